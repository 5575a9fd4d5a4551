// Greedy (temperature 0) mode of fsr_spec_accept: Sec. 2.1's accept-until-first-mismatch rule with
// an arg-max target.  A draft is accepted iff it is the arg-max token of its target row (lowest id
// among equal maxima); the token after the accepted run is the arg-max of the next target row.
//
// The cost is one streaming pass over the target rows (4 V bytes each).  Row after row would put a memory round trip per
// accepted draft on the critical path, so all rows are read at once; but a large call starts them in the order of their
// positions, those of all requests' first drafts before any of a second one, and a workgroup whose request is known to have a
// mismatch before its row leaves at once.  A mismatch is known as soon as any workgroup of the row has met a score above the
// draft's own, long before the row is done.  A small call has most rows in flight before anything is known, and the asking
// and telling costs it more than the rows (kSkipMinPieces).
// greedy_argmax_kernel: every workgroup folds a 16 KB piece of a row into a 64-bit key (value made order-preserving << 32 |
// ~index) and merges it into the row's key with one atomic max, which yields the largest value and, among equals, the
// lowest index.
// Measured, us a call (three launches in a graph), 1-8 drafts of which about 40 % match, all rows read / rows left out, by the
// pieces the call can hold: vocabulary 152064: 32 requests (10.9 k) 24.0 / 25.4, 48 (16.4 k) 34.0 / 30.0, 128 81 / 38;
// 128256: 16 requests 16.1 / 17.7, 48 (13.8 k) 28.9 / 31.4, 64 (18.4 k) 34.3 / 33.0, 256 123 / 60; 64000: 32 requests 13.2 /
// 22.8, 96 (13.8 k) 27.4 / 29.0, 128 (18.4 k) 33.8 / 26.5; 32000: 64 requests 14.9 / 24.0, 192 (13.8 k) 28.6 / 27.7, 256
// (18.4 k) 36.0 / 26.6.  Workgroups that go through a request's positions one after the other read less but wait more: 39 us
// at 64 requests, 176 us at 384.
#include <climits>
#include <cstdint>

#include "common.hpp"
#include "device_utils.hpp"
#include "greedy_accept.hpp"

namespace fsr {
namespace {

constexpr int kThreads = 256;
constexpr int kChunk = 4096;  // scores of a piece
constexpr int kQuads = kChunk / kThreads / 4;
constexpr int kSkipMinPieces = 16384;  // pieces a call must be able to hold for rows behind a mismatch to be left out

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)), __aligned__(4))) uint32_t gu32x4;  // at any element of a row

// fp32 bits -> unsigned integer with the same order (-0 and +0 map to the same key; a NaN never wins
// against a number: it takes the key of minus infinity).
__device__ __forceinline__ uint32_t ordered_bits(uint32_t b) {
    if ((b << 1) == 0) b = 0;  // -0 -> +0
    if ((b & 0x7fffffffu) > 0x7f800000u) b = 0xff800000u;  // NaN -> -inf
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ unsigned long long make_key(uint32_t bits, int idx) {
    return ((unsigned long long)ordered_bits(bits) << 32) | (uint32_t)(0xffffffffu - (uint32_t)idx);
}
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)k, o, kWave), hi = __shfl_xor((uint32_t)(k >> 32), o, kWave);
        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
        k = other > k ? other : k;
    }
    return k;
}

// A request whose row counts do not fit the call is flagged by `decide`; none of its rows or drafts is looked at (a call with
// S_max = 0 has no drafts to read: draft_tokens may be null).
__device__ __forceinline__ bool refused(int t0, int t_i, int d_i, int S_max, int R_cap) {
    return d_i < 0 || d_i > S_max || t_i < d_i || t_i > d_i + 1 || t0 < 0 || t0 + t_i > R_cap;
}

// first_miss [B]: position of the first mismatch known so far (the accepted_len output serves until `decide` fills it)
__global__ __launch_bounds__(kThreads) void greedy_init_kernel(unsigned long long* keys, int32_t* first_miss, int n, int B) {
    const int r = blockIdx.x * kThreads + threadIdx.x;
    if (r < n) keys[r] = 0ull;
    if (r < B) first_miss[r] = INT_MAX;
}

// grid (pieces, B (S_max + 1)).  SKIP: workgroup row y takes position y / B of request y % B and leaves out what lies behind a
// known mismatch; else it takes the call's row y.
template <bool SKIP>
__global__ __launch_bounds__(kThreads) void greedy_argmax_kernel(
    const float* __restrict__ target, const int32_t* __restrict__ draft_tokens, const int32_t* __restrict__ cu_t,
    const int32_t* __restrict__ cu_d, const int32_t* __restrict__ t_rows, const int32_t* __restrict__ d_rows,
    unsigned long long* keys, int32_t* first_miss, int B, int V, int S_max, int R_cap) {
    __shared__ unsigned long long part[kThreads / 64];
    __shared__ int s_miss;
    int r = blockIdx.y, i = 0, j = 0, d0 = 0, d_i = 0;  // r: call-row on the target side
    if constexpr (SKIP) {
        j = r / B;
        i = r - j * B;
        const int t0 = cu_t[i], t_i = cu_t[i + 1] - t0;
        d0 = cu_d[i];
        d_i = cu_d[i + 1] - d0;
        r = t0 + j;
        if (j >= t_i || r >= cu_t[B] || refused(t0, t_i, d_i, S_max, R_cap)) return;
        if (j > 0) {  // one lane asks: the words of all requests lie in a few cache lines that every workgroup wants
            if (threadIdx.x == 0) s_miss = __hip_atomic_load(first_miss + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (s_miss < j) return;
        }
    } else if (r >= cu_t[B]) {
        return;
    }
    const float* z = target + (size_t)(t_rows ? t_rows[r] : r) * V;
    const int v0 = blockIdx.x * kChunk;
    u32x4 x[kQuads];
    if (v0 + kChunk <= V) {
#pragma unroll
        for (int q = 0; q < kQuads; ++q)  // a row is streamed once
            x[q] = __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(z + v0 + (q * kThreads + threadIdx.x) * 4));
    } else {  // past the end: minus infinity at an index that loses against every token
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const int v = v0 + (q * kThreads + threadIdx.x) * 4;
            if (v + 3 < V) x[q] = __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(z + v));
            else x[q] = u32x4{0xff800000u, 0xff800000u, 0xff800000u, 0xff800000u};
        }
        const int tail = V & ~3;  // (v0 is a multiple of four, so only the row's last quad is not whole)
        if (tail < V && (tail - v0) / 4 % kThreads == (int)threadIdx.x) {
#pragma unroll
            for (int q = 0; q < kQuads; ++q)
                if (v0 + (q * kThreads + (int)threadIdx.x) * 4 == tail)
#pragma unroll
                    for (int u = 0; u < 3; ++u)
                        if (tail + u < V) x[q][u] = __builtin_bit_cast(uint32_t, z[tail + u]);
        }
    }
    // the key of the draft this row verifies: larger than any if there is none, smaller for an id outside the vocabulary
    unsigned long long drafted = ~0ull;
    if (SKIP && d0 >= 0 && j < d_i && d0 + j < cu_d[B]) {
        const int t = draft_tokens[d_rows ? d_rows[d0 + j] : d0 + j];
        drafted = t < 0 || t >= V ? 0ull : make_key(__builtin_bit_cast(uint32_t, z[t]), t);
    }
    unsigned long long best = 0ull;
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
        const int v = v0 + (q * kThreads + threadIdx.x) * 4;
        const uint32_t w0 = x[q][0], w1 = x[q][1], w2 = x[q][2], w3 = x[q][3];
        unsigned long long c = make_key(w0, v);
        const unsigned long long c1 = make_key(w1, v + 1), c2 = make_key(w2, v + 2), c3 = make_key(w3, v + 3);
        c = c1 > c ? c1 : c;
        c = c2 > c ? c2 : c;
        c = c3 > c ? c3 : c;
        best = c > best ? c : best;
    }
    best = wave_max_u64(best);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kThreads / 64; ++w) best = part[w] > best ? part[w] : best;
        if (SKIP && best > drafted) atomicMin(first_miss + i, j);
        atomicMax(keys + r, best);
    }
}

__global__ __launch_bounds__(kThreads) void greedy_decide_kernel(const int32_t* __restrict__ draft_tokens,
                                                                 const int32_t* __restrict__ cu_t,
                                                                 const int32_t* __restrict__ cu_d,
                                                                 const int32_t* __restrict__ d_rows,
                                                                 const unsigned long long* __restrict__ keys,
                                                                 int32_t* accepted_len, int32_t* n_emitted,
                                                                 int32_t* emitted, int B, int S_max, int R_cap) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= B) return;
    const int d_i = cu_d[i + 1] - cu_d[i], t_i = cu_t[i + 1] - cu_t[i];
    int32_t* em = emitted + (size_t)i * (S_max + 1);
    for (int s = 0; s <= S_max; ++s) em[s] = -1;
    if (refused(cu_t[i], t_i, d_i, S_max, R_cap)) {
        accepted_len[i] = -1;
        n_emitted[i] = -1;
        return;
    }
    auto choice = [&](int n) { return (int)(0xffffffffu - (uint32_t)keys[cu_t[i] + n]); };
    int n = 0, tok = -1;
    while (n < d_i) {
        const long long dr = d_rows ? d_rows[cu_d[i] + n] : cu_d[i] + n;
        const int c = choice(n);
        if (draft_tokens[dr] != c) {
            tok = c;
            break;
        }
        em[n] = c;
        ++n;
    }
    if (n == d_i && t_i == d_i + 1) tok = choice(d_i);
    if (tok >= 0) em[n] = tok;
    accepted_len[i] = n;
    n_emitted[i] = n + (tok >= 0 ? 1 : 0);
}

}  // namespace

size_t greedy_workspace_bytes(const fsr_accept_params& p) {
    return align_up((size_t)p.B * (size_t)(p.S_max + 1) * sizeof(unsigned long long), 256);
}

int greedy_accept_launch(const float* target, const int32_t* draft_tokens, const int32_t* cu_t, const int32_t* cu_d,
                         const int32_t* t_rows, const int32_t* d_rows, int32_t* accepted_len, int32_t* n_emitted,
                         int32_t* emitted, const fsr_accept_params& p, void* workspace, hipStream_t s) {
    unsigned long long* keys = (unsigned long long*)workspace;
    const int R_cap = p.B * (p.S_max + 1);
    int rc;
    hipLaunchKernelGGL(greedy_init_kernel, dim3((R_cap + kThreads - 1) / kThreads), dim3(kThreads), 0, s, keys, accepted_len, R_cap, p.B);
    if ((rc = check_launch("greedy_init_kernel")) != FSR_OK) return rc;
    const int pieces = (p.V + kChunk - 1) / kChunk;
    const bool skip = (long long)R_cap * pieces >= kSkipMinPieces;
    hipLaunchKernelGGL(skip ? greedy_argmax_kernel<true> : greedy_argmax_kernel<false>, dim3(pieces, R_cap), dim3(kThreads), 0, s, target,
                       draft_tokens, cu_t, cu_d, t_rows, d_rows, keys, accepted_len, p.B, p.V, p.S_max, R_cap);
    if ((rc = check_launch("greedy_argmax_kernel")) != FSR_OK) return rc;
    hipLaunchKernelGGL(greedy_decide_kernel, dim3((p.B + kThreads - 1) / kThreads), dim3(kThreads), 0, s, draft_tokens, cu_t,
                       cu_d, d_rows, keys, accepted_len, n_emitted, emitted, p.B, p.S_max, R_cap);
    return check_launch("greedy_decide_kernel");
}

}  // namespace fsr
