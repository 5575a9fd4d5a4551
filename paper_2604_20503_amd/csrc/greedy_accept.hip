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
// greedy_argmax_kernel: every workgroup finds the largest score of a 32 or 64 KB piece of a row and its lowest place, and merges
// them as a 64-bit key (value made order-preserving << 32 | ~index) into the row's key with one atomic max, which yields the largest
// value and, among equals, the lowest index.  Most workgroups of a large call are those of rows that are left out, and each costs two
// memory round trips before it may leave: the largest calls take 64 KB pieces.  With fewer, smaller pieces tell of a mismatch sooner.
// Telling costs too: the words of 32 requests share a cache line, and every atomic on one waits for those before it.  Below a bad
// guess thousands of scores, in every piece, are larger than the draft's: such a piece (scores of several of its waves are) first
// merges its key and tells only if the row's key of before was not above the draft's already.  A near miss is told at once.
// Measured, us a call, 1-8 drafts of which 40 % match and the others are their row's second-best token / a random one:
//   all rows read, by pieces of 64 KB the call can hold, pieces of 16 KB (256 threads) / 32 / 64 KB: vocabulary 32000: 1 request (18)
//   7.4 / 7.3 / 8.1, 4 (72) 8.9 / 8.0 / 8.7, 24 (432) 10.9 / 9.8 / 10.8, 48 (864) 13.3 / 11.7 / 12.1;  64000: 1 (36) 8.1 / 7.7 / 8.4, 16 (576)
//   12.8 / 11.1 / 11.4;  128256: 1 (72) 7.4 / 7.5 / 8.2, 2 (144) 10.4 / 9.0 / 8.8, 8 (576) 12.0 / 9.8 / 9.2, 16 (1152) 16.3 / 13.7 / 13.2, 24
//   (1728) 22.4 / 18.9 / 18.6;
//   all rows read in pieces of 32 KB / rows left out, near misses, bad guesses (told by every piece): 128256: 48 requests (3456) 29 / 23.1,
//   26.7 (51), all match 29 / 31;  64 (4608) 35 / 24.9, 27.0 (51), all match 35 / 39;  100 (7200) 50 / 29.7, 30.5 (40);  152064: 128 (11520)
//   76 / 39.7, 40.0 (51);  128256: 384 (27648) 167 / 67.4, 65.8 (68).  (Told after the merge by every piece: 64 requests 26.3, 25.0.)
//   rows left out, pieces of 16 KB / 32 / 64 KB, with the compaction: 128256: 64 requests (4608) 40.0 / 34.6 / 36.3, 100 (7200) 37.6 / 36.6 /
//   40.3, 160 (11520) 48.7 / 47.7 / 47.9, 384 (27648) 101 / 101 / 85; 152064: 250 (22500) 78 / 78 / 68; 32000: 380 (6840) 42.8 / 39.5 / 41.1.
// At 64 requests 50 MB are read: what is left is the chain of workgroups, not the bytes.  Workgroups that go through a request's
// positions one after the other read less but wait more: 45 us at 64 requests, 139 us at 384.
#include <climits>
#include <cstdint>

#include "common.hpp"
#include "device_utils.hpp"
#include "greedy_accept.hpp"

namespace fsr {
namespace {

constexpr int kThreads = 256;
constexpr int kRowThreads = 512;                  // threads that take a piece of a row
// 16-byte loads of such a thread, all in flight together: four or eight, i.e. pieces of 32 or 64 KB
template <int QUADS>
constexpr int kChunk = kRowThreads * QUADS * 4;  // scores of a piece
constexpr int kLongPieces = 12288;    // 64 KB pieces a call must be able to hold for pieces of that size where rows are left out
constexpr int kSkipMinPieces = 3072;  // 64 KB pieces a call must be able to hold for rows behind a mismatch to be left out
constexpr int kShortRow = 98304;      // where none is left out: scores of a row up to which its pieces are of 32 KB, ...
constexpr int kFewPieces = 128;       // ... and 64 KB pieces up to which a call's are

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

// A thread's scores of a piece are the quads q * kRowThreads + thread.
// Send for the scores v0 .. v0 + kChunk - 1 of row z.
template <int kQuads>
__device__ __forceinline__ void load_piece(const float* __restrict__ z, int v0, int V, u32x4 (&x)[kQuads]) {
    if (v0 + kChunk<kQuads> <= V) {
#pragma unroll
        for (int q = 0; q < kQuads; ++q)  // a row is streamed once
            x[q] = __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(z + v0 + (q * kRowThreads + threadIdx.x) * 4));
    } else {  // past the end: minus infinity at an index that loses against every token
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const int v = v0 + (q * kRowThreads + threadIdx.x) * 4;
            if (v + 3 < V) x[q] = __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(z + v));
            else x[q] = u32x4{0xff800000u, 0xff800000u, 0xff800000u, 0xff800000u};
        }
        const int tail = V & ~3;  // (v0 is a multiple of four, so only the row's last quad is not whole)
        if (tail < V && (tail - v0) / 4 % kRowThreads == (int)threadIdx.x) {
#pragma unroll
            for (int q = 0; q < kQuads; ++q)
                if (v0 + (q * kRowThreads + (int)threadIdx.x) * 4 == tail)
#pragma unroll
                    for (int u = 0; u < 3; ++u)
                        if (tail + u < V) x[q][u] = __builtin_bit_cast(uint32_t, z[tail + u]);
        }
    }
}

// Key of the piece's largest score and its lowest place, valid in thread 0; ends behind a barrier.  The largest value first (a
// NaN counts as minus infinity, -0 equals +0), by plain maxima, and only then, in the waves that hold it, the lowest place: one
// or two instructions a score where folding (value, place) keys took ten.
template <int kQuads>
__device__ __forceinline__ unsigned long long piece_key(const u32x4 (&x)[kQuads], int v0, float* s_top, int* s_at) {
    constexpr int kW = kRowThreads / 64;
    float top = -INFINITY;
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
        const uint32_t w0 = x[q][0], w1 = x[q][1], w2 = x[q][2], w3 = x[q][3];
        top = fmaxf(top, fmaxf(__builtin_bit_cast(float, w0), __builtin_bit_cast(float, w1)));
        top = fmaxf(top, fmaxf(__builtin_bit_cast(float, w2), __builtin_bit_cast(float, w3)));
    }
    top = wave_max(top);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0) s_top[w] = top;
    __syncthreads();
    float most = s_top[0];
#pragma unroll
    for (int k = 1; k < kW; ++k) most = fmaxf(most, s_top[k]);
    int at = INT_MAX;
    if (top == most) {
#pragma unroll
        for (int q = kQuads - 1; q >= 0; --q) {
            const uint32_t wq[4] = {x[q][0], x[q][1], x[q][2], x[q][3]};
#pragma unroll
            for (int u = 3; u >= 0; --u) {  // (nothing but minus infinities and NaN: the first place)
                const float f = __builtin_bit_cast(float, wq[u]);
                if (f == most || most == -INFINITY) at = v0 + (q * kRowThreads + (int)threadIdx.x) * 4 + u;
            }
        }
        at = wave_min_i(at);
    }
    if ((threadIdx.x & 63) == 0) s_at[w] = at;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kW; ++k) at = min(at, s_at[k]);
    return make_key(__builtin_bit_cast(uint32_t, most), at);
}

// grid (pieces, B (S_max + 1)).  SKIP: workgroup row y takes position y / B of request y % B and leaves out what lies behind a
// known mismatch; else it takes the call's row y.
template <bool SKIP, int kQuads>
__global__ __launch_bounds__(kRowThreads) void greedy_argmax_kernel(
    const float* __restrict__ target, const int32_t* __restrict__ draft_tokens, const int32_t* __restrict__ cu_t,
    const int32_t* __restrict__ cu_d, const int32_t* __restrict__ t_rows, const int32_t* __restrict__ d_rows,
    unsigned long long* keys, int32_t* first_miss, int B, int V, int S_max, int R_cap) {
    __shared__ float s_top[kRowThreads / 64];
    __shared__ int s_at[kRowThreads / 64];
    __shared__ int s_miss;
    int r = blockIdx.y, i = 0, j = 0, d0 = 0, d_i = 0;  // r: call-row on the target side
    if constexpr (SKIP) {
        j = r / B;
        i = r - j * B;
        // one lane asks (the words of all requests lie in a few cache lines that every workgroup wants), with the offsets
        // still on their way: most workgroups of a large call do nothing else
        if (threadIdx.x == 0) s_miss = __hip_atomic_load(first_miss + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int t0 = cu_t[i], t_i = cu_t[i + 1] - t0;
        d0 = cu_d[i];
        d_i = cu_d[i + 1] - d0;
        r = t0 + j;
        if (j >= t_i || r >= cu_t[B] || refused(t0, t_i, d_i, S_max, R_cap)) return;
        __syncthreads();
        if (s_miss < j) return;
    } else if (r >= cu_t[B]) {
        return;
    }
    const float* z = target + (size_t)(t_rows ? t_rows[r] : r) * V;
    const int v0 = blockIdx.x * kChunk<kQuads>;
    u32x4 x[kQuads];
    load_piece(z, v0, V, x);
    // the key of the draft this row verifies: larger than any if there is none, smaller for an id outside the vocabulary
    unsigned long long drafted = ~0ull;
    float guess = -INFINITY;
    if (SKIP && d0 >= 0 && j < d_i && d0 + j < cu_d[B]) {
        const int t = draft_tokens[d_rows ? d_rows[d0 + j] : d0 + j];
        if (t >= 0 && t < V) guess = z[t];
        drafted = t < 0 || t >= V ? 0ull : make_key(__builtin_bit_cast(uint32_t, guess), t);
    }
    const unsigned long long best = piece_key(x, v0, s_top, s_at);
    if (threadIdx.x == 0) {
        int above = 0;  // waves of the piece with a score above the draft's own
        if (SKIP && best > drafted) {
#pragma unroll
            for (int k = 0; k < kRowThreads / 64; ++k) above += !(s_top[k] <= guess);
        }
        if (above > 1 && blockIdx.x != 0) {  // (a wait for the key of before, which a near miss is spared)
            if (atomicMax(keys + r, best) <= drafted) atomicMin(first_miss + i, j);
        } else {
            if (SKIP && best > drafted) atomicMin(first_miss + i, j);
            atomicMax(keys + r, best);
        }
    }
}

__global__ __launch_bounds__(kThreads) void greedy_decide_kernel(const int32_t* __restrict__ draft_tokens,
                                                                 const int32_t* __restrict__ cu_t,
                                                                 const int32_t* __restrict__ cu_d,
                                                                 const int32_t* __restrict__ d_rows,
                                                                 const unsigned long long* __restrict__ keys,
                                                                 int32_t* accepted_len, int32_t* n_emitted,
                                                                 int32_t* emitted, int B, int S_max, int R_cap) {
    // one wave per request, lane n tests draft n: what they read is in flight together
    const int i = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= B) return;
    const int t0 = cu_t[i], t_i = cu_t[i + 1] - t0, d0 = cu_d[i], d_i = cu_d[i + 1] - d0;
    int32_t* em = emitted + (size_t)i * (S_max + 1);
    if (refused(t0, t_i, d_i, S_max, R_cap)) {
        for (int s = lane; s <= S_max; s += 64) em[s] = -1;
        if (lane == 0) {
            accepted_len[i] = -1;
            n_emitted[i] = -1;
        }
        return;
    }
    int n = d_i, tok = -1;  // accepted drafts, and the token behind them
    for (int n0 = 0; n0 < t_i; n0 += 64) {
        const int k = n0 + lane;
        int choice = -1, drafted = -1;
        if (k < t_i) choice = (int)(0xffffffffu - (uint32_t)keys[t0 + k]);
        if (k < d_i) drafted = draft_tokens[d_rows ? d_rows[d0 + k] : d0 + k];
        // the run ends at the first mismatch, or at the row behind the last draft
        const unsigned long long ends = __builtin_amdgcn_ballot_w64(k < t_i && (k >= d_i || choice != drafted));
        const int first = ends ? (int)__builtin_ctzll(ends) : 64;
        if (k < t_i && lane < first) em[k] = choice;
        if (ends) {
            n = n0 + first;
            tok = __shfl(choice, first, 64);
            break;
        }
    }
    for (int s = n + lane; s <= S_max; s += 64) em[s] = s == n ? tok : -1;
    if (lane == 0) {
        accepted_len[i] = n;
        n_emitted[i] = n + (tok >= 0 ? 1 : 0);
    }
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
    auto launch = [&](auto kernel, int chunk) {
        hipLaunchKernelGGL(kernel, dim3((p.V + chunk - 1) / chunk, R_cap), dim3(kRowThreads), 0, s, target, draft_tokens, cu_t, cu_d, t_rows,
                           d_rows, keys, accepted_len, p.B, p.V, p.S_max, R_cap);
    };
    const long long pieces = (long long)R_cap * ((p.V + kChunk<8> - 1) / kChunk<8>);
    if (pieces < kSkipMinPieces && (p.V <= kShortRow || pieces <= kFewPieces)) launch(greedy_argmax_kernel<false, 4>, kChunk<4>);
    else if (pieces < kSkipMinPieces) launch(greedy_argmax_kernel<false, 8>, kChunk<8>);
    else if (pieces < kLongPieces) launch(greedy_argmax_kernel<true, 4>, kChunk<4>);
    else launch(greedy_argmax_kernel<true, 8>, kChunk<8>);
    if ((rc = check_launch("greedy_argmax_kernel")) != FSR_OK) return rc;
    hipLaunchKernelGGL(greedy_decide_kernel, dim3((p.B + kThreads / 64 - 1) / (kThreads / 64)), dim3(kThreads), 0, s, draft_tokens, cu_t,
                       cu_d, d_rows, keys, accepted_len, n_emitted, emitted, p.B, p.S_max, R_cap);
    return check_launch("greedy_decide_kernel");
}

}  // namespace fsr
