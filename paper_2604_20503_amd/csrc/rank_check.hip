// Early-exit rank check (Sec. 3.2: intermediate scores predict a rejection when the draft is not
// among their K best tokens; Sec. 4: decided by counting the scores above the draft's own, without
// building the set of the K best).
//
// The work is one pass over the score row of every draft that still has an active row: count the
// scores strictly above the draft's own.  That is HBM streaming with a trivial reduction.
//   rank_check_kernel   one launch, one workgroup per draft: it streams the row with 16-byte loads (at any alignment: the
//                       hardware takes vectors at element addresses), the next four of every thread in flight while four
//                       are counted, and writes the draft's rank and its row's mask itself.  Long rows and those of few
//                       drafts get 1024 threads, others, which a workgroup is through with in a few rounds, 512.
//   rank_init_kernel    rank[d] = 0 for drafts with an active row and a valid token id, -1 for drafts without a row, V for
//                       ids outside the vocabulary;
//   rank_count_kernel   rank[d] += #{v in chunk : z[row][v] > z[row][draft]}, grid (32 KB piece of a row) x (draft), a piece's
//                       loads all in flight together, one integer atomic per workgroup;
//   rank_mask_kernel    keep[row] from the ranks (first row of a request always kept): three launches, for a few hundred
//                       rows of 384 KB or more, a few dozen of 320 KB or a few of 288, which one workgroup each would take too
//                       long, or on too few of the compute units, to read (see pieces_below).
// What bounds it is reading the rows once there are enough of them, and one row's stream through one workgroup where there are
// few.  Drafts may have lost their rows to an earlier check, and the caller's capacities need not say so.
// Measured, us a call in a graph, caches cold, drafts of the call and rows that are live, three launches / one of 1024 threads /
// of 512:
// (256 threads: 4032 all of 256 KB 160, of 513 KB 315; 2054, 508 live of 513 KB 75; 3976 all of 64 KB 43.5, 355 live 12.1, there with 512 13.9)
//   64 KB rows (32000 bf16): 73, 57 live 8.0 / 4.8 / 4.9;  718 all 16.2 / 12.3 / 11.2;  718, 43 live 9.3 / 5.9 / 5.2;  3976 all 47.4 /
//   51.0 / 41.7;  128 KB rows (32000 fp32): 493 all 17.3 / 13.4 / 13.4;  4006 all 82.3 / 79.9 / 79.1;  4006, 205 live 19.9 / 19.5 / 13.6;
//   256 KB rows (128256 bf16): 83 all 11.2 / 10.5 / 10.7;  279, 69 live 10.9 / 9.5 / 10.2;  471 all 26.3 / 22.9 / 23.0;  716 all 35.4 / 32.0 /
//   33.2;  716, 45 live 11.5 / 13.5 / 13.4;  1427 all 63.2 / 58.4 / 60.2;  1427, 416 live 26.3 / 24.6 / 26.1;  2040 all 85.0 / 79.9 / 82.7;
//   304 KB rows (152064 bf16), three launches / one: 2 requests of 1 to 4 drafts 7.8 / 8.7, 4, half of them live, 8.2 / 9.1, 8 all 9.3 / 8.7, 16
//   all 10.9 / 9.6;  340 KB (170000 bf16): 2 requests 7.8 / 9.1, 16 all 10.2 / 10.7, half live 8.8 / 10.1, 24 all 12.3 / 11.3;  380 KB: 2 requests
//   7.9 / 9.8, 16 all 10.5 / 11.2, half live 9.0 / 11.5, 24 all 13.1 / 12.6;
//   513 KB rows (128256 fp32): 79 all 15.6 / 16.0 / 16.8;  79, 19 live 9.0 / 12.3 / 14.3;  289, 93 live 15.1 / 23.2 / 23.1;  491 all 48.7 /
//   41.2 / 41.8;  491, 123 live 19.0 / 24.4 / 24.8;  722 all 66.6 / 58.9 / 61.2;  722, 183 live 24.3 / 26.0 / 26.1;  990, 247 live 30.2 / 28.5 /
//   43.3;  1431 all 121 / 111 / 115;  2054 all 168 / 163 / 167;  2054, 508 live 51.5 / 47.2 / 53.6.
#include <algorithm>
#include <cstdint>

#include "common.hpp"
#include "device_utils.hpp"

namespace fsr {
namespace {

constexpr int kLoads = 4;       // 16-byte loads of a thread that are counted together; as many more are in flight
constexpr int kThreads = 256;   // of the three launches
constexpr int kPieceLoads = 8;  // 16-byte loads of a thread, all in flight together
constexpr int kChunkBytes = kThreads * kPieceLoads * 16;  // a workgroup's piece of a row
// Live rows that a call can have, by the bytes of a row, below which its rows are cut into pieces, if it has no more drafts than
// kPiecesDrafts (the launches before and after look at every draft).
int pieces_below(long long row_bytes) { return row_bytes >= 384 << 10 ? 512 : row_bytes >= 320 << 10 ? 48 : row_bytes >= 288 << 10 ? 12 : 0; }
constexpr int kPiecesDrafts = 1536;
constexpr int kLongRow = 192 << 10;    // bytes of a row from which it gets 1024 threads, ...
constexpr int kFewDrafts = 512;        // ... and drafts up to which it does in any case
constexpr int kMaskRows = 256;  // rows without a draft that one of the further workgroups looks after

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)), __aligned__(2))) uint32_t gu32x4;  // at any element of a row

struct RankArgs {
    const void* logits;
    const int32_t* draft_tokens;
    const int32_t* cu_q;
    const int32_t* cu_d;
    int32_t* rank;
    uint8_t* keep;
    int B, V, K, N_cap, D_cap;
};

// Largest i with cu[i] <= x, skipping empty requests to the right (cu is non-decreasing, cu[0] = 0).
__device__ __forceinline__ int owner(const int32_t* __restrict__ cu, int B, int x) {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// The same by a whole wave: every lane looks at one of 64 places at a time, so a search is one memory round trip per factor
// of 64 instead of one per factor of two.
__device__ __forceinline__ int owner_by_wave(const int32_t* __restrict__ cu, int B, int x) {
    const int lane = threadIdx.x & 63;
    int lo = 0, n = B;  // the answer lies in [lo, lo + n)
    while (n > 1) {
        const int step = (n + 63) / 64, at = lo + lane * step;
        const unsigned long long below = __builtin_amdgcn_ballot_w64(lane * step < n && cu[at] <= x);
        const int k = below ? 63 - (int)__builtin_clzll(below) : 0;  // the last such place (cu is non-decreasing)
        n = min(step, n - k * step);
        lo += k * step;
    }
    return lo;
}

template <typename T>
__device__ __forceinline__ float score(const void* base, size_t idx);
template <>
__device__ __forceinline__ float score<float>(const void* base, size_t idx) {
    return reinterpret_cast<const float*>(base)[idx];
}
template <>
__device__ __forceinline__ float score<uint16_t>(const void* base, size_t idx) {
    return __builtin_bit_cast(float, (uint32_t)reinterpret_cast<const uint16_t*>(base)[idx] << 16);
}

// How many of the two bf16 scores packed in w exceed x.
__device__ __forceinline__ int above_pair(uint32_t w, float x) {
    return (__builtin_bit_cast(float, w << 16) > x) + (__builtin_bit_cast(float, w & 0xffff0000u) > x);
}

// Score row of draft d, or -1 if the draft has no active row (its rows were pruned earlier).
__device__ __forceinline__ int row_of_draft(const RankArgs& a, int d) {
    const int i = owner(a.cu_d, a.B, d);
    const int j = d - a.cu_d[i];
    return j < a.cu_q[i + 1] - a.cu_q[i] ? a.cu_q[i] + j : -1;
}

__global__ __launch_bounds__(kThreads) void rank_init_kernel(RankArgs a) {
    const int d = blockIdx.x * kThreads + threadIdx.x;
    if (d >= a.D_cap || d >= a.cu_d[a.B]) return;
    const int row = row_of_draft(a, d);
    const int tok = a.draft_tokens[d];
    a.rank[d] = row < 0 ? -1 : (tok < 0 || tok >= a.V) ? a.V : 0;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void rank_count_kernel(RankArgs a) {
    __shared__ int part[kThreads / 64];
    const int d = blockIdx.y;
    if (d >= a.cu_d[a.B]) return;
    const int i = owner_by_wave(a.cu_d, a.B, d), j = d - a.cu_d[i];
    const int row = j < a.cu_q[i + 1] - a.cu_q[i] ? a.cu_q[i] + j : -1;
    const int tok = a.draft_tokens[d];
    if (row < 0 || row >= a.N_cap || tok < 0 || tok >= a.V) return;  // uniform for the workgroup
    constexpr int kPer = 16 / sizeof(T);  // scores per 16-byte load
    const T* z = reinterpret_cast<const T*>(a.logits) + (size_t)row * a.V;
    const int v0 = blockIdx.x * (kChunkBytes / (int)sizeof(T));
    u32x4 w[kPieceLoads];
    const bool whole = a.V - v0 >= kChunkBytes / (int)sizeof(T);
    const int last = a.V - v0 - kPer;  // of the row's last piece: where its last whole load may start
    if (whole) {
#pragma unroll
        for (int k = 0; k < kPieceLoads; ++k)  // a row is streamed once
            w[k] = __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(z + v0 + (k * kThreads + threadIdx.x) * kPer));
    } else if (a.V >= kPer) {
        // loads past the row's end are moved back to its last whole one, so that all are unconditional and in flight
        // together here too, and what they bring is left out
#pragma unroll
        for (int k = 0; k < kPieceLoads; ++k)
            w[k] = *reinterpret_cast<const gu32x4*>(z + (v0 + min((k * kThreads + (int)threadIdx.x) * kPer, last)));
    }
    const float mine = score<T>(z, tok);
    int count = 0;
    auto add = [&](u32x4 x) {
        // elements go to scalars first: __builtin_bit_cast applied to a vector-element expression was
        // seen to read element 0 for every index
        const uint32_t w0 = x[0], w1 = x[1], w2 = x[2], w3 = x[3];
        if constexpr (sizeof(T) == 4) {
            count += (__builtin_bit_cast(float, w0) > mine) + (__builtin_bit_cast(float, w1) > mine) +
                     (__builtin_bit_cast(float, w2) > mine) + (__builtin_bit_cast(float, w3) > mine);
        } else {
            count += above_pair(w0, mine) + above_pair(w1, mine) + above_pair(w2, mine) + above_pair(w3, mine);
        }
    };
    if (whole) {
#pragma unroll
        for (int k = 0; k < kPieceLoads; ++k) add(w[k]);
    } else {
#pragma unroll
        for (int k = 0; k < kPieceLoads; ++k)
            if ((k * kThreads + (int)threadIdx.x) * kPer <= last) add(w[k]);
    }
    const int tail = a.V - a.V % kPer + (int)threadIdx.x;  // (pieces are whole loads: what is left over ends the row's last one)
    if ((int)threadIdx.x < a.V % kPer && tail >= v0 && tail < v0 + kChunkBytes / (int)sizeof(T)) count += score<T>(z, tail) > mine;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o, kWave);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) total += part[w];
        if (total) atomicAdd(a.rank + d, total);
    }
}

__global__ __launch_bounds__(kThreads) void rank_mask_kernel(RankArgs a) {
    const int row = blockIdx.x * kThreads + threadIdx.x;
    if (row >= a.N_cap || row >= a.cu_q[a.B]) return;
    const int i = owner(a.cu_q, a.B, row);
    const int j = row - a.cu_q[i];  // the row's input is draft j - 1 of the request
    uint8_t keep = 1;
    if (j >= 1 && j - 1 < a.cu_d[i + 1] - a.cu_d[i]) keep = a.rank[a.cu_d[i] + j - 1] < a.K ? 1 : 0;
    a.keep[row] = keep;
}

// Workgroup d < D_cap: rank[d], and keep[row] of the row that carries the draft.  The workgroups behind those: keep = 1 for
// the rows that carry no draft (a request's first row; rows past its last draft).
template <typename T, int THREADS>
__global__ __launch_bounds__(THREADS) void rank_check_kernel(RankArgs a) {
    __shared__ int part[THREADS / 64];
    if (blockIdx.x >= (unsigned)a.D_cap) {
        const int row = (blockIdx.x - a.D_cap) * kMaskRows + threadIdx.x;
        if (threadIdx.x >= kMaskRows || row >= a.N_cap || row >= a.cu_q[a.B]) return;
        const int i = owner(a.cu_q, a.B, row);
        const int j = row - a.cu_q[i];  // the row's input is draft j - 1 of the request
        if (j < 1 || j - 1 >= a.cu_d[i + 1] - a.cu_d[i]) a.keep[row] = 1;
        return;
    }
    const int d = blockIdx.x;
    if (d >= a.cu_d[a.B]) return;
    const int i = owner_by_wave(a.cu_d, a.B, d), j = d - a.cu_d[i];
    const int q0 = a.cu_q[i], q1 = a.cu_q[i + 1];
    const int row = j < q1 - q0 ? q0 + j : -1;
    const int tok = a.draft_tokens[d];
    // -1 without an active row (its rows were pruned earlier), V for an id outside the vocabulary, 0 for a row past N_cap
    int rank = row < 0 ? -1 : (tok < 0 || tok >= a.V) ? a.V : 0;
    if (rank == 0 && row < a.N_cap) {  // uniform for the workgroup
        constexpr int kPer = 16 / sizeof(T);                 // scores per 16-byte load
        constexpr int kPiece = THREADS * kLoads * kPer;      // scores the workgroup counts between two waits
        const T* z = reinterpret_cast<const T*>(a.logits) + (size_t)row * a.V;
        const float mine = score<T>(z, tok);
        int count = 0;
        auto add = [&](u32x4 x) {
            // elements go to scalars first: __builtin_bit_cast applied to a vector-element expression was
            // seen to read element 0 for every index
            const uint32_t w0 = x[0], w1 = x[1], w2 = x[2], w3 = x[3];
            if constexpr (sizeof(T) == 4) {
                count += (__builtin_bit_cast(float, w0) > mine) + (__builtin_bit_cast(float, w1) > mine) +
                         (__builtin_bit_cast(float, w2) > mine) + (__builtin_bit_cast(float, w3) > mine);
            } else {
                count += above_pair(w0, mine) + above_pair(w1, mine) + above_pair(w2, mine) + above_pair(w3, mine);
            }
        };
        const int n_vec = a.V / kPer;  // whole loads of the row
        u32x4 w[2][kLoads];
        // loads past the row's last whole one are moved back to it, so that all are unconditional, and what they bring is
        // left out
        auto issue = [&](u32x4 (&x)[kLoads], int p) {
#pragma unroll
            for (int k = 0; k < kLoads; ++k)  // a row is streamed once
                x[k] = __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(
                    z + (size_t)min(p * THREADS * kLoads + k * THREADS + (int)threadIdx.x, n_vec - 1) * kPer));
        };
        auto take = [&](const u32x4 (&x)[kLoads], int p) {
            if ((p + 1) * THREADS * kLoads <= n_vec) {
#pragma unroll
                for (int k = 0; k < kLoads; ++k) add(x[k]);
            } else {
#pragma unroll
                for (int k = 0; k < kLoads; ++k)
                    if (p * THREADS * kLoads + k * THREADS + (int)threadIdx.x < n_vec) add(x[k]);
            }
        };
        if (n_vec > 0) {
            const int n_piece = (a.V + kPiece - 1) / kPiece;
            issue(w[0], 0);
            for (int p = 0; p < n_piece; p += 2) {
                if (p + 1 < n_piece) issue(w[1], p + 1);
                take(w[0], p);
                if (p + 1 >= n_piece) break;
                if (p + 2 < n_piece) issue(w[0], p + 2);
                take(w[1], p + 1);
            }
        }
        const int tail = n_vec * kPer + (int)threadIdx.x;
        if (tail < a.V) count += score<T>(z, tail) > mine;  // (fewer than kPer scores)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o, kWave);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = count;
        __syncthreads();
#pragma unroll
        for (int w_ = 0; w_ < THREADS / 64; ++w_) rank += part[w_];
    }
    if (threadIdx.x == 0) {
        a.rank[d] = rank;
        const int own = q0 + j + 1;  // the row whose input the draft is
        if (own < q1 && own < a.N_cap) a.keep[own] = rank < a.K ? 1 : 0;
    }
}

}  // namespace
}  // namespace fsr

using namespace fsr;

extern "C" int fsr_topk_rank_check(const void* logits, const int32_t* draft_tokens, const int32_t* cu_q,
                                   const int32_t* cu_d, int32_t* rank, uint8_t* keep_mask,
                                   const fsr_rank_params* p, void* stream) {
    if (!p) return fail(FSR_EINVAL, "fsr_topk_rank_check: params is null");
    if (p->B < 0 || p->N_cap < 0 || p->D_cap < 0 || p->V <= 0 || p->K < 0 || p->reserved != 0)
        return fail(FSR_EINVAL, "fsr_topk_rank_check: B=%d N_cap=%d D_cap=%d V=%d K=%d reserved=%d", p->B, p->N_cap, p->D_cap,
                    p->V, p->K, p->reserved);
    if (p->dtype != FSR_F32 && p->dtype != FSR_BF16) return fail(FSR_EUNSUP, "fsr_topk_rank_check: dtype=%d", p->dtype);
    if (p->B == 0 || p->N_cap == 0) return FSR_OK;
    if (!logits || !cu_q || !cu_d || !keep_mask || (p->D_cap > 0 && (!draft_tokens || !rank)))
        return fail(FSR_EINVAL, "fsr_topk_rank_check: null pointer among logits/draft_tokens/cu_q/cu_d/rank/keep_mask");
    if (p->D_cap > 65535) return fail(FSR_EUNSUP, "fsr_topk_rank_check: D_cap=%d exceeds 65535 drafts per call", p->D_cap);
    if ((uintptr_t)logits & (p->dtype == FSR_F32 ? 3 : 1)) return fail(FSR_EINVAL, "fsr_topk_rank_check: logits misaligned");
    hipStream_t s = (hipStream_t)stream;
    RankArgs a;
    a.logits = logits; a.draft_tokens = draft_tokens; a.cu_q = cu_q; a.cu_d = cu_d; a.rank = rank; a.keep = keep_mask;
    a.B = p->B; a.V = p->V; a.K = p->K; a.N_cap = p->N_cap; a.D_cap = p->D_cap;
    const bool f32 = p->dtype == FSR_F32;
    const long long row_bytes = (long long)p->V * (f32 ? 4 : 2);
    // (rows of logits that exist bound the live drafts; both sides measured at the top)
    if (p->D_cap > 0 && std::min(p->D_cap, p->N_cap) < pieces_below(row_bytes) && p->D_cap <= kPiecesDrafts) {
        hipLaunchKernelGGL(rank_init_kernel, dim3((p->D_cap + kThreads - 1) / kThreads), dim3(kThreads), 0, s, a);
        const int piece = kChunkBytes / (f32 ? 4 : 2);
        const dim3 pieces((p->V + piece - 1) / piece, p->D_cap);
        if (f32) hipLaunchKernelGGL(rank_count_kernel<float>, pieces, dim3(kThreads), 0, s, a);
        else hipLaunchKernelGGL(rank_count_kernel<uint16_t>, pieces, dim3(kThreads), 0, s, a);
        hipLaunchKernelGGL(rank_mask_kernel, dim3((p->N_cap + kThreads - 1) / kThreads), dim3(kThreads), 0, s, a);
        return check_launch("fsr_topk_rank_check");
    }
    const dim3 grid((unsigned)p->D_cap + (p->N_cap + kMaskRows - 1) / kMaskRows);
#define FSR_RANK(T, THREADS) hipLaunchKernelGGL((rank_check_kernel<T, THREADS>), grid, dim3(THREADS), 0, s, a)
    if (row_bytes >= kLongRow || p->D_cap <= kFewDrafts) {
        if (f32) FSR_RANK(float, 1024); else FSR_RANK(uint16_t, 1024);
    } else {
        if (f32) FSR_RANK(float, 512); else FSR_RANK(uint16_t, 512);
    }
#undef FSR_RANK
    return check_launch("fsr_topk_rank_check");
}
