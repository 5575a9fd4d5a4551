// prune_compact / prune_restore / frontier state kernels (integer work, bit-exact).
//
// The ragged metadata of a verification batch is a few KB (B <= a few thousand requests,
// N <= a few thousand rows), so the offsets and row maps are produced by ONE workgroup that
// walks the requests in tiles of 1024 with a running carry: latency-bound, no inter-block
// synchronisation.  The optional payload gather is the only part that moves real bytes: its workgroups
// (a window of output rows each) work the offsets out once more for themselves, which takes as long as
// it takes the one that writes the maps, instead of waiting for that one in a second launch.
// What bounds that is the chain of loads, scan and copy, so a call of up to 4096 rows gets one workgroup per compute unit
// (255 beside the maps' own) and a small one a row to a workgroup; with more rows twice as many.  Where that is too much for
// the workgroups the rows are moved by a second launch, which cuts wide ones across.
// Measured, us a call, 45 % / 90 % of the rows kept, windows of at least 8 rows in up to 511 workgroups / this / in two launches:
//   64 rows of 8 KB 6.5, 6.7 / 4.7, 4.9 / 6.2, 6.3;  700 7.0, 7.9 / 5.6, 6.7 / 6.6, 7.8;  1400 7.8, 9.1 / 7.4, 9.1 / 7.8, 9.3;
//   64 of 16 KB 8.9, 9.1 / 5.0, 5.2 / 6.3, 6.4;  64 of 32 KB 13.6, 13.8 / 5.5, 5.9 / 6.4, 6.7;  20000 of 8 KB 42, 70 / 42, 70 / 47, 69.
//   In two launches now: 3000 of 8 KB 10.4, 19.7 / 9.4, 16.3 (one launch of 255 10.2, 16.9, with 60 % kept 14.6 and in two 12.4);
//   1400 of 16 KB 12.3, 17.2 / 9.7, 14.9;  64 of 64 KB 24.1, 24.3 / 6.8, 7.6;  64 of 513 KB, 80 % kept, 172 / 13.
// Requests of many rows, 70 % kept up to the first that is not, all mask bytes looked at / up to that row (and the copying workgroups
// not going through rows that they do not take): 64 requests of 20 to 40 rows 11.0 / 8.4, with 8 KB rows 13.3 / 8.8, 250 12.6 / 10.8,
// 19.6 / 15.4, 250 of 100 to 120 31 / 22, 43 / 24.
// 255 against 511 workgroups: 700 rows of 8 KB 5.6, 6.7 / 5.8, 8.3;  20000 rows of 4 KB 33.9, 39.5 / 26.5, 40.5.
#include <algorithm>

#include "common.hpp"
#include "device_utils.hpp"

namespace fsr {

namespace {

constexpr int kScanThreads = 1024;

// Exclusive scan of one value per thread over the block; returns the exclusive prefix and sets `total`.  smem holds two
// buffers of kScanThreads / 64 values; `turn` says which one is used (a buffer is written again two scans later at the
// earliest, with a barrier in between).  Lanes move data by DPP and every wave adds up the waves before it for itself: one
// barrier and no LDS round trips but one.
__device__ __forceinline__ int block_exclusive_scan(int v, int (*smem)[kScanThreads / 64], int& turn, int& total) {
    constexpr int kW = kScanThreads / 64;
    static_assert(kW == 16, "the waves' sums are one row of lanes");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int inc = wave_inclusive_scan_dpp(v);
    int* sums = smem[turn];
    turn ^= 1;
    if (lane == 63) sums[w] = inc;
    __syncthreads();
    const int before = wave_inclusive_scan_dpp(lane < kW ? sums[lane] : 0);
    total = __builtin_amdgcn_readlane(before, kW - 1);
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int base = wu > 0 ? __builtin_amdgcn_readlane(before, max(wu - 1, 0)) : 0;
    return base + inc - v;
}

// Whether rows r0 .. r1 - 1 (mask bytes) are kept, until f says that no further one matters; the bytes of eight rows are sent
// for together.
template <typename F>
__device__ __forceinline__ void for_kept(const uint8_t* __restrict__ keep, int r0, int r1, F&& f) {
    bool more = true;
    for (int r = r0; r < r1 && more; r += 8) {
        uint8_t k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) k[u] = keep[min(r + u, r1 - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (r + u < r1) more = f(r + u, k[u] != 0);
    }
}

struct CompactArgs {
    // keep: the mask; or, when accepted_len is given instead, request i keeps its rows 0 .. accepted_len[i]
    // (the survivors of an accept step; always suffix-closed) and keep_out, if not null, receives that mask.
    const uint8_t* keep;
    const int32_t* accepted_len;
    uint8_t* keep_out;
    const int32_t* cu_q;
    int32_t* new_cu_q;
    int32_t* new_q_lens;
    int32_t* src_row;
    int32_t* dst_row;
    int32_t* n_active;
    int32_t* active_ids;
    int B, N_cap, suffix_close;
    const void* in;  // payload rows of row_vecs vectors, or null
    void* out;
    size_t row_vecs;
    int window;      // output rows of a copying workgroup
};

constexpr int kMaxWindow = 4096;
constexpr int kFewRows = 4096;  // up to so many rows one copying workgroup per compute unit, else as many as run at once

// Whether a payload is copied by the launch that writes the maps: it saves the second launch, but copies at a workgroup's pace
// and before anybody knows how many rows were kept (both sides measured at the top).
constexpr size_t kOneLaunchBytes = 16 << 20, kOneLaunchRow = 32768;
constexpr size_t kNarrowRow = 12288, kManyRows = 6144;  // many narrow rows: the second launch's workgroups per row cost more
bool one_launch(size_t rows, size_t row_bytes) {
    return (row_bytes <= kOneLaunchRow && rows * row_bytes <= kOneLaunchBytes) || (row_bytes <= kNarrowRow && rows > kManyRows);
}

// Workgroup 0 writes the maps; workgroup 1 + k copies the output rows k * window .. of the payload.
template <typename VecT>
__global__ __launch_bounds__(kScanThreads) void prune_compact_kernel(CompactArgs a) {
    __shared__ int smem[2][kScanThreads / 64];
    int turn = 0;
    __shared__ int src_of[kMaxWindow];  // input row of the window's output rows
    const bool maps = blockIdx.x == 0;
    const long long lo = maps ? 0 : (long long)(blockIdx.x - 1) * a.window;  // (N_cap < 2^31: past the end it may exceed an int)
    const int B = a.B, N_cap = a.N_cap;
    int row_carry = 0, act_carry = 0;
    const int N = B > 0 ? min(max(a.cu_q[B], 0), N_cap) : 0;
    if (lo > N) return;
    for (int base = 0; base < B; base += kScanThreads) {
        const int i = base + threadIdx.x;
        int kept = 0, r0 = 0, r1 = 0;
        if (i < B) {
            r0 = min(max(a.cu_q[i], 0), N_cap);  // offsets beyond the allocated rows are cut off
            r1 = min(max(a.cu_q[i + 1], r0), N_cap);
            if (a.accepted_len) {
                kept = min(max(a.accepted_len[i] + 1, 0), r1 - r0);
            } else {
                bool open = true;  // suffix_close: no row so far was dropped
                for_kept(a.keep, r0, r1, [&](int, bool k) {
                    kept += k && open;
                    open = open && (k || !a.suffix_close);
                    return open;
                });
            }
        }
        int tile_rows, tile_act = 0;
        const int off = row_carry + block_exclusive_scan(kept, smem, turn, tile_rows);
        if (maps) {
            const int aoff = act_carry + block_exclusive_scan(kept > 0 ? 1 : 0, smem, turn, tile_act);
            if (i < B) {
                a.new_cu_q[i] = off;
                a.new_q_lens[i] = kept;
                if (kept > 0) a.active_ids[aoff] = i;
            }
        }
        const bool wanted = i < B && (maps || (off < lo + a.window && off + kept > lo));
        if (wanted && (a.accepted_len || a.suffix_close)) {  // the request's first rows
            if (maps) {
                for (int r = r0; r < r1; ++r) {
                    const bool k = r - r0 < kept;
                    if (a.keep_out) a.keep_out[r] = k ? 1 : 0;
                    if (k) a.src_row[off + (r - r0)] = r;
                    a.dst_row[r] = k ? off + (r - r0) : -1;
                }
            } else {
                const int o1 = (int)min((long long)off + kept, lo + a.window);
                for (int o = (int)max((long long)off, lo); o < o1; ++o) src_of[o - lo] = r0 + (o - off);
            }
        } else if (wanted) {
            int o = off;
            for_kept(a.keep, r0, r1, [&](int r, bool k) {
                if (maps) {
                    if (k) a.src_row[o] = r;
                    a.dst_row[r] = k ? o : -1;
                } else if (k && o >= lo && o < lo + a.window) {
                    src_of[o - lo] = r;
                }
                o += k;
                return true;
            });
        }
        row_carry += tile_rows;
        act_carry += tile_act;
        if (!maps && row_carry >= lo + a.window) break;  // the window is complete
    }
    if (maps) {
        if (threadIdx.x == 0) {
            a.new_cu_q[B] = row_carry;
            a.n_active[0] = act_carry;
        }
        for (int r = row_carry + threadIdx.x; r < N_cap; r += kScanThreads) a.src_row[r] = -1;
        for (int r = N + threadIdx.x; r < N_cap; r += kScanThreads) a.dst_row[r] = -1;
        for (int k = act_carry + threadIdx.x; k < B; k += kScanThreads) a.active_ids[k] = -1;
        return;
    }
    __syncthreads();
    const int n = (int)min(max(min(row_carry, N_cap) - lo, 0LL), (long long)a.window);
    // a wave takes pieces of four vectors a lane, all in flight together
    constexpr int kPer = 4, kPiece = 64 * kPer, kWavesCopy = kScanThreads / 64;
    const size_t pieces = (a.row_vecs + kPiece - 1) / kPiece;
    const int lane = threadIdx.x & 63;
    for (size_t u = threadIdx.x >> 6; u < (size_t)n * pieces; u += kWavesCopy) {
        const size_t r = u / pieces, v0 = (u - r * pieces) * kPiece + lane;
        const VecT* src = reinterpret_cast<const VecT*>(a.in) + (size_t)src_of[r] * a.row_vecs;
        VecT* dst = reinterpret_cast<VecT*>(a.out) + (size_t)(lo + r) * a.row_vecs;
        if (v0 - lane + kPiece <= a.row_vecs) {
            VecT x[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) x[e] = src[v0 + 64 * e];
#pragma unroll
            for (int e = 0; e < kPer; ++e) dst[v0 + 64 * e] = x[e];
        } else {
            for (size_t v = v0; v < a.row_vecs; v += 64) dst[v] = src[v];
        }
    }
}

// Rows 0 .. n_new[0] - 1 of the compact side: out[r'] = in[src_row[r']] (GATHER), or out[src_row[r']] = in[r'], where rows of
// `out` that no r' maps to keep their contents.
template <typename VecT, bool GATHER>
__global__ __launch_bounds__(256) void move_rows_kernel(const VecT* __restrict__ in, VecT* __restrict__ out,
                                                        const int32_t* __restrict__ src_row, const int32_t* __restrict__ n_new,
                                                        size_t row_vecs, int N_cap) {
    const int n = min(n_new[0], N_cap);
    for (int r = blockIdx.x; r < n; r += gridDim.x) {
        const int d = src_row[r];
        if (d < 0 || d >= N_cap) continue;
        const VecT* src = in + (size_t)(GATHER ? d : r) * row_vecs;
        VecT* dst = out + (size_t)(GATHER ? r : d) * row_vecs;
        for (size_t v = (size_t)blockIdx.y * blockDim.x + threadIdx.x; v < row_vecs; v += (size_t)gridDim.y * blockDim.x)
            dst[v] = src[v];
    }
}

template <typename VecT>
__global__ __launch_bounds__(256) void restore_rows_kernel(const VecT* __restrict__ compact,
                                                           const int32_t* __restrict__ dst_row,
                                                           VecT* __restrict__ restored, uint8_t* __restrict__ has_value,
                                                           size_t row_vecs, int N, VecT pad) {
    for (int r = blockIdx.x; r < N; r += gridDim.x) {
        const int s = dst_row[r];
        VecT* dst = restored + (size_t)r * row_vecs;
        if (s >= 0) {
            const VecT* src = compact + (size_t)s * row_vecs;
            for (size_t v = (size_t)blockIdx.y * blockDim.x + threadIdx.x; v < row_vecs; v += (size_t)gridDim.y * blockDim.x)
                dst[v] = src[v];
        } else {
            for (size_t v = (size_t)blockIdx.y * blockDim.x + threadIdx.x; v < row_vecs; v += (size_t)gridDim.y * blockDim.x)
                dst[v] = pad;
        }
        if (has_value && blockIdx.y == 0 && threadIdx.x == 0) has_value[r] = s >= 0 ? 1 : 0;
    }
}

// keep[r] = 1 for rows 0 .. accepted_len[i] of request i (the rows whose tokens stay committed after
// the accept step: the last committed token and the accepted drafts), 0 for the rejected suffix.
__global__ void survivor_mask_kernel(const int32_t* __restrict__ accepted_len, const int32_t* __restrict__ cu_q,
                                     uint8_t* __restrict__ keep, int B, int N_cap) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    const int r0 = min(max(cu_q[i], 0), N_cap), r1 = min(max(cu_q[i + 1], r0), N_cap);
    const int n = accepted_len[i];
    for (int r = r0; r < r1; ++r) keep[r] = (r - r0 <= n) ? 1 : 0;
}

__global__ void frontier_init_kernel(const int32_t* __restrict__ spec_lens, int32_t* pos, int32_t* active,
                                     int32_t* n_out, int32_t* acc_total, int32_t* out_tokens, int B, int out_stride) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    pos[i] = 0;
    active[i] = 1;
    n_out[i] = 0;
    acc_total[i] = 0;
    for (int s = 0; s < out_stride; ++s) out_tokens[(size_t)i * out_stride + s] = -1;
}

__global__ void frontier_plan_kernel(const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ spec_lens,
                                     const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_d,
                                     const int32_t* __restrict__ pos, const int32_t* __restrict__ active,
                                     const int32_t* __restrict__ chunk_len, uint8_t* __restrict__ t_mask,
                                     uint8_t* __restrict__ d_mask, int32_t* __restrict__ chunk_ctx, int B,
                                     int N_t_cap, int N_d_cap) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    const int t0 = cu_q[i], t1 = min(cu_q[i + 1], N_t_cap), d0 = cu_d[i], d1 = min(cu_d[i + 1], N_d_cap);
    const int s = spec_lens[i], p = pos[i];
    int nk = 0, nt = 0;
    if (active[i]) {
        nk = max(0, min(chunk_len[i], s - p));
        // the bonus row rides with the chunk that verifies the last draft (or is the only
        // row of a request without drafts)
        const bool last = (p + nk == s) && (nk > 0 || s == 0);
        nt = nk + (last ? 1 : 0);
    }
    for (int r = t0; r < t1; ++r) t_mask[r] = (r - t0 >= p && r - t0 < p + nt) ? 1 : 0;
    for (int r = d0; r < d1; ++r) d_mask[r] = (r - d0 >= p && r - d0 < p + nk) ? 1 : 0;
    chunk_ctx[i] = ctx_lens[i] + p;
}

__global__ void frontier_commit_kernel(const int32_t* __restrict__ spec_lens, const int32_t* __restrict__ chunk_len,
                                       const int32_t* __restrict__ accepted_len, const int32_t* __restrict__ n_emitted,
                                       const int32_t* __restrict__ emitted, int emitted_stride, int32_t* pos,
                                       int32_t* active, int32_t* n_out, int32_t* acc_total, int32_t* out_tokens, int B,
                                       int out_stride) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    if (!active[i]) return;
    const int s = spec_lens[i], p = pos[i];
    const int nk = max(0, min(chunk_len[i], s - p));
    const int ne = max(0, min(n_emitted[i], emitted_stride));
    int o = n_out[i];
    for (int e = 0; e < ne && o < out_stride; ++e, ++o) out_tokens[(size_t)i * out_stride + o] = emitted[(size_t)i * emitted_stride + e];
    n_out[i] = o;
    const int a = accepted_len[i];
    acc_total[i] += max(a, 0);
    pos[i] = p + nk;
    if (a < nk || p + nk >= s) active[i] = 0;
}

template <typename F>
int launch_by_width(size_t row_bytes, const void* a, const void* b, F&& f) {
    const uintptr_t bits = (uintptr_t)a | (uintptr_t)b | (uintptr_t)row_bytes;
    if ((bits & 15) == 0) return f(uint4{}, row_bytes / 16);
    return f(uint32_t{}, row_bytes / 4);
}

template <bool GATHER>
int move_rows(const void* in, void* out, const int32_t* src_row, const int32_t* n_new, size_t row_bytes, int N_cap, hipStream_t s) {
    return launch_by_width(row_bytes, in, out, [&](auto tag, size_t row_vecs) {
        using VecT = decltype(tag);
        const unsigned gy = (unsigned)std::min<size_t>(std::max<size_t>(1, (row_vecs + 255) / 256), 64);
        const unsigned gx = (unsigned)std::min(N_cap, 65535);
        hipLaunchKernelGGL((move_rows_kernel<VecT, GATHER>), dim3(gx, gy), dim3(256), 0, s, (const VecT*)in, (VecT*)out, src_row, n_new,
                           row_vecs, N_cap);
        return check_launch("move_rows_kernel");
    });
}

struct Span {
    const void* at;
    size_t bytes;
};
bool overlap(const Span& a, const Span& b) {
    const uintptr_t x = (uintptr_t)a.at, y = (uintptr_t)b.at;
    return x && y && x < y + b.bytes && y < x + a.bytes;
}

}  // namespace
}  // namespace fsr

using namespace fsr;

namespace {
// Both compaction entry points: the kept rows come from keep_mask, or from accepted_len (then keep_out, nullable,
// receives the mask and the rule is suffix-closed by construction).
int compact_call(const char* who, const uint8_t* keep_mask, const int32_t* accepted_len, uint8_t* keep_out, const int32_t* cu_q,
                 int32_t* new_cu_q, int32_t* new_q_lens, int32_t* src_row, int32_t* dst_row, int32_t* n_active,
                 int32_t* active_ids, const void* payload_in, void* payload_out, size_t row_bytes, const fsr_prune_params* p,
                 void* stream) {
    if (!p) return fail(FSR_EINVAL, "%s: params is null", who);
    if (p->B < 0 || p->N_cap < 0 || p->reserved != 0) return fail(FSR_EINVAL, "%s: B=%d N_cap=%d reserved=%d", who, p->B, p->N_cap, p->reserved);
    if (!cu_q || !new_cu_q || !n_active) return fail(FSR_EINVAL, "%s: cu_q/new_cu_q/n_active is null", who);
    if (p->B > 0 && (!new_q_lens || !active_ids)) return fail(FSR_EINVAL, "%s: new_q_lens/active_ids is null", who);
    if (p->N_cap > 0 && ((!keep_mask && !accepted_len) || !src_row || !dst_row))
        return fail(FSR_EINVAL, "%s: %s/src_row/dst_row is null", who, accepted_len || keep_out ? "accepted_len" : "keep_mask");
    if ((payload_in == nullptr) != (payload_out == nullptr)) return fail(FSR_EINVAL, "%s: payload_in and payload_out must both be given or both be null", who);
    if (payload_in && (row_bytes == 0 || row_bytes % 4 != 0)) return fail(FSR_ESHAPE, "%s: row_bytes=%zu must be a positive multiple of 4", who, row_bytes);
    if (payload_in && payload_in == payload_out) return fail(FSR_EINVAL, "%s: payload gather cannot run in place", who);
    hipStream_t s = (hipStream_t)stream;
    CompactArgs a{keep_mask, accepted_len, keep_out, cu_q, new_cu_q, new_q_lens, src_row, dst_row, n_active, active_ids, p->B, p->N_cap,
                  accepted_len ? 1 : p->suffix_close, nullptr, nullptr, 0, 0};
    const size_t B = p->B, N = p->N_cap;
    // The copying workgroups read the offsets, the mask (or lengths) and the payload while the first one writes the maps: where
    // these share memory (a batch re-packed in place: new_cu_q is cu_q, new_q_lens accepted_len) the maps come first, and the
    // rows in a launch behind them that reads nothing but src_row.
    const Span reads[] = {{cu_q, (B + 1) * 4}, {keep_mask, N}, {accepted_len, B * 4}, {payload_in, N * row_bytes}};
    const Span maps[] = {{new_cu_q, (B + 1) * 4}, {new_q_lens, B * 4}, {src_row, N * 4}, {dst_row, N * 4}, {n_active, 4}, {active_ids, B * 4}, {keep_out, N}};
    bool shared = false;
    for (const Span& r : reads) {
        for (const Span& w : maps) shared |= overlap(r, w);
        if (r.at != payload_in) shared |= overlap(r, Span{payload_out, N * row_bytes});
    }
    if (!payload_in || N == 0 || shared || !one_launch(N, row_bytes)) {
        hipLaunchKernelGGL(prune_compact_kernel<uint32_t>, dim3(1), dim3(kScanThreads), 0, s, a);
        const int rc = check_launch("prune_compact_kernel");
        if (rc != FSR_OK || !payload_in || N == 0) return rc;
        return move_rows<true>(payload_in, payload_out, src_row, new_cu_q + p->B, row_bytes, p->N_cap, s);
    }
    a.in = payload_in;
    a.out = payload_out;
    a.window = std::min(p->N_cap / (p->N_cap <= kFewRows ? 255 : 511) + 1, kMaxWindow);
    return launch_by_width(row_bytes, payload_in, payload_out, [&](auto tag, size_t row_vecs) {
        using VecT = decltype(tag);
        a.row_vecs = row_vecs;
        hipLaunchKernelGGL(prune_compact_kernel<VecT>, dim3(1 + (p->N_cap - 1) / a.window + 1), dim3(kScanThreads), 0, s, a);
        return check_launch("prune_compact_kernel");
    });
}
}  // namespace

extern "C" int fsr_prune_compact(const uint8_t* keep_mask, const int32_t* cu_q, int32_t* new_cu_q,
                                 int32_t* new_q_lens, int32_t* src_row, int32_t* dst_row, int32_t* n_active,
                                 int32_t* active_ids, const void* payload_in, void* payload_out, size_t row_bytes,
                                 const fsr_prune_params* p, void* stream) {
    return compact_call("fsr_prune_compact", keep_mask, nullptr, nullptr, cu_q, new_cu_q, new_q_lens, src_row, dst_row, n_active,
                        active_ids, payload_in, payload_out, row_bytes, p, stream);
}

extern "C" int fsr_survivor_compact(const int32_t* accepted_len, const int32_t* cu_q, uint8_t* keep_mask, int32_t* new_cu_q,
                                    int32_t* new_q_lens, int32_t* src_row, int32_t* dst_row, int32_t* n_active,
                                    int32_t* active_ids, const void* payload_in, void* payload_out, size_t row_bytes,
                                    const fsr_prune_params* p, void* stream) {
    if (p && p->B > 0 && !accepted_len) return fail(FSR_EINVAL, "fsr_survivor_compact: accepted_len is null");
    return compact_call("fsr_survivor_compact", nullptr, accepted_len, keep_mask, cu_q, new_cu_q, new_q_lens, src_row, dst_row,
                        n_active, active_ids, payload_in, payload_out, row_bytes, p, stream);
}

extern "C" int fsr_prune_restore(const void* compact, const int32_t* dst_row, void* restored, uint8_t* has_value,
                                 size_t row_bytes, int32_t N, uint32_t pad_word, void* stream) {
    if (N < 0) return fail(FSR_EINVAL, "fsr_prune_restore: N=%d", N);
    if (N == 0) return FSR_OK;
    if (!compact || !dst_row || !restored) return fail(FSR_EINVAL, "fsr_prune_restore: null pointer");
    if (row_bytes == 0 || row_bytes % 4 != 0) return fail(FSR_ESHAPE, "fsr_prune_restore: row_bytes=%zu must be a positive multiple of 4", row_bytes);
    if (compact == restored) return fail(FSR_EINVAL, "fsr_prune_restore: cannot run in place");
    hipStream_t s = (hipStream_t)stream;
    return launch_by_width(row_bytes, compact, restored, [&](auto tag, size_t row_vecs) {
        using VecT = decltype(tag);
        VecT pad;
        if constexpr (sizeof(VecT) == 16) pad = uint4{pad_word, pad_word, pad_word, pad_word};
        else pad = pad_word;
        const unsigned gy = (unsigned)std::min<size_t>(std::max<size_t>(1, (row_vecs + 255) / 256), 64);
        const unsigned gx = (unsigned)std::min(N, 65535);
        hipLaunchKernelGGL(restore_rows_kernel<VecT>, dim3(gx, gy), dim3(256), 0, s, (const VecT*)compact, dst_row,
                           (VecT*)restored, has_value, row_vecs, N, pad);
        return check_launch("restore_rows_kernel");
    });
}

extern "C" int fsr_prune_scatter(const void* compact, const int32_t* src_row, const int32_t* n_rows, void* out,
                                 size_t row_bytes, int32_t N_cap, void* stream) {
    if (N_cap < 0) return fail(FSR_EINVAL, "fsr_prune_scatter: N_cap=%d", N_cap);
    if (N_cap == 0) return FSR_OK;
    if (!compact || !src_row || !n_rows || !out) return fail(FSR_EINVAL, "fsr_prune_scatter: null pointer");
    if (row_bytes == 0 || row_bytes % 4 != 0) return fail(FSR_ESHAPE, "fsr_prune_scatter: row_bytes=%zu must be a positive multiple of 4", row_bytes);
    if (compact == out) return fail(FSR_EINVAL, "fsr_prune_scatter: cannot run in place");
    return move_rows<false>(compact, out, src_row, n_rows, row_bytes, N_cap, (hipStream_t)stream);
}

extern "C" int fsr_survivor_mask(const int32_t* accepted_len, const int32_t* cu_q, uint8_t* keep_mask, int32_t B,
                                 int32_t N_cap, void* stream) {
    if (B < 0 || N_cap < 0) return fail(FSR_EINVAL, "fsr_survivor_mask: B=%d N_cap=%d", B, N_cap);
    if (B == 0 || N_cap == 0) return FSR_OK;
    if (!accepted_len || !cu_q || !keep_mask) return fail(FSR_EINVAL, "fsr_survivor_mask: null pointer");
    hipLaunchKernelGGL(survivor_mask_kernel, dim3((B + 255) / 256), dim3(256), 0, (hipStream_t)stream, accepted_len, cu_q,
                       keep_mask, B, N_cap);
    return check_launch("survivor_mask_kernel");
}

extern "C" int fsr_frontier_init(const int32_t* spec_lens, int32_t* pos, int32_t* active, int32_t* n_out,
                                 int32_t* acc_total, int32_t* out_tokens, int32_t B, int32_t out_stride, void* stream) {
    if (B < 0 || out_stride < 0) return fail(FSR_EINVAL, "fsr_frontier_init: B=%d out_stride=%d", B, out_stride);
    if (B == 0) return FSR_OK;
    if (!spec_lens || !pos || !active || !n_out || !acc_total || !out_tokens) return fail(FSR_EINVAL, "fsr_frontier_init: null pointer");
    hipLaunchKernelGGL(frontier_init_kernel, dim3((B + 255) / 256), dim3(256), 0, (hipStream_t)stream, spec_lens, pos, active,
                       n_out, acc_total, out_tokens, B, out_stride);
    return check_launch("frontier_init_kernel");
}

extern "C" int fsr_frontier_plan(const int32_t* ctx_lens, const int32_t* spec_lens, const int32_t* cu_q,
                                 const int32_t* cu_d, const int32_t* pos, const int32_t* active,
                                 const int32_t* chunk_len, uint8_t* t_mask, uint8_t* d_mask, int32_t* chunk_ctx,
                                 int32_t B, int32_t N_t_cap, int32_t N_d_cap, void* stream) {
    if (B < 0 || N_t_cap < 0 || N_d_cap < 0) return fail(FSR_EINVAL, "fsr_frontier_plan: B=%d N_t_cap=%d N_d_cap=%d", B, N_t_cap, N_d_cap);
    if (B == 0) return FSR_OK;
    if (!ctx_lens || !spec_lens || !cu_q || !cu_d || !pos || !active || !chunk_len || !chunk_ctx) return fail(FSR_EINVAL, "fsr_frontier_plan: null pointer");
    if ((N_t_cap > 0 && !t_mask) || (N_d_cap > 0 && !d_mask)) return fail(FSR_EINVAL, "fsr_frontier_plan: mask is null");
    hipLaunchKernelGGL(frontier_plan_kernel, dim3((B + 255) / 256), dim3(256), 0, (hipStream_t)stream, ctx_lens, spec_lens, cu_q,
                       cu_d, pos, active, chunk_len, t_mask, d_mask, chunk_ctx, B, N_t_cap, N_d_cap);
    return check_launch("frontier_plan_kernel");
}

extern "C" int fsr_frontier_commit(const int32_t* spec_lens, const int32_t* chunk_len, const int32_t* accepted_len,
                                   const int32_t* n_emitted, const int32_t* emitted, int32_t emitted_stride,
                                   int32_t* pos, int32_t* active, int32_t* n_out, int32_t* acc_total,
                                   int32_t* out_tokens, int32_t B, int32_t out_stride, void* stream) {
    if (B < 0 || emitted_stride < 1 || out_stride < 1) return fail(FSR_EINVAL, "fsr_frontier_commit: B=%d emitted_stride=%d out_stride=%d", B, emitted_stride, out_stride);
    if (B == 0) return FSR_OK;
    if (!spec_lens || !chunk_len || !accepted_len || !n_emitted || !emitted || !pos || !active || !n_out || !acc_total || !out_tokens)
        return fail(FSR_EINVAL, "fsr_frontier_commit: null pointer");
    hipLaunchKernelGGL(frontier_commit_kernel, dim3((B + 255) / 256), dim3(256), 0, (hipStream_t)stream, spec_lens, chunk_len,
                       accepted_len, n_emitted, emitted, emitted_stride, pos, active, n_out, acc_total, out_tokens, B, out_stride);
    return check_launch("frontier_commit_kernel");
}
