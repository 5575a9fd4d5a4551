// Verification attention (Sec. 2.1 / 3.1) for the shapes the stream kernel of verify_attention.hip is not built for:
// fp32 inputs, heads of 64, page sizes other than 16, more than 16 query heads per KV head, very large batches.
// Nothing is handed from one workgroup to another, so the call needs no workspace, except that bf16 items of a small call, and
// the long ones of a larger call, are cut into pieces of their keys where the caller brings scratch memory for them.
//
// What bounds it is reading K and V (bf16) or the fp32 matrix instructions (fp32), so the work is laid out to read a
// request's keys once per KV head: one workgroup per (request, KV head, group of up to 16 * MT query rows), its waves
// take the keys' tiles in turn and are merged through LDS at the end.  Longer suffixes than a group holds are further
// workgroups (grid.z), or further rounds of the same one where there are more groups than workgroups.  A ragged
// batch loads the compute units unevenly, but a compute unit draws about twice its even share of the HBM bandwidth
// when others are idle, which covers a longest context of twice the mean.
//   bf16: 32-key tiles.  Whole key rows are loaded (1 KB of consecutive bytes per load, each lane 16) and put through
//     wave-private swizzled LDS tiles, from which K is read as matrix operand and V transposed; while a tile is worked
//     on, the next one is in flight in registers, and the places of the keys of the one after it.  Probabilities go to
//     the matrix cores as three bf16 terms, which together are the fp32 value exactly (two terms, 17 bits: 39 instead of
//     42 us at the first shape below, but errors of 4e-6 of the largest value before the output's rounding, not 5e-7).
//     A wave spends about as many cycles on its vector instructions as on waiting, so two waves per SIMD matter more
//     than a second tile in flight: at 32 requests of 256 to 4096 tokens, 8 KV heads, D = 64, bf16, and two terms, 36 us
//     as built, 45 us with two tiles in flight (the registers spill), 59 us with four waves of 512 registers.
//   fp32: 16-key tiles on v_mfma_f32_16x16x4_f32, operands straight from memory in the operand layout.
// All global accesses are declared with the element's alignment only (the hardware takes unaligned vectors).
//
// Measured, us a call, against one wave per (row, query head) with vector FMAs, which re-reads the keys for each of them:
//   bf16 D = 64, 32/8 heads, 32 requests of 256-4096 tokens, 1-8 drafts      718 -> 42
//   bf16 D = 64, 32/8 heads, 1 request of 8192 tokens, no drafts             317 -> 54 (eight workgroups in all)
//   bf16 D = 64, 32/32 heads, 64 requests of 256-4096 tokens, 0-7 drafts     1282 -> 193
//   bf16 D = 128, 64/2 heads, 16 requests of 1024-2048 tokens, 1-8 drafts    761 -> 64
//   fp32 D = 128, 32/8 heads, 32 requests of 1024-2048 tokens, 1-8 drafts    1586 -> 142
//   fp32 D = 64, 8/2 heads, 4 requests of 64-256 tokens, 0-4 drafts          20 -> 9 (kernel)
#include "attend_items.hpp"

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "device_utils.hpp"

namespace fsr {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
// 16 bytes of global memory aligned to the element type only
typedef __attribute__((__vector_size__(16), __aligned__(2))) uint32_t gu32x4;
typedef __attribute__((__vector_size__(16), __aligned__(4))) float gf32x4;

constexpr double kLog2e = 1.4426950408889634074;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kMaxSplits = 8;
constexpr int kSplitKeys = 512;            // an item is not cut into pieces of fewer keys
constexpr long long kSplitGroups = 256;    // workgroups a call is brought up to by cutting items: one per compute unit
// Calls of many items cut the longest by their lengths, see BalancedPieces and, for the rule, layout_of.  us a call: a base of 2 /
// 4 / 8 for a tile 48 requests of 256-4096 tokens 56.6 / 56.6 / 63.3, 20 28.4 / 28.5 / 30.0, 40 log-normal 54.9 / 59.2 / 59.7, 16/16 heads, 16 of
// 256-4096 35.1 / 32.8 / 32.8; pieces of 4 / 8 / 16 tiles 32 of up to 2048 25.2 / 25.2 / 26.2, others alike.
constexpr int kBalancedMaxB = 64;          // a request per lane
constexpr int kBalancedKeys = 1536;        // keys from which an item is worth cutting
constexpr int kPieceTiles = 8;             // least tiles of a piece that is handed over
constexpr float kTileBase = 4.0f;          // a tile costs this + the query tiles that ride on it
constexpr float kWorthCutting = 110.0f;    // what cutting has to take off at least, in those costs of four waves
enum : int { kWhole = 0, kEven = 1, kBalanced = 2 };  // how items are cut

struct ItemArgs {
    const void* q;
    const void* k;
    const void* v;
    const int32_t* bt;
    const int32_t* ctx;
    const int32_t* cu_q;
    void* out;
    float* lse;
    int B, N_cap, H_q, H_kv, G, P, p_shift, max_pages, n_pages;  // p_shift: log2(P), or -1 if P is no power of two
    int out_bf16;
    long long page_stride, slot_stride, head_stride;  // of the caches, in bytes
    // bf16: an item is cut into up to `splits` pieces of at least kSplitKeys keys, handed over through the workspace
    int splits;
    int places;      // balanced pieces: how many a call has at most, two to a workgroup
    float* part_o;   // [items * splits, or places][16 * MTMAX][D] unnormalised sums of the pieces
    float* part_ml;  // [items * splits, or places][16 * MTMAX][4] exponent reference (log2), sum, call tag, unused
    unsigned long long* arrivals;  // [items] (call id << 16 | pieces that have arrived)
    unsigned long long call_id;
    float scale_log2, scale_rest;  // softmax scale times log2(e), and (times ln 2) what rounding took off it
};

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ __forceinline__ void lds_fence() {  // orders a wave's own LDS accesses (it issues them in order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

template <bool BF16, int D, int MT, int CUT>
struct Map {
    // waves of a workgroup: eight at 256 registers each, or four at 512 where a tile in flight and the accumulators
    // need more than that (measured by the compiler's spill counts)
    static constexpr bool kLarge = D == 128 || MT == 4;
    static constexpr int kW = kLarge ? 4 : 8;
    static constexpr int kParts = CUT == kBalanced ? 2 : 1;  // items that a workgroup may work on side by side
    static constexpr int kThreads = kW * 64;
    static constexpr int kPerSimd = kLarge ? 1 : 2;          // waves that share a SIMD
    static constexpr int kElem = BF16 ? 2 : 4;
    static constexpr int kTile = BF16 ? 32 : 16;             // keys of a wave tile
    static constexpr int kKt = kTile / 16;
    static constexpr int kRow = D * kElem;                   // bytes of a key row
    static constexpr int kQPieces = kRow / 64;               // 1 KB operand pieces of a query tile (64 B of each of 16 rows)
    static constexpr int kStage = BF16 ? kW * 2 * kTile * kRow : 0;  // K and V tiles of the waves
    static constexpr int kRedStride = D + 4;                 // floats
    static constexpr int kRed = kW * 16 * kRedStride * 4;    // one query tile's accumulators of all waves
    static constexpr int kShared = kStage > kRed ? kStage : kRed;
    static constexpr int kMl = kShared;                      // references and sums of all waves
    static constexpr int kQ = kMl + 2 * kW * 16 * MT * 4;
    static constexpr int kSmem = kQ + kParts * MT * kQPieces * 1024;
};

// LDS places of 16-byte chunk ch of key row `row`, such that the accesses of 16 lanes cover all banks: K is written and
// read row by row and chunk by chunk, V read transposed in pieces of two neighbouring chunks.
template <int D>
__device__ __forceinline__ int k_off(int row, int ch) {
    return D == 64 ? row * 128 + ((ch ^ ((row >> 1) & 7)) << 4) : row * 256 + ((ch ^ (row & 15)) << 4);
}
template <int D>
__device__ __forceinline__ int v_off(int row, int ch) {
    return D == 64 ? row * 128 + ((ch ^ (((row >> 1) & 3) << 1)) << 4) : row * 256 + ((ch ^ ((row & 7) << 1)) << 4);
}

template <bool NT>
__device__ __forceinline__ u32x4 load16(const char* p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const gu32x4*>(p));
    else return *reinterpret_cast<const gu32x4*>(p);
}

// Stores through to memory, past the die's L2, for what another workgroup of the launch reads.
__device__ __forceinline__ void store_device(float* base, long long at, f32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000),
                                           (int)(at * 4), 0, 16);
}

__device__ __forceinline__ void write_out(const ItemArgs& a, size_t at, float x) {
    if (a.out_bf16) reinterpret_cast<uint16_t*>(a.out)[at] = to_bf16(x);
    else reinterpret_cast<float*>(a.out)[at] = x;
}

// The pieces of an item's rows m0 .. m0 + rows - 1, slots slot0, next, next + step, .., n of them, to the rows themselves: four
// values of a row to a thread at a time.  Ordinary loads: a slot was stored through to memory before its piece was counted, is written and
// read once per launch, and caches start a launch without older copies.  A slot that this call did not write makes its rows NaN.
template <int D, int ROWS>
__device__ __forceinline__ void combine_pieces(const ItemArgs& a, int g, int q0, int m0, int rows, int slot0, int next, int step, int n,
                                               int thread, int threads) {
    for (int e = thread; e < rows * (D / 4); e += threads) {
        const int m = e / (D / 4), d0 = (e % (D / 4)) * 4;
        f32x4 ml[kMaxSplits], o[kMaxSplits];
#pragma unroll
        for (int k = 0; k < kMaxSplits; ++k) {  // past the last piece: it again, left out below
            const int p = min(k, n - 1);
            const long long row = (long long)(p == 0 ? slot0 : next + (p - 1) * step) * ROWS + m;
            ml[k] = *reinterpret_cast<const f32x4*>(a.part_ml + row * 4);
            o[k] = *reinterpret_cast<const f32x4*>(a.part_o + row * D + d0);
        }
        float top = -INFINITY, sum = 0.0f;
#pragma unroll
        for (int k = 0; k < kMaxSplits; ++k)
            if (k < n) top = fmaxf(top, ml[k][0]);
        const float ref = top == -INFINITY ? 0.0f : top;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kMaxSplits; ++k) {
            const float tag = ml[k][2];
            float w = exp2_fast(ml[k][0] - ref);
            if (__builtin_bit_cast(uint32_t, tag) != (uint32_t)a.call_id) w = __builtin_nanf("");
            if (k < n) {
                sum = fmaf(ml[k][1], w, sum);
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[u] = fmaf(o[k][u], w, acc[u]);
            }
        }
        const int j = (m0 + m) / a.G, h = g * a.G + (m0 + m) % a.G;
        const size_t at = ((size_t)(q0 + j) * a.H_q + h) * D + d0;
        const float inv = 1.0f / sum;
#pragma unroll
        for (int u = 0; u < 4; ++u) write_out(a, at + u, acc[u] * inv);
        if (a.lse && d0 == 0) a.lse[(size_t)(q0 + j) * a.H_q + h] = top * kLn2 + logf(sum);
    }
}

// Who works on a piece: the waves of the workgroup, all on one or (balanced) on two consecutive ones, or each four on one; the item's
// keys are shared by `of` such parts.
struct Part {
    int waves, of;
    int slot;  // (evenly cut) of the piece in the workspace
};

// Query rows m0 .. of item (request i, KV head g), at most 16 * MT of them: stream the keys they see (piece sp of n_sp of
// them), merge the waves, write the rows (or the piece's sums to the workspace).  MTMAX: what the LDS is laid out for.
template <bool BF16, int D, int MTMAX, int MT, bool NT, int CUT>
__device__ __forceinline__ void attend_group(const ItemArgs& a, char* smem, int i, int g, int q0, int M, int c, int m0, int sp, int n_sp,
                                             const Part& part) {
    typedef Map<BF16, D, MTMAX, CUT> L;
    constexpr bool SPLIT = CUT != kWhole;
    constexpr int kTile = L::kTile, kKt = L::kKt, kDB = D / 16, kW = L::kW;
    const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6), lg = lane >> 4, li = lane & 15;
    const int kv_cap = (int)min((long long)a.max_pages * a.P, 1LL << 30);
    const int32_t* bt = a.bt + (size_t)i * a.max_pages;
    const char* kc = reinterpret_cast<const char*>(a.k) + (size_t)g * a.head_stride;
    const char* vc = reinterpret_cast<const char*>(a.v) + (size_t)g * a.head_stride;
    // the waves of the item: all, or four of them; this one's place among them
    const int n_waves = CUT == kBalanced ? part.waves : kW, wi = CUT == kBalanced ? w & (n_waves - 1) : w;
    char* qbuf = smem + L::kQ + (CUT == kBalanced && wi != w ? MT * L::kQPieces * 1024 : 0);
    float* red_m = reinterpret_cast<float*>(smem + L::kMl);  // [kW][16 * MT]
    float* red_l = red_m + kW * 16 * MT;
    char* kbuf = smem + w * 2 * kTile * L::kRow;  // the wave's tiles (bf16)
    char* vbuf = kbuf + kTile * L::kRow;

    const int rows = min(16 * MT, M - m0);
    const int first_lim = c + m0 / a.G;                           // last key the group's first row sees
    int kend = min(c + (m0 + rows - 1) / a.G + 1, kv_cap);  // keys any row of the group sees
    int kb0 = wi * kTile;
    if (SPLIT && part.of > 1) {  // the piece's even share of their tiles (at most 2^30 keys and eight pieces: the products fit 32 bits)
        const unsigned n_tiles = (unsigned)(kend + kTile - 1) / kTile;
        const int upto = sp + (CUT == kBalanced ? part.waves >> 2 : 1);
        kb0 += (int)(n_tiles * sp / n_sp) * kTile;
        if (upto < n_sp) kend = (int)(n_tiles * upto / n_sp) * kTile;
    }
    const int step = n_waves * kTile;
    const int nw = rows > 0 && kb0 < kend ? (kend - kb0 + step - 1) / step : 0;
    // the wave's first n_plain tiles lie wholly below every row's causal limit
    const int below = min(first_lim + 1, kend) - kTile - kb0;
    // (none where the group has no rows: the other item of the workgroup has more rounds, and this one has loaded nothing)
    const int n_plain = min(nw, below < 0 ? 0 : below / step + 1);

    // ---- query operands to LDS: piece (mt, s) holds for lane (li, lg) 16 bytes of row mt * 16 + li
    for (int pr = wi; pr < MT * L::kQPieces; pr += n_waves) {
        const int m = m0 + (pr / L::kQPieces) * 16 + li;
        const bool ok = m < M;
        const int mv = ok ? m : m0 < M ? m0 : 0;  // (the other item of the workgroup may have more rounds than this one)
        const int j = mv / a.G, gq = mv % a.G;
        const char* src = reinterpret_cast<const char*>(a.q) + ((size_t)(q0 + j) * a.H_q + g * a.G + gq) * L::kRow +
                          64 * (pr % L::kQPieces) + 16 * lg;
        u32x4 x = *reinterpret_cast<const gu32x4*>(src);
        if (!ok) x = u32x4{0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(qbuf + (pr * 64 + lane) * 16) = x;
    }
    int lim[MT];  // last key that query row mt * 16 + li sees
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = mt * 16 + li;
        lim[mt] = m < rows ? min(c + (m0 + m) / a.G, kv_cap - 1) : -1;
    }

    // ---- key rows: lane l looks up the place of key kb + l % kTile of a tile (keys past the end: the last one)
    uint32_t at_lo = 0, at_hi = 0;
    auto look_up = [&](int t) {
        const int key = max(min(kb0 + t * step + (lane & (kTile - 1)), kend - 1), 0);
        const int pg = a.p_shift >= 0 ? key >> a.p_shift : key / a.P;
        const int page = min(max(bt[pg], 0), a.n_pages - 1);
        const long long at = page * a.page_stride + (key - pg * a.P) * a.slot_stride;
        at_lo = (uint32_t)at;
        at_hi = (uint32_t)((unsigned long long)at >> 32);
    };
    auto row_at = [&](int r) {  // byte offset of key row r of the tile looked up last
        return (long long)(((unsigned long long)(uint32_t)__shfl((int)at_hi, r, 64) << 32) | (uint32_t)__shfl((int)at_lo, r, 64));
    };
    // registers of a tile in flight.  bf16: load n covers rows n * kRpl + lane / kCh, 16-byte chunk lane % kCh.
    // fp32: K is the matrix operand itself (row li, floats 16 s + 4 lg ..), V[e][db] = V[key 4 lg + e][16 db + li].
    constexpr int kCh = D * 2 / 16, kRpl = 64 / kCh, kLoads = BF16 ? kTile / kRpl : 1;
    u32x4 kr[BF16 ? kLoads : 1], vr[BF16 ? kLoads : 1];
    f32x4 kf[BF16 ? 1 : D / 16];
    float vf[BF16 ? 1 : 4][BF16 ? 1 : kDB];
    auto issue = [&]() {
        if constexpr (BF16) {
            long long at[kLoads];
#pragma unroll
            for (int n = 0; n < kLoads; ++n) at[n] = row_at(n * kRpl + lane / kCh) + (lane % kCh) * 16;
#pragma unroll
            for (int n = 0; n < kLoads; ++n) kr[n] = load16<NT>(kc + at[n]);
#pragma unroll
            for (int n = 0; n < kLoads; ++n) vr[n] = load16<NT>(vc + at[n]);
        } else {
            const char* kp = kc + row_at(li) + 16 * lg;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) kf[s] = *reinterpret_cast<const gf32x4*>(kp + 64 * s);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const char* vp = vc + row_at(4 * lg + e) + 4 * li;
#pragma unroll
                for (int db = 0; db < kDB; ++db) vf[e][db] = *reinterpret_cast<const float*>(vp + 64 * db);
            }
        }
    };

    float m_run[MT], l_run[MT];
    f32x4 acc[MT][kDB];
    auto start = [&]() {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            m_run[mt] = -INFINITY;
            l_run[mt] = 0.0f;
#pragma unroll
            for (int db = 0; db < kDB; ++db) acc[mt][db] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (nw > 0) {
            look_up(0);
            issue();
            look_up(min(1, nw - 1));
        }
    };
    // One tile.  masked: some row does not see all of its keys.  careful: V may hold Inf or NaN, which must reach
    // exactly the rows that see their key, and an infinite value must meet the whole probability and not its zero
    // parts: the sum is formed without the matrix cores.  V may also be so large that it must not meet a probability
    // above 1: the references are the largest scores.
    auto tile = [&](int t, auto masked_, auto careful_) {
        constexpr bool masked = decltype(masked_)::value, careful = decltype(careful_)::value;
        const int kb = kb0 + t * step;
        // ---- scores: s[mt][kt][e] = key kb + 16 kt + 4 lg + e, query row mt * 16 + li
        f32x4 s[MT][kKt];
        float vt[BF16 ? 1 : 4][BF16 ? 1 : kDB];
        if constexpr (BF16) {
#pragma unroll
            for (int n = 0; n < kLoads; ++n) {
                const int row = n * kRpl + lane / kCh, ch = lane % kCh;
                *reinterpret_cast<u32x4*>(kbuf + k_off<D>(row, ch)) = kr[n];
                *reinterpret_cast<u32x4*>(vbuf + v_off<D>(row, ch)) = vr[n];
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                f32x4 chain[4];  // four shorter sums: less rounding, and the matrix instructions need not wait for each other
#pragma unroll
                for (int e = 0; e < 4; ++e) chain[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ss = 0; ss < D / 16; ++ss) {
                    const f32x4 qop = *reinterpret_cast<const f32x4*>(qbuf + ((mt * L::kQPieces + ss) * 64 + lane) * 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        chain[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[ss][e], qop[e], chain[e], 0, 0, 0);
                }
                s[mt][0] = (chain[0] + chain[1]) + (chain[2] + chain[3]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int db = 0; db < kDB; ++db) vt[e][db] = vf[e][db];
        }
        if (t + 1 < nw) {  // the registers are free: send for the next tile, look up the keys of the one after it
            issue();
            look_up(min(t + 2, nw - 1));
        }
        if constexpr (BF16) {
            lds_fence();
            bf16x8 kop[2][D / 32];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int kk = 0; kk < D / 32; ++kk)
                    kop[h][kk] = *reinterpret_cast<const bf16x8*>(kbuf + k_off<D>(16 * h + li, 4 * kk + lg));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                s[mt][0] = s[mt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < D / 32; ++kk) {
                    const bf16x8 qop = *reinterpret_cast<const bf16x8*>(qbuf + ((mt * L::kQPieces + kk) * 64 + lane) * 16);
                    s[mt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[0][kk], qop, s[mt][0], 0, 0, 0);
                    s[mt][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[1][kk], qop, s[mt][1], 0, 0, 0);
                }
            }
        }
        // ---- masking, exponent references (raised, with a rescale, only when a score exceeds one by 2^8)
        float x[MT][4 * kKt], top[MT];
        bool raise = false;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            top[mt] = -INFINITY;
#pragma unroll
            for (int kt = 0; kt < kKt; ++kt)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float z = s[mt][kt][e];
                    if (masked && kb + 16 * kt + 4 * lg + e > lim[mt]) z = -INFINITY;
                    x[mt][kt * 4 + e] = z;
                    top[mt] = fmaxf(top[mt], z);
                }
            top[mt] *= a.scale_log2;
            raise |= top[mt] > m_run[mt] + (careful ? 0.0f : 8.0f);
        }
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float up = fmaxf(top[mt], __shfl_xor(top[mt], 16, 64));
                up = fmaxf(up, __shfl_xor(up, 32, 64));
                const float m_new = fmaxf(m_run[mt], up);
                const float alpha = m_new == -INFINITY ? 1.0f : exp2_fast(m_run[mt] - m_new);
                m_run[mt] = m_new;
                l_run[mt] *= alpha;
#pragma unroll
                for (int db = 0; db < kDB; ++db) acc[mt][db] *= alpha;
            }
        }
        // ---- probabilities in place of the scores; what rounding took off the scale comes back as a factor near 1
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const float neg_m = m_run[mt] == -INFINITY ? 0.0f : -m_run[mt];
            float sum = 0.0f;
#pragma unroll
            for (int e = 0; e < 4 * kKt; ++e) {
                float p = exp2_fast(fmaf(x[mt][e], a.scale_log2, neg_m));
                p = fmaf(p, fmaxf(x[mt][e], -1e30f) * a.scale_rest, p);
                x[mt][e] = p;
                sum += p;
            }
            l_run[mt] += sum;
        }
        // ---- O^T += V^T P^T
        if constexpr (careful) {
#pragma unroll 1
            for (int quad = 0; quad < 4; ++quad)
#pragma unroll
                for (int kt = 0; kt < kKt; ++kt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r = 16 * kt + 4 * quad + e;  // key row of the tile
#pragma unroll
                        for (int db = 0; db < kDB; ++db) {
                            float v4[4];
                            if constexpr (BF16) {
                                const uint2 t2 = *reinterpret_cast<const uint2*>(vbuf + v_off<D>(r, 2 * db + (lg >> 1)) + (lg & 1) * 8);
                                v4[0] = __builtin_bit_cast(float, t2.x << 16);
                                v4[1] = __builtin_bit_cast(float, t2.x & 0xffff0000u);
                                v4[2] = __builtin_bit_cast(float, t2.y << 16);
                                v4[3] = __builtin_bit_cast(float, t2.y & 0xffff0000u);
                            } else {
#pragma unroll
                                for (int u = 0; u < 4; ++u) v4[u] = __shfl(vt[e][db], quad * 16 + 4 * lg + u, 64);
                            }
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt) {
                                const float p = __shfl(x[mt][kt * 4 + e], quad * 16 + li, 64);
                                if (kb + r <= lim[mt]) {
#pragma unroll
                                    for (int u = 0; u < 4; ++u) acc[mt][db][u] = fmaf(p, v4[u], acc[mt][db][u]);
                                }
                            }
                        }
                    }
        } else if constexpr (BF16) {
            bf16x8 vop[kDB];  // element e < 4: key 4 lg + e, e >= 4: key 16 + 4 lg + (e - 4), at d = 16 db + li
#pragma unroll
            for (int db = 0; db < kDB; ++db) {
                const int off = v_off<D>(4 * lg + (li >> 2), 2 * db + ((li & 3) >> 1)) + (li & 1) * 8;
                const s16x4 t0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vbuf + off));
                const s16x4 t1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vbuf + off + 16 * L::kRow));
                vop[db] = __builtin_bit_cast(bf16x8, s16x8{t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]});
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                // x = hi + lo + rest exactly: hi and lo by truncation, 8 bits each
                uint32_t hi[4], lo[4], rest[4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    uint32_t b0 = __builtin_bit_cast(uint32_t, x[mt][e]), b1 = __builtin_bit_cast(uint32_t, x[mt][e + 1]);
                    hi[e >> 1] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                    const float r0 = x[mt][e] - __builtin_bit_cast(float, b0 & 0xffff0000u);
                    const float r1 = x[mt][e + 1] - __builtin_bit_cast(float, b1 & 0xffff0000u);
                    b0 = __builtin_bit_cast(uint32_t, r0);
                    b1 = __builtin_bit_cast(uint32_t, r1);
                    lo[e >> 1] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                    b0 = __builtin_bit_cast(uint32_t, r0 - __builtin_bit_cast(float, b0 & 0xffff0000u));
                    b1 = __builtin_bit_cast(uint32_t, r1 - __builtin_bit_cast(float, b1 & 0xffff0000u));
                    rest[e >> 1] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                }
                const bf16x8 ph = __builtin_bit_cast(bf16x8, u32x4{hi[0], hi[1], hi[2], hi[3]});
                const bf16x8 pl = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], lo[2], lo[3]});
                const bf16x8 pr = __builtin_bit_cast(bf16x8, u32x4{rest[0], rest[1], rest[2], rest[3]});
#pragma unroll
                for (int db = 0; db < kDB; ++db) {
                    acc[mt][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[db], pr, acc[mt][db], 0, 0, 0);
                    acc[mt][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[db], pl, acc[mt][db], 0, 0, 0);
                    acc[mt][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[db], ph, acc[mt][db], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int db = 0; db < kDB; ++db)
                        acc[mt][db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vt[e][db], x[mt][e], acc[mt][db], 0, 0, 0);
        }
        if constexpr (BF16) lds_fence();  // the next tile's stores must not overtake this tile's reads
    };
    start();
    __syncthreads();  // the query operands are staged
    int t = 0;
#pragma unroll 1
    for (; t < n_plain; ++t) tile(t, std::false_type{}, std::false_type{});
#pragma unroll 1
    for (; t < nw; ++t) tile(t, std::true_type{}, std::false_type{});
    // an accumulator that is not finite, or so large that the sum over the waves might not be (each may lie 2^8 above what
    // references without slack give): once more from the start, with care (0 * x is NaN for exactly those)
    float zero = 0.0f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int u = 0; u < 4; ++u) zero = fmaf(acc[mt][db][u] * 0x1p14f, 0.0f, zero);
    if (__builtin_amdgcn_ballot_w64(!(zero == 0.0f)) != 0) {
        start();
#pragma unroll 1
        for (t = 0; t < nw; ++t) tile(t, std::true_type{}, std::true_type{});
    }

    // ---- merge the waves, one query tile at a time
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        l_run[mt] += __shfl_xor(l_run[mt], 16, 64);
        l_run[mt] += __shfl_xor(l_run[mt], 32, 64);
        if (lg == 0) {
            red_m[w * 16 * MT + mt * 16 + li] = m_run[mt];
            red_l[w * 16 * MT + mt * 16 + li] = l_run[mt];
        }
    }
    float* red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        __syncthreads();  // every wave is done with what lies here: its K/V tiles, the previous query tile's sums
#pragma unroll
        for (int db = 0; db < kDB; ++db)
            *reinterpret_cast<f32x4*>(red + (w * 16 + li) * L::kRedStride + db * 16 + 4 * lg) = acc[mt][db];
        __syncthreads();
        // the item's threads sum kPer consecutive values of one row each
        auto sum_rows = [&](auto waves_, int thread, int first) {
            constexpr int kWaves = decltype(waves_)::value, kPer = 16 * D / (64 * kWaves);
            if constexpr (BF16) asm volatile("" : "+v"(thread));  // or the offsets below are made at the kernel's start and spilled
            const int row = thread / (D / kPer), d0 = (thread % (D / kPer)) * kPer, m = mt * 16 + row;
            float top = -INFINITY;
#pragma unroll
            for (int ww = 0; ww < kWaves; ++ww) top = fmaxf(top, red_m[(first + ww) * 16 * MT + m]);
            const float ref = top == -INFINITY ? 0.0f : top;
            float sum = 0.0f, o[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) o[u] = 0.0f;
#pragma unroll
            for (int ww = 0; ww < kWaves; ++ww) {
                const float e = exp2_fast(red_m[(first + ww) * 16 * MT + m] - ref);  // 0 for a wave that saw no key of the row
                sum = fmaf(red_l[(first + ww) * 16 * MT + m], e, sum);
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const float part_o = red[((first + ww) * 16 + row) * L::kRedStride + d0 + u];
                    o[u] = fmaf(part_o, e, o[u]);
                }
            }
            if (SPLIT && part.of > 1 && m < rows) {
                const int slot = CUT == kBalanced ? 2 * blockIdx.x + (first > 0 ? 1 : 0) : part.slot;
                const long long at = (long long)slot * (16 * MTMAX) + m;
                if constexpr (kPer >= 4) {
#pragma unroll
                    for (int u = 0; u < kPer; u += 4) store_device(a.part_o, at * D + d0 + u, f32x4{o[u], o[u + 1], o[u + 2], o[u + 3]});
                } else {  // two neighbours make a vector
                    static_assert(kPer == 2 || kPer >= 4, "a thread's values are whole vectors or half of one");
                    const float o2 = __shfl_down(o[0], 1, 64), o3 = __shfl_down(o[1], 1, 64);
                    if (d0 % 4 == 0) store_device(a.part_o, at * D + d0, f32x4{o[0], o[1], o2, o3});
                }
                if (d0 == 0) store_device(a.part_ml, at * 4, f32x4{top, sum, __builtin_bit_cast(float, (uint32_t)a.call_id), 0.0f});
            } else if (m < rows) {
                const int j = (m0 + m) / a.G, h = g * a.G + (m0 + m) % a.G;
                const size_t at = ((size_t)(q0 + j) * a.H_q + h) * D + d0;
                const float inv = 1.0f / sum;
#pragma unroll
                for (int u = 0; u < kPer; ++u) write_out(a, at + u, o[u] * inv);
                if (a.lse && d0 == 0) a.lse[(size_t)(q0 + j) * a.H_q + h] = top * kLn2 + logf(sum);
            }
        };
        if constexpr (CUT == kBalanced) {
            if (part.waves == 4) sum_rows(std::integral_constant<int, 4>{}, threadIdx.x & 255, w & 4);
            else sum_rows(std::integral_constant<int, kW>{}, threadIdx.x, 0);
        } else {
            sum_rows(std::integral_constant<int, kW>{}, threadIdx.x, 0);
        }
    }
}

// Balanced pieces: every item is cut into as many as it takes for none to last longer than a
// common time, the shortest that leaves no more pieces than there are places for four waves.  A workgroup holds two places.
// The items of an even number of pieces come first, so that theirs lie side by side: a workgroup whose two places hold pieces of
// one item works on both with all of its waves.  Every wave works this out for itself, from the lengths in its lanes.  Where
// there is little to gain every item has a workgroup to itself, the search is left out and what runs is the code of whole items: code
// that a workgroup runs once costs its fetch, 2 us with the search, the arguments in the order of their use and a stack frame, 0.5 to 1 us
// without but with four or eight waves to an item and its place looked up.
// D = 64, 32/8 heads, 1-7 drafts, us a call over the caches of 12 layers in turn, an item per workgroup / balanced, always searched /
// like this (gain): 20 requests of 256-4096 tokens 38.8 / 29.7 / 29.7 (242), 24 38.6 / 32.2 / 32.4, 32 40.4 / 35.0 / 34.9 (207), 48 64.1 /
// 53.6 / 53.7; 32 with log-normal contexts 34.6 / 24.8 / 24.7 (245); 16/16 heads, 10 of up to 3500 25.1 / 19.0 / 18.8 (173), 16 of
// 256-4096 35.1 / 33.2 / 33.3 (132); 20 of up to 2048 24.2 / 23.2 / 23.2 (124), 26 of up to 2600 28.0 / 27.7 / 27.7 (131), 32 of up
// to 3000 32.2 / 32.3 / 32.1 (132), of up to 2600 29.6 / 30.2 / 30.2 (115); 26 of up to 2048 25.1 / 26.0 / 24.9 (107), 32 of up to 2048
// 25.1 / 26.6 / 25.1 (101), up to 1024 16.2 / 20.5 / 16.3 (42), up to 256 9.7 / 11.7 / 9.7 (15); equal lengths, 20 of 1600 22.3 /
// 26.0 / 22.3 (62), 24 of 2176 27.4 / 29.8 / 27.7 (60), 32 of 2176 32.1 / 33.6 / 32.2 (12), 48 55.0 / 49.6 / 49.5.  Workgroups
// of four waves, two to a compute unit, in place of two items side by side in one of eight: 32 of 2176 37.1, and 14 us for 32 of up to 256.
__device__ __forceinline__ int small_quotient(int x, int d) {  // x / d, both the same in every lane
    return uniform((int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)d)));
}
struct Piece {
    int i, g, sp, n_sp, place0;  // piece sp of the n_sp of request i's item for KV head g, the first of which has place0
    int q0, q_len, c;            // the request's rows and context
};
template <int MTMAX, bool WHOLE>  // WHOLE: there are no more items than workgroups
struct BalancedPieces {
    int k, from, upto;  // the lane's request: pieces of an item, places of all of its items
    int q0, ql, c;      // its rows and context
    bool whole;         // every item has a workgroup to itself

    __device__ __forceinline__ explicit BalancedPieces(const ItemArgs& a) {
        const int lane = threadIdx.x & 63;
        q0 = ql = c = 0;
        if (lane < a.B) {
            q0 = a.cu_q[lane];
            ql = min(a.cu_q[lane + 1], a.N_cap) - q0;
            c = a.ctx[lane];
        }
        // (the other arguments are sent for while these come: later each would be another round trip)
        asm volatile("" ::"s"(a.q), "s"(a.k), "s"(a.v), "s"(a.bt), "s"(a.H_q), "s"(a.G), "s"(a.n_pages), "s"(a.page_stride), "s"(a.slot_stride), "s"(a.head_stride), "s"(a.p_shift));
        // rows beyond the caller's bound are further rounds (a slot would be written twice: no pieces then)
        const int M = max(ql, 0) * a.G, mt = (M + 15) >> 4, rounds = (mt + MTMAX - 1) / MTMAX;
        const int tiles = (min(max(c, 0), (int)min((long long)a.max_pages * a.P, 1LL << 30)) + ql + 31) >> 5;
        const float work = (float)tiles * (kTileBase * (float)rounds + (float)mt);
        const float longest = __builtin_bit_cast(float, wave_max_positive(__builtin_bit_cast(int, work)));
        const float share = work * __builtin_amdgcn_rcpf(longest);
        // With an item to a workgroup the call lasts as long as its longest; cut, no less than its share of the sum.
        const float sum = (float)wave_sum_i((int)(share * 65536.0f)) * (1.0f / 65536.0f);
        const float gain = longest * (0.5f - sum * (float)a.H_kv * __builtin_amdgcn_rcpf((float)a.places));
        whole = WHOLE && __builtin_amdgcn_ballot_w64(gain > kWorthCutting) == 0;
        k = from = upto = 0;
        if (whole) return;
        // two lie side by side and cost nothing; more have to be long enough to be worth handing over
        const int most = ql <= 0 ? 0 : rounds > 1 ? 1 : min(kMaxSplits, max(tiles / kPieceTiles, min(tiles, 2)));
        // times from the longest item's down to an eighth of it, 32 in equal ratios, by bisection; lane n holds longest / time n
        // (to a quarter / eighth / sixteenth, us a call: 20 requests 31.3 / 28.5 / 30.0, 32 of up to 2048 24.8 / 25.2 / 24.9, others alike)
        const float ratios = exp2_fast((float)lane * (3.0f / 31.0f));
        auto pieces = [=](int n) {
            const float r = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ratios), n));
            return min(most, max((int)__builtin_ceilf(share * r - 1e-4f), 1));
        };
        int lo = 0;
#pragma unroll
        for (int bit = 16; bit > 0; bit >>= 1)  // largest n that fits; n = 0, nothing is cut, always does
            if (wave_sum_i(pieces(lo + bit)) * a.H_kv <= a.places) lo += bit;
        k = pieces(lo);
        const int even = (k & 1) == 0 ? k * a.H_kv : 0, odd = k * a.H_kv - even;
        const int upto_even = wave_inclusive_scan_dpp(even), upto_odd = wave_inclusive_scan_dpp(odd);
        upto = even > 0 ? upto_even : odd > 0 ? __builtin_amdgcn_readlane(upto_even, 63) + upto_odd : 0;
        from = upto - k * a.H_kv;
    }
    // What lies at a place; n_sp = 0: nothing.
    __device__ __forceinline__ Piece at(int place) const {
        Piece p{0, 0, 0, 0, 0, 0, 0, 0};
        const unsigned long long mine = __builtin_amdgcn_ballot_w64(place < upto && place >= from);
        if (mine == 0) return p;
        p.i = __builtin_ctzll(mine);
        p.n_sp = __builtin_amdgcn_readlane(k, p.i);
        const int first = __builtin_amdgcn_readlane(from, p.i);
        p.g = small_quotient(place - first, p.n_sp);
        p.place0 = first + p.g * p.n_sp;
        p.sp = place - p.place0;
        p.q0 = __builtin_amdgcn_readlane(q0, p.i);
        p.q_len = __builtin_amdgcn_readlane(ql, p.i);
        p.c = __builtin_amdgcn_readlane(c, p.i);
        return p;
    }
};

// attend_group for as many query tiles as the group really has: mt_group rows of whoever shares the workgroup, from m0 on.
template <bool BF16, int D, int MTMAX, bool NT, int CUT>
__device__ __forceinline__ void attend_rows(const ItemArgs& a, char* smem, int i, int g, int q0, int M, int c, int m0, int mt_group, int sp, int n_sp,
                                            const Part& part) {
    const int mt = (min(mt_group - m0, 16 * MTMAX) + 15) >> 4;
    if constexpr (MTMAX >= 4)
        if (mt == 4) attend_group<BF16, D, MTMAX, 4, NT, CUT>(a, smem, i, g, q0, M, c, m0, sp, n_sp, part);
    if constexpr (MTMAX >= 3)
        if (mt == 3) attend_group<BF16, D, MTMAX, 3, NT, CUT>(a, smem, i, g, q0, M, c, m0, sp, n_sp, part);
    if constexpr (MTMAX >= 2)
        if (mt == 2) attend_group<BF16, D, MTMAX, 2, NT, CUT>(a, smem, i, g, q0, M, c, m0, sp, n_sp, part);
    if (mt == 1) attend_group<BF16, D, MTMAX, 1, NT, CUT>(a, smem, i, g, q0, M, c, m0, sp, n_sp, part);
    __syncthreads();  // before the next group's query operands and tiles
}

// CUT: one group per item, whose keys are cut into pieces -- evenly, grid.z of them, or by BalancedPieces; else grid.z counts the groups.
// WHOLE: see BalancedPieces.
template <bool BF16, int D, int MTMAX, bool NT, int CUT, bool WHOLE = false>
__global__ __launch_bounds__((Map<BF16, D, MTMAX, CUT>::kThreads), (Map<BF16, D, MTMAX, CUT>::kPerSimd)) void attend_items_kernel(ItemArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int kW = Map<BF16, D, MTMAX, CUT>::kW;
    int g = blockIdx.x, i = blockIdx.y, n_sp = 1, sp = 0, z = blockIdx.z, nz = gridDim.z, mt_group = 0;
    Part part{kW, 1, 0};
    bool cut = true;
    int q0, q_len, c;
    // what is needed again behind the keys' loops, of each half (scalar registers are short in them)
    __shared__ int s_place0[2], s_word[2];
    if constexpr (CUT == kBalanced) {
        const BalancedPieces<MTMAX, WHOLE> bp(a);
        z = 0;
        nz = 1;
        if constexpr (WHOLE) {
            if (bp.whole) {
                i = small_quotient(blockIdx.x, a.H_kv);
                g = blockIdx.x - i * a.H_kv;
                if (i >= a.B) return;
                q0 = __builtin_amdgcn_readlane(bp.q0, i);
                q_len = __builtin_amdgcn_readlane(bp.ql, i);
                c = __builtin_amdgcn_readlane(bp.c, i);
                const int M = q_len * a.G;
                for (int m0 = 0; m0 < M; m0 += 16 * MTMAX) attend_rows<BF16, D, MTMAX, NT, kWhole>(a, smem, i, g, q0, M, c, m0, M, 0, 1, part);
                return;
            }
        }
        const int half = uniform(threadIdx.x >> 8);
        const Piece p0 = bp.at(2 * blockIdx.x), p1 = bp.at(2 * blockIdx.x + 1);
        if (p0.n_sp == 0 && p1.n_sp == 0) return;
        const bool joint = p0.n_sp > 0 && p1.n_sp > 0 && p0.place0 == p1.place0;
        const Piece p = joint || half == 0 ? p0 : p1;
        i = p.i; g = p.g; sp = p.sp; n_sp = p.n_sp;
        part.waves = joint ? 8 : 4;
        auto parts_of = [](const Piece& x) { return x.n_sp > 0 ? ((x.place0 + x.n_sp - 1) >> 1) - (x.place0 >> 1) + 1 : 1; };
        part.of = parts_of(p);
        cut = parts_of(p0) > 1 || parts_of(p1) > 1;
        if ((threadIdx.x & 255) == 0) {
            s_place0[half] = p.place0;
            s_word[half] = p.i * a.H_kv + p.g;
        }
        // the same number of query tiles for both, so that their barriers meet (an empty place has no rows)
        mt_group = max(p0.q_len, p1.q_len) * a.G;
        q0 = p.q0; q_len = p.q_len; c = p.c;
    } else {
        q0 = a.cu_q[i];
        q_len = min(a.cu_q[i + 1], a.N_cap) - q0;
        c = a.ctx[i];
    }
    const int M = q_len * a.G;
    if (CUT != kBalanced && q_len <= 0) return;
    if constexpr (CUT == kEven) {
        // (rows beyond the caller's bound are further rounds: a slot would be written twice, so no pieces then)
        const int seen = (int)min((long long)c + q_len, min((long long)a.max_pages * a.P, 1LL << 30));
        if (M <= 16 * MTMAX) n_sp = max(1, min((int)gridDim.z, seen / kSplitKeys));
        sp = blockIdx.z;
        if (sp >= n_sp) return;
        part.of = n_sp;
        part.slot = uniform((i * a.H_kv + g) * nz + sp);  // (here: the grid's size is a load, and a round trip behind the keys' loops)
        z = 0;
        nz = 1;
    }
    if (CUT != kBalanced) mt_group = M;
    for (int m0 = z * 16 * MTMAX; m0 < mt_group; m0 += nz * 16 * MTMAX)
        attend_rows<BF16, D, MTMAX, NT, CUT>(a, smem, i, g, q0, M, c, m0, mt_group, sp, n_sp, part);
    if constexpr (CUT != kWhole) {
        __shared__ int s_last[2];
        if (CUT == kEven ? n_sp == 1 : !cut) return;
        const int half = CUT == kBalanced ? uniform(threadIdx.x >> 8) & (part.waves == 4 ? 1 : 0) : 0;
        const int thread = CUT == kBalanced && part.waves == 4 ? threadIdx.x & 255 : threadIdx.x;
        const int word = CUT == kBalanced ? uniform(s_word[half]) : i * a.H_kv + g;
        const int slot0 = CUT == kBalanced ? uniform(s_place0[half]) : part.slot - sp;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the piece is in memory once every wave's stores are acknowledged
        __syncthreads();
        if (thread == 0) s_last[half] = part.of > 1 && count_arrival(a.arrivals + word, a.call_id) == part.of;
        __syncthreads();
        if (!s_last[half]) return;
        combine_pieces<D, 16 * MTMAX>(a, g, q0, 0, M, slot0, CUT == kBalanced ? 2 * ((slot0 >> 1) + 1) : slot0 + 1, CUT == kBalanced ? 2 : 1,
                                      part.of, thread, CUT == kBalanced ? 64 * part.waves : 64 * kW);
        if (thread == 0) __atomic_store_n(a.arrivals + word, a.call_id << 16, __ATOMIC_RELAXED);  // for a graph's next replay
    }
}

template <bool BF16, int D, int MT, bool NT, int CUT, bool WHOLE = false>
void launch_as(const ItemArgs& a, unsigned z, hipStream_t s) {
    typedef Map<BF16, D, MT, CUT> L;
    const dim3 grid = CUT == kBalanced ? dim3((unsigned)(a.places / 2)) : dim3((unsigned)a.H_kv, (unsigned)a.B, z);
    hipLaunchKernelGGL((attend_items_kernel<BF16, D, MT, NT, CUT, WHOLE>), grid, dim3(L::kThreads), L::kSmem, s, a);
}

template <bool BF16, int D, int MT>
int launch(const ItemArgs& a, unsigned groups, hipStream_t s) {
    // keys that one workgroup reads once bypass the caches' replacement (non-temporal); further groups of a request
    // find them in the caches.  D = 64, 32/8 heads, 256 to 4096 tokens, us a call over the caches of 24 layers in turn,
    // non-temporal / plain: 16 requests 38.2 / 39.8, 64 70.6 / 78.2, 128 125 / 140, 32/32 heads 64 requests 191 / 216, one
    // request of 8192 tokens 55.2 / 55.7.  (Called again and again on one pair of caches that the last level holds, the
    // plain loads win at the small end: one request of 8192 tokens 54.0 / 47.3.)
    if constexpr (BF16) {
        if (a.places > 0) {
            if constexpr (!Map<true, D, MT, kBalanced>::kLarge) {
                if (2 * a.B * a.H_kv <= a.places) launch_as<true, D, MT, true, kBalanced, true>(a, 1, s);
                else launch_as<true, D, MT, true, kBalanced>(a, 1, s);
            }
        } else if (a.splits > 1) launch_as<true, D, MT, true, kEven>(a, (unsigned)a.splits, s);
        else if (groups == 1) launch_as<true, D, MT, true, kWhole>(a, 1, s);
        else launch_as<true, D, MT, false, kWhole>(a, groups, s);
    } else {
        launch_as<false, D, MT, false, kWhole>(a, groups, s);
    }
    return check_launch("attend_items_kernel");
}

// How a call is laid out.
struct Layout {
    int mt;           // query tiles of a group
    unsigned groups;  // workgroups an item's rows are dealt to
    int splits;       // pieces an item's keys are cut into at most
    int places;       // > 0: items are cut by their lengths, into this many pieces in all
    size_t bytes_o, bytes_ml, bytes_cnt;
};
Layout layout_of(const fsr_attn_params& p) {
    // query rows a KV head of one request can have: the caller's bound on its rows, or all rows of the call
    const bool bounded = p.max_q_len > 0;
    const long long rows = (long long)(p.H_q / p.H_kv) * (bounded ? std::min(p.max_q_len, p.N_cap) : p.N_cap);
    const int most_tiles = p.D == 64 ? 4 : 3;  // query tiles a wave holds (three at D = 128 spill some 30 registers, outside the loops' sums)
    Layout l{};
    l.mt = (int)std::max(1LL, std::min<long long>(most_tiles, (rows + 15) / 16));
    // An item gets as many workgroups as its rows need groups, up to 64; each may take several, and one without rows leaves
    // at once.  Where the caller has not said how many rows a request has, one may have all of the call's, and the bound is
    // as many as leave the call some thousands (at least four an item).  Without a hint, us a call with four an item / like
    // this: 32/1 heads of 64, one request of 64 rows and 8192 tokens 1039 / 141, 32/8 heads, one of 256 rows and 4096 tokens
    // 283 / 77, one of 1024 rows 1207 / 165, 128 of 2 to 9 rows 114 / 114; fp32, 8/2 heads, 512 of 2 to 9 rows 57 / 57.
    const long long items = std::max(1LL, (long long)p.B * p.H_kv), most = bounded ? 64 : std::max(4LL, std::min(64LL, 4096 / items));
    l.groups = (unsigned)std::max(1LL, std::min(most, (rows + 16 * l.mt - 1) / (16 * l.mt)));
    // Pieces of an item's keys, where a call has fewer items than the device has compute units.  Not more: one workgroup runs on
    // a compute unit at a time, and a second one waits for the first before it sends for anything.  D = 64, 32/8 heads, us of 3
    // layers with no pieces / up to 256 / 512 / 1024 workgroups: one request of 8192 tokens 164 / 66 / 66 / 66, 4 of 256 to 4096
    // 89 / 62 / 62 / 62, 16 of 256 to 8192 194 / 132 / 143 / 174, 32 of 256 to 4096 128 / 128 / 144 / 176.  On a stream that owns
    // part of the device max_workgroups says how many units there are, us a layer with no pieces / up to 256 workgroups / up to the
    // units owned: 32 units, 4 requests of 256 to 4096 37 / 76 / 35, 16 122 / 162 / 120, one of 8192 71 / 37 / 29; 128 units, 4 48 / 37 / 27.
    l.splits = 1;
    if (p.dtype == FSR_BF16 && l.groups == 1) {
        const long long keys = (long long)p.max_pages * p.P;
        const long long units = p.max_workgroups > 0 ? std::min<long long>(p.max_workgroups, kSplitGroups) : kSplitGroups;
        l.splits = (int)std::max(1LL, std::min({(long long)kMaxSplits, keys / kSplitKeys, units / items}));
        // From more items than half the units to one and a half times as many, heads of 64 (eight waves a workgroup): balanced by
        // length.  With fewer even pieces do as well (16 requests 26.5 / 26.6), with more the units have several items anyway (56
        // requests 68.7 / 71.5).  Tables of so few pages hold nothing that is worth it (see kWorthCutting).
        if (p.D == 64 && l.mt < 4 && p.B > 1 && p.B <= kBalancedMaxB && keys >= kBalancedKeys && 2 * items > units && 2 * items <= 3 * units) {
            l.places = (int)(2 * units);
            l.splits = 1;
        }
    }
    const size_t slots = l.places > 0 ? (size_t)l.places : (size_t)items * l.splits, row = (size_t)16 * l.mt;
    if (l.splits > 1 || l.places > 0) {
        l.bytes_o = align_up(slots * row * p.D * sizeof(float), 256);
        l.bytes_ml = align_up(slots * row * 4 * sizeof(float), 256);
        l.bytes_cnt = align_up((size_t)items * sizeof(unsigned long long), 256);  // (no more items than places)
    }
    return l;
}

template <bool BF16, int D>
int launch_mt(const ItemArgs& a, const Layout& l, hipStream_t s) {
    switch (l.mt) {
        case 1: return launch<BF16, D, 1>(a, l.groups, s);
        case 2: return launch<BF16, D, 2>(a, l.groups, s);
        case 3: return launch<BF16, D, 3>(a, l.groups, s);
        default: return launch<BF16, D, D == 64 ? 4 : 3>(a, l.groups, s);
    }
}

}  // namespace

// For as many slots as any batch uses, so that the size covers smaller batches and fewer rows a request too (which are cut into more
// pieces): heads of 64 two slots a workgroup of up to three query tiles, which is more than one of four.
size_t attend_items_workspace_bytes(const fsr_attn_params& p) {
    if (p.dtype != FSR_BF16) return 0;
    const size_t slots = (p.D == 64 ? 2 : 1) * (size_t)kSplitGroups, rows = slots * 16 * std::min(layout_of(p).mt, 3);
    return align_up(rows * p.D * sizeof(float), 256) + align_up(rows * 4 * sizeof(float), 256) +
           align_up(slots * sizeof(unsigned long long), 256);
}

int attend_items_launch(const void* q, const void* k_cache, const void* v_cache, const int32_t* block_tables,
                        const int32_t* ctx_lens, const int32_t* cu_q, void* out, float* lse, const fsr_attn_params* p,
                        void* workspace, size_t ws_bytes, hipStream_t s, const char* who) {
    if (p->N_cap > 65535) return fail(FSR_EUNSUP, "%s: the scratch-free path is limited to N_cap <= 65535 rows", who);
    ItemArgs a;
    const long long e = p->dtype == FSR_BF16 ? 2 : 4, row = p->D * e;
    a.q = q; a.k = k_cache; a.v = v_cache; a.bt = block_tables; a.ctx = ctx_lens; a.cu_q = cu_q; a.out = out; a.lse = lse;
    a.B = p->B; a.N_cap = p->N_cap; a.H_q = p->H_q; a.H_kv = p->H_kv; a.G = p->H_q / p->H_kv; a.P = p->P;
    a.max_pages = p->max_pages; a.n_pages = p->n_pages;
    a.p_shift = (p->P & (p->P - 1)) == 0 ? __builtin_ctz((unsigned)p->P) : -1;
    a.out_bf16 = p->out_dtype == FSR_BF16;
    a.page_stride = (long long)p->P * p->H_kv * row;
    const bool token_major = p->kv_layout == FSR_KV_TOKEN_MAJOR;
    a.slot_stride = token_major ? p->H_kv * row : row;
    a.head_stride = token_major ? row : p->P * row;
    a.scale_log2 = p->scale * (float)kLog2e;
    a.scale_rest = (float)(p->scale - a.scale_log2 / kLog2e);
    Layout l = layout_of(*p);
    // a caller without (enough) scratch memory gets one workgroup per group
    if ((l.splits > 1 || l.places > 0) && (!workspace || ((uintptr_t)workspace & 255) || ws_bytes < l.bytes_o + l.bytes_ml + l.bytes_cnt)) l.splits = 1, l.places = 0;
    a.splits = l.splits;
    a.places = l.places;
    a.part_o = (float*)workspace;
    a.part_ml = (float*)((char*)workspace + l.bytes_o);
    a.arrivals = (unsigned long long*)((char*)workspace + l.bytes_o + l.bytes_ml);
    a.call_id = l.splits > 1 || l.places > 0 ? next_call_id() : 0;
    if (p->dtype == FSR_BF16) return p->D == 64 ? launch_mt<true, 64>(a, l, s) : launch_mt<true, 128>(a, l, s);
    return p->D == 64 ? launch_mt<false, 64>(a, l, s) : launch_mt<false, 128>(a, l, s);
}

}  // namespace fsr
