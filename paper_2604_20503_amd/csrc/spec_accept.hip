// spec_accept: accept / reject of drafted tokens with recovery or bonus token.
//
// Rule (Sec. 2.1 of the paper; the mismatch test and resampling distribution are those of
// speculative sampling): accept drafts while u * q(x) < p(x); at the first rejection draw
// one token from the normalised positive part of p - q; if everything is accepted and the
// call carries the extra target row, draw the bonus token from it.
//
// Work split.  A verification batch has few requests (16 .. 512) but a vocabulary of
// ~1.3e5, so one workgroup per request cannot fill the chip: every vocabulary row is cut
// into chunks of kChunk tokens and the vocabulary-wide sums are two-level.
//   stats    (LOGITS mode only) per row and group of 1-8 chunks: a reference and the sum of exp(z / T - reference) in
//            fp64.  The rows of all requests' first drafts come first in the grid, then those of their second drafts
//            and so on; the workgroup that finishes a draft's two rows last tests the draft, and rows behind a
//            rejected draft that have not been started by then are left out (only rows 0 .. n of a request are
//            needed, n = accepted drafts)
//   decide   per request, one wave: the accept tests, one lane per draft with all gathers in flight
//            together (LOGITS mode: the outcome that `stats` has found); picks the row pair to sample from and
//            records it
//   sample   grid (chunks, requests): every workgroup sums the fp64 mass of its chunks of the residual or of the target
//            row (of the target row too where there is no residual, for the draw if there is none anywhere); the
//            workgroup of a request that finishes last (found by an arrival counter that `decide` has zeroed) draws the
//            token: prefix over the chunk masses -> chunk holding u * R -> scan inside that chunk
// Only the rows the outcome needs are streamed: one target row (bonus) or one target and
// one draft row (rejection) per request -- the algorithmic minimum in PROBS mode.
// All masses are accumulated in fp64 so that the chosen token matches a sequential fp64
// scan except when u * R lies within rounding of a CDF step.
#include <algorithm>
#include <cfloat>
#include <climits>

#include "common.hpp"
#include "device_utils.hpp"
#include "greedy_accept.hpp"
#include "temp_scale.hpp"

namespace fsr {
namespace {

constexpr int kChunk = 4096;        // vocabulary tokens per chunk
constexpr int kThreads = 256;       // threads per block in stats / partials / select
constexpr int kPerThread = kChunk / kThreads;  // 16 contiguous tokens per thread in select
constexpr int kMaxStatGroup = 8;    // LOGITS mode: most chunks whose softmax statistics one workgroup folds into one (reference, sum) pair
constexpr int kSkipMinRows = 2048;  // LOGITS mode: rows a call must be able to hold for rows behind a rejection to be left out
constexpr double kStatSlack = 100.0;  // LOGITS mode, temperatures out of all range: exponents the statistics let grow before they change their reference
constexpr int kMaxSampleGroup = 8;  // accept_sample: most consecutive chunks that a workgroup takes (see sample_group_of)

enum : int { kCaseNone = 0, kCaseResidual = 1, kCaseTarget = 2 };

// What `decide` hands to the later kernels, one per request.
struct Decision {
    long long t_row;  // storage row of the target distribution to sample from
    long long d_row;  // storage row of the draft distribution (residual case)
    double m_t, Z_t;  // LOGITS mode: exponent reference (at most 100 below the maximum) and partition sum of the target row
    double m_d, Z_d;  // ... of the draft row
    int kind;         // kCase*
    int n;            // accepted drafts
};
// LOGITS mode, how a row's masses in a draw are formed: exp(z / T) / 2^shift by exp_of_logit (direct; `shift` brings the row's
// largest near 1), else exp(z / T - m).  A direct row takes logits from `lowest` on as they are; one below that is masked
// if its mass is 0 in fp64, and hardly ever anything else.
struct RowScale {
    double shift;
    double rest;   // m - shift ln2, 0 if not direct: a mass is exp(z / T - m + rest)
    float lowest;
    float masked;  // below this a logit of a direct row is masked whatever the roundings
};
struct DrawScale {
    RowScale t, d;
    double ratio;  // one unit of the draft row's masses in those of the target row
    int direct;
    int unused;
};

struct Workspace {
    Decision* dec;       // [B]
    double* mass_res;    // [B, n_chunks]
    double* mass_tgt;    // [B, n_chunks]
    double* stat_t;      // [R_t_cap, n_stat_groups, 2]  (LOGITS)
    double* stat_d;      // [R_d_cap, n_stat_groups, 2]
    DrawScale* scale;    // [B] (LOGITS)
    unsigned int* arrivals;  // [B] chunk workgroups of the request that have finished (zeroed by decide)
    int stat_group;          // chunks per (reference, sum) pair in this call (set at launch)
    // LOGITS mode, while the statistics of a large call are made (the memory is that of the chunk masses, which come
    // later): 2 * n_chunks 32-bit words per request from mass_res on, word 0 the first rejected draft, word 1 + j the
    // workgroups that have finished rows j (accept_clear_kernel sets them up).  0: `decide` tests the drafts.
    int skip;
};

__host__ __device__ inline int n_chunks_of(int V) { return (V + kChunk - 1) / kChunk; }
__host__ __device__ inline int n_stat_groups_of(int V, int group) { return (n_chunks_of(V) + group - 1) / group; }

size_t carve(const fsr_accept_params& p, char* base, Workspace* w) {
    const size_t nc = (size_t)n_chunks_of(p.V), B = (size_t)p.B;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* ptr = base ? base + off : nullptr;
        off += align_up(bytes, 256);
        return ptr;
    };
    Workspace tmp;
    tmp.dec = (Decision*)take(B * sizeof(Decision));
    tmp.mass_res = (double*)take(B * nc * sizeof(double));
    tmp.mass_tgt = (double*)take(B * nc * sizeof(double));
    tmp.arrivals = (unsigned int*)take(B * sizeof(unsigned int));
    tmp.skip = 0;
    tmp.stat_group = kMaxStatGroup;
    if (p.mode == FSR_LOGITS) {
        const size_t nsg = nc;  // room for one pair per chunk; a call folds 1, 2, 4 or 8 chunks into a pair
        tmp.stat_t = (double*)take(B * (size_t)(p.S_max + 1) * nsg * 2 * sizeof(double));
        tmp.stat_d = (double*)take(B * (size_t)p.S_max * nsg * 2 * sizeof(double));
        tmp.scale = (DrawScale*)take(B * sizeof(DrawScale));
    } else {
        tmp.stat_t = tmp.stat_d = nullptr;
        tmp.scale = nullptr;
    }
    if (w) *w = tmp;
    return off;
}

constexpr unsigned kNoRejection = 0xffffffffu;
// The request's words of the statistics (see Workspace::skip).
__device__ __forceinline__ unsigned* stat_words(const Workspace& ws, int i, int nc) {
    return reinterpret_cast<unsigned*>(ws.mass_res + (size_t)i * nc);
}
__global__ __launch_bounds__(kThreads) void accept_clear_kernel(Workspace ws, int n_words, int nc) {
    const int w = blockIdx.x * kThreads + threadIdx.x;
    if (w < n_words) stat_words(ws, 0, nc)[w] = w % (2 * nc) == 0 ? kNoRejection : 0u;
}

// Rows are fp32, or bf16 stored as 16-bit patterns (the upper half of an fp32).
__device__ __forceinline__ float to_float(float x) { return x; }
__device__ __forceinline__ float to_float(uint16_t x) { return __builtin_bit_cast(float, (uint32_t)x << 16); }
// Four consecutive values of a row, wherever they start: the hardware takes vectors that are aligned to their elements only,
// and most rows of an odd vocabulary start in the middle of one.  Against element by element for such rows, vocabulary
// 152063, 1 to 7 drafts, us a call: PROBS 16 requests 23.2 / 17.0, 128 55.3 / 29.0, 384 120 / 83; LOGITS 16 in bf16 58 / 41.5, 128
// in bf16 350 / 182, 384 in fp32 476 / 375.
typedef __attribute__((__vector_size__(16), __aligned__(4))) float row_f32x4;
typedef __attribute__((__vector_size__(8), __aligned__(2))) uint16_t row_u16x4;
template <bool NT = false>  // with the non-temporal hint
__device__ __forceinline__ row_f32x4 raw_quad(const float* __restrict__ row, int e) {
    const row_f32x4* p = reinterpret_cast<const row_f32x4*>(row + e);
    return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT = false>
__device__ __forceinline__ row_u16x4 raw_quad(const uint16_t* __restrict__ row, int e) {
    const row_u16x4* p = reinterpret_cast<const row_u16x4*>(row + e);
    return NT ? __builtin_nontemporal_load(p) : *p;
}
template <typename RT>
__device__ __forceinline__ void load_quad_vec(const RT* __restrict__ row, int e, float (&x)[4]) {
    const auto t = raw_quad(row, e);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = to_float(t[k]);
}
// The same where some of the four may lie past the vocabulary: `fill` stands for those.
template <typename RT>
__device__ __forceinline__ void load_quad(const RT* __restrict__ row, int e, int V, float (&x)[4], float fill = 0.0f) {
    if (e + 3 < V) {
        load_quad_vec(row, e, x);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (e + k < V) ? to_float(row[e + k]) : fill;
    }
}

// Constants of exp_softmax, made once per kernel.  The empty asm statements pin each one to a scalar register pair
// (the leading coefficient to a vector pair) and hide its value from the compiler, which otherwise rebuilds every
// constant with move instructions in front of each use: that doubles the instruction count of the polynomial.
struct ExpConsts {
    double floor, log2e, nln2_hi, nln2_lo, magic, c10, c9, c8, c7, c6, c5, c4, c3, c2, c1;
};
__device__ __forceinline__ ExpConsts exp_consts() {
    ExpConsts k;
    k.floor = -800.0;  // below it exp is 0 in fp64
    k.log2e = 1.4426950408889634074;
    k.nln2_hi = -6.93147180369123816490e-01;  // high part of ln2: its last 21 bits are zero, so k * hi is exact for |k| < 2^21
    k.nln2_lo = -1.90821492927058770002e-10;
    k.magic = 6755399441055744.0;  // 1.5 * 2^52: adding it rounds to an integer and leaves that integer in the low word
    // the polynomial of degree 10 that equals exp at the 11 Chebyshev nodes of [-ln2/2, ln2/2] (widened by 0.05 %),
    // solved in 80-bit arithmetic and rounded to fp64: 3e-16 from exp over the interval, 5e-16 as evaluated
    k.c10 = 2.7626457017679406e-07;
    k.c9 = 2.7640263805714195e-06;
    k.c8 = 2.480150410776298e-05;
    k.c7 = 0.00019841170070855952;
    k.c6 = 0.0013888888932672718;
    k.c5 = 0.008333333385825259;
    k.c4 = 0.041666666666572656;
    k.c3 = 0.16666666666553953;
    k.c2 = 0.5000000000000006;
    k.c1 = 1.0000000000000069;
    asm volatile("" : "+s"(k.log2e), "+s"(k.nln2_hi), "+s"(k.nln2_lo), "+s"(k.floor), "+v"(k.c10), "+v"(k.magic));
    asm volatile("" : "+s"(k.c9), "+s"(k.c8), "+s"(k.c7), "+s"(k.c6), "+s"(k.c5));
    asm volatile("" : "+s"(k.c4), "+s"(k.c3), "+s"(k.c2), "+s"(k.c1));
    return k;
}

// exp(x) in fp64 for the arguments a softmax produces (x up to about 100 after the row's reference is taken off; a few
// hundred work too; x below -745, -inf included, gives 0, and so does NaN: such a logit counts as masked).
// x = k ln2 + r with |r| <= ln2 / 2: k by adding 1.5 * 2^52 to x log2(e), which rounds to the integer and leaves it
// in the sum's low word; ln2 in two parts so that r is exact to the last bit; exp(r) by a polynomial of degree 10
// (5e-16 relative); times 2^k by ldexp, which also makes the subnormal results and the final 0.  16 instructions,
// all of them issued at the full fp64 rate, where the library routine takes several times as many: the per-element
// exp is what bounds the LOGITS-mode kernels.
__device__ __forceinline__ double exp_softmax(double x, const ExpConsts& k) {
    x = fmax(x, k.floor);
    const double t = fma(x, k.log2e, k.magic);
    const double kf = t - k.magic;
    double r = fma(kf, k.nln2_hi, x);
    r = fma(kf, k.nln2_lo, r);
    double p = fma(k.c10, r, k.c9);
    p = fma(p, r, k.c8);
    p = fma(p, r, k.c7);
    p = fma(p, r, k.c6);
    p = fma(p, r, k.c5);
    p = fma(p, r, k.c4);
    p = fma(p, r, k.c3);
    p = fma(p, r, k.c2);
    p = fma(p, r, k.c1);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)(uint32_t)__builtin_bit_cast(unsigned long long, t));
}
// exp for the loops over whole rows, where its instruction count is the kernel's time: x = n ln2 / 256 + r with
// |r| <= ln2 / 512, 2^(n/256) from a table of 256 values in LDS and four terms of the series in r: 13 instructions and a
// table look-up where exp_softmax takes 16, and closer to exp (2.3e-16).  The integer n sits in the low word of the
// rounding sum; the table's high words are stored less j << 12, so that one shift-and-add of n puts 2^(n / 256) together.
// Measured, statistics of 512 requests x 152064 logits (about 2.9 GB of rows, bound by the vector ALUs): 693 -> 557 us, with
// the references that need no rescaling per chunk.
// Arguments below kExpTableFloor (and NaN) count as that floor: 1e-304, so that the exponent stays a normal one.
constexpr double kExpTableFloor = -700.0;
__device__ const double kExp2Table[256] = {
#include "exp_table.inc"
};
struct ExpTable {
    const uint2* tab;  // LDS
    double c, nl_hi, nl_lo, magic, c4, c3, floor;
};
// The thread's entry of the table that a workgroup keeps in LDS.  Loaded before the rows are sent for, stored behind that:
// loads return in order, and the table must not wait for the rows, nor they for it.
static_assert(kThreads == 256, "a thread brings one entry of the table");
__device__ __forceinline__ uint2 exp_table_entry() {
    const unsigned long long v = __builtin_bit_cast(unsigned long long, kExp2Table[threadIdx.x]);
    return make_uint2((uint32_t)v, (uint32_t)(v >> 32) - (threadIdx.x << 12));
}
__device__ __forceinline__ ExpTable exp_table(const uint2* tab) {
    ExpTable k;
    k.tab = tab;
    k.c = 369.3299304675746;            // 256 / ln2
    k.nl_hi = -0.00270760617331689;     // -ln2 / 256 in two parts, the high one with 21 zero bits at its end
    k.nl_lo = -7.453964567463233e-13;
    k.magic = 6755399441055744.0;       // 1.5 * 2^52
    k.c4 = 1.0 / 24.0;
    k.c3 = 1.0 / 6.0;
    k.floor = kExpTableFloor;
    asm volatile("" : "+s"(k.floor), "+s"(k.c), "+s"(k.nl_hi), "+s"(k.nl_lo), "+s"(k.c4), "+v"(k.c3), "+v"(k.magic));
    return k;
}
__device__ __forceinline__ double exp_lookup(double x, const ExpTable& k) {
    x = fmax(x, k.floor);
    const double t = fma(x, k.c, k.magic);
    const double kf = t - k.magic;
    const uint32_t n = (uint32_t)__builtin_bit_cast(unsigned long long, t);
    const uint2 e = k.tab[n & 255u];
    double r = fma(kf, k.nl_hi, x);
    r = fma(kf, k.nl_lo, r);
    const double p = fma(fma(fma(r, k.c4, k.c3), r, 0.5), r, 1.0);
    const double pow2 = __builtin_bit_cast(double, ((unsigned long long)(e.y + (n << 12)) << 32) | e.x);
    return fma(pow2 * r, p, pow2);
}
// exp(z / T) for the logits themselves, with no reference taken off: z / T = n ln2 / 256 + r again, but in units of ln2 / 256, so
// that one multiply-add rounds to n, one subtraction and two multiply-adds give r (256 / (T ln2) in two parts, the high one of 29
// bits, whose product with a logit is exact), four the series and a fifth adds the value to a sum: 12 instructions and a
// look-up where exp_lookup and its argument take 16.  Errors against exp(z / T), logits N(0, 2^2): 3.0e-16 at most, 8.3e-17
// root mean square, at every T (by way of z * (1 / T) 1.9e-16 and 6.6e-17 at T = 1, 1.0e-15 and 1.9e-16 at 0.7, 7.9e-15 and 2.2e-15
// at 0.05, where 1 / T is rounded).  A shift by a whole power of two costs nothing: it goes into the constant that rounds, so that the
// low word of the sum is n less 256 shift.  For |z / T - shift ln2| up to 700 or so, where 2^n is a normal number, and
// |z / T| up to kWidest, where n is exact.
struct ExpDirect {
    const uint2* tab;  // LDS
    double c, c_hi, c_lo, magic, a4, a3, a2, a1;
};
__device__ __forceinline__ ExpDirect exp_direct(const uint2* tab, const TempScale& ts) {
    ExpDirect k;
    k.tab = tab;
    k.c = ts.c;
    k.c_hi = ts.c_hi;
    k.c_lo = ts.c_lo;
    k.magic = 6755399441055744.0;  // 1.5 * 2^52
    k.a4 = 2.239395190875157e-12;  // (ln2 / 256)^n / n!
    k.a3 = 3.3083026805413713e-09;
    k.a2 = 3.6655655969101062e-06;
    k.a1 = 0.0027076061740622863;
    asm volatile("" : "+s"(k.c), "+s"(k.c_hi), "+s"(k.c_lo), "+s"(k.a4), "+v"(k.a3), "+s"(k.a2), "+s"(k.a1), "+v"(k.magic));
    return k;
}
constexpr double kWidest = 5e12;  // 256 / ln2 times it is below 2^51
constexpr double kRound = 6755399441055744.0;
__device__ __forceinline__ ExpDirect shifted(ExpDirect k, double shift) {
    k.magic = kRound - 256.0 * shift;
    return k;
}
constexpr double kLn2Hi = 6.93147180369123816490e-01, kLn2Lo = 1.90821492927058770002e-10;  // ln2 in two parts, see ExpConsts
__device__ __forceinline__ double less_shift(double m, double shift) { return fma(-shift, kLn2Lo, fma(-shift, kLn2Hi, m)); }
// exp(z / T) / 2^shift = power * series
struct ExpParts {
    double power, series;
};
__device__ __forceinline__ ExpParts exp_of_logit(double x, const ExpDirect& k) {
    const double t = fma(x, k.c, k.magic);
    const double n = t - k.magic;
    const uint32_t low = (uint32_t)__builtin_bit_cast(unsigned long long, t);
    const uint2 e = k.tab[low & 255u];
    const double r = fma(x, k.c_lo, fma(x, k.c_hi, -n));
    ExpParts p;
    p.power = __builtin_bit_cast(double, ((unsigned long long)(e.y + (low << 12)) << 32) | e.x);
    p.series = fma(fma(fma(fma(k.a4, r, k.a3), r, k.a2), r, k.a1), r, 1.0);
    return p;
}
// Largest magnitude, largest and smallest of three (one instruction each; a quiet NaN is passed over, a signalling one too in waves
// that have called pass_over_nans, and else hides the value beside it).
__device__ __forceinline__ float max3_abs(float m, float x, float y) {
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(x), "v"(y));
    return m;
}
__device__ __forceinline__ float max3(float m, float x, float y) {
    asm("v_max3_f32 %0, %1, %2, %0" : "+v"(m) : "v"(x), "v"(y));
    return m;
}
__device__ __forceinline__ float min3(float m, float x, float y) {
    asm("v_min3_f32 %0, %1, %2, %0" : "+v"(m) : "v"(x), "v"(y));
    return m;
}
__device__ __forceinline__ float max2(float x, float y) {  // (fmaxf quiets its operands first)
    float m;
    asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(x), "v"(y));
    return m;
}
// The IEEE bit of the wave's mode off (bit 9 of hardware register 1): minima and maxima return the operand that is no NaN whatever
// kind of NaN the other is.
__device__ __forceinline__ void pass_over_nans() { __builtin_amdgcn_s_setreg(1 | 9 << 6, 0); }
// A value that is the same in every lane, said so.
__device__ __forceinline__ float uniform(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ double uniform(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)b), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Largest of the wave's values, in every lane.  (The value may come from asm, which the compiler does not keep two instructions
// away from a DPP read: an instruction of its own first.)
__device__ __forceinline__ float wave_top(float v) {
    v = __builtin_canonicalizef(v);
    auto step = [&](auto ctrl, auto rows) {
        const int b = __builtin_bit_cast(int, v);
        v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
// The least float that is not below x.
__device__ __forceinline__ float float_up(double x) {
    const float f = (float)x;
    if (!((double)f < x)) return f;
    const uint32_t b = __builtin_bit_cast(uint32_t, f);
    return f == 0.0f ? __builtin_bit_cast(float, 1u) : __builtin_bit_cast(float, f < 0.0f ? b - 1u : b + 1u);
}
constexpr double kLn2 = 0.6931471805599453, kAmple = 1.9151695967140057e-174;  // exp(-400)
constexpr double kExpZero = -746.0;  // exp of it and of anything less is 0 in fp64
// The constants for a kernel of the given mode: PROBS mode never evaluates exp and gets an empty set.
template <int MODE>
__device__ __forceinline__ ExpConsts exp_consts_for() {
    if constexpr (MODE == FSR_LOGITS) return exp_consts();
    else return ExpConsts{};
}

// z / T - m.  Beyond kWidest the two differ by whole units or not at all, and m is the rounded quotient of one of the row's
// logits: a multiply-add would leave its rounding behind where there is no difference.  (An infinite m is that of a row without
// any mass: NaN or infinite, which counts as none.)
__device__ __forceinline__ double less_reference(float z, double inv_T, double m) {
    const double d = fma((double)z, inv_T, -m);
    return fabs(m) > kWidest && fabs(m) < INFINITY && __dmul_rn((double)z, inv_T) == m ? 0.0 : d;
}

// Probability of one entry in fp64: the value itself, or exp(z / T - m) / Z with the two divisions as products
// by 1 / T and 1 / Z (loop invariants the compiler hoists).  m is a reference that the row's statistics have kept, at most
// kStatSlack below the largest z / T, and Z the sum relative to the same m.
template <int MODE>
__device__ __forceinline__ double prob_of(float x, double T, double m, double Z, const ExpConsts& ek) {
    if constexpr (MODE == FSR_PROBS) {
        return (double)x;
    } else {
        return exp_softmax(less_reference(x, 1.0 / T, m), ek) * (1.0 / Z);
    }
}

// 8-byte values that another workgroup of the same launch reads: stored through to memory / loaded past the caches
__device__ __forceinline__ void publish_f64(double* p, double v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double fetch_f64(const double* p) {
    return __builtin_bit_cast(double, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT));
}

// One step of a reduction over each half of the wave by DPP (see wave_sum_to_last): the lane's value, or `none` where the
// control has no lane to take one from.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v, double none) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v), z = __builtin_bit_cast(unsigned long long, none);
    const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)z, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(z >> 32), (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}
// Lane 31 ends with the fold of lanes 0 .. 31, lane 63 with that of lanes 32 .. 63.
template <typename F>
__device__ __forceinline__ double fold_halves(double v, double none, F&& f) {
    v = f(v, dpp_f64<0x111, 0xf>(v, none));
    v = f(v, dpp_f64<0x112, 0xf>(v, none));
    v = f(v, dpp_f64<0x114, 0xf>(v, none));
    v = f(v, dpp_f64<0x118, 0xf>(v, none));
    return f(v, dpp_f64<0x142, 0xa>(v, none));
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, lane), hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

struct RowStat {
    double m, Z;  // largest reference, partition sum relative to it
};
// Combine the chunk statistics of two rows, one in each half of the wave (all lanes call it; stat_b may be stat_a).  FRESH: the
// statistics were made by other workgroups of this launch.
template <bool FRESH>
__device__ __forceinline__ void combine_stats(const double* __restrict__ stat_a, const double* __restrict__ stat_b, int nc,
                                              const ExpConsts& ek, RowStat& ra, RowStat& rb) {
    const int lane = threadIdx.x & 63, l = lane & 31;
    const double* stat = lane < 32 ? stat_a : stat_b;
    auto at = [&](int k) { return FRESH ? fetch_f64(stat + k) : stat[k]; };
    // the first two pairs of a lane stay in registers (rows of up to 64 groups, i.e. nearly all)
    double m0 = -INFINITY, m1 = -INFINITY, s0 = 0.0, s1 = 0.0;
    if (l < nc) {
        m0 = at(2 * l);
        s0 = at(2 * l + 1);
    }
    if (l + 32 < nc) {
        m1 = at(2 * (l + 32));
        s1 = at(2 * (l + 32) + 1);
    }
    double mm = fmax(m0, m1);
    for (int c = l + 64; c < nc; c += 32) mm = fmax(mm, at(c * 2));
    mm = fold_halves(mm, -INFINITY, [](double x, double y) { return fmax(x, y); });
    ra.m = lane_f64(mm, 31);
    rb.m = lane_f64(mm, 63);
    mm = lane < 32 ? ra.m : rb.m;
    double z = 0.0;
    if (l < nc) z = s0 * exp_softmax(m0 - mm, ek);
    if (l + 32 < nc) z += s1 * exp_softmax(m1 - mm, ek);
    for (int c = l + 64; c < nc; c += 32) z += at(c * 2 + 1) * exp_softmax(at(c * 2) - mm, ek);
    z = fold_halves(z, 0.0, [](double x, double y) { return x + y; });
    ra.Z = lane_f64(z, 31);
    rb.Z = lane_f64(z, 63);
}
// ---------------------------------------------------------------------------------------
// LOGITS mode: per row and group of ws.stat_group chunks, a reference and the sum of exp(z / T - reference), fp64.
// grid = (n_stat_groups, (2 * S_max + 1) * B): workgroup row k * B + i takes, of request i, target row k / 2 for even k and
// draft row k / 2 for odd k, so that the rows of the first drafts are all started before any row of a second draft.
// Each lane sums exp(z / T) itself over its own elements (16 per chunk) as long as the wave's are within reach (600 temperatures of
// 0), and exp(z / T) / 2^shift from then on: the shift is the wave's, by the largest logit of the chunk that called for it, and moves
// only when one lies 600 temperatures further up, so the chunks of a group need no exchange between lanes but then; lanes and waves are
// combined once, at the end.  Any reference gives the same probabilities; it has to keep the exponents in range.
// us a launch, 128 requests x 128256 in fp32, a reference taken off every logit / from the logits themselves where those are within
// reach and else read again / like this: T = 0.005 95 / 181 / 86, all but 50 logits a row masked by -1e9 64 / 117 / 59, T = 1 118 /
// 105 / 101; 16 requests 26 / 41 / 25, 24.5 / 35 / 25, 26 / 22 / 22.  Registers decide: calls of few rows are workgroups' latencies, and
// 1 to 3 us slower with five waves per SIMD than with six (in fp32 the spills of seven cost as much; in bf16, us a call with six / seven, 64
// requests x 128256 96.6 / 95.8, 16 with all but 50 logits masked 41.5 / 40.6); those that leave rows out are 3 % faster with five.
// The rows are read once here, with the non-temporal hint (512 requests x 152064 in fp32: call 533 us without, 508 with).  What
// bounds it is both the rows' bytes and the fp64 instructions: 512 requests 455 us a launch with a reference taken off every logit
// and ordinary loads, 394 like this (about 2.3 GB; vector ALUs 70 % busy); 16 requests x 128256 in bf16 23.8 / 18.4.
// ---------------------------------------------------------------------------------------
template <typename RT, bool SKIP>  // SKIP: rows behind a rejection are left out (ws.skip)
__global__ __launch_bounds__(kThreads, SKIP ? 5 : sizeof(RT) == 2 ? 7 : 6) void accept_stats_kernel(
    const RT* __restrict__ z_target, const RT* __restrict__ z_draft, const int32_t* __restrict__ draft_tokens,
    const float* __restrict__ u_accept, const int32_t* __restrict__ cu_t, const int32_t* __restrict__ cu_d,
    const int32_t* __restrict__ t_rows, const int32_t* __restrict__ d_rows, Workspace ws, int B, int V, int S_max, double T,
    TempScale ts) {
    __shared__ double s_sum[kThreads / 64], s_direct[kThreads / 64], s_shift[kThreads / 64];
    __shared__ float s_max[kThreads / 64];
    __shared__ uint2 s_exp[256];
    __shared__ int s_behind, s_last;
    pass_over_nans();
    const int nc = n_chunks_of(V), nsg = n_stat_groups_of(V, ws.stat_group);
    const int k = blockIdx.y / B, i = blockIdx.y - k * B, j = k >> 1;
    const int t0 = cu_t[i], t_i = cu_t[i + 1] - t0, d0 = cu_d[i], d_i = cu_d[i + 1] - d0;
    const RT* rows;
    double* stat;
    if ((k & 1) == 0) {
        const long long r = (long long)t0 + j;
        // no such row, or past what the workspace or the caller's row map holds (offsets of an invalid call)
        if (j >= t_i || t0 < 0 || r >= (long long)B * (S_max + 1) || r >= cu_t[B]) return;
        rows = z_target + (size_t)(t_rows ? t_rows[r] : r) * V;
        stat = ws.stat_t + (size_t)r * nsg * 2;
    } else {
        const long long r = (long long)d0 + j;
        if (j >= d_i || d0 < 0 || r >= (long long)B * S_max || r >= cu_d[B]) return;
        rows = z_draft + (size_t)(d_rows ? d_rows[r] : r) * V;
        stat = ws.stat_d + (size_t)r * nsg * 2;
    }
    const int c_first = blockIdx.x * ws.stat_group, c_end = min(nc, c_first + ws.stat_group);
    const int c_whole = min(c_end, V / kChunk);  // chunks before it are whole
    // (as they come from memory: made floats where they are loaded, 16-bit ones take twice the registers, and are waited for there:
    // us a launch, 16 requests x 128256 20.0 / 18.4)
    typedef decltype(raw_quad<true>(rows, 0)) Raw;
    Raw va[kPerThread / 4], vb[kPerThread / 4];
    auto load_chunk = [&](int c, Raw (&v)[kPerThread / 4]) {
#pragma unroll
        for (int q = 0; q < kPerThread / 4; ++q) v[q] = raw_quad<true>(rows, c * kChunk + (q * kThreads + threadIdx.x) * 4);
    };
    auto load_checked = [&](int c, float (&v)[kPerThread]) {
#pragma unroll
        for (int q = 0; q < kPerThread / 4; ++q) {
            float x[4];
            load_quad(rows, c * kChunk + (q * kThreads + (int)threadIdx.x) * 4, V, x, -INFINITY);
#pragma unroll
            for (int u = 0; u < 4; ++u) v[q * 4 + u] = x[u];
        }
    };
    const uint2 entry = exp_table_entry();
    if (!SKIP && c_first < c_whole) load_chunk(c_first, va);  // (in flight while the table is filled)
    // If a draft before this row's has been rejected, nothing will read the row's statistics.  One lane asks for the whole
    // workgroup: other workgroups may lower the word at any time, and waves that asked for themselves could differ.
    if (threadIdx.x == 0)
        s_behind = SKIP && j > 0 &&
                   __hip_atomic_load(stat_words(ws, i, nc), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (unsigned)j;
    s_exp[threadIdx.x] = entry;
    __syncthreads();
    if (s_behind) return;
    if (SKIP && c_first < c_whole) load_chunk(c_first, va);
    float mz = -INFINITY;  // of logits that no shift fits: a reference, one of them,
    double sum = 0.0;      // and the sum of exp(z / T - mz / T) over those of them in this lane
    double direct = 0.0, shift = 0.0;  // sum of exp(z / T) / 2^shift over this lane's other elements; the shift is the wave's
    if (ts.reach > 0.0f) {
        ExpDirect ed = exp_direct(s_exp, ts);
        float plain = ts.reach;  // up to which logits are taken without a look at the shift: none once there is one
        double lowest = -kReach * T;  // the shift less 600
        float highest = ts.reach, significant = (float)(-500.0 / kReach) * ts.reach;  // and 600 more, 500 less
        auto add_chunk = [&](const float (&v)[kPerThread]) {
            float top = 0.0f;
#pragma unroll
            for (int u = 0; u < kPerThread; u += 2) top = max3_abs(top, v[u], v[u + 1]);
            if (__builtin_amdgcn_ballot_w64(!(top <= plain)) == 0) {
                const double before = direct;
#pragma unroll
                for (int u = 0; u < kPerThread; ++u) {
                    const ExpParts e = exp_of_logit((double)v[u], ed);
                    direct = fma(e.power, e.series, direct);
                }
                if (__builtin_amdgcn_ballot_w64(direct != direct) == 0) return;
                direct = before;  // a NaN logit counts as masked
            }
            float hi = -INFINITY;
#pragma unroll
            for (int u = 0; u < kPerThread; u += 2) hi = max3(hi, v[u], v[u + 1]);
            const bool low = __builtin_amdgcn_ballot_w64(hi >= significant) == 0;
            // masked logits only, or nothing beside what the wave has seen
            if (low && (__builtin_amdgcn_ballot_w64(hi != -INFINITY) == 0 || __builtin_amdgcn_ballot_w64(direct >= kAmple) != 0)) return;
            if (low || __builtin_amdgcn_ballot_w64(hi > highest) != 0) {  // a shift by the largest
                double T_ = T, c = ts.c;
                asm volatile("" : "+s"(T_), "+s"(c));  // or what follows is worked out in front of the loop, and kept in registers
                const float m = wave_top(hi);
                if (!(fabs((double)m) <= kWidest * T_)) {
                    // Floats of such a size lie 6e5 temperatures apart: exp of the next is 0.
                    if (m > mz) {
                        mz = m;
                        sum = 0.0;
                    }
                    int n = 0;
#pragma unroll
                    for (int u = 0; u < kPerThread; ++u) n += v[u] == mz ? 1 : 0;
                    sum += (double)n;
                    return;
                }
                // (no further down than the sum allows)
                const double at = __builtin_amdgcn_ballot_w64(direct > 0.0) != 0 ? fmax((double)m, lowest) : (double)m;
                const double to = uniform(rint(at * (c / 256.0)));
                direct = ldexp(direct, (int)fmin(fmax(shift - to, -5000.0), 5000.0));
                shift = to;
                plain = -1.0f;
                ed.magic = kRound - 256.0 * to;
                lowest = uniform((to * kLn2 - kReach) * T_);
                highest = uniform(-float_up(-(to * kLn2 + kReach) * T_));
                significant = uniform(float_up((to * kLn2 - 500.0) * T_));
            }
            // What is masked (-inf, NaN), or far below the rest, adds exp(-600) where something has added exp(-500) at least.
#pragma unroll
            for (int u = 0; u < kPerThread; ++u) {
                const ExpParts e = exp_of_logit(fmax((double)v[u], lowest), ed);
                direct = fma(e.power, e.series, direct);
            }
        };
        auto add_raw = [&](const Raw (&r)[kPerThread / 4]) {
            float v[kPerThread];
#pragma unroll
            for (int u = 0; u < kPerThread; ++u) v[u] = to_float(r[u / 4][u % 4]);
            add_chunk(v);
        };
        // Whole chunks: four vector loads per lane and chunk, all in flight together, the next chunk's issued before this one's
        // arithmetic, and only such loads in the loop: mixed with bounds-checked ones the compiler orders each vector load behind
        // all loads before it.
#pragma unroll 1
        for (int c = c_first; c < c_whole; c += 2) {
            if (c + 1 < c_whole) load_chunk(c + 1, vb);
            add_raw(va);
            if (c + 1 >= c_whole) break;
            if (c + 2 < c_whole) load_chunk(c + 2, va);
            add_raw(vb);
        }
        if (c_whole < c_end) {  // the chunk that holds the vocabulary's ragged end
            float v[kPerThread];
            load_checked(c_whole, v);
            add_chunk(v);
        }
    } else {  // a temperature out of all range: against a reference of the lane's own
        const ExpTable et = exp_table(s_exp);
        const double inv_T = 1.0 / T;
        float limit = -INFINITY;  // a logit above this makes a new reference
#pragma unroll 1
        for (int c = c_first; c < c_end; ++c) {
            float v[kPerThread];
            load_checked(c, v);
            float mx = v[0];
#pragma unroll
            for (int u = 1; u < kPerThread; ++u) mx = fmaxf(mx, v[u]);
            if (mx > limit) {
                if (mz != -INFINITY) sum *= exp_lookup(((double)mz - (double)mx) * inv_T, et);
                mz = mx;
                limit = mx + (float)(kStatSlack * T);
            }
            // (a masked logit -- -inf, NaN, past V -- or one far below the reference adds 1e-304)
#pragma unroll
            for (int u = 0; u < kPerThread; ++u) sum += exp_lookup(((double)v[u] - (double)mz) * inv_T, et);
        }
    }
    const ExpConsts ek = exp_consts();
    // lanes -> wave -> workgroup, each time against the common maximum
    const double inv_T = 1.0 / T;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    direct = wave_sum_to_last(direct);
    float mw = -INFINITY;
    if (__builtin_amdgcn_ballot_w64(mz != -INFINITY) != 0) {
        mw = wave_max(mz);
        sum = mz == -INFINITY ? 0.0 : sum * exp_softmax(((double)mz - (double)mw) * inv_T, ek);
        sum = wave_sum_to_last(sum);
    }
    if (lane == 63) {
        s_max[w] = mw;
        s_sum[w] = sum;
        s_direct[w] = direct;
        s_shift[w] = shift;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const float mg = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
        double mgT = -INFINITY, tot = (s_direct[0] + s_direct[1]) + (s_direct[2] + s_direct[3]);
        if (mg == -INFINITY && s_shift[0] == 0.0 && s_shift[1] == 0.0 && s_shift[2] == 0.0 && s_shift[3] == 0.0) {
            if (tot > 0.0) {  // a reference below the sum's largest term, which is at least 2^-15 of it
                mgT = kLn2 * (double)(ilogb(tot) - 16);
                tot *= exp_softmax(-mgT, ek);
            }
        } else {
            double out = 0.0, most = -INFINITY;
            tot = 0.0;
#pragma unroll 1
            for (int q = 0; q < kThreads / 64; ++q) {
                if (s_max[q] != -INFINITY) out += s_sum[q] * exp_softmax(((double)s_max[q] - (double)mg) * inv_T, ek);
                if (s_direct[q] > 0.0) most = fmax(most, s_shift[q]);
            }
#pragma unroll 1
            for (int q = 0; q < kThreads / 64; ++q)
                if (s_direct[q] > 0.0) tot += ldexp(s_direct[q], (int)fmax(s_shift[q] - most, -5000.0));
            if (mg != -INFINITY) mgT = (double)mg * inv_T;
            if (tot > 0.0) {
                const int up = ilogb(tot) - 16;
                most += (double)up;
                const double md = most * kLn2, top = fmax(mgT, md);
                // (md is rounded)
                tot = ldexp(tot, -up) * exp_softmax((mgT > md ? md - mgT : 0.0) - less_shift(md, most), ek) +
                      out * exp_softmax(mgT < md ? mgT - md : 0.0, ek);
                mgT = top;
            } else {
                tot = out;
            }
        }
        publish_f64(stat + blockIdx.x * 2, mgT);  // -inf for a group of masked logits only
        publish_f64(stat + blockIdx.x * 2 + 1, tot);
        s_last = 0;
        if (SKIP && j < d_i && j < S_max) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the pair is in memory before it is counted
            s_last = atomicAdd(stat_words(ws, i, nc) + 1 + j, 1u) + 1 == 2u * nsg;
        }
    }
    if (!SKIP || j >= d_i || j >= S_max) return;
    __syncthreads();
    if (!s_last || threadIdx.x >= 64) return;
    // the draft's rows are done (both lie inside the workspace and the row maps: their workgroups have checked): test it
    const long long rt = (long long)t0 + j, rd = (long long)d0 + j;
    RowStat st, sd;
    combine_stats<true>(ws.stat_t + (size_t)rt * nsg * 2, ws.stat_d + (size_t)rd * nsg * 2, nsg, ek, st, sd);
    const long long tr = t_rows ? t_rows[rt] : rt, dr = d_rows ? d_rows[rd] : rd;
    const int x = min(max(draft_tokens[dr], 0), V - 1);
    const double px = prob_of<FSR_LOGITS>(to_float(z_target[(size_t)tr * V + x]), T, st.m, st.Z, ek);
    const double qx = prob_of<FSR_LOGITS>(to_float(z_draft[(size_t)dr * V + x]), T, sd.m, sd.Z, ek);
    if (threadIdx.x == 0 && !((double)u_accept[dr] * qx < px)) atomicMin(stat_words(ws, i, nc), (unsigned)j);
}

constexpr double kBesideFar = 2.65e-261;  // exp(-600): a mass beside which 4096 of exp(-688) are nothing
// (a row's largest z / T lies at most 100 above its reference)
__device__ __forceinline__ RowScale row_scale(double m, double T, bool direct) {
    if (!direct) return RowScale{0.0, 0.0, 0.0f, 0.0f};
    const double shift = rint(m * 1.4426950408889634), zero = (m + kExpZero) * T;
    return RowScale{shift, less_shift(m, shift), float_up((shift * kLn2 + kExpTableFloor) * T), (float)(zero - 1e-6 * fabs(zero))};
}
__device__ __forceinline__ DrawScale draw_scale(const Decision& dec, double T, const TempScale& ts, const ExpConsts& ek) {
    const bool residual = dec.kind == kCaseResidual;
    const bool direct = ts.reach > 0.0f && fabs(dec.m_t) <= kWidest && (!residual || fabs(dec.m_d) <= kWidest);
    DrawScale sc{row_scale(dec.m_t, T, direct), row_scale(dec.m_d, T, direct && residual), 1.0, direct, 0};
    if (residual) sc.ratio = dec.Z_t / dec.Z_d * exp_softmax(sc.t.rest - sc.d.rest, ek);
    return sc;
}
// One logit of a direct row: its mass if it is not below `lowest`, else 0, and far if it may have one all the same.
__device__ __forceinline__ double mass_or_zero(float z, const RowScale& sc, const ExpDirect& ed, bool& far) {
    const bool in = z >= sc.lowest;
    far |= !in && z > sc.masked;
    const ExpParts e = exp_of_logit((double)max2(z, sc.lowest), ed);
    return in ? e.power * e.series : 0.0;
}
// Masses of four entries of a row in a draw: the probabilities themselves, or as RowScale says.
template <int MODE>
__device__ __forceinline__ void token_masses(const float (&z)[4], double inv_T, bool direct, const RowScale& sc,
                                             double m, const ExpDirect& ed, double (&mass)[4]) {
    if constexpr (MODE == FSR_PROBS) {
#pragma unroll
        for (int k = 0; k < 4; ++k) mass[k] = (double)z[k];
    } else {
        bool far = !direct;
        if (direct) {
#pragma unroll
            for (int k = 0; k < 4; ++k) mass[k] = mass_or_zero(z[k], sc, ed, far);
        }
        if (__builtin_amdgcn_ballot_w64(far) != 0) {  // hardly ever: one copy of exp_softmax, its constants made here
            const ExpConsts ek = exp_consts();
#pragma unroll 1
            for (int k = 0; k < 4; ++k) {
                const float zk = k == 0 ? z[0] : k == 1 ? z[1] : k == 2 ? z[2] : z[3];
                const bool take = !direct || (!(zk >= sc.lowest) && zk > sc.masked);
                if (__builtin_amdgcn_ballot_w64(take) == 0) continue;
                const double x = less_reference(zk, inv_T, m), v = x > kExpZero ? exp_softmax(x + sc.rest, ek) : 0.0;
#pragma unroll
                for (int u = 0; u < 4; ++u) mass[u] = take && u == k ? v : mass[u];
            }
        }
    }
}
// Residual p - q of two masses, in units of p's row; ratio: what one unit of q's row is in those.  Equal rows have a ratio of
// exactly 1 and leave exactly 0.
__device__ __forceinline__ double residual_of(double p, double q, double ratio) { return fma(-q, ratio, p); }
// Masses of 4 consecutive tokens starting at e for a draw from the row or from the residual (bounds-checked); their sum in
// the target row is added to `target`.
template <int MODE, typename RT>
__device__ __forceinline__ void quad_masses(bool residual, const RT* __restrict__ trow, const RT* __restrict__ drow, int e, int V,
                                            double inv_T, const Decision& dec,
                                            const DrawScale& sc, const ExpDirect& et, const ExpDirect& ed, double (&mass)[4], double& target) {
    constexpr float kNothing = MODE == FSR_LOGITS ? -INFINITY : 0.0f;  // past the vocabulary
    float a[4], b[4];
    load_quad(trow, e, V, a, kNothing);
    if (residual) load_quad(drow, e, V, b, kNothing);
    token_masses<MODE>(a, inv_T, sc.direct, sc.t, dec.m_t, et, mass);
    target += (mass[0] + mass[1]) + (mass[2] + mass[3]);
    if (residual) {
        double q[4];
        token_masses<MODE>(b, inv_T, sc.direct, sc.d, dec.m_d, ed, q);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double r = residual_of(mass[k], q[k], sc.ratio);
            mass[k] = r > 0.0 ? r : 0.0;
        }
    }
}

__device__ __forceinline__ double shfl_f64(double v, int src) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const uint32_t lo = __shfl((uint32_t)b, src, 64), hi = __shfl((uint32_t)(b >> 32), src, 64);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ long long shfl_i64(long long v, int src) {
    const uint32_t lo = __shfl((uint32_t)v, src, 64), hi = __shfl((uint32_t)((unsigned long long)v >> 32), src, 64);
    return (long long)(((unsigned long long)hi << 32) | lo);
}
// ---------------------------------------------------------------------------------------
// decide: PROBS mode, and where the statistics have found the outcome: one wave per request, lane n tests draft n.  LOGITS mode
// otherwise: one wave per draft (in rounds of the workgroup's waves, one more for the row behind the last draft), its lanes hold
// the row pair's statistics, so that a test is one memory round trip and two reductions; or, where that would be many rounds
// for rows of few pairs, a lane per draft that folds them four at a time, one round trip each (see decide_waves_of).
// ---------------------------------------------------------------------------------------
// combine_stats by one lane on its own (every lane of the wave works on a different row): the pairs four at a time, all
// eight loads of a batch in flight together, folded with a running maximum.
__device__ __forceinline__ RowStat combine_stats_lane(const double* __restrict__ stat, int nc, const ExpConsts& ek) {
    double mm = -INFINITY, z = 0.0;
    for (int c0 = 0; c0 < nc; c0 += 4) {
        double mc[4], sc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = min(c0 + u, nc - 1);
            mc[u] = stat[c * 2];
            sc[u] = stat[c * 2 + 1];
        }
        double mb = mc[0];
#pragma unroll
        for (int u = 1; u < 4; ++u) mb = fmax(mb, c0 + u < nc ? mc[u] : -INFINITY);
        if (mb > mm) {
            z = mm == -INFINITY ? 0.0 : z * exp_softmax(mm - mb, ek);
            mm = mb;
        }
        if (mm != -INFINITY) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (c0 + u < nc) z += sc[u] * exp_softmax(mc[u] - mm, ek);
        }
    }
    return RowStat{mm, z};
}
constexpr int kDecideWaves = 12;
// Waves of a request's workgroup (LOGITS mode, drafts not yet tested): twelve rows a round, or one wave with a lane per row.
// Measured, us a call with a lane / a wave per draft: one round: 16 requests of 8 drafts x 128256 bf16 51.8 / 48.3, 4 of 4 x 152064
// fp32 34.9 / 24.2, 2 of 8 x 32000 19.0 / 18.4; 32 pairs a row: two rounds, 8 of 12 x 128256 bf16 52.5 / 46.0, three, one of 24 31.4
// / 28.8; 16 pairs, three rounds, 8 of 24 60.1 / 61.7; 8 pairs, vocabulary 32000: two rounds, 2 of 16 20.2 / 22.3, three, of 32
// 22.4 / 28.8, six, of 64 27.9 / 43.5; one pair, one round, 60 of 11 x 4000 25.0 / 26.0.
int decide_waves_of(int S_max, int pairs) {
    const int rounds = (S_max + kDecideWaves) / kDecideWaves;
    return (rounds == 1 && pairs > 4) || 8 * rounds <= pairs ? std::min(kDecideWaves, S_max + 1) : 1;
}
// What a wave finds out about a draft, or (test unused) the row behind the last one.
struct DraftTest {
    long long t_row, d_row;
    double m_t, Z_t, m_d, Z_d;
    int x, ok;
};
template <int MODE, typename RT>
__global__ __launch_bounds__(MODE == FSR_LOGITS ? 64 * kDecideWaves : 64) void accept_decide_kernel(
    const RT* __restrict__ p_target, const RT* __restrict__ p_draft, const int32_t* __restrict__ draft_tokens,
    const float* __restrict__ u_accept, const int32_t* __restrict__ cu_t, const int32_t* __restrict__ cu_d,
    const int32_t* __restrict__ t_rows, const int32_t* __restrict__ d_rows, int32_t* __restrict__ accepted_len,
    int32_t* __restrict__ n_emitted, int32_t* __restrict__ emitted, Workspace ws, int B, int V, int S_max, double T, TempScale ts) {
    const int i = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int nsg = n_stat_groups_of(V, ws.stat_group);
    const int t0 = cu_t[i], t_i = cu_t[i + 1] - t0, d0 = cu_d[i], d_i = cu_d[i + 1] - d0;
    int32_t* em = emitted + (size_t)i * (S_max + 1);
    Decision dec;
    dec.kind = kCaseNone;
    dec.n = 0;
    dec.t_row = dec.d_row = 0;
    dec.m_t = dec.m_d = 0.0;
    dec.Z_t = dec.Z_d = 1.0;
    if (threadIdx.x == 0) ws.arrivals[i] = 0u;
    // the per-row statistics hold B*(S_max+1) target and B*S_max draft rows: a call whose offsets
    // run past that (only possible after an invalid request) is refused for the requests beyond
    const bool fits = (long long)t0 + t_i <= (long long)B * (S_max + 1) && (long long)d0 + d_i <= (long long)B * S_max;
    if (d_i < 0 || d_i > S_max || t_i < d_i || t_i > d_i + 1 || t0 < 0 || d0 < 0 || !fits) {
        for (int s = threadIdx.x; s <= S_max; s += blockDim.x) em[s] = -1;
        if (threadIdx.x == 0) {
            accepted_len[i] = -1;
            n_emitted[i] = -1;
            ws.dec[i] = dec;
        }
        return;
    }
    const ExpConsts ek = exp_consts_for<MODE>();
    int n = d_i;  // accepted drafts
    if (MODE == FSR_LOGITS && ws.skip) {
        n = (int)min(*stat_words(ws, i, n_chunks_of(V)), (unsigned)d_i);
        for (int k = lane; k < n; k += 64) em[k] = min(max(draft_tokens[d_rows ? d_rows[d0 + k] : d0 + k], 0), V - 1);
        if (n < d_i) {
            dec.kind = kCaseResidual;
            dec.t_row = t_rows ? t_rows[t0 + n] : t0 + n;
            dec.d_row = d_rows ? d_rows[d0 + n] : d0 + n;
            RowStat st, sd;
            combine_stats<false>(ws.stat_t + (size_t)(t0 + n) * nsg * 2, ws.stat_d + (size_t)(d0 + n) * nsg * 2, nsg, ek, st, sd);
            dec.m_t = st.m; dec.Z_t = st.Z;
            dec.m_d = sd.m; dec.Z_d = sd.Z;
        }
    } else if (MODE == FSR_LOGITS && n_waves > 1) {
        __shared__ DraftTest s_test[kDecideWaves];
        for (int n0 = 0; n0 < t_i && n == d_i; n0 += n_waves) {
            const int k = n0 + w;
            if (k < t_i) {
                DraftTest t{};
                t.t_row = t_rows ? t_rows[t0 + k] : t0 + k;
                t.ok = 1;
                const double* stat_t = ws.stat_t + (size_t)(t0 + k) * nsg * 2;
                RowStat st, sd;
                if (k < d_i) {
                    t.d_row = d_rows ? d_rows[d0 + k] : d0 + k;
                    t.x = min(max(draft_tokens[t.d_row], 0), V - 1);
                    const double u = (double)u_accept[t.d_row];
                    const float z_t = to_float(p_target[(size_t)t.t_row * V + t.x]), z_d = to_float(p_draft[(size_t)t.d_row * V + t.x]);
                    combine_stats<false>(stat_t, ws.stat_d + (size_t)(d0 + k) * nsg * 2, nsg, ek, st, sd);
                    t.ok = u * prob_of<MODE>(z_d, T, sd.m, sd.Z, ek) < prob_of<MODE>(z_t, T, st.m, st.Z, ek);
                    t.m_d = sd.m; t.Z_d = sd.Z;
                } else {
                    combine_stats<false>(stat_t, stat_t, nsg, ek, st, sd);
                }
                t.m_t = st.m; t.Z_t = st.Z;
                if (lane == 0) s_test[w] = t;
            }
            __syncthreads();
            const int here = min(n_waves, t_i - n0);
            for (int q = 0; q < here; ++q) {  // (the same in every wave)
                const DraftTest& t = s_test[q];
                if (n0 + q < d_i && t.ok) {
                    if (threadIdx.x == 0) em[n0 + q] = t.x;
                    continue;
                }
                dec.kind = n0 + q < d_i ? kCaseResidual : kCaseTarget;
                n = n0 + q;
                dec.t_row = t.t_row; dec.m_t = t.m_t; dec.Z_t = t.Z_t;
                if (dec.kind == kCaseResidual) {
                    dec.d_row = t.d_row; dec.m_d = t.m_d; dec.Z_d = t.Z_d;
                }
                break;
            }
            if (dec.kind != kCaseNone) break;
            __syncthreads();  // before the next round's results
        }
        if (w != 0) return;
    } else {
        for (int n0 = 0; n0 < d_i && n == d_i; n0 += 64) {
            const int k = n0 + lane;
            const bool live = k < d_i;
            long long tr = 0, dr = 0;
            RowStat st{0.0, 1.0}, sd{0.0, 1.0};
            int x = 0;
            bool ok = true;
            if (live) {
                tr = t_rows ? t_rows[t0 + k] : t0 + k;
                dr = d_rows ? d_rows[d0 + k] : d0 + k;
                x = min(max(draft_tokens[dr], 0), V - 1);
                const double u = (double)u_accept[dr];
                if constexpr (MODE == FSR_LOGITS) {
                    st = combine_stats_lane(ws.stat_t + (size_t)(t0 + k) * nsg * 2, nsg, ek);
                    sd = combine_stats_lane(ws.stat_d + (size_t)(d0 + k) * nsg * 2, nsg, ek);
                }
                const double px = prob_of<MODE>(to_float(p_target[(size_t)tr * V + x]), T, st.m, st.Z, ek);
                const double qx = prob_of<MODE>(to_float(p_draft[(size_t)dr * V + x]), T, sd.m, sd.Z, ek);
                ok = u * qx < px;
            }
            const unsigned long long rejected = __builtin_amdgcn_ballot_w64(live && !ok);
            const int first = rejected ? (int)__builtin_ctzll(rejected) : 64;
            if (live && lane < first) em[k] = x;  // accepted drafts of this round of 64
            if (rejected) {
                n = n0 + first;
                dec.kind = kCaseResidual;
                dec.t_row = shfl_i64(tr, first);
                dec.d_row = shfl_i64(dr, first);
                dec.m_t = shfl_f64(st.m, first); dec.Z_t = shfl_f64(st.Z, first);
                dec.m_d = shfl_f64(sd.m, first); dec.Z_d = shfl_f64(sd.Z, first);
            }
        }
    }
    dec.n = n;
    if (dec.kind == kCaseNone && n == d_i && t_i == d_i + 1) {
        dec.kind = kCaseTarget;
        dec.t_row = t_rows ? t_rows[t0 + d_i] : t0 + d_i;
        if constexpr (MODE == FSR_LOGITS) {
            const double* stat_t = ws.stat_t + (size_t)(t0 + d_i) * nsg * 2;
            RowStat st, sd;
            combine_stats<false>(stat_t, stat_t, nsg, ek, st, sd);
            dec.m_t = st.m; dec.Z_t = st.Z;
        }
    }
    for (int s = n + lane; s <= S_max; s += 64) em[s] = -1;
    if constexpr (MODE == FSR_LOGITS) {
        const DrawScale sc = draw_scale(dec, T, ts, ek);  // (here, once, and not in every workgroup that sums a part of the rows)
        if (lane == 0) ws.scale[i] = sc;
    }
    if (lane == 0) {
        accepted_len[i] = n;
        n_emitted[i] = n;  // the sampling kernel adds the drawn token
        ws.dec[i] = dec;
    }
}

// ---------------------------------------------------------------------------------------
// sample: request i = blockIdx.y; this workgroup owns chunks group * blockIdx.x .. + group - 1 of the
// vocabulary (SINGLE: group is 1).  grid = (ceil(n_chunks / group), B)
// Where a wave meets no residual in a chunk it sums the target row's masses as well, in case there is none anywhere (a
// drafted token without probability, rows that are equal otherwise); left to the request's last workgroup, such a call of
// 16 requests took 57 us in place of 17 (PROBS) and 127 in place of 50 (LOGITS), one of 128 requests 76 in place of 31 and
// 210 in place of 116.  LOGITS: four waves per SIMD, 128 registers (133 and three: 573 in place of 560 us a call of 512).
// A large call is bound by the rows' bytes (PROBS) or by fp64 instructions (LOGITS: exp by table look-up, see exp_of_logit);
// a small one is a latency chain (decision, rows, sums, arrival, chunk search, chunk scan), so what lies on it is kept
// short: sums over a wave by DPP, the search over the chunk masses by one wave.  Measured, us a launch before / after:
// PROBS 16 requests 17.6 / 13.4, chunks of 512 requests' drafts (mean of four) 47.5 / 39.3; LOGITS 16 requests in bf16
// 20.8 / 16.4, 512 requests 183 / 148.  The scales of the rows are worked out by `decide`, and what is hardly ever needed has one copy of
// exp_softmax: a small call pays for code that it fetches (4 requests, LOGITS: 80 KB of it 24.0 us, 48 KB 23.1).  LOGITS calls with masked logits, 128 requests x 128256 in fp32, us a call with such
// chunks read again by the checked path / summed from the registers: all but 50 logits of a row masked 171 / 158, every
// second one 164 / 141.  Exponents spread over several hundred, us a launch with every chunk that holds one below exp(-700) read again / only
// where a wave has nothing beside them: 128 requests T = 0.02 97 / 59, 16 requests 26.6 / 23.7.  References beyond 580 by the
// checked path / by the shift: T = 0.005 82 / 69, 29.7 / 24.2.
// ---------------------------------------------------------------------------------------
template <int MODE, typename RT, bool SINGLE>
__global__ __launch_bounds__(kThreads, MODE == FSR_LOGITS ? 4 : 1) void accept_sample_kernel(
    const RT* __restrict__ p_target, const RT* __restrict__ p_draft, const float* __restrict__ u_sample,
    int32_t* __restrict__ n_emitted, int32_t* __restrict__ emitted, Workspace ws, int V, int S_max, double T, TempScale ts,
    int group) {
    constexpr int kMost = SINGLE ? 1 : kMaxSampleGroup;
    __shared__ double s_part[kThreads / 64][kMost], s_part_t[kThreads / 64][kMost];
    __shared__ double s_wave[kThreads / 64];
    __shared__ int s_i[kThreads / 64];
    __shared__ double s_base, s_thr;
    __shared__ int s_chunk, s_fallback, s_last;
    __shared__ uint2 s_exp[MODE == FSR_LOGITS ? 256 : 1];
    const int nc = n_chunks_of(V), i = blockIdx.y;
    if (SINGLE) group = 1;
    const int c_first = blockIdx.x * group, n_here = min(group, nc - c_first);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t* em = emitted + (size_t)i * (S_max + 1);
    Decision dec = ws.dec[i];
    dec.kind = __builtin_amdgcn_readfirstlane(dec.kind);  // the same in every lane: say so, branches on it stay scalar
    if (dec.kind == kCaseNone) return;
    DrawScale sc{{}, {}, 1.0, 0, 0};
    if constexpr (MODE == FSR_LOGITS) sc = ws.scale[i];
    sc.direct = __builtin_amdgcn_readfirstlane(sc.direct);

    // ---- 2. fp64 mass of this workgroup's chunks of the sampling distribution
    const RT* trow = p_target + (size_t)dec.t_row * V;
    const RT* drow = p_draft + (size_t)dec.d_row * V;
    const double inv_T = 1.0 / T;
    // whole chunks go through code that has only vector loads; a row without a direct form (see RowScale) through the checked one
    const bool residual = dec.kind == kCaseResidual;
    const int n_whole = MODE == FSR_PROBS || sc.direct ? min(n_here, max(0, V / kChunk - c_first)) : 0;
    float ta[kPerThread], da[kPerThread];
    auto load_rows = [&](int c, float (&t)[kPerThread], float (&d)[kPerThread]) {
#pragma unroll
        for (int k = 0; k < kPerThread / 4; ++k) {
            const int e = c * kChunk + (k * kThreads + threadIdx.x) * 4;
            float x[4], y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            load_quad_vec(trow, e, x);
            if (residual) load_quad_vec(drow, e, y);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                t[4 * k + u] = x[u];
                d[4 * k + u] = y[u];
            }
        }
    };
    uint2 entry{};
    if constexpr (MODE == FSR_LOGITS) entry = exp_table_entry();
    if (n_whole > 0) load_rows(c_first, ta, da);  // (in flight while the table is filled)
    if constexpr (MODE == FSR_LOGITS) __builtin_amdgcn_sched_barrier(0);
    // A draw needs no normalisation: its masses are relative to each other only.
    ExpDirect et{}, ed{};  // of the target row and of the draft row
    if constexpr (MODE == FSR_LOGITS) {
        s_exp[threadIdx.x] = entry;
        ed = exp_direct(s_exp, ts);
        et = shifted(ed, sc.t.shift);
        ed = shifted(ed, sc.d.shift);
        __syncthreads();
    }
    // A workgroup takes `group` consecutive chunks: the chain every workgroup goes through (decision record,
    // row loads, reduction, store-through, arrival count) is paid once per 128 KB instead of once per 32 KB.
    auto chunk_mass_checked = [&](int c, double& target) __attribute__((always_inline)) {  // any chunk, element by element
        double r = 0.0;
        target = 0.0;
#pragma unroll
        for (int k = 0; k < kPerThread / 4; ++k) {
            double m[4];
            quad_masses<MODE, RT>(dec.kind == kCaseResidual, trow, drow, c * kChunk + (k * kThreads + threadIdx.x) * 4, V,
                                  inv_T, dec, sc, et, ed, m, target);
            r += (m[0] + m[1]) + (m[2] + m[3]);
        }
        return r;
    };
    {
        // whole chunks first, through code that has only vector loads (the next chunk's issued before
        // this chunk's arithmetic); then the chunk with the vocabulary's ragged end,
        // bounds-checked.  A chunk's mass goes to LDS as soon as the wave has it.
        unsigned todo = ((1u << n_here) - 1u) & ~((1u << n_whole) - 1u);  // chunks left to the checked path
        // A wave's masses of chunk cc to LDS.  Only a residual that is zero everywhere needs the target row's: a wave sums
        // those where it has met no residual.
        auto put = [&](int cc, double r, double target) {
            const bool none = residual && __builtin_amdgcn_ballot_w64(r > 0.0) == 0;
            r = wave_sum_to_last(r);
            if (none) target = wave_sum_to_last(target);
            if (lane == 63) {
                s_part[w][cc] = r;
                if (residual) s_part_t[w][cc] = none ? target : 0.0;
            }
        };
        auto sum_chunk = [&](int cc, const float (&t)[kPerThread], const float (&d)[kPerThread]) {
            double r = 0.0, target = 0.0;
            if constexpr (MODE == FSR_LOGITS) {
                // Without a check per token where no logit of the wave lies below its row's `lowest`; where some do, those counted
                // as 0: they are masked (-inf, NaN, or so low that exp is 0), or have a mass of less than exp(-688), which
                // is nothing beside a sum of exp(-600); the checked path where the wave has neither.  Otherwise the values are
                // those of token_masses.
                bool far = false;
                auto sum = [&](auto masked) {
                    auto mass = [&](float z, const RowScale& rs, const ExpDirect& k) {
                        if constexpr (decltype(masked)::value) {
                            return mass_or_zero(z, rs, k, far);
                        } else {
                            const ExpParts e = exp_of_logit((double)z, k);
                            return e.power * e.series;
                        }
                    };
                    double acc = 0.0;
#pragma unroll
                    for (int u = 0; u < kPerThread; ++u) {
                        if (residual) {
                            const double x = residual_of(mass(t[u], sc.t, et), mass(d[u], sc.d, ed), sc.ratio);
                            acc += x < 0.0 ? 0.0 : x;  // (keeps a NaN)
                        } else {
                            acc += mass(t[u], sc.t, et);
                        }
                    }
                    return acc;
                };
                float lo_t = t[0], lo_d = residual ? d[0] : INFINITY;
#pragma unroll
                for (int u = 1; u + 1 < kPerThread; u += 2) lo_t = min3(lo_t, t[u], t[u + 1]);
                lo_t = min3(lo_t, t[kPerThread - 1], lo_t);
                if (residual) {
#pragma unroll
                    for (int u = 1; u + 1 < kPerThread; u += 2) lo_d = min3(lo_d, d[u], d[u + 1]);
                    lo_d = min3(lo_d, d[kPerThread - 1], lo_d);
                }
                const float low_d = residual ? sc.d.lowest : -INFINITY;
                bool plain = __builtin_amdgcn_ballot_w64(!(lo_t >= sc.t.lowest && lo_d >= low_d)) == 0;
                if (plain) {
                    r = sum(std::false_type{});
                    plain = __builtin_amdgcn_ballot_w64(r != r) == 0;  // a NaN logit counts as masked
                }
                if (!plain) {
                    r = sum(std::true_type{});
                    if (__builtin_amdgcn_ballot_w64(far) != 0 && __builtin_amdgcn_ballot_w64(r > kBesideFar) == 0) {
                        todo |= 1u << cc;
                        return;
                    }
                }
                if (residual && __builtin_amdgcn_ballot_w64(r > 0.0) == 0) {
#pragma unroll
                    for (int u = 0; u < kPerThread; ++u) {
                        float z = t[u];
                        asm volatile("" : "+v"(z));  // or the compiler keeps sixteen masses of the loop above in registers
                        target += mass_or_zero(z, sc.t, et, far);
                    }
                }
            } else if (residual) {
#pragma unroll
                for (int k = 0; k < kPerThread; k += 4) {
                    double m[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const double x = (double)t[k + u] - (double)d[k + u];
                        m[u] = x > 0.0 ? x : 0.0;
                    }
                    r += (m[0] + m[1]) + (m[2] + m[3]);
                    target += ((double)t[k] + (double)t[k + 1]) + ((double)t[k + 2] + (double)t[k + 3]);
                }
            } else {
#pragma unroll
                for (int k = 0; k < kPerThread; k += 4)
                    r += ((double)t[k] + (double)t[k + 1]) + ((double)t[k + 2] + (double)t[k + 3]);
            }
            put(cc, r, target);
        };
        if (n_whole > 0) {
            float tb[kPerThread], db[kPerThread];
#pragma unroll 1
            for (int cc = 0; cc < n_whole; cc += 2) {
                if (cc + 1 < n_whole) load_rows(c_first + cc + 1, tb, db);
                sum_chunk(cc, ta, da);
                if (cc + 1 >= n_whole) break;
                if (cc + 2 < n_whole) load_rows(c_first + cc + 2, ta, da);
                sum_chunk(cc + 1, tb, db);
            }
        }
#pragma unroll 1
        while (todo) {
            const int cs = __builtin_ctz(todo);
            todo &= todo - 1;
            double target;
            const double r = chunk_mass_checked(c_first + cs, target);
            put(cs, r, target);
        }
        __syncthreads();
        if (w == 0) {
            if (lane < n_here) {
                double r = 0.0;
#pragma unroll
                for (int k = 0; k < kThreads / 64; ++k) r += s_part[k][lane];
                publish_f64(ws.mass_res + (size_t)i * nc + c_first + lane, r);
                if (residual && !(r > 0.0))
                    publish_f64(ws.mass_tgt + (size_t)i * nc + c_first + lane,
                                (s_part_t[0][lane] + s_part_t[1][lane]) + (s_part_t[2][lane] + s_part_t[3][lane]));
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // all are in memory before the arrivals are counted
            if (lane == 0) s_last = atomicAdd(ws.arrivals + i, (unsigned)n_here) + (unsigned)n_here == (unsigned)nc;
        }
        __syncthreads();
        if (!s_last) return;
    }

    // ---- 3. the request's last workgroup draws the token: total mass and the chunk that holds u * R, by one wave (lane
    // l takes chunks l, l + 64, ...; the masses come from memory, other workgroups wrote them)
    auto search = [&](const double* masses, bool last_resort) {  // false: no mass at all
        double v0 = 0.0, inc0 = 0.0, R = 0.0;
        for (int c0 = 0; c0 < nc; c0 += 64) {
            const double v = c0 + lane < nc ? fetch_f64(masses + c0 + lane) : 0.0, inc = wave_inclusive_scan(v);
            if (c0 == 0) {
                v0 = v;
                inc0 = inc;
            }
            R += shfl_f64(inc, 63);
        }
        if (!(R > 0.0) && !last_resort) return false;
        const double thr = (double)u_sample[i] * R;
        double carry = 0.0, base = 0.0;
        int chunk = -1, last_pos = 0;
        double last_base = 0.0;
        for (int c0 = 0; c0 < nc; c0 += 64) {
            const double v = c0 == 0 ? v0 : c0 + lane < nc ? fetch_f64(masses + c0 + lane) : 0.0;
            const double inc = c0 == 0 ? inc0 : wave_inclusive_scan(v);
            const double up = __shfl_up(inc, 1, 64), before = carry + (lane == 0 ? 0.0 : up);
            const unsigned long long with_mass = __builtin_amdgcn_ballot_w64(v > 0.0);
            const unsigned long long past = __builtin_amdgcn_ballot_w64(v > 0.0 && carry + inc > thr);
            if (past) {
                chunk = c0 + (int)__builtin_ctzll(past);
                base = shfl_f64(before, chunk - c0);
                break;
            }
            if (with_mass) {
                last_pos = c0 + 63 - (int)__builtin_clzll(with_mass);
                last_base = shfl_f64(before, last_pos - c0);
            }
            carry += shfl_f64(inc, 63);
        }
        if (chunk < 0) {  // rounding left no chunk: the last chunk with mass
            chunk = last_pos;
            base = last_base;
        }
        if (lane == 0) {
            s_base = base;
            s_thr = thr;
            s_chunk = chunk;
        }
        return true;
    };
    if (w == 0) {
        const bool found = search(ws.mass_res + (size_t)i * nc, false);
        if (lane == 0) s_fallback = !found;
    }
    __syncthreads();
    if (s_fallback) {  // the residual is all zero: sample from the target row itself
        if (w == 0) search((dec.kind == kCaseResidual ? ws.mass_tgt : ws.mass_res) + (size_t)i * nc, true);
        dec.kind = kCaseTarget;
        __syncthreads();
    }
    const double thr = s_thr;
    const int cs = s_chunk;

    // scan inside the chunk: thread t owns tokens [16 t, 16 t + 16) of the chunk
    const int e0 = cs * kChunk + threadIdx.x * kPerThread;
    double mass[kPerThread];
    double local = 0.0, unused = 0.0;
#pragma unroll
    for (int k = 0; k < kPerThread / 4; ++k) {
        double m[4];
        quad_masses<MODE, RT>(dec.kind == kCaseResidual, trow, drow, e0 + 4 * k, V, inv_T, dec, sc, et, ed, m, unused);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            mass[4 * k + j] = m[j];
            local += m[j];
        }
    }
    const double inc = wave_inclusive_scan(local);
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    double run = s_base + (inc - local);
    for (int k = 0; k < w; ++k) run += s_wave[k];
    int hit = INT_MAX, last_pos = -1;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        run += mass[k];
        if (mass[k] > 0.0) {
            last_pos = e0 + k;
            if (run > thr && hit == INT_MAX) hit = e0 + k;
        }
    }
    hit = wave_min_i(hit);
    last_pos = wave_max_i(last_pos);
    __syncthreads();
    if (lane == 0) s_i[w] = hit;
    __syncthreads();
    hit = min(min(s_i[0], s_i[1]), min(s_i[2], s_i[3]));
    __syncthreads();
    if (lane == 0) s_i[w] = last_pos;
    __syncthreads();
    last_pos = max(max(s_i[0], s_i[1]), max(s_i[2], s_i[3]));
    if (threadIdx.x == 0) {
        int tok = hit != INT_MAX ? hit : last_pos;
        if (tok < 0) tok = 0;  // only if no token of the row has any mass; keeps the id in range
        em[dec.n] = tok;
        n_emitted[i] = dec.n + 1;
    }
}

// Chunks per workgroup of accept_sample.
// PROBS: a compute unit holds four of its workgroups, and they are alike, so what counts is how many times over the device is
// filled and what one workgroup takes: its chunks and about two more for the chain it goes through.  Vocabulary 128256, us a
// call with 1, 2, 4 or 8 chunks, as many as leave 1024 workgroups / like this: 16 requests 16.9 / 16.9, 48 23.3 / 18.5, 96 24.4 /
// 22.2, 256 48.6 / 48.2; 152064, 128 28.9 / 29.2, 384 82 / 82.  Beyond two rounds of the largest workgroups the places are taken as
// they come free (some requests have nothing to sample) and most chunks a workgroup are best: the draw of a chunked step of
// 512 requests 40.3 us with 8, 45.6 with the 10 that would make it two rounds.  One chunk / two / three for the chain: 384 x 152064 75.6 /
// 72.1 / 72.0, 30 sizes of 16 to 512 requests and 32000 to 152064 tokens otherwise alike.
// LOGITS: the chain is a smaller part: 96 requests 119.6 / 116.8, 128 165 / 167, 512 503 / 509.
constexpr int kSamplePlaces = 1024;
int sample_group_of(int mode, int B, int nc) {
    if (mode == FSR_LOGITS) {
        int g = 8;
        while (g > 1 && (long long)B * ((nc + g - 1) / g) < kSamplePlaces) g >>= 1;
        return g;
    }
    if ((long long)B * ((nc + kMaxSampleGroup - 1) / kMaxSampleGroup) > 2 * kSamplePlaces) return kMaxSampleGroup;
    int best = 1;
    long long least = LLONG_MAX;
    for (int g = 1; g <= kMaxSampleGroup; ++g) {
        const long long groups = (long long)B * ((nc + g - 1) / g), cost = (groups + kSamplePlaces - 1) / kSamplePlaces * (std::min(g, nc) + 2);
        if (cost < least) {
            least = cost;
            best = g;
        }
    }
    return best;
}

template <int MODE, typename RT>
int launch_all(const RT* p_target, const RT* p_draft, const int32_t* draft_tokens, const float* u_accept,
               const float* u_sample, const int32_t* cu_t, const int32_t* cu_d, const int32_t* t_rows,
               const int32_t* d_rows, int32_t* accepted_len, int32_t* n_emitted, int32_t* emitted,
               const fsr_accept_params& p, const Workspace& ws_in, hipStream_t s) {
    Workspace ws = ws_in;
    const int nc = n_chunks_of(p.V);
    const double T = p.temperature;
    const TempScale ts = MODE == FSR_LOGITS ? temp_scale(T) : TempScale{};
    int rc;
    if (MODE == FSR_LOGITS) {
        const int rows_cap = p.B * (2 * p.S_max + 1);
        // chunks per workgroup: as many as leave the device a few thousand workgroups (a small call is a latency
        // chain per workgroup, and more of them in parallel is what shortens it)
        int sg = kMaxStatGroup;
        while (sg > 1 && (long long)rows_cap * n_stat_groups_of(p.V, sg) < 4096) sg >>= 1;
        ws.stat_group = sg;
        // Leaving rows out is worth its clearing launch and the counting where there are many rows; a small call has all
        // its rows in flight at once.  Vocabulary 128256, 1-8 drafts, fp32, us a call with / without: 16 requests 62.8 /
        // 52.2, 64 requests (1088 rows) 103.5 / 102.3, 128 requests (2176 rows) 170.6 / 182.4, 256 requests 284 / 336.
        if (rows_cap >= kSkipMinRows && p.S_max + 1 <= 2 * nc) {
            ws.skip = 1;
            const int n_words = p.B * 2 * nc;
            hipLaunchKernelGGL(accept_clear_kernel, dim3((n_words + kThreads - 1) / kThreads), dim3(kThreads), 0, s, ws, n_words, nc);
            if ((rc = check_launch("accept_clear_kernel")) != FSR_OK) return rc;
        }
        hipLaunchKernelGGL((ws.skip ? accept_stats_kernel<RT, true> : accept_stats_kernel<RT, false>), dim3(n_stat_groups_of(p.V, sg), rows_cap),
                           dim3(kThreads), 0, s, p_target, p_draft, draft_tokens, u_accept, cu_t, cu_d, t_rows, d_rows, ws, p.B, p.V, p.S_max, T, ts);
        if ((rc = check_launch("accept_stats_kernel")) != FSR_OK) return rc;
    }
    const int decide_waves = MODE == FSR_LOGITS && !ws.skip ? decide_waves_of(p.S_max, n_stat_groups_of(p.V, ws.stat_group)) : 1;
    hipLaunchKernelGGL((accept_decide_kernel<MODE, RT>), dim3(p.B), dim3(64 * decide_waves), 0, s, p_target, p_draft, draft_tokens, u_accept, cu_t,
                       cu_d, t_rows, d_rows, accepted_len, n_emitted, emitted, ws, p.B, p.V, p.S_max, T, ts);
    if ((rc = check_launch("accept_decide_kernel")) != FSR_OK) return rc;
    const int group = sample_group_of(MODE, p.B, nc);
    const dim3 grid((nc + group - 1) / group, p.B), block(kThreads);
    if (group == 1)
        hipLaunchKernelGGL((accept_sample_kernel<MODE, RT, true>), grid, block, 0, s, p_target, p_draft, u_sample, n_emitted, emitted, ws, p.V,
                           p.S_max, T, ts, group);
    else
        hipLaunchKernelGGL((accept_sample_kernel<MODE, RT, false>), grid, block, 0, s, p_target, p_draft, u_sample, n_emitted, emitted, ws, p.V,
                           p.S_max, T, ts, group);
    return check_launch("accept_sample_kernel");
}

int validate(const fsr_accept_params* p, const char* who) {
    if (!p) return fail(FSR_EINVAL, "%s: params is null", who);
    if (p->B < 0 || p->V <= 0 || p->S_max < 0 || p->reserved2 != 0)
        return fail(FSR_EINVAL, "%s: B=%d V=%d S_max=%d reserved2=%d", who, p->B, p->V, p->S_max, p->reserved2);
    if (p->dtype != FSR_F32 && p->dtype != FSR_BF16) return fail(FSR_EUNSUP, "%s: dtype=%d", who, p->dtype);
    if (p->dtype == FSR_BF16 && p->mode == FSR_GREEDY) return fail(FSR_EUNSUP, "%s: greedy mode takes fp32 rows", who);
    if (p->mode != FSR_PROBS && p->mode != FSR_LOGITS && p->mode != FSR_GREEDY) return fail(FSR_EUNSUP, "%s: mode=%d", who, p->mode);
    if (p->mode == FSR_LOGITS && !(p->temperature > 0.0)) return fail(FSR_EINVAL, "%s: temperature=%g must be > 0", who, p->temperature);
    if ((long long)p->B * (2LL * p->S_max + 1) > 65535) return fail(FSR_EUNSUP, "%s: B*(2*S_max+1)=%lld exceeds 65535 rows per call", who, (long long)p->B * (2LL * p->S_max + 1));
    return FSR_OK;
}

}  // namespace
}  // namespace fsr

using namespace fsr;

extern "C" int fsr_accept_workspace_bytes(const fsr_accept_params* p, size_t* out_bytes) {
    int rc = validate(p, "fsr_accept_workspace_bytes");
    if (rc != FSR_OK) return rc;
    if (!out_bytes) return fail(FSR_EINVAL, "fsr_accept_workspace_bytes: out_bytes is null");
    *out_bytes = p->mode == FSR_GREEDY ? greedy_workspace_bytes(*p) : carve(*p, nullptr, nullptr);
    return FSR_OK;
}

extern "C" int fsr_spec_accept(const void* p_target, const void* p_draft, const int32_t* draft_tokens,
                               const float* u_accept, const float* u_sample, const int32_t* cu_t, const int32_t* cu_d,
                               const int32_t* t_rows, const int32_t* d_rows, int32_t* accepted_len, int32_t* n_emitted,
                               int32_t* emitted, const fsr_accept_params* p, void* workspace, size_t ws_bytes,
                               void* stream) {
    int rc = validate(p, "fsr_spec_accept");
    if (rc != FSR_OK) return rc;
    if (p->B == 0) return FSR_OK;
    if (p->mode == FSR_GREEDY) {
        if (!p_target || !cu_t || !cu_d || !accepted_len || !n_emitted || !emitted)
            return fail(FSR_EINVAL, "fsr_spec_accept: null pointer among p_target/cu_t/cu_d/outputs");
        if (p->S_max > 0 && !draft_tokens) return fail(FSR_EINVAL, "fsr_spec_accept: draft_tokens is null with S_max=%d", p->S_max);
        const size_t need_g = greedy_workspace_bytes(*p);
        if (!workspace || ws_bytes < need_g) return fail(FSR_EWS, "fsr_spec_accept: workspace %zu bytes, need %zu", ws_bytes, need_g);
        if ((uintptr_t)workspace & 255) return fail(FSR_EWS, "fsr_spec_accept: workspace must be 256-byte aligned");
        return greedy_accept_launch((const float*)p_target, draft_tokens, cu_t, cu_d, t_rows, d_rows, accepted_len, n_emitted, emitted, *p,
                                    workspace, (hipStream_t)stream);
    }
    if (!p_target || !u_sample || !cu_t || !cu_d || !accepted_len || !n_emitted || !emitted)
        return fail(FSR_EINVAL, "fsr_spec_accept: null pointer among p_target/u_sample/cu_t/cu_d/outputs");
    if (p->S_max > 0 && (!p_draft || !draft_tokens || !u_accept))
        return fail(FSR_EINVAL, "fsr_spec_accept: p_draft/draft_tokens/u_accept is null with S_max=%d", p->S_max);
    Workspace ws;
    const size_t need = carve(*p, (char*)workspace, &ws);
    if (!workspace || ws_bytes < need) return fail(FSR_EWS, "fsr_spec_accept: workspace %zu bytes, need %zu", ws_bytes, need);
    if ((uintptr_t)workspace & 255) return fail(FSR_EWS, "fsr_spec_accept: workspace must be 256-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    // a request without drafts never dereferences the draft arrays; give the kernels a valid base
    if (!p_draft) p_draft = p_target;
    if (p->dtype == FSR_BF16) {
        const uint16_t* pt = (const uint16_t*)p_target;
        const uint16_t* pd = (const uint16_t*)p_draft;
        if (p->mode == FSR_LOGITS)
            return launch_all<FSR_LOGITS>(pt, pd, draft_tokens, u_accept, u_sample, cu_t, cu_d, t_rows, d_rows, accepted_len,
                                          n_emitted, emitted, *p, ws, s);
        return launch_all<FSR_PROBS>(pt, pd, draft_tokens, u_accept, u_sample, cu_t, cu_d, t_rows, d_rows, accepted_len,
                                     n_emitted, emitted, *p, ws, s);
    }
    const float* pt = (const float*)p_target;
    const float* pd = (const float*)p_draft;
    if (p->mode == FSR_LOGITS)
        return launch_all<FSR_LOGITS>(pt, pd, draft_tokens, u_accept, u_sample, cu_t, cu_d, t_rows, d_rows, accepted_len,
                                      n_emitted, emitted, *p, ws, s);
    return launch_all<FSR_PROBS>(pt, pd, draft_tokens, u_accept, u_sample, cu_t, cu_d, t_rows, d_rows, accepted_len,
                                 n_emitted, emitted, *p, ws, s);
}
