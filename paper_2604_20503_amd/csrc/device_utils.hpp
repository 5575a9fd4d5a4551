// Wavefront-level (64 lanes) reductions and scans, and the arrival counter several kernels use to
// find out which workgroup is the last of a group to finish.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace fsr {

constexpr int kWave = 64;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Sum over the wave, valid in lane 63 only: lanes move data by DPP, which costs a few vector instructions per step where
// a shuffle waits for the LDS.
__device__ __forceinline__ double wave_sum_to_last(double v) {
    auto step = [&](auto ctrl, auto rows) {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        v += __builtin_bit_cast(double, ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});  // lanes 1, 2, 4, 8 to the left in a row of 16
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});  // lane 15 of a row to the next row
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});  // lane 31 to the upper half
    return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, kWave));
    return v;
}

// Inclusive scan across the 64 lanes of a wave.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        T up = __shfl_up(v, o, kWave);
        if (lane >= o) v += up;
    }
    return v;
}

// The same by DPP: no round trip through LDS per step.
__device__ __forceinline__ int wave_inclusive_scan_dpp(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // lanes 1, 2, 4, 8 to the left in a row of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // lane 15 of a row to the next row
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // lane 31 to the upper half
    return v;
}
// Largest of values that are not negative (floats of that kind keep their order as bits), in every lane.
__device__ __forceinline__ int wave_max_positive(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, kWave - 1);
}
__device__ __forceinline__ int wave_sum_i(int v) { return __builtin_amdgcn_readlane(wave_inclusive_scan_dpp(v), kWave - 1); }

// Count one more arrival on a 64-bit word that holds (call id << 16 | count).  A word left by another
// call (or never written) counts as zero, so the memory it lives in needs no clearing between calls
// and HIP-graph replays work.  Returns the count including this arrival.  Device scope.
// One round trip to memory where others of the call have arrived before (whoever comes last waits for nothing else): the word is
// added to before it is known whose it is, and one of another call's is replaced by this call's, whichever arrival manages that.
__device__ __forceinline__ int count_arrival(unsigned long long* word, unsigned long long call_id) {
    for (;;) {
        const unsigned long long seen = atomicAdd(word, 1ull);
        if ((seen >> 16) == call_id) return (int)(seen & 0xffffu) + 1;
        unsigned long long stale = seen + 1;
        for (;;) {
            const unsigned long long prev = atomicCAS(word, stale, (call_id << 16) | 1);
            if (prev == stale) return 1;
            if ((prev >> 16) == call_id) break;  // another arrival has: count on its word
            stale = prev;
        }
    }
}

}  // namespace fsr
