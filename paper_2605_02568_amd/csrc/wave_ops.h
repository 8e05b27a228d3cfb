// Reductions and scans over the 64 lanes of a wave on the vector ALU's own lane moves (DPP): about 8
// cycles a step, where a step through the LDS permute of __shfl waits for an LDS round trip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace si {

// Lane 63 ends up with op over all lanes, lane l with op over lanes 0..l (op associative, commutative).
template <typename T, typename Op>
__device__ __forceinline__ T wave_scan(T x, T identity, Op op) {
    static_assert(sizeof(T) == 4, "one register");
#define SI_DPP_STEP(CTRL, ROWS)                                                                              \
    x = op(x, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, identity),           \
                                                                __builtin_bit_cast(int, x), CTRL, ROWS, 0xf, false)));
    SI_DPP_STEP(0x111, 0xf)  // row_shr:1, :2, :4, :8 inside each row of 16 lanes
    SI_DPP_STEP(0x112, 0xf)
    SI_DPP_STEP(0x114, 0xf)
    SI_DPP_STEP(0x118, 0xf)
    SI_DPP_STEP(0x142, 0xa)  // last lane of rows 0 and 2 to rows 1 and 3
    SI_DPP_STEP(0x143, 0xc)  // lane 31 to rows 2 and 3
#undef SI_DPP_STEP
    return x;
}
template <typename T>
__device__ __forceinline__ T lane_value(T x, int lane) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ int wave_prefix_sum(int x) {  // inclusive
    return wave_scan(x, 0, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int wave_max(int x) {
    return lane_value(wave_scan(x, static_cast<int>(0x80000000), [](int a, int b) { return max(a, b); }), 63);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
    return lane_value(wave_scan(x, 0u, [](uint32_t a, uint32_t b) { return a | b; }), 63);
}
__device__ __forceinline__ uint32_t wave_and(uint32_t x) {
    return lane_value(wave_scan(x, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return a & b; }), 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    return lane_value(wave_scan(x, 0u, [](uint32_t a, uint32_t b) { return max(a, b); }), 63);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    return lane_value(wave_scan(x, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return min(a, b); }), 63);
}
__device__ __forceinline__ float wave_max(float x) {
    return lane_value(wave_scan(x, -__builtin_huge_valf(), [](float a, float b) { return fmaxf(a, b); }), 63);
}
__device__ __forceinline__ float wave_min(float x) {
    return lane_value(wave_scan(x, __builtin_huge_valf(), [](float a, float b) { return fminf(a, b); }), 63);
}
__device__ __forceinline__ float wave_sum(float x) {
    return lane_value(wave_scan(x, 0.0f, [](float a, float b) { return a + b; }), 63);
}

}  // namespace si
