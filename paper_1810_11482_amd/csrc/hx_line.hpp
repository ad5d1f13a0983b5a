// Steps of a line held in a wave's registers, shared by the 1D kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hx {
namespace {

// DPP controls of the wave-wide shifts: lane i reads lane i-1 (shr) or i+1 (shl);
// the lane with no source reads 0.
constexpr int DPP_WAVE_SHL1 = 0x130;
constexpr int DPP_WAVE_SHR1 = 0x138;

template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

// One step of a whole wave tile, in place on the lane-contiguous registers a.
// The cell left of a lane's first comes from the lane below, the cell right of
// its last from the lane above (DPP wave shifts of the old values).  The
// neighbour sum of cell j+1 is formed from the old a[j] before a[j] is
// overwritten, so one array and two short-lived temporaries suffice and the
// register assignment is the same after every step (no register moves).  Per
// cell: s = l + rt; d = fma(-2, c, s); c' = fma(r, d, c).  Cells outside a
// zero-Dirichlet end are reset to 0 after the step.
template <typename T, int C>
__device__ __forceinline__ void step_tile(T (&a)[C], T k, bool zero_lo, bool zero_hi,
                                          int64_t lbase, int64_t n) {
    const T left = dpp_move<DPP_WAVE_SHR1>(a[C - 1]);
    const T right = dpp_move<DPP_WAVE_SHL1>(a[0]);
    T s_cur = left + (C > 1 ? a[1] : right);
#pragma unroll
    for (int j = 0; j < C; ++j) {
        T s_next = T(0);
        if (j + 1 < C) s_next = a[j] + (j + 2 < C ? a[j + 2] : right);
        const T d = fmaT(T(-2), a[j], s_cur);
        a[j] = fmaT(k, d, a[j]);
        s_cur = s_next;
    }
    if (zero_lo || zero_hi) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int64_t g = lbase + j;
            if ((zero_lo && g < 0) || (zero_hi && g >= n)) a[j] = T(0);
        }
    }
}

// One step of the rescaled form (see set_rate_1d): w' = w + b (w_l + w_r).
// Same register discipline as step_tile: one add and one fma per cell.
template <typename T, int C>
__device__ __forceinline__ void step_tile_scaled(T (&a)[C], T b, bool zero_lo, bool zero_hi,
                                                 int64_t lbase, int64_t n) {
    const T left = dpp_move<DPP_WAVE_SHR1>(a[C - 1]);
    const T right = dpp_move<DPP_WAVE_SHL1>(a[0]);
    T s_cur = left + (C > 1 ? a[1] : right);
#pragma unroll
    for (int j = 0; j < C; ++j) {
        T s_next = T(0);
        if (j + 1 < C) s_next = a[j] + (j + 2 < C ? a[j + 2] : right);
        a[j] = fmaT(b, s_cur, a[j]);
        s_cur = s_next;
    }
    if (zero_lo || zero_hi) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int64_t g = lbase + j;
            if ((zero_lo && g < 0) || (zero_hi && g >= n)) a[j] = T(0);
        }
    }
}

template <typename T, int C>
__device__ __forceinline__ void scale_tile(T (&a)[C], T f) {
#pragma unroll
    for (int j = 0; j < C; ++j) a[j] *= f;
}

}  // namespace
}  // namespace hx
