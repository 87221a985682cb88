// Cross-lane sums inside a wavefront on the vector ALUs (DPP moves and the
// gfx950 permlane swaps) instead of LDS-routed shuffles: a shuffle costs an
// LDS round trip per step, six in a row for a 64-lane sum, which is most of
// the time of a row of a few hundred entries.
#pragma once

#include "sk_internal.h"

namespace sk {

// DPP controls: lane l reads lane 15 - l of its row of 16, 7 - l of its half
// row, l ^ 2 and l ^ 1 of its quad.
constexpr int kDppRowMirror = 0x140, kDppHalfMirror = 0x141, kDppXor2 = 0x4e, kDppXor1 = 0xb1;

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// a and b of both halves of the wave (of each pair of 16-lane rows): lanes
// with bit 5 (bit 4) clear get the pair's sum of a, the others that of b, in
// float64.
__device__ __forceinline__ double swap_add32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return (double)__uint_as_float(r[0]) + (double)__uint_as_float(r[1]);
}
__device__ __forceinline__ double swap_add32(double a, double b) {
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double swap_add16(double a, double b) {
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
// The same across the halves of a 16-lane row (bit 3) and of a half row
// (bit 2), whose partner lane is the mirror image.
template <int CTRL>
__device__ __forceinline__ double fold_add(double a, double b, bool hi) {
    const double keep = hi ? b : a, send = hi ? a : b;
    return keep + dpp_mov<CTRL>(send);
}

// Sums of 16 values over the 64 lanes at once, added in float64: lane l gets
// the sum of f(l / 4) over the lanes. Each step halves the values a lane
// carries instead of adding all of them across the wave: 17 adds instead of
// 6 * 16.
template <class Fn>
__device__ __forceinline__ double wave_sums16(Fn f, int lane) {
    constexpr int R = 16;
    double a[R / 2], b[R / 4];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
        a[k] = swap_add32(f(k), f(k + R / 2));
        if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = 0; k < R / 4; ++k) b[k] = swap_add16(a[k], a[k + R / 4]);
    const double c0 = fold_add<kDppRowMirror>(b[0], b[2], (lane & 8) != 0);
    const double c1 = fold_add<kDppRowMirror>(b[1], b[3], (lane & 8) != 0);
    double s = fold_add<kDppHalfMirror>(c0, c1, (lane & 4) != 0);
    s += dpp_mov<kDppXor2>(s);
    s += dpp_mov<kDppXor1>(s);
    return s;
}

// The same for 8 values: lane l gets the sum of f(l / 8).
template <class Fn>
__device__ __forceinline__ double wave_sums8(Fn f, int lane) {
    double a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float x = f(k), y = f(k + 4);
        a[k] = swap_add32(x, y);
        __builtin_amdgcn_sched_barrier(0);  // a pair of values in hand at a time
    }
    const double b0 = swap_add16(a[0], a[2]), b1 = swap_add16(a[1], a[3]);
    double s = fold_add<kDppRowMirror>(b0, b1, (lane & 8) != 0);
    s += dpp_mov<kDppHalfMirror>(s);
    s += dpp_mov<kDppXor2>(s);
    s += dpp_mov<kDppXor1>(s);
    return s;
}

// The largest v over the 64 lanes, in every lane.
__device__ __forceinline__ float wave_max_v(float v) {
    v = fmaxf(v, dpp_mov<kDppXor1>(v));
    v = fmaxf(v, dpp_mov<kDppXor2>(v));
    v = fmaxf(v, dpp_mov<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_mov<kDppRowMirror>(v));
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float readlane_v(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double readlane_v(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

}  // namespace sk
