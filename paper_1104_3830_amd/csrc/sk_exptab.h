// Exact integer exponents and the LDS table of exp(E) shared by the
// log-domain kernels (sweeps, single pass, exact recompute).
#pragma once

#include <climits>

#include "sk_internal.h"

namespace sk {

// Every exponent the sweeps evaluate splits exactly into an integer part
// E_ij = p w_ij + F_i + G_j and the fractions phi_i, gam_j:
//   x_ij = exp(E_ij) * exp(phi_i) * exp(gam_j).
// exp(E) for integer E is read from a table in LDS, correctly rounded to
// float32; the fraction factors are one value per row and per column. Entries
// with E <= kTabLo contribute exp(-88) < 2^-126 (dropped: a sum in the safe
// range [2^-64, 2^64] of at most 16384 such terms changes by less than one
// part in 2^40); E >= kTabHi reads +inf, which sends the row or column to the
// exact max-shifted recompute. Integer arithmetic is exact: with p <= 2048
// and |w| < 2^15, |4 E| < 2^31.
constexpr int kTabLo = -88;
constexpr int kTabHi = 80;
constexpr int kTabN = kTabHi - kTabLo + 1;  // 169 entries
constexpr int kTabMaxOff = 4 * (kTabN - 1);  // byte offset of the +inf entry

// The table itself, formed at compile time: exp(k) as a product of the powers
// e^(2^b) of k's bits (each within half an ulp of float64, so a product of
// seven rounds to the float32 nearest exp(k)). A kernel that formed it with
// the FP64 exp spent 0.5-1 us of every launch on it before its first barrier.
struct ExpTable {
    float v[kTabN];
};
constexpr ExpTable make_exp_table() {
    constexpr double pw[7] = {2.718281828459045,      7.38905609893065,       54.598150033144236, 2980.9579870417283,
                              8886110.520507872,      78962960182680.69,      6.235149080811617e27};
    ExpTable t{};
    t.v[0] = 0.f;
    t.v[kTabN - 1] = __builtin_inff();
    for (int k = 1; k < kTabN - 1; ++k) {
        const int e = k + kTabLo, a = e < 0 ? -e : e;
        double x = 1.0;
        for (int b = 0; b < 7; ++b)
            if ((a >> b) & 1) x *= pw[b];
        t.v[k] = (float)(e < 0 ? 1.0 / x : x);
    }
    return t;
}
static __constant__ const ExpTable kExpTable = make_exp_table();

__device__ __forceinline__ void fill_exp_table(float *tab) {
    for (int k = threadIdx.x; k < kTabN; k += blockDim.x) tab[k] = kExpTable.v[k];
}

// Table read at a byte offset already clamped to [0, kTabMaxOff].
__device__ __forceinline__ float tab_at(const float *tab, int off) {
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(tab) + off);
}

// Byte offset of exp(E) with 4 E - 4 kTabLo = 4 p w + A + B (A, B prescaled);
// a sum outside int32 wraps.
__device__ __forceinline__ int tab_off(int p4, int w, int A, int B) {
    const int t = (int)((unsigned)__mul24(p4, w) + (unsigned)A + (unsigned)B);
    return min(max(t, 0), kTabMaxOff);
}

// Unpacks 8 int16 from a 16-byte vector as int32.
__device__ __forceinline__ void unpack8i(const int4 v, int (&w)[8]) {
    w[0] = (int)(short)(v.x & 0xffff); w[1] = v.x >> 16;
    w[2] = (int)(short)(v.y & 0xffff); w[3] = v.y >> 16;
    w[4] = (int)(short)(v.z & 0xffff); w[5] = v.z >> 16;
    w[6] = (int)(short)(v.w & 0xffff); w[7] = v.w >> 16;
}

__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, kWave));
    return v;
}

}  // namespace sk
