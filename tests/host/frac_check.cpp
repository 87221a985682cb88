// sk_frac.h on the host: -log S = k + f leaves a fraction that reading it back
// does not move, and is right to the rounding of float32; other splits of a
// logarithm are read as a fraction of at most 1/2. The two hardware functions stand as their C counterparts, the
// reciprocal also a unit in the last place off either way.
#include <cmath>
#include <cstdio>
#include <cstdlib>

static int g_ulps = 0;  // error of the reciprocal
static float shim_rcp(float x) {
    float r = 1.f / x;
    for (int k = 0; k < std::abs(g_ulps); ++k) r = std::nextafterf(r, g_ulps > 0 ? INFINITY : -INFINITY);
    return r;
}
static float shim_mant(float x) {
    int e;
    return std::frexp(x, &e);
}
static int shim_exp(float x) {
    int e;
    std::frexp(x, &e);
    return e;
}
#define __builtin_amdgcn_frexp_mantf shim_mant
#define __builtin_amdgcn_frexp_expf shim_exp
#define __builtin_amdgcn_rcpf shim_rcp
#include "sk_frac.h"

int main() {
    long checked = 0, near = 0;
    double worst = 0.0;
    auto one = [&](double S) {
        int k;
        const float f = sk::neg_log_split(S, k);
        int k2 = k;
        float f2 = f;
        sk::unit_frac(k2, f2);
        if (!(std::fabs(f) <= 0.5001f) || k2 != k || f2 != f) {
            std::printf("S = %.17g: k %d f %.9g\n", S, k, f);
            std::exit(1);
        }
        worst = std::fmax(worst, std::fabs((double)k + (double)f + std::log(S)));
        near += std::fabs(f) > 0.4999f;
        ++checked;
    };
    for (g_ulps = -1; g_ulps <= 1; ++g_ulps) {
        // logarithms around every half integer of the range, where k is chosen
        for (int h = -44; h < 44; ++h)
            for (int s = -400; s <= 400; ++s) one(std::exp(h + 0.5 + s * 2.5e-7));
        // and over all of it
        for (int s = 0; s < 200000; ++s) one(std::exp2(-64.0 + 128.0 * s / 200000.0));
    }
    for (int s = -4000; s <= 4000; ++s) {
        int k = 7;
        float f = 0.013f * (float)s;
        const double x = 7.0 + (double)f;
        const bool split = std::fabs(f) <= 0.5f;
        const float f0 = f;
        sk::unit_frac(k, f);
        if (!(std::fabs(f) <= 0.51f) || (double)k + (double)f != x || (split && (k != 7 || f != f0))) {
            std::printf("split %g: %d %.9g\n", x, k, f);
            return 1;
        }
    }
    std::printf("ok checked=%ld near=%ld worst=%.3g\n", checked, near, worst);
    // two float32 roundings below 1/2 and of the reciprocal's product
    return worst <= 4 * 0x1p-25 && near > 100000 ? 0 : 2;
}
