// The real-weight exact solver from potentials of another size than the
// weights (small weights kept of a matrix with large ones, or all equal): the
// permutation and its weight are those of the solve without a start, and a
// start that was replaced serves the next solve.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "sk_hostsolve.h"

#define CHECK(c)                                                                            \
    do {                                                                                    \
        if (!(c)) {                                                                         \
            std::printf("failed line %d: %s (n %d weights %g start %g)\n", __LINE__, #c, n, ws, vs); \
            std::exit(1);                                                                   \
        }                                                                                   \
    } while (0)

int main() {
    std::mt19937_64 rng(11);
    int solved = 0;
    for (int trial = 0; trial < 40; ++trial)
        for (const double ws : {1.0, 1e-4, 1e-8, 1e-12, 1e-30, 0.0})
            for (const double vs : {0.0, 1.0, 1e3, 1e6}) {
                const int n = trial % 4 == 0 ? 1 + trial % 7 : 20 + (int)(rng() % 80);
                std::uniform_real_distribution<double> U(0.0, 1.0);
                std::vector<int64_t> rp{0};
                std::vector<int32_t> col;
                std::vector<float> w;
                for (int i = 0; i < n; ++i) {
                    for (int j = 0; j < n; ++j)
                        if (U(rng) < 0.15 || j == (i + 3) % n) {
                            col.push_back(j);
                            w.push_back((float)(-ws * U(rng)));
                        }
                    rp.push_back((int64_t)col.size());
                }
                std::vector<int32_t> hint((size_t)n), p0((size_t)n), p1((size_t)n);
                for (int32_t &h : hint) h = (int32_t)(rng() % (uint64_t)n);
                double w0 = 0, w1 = 0;
                CHECK(sk::solve_real_impl(n, rp.data(), col.data(), w.data(), hint.data(), nullptr, p0.data(), &w0) == SK_OK);
                sk::MatchStart s;
                s.v.resize((size_t)n);
                for (double &v : s.v) v = vs * (2 * U(rng) - 1);
                for (int again = 0; again < 2; ++again) {
                    CHECK(sk::solve_real_impl(n, rp.data(), col.data(), w.data(), hint.data(), &s, p1.data(), &w1) == SK_OK);
                    CHECK(p1 == p0 && w1 == w0);
                }
                ++solved;
            }
    std::printf("ok solved=%d\n", solved);
    return 0;
}
