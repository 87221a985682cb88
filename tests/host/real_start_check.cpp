// The real-weight exact solver from given potentials: whatever the start
// (none, good, far off, of another instance), the permutation and its weight
// are those of the solve without one, on weights without ties and on weights
// full of them, and an instance without a matching stays without one.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "sk_hostsolve.h"

#define CHECK(c)                                                      \
    do {                                                              \
        if (!(c)) {                                                   \
            std::printf("failed line %d: %s (n %d)\n", __LINE__, #c, n); \
            std::exit(1);                                             \
        }                                                             \
    } while (0)

int main() {
    std::mt19937_64 rng(5);
    int solved = 0, infeasible = 0;
    for (int trial = 0; trial < 300; ++trial) {
        const int n = trial % 3 == 0 ? 1 + trial % 9 : 20 + (int)(rng() % 130);
        const bool ties = trial % 2;
        const double density = n < 10 ? 0.5 : 0.05 + 0.3 * (double)(trial % 5) / 4;
        std::uniform_real_distribution<double> U(0.0, 1.0);
        std::vector<int64_t> rp{0};
        std::vector<int32_t> col;
        std::vector<float> w;
        for (int i = 0; i < n; ++i) {
            for (int j = 0; j < n; ++j)
                if (U(rng) < density || j == (i + 3) % n) {
                    col.push_back(j);
                    w.push_back(ties ? (float)(int)(8 * U(rng)) - 4 : (float)(-10 * U(rng)));
                }
            rp.push_back((int64_t)col.size());
        }
        std::vector<int32_t> hint((size_t)n), p0((size_t)n, -1), p1((size_t)n, -1);
        for (int32_t &h : hint) h = (int32_t)(rng() % (uint64_t)n);
        double w0 = 0, w1 = 0;
        const sk_status st = sk::solve_real_impl(n, rp.data(), col.data(), w.data(), hint.data(), nullptr, p0.data(), &w0);
        sk::MatchStart kept;
        for (int start = 0; start < 5; ++start) {
            sk::MatchStart s;
            s.v.assign((size_t)n, 0.0);
            if (start == 1)
                for (double &v : s.v) v = 20 * U(rng) - 10;
            if (start == 2) s = kept;  // its own optimum
            if (start == 3) {          // its own potentials, another matching
                s = kept;
                for (int32_t &c : s.col) c = (int32_t)(rng() % (uint64_t)n);
            }
            if (start == 4)
                for (double &v : s.v) v = 1e6 * U(rng);
            if (s.v.empty()) s.v.assign((size_t)n, 0.0);
            CHECK(sk::solve_real_impl(n, rp.data(), col.data(), w.data(), hint.data(), &s, p1.data(), &w1) == st);
            if (st != SK_OK) continue;
            CHECK(p1 == p0 && w1 == w0);
            CHECK(s.v.size() == (size_t)n && s.col.size() == (size_t)n);
            if (start == 1) kept = s;
        }
        ++(st == SK_OK ? solved : infeasible);
        // the same pattern without the column that row n - 1 needs
        if (n > 1) {
            const int64_t last = rp[(size_t)n - 1];
            for (int64_t e = last; e < rp[(size_t)n]; ++e) col[(size_t)e] = col[0];
            for (int64_t e = 0; e < rp[1]; ++e) col[(size_t)e] = col[0];
            sk::MatchStart s;
            s.v.assign((size_t)n, 0.0);
            CHECK(sk::solve_real_impl(n, rp.data(), col.data(), w.data(), hint.data(), &s, p1.data(), &w1) ==
                  SK_EINFEASIBLE);
            ++infeasible;
        }
    }
    std::printf("ok solved=%d infeasible=%d\n", solved, infeasible);
    return 0;
}
