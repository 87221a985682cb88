// Host exact solvers of the reduced instance (no device code), shared by the
// scaling paths and the C entry points.
#pragma once
#include <cstdint>
#include <vector>

#include "../../include/sk.h"

namespace sk {

// sk_solve_reduced with a column per row to try first in the greedy start
// of the matching (nullptr: none).
sk_status solve_reduced_seeded(const sk_csr *csr, const int32_t *hint, int32_t *perm,
                               int64_t *weight);

// Where solve_real_impl starts, and afterwards where it ended: the column
// potentials in units of w (n finite values), and per row the column of an
// optimal matching that goes with them (empty: none).
struct MatchStart {
    std::vector<double> v;
    std::vector<int32_t> col;
};

// Maximum-weight perfect matching of the CSR (rp, col, w) with float weights
// by shortest augmenting paths; hint as above, start optional. SK_EINVAL for
// a malformed CSR or a non-finite weight, SK_EINFEASIBLE when no perfect
// matching exists (start then keeps what it was).
sk_status solve_real_impl(int n, const int64_t *rp, const int32_t *col, const float *w,
                          const int32_t *hint, MatchStart *start, int32_t *perm, double *weight);

}  // namespace sk
