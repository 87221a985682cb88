// Exact maximum-weight perfect matching of a reduced instance with real
// (float) weights, the exact step of Section 4.2 for real-valued log-weights.
// Host code only, no device calls.
//
// What bounds it: the searches, one per row that the start leaves free. From
// column potentials 0 that is some 40 % of the rows, and a late search settles
// most of the instance; the scaling's log v / p are within its residual of
// optimal ones, and the optimum of the evaluation before is within a pivot or
// two. The eleven evaluations of a Euclidean instance (n = 1000, p = 100, 150,
// .. 600, 20800 entries falling to 3950) take 4.2 ms, the first 2.6 of them,
// where starts from 0 took 146 ms, the first 32; the 32 of a random one (log
// uniform weights, 258000 entries falling to 41000) 75 where they took 1840.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <functional>
#include <utility>
#include <vector>

#include "sk_hostsolve.h"

namespace sk {
namespace {

struct Matching {
    std::vector<double> u, v;
    std::vector<int32_t> row_of, col_of;
    std::vector<int64_t> edge_of;  // CSR position of a row's matched entry
};

// Row reduction: a free row takes the column of its least reduced cost, whose
// potential falls until the row's next best is as good, and the row that held
// it looks for another. Most of what a good start leaves free is settled here,
// a row at a time instead of a search; the budget bounds what equal or nearly
// equal entries can cost, and the searches do the rest.
void reduce_rows(int n, const int64_t *rp, const int32_t *col, const float *w, Matching &M) {
    const double INF = INFINITY;
    int64_t budget = 4 * (int64_t)n;
    for (int f = 0; f < n; ++f) {
        for (int i = f; i >= 0 && M.col_of[i] < 0 && budget > 0; --budget) {
            double m1 = INF, m2 = INF;
            int64_t e1 = rp[i];
            for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
                const double r = -(double)w[e] - M.v[col[e]];
                if (r < m1) {
                    m2 = m1;
                    m1 = r;
                    e1 = e;
                } else if (r < m2) {
                    m2 = r;
                }
            }
            const int j = col[e1], k = M.row_of[j];
            // the only entry, or no better than the next where another row holds it
            if (m2 == INF || (k >= 0 && !(m1 < m2))) break;
            M.v[j] -= m2 - m1;
            M.u[i] = m2;
            M.row_of[j] = i;
            M.col_of[i] = j;
            M.edge_of[i] = e1;
            if (k >= 0) M.col_of[k] = -1;
            i = k;
        }
    }
    // a free row's potential is its least reduced cost
    for (int i = 0; i < n; ++i) {
        if (M.col_of[i] >= 0) continue;
        double m = INF;
        for (int64_t e = rp[i]; e < rp[i + 1]; ++e) m = std::min(m, -(double)w[e] - M.v[col[e]]);
        M.u[i] = m;
    }
}

// Sparse shortest augmenting paths (Dijkstra with row and column potentials)
// minimising sum c with c = -w, i.e. maximising sum w, from the column
// potentials M.v. Invariant: reduced costs c_ij - u_i - v_j >= 0 on every
// entry and = 0 on matched ones. After a search from free row i0 that reaches
// a free column at distance d*, the potentials of the nodes it finalised move
// by (their distance - d*), which keeps the invariant and makes the
// augmenting path tight.
sk_status augment_all(int n, const int64_t *rp, const int32_t *col, const float *w, const int32_t *hint,
                      const MatchStart *start, double slack, Matching &M) {
    const double INF = INFINITY;
    std::vector<double> &u = M.u, &v = M.v;
    std::vector<int32_t> &row_of = M.row_of, &col_of = M.col_of;
    std::vector<int64_t> &edge_of = M.edge_of;
    u.assign((size_t)n, 0.0);
    row_of.assign((size_t)n, -1);
    col_of.assign((size_t)n, -1);
    edge_of.assign((size_t)n, -1);
    for (int i = 0; i < n; ++i) {
        double m = INF;
        for (int64_t e = rp[i]; e < rp[i + 1]; ++e) m = std::min(m, -(double)w[e] - v[col[e]]);
        u[i] = m;
    }
    auto match = [&](int i, int64_t e) {
        col_of[i] = col[e];
        row_of[col[e]] = i;
        edge_of[i] = e;
    };
    // the matching that the potentials come with, where it is still optimal
    if (start && !start->col.empty())
        for (int i = 0; i < n; ++i)
            for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
                if (col[e] != start->col[i]) continue;
                const double c = -(double)w[e] - v[col[e]];
                if (c <= u[i] + slack && row_of[col[e]] < 0) {
                    u[i] = c;
                    match(i, e);
                }
                break;
            }
    // greedy start on tight entries, the hinted column first
    for (int i = 0; i < n; ++i) {
        if (col_of[i] >= 0) continue;
        int64_t pick = -1;
        for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
            if (-(double)w[e] - v[col[e]] != u[i] || row_of[col[e]] >= 0) continue;
            if (pick < 0 || (hint && col[e] == hint[i])) pick = e;
        }
        if (pick >= 0) match(i, pick);
    }
    if (start) reduce_rows(n, rp, col, w, M);
    std::vector<double> dist((size_t)n, INF);
    std::vector<int32_t> pred((size_t)n, -1);
    std::vector<int64_t> pred_edge((size_t)n, -1);
    std::vector<char> done((size_t)n, 0);
    using Item = std::pair<double, int32_t>;
    std::vector<Item> heap;  // a min-heap in (distance, column)
    std::vector<int32_t> touched, finalized;
    for (int i0 = 0; i0 < n; ++i0) {
        if (col_of[i0] >= 0) continue;
        double bound = INF;  // least distance of a free column so far
        auto relax = [&](int i, double di) {
            for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
                const int j = col[e];
                const double r = std::max(0.0, -(double)w[e] - u[i] - v[j]);
                const double nd = di + r;
                // a column farther than the bound is never taken off the heap
                if (nd > bound || done[j] || !(nd < dist[j])) continue;
                if (dist[j] == INF) touched.push_back(j);
                dist[j] = nd;
                pred[j] = i;
                pred_edge[j] = e;
                if (row_of[j] < 0) bound = nd;
                heap.push_back({nd, j});
                std::push_heap(heap.begin(), heap.end(), std::greater<Item>());
            }
        };
        relax(i0, 0.0);
        int sink = -1;
        double dsink = 0.0;
        while (!heap.empty()) {
            const Item it = heap.front();
            std::pop_heap(heap.begin(), heap.end(), std::greater<Item>());
            heap.pop_back();
            const int j = it.second;
            if (done[j] || it.first > dist[j]) continue;
            done[j] = 1;
            finalized.push_back(j);
            if (row_of[j] < 0) {
                sink = j;
                dsink = it.first;
                break;
            }
            relax(row_of[j], it.first);
        }
        if (sink < 0) return SK_EINFEASIBLE;
        for (int j : finalized) {
            if (j == sink) continue;
            const double delta = dist[j] - dsink;  // <= 0
            v[j] += delta;
            u[row_of[j]] -= delta;
        }
        u[i0] += dsink;
        // augment along the search tree
        for (int j = sink;;) {
            const int i = pred[j];
            const int jn = col_of[i];
            col_of[i] = j;
            row_of[j] = i;
            edge_of[i] = pred_edge[j];
            if (i == i0) break;
            j = jn;
        }
        for (int j : touched) dist[j] = INF;
        for (int j : finalized) done[j] = 0;
        touched.clear();
        finalized.clear();
        heap.clear();
    }
    return SK_OK;
}

// Whether the potentials prove M the optimum and no other perfect matching
// within tol of it. exact: whether they are precise enough to, that is whether
// what their rounding leaves open stays below tol / 2: over the rows (a
// matching has one entry in each), the most by which a reduced cost of the row
// can be below 0 and its matched one's off 0, with the rounding of their two
// subtractions. It grows with the potentials and not with the weights. Another
// matching would need a cycle of rows, each with an entry of reduced cost
// <= tol in the next one's column. Rows that none is left to point at are
// taken away until all are gone or a cycle stays.
bool unique_within(int n, const int64_t *rp, const int32_t *col, const float *w, const Matching &M, double tol,
                   bool &exact) {
    constexpr double kUlp = 0x1p-52;
    std::vector<int32_t> into((size_t)n, 0), queue;
    double slack = 0.0;
    for (int i = 0; i < n; ++i) {
        double below = 0.0;
        for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
            const double c = -(double)w[e] - M.u[i], r = c - M.v[col[e]];
            const double err = kUlp * (std::fabs(c) + std::fabs(r));
            below = std::max(below, err - r);
            if (e == M.edge_of[i]) slack += std::fabs(r) + err;
            if (r <= tol && M.row_of[col[e]] != i) ++into[M.row_of[col[e]]];
        }
        slack += below;
    }
    exact = slack <= 0.5 * tol;
    if (!exact) return false;
    queue.reserve((size_t)n);
    for (int i = 0; i < n; ++i)
        if (into[i] == 0) queue.push_back(i);
    for (size_t h = 0; h < queue.size(); ++h) {
        const int i = queue[h];
        for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
            const int k = M.row_of[col[e]];
            if (k != i && -(double)w[e] - M.u[i] - M.v[col[e]] <= tol && --into[k] == 0) queue.push_back(k);
        }
    }
    return queue.size() == (size_t)n;
}

}  // namespace

// Any start gives an optimal matching, and one that is unique is the same from
// all. Where others come within kTieTol (of the largest |w|: below a float32
// step of the larger weights) the choice would hang on the start, so the
// search is done again from potentials 0, which decides there. So it is where
// the potentials are so large beside the weights that their rounding takes
// more than half of that (small weights kept of a matrix whose others are
// not, a far start): then they neither prove the matching nor its uniqueness.
sk_status solve_real_impl(int n, const int64_t *rp, const int32_t *col, const float *w, const int32_t *hint,
                          MatchStart *start, int32_t *perm, double *weight) {
    constexpr double kTieTol = 1e-9, kSlack = 1e-13;
    if (n <= 0) return SK_EINVAL;
    double wmax = 0.0;
    for (int i = 0; i < n; ++i) {
        if (rp[i + 1] < rp[i]) return SK_EINVAL;
        if (rp[i + 1] == rp[i]) return SK_EINFEASIBLE;
        for (int64_t e = rp[i]; e < rp[i + 1]; ++e) {
            if (col[e] < 0 || col[e] >= n || !(w[e] > -INFINITY && w[e] < INFINITY)) return SK_EINVAL;
            wmax = std::max(wmax, std::fabs((double)w[e]));
        }
    }
    Matching M;
    bool solved = false, exact = true;
    if (start) {
        M.v = start->v;
        const sk_status st = augment_all(n, rp, col, w, hint, start, kSlack * wmax, M);
        if (st != SK_OK) return st;
        solved = unique_within(n, rp, col, w, M, kTieTol * wmax, exact);
        start->v = M.v;
        start->col = M.col_of;
    }
    if (!solved) {
        M.v.assign((size_t)n, 0.0);
        const sk_status st = augment_all(n, rp, col, w, hint, nullptr, 0.0, M);
        if (st != SK_OK) return st;
        if (!exact) {  // the next start is this one's optimum
            start->v = M.v;
            start->col = M.col_of;
        }
    }
    double total = 0.0;
    for (int i = 0; i < n; ++i) {
        perm[i] = M.col_of[i];
        total += (double)w[M.edge_of[i]];
    }
    *weight = total;
    return SK_OK;
}

}  // namespace sk

extern "C" sk_status sk_solve_reduced_real(const sk_csr_real *csr, int32_t *perm, double *weight) {
    if (!csr || !perm || !weight || !csr->row_ptr || csr->n < 1) return SK_EINVAL;
    if (csr->row_ptr[0] != 0 || csr->row_ptr[csr->n] != csr->nnz) return SK_EINVAL;
    if (csr->nnz > 0 && (!csr->col || !csr->w)) return SK_EINVAL;
    return sk::solve_real_impl(csr->n, csr->row_ptr, csr->col, csr->w, nullptr, nullptr, perm, weight);
}
