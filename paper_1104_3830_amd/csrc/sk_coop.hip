// The resident iteration of sk_coop.h over int16 log-weights.
#include <cstddef>

#include "sk_coop.h"

namespace sk {
namespace {

// Terms from the exponent table, formed anew in every iteration (see
// sk_coop.h). SENT: W holds absent entries.
template <int CH, bool SENT>
struct CoopInt {
    static constexpr bool kKeep = false;
    struct Lds {
        // the rows of W, a thread's 8 columns of a row per entry: in registers
        // they would not fit beside the terms
        int4 w[kCoopR * CH][kCoopThreads];
        float tab[kTabN];
    };
    int p4;

    static __device__ __forceinline__ int col_code(int G, bool on) { return on ? 4 * G : kPadExp4; }

    __device__ __forceinline__ void load(const Inst &I, Lds &L, int rw, int t) {
        const int n = I.n, lane = t % kWave;
#pragma unroll
        for (int k = 0; k < kCoopR; ++k) {
            const int16_t *wr = I.W + (int64_t)min(rw + k, n - 1) * I.pitch;
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                const int j0 = 512 * q + 8 * lane;
                int4 v = make_int4(0, 0, 0, 0);
                if (I.vec8) {
                    if (j0 < n) v = gload<false>(reinterpret_cast<const int4 *>(wr + j0));
                } else if (j0 < n) {
                    // n % 8 == 0 here: the chunk is inside the row
                    unsigned h[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) h[c] = (unsigned)(uint16_t)wr[j0 + c];
                    v = make_int4((int)(h[0] | h[1] << 16), (int)(h[2] | h[3] << 16), (int)(h[4] | h[5] << 16),
                                  (int)(h[6] | h[7] << 16));
                }
                L.w[k * CH + q][t] = v;
            }
        }
        fill_exp_table(L.tab);
    }
    __device__ __forceinline__ void begin(const Inst &, int p) { p4 = 4 * p; }

    // rows past the matrix: every exponent 4 (p w + G_j) + kPadExp4 clamps to
    // the table's zero entry (in padding columns the sum may wrap, and what
    // these add to each other is not used)
    __device__ __forceinline__ void row_terms(const Lds &L, int k, int t, bool on, int F, const int (&A)[8 * CH],
                                              float *e) {
        const int B = on ? 4 * (F - kTabLo) : kPadExp4;
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            int w[8];
            unpack8i(L.w[k * CH + q][t], w);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float x = tab_at(L.tab, tab_off(p4, w[c], A[8 * q + c], B));
                if (SENT) x = w[c] == SK_SENTINEL ? 0.f : x;
                e[8 * q + c] = x;
            }
        }
    }

    // The sum of a row that left the safe range relative to
    // M = max_j (p w_ij + F_i + G_j); false for an empty row.
    __device__ __forceinline__ bool rescue_row(const Inst &I, const CoopLds<CH> &L, const Lds &LP, int row, int F,
                                               int lane, int n8, double &S, int &M) {
        const int n = I.n, F4 = 4 * F;
        const int16_t *wr = I.W + (int64_t)row * I.pitch;
        int m4 = INT_MIN;
        for (int j = lane; j < n; j += kWave) {
            const int w = (int)wr[j];
            if (w != SK_SENTINEL) m4 = max(m4, __mul24(p4, w) + L.cp[swz8(j, n8)].a + F4);
        }
        m4 = wave_max_i(m4);
        if (m4 == INT_MIN) return false;
        const int B = F4 - (m4 & ~3) - 4 * kTabLo;  // m4 is a multiple of 4
        double s = 0.0;
        for (int j = lane; j < n; j += kWave) {
            const int w = (int)wr[j];
            if (w == SK_SENTINEL) continue;
            const ColPot c = L.cp[swz8(j, n8)];
            s = fma((double)tab_at(LP.tab, tab_off(p4, w, c.a, B)), (double)c.g, s);
        }
        S = wave_sum_d(s);
        M = m4 >> 2;
        return true;
    }
};

template <int CH, bool SENT>
__device__ __forceinline__ void coop_int(const Inst &I, int budget, CoopGiveUp give_up, CoopLds<CH> &L,
                                         typename CoopInt<CH, SENT>::Lds &LP) {
    coop_run<CoopInt<CH, SENT>, CH>(I, L, LP, budget, give_up);
}

template <int CH>
__global__ __launch_bounds__(kCoopThreads, 1) void k_coop(const Inst *__restrict__ insts, int budget,
                                                          CoopGiveUp give_up) {
    __shared__ CoopLds<CH> L;
    // (one layout whether W holds absent entries or not)
    __shared__ typename CoopInt<CH, false>::Lds LP;
    const Inst &I = insts[0];
    if (__builtin_amdgcn_readfirstlane(I.ctl->state) != ST_RUNNING) return;
    if (__builtin_amdgcn_readfirstlane(I.ctl->sent) != 0u)
        coop_int<CH, true>(I, budget, give_up, L, reinterpret_cast<typename CoopInt<CH, true>::Lds &>(LP));
    else
        coop_int<CH, false>(I, budget, give_up, L, LP);
}

// Takes the launch's result over if every workgroup left its share; otherwise
// the second copy of the row potentials gets the start's state back.
__global__ __launch_bounds__(256) void k_coop_commit(const Inst *__restrict__ insts, int nblk) {
    const Inst &I = insts[0];
    const int n = I.n, i = blockIdx.x * blockDim.x + threadIdx.x;
    CoopHdr *hdr = reinterpret_cast<CoopHdr *>(I.coop);
    const bool ok = hdr->done == (uint32_t)nblk;
    if (ok && i < n) {
        I.F[0][i] = I.F[1][i];
        I.phi[0][i] = I.phi[1][i];
        I.G[i] = I.G2[i];
        I.gam[i] = I.gam2[i];
    } else if (i < n && I.ctl->state == ST_RUNNING) {
        I.F[1][i] = I.F[0][i];
        I.phi[1][i] = I.phi[0][i];
    }
    if (blockIdx.x > 0 || threadIdx.x >= kWave) return;
    Ctl *c = I.ctl;
    const Ctl *d = I.ctl2;
    const int stage0 = c->stage, state0 = c->state;
    if (state0 != ST_RUNNING) return;
    if (ok) {
        const int s = stage0 + (int)threadIdx.x;
        if (s <= d->stage && s < SK_MAX_LADDER) c->stage_iters[s] += d->stage_iters[s];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (ok) {
            c->err |= d->err;
            c->state = d->state;
            c->stage = d->stage;
            c->p = d->p;
            c->iter = d->iter;
            c->capped += d->capped;
            c->iters_total += d->iters_total;
            c->last_res = d->last_res;
        }
        c->coop = ok ? d->coop : kCoopFailed;
    }
}

// A cleared exchange area (sequence numbers start at 1), and the count of
// workgroups of a launch.
__global__ __launch_bounds__(256) void k_coop_clear(const Inst *__restrict__ insts, size_t words) {
    CoopWord *p = reinterpret_cast<CoopWord *>(insts[0].coop);
    for (size_t i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}
__global__ void k_coop_begin(const Inst *__restrict__ insts) {
    reinterpret_cast<CoopHdr *>(insts[0].coop)->done = 0u;
}

}  // namespace

size_t coop_bytes(int n) { return 8 * coop_words(n); }

hipError_t launch_coop_clear(const Inst *d_insts, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_coop_clear, dim3(256), dim3(256), 0, st, d_insts, coop_words(n));
    return hipGetLastError();
}

hipError_t launch_coop(const Inst *d_insts, int n, int real, int budget, CoopGiveUp give_up, hipStream_t st) {
    const int nblk = (n + kMidRows - 1) / kMidRows;
    hipLaunchKernelGGL(k_coop_begin, dim3(1), dim3(1), 0, st, d_insts);
    if (real)
        launch_coop_real(d_insts, n, nblk, budget, give_up, st);
    else if (n <= 512)
        hipLaunchKernelGGL(k_coop<1>, dim3(nblk), dim3(kCoopThreads), 0, st, d_insts, budget, give_up);
    else
        hipLaunchKernelGGL(k_coop<2>, dim3(nblk), dim3(kCoopThreads), 0, st, d_insts, budget, give_up);
    hipLaunchKernelGGL(k_coop_commit, dim3((n + 255) / 256), dim3(256), 0, st, d_insts, nblk);
    return hipGetLastError();
}

}  // namespace sk
