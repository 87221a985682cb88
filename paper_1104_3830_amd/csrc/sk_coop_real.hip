// The resident iteration of sk_coop.h over real-valued log-weights
// (sk_real.h).
//
// A term exp(p (w_ij - wref) + F_i + G_j) has its exponent in FP64, some
// twenty instructions where an int16 one has four and a table read, so the
// terms stay in registers and only those of moved rows and columns are formed
// again. Only one instance at a time takes this path, so its sums have no
// other kernel to agree with. At n = 1000 (Euclidean weights, 632 iterations)
// an iteration takes 8.4 us, of which the two exchanges are 3.6, where the
// sweeps' four launches took 30 (row sweep 14.4, column sweep 7.1, finalise
// 4.6, end of iteration 3.7).
#include "sk_coop.h"
#include "sk_real.h"

namespace sk {
namespace {

// 2^e2 in float32: the fraction's exponential to half an ulp, since a kept
// term enters every iteration with the same error.
__device__ __forceinline__ float pow2_frac(double e2) {
    const double m = rint(e2);
    const float x = (float)((e2 - m) * kLn2D);
    return ldexpf(exp_frac(x), sat_i32(m));
}

template <int CH>
struct CoopReal {
    static constexpr bool kKeep = true;
    struct Lds {
        // the rows of W, 4 of a thread's columns of a row per entry; -inf
        // outside the matrix
        float4 w[kCoopR * CH * 2][kCoopThreads];
    };
    double p2, wref;

    static __device__ __forceinline__ int col_code(int G, bool) { return G; }

    __device__ __forceinline__ void load(const Inst &I, Lds &L, int rw, int t) {
        const int n = I.n, lane = t % kWave;
#pragma unroll
        for (int k = 0; k < kCoopR; ++k) {
            const float *wr = I.Wr + (int64_t)min(rw + k, n - 1) * I.pitch;
#pragma unroll
            for (int h = 0; h < 2 * CH; ++h) {
                const int j0 = 512 * (h / 2) + 8 * lane + 4 * (h % 2);
                float x[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) x[c] = rw + k < n && j0 + c < n ? wr[j0 + c] : -INFINITY;
                L.w[k * CH * 2 + h][t] = make_float4(x[0], x[1], x[2], x[3]);
            }
        }
        wref = (double)I.wref;
    }
    __device__ __forceinline__ void begin(const Inst &I, int p) { p2 = (double)p * I.pscale * kLog2eD; }

    __device__ __forceinline__ float term(float w, int FG) const {
        const float x = pow2_frac(fma(p2, (double)w - wref, (double)FG * kLog2eD));
        return w == -INFINITY ? 0.f : x;
    }
    __device__ __forceinline__ void row_terms(const Lds &L, int k, int t, bool, int F, const int (&A)[8 * CH],
                                              float *e) {
#pragma unroll
        for (int h = 0; h < 2 * CH; ++h) {
            const float4 v = L.w[k * CH * 2 + h][t];
            e[4 * h] = term(v.x, F + A[4 * h]);
            e[4 * h + 1] = term(v.y, F + A[4 * h + 1]);
            e[4 * h + 2] = term(v.z, F + A[4 * h + 2]);
            e[4 * h + 3] = term(v.w, F + A[4 * h + 3]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // column c of the lane over the wave's rows
    template <int R, int C, int RL>
    __device__ __forceinline__ void col_terms(const Lds &L, int c, int t, int, int F, int a, float (&e)[R * C]) {
        float w[R];
#pragma unroll
        for (int k = 0; k < R; ++k) w[k] = reinterpret_cast<const float *>(&L.w[k * CH * 2 + c / 4][t])[c % 4];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            e[k * C + c] = term(w[k], __builtin_amdgcn_readlane(F, k * RL) + a);
            if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }

    // The sum of a row that left the safe range relative to
    // M = rint(max_j (p w'_ij + F_i + G_j)); false for an empty row.
    __device__ __forceinline__ bool rescue_row(const Inst &I, const CoopLds<CH> &L, const Lds &, int row, int F, int lane,
                                               int n8, double &S, int &M) {
        const int n = I.n;
        const float *wr = I.Wr + (int64_t)row * I.pitch;
        double m2 = -INFINITY;
        for (int j = lane; j < n; j += kWave)
            if (wr[j] != -INFINITY)
                m2 = fmax(m2, fma(p2, (double)wr[j] - wref, (double)(F + L.cp[swz8(j, n8)].a) * kLog2eD));
        m2 = wave_max_d(m2);
        if (m2 == -INFINITY) return false;
        M = (int)rint(m2 * kLn2D);
        double s = 0.0;
        for (int j = lane; j < n; j += kWave) {
            const ColPot c = L.cp[swz8(j, n8)];
            s = fma((double)term(wr[j], F - M + c.a), (double)c.g, s);
        }
        S = wave_sum_d(s);
        return true;
    }
};

template <int CH>
__global__ __launch_bounds__(kCoopThreads, 1) void k_coop_real(const Inst *__restrict__ insts, int budget,
                                                               CoopGiveUp give_up) {
    __shared__ CoopLds<CH> L;
    __shared__ typename CoopReal<CH>::Lds LP;
    const Inst &I = insts[0];
    if (__builtin_amdgcn_readfirstlane(I.ctl->state) != ST_RUNNING) return;
    coop_run<CoopReal<CH>, CH>(I, L, LP, budget, give_up);
}

}  // namespace

void launch_coop_real(const Inst *d_insts, int n, int nblk, int budget, CoopGiveUp give_up, hipStream_t st) {
    if (n <= 512)
        hipLaunchKernelGGL(k_coop_real<1>, dim3(nblk), dim3(kCoopThreads), 0, st, d_insts, budget, give_up);
    else
        hipLaunchKernelGGL(k_coop_real<2>, dim3(nblk), dim3(kCoopThreads), 0, st, d_insts, budget, give_up);
}

}  // namespace sk
