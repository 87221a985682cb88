// Sinkhorn iteration of instances with n <= kSmallN in one launch: one
// workgroup holds the whole instance and runs iteration after iteration, stage
// after stage, up to a budget of iterations.
//
// What bounds it. An iteration of such an instance is at most 2 * 65536
// multiply-adds, far below the launch chain of the sweeps (row sweep, column
// sweep, finalise, end of iteration: 18-20 us per iteration at n = 64 on an
// otherwise idle chip, all of it launch and memory latency). Here it is the
// latency of two barriers, two cross-lane reductions and the matrix pass:
// 1.3 us per iteration at n = 64, 2.1 at 100, 2.6 at 160, 5.0 at 256 (there the
// issue of some 700 instructions in each of 16 waves). Waves of 16 rows rather
// than 4 at n = 64: four times fewer waves issue the logarithm and exponential
// of a row step (1.7 us with 16 waves of 4 rows).
//
// Layout. Wave w owns rows R w .. R w + R - 1, lane l columns l + 64 c, so a
// thread holds R x C entries e = exp(p w_ij + F_i + G_j) of the exponent table
// in registers. With the integer parts unchanged, e is the same from one
// iteration to the next, so a sweep is one multiply-add per entry; only the
// entries of a row whose F_i moved, and of a column whose G_j moved, are read
// from the table again. The log-weights are packed in pairs, in registers up
// to n = 128 and in LDS above (128 KiB at n = 256), where 64 entries and 32
// pairs per thread would not fit the 128 registers of a 1024-thread workgroup.
#include "sk_frac.h"
#include "sk_rowsweep.h"
#include "sk_wave.h"

namespace sk {
namespace {

constexpr int kRows = 16;  // rows per wave

template <int C, class T>
struct SmallLds {
    static constexpr int kCols = kWave * C, kWaves = 4 * C, kStride = kCols + 4;

    float tab[kTabN];
    alignas(16) float wres[kWaves];  // residual maximum per wave
    T part[kWaves * kStride];        // column partials per wave
    int ca[kCols];                   // 4 G_j
    T cg[kCols];                     // exp(gam_j)
    // exact recompute of columns: the rows' new potentials, the flagged
    // columns and their new potentials
    int rF4[kCols];
    T rr[kCols];
    int list[kCols];
    int newG[kCols];
    float newg[kCols];
    unsigned flagged, err;
};

// C columns per lane and 4 C waves: n <= 64 C. WLDS: the packed weights in LDS
// (pairs of one thread a workgroup's threads apart). T: type of the terms and
// of a thread's part of a sum; sums across threads are float64 (a sum's
// roundings repeat from one iteration to the next, and a slowly converging
// instance adds them up).
template <int C, bool WLDS, class T>
__device__ __forceinline__ void small_run(const Inst &I, SmallLds<C, T> &L, unsigned *wlds, int budget) {
    constexpr int R = kRows, NW = 4 * C, NT = NW * kWave, PS = SmallLds<C, T>::kStride;
    constexpr int RL = kWave / R;  // lanes that carry one row's state
    constexpr int NP = C * R / 2;
    static_assert(C * R % 2 == 0, "pairs of entries");
    const int t = (int)threadIdx.x, lane0 = t % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    Ctl *ctl = I.ctl;
    const int n = I.n;
    const float tol = I.tol;
    int iter = __builtin_amdgcn_readfirstlane(ctl->iter);
    int stage = __builtin_amdgcn_readfirstlane(ctl->stage);
    int p = __builtin_amdgcn_readfirstlane(ctl->p);
    float last_res = ctl->last_res;
    int done = 0, stage_done = 0;  // iterations of this launch, of them in this stage

    // the row whose state this lane carries, and the column whose partial
    // sums this thread and its quad add
    const int row = wave * R + lane0 / RL;
    const bool row_on = row < n;
    const int colj = t >> 2;
    const bool col_on = colj < n;
    int F = 0, G = 0;
    float phi = 0.f, gam = 0.f;
    if (row_on) {
        F = I.F[iter & 1][row];
        phi = I.phi[iter & 1][row];
    }
    if (col_on) {
        G = I.G[colj];
        gam = I.gam[colj];
    }
    // a caller's starting potentials may split their logarithm in any way
    unit_frac(F, phi);
    unit_frac(G, gam);
    // entries outside the matrix are absent ones
    unsigned wp[WLDS ? 1 : NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        unsigned x = 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = (2 * q + h) / C, c = (2 * q + h) % C;
            const int r = wave * R + k, j = lane0 + kWave * c;
            int w = SK_SENTINEL;
            if (r < n && j < n) w = (int)I.W[(int64_t)r * I.pitch + j];
            x |= (unsigned)(w & 0xffff) << (16 * h);
        }
        if constexpr (WLDS) wlds[q * NT + t] = x;
        else wp[q] = x;
    }
    if (t == 0) {
        L.flagged = 0u;
        L.err = ctl->err;
    }
    if (t < kWave * C) {
        L.ca[t] = 0;
        L.cg[t] = 0;
    }
    fill_exp_table(L.tab);
    __syncthreads();
    auto publish = [&]() {
        if (col_on && (t & 3) == 0) {
            L.ca[colj] = 4 * G;
            exp_frac(gam, L.cg[colj]);
        }
    };
    publish();
    __syncthreads();

    int A[C];
    T g[C];
    T e[C * R];
    int p4 = 4 * p;
    auto term = [&](int k, int c, int B) {
        const int q = k * C + c;
        unsigned x;
        if constexpr (WLDS) x = wlds[(q >> 1) * NT + t];
        else x = wp[q >> 1];
        const int w = (q & 1) ? (int)x >> 16 : (int)(short)(x & 0xffff);
        const float v = tab_at(L.tab, tab_off(p4, w, A[c], B));
        return w == SK_SENTINEL ? 0.f : v;
    };
    auto load_cols = [&]() {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            A[c] = L.ca[lane0 + kWave * c];
            g[c] = L.cg[lane0 + kWave * c];
        }
    };
    // scheduling barriers keep the table reads of a few rows in flight at a
    // time (all of them at once take more registers than there are)
    auto all_terms = [&]() {
        const int B = 4 * (F - kTabLo);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int Bk = __builtin_amdgcn_readlane(B, k * RL);
#pragma unroll
            for (int c = 0; c < C; ++c) e[k * C + c] = term(k, c, Bk);
            if (C * (k + 1) % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        }
    };
    load_cols();
    all_terms();

    T rc;  // exp(phi_i) of the current iterate
    exp_frac(phi, rc);
    int state = ST_RUNNING, capped = 0;
    while (done < budget) {
        // opaque copies: what follows from the packed weights and from the
        // lane is formed where it is used, not kept across iterations
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        if constexpr (!WLDS) {
#pragma unroll
            for (int q = 0; q < NP; ++q) asm volatile("" : "+v"(wp[q]));
        }
        // ---- row step: S_i = sum_j e_ij exp(gam_j)
        double S = wave_sums16(
            [&](int k) {
                T s = e[k * C] * g[0];
#pragma unroll
                for (int c = 1; c < C; ++c) s = fma(e[k * C + c], g[c], s);
                return s;
            },
            lane);
        int M = 0;
        uint64_t bad = __ballot(row_on && !(S >= (double)kSafeLo && S <= (double)kSafeHi));
        while (bad != 0ull) {
            // exact max-shifted recompute (Section 4.1.2) of a row whose sum
            // left the safe range: M = max_j (p w_ij + F_i + G_j)
            const int k = (__ffsll((unsigned long long)bad) - 1) / RL;
            bad &= ~(((1ull << RL) - 1ull) << (k * RL));
            const int16_t *wr = I.W + (int64_t)(wave * R + k) * I.pitch;
            const int F4 = 4 * __builtin_amdgcn_readlane(F, k * RL);
            int m4 = INT_MIN;
            for (int j = lane; j < n; j += kWave)
                if (wr[j] != SK_SENTINEL) m4 = max(m4, __mul24(p4, (int)wr[j]) + L.ca[j] + F4);
            m4 = wave_max_i(m4);
            double s = 0;
            if (m4 == INT_MIN) {
                if (lane == 0) atomicOr(&L.err, (unsigned)ERR_EMPTY_ROW);
                s = 1;
            } else {
                const int B = F4 - (m4 & ~3) - 4 * kTabLo;  // m4 is a multiple of 4
                for (int j = lane; j < n; j += kWave)
                    if (wr[j] != SK_SENTINEL)
                        s = fma((double)tab_at(L.tab, tab_off(p4, (int)wr[j], L.ca[j], B)), (double)L.cg[j], s);
                s = wave_sum_d(s);
            }
            if (lane / RL == k) {
                S = s;
                M = m4 == INT_MIN ? 0 : m4 >> 2;
            }
        }
        // log u_i <- F_i - M - log S;  r_i = exp(phi_i + M) S
        int kr;
        float phin = neg_log_split(S, kr);
        const int Fn = row_on ? F - M + kr : F;
        phin = row_on ? phin : 0.f;
        float ri = (float)((double)rc * S - 1.0);
        if (M != 0) ri = ex2(fmaf((float)M, kLog2e, lg2((float)((double)rc * S)))) - 1.f;
        const float res = wave_max_v(row_on ? fabsf(ri) : 0.f);
        T rn;
        exp_frac(phin, rn);
        rn = row_on ? rn : (T)0;
        const uint64_t moved = __ballot(Fn != F);
        if (moved != 0ull) {
            const int B = 4 * (Fn - kTabLo);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if (!((moved >> (k * RL)) & 1ull)) continue;
                const int Bk = __builtin_amdgcn_readlane(B, k * RL);
#pragma unroll
                for (int c = 0; c < C; ++c) e[k * C + c] = term(k, c, Bk);
            }
        }
        // ---- column partials: sum over the wave's rows of e_ij exp(phi_i)
        T acc[C];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const T rk = readlane_v(rn, k * RL);
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = k == 0 ? e[c] * rk : fma(e[k * C + c], rk, acc[c]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) L.part[wave * PS + lane + kWave * c] = acc[c];
        if (lane == 0) L.wres[wave] = res;
        __syncthreads();
        float rmax = 0.f;
#pragma unroll
        for (int q = 0; q < NW; q += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(&L.wres[q]);
            rmax = fmaxf(rmax, fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)));
        }
        const bool conv = iter >= 1 && rmax < tol;
        if (!conv) {
            // ---- column step: log v_j <- G_j - log sum
            bool flag = false;
            if (col_on) {
                const T *q = &L.part[C * (t & 3) * PS + colj];
                double s = (double)q[0];
#pragma unroll
                for (int k = 1; k < C; ++k) s += (double)q[k * PS];
                s += dpp_mov<kDppXor1>(s);
                s += dpp_mov<kDppXor2>(s);
                flag = !(s >= (double)kSafeLo && s <= (double)kSafeHi);
                if (!flag) {
                    int k;
                    gam = neg_log_split(s, k);
                    G += k;
                    publish();
                } else if ((t & 3) == 0) {
                    L.list[atomicAdd(&L.flagged, 1u)] = colj;
                }
            }
            __syncthreads();
            const int nf = (int)L.flagged;
            if (nf > 0) {
                // exact max-shifted recompute of the flagged columns, one per
                // wave at a time: M = max_i (p w_ij + F_i + G_j), then
                // log v_j <- G_j - M - log sum_i exp(p w_ij + log u_i + G_j - M)
                if (row_on && lane % RL == 0) {
                    L.rF4[row] = 4 * Fn;
                    L.rr[row] = rn;
                }
                __syncthreads();
                for (int q = wave; q < nf; q += NW) {
                    const int j = L.list[q];
                    const int a = L.ca[j];
                    int m4 = INT_MIN;
                    for (int r = lane; r < n; r += kWave) {
                        const int w = (int)I.W[(int64_t)r * I.pitch + j];
                        if (w != SK_SENTINEL) m4 = max(m4, __mul24(p4, w) + a + L.rF4[r]);
                    }
                    m4 = wave_max_i(m4);
                    if (m4 == INT_MIN) {
                        if (lane == 0) {
                            atomicOr(&L.err, (unsigned)ERR_EMPTY_COL);
                            L.newG[j] = a >> 2;
                            L.newg[j] = 0.f;
                        }
                        continue;
                    }
                    double s = 0;
                    for (int r = lane; r < n; r += kWave) {
                        const int w = (int)I.W[(int64_t)r * I.pitch + j];
                        if (w == SK_SENTINEL) continue;
                        const int B = L.rF4[r] - (m4 & ~3) - 4 * kTabLo;
                        s = fma((double)tab_at(L.tab, tab_off(p4, w, a, B)), (double)L.rr[r], s);
                    }
                    s = wave_sum_d(s);
                    if (lane == 0) {
                        int k;
                        L.newg[j] = neg_log_split(s, k);
                        L.newG[j] = (a >> 2) - (m4 >> 2) + k;
                    }
                }
                __syncthreads();
                if (flag) {
                    G = L.newG[colj];
                    gam = L.newg[colj];
                    publish();
                }
                if (t == 0) L.flagged = 0u;
                __syncthreads();
            }
        }
        if ((L.err & (ERR_EMPTY_ROW | ERR_EMPTY_COL)) != 0u) {
            state = ST_ERROR;
            break;
        }
        bool stage_end = conv;
        if (conv) {
            last_res = rmax;
        } else {
            // commit of the iteration
            F = Fn;
            phi = phin;
            rc = rn;
            if (iter >= 1) last_res = rmax;
            ++iter;
            ++done;
            ++stage_done;
            stage_end = (int64_t)iter >= I.max_iters;
            if (stage_end) ++capped;
        }
        if (stage_end) {
            if (t == 0) ctl->stage_iters[stage] += stage_done;
            stage_done = 0;
            if (I.pause || stage + 1 >= I.n_p) {
                state = I.pause ? ST_STAGE_END : ST_DONE;
                break;
            }
            // the next p, with p^-1 log u and p^-1 log v held (FP64)
            const int p1 = I.ladder[stage + 1];
            const double ratio = (double)p1 / (double)I.ladder[stage];
            const double f = ((double)F + (double)phi) * ratio, kf = rint(f);
            F = (int)kf;
            phi = (float)(f - kf);
            exp_frac(phi, rc);
            const double gg = ((double)G + (double)gam) * ratio, kg = rint(gg);
            G = (int)kg;
            gam = (float)(gg - kg);
            ++stage;
            p = p1;
            iter = 0;
            __syncthreads();  // every wave is past its last read of the columns
            publish();
            __syncthreads();
            p4 = 4 * p;
            load_cols();
            all_terms();
            continue;
        }
        // ---- the columns as the next row step sees them
        unsigned ch = 0u;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int a = L.ca[lane + kWave * c];
            if (a != A[c]) ch |= 1u << c;
            A[c] = a;
            g[c] = L.cg[lane + kWave * c];
        }
        if (__ballot(ch != 0u) != 0ull) {
            const int B = 4 * (F - kTabLo);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (__ballot((ch >> c) & 1u) == 0ull) continue;
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    e[k * C + c] = term(k, c, __builtin_amdgcn_readlane(B, k * RL));
                    if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    // ---- back to the instance's buffers, as the sweeps leave them
    if (row_on && lane0 % RL == 0) {
        I.F[iter & 1][row] = F;
        I.phi[iter & 1][row] = phi;
    }
    if (col_on && (t & 3) == 0) {
        I.G[colj] = G;
        I.gam[colj] = gam;
    }
    if (t == 0) {
        if (stage_done > 0) ctl->stage_iters[stage] += stage_done;
        ctl->err = L.err;
        ctl->state = state;
        ctl->stage = stage;
        ctl->p = p;
        ctl->iter = iter;
        ctl->capped += capped;
        ctl->iters_total += done;
        ctl->last_res = last_res;
    }
}

// Workgroup b: the instance small_idx of insts[first + b].
template <int C, bool WLDS, class T>
__global__ __launch_bounds__(4 * C * kWave) void k_small(const Inst *__restrict__ insts, int first, int budget) {
    __shared__ SmallLds<C, T> L;
    extern __shared__ unsigned wlds[];
    const Inst &I = insts[insts[first + blockIdx.x].small_idx];
    if (__builtin_amdgcn_readfirstlane(I.ctl->state) != ST_RUNNING) return;
    small_run<C, WLDS, T>(I, L, wlds, budget);
}

constexpr int wlds_bytes(int C) { return 4 * C * kWave * (C * kRows / 2) * (int)sizeof(unsigned); }

template <int C, bool WLDS, class T>
void launch_class(const Inst *d_insts, int first, int count, int budget, hipStream_t st) {
    if (count > 0)
        hipLaunchKernelGGL((k_small<C, WLDS, T>), dim3(count), dim3(4 * C * kWave), WLDS ? wlds_bytes(C) : 0, st,
                           d_insts, first, budget);
}

}  // namespace

hipError_t launch_small(const Inst *d_insts, const int *counts, int budget, hipStream_t st) {
    int first = 0;
    launch_class<4, true, float>(d_insts, first, counts[3], budget, st);
    first += counts[3];
    launch_class<3, true, float>(d_insts, first, counts[2], budget, st);
    first += counts[2];
    launch_class<2, false, double>(d_insts, first, counts[1], budget, st);
    first += counts[1];
    launch_class<1, false, double>(d_insts, first, counts[0], budget, st);
    return hipGetLastError();
}

hipError_t set_small_attributes() {
    const hipError_t e = hipFuncSetAttribute((const void *)k_small<4, true, float>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, wlds_bytes(4));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_small<3, true, float>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, wlds_bytes(3));
}

}  // namespace sk
