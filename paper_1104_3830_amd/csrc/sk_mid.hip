// Sinkhorn iteration of instances with kSmallN < n <= kMidN in one launch per
// iteration: batches, and one instance alone where the resident iteration of
// sk_coop.h (7.5 us at n = 1003) gave up.
//
// What bounds it. Such a matrix (2 MB at n = 1024) sits in the L2 caches and
// takes about a microsecond to sweep, but an iteration of the sweeps is four
// dependent launches (35 us at n = 1003: column sweep 18.9, row sweep 7.9,
// finalise 4.7, end of iteration 4.0). Here a workgroup takes blocks of 32
// rows, which it loads once for both steps, and what needs the whole matrix
// happens at the start of the next launch, in every workgroup alike: the
// residual maximum and the controller's decision, the column sums over the
// blocks' partials and the column step. An iteration is one launch, 12.0 us
// at n = 1003 (latency: four waves on each of 32 compute units).
//
// A batch has too many blocks for each to read all partials (n / 32 of n
// floats, twice the block's own 64 n bytes of W at n = 1024): above
// kMidFoldUnits blocks k_mid_columns takes the column step once per instance,
// and a workgroup sweeps a run of blocks, the next one's rows in flight. The
// 102 + 102 instances of n in 257..1024 of a 512-instance batch: 39 + 15 us
// and 8 us for the column step, where the sweeps took 108 + 15 us (with the
// rest of the batch). The arithmetic and its order are the same either way.
//
// Four waves of 8 rows: the row step's reduction, logarithm and exponentials
// are issued once per wave whatever its rows, some 200 instructions beside 6.5
// per 64 entries; with 16 waves of 2 rows the wide instances took 58 us.
//
// Two copies of everything that crosses a launch (column partials, residuals,
// controller, potentials), used in turn: a launch reads copy `in` and writes
// the other. Launches come in pairs, so the host always finds copy 0 current.
#include <climits>
#include <cstddef>

#include "sk_frac.h"
#include "sk_rowsweep.h"
#include "sk_wave.h"

namespace sk {
namespace {

constexpr int kMidWaves = 4, kMidThreads = kMidWaves * kWave;
constexpr int kR = kMidRows / kMidWaves;  // rows per wave
constexpr int kRL = kWave / kR;           // lanes that carry one row's state
constexpr int kCT = 4;                    // consecutive columns per thread in the column step
static_assert(kR == 8 && kCT * kMidThreads >= kMidN, "wave_sums8, every column has a thread");

// FOLD launches have one block of rows per workgroup.
template <int CH, bool FOLD>
struct MidLds {
    static constexpr int kCols = 512 * CH;
    float tab[kTabN];
    ColPot cp[kCols];              // swizzled (swz8)
    alignas(16) float part[FOLD ? 1 : 2][kMidWaves][kCols];  // column partials per wave
    float wres[FOLD ? 1 : 2][kMidWaves];
    unsigned err;
};
struct MidColLds {
    float tab[kTabN];
    int list[kMidN];  // columns outside the safe range
    int newG[kMidN];  // their exact recompute
    float newg[kMidN];
    unsigned flagged, newerr;
};

// What a launch finds of the iteration before it, the same in every
// workgroup: whether one is pending, its residual and whether it converged.
struct MidState {
    bool pending, conv;
    int stage, iter, p;
    float rm;
};
__device__ __forceinline__ MidState mid_state(const Inst &I, const Ctl *ci, float r) {
    MidState s;
    s.pending = __builtin_amdgcn_readfirstlane(ci->pending) != 0u;
    s.stage = __builtin_amdgcn_readfirstlane(ci->stage);
    s.iter = __builtin_amdgcn_readfirstlane(ci->iter);
    s.p = __builtin_amdgcn_readfirstlane(ci->p);
    s.rm = wave_max_v(r);
    s.conv = s.pending && s.iter >= 1 && s.rm < I.tol;
    return s;
}
// Whether the stage ends with the pending iteration, and the factor on the
// potentials if another one follows.
__device__ __forceinline__ bool mid_stage_end(const Inst &I, const MidState &s) {
    return s.conv || (s.pending && (int64_t)s.iter + 1 >= I.max_iters);
}
__device__ __forceinline__ bool mid_next_stage(const Inst &I, const MidState &s, double &ratio) {
    if (!mid_stage_end(I, s) || I.pause || s.stage + 1 >= I.n_p) return false;
    ratio = (double)I.ladder[s.stage + 1] / (double)I.ladder[s.stage];
    return true;
}
// k + f scaled, in FP64.
__device__ __forceinline__ void scale_pot(double ratio, int &k, float &f) {
    const double x = ((double)k + (double)f) * ratio, r = rint(x);
    k = (int)r;
    f = (float)(x - r);
}

// The residual of workgroup `lane`, for mid_state.
__device__ __forceinline__ float mid_residual(const Inst &I, int in, int nblk, int lane) {
    return lane < nblk ? I.res_slots[in * kMidMaxBlocks + lane] : 0.f;
}

// A thread's columns kCT t .. kCT t + 3 as it finds them: their potentials
// (copy `from`), and the partials of their sums, all requested at once (past
// the last one it is read again). The arrays' rows are padded to whole
// vectors; what the padding holds is not used.
struct MidCol {
    int4 G;
    float4 gam;
};
__device__ __forceinline__ MidCol mid_load_column(const Inst &I, int from) {
    const int j = min(kCT * (int)threadIdx.x, (I.n - 1) / kCT * kCT);
    MidCol c;
    c.G = *reinterpret_cast<const int4 *>((from ? I.G2 : I.G) + j);
    c.gam = *reinterpret_cast<const float4 *>((from ? I.gam2 : I.gam) + j);
    return c;
}
__device__ __forceinline__ void mid_load_partials(const Inst &I, int in, int nblk, int64_t slot,
                                                  float4 (&x)[kMidMaxBlocks]) {
    const int j = min(kCT * (int)threadIdx.x, (I.n - 1) / kCT * kCT);
    const float *q = I.colpart + (int64_t)in * nblk * slot + j;
#pragma unroll
    for (int b = 0; b < kMidMaxBlocks; ++b)
        x[b] = *reinterpret_cast<const float4 *>(q + (int64_t)min(b, nblk - 1) * slot);
}

// The pending column step for the thread's columns and the continuation to the
// next stage: G, gam as the next row step takes them. Every thread of the
// workgroup calls it; L.newerr is set for an empty column.
__device__ __forceinline__ void mid_columns(const Inst &I, MidColLds &L, const MidState &s,
                                            const float4 (&x)[kMidMaxBlocks], int in, int nblk, int (&G)[kCT],
                                            float (&gam)[kCT]) {
    const int t = (int)threadIdx.x, lane = t % kWave, wave = t / kWave, n = I.n, j0 = kCT * t;
    if (t == 0) {
        L.flagged = 0u;
        L.newerr = 0u;
    }
    fill_exp_table(L.tab);
    double T[kCT] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < kMidMaxBlocks; ++b) {
        T[0] += b < nblk ? (double)x[b].x : 0.0;
        T[1] += b < nblk ? (double)x[b].y : 0.0;
        T[2] += b < nblk ? (double)x[b].z : 0.0;
        T[3] += b < nblk ? (double)x[b].w : 0.0;
    }
    __syncthreads();
    if (s.pending && !s.conv) {
        unsigned bad = 0u;
#pragma unroll
        for (int c = 0; c < kCT; ++c) {
            if (j0 + c >= n) continue;
            if (!(T[c] >= (double)kSafeLo && T[c] <= (double)kSafeHi)) {
                bad |= 1u << c;
                L.list[atomicAdd(&L.flagged, 1u)] = j0 + c;
                L.newG[j0 + c] = G[c];
            } else {
                int k;
                gam[c] = neg_log_split(T[c], k);
                G[c] += k;
            }
        }
        __syncthreads();
        const int nf = (int)L.flagged;
        if (nf > 0) {
            // exact max-shifted recompute (Section 4.1.2), one column per
            // wave at a time: M = max_i (p w_ij + F_i + G_j), then
            // log v_j <- G_j - M - log sum_i exp(p w_ij + log u_i + G_j - M)
            const int p4 = 4 * s.p;
            for (int qi = wave; qi < nf; qi += kMidWaves) {
                const int j = L.list[qi];
                const int a = 4 * L.newG[j];
                int m4 = INT_MIN;
                for (int rr = lane; rr < n; rr += kWave) {
                    const int w = (int)I.W[(int64_t)rr * I.pitch + j];
                    if (w != SK_SENTINEL) m4 = max(m4, __mul24(p4, w) + a + 4 * I.F[in][rr]);
                }
                m4 = wave_max_i(m4);
                if (m4 == INT_MIN) {
                    if (lane == 0) {
                        atomicOr(&L.newerr, (unsigned)ERR_EMPTY_COL);
                        L.newg[j] = 0.f;
                    }
                    continue;
                }
                double sum = 0.0;
                for (int rr = lane; rr < n; rr += kWave) {
                    const int w = (int)I.W[(int64_t)rr * I.pitch + j];
                    if (w == SK_SENTINEL) continue;
                    const int B = 4 * I.F[in][rr] - (m4 & ~3) - 4 * kTabLo;
                    sum = fma((double)tab_at(L.tab, tab_off(p4, w, a, B)), (double)exp_frac(I.phi[in][rr]), sum);
                }
                sum = wave_sum_d(sum);
                if (lane == 0) {
                    int k;
                    L.newg[j] = neg_log_split(sum, k);
                    L.newG[j] = (a >> 2) - (m4 >> 2) + k;
                }
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < kCT; ++c)
                if ((bad >> c) & 1u) {
                    G[c] = L.newG[j0 + c];
                    gam[c] = L.newg[j0 + c];
                }
        }
    }
    double ratio;
    const bool next = mid_next_stage(I, s, ratio);
#pragma unroll
    for (int c = 0; c < kCT; ++c) {
        // a caller's starting potentials may split their logarithm in any way
        unit_frac(G[c], gam[c]);
        if (next) scale_pot(ratio, G[c], gam[c]);
    }
}
// The thread's columns into a copy of the column potentials.
__device__ __forceinline__ void mid_store_column(const Inst &I, int to, const int (&G)[kCT], const float (&gam)[kCT]) {
    const int j0 = kCT * (int)threadIdx.x;
#pragma unroll
    for (int c = 0; c < kCT; ++c)
        if (j0 + c < I.n) {
            (to ? I.G2 : I.G)[j0 + c] = G[c];
            (to ? I.gam2 : I.gam)[j0 + c] = gam[c];
        }
}

// CH: chunks of 512 columns (8 consecutive per lane). SENT: W holds absent
// entries. FOLD: the pending column step is taken here (else k_mid_columns
// has taken it and left the new column potentials in copy `out`).
template <int CH, bool SENT, bool FOLD>
__device__ __forceinline__ void mid_run(const Inst &I, MidLds<CH, FOLD> &L, MidColLds *LC, int row0, int count, int in) {
    constexpr int C = 8 * CH;
    const int t = (int)threadIdx.x, lane = t % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int n = I.n, n8 = pad8(n) >> 3, nblk = (n + kMidRows - 1) / kMidRows, blk = row0 / kMidRows;
    const int64_t slot = pad8(n);  // floats of one block's partials
    const int out = in ^ 1;
    const Ctl *ci = in ? I.ctl2 : I.ctl;
    Ctl *co = in ? I.ctl : I.ctl2;
    float *pout = I.colpart + ((int64_t)out * nblk + blk) * slot;
    const int blk_end = blk + (FOLD ? 1 : count);  // this workgroup's blocks of rows

    // ---- what the launch reads, requested before it is needed
    // (without FOLD, k_mid_columns has left copy `out` of the columns)
    const MidCol col = mid_load_column(I, FOLD ? in : out);
    float4 x[FOLD ? kMidMaxBlocks : 1];
    if constexpr (FOLD) mid_load_partials(I, in, nblk, slot, x);
    const float rres = mid_residual(I, in, nblk, lane);
    // controller words `lane` and 64 + `lane`
    constexpr int kWords = (int)(sizeof(Ctl) / 4);
    static_assert(kWords <= 2 * kWave, "two words per lane");
    uint32_t cw[2] = {0u, 0u};
    const bool writer = blk == 0 && wave == 0;
    if (writer)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (lane + kWave * h < kWords) cw[h] = reinterpret_cast<const uint32_t *>(ci)[lane + kWave * h];
    // read by one thread: a row step of another workgroup may set it during
    // this launch, and the workgroup has to decide as one
    if (t == 0) L.err = I.ctl->err;
    // a block's share of this thread: the row whose state its lane carries
    // (both copies), and the wave's rows of W
    int Fi, Fo;
    float phii, phio;
    int4 wv[kR * CH];
    auto load_block = [&](int b) {
        const int r = min(b * kMidRows + wave * kR + lane / kRL, n - 1);
        Fi = I.F[in][r];
        phii = I.phi[in][r];
        Fo = I.F[out][r];
        phio = I.phi[out][r];
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const int16_t *wr = I.W + (int64_t)min(b * kMidRows + wave * kR + k, n - 1) * I.pitch;
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
                wv[k * CH + q] = v;
            }
        }
    };
    load_block(blk);
    const MidState st = mid_state(I, ci, rres);
    fill_exp_table(L.tab);
    int G[kCT] = {col.G.x, col.G.y, col.G.z, col.G.w};
    float gam[kCT] = {col.gam.x, col.gam.y, col.gam.z, col.gam.w};
    if constexpr (FOLD) mid_columns(I, *LC, st, x, in, nblk, G, gam);
    __syncthreads();
    const unsigned newerr = FOLD ? LC->newerr : 0u;

    // ---- the decision on the pending iteration, in every workgroup alike
    int state = ST_RUNNING, stage = st.stage, iter = st.iter, p = st.p;
    const int did = st.pending && !st.conv ? 1 : 0;
    const bool end = mid_stage_end(I, st), failed = (L.err | newerr) & (ERR_EMPTY_ROW | ERR_EMPTY_COL);
    double ratio = 1.0;
    bool next = false;
    if (failed && st.pending) {
        state = ST_ERROR;
    } else {
        iter += did;
        next = mid_next_stage(I, st, ratio);
        if (next) {
            p = I.ladder[++stage];
            iter = 0;
        } else if (end) {
            state = I.pause ? ST_STAGE_END : ST_DONE;
        }
    }
    // the row potentials of the block in hand as this iteration finds them:
    // converged, the last row step is not taken; the next p holds
    // p^-1 log u (FP64)
    auto row_state = [&](int &F, float &phi) {
        F = st.conv ? Fo : Fi;
        phi = st.conv ? phio : phii;
        unit_frac(F, phi);
        if (next) scale_pot(ratio, F, phi);
    };
    if (writer) {
        // the controller, a word per lane (err is kept in copy 0 alone)
        const bool ok = state != ST_ERROR;
        const float last = ok && st.pending && st.iter >= 1 ? st.rm : __uint_as_float(0u);
        const bool has_last = ok && st.pending && st.iter >= 1;
        const int inc = ok ? did : 0;
        constexpr int kIters = (int)(offsetof(Ctl, stage_iters) / 4);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int w = lane + kWave * h;
            const uint32_t below = h ? 0u : (uint32_t)__shfl_up((int)cw[0], 1, kWave);
            uint32_t low = below;  // the low half of a 64-bit count
            if (h) {
                const uint32_t up = (uint32_t)__shfl_up((int)cw[1], 1, kWave);
                low = lane == 0 ? (uint32_t)__shfl((int)cw[0], kWave - 1, kWave) : up;
            }
            uint32_t v = cw[h];
            const uint32_t carry = inc && low == 0xffffffffu ? 1u : 0u;
            if (w == (int)(offsetof(Ctl, state) / 4)) v = (uint32_t)state;
            if (w == (int)(offsetof(Ctl, stage) / 4)) v = (uint32_t)stage;
            if (w == (int)(offsetof(Ctl, p) / 4)) v = (uint32_t)p;
            if (w == (int)(offsetof(Ctl, iter) / 4)) v = (uint32_t)iter;
            if (w == (int)(offsetof(Ctl, capped) / 4)) v += ok && end && !st.conv ? 1u : 0u;
            if (w == (int)(offsetof(Ctl, iters_total) / 4)) v += (uint32_t)inc;
            if (w == (int)(offsetof(Ctl, iters_total) / 4) + 1) v += carry;
            if (w == (int)(offsetof(Ctl, last_res) / 4) && has_last) v = __float_as_uint(last);
            if (w == (int)(offsetof(Ctl, pending) / 4)) v = state == ST_RUNNING ? 1u : 0u;
            if (w == kIters + 2 * st.stage) v += (uint32_t)inc;
            if (w == kIters + 2 * st.stage + 1) v += carry;
            if (w < kWords && w != (int)(offsetof(Ctl, err) / 4)) reinterpret_cast<uint32_t *>(co)[w] = v;
        }
        if (lane == 0 && newerr) atomicOr(&I.ctl->err, newerr);
    }
    if (FOLD && kCT * t / kMidRows == blk) mid_store_column(I, out, G, gam);
    if (state != ST_RUNNING) {
        // both copies of the row potentials hold the result (a column
        // recompute of another workgroup may still read copy `in`, but only
        // where the row step was taken, and then it holds this value already)
        for (int b = blk; b < blk_end; ++b) {
            if (b > blk) load_block(b);
            int F;
            float phi;
            row_state(F, phi);
            const int r = b * kMidRows + wave * kR + lane / kRL;
            if (r < n && lane % kRL == 0) {
                I.F[out][r] = F;
                I.phi[out][r] = phi;
                if (st.conv) {
                    I.F[in][r] = F;
                    I.phi[in][r] = phi;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < kCT; ++c) {
        const int j = kCT * t + c;
        if (j >= 8 * n8) continue;
        ColPot k;
        k.a = j < n ? 4 * G[c] : kPadExp4;
        k.g = j < n ? exp_frac(gam[c]) : 0.f;
        L.cp[swz8(j, n8)] = k;
    }
    __syncthreads();

    float e[kR * C];
    const int p4 = 4 * p;
    for (int b = blk; b < blk_end; ++b) {
        const int rw = b * kMidRows + wave * kR;  // the wave's first row
        const int r = rw + lane / kRL;
        const bool row_on = r < n;
        int F;
        float phi;
        row_state(F, phi);
        // ---- row step: S_i = sum_j e_ij exp(gam_j). The lane's columns are
        // read again for every block: kept over the column step they would not
        // fit the registers beside the terms and the next block's rows
        int A[C], ln = lane;
        float g[C];
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const bool on = 512 * q + 8 * ln < n;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const ColPot k = L.cp[on ? c * n8 + 64 * q + ln : 0];
                A[8 * q + c] = on ? k.a : kPadExp4;
                g[8 * q + c] = on ? k.g : 0.f;
            }
        }
        // rows past the matrix: every exponent 4 (p w + G_j) + kPadExp4 clamps
        // to the table's zero entry (in padding columns the sum may wrap, and
        // what these add to each other is not used)
        const int Boff = row_on ? 4 * (F - kTabLo) : kPadExp4;
        auto row_terms = [&](int k, int B) {
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                int w[8];
                unpack8i(wv[k * CH + q], w);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    float x = tab_at(L.tab, tab_off(p4, w[c], A[8 * q + c], B));
                    if (SENT) x = w[c] == SK_SENTINEL ? 0.f : x;
                    e[k * C + 8 * q + c] = x;
                }
            }
        };
        double S = wave_sums8([&](int k) {
            row_terms(k, __builtin_amdgcn_readlane(Boff, k * kRL));
            float s = e[k * C] * g[0];
#pragma unroll
            for (int c = 1; c < C; ++c) s = fmaf(e[k * C + c], g[c], s);
            return s;
        }, lane);
        int M = 0;
        uint64_t off = __ballot(row_on && !(S >= (double)kSafeLo && S <= (double)kSafeHi));
        while (off != 0ull) {
            // exact max-shifted recompute of a row whose sum left the safe range
            const int k = (__ffsll((unsigned long long)off) - 1) / kRL;
            off &= ~(((1ull << kRL) - 1ull) << (k * kRL));
            const int16_t *wr = I.W + (int64_t)(rw + k) * I.pitch;
            const int F4 = 4 * __builtin_amdgcn_readlane(F, k * kRL);
            int m4 = INT_MIN;
            for (int j = lane; j < n; j += kWave) {
                const int w = (int)wr[j];
                if (w != SK_SENTINEL) m4 = max(m4, __mul24(p4, w) + L.cp[swz8(j, n8)].a + F4);
            }
            m4 = wave_max_i(m4);
            double s = 0.0;
            if (m4 == INT_MIN) {
                if (lane == 0) atomicOr(&I.ctl->err, (unsigned)ERR_EMPTY_ROW);
                s = 1.0;
            } else {
                const int B = F4 - (m4 & ~3) - 4 * kTabLo;
                for (int j = lane; j < n; j += kWave) {
                    const int w = (int)wr[j];
                    if (w == SK_SENTINEL) continue;
                    const ColPot c = L.cp[swz8(j, n8)];
                    s = fma((double)tab_at(L.tab, tab_off(p4, w, c.a, B)), (double)c.g, s);
                }
                s = wave_sum_d(s);
            }
            if (lane / kRL == k) {
                S = s;
                M = m4 == INT_MIN ? 0 : m4 >> 2;
            }
        }
        // log u_i <- F_i - M - log S;  r_i = exp(phi_i + M) S
        int kr;
        const float phin = neg_log_split(S, kr);
        const int Fn = row_on ? F - M + kr : F;
        const double rs = (double)exp_frac(phi) * S;
        float ri = (float)(rs - 1.0);
        if (M != 0) ri = ex2(fmaf((float)M, kLog2e, lg2((float)rs))) - 1.f;
        const float res = wave_max_v(row_on ? fabsf(ri) : 0.f);
        const float rn = row_on ? exp_frac(phin) : 0.f;
        if (row_on && lane % kRL == 0) {
            I.F[out][r] = Fn;
            I.phi[out][r] = phin;
        }
        const uint64_t moved = __ballot(Fn != F);
        if (moved != 0ull) {
            const int B = 4 * (Fn - kTabLo);
#pragma unroll
            for (int k = 0; k < kR; ++k)
                if ((moved >> (k * kRL)) & 1ull) row_terms(k, __builtin_amdgcn_readlane(B, k * kRL));
        }
        // the next block's rows, in flight during the rest of this one
        if (b + 1 < blk_end) load_block(b + 1);
        // ---- column partials: sum over the block's rows of e_ij exp(phi_i)
        float acc[C];
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const float rk = readlane_v(rn, k * kRL);
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = k == 0 ? e[c] * rk : fmaf(e[k * C + c], rk, acc[c]);
        }
        // two buffers in turn: a wave writes one while others may still read
        // the other, and the barrier between keeps them a block apart
        auto &part = L.part[FOLD ? 0 : (b - blk) & 1];
        float *wres = L.wres[FOLD ? 0 : (b - blk) & 1];
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            float4 *dst = reinterpret_cast<float4 *>(&part[wave][512 * q + 8 * lane]);
            dst[0] = make_float4(acc[8 * q], acc[8 * q + 1], acc[8 * q + 2], acc[8 * q + 3]);
            dst[1] = make_float4(acc[8 * q + 4], acc[8 * q + 5], acc[8 * q + 6], acc[8 * q + 7]);
        }
        if (lane == 0) wres[wave] = res;
        __syncthreads();
        if (kCT * t < n) {
            double a[kCT] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int w = 0; w < kMidWaves; ++w) {
                const float4 y = *reinterpret_cast<const float4 *>(&part[w][kCT * t]);
                a[0] += (double)y.x;
                a[1] += (double)y.y;
                a[2] += (double)y.z;
                a[3] += (double)y.w;
            }
            *reinterpret_cast<float4 *>(pout + kCT * t) = make_float4((float)a[0], (float)a[1], (float)a[2], (float)a[3]);
        }
        pout += slot;
        if (t == 0) {
            float m = wres[0];
#pragma unroll
            for (int w = 1; w < kMidWaves; ++w) m = fmaxf(m, wres[w]);
            I.res_slots[out * kMidMaxBlocks + b] = m;
        }
    }
}

// An instance that has ended: the other copies follow.
__device__ __forceinline__ void mid_follow(const Inst &I, int row0, int count, int in) {
    const Ctl *ci = in ? I.ctl2 : I.ctl;
    Ctl *co = in ? I.ctl : I.ctl2;
    const int t = (int)threadIdx.x, j = row0 + t;
    if (t < kMidRows * count && j < I.n) {
        (in ? I.G : I.G2)[j] = (in ? I.G2 : I.G)[j];
        (in ? I.gam : I.gam2)[j] = (in ? I.gam2 : I.gam)[j];
    }
    if (row0 == 0) {
        constexpr int kErr = (int)(offsetof(Ctl, err) / 4);
        for (int w = t; w < (int)(sizeof(Ctl) / 4); w += kMidThreads)
            if (w != kErr) reinterpret_cast<uint32_t *>(co)[w] = reinterpret_cast<const uint32_t *>(ci)[w];
    }
}

template <int CH, bool FOLD>
__global__ __launch_bounds__(kMidThreads, FOLD ? 1 : 2) void k_mid(const Inst *__restrict__ insts,
                                                   const RowUnit *__restrict__ units, int in) {
    __shared__ MidLds<CH, FOLD> L;
    __shared__ std::conditional_t<FOLD, MidColLds, int> LC;
    // one instance: its blocks in order, no table to read first
    int inst = 0, row0 = kMidRows * (int)blockIdx.x, count = 1;
    if (units) {
        const RowUnit un = units[blockIdx.x];
        inst = un.inst;
        row0 = un.row0 & 0xffff;
        count = un.row0 >> 16;
    }
    const Inst &I = insts[inst];
    const Ctl *ci = in ? I.ctl2 : I.ctl;
    if (__builtin_amdgcn_readfirstlane(ci->state) != ST_RUNNING) {
        mid_follow(I, row0, count, in);
        return;
    }
    MidColLds *lc = nullptr;
    if constexpr (FOLD) lc = &LC;
    if (__builtin_amdgcn_readfirstlane(ci->sent) != 0u) mid_run<CH, true, FOLD>(I, L, lc, row0, count, in);
    else mid_run<CH, false, FOLD>(I, L, lc, row0, count, in);
}

// The column step on its own, a workgroup per instance (insts[b].mid_idx).
__global__ __launch_bounds__(kMidThreads) void k_mid_columns(const Inst *__restrict__ insts, int in) {
    __shared__ MidColLds L;
    const Inst &I = insts[insts[blockIdx.x].mid_idx];
    const Ctl *ci = in ? I.ctl2 : I.ctl;
    if (__builtin_amdgcn_readfirstlane(ci->state) != ST_RUNNING) return;  // k_mid lets the copies follow
    const int nblk = (I.n + kMidRows - 1) / kMidRows, t = (int)threadIdx.x;
    const MidCol col = mid_load_column(I, in);
    float4 x[kMidMaxBlocks];
    mid_load_partials(I, in, nblk, pad8(I.n), x);
    const MidState st = mid_state(I, ci, mid_residual(I, in, nblk, t % kWave));
    int G[kCT] = {col.G.x, col.G.y, col.G.z, col.G.w};
    float gam[kCT] = {col.gam.x, col.gam.y, col.gam.z, col.gam.w};
    mid_columns(I, L, st, x, in, nblk, G, gam);
    mid_store_column(I, in ^ 1, G, gam);
    __syncthreads();
    if (t == 0 && L.newerr) atomicOr(&I.ctl->err, L.newerr);
}

}  // namespace

hipError_t launch_mid_pair(const Inst *d_insts, const RowUnit *d_units, int nwide, int nnarrow, int ninst, int fold,
                           hipStream_t st) {
    const RowUnit *narrow = d_units ? d_units + nwide : nullptr;
    for (int in = 0; in < 2; ++in) {
        if (fold) {
            if (nwide > 0)
                hipLaunchKernelGGL((k_mid<2, true>), dim3(nwide), dim3(kMidThreads), 0, st, d_insts, d_units, in);
            if (nnarrow > 0)
                hipLaunchKernelGGL((k_mid<1, true>), dim3(nnarrow), dim3(kMidThreads), 0, st, d_insts, narrow, in);
            continue;
        }
        hipLaunchKernelGGL(k_mid_columns, dim3(ninst), dim3(kMidThreads), 0, st, d_insts, in);
        if (nwide > 0)
            hipLaunchKernelGGL((k_mid<2, false>), dim3(nwide), dim3(kMidThreads), 0, st, d_insts, d_units, in);
        if (nnarrow > 0)
            hipLaunchKernelGGL((k_mid<1, false>), dim3(nnarrow), dim3(kMidThreads), 0, st, d_insts, narrow, in);
    }
    return hipGetLastError();
}

}  // namespace sk
