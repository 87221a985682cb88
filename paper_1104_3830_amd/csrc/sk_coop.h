// Sinkhorn iteration of one instance with kSmallN < n <= kMidN inside one
// launch: a workgroup per 32 rows, all of them resident at once, exchanging
// column sums and column potentials through global memory.
//
// What bounds it. One launch per iteration (sk_mid.hip) takes 12.0 us at
// n = 1003, most of it the launch itself and the loads at its start. Here an
// iteration is the row and column step on rows that stay on chip and two
// exchanges: each workgroup publishes its partial column sums, the owner of 32
// columns adds them and publishes the columns' new potentials. 7.5 us at
// n = 1003: two such exchanges take 3.6 us between 32 workgroups on 32 compute
// units of any XCD (4.5 us with all of them on one XCD, whose channels then
// carry all of the traffic), the steps the rest. The arithmetic and its order
// are those of sk_mid.hip, bit for bit.
// Keeping the terms exp(p w_ij + F_i + G_j) from one iteration to the next, as
// sk_small.hip does, did not pay: with a thousand columns some G_j moves in
// nearly every iteration, and reading the moved columns' terms one by one
// took 9.7 us.
//
// An exchange. Every published value is one 64-bit word that carries its own
// sequence number, stored and polled with relaxed agent-scope atomics, so no
// fence and no separate flag is needed: a reader spins on the word itself.
// Two buffers in turn: a word of sequence s + 2 is written only after its
// writer has seen every word of s + 1, whose writers had read all of s.
//
// Every wait is bounded: a workgroup that runs out of polls (the others could
// not become resident) leaves without its share of the result, and the commit
// kernel then drops the whole launch. Shares go to the second copies of the
// potentials; the first row copy always holds the state a launch starts from,
// and the commit of a dropped launch writes it over what others may have left
// in the second (which the sweeps read at an odd iteration). The caller goes
// on with the launch-per-iteration kernel, or the sweeps.
#pragma once

#include <climits>

#include "sk_frac.h"
#include "sk_rowsweep.h"
#include "sk_wave.h"

namespace sk {

constexpr int kCoopWaves = 4, kCoopThreads = kCoopWaves * kWave;
constexpr int kCoopR = kMidRows / kCoopWaves;  // rows per wave
constexpr int kCoopRL = kWave / kCoopR;        // lanes that carry one row's state
constexpr int kCoopCT = 4;                     // words a thread publishes and polls
// Polls of one word before a workgroup gives up (each a memory round trip of
// about a microsecond).
constexpr int kCoopSpins = 1 << 20;

// Header of the exchange area: workgroups that have left their share, and the
// last sequence number.
struct CoopHdr {
    uint32_t done, seq;
    uint32_t pad[30];
};
// Words of the exchange area after the header: two buffers each of the
// blocks' partials [block][column], the columns' potentials and the blocks'
// residuals.
__host__ __device__ constexpr size_t coop_words(int n) {
    const size_t nb = (size_t)((n + kMidRows - 1) / kMidRows);
    return sizeof(CoopHdr) / 8 + 2 * (nb * (size_t)pad8(n) + (size_t)pad8(n) + kMidMaxBlocks);
}

using CoopWord = unsigned long long;
__device__ __forceinline__ void coop_put(CoopWord *p, CoopWord v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ CoopWord coop_get(const CoopWord *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sequence number of a word: the upper half, or for column potentials the low
// four bits of the half that holds G. G has 28 bits there, fewer than the int32
// it is kept in (a cold start reaches 0.7 of 2^27, and a caller's starting
// potentials may split log u_i + log v_j anywhere): a column outside them
// leaves the iteration to the launched kernels, as one whose sum left the safe
// range does.
struct CoopSeq32 {
    static __device__ __forceinline__ bool ok(CoopWord x, uint32_t s) { return (uint32_t)(x >> 32) == s; }
};
struct CoopSeq4 {
    static __device__ __forceinline__ bool ok(CoopWord x, uint32_t s) { return ((uint32_t)(x >> 32) & 15u) == (s & 15u); }
};
// Polls the K words p(0) .. p(K - 1), all in flight together, until each has
// sequence number s. False when the spins ran out.
template <int K, class Seq, class P>
__device__ __forceinline__ bool coop_poll(P p, uint32_t s, int spins, CoopWord (&x)[K]) {
    for (int spin = 0; spin < spins; ++spin) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < K; ++k) x[k] = coop_get(p(k));
#pragma unroll
        for (int k = 0; k < K; ++k) all &= Seq::ok(x[k], s);
        if (all) return true;
    }
    return false;
}

template <int CH>
struct CoopLds {
    static constexpr int kCols = 512 * CH;
    ColPot cp[kCols];                            // code of G_j and exp(gam_j), swizzled (swz8)
    alignas(16) float part[kCoopWaves][kCols];   // column partials per wave
    float slot[kMidMaxBlocks][kMidRows];         // the blocks' partials of the owned columns
    float wres[kCoopWaves];
    float rmax;
    unsigned fail, err, bail;
};

constexpr uint32_t kCoopErr = 0xffffffffu;         // residual word of a block with an empty row
constexpr int kCoopBail = -(1 << 27);              // G of a column that leaves the iteration to other kernels

// Pol: the kind of weights. CH: chunks of 512 columns, 8 consecutive columns
// of each per lane. Pol::kKeep: the terms are kept from one iteration to the
// next, and only those of rows and columns whose integer parts moved are
// formed again (terms that cost more than their table read).
template <class Pol, int CH>
__device__ __forceinline__ void coop_run(const Inst &I, CoopLds<CH> &L, typename Pol::Lds &LP, int budget,
                                         CoopGiveUp give_up) {
    constexpr int C = 8 * CH, R = kCoopR, RL = kCoopRL;
    const int t = (int)threadIdx.x, lane0 = t % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int n = I.n, n8 = pad8(n) >> 3, nblk = (int)gridDim.x, blk = (int)blockIdx.x;
    const float tol = I.tol;
    const int spins = give_up.polls > 0 ? give_up.polls : kCoopSpins;
    if (give_up.polls > 0 && blk == give_up.workgroup) return;
    Ctl *ctl = I.ctl;
    CoopHdr *hdr = reinterpret_cast<CoopHdr *>(I.coop);
    CoopWord *base = reinterpret_cast<CoopWord *>(I.coop) + sizeof(CoopHdr) / 8;
    const int64_t slot = pad8(n);
    CoopWord *const wpart = base, *const wcol = wpart + 2 * nblk * slot, *const wresid = wcol + 2 * slot;
    int iter = __builtin_amdgcn_readfirstlane(ctl->iter);
    int stage = __builtin_amdgcn_readfirstlane(ctl->stage);
    int p = __builtin_amdgcn_readfirstlane(ctl->p);
    uint32_t seq = __builtin_amdgcn_readfirstlane(hdr->seq);
    float last_res = ctl->last_res;
    int done = 0, capped = 0, state = ST_RUNNING;
    int64_t st_iters = 0;  // of the stage in hand, by this launch

    // the row whose state this lane carries, and the column of threads below 32
    const int rw = blk * kMidRows + wave * R, r = rw + lane0 / RL;
    const bool row_on = r < n;
    const int jo = blk * kMidRows + t;
    const bool own = t < kMidRows && jo < n;
    int F = 0, G = 0;
    float phi = 0.f, gam = 0.f;
    if (row_on) {
        F = I.F[0][r];
        phi = I.phi[0][r];
    }
    if (own) {
        G = I.G[jo];
        gam = I.gam[jo];
    }
    unit_frac(F, phi);
    unit_frac(G, gam);
    Pol pol;
    pol.load(I, LP, rw, t);
    if (t == 0) {
        L.fail = 0u;
        L.bail = 0u;
        L.err = ctl->err & (ERR_EMPTY_ROW | ERR_EMPTY_COL);
    }
    auto stage_col = [&](int j, int Gj, float gj) {
        ColPot k;
        k.a = Pol::col_code(Gj, j < n);
        k.g = j < n ? exp_frac(gj) : 0.f;
        L.cp[swz8(j, n8)] = k;
    };
#pragma unroll
    for (int q = 0; q < kCoopCT; ++q) {
        const int j = kCoopCT * t + q;
        if (j >= 8 * n8) continue;
        int Gj = j < n ? I.G[j] : 0;
        float gj = j < n ? I.gam[j] : 0.f;
        unit_frac(Gj, gj);
        stage_col(j, Gj, gj);
    }
    __syncthreads();

    int A[C];
    float g[C], e[R * C];
    pol.begin(I, p);
    auto row_terms = [&](int k, int Fk) {
        pol.row_terms(LP, k, t, rw + k < n, Fk, A, e + k * C);
    };
    // the lane's columns; the bits of those whose integer part moved
    auto load_cols = [&](int lane) {
        unsigned moved = 0u;
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const bool on = 512 * q + 8 * lane < n;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const ColPot k = L.cp[on ? c * n8 + 64 * q + lane : 0];
                const int a = on ? k.a : Pol::col_code(0, false);
                if (Pol::kKeep && a != A[8 * q + c]) moved |= 1u << (8 * q + c);
                A[8 * q + c] = a;
                g[8 * q + c] = on ? k.g : 0.f;
            }
        }
        return moved;
    };
    auto all_terms = [&]() {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            row_terms(k, __builtin_amdgcn_readlane(F, k * RL));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    bool fresh = true;  // kKeep: every term is to be formed
    float rc = exp_frac(phi);  // exp(phi_i) of the current iterate

    while (done < budget) {
        ++seq;
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        // ---- row step: S_i = sum_j e_ij exp(gam_j)
        const unsigned ch = load_cols(lane);
        if constexpr (Pol::kKeep) {
            if (fresh) {
                all_terms();
                fresh = false;
            } else if (__ballot(ch != 0u) != 0ull) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if (__ballot((ch >> c) & 1u) == 0ull) continue;
                    pol.template col_terms<R, C, RL>(LP, c, t, n - rw, F, A[c], e);
                }
            }
        }
        double S = wave_sums8(
            [&](int k) {
                if constexpr (!Pol::kKeep) row_terms(k, __builtin_amdgcn_readlane(F, k * RL));
                float s = e[k * C] * g[0];
#pragma unroll
                for (int c = 1; c < C; ++c) s = fmaf(e[k * C + c], g[c], s);
                return s;
            },
            lane);
        int M = 0;
        uint64_t off = __ballot(row_on && !(S >= (double)kSafeLo && S <= (double)kSafeHi));
        while (off != 0ull) {
            // exact max-shifted recompute of a row whose sum left the safe range
            const int k = (__ffsll((unsigned long long)off) - 1) / RL;
            off &= ~(((1ull << RL) - 1ull) << (k * RL));
            int Mk;
            double s;
            if (!pol.rescue_row(I, L, LP, rw + k, __builtin_amdgcn_readlane(F, k * RL), lane, n8, s, Mk)) {
                if (lane == 0) atomicOr(&L.err, (unsigned)ERR_EMPTY_ROW);
                s = 1.0;
                Mk = 0;
            }
            if (lane / RL == k) {
                S = s;
                M = Mk;
            }
        }
        // log u_i <- F_i - M - log S;  r_i = exp(phi_i + M) S
        int kr;
        const float phin = neg_log_split(S, kr);
        const int Fn = row_on ? F - M + kr : F;
        const double rs = (double)rc * S;
        float ri = (float)(rs - 1.0);
        if (M != 0) ri = ex2(fmaf((float)M, kLog2e, lg2((float)rs))) - 1.f;
        const float res = wave_max_v(row_on ? fabsf(ri) : 0.f);
        const float rn = row_on ? exp_frac(phin) : 0.f;
        const uint64_t moved = __ballot(Fn != F);
        if (moved != 0ull) {
#pragma unroll
            for (int k = 0; k < R; ++k)
                if ((moved >> (k * RL)) & 1ull) row_terms(k, __builtin_amdgcn_readlane(Fn, k * RL));
        }
        // ---- column partials: sum over the block's rows of e_ij exp(phi_i)
        float acc[C];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const float rk = readlane_v(rn, k * RL);
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = k == 0 ? e[c] * rk : fmaf(e[k * C + c], rk, acc[c]);
        }
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            float4 *dst = reinterpret_cast<float4 *>(&L.part[wave][512 * q + 8 * lane]);
            dst[0] = make_float4(acc[8 * q], acc[8 * q + 1], acc[8 * q + 2], acc[8 * q + 3]);
            dst[1] = make_float4(acc[8 * q + 4], acc[8 * q + 5], acc[8 * q + 6], acc[8 * q + 7]);
        }
        if (lane == 0) L.wres[wave] = res;
        __syncthreads();
        // ---- first exchange: partial column sums, residuals
        const CoopWord tag = (CoopWord)seq << 32;
        const int buf = (int)(seq & 1u);
        if (kCoopCT * t < n) {
            double a[kCoopCT] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int w = 0; w < kCoopWaves; ++w) {
                const float4 y = *reinterpret_cast<const float4 *>(&L.part[w][kCoopCT * t]);
                a[0] += (double)y.x;
                a[1] += (double)y.y;
                a[2] += (double)y.z;
                a[3] += (double)y.w;
            }
            CoopWord *dst = wpart + ((int64_t)buf * nblk + blk) * slot + kCoopCT * t;
#pragma unroll
            for (int q = 0; q < kCoopCT; ++q)
                if (kCoopCT * t + q < n) coop_put(dst + q, tag | __float_as_uint((float)a[q]));
        }
        if (t == 0) {
            const float m = fmaxf(fmaxf(L.wres[0], L.wres[1]), fmaxf(L.wres[2], L.wres[3]));
            coop_put(wresid + buf * kMidMaxBlocks + blk, tag | (L.err ? kCoopErr : __float_as_uint(m)));
        }
        bool good = true;
        {
            // the owned columns' partials: column t % 32 of blocks t / 32 + 8 q
            // (blocks and columns past the last are those again)
            const int jc = min(blk * kMidRows + t % kMidRows, n - 1);
            const CoopWord *src = wpart + (int64_t)buf * nblk * slot + jc;
            CoopWord x[kMidMaxBlocks * kMidRows / kCoopThreads];
            constexpr int K = kMidMaxBlocks * kMidRows / kCoopThreads, Q = kCoopThreads / kMidRows;
            good &= coop_poll<K, CoopSeq32>(
                [&](int k) { return src + (int64_t)min(t / kMidRows + Q * k, nblk - 1) * slot; }, seq, spins, x);
#pragma unroll
            for (int k = 0; k < K; ++k) L.slot[t / kMidRows + Q * k][t % kMidRows] = __uint_as_float((uint32_t)x[k]);
        }
        if (wave == kCoopWaves - 1) {
            CoopWord x[1];
            good &= coop_poll<1, CoopSeq32>(
                [&](int) { return wresid + buf * kMidMaxBlocks + min(lane, nblk - 1); }, seq, spins, x);
            const uint32_t b = (uint32_t)x[0];
            const float m = wave_max_v(b == kCoopErr ? 0.f : __uint_as_float(b));
            if (b == kCoopErr) L.err = ERR_EMPTY_ROW;
            if (lane == 0) L.rmax = m;
        }
        if (!good) L.fail = 1u;
        __syncthreads();
        if (L.fail) return;
        const bool error = L.err != 0u;
        const float rmax = L.rmax;
        const bool conv = iter >= 1 && rmax < tol;
        // ---- the decision, in every workgroup alike
        const bool end = !error && (conv || (int64_t)iter + 1 >= I.max_iters);
        const bool next = end && !I.pause && stage + 1 < I.n_p;
        const double ratio = next ? (double)I.ladder[stage + 1] / (double)I.ladder[stage] : 1.0;
        // ---- column step of the owned columns
        int Gn = G;
        float gamn = gam;
        bool flag = false;
        if (own && !conv) {
            double T = 0.0;
            for (int b0 = 0; b0 < nblk; b0 += 8) {
                float y[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) y[b] = L.slot[b0 + b][t];
#pragma unroll
                for (int b = 0; b < 8; ++b) T += b0 + b < nblk ? (double)y[b] : 0.0;
            }
            flag = !(T >= (double)kSafeLo && T <= (double)kSafeHi);
            int k;
            gamn = neg_log_split(T, k);
            Gn = G + k;
        }
        if (next) {
            // the next p, with p^-1 log v held (FP64)
            const double x = ((double)Gn + (double)gamn) * ratio, k = rint(x);
            Gn = (int)k;
            gamn = (float)(x - k);
        }
        flag |= own && (Gn <= kCoopBail || Gn >= -kCoopBail);
        if (error) {
            state = ST_ERROR;
            break;
        }
        // ---- second exchange: the columns' new potentials
        if (own) {
            const uint32_t hi = ((uint32_t)(flag ? kCoopBail : Gn) << 4) | (seq & 15u);
            coop_put(wcol + buf * slot + jo, (CoopWord)hi << 32 | __float_as_uint(gamn));
        }
        {
            CoopWord x[kCoopCT];
            good = kCoopCT * t >= n || coop_poll<kCoopCT, CoopSeq4>(
                [&](int k) { return wcol + buf * slot + min(kCoopCT * t + k, n - 1); }, seq, spins, x);
            if (!good) L.fail = 1u;
#pragma unroll
            for (int q = 0; q < kCoopCT; ++q) {
                const int j = kCoopCT * t + q;
                if (j >= 8 * n8) continue;
                const int Gj = kCoopCT * t < n ? (int)(uint32_t)(x[q] >> 32) >> 4 : 0;
                if (kCoopCT * t < n && Gj == kCoopBail) L.bail = 1u;
                stage_col(j, Gj, kCoopCT * t < n ? __uint_as_float((uint32_t)x[q]) : 0.f);
            }
        }
        __syncthreads();
        if (L.fail) return;
        if (L.bail) break;  // this iteration is left to the launch-per-iteration kernel
        // ---- commit
        G = Gn;
        gam = gamn;
        if (conv) {
            last_res = rmax;
        } else {
            F = Fn;
            phi = phin;
            rc = rn;
            if (iter >= 1) last_res = rmax;
            ++iter;
            ++done;
            ++st_iters;
            capped += end ? 1 : 0;
        }
        if (end) {
            if (!next) {
                state = I.pause ? ST_STAGE_END : ST_DONE;
                break;
            }
            if (blk == 0 && t == 0) I.ctl2->stage_iters[stage] = st_iters;
            st_iters = 0;
            const double x = ((double)F + (double)phi) * ratio, k = rint(x);
            F = (int)k;
            phi = (float)(x - k);
            rc = exp_frac(phi);
            ++stage;
            p = I.ladder[stage];
            pol.begin(I, p);
            fresh = true;
            iter = 0;
        }
    }
    if (blk == give_up.workgroup) return;
    // ---- this workgroup's share, into the second copies (k_coop_commit)
    if (row_on && lane0 % RL == 0) {
        I.F[1][r] = F;
        I.phi[1][r] = phi;
    }
    if (own) {
        I.G2[jo] = G;
        I.gam2[jo] = gam;
    }
    if (t == 0) {
        if (blk == 0) {
            // what the launch adds to the controller
            Ctl *c = I.ctl2;
            c->stage_iters[stage] = st_iters;
            c->err = L.err;
            c->state = state;
            c->stage = stage;
            c->p = p;
            c->iter = iter;
            c->capped = capped;
            c->iters_total = done;
            c->last_res = last_res;
            c->coop = L.bail ? kCoopBailed : kCoopOk;
            hdr->seq = seq;
        }
        atomicAdd(&hdr->done, 1u);
    }
}

}  // namespace sk
