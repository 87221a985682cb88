// Host runtime of libsk: contexts, arena planning, the stage controller that
// drives the sweep kernels, the FP64 recheck and certificate, pruning, and the
// C ABI entry points declared in include/sk.h.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "sk_internal.h"
#include "sk_runtime.h"

namespace sk {

// ---------------------------------------------------------------- planning

// Tuned segment heights (sk_set_tile_table); empty = built-in rule.
static std::vector<std::pair<int32_t, int32_t>> g_tile_table;

TilePlan plan_tiles(int32_t n, int vec8) {
    TilePlan t;
    t.tile_cols = vec8 ? kColTile8 : kColTile1;
    t.ntiles = (n + t.tile_cols - 1) / t.tile_cols;
    for (const auto &e : g_tile_table) {
        if (n <= e.first) {
            t.seg_rows = std::min(e.second, std::max(16, (n + 15) / 16 * 16));
            t.nseg = (n + t.seg_rows - 1) / t.seg_rows;
            return t;
        }
    }
    // Column-sweep segment height: aim for ~1024 work units per sweep, but
    // keep each unit at >= 128 rows so the fixed-slot partials stay a small
    // fraction of the matrix traffic.
    int64_t want = ((int64_t)n * t.ntiles + 1023) / 1024;
    int seg = (int)std::min<int64_t>(kMaxSegRows, std::max<int64_t>(128, (want + 15) / 16 * 16));
    seg = std::min(seg, std::max(16, (n + 15) / 16 * 16));
    t.seg_rows = seg;
    t.nseg = (n + seg - 1) / seg;
    return t;
}


// Sizes iterated by k_mid, and its column-partial slots (two copies).
static bool mid_size(int32_t n) { return n > kSmallN && n <= kMidN; }
static size_t mid_slots(int32_t n) { return 2 * (size_t)((n + kMidRows - 1) / kMidRows); }

size_t instance_bytes(int32_t n, int vec8, int storage, int fused, int mid) {
    TilePlan t = plan_tiles(n, vec8);
    const bool kstore = storage == SK_K_BF16 || storage == SK_K_F32;
    const bool is_mid = mid && mid_size(n) && !kstore;
    size_t b = 0;
    b += align_up(sizeof(int32_t) * n, 256) * 3;  // F[2], G
    b += align_up(sizeof(float) * n, 256) * 3;    // phi[2], gam
    const size_t slots = fused ? std::max(t.nseg, kFusedSlots) : t.nseg;
    b += align_up(sizeof(float) * std::max(slots * n, is_mid ? mid_slots(n) * pad8(n) : 0), 256);
    b += align_up(sizeof(uint32_t) * n, 256);
    b += align_up(sizeof(Ctl), 256);
    b += align_up(sizeof(float) * std::max((n + kRowWaves - 1) / kRowWaves, kFusedSlots), 256) * 2;
    b += align_up(sizeof(float) * n, 256);  // rres
    b += align_up(sizeof(uint32_t) * kRowResSlots * kRowResStride, 256);  // rowres
    if (n > kLdsMaxN) b += align_up(8 * (size_t)pad8(n), 256);  // colpack
    if (is_mid) b += align_up(sizeof(Ctl), 256) + align_up(sizeof(int32_t) * n, 256) + align_up(sizeof(float) * n, 256);
    if (kstore) {
        const size_t es = storage == SK_K_BF16 ? 2 : 4;
        const size_t kp = (size_t)(n + 7) / 8 * 8;
        b += align_up(es * (size_t)n * kp, 256);
        b += align_up(sizeof(float) * n, 256) * 3;  // a[2], b
    }
    return b;
}

// Row segments of the FP64 check's column pass.
static int check_seg_rows(int32_t n, const TilePlan &t) { return n <= kCheckShortN ? kCheckShortSeg : t.seg_rows; }
static int check_segs(int32_t n, const TilePlan &t) {
    const int seg = check_seg_rows(n, t);
    return (n + seg - 1) / seg;
}
// Segments whose column partials an instance's check scratch holds: the check
// of a stored K sums the column sweep's segments, which a tuned table makes
// shorter than the int16 check's.
static int check_slots(int32_t n, const TilePlan &t) { return std::max(check_segs(n, t), t.nseg); }
// Doubles of check scratch for a batch: all instances at once up to 32 MiB
// (more go in groups), at least the largest instance's.
static size_t check_scratch(size_t largest, size_t sum) {
    return std::max(largest, std::min(sum, (size_t)(32 << 20) / sizeof(double)));
}

// The library's 8-wide copy of a W whose n is not a multiple of 8.
size_t pad_copy_bytes(int32_t n) {
    return (n % 8) ? align_up(sizeof(int16_t) * (size_t)n * (size_t)pad8(n), 256) : 0;
}

size_t shared_bytes(int32_t count, const int32_t *n) {
    int64_t rows = 0, cols = 0, nmax = 0, fins = 0, mids = 0, ccols = 0;
    size_t chk_max = 0, chk_sum = 0;
    for (int k = 0; k < count; ++k) {
        // an instance takes the 8-wide plan unless its W is misaligned
        // (then the 1-wide plan: no more slots, more column units)
        TilePlan t = plan_tiles(n[k], 1), t1 = plan_tiles(n[k], 0);
        const size_t chk = check_doubles(n[k], check_slots(n[k], t));
        chk_max = std::max(chk_max, chk);
        chk_sum += chk;
        ccols += (int64_t)((n[k] + kColTile8 - 1) / kColTile8) * check_segs(n[k], t);
        rows += (n[k] + kRowWaves - 1) / kRowWaves;
        cols += std::max<int64_t>((int64_t)t.ntiles * t.nseg, (int64_t)t1.ntiles * t1.nseg);
        fins += (n[k] + kFinCols - 1) / kFinCols;
        if (mid_size(n[k])) mids += (n[k] + kMidRows - 1) / kMidRows;
        nmax = std::max<int64_t>(nmax, n[k]);
    }
    size_t b = 0;
    b += align_up(sizeof(Inst) * count, 256);
    b += align_up(sizeof(Ctl) * count, 256);
    b += align_up(sizeof(double) * 4 * count, 256) + align_up(sizeof(int64_t) * count, 256);
    b += align_up(sizeof(RowUnit) * rows, 256);
    b += align_up(sizeof(ColUnit) * cols, 256);
    b += align_up(sizeof(FinUnit) * fins, 256);
    if (mids > 0) b += align_up(sizeof(RowUnit) * mids, 256);
    b += align_up(sizeof(double) * check_scratch(chk_max, chk_sum), 256);
    if (count > 1) b += align_up(sizeof(ColUnit) * ccols, 256);
    b += align_up(sizeof(int64_t) * (nmax + 1), 256);  // prune row counts
    b += align_up(sizeof(int32_t) * (kMaxRowGrid + 1), 256);  // row-sweep workgroup bounds
    return b;
}



const char *kKernelNames[KID_COUNT] = {"init", "row_sweep", "col_sweep", "check_rows",
                                       "check_cols", "prune_count", "scan", "prune_fill",
                                       "absorb", "row_sweep_k", "col_sweep_k", "fold_k",
                                       "row_sweep:detect", "col_sweep:detect", "row_sweep:idle",
                                       "col_sweep:idle", "row_sweep_k:detect",
                                       "col_sweep_k:detect", "row_sweep_k:idle",
                                       "col_sweep_k:idle", "fused", "fused:detect", "fused:idle",
                                       "nt_product", "nt_step", "nt_product:idle",
                                       "nt_step:idle", "pad_copy", "small", "mid"};

hipEvent_t Profiler::take() {
    if (!pool.empty()) {
        hipEvent_t e = pool.back();
        pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
    return e;
}
hipEvent_t Profiler::kernel_stamp(int *idx) {
    *idx = -1;
    if (!on) return nullptr;
    hipEvent_t e = take();
    if (!e) return nullptr;
    stamps.push_back(e);
    *idx = (int)stamps.size() - 1;
    return e;
}
int Profiler::stamp(hipStream_t st) {
    if (!on) return -1;
    hipEvent_t e = take();
    if (!e) return -1;
    if (hipEventRecord(e, st) != hipSuccess) {
        pool.push_back(e);
        return -1;
    }
    stamps.push_back(e);
    return (int)stamps.size() - 1;
}
void Profiler::add(int id, int from, int to) {
    if (from >= 0 && to >= 0) pending.push_back({id, {from, to}});
}
void Profiler::begin(hipStream_t st, int id) {
    if (!on) return;
    cur_id = id;
    cur_start = stamp(st);
}
void Profiler::end(hipStream_t st) {
    if (!on || cur_start < 0) return;
    add(cur_id, cur_start, stamp(st));
    cur_start = -1;
}
void Profiler::drain() {
    for (auto &p : pending) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, stamps[p.second.first], stamps[p.second.second]) == hipSuccess) {
            launches[p.first] += 1;
            total_ms[p.first] += ms;
        }
    }
    for (hipEvent_t e : stamps) pool.push_back(e);
    stamps.clear();
    pending.clear();
    cur_start = -1;
    iter_end_stamp = -1;
}
void Profiler::reset() {
    drain();
    for (int k = 0; k < KID_COUNT; ++k) {
        launches[k] = 0;
        total_ms[k] = 0.0;
    }
}
Profiler::~Profiler() {
    for (auto e : stamps) (void)hipEventDestroy(e);
    for (auto e : pool) (void)hipEventDestroy(e);
}

}  // namespace sk

using namespace sk;

sk_status sk_set_tile_table(const int32_t *n_max, const int32_t *seg_rows, int32_t count) {
    if (count < 0 || (count > 0 && (!n_max || !seg_rows))) return SK_EINVAL;
    std::vector<std::pair<int32_t, int32_t>> t;
    for (int k = 0; k < count; ++k) {
        if (seg_rows[k] < 16 || seg_rows[k] > kMaxSegRows || seg_rows[k] % 16 != 0) return SK_EINVAL;
        if (k > 0 && n_max[k] <= n_max[k - 1]) return SK_EINVAL;
        t.push_back({n_max[k], seg_rows[k]});
    }
    g_tile_table = t;
    return SK_OK;
}

// For tests alone, not part of the ABI: the context's resident launch number
// `launch` from here is given up as CoopGiveUp says.
extern "C" void sk_test_resident_give_up(sk_ctx *ctx, int launch, int workgroup, int polls) {
    std::lock_guard<std::mutex> g(ctx->mu);
    ctx->give_up_launch = launch;
    ctx->give_up.workgroup = workgroup;
    ctx->give_up.polls = polls;
}

sk_status sk_profile_enable(sk_ctx *ctx, int enable) {
    if (!ctx) return SK_EINVAL;
    std::lock_guard<std::mutex> g(ctx->mu);
    (void)hipStreamSynchronize(ctx->stream);
    ctx->prof.reset();
    ctx->prof.on = enable != 0;
    return SK_OK;
}

int32_t sk_profile_read(sk_ctx *ctx, sk_kernel_stat *out, int32_t max) {
    if (!ctx) return -1;
    std::lock_guard<std::mutex> g(ctx->mu);
    (void)hipStreamSynchronize(ctx->stream);
    ctx->prof.drain();
    int32_t k = 0;
    for (int id = 0; id < KID_COUNT; ++id) {
        if (ctx->prof.launches[id] == 0) continue;
        if (out && k < max) {
            memset(&out[k], 0, sizeof out[k]);
            snprintf(out[k].name, sizeof out[k].name, "%s", kKernelNames[id]);
            out[k].launches = ctx->prof.launches[id];
            out[k].total_ms = ctx->prof.total_ms[id];
        }
        ++k;
    }
    return k;
}

// ---------------------------------------------------------------- context

static std::mutex g_attr_mu;
static bool g_attr_done = false;

size_t sk_potentials_bytes(int32_t n) { return n > 0 ? (size_t)16 * n : 0; }

size_t sk_arena_bytes(int32_t n, int32_t storage) {
    if (n <= 0 || n > kMaxN) return 0;
    return instance_bytes(n, 1, storage, 1) + pad_copy_bytes(n) + shared_bytes(1, &n) +
           newton_bytes(n) + 4096;
}

size_t sk_batch_arena_bytes(int32_t count, const int32_t *n, int32_t storage) {
    if (count <= 0 || !n) return 0;
    for (int k = 0; k < count; ++k)
        if (n[k] <= 0 || n[k] > (count == 1 ? kMaxN : kLdsMaxN)) return 0;
    size_t b = shared_bytes(count, n) + 4096;
    for (int k = 0; k < count; ++k) b += instance_bytes(n[k], 1, storage) + pad_copy_bytes(n[k]);
    return b;
}

sk_status sk_create(sk_ctx **out, int device, void *hip_stream, void *arena_dev_ptr,
                    size_t arena_bytes) {
    if (!out) return SK_EINVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return SK_EDEVICE;
    if (hipSetDevice(device) != hipSuccess) return SK_EDEVICE;
    // the static scratch of sk_scale_static: its address on this device
    if (static_scratch_init(device) != hipSuccess) return SK_EDEVICE;
    {
        std::lock_guard<std::mutex> g(g_attr_mu);
        if (!g_attr_done) {
            if (set_kernel_attributes() != hipSuccess) return SK_EDEVICE;
            if (set_k_attributes() != hipSuccess) return SK_EDEVICE;
            if (set_small_attributes() != hipSuccess) return SK_EDEVICE;
            if (set_real_attributes() != hipSuccess) return SK_EDEVICE;
            g_attr_done = true;
        }
    }
    sk_ctx *c = new sk_ctx();
    c->device = device;
    c->stream = (hipStream_t)hip_stream;
    c->arena = (char *)arena_dev_ptr;
    c->arena_bytes = arena_dev_ptr ? arena_bytes : 0;
    (void)hipDeviceGetAttribute(&c->num_cus, hipDeviceAttributeMultiprocessorCount, device);
    if (c->num_cus <= 0) c->num_cus = 256;
    if (hipHostMalloc((void **)&c->h_ctl, sizeof(Ctl) * kMaxBatch, hipHostMallocDefault) !=
            hipSuccess ||
        hipHostMalloc((void **)&c->h_checkout, sizeof(double) * 4 * kMaxBatch,
                      hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void **)&c->h_nnz, sizeof(int64_t) * kMaxBatch, hipHostMallocDefault) !=
            hipSuccess) {
        delete c;
        return SK_EDEVICE;
    }
    *out = c;
    return SK_OK;
}

sk_status sk_destroy(sk_ctx *ctx) {
    if (!ctx) return SK_EINVAL;
    serve_stop(ctx);
    (void)hipSetDevice(ctx->device);
    (void)hipStreamSynchronize(ctx->stream);
    if (ctx->h_ctl) (void)hipHostFree(ctx->h_ctl);
    if (ctx->h_checkout) (void)hipHostFree(ctx->h_checkout);
    if (ctx->h_nnz) (void)hipHostFree(ctx->h_nnz);
    if (ctx->h_csr) (void)hipHostFree(ctx->h_csr);
    delete ctx;
    return SK_OK;
}

const char *sk_last_error(const sk_ctx *ctx) { return ctx ? ctx->err.c_str() : "null context"; }

sk_status sk::fail(sk_ctx *ctx, sk_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    ctx->err = buf;
    return st;
}

sk_status sk::check_size(sk_ctx *ctx, int32_t n, const sk_params *p) {
    if (n < 1 || n > kMaxN) return fail(ctx, SK_EINVAL, "n = %d outside [1, %d]", n, kMaxN);
    if (n > kLdsMaxN && p && (p->storage != SK_W_I16 || p->fused || p->method != SK_SINKHORN))
        return fail(ctx, SK_EINVAL,
                    "n = %d above %d: only the two-sweep Sinkhorn iteration on int16 W (storage 0, not fused)",
                    n, kLdsMaxN);
    return SK_OK;
}

sk_status sk::check_params(sk_ctx *ctx, const sk_params *p, bool real) {
    if (!p) return fail(ctx, SK_EINVAL, "params is NULL");
    if (p->n_p < 1 || p->n_p > SK_MAX_LADDER)
        return fail(ctx, SK_EINVAL, "n_p must be in [1, %d]", SK_MAX_LADDER);
    for (int k = 0; k < p->n_p; ++k)
        if (p->p_ladder[k] < 1 || p->p_ladder[k] > 2048)
            return fail(ctx, SK_EINVAL, "p_ladder[%d] = %d outside [1, 2048]", k, p->p_ladder[k]);
    if (!(p->tol >= 0.0)) return fail(ctx, SK_EINVAL, "tol must be >= 0");
    if (p->max_iters_per_stage < 1) return fail(ctx, SK_EINVAL, "max_iters_per_stage must be >= 1");
    if (p->storage < SK_W_I16 || p->storage > SK_K_F32) return fail(ctx, SK_EINVAL, "bad storage");
    if (!(p->deform_a >= 0.0) || p->deform_a > 1e6)
        return fail(ctx, SK_EINVAL, "deform_a must be in [0, 1e6]");
    if (p->deform_a > 0.0 && p->storage != SK_W_I16)
        return fail(ctx, SK_EINVAL, "the deformed iteration sweeps int16 W");
    if (p->method != SK_SINKHORN && p->method != SK_NEWTON) return fail(ctx, SK_EINVAL, "bad method");
    if (p->method == SK_NEWTON && (p->storage != SK_W_I16 || p->fused || p->deform_a > 0.0))
        return fail(ctx, SK_EINVAL, "Newton scaling runs on int16 W, two-pass, undeformed");
    if (p->prescale != 0 && p->prescale != 1) return fail(ctx, SK_EINVAL, "prescale must be 0 or 1");
    if (!real && p->prescale)
        return fail(ctx, SK_EINVAL, "prescaling needs real-valued weights (sk_scale_real / sk_solve_real)");
    if (real && (p->storage != SK_W_I16 || p->fused || p->method != SK_SINKHORN))
        return fail(ctx, SK_EINVAL,
                    "real-valued weights run the two-sweep Sinkhorn iteration on W (storage 0, not fused)");
    return SK_OK;
}

// ---------------------------------------------------------------- batch plan

// What an iteration leaves behind and the next stage does not read: the column
// partials, and k_mid's second copies.
static bool carve_scratch(Bump &bump, Inst &I) {
    const size_t nn = (size_t)I.n;
    const size_t slots = I.fused ? std::max(I.nseg, kFusedSlots) : I.nseg;
    I.colpart = bump.take<float>(I.mid ? mid_slots(I.n) * pad8(I.n) : slots * nn);
    if (!I.colpart) return false;
    if (!I.mid) return true;
    I.ctl2 = bump.take<Ctl>(1);
    I.G2 = bump.take<int32_t>(nn);
    I.gam2 = bump.take<float>(nn);
    return I.ctl2 && I.G2 && I.gam2;
}

// Fills the descriptor of one instance and carves its buffers from `bump`.
bool sk::carve_instance(Bump &bump, const int16_t *W, int64_t pitch, int32_t nn,
                        const sk_params *prm, Inst &I, const float *Wr, bool mid_ok, bool scratch) {
    I = Inst{};
    I.W = W;
    I.pitch = pitch;
    I.n = nn;
    I.pscale = 1.0;
    // 8-wide loads read whole aligned 16-byte chunks up to column pad8(n):
    // inside each row when pitch >= pad8(n), and for the last row inside the
    // aligned chunk that holds its last entry
    I.vec8 = (pitch % 8 == 0) && (pitch >= pad8(nn)) && ((uintptr_t)W % 16 == 0);
    if (Wr) {
        // real-valued: 16-byte loads of 4 floats when every row is whole
        // 16-byte chunks
        I.W = nullptr;
        I.Wr = Wr;
        I.vec8 = (nn % 4 == 0) && (pitch % 4 == 0) && ((uintptr_t)Wr % 16 == 0);
    } else if (!I.vec8 && nn % 8 != 0) {
        // the library's padded copy (filled by k_pad_copy before the input scan)
        int16_t *cp = bump.take<int16_t>((size_t)nn * pad8(nn));
        if (!cp) return false;
        I.Wsrc = W;
        I.src_pitch = pitch;
        I.W = cp;
        I.pitch = pad8(nn);
        I.vec8 = 1;
    }
    TilePlan t = plan_tiles(nn, Wr ? 1 : I.vec8);
    if (Wr) {
        t.tile_cols = kRealTile;
        t.ntiles = (nn + kRealTile - 1) / kRealTile;
    }
    I.nseg = t.nseg;
    I.seg_rows = t.seg_rows;
    I.ntiles = t.ntiles;
    I.tile_cols = t.tile_cols;
    I.n_p = prm->n_p;
    for (int s = 0; s < prm->n_p; ++s) I.ladder[s] = prm->p_ladder[s];
    I.tol = (float)prm->tol;
    I.max_iters = prm->max_iters_per_stage;
    I.storage = prm->storage;
    I.fused = prm->fused ? 1 : 0;
    I.deform_a = prm->deform_a > 0.0 ? prm->deform_a : 0.0;
    I.fused_grid = std::min(kFusedSlots, std::max(1, nn / 2));
    // by size and options, so that a result does not depend on what else is in
    // the batch (the deformed iteration moves p, and with it every entry, each
    // time: it stays with the sweeps). Only an arena without the room for
    // k_mid's column partials (64 floats per column at n = 1024, where the
    // sweeps need 8 or fewer) leaves its sizes to the sweeps: !mid_ok.
    const bool onchip = !Wr && prm->storage == SK_W_I16 && !prm->fused && prm->method == SK_SINKHORN &&
                        I.deform_a <= 0.0;
    I.small = onchip && nn <= kSmallN;
    I.mid = onchip && mid_ok && mid_size(nn);
    for (int b = 0; b < 2; ++b) {
        I.F[b] = bump.take<int32_t>(nn);
        I.phi[b] = bump.take<float>(nn);
    }
    I.G = bump.take<int32_t>(nn);
    I.gam = bump.take<float>(nn);
    if (scratch && !carve_scratch(bump, I)) return false;
    I.rescue = bump.take<uint32_t>(nn);
    I.ctl = bump.take<Ctl>(1);
    const int nrows_units = (nn + kRowWaves - 1) / kRowWaves;
    I.ncolslots = I.fused ? I.fused_grid : t.nseg;
    I.res_slots = bump.take<float>(std::max(nrows_units, kFusedSlots));
    if (prm->storage != SK_W_I16) {
        I.drift_slots = bump.take<float>(std::max(nrows_units, kFusedSlots));
        if (!I.drift_slots) return false;
    }
    I.rres = bump.take<float>(nn);
    I.rowres = bump.take<uint32_t>((size_t)kRowResSlots * kRowResStride);
    if (!I.res_slots || !I.rres || !I.rowres) return false;
    if (nn > kLdsMaxN && !Wr) {
        I.colpack = bump.take<int2>((size_t)pad8(nn));
        if (!I.colpack) return false;
    }
    if (!I.F[0] || !I.F[1] || !I.phi[0] || !I.phi[1] || !I.G || !I.gam || !I.rescue || !I.ctl) return false;
    I.kpitch = (nn + 7) / 8 * 8;
    if (prm->storage != SK_W_I16) {
        const size_t es = prm->storage == SK_K_BF16 ? 2 : 4;
        I.K = bump.take<char>(es * (size_t)nn * I.kpitch);
        I.a[0] = bump.take<float>(nn);
        I.a[1] = bump.take<float>(nn);
        I.b = bump.take<float>(nn);
        if (!I.K || !I.a[0] || !I.a[1] || !I.b) return false;
    }
    return true;
}

// Work-unit tables, shared scratch and launch grids for the instances in B.h_insts.
sk_status sk::finish_tables(sk_ctx *ctx, Bump &bump, Batch &B, bool lean, bool solve) {
    B.count = (int)B.h_insts.size();
    // matrix loads take the non-temporal hint only when the batch's matrices
    // cannot stay in the last-level cache between passes
    size_t mbytes = 0;
    for (const Inst &I : B.h_insts) {
        const size_t es = (I.storage == SK_K_F32 || I.Wr) ? 4 : 2;
        mbytes += es * (size_t)I.n * (size_t)(I.storage == SK_W_I16 ? I.pitch : (I.n + 7) / 8 * 8);
    }
    for (Inst &I : B.h_insts) I.nt = mbytes > kNtBytes ? 1 : 0;
    B.h_rows.clear();
    B.h_cols.clear();
    B.h_fins.clear();
    B.h_ccols.clear();
    B.order.clear();
    B.row_at.assign((size_t)B.count + 1, 0);
    B.ccol_at.assign((size_t)B.count + 1, 0);
    B.fin_at.assign((size_t)B.count + 1, 0);
    B.nmax = B.sweep_nmax = 0;
    B.nsweep = B.nsmall = 0;
    for (int &c : B.small_class) c = 0;
    B.h_mid.clear();
    B.nmid = B.mid_wide = 0;
    for (int k = 0; k < B.count; ++k) {
        const Inst &I = B.h_insts[k];
        B.nmax = std::max(B.nmax, I.n);
        if (I.small) {
            B.nsmall += 1;
            B.small_class[(I.n - 1) / kWave] += 1;
        }
        if (I.mid) B.h_insts[B.nmid++].mid_idx = k;
        if (I.small || I.mid) continue;
        B.order.push_back(k);
        for (int s = 0; s < I.nseg; ++s)
            for (int tt = 0; tt < I.ntiles; ++tt) B.h_cols.push_back(ColUnit{k, tt, s, 0});
        B.sweep_nmax = std::max(B.sweep_nmax, I.n);
        B.nsweep += 1;
    }
    for (int k = 0; k < B.count; ++k)
        if (B.h_insts[k].small || B.h_insts[k].mid) B.order.push_back(k);
    size_t chk_max = 0, chk_sum = 0;
    for (int q = 0; q < B.count; ++q) {
        const int k = B.order[q];
        Inst &I = B.h_insts[k];
        const TilePlan t{I.tile_cols, I.ntiles, I.seg_rows, I.nseg};
        I.chk_seg = lean ? I.seg_rows : check_seg_rows(I.n, t);
        I.chk_nseg = lean ? I.nseg : check_segs(I.n, t);
        if (q == B.nsweep) {
            B.nsweep_rows = (int)B.h_rows.size();
            B.nsweep_fins = (int)B.h_fins.size();
        }
        B.h_insts[q].ord_idx = k;
        B.row_at[q] = (int)B.h_rows.size();
        B.ccol_at[q] = (int)B.h_ccols.size();
        B.fin_at[q] = (int)B.h_fins.size();
        for (int r = 0; r < I.n; r += kRowWaves) B.h_rows.push_back(RowUnit{k, r});
        for (int g = 0; g * kFinCols < I.n; ++g) B.h_fins.push_back(FinUnit{k, g});
        if (B.count > 1 && !lean)
            for (int s = 0; s < I.chk_nseg; ++s)
                for (int tt = 0; tt * kColTile8 < I.n; ++tt) B.h_ccols.push_back(ColUnit{k, tt, s, 0});
        const size_t chk = check_doubles(I.n, std::max(I.chk_nseg, I.nseg));
        chk_max = std::max(chk_max, chk);
        chk_sum += chk;
    }
    B.row_at[B.count] = (int)B.h_rows.size();
    B.ccol_at[B.count] = (int)B.h_ccols.size();
    B.fin_at[B.count] = (int)B.h_fins.size();
    if (B.nsweep == B.count) {
        B.nsweep_rows = (int)B.h_rows.size();
        B.nsweep_fins = (int)B.h_fins.size();
    }
    // a run of blocks per workgroup such that each launch has about the two
    // workgroups per compute unit that are resident at once (the blocks of a
    // run share the staging of the column potentials)
    int mblocks[2] = {0, 0};
    for (int q = 0; q < B.nmid; ++q) {
        const int nn = B.h_insts[B.h_insts[q].mid_idx].n;
        mblocks[nn > 512] += (nn + kMidRows - 1) / kMidRows;
    }
    B.mid_fold = mblocks[0] + mblocks[1] <= kMidFoldUnits;
    for (const bool wide : {true, false}) {
        const int run =
            B.mid_fold ? 1 : std::max(1, std::min(kMidRun, (mblocks[wide] + 2 * ctx->num_cus - 1) / (2 * ctx->num_cus)));
        for (int q = 0; q < B.nmid; ++q) {
            const int k = B.h_insts[q].mid_idx, nn = B.h_insts[k].n;
            if ((nn > 512) != wide) continue;
            const int nb = (nn + kMidRows - 1) / kMidRows;
            for (int b = 0; b < nb; b += run)
                B.h_mid.push_back(RowUnit{k, kMidRows * b | std::min(run, nb - b) << 16});
        }
        if (wide) B.mid_wide = (int)B.h_mid.size();
    }
    int at[kSmallClasses];
    for (int c = kSmallClasses - 1, first = 0; c >= 0; --c) {
        at[c] = first;
        first += B.small_class[c];
    }
    for (int k = 0; k < B.count; ++k) {
        const Inst &I = B.h_insts[k];
        if (I.small) B.h_insts[at[(I.n - 1) / kWave]++].small_idx = k;
    }
    B.d_insts = bump.take<Inst>(B.count);
    B.d_ctl_all = bump.take<Ctl>(B.count);
    B.d_checkout = bump.take<double>(4 * (size_t)B.count);
    B.d_nnz = bump.take<int64_t>(B.count);
    B.d_rows = bump.take<RowUnit>(B.h_rows.size());
    B.d_cols = bump.take<ColUnit>(B.h_cols.size());
    B.d_fins = bump.take<FinUnit>(B.h_fins.size());
    B.d_mid = nullptr;  // (an instance alone needs none)
    if (B.count > 1 && !B.h_mid.empty() && !(B.d_mid = bump.take<RowUnit>(B.h_mid.size())))
        return fail(ctx, SK_ENOMEM, "arena too small for the batch tables");
    B.d_counts = bump.take<int64_t>(B.nmax + 1);
    B.d_ccols = B.h_ccols.empty() ? nullptr : bump.take<ColUnit>(B.h_ccols.size());
    if ((!B.h_ccols.empty() && !B.d_ccols) || !B.d_insts || !B.d_rows || !B.d_cols ||
        !B.d_fins || !B.d_counts || !B.d_ctl_all || !B.d_checkout || !B.d_nnz)
        return fail(ctx, SK_ENOMEM, "arena too small for the batch tables");
    // grids: row sweep stages pad8(n) columns of potentials (8 B each) in LDS
    // (above kLdsMaxN it reads them from the instance's packed buffer)
    const size_t lds = B.nmax > kLdsMaxN ? 0 : sizeof(float2) * (size_t)pad8(B.nmax);
    const int per_cu = lds <= 32768 ? 2 : 1;
    B.row_lds = lds;
    B.row_lds_k = sizeof(float) * (size_t)((B.nmax + 7) / 8 * 8);
    B.row_grid = (int)std::max<size_t>(
        1, std::min<size_t>({B.nsweep > 0 ? (size_t)B.nsweep_rows : B.h_rows.size(), (size_t)ctx->num_cus * per_cu, (size_t)kMaxRowGrid}));
    // one workgroup per CU: with two (and four loads in flight per lane) the
    // BF16 row sweep at n = 16384 ran 99 us instead of 89 us, more
    // concurrent row streams than HBM serves well
    const int per_cu_k = 1;
    B.row_grid_k = (int)std::max<size_t>(1, std::min<size_t>(B.h_rows.size(), (size_t)ctx->num_cus * per_cu_k));
    for (Inst &I : B.h_insts) I.kres_slots = B.row_grid_k;
    // Row-sweep ranges: contiguous runs of row units of about equal cost, so
    // that a batch of mixed sizes does not wait on the workgroups that drew
    // the large instances (an even split by count ran the 512-instance batch
    // of n in [32, 1024] 24% slower). Costs in hundredths of a step: a unit
    // (one row per wave) takes one step per 512 columns of its rows (one
    // 16-byte load per lane covers 512); of five cost models timed on that
    // batch this was the best (charging the staging of an instance's column
    // data, or a constant per unit, did not help).
    // Integer costs: equal units split exactly evenly.
    constexpr int64_t kCostCols = 512;
    {
        const size_t nu = (size_t)B.nsweep_rows;
        const int g = B.row_grid;
        std::vector<int64_t> cost(nu);
        int64_t total = 0;
        for (size_t q = 0; q < nu; ++q) {
            const int64_t nn = B.h_insts[B.h_rows[q].inst].n;
            const int64_t c = 100 * ((nn + kCostCols - 1) / kCostCols);
            cost[q] = c;
            total += c;
        }
        B.h_row_bounds.assign((size_t)g + 1, (int32_t)nu);
        B.h_row_bounds[0] = 0;
        int b = 0;
        int64_t acc = 0;
        for (size_t q = 0; q < nu && b + 1 < g; ++q) {
            acc += cost[q];
            while (b + 1 < g && acc * g >= total * (b + 1)) B.h_row_bounds[++b] = (int32_t)(q + 1);
        }
        B.d_row_bounds = bump.take<int32_t>((size_t)g + 1);
        if (!B.d_row_bounds) return fail(ctx, SK_ENOMEM, "arena too small for the batch tables");
    }
    if (solve) {
        B.d_rp = bump.take<int64_t>((size_t)B.nmax + 1);
        B.d_hint = bump.take<int32_t>((size_t)B.nmax);
        if (!B.d_rp || !B.d_hint) return fail(ctx, SK_ENOMEM, "arena too small for the reduced matrix (row pointers)");
    }
    B.scratch_at = align_up(bump.off, 256);
    if (B.count == 1 && !B.h_insts[0].colpart && !carve_scratch(bump, B.h_insts[0]))
        return fail(ctx, SK_ENOMEM, "arena too small for the column partials");
    // the check's scratch: consecutive instances share it group by group
    size_t chk_cap = lean ? chk_max : check_scratch(chk_max, chk_sum);
    B.d_chk = bump.take<double>(chk_cap);
    if (!B.d_chk) {
        chk_cap = chk_max;
        B.d_chk = bump.take<double>(chk_cap);
    }
    if (!B.d_chk) return fail(ctx, SK_ENOMEM, "arena too small for the batch tables");
    B.chk_end.clear();
    size_t chk_used = 0;
    for (int q = 0; q < B.count; ++q) {
        Inst &I = B.h_insts[B.order[q]];
        const size_t chk = check_doubles(I.n, std::max(I.chk_nseg, I.nseg));
        if (chk_used + chk > chk_cap || (lean && q > 0)) {
            B.chk_end.push_back(q);
            chk_used = 0;
        }
        I.chk = B.d_chk + chk_used;
        chk_used += chk;
    }
    B.chk_end.push_back(B.count);
    B.col_grid = (int)std::max<size_t>(1, std::min<size_t>(B.h_cols.size(), (size_t)ctx->num_cus * 8));
    return SK_OK;
}

// The exchange area of the resident iteration (one instance), and for
// real-valued weights the second copies it needs: at the arena's end, and only
// if what is left has the room. Where it has not, or where the reduced matrix
// needs the room later (more_room), the instance takes a launch per iteration,
// an int16 one with the same results.
void sk::take_resident(const Bump &bump, Batch &B) {
    B.coop = false;
    B.reserved = 0;
    if (B.count != 1) return;
    Inst &I = B.h_insts[0];
    if (!I.mid && !(I.Wr && I.n <= kMidN && I.deform_a <= 0.0)) return;
    const size_t copies = I.Wr ? align_up(sizeof(Ctl), 256) + 2 * align_up(sizeof(float) * (size_t)I.n, 256) : 0;
    const size_t bytes = align_up(coop_bytes(I.n), 256) + copies;
    if (align_up(bump.off, 256) + bytes > bump.cap) return;
    const size_t at = (bump.cap - bytes) / 256 * 256;
    if (at < bump.off) return;
    Bump area{bump.base, bump.cap, at};
    if (I.Wr) {
        I.ctl2 = area.take<Ctl>(1);
        I.G2 = area.take<int32_t>(I.n);
        I.gam2 = area.take<float>(I.n);
    }
    I.coop = area.take<char>(coop_bytes(I.n));
    B.reserved = bump.cap - at;
    B.coop = true;
}

bool sk::more_room(Batch &B, Bump &rest) {
    if (B.scratch_at != 0 && rest.off > B.scratch_at) {
        rest.off = B.scratch_at;
        return true;
    }
    if (B.reserved == 0) return false;
    rest.cap += B.reserved;
    B.reserved = 0;
    B.coop = false;
    return true;
}

sk_status sk::plan_batch(sk_ctx *ctx, Bump &bump, int count, const int16_t *const *W,
                         const int64_t *pitch, const int32_t *n, const sk_params *prm,
                         Batch &B, bool solve) {
    // an arena without the room for all of it: what the sweeps need, of the
    // batch tables the least. Newton's vectors follow the plan, which
    // leaves them as much as there can be.
    const bool one = count == 1, newton = prm->method == SK_NEWTON;
    const std::string err = ctx->err;  // a plan that did not fit is no error of the call
    sk_status st = SK_ENOMEM;
    for (int lean = newton ? 1 : 0; lean < 2; ++lean) {
        Bump b = bump;
        B.h_insts.assign(count, Inst{});
        int k = 0;
        while (k < count && carve_instance(b, W[k], pitch[k], n[k], prm, B.h_insts[k], nullptr, !lean, !one)) ++k;
        st = k < count ? fail(ctx, SK_ENOMEM, "arena too small for instance %d (n=%d)", k, n[k])
                       : finish_tables(ctx, b, B, lean != 0, solve);
        if (st == SK_OK) {
            ctx->err = err;
            bump = b;
            take_resident(bump, B);
            if (newton) B.scratch_at = 0;
        }
        if (st != SK_ENOMEM) break;
    }
    return st;
}

sk_status sk::upload_batch(sk_ctx *ctx, Batch &B) {
    HIPCHK(ctx, hipMemcpyAsync(B.d_insts, B.h_insts.data(), sizeof(Inst) * B.count,
                               hipMemcpyHostToDevice, ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(B.d_rows, B.h_rows.data(), sizeof(RowUnit) * B.h_rows.size(),
                               hipMemcpyHostToDevice, ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(B.d_row_bounds, B.h_row_bounds.data(),
                               sizeof(int32_t) * B.h_row_bounds.size(), hipMemcpyHostToDevice,
                               ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(B.d_fins, B.h_fins.data(), sizeof(FinUnit) * B.h_fins.size(),
                               hipMemcpyHostToDevice, ctx->stream));
    if (!B.h_ccols.empty())
        HIPCHK(ctx, hipMemcpyAsync(B.d_ccols, B.h_ccols.data(), sizeof(ColUnit) * B.h_ccols.size(),
                                   hipMemcpyHostToDevice, ctx->stream));
    if (B.nsweep > 0)
        HIPCHK(ctx, hipMemcpyAsync(B.d_cols, B.h_cols.data(), sizeof(ColUnit) * B.h_cols.size(),
                                   hipMemcpyHostToDevice, ctx->stream));
    if (B.d_mid)
        HIPCHK(ctx, hipMemcpyAsync(B.d_mid, B.h_mid.data(), sizeof(RowUnit) * B.h_mid.size(),
                                   hipMemcpyHostToDevice, ctx->stream));
    bool pads = false;
    for (const Inst &I : B.h_insts) pads |= I.Wsrc != nullptr;
    if (pads)
        HIPCHK(ctx, PROF(ctx, KID_PAD_COPY, launch_pad_copy(B.d_insts, B.d_rows, (int)B.h_rows.size(),
                                                            B.row_grid, ctx->stream)));
    return SK_OK;
}

// Initial control blocks and the input scan (cold start or warm start).
sk_status sk::start_batch(sk_ctx *ctx, Batch &B, const sk_params *prm, void *const *pot_in) {
    HIPCHK(ctx, launch_reset_ctl(B.d_insts, nullptr, B.count, ctx->stream));
    if (B.coop) HIPCHK(ctx, launch_coop_clear(B.d_insts, B.h_insts[0].n, ctx->stream));
    if (prm->warm_start) {
        const bool one = B.count == 1;
        HIPCHK(ctx, launch_copy_pot(B.d_insts, one ? nullptr : B.d_fins, 0, (int)B.h_fins.size(),
                                    one ? pot_in[0] : nullptr, 1, ctx->stream));
    }
    if (B.h_insts[0].Wr)
        HIPCHK(ctx, PROF(ctx, KID_INIT, launch_init_real(B.d_insts, B.d_rows, (int)B.h_rows.size(),
                                                         B.row_grid, prm->warm_start ? 0 : 1, ctx->stream)));
    else
        HIPCHK(ctx, PROF(ctx, KID_INIT, launch_init(B.d_insts, B.d_rows, (int)B.h_rows.size(), B.row_grid,
                                                    prm->warm_start ? 0 : 1, ctx->stream)));
    return SK_OK;
}

sk_status sk::read_ctl(sk_ctx *ctx, Batch &B) {
    if (B.count == 1) {
        HIPCHK(ctx, hipMemcpyAsync(&ctx->h_ctl[0], B.h_insts[0].ctl, sizeof(Ctl),
                                   hipMemcpyDeviceToHost, ctx->stream));
    } else {
        HIPCHK(ctx, launch_gather_ctl(B.d_insts, B.count, B.d_ctl_all, ctx->stream));
        HIPCHK(ctx, hipMemcpyAsync(ctx->h_ctl, B.d_ctl_all, sizeof(Ctl) * B.count,
                                   hipMemcpyDeviceToHost, ctx->stream));
    }
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    return SK_OK;
}

// One Sinkhorn iteration over every running instance of the batch.
sk_status sk::iterate_i16(sk_ctx *ctx, Batch &B, bool chained) {
    Profiler &pf = ctx->prof;
    if (B.count == 1 && B.h_insts[0].fused) {
        const Inst &I = B.h_insts[0];
        HIPCHK(ctx, PROF(ctx, KID_FUSED, launch_fused(B.d_insts, 0, I.n, I.fused_grid, SK_W_I16,
                                                      I.nt, ctx->stream)));
        HIPCHK(ctx, launch_finalize(B.d_insts, B.count == 1 ? nullptr : B.d_fins, B.nsweep_fins, kFinOnePass, ctx->stream));
        pf.iter_end_stamp = -1;
        return SK_OK;
    }
    // timed: the two sweeps. Each launch records its own end stamp; the row
    // sweep is timed from the previous iteration's end stamp when this call
    // follows it directly, else from a marker.
    const Inst &I0 = B.h_insts[0];
    // n > kLdsMaxN (one instance): the row sweep reads the column entries
    // packed here (timed with it)
    const int gcol = B.count == 1 && I0.colpack != nullptr;
    const int s0 = chained && !gcol && pf.iter_end_stamp >= 0 ? pf.iter_end_stamp : pf.stamp(ctx->stream);
    if (gcol) HIPCHK(ctx, launch_col_pack(B.d_insts, 0, I0.n, 0, ctx->stream));
    const int nt = B.count > 0 ? B.h_insts[0].nt : 0;  // the same for the whole batch
    int s1, s2, s3;
    hipEvent_t e1 = pf.kernel_stamp(&s1);
    if (I0.Wr)
        HIPCHK(ctx, launch_row_sweep_real(B.d_insts, B.d_rows, (int)B.h_rows.size(), B.row_grid,
                                          B.row_lds, nt, I0.vec8, ctx->stream, e1));
    else
        HIPCHK(ctx, launch_row_sweep(B.d_insts, B.d_rows, B.nsweep_rows, B.d_row_bounds, B.row_grid,
                                     B.row_lds, nt, B.sweep_nmax <= kShortRowN, gcol, ctx->stream, e1));
    hipEvent_t e2 = pf.kernel_stamp(&s2);
    if (I0.Wr)
        HIPCHK(ctx, launch_col_sweep_real(B.d_insts, B.d_cols, (int)B.h_cols.size(), B.col_grid, nt,
                                          I0.vec8, ctx->stream, e2));
    else
        HIPCHK(ctx, launch_col_sweep(B.d_insts, B.d_cols, (int)B.h_cols.size(), B.col_grid, nt,
                                     B.sweep_nmax <= kShortRowN, ctx->stream, e2));
    pf.add(KID_ROW, s0, s1);
    pf.add(KID_COL, s1, s2);
    hipEvent_t e3 = pf.kernel_stamp(&s3);
    HIPCHK(ctx, launch_finalize(B.d_insts, B.count == 1 ? nullptr : B.d_fins, B.nsweep_fins, 0, ctx->stream, e3));
    pf.iter_end_stamp = s3;
    return SK_OK;
}

sk_status sk::iterate_small(sk_ctx *ctx, Batch &B, int budget) {
    if (B.nsmall == 0) return SK_OK;
    HIPCHK(ctx, PROF(ctx, KID_SMALL, launch_small(B.d_insts, B.small_class, budget, ctx->stream)));
    return SK_OK;
}

sk_status sk::iterate_mid(sk_ctx *ctx, Batch &B, int count) {
    if (B.h_mid.empty()) return SK_OK;
    for (int k = 0; k < count; k += 2)
        HIPCHK(ctx, PROF(ctx, KID_MID, launch_mid_pair(B.d_insts, B.count == 1 ? nullptr : B.d_mid, B.mid_wide,
                                                  (int)B.h_mid.size() - B.mid_wide, B.nmid, B.mid_fold,
                                                  ctx->stream)));
    return SK_OK;
}

// Iterations per launch of the small instances: a launch of a few
// milliseconds at most, so that a long ladder stays in the host's hands (a
// read-back per launch, ~15 us).
static constexpr int kSmallBudget = 2048;

// Runs the ladder of every instance to completion (device-side stopping).
// With timing on, launches are tagged afterwards: a triple (row, column,
// end) either did an iteration, or only detected that a stage had converged
// (its column sweep does no sums), or came after every instance finished.
sk_status sk::run_batch_i16(sk_ctx *ctx, Batch &B, const sk_params *prm, int first_stage) {
    const int check = std::max(1, prm->check_every);
    const int64_t bound = (prm->max_iters_per_stage + 1) * prm->n_p + 1;
    const size_t pstart = ctx->prof.pending.size();
    int64_t launched = 0;
    // Launch blocks between two looks at the controllers: a launch after the
    // end costs some 8 us at n = 4096 and 20 at n = 32768, a look some 20. A
    // stage takes at least two launches (an iteration, and the one that finds
    // it converged), so the first block is that long for the whole ladder;
    // the next ones are as long as the stages left take if each is like the
    // one before (they rarely take less), up to check_every. n = 4096,
    // planted, 12 launches: 738 us with a first block of 32, 539 now. For an
    // instance paused at each stage end the first block is the previous
    // stage's length, the next ones kTailBlock.
    constexpr int kTailBlock = 8;
    int blk = prm->deform_a > 0.0 ? check : std::min(check, 2 * std::max(1, prm->n_p - first_stage));
    auto left = [&](const Inst &I, const Ctl &c) -> int64_t {
        if (I.deform_a > 0.0) return check;  // one long stage
        if (I.pause || c.stage == 0) return kTailBlock;
        const int64_t stage = c.stage_iters[c.stage - 1] + 1;
        return std::max<int64_t>(2, stage - c.stage_iters[c.stage]) + (I.n_p - 1 - c.stage) * stage;
    };
    bool swept = B.nsweep > 0, mid = !B.h_mid.empty();  // they have a running instance
    if (B.count == 1 && B.h_insts[0].pause)
        blk = first_stage == 0 ? check : (int)std::min<int64_t>(check, std::max<int64_t>(
                                                4, ctx->h_ctl[0].stage_iters[first_stage - 1] + 2));
    for (;;) {
        if (swept && !B.coop)
            for (int k = 0; k < blk; ++k) {
                sk_status s = iterate_i16(ctx, B, k > 0);
                if (s != SK_OK) return s;
            }
        sk_status s = SK_OK;
        if (B.coop)
            HIPCHK(ctx, PROF(ctx, KID_MID, launch_coop(B.d_insts, B.nmax, B.h_insts[0].Wr != nullptr, kSmallBudget,
                                                       ctx->give_up_launch-- == 0 ? ctx->give_up : CoopGiveUp{},
                                                       ctx->stream)));
        else if (mid)
            s = iterate_mid(ctx, B, blk);
        if (s == SK_OK) s = iterate_small(ctx, B, kSmallBudget);
        if (s != SK_OK) return s;
        // every running instance has moved on by its block
        launched += (swept || mid) && !B.coop ? blk : kSmallBudget;
        if ((s = read_ctl(ctx, B)) != SK_OK) return s;
        // its workgroups were not all resident, or a column needs the exact
        // max shift: the rest of the run takes a launch per iteration
        if (B.coop && ctx->h_ctl[0].coop != kCoopOk) {
            B.coop = false;
            launched = 0;
        }
        bool running = false;
        int64_t want = 0;
        swept = mid = false;
        for (int k = 0; k < B.count; ++k) {
            const Ctl &c = ctx->h_ctl[k];
            if (c.state != ST_RUNNING) continue;
            running = true;
            const Inst &I = B.h_insts[k];
            if (I.small) continue;
            (I.mid ? mid : swept) = true;
            want = std::max(want, left(I, c));
        }
        if (!running) break;
        if (launched > bound) return fail(ctx, SK_EDEVICE, "stage controller did not terminate");
        blk = (int)std::min<int64_t>(check, want);
    }
    if (ctx->prof.on) {
        // triple index of each convergence detection, and the number of
        // triples that advanced some instance
        std::vector<int64_t> detect;
        int64_t working = 0;
        for (int k = 0; k < B.count; ++k) {
            if (B.h_insts[k].small || B.h_insts[k].mid) continue;
            const Ctl &c = ctx->h_ctl[k];
            int64_t t = 0;
            for (int s = first_stage; s <= std::min(c.stage, prm->n_p - 1); ++s) {
                t += c.stage_iters[s];
                const bool conv = c.stage_iters[s] < prm->max_iters_per_stage &&
                                  (s < c.stage || c.state == ST_DONE || c.state == ST_STAGE_END);
                if (conv) {
                    if (B.count == 1) detect.push_back(t);
                    t += 1;
                }
            }
            working = std::max(working, t);
        }
        if (B.count > 1) detect.clear();
        auto tagger = [&](int det, int idle) {
            return [&, det, idle](int64_t t) {
                if (t >= working) return idle;
                for (int64_t d : detect)
                    if (d == t) return det;
                return -1;
            };
        };
        ctx->prof.retag(pstart, KID_ROW, tagger(KID_ROW_DETECT, KID_ROW_IDLE));
        ctx->prof.retag(pstart, KID_COL, tagger(KID_COL_DETECT, KID_COL_IDLE));
        ctx->prof.retag(pstart, KID_FUSED, tagger(KID_FUSED_DETECT, KID_FUSED_IDLE));
    }
    return SK_OK;
}

// FP64 recheck of the batch's one instance (enqueued): row and column sums of
// the balanced matrix and the certificate terms, reduced on the device into
// B.d_checkout.
sk_status sk::enqueue_check(sk_ctx *ctx, Batch &B, const CheckCounts *cc) {
    const Inst &I = B.h_insts[0];
    const int nn = I.n;
    const int nunits = (int)B.h_rows.size(), nfins = (int)B.h_fins.size();
    const int grid = std::min(nunits, ctx->num_cus * 2);
    if (I.Wr) {
        HIPCHK(ctx, PROF(ctx, KID_CHECK_ROWS,
                         launch_check_real(B.d_insts, B.d_rows, nunits, grid, 0, nn, I.chk_nseg, I.chk,
                                           I.chk + check_stride(nn), cc ? cc->logt : 0.0,
                                           cc ? cc->counts : nullptr, cc ? cc->hint : nullptr,
                                           I.chk + 3 * check_stride(nn), ctx->stream)));
        HIPCHK(ctx, launch_check_sums(B.d_insts, nullptr, 0, nfins, 0, 1, 0, B.d_checkout, ctx->stream));
        return SK_OK;
    }
    // n > kLdsMaxN: the row pass reads (G_j, gam_j) packed in I.colpack
    const int gcol = I.colpack != nullptr;
    if (gcol) HIPCHK(ctx, launch_col_pack(B.d_insts, 0, nn, 1, ctx->stream));
    HIPCHK(ctx, PROF(ctx, KID_CHECK_ROWS,
                     launch_check_rows(B.d_insts, B.d_rows, nunits, grid, 0, cc ? cc->logt : 0.0,
                                       cc ? cc->counts : nullptr, cc ? cc->hint : nullptr, gq_lds_bytes(nn), I.nt,
                                       gcol, ctx->stream)));
    const int ncols = (nn + kColTile8 - 1) / kColTile8 * I.chk_nseg;
    HIPCHK(ctx, PROF(ctx, KID_CHECK_COLS,
                     launch_check_cols(B.d_insts, nullptr, 0, ncols, 0, I.nt, ctx->stream)));
    HIPCHK(ctx, launch_check_sums(B.d_insts, nullptr, 0, nfins, 0, 1, 0, B.d_checkout, ctx->stream));
    return SK_OK;
}

// The same for every instance of a batch (int16 W, n <= kLdsMaxN) that is not
// running, a launch of each kernel per group of instances that fits the
// scratch (separate launches per instance: 40 us each, 20 ms of the 28 ms of a
// 512-instance planted batch).
sk_status sk::enqueue_checks(sk_ctx *ctx, Batch &B) {
    if (B.count == 1 && B.h_insts[0].colpack) return enqueue_check(ctx, B);
    int q0 = 0;
    for (const int q1 : B.chk_end) {
        int nmax = 0;
        for (int q = q0; q < q1; ++q) nmax = std::max(nmax, B.h_insts[B.order[q]].n);
        const int nrows = B.row_at[q1] - B.row_at[q0];
        const int nt = B.h_insts[0].nt;  // the same for the whole batch
        // short rows: two workgroups per CU (their column data fits twice)
        const int grid = std::min(nrows, ctx->num_cus * 2);
        HIPCHK(ctx, PROF(ctx, KID_CHECK_ROWS,
                         launch_check_rows(B.d_insts, B.d_rows + B.row_at[q0], nrows, grid, 1, 0.0, nullptr, nullptr,
                                           gq_lds_bytes(nmax), nt, 0, ctx->stream)));
        const bool one = B.h_ccols.empty();  // no table: the group is one instance
        const int k0 = B.order[q0];
        const int ncols = one ? (nmax + kColTile8 - 1) / kColTile8 * B.h_insts[k0].chk_nseg
                              : B.ccol_at[q1] - B.ccol_at[q0];
        HIPCHK(ctx, PROF(ctx, KID_CHECK_COLS,
                         launch_check_cols(B.d_insts, one ? nullptr : B.d_ccols + B.ccol_at[q0], k0, ncols, 1, nt,
                                           ctx->stream)));
        HIPCHK(ctx, launch_check_sums(B.d_insts, B.d_fins + B.fin_at[q0], 0, B.fin_at[q1] - B.fin_at[q0], q0, q1 - q0,
                                      1, B.d_checkout, ctx->stream));
        q0 = q1;
    }
    return SK_OK;
}

// Proposition prop:aoc with log d_r = log u, log d_c = log v: log u cancels,
// UB = p^-1 (sum_i max_j (p w_ij + log v_j) - sum_j log v_j).
void sk::report_from_check(const double *o, double p, sk_report *rep, int n, double wref) {
    rep->residual_fp64 = o[0];
    rep->col_residual_fp64 = o[1];
    rep->residual_exact_fp64 = o[0];
    rep->col_residual_exact_fp64 = o[1];
    rep->ub = (o[2] - o[3]) / p + (double)n * wref;
}

void sk::fill_report(const Ctl &c, sk_report *rep) {
    rep->residual_fp32 = c.last_res;
    rep->iters_total = c.iters_total;
    for (int s = 0; s < SK_MAX_LADDER; ++s) rep->iters_stage[s] = c.stage_iters[s];
    rep->p_final = c.p;
    rep->stages_capped = c.capped;
}

sk_status sk::copy_potentials_out(sk_ctx *ctx, Batch &B, void *pot) {
    const bool one = pot != nullptr;
    HIPCHK(ctx, launch_copy_pot(B.d_insts, one ? nullptr : B.d_fins, 0, (int)B.h_fins.size(), pot, 0, ctx->stream));
    return SK_OK;
}

sk_status sk::status_of(const Ctl &c) {
    if (c.err & (ERR_EMPTY_ROW | ERR_EMPTY_COL)) return SK_ENOSUPPORT;
    if (c.err & ERR_NEWTON) return SK_EDEVICE;
    if (c.capped) return SK_ENOCONV;
    return SK_OK;
}

// The sweeps form the exponent 4 (p w_ij + F_i + G_j) in int32 (the byte
// offset of exp(E) in the LDS table), with p w from v_mul_i32_i24. Valid
// weights lie in [-16384, 16383]; p <= 2048 keeps |4 p w| <= 2^27, so with
// the potentials' integer parts (a few p times the weight range) and the
// padding columns' kPadExp4 = -2^30 every sum stays inside int32 and every
// exponent is exact.
sk_status sk::check_range(sk_ctx *ctx, const sk_params *prm) {
    int pmax = 0;
    for (int s = 0; s < prm->n_p; ++s) pmax = std::max(pmax, prm->p_ladder[s]);
    if ((int64_t)pmax * 16384 > ((int64_t)1 << 25))
        return fail(ctx, SK_EINVAL, "p = %d: p * 16384 exceeds 2^25 (exact int32 exponents)", pmax);
    return SK_OK;
}

sk_status sk::scale_impl(sk_ctx *ctx, int count, const int16_t *const *W, const int32_t *n,
                         const sk_params *prm, void *const *pot, sk_report *reports, char *arena,
                         size_t arena_bytes) {
    auto t0 = std::chrono::steady_clock::now();
    if (serving(ctx)) return fail(ctx, SK_EINVAL, "context is serving; blocking calls are disabled");
    ctx->absorbs = 0;
    sk_status st = check_params(ctx, prm);
    if (st != SK_OK) return st;
    if (count < 1 || count > kMaxBatch) return fail(ctx, SK_EINVAL, "count must be in [1, %d]", kMaxBatch);
    std::vector<int64_t> pitch(count);
    for (int k = 0; k < count; ++k) {
        if (!W[k] || !pot[k]) return fail(ctx, SK_EINVAL, "null W or potentials for instance %d", k);
        if (count == 1) {
            if ((st = check_size(ctx, n[0], prm)) != SK_OK) return st;
        } else if (n[k] < 1 || n[k] > kLdsMaxN) {
            return fail(ctx, SK_EINVAL, "n[%d] = %d outside [1, %d] (a batch; one larger instance goes to sk_scale)",
                        k, n[k], kLdsMaxN);
        }
        pitch[k] = n[k];
    }
    if (prm->storage != SK_W_I16 && count != 1)
        return fail(ctx, SK_EINVAL, "stored-K storages are single-instance");
    if (prm->fused && count != 1)
        return fail(ctx, SK_EINVAL, "the single-pass iteration is single-instance");
    if (prm->fused && prm->storage == SK_W_I16 && (n[0] % 8 != 0 || (uintptr_t)W[0] % 16 != 0))
        return fail(ctx, SK_EINVAL, "the single-pass iteration over int16 W needs n %% 8 == 0");
    if ((st = check_range(ctx, prm)) != SK_OK) return st;
    HIPCHK(ctx, hipSetDevice(ctx->device));
    Bump bump{arena, arena_bytes};
    Batch &B = ctx->scratch_batch;
    if ((st = plan_batch(ctx, bump, count, W, pitch.data(), n, prm, B)) != SK_OK) return st;
    for (int k = 0; k < count; ++k) B.h_insts[k].pot = pot[k];
    if ((st = upload_batch(ctx, B)) != SK_OK) return st;
    if ((st = start_batch(ctx, B, prm, pot)) != SK_OK) return st;
    if (prm->method == SK_NEWTON) {
        if (count != 1) return fail(ctx, SK_EINVAL, "Newton scaling is single-instance");
        if ((st = run_newton_i16(ctx, B, prm, bump)) != SK_OK) return st;
        if ((st = read_ctl(ctx, B)) != SK_OK) return st;
    } else if (prm->storage == SK_W_I16) {
        if ((st = run_batch_i16(ctx, B, prm)) != SK_OK) return st;
    } else {
        if ((st = run_single_k(ctx, B, prm)) != SK_OK) return st;
    }
    sk_status result = SK_OK;
    // FP64 checks of every instance, reduced on the device; one copy back
    bool any_check = false;
    for (int k = 0; k < count; ++k) any_check |= !(ctx->h_ctl[k].err & (ERR_EMPTY_ROW | ERR_EMPTY_COL));
    if (any_check) {
        st = count == 1 ? enqueue_check(ctx, B) : enqueue_checks(ctx, B);
        if (st != SK_OK) return st;
        HIPCHK(ctx, hipMemcpyAsync(ctx->h_checkout, B.d_checkout, sizeof(double) * 4 * count,
                                   hipMemcpyDeviceToHost, ctx->stream));
    }
    if ((st = copy_potentials_out(ctx, B, count == 1 ? pot[0] : nullptr)) != SK_OK) return st;
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    for (int k = 0; k < count; ++k) {
        const Ctl &c = ctx->h_ctl[k];
        sk_report rep;
        memset(&rep, 0, sizeof rep);
        fill_report(c, &rep);
        rep.absorbs = ctx->absorbs;
        if (!(c.err & (ERR_EMPTY_ROW | ERR_EMPTY_COL))) {
            report_from_check(ctx->h_checkout + 4 * (size_t)k, c.p, &rep);
            if (prm->storage != SK_W_I16 && !std::isnan(ctx->k_res_rows)) {
                rep.residual_fp64 = ctx->k_res_rows;
                rep.col_residual_fp64 = ctx->k_res_cols;
            }
        }
        rep.seconds = 0;
        if (reports) reports[k] = rep;
        sk_status sk = status_of(c);
        if (sk == SK_ENOSUPPORT || sk == SK_EDEVICE) result = sk;
        else if (sk == SK_ENOCONV && result == SK_OK) result = SK_ENOCONV;
    }
    const double secs =
        std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (reports)
        for (int k = 0; k < count; ++k) reports[k].seconds = secs;
    if (result == SK_ENOSUPPORT) fail(ctx, result, "a row or column of A has no entry");
    else if (result == SK_EDEVICE) fail(ctx, result, "Newton scaling broke down");
    else if (result == SK_ENOCONV) fail(ctx, result, "a stage hit max_iters_per_stage");
    return result;
}

sk_status sk_scale(sk_ctx *ctx, const int16_t *W, int32_t n, const sk_params *params,
                   void *potentials, sk_report *report) {
    if (!ctx) return SK_EINVAL;
    std::lock_guard<std::mutex> g(ctx->mu);
    const int16_t *Ws[1] = {W};
    void *pots[1] = {potentials};
    return scale_impl(ctx, 1, Ws, &n, params, pots, report, ctx->arena, ctx->arena_bytes);
}

sk_status sk_scale_batch(sk_ctx *ctx, int32_t count, const int16_t *const *W, const int32_t *n,
                         const sk_params *params, void *const *potentials, sk_report *reports) {
    if (!ctx) return SK_EINVAL;
    if (!W || !n || !potentials) return fail(ctx, SK_EINVAL, "null array argument");
    std::lock_guard<std::mutex> g(ctx->mu);
    return scale_impl(ctx, count, W, n, params, potentials, reports, ctx->arena, ctx->arena_bytes);
}

// ---------------------------------------------------------------- prune

sk_status sk_prune(sk_ctx *ctx, const int16_t *W, int32_t n, const void *potentials,
                   const sk_params *params, sk_csr *csr) {
    if (!ctx) return SK_EINVAL;
    std::lock_guard<std::mutex> g(ctx->mu);
    if (serving(ctx)) return fail(ctx, SK_EINVAL, "context is serving; blocking calls are disabled");
    sk_status st = check_params(ctx, params);
    if (st != SK_OK) return st;
    if (!W || !potentials || !csr || !csr->row_ptr)
        return fail(ctx, SK_EINVAL, "null argument");
    if (n < 1 || n > kMaxN) return fail(ctx, SK_EINVAL, "n = %d outside [1, %d]", n, kMaxN);
    if (!(params->threshold > 0.0)) return fail(ctx, SK_EINVAL, "threshold must be > 0");
    HIPCHK(ctx, hipSetDevice(ctx->device));
    Bump bump{ctx->arena, ctx->arena_bytes};
    Batch &B = ctx->scratch_batch;
    const int16_t *Ws[1] = {W};
    int64_t pitch = n;
    sk_params p1 = *params;
    p1.storage = SK_W_I16;
    if ((st = plan_batch(ctx, bump, 1, Ws, &pitch, &n, &p1, B)) != SK_OK) return st;
    // point the descriptor at the caller's potentials
    Inst &I = B.h_insts[0];
    char *pot = (char *)potentials;
    I.F[0] = I.F[1] = (int32_t *)pot;
    I.phi[0] = I.phi[1] = (float *)(pot + 4 * (size_t)n);
    I.G = (int32_t *)(pot + 8 * (size_t)n);
    I.gam = (float *)(pot + 12 * (size_t)n);
    if ((st = upload_batch(ctx, B)) != SK_OK) return st;
    Ctl c;
    memset(&c, 0, sizeof c);
    c.state = ST_DONE;
    c.p = params->p_ladder[params->n_p - 1];
    ctx->h_ctl[0] = c;
    HIPCHK(ctx, hipMemcpyAsync(I.ctl, &ctx->h_ctl[0], sizeof(Ctl), hipMemcpyHostToDevice,
                               ctx->stream));
    const double logt = std::log(params->threshold);
    const int nunits = (int)B.h_rows.size();
    const int gcol = I.colpack != nullptr;  // n > kLdsMaxN: (G_j, gam_j) packed
    if (gcol) HIPCHK(ctx, launch_col_pack(B.d_insts, 0, n, 1, ctx->stream));
    HIPCHK(ctx, PROF(ctx, KID_PRUNE_COUNT, launch_prune_count(B.d_insts, B.d_rows, nunits, B.row_grid, logt, B.d_counts,
                                   gq_lds_bytes(n), B.h_insts[0].nt, gcol, ctx->stream)));
    HIPCHK(ctx, PROF(ctx, KID_SCAN, launch_scan(B.d_counts, csr->row_ptr, n, ctx->stream)));
    int64_t total = 0;
    HIPCHK(ctx, hipMemcpyAsync(&total, csr->row_ptr + n, sizeof(int64_t), hipMemcpyDeviceToHost,
                               ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    const int64_t cap = csr->nnz;
    csr->n = n;
    csr->nnz = total;
    if (total > cap) return fail(ctx, SK_ENOMEM, "reduced matrix has %lld entries, capacity %lld",
                                 (long long)total, (long long)cap);
    if (total > 0) {
        if (!csr->col || !csr->w) return fail(ctx, SK_EINVAL, "null col/w buffers");
        HIPCHK(ctx, PROF(ctx, KID_PRUNE_FILL, launch_prune_fill(B.d_insts, B.d_rows, nunits, B.row_grid, logt, csr->row_ptr,
                                      csr->col, csr->w, gq_lds_bytes(n), B.h_insts[0].nt, gcol, ctx->stream)));
    }
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    return SK_OK;
}
