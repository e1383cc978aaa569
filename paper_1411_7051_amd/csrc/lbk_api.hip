// lbk_api.hip -- host side of the C ABI declared in include/lbk.h: argument
// validation, workspace carve-up, launch sequencing on the caller's stream,
// FP64 diagnostics and state save/load.  No kernels live here.
#include "lbk_adjoint.h"
#include "lbk_host.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace lbk;

namespace {
thread_local std::string g_err;
} // namespace

lbk_status lbk::fail(lbk_status s, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

namespace {

size_t elem_size(int storage) { return storage == LBK_F32 ? 4 : 2; }

WsLayout layout_of(const lbk_desc &d)
{
    WsLayout L{};
    L.pitch = (int)align_up((size_t)d.nx, 64);
    const size_t es = elem_size(d.storage), p = (size_t)L.pitch;
    L.lay.row = p * (4 + 9 * es);
    L.lay.h_off = (uint32_t)(p * 4);
    L.lay.h_slot = (uint32_t)(p * es);
    L.mlay.row = 3 * p * 4;
    L.mlay.slot = (uint32_t)(p * 4);
    L.level_bytes = L.lay.row * (size_t)d.ny;
    const size_t f32 = p * (size_t)d.ny * 4;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    L.level[0] = take(L.level_bytes);
    L.level[1] = take(L.level_bytes);
    L.med = take(L.mlay.row * (size_t)d.ny);
    L.uxp = take(f32);
    L.uyp = take(f32);
    Geom g{d.nx, d.ny, L.pitch};
    L.blocks = launch_of(g).blocks;
    L.partials = take((size_t)8 * L.blocks * sizeof(double));
    L.total = o;
    return L;
}

lbk_status check_desc(const lbk_desc *d)
{
    if (!d)
        return fail(LBK_ERR_INVALID_ARG, "desc is NULL");
    if (d->nx < 1 || d->ny < 1)
        return fail(LBK_ERR_INVALID_ARG, "nx, ny must be >= 1 (got %d, %d)", d->nx, d->ny);
    if ((int64_t)align_up((size_t)d->nx, 64) * d->ny > (int64_t)1 << 30)
        return fail(LBK_ERR_UNSUPPORTED, "lattice of %d x %d exceeds 2^30 nodes", d->nx, d->ny);
    // kernels reach every row block through a buffer resource with 32-bit
    // offsets; the widest row (an FP32 state row, 40 B per node) must fit
    if ((uint64_t)align_up((size_t)d->nx, 64) * 40 > 0xFFFFFFFFull)
        return fail(LBK_ERR_UNSUPPORTED, "rows of %d nodes exceed the 4 GiB a row block may span",
                    d->nx);
    if (d->bc_x < 0 || d->bc_x > 2 || d->bc_y < 0 || d->bc_y > 1)
        return fail(LBK_ERR_INVALID_ARG, "bc_x must be 0..2 and bc_y 0..1 (got %d, %d)",
                    d->bc_x, d->bc_y);
    if (d->storage < 0 || d->storage > 2)
        return fail(LBK_ERR_INVALID_ARG, "storage must be 0..2 (got %d)", d->storage);
    if (!(d->tau > 0.5) || !isfinite(d->tau))
        return fail(LBK_ERR_INVALID_ARG, "tau must be > 1/2 (got %g)", d->tau);
    if (!isfinite(d->gx) || !isfinite(d->gy) || !isfinite(d->f_eps) || d->f_eps < 0)
        return fail(LBK_ERR_INVALID_ARG, "gx, gy, f_eps must be finite, f_eps >= 0");
    if (d->bc_x == LBK_BC_PRESSURE) {
        if (d->nx < 3)
            return fail(LBK_ERR_INVALID_ARG, "pressure boundaries need nx >= 3");
    }
    if ((d->bc_x == LBK_BC_PRESSURE || d->init == 1) &&
        (!(d->rho_in > 0) || !(d->rho_out > 0) || !isfinite(d->rho_in) || !isfinite(d->rho_out)))
        return fail(LBK_ERR_INVALID_ARG, "rho_in, rho_out must be positive and finite");
    if (d->init != 0 && d->init != 1)
        return fail(LBK_ERR_INVALID_ARG, "init must be 0 or 1");
    if (d->init == 0 && (!(d->rho0 > 0) || !isfinite(d->rho0)))
        return fail(LBK_ERR_INVALID_ARG, "rho0 must be positive and finite");
    if (!(d->rho_ref > 0) || !isfinite(d->rho_ref))
        return fail(LBK_ERR_INVALID_ARG, "rho_ref must be positive and finite");
    if (d->check_every < 0)
        return fail(LBK_ERR_INVALID_ARG, "check_every must be >= 0");
    if (d->correlation < 0 || d->correlation > 2)
        return fail(LBK_ERR_INVALID_ARG, "correlation must be 0..2 (got %d)", d->correlation);
    if (!(d->slip_b <= 0.0) || !isfinite(d->slip_b))
        return fail(LBK_ERR_INVALID_ARG, "slip_b must be finite and <= 0 (got %g)", d->slip_b);
    if (d->pass_mode < LBK_PASS_AUTO || d->pass_mode > LBK_PASS_THREE_STEP)
        return fail(LBK_ERR_INVALID_ARG, "pass_mode must be 0..3 (got %d)", d->pass_mode);
    if (d->band < 0 || d->band > 1024)
        return fail(LBK_ERR_INVALID_ARG, "band must be 0..1024 (got %d)", d->band);
    return LBK_OK;
}

// Split a double into hi + lo floats with hi + lo == v to ~2^-48 relative.
void split(double v, float &hi, float &lo)
{
    hi = (float)v;
    lo = (float)(v - (double)hi);
}

} // namespace

// Shape and steps of tile passes over one or several lattices: the least
// predicted time per step.  A launch costs about 4.2 us (dispatch, the latency
// of the loads, the drain of the stores); every tile of a compute unit's share
// takes 0.103 us per row it loads and 0.043 us per row update; and 0.07 us per
// row update of one tile is what the barriers leave exposed whatever the
// share.  The constants fit the FP32 times of ten shapes on lattices from
// 33 x 21 to 4096 x 4096 within about 10% (16-bit ones run alike), which
// orders the shapes right where they differ: us a step, chosen against the next
// candidate kind, 64 x 32: 2.1 (8 x 1 rows, 3 steps) / 2.5 (12 x 1, 4);
// 256 x 256: 2.4 (16 x 1, 5) / 2.5 (8 x 2, 5); 777 x 333: 4.2 (16 x 1, 3) / 4.7
// (16 x 2, 5); 1024 x 512: 6.2 (16 x 2, 5) / 6.9 (16 x 1, 3); 1024 x 1024: 9.6
// (12 x 2, 4) / 10.4 (16 x 2, 5); 4096 x 4096: 99 (16 x 2, 4) / 106 (12 x 2, 4).
TilePlan lbk::tile_plan(const int *nx, const int *ny, int n)
{
    static const TilePlan cand[] = {{{8, 1}, 3},  {{12, 1}, 3}, {{12, 1}, 4}, {{16, 1}, 3},
                                    {{16, 1}, 4}, {{16, 1}, 5}, {{8, 2}, 3},  {{12, 2}, 4},
                                    {{16, 2}, 4}, {{16, 2}, 5}};
    const double cus = 256;
    TilePlan best = cand[0];
    double best_us = INFINITY;
    for (const TilePlan &p : cand) {
        double tiles = 0;
        for (int i = 0; i < n; ++i)
            tiles += (double)tile_strips(nx[i], p) * tile_bands(ny[i], p);
        // tiles of the busiest compute unit: whole ones while they are few
        const double q = tiles <= 8 * cus ? ceil(tiles / cus) : tiles / cus;
        const int H = p.tile.waves * p.tile.rows;
        const int rows = p.steps * (H - 1 - p.steps); // row updates: H - 2 - 2 k at step k
        const double us = (4.2 + q * (0.103 * H + 0.043 * rows) + 0.07 * rows) / p.steps;
        if (us < best_us) {
            best_us = us;
            best = p;
        }
    }
    best.us = best_us;
    return best;
}

double lbk::tile_us(const TilePlan &p, int storage, double model, const int *nx,
                    const int *ny, int n)
{
    const int H = p.tile.waves * p.tile.rows, own_x = 64 - 2 * p.steps, own_y = H - 2 * p.steps;
    const double level = 4.0 + 9.0 * elem_size(storage); // bytes of a node's state
    double bytes = 0;
    for (int i = 0; i < n; ++i)
        bytes += (double)tile_strips(nx[i], p) * tile_bands(ny[i], p) *
                 (64.0 * H * (level + 12.0) + (double)own_x * std::min(own_y, ny[i]) * level);
    return std::max(p.us * model, bytes / p.steps / 5.3e6); // 5.3 TB/s
}

// Whether tile passes lead on a lattice: everywhere but
//
// - where a single band of the passes they replace covers a lattice of a few
//   rows, which those then march along without recomputing any, while a tile
//   loads 8 to 16 rows for the few it stores.  The predicted times (us a step, n
//   the nodes) are fits to lattices 24,576 to 4,194,304 wide, right within 8%
//   where they decide: us a step, tile passes against the others, 32768 x 1
//   2.7 / 4.1 and 131072 x 1 5.7 / 4.6 (FP32), 98304 x 3 5.9 / 6.1 and 262144 x 3
//   12.8 / 10.9 (FP16), 524288 x 2 18.5 / 12.0, 1048576 x 8 68 / 73 and
//   1048576 x 5 61 / 51 (FP32), 1048576 x 12 98 / 79 and 1048576 x 16 101 / 101
//   (FP16).  The Forchheimer term costs a tile's redundant updates more than a
//   pass that waits for memory: 262144 x 2 13.8 / 11.1 with it, 10.1 / 10.9
//   without;
// - with the Forchheimer term, 16-bit storage and pressure columns (whose strips
//   then hold their compute units longest) on lattices that single sweeps read
//   from the on-package cache: 777 x 333 5.7 / 6.5, 512 x 512 5.7 / 5.5,
//   1024 x 512 9.5 / 7.5, 1024 x 1024 15.1 / 13.9, 1400 x 1400 23.3 / 23.4.
static bool tiles_lead(const lbk_desc &d, const Physics &ph, const TilePlan &p)
{
    const double n = (double)d.nx * d.ny;
    const bool f32 = d.storage == LBK_F32, forch = ph.feps != 0.0f;
    if (forch && !f32 && d.bc_x == LBK_BC_PRESSURE && d.ny > 8 && n >= 1 << 18 && n < 3 << 19)
        return false;
    double us = INFINITY;
    if (n >= (double)three_step_nodes(d.storage)) {
        if (d.ny < fwd_band3(d) + forch)
            us = 1e-6 * n * (f32 ? 7.5 + 7.5 / d.ny : 6.1 + 8.0 / d.ny) *
                 (!forch ? 1.0 : f32 ? 1.12 : 1.3);
    } else if (n >= (double)two_step_nodes(d.storage)) {
        if (d.ny < fwd_band(d) + forch)
            us = 1.0 + 1e-6 * n * (f32 ? 11.0 : 8.0) * (!forch ? 1.0 : f32 ? 1.08 : 1.2);
    } else if (d.ny <= 8) {
        us = std::max(3.7, 3.3 + 1e-6 * n * (f32 ? 14.5 : 9.7));
    }
    const double model = forch ? 1.4 : ph.standard ? 1.0 : 1.03;
    return tile_us(p, d.storage, model, &d.nx, &d.ny, 1) <= us;
}

// The next launch of `left` >= 1 steps.  Tile passes share the steps evenly
// (22 steps at up to 5 a launch are two fives and three fours; a whole pass has
// three steps or more, so none gets one); three-step passes leave a remainder to
// a two-step pass or a single sweep.  Every pass is bitwise the single sweeps it
// replaces.
Pass lbk::next_pass(const lbk_lattice *lat, int64_t left)
{
    if (left > 1 && tile_pass(lat)) {
        const TilePlan &p = lat->plan;
        const int64_t launches = (left + p.steps - 1) / p.steps;
        return Pass{PASS_TILE, (int)((left + launches - 1) / launches), p.tile};
    }
    if (left > 2 && three_step_pass(lat))
        return Pass{PASS_THREE, 3, {}};
    if (left > 1 && two_step_pass(lat))
        return Pass{PASS_TWO, 2, {}};
    return Pass{PASS_ONE, 1, {}};
}

hipError_t lbk::launch_pass(const lbk_lattice *lat, const Pass &p, const char *src, char *dst,
                            float *hist, size_t hist_bytes, hipStream_t st)
{
    const lbk_desc &d = lat->d;
    auto slot = [&](int k) {
        return hist ? reinterpret_cast<float *>(reinterpret_cast<char *>(hist) + k * hist_bytes)
                    : nullptr;
    };
    switch (p.kind) {
    case PASS_TILE:
        return launch_tile(d.storage, d.bc_x, d.bc_y, src, dst, lat->L.lay, lat->med(),
                           lat->L.mlay, lat->g, lat->ph, lat->s(), lat->inv_s(), p.tile, p.steps,
                           hist, hist_bytes, st);
    case PASS_THREE:
        return launch_sweep3x(d.storage, d.bc_x, d.bc_y, src, dst, lat->L.lay, lat->med(),
                              lat->L.mlay, lat->g, lat->ph, lat->s(), lat->inv_s(), fwd_band3(d),
                              slot(0), slot(1), slot(2), st);
    case PASS_TWO:
        return launch_sweep2(d.storage, d.bc_x, d.bc_y, src, dst, lat->L.lay, lat->med(),
                             lat->L.mlay, lat->g, lat->ph, lat->s(), lat->inv_s(), fwd_band(d),
                             slot(0), slot(1), st);
    default:
        return launch_sweep(d.storage, d.bc_x, d.bc_y, src, dst, lat->L.lay, lat->med(),
                            lat->L.mlay, lat->g, lat->ph, lat->s(), lat->inv_s(), hist, st);
    }
}

// n steps of the lattice on stream st.
lbk_status lbk::advance(lbk_lattice *lat, int64_t n, hipStream_t st)
{
    for (int64_t i = 0; i < n;) {
        const Pass p = next_pass(lat, n - i);
        const int nxt = lat->cur ^ 1;
        HIP_TRY(launch_pass(lat, p, lat->state(lat->cur), lat->state(nxt), nullptr, 0, st));
        lat->cur = nxt;
        lat->t += p.steps;
        ++lat->version;
        i += p.steps;
    }
    return LBK_OK;
}

namespace {

// Pool of result slots: slabs of pinned memory that every device can write,
// kSlots slots each.  A slab without a taken slot is freed unless it is the
// only one, so the pool holds at most one page beyond what its users hold.
constexpr size_t kSlotBytes = 16 * sizeof(double);
constexpr int kSlots = 32;
struct Slab {
    char *base = nullptr;
    uint32_t taken = 0; // bit per slot
};
std::mutex g_slab_mu;
std::vector<Slab> &slabs()
{
    static std::vector<Slab> *v = new std::vector<Slab>(); // outlives every handle
    return *v;
}

} // namespace

bool lbk::HostSums::alloc()
try {
    std::lock_guard<std::mutex> lock(g_slab_mu);
    std::vector<Slab> &v = slabs();
    Slab *s = nullptr;
    for (Slab &c : v)
        if (c.taken != 0xFFFFFFFFu)
            s = &c;
    if (!s) {
        v.reserve(v.size() + 1);
        Slab n;
        if (hipHostMalloc((void **)&n.base, kSlots * kSlotBytes,
                          hipHostMallocCoherent | hipHostMallocPortable) != hipSuccess)
            return false;
        v.push_back(n);
        s = &v.back();
    }
    const int k = __builtin_ctz(~s->taken);
    s->taken |= 1u << k;
    sums = reinterpret_cast<double *>(s->base + k * kSlotBytes);
    memset(sums, 0, kSlotBytes);
    done = reinterpret_cast<uint64_t *>(sums + 8);
    seq = 0;
    return true;
} catch (...) { // no memory for the pool's list
    return false;
}

void lbk::HostSums::release()
{
    if (!sums)
        return;
    std::lock_guard<std::mutex> lock(g_slab_mu);
    std::vector<Slab> &v = slabs();
    const char *p = reinterpret_cast<const char *>(sums);
    sums = nullptr;
    for (size_t i = 0; i < v.size(); ++i) {
        if (p < v[i].base || p >= v[i].base + kSlots * kSlotBytes)
            continue;
        v[i].taken &= ~(1u << ((p - v[i].base) / kSlotBytes));
        if (v[i].taken == 0 && v.size() > 1) {
            (void)hipHostFree(v[i].base);
            v.erase(v.begin() + i);
        }
        return;
    }
}

lbk_status lbk::HostSums::fetch(const double *partials, int slots, int blocks,
                                unsigned max_mask, hipStream_t st)
{
    HIP_TRY(launch_finish(partials, slots, blocks, max_mask, sums, done, ++seq, st));
    auto arrived = [&] {
        for (int k = 0; k < slots; ++k)
            if (__atomic_load_n(&done[k], __ATOMIC_ACQUIRE) != seq)
                return false;
        return true;
    };
    // poll for a bounded time, then wait for the stream (which also reports
    // an error that kept the kernel from running)
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(2);
    while (!arrived()) {
        for (int i = 0; i < 32; ++i)
            __builtin_ia32_pause();
        if (std::chrono::steady_clock::now() > until) {
            HIP_TRY(hipStreamSynchronize(st));
            break;
        }
    }
    return LBK_OK;
}

// Run a reduction's finish kernel and bring `slots` doubles to lat->host.
lbk_status lbk::fetch(lbk_lattice *lat, int slots, unsigned max_mask)
{
    return lat->out.fetch(lat->partials(), slots, lat->L.blocks, max_mask, lat->stream);
}

// NaN/Inf check of the current state; for FP16 also re-centre the scale so
// the largest stored magnitude sits near 2^12 (exact power-of-two rescale).
lbk_status lbk::check_state(lbk_lattice *lat)
{
    char *s = lat->state(lat->cur);
    HIP_TRY(launch_state_sums(lat->d.storage, s, lat->L.lay, lat->g, lat->inv_s(),
                              lat->partials(), lat->stream));
    lbk_status st = fetch(lat, ST_SLOTS, 1u << ST_HMAX);
    if (st != LBK_OK)
        return st;
    if (lat->host[ST_BAD] != 0.0 || !isfinite(lat->host[ST_MASS]))
        return fail(LBK_ERR_NONFINITE, "non-finite value in the state after %lld steps",
                    (long long)lat->t);
    if (lat->d.storage == LBK_F16 && lat->host[ST_HMAX] > 0.0) {
        int e;
        frexp(lat->host[ST_HMAX] * ldexp(1.0, lat->scale_exp), &e); // stored max in [2^(e-1), 2^e)
        const int target = 13;                                       // max in [2^12, 2^13)
        if (e > 14 || e < 10) {
            int k = target - e;
            if (lat->scale_exp + k > 100)
                k = 100 - lat->scale_exp;
            if (k != 0) {
                HIP_TRY(launch_rescale(lat->d.storage, s, lat->L.lay, lat->g, k, lat->stream));
                lat->scale_exp += k;
                ++lat->version;
            }
        }
    }
    return LBK_OK;
}

extern "C" {

lbk_status lbk_desc_default(lbk_desc *d)
{
    if (!d)
        return fail(LBK_ERR_INVALID_ARG, "desc is NULL");
    memset(d, 0, sizeof *d);
    d->nx = d->ny = 1;
    d->bc_x = d->bc_y = LBK_BC_PERIODIC;
    d->storage = LBK_F32;
    d->kn_local = 1;
    d->init = 0;
    d->check_every = 100;
    d->tau = 0.8;
    d->rho_in = d->rho_out = d->rho0 = d->rho_ref = 1.0;
    d->slip_b = -1.0;
    d->correlation = LBK_FC_BKC;
    return LBK_OK;
}

lbk_status lbk_workspace_size(const lbk_desc *d, size_t *bytes)
{
    lbk_status s = check_desc(d);
    if (s != LBK_OK)
        return s;
    if (!bytes)
        return fail(LBK_ERR_INVALID_ARG, "bytes is NULL");
    *bytes = layout_of(*d).total;
    return LBK_OK;
}

lbk_status lbk_create(const lbk_desc *d, const float *eps, const float *k, const float *kn0,
                      void *workspace, size_t ws_bytes, void *stream, lbk_lattice **out)
{
    if (!out)
        return fail(LBK_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    lbk_status s = check_desc(d);
    if (s != LBK_OK)
        return s;
    if (!eps || !k)
        return fail(LBK_ERR_INVALID_ARG, "eps and k are required");
    if (!workspace || ((uintptr_t)workspace & 255u))
        return fail(LBK_ERR_INVALID_ARG, "workspace must be non-NULL and 256-byte aligned");
    WsLayout L = layout_of(*d);
    if (ws_bytes < L.total)
        return fail(LBK_ERR_OOM, "workspace of %zu bytes < %zu needed", ws_bytes, L.total);
    int dev = -1;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
        return fail(LBK_ERR_DEVICE, "no HIP device");
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(LBK_ERR_DEVICE, "device %s is not gfx950", prop.gcnArchName);

    lbk_lattice *lat = new (std::nothrow) lbk_lattice();
    if (!lat)
        return fail(LBK_ERR_OOM, "host allocation failed");
    lat->d = *d;
    lat->L = L;
    lat->g = Geom{d->nx, d->ny, L.pitch};
    lat->stream = static_cast<hipStream_t>(stream);
    lat->device = dev;
    lat->ws = static_cast<char *>(workspace);
    lat->cur = 0;
    lat->t = 0;
    lat->version = 0;
    lat->scale_exp = d->storage == LBK_F16 ? 20 : 0;
    lat->have_prev = false;
    if (!lat->out.alloc()) {
        delete lat;
        return fail(LBK_ERR_DEVICE, "pinned host allocation failed");
    }
    lat->host = lat->out.sums;
    auto cleanup = [&](lbk_status st) {
        lat->out.release();
        delete lat;
        return st;
    };

    const double nu = (d->tau - 0.5) / 3.0;
    Physics &ph = lat->ph;
    ph.omega = (float)(1.0 / d->tau);
    ph.guo = (float)(1.0 - 0.5 / d->tau);
    ph.gx = (float)d->gx;
    ph.gy = (float)d->gy;
    ph.feps = (float)d->f_eps;
    ph.inv_nu = (float)(1.0 / nu);
    ph.rho_ref = (float)d->rho_ref;
    split(d->rho_in, ph.rin_hi, ph.rin_lo);
    split(d->rho_out, ph.rout_hi, ph.rout_lo);
    ph.kn_local = d->kn_local ? 1 : 0;
    ph.corr = d->correlation;
    ph.slip_nb = (float)(-d->slip_b);
    ph.slip_c = (float)(4.0 - d->slip_b);
    ph.derive();
    lat->plan = tile_plan(&d->nx, &d->ny, 1);
    lat->tiles_lead = tiles_lead(*d, ph, lat->plan);

    char *ws = lat->ws;
    char *med = lat->med();
    const size_t row = (size_t)d->nx * sizeof(float), mrow = L.mlay.row;
    hipStream_t st = lat->stream;
    auto hip_ok = [&](hipError_t e, const char *what) {
        if (e == hipSuccess)
            return true;
        fail(LBK_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
        return false;
    };
    // raw fields into the medium slots (eps, k, kn0), then k -> drag
    if (!hip_ok(hipMemsetAsync(ws, 0, L.total, st), "clear workspace") ||
        !hip_ok(hipMemcpy2DAsync(med, mrow, eps, row, row, d->ny, hipMemcpyDefault, st), "eps") ||
        !hip_ok(hipMemcpy2DAsync(med + L.mlay.slot, mrow, k, row, row, d->ny, hipMemcpyDefault,
                                 st), "k") ||
        (kn0 && !hip_ok(hipMemcpy2DAsync(med + 2 * L.mlay.slot, mrow, kn0, row, row, d->ny,
                                         hipMemcpyDefault, st), "kn0")) ||
        !hip_ok(launch_fields(med, L.mlay, lat->g, nu, lat->partials(), st), "fields kernel"))
        return cleanup(LBK_ERR_DEVICE);
    if ((s = fetch(lat, FLD_SLOTS, 0)) != LBK_OK)
        return cleanup(s);
    if (lat->host[FLD_BAD] != 0.0)
        return cleanup(fail(LBK_ERR_INVALID_ARG,
                            "%.0f field values out of range (need 0<=eps<=1, k>0 or +inf, "
                            "kn0>=0 finite)",
                            lat->host[FLD_BAD]));
    // mean porosity of the pressure columns (for the global permeability)
    lat->eps_b = d->bc_x == LBK_BC_PRESSURE ? lat->host[FLD_EPS] / (2.0 * d->ny) : 0.0;
    if (!hip_ok(launch_init_state(d->storage, lat->state(0), L.lay, lat->g, d->init, d->rho0,
                                  d->rho_in, d->rho_out, lat->s(), st), "init kernel") ||
        !hip_ok(hipStreamSynchronize(st), "sync"))
        return cleanup(LBK_ERR_DEVICE);
    *out = lat;
    return LBK_OK;
}

lbk_status lbk_destroy(lbk_lattice *lat)
{
    if (!lat)
        return LBK_OK;
    lat->out.release();
    delete lat;
    return LBK_OK;
}

lbk_status lbk_step(lbk_lattice *lat, int64_t n)
{
    if (!lat)
        return fail(LBK_ERR_INVALID_ARG, "lattice is NULL");
    if (n < 0)
        return fail(LBK_ERR_INVALID_ARG, "n must be >= 0");
    const lbk_desc &d = lat->d;
    Range range("lbk_step");
    while (n > 0) {
        // checks fall on multiples of check_every in the lattice's own time,
        // so a run resumed from a saved state checks where the original did
        int64_t chunk = n;
        if (d.check_every > 0)
            chunk = std::min(chunk, d.check_every - lat->t % d.check_every);
        lbk_status s = advance(lat, chunk, lat->stream);
        if (s != LBK_OK)
            return s;
        n -= chunk;
        if (d.check_every > 0 && lat->t % d.check_every == 0 && (s = check_state(lat)) != LBK_OK)
            return s;
    }
    return LBK_OK;
}

lbk_status lbk_time(const lbk_lattice *lat, int64_t *t)
{
    if (!lat || !t)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    *t = lat->t;
    return LBK_OK;
}

lbk_status lbk_steps_per_launch(const lbk_lattice *lat, int32_t *steps)
{
    if (!lat || !steps)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    *steps = three_step_pass(lat) ? 3 : (two_step_pass(lat) ? 2 : 1);
    return LBK_OK;
}

lbk_status lbk_tile_steps(const lbk_lattice *lat, int32_t *steps)
{
    if (!lat || !steps)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    *steps = tile_pass(lat) ? lat->plan.steps : 0;
    return LBK_OK;
}

lbk_status lbk_read_macroscopic(lbk_lattice *lat, float *rho, float *ux, float *uy)
{
    if (!lat)
        return fail(LBK_ERR_INVALID_ARG, "lattice is NULL");
    const lbk_desc &d = lat->d;
    HIP_TRY(launch_macro(d.storage, d.bc_x, d.bc_y, lat->state(lat->cur), lat->L.lay,
                         lat->med(), lat->L.mlay, lat->g, lat->ph, lat->s(), lat->inv_s(), rho, ux, uy,
                         lat->stream));
    return LBK_OK;
}

lbk_status lbk_read_populations(lbk_lattice *lat, double *f)
{
    if (!lat || !f)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    HIP_TRY(launch_populations(lat->d.storage, lat->state(lat->cur), lat->L.lay, lat->g,
                               lat->inv_s(), f, lat->stream));
    return LBK_OK;
}

} // extern "C"

bool lbk::has_drive(const lbk_desc &d)
{
    return d.bc_x == LBK_BC_PRESSURE ? d.rho_in != d.rho_out : d.gx != 0.0;
}

double lbk::k_app_of(const lbk_lattice *lat, const double *sums)
{
    const lbk_desc &d = lat->d;
    const double n = (double)d.nx * d.ny, nu = (d.tau - 0.5) / 3.0;
    if (!has_drive(d))
        return NAN;
    if (d.bc_x == LBK_BC_PRESSURE)
        return lat->eps_b * nu * (d.nx - 1) * (sums[MAC_FLUX] / n) /
               ((1.0 / 3.0) * (d.rho_in - d.rho_out));
    return nu * (sums[MAC_UX] / n) / d.gx;
}

lbk_status lbk::macro_sums(lbk_lattice *lat, bool residual, bool mass)
{
    const lbk_desc &d = lat->d;
    char *ws = lat->ws;
    float *uxp = residual ? reinterpret_cast<float *>(ws + lat->L.uxp) : nullptr;
    float *uyp = residual ? reinterpret_cast<float *>(ws + lat->L.uyp) : nullptr;
    HIP_TRY(launch_macro_sums(d.storage, d.bc_x, d.bc_y, lat->state(lat->cur), lat->L.lay,
                              lat->med(), lat->L.mlay, lat->g, lat->ph, lat->s(), lat->inv_s(),
                              uxp, uyp, mass, lat->partials(), lat->stream));
    return fetch(lat, MAC_SLOTS, 0);
}

extern "C" {

lbk_status lbk_apparent_permeability(lbk_lattice *lat, double *k_app)
{
    if (!lat || !k_app)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    if (!has_drive(lat->d))
        return fail(LBK_ERR_INVALID_ARG, "the global permeability needs rho_in != rho_out "
                                         "(pressure drive) or gx != 0");
    lbk_status s = macro_sums(lat, false, false);
    if (s != LBK_OK)
        return s;
    *k_app = k_app_of(lat, lat->host);
    return LBK_OK;
}

lbk_status lbk_diagnostics(lbk_lattice *lat, double *mass, double *flux_x, double *residual)
{
    if (!lat)
        return fail(LBK_ERR_INVALID_ARG, "lattice is NULL");
    lbk_status s = macro_sums(lat, true, mass != nullptr);
    if (s != LBK_OK)
        return s;
    const double flux = lat->host[MAC_FLUX];
    // relative change of the velocity field; a field that is zero now and
    // was zero before has not changed (0), one that fell to zero changed
    // by everything it had (+inf)
    const double du2 = lat->host[MAC_DU2], u2 = lat->host[MAC_U2];
    const double res = !lat->have_prev ? INFINITY
                       : u2 > 0.0      ? sqrt(du2 / u2)
                       : du2 > 0.0     ? INFINITY
                                       : 0.0;
    lat->have_prev = true;
    if (flux_x)
        *flux_x = flux;
    if (residual)
        *residual = res;
    if (mass)
        *mass = lat->host[MAC_MASS];
    return LBK_OK;
}

// Saved state: a 64-byte header (magic, step count, FP16 scale exponent,
// sizes) followed by the current time level (density and deviations).
static const uint64_t kMagic = 0x6c626b7374617465ull; // "lbkstate"

lbk_status lbk_state_size(const lbk_lattice *lat, size_t *bytes)
{
    if (!lat || !bytes)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    *bytes = 64 + lat->L.level_bytes;
    return LBK_OK;
}

lbk_status lbk_save_state(lbk_lattice *lat, void *dst)
{
    if (!lat || !dst)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    size_t bytes;
    lbk_state_size(lat, &bytes);
    int64_t hdr[8] = {(int64_t)kMagic, lat->t, lat->scale_exp, (int64_t)bytes,
                      lat->d.nx,       lat->d.ny, lat->d.storage, 0};
    HIP_TRY(hipStreamSynchronize(lat->stream));
    HIP_TRY(hipMemcpy(dst, hdr, sizeof hdr, hipMemcpyDefault));
    HIP_TRY(hipMemcpyAsync(static_cast<char *>(dst) + 64, lat->state(lat->cur), bytes - 64,
                           hipMemcpyDefault, lat->stream));
    return LBK_OK;
}

lbk_status lbk_load_state(lbk_lattice *lat, const void *src)
{
    if (!lat || !src)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    size_t bytes;
    lbk_state_size(lat, &bytes);
    int64_t hdr[8];
    HIP_TRY(hipStreamSynchronize(lat->stream));
    HIP_TRY(hipMemcpy(hdr, src, sizeof hdr, hipMemcpyDefault));
    if (hdr[0] != (int64_t)kMagic || hdr[3] != (int64_t)bytes || hdr[4] != lat->d.nx ||
        hdr[5] != lat->d.ny || hdr[6] != lat->d.storage)
        return fail(LBK_ERR_INVALID_ARG, "state does not match this lattice");
    HIP_TRY(hipMemcpyAsync(lat->state(lat->cur), static_cast<const char *>(src) + 64,
                           bytes - 64, hipMemcpyDefault, lat->stream));
    lat->t = hdr[1];
    lat->scale_exp = (int)hdr[2];
    ++lat->version;
    lat->have_prev = false;
    return LBK_OK;
}

lbk_status lbk_correction_factor(int32_t correlation, double slip_b, const double *kn,
                                 double *fc, size_t n)
{
    if ((n && (!kn || !fc)))
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    if (correlation < 0 || correlation > 2)
        return fail(LBK_ERR_INVALID_ARG, "correlation must be 0..2 (got %d)", correlation);
    if (!(slip_b <= 0.0) || !isfinite(slip_b))
        return fail(LBK_ERR_INVALID_ARG, "slip_b must be finite and <= 0");
    for (size_t i = 0; i < n; ++i) {
        const double k = kn[i];
        if (!(k >= 0.0) || !isfinite(k))
            return fail(LBK_ERR_INVALID_ARG, "Kn[%zu] = %g is not finite and >= 0", i, k);
        double f = 1.0;
        if (k > 0.0 && correlation == LBK_FC_KLINKENBERG) {
            f = 1.0 + 4.0 * k;
        } else if (k > 0.0 && correlation == LBK_FC_BKC) {
            const double alpha = 1.358 / (1.0 + 0.170 * pow(k, -0.4348));
            f = (1.0 + alpha * k) * (1.0 + 4.0 * k / (1.0 - slip_b * k));
        }
        fc[i] = f;
    }
    return LBK_OK;
}

const char *lbk_last_error(void) { return g_err.c_str(); }

} // extern "C"

// ------------------------------------------------------------ gradients

lbk_status lbk::adj_plan(const lbk_lattice *lat, int64_t n, int64_t c1, int64_t c2,
                         AdjPlan &P)
{
    if (n < 1 || c1 < 1 || c2 < 1 || c2 > c1)
        return fail(LBK_ERR_INVALID_ARG,
                    "need n_steps >= 1 and 1 <= hist_len <= ckpt_every (got %lld, %lld, %lld)",
                    (long long)n, (long long)c1, (long long)c2);
    P = AdjPlan{};
    P.n = n;
    P.c1 = c1;
    P.c2 = c2;
    P.two_level = c2 < c1 && c2 < n;
    P.k1 = (n + c1 - 1) / c1;
    P.k2 = P.two_level ? (c1 + c2 - 1) / c2 : 0;
    P.hlen = P.two_level ? c2 : (c1 < n ? c1 : n);
    const int64_t rows = lat->d.ny;
    P.level_bytes = lat->L.level_bytes;
    P.hist_bytes = (size_t)rows * 3 * lat->L.pitch * 4;
    P.lam_bytes = (size_t)rows * 9 * lat->L.pitch * 4;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    P.outer = take(P.level_bytes * (size_t)P.k1);
    P.rec = take(2 * P.level_bytes);
    P.hist = take(P.hist_bytes * (size_t)(P.hlen + 1));
    P.lam = take(2 * P.lam_bytes);
    P.grad = take((size_t)rows * lat->L.pitch * 8);
    P.seg = take((size_t)rows * lat->L.pitch * 4);
    P.grad2 = take((size_t)rows * lat->L.pitch * 8);
    P.seg2 = take((size_t)rows * lat->L.pitch * 4);
    P.inner_seg = P.level_bytes * (size_t)P.k2;
    P.inner = take(P.inner_seg);
    P.keep = P.two_level ? 1 : 0;
    P.total = o;
    return LBK_OK;
}

void lbk::adj_keep(AdjPlan &P, size_t ws_bytes)
{
    if (!P.two_level || ws_bytes < P.total)
        return;
    const size_t extra = (ws_bytes - P.total) / P.inner_seg;
    P.keep = std::min<int64_t>(P.k1, 1 + (int64_t)std::min<size_t>(extra, (size_t)P.k1));
    P.total += (size_t)(P.keep - 1) * P.inner_seg;
}

int64_t lbk::adj_rebuild_steps(const AdjPlan &P)
{
    if (!P.two_level)
        return 0;
    int64_t steps = 0;
    for (int64_t k = 0; k < P.k1 - P.keep; ++k) {
        const int64_t len = std::min(P.c1, P.n - k * P.c1);
        steps += ((len + P.c2 - 1) / P.c2 - 1) * P.c2; // sweep to the last inner start
    }
    return steps;
}

double lbk::objective_weights(const lbk_lattice *lat, int objective, const double *sums,
                              double &a1, double &a2, int &outlet)
{
    const lbk_desc &d = lat->d;
    const double nodes = (double)d.nx * d.ny, nu = (d.tau - 0.5) / 3.0;
    if (objective == LBK_OBJ_OUTLET_FLUX) {
        a1 = 1.0;
        a2 = 0.0;
        outlet = 1;
        return sums[MAC_QOUT];
    }
    outlet = 0;
    if (d.bc_x == LBK_BC_PRESSURE) {
        a1 = lat->eps_b * nu * (d.nx - 1) / ((1.0 / 3.0) * (d.rho_in - d.rho_out) * nodes);
        a2 = 0.0;
        return a1 * sums[MAC_FLUX];
    }
    a1 = 0.0;
    a2 = nu / (d.gx * nodes);
    return a2 * sums[MAC_UX];
}

lbk_status lbk::check_objective(const lbk_lattice *lat, int objective)
{
    const lbk_desc &d = lat->d;
    if (objective != LBK_OBJ_PERMEABILITY && objective != LBK_OBJ_OUTLET_FLUX)
        return fail(LBK_ERR_INVALID_ARG, "unknown objective %d", objective);
    if (objective == LBK_OBJ_PERMEABILITY && !has_drive(d))
        return fail(LBK_ERR_INVALID_ARG, "the global permeability needs rho_in != rho_out "
                                         "(pressure drive) or gx != 0");
    return LBK_OK;
}

extern "C" lbk_status lbk_adjoint_workspace_size(const lbk_lattice *lat, int64_t n_steps,
                                                 int64_t ckpt_every, int64_t hist_len,
                                                 size_t *bytes)
{
    if (!lat || !bytes)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    AdjPlan P;
    lbk_status s = adj_plan(lat, n_steps, ckpt_every, hist_len, P);
    if (s != LBK_OK)
        return s;
    *bytes = P.total;
    return LBK_OK;
}

extern "C" lbk_status lbk_adjoint_plan(const lbk_lattice *lat, int64_t n_steps,
                                       int64_t ckpt_every, size_t budget_bytes,
                                       int64_t *hist_len, size_t *bytes)
{
    if (!lat || !hist_len)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    if (n_steps < 1 || ckpt_every < 1)
        return fail(LBK_ERR_INVALID_ARG, "need n_steps >= 1 and ckpt_every >= 1");
    const int64_t c1 = std::min(ckpt_every, n_steps);
    // fewest sweeps spent rebuilding inner checkpoints; among equals, the
    // longest history (fewest segments)
    int64_t prev = -1, best_h = -1, best_cost = -1;
    size_t best_bytes = 0;
    for (int64_t m = 1; m <= c1; ++m) {
        const int64_t h = (c1 + m - 1) / m;
        if (h == prev)
            continue;
        prev = h;
        AdjPlan P;
        lbk_status s = adj_plan(lat, n_steps, c1, h, P);
        if (s != LBK_OK)
            return s;
        if (P.total > budget_bytes)
            continue;
        adj_keep(P, budget_bytes);
        const int64_t cost = adj_rebuild_steps(P);
        if (best_h < 0 || cost < best_cost) {
            best_h = h;
            best_cost = cost;
            best_bytes = P.total;
        }
        if (cost == 0)
            break;
    }
    if (best_h < 0)
        return fail(LBK_ERR_OOM, "no checkpoint plan for %lld steps every %lld fits in %zu bytes",
                    (long long)n_steps, (long long)c1, budget_bytes);
    *hist_len = best_h;
    if (bytes)
        *bytes = best_bytes;
    return LBK_OK;
}

// n >= 1 steps from src to dst (nullptr: to one of the levels lv) by way of the
// levels lv, one of which src may be; src becomes where the state is then.
static hipError_t lead(const lbk_lattice *lat, char *&src, int64_t n, char *const (&lv)[2],
                       char *dst, hipStream_t st)
{
    while (n > 0) {
        const Pass p = next_pass(lat, n);
        char *to = dst && p.steps == n ? dst : lv[src == lv[0] ? 1 : 0];
        const hipError_t e = launch_pass(lat, p, src, to, nullptr, 0, st);
        if (e != hipSuccess)
            return e;
        src = to;
        n -= p.steps;
    }
    return hipSuccess;
}

extern "C" lbk_status lbk_adjoint_forward(lbk_lattice *lat, int objective, int64_t n_steps,
                                          int64_t ckpt_every, int64_t hist_len, void *ws,
                                          size_t ws_bytes, double *J)
{
    if (!lat || !ws || !J)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    Range range("adjoint forward");
    lbk_status s0 = check_objective(lat, objective);
    if (s0 != LBK_OK)
        return s0;
    if ((uintptr_t)ws & 255u)
        return fail(LBK_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
    AdjPlan P;
    lbk_status s = adj_plan(lat, n_steps, ckpt_every, hist_len, P);
    if (s != LBK_OK)
        return s;
    if (ws_bytes < P.total)
        return fail(LBK_ERR_OOM, "adjoint workspace of %zu bytes < %zu needed", ws_bytes,
                    P.total);
    adj_keep(P, ws_bytes);
    lat->adj.valid = false;
    char *w = static_cast<char *>(ws);
    hipStream_t st = lat->stream;
    P.t0 = lat->t;
    // Segment by segment from checkpoint to checkpoint: the last pass before a
    // checkpoint writes it, the first one after it reads it, so only the first
    // is a copy (67 us a checkpoint of 2048 x 2048).  The last `keep` segments
    // are reversed first: their inner checkpoints are kept now rather than
    // recomputed in the backward pass.
    char *lv[2] = {lat->state(0), lat->state(1)};
    char *src = w + P.outer;
    HIP_TRY(hipMemcpyAsync(src, lat->state(lat->cur), P.level_bytes, hipMemcpyDeviceToDevice, st));
    for (int64_t t = 0; t < P.n;) {
        const int64_t k = t / P.c1, kept = k - (P.k1 - P.keep);
        const int64_t run = P.two_level && kept >= 0 ? P.c2 : P.c1;
        const int64_t end = std::min(std::min(P.n, (k + 1) * P.c1), t + run);
        char *dst = nullptr;
        if (end < P.n && end == (k + 1) * P.c1)
            dst = w + P.outer + (size_t)(k + 1) * P.level_bytes;
        else if (end < P.n)
            dst = w + P.inner + (size_t)kept * P.inner_seg +
                  (size_t)((end - k * P.c1) / P.c2) * P.level_bytes;
        HIP_TRY(lead(lat, src, end - t, lv, dst, st));
        t = end;
    }
    lat->cur = src == lv[1];
    lat->t += P.n;
    ++lat->version;
    if ((s = macro_sums(lat, false, false)) != LBK_OK)
        return s;
    P.objective = objective;
    *J = objective_weights(lat, objective, lat->host, P.a1, P.a2, P.outlet);
    P.ws = ws;
    P.valid = true;
    lat->adj = P;
    return LBK_OK;
}

// The tile of a reverse pass (launch_adjoint_tile) of `steps` steps at most:
// while every tile has a CU of its own a pass costs its launch and its chain
// of steps, so the most steps whose tiles number at most the device's 256 CUs
// (16 waves of one row, then of two); on larger lattices the bytes of the tiles
// count, and two workgroups a CU, one loading while the other computes.  us a step:
//   384 x 256    2.9 (16, 1, 4)  3.3 (8, 2, 4)   3.3 (16, 1, 3)
//   333 x 100    2.4 (16, 1, 6)  2.6 (16, 1, 5)  2.9 (16, 1, 4)
//   1024 x 512   8.5 (16, 2, 5)  8.9 (8, 2, 3)   10.1 (16, 1, 3)
//   2048 x 512   14.5 (8, 2, 3)  15.3 (16, 2, 5) 17 (12, 1, 3)
//   2048 x 2048  49.3 (8, 2, 3)  51.2 (16, 2, 5) 57.5 (12, 1, 3)
static TilePlan rev_tile_plan(const lbk_lattice *lat)
{
    const bool one_row = rev_model(lat->ph) == REV_FORCH;
    const TilePlan plans[] = {{{16, 1}, 6}, {{16, 1}, 4}, {{16, 2}, 5}};
    for (const TilePlan &p : plans) {
        const int64_t own_x = 64 - 2 * p.steps, own_y = p.tile.waves * p.tile.rows - 2 * p.steps;
        const int64_t tiles = ((lat->d.nx + own_x - 1) / own_x) * ((lat->d.ny + own_y - 1) / own_y);
        if (tiles <= 256 && !(one_row && p.tile.rows > 1))
            return p;
    }
    return one_row ? TilePlan{{12, 1}, 3} : TilePlan{{8, 2}, 3};
}

// Whether the automatic mode's reverse steps take tile passes of that plan:
// everywhere but where the rows its bands have room for are many times the
// lattice's and the tiles too many to run side by side; the lattice's own rows
// are then read once instead.  us a step, tile passes against single steps or
// pairs: 16384 x 1 4.8 / 5.6, 65536 x 1 8.5 / 6.8 and 524288 x 1 45 / 13,
// 32768 x 4 6.6 / 7.3, 131072 x 4 14.2 / 12.8 and 524288 x 4 56 / 45,
// 65536 x 5 8.8 / 9.6, 262144 x 5 30 / 30 and 524288 x 5 68 / 55,
// 262144 x 11 69 / 79 and 524288 x 11 129 / 113, 524288 x 7 72 / 78.  With the
// Forchheimer term, whose updates cost more, a quarter of unused room is too much
// (a backward pass, us a step: 131072 x 3 24 / 21, 524288 x 7 154 / 135,
// 524288 x 13 258 / 206), between walls a sixth (524288 x 5 129 / 114, 524288 x 7
// 216 / 124).
static bool rev_tiles_lead(const lbk_lattice *lat, const TilePlan &p)
{
    const lbk_desc &d = lat->d;
    const int own_y = p.tile.waves * p.tile.rows - 2 * p.steps;
    const int64_t bands = tile_bands(d.ny, p), tiles = tile_strips(d.nx, p) * bands;
    const int64_t nodes = (int64_t)d.nx * d.ny;
    const double room = (double)bands * own_y / d.ny;
    if (lat->ph.feps != 0.0f)
        return room < (d.bc_y == LBK_BC_WALL ? 1.15 : 1.25) || tiles <= (room < 2.0 ? 2000 : 600);
    if (room >= 2.5)
        return tiles <= 600;
    if (room >= 2.0)
        return nodes < (int64_t)1 << 21;
    return room <= 1.6 || nodes < (int64_t)1 << 22;
}

extern "C" lbk_status lbk_adjoint_backward(lbk_lattice *lat, void *ws, size_t ws_bytes,
                                           float *dJ_dlnk, float *dJ_dlnkn0)
{
    if (!lat || !ws || !dJ_dlnk)
        return fail(LBK_ERR_INVALID_ARG, "NULL argument");
    AdjPlan &P = lat->adj;
    if (!P.valid || P.ws != ws || ws_bytes < P.total)
        return fail(LBK_ERR_INVALID_ARG, "no matching lbk_adjoint_forward for this workspace");
    if (lat->t != P.t0 + P.n)
        return fail(LBK_ERR_INVALID_ARG, "the lattice moved since lbk_adjoint_forward");
    const lbk_desc &d = lat->d;
    hipStream_t st = lat->stream;
    char *w = static_cast<char *>(ws);
    auto level = [&](size_t off, int64_t k) { return w + off + (size_t)k * P.level_bytes; };
    auto histp = [&](int64_t k) {
        return reinterpret_cast<float *>(w + P.hist + (size_t)k * P.hist_bytes);
    };
    float *lam[2] = {reinterpret_cast<float *>(w + P.lam),
                     reinterpret_cast<float *>(w + P.lam + P.lam_bytes)};
    double *grad = reinterpret_cast<double *>(w + P.grad);
    float *seg = reinterpret_cast<float *>(w + P.seg);
    const bool kn = dJ_dlnkn0 != nullptr;
    double *grad2 = reinterpret_cast<double *>(w + P.grad2);
    float *seg2 = kn ? reinterpret_cast<float *>(w + P.seg2) : nullptr;
    char *rec[2] = {level(P.rec, 0), level(P.rec, 1)};
    // rebuilt inner checkpoints (no history) and recorded segments take
    // lbk_step's passes, the reverse steps tile passes or pairs likewise
    const TilePlan rev = rev_tile_plan(lat);
    const bool tile = d.pass_mode == LBK_PASS_AUTO && d.band == 0 && rev_tiles_lead(lat, rev);
    const bool two = two_step_pass(lat);
    const float a1 = (float)P.a1, a2 = (float)P.a2;

    HIP_TRY(hipMemsetAsync(grad, 0, (size_t)d.ny * lat->L.pitch * 8, st));
    HIP_TRY(hipMemsetAsync(seg, 0, (size_t)d.ny * lat->L.pitch * 4, st));
    if (kn) {
        HIP_TRY(hipMemsetAsync(grad2, 0, (size_t)d.ny * lat->L.pitch * 8, st));
        HIP_TRY(hipMemsetAsync(seg2, 0, (size_t)d.ny * lat->L.pitch * 4, st));
    }
    // read-out of J at step n: linearisation point of the pull of S_n
    HIP_TRY(launch_pass(lat, Pass{PASS_ONE, 1, {}}, lat->state(lat->cur), rec[0], histp(0),
                        P.hist_bytes, st));
    HIP_TRY(launch_adjoint(d.bc_x, d.bc_y, nullptr, lam[0], histp(0), lat->med(), lat->L.mlay,
                           seg, seg2, lat->g, lat->ph, 1, a1, a2, P.outlet, st));
    int cur = 0;
    for (int64_t k = P.k1 - 1; k >= 0; --k) {
        const int64_t a = k * P.c1, b = std::min(P.n, a + P.c1);
        int64_t nseg = 1;
        // inner checkpoints of this segment: kept by the forward pass, or
        // rebuilt into the first kept segment's slots (free by now, since
        // the kept segments are the last ones and reversed first; its own are
        // gone once a pass has done so)
        const int64_t kept = k - (P.k1 - P.keep);
        const size_t inner = P.inner + (size_t)(kept > 0 ? kept : 0) * P.inner_seg;
        if (P.two_level && (kept > 0 || (kept == 0 && !P.reused))) {
            nseg = (b - a + P.c2 - 1) / P.c2;
        } else if (P.two_level) {
            P.reused = true;
            // rebuild the inner checkpoints of this outer segment (the first
            // is the outer one; the last inner segment needs no further state)
            Range range("adjoint rebuild");
            char *src = level(P.outer, k);
            nseg = (b - a + P.c2 - 1) / P.c2;
            for (int64_t j = 1; j < nseg; ++j)
                HIP_TRY(lead(lat, src, P.c2, rec, level(inner, j), st));
        }
        for (int64_t j = nseg - 1; j >= 0; --j) {
            const int64_t a2s = P.two_level ? a + j * P.c2 : a;
            const int64_t b2s = P.two_level ? std::min(b, a2s + P.c2) : b;
            const char *src = j > 0 ? level(inner, j) : level(P.outer, k);
            // recompute the segment, recording each step's linearisation point
            int r = 0;
            {
                Range range("adjoint recompute");
                for (int64_t t = a2s; t < b2s;) {
                    const char *from = t == a2s ? src : rec[r];
                    const Pass p = next_pass(lat, b2s - t);
                    HIP_TRY(launch_pass(lat, p, from, rec[r ^ 1], histp(t - a2s + 1),
                                        P.hist_bytes, st));
                    t += p.steps;
                    r ^= 1;
                }
            }
            Range range("adjoint reverse");
            for (int64_t t = b2s; t > a2s;) {
                if (tile && t - 1 > a2s) {
                    const int n = (int)std::min<int64_t>(rev.steps, t - a2s);
                    HIP_TRY(launch_adjoint_tile(d.bc_x, d.bc_y, lam[cur], lam[cur ^ 1],
                                                histp(t - a2s), P.hist_bytes, lat->med(),
                                                lat->L.mlay, seg, seg2, lat->g, lat->ph, rev.tile,
                                                n, st));
                    t -= n;
                } else if (two && t - 1 > a2s) {
                    HIP_TRY(launch_adjoint2(d.bc_x, d.bc_y, lam[cur], lam[cur ^ 1],
                                            histp(t - a2s), histp(t - 1 - a2s), lat->med(),
                                            lat->L.mlay, seg, seg2, lat->g, lat->ph,
                                            rev_band(d), st));
                    t -= 2;
                } else {
                    HIP_TRY(launch_adjoint(d.bc_x, d.bc_y, lam[cur], lam[cur ^ 1],
                                           histp(t - a2s), lat->med(), lat->L.mlay, seg, seg2,
                                           lat->g, lat->ph, 0, a1, a2, P.outlet, st));
                    --t;
                }
                cur ^= 1;
            }
            HIP_TRY(launch_grad_fold(seg, grad, lat->g, st));
            if (kn)
                HIP_TRY(launch_grad_fold(seg2, grad2, lat->g, st));
        }
    }
    HIP_TRY(launch_grad_out(grad, dJ_dlnk, lat->g, st));
    if (kn)
        HIP_TRY(launch_grad_out(grad2, dJ_dlnkn0, lat->g, st));
    return LBK_OK;
}
