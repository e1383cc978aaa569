// lbk_adjoint.hip -- reverse-mode (discrete adjoint) sweep of the Klinkenberg
// lattice Boltzmann step, for gradients of a scalar read-out J of the state
// after N steps with respect to the log-permeability field ln k(x) and,
// optionally, the log base-Knudsen field ln kn0(x).
//
// The forward step n is  f^n = B(P(S_{n-1})),  S_n = C(f^n; ln k)  with P the
// pull (a permutation, bounce-back included), B the pressure-column override
// and C the per-node BGK/Guo collide (Eqs. 12, 14, 15, 17, 8, 3, 6-7).
// Given mu_n = dJ/dS_n, one reverse step computes
//   lam_f(x) = (dC/df)(x)^T mu_n(x)          (local, 9 -> 9)
//   grad(x) += (dC/d ln k)(x)^T mu_n(x)
//   mu_{n-1} = P^T B^T lam_f                 (the push: each source slot of
//                                             S_{n-1} has exactly one reader)
// C depends on f only through rho = sum f and j = sum f e, so
//   lam_f_k = (1 - omega) mu_k + G_rho + e_k . G_j
// with G_rho, G_j the total derivatives of Psi = sum_i mu_i (omega f^eq_i + F_i)
// through u(rho, j, ln k), F = -A u - B |u| u + eps G (Eq. 2; B = 0 without
// the Forchheimer term), A = eps nu / (k f_c(Kn)) and
// Kn = kn0 rho_ref / rho (so dA/d ln k = -A and dA/d ln kn0 =
// -A Kn f_c'(Kn) / f_c, which varies with rho from step to step and needs a
// gradient plane of its own); the linearisation point (rho, j) of every step is
// the history written by the recomputing forward sweep.  The read-out of J
// (global permeability or outlet flux) is the same local map with Psi the
// node's share of J and no (1 - omega) mu term.
//
// Pressure columns: the boundary node's populations are a function of its
// neighbour's (non-equilibrium extrapolation), so the thread of the
// neighbouring column also carries the boundary node's adjoint and adds
// B^T to its own; boundary threads only clear the adjoint slots whose
// forward values were discarded.
//
// Layouts (row blocks, `pitch` elements per slot, FP32): adjoint state
// [y][9][pitch]; history [y][pitch][3] = (rho, jx, jy) per node; gradient
// [y][pitch] (one plane per parameter field) accumulated in FP32 over one
// recomputed segment (at most a few hundred steps) and folded into an FP64
// total at the segment's end.  The
// adjoint state and the history are each read once, so they stream
// nontemporally.  With the Forchheimer term on, the quadratic velocity solve
// of Eq. 2 is differentiated as well (template flag FC; without it the
// Darcy path alone is compiled).
#include "lbk_adjoint_dev.h"

namespace lbk {

// One reverse step (or, with terminal != 0, the read-out of J).
//   mu_in  [y][9][pitch]  adjoint of S_n (ignored when terminal)
//   mu_out [y][9][pitch]  adjoint of S_{n-1} (written by push)
//   hist   [y][pitch][3]  (rho, jx, jy) of step n's post-stream populations
//   grad   [y][pitch]     FP32, accumulates d J / d ln k over a segment
//   grad2  [y][pitch]     FP32, d J / d ln kn0 likewise (KN only)
// Objective: J = sum_x a1(x) rho u_x + a2 u_x with a1(x) = a1 (all nodes,
// or only column nx-1 when outlet != 0) and a2 uniform.
template <int BCX, int BCY, bool KN, bool FC>
__device__ __forceinline__ void adjoint_node(const float *mu_in, float *mu_out, const float *hist,
                                             const char *med, const MLayout &mlay, float *grad,
                                             float *grad2, const Geom &g, const Physics &ph,
                                             int terminal, float a1, float a2, int outlet, int y,
                                             uint32_t x)
{
    const uint32_t nx = (uint32_t)g.nx;
    const uint64_t lrow = 9ull * g.pitch * 4, hrow = 3ull * g.pitch * 4;
    const uint32_t slot = (uint32_t)g.pitch * 4; // bytes per FP32 slot
    const Rsrc hr = rsrc_row(hist, hrow, y);
    const Rsrc mr = make_rsrc(med + (uint64_t)y * mlay.row, (uint32_t)mlay.row);
    const Rsrc lin = rsrc_row(mu_in, lrow, y);
    float *grow_p = grad + (uint64_t)y * g.pitch;
    float *grow_k = KN ? grad2 + (uint64_t)y * g.pitch : nullptr;

    auto load_node = [&](uint32_t xx) {
        float h[3];
        ld_hist<kNT>(hr, xx * 12, h);
        return node_fwd<FC>(ph, h[0], h[1], h[2], ld_f32(mr, xx * 4, 0),
                            ld_f32(mr, xx * 4, mlay.slot), ld_f32(mr, xx * 4, 2 * mlay.slot));
    };
    auto node_adj = [&](const NodeFwd &n, uint32_t xx, float (&lf)[9]) {
        if (terminal) {
            const float a = (!outlet || xx == nx - 1) ? a1 : 0.0f;
            return readout_adj<FC>(ph, n, a, a2, lf);
        }
        float mu[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            mu[i] = ld_f32_nt(lin, xx * 4, i * slot);
        return collide_adj<FC>(ph, n, mu, lf);
    };
    // each gradient entry has exactly one writer per launch
    auto add_grad = [&](uint32_t xx, float v, float vk) {
        grow_p[xx] += v;
        if (KN)
            grow_k[xx] += vk;
    };

    // rows the push writes into: source of direction i is (x - e_ix, y - e_iy)
    int ym = y - 1, yp = y + 1;
    bool wym = false, wyp = false;
    if (BCY == BC_PERIODIC) {
        ym = (y == 0) ? g.ny - 1 : ym;
        yp = (y == g.ny - 1) ? 0 : yp;
    } else {
        // scalar wall flags (the row is the workgroup's): keeps the selects
        // of the pushed rows' buffer resources scalar
        wym = __builtin_amdgcn_readfirstlane(y == 0 ? 1 : 0) != 0;
        wyp = __builtin_amdgcn_readfirstlane(y == g.ny - 1 ? 1 : 0) != 0;
        ym = wym ? y : ym;
        yp = wyp ? y : yp;
    }
    const Rsrc orow[3] = {rsrc_row(mu_out, lrow, ym), rsrc_row(mu_out, lrow, y),
                          rsrc_row(mu_out, lrow, yp)};

    float lf[9];
    const bool bnode = (BCX == BC_PRESSURE) && (x == 0 || x == nx - 1);
    if (bnode) {
        // forward values pulled into this node were discarded: clear the
        // slots it would push to, and the slots whose destination lies
        // outside the lattice
#pragma unroll
        for (int i = 0; i < 9; ++i)
            lf[i] = 0.0f;
    } else {
        const NodeFwd n = load_node(x);
        const Grads G = node_adj(n, x, lf);
        float gl = G.lnk, gk = G.lnkn;
        if (BCX == BC_PRESSURE && (x == 1 || x == nx - 2)) {
            // carry the boundary node next door (x = 0 or nx-1)
            const uint32_t xb = (x == 1) ? 0 : nx - 1;
            {
                const NodeFwd b = load_node(xb);
                float lb[9];
                const Grads Gb = node_adj(b, xb, lb);
                add_grad(xb, Gb.lnk, Gb.lnkn);
                const float2 gn = nee_adj<FC>(ph, n, b.rho, b.ie, lb, lf);
                gl += gn.x;
                gk += gn.y;
            }
            if (nx == 3) {
                // x = 1 is the neighbour of both columns: the outlet too
                const NodeFwd b = load_node(2);
                float lb[9];
                const Grads Gb = node_adj(b, 2, lb);
                add_grad(2, Gb.lnk, Gb.lnkn);
                const float2 gn = nee_adj<FC>(ph, n, b.rho, b.ie, lb, lf);
                gl += gn.x;
                gk += gn.y;
            }
        }
        add_grad(x, gl, gk);
    }

    // push: mu_out[i](x - e_i) = lf_i, bounce-back at walls.  The pushed
    // stores keep the default cache policy: a wave's shifted store covers
    // parts of two cache lines whose other parts the neighbouring wave
    // writes, and L2 merges them (3% less gradient time than streaming
    // stores on the 8192^2 shale)
    uint32_t xm = x - 1, xp = x + 1;
    bool wxm = false, wxp = false;
    if (BCX == BC_PERIODIC) {
        xm = (x == 0) ? nx - 1 : xm;
        xp = (x == nx - 1) ? 0 : xp;
    } else if (BCX == BC_WALL) {
        wxm = (x == 0);
        wxp = (x == nx - 1);
    } else {
        wxm = (x == 0); // pressure: nothing beyond the end columns
        wxp = (x == nx - 1);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int ex = ex_of(i), ey = ey_of(i);
        const bool wall_y = (ey == 1 && wym) || (ey == -1 && wyp); // uniform
        const bool out_x = (ex == 1 && wxm) || (ex == -1 && wxp);  // per lane
        const int ry = ey == 1 ? 0 : (ey == -1 ? 2 : 1);
        const uint32_t tx = ex == 1 ? xm : (ex == -1 ? xp : x);
        if (BCX == BC_PRESSURE) {
            if (out_x)
                continue; // source outside the lattice
            if (wall_y)
                st_f32(orow[1], x * 4, opp_of(i) * slot, lf[i], false);
            else
                st_f32(orow[ry], tx * 4, i * slot, lf[i], false);
        } else {
            if (wall_y || out_x)
                st_f32(orow[1], x * 4, opp_of(i) * slot, lf[i], false);
            else
                st_f32(orow[ry], tx * 4, i * slot, lf[i], false);
        }
    }
    if (BCX == BC_PRESSURE && bnode) {
        // slots of this node whose forward destination lies outside
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const int ex = ex_of(i);
            if ((x == 0 && ex == -1) || (x == nx - 1 && ex == 1))
                st_f32(orow[1], x * 4, i * slot, 0.0f, false);
        }
    }
}

template <int BCX, int BCY, bool KN, bool FC>
__global__ __launch_bounds__(256) void adjoint_kernel(const float *mu_in, float *mu_out,
                                                       const float *hist, const char *med,
                                                       MLayout mlay, float *grad, float *grad2,
                                                       Geom g, Physics ph, int terminal,
                                                       float a1, float a2, int outlet, int bpr)
{
    const int L = xcd_remap_a(blockIdx.x, gridDim.x);
    const int y = L / bpr;
    const uint32_t x = (uint32_t)(L - y * bpr) * 256 + threadIdx.x;
    if (x >= (uint32_t)g.nx)
        return;
    adjoint_node<BCX, BCY, KN, FC>(mu_in, mu_out, hist, med, mlay, grad, grad2, g, ph, terminal, a1,
                               a2, outlet, y, x);
}

// ------------------------------------------------ two reverse steps per pass
//
// adjoint2_kernel takes mu_n to mu_{n-2} in one pass, bitwise what two
// adjoint_kernel launches through mu_{n-1} give, with mu_{n-1} never
// leaving registers.  In gather form a reverse step reads
//   mu_{n-1}(x, j) = lam_f_j(x + e_j),
// lam_f_{opp j}(x) where x + e_j lies beyond a wall (bounce-back), and 0
// where x + e_j lies beyond a pressure column; lam_f itself is local to its
// node (plus, at the column next to a pressure column, that column's
// contribution through the non-equilibrium extrapolation).  As in the
// forward two-step pass, a wave holds a strip of 64 columns (60 of its own
// and two halo columns on either side, x neighbours through DPP lane shifts)
// and marches down a band of rows; lam_f of step n, mu_{n-1} and lam_f of
// step n-1 of the rows around the current one stay in registers, and each
// gradient entry collects both steps' terms before it is written once.
namespace {

// A row's inputs at this lane's column, in two parts loaded at different
// times: what the reverse of step n needs (mu_n, the history of step n and
// the medium) and what the reverse of step n - 1 adds (the history of step
// n - 1 and the medium again).  Each part is loaded straight into the
// registers where it is used, and nothing loaded is copied to another
// register, so no load is waited for before its use.
struct RowA {
    float mu[9], h1[3], md[3];
};
struct RowB {
    float h0[3], md[3];
};
// After the reverse of step n, and after that of step n - 1: lam_f and the
// gradient terms.
struct AMid {
    float lf[9], gl, gk;
};

} // namespace

// Two reverse steps: mu_in = mu_n -> mu_out = mu_{n-2}, hist1 / hist0 the
// histories of steps n and n - 1, grad / grad2 as in adjoint_node.  Rows
// are marched in bands of `band`; a block holds four strips.
// The pass of one wave: strip `strip` of band `bnd` of one lattice.
template <int BCX, int BCY, bool KN, bool FC>
__device__ __forceinline__ void adjoint2_strip(
    const float *__restrict__ mu_in, float *__restrict__ mu_out, const float *__restrict__ hist1,
    const float *__restrict__ hist0, const char *__restrict__ med, const MLayout &mlay,
    float *__restrict__ grad, float *__restrict__ grad2, const Geom &g, const Physics &ph,
    int band, int bnd, int strip)
{
    const int lane = (int)(threadIdx.x & 63);
    const int nx = g.nx, ny = g.ny;
    const int nstrips = (nx + kStrip2 - 1) / kStrip2;
    if (strip >= nstrips)
        return; // the whole wave
    // Strip s owns columns [c0, c1).  With pressure columns the last strip
    // starts at most at nx - 4: the column next to the outlet then never
    // sits at lane 63 of a strip that owns the column two to its left, whose
    // result would need the outlet column's values from beyond the wave.
    int c0 = strip * kStrip2, c1 = min(c0 + kStrip2, nx);
    if (BCX == BC_PRESSURE) {
        const int cl = max(0, min(kStrip2 * (nstrips - 1), nx - 4));
        if (strip == nstrips - 1)
            c0 = cl;
        else if (strip == nstrips - 2)
            c1 = cl;
    }
    const int xr = c0 - 2 + lane;
    const bool owned = xr >= c0 && xr < c1;
    ALanes ln;
    if (BCX == BC_PERIODIC)
        ln.x = (uint32_t)(((xr % nx) + nx) % nx);
    else
        ln.x = (uint32_t)(xr < 0 ? 0 : (xr >= nx ? nx - 1 : xr)); // beyond: unused copies
    ln.wxm = BCX == BC_WALL && xr == 0;
    ln.wxp = BCX == BC_WALL && xr == nx - 1;
    ln.first = BCX == BC_PRESSURE && xr == 0;
    ln.last = BCX == BC_PRESSURE && xr == nx - 1;
    ln.cl = BCX == BC_PRESSURE && nx >= 3 && xr == 1;
    ln.cr = BCX == BC_PRESSURE && nx >= 3 && xr == nx - 2;
    ln.has_b = BCX == BC_PRESSURE && (strip == 0 || strip >= nstrips - 2);
    ln.bgrad = nx >= 3;
    const int y0 = bnd * band, y1 = min(y0 + band, ny);
    auto exists = [&](int y) { return BCY == BC_PERIODIC || (y >= 0 && y < ny); };
    auto wrap = [&](int y) { return BCY == BC_PERIODIC ? ((y % ny) + ny) % ny : y; };
    // a row that always exists (beyond a wall: the nearest row, loaded but
    // never used, since the gather bounces back there)
    auto held = [&](int y) {
        return BCY == BC_PERIODIC ? wrap(y) : (y < 0 ? 0 : (y >= ny ? ny - 1 : y));
    };
    auto wall_lo = [&](int y) { return BCY == BC_WALL && y == 0; };
    auto wall_hi = [&](int y) { return BCY == BC_WALL && y == ny - 1; };
    // Unconditional stores (see sweep2_kernel): a lane that does not own
    // its column repeats the store of the wave's first owning lane.
    const uint64_t om = __builtin_amdgcn_ballot_w64(owned);
    if (om == 0)
        return;
    const int q = (int)__builtin_ctzll(om);
    const uint32_t xq = (uint32_t)__builtin_amdgcn_readlane((int)ln.x, q);
    const uint32_t xst = owned ? ln.x : xq;
    auto same = [&](float v) {
        const float vq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), q));
        return owned ? v : vq;
    };

    const uint64_t lrow = 9ull * g.pitch * 4, hrow = 3ull * g.pitch * 4;
    const uint64_t grow = (uint64_t)g.pitch * 4;
    const uint32_t slot = (uint32_t)g.pitch * 4;
    const uint32_t xo = ln.x * 4;
    // Loads keep the default cache policy: a strip's first and last cache
    // lines are shared with the neighbouring strips, which read them about
    // the same time.
    // The march loads ahead of its needs; rows past them (first parts
    // beyond y1 + 1, second parts beyond y1: the last output row's) get
    // empty buffer resources, so their loads return 0 without touching
    // memory.
    auto row_of = [&](const void *base, uint64_t bytes, int yh, bool live) {
        return make_rsrc(static_cast<const char *>(base) + (uint64_t)yh * bytes,
                         live ? (uint32_t)bytes : 0u);
    };
    auto load_a = [&](int y, RowA &r) {
        const int yh = held(y);
        const bool live = y <= y1 + 1;
        const Rsrc lr = row_of(mu_in, lrow, yh, live);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            r.mu[i] = ld_f32(lr, xo, i * slot);
        const Rsrc hr = row_of(hist1, hrow, yh, live), mr = row_of(med, mlay.row, yh, live);
        ld_hist<0>(hr, ln.x * 12, r.h1);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            r.md[k] = ld_f32(mr, xo, k * mlay.slot);
    };
    auto load_b = [&](int y, RowB &r) {
        const int yh = held(y);
        const bool live = y <= y1;
        const Rsrc hr = row_of(hist0, hrow, yh, live), mr = row_of(med, mlay.row, yh, live);
        ld_hist<0>(hr, ln.x * 12, r.h0);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            r.md[k] = ld_f32(mr, xo, k * mlay.slot);
    };
    auto step_a = [&](const RowA &r, AMid &a) {
        local_adj<BCX, FC>(ph, r.mu, r.h1, r.md, ln, a.lf, a.gl, a.gk);
    };
    auto step_b = [&](int y, const AMid &dn, const AMid &c, const AMid &up, const RowB &r,
                      AMid &b) {
        float mu[9];
        gather<BCX>(dn.lf, c.lf, up.lf, wall_lo(y), wall_hi(y), ln, mu);
        local_adj<BCX, FC>(ph, mu, r.h0, r.md, ln, b.lf, b.gl, b.gk);
    };
    // Output row y from lam_f of step n - 1 of rows y - 1 .. y + 1; the
    // gradient entries add the terms of step n (a) and then of step n - 1
    // (c), in the order of two single reverse steps.
    auto emit = [&](int y, const AMid &dn, const AMid &c, const AMid &up, const AMid &a,
                    float gp, float gk) {
        float mu[9];
        gather<BCX>(dn.lf, c.lf, up.lf, wall_lo(y), wall_hi(y), ln, mu);
        const Rsrc orow = rsrc_row(mu_out, lrow, y);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            st_f32(orow, xst * 4, i * slot, same(mu[i]), false);
        st_f32(rsrc_row(grad, grow, y), xst * 4, 0, same((gp + a.gl) + c.gl), false);
        if (KN)
            st_f32(rsrc_row(grad2, grow, y), xst * 4, 0, same((gk + a.gk) + c.gk), false);
    };

    // For output row y: lam_f of step n of rows y .. y + 2 (A slots), of
    // step n - 1 of rows y - 1 .. y + 1 (B slots).  The first input parts
    // of rows y + 2 .. y + 4 and the second parts of rows y + 1 .. y + 3 are
    // in flight (three slots each, reloaded as soon as consumed).
    RowA P, Q, S;
    RowB U, V, W;
    AMid A0{}, A1{}, A2{}, B0{}, B1{}, B2{};
    load_a(y0 - 2, P);
    load_a(y0 - 1, Q);
    load_a(y0, S);
    load_b(y0 - 1, U);
    load_b(y0, V);
    load_b(y0 + 2, W);
    if (exists(y0 - 2))
        step_a(P, A0);
    load_a(y0 + 1, P);
    if (exists(y0 - 1))
        step_a(Q, A1);
    load_a(y0 + 2, Q);
    step_a(S, A2);
    load_a(y0 + 3, S);
    if (exists(y0 - 1))
        step_b(wrap(y0 - 1), A0, A1, A2, U, B0);
    load_b(y0 + 1, U);
    if (exists(y0 + 1))
        step_a(P, A0);
    load_a(y0 + 4, P);
    step_b(y0, A1, A2, A0, V, B1);
    load_b(y0 + 3, V);
    // One output row y, the slots in rotated roles (period 3).
    // The gradient entries of row y are read at the start of its row, a
    // whole row's arithmetic before they are needed.
    auto row = [&](int y, RowA &ra, AMid &na, const AMid &adn, const AMid &ac, RowB &rb,
                   AMid &nb, const AMid &bdn, const AMid &bc) {
        const float gp = ld_f32(rsrc_row(grad, grow, y), xo, 0);
        const float gk = KN ? ld_f32(rsrc_row(grad2, grow, y), xo, 0) : 0.0f;
        if (exists(y + 2))
            step_a(ra, na);
        load_a(y + 5, ra);
        if (exists(y + 1))
            step_b(wrap(y + 1), adn, ac, na, rb, nb);
        load_b(y + 4, rb);
        emit(y, bdn, bc, nb, adn, gp, gk);
    };
    // Whole periods in the loop, the last one or two rows after it: a loop
    // with exits between its rows made the compiler copy loaded values at
    // the back edge, waiting there for the loads just issued.
    int y = y0;
    for (; y + 3 <= y1; y += 3) {
        row(y, Q, A1, A2, A0, U, B2, B0, B1);
        row(y + 1, S, A2, A0, A1, W, B0, B1, B2);
        row(y + 2, P, A0, A1, A2, V, B1, B2, B0);
    }
    if (y < y1) {
        row(y, Q, A1, A2, A0, U, B2, B0, B1);
        if (y + 1 < y1)
            row(y + 1, S, A2, A0, A1, W, B0, B1, B2);
    }
}

template <int BCX, int BCY, bool KN, bool FC>
__global__ __launch_bounds__(256) void adjoint2_kernel(
    const float *__restrict__ mu_in, float *__restrict__ mu_out, const float *__restrict__ hist1,
    const float *__restrict__ hist0, const char *__restrict__ med, MLayout mlay,
    float *__restrict__ grad, float *__restrict__ grad2, Geom g, Physics ph, int band, int groups)
{
    // logical block: band-major, four strips (one per wave) per block
    const int L = xcd_remap_a(blockIdx.x, gridDim.x);
    const int bnd = L / groups;
    const int strip = (L - bnd * groups) * 4 + (int)(threadIdx.x >> 6);
    adjoint2_strip<BCX, BCY, KN, FC>(mu_in, mu_out, hist1, hist0, med, mlay, grad, grad2, g, ph,
                                     band, bnd, strip);
}

// total += seg; seg = 0 (end of a recomputed segment)
__global__ __launch_bounds__(256) void grad_fold_kernel(float *seg, double *total, Geom g,
                                                         int bpr)
{
    const int L = xcd_remap_a(blockIdx.x, gridDim.x);
    const int y = L / bpr;
    const int x = (L - y * bpr) * 256 + threadIdx.x;
    if (x >= g.nx)
        return;
    const int64_t c = (int64_t)y * g.pitch + x;
    total[c] += (double)seg[c];
    seg[c] = 0.0f;
}

__global__ __launch_bounds__(256) void grad_out_kernel(const double *grad, float *out, Geom g,
                                                        int bpr)
{
    const int L = xcd_remap_a(blockIdx.x, gridDim.x);
    const int y = L / bpr;
    const int x = (L - y * bpr) * 256 + threadIdx.x;
    if (x >= g.nx)
        return;
    out[(int64_t)y * g.nx + x] = (float)grad[(int64_t)y * g.pitch + x];
}

template <int BCX, int BCY>
static hipError_t adj_t(const float *mu_in, float *mu_out, const float *hist, const char *med,
                        const MLayout &mlay, float *grad, float *grad2, const Geom &g,
                        const Physics &ph, int terminal, float a1, float a2, int outlet,
                        hipStream_t st)
{
    const int bpr = (g.nx + 255) / 256;
#define LBK_ADJK(KN, FC)                                                                     \
    hipLaunchKernelGGL((adjoint_kernel<BCX, BCY, KN, FC>), dim3(bpr * g.ny), dim3(256), 0, st, \
                       mu_in, mu_out, hist, med, mlay, grad, grad2, g, ph, terminal, a1, a2,   \
                       outlet, bpr)
    const bool fc = ph.feps != 0.0f;
    if (grad2 && fc)
        LBK_ADJK(true, true);
    else if (grad2)
        LBK_ADJK(true, false);
    else if (fc)
        LBK_ADJK(false, true);
    else
        LBK_ADJK(false, false);
#undef LBK_ADJK
    return hipGetLastError();
}

hipError_t launch_adjoint(int bcx, int bcy, const float *mu_in, float *mu_out, const float *hist,
                          const char *med, const MLayout &mlay, float *grad, float *grad2,
                          const Geom &g, const Physics &ph, int terminal, float a1, float a2,
                          int outlet, hipStream_t st)
{
#define LBK_ADJ(X, Y)                                                                        \
    adj_t<X, Y>(mu_in, mu_out, hist, med, mlay, grad, grad2, g, ph, terminal, a1, a2, outlet, st)
    switch (bcx * 2 + bcy) {
    case 0: return LBK_ADJ(BC_PERIODIC, BC_PERIODIC);
    case 1: return LBK_ADJ(BC_PERIODIC, BC_WALL);
    case 2: return LBK_ADJ(BC_WALL, BC_PERIODIC);
    case 3: return LBK_ADJ(BC_WALL, BC_WALL);
    case 4: return LBK_ADJ(BC_PRESSURE, BC_PERIODIC);
    case 5: return LBK_ADJ(BC_PRESSURE, BC_WALL);
    default: return hipErrorInvalidValue;
    }
#undef LBK_ADJ
}

template <int BCX, int BCY>
static hipError_t adj2_t(const float *mu_in, float *mu_out, const float *hist1,
                         const float *hist0, const char *med, const MLayout &mlay, float *grad,
                         float *grad2, const Geom &g, const Physics &ph, int band, hipStream_t st)
{
    const int nstrips = (g.nx + kStrip2 - 1) / kStrip2;
    const int groups = (nstrips + 3) / 4;
    const int blocks = groups * ((g.ny + band - 1) / band);
#define LBK_ADJ2K(KN, FC)                                                                    \
    hipLaunchKernelGGL((adjoint2_kernel<BCX, BCY, KN, FC>), dim3(blocks), dim3(256), 0, st,    \
                       mu_in, mu_out, hist1, hist0, med, mlay, grad, grad2, g, ph, band, groups)
    const bool fc = ph.feps != 0.0f;
    if (grad2 && fc)
        LBK_ADJ2K(true, true);
    else if (grad2)
        LBK_ADJ2K(true, false);
    else if (fc)
        LBK_ADJ2K(false, true);
    else
        LBK_ADJ2K(false, false);
#undef LBK_ADJ2K
    return hipGetLastError();
}

hipError_t launch_adjoint2(int bcx, int bcy, const float *mu_in, float *mu_out,
                           const float *hist1, const float *hist0, const char *med,
                           const MLayout &mlay, float *grad, float *grad2, const Geom &g,
                           const Physics &ph, int band, hipStream_t st)
{
    if (band < 1 || mu_in == mu_out)
        return hipErrorInvalidValue;
#define LBK_ADJ2(X, Y)                                                                       \
    adj2_t<X, Y>(mu_in, mu_out, hist1, hist0, med, mlay, grad, grad2, g, ph, band, st)
    switch (bcx * 2 + bcy) {
    case 0: return LBK_ADJ2(BC_PERIODIC, BC_PERIODIC);
    case 1: return LBK_ADJ2(BC_PERIODIC, BC_WALL);
    case 2: return LBK_ADJ2(BC_WALL, BC_PERIODIC);
    case 3: return LBK_ADJ2(BC_WALL, BC_WALL);
    case 4: return LBK_ADJ2(BC_PRESSURE, BC_PERIODIC);
    case 5: return LBK_ADJ2(BC_PRESSURE, BC_WALL);
    default: return hipErrorInvalidValue;
    }
#undef LBK_ADJ2
}

hipError_t launch_grad_fold(float *seg, double *total, const Geom &g, hipStream_t st)
{
    const int bpr = (g.nx + 255) / 256;
    hipLaunchKernelGGL(grad_fold_kernel, dim3(bpr * g.ny), dim3(256), 0, st, seg, total, g, bpr);
    return hipGetLastError();
}

hipError_t launch_grad_out(const double *grad, float *out, const Geom &g, hipStream_t st)
{
    const int bpr = (g.nx + 255) / 256;
    hipLaunchKernelGGL(grad_out_kernel, dim3(bpr * g.ny), dim3(256), 0, st, grad, out, g, bpr);
    return hipGetLastError();
}

// ------------------------------------------------------ batched gradients
//
// The same reverse step, fold and output over a batch's tile list (tiles of
// blockDim.x by rows, one workgroup per tile); each sample's regions come
// from its descriptor, copied to registers before the first store.

__device__ __forceinline__ bool adj_tile(const AdjSampleDesc *__restrict__ samples,
                                         const int *__restrict__ tile_sample, int rows,
                                         AdjSampleDesc &sd, uint32_t &x, int &y0, int &y1)
{
    const int t = xcd_remap_a(blockIdx.x, gridDim.x);
    sd = samples[tile_sample[t]];
    const int rel = t - sd.one.tile0;
    const int ty = rel / sd.one.tpr;
    x = (uint32_t)(rel - ty * sd.one.tpr) * blockDim.x + threadIdx.x;
    y0 = ty * rows;
    y1 = min(y0 + rows, sd.g.ny);
    return x < (uint32_t)sd.g.nx;
}

// lam_in < 0: the terminal read-out (writes lam[0]); else lam[lam_in] ->
// lam[lam_in ^ 1].  hist_slot: the history of the step being reversed.
template <int BCX, int BCY, bool KN, bool FC>
__global__ __launch_bounds__(256) void batch_adjoint_kernel(
    const AdjSampleDesc *__restrict__ samples, const int *__restrict__ tile_sample, int rows,
    int lam_in, int hist_slot)
{
    AdjSampleDesc sd;
    uint32_t x;
    int y0, y1;
    if (!adj_tile(samples, tile_sample, rows, sd, x, y0, y1))
        return;
    const bool terminal = lam_in < 0;
    const float *mu_in = terminal ? nullptr : (lam_in ? sd.lam[1] : sd.lam[0]);
    float *mu_out = terminal ? sd.lam[0] : (lam_in ? sd.lam[0] : sd.lam[1]);
    const float *hist = reinterpret_cast<const float *>(reinterpret_cast<const char *>(sd.hist) +
                                                        (uint64_t)hist_slot * sd.hist_bytes);
    for (int y = y0; y < y1; ++y)
        adjoint_node<BCX, BCY, KN, FC>(mu_in, mu_out, hist, sd.med, sd.mlay, sd.seg, sd.seg2, sd.g,
                                   sd.ph, terminal ? 1 : 0, sd.a1, sd.a2, sd.outlet, y, x);
}

// Two reverse steps of every sample, lam[lam_in] -> lam[lam_in ^ 1], the
// histories in slots hist_slot (the later step) and hist_slot - 1: tiles of
// four strips by `band` rows (the batch's two-step tiling: sd.two gives a
// sample's first tile and its groups of four strips per band).
template <int BCX, int BCY, bool KN, bool FC>
__global__ __launch_bounds__(256) void batch_adjoint2_kernel(
    const AdjSampleDesc *__restrict__ samples, const int *__restrict__ tile_sample, int band,
    int lam_in, int hist_slot)
{
    const int t = xcd_remap_a(blockIdx.x, gridDim.x);
    const AdjSampleDesc sd = samples[tile_sample[t]];
    const int rel = t - sd.two.tile0;
    const int bnd = rel / sd.two.tpr;
    const int strip = (rel - bnd * sd.two.tpr) * 4 + (int)(threadIdx.x >> 6);
    const float *mu_in = lam_in ? sd.lam[1] : sd.lam[0];
    float *mu_out = lam_in ? sd.lam[0] : sd.lam[1];
    const char *h = reinterpret_cast<const char *>(sd.hist);
    const float *hist1 = reinterpret_cast<const float *>(h + (uint64_t)hist_slot * sd.hist_bytes);
    const float *hist0 =
        reinterpret_cast<const float *>(h + (uint64_t)(hist_slot - 1) * sd.hist_bytes);
    adjoint2_strip<BCX, BCY, KN, FC>(mu_in, mu_out, hist1, hist0, sd.med, sd.mlay, sd.seg,
                                     KN ? sd.seg2 : nullptr, sd.g, sd.ph, band, bnd, strip);
}

// op 0: clear the segment and total planes; 1: fold segment into total;
// 2: write the totals to the output planes.  kn: the ln kn0 plane too.
__global__ __launch_bounds__(256) void batch_grad_kernel(const AdjSampleDesc *__restrict__ samples,
                                                         const int *__restrict__ tile_sample,
                                                         int rows, int op, int kn)
{
    AdjSampleDesc sd;
    uint32_t x;
    int y0, y1;
    if (!adj_tile(samples, tile_sample, rows, sd, x, y0, y1))
        return;
    for (int y = y0; y < y1; ++y) {
        const int64_t c = (int64_t)y * sd.g.pitch + x, o = (int64_t)y * sd.g.nx + x;
        for (int p = 0; p < (kn ? 2 : 1); ++p) {
            float *seg = p ? sd.seg2 : sd.seg;
            double *tot = p ? sd.grad2 : sd.grad;
            if (op == 0) {
                seg[c] = 0.0f;
                tot[c] = 0.0;
            } else if (op == 1) {
                tot[c] += (double)seg[c];
                seg[c] = 0.0f;
            } else {
                (p ? sd.out2 : sd.out)[o] = (float)tot[c];
            }
        }
    }
}

template <int BCX, int BCY>
static hipError_t batch_adj_t(const AdjSampleDesc *samples, const int *tile_sample, int ntiles,
                              int tile_x, int rows, int lam_in, int hist_slot, int kn, int fc,
                              hipStream_t st)
{
#define LBK_BADJK(KN, FC)                                                                    \
    hipLaunchKernelGGL((batch_adjoint_kernel<BCX, BCY, KN, FC>), dim3(ntiles), dim3(tile_x), 0, \
                       st, samples, tile_sample, rows, lam_in, hist_slot)
    if (kn && fc)
        LBK_BADJK(true, true);
    else if (kn)
        LBK_BADJK(true, false);
    else if (fc)
        LBK_BADJK(false, true);
    else
        LBK_BADJK(false, false);
#undef LBK_BADJK
    return hipGetLastError();
}

hipError_t launch_batch_adjoint(int bcx, int bcy, const AdjSampleDesc *samples,
                                const int *tile_sample, int ntiles, int tile_x, int rows,
                                int lam_in, int hist_slot, int kn, int fc, hipStream_t st)
{
    if (tile_x < 64 || tile_x > 256 || (tile_x & 63) || rows < 1 || ntiles < 0)
        return hipErrorInvalidValue;
    if (ntiles == 0)
        return hipSuccess;
#define LBK_BADJ(X, Y)                                                                       \
    batch_adj_t<X, Y>(samples, tile_sample, ntiles, tile_x, rows, lam_in, hist_slot, kn, fc, st)
    switch (bcx * 2 + bcy) {
    case 0: return LBK_BADJ(BC_PERIODIC, BC_PERIODIC);
    case 1: return LBK_BADJ(BC_PERIODIC, BC_WALL);
    case 2: return LBK_BADJ(BC_WALL, BC_PERIODIC);
    case 3: return LBK_BADJ(BC_WALL, BC_WALL);
    case 4: return LBK_BADJ(BC_PRESSURE, BC_PERIODIC);
    case 5: return LBK_BADJ(BC_PRESSURE, BC_WALL);
    default: return hipErrorInvalidValue;
    }
#undef LBK_BADJ
}

template <int BCX, int BCY>
static hipError_t batch_adj2_t(const AdjSampleDesc *samples, const int *tile_sample, int ntiles,
                               int band, int lam_in, int hist_slot, int kn, int fc,
                               hipStream_t st)
{
#define LBK_BADJ2K(KN, FC)                                                                   \
    hipLaunchKernelGGL((batch_adjoint2_kernel<BCX, BCY, KN, FC>), dim3(ntiles), dim3(256), 0,  \
                       st, samples, tile_sample, band, lam_in, hist_slot)
    if (kn && fc)
        LBK_BADJ2K(true, true);
    else if (kn)
        LBK_BADJ2K(true, false);
    else if (fc)
        LBK_BADJ2K(false, true);
    else
        LBK_BADJ2K(false, false);
#undef LBK_BADJ2K
    return hipGetLastError();
}

hipError_t launch_batch_adjoint2(int bcx, int bcy, const AdjSampleDesc *samples,
                                 const int *tile_sample, int ntiles, int band, int lam_in,
                                 int hist_slot, int kn, int fc, hipStream_t st)
{
    if (ntiles < 0 || band < 1 || lam_in < 0 || lam_in > 1 || hist_slot < 1)
        return hipErrorInvalidValue;
    if (ntiles == 0)
        return hipSuccess;
#define LBK_BADJ2(X, Y) batch_adj2_t<X, Y>(samples, tile_sample, ntiles, band, lam_in, hist_slot, kn, fc, st)
    switch (bcx * 2 + bcy) {
    case 0: return LBK_BADJ2(BC_PERIODIC, BC_PERIODIC);
    case 1: return LBK_BADJ2(BC_PERIODIC, BC_WALL);
    case 2: return LBK_BADJ2(BC_WALL, BC_PERIODIC);
    case 3: return LBK_BADJ2(BC_WALL, BC_WALL);
    case 4: return LBK_BADJ2(BC_PRESSURE, BC_PERIODIC);
    case 5: return LBK_BADJ2(BC_PRESSURE, BC_WALL);
    default: return hipErrorInvalidValue;
    }
#undef LBK_BADJ2
}

hipError_t launch_batch_grad(const AdjSampleDesc *samples, const int *tile_sample, int ntiles,
                             int tile_x, int rows, int op, int kn, hipStream_t st)
{
    if (tile_x < 64 || tile_x > 256 || (tile_x & 63) || rows < 1 || ntiles < 0 || op < 0 ||
        op > 2)
        return hipErrorInvalidValue;
    if (ntiles == 0)
        return hipSuccess;
    hipLaunchKernelGGL(batch_grad_kernel, dim3(ntiles), dim3(tile_x), 0, st, samples,
                       tile_sample, rows, op, kn);
    return hipGetLastError();
}

} // namespace lbk
