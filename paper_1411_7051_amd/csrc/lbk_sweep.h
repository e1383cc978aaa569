// lbk_sweep.h -- the node update of the D2Q9 sweep as the kernels share it:
// the post-stream state of a node with the pressure-column override
// (pulled from HBM, or from rows held in registers), the full update of a
// node, and the history record of the adjoint.
#pragma once

#include "lbk_kernels.h"

namespace lbk {

// Hardware block b lands on XCD b % 8; give XCD j the j-th contiguous chunk
// of logical blocks.  A bijection on [0, nb) for any nb.
__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    const int j = b & 7, idx = b >> 3;
    return j * q + (j < r ? j : r) + idx;
}

// Row and column of this thread's node; y is uniform across the block.
struct Node {
    int y;
    uint32_t x;
    int L; // logical block index
};
__device__ __forceinline__ Node node_of(int bpr)
{
    Node n;
    n.L = xcd_remap(blockIdx.x, gridDim.x);
    n.y = n.L / bpr;
    n.x = (uint32_t)(n.L - n.y * bpr) * kBlock + threadIdx.x;
    return n;
}

// Medium of row y: eps, drag and kn0 at x.
struct Med {
    Rsrc r;
    uint32_t slot, slot2; // byte offsets of the drag and kn0 slots
    __device__ __forceinline__ float eps(uint32_t x) const { return ld_f32(r, x * 4, 0); }
    __device__ __forceinline__ float drag(uint32_t x) const { return ld_f32(r, x * 4, slot); }
    __device__ __forceinline__ float kn0(uint32_t x) const { return ld_f32(r, x * 4, slot2); }
};

// Pressure-column override (non-equilibrium extrapolation from the
// neighbouring column): on entry d, rho, inc, r are the neighbour's pulled
// deviations, density and density residual and en, dragn, kn0n its medium;
// on return d holds the boundary node's deviations relative to the imposed
// density rb (returned), inc = 0 and r its density residual:
//   f_i = f_eq_i(rho_b, u_n; eps_b) + f_i(n) - f_eq_i(rho_n, u_n; eps_n)
// eb and en are what the model's nodes carry: eps, or 1 / eps under MODEL_STD.
template <typename T, int MODEL>
__device__ __forceinline__ float extrapolate(const Physics &ph, float s, float inv_s, bool in,
                                             float eb, float en, float dragn, float kn0n,
                                             float rho, float (&d)[9], float &inc, float &r)
{
    float jx, jy, ux, uy, Fx, Fy;
    momentum(d, jx, jy);
    if (Elem<T>::kScaled) {
        jx *= inv_s;
        jy *= inv_s;
    }
    velocity<MODEL>(ph, rho, jx, jy, en, dragn, kn0n, true, ux, uy, Fx, Fy);
    const float rb = in ? ph.rin_hi : ph.rout_hi;
    const float rbl = in ? ph.rin_lo : ph.rout_lo;
    // f_eq_i(rho_b, u; eps_b) - f_eq_i(rho_n, u; eps_n) of Eq. 14 as
    // w_i [a e.u + b (4.5 (e.u)^2 - 1.5 u.u)], each equilibrium's
    // deviation from w_i rho vanishing at eps = 0
    const bool sb = !(eb > 0.0f), sn = !(en > 0.0f);
    const float a = 3.0f * ((sb ? 0.0f : rb) - (sn ? 0.0f : rho));
    const float ib = MODEL == MODEL_STD ? eb : __builtin_amdgcn_rcpf(eb);
    const float in_ = MODEL == MODEL_STD ? en : __builtin_amdgcn_rcpf(en);
    const float b = (sb ? 0.0f : rb * ib) - (sn ? 0.0f : rho * in_);
    const float uu = ux * ux + uy * uy;
    const float c = (rbl - r) - inc; // w_i (rbl - r) - w_i inc, over w_i
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        // physical deviation of the boundary node from w_i rb
        const float eu = edot(ex_of(i), ey_of(i), 0, ux, uy, 0.0f);
        const float q = c + b * (4.5f * eu * eu - 1.5f * uu) + a * eu;
        const float v = w_of(i) * q + (Elem<T>::kScaled ? d[i] * inv_s : d[i]);
        sum += v;
        d[i] = Elem<T>::kScaled ? v * s : v;
    }
    inc = 0.0f;
    r = sum;
    return rb;
}

// Post-stream deviations d_i (storage unit) of node (x, y) after the
// boundary override, relative to rho - inc; returns the FP32 density rho
// and sets inc and the density residual r (physical unit).  A pressure-
// column node pulls at its neighbour xn with the same code as every other
// lane, so that only the extrapolation itself diverges (narrow samples of
// a batch have boundary lanes in a large share of their waves).
template <typename T, int BCX>
__device__ __forceinline__ float post_stream(const Rows &R, const Layout &L, const Med &md,
                                             const Geom &g, const Physics &ph, float s,
                                             float inv_s, uint32_t x, float (&d)[9], float &inc,
                                             float &r)
{
    const bool bnode = BCX == BC_PRESSURE && (x == 0 || x == (uint32_t)g.nx - 1);
    const uint32_t xs = !bnode ? x : (x == 0 ? 1u : (uint32_t)g.nx - 2);
    float rc;
    pull<T, BCX>(R, L, g, s, xs, rc, d);
    const float rho = density<T>(rc, d, inv_s, inc, r);
    if (BCX == BC_PRESSURE && bnode) {
        const float en = md.eps(xs), eb = md.eps(x);
        return extrapolate<T, MODEL_GEN>(ph, s, inv_s, x == 0, eb, en, md.drag(xs), md.kn0(xs),
                                         rho, d, inc, r);
    }
    return rho;
}

// Linearisation point (rho, jx, jy) of one step at node (x, y) into a
// history slot [y][pitch][3] (FP32, the node's three values together), for
// the adjoint; nt: streaming stores.
__device__ __forceinline__ void record(float *hist, const Geom &g, int y, uint32_t x, float rho,
                                       float jx, float jy, bool nt = true)
{
    const uint32_t hrow = 3u * (uint32_t)g.pitch * 4u;
    const Rsrc hr = make_rsrc(reinterpret_cast<char *>(hist) + (uint64_t)y * hrow, hrow);
    if (nt)
        st_hist<kNT>(hr, x * 12, rho, jx, jy);
    else
        st_hist<0>(hr, x * 12, rho, jx, jy);
}

// Full update of node (x, y): pull, boundary override, moments, velocity,
// collide, store; with HIST also the step's linearisation point.
template <typename T, int BCX, int BCY, bool HIST>
__device__ __forceinline__ void sweep_node(const char *src, char *dst, const Layout &lay,
                                           const char *med, const MLayout &mlay, const Geom &g,
                                           const Physics &ph, float s, float inv_s, float *hist,
                                           int y, uint32_t x)
{
    const Rows R = rows_of<BCY>(src, lay, g, y);
    const Med md{med_row(med, mlay, y), mlay.slot, 2 * mlay.slot};
    float d[9], inc, r;
    const float rho = post_stream<T, BCX>(R, lay, md, g, ph, s, inv_s, x, d, inc, r);
    float jx, jy, ux, uy, Fx, Fy;
    momentum(d, jx, jy);
    if (Elem<T>::kScaled) {
        jx *= inv_s;
        jy *= inv_s;
    }
    if (HIST)
        record(hist, g, y, x, rho, jx, jy);
    const float eps = md.eps(x);
    const bool solids = any_lane(!(eps > 0.0f));
    velocity<MODEL_GEN>(ph, rho, jx, jy, eps, md.drag(x), md.kn0(x), solids, ux, uy, Fx, Fy);
    float hs[9];
    collide<T, MODEL_GEN>(ph, rho, inc, r, d, ux, uy, Fx, Fy, eps, solids, s, hs);
    const Rsrc out = make_rsrc(dst + (uint64_t)y * lay.row, (uint32_t)lay.row);
    st_f32(out, x * 4, 0, rho, true);
    constexpr uint32_t es = sizeof(T);
#pragma unroll
    for (int i = 0; i < 9; ++i)
        Elem<T>::st(out, x * es, lay.h_off + i * lay.h_slot, hs[i]);
}

// ------------------------------------------- updates of rows in registers

// One node of a level as a pull reads it: density and deviations (storage
// unit, as stored), with the node's medium.
template <typename T> struct Mid {
    float rho;
    typename Elem<T>::Reg h[9];
    float e, drag, kn0; // e = eps, or 1 / eps under MODEL_STD (0 where eps = 0)
};

// Node (x, y) of a stored level and its medium.  A row the march loads
// ahead but will not use (live = false, uniform) gets empty buffer
// resources: its loads return 0 without touching memory.
template <typename T, int MODEL = MODEL_GEN>
__device__ __forceinline__ void load_node(const char *src, const Layout &lay, const char *med,
                                          const MLayout &mlay, int y, uint32_t x, Mid<T> &m,
                                          bool live = true)
{
    const Rsrc row = make_rsrc(src + (uint64_t)y * lay.row, live ? (uint32_t)lay.row : 0u);
    // default cache policy: a strip's 64-column loads share their first and
    // last cache lines with the neighbouring strips, which read them about
    // the same time (nontemporal loads fetched those lines twice)
    m.rho = ld_f32(row, x * 4, 0);
    constexpr uint32_t es = sizeof(T);
#pragma unroll
    for (int i = 0; i < 9; ++i)
        m.h[i] = Elem<T>::template ldr<0>(row, x * es, lay.h_off + i * lay.h_slot);
    const Rsrc mr = make_rsrc(med + (uint64_t)y * mlay.row, live ? (uint32_t)mlay.row : 0u);
    m.e = ld_f32(mr, x * 4, 0);
    if (MODEL == MODEL_STD)
        m.e = m.e > 0.0f ? __builtin_amdgcn_rcpf(m.e) : 0.0f;
    m.drag = ld_f32(mr, x * 4, mlay.slot);
    m.kn0 = ld_f32(mr, x * 4, 2 * mlay.slot);
}

// The pull of this lane's node from the rows y - 1 (dn), y (c) and y + 1 (up)
// of the previous level: the arithmetic of pull() with the neighbour values
// taken from registers and adjacent lanes.
template <typename T, int BCX>
__device__ __forceinline__ void pull_mid(const Mid<T> &dn, const Mid<T> &c, const Mid<T> &up, bool wym,
                                         bool wyp, bool wxm, bool wxp, float s, float &rc,
                                         float (&d)[9])
{
    rc = c.rho;
    d[0] = Elem<T>::val(c.h[0]);
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const int ex = ex_of(i), ey = ey_of(i);
        const bool wall_y = (ey == 1 && wym) || (ey == -1 && wyp); // uniform
        const Mid<T> &m = ey == 1 ? dn : (ey == -1 ? up : c);
        const float ws = Elem<T>::kScaled ? w_of(i) * s : w_of(i);
        // the shift of rho folds into the subtraction, the widening of an
        // FP16 h into the FMA
        float df = (ex == 1 ? lane_from<1>(m.rho) : (ex == -1 ? lane_from<-1>(m.rho) : m.rho)) - rc;
        auto h = ex == 1 ? lane_from<1>(m.h[i]) : (ex == -1 ? lane_from<-1>(m.h[i]) : m.h[i]);
        // a wall bounces the pull back: a select, not a branch, so that no
        // control flow splits the row's loads from their uses
        if (ey != 0) {
            df = wall_y ? 0.0f : df;
            h = wall_y ? c.h[opp_of(i)] : h;
        }
        d[i] = ws * df + Elem<T>::val(h);
        if (BCX == BC_WALL) {
            const bool wall_x = (ex == 1 && wxm) || (ex == -1 && wxp); // per lane, edges only
            if (wall_x)
                d[i] = Elem<T>::val(c.h[opp_of(i)]);
        }
    }
}

// Lane-dependent facts of a strip: which column a lane holds and what kind.
struct Lanes {
    uint32_t x;     // the lane's column, wrapped (periodic) or clamped
    bool wxm, wxp;  // x walls on either side of the column
    bool bin, bout; // the inlet / outlet pressure column
    int has_b;      // uniform: the wave may hold a pressure column
};

// One step of this lane's node at row y from three rows of the previous
// level in registers: pull, pressure-column override from the neighbouring
// lane's pull, moments, velocity and collide -- sweep_node's update.
// Returns the new density, the unrounded deviations hs and, for the
// history, (jx, jy).
template <typename T, int BCX, int MODEL = MODEL_GEN>
__device__ __forceinline__ float step_from(const Physics &ph, float s, float inv_s, const Mid<T> &dn,
                                           const Mid<T> &c, const Mid<T> &up, bool wym, bool wyp,
                                           const Lanes &ln, bool any_solid, float (&hs)[9],
                                           float &jx, float &jy)
{
    float d[9], rc, inc, r;
    pull_mid<T, BCX>(dn, c, up, wym, wyp, ln.wxm, ln.wxp, s, rc, d);
    float en = 0.0f, dragn = 0.0f, kn0n = 0.0f;
    if (BCX == BC_PRESSURE && ln.has_b) {
        // a pressure column pulls at its neighbour: take that lane's pull
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const float lf = lane_from<-1>(d[i]), rf = lane_from<1>(d[i]);
            d[i] = ln.bin ? lf : (ln.bout ? rf : d[i]);
        }
        const float rl = lane_from<-1>(rc), rr = lane_from<1>(rc);
        rc = ln.bin ? rl : (ln.bout ? rr : rc);
        const float el = lane_from<-1>(c.e), er = lane_from<1>(c.e);
        const float dl = lane_from<-1>(c.drag), dr = lane_from<1>(c.drag);
        const float kl = lane_from<-1>(c.kn0), kr = lane_from<1>(c.kn0);
        en = ln.bin ? el : er;
        dragn = ln.bin ? dl : dr;
        kn0n = ln.bin ? kl : kr;
    }
    float rho = density<T>(rc, d, inv_s, inc, r);
    if (BCX == BC_PRESSURE && (ln.bin || ln.bout))
        rho = extrapolate<T, MODEL>(ph, s, inv_s, ln.bin, c.e, en, dragn, kn0n, rho, d, inc, r);
    momentum(d, jx, jy);
    if (Elem<T>::kScaled) {
        jx *= inv_s;
        jy *= inv_s;
    }
    float ux, uy, Fx, Fy;
    velocity<MODEL>(ph, rho, jx, jy, c.e, c.drag, c.kn0, any_solid, ux, uy, Fx, Fy);
    collide<T, MODEL>(ph, rho, inc, r, d, ux, uy, Fx, Fy, c.e, any_solid, s, hs);
    return rho;
}

// First step of row y: the intermediate node as the second step reads it.
template <typename T, int BCX, bool HIST>
__device__ __forceinline__ void first_step(const Physics &ph, float s, float inv_s, const Geom &g,
                                           const Mid<T> &dn, const Mid<T> &c, const Mid<T> &up,
                                           bool wym, bool wyp, const Lanes &ln, int y, float *hist,
                                           bool rec, Mid<T> &m)
{
    float hs[9], jx, jy;
    m.rho = step_from<T, BCX>(ph, s, inv_s, dn, c, up, wym, wyp, ln, any_lane(!(c.e > 0.0f)), hs,
                              jx, jy);
    if (HIST && rec)
        record(hist, g, y, ln.x, m.rho, jx, jy, false);
#pragma unroll
    for (int i = 0; i < 9; ++i)
        m.h[i] = Elem<T>::reg(hs[i]);
    m.e = c.e;
    m.drag = c.drag;
    m.kn0 = c.kn0;
}

// Dispatch a (storage, bc_x, bc_y) triple to a template instance.
#define LBK_DISPATCH_BC(FN, T, ...)                                                          \
    switch (bcx * 2 + bcy) {                                                                 \
    case 0: return FN<T, BC_PERIODIC, BC_PERIODIC>(__VA_ARGS__);                             \
    case 1: return FN<T, BC_PERIODIC, BC_WALL>(__VA_ARGS__);                                 \
    case 2: return FN<T, BC_WALL, BC_PERIODIC>(__VA_ARGS__);                                 \
    case 3: return FN<T, BC_WALL, BC_WALL>(__VA_ARGS__);                                     \
    case 4: return FN<T, BC_PRESSURE, BC_PERIODIC>(__VA_ARGS__);                             \
    case 5: return FN<T, BC_PRESSURE, BC_WALL>(__VA_ARGS__);                                 \
    default: return hipErrorInvalidValue;                                                    \
    }

#define LBK_DISPATCH(FN, ...)                                                                \
    switch (storage) {                                                                       \
    case 0: LBK_DISPATCH_BC(FN, float, __VA_ARGS__)                                          \
    case 1: LBK_DISPATCH_BC(FN, __half, __VA_ARGS__)                                         \
    case 2: LBK_DISPATCH_BC(FN, __hip_bfloat16, __VA_ARGS__)                                 \
    default: return hipErrorInvalidValue;                                                    \
    }

} // namespace lbk
