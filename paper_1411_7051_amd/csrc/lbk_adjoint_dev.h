// lbk_adjoint_dev.h -- one reverse step of a node as the reverse kernels share
// it: the adjoint of the collide (and of the read-out of J, and of the
// pressure-column override), and the gather form of the adjoint of the pull
// on values held in registers.  lbk_adjoint.hip derives the formulas.
//
// A step of a node in Darcy form takes about 150 vector instructions and five
// transcendental ones; with the partials of each term formed by itself, eight
// reciprocals and rho applied and divided out again it was 240.  The marching
// pairs of 2048 x 2048 went from 64.0 to 61.8 us a step, single steps of 64 x
// 32 from 5.1 to 4.4.
#pragma once

#include "lbk_adjoint.h"
#include "lbk_kernels.h"

namespace lbk {

namespace {

__device__ __forceinline__ int xcd_remap_a(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    const int j = b & 7, idx = b >> 3;
    return j * q + (j < r ? j : r) + idx;
}

// Forward quantities of one node's velocity solve, as in velocity() of the
// sweep, plus what the adjoint needs: dA/d ln kn0 and, through the local Kn,
// dA/drho = drho_k dA/d ln kn0 / rho with drho_k = -1 or 0.
struct NodeFwd {
    float rho, rinv, jx, jy, ie, A, B, c0, g, ag, ux, uy, un, Fx, Fy, dA_dlnkn;
    bool solid, any_solid; // any_solid: uniform, whether a lane is solid
};

// M: what of the model a kernel is compiled for.  With REV_STD the eps given
// is 1 / eps (0 where eps = 0).
__device__ __forceinline__ float inv_eps(float eps)
{
    return eps > 0.0f ? __builtin_amdgcn_rcpf(eps) : 0.0f;
}

template <int M>
__device__ __forceinline__ NodeFwd node_fwd(const Physics &ph, float rho, float jx, float jy,
                                            float e, float drag, float kn0)
{
    NodeFwd n;
    n.rho = rho;
    n.jx = jx;
    n.jy = jy;
    n.solid = !(e > 0.0f);
    n.any_solid = any_lane(n.solid);
    // hardware reciprocals, as in the sweep's velocity solve
    n.ie = M == REV_STD ? e : inv_eps(e);
    n.rinv = __builtin_amdgcn_rcpf(rho);
    // f_c = den / num, as in the sweep, and ndr = num f_c'(Kn) / f_c.
    // For Eqs. 6-7, f_c = P1 P2 with P1 = p1/a, a = t + 0.170, t = Kn^0.4348,
    // p1 = a + 1.358 t Kn, and P2 = p2/q, p2 = 1 + (4 - b) Kn, q = 1 - b Kn:
    // P1' = 1.358 t (t + 1.4348 * 0.170)/a^2 and P2' = 4/q^2, so
    // f_c'/f_c = 1.358 t (t + 0.243916)/(a p1) + 4/(q p2), over the common
    // denominator num den = a q p1 p2: one reciprocal, r = 1 / den.  r goes into
    // each product before the large factors meet, so that nothing overflows
    // before den itself does (~ Kn^2.43, from Kn = 3e15 on).  For Eqs. 4-5,
    // f_c' = 4.
    const float kn = M == REV_STD ? kn0 * n.rinv
                                  : (ph.kn_local ? kn0 * (ph.rho_ref * n.rinv) : kn0);
    float num = 1.0f, den = 1.0f, r = 1.0f, ndr = 0.0f;
    if (M == REV_STD || ph.corr == CORR_BKC) {
        const float t = fc_pow(kn);
        fc_bkc(ph, kn, t, num, den);
        r = __builtin_amdgcn_rcpf(den);
        const float a = t + 0.170f, tt = 1.358f * t;
        const float p1 = a + tt * kn, p2 = 1.0f + ph.slip_c * kn, q = 1.0f + ph.slip_nb * kn;
        ndr = tt * (t + 0.243916f) * q * (p2 * r) + 4.0f * a * (p1 * r);
    } else if (ph.corr == CORR_KLINKENBERG) {
        fc_parts_t(ph, kn, 0.0f, num, den);
        r = __builtin_amdgcn_rcpf(den);
        ndr = 4.0f * r;
    }
    const float dn = drag * num;
    n.A = dn * r; // drag / f_c
    // dA/d ln kn0 = -A Kn f_c'(Kn) / f_c = -drag Kn ndr / den
    n.dA_dlnkn = -(kn * ndr * r) * drag;
    float vx = jx * n.rinv, vy = jy * n.rinv, egx = 0.0f, egy = 0.0f;
    if (M != REV_STD) {
        egx = e * ph.gx;
        egy = e * ph.gy;
        vx += 0.5f * egx;
        vy += 0.5f * egy;
    }
    n.B = n.un = 0.0f;
    n.c0 = 1.0f + 0.5f * n.A;
    if (M != REV_FORCH || ph.feps == 0.0f) {
        const float R2 = 2.0f * __builtin_amdgcn_rcpf(2.0f * den + dn);
        n.g = den * R2; // 1 / (1 + A/2)
        n.ag = dn * R2; // A g
    } else {
        // Forchheimer (Eq. 2): c0 u + (B/2) |u| u = v, B = eps F_eps / sqrt(k_a),
        // the positive root as in the forward velocity solve
        n.B = ph.feps * __builtin_sqrtf(e * n.A * ph.inv_nu);
        const float wn = __builtin_sqrtf(vx * vx + vy * vy);
        n.g = 2.0f / (n.c0 + __builtin_sqrtf(n.c0 * n.c0 + 2.0f * n.B * wn));
        n.ag = n.A * n.g;
    }
    n.ux = n.g * vx;
    n.uy = n.g * vy;
    n.Fx = egx - n.ag * vx;
    n.Fy = egy - n.ag * vy;
    if (M == REV_FORCH) {
        n.un = n.solid || ph.feps == 0.0f ? 0.0f
                                          : __builtin_sqrtf(n.ux * n.ux + n.uy * n.uy);
        n.Fx -= n.B * n.un * n.ux;
        n.Fy -= n.B * n.un * n.uy;
    }
    if (uniform_branch(n.any_solid)) {
        n.ux = n.solid ? 0.0f : n.ux;
        n.uy = n.solid ? 0.0f : n.uy;
        n.Fx = n.solid ? -2.0f * jx * n.rinv : n.Fx;
        n.Fy = n.solid ? -2.0f * jy * n.rinv : n.Fy;
    }
    return n;
}

// w-weighted moments of a 9-vector: L0 = sum w l, L1 = sum w l e,
// L2 = sum w l e e (symmetric; xx, yy, xy), from the sums and differences
// of opposite directions, each weight class applied once.
struct Mom {
    float m0, m1x, m1y, mxx, myy, mxy;
};
__device__ __forceinline__ Mom moments(const float (&l)[9])
{
    // e_5 = (1, 1), e_6 = (-1, 1), e_7 = (-1, -1), e_8 = (1, -1)
    const float a13 = l[1] + l[3], d13 = l[1] - l[3];
    const float a24 = l[2] + l[4], d24 = l[2] - l[4];
    const float a57 = l[5] + l[7], d57 = l[5] - l[7];
    const float a68 = l[6] + l[8], d68 = l[6] - l[8];
    const float sd = a57 + a68;
    const float w0 = w_of(0), w1 = w_of(1), w2 = w_of(5);
    Mom m;
    m.m0 = w0 * l[0] + w1 * (a13 + a24) + w2 * sd;
    m.m1x = w1 * d13 + w2 * (d57 - d68);
    m.m1y = w1 * d24 + w2 * (d57 + d68);
    m.mxx = w1 * a13 + w2 * sd;
    m.myy = w1 * a24 + w2 * sd;
    m.mxy = w2 * (a57 - a68);
    return m;
}

// out_i = k v_i + c + e_i . (gx, gy) for the nine directions (v = NULL: k
// v_i left out), the direction-class sums formed once.
template <bool V>
__device__ __forceinline__ void spread(float k, const float *v, float c, float gx, float gy,
                                       float (&out)[9])
{
    const float px = c + gx, mx = c - gx;
    const float t[9] = {c, px, c + gy, mx, c - gy, px + gy, mx + gy, mx - gy, px - gy};
#pragma unroll
    for (int i = 0; i < 9; ++i)
        out[i] = V ? k * v[i] + t[i] : t[i];
}

// Chain rule from the partials of a node function Psi = rho psi(rho, u, F)
// to its total derivatives with respect to rho, j and ln k through the node's
// velocity solve.  Pr is the explicit dPsi/drho, (pux, puy) = psi_u and
// (pfx, pfy) = psi_F: the partials of Psi over rho, so that rho and the 1 / rho
// of dv/dj = 1 / rho cancel instead of being applied one after the other.
struct Grads {
    float rho, jx, jy, lnk, lnkn;
};
template <int M>
__device__ __forceinline__ Grads chain(const Physics &ph, const NodeFwd &n, float Pr, float pux,
                                       float puy, float pfx, float pfy)
{
    Grads G;
    // The velocity solves M(u) = c0 u + (B/2) |u| u = v, v = j / rho + eps G / 2,
    // c0 = 1 + A/2, and F = eps G - A u - B |u| u.  With T = dPsi/du through
    // u and F(u) at fixed A, B, and K = dM/du = a I + (B/2) u u^T / |u|,
    // a = c0 + B |u| / 2: dPsi/dv = S = K^-1 T, dPsi/dj = S / rho, and
    // dPsi/dA = -(S.u / 2 + Psi_F.u) = GA, dPsi/dB = |u| GA.  B ~ sqrt(A), so
    // the B path adds GA |u| B / (2 A) per unit of dA.  Darcy (B = 0): S = T / c0.
    const float pfu = pfx * n.ux + pfy * n.uy;
    float sx, sy, fac = 1.0f;
    if (M != REV_FORCH || n.B == 0.0f) {
        sx = n.g * pux - n.ag * pfx;
        sy = n.g * puy - n.ag * pfy;
    } else {
        const float un = n.un, hb = 0.5f * n.B * un;
        const float q = un > 0.0f ? pfu * __builtin_amdgcn_rcpf(un) : 0.0f; // u.psi_F / |u|
        const float tx = pux - n.A * pfx - n.B * (un * pfx + q * n.ux);
        const float ty = puy - n.A * pfy - n.B * (un * pfy + q * n.uy);
        const float a = n.c0 + hb;
        // K^-1 = (I - b/(a + b) u u^T / |u|^2) / a with b = B |u| / 2
        const float kap =
            un > 0.0f ? 0.5f * n.B * __builtin_amdgcn_rcpf((a + hb) * un) : 0.0f;
        const float ut = n.ux * tx + n.uy * ty, ia = __builtin_amdgcn_rcpf(a);
        sx = ia * (tx - kap * ut * n.ux);
        sy = ia * (ty - kap * ut * n.uy);
        fac = n.A > 0.0f ? 1.0f + un * n.B * __builtin_amdgcn_rcpf(2.0f * n.A) : 1.0f;
    }
    const float vx = n.jx * n.rinv, vy = n.jy * n.rinv;
    float ga = -0.5f * (sx * n.ux + sy * n.uy) - pfu; // GA / rho
    if (M == REV_FORCH)
        ga *= fac;
    G.jx = sx;
    G.jy = sy;
    G.rho = Pr - (sx * vx + sy * vy);
    if (M == REV_STD || ph.kn_local)
        G.rho -= n.dA_dlnkn * ga;
    const float rga = n.rho * ga;
    G.lnk = -n.A * rga; // dA / d ln k = -A
    G.lnkn = n.dA_dlnkn * rga;
    if (uniform_branch(n.any_solid)) {
        // u = 0, F = -2 j / rho
        G.jx = n.solid ? -2.0f * pfx : G.jx;
        G.jy = n.solid ? -2.0f * pfy : G.jy;
        G.rho = n.solid ? Pr + 2.0f * (pfx * vx + pfy * vy) : G.rho;
        G.lnk = n.solid ? 0.0f : G.lnk;
        G.lnkn = n.solid ? 0.0f : G.lnkn;
    }
    return G;
}

// Adjoint of the collide at one node: lam_f from mu (the adjoint of the
// post-collision populations) and the sensitivity to ln k.
template <int M>
__device__ __forceinline__ Grads collide_adj(const Physics &ph, const NodeFwd &n,
                                             const float (&mu)[9], float (&lf)[9])
{
    const Mom L = moments(mu);
    const float om = ph.omega, cg = ph.guo, ie = n.ie;
    const float ux = n.ux, uy = n.uy, Fx = n.Fx, Fy = n.Fy;
    // psi = omega [L0 + 3 L1.u + u.Q.u / 2] + g [3 L1.F + u.Q.F] with the
    // symmetric Q = (9 L2 - 3 L0 I) / eps, and a = 3 L1 + Q u:
    // psi = omega [L0 + (a.u + 3 L1.u) / 2] + g a.F, psi_u = omega a + g Q F,
    // psi_F = g a
    const float l3 = 3.0f * L.m0;
    const float qxx = ie * (9.0f * L.mxx - l3), qyy = ie * (9.0f * L.myy - l3);
    const float qxy = ie * (9.0f * L.mxy);
    const float ax = 3.0f * L.m1x + (qxx * ux + qxy * uy);
    const float ay = 3.0f * L.m1y + (qxy * ux + qyy * uy);
    const float cx = qxx * Fx + qxy * Fy, cy = qxy * Fx + qyy * Fy;
    const float au = ax * ux + ay * uy, af = ax * Fx + ay * Fy;
    const float lu = L.m1x * ux + L.m1y * uy;
    const float Pr = om * (L.m0 + 0.5f * au + 1.5f * lu) + cg * af; // psi = dPsi/drho
    const Grads G = chain<M>(ph, n, Pr, om * ax + cg * cx, om * ay + cg * cy, cg * ax, cg * ay);
    spread<true>(ph.keep, mu, G.rho, G.jx, G.jy, lf);
    return G;
}

// Adjoint of the read-out share of J at one node, J_x = a1 rho u_x + a2 u_x.
template <int M>
__device__ __forceinline__ Grads readout_adj(const Physics &ph, const NodeFwd &n, float a1,
                                             float a2, float (&lf)[9])
{
    Grads G{0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (!n.solid && (a1 != 0.0f || a2 != 0.0f))
        G = chain<M>(ph, n, a1 * n.ux, a1 + a2 * n.rinv, 0.0f, 0.0f, 0.0f);
    spread<false>(0.0f, nullptr, G.rho, G.jx, G.jy, lf);
    return G;
}

// Adjoint of the pressure-column override
//   f_i(b) = f_eq_i(rho_b, u_n; eps_b) + f_i(n) - f_eq_i(rho_n, u_n; eps_n)
// with respect to the neighbour's post-stream populations f(n) (through
// f(n) itself, rho_n, j_n and u_n(rho_n, j_n, ln k_n)).  Adds to lfn and
// returns the neighbour's ln k and ln kn0 sensitivities.
template <int M>
__device__ __forceinline__ float2 nee_adj(const Physics &ph, const NodeFwd &n, float rho_b,
                                         float ie_b, const float (&lb)[9], float (&lfn)[9])
{
    const Mom L = moments(lb);
    const float ux = n.ux, uy = n.uy, ie = n.ie;
    // Phi(rho, eps) = sum_i lb_i f_eq_i = rho [L0 + 3 L1.u + u.Q.u / 2] with
    // Q as in collide_adj; for eps = 0 it is rho L0.
    const float l3 = 3.0f * L.m0;
    const float pxx = 9.0f * L.mxx - l3, pyy = 9.0f * L.myy - l3, pxy = 9.0f * L.mxy;
    const float px = pxx * ux + pxy * uy, py = pxy * ux + pyy * uy;
    const float lx = 3.0f * L.m1x, ly = 3.0f * L.m1y;
    const float rb = ie_b > 0.0f ? rho_b * n.rinv : 0.0f; // rho_b / rho_n
    const float hx = rb * (lx + ie_b * px) - (lx + ie * px);
    const float hy = rb * (ly + ie_b * py) - (ly + ie * py);
    const float phin = // Phi_n / rho_n
        n.solid ? L.m0 : L.m0 + (lx * ux + ly * uy) + 0.5f * ie * (px * ux + py * uy);
    // Psi = Phi_b(u) - Phi_n(rho_n, u): explicit d/drho_n = -Phi_n / rho_n,
    // d/du = Hu; no direct force dependence.
    const Grads G = chain<M>(ph, n, -phin, hx, hy, 0.0f, 0.0f);
    float gx = G.jx, gy = G.jy, gr = G.rho, gl = G.lnk, gk = G.lnkn;
    if (n.solid) { // u_n = 0 does not move with f(n)
        gx = gy = gl = gk = 0.0f;
        gr = -phin;
    }
    float add[9];
    spread<true>(1.0f, lb, gr, gx, gy, add);
#pragma unroll
    for (int i = 0; i < 9; ++i)
        lfn[i] += add[i];
    return make_float2(gl, gk);
}

__device__ __forceinline__ Rsrc rsrc_row(const void *base, uint64_t row_bytes, int y)
{
    return make_rsrc(static_cast<const char *>(base) + (uint64_t)y * row_bytes,
                     (uint32_t)row_bytes);
}

// Lane-dependent facts of a strip of the reverse pass.
struct ALanes {
    uint32_t x;         // the lane's column, wrapped (periodic) or clamped
    bool wxm, wxp;      // wall x: the column is the first / last
    bool first, last;   // pressure x: the inlet / outlet column
    bool cl, cr;        // pressure x: the column next to the inlet / outlet
    bool has_b;         // uniform: the wave may hold any of these
    bool bgrad;         // pressure columns receive gradient terms (nx >= 3)
};

// lam_f and the ln k / ln kn0 terms of one reverse step at this lane's node
// (adjoint_node's arithmetic, with a pressure column's contribution taken
// from the neighbouring lane rather than recomputed).
template <int BCX, int M>
__device__ __forceinline__ void local_adj(const Physics &ph, const float (&mu)[9], const float (&h)[3],
                                          const float (&md)[3], const ALanes &ln,
                                          float (&lf)[9], float &gl, float &gk)
{
    const NodeFwd n = node_fwd<M>(ph, h[0], h[1], h[2], md[0], md[1], md[2]);
    const Grads G = collide_adj<M>(ph, n, mu, lf);
    gl = G.lnk;
    gk = G.lnkn;
    if (BCX != BC_PRESSURE)
        return;
    if (ln.has_b) {
        // the pressure columns' lam_f as computed so far (never changed by
        // the carries below, which only touch the columns next to them)
        float lb[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            lb[i] = lane_from<1>(lf[i]);
        float rb = lane_from<1>(n.rho), eb = lane_from<1>(n.ie);
        if (ln.cl) {
            const float2 q = nee_adj<M>(ph, n, rb, eb, lb, lf);
            gl += q.x;
            gk += q.y;
        }
#pragma unroll
        for (int i = 0; i < 9; ++i)
            lb[i] = lane_from<-1>(lf[i]);
        rb = lane_from<-1>(n.rho);
        eb = lane_from<-1>(n.ie);
        if (ln.cr) {
            const float2 q = nee_adj<M>(ph, n, rb, eb, lb, lf);
            gl += q.x;
            gk += q.y;
        }
    }
    if (ln.first || ln.last) {
        // forward values pulled into a pressure column are discarded
#pragma unroll
        for (int i = 0; i < 9; ++i)
            lf[i] = 0.0f;
        if (!ln.bgrad)
            gl = gk = 0.0f;
    }
}

// mu of this lane's node from lam_f of rows y - 1 (dn), y (c), y + 1 (up).
// wym / wyp: the row below / above lies beyond a wall.
template <int BCX>
__device__ __forceinline__ void gather(const float (&dn)[9], const float (&c)[9],
                                       const float (&up)[9], bool wym, bool wyp,
                                       const ALanes &ln, float (&mu)[9])
{
    mu[0] = c[0];
#pragma unroll
    for (int j = 1; j < 9; ++j) {
        const int ex = ex_of(j), ey = ey_of(j);
        const bool wall_y = (ey == 1 && wyp) || (ey == -1 && wym); // uniform
        const float(&r)[9] = ey == 1 ? up : (ey == -1 ? dn : c);
        float v;
        if (wall_y)
            v = c[opp_of(j)];
        else if (ex == 1)
            v = lane_from<-1>(r[j]);
        else if (ex == -1)
            v = lane_from<1>(r[j]);
        else
            v = r[j];
        if (BCX == BC_WALL) {
            const bool out_x = (ex == 1 && ln.wxp) || (ex == -1 && ln.wxm);
            if (out_x)
                v = c[opp_of(j)];
        }
        if (BCX == BC_PRESSURE) {
            const bool out_x = (ex == 1 && ln.last) || (ex == -1 && ln.first);
            if (out_x)
                v = 0.0f;
        }
        mu[j] = v;
    }
}

} // namespace

} // namespace lbk
