// lbk_adjoint_tile.hip -- several reverse steps of a lattice in one launch:
// the tile pass of the forward sweep run backwards.
//
// A workgroup of W waves holds the adjoint state of a tile of 64 columns by
// W x R rows in registers, takes it K steps back and stores the nodes K or more
// away from its edges.  Per step it reads the 12 B history of each node (one
// step ahead of its use), forms lam_f of every row still wanted, exchanges the
// first and last rows' crossing components between waves through LDS (two
// alternating buffers, one barrier a step) and gathers the next adjoint state.
// The gradient terms of all K steps are added in registers, in the order of
// single reverse steps, and written once.  Bitwise K single reverse steps.
//
// What bounds it: on a large lattice the bytes of the tiles (152 B a node of a
// tile and pass of three steps, 64 B per node and step with the halos, at 5.4
// TB/s); on a small one the launch and the chain of steps, as in the forward
// pass.  Two rows a wave keep 98 registers, four waves a SIMD; at 96 and five
// waves a SIMD (a few spills) nothing was gained.  Measured against the
// marching pairs (two waves a SIMD): 50 us a step for 60 at 2048 x 2048, 179 for
// 216 at 4096 x 4096, 14.6 for 24 at 2048 x 512 (22 in single steps); against
// single steps 2.9 us for 5.5 at 384 x 256, 2.2 for 4.4 at 64 x 32.
// Tiles in the order of rows of tiles: columns of tiles first (1, 2, 4 or 8
// strips wide) was slower, 55 to 57 us at 2048 x 2048 where rows took 50.
#include "lbk_adjoint_dev.h"

namespace lbk {

namespace {

// What a wave's first and last rows give the rows below and above them.
struct AEdges {
    float first[3][64], last[3][64]; // lam_f 2, 5, 6 and 4, 7, 8
};
constexpr size_t kATileLds = 2 * (size_t)kTileMaxWaves * sizeof(AEdges);

// EDGE: rows at a wall may be among the tile's.
template <int BCX, int BCY, bool KN, int M, int R, bool EDGE>
__device__ __forceinline__ void adj_tile(const float *__restrict__ mu_in,
                                         float *__restrict__ mu_out,
                                         const float *__restrict__ hist, uint64_t hist_bytes,
                                         const char *__restrict__ med, const MLayout &mlay,
                                         float *__restrict__ grad, float *__restrict__ grad2,
                                         const Geom &g, const Physics &ph, int steps, int strip,
                                         int band, AEdges *__restrict__ edges)
{
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    const int nx = g.nx, ny = g.ny;
    const int own_x = 64 - 2 * steps, H = waves * R, own_y = H - 2 * steps;
    const int nstrips = (nx + own_x - 1) / own_x;
    // Strip s owns columns [c0, c1).  A pressure column's contribution goes
    // to the column next to it, one lane further than a gather reaches: with
    // the column next to the outlet on lane 63 its values would be wrong from
    // the first step on, and the strip's last column after the last, so the
    // last strip starts at most at nx - 2 - steps and the one before ends there.
    int c0 = strip * own_x, c1 = min(c0 + own_x, nx);
    if (BCX == BC_PRESSURE) {
        const int cl = max(0, min(own_x * (nstrips - 1), nx - 2 - steps));
        if (strip == nstrips - 1)
            c0 = cl;
        else if (strip == nstrips - 2)
            c1 = cl;
    }
    const int xr = c0 - steps + lane;
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
    ln.has_b = BCX == BC_PRESSURE &&
               __builtin_amdgcn_ballot_w64(ln.first || ln.last || ln.cl || ln.cr) != 0;
    ln.bgrad = nx >= 3;
    const int y0 = band * own_y, y1 = min(y0 + own_y, ny);
    const int j0 = wave * R;
    auto row_of = [&](int j) { return y0 - steps + j; };
    // a row that always exists; rows beyond a wall hold copies that the
    // gather never reads
    auto held = [&](int y) {
        if (BCY != BC_PERIODIC)
            return y < 0 ? 0 : (y >= ny ? ny - 1 : y);
        while (y < 0)
            y += ny;
        while (y >= ny)
            y -= ny;
        return y;
    };
    const uint64_t lrow = 9ull * g.pitch * 4, hrow = 3ull * g.pitch * 4;
    const uint64_t grow = (uint64_t)g.pitch * 4;
    const uint32_t slot = (uint32_t)g.pitch * 4;
    const uint32_t xo = ln.x * 4;
    auto load_hist = [&](int k, float (&h)[R][3]) {
        const char *base = reinterpret_cast<const char *>(hist) - (uint64_t)k * hist_bytes;
#pragma unroll
        for (int r = 0; r < R; ++r)
            ld_hist<0>(rsrc_row(base, hrow, held(row_of(j0 + r))), ln.x * 12, h[r]);
    };
    float mu[R][9], md[R][3], gp[R], gk[R], ha[R][3], hb[R][3];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = row_of(j0 + r), yh = held(y);
        const Rsrc lr = rsrc_row(mu_in, lrow, yh);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            mu[r][i] = ld_f32(lr, xo, i * slot);
        const Rsrc mr = rsrc_row(med, mlay.row, yh);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            md[r][k] = ld_f32(mr, xo, k * mlay.slot);
        if (M == REV_STD)
            md[r][0] = inv_eps(md[r][0]);
        const bool mine = y >= y0 && y < y1;
        gp[r] = mine ? ld_f32(rsrc_row(grad, grow, yh), xo, 0) : 0.0f;
        gk[r] = KN && mine ? ld_f32(rsrc_row(grad2, grow, yh), xo, 0) : 0.0f;
    }
    load_hist(0, ha);
    // The first wave's lower and the last wave's upper neighbours lie outside
    // the tile: they read their own edges, into rows that are never stored.
    AEdges *const mine = edges + wave;
    const float(*const below)[64] = wave > 0 ? edges[wave - 1].last : mine->last;
    const float(*const above)[64] = wave < waves - 1 ? edges[wave + 1].first : mine->first;
    // Reverse step k; the buffer of the edges is k & 1, a constant of the code.
    auto step = [&](int k, auto parity, float (&h)[R][3], float (&hn)[R][3]) {
        constexpr int P = decltype(parity)::value * kTileMaxWaves;
        constexpr int PF = P * (int)(sizeof(AEdges) / sizeof(float[64]));
        if (k + 1 < steps)
            load_hist(k + 1, hn);
        // lam_f is wanted of rows k .. H - 1 - k, the next state of one less
        // on either side
        const int lo = k, hi = H - 1 - k;
        float lf[R][9];
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (j0 + r >= lo && j0 + r <= hi) {
                float gl, gn;
                local_adj<BCX, M>(ph, mu[r], h[r], md[r], ln, lf[r], gl, gn);
                gp[r] += gl;
                if (KN)
                    gk[r] += gn;
            }
        AEdges &m = mine[P];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            m.first[i][lane] = lf[0][i == 0 ? 2 : (i == 1 ? 5 : 6)];
            m.last[i][lane] = lf[R - 1][i == 0 ? 4 : (i == 1 ? 7 : 8)];
        }
        __syncthreads();
        if (j0 + R <= lo + 1 || j0 > hi - 1)
            return;
        float dn[9], up[9]; // the components a gather reads of them
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            dn[i == 0 ? 4 : (i == 1 ? 7 : 8)] = below[PF + i][lane];
            up[i == 0 ? 2 : (i == 1 ? 5 : 6)] = above[PF + i][lane];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = row_of(j0 + r);
            gather<BCX>(r > 0 ? lf[r - 1] : dn, lf[r], r + 1 < R ? lf[r + 1] : up, EDGE && y == 0,
                        EDGE && y == ny - 1, ln, mu[r]);
        }
    };
    for (int k = 0; k < steps; k += 2) {
        step(k, std::integral_constant<int, 0>{}, ha, hb);
        if (k + 1 < steps)
            step(k + 1, std::integral_constant<int, 1>{}, hb, ha);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = row_of(j0 + r);
        if (y < y0 || y >= y1)
            continue;
        if (owned) {
            const Rsrc out = rsrc_row(mu_out, lrow, y);
#pragma unroll
            for (int i = 0; i < 9; ++i)
                st_f32(out, xo, i * slot, mu[r][i], false);
            st_f32(rsrc_row(grad, grow, y), xo, 0, gp[r], false);
            if (KN)
                st_f32(rsrc_row(grad2, grow, y), xo, 0, gk[r], false);
        }
    }
}

} // namespace

template <int BCX, int BCY, bool KN, int M, int R>
__global__ __launch_bounds__(kTileMaxWaves * 64, 4) void adjoint_tile_kernel(
    const float *__restrict__ mu_in, float *__restrict__ mu_out, const float *__restrict__ hist,
    uint64_t hist_bytes, const char *__restrict__ med, MLayout mlay, float *__restrict__ grad,
    float *__restrict__ grad2, Geom g, Physics ph, int steps, int strips)
{
    extern __shared__ AEdges aedges[]; // [parity][kTileMaxWaves]
    const int L = xcd_remap_a(blockIdx.x, gridDim.x);
    const int band = L / strips, strip = L - band * strips;
    const int H = (int)(blockDim.x >> 6) * R, top = band * (H - 2 * steps) - steps;
    if (BCY == BC_WALL && (top <= 0 || top + H >= g.ny))
        adj_tile<BCX, BCY, KN, M, R, BCY == BC_WALL>(mu_in, mu_out, hist, hist_bytes, med, mlay,
                                                     grad, grad2, g, ph, steps, strip, band,
                                                     aedges);
    else
        adj_tile<BCX, BCY, KN, M, R, false>(mu_in, mu_out, hist, hist_bytes, med, mlay, grad,
                                            grad2, g, ph, steps, strip, band, aedges);
}

// REV_FORCH is compiled for one row a wave only: with its registers two rows
// gain nothing.
#define LBK_ATILE_RKF(LAUNCH)                                                                \
    if (model == REV_FORCH) {                                                                \
        if (kn)                                                                              \
            LAUNCH(true, REV_FORCH, 1);                                                      \
        else                                                                                 \
            LAUNCH(false, REV_FORCH, 1);                                                     \
    } else if (model == REV_STD) {                                                           \
        LBK_ATILE_RK(LAUNCH, REV_STD)                                                        \
    } else {                                                                                 \
        LBK_ATILE_RK(LAUNCH, REV_DARCY)                                                      \
    }                                                                                        \
    return hipGetLastError();
#define LBK_ATILE_RK(LAUNCH, MODEL)                                                          \
    if (rows == 1) {                                                                         \
        if (kn)                                                                              \
            LAUNCH(true, MODEL, 1);                                                          \
        else                                                                                 \
            LAUNCH(false, MODEL, 1);                                                         \
    } else {                                                                                 \
        if (kn)                                                                              \
            LAUNCH(true, MODEL, 2);                                                          \
        else                                                                                 \
            LAUNCH(false, MODEL, 2);                                                         \
    }

#define LBK_ATILE_BC(FN, ...)                                                                \
    switch (bcx * 2 + bcy) {                                                                 \
    case 0: return FN<BC_PERIODIC, BC_PERIODIC>(__VA_ARGS__);                                \
    case 1: return FN<BC_PERIODIC, BC_WALL>(__VA_ARGS__);                                    \
    case 2: return FN<BC_WALL, BC_PERIODIC>(__VA_ARGS__);                                    \
    case 3: return FN<BC_WALL, BC_WALL>(__VA_ARGS__);                                        \
    case 4: return FN<BC_PRESSURE, BC_PERIODIC>(__VA_ARGS__);                                \
    case 5: return FN<BC_PRESSURE, BC_WALL>(__VA_ARGS__);                                    \
    default: return hipErrorInvalidValue;                                                    \
    }

template <int BCX, int BCY>
static hipError_t adj_tile_t(const float *mu_in, float *mu_out, const float *hist,
                             uint64_t hist_bytes, const char *med, const MLayout &mlay,
                             float *grad, float *grad2, const Geom &g, const Physics &ph,
                             const Tile &t, int steps, hipStream_t st)
{
    const int own_x = 64 - 2 * steps, own_y = t.waves * t.rows - 2 * steps, rows = t.rows;
    const int strips = (g.nx + own_x - 1) / own_x, bands = (g.ny + own_y - 1) / own_y;
    const bool kn = grad2 != nullptr;
    const int model = rev_model(ph);
#define LBK_ATILE(KN, M, R)                                                                 \
    hipLaunchKernelGGL((adjoint_tile_kernel<BCX, BCY, KN, M, R>),                           \
                       dim3((unsigned)(strips * bands)), dim3(t.waves * 64), kATileLds, st,  \
                       mu_in, mu_out, hist, hist_bytes, med, mlay, grad, grad2, g, ph, steps, \
                       strips)
    LBK_ATILE_RKF(LBK_ATILE)
#undef LBK_ATILE
}

hipError_t launch_adjoint_tile(int bcx, int bcy, const float *mu_in, float *mu_out,
                               const float *hist, uint64_t hist_bytes, const char *med,
                               const MLayout &mlay, float *grad, float *grad2, const Geom &g,
                               const Physics &ph, const Tile &t, int steps, hipStream_t st)
{
    const bool fits = t.waves >= 2 && t.waves <= kTileMaxWaves && (t.rows == 1 || t.rows == 2) &&
                      (t.rows == 1 || rev_model(ph) != REV_FORCH) && steps >= 1 &&
                      2 * steps < 64 && 2 * steps < t.waves * t.rows;
    if (!fits || bcy < 0 || bcy > 1)
        return hipErrorInvalidValue;
    LBK_ATILE_BC(adj_tile_t, mu_in, mu_out, hist, hist_bytes, med, mlay, grad, grad2, g, ph, t,
                 steps, st)
}

} // namespace lbk
