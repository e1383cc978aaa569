// lbk_tile.h -- the tile pass: several time steps of a lattice in one launch.
//
// Below about a million nodes a sweep is not bound by HBM (its levels stay in
// the on-package cache) but by what surrounds the arithmetic: a launch, the
// latency of one wave's loads, the drain of its stores.  A 64 x 32 lattice
// took 3.0 us a step and 1024 x 512 10.2 us, where the arithmetic of the
// latter is 2.7 us of the device's vector issue.  The tile pass pays for
// launch, load and store once per K steps: a workgroup loads a tile of 64
// columns by W x R rows (W waves, R rows each, the whole tile in registers),
// advances it K steps and stores the nodes K or more away from the tile's
// edges, which are the ones whose neighbourhood it held.  Within a step the x
// neighbours come from the adjacent lanes (DPP), the y neighbours from the
// wave's own rows and, across waves, from LDS: a wave leaves the densities and
// the three populations that move on of its first and last row there, in two
// alternating buffers, so one barrier a step is enough.  The rows and columns
// around a tile are advanced by the neighbouring tiles too; a wave whose rows
// no longer reach a stored node rests.
//
// Each step is the node update of the single sweep on values rounded as a
// store would round them, so K steps are bitwise K single sweeps.
//
// What bounds it: on lattices that fill the device, the vector issue (on
// 4096 x 4096 85 to 86% of the issue slots at FP32, beside 4.8 TB/s of HBM
// traffic, 96 to 97% at FP16 and 99% at BF16; 16 x 2 rows and K = 4 make 1.30
// updates per node and step), with eight waves per SIMD: FP32 95 us a step there
// against 124 in three-step marching passes (three waves per SIMD), 174 in
// two-step passes and 234 in single sweeps, FP16 95 against 106, 123 and 149 (one
// device; another took 99 and 97); on small ones a launch's fixed 4 us.  Two rows
// a wave are what 64 registers hold (with three or four the device runs half
// the waves, which measured slower at every size).  What an update does not
// need is kept out of it: a row beyond the rows still wanted is skipped, LDS
// addresses are constants of the code (the two buffers' steps are unrolled),
// only tiles at a wall carry the bounce-back selects and only waves that hold a
// pressure column the exchange with its neighbour (a sixth of the time in all,
// with the next).  MODEL_STD, the default model under a pressure drive, is
// compiled apart: 148 vector instructions an update at FP32, loads and stores of
// the tile included.
#pragma once

#include "lbk_sweep.h"

namespace lbk {

// What one wave's row gives its y neighbour in another wave: the density and
// the populations that cross (4, 7, 8 downwards from its first row, 2, 5, 6
// upwards from its last), Elem<T>::Reg as bits.
struct Edge {
    float rho[64];
    uint32_t h[3][64];
};
// The edges a workgroup exchanges at one step: [parity][wave], its first and
// last rows.
struct Edges {
    Edge first, last;
};
__device__ __forceinline__ uint32_t reg_bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t reg_bits(uint32_t v) { return v; }
__device__ __forceinline__ void bits_reg(uint32_t b, float &v) { v = __uint_as_float(b); }
__device__ __forceinline__ void bits_reg(uint32_t b, uint32_t &v) { v = b; }
constexpr size_t kTileLds = 2 * (size_t)kTileMaxWaves * sizeof(Edges);

// One workgroup's tile: strip `strip` by band `band` of a lattice cut for
// `halo` >= steps halo nodes on each side (waves, R), advanced `steps` steps.
// EDGE: rows at a wall may be among the tile's (the selects of the bounce-back
// are twelve instructions a row update that other tiles are spared).
template <typename T, int BCX, int BCY, bool HIST, int R, int MODEL, bool EDGE>
__device__ __forceinline__ void tile_advance(const char *__restrict__ src, char *__restrict__ dst,
                                           const Layout &lay, const char *__restrict__ med,
                                           const MLayout &mlay, const Geom &g, const Physics &ph,
                                           float s, float inv_s, int halo, int org, int steps,
                                           int strip, int band, float *__restrict__ hist,
                                           uint64_t hist_bytes, Edges *__restrict__ edges)
{
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    const int own_x = 64 - 2 * halo, H = waves * R, own_y = H - 2 * halo;
    const int nstrips = (g.nx + own_x - 1) / own_x;
    if (strip >= nstrips)
        return; // the whole workgroup
    // org > 0: that many columns of the outlet's end lie left of the inlet in
    // strip 0, which then holds both pressure columns.  Nothing is pulled across
    // this seam, as a pressure column takes its neighbour's pull.
    const int xr = strip * own_x - org - halo + lane;
    Lanes ln;
    if (BCX == BC_PERIODIC)
        ln.x = (uint32_t)(((xr % g.nx) + g.nx) % g.nx);
    else // beyond: unused copies
        ln.x = (uint32_t)(xr < 0 ? (org ? xr + g.nx : 0) : (xr >= g.nx ? g.nx - 1 : xr));
    // Without the seam, as in the marching passes, an outlet column at the
    // first lane of a strip is left to the previous strip, which completes its
    // neighbour's pull.
    bool owned = lane >= halo && lane < halo + own_x && xr < g.nx - org;
    if (BCX == BC_PRESSURE && !org && xr == g.nx - 1)
        owned = lane >= halo + 1 && lane <= halo + own_x;
    ln.wxm = BCX == BC_WALL && ln.x == 0;
    ln.wxp = BCX == BC_WALL && ln.x == (uint32_t)g.nx - 1;
    ln.bin = BCX == BC_PRESSURE && xr == 0;
    ln.bout = BCX == BC_PRESSURE && xr == (org ? -1 : g.nx - 1);
    ln.has_b = BCX == BC_PRESSURE && any_lane(ln.bin || ln.bout) ? 1 : 0;
    const int y0 = band * own_y, y1 = min(y0 + own_y, g.ny);
    // tile row j is the lattice's row y0 - halo + j; rows beyond a wall
    // hold copies that the bounce-back never reads
    const int j0 = wave * R;
    auto row_of = [&](int j) { return y0 - halo + j; };
    auto held = [&](int y) {
        if (BCY != BC_PERIODIC)
            return y < 0 ? 0 : (y >= g.ny ? g.ny - 1 : y);
        while (y < 0) // uniform; more than once only where ny is below the tile's rows
            y += g.ny;
        while (y >= g.ny)
            y -= g.ny;
        return y;
    };
    Mid<T> a[R];
    int solids = 0; // whether any of the wave's nodes is impermeable (an int: a
                    // flag kept as a lane mask costs two instructions a test)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        load_node<T, MODEL>(src, lay, med, mlay, held(row_of(j0 + r)), ln.x, a[r]);
        solids |= any_lane(!(a[r].e > 0.0f)) ? 1 : 0;
    }
    // The first wave's lower and the last wave's upper neighbours lie outside
    // the tile: they read their own edges, into rows that are never stored.
    Edges *const mine = edges + wave;
    const Edge *const below = wave > 0 ? &edges[wave - 1].last : &mine->last;
    const Edge *const above = wave < waves - 1 ? &edges[wave + 1].first : &mine->first;
    // Step k; P = k & 1 is the buffer of the edges, a constant of the code, so
    // that no LDS address is computed in the loop.
    auto step = [&](int k, auto parity) {
        constexpr int P = decltype(parity)::value * kTileMaxWaves; // edges per buffer
        Edges &m = mine[P];
        m.first.rho[lane] = a[0].rho;
        m.first.h[0][lane] = reg_bits(a[0].h[4]);
        m.first.h[1][lane] = reg_bits(a[0].h[7]);
        m.first.h[2][lane] = reg_bits(a[0].h[8]);
        m.last.rho[lane] = a[R - 1].rho;
        m.last.h[0][lane] = reg_bits(a[R - 1].h[2]);
        m.last.h[1][lane] = reg_bits(a[R - 1].h[5]);
        m.last.h[2][lane] = reg_bits(a[R - 1].h[6]);
        __syncthreads();
        // rows k + 1 .. H - 2 - k of the tile are complete after this step;
        // the others have nothing to do
        const int lo = k + 1, hi = H - 2 - k;
        if (j0 + R <= lo || j0 > hi)
            return;
        const Edge &d = reinterpret_cast<const Edges *>(below)[P].first;
        const Edge &u = reinterpret_cast<const Edges *>(above)[P].first;
        Mid<T> dn, up; // the values a pull reads of them
        dn.rho = d.rho[lane];
        bits_reg(d.h[0][lane], dn.h[2]);
        bits_reg(d.h[1][lane], dn.h[5]);
        bits_reg(d.h[2][lane], dn.h[6]);
        up.rho = u.rho[lane];
        bits_reg(u.h[0][lane], up.h[4]);
        bits_reg(u.h[1][lane], up.h[7]);
        bits_reg(u.h[2][lane], up.h[8]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const Mid<T> old = a[r];
            if (R == 1 || (j0 + r >= lo && j0 + r <= hi)) {
                const int y = row_of(j0 + r);
                float hs[9], jx, jy;
                const float rho = step_from<T, BCX, MODEL>(
                    ph, s, inv_s, dn, old, r + 1 < R ? a[r + 1] : up, EDGE && y == 0,
                    EDGE && y == g.ny - 1, ln, solids != 0, hs, jx, jy);
                if (HIST && owned && y >= y0 && y < y1)
                    record(reinterpret_cast<float *>(reinterpret_cast<char *>(hist) +
                                                     (uint64_t)k * hist_bytes),
                           g, y, ln.x, rho, jx, jy, false);
                a[r].rho = rho;
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    a[r].h[i] = Elem<T>::reg(hs[i]);
            }
            dn = old;
        }
    };
    for (int k = 0; k < steps; k += 2) {
        step(k, std::integral_constant<int, 0>{});
        if (k + 1 < steps)
            step(k + 1, std::integral_constant<int, 1>{});
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = row_of(j0 + r);
        if (y < y0 || y >= y1)
            continue;
        if (owned) {
            const Rsrc out = make_rsrc(dst + (uint64_t)y * lay.row, (uint32_t)lay.row);
            st_f32(out, ln.x * 4, 0, a[r].rho, false);
            constexpr uint32_t es = sizeof(T);
#pragma unroll
            for (int i = 0; i < 9; ++i)
                Elem<T>::template str<0>(out, ln.x * es, lay.h_off + i * lay.h_slot, a[r].h[i]);
        }
    }
}

template <typename T, int BCX, int BCY, bool HIST, int R, int MODEL>
__device__ __forceinline__ void tile_steps(const char *__restrict__ src, char *__restrict__ dst,
                                           const Layout &lay, const char *__restrict__ med,
                                           const MLayout &mlay, const Geom &g, const Physics &ph,
                                           float s, float inv_s, int halo, int org, int steps,
                                           int strip, int band, float *__restrict__ hist,
                                           uint64_t hist_bytes, Edges *__restrict__ edges)
{
    const int H = (int)(blockDim.x >> 6) * R, top = band * (H - 2 * halo) - halo;
    if (BCY == BC_WALL && (top <= 0 || top + H >= g.ny))
        tile_advance<T, BCX, BCY, HIST, R, MODEL, BCY == BC_WALL>(
            src, dst, lay, med, mlay, g, ph, s, inv_s, halo, org, steps, strip, band, hist,
            hist_bytes, edges);
    else
        tile_advance<T, BCX, BCY, HIST, R, MODEL, false>(src, dst, lay, med, mlay, g, ph, s,
                                                         inv_s, halo, org, steps, strip, band, hist,
                                                         hist_bytes, edges);
}

} // namespace lbk
