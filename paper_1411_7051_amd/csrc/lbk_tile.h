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
// What bounds it: on lattices that fill the device, the vector issue (16 x 2
// rows and K = 4 recompute 1.33 updates per node and step and keep eight waves
// per SIMD: 4096 x 4096 FP32 runs at 108 us a step, against 128 in three-step
// marching passes with three waves per SIMD, 176 in two-step passes and 237 in
// single sweeps); on small ones a launch's fixed 4 us.  Two rows a wave are
// what 64 registers hold (a third makes the device run four waves per SIMD
// instead of eight, which measured slower at every size).  MODEL_STD, the
// default model under a pressure drive, is compiled apart: 57 instead of 64
// registers and about 145 instead of 165 vector instructions an update (108
// against 119 us).
#pragma once

#include "lbk_sweep.h"

namespace lbk {

// What one wave's row gives its y neighbour in another wave: the density and
// the populations that cross (2, 5, 6 upwards, 4, 7, 8 downwards).
struct Edge {
    float rho[64];
    uint32_t h[3][64]; // Elem<T>::Reg as bits
};
__device__ __forceinline__ uint32_t reg_bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t reg_bits(uint32_t v) { return v; }
__device__ __forceinline__ void bits_reg(uint32_t b, float &v) { v = __uint_as_float(b); }
__device__ __forceinline__ void bits_reg(uint32_t b, uint32_t &v) { v = b; }

// One workgroup's tile: strip `strip` by band `band` of a lattice cut for
// `halo` >= steps halo nodes on each side (waves, R), advanced `steps` steps.
template <typename T, int BCX, int BCY, bool HIST, int R, int MODEL>
__device__ __forceinline__ void tile_steps(const char *__restrict__ src, char *__restrict__ dst,
                                           const Layout &lay, const char *__restrict__ med,
                                           const MLayout &mlay, const Geom &g, const Physics &ph,
                                           float s, float inv_s, int halo, int steps, int strip,
                                           int band, float *__restrict__ hist,
                                           uint64_t hist_bytes, Edge *__restrict__ edges)
{
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    const int own_x = 64 - 2 * halo, H = waves * R, own_y = H - 2 * halo;
    const int nstrips = (g.nx + own_x - 1) / own_x;
    if (strip >= nstrips)
        return; // the whole workgroup
    const int xr = strip * own_x - halo + lane;
    Lanes ln;
    if (BCX == BC_PERIODIC)
        ln.x = (uint32_t)(((xr % g.nx) + g.nx) % g.nx);
    else
        ln.x = (uint32_t)(xr < 0 ? 0 : (xr >= g.nx ? g.nx - 1 : xr)); // beyond: unused copies
    // As in the marching passes, an outlet column at the first lane of a
    // strip is left to the previous strip, which completes its neighbour's
    // pull.
    bool owned = lane >= halo && lane < halo + own_x && xr < g.nx;
    if (BCX == BC_PRESSURE && xr == g.nx - 1)
        owned = lane >= halo + 1 && lane <= halo + own_x;
    ln.wxm = BCX == BC_WALL && ln.x == 0;
    ln.wxp = BCX == BC_WALL && ln.x == (uint32_t)g.nx - 1;
    ln.bin = BCX == BC_PRESSURE && xr == 0;
    ln.bout = BCX == BC_PRESSURE && xr == g.nx - 1;
    ln.has_b = BCX == BC_PRESSURE && any_lane(ln.bin || ln.bout);
    const int y0 = band * own_y, y1 = min(y0 + own_y, g.ny);
    // tile row j is the lattice's row y0 - halo + j; rows beyond a wall
    // hold copies that the bounce-back never reads
    const int j0 = wave * R;
    auto row_of = [&](int j) { return y0 - halo + j; };
    auto held = [&](int y) {
        return BCY == BC_PERIODIC ? ((y % g.ny) + g.ny) % g.ny
                                  : (y < 0 ? 0 : (y >= g.ny ? g.ny - 1 : y));
    };
    Mid<T> a[R];
    bool solids = false; // whether any of the wave's nodes is impermeable
#pragma unroll
    for (int r = 0; r < R; ++r) {
        load_node<T, MODEL>(src, lay, med, mlay, held(row_of(j0 + r)), ln.x, a[r]);
        solids = solids || any_lane(!(a[r].e > 0.0f));
    }
    Edge *lo = edges, *hi = edges + 2 * waves; // [parity][wave]: first and last rows
    for (int k = 0; k < steps; ++k) {
        const int p = (k & 1) * waves;
        if (waves > 1) {
            Edge &f = lo[p + wave], &l = hi[p + wave];
            f.rho[lane] = a[0].rho;
            f.h[0][lane] = reg_bits(a[0].h[4]);
            f.h[1][lane] = reg_bits(a[0].h[7]);
            f.h[2][lane] = reg_bits(a[0].h[8]);
            l.rho[lane] = a[R - 1].rho;
            l.h[0][lane] = reg_bits(a[R - 1].h[2]);
            l.h[1][lane] = reg_bits(a[R - 1].h[5]);
            l.h[2][lane] = reg_bits(a[R - 1].h[6]);
            __syncthreads();
        }
        // rows k + 1 .. H - 2 - k of the tile are complete after this step; a
        // wave with none of them, or none in the lattice's rows that remain
        // to be stored, has nothing to do
        if (j0 + R <= k + 1 || j0 > H - 2 - k)
            continue;
        Mid<T> dn = a[0], up = a[R - 1];
        if (wave > 0) {
            const Edge &e = hi[p + wave - 1];
            dn.rho = e.rho[lane];
            bits_reg(e.h[0][lane], dn.h[2]);
            bits_reg(e.h[1][lane], dn.h[5]);
            bits_reg(e.h[2][lane], dn.h[6]);
        }
        if (wave < waves - 1) {
            const Edge &e = lo[p + wave + 1];
            up.rho = e.rho[lane];
            bits_reg(e.h[0][lane], up.h[4]);
            bits_reg(e.h[1][lane], up.h[7]);
            bits_reg(e.h[2][lane], up.h[8]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = row_of(j0 + r);
            const Mid<T> old = a[r];
            float hs[9], jx, jy;
            const float rho = step_from<T, BCX, MODEL>(
                ph, s, inv_s, dn, old, r + 1 < R ? a[r + 1] : up, BCY == BC_WALL && y == 0,
                BCY == BC_WALL && y == g.ny - 1, ln, solids, hs, jx, jy);
            if (HIST && owned && y >= y0 && y < y1)
                record(reinterpret_cast<float *>(reinterpret_cast<char *>(hist) +
                                                 (uint64_t)k * hist_bytes),
                       g, y, ln.x, rho, jx, jy, false);
            a[r].rho = rho;
#pragma unroll
            for (int i = 0; i < 9; ++i)
                a[r].h[i] = Elem<T>::reg(hs[i]);
            dn = old;
        }
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

} // namespace lbk
