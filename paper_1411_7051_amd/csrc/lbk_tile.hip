// lbk_tile.hip -- the tile pass (lbk_tile.h) of one lattice.
#include "lbk_tile.h"

namespace lbk {

template <typename T, int BCX, int BCY, bool HIST, int R, int MODEL>
__global__ __launch_bounds__(kTileMaxWaves * 64, 8) void tile_kernel(
    const char *__restrict__ src, char *__restrict__ dst, Layout lay,
    const char *__restrict__ med, MLayout mlay, Geom g, Physics ph, float s, float inv_s,
    int steps, int strips, float *__restrict__ hist, uint64_t hist_bytes)
{
    extern __shared__ Edges edges[]; // [parity][kTileMaxWaves]
    const int L = xcd_remap(blockIdx.x, gridDim.x);
    const int band = L / strips, strip = L - band * strips;
    tile_steps<T, BCX, BCY, HIST, R, MODEL>(src, dst, lay, med, mlay, g, ph, s, inv_s, steps, 0,
                                            steps, strip, band, hist, hist_bytes, edges);
}

template <typename T, int BCX, int BCY>
static hipError_t tile_t(const char *src, char *dst, const Layout &lay, const char *med,
                         const MLayout &mlay, const Geom &g, const Physics &ph, float s,
                         float inv_s, const Tile &t, int steps, float *hist, uint64_t hist_bytes,
                         hipStream_t st)
{
    const int own_x = 64 - 2 * steps, own_y = t.waves * t.rows - 2 * steps;
    const int strips = (g.nx + own_x - 1) / own_x, bands = (g.ny + own_y - 1) / own_y;
    const dim3 grid((unsigned)(strips * bands)), block(t.waves * 64);
    const size_t lds = kTileLds;
#define LBK_TILE(HIST, R)                                                                    \
    do {                                                                                     \
        if (BCX == BC_PRESSURE && ph.standard)                                               \
            hipLaunchKernelGGL((tile_kernel<T, BCX, BCY, HIST, R,                            \
                                            BCX == BC_PRESSURE ? MODEL_STD : MODEL_GEN>),    \
                               grid, block, lds, st, src, dst, lay, med, mlay, g, ph, s,     \
                               inv_s, steps, strips, hist, hist_bytes);                      \
        else                                                                                 \
            hipLaunchKernelGGL((tile_kernel<T, BCX, BCY, HIST, R, MODEL_GEN>), grid, block,  \
                               lds, st, src, dst, lay, med, mlay, g, ph, s, inv_s, steps,    \
                               strips, hist, hist_bytes);                                    \
    } while (0)
    if (t.rows == 1) {
        if (hist)
            LBK_TILE(true, 1);
        else
            LBK_TILE(false, 1);
    } else {
        if (hist)
            LBK_TILE(true, 2);
        else
            LBK_TILE(false, 2);
    }
#undef LBK_TILE
    return hipGetLastError();
}

hipError_t launch_tile(int storage, int bcx, int bcy, const char *src, char *dst,
                       const Layout &lay, const char *med, const MLayout &mlay, const Geom &g,
                       const Physics &ph, float s, float inv_s, const Tile &t, int steps,
                       float *hist, uint64_t hist_bytes, hipStream_t st)
{
    if (bcy < 0 || bcy > 1 || steps < 1 || t.waves < 2 || t.waves > kTileMaxWaves ||
        (t.rows != 1 && t.rows != 2) || 64 - 2 * steps < 1 ||
        t.waves * t.rows - 2 * steps < 1)
        return hipErrorInvalidValue;
    LBK_DISPATCH(tile_t, src, dst, lay, med, mlay, g, ph, s, inv_s, t, steps, hist, hist_bytes,
                 st)
}

} // namespace lbk
