// lbk_tile_batch.hip -- the tile pass (lbk_tile.h) over every sample of a
// batch: one workgroup per entry of a tile list cut for the batch's tile shape
// and step count.  A pass of fewer steps uses the same list.
#include "lbk_tile.h"

namespace lbk {

template <typename T, int BCX, int BCY, int R, int MODEL>
__global__ __launch_bounds__(kTileMaxWaves * 64, 8) void batch_tile_kernel(
    const SampleDesc *__restrict__ samples, const int *__restrict__ tile_sample, int halo,
    int steps, int parity, int seam)
{
    extern __shared__ Edges edges[];
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    const SampleDesc sd = samples[tile_sample[t]];
    const int rel = t - sd.tile0;
    const int band = rel / sd.tpr, strip = rel - band * sd.tpr;
    tile_steps<T, BCX, BCY, false, R, MODEL>(
        parity ? sd.state[1] : sd.state[0], parity ? sd.state[0] : sd.state[1], sd.lay, sd.med,
        sd.mlay, sd.g, sd.ph, sd.s, sd.inv_s, halo, sd.g.nx >= 64 ? seam : 0, steps, strip, band,
        nullptr, 0, edges);
}

template <typename T, int BCX, int BCY, int R, int MODEL, bool HIST>
__global__ __launch_bounds__(kTileMaxWaves * 64, 8) void batch_rec_tile_kernel(
    const AdjSampleDesc *__restrict__ samples, const int *__restrict__ tile_sample, int halo,
    int steps, LevelSel src_sel, LevelSel dst_sel, int hist_slot, int seam)
{
    extern __shared__ Edges edges[];
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    const AdjSampleDesc sd = samples[tile_sample[t]];
    const int rel = t - sd.tile.tile0;
    const int band = rel / sd.tile.tpr, strip = rel - band * sd.tile.tpr;
    auto region = [&](int r) {
        return r == ADJ_CUR ? sd.region[0]
                            : (r == ADJ_OUTER ? sd.region[1]
                                              : (r == ADJ_INNER ? sd.region[2] : sd.region[3]));
    };
    const char *src = region(src_sel.region) + (uint64_t)src_sel.index * sd.level_bytes;
    char *dst = region(dst_sel.region) + (uint64_t)dst_sel.index * sd.level_bytes;
    float *hist = HIST ? reinterpret_cast<float *>(reinterpret_cast<char *>(sd.hist) +
                                                   (uint64_t)hist_slot * sd.hist_bytes)
                       : nullptr;
    tile_steps<T, BCX, BCY, HIST, R, MODEL>(src, dst, sd.lay, sd.med, sd.mlay, sd.g, sd.ph, sd.s,
                                            sd.inv_s, halo, sd.g.nx >= 64 ? seam : 0, steps, strip, band,
                                            hist,
                                            sd.hist_bytes, edges);
}

namespace {

// The columns of a sample's outlet end that lie left of its inlet in its first
// strip (tile_advance's org), for samples of 64 columns and more, so that the
// strip's columns are distinct; the other strips' halos end short of them.  One
// strip instead of two then pays for the pressure columns, which double the
// instructions of a row update.  Worth it where the instructions of all tiles
// count: 16 FP16 samples of 900 x 900 87.8 us a step with the ends apart, 82.1
// together.  Where a compute unit has a tile or two the slowest tile
// counts.  One lattice keeps its ends apart: the choice at run time cost its
// kernel 2 to 4% where it gained nothing (1024 x 512 6.55 us a step, with it 6.71).
int seam_of(int bcx, int halo, int ntiles)
{
    return bcx == BC_PRESSURE && halo <= 14 && ntiles > 1024 ? 16 : 0;
}

// Call f with the template arguments (R, MODEL) as integral constants.
template <int BCX, typename F> void pick(int rows, int standard, F f)
{
    using one = std::integral_constant<int, 1>;
    using two = std::integral_constant<int, 2>;
    using gen = std::integral_constant<int, MODEL_GEN>;
    using std_ = std::integral_constant<int, BCX == BC_PRESSURE ? MODEL_STD : MODEL_GEN>;
    const bool s = BCX == BC_PRESSURE && standard;
    if (rows == 1) {
        if (s)
            f(one{}, std_{});
        else
            f(one{}, gen{});
    } else {
        if (s)
            f(two{}, std_{});
        else
            f(two{}, gen{});
    }
}

bool valid(int bcy, const Tile &t, int halo, int steps, int ntiles)
{
    return bcy >= 0 && bcy <= 1 && t.waves >= 2 && t.waves <= kTileMaxWaves &&
           (t.rows == 1 || t.rows == 2) && steps >= 1 && halo >= steps && 64 - 2 * halo >= 1 &&
           t.waves * t.rows - 2 * halo >= 1 && ntiles >= 0;
}

} // namespace

template <typename T, int BCX, int BCY>
static hipError_t batch_tile_t(const SampleDesc *samples, const int *tile_sample, int ntiles,
                               int parity, const Tile &t, int halo, int steps, int standard,
                               hipStream_t st)
{
    const int seam = seam_of(BCX, halo, ntiles);
    pick<BCX>(t.rows, standard, [&](auto r, auto m) {
        hipLaunchKernelGGL((batch_tile_kernel<T, BCX, BCY, decltype(r)::value,
                                              decltype(m)::value>),
                           dim3(ntiles), dim3(t.waves * 64), kTileLds, st,
                           samples, tile_sample, halo, steps, parity, seam);
    });
    return hipGetLastError();
}

template <typename T, int BCX, int BCY>
static hipError_t batch_rec_tile_t(const AdjSampleDesc *samples, const int *tile_sample,
                                   int ntiles, const Tile &t, int halo, int steps, int standard,
                                   LevelSel src, LevelSel dst, int hist_slot, hipStream_t st)
{
    const int seam = seam_of(BCX, halo, ntiles);
    pick<BCX>(t.rows, standard, [&](auto r, auto m) {
        constexpr int R = decltype(r)::value, M = decltype(m)::value;
        if (hist_slot >= 0)
            hipLaunchKernelGGL((batch_rec_tile_kernel<T, BCX, BCY, R, M, true>), dim3(ntiles),
                               dim3(t.waves * 64), kTileLds, st, samples,
                               tile_sample, halo, steps, src, dst, hist_slot, seam);
        else
            hipLaunchKernelGGL((batch_rec_tile_kernel<T, BCX, BCY, R, M, false>), dim3(ntiles),
                               dim3(t.waves * 64), kTileLds, st, samples,
                               tile_sample, halo, steps, src, dst, hist_slot, seam);
    });
    return hipGetLastError();
}

hipError_t launch_batch_tile(int storage, int bcx, int bcy, const SampleDesc *samples,
                             const int *tile_sample, int ntiles, int parity, const Tile &t,
                             int halo, int steps, int standard, hipStream_t st)
{
    if (!valid(bcy, t, halo, steps, ntiles))
        return hipErrorInvalidValue;
    if (ntiles == 0)
        return hipSuccess;
    LBK_DISPATCH(batch_tile_t, samples, tile_sample, ntiles, parity, t, halo, steps, standard, st)
}

hipError_t launch_batch_rec_tile(int storage, int bcx, int bcy, const AdjSampleDesc *samples,
                                 const int *tile_sample, int ntiles, const Tile &t, int halo,
                                 int steps, int standard, LevelSel src, LevelSel dst,
                                 int hist_slot, hipStream_t st)
{
    if (!valid(bcy, t, halo, steps, ntiles) || src.region < 0 || src.region > 3 ||
        dst.region < 0 || dst.region > 3)
        return hipErrorInvalidValue;
    if (ntiles == 0)
        return hipSuccess;
    LBK_DISPATCH(batch_rec_tile_t, samples, tile_sample, ntiles, t, halo, steps, standard, src,
                 dst, hist_slot, st)
}

} // namespace lbk
