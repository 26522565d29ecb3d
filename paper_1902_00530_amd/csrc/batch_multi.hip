// Batched sweeps of small lattices with several steps per launch: the tile body
// of multi.h over a list of tiles of many lattices.
#include "batch.h"
#include "multi.h"

namespace lbm {

template <class LP, int M, int F>
__global__ __launch_bounds__(multi_lanes(M)) void k_batch_multi(const BatchTile *__restrict__ tiles,
                                                          const LatDesc *__restrict__ lats,
                                                          const Ctrl *__restrict__ ctrl, MultiGeom g, int step_off,
                                                          int launch_off)
{
    __shared__ float lds[multi_lds<LP, M>()];
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    multi_tile<LP, M, F>(L.buf[par], L.buf[par ^ 1], a, g, tl.tx * g.tx, tl.ty * g.ty,
                         (uint64_t)(ctrl->t0 + step_off), lds);
}

template <class LP, int F>
static hipError_t launch_f(int model, const MultiGeom &g, int64_t ntiles, const BatchTile *tiles, const LatDesc *lats,
                           const Ctrl *ctrl, int step_off, int launch_off, hipStream_t s)
{
    const dim3 grd((unsigned)ntiles), blk(multi_lanes(model));
    if (model == kMips)
        hipLaunchKernelGGL((k_batch_multi<LP, kMips, F>), grd, blk, 0, s, tiles, lats, ctrl, g, step_off, launch_off);
    else if (model == kCil)
        hipLaunchKernelGGL((k_batch_multi<LP, kCil, F>), grd, blk, 0, s, tiles, lats, ctrl, g, step_off, launch_off);
    else
        hipLaunchKernelGGL((k_batch_multi<LP, kPassive, F>), grd, blk, 0, s, tiles, lats, ctrl, g, step_off,
                           launch_off);
    return hipGetLastError();
}

hipError_t launch_batch_multi(int lattice, int model, int storage, int flags, const MultiGeom &g, int64_t ntiles,
                              const BatchTile *tiles, const LatDesc *lats, const Ctrl *ctrl, int step_off,
                              int launch_off, hipStream_t s)
{
    return with_flags(flags, [&](auto fl) {
        constexpr int F = decltype(fl)::value;
        if (lattice == LBM_D2Q9)
            return storage == kF32 ? launch_f<MultiQ9<kF32>, F>(model, g, ntiles, tiles, lats, ctrl, step_off,
                                                               launch_off, s)
                                   : hipErrorInvalidValue;
        return with_storage(storage, [&](auto st) {
            return launch_f<MultiQ7<decltype(st)::value>, F>(model, g, ntiles, tiles, lats, ctrl, step_off, launch_off,
                                                            s);
        });
    });
}

}  // namespace lbm
