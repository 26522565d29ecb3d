// lbm_step's several-steps-per-launch kernels for small square (D2Q9) lattices:
// the tile body of multi.h over one lattice, the step index from the step clock.
#include "internal.h"
#include "multi.h"

namespace lbm {

template <class LP, int M, int F>
__global__ __launch_bounds__(multi_lanes(M)) void k_q9_multi(const void *__restrict__ src, void *__restrict__ dst,
                                                       StepArgs a, MultiGeom g, StepClock *__restrict__ clk, int slot)
{
    __shared__ float lds[multi_lds<LP, M>()];
    const uint64_t t = clock_read(clk, slot);
    multi_tile<LP, M, F>(src, dst, a, g, blockIdx.x * g.tx, blockIdx.y * g.ty, t, lds);
    clock_advance(clk, slot, t, g.T);
}

template <int ST, int F>
static hipError_t launch_q9_sf(const lbm_params &p, const StepArgs &a, const MultiGeom &g, const void *src, void *dst,
                               StepClock *clk, int slot, hipStream_t s)
{
    using LP = MultiQ9<ST>;
    const dim3 grd((p.nx + g.tx - 1) / g.tx, (p.ny + g.ty - 1) / g.ty), blk(multi_lanes(p.model));
    if (p.model == kMips)
        hipLaunchKernelGGL((k_q9_multi<LP, kMips, F>), grd, blk, 0, s, src, dst, a, g, clk, slot);
    else if (p.model == kCil)
        hipLaunchKernelGGL((k_q9_multi<LP, kCil, F>), grd, blk, 0, s, src, dst, a, g, clk, slot);
    else
        hipLaunchKernelGGL((k_q9_multi<LP, kPassive, F>), grd, blk, 0, s, src, dst, a, g, clk, slot);
    return hipGetLastError();
}

hipError_t launch_multi_q9(const lbm_params &p, const StepArgs &a, const MultiChoice &c, int steps, const void *src,
                           void *dst, StepClock *clk, int slot, hipStream_t s)
{
    const MultiGeom g = multi_geom(p.model, steps, c.tx, c.ty);
    return with_flags(step_flags(a), [&](auto fl) {
        constexpr int F = decltype(fl)::value;
        switch (p.storage) {
        case kF32: return launch_q9_sf<kF32, F>(p, a, g, src, dst, clk, slot, s);
        case kBf16Dev: return launch_q9_sf<kBf16Dev, F>(p, a, g, src, dst, clk, slot, s);
        case kF16Dev: return launch_q9_sf<kF16Dev, F>(p, a, g, src, dst, clk, slot, s);
        }
        return hipErrorInvalidValue;
    });
}

}  // namespace lbm
