// lbm_step's two-steps-per-launch kernels on the triangular lattice: the tile
// bodies of step2.h over one lattice, the step index from the step clock.
#include "internal.h"
#include "step2.h"

namespace lbm {

template <int M, int S, int F, int TY>
__global__ __launch_bounds__(256) void k_step2_local(const void *__restrict__ src, void *__restrict__ dst, StepArgs a,
                                                     StepClock *__restrict__ clk, int slot, int stream)
{
    __shared__ float mid[MidLayout<TY>::kSize];
    const uint64_t t = clock_read(clk, slot);
    int txi, tyi;
    row_group_tile(txi, tyi);
    if (tyi * TY >= a.ny)  // padding tile rows of the last group: the whole block
        return;
    step2_tile<M, S, F, TY, 4>(src, dst, a, txi * 64, tyi * TY, t, stream != 0, mid);
    clock_advance(clk, slot, t, 2);
}

template <int S, int F, int TY, int NW>
__global__ __launch_bounds__(64 * NW) void k_step2_mips(const void *__restrict__ src, void *__restrict__ dst, StepArgs a,
                                                    StepClock *__restrict__ clk, int slot, int stream)
{
    __shared__ float lds[mips2_lds<Mips2Q7<S>, TY>()];
    const uint64_t t = clock_read(clk, slot);
    int txi, tyi;
    row_group_tile(txi, tyi);
    if (tyi * TY >= a.ny)
        return;
    step2_mips_tile<Mips2Q7<S>, F, TY, NW>(src, dst, a, txi * 64, tyi * TY, t, stream != 0, lds);
    clock_advance(clk, slot, t, 2);
}

template <int S, int F>
static hipError_t launch_sf(const lbm_params &p, const StepArgs &a, int ty, const void *src, void *dst, StepClock *clk,
                            int slot, hipStream_t s)
{
    const int stream = 2ull * Planes<S>::bytes(a.plane) > kStreamStateBytes;
    const dim3 grd = row_group_grid((p.nx + 63) / 64, (p.ny + ty - 1) / ty);
    if (p.model == kMips) {
        hipLaunchKernelGGL((k_step2_mips<S, F, 16, 8>), grd, dim3(512), 0, s, src, dst, a, clk, slot, stream);
    } else if (p.model == kCil) {
        if (ty == 8)
            hipLaunchKernelGGL((k_step2_local<kCil, S, F, 8>), grd, dim3(256), 0, s, src, dst, a, clk, slot, stream);
        else
            hipLaunchKernelGGL((k_step2_local<kCil, S, F, 16>), grd, dim3(256), 0, s, src, dst, a, clk, slot, stream);
    } else {
        if (ty == 8)
            hipLaunchKernelGGL((k_step2_local<kPassive, S, F, 8>), grd, dim3(256), 0, s, src, dst, a, clk, slot, stream);
        else
            hipLaunchKernelGGL((k_step2_local<kPassive, S, F, 16>), grd, dim3(256), 0, s, src, dst, a, clk, slot, stream);
    }
    return hipGetLastError();
}

hipError_t launch_step2(const lbm_params &p, const StepArgs &a, int rows, const void *src, void *dst, StepClock *clk,
                        int slot, hipStream_t s)
{
    return with_storage(p.storage, [&](auto st) {
        return with_flags(step_flags(a), [&](auto fl) {
            return launch_sf<decltype(st)::value, decltype(fl)::value>(p, a, rows, src, dst, clk, slot, s);
        });
    });
}

}  // namespace lbm
