// lbm_step's two-steps-per-launch kernels on the square lattice (D2Q9): the
// tile bodies of step2.h over one lattice, the step index from the step clock.
#include "internal.h"
#include "step2.h"

namespace lbm {

template <int M, int S, int F, int TY, int NW>
__global__ __launch_bounds__(64 * NW) void k_q9_step2_local(const typename Store<S>::T *__restrict__ src,
                                                        typename Store<S>::T *__restrict__ dst, StepArgs a,
                                                        StepClock *__restrict__ clk, int slot, int stream)
{
    __shared__ float mid[Q9MidLayout<TY>::kSize];
    const uint64_t t = clock_read(clk, slot);
    int txi, tyi;
    row_group_tile(txi, tyi);
    if (tyi * TY >= a.ny)  // padding tile rows of the last group: the whole block
        return;
    q9_step2_tile<M, S, F, TY, NW>(src, dst, a, txi * 64, tyi * TY, t, stream != 0, mid);
    clock_advance(clk, slot, t, 2);
}

template <int S, int F, int TY, int NW>
__global__ __launch_bounds__(64 * NW) void k_q9_step2_mips(const void *__restrict__ src, void *__restrict__ dst,
                                                       StepArgs a, StepClock *__restrict__ clk, int slot, int stream)
{
    __shared__ float lds[mips2_lds<Mips2Q9<S>, TY>()];
    const uint64_t t = clock_read(clk, slot);
    int txi, tyi;
    row_group_tile(txi, tyi);
    if (tyi * TY >= a.ny)
        return;
    step2_mips_tile<Mips2Q9<S>, F, TY, NW>(src, dst, a, txi * 64, tyi * TY, t, stream != 0, lds);
    clock_advance(clk, slot, t, 2);
}

template <int S, int F>
static hipError_t launch_q9_sf(const lbm_params &p, const StepArgs &a, int rows, const void *src, void *dst, StepClock *clk,
                               int slot, hipStream_t s)
{
    using T = typename Store<S>::T;
    const int stream = 2ull * 9ull * (uint64_t)a.plane * sizeof(T) > kStreamStateBytes;
    const dim3 grd = row_group_grid((p.nx + 63) / 64, (p.ny + rows - 1) / rows);
    const T *in = (const T *)src;
    T *out = (T *)dst;
    if (p.model == kMips) {
        if (rows == 16)
            hipLaunchKernelGGL((k_q9_step2_mips<S, F, 16, 8>), grd, dim3(512), 0, s, src, dst, a, clk, slot, stream);
        else
            hipLaunchKernelGGL((k_q9_step2_mips<S, F, 24, 8>), grd, dim3(512), 0, s, src, dst, a, clk, slot, stream);
        return hipGetLastError();
    }
    auto local = [&](auto model) {
        constexpr int M = decltype(model)::value;
        if (rows == 8)
            hipLaunchKernelGGL((k_q9_step2_local<M, S, F, 8, 4>), grd, dim3(256), 0, s, in, out, a, clk, slot, stream);
        else
            hipLaunchKernelGGL((k_q9_step2_local<M, S, F, 16, 4>), grd, dim3(256), 0, s, in, out, a, clk, slot, stream);
    };
    if (p.model == kCil)
        local(IntTag<kCil>{});
    else
        local(IntTag<kPassive>{});
    return hipGetLastError();
}

hipError_t launch_step2_q9(const lbm_params &p, const StepArgs &a, int rows, const void *src, void *dst, StepClock *clk,
                           int slot, hipStream_t s)
{
    return with_flags(step_flags(a), [&](auto fl) {
        constexpr int F = decltype(fl)::value;
        switch (p.storage) {
        case kF32: return launch_q9_sf<kF32, F>(p, a, rows, src, dst, clk, slot, s);
        case kBf16Dev: return launch_q9_sf<kBf16Dev, F>(p, a, rows, src, dst, clk, slot, s);
        case kF16Dev: return launch_q9_sf<kF16Dev, F>(p, a, rows, src, dst, clk, slot, s);
        }
        return hipErrorInvalidValue;
    });
}

}  // namespace lbm
