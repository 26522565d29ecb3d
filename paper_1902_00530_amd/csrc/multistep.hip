// lbm_step's several-steps-per-launch kernels for small triangular lattices (the
// tile body of multi.h over one lattice, the step index from the step clock),
// and the choice of the launch geometry.
#include <algorithm>

#include "internal.h"
#include "multi.h"

namespace lbm {

template <class LP, int M, int F>
__global__ __launch_bounds__(multi_lanes(M)) void k_multi(const void *__restrict__ src, void *__restrict__ dst, StepArgs a,
                                                    MultiGeom g, StepClock *__restrict__ clk, int slot)
{
    __shared__ float lds[multi_lds<LP, M>()];
    const uint64_t t = clock_read(clk, slot);
    multi_tile<LP, M, F>(src, dst, a, g, blockIdx.x * g.tx, blockIdx.y * g.ty, t, lds);
    clock_advance(clk, slot, t, g.T);
}

MultiGeom multi_geom(int model, int T, int tx, int ty)
{
    MultiGeom g{};
    const int r = model == kMips ? 2 : 1;
    g.T = T;
    g.tx = tx;
    g.ty = ty;
    g.w = tx + 2 * r * T;
    g.h = ty + 2 * r * T;
    for (int k = 0; k <= T; ++k)
        g.mag[k] = (1u << 22) / (uint32_t)(g.w - 2 * r * k) + 1u;
    return g;
}

// The steps per launch and the tile with the least time per step by this model
// of a launch, in us: 3.5 for the launch and the region's load, and per step
// 0.4 (MIPS 0.5) of latency (LDS, two barriers) plus 0.3 (0.4) for every wave
// of the step's box that a SIMD of the fullest CU runs (at least one).  Fitted
// to the measured times of 18 lattices from 32^2 to 512^2 on up to 50
// geometries each: where one block a CU is enough, the choice is within 2% of
// the fastest geometry measured.  CIL 64^2: 4x4 tiles, 8 steps, 2.40 -> 1.10 us
// a step against one step per launch; 128^2: 8x8, 8 steps, 2.40 -> 1.24; 256^2:
// 16x16, 8 steps, 2.60 -> 1.74; MIPS 64^2: 4x4, 6 steps, 3.04 -> 1.52; 128^2:
// 8x8, 5 steps, 3.14 -> 1.75; 256^2: 16x16, 4 steps, 3.46 -> 2.36.
MultiChoice multi_choose(int model, const MultiSize *sizes, int n)
{
    const int r = model == kMips ? 2 : 1, t_max = model == kMips ? 6 : kMultiMaxT;
    const double lat = model == kMips ? 0.5 : 0.4, wave = model == kMips ? 0.4 : 0.3;
    MultiChoice best{};
    for (int tx = 4; tx <= 32; tx += 2)
        for (int ty = 4; ty <= 32; ty += 2) {
            int64_t blocks = 0;
            for (int l = 0; l < n; ++l)
                blocks += (int64_t)sizes[l].count * ((sizes[l].nx + tx - 1) / tx) * ((sizes[l].ny + ty - 1) / ty);
            if (blocks > kMultiMaxTiles)
                continue;
            const int64_t per_cu = (blocks + 255) / 256;
            double t = 3.5;
            for (int T = 1; T <= t_max; ++T) {
                const int w = tx + 2 * r * T, h = ty + 2 * r * T;
                if (w * h > kMultiSites)
                    break;
                // one more step at the start: the box it adds is the largest
                const int waves = ((w - 2 * r) * (h - 2 * r) + 63) / 64;
                t += lat + wave * std::max(1.0, 0.25 * (double)per_cu * waves);
                if (T > 1 && (best.T == 0 || t / T < best.us)) {
                    best.T = T;
                    best.tx = tx;
                    best.ty = ty;
                    best.us = t / T;
                }
            }
        }
    return best;
}

// Lattices of up to these many sites take the several-steps form: beyond them
// two steps on the large tiles of step2.h are as fast.  Measured, us per step
// (best several-steps geometry against the other forms' best): CIL 384^2 2.70
// against 2.91, 512^2 3.50 / 3.31; MIPS 256^2 2.36 / 3.45, 384^2 3.93 / 3.85;
// D2Q9 CIL 384^2 3.17 / 3.66; D2Q9 MIPS 128^2 1.90 / 3.83, 384^2 4.27 / 4.34.
// Two rows count as the four of the lowest tile in the local models (against one
// step per launch: CIL 40000x2 3.8 / 4.0, 80000x2 7.9 / 6.2; MIPS 40000x2 9.0 / 15.7).
MultiChoice multi_for_lattice(const lbm_params &p, const StepArgs &a)
{
    const int64_t most = p.model != LBM_MIPS ? 5 << 15 : p.lattice == LBM_D2Q9 ? 1 << 17 : 3 << 15;
    if (a.pitch != p.nx || (int64_t)p.nx * std::max(p.ny, p.model == LBM_MIPS ? 2 : 4) > most)
        return MultiChoice{};
    const MultiSize size{p.nx, p.ny, 1};
    return multi_choose(p.model, &size, 1);
}

hipError_t launch_multi(const lbm_params &p, const StepArgs &a, const MultiChoice &c, int steps, const void *src, void *dst,
                        StepClock *clk, int slot, hipStream_t s)
{
    const MultiGeom g = multi_geom(p.model, steps, c.tx, c.ty);
    const dim3 grd((p.nx + g.tx - 1) / g.tx, (p.ny + g.ty - 1) / g.ty), blk(multi_lanes(p.model));
    return with_storage(p.storage, [&](auto st) {
        using LP = MultiQ7<decltype(st)::value>;
        return with_flags(step_flags(a), [&](auto fl) {
            constexpr int F = decltype(fl)::value;
            if (p.model == kMips)
                hipLaunchKernelGGL((k_multi<LP, kMips, F>), grd, blk, 0, s, src, dst, a, g, clk, slot);
            else if (p.model == kCil)
                hipLaunchKernelGGL((k_multi<LP, kCil, F>), grd, blk, 0, s, src, dst, a, g, clk, slot);
            else
                hipLaunchKernelGGL((k_multi<LP, kPassive, F>), grd, blk, 0, s, src, dst, a, g, clk, slot);
            return hipGetLastError();
        });
    });
}

}  // namespace lbm
