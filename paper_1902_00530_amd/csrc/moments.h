// Sums of one moments tile (256 columns x 16 rows of a lattice), shared by the
// single-lattice (moments.hip) and the batched (batch.hip) sampling kernels.
//
// A lane takes R rows of a column, four rows' populations loaded before the
// first is used.  R = 4, 1024 lanes: where the tiles are few (mom_few_tiles) and
// one lane walking 16 rows would wait on memory with one wave a SIMD: 1024^2
// with its fields written (42 MB, 8.5 us at the rate of a large copy) 17.4 us
// with 16 rows, one load at a time, 11.0 with four.  R = 16, 256 lanes, takes a
// quarter of the lane sums: 4000 x 3000 in BF16 80 us against 92.
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

constexpr int kMomCols = 256, kMomRows = 16;  // columns and rows of a tile
constexpr int kMomParts = 5;                   // M, Jx, Jy, sum |j|, nonfinite

constexpr int mom_lanes(int R) { return kMomCols * kMomRows / R; }
// four rows a lane: up to four tiles a CU
inline bool mom_few_tiles(int64_t tiles) { return tiles <= 1024; }

template <int R>
struct MomLds {
    double col[kMomRows / R][kMomCols];
    double part[mom_lanes(R) / 64][kMomParts];
};

__device__ __forceinline__ double mom_wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_down(v, off, 64);
    return v;
}

// The tile at column x0 and row y0: load(f, x, y) the streamed populations of a
// site, moments(f, rho, jx, jy) its fields, out(x, y, rho, jx, jy) takes them;
// part: the tile's five sums, col: the tile's column sums of rho (col[x - x0]).
// Fixed order: rows of a lane, then lanes of a wave, then waves; for a column
// the rows of a lane, then its lanes.
template <int R, int Q, class Load, class Moments, class Out>
__device__ __forceinline__ void moments_tile(MomLds<R> &lds, int nx, int ny, int x0, int y0, Load load, Moments moments,
                                             Out out, double *__restrict__ part, double *__restrict__ col)
{
    constexpr int B = 4, NW = mom_lanes(R) / 64;  // rows loaded at a time, waves
    const int c = threadIdx.x % kMomCols, group = threadIdx.x / kMomCols;
    const int x = x0 + c;
    double acc[kMomParts] = {0.0, 0.0, 0.0, 0.0, 0.0}, sum = 0.0;
    if (x < nx)
        for (int y1 = y0 + group * R; y1 < min(y0 + group * R + R, ny); y1 += B) {
            float f[B][Q];
#pragma unroll
            for (int r = 0; r < B; ++r)
                load(f[r], x, min(y1 + r, ny - 1));
#pragma unroll
            for (int r = 0; r < B; ++r) {
                if (y1 + r >= ny)
                    break;
                float rho, jx, jy;
                moments(f[r], rho, jx, jy);
                bool finite = true;
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    finite = finite && isfinite(f[r][i]);
                const double dr = rho, dx = jx, dy = jy;
                acc[0] += dr;
                acc[1] += dx;
                acc[2] += dy;
                acc[3] += sqrt(dx * dx + dy * dy);
                acc[4] += finite ? 0.0 : 1.0;
                sum += dr;
                out(x, y1 + r, rho, jx, jy);
            }
        }
    if (R < kMomRows)
        lds.col[group][c] = sum;
    else if (x < nx)
        col[c] = sum;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kMomParts; ++k)
        acc[k] = mom_wave_sum(acc[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kMomParts; ++k)
            lds.part[wave][k] = acc[k];
    __syncthreads();
    if (R < kMomRows && group == 0 && x < nx) {
        double v = lds.col[0][c];
#pragma unroll
        for (int g = 1; g < kMomRows / R; ++g)
            v += lds.col[g][c];
        col[c] = v;
    }
    if (threadIdx.x >= mom_lanes(R) - kMomParts) {
        const int k = threadIdx.x - (mom_lanes(R) - kMomParts);
        double v = lds.part[0][k];
#pragma unroll
        for (int w = 1; w < NW; ++w)
            v += lds.part[w][k];
        part[k] = v;
    }
}

}  // namespace lbm
