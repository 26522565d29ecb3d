// Sums of one moments tile (256 columns x 16 rows of a lattice), shared by the
// single-lattice (moments.hip) and the batched (batch.hip) sampling kernels.
//
// A lane takes R rows of a column.  R = 4, 1024 lanes, every row loaded before the
// first is used: where the tiles are no more than the CUs (mom_few_tiles) and one lane
// walking 16 rows would wait on memory with one wave a SIMD.  R = 16, 256 lanes, row by
// row, where more tiles hide each other's loads: it needs half the registers and passes
// no sums between lanes.  lbm_moments with its fields, us, R = 16 / 4: F32 512^2 (64
// tiles) 16.4 / 13.1, 1024^2 (256) 26.1 / 21.1, 1024x1280 (320) 25.4 / 25.4, 1448^2 (546)
// 31.8 / 37.1, 2000^2 (1000) 46.5 / 52.4; BF16 1024^2 25.5 / 20.1, 2000^2 40.1 / 47.6.
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

constexpr int kMomCols = 256, kMomRows = 16;  // columns and rows of a tile
constexpr int kMomParts = 5;                   // M, Jx, Jy, sum |j|, nonfinite

constexpr int mom_lanes(int R) { return kMomCols * kMomRows / R; }
// four rows a lane: up to a tile a CU
inline bool mom_few_tiles(int64_t tiles) { return tiles <= 256; }

template <int R>
struct MomLds {
    double acc[R < kMomRows ? kMomParts : 1][kMomCols];  // the columns' sums so far
    double part[kMomCols / 64][kMomParts];
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
// One order for every R, so that a lattice's sums do not depend on how many tiles
// its batch has: the rows of a column in turn (R < 16: passed on from one lane's rows
// to the next lane's), then the columns of a wave, then waves.
template <int R, int Q, class Load, class Moments, class Out>
__device__ __forceinline__ void moments_tile(MomLds<R> &lds, int nx, int ny, int x0, int y0, Load load, Moments moments,
                                             Out out, double *__restrict__ part, double *__restrict__ col)
{
    constexpr int G = kMomRows / R, B = G == 1 ? 1 : R;  // lanes of a column, rows loaded at a time
    const int c = threadIdx.x % kMomCols, group = threadIdx.x / kMomCols;
    const int x = x0 + c;
    double acc[kMomParts] = {0.0, 0.0, 0.0, 0.0, 0.0}, v[B][kMomParts];
    int rows = 0;  // of the B last loaded
    auto add = [&]() {
#pragma unroll
        for (int r = 0; r < B; ++r)
            if (r < rows)
#pragma unroll
                for (int k = 0; k < kMomParts; ++k)
                    acc[k] += v[r][k];
    };
    if (x < nx)
        for (int y1 = y0 + group * R; y1 < min(y0 + group * R + R, ny); y1 += B) {
            float f[B][Q];
#pragma unroll
            for (int r = 0; r < B; ++r)
                load(f[r], x, min(y1 + r, ny - 1));
            rows = min(B, ny - y1);
#pragma unroll
            for (int r = 0; r < B; ++r) {
                if (r >= rows)
                    break;
                float rho, jx, jy;
                moments(f[r], rho, jx, jy);
                bool finite = true;
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    finite = finite && isfinite(f[r][i]);
                const double dx = jx, dy = jy;
                v[r][0] = rho;
                v[r][1] = dx;
                v[r][2] = dy;
                v[r][3] = sqrt(dx * dx + dy * dy);
                v[r][4] = finite ? 0.0 : 1.0;
                out(x, y1 + r, rho, jx, jy);
            }
            if (G == 1)
                add();
        }
#pragma unroll
    for (int g = 0; g < G && G > 1; ++g) {
        if (group == g) {
            if (g > 0)
#pragma unroll
                for (int k = 0; k < kMomParts; ++k)
                    acc[k] = lds.acc[k][c];
            add();
            if (g < G - 1)
#pragma unroll
                for (int k = 0; k < kMomParts; ++k)
                    lds.acc[k][c] = acc[k];
        }
        if (g < G - 1)
            __syncthreads();
    }
    if (group == G - 1) {
        if (x < nx)
            col[c] = acc[0];
#pragma unroll
        for (int k = 0; k < kMomParts; ++k)
            acc[k] = mom_wave_sum(acc[k]);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int k = 0; k < kMomParts; ++k)
                lds.part[c >> 6][k] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x < kMomParts)
        part[threadIdx.x] = ((lds.part[0][threadIdx.x] + lds.part[1][threadIdx.x]) + lds.part[2][threadIdx.x]) +
                            lds.part[3][threadIdx.x];
}

}  // namespace lbm
