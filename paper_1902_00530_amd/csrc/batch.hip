// Batched sweeps: many independent lattices of different sizes and
// parameters advanced together (one kernel launch per step, or per two steps,
// covers every lattice), with FP64 observables sampled every sample_every
// steps.
//
// Work list.  Each lattice is cut into TX x TY tiles; the list of all tiles
// of all lattices is built on the host.  Within a lattice, tiles are listed
// in groups of eight tile rows, column by column, so that tile list position
// b runs on XCD b mod 8 and a whole row of tiles stays on one XCD (the same
// order as the single-lattice kernel).  A block reads its tile and its
// lattice's descriptor with scalar loads and runs the same site body as the
// single-lattice kernel, so a batch member gives bit-for-bit the result of
// the single-lattice call with the same seed.
//
// Two steps per launch.  The two-step tile bodies (step2.h) read and write the
// state once per two updates, the first step's results staying in LDS.
//
// Step loop.  One sample period (its step kernels, the sampling kernels, one
// counter update) is captured once in a HIP graph and replayed; the step
// index and the buffer parity come from a small control block in device
// memory that the last node advances, so no kernel arguments change between
// replays and no kernel waits on another workgroup.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <tuple>
#include <type_traits>
#include <vector>

#include "batch.h"
#include "moments.h"
#include "step2.h"

namespace lbm {

// ---------------------------------------------------------------------------
// Step kernels over the tile list.  step_off: steps of this sample period
// before this launch; launch_off: launches before it (the buffer parity).
// ---------------------------------------------------------------------------
template <int M, int ST, int F>
__global__ __launch_bounds__(256) void k_batch_step(const BatchTile *__restrict__ tiles,
                                                    const LatDesc *__restrict__ lats,
                                                    const Ctrl *__restrict__ ctrl, int step_off, int launch_off)
{
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int64_t t = ctrl->t0 + step_off;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x = tl.tx * blockDim.x + threadIdx.x;
    const int y = tl.ty * blockDim.y + threadIdx.y;
    if (x >= a.nx || y >= a.ny)
        return;
    const uint32_t plane = (uint32_t)a.plane;
    const __amdgpu_buffer_rsrc_t src = buffer_rsrc(L.buf[par], (uint32_t)Planes<ST>::bytes(plane));
    const __amdgpu_buffer_rsrc_t dst = buffer_rsrc(L.buf[par ^ 1], (uint32_t)Planes<ST>::bytes(plane));
    const PullSources32 g_src = pull_sources32(a, x, y);
    float f[7];
#pragma unroll
    for (int i = 0; i < 7; ++i)
        f[i] = Planes<ST>::load(src, g_src.idx[i], 0u, i, plane, a);
    float rho, jx, jy, ux, uy;
    site_moments(f, rho, jx, jy);
    local_ustar<M>(a, rho, jx, jy, ux, uy);
    // batch buffers have pitch nx, so the own offset is the site index
    const uint32_t own = g_src.idx[0];
    site_collide<F, ST>(a, f, rho, ux, uy, own, (uint32_t)((uint64_t)t & 0xffffffffu), (uint32_t)((uint64_t)t >> 32));
    store7<ST>(L.stream != 0, dst, own, 0u, plane, f, a);
}

// MIPS over a list of 64 x ROWS tiles (the tile body of the single-lattice
// MIPS kernel, mips_tile_step), one step per launch.
template <int ST, int F, int ROWS>
__global__ __launch_bounds__(256) void k_batch_step_mips(const BatchTile *__restrict__ tiles,
                                                         const LatDesc *__restrict__ lats,
                                                         const Ctrl *__restrict__ ctrl, int step_off, int launch_off)
{
    __shared__ float srho[mips_tile_lds(ROWS)];
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int64_t t = ctrl->t0 + step_off;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x0 = tl.tx * 64, y0 = tl.ty * ROWS;
    if (x0 >= a.nx || y0 >= a.ny)  // whole-block exit, before the barrier
        return;
    const uint32_t bytes = (uint32_t)Planes<ST>::bytes(a.plane);
    mips_tile_step<ST, F, ROWS>(buffer_rsrc(L.buf[par], bytes), buffer_rsrc(L.buf[par ^ 1], bytes), a, x0, y0,
                            (uint32_t)((uint64_t)t & 0xffffffffu), (uint32_t)((uint64_t)t >> 32), srho);
}

// Whole lattices resident in LDS (D2Q7, at most kResidentSites sites each):
// one workgroup of 1024 lanes per lattice runs every step of the launch
// without leaving its CU.  The state is read from HBM once; each step pulls
// every site's populations out of LDS into registers (for MIPS also putting
// each site's density into LDS), waits, collides with the site body of the
// tile kernels and writes the populations back to LDS in place; after the
// last step the state goes to HBM, into the buffer the step count's parity
// names (as after the same number of one-step launches).  A lattice of the
// paper's size (90 x 30) then costs one CU for a whole sample period instead
// of a launch per step.  Results equal the tile kernels' bit for bit.
constexpr int kResidentSites = 4096;
constexpr int kResidentLanes = 1024;
constexpr int kResidentPer = (kResidentSites + kResidentLanes - 1) / kResidentLanes;  // sites per lane

template <int M, int ST, int F>
__global__ __launch_bounds__(kResidentLanes) void k_batch_resident(const LatDesc *__restrict__ lats,
                                                                  const Ctrl *__restrict__ ctrl, int steps)
{
    using T = typename Store<ST>::T;
    __shared__ float st[8 * kResidentSites];  // plane i of the state at i * S, densities at 7 * S
    const LatDesc &L = lats[blockIdx.x];
    const StepArgs a = L.a;  // pitch nx: plane i holds S = nx * ny contiguous elements
    const int S = a.nx * a.ny;
    const int par = (int)(ctrl->k0 & 1);
    const T *__restrict__ src = (const T *)L.buf[par];
    T *__restrict__ dst = (T *)L.buf[par ^ (steps & 1)];
    const int tid = threadIdx.x;
    float *rho_l = st + 7 * S;
    // the state is kept in LDS as stored (16-bit storages: the stored bits),
    // so every step rounds and widens exactly as lbm_step's loads and stores;
    // with a float32 rest plane (kBf16R32) as the values the storage gives
    // back, in float32
    constexpr bool kFloatLds = ST == kBf16R32;
    T *sv = (T *)st;
#pragma unroll
    for (int i = 0; i < 7; ++i)
        for (int e = tid; e < S; e += kResidentLanes) {
            if constexpr (kFloatLds)
                st[i * S + e] = Planes<ST>::ld(src, e, i, a.plane, a);
            else
                sv[i * S + e] = src[(int64_t)i * a.plane + e];
        }
    // this lane's sites s = tid + j * 1024 and their coordinates
    int sx[kResidentPer], sy[kResidentPer];
#pragma unroll
    for (int j = 0; j < kResidentPer; ++j) {
        const int s = tid + j * kResidentLanes;
        sy[j] = s / a.nx;
        sx[j] = s - sy[j] * a.nx;
    }
    __syncthreads();
    const int64_t t0 = ctrl->t0;
    for (int k = 0; k < steps; ++k) {
        const uint64_t t = (uint64_t)(t0 + k);
        const uint32_t tlo = (uint32_t)(t & 0xffffffffu), thi = (uint32_t)(t >> 32);
        float f[kResidentPer][7], rho[kResidentPer], jx[kResidentPer], jy[kResidentPer];
#pragma unroll
        for (int j = 0; j < kResidentPer; ++j) {
            const int s = tid + j * kResidentLanes;
            if (s < S) {
                const PullSources32 q = pull_sources32(a, sx[j], sy[j]);
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    if constexpr (kFloatLds)
                        f[j][i] = st[i * S + (int)q.idx[i]];
                    else
                        f[j][i] = Store<ST>::widen(sv[i * S + (int)q.idx[i]], i == 0 ? a.wr0 : a.wr1);
                }
                site_moments(f[j], rho[j], jx[j], jy[j]);
                if (M == kMips)
                    rho_l[s] = rho[j];
            }
        }
        __syncthreads();  // every pull done (the state may be overwritten), densities in place
#pragma unroll
        for (int j = 0; j < kResidentPer; ++j) {
            const int s = tid + j * kResidentLanes;
            if (s < S) {
                float ux, uy;
                if (M == kMips) {
                    // density at r + e_i: the pull source of the opposite population
                    const PullSources32 q = pull_sources32(a, sx[j], sy[j]);
                    float nb[7];
                    nb[0] = rho[j];
                    nb[1] = rho_l[q.idx[4]];
                    nb[2] = rho_l[q.idx[5]];
                    nb[3] = rho_l[q.idx[6]];
                    nb[4] = rho_l[q.idx[1]];
                    nb[5] = rho_l[q.idx[2]];
                    nb[6] = rho_l[q.idx[3]];
                    mips_ustar(a, rho[j], nb, ux, uy);
                } else {
                    local_ustar<M>(a, rho[j], jx[j], jy[j], ux, uy);
                }
                site_collide<F, ST>(a, f[j], rho[j], ux, uy, (uint32_t)s, tlo, thi);
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    if constexpr (kFloatLds)
                        st[i * S + s] = Planes<ST>::round(f[j][i], i, a);
                    else
                        sv[i * S + s] = Store<ST>::narrow(f[j][i], i == 0 ? a.wr0 : a.wr1);
                }
            }
        }
        __syncthreads();  // the step's writes precede the next step's pulls
    }
#pragma unroll
    for (int i = 0; i < 7; ++i)
        for (int e = tid; e < S; e += kResidentLanes) {
            if constexpr (kFloatLds)
                Planes<ST>::st(dst, e, i, a.plane, st[i * S + e], a);
            else
                dst[(int64_t)i * a.plane + e] = sv[i * S + e];
        }
}

// The same for the square lattice (D2Q9): nine planes and the densities, at
// most kResidentSitesQ9 sites (120 KiB of LDS), the site body of the D2Q9
// tile kernels (q9_moments, local_ustar or q9_mips_ustar, q9_collide).
constexpr int kResidentSitesQ9 = 3072;
constexpr int kResidentPerQ9 = (kResidentSitesQ9 + kResidentLanes - 1) / kResidentLanes;

template <int M, int F>
__global__ __launch_bounds__(kResidentLanes) void k_batch_resident_q9(const LatDesc *__restrict__ lats,
                                                                     const Ctrl *__restrict__ ctrl, int steps)
{
    __shared__ float st[10 * kResidentSitesQ9];  // plane i of the state at i * S, densities at 9 * S
    const LatDesc &L = lats[blockIdx.x];
    const StepArgs a = L.a;  // pitch nx: plane i holds S = nx * ny contiguous floats
    const int S = a.nx * a.ny;
    const int par = (int)(ctrl->k0 & 1);
    const float *__restrict__ src = (const float *)L.buf[par];
    float *__restrict__ dst = (float *)L.buf[par ^ (steps & 1)];
    const int tid = threadIdx.x;
    float *rho_l = st + 9 * S;
#pragma unroll
    for (int i = 0; i < 9; ++i)
        for (int e = tid; e < S; e += kResidentLanes)
            st[i * S + e] = src[(int64_t)i * a.plane + e];
    int sx[kResidentPerQ9], sy[kResidentPerQ9];
#pragma unroll
    for (int j = 0; j < kResidentPerQ9; ++j) {
        const int s = tid + j * kResidentLanes;
        sy[j] = s / a.nx;
        sx[j] = s - sy[j] * a.nx;
    }
    __syncthreads();
    const int64_t t0 = ctrl->t0;
    for (int k = 0; k < steps; ++k) {
        const uint64_t t = (uint64_t)(t0 + k);
        const uint32_t tlo = (uint32_t)(t & 0xffffffffu), thi = (uint32_t)(t >> 32);
        float f[kResidentPerQ9][9], rho[kResidentPerQ9], jx[kResidentPerQ9], jy[kResidentPerQ9];
#pragma unroll
        for (int j = 0; j < kResidentPerQ9; ++j) {
            const int s = tid + j * kResidentLanes;
            if (s < S) {
                const Q9Sources q = q9_sources(a, sx[j], sy[j]);
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    f[j][i] = st[i * S + (int)q.idx[i]];
                q9_moments(f[j], rho[j], jx[j], jy[j]);
                if (M == kMips)
                    rho_l[s] = rho[j];
            }
        }
        __syncthreads();  // every pull done (the state may be overwritten), densities in place
#pragma unroll
        for (int j = 0; j < kResidentPerQ9; ++j) {
            const int s = tid + j * kResidentLanes;
            if (s < S) {
                float ux, uy;
                if (M == kMips) {
                    // density at r + e_i: the pull source of the opposite population
                    const Q9Sources q = q9_sources(a, sx[j], sy[j]);
                    float nb[9];
                    nb[0] = rho[j];
                    nb[1] = rho_l[q.idx[3]];
                    nb[2] = rho_l[q.idx[4]];
                    nb[3] = rho_l[q.idx[1]];
                    nb[4] = rho_l[q.idx[2]];
                    nb[5] = rho_l[q.idx[7]];
                    nb[6] = rho_l[q.idx[8]];
                    nb[7] = rho_l[q.idx[5]];
                    nb[8] = rho_l[q.idx[6]];
                    q9_mips_ustar(a, rho[j], nb, ux, uy);
                } else {
                    local_ustar<M>(a, rho[j], jx[j], jy[j], ux, uy);
                }
                q9_collide<F>(a, f[j], rho[j], ux, uy, (uint32_t)s, tlo, thi);
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    st[i * S + s] = f[j][i];
            }
        }
        __syncthreads();  // the step's writes precede the next step's pulls
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
        for (int e = tid; e < S; e += kResidentLanes)
            dst[(int64_t)i * a.plane + e] = st[i * S + e];
}

// The square lattice (D2Q9) over the tile list: the single-lattice site body
// (passive, CIL) and MIPS tile body, one step per launch.
template <int M, int F>
__global__ __launch_bounds__(256) void k_batch_q9_step(const BatchTile *__restrict__ tiles,
                                                       const LatDesc *__restrict__ lats,
                                                       const Ctrl *__restrict__ ctrl, int step_off, int launch_off)
{
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int64_t t = ctrl->t0 + step_off;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x = tl.tx * blockDim.x + threadIdx.x;
    const int y = tl.ty * blockDim.y + threadIdx.y;
    if (x >= a.nx || y >= a.ny)
        return;
    q9_site_step<M, kF32, F>((const float *)L.buf[par], (float *)L.buf[par ^ 1], a, x, y,
                             (uint32_t)((uint64_t)t & 0xffffffffu), (uint32_t)((uint64_t)t >> 32));
}

template <int F>
__global__ __launch_bounds__(256) void k_batch_q9_step_mips(const BatchTile *__restrict__ tiles,
                                                            const LatDesc *__restrict__ lats,
                                                            const Ctrl *__restrict__ ctrl, int step_off, int launch_off)
{
    __shared__ float srho[(kQ9MipsRows + 2) * 66];
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int64_t t = ctrl->t0 + step_off;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x0 = tl.tx * 64, y0 = tl.ty * kQ9MipsRows;
    if (x0 >= a.nx || y0 >= a.ny)  // whole-block exit, before the barrier
        return;
    q9_mips_tile_step<kF32, F>((const float *)L.buf[par], (float *)L.buf[par ^ 1], a, x0, y0,
                               (uint32_t)((uint64_t)t & 0xffffffffu), (uint32_t)((uint64_t)t >> 32), srho);
}

// Two steps per launch over the tile list (the tile bodies of step2.h): local
// models, the square lattice, and MIPS on either lattice.  A tile past its
// lattice's edge exits as a whole block, before any barrier.
template <int M, int F, int TY, int NW>
__global__ __launch_bounds__(64 * NW) void k_batch_q9_step2(const BatchTile *__restrict__ tiles,
                                                            const LatDesc *__restrict__ lats,
                                                            const Ctrl *__restrict__ ctrl, int step_off,
                                                            int launch_off)
{
    __shared__ float mid[Q9MidLayout<TY>::kSize];
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x0 = tl.tx * 64, y0 = tl.ty * TY;
    if (x0 >= a.nx || y0 >= a.ny)
        return;
    q9_step2_tile<M, kF32, F, TY, NW>((const float *)L.buf[par], (float *)L.buf[par ^ 1], a, x0, y0,
                                      (uint64_t)(ctrl->t0 + step_off), L.stream != 0, mid);
}

template <int M, int ST, int F, int TY, int NW>
__global__ __launch_bounds__(64 * NW) void k_batch_step2(const BatchTile *__restrict__ tiles,
                                                     const LatDesc *__restrict__ lats,
                                                     const Ctrl *__restrict__ ctrl, int step_off, int launch_off)
{
    __shared__ float mid[MidLayout<TY>::kSize];
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x0 = tl.tx * 64, y0 = tl.ty * TY;
    if (x0 >= a.nx || y0 >= a.ny)
        return;
    step2_tile<M, ST, F, TY, NW>(L.buf[par], L.buf[par ^ 1], a, x0, y0, (uint64_t)(ctrl->t0 + step_off),
                                 L.stream != 0, mid);
}

template <class LP, int F, int TY, int NW>
__global__ __launch_bounds__(64 * NW) void k_batch_step2_mips(const BatchTile *__restrict__ tiles,
                                                          const LatDesc *__restrict__ lats,
                                                          const Ctrl *__restrict__ ctrl, int step_off, int launch_off)
{
    __shared__ float lds[mips2_lds<LP, TY>()];
    const BatchTile tl = tiles[blockIdx.x];
    const LatDesc &L = lats[tl.lat];
    const StepArgs a = L.a;
    const int par = (int)((ctrl->k0 + launch_off) & 1);
    const int x0 = tl.tx * 64, y0 = tl.ty * TY;
    if (x0 >= a.nx || y0 >= a.ny)
        return;
    step2_mips_tile<LP, F, TY, NW>(L.buf[par], L.buf[par ^ 1], a, x0, y0, (uint64_t)(ctrl->t0 + step_off),
                                   L.stream != 0, lds);
}

// ---------------------------------------------------------------------------
// Sampling: per moments tile (256 columns x 16 rows of one lattice) FP64
// partial sums of M, Jx, Jy, sum |j|, nonfinite and per-column density sums
// of the streamed populations; then per lattice the fixed-order totals.
// ---------------------------------------------------------------------------
// Q = 7 (triangular) or 9 (square lattice, F32 storage only).  Block b
// takes moments tile base + b (a launch may cover one lattice group).
template <int Q, int ST, int R>
__global__ __launch_bounds__(mom_lanes(R)) void k_batch_moments(const MomTile *__restrict__ mt,
                                                             const LatDesc *__restrict__ lats,
                                                             const Ctrl *__restrict__ ctrl, int node, int base,
                                                             double *__restrict__ part, double *__restrict__ colpart)
{
    __shared__ MomLds<R> lds;
    const int tile = base + (int)blockIdx.x;
    const MomTile m = mt[tile];
    const LatDesc &L = lats[m.lat];
    const StepArgs a = L.a;
    const int par = (int)((ctrl->k0 + node) & 1);
    const uint32_t plane = (uint32_t)a.plane;
    const void *buf = L.buf[par];
    moments_tile<R, Q>(
        lds, a.nx, a.ny, m.cx * kMomCols, m.cy * kMomRows,
        [&](float *f, int x, int y) {
            if constexpr (Q == 7) {
                const __amdgpu_buffer_rsrc_t src = buffer_rsrc(buf, (uint32_t)Planes<ST>::bytes(plane));
                const PullSources32 g = pull_sources32(a, x, y);
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    f[i] = Planes<ST>::load(src, g.idx[i], 0u, i, plane, a);
            } else {
                const Q9Sources g = q9_sources(a, x, y);
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    f[i] = BufIO<float>::load(q9_plane_rsrc((const float *)buf, i, plane), g.idx[i], 0u);
            }
        },
        [](const float *f, float &rho, float &jx, float &jy) {
            if constexpr (Q == 7)
                site_moments(f, rho, jx, jy);
            else
                q9_moments(f, rho, jx, jy);
        },
        [](int, int, float, float, float) {}, part + (int64_t)tile * kMomParts,
        colpart + L.col_off + (int64_t)m.cy * a.nx + m.cx * kMomCols);
}

// Column means rho_y(x) of every lattice: one thread per column (grid y =
// lattice), the column's row-block partials added in row order.  Many
// blocks, so a sample of a few large lattices does not wait on a handful of
// CUs walking every column.
__global__ __launch_bounds__(256) void k_batch_colmeans(const LatDesc *__restrict__ lats,
                                                        const double *__restrict__ colpart,
                                                        double *__restrict__ colmean)
{
    const LatDesc &L = lats[blockIdx.y];
    const int nx = L.a.nx;
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= nx)
        return;
    const double *cp = colpart + L.col_off + x;
    double c = 0.0;
#pragma unroll 16
    for (int r = 0; r < L.nrb; ++r)
        c += cp[(int64_t)r * nx];
    colmean[L.cm_off + x] = c / (double)L.a.ny;
}

// One block per lattice: totals of its tiles, the mean of its column means
// and their variance; writes 8 doubles {M, Jx, Jy, sum|j|, nonfinite, mean,
// var, step} of sample s.
__global__ __launch_bounds__(256) void k_batch_final(const LatDesc *__restrict__ lats, const Ctrl *__restrict__ ctrl,
                                                     int node, const double *__restrict__ part,
                                                     const double *__restrict__ colmean,
                                                     double *__restrict__ results, int n_samples)
{
    __shared__ double lds[4][6];
    __shared__ double mean_s;
    const LatDesc &L = lats[blockIdx.x];
    const int nx = L.a.nx;
    const double *cm = colmean + L.cm_off;
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < L.mt_count; b += blockDim.x)
#pragma unroll
        for (int k = 0; k < 5; ++k)
            v[k] += part[(int64_t)(L.mt_begin + b) * 5 + k];
    for (int x = threadIdx.x; x < nx; x += blockDim.x)
        v[5] += cm[x];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        v[k] = mom_wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k)
            lds[w][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
        mean_s = (((lds[0][5] + lds[1][5]) + lds[2][5]) + lds[3][5]) / (double)nx;
    __syncthreads();
    const double mean = mean_s;
    double q = 0.0;
    for (int x = threadIdx.x; x < nx; x += blockDim.x) {
        const double d = cm[x] - mean;
        q += d * d;
    }
    q = mom_wave_sum(q);
    __shared__ double lq[4];
    if (lane == 0)
        lq[w] = q;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t s = ctrl->sample;
        if (s < n_samples) {
            double *r = results + ((int64_t)blockIdx.x * n_samples + s) * 8;
#pragma unroll
            for (int k = 0; k < 5; ++k)
                r[k] = ((lds[0][k] + lds[1][k]) + lds[2][k]) + lds[3][k];
            r[5] = mean;
            r[6] = (((lq[0] + lq[1]) + lq[2]) + lq[3]) / (double)nx;
            r[7] = (double)(ctrl->t0 + node);
        }
    }
}

// The density change of the paper's protocol (appendix "Simulation procedure
// for results"): every population of lattice l gains drho_l / Q, in the
// buffer that holds the state after this period's steps; per moments tile.
template <int Q, int ST>
__global__ __launch_bounds__(256) void k_batch_add_density(const MomTile *__restrict__ mt,
                                                           const LatDesc *__restrict__ lats,
                                                           const Ctrl *__restrict__ ctrl, int node)
{
    const MomTile m = mt[blockIdx.x];
    const LatDesc &L = lats[m.lat];
    const float add = L.add;
    if (add == 0.0f)
        return;
    const StepArgs &a = L.a;
    const int par = (int)((ctrl->k0 + node) & 1);
    using T = typename Store<ST>::T;
    T *f = (T *)L.buf[par];
    const int x = m.cx * 256 + threadIdx.x;
    if (x >= a.nx)
        return;
    const int ye = min(m.cy * kMomRows + kMomRows, a.ny);
    for (int y = m.cy * kMomRows; y < ye; ++y)
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int64_t e = (int64_t)y * a.pitch + x;
            if constexpr (Q == 7) {
                Planes<ST>::st(f, e, i, a.plane, Planes<ST>::ld(f, e, i, a.plane, a) + add, a);
            } else {
                T *p = f + (size_t)i * (size_t)a.plane + (size_t)e;
                *p = Store<ST>::narrow(Store<ST>::widen(*p, 0.0f) + add, 0.0f);
            }
        }
}

__global__ void k_batch_advance(Ctrl *ctrl, int64_t steps, int sampled)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        ctrl->t0 += steps;
        ctrl->k0 += steps;
        ctrl->sample += sampled;
    }
}

__global__ void k_batch_set_ctrl(Ctrl *ctrl, int64_t t0)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        ctrl->t0 = t0;
        ctrl->k0 = 0;
        ctrl->sample = 0;
        ctrl->pad = 0;
    }
}

// ---------------------------------------------------------------------------
// Host side: layout of the workspace, tile lists, tile-shape tuning.
// ---------------------------------------------------------------------------
static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct Layout {
    size_t lat, tiles, mtiles, ctrl, part, colpart, colmean, tiles3, results, total;
    int64_t n_tiles1, n_tiles2, n_tiles3, n_mtiles, colpart_n, colmean_n;
};

// Work-tile shapes: sites across, rows, steps per launch.  Shapes 0..4 serve
// the local models (CIL, passive); MIPS takes the two-step shapes 3 and 4
// (64 x 8, 64 x 16; D2Q9 also 7, 64 x 24) and, for single steps, shape 6
// (D2Q7, 64 x 4) or 5 (D2Q9, 64 x 16); each model's shapes are tuned among
// themselves.
struct Shape {
    int tx, ty, steps;
};
constexpr int kNumShapes = 8;
constexpr int kNumTuned = 5;
constexpr int kMipsShape = 5, kMipsShape4 = 6, kMipsShape24 = 7;
static const Shape kShapes[kNumShapes] = {{256, 1, 1}, {128, 2, 1}, {64, 4, 1}, {64, 8, 2},
                                          {64, 16, 2}, {64, 16, 1}, {64, 4, 1}, {64, 24, 2}};
// the forms that tile_rows names (the others are the tuning's own)
static bool named_shape(int k) { return k != kMipsShape24 && k <= kNumShapes; }
constexpr int64_t kChunk = 1024;  // steps per captured graph, at most
constexpr int64_t kBranchLaunches = 10;  // launches of a graph that may run as two branches, at least
// the LDS-resident form (k_batch_resident): no tile list, every step of a
// graph chunk in one launch; a tuning launch runs an odd number of steps, so
// it writes the second buffer like the tile shapes' tuning launches
constexpr int kResident = kNumShapes;
constexpr int kResidentTuneSteps = 63;
// the several-steps form on small tiles (multi.h): a tile list of its own
// geometry, up to MultiChoice::T steps per launch
constexpr int kMulti = kNumShapes + 1;

static bool resident_fits(const lbm_params *ps, int n)
{
    for (int l = 0; l < n; ++l)
        if ((int64_t)ps[l].nx * ps[l].ny > (ps[l].lattice == LBM_D2Q9 ? kResidentSitesQ9 : kResidentSites))
            return false;
    return true;
}

// The shapes that a batch of this model and lattice may take (tuned among
// themselves): MIPS 64x8 and 64x16 with two steps per launch, D2Q7 also 64x4 with
// one, D2Q9 also 64x24; the local models shapes 0..4.
static std::vector<int> batch_shapes(const lbm_params &p)
{
    if (p.model == LBM_MIPS)
        return p.lattice == LBM_D2Q9 ? std::vector<int>{3, 4, kMipsShape24} : std::vector<int>{kMipsShape4, 3, 4};
    std::vector<int> v(kNumTuned);
    for (int k = 0; k < kNumTuned; ++k)
        v[k] = k;
    return v;
}

static int64_t count_tiles(const lbm_params *ps, int n, int tx, int ty)
{
    int64_t c = 0;
    for (int l = 0; l < n; ++l) {
        const int64_t ntx = (ps[l].nx + tx - 1) / tx, nty = (ps[l].ny + ty - 1) / ty;
        c += ntx * ((nty + 7) / 8) * 8;  // rows padded to whole groups of eight
    }
    return c;
}

// The several-steps form of this batch, T = 0 where it has none: batches of up
// to 2^20 sites (larger ones fill the GPU with the tile forms; the tuning times
// it against them).  Twelve 90 x 30 MIPS lattices 3.25 (resident in LDS, 12 of
// 256 CUs) -> 2.14 us a step, fifty 180 x 60 CIL lattices 6.1 (two steps per
// launch, 64 x 8 tiles) -> 5.3.
constexpr int64_t kMultiBatchSites = 1 << 20;

static MultiChoice multi_for_batch(const lbm_params *ps, int n)
{
    int64_t sites = 0;
    std::map<std::pair<int, int>, int> hist;
    for (int l = 0; l < n; ++l) {
        sites += (int64_t)ps[l].nx * ps[l].ny;
        if (sites > kMultiBatchSites)
            return MultiChoice{};
        hist[{ps[l].nx, ps[l].ny}]++;
    }
    std::vector<MultiSize> v;
    for (const auto &h : hist)
        v.push_back(MultiSize{h.first.first, h.first.second, h.second});
    return multi_choose(ps[0].model, v.data(), (int)v.size());
}

// its tiles: one list of every lattice's tiles, lattice by lattice, no padding
static int64_t count_multi_tiles(const lbm_params *ps, int n, const MultiChoice &c)
{
    int64_t t = 0;
    for (int l = 0; l < n && c.T; ++l)
        t += (int64_t)((ps[l].nx + c.tx - 1) / c.tx) * ((ps[l].ny + c.ty - 1) / c.ty);
    return t;
}

static std::vector<BatchTile> build_multi_tiles(const lbm_params *ps, int n, const MultiChoice &c)
{
    std::vector<BatchTile> v;
    for (int l = 0; l < n; ++l)
        for (int y = 0; y * c.ty < ps[l].ny; ++y)
            for (int x = 0; x * c.tx < ps[l].nx; ++x)
                v.push_back(BatchTile{l, (int16_t)x, (int16_t)y});
    return v;
}

// Lattices are independent, so a chunk of steps may run lattice group by
// lattice group: every launch of the chunk for the first group, then for the
// next.  A group's two buffers then stay in the 256 MiB Infinity Cache across
// the chunk's launches instead of streaming from HBM every step.  The batch
// takes the fewest groups of at most kCacheGroupBytes (as measured, larger
// groups of fewer launches beat smaller ones down to that size), cut into
// consecutive lattices of about equal bytes.
constexpr uint64_t kCacheGroupBytes = 240ull << 20;

// bytes of a lattice's two population buffers (pitch nx)
static uint64_t state_bytes(const lbm_params &p)
{
    const uint64_t per_site = p.lattice == LBM_D2Q9 ? (p.storage == LBM_F32 ? 36ull : 18ull)
                              : p.storage == LBM_F32        ? 28ull
                              : p.storage == LBM_BF16_DEV_R32 ? 16ull
                                                              : 14ull;
    return 2ull * per_site * (uint64_t)p.nx * p.ny;
}

static std::vector<int> cache_groups(const lbm_params *ps, int n)
{
    std::vector<uint64_t> b(n);
    uint64_t total = 0;
    for (int l = 0; l < n; ++l) {
        b[l] = state_bytes(ps[l]);
        total += b[l];
    }
    const uint64_t ng = (total + kCacheGroupBytes - 1) / kCacheGroupBytes;
    const uint64_t target = (total + ng - 1) / ng;
    std::vector<int> first{0};  // first lattice of each group, then n
    uint64_t cum = 0, in_group = 0;
    for (int l = 0; l < n; ++l) {
        const uint64_t cut = (uint64_t)(first.size()) * target;  // where the next group begins
        if (l > first.back() && (cum >= cut || in_group + b[l] > kCacheGroupBytes)) {
            first.push_back(l);
            in_group = 0;
        }
        cum += b[l];
        in_group += b[l];
    }
    first.push_back(n);
    return first;
}

// The lattice at which a group of them (consecutive lattices first .. last - 1)
// is cut into two branches of about equal sites; last where there is only one.
static int branch_cut(const lbm_params *ps, int first, int last)
{
    auto sites = [&](int l) { return (int64_t)ps[l].nx * ps[l].ny; };
    int64_t total = 0, cum = 0;
    for (int l = first; l < last; ++l)
        total += sites(l);
    for (int l = first; l + 1 < last; ++l) {
        cum += sites(l);
        if (2 * cum + sites(l + 1) > total)  // cutting after the next one is further from the middle
            return l + 1;
    }
    return last - 1 > first ? last - 1 : last;
}

static Layout layout(const lbm_params *ps, int n, int64_t n_samples)
{
    Layout L{};
    L.n_tiles3 = kMultiMaxTiles;
    // room for the list of one single-step shape and one two-step shape
    L.n_tiles1 = 0;
    L.n_tiles2 = 0;
    for (int k = 0; k < kNumShapes; ++k) {
        int64_t &m = kShapes[k].steps == 1 ? L.n_tiles1 : L.n_tiles2;
        m = std::max(m, count_tiles(ps, n, kShapes[k].tx, kShapes[k].ty));
    }
    L.n_mtiles = 0;
    L.colpart_n = 0;
    L.colmean_n = 0;
    for (int l = 0; l < n; ++l) {
        const int64_t cx = (ps[l].nx + 255) / 256, cy = (ps[l].ny + kMomRows - 1) / kMomRows;
        L.n_mtiles += cx * cy;
        L.colpart_n += cy * ps[l].nx;
        L.colmean_n += ps[l].nx;
    }
    size_t off = 0;
    L.lat = off;
    off = align256(off + sizeof(LatDesc) * n);
    L.tiles = off;
    off = align256(off + sizeof(BatchTile) * (L.n_tiles1 + L.n_tiles2));
    L.mtiles = off;
    off = align256(off + sizeof(MomTile) * L.n_mtiles);
    L.ctrl = off;
    off = align256(off + sizeof(Ctrl));
    L.part = off;
    off = align256(off + sizeof(double) * 5 * L.n_mtiles);
    L.colpart = off;
    off = align256(off + sizeof(double) * L.colpart_n);
    L.colmean = off;
    off = align256(off + sizeof(double) * L.colmean_n);
    // room for the largest list, whatever the lattices and their model: part of a
    // batch never needs more workspace than the batch
    L.tiles3 = off;
    off = align256(off + sizeof(BatchTile) * L.n_tiles3);
    L.results = off;
    off = align256(off + sizeof(double) * 8 * (size_t)n * (size_t)std::max<int64_t>(n_samples, 1));
    L.total = off;
    return L;
}

// Tile list of one shape, row-group order per lattice; tiles in the padding
// rows of a lattice's last group point past the lattice and exit at once.
static std::vector<BatchTile> build_tiles(const lbm_params *ps, int n, int tx, int ty)
{
    std::vector<BatchTile> v;
    for (int l = 0; l < n; ++l) {
        const int ntx = (ps[l].nx + tx - 1) / tx, nty = (ps[l].ny + ty - 1) / ty;
        for (int g = 0; g < (nty + 7) / 8; ++g)
            for (int c = 0; c < ntx; ++c)
                for (int r = 0; r < 8; ++r)
                    v.push_back(BatchTile{l, (int16_t)c, (int16_t)(8 * g + r)});
    }
    return v;
}

static int sweep_flags(const lbm_params *ps, int n)
{
    const int f = step_flags(make_step_args(ps[0], ps[0].nx));
    for (int l = 1; l < n; ++l)
        if (step_flags(make_step_args(ps[l], ps[l].nx)) != f)
            return -1;
    return f;
}

template <int M, int ST, int F>
static hipError_t launch_batch_step_mf(int shape, int64_t ntiles, const BatchTile *tiles, const LatDesc *lats,
                                       const Ctrl *ctrl, int step_off, int launch_off, hipStream_t s)
{
    const Shape &sh = kShapes[shape];
    if (sh.steps == 1)
        hipLaunchKernelGGL((k_batch_step<M, ST, F>), dim3((unsigned)ntiles), dim3(sh.tx, sh.ty), 0, s, tiles, lats,
                           ctrl, step_off, launch_off);
    else if (sh.ty == 8)
        hipLaunchKernelGGL((k_batch_step2<M, ST, F, 8, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles, lats, ctrl,
                           step_off, launch_off);
    else
        hipLaunchKernelGGL((k_batch_step2<M, ST, F, 16, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles, lats,
                           ctrl, step_off, launch_off);
    return hipGetLastError();
}

template <int ST, int F>
static hipError_t launch_batch_mips_f(int shape, int64_t ntiles, const BatchTile *tiles, const LatDesc *lats,
                                      const Ctrl *ctrl, int step_off, int launch_off, hipStream_t s)
{
    if (kShapes[shape].steps == 2 && kShapes[shape].ty == 8)
        hipLaunchKernelGGL((k_batch_step2_mips<Mips2Q7<ST>, F, 8, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles,
                           lats, ctrl, step_off, launch_off);
    else if (kShapes[shape].steps == 2)
        hipLaunchKernelGGL((k_batch_step2_mips<Mips2Q7<ST>, F, 16, 8>), dim3((unsigned)ntiles), dim3(512), 0, s,
                           tiles, lats, ctrl, step_off, launch_off);
    else if (shape == kMipsShape4)
        hipLaunchKernelGGL((k_batch_step_mips<ST, F, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles, lats, ctrl,
                           step_off, launch_off);
    else
        hipLaunchKernelGGL((k_batch_step_mips<ST, F, kMipsRows>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles,
                           lats, ctrl, step_off, launch_off);
    return hipGetLastError();
}

// Every lattice of the batch in one CU's LDS (D2Q9: F32 storage only).
static hipError_t launch_resident(int lattice, int model, int storage, int flags, int n, const LatDesc *lats,
                                  const Ctrl *ctrl, int steps, hipStream_t s)
{
    const dim3 grd((unsigned)n), blk(kResidentLanes);
    return with_storage(storage, [&](auto st) {
        constexpr int ST = decltype(st)::value;
        return with_flags(flags, [&](auto fl) {
            constexpr int F = decltype(fl)::value;
            if (lattice == LBM_D2Q9) {
                if (ST != kF32)
                    return hipErrorInvalidValue;
                if (model == LBM_MIPS)
                    hipLaunchKernelGGL((k_batch_resident_q9<kMips, F>), grd, blk, 0, s, lats, ctrl, steps);
                else if (model == LBM_CIL)
                    hipLaunchKernelGGL((k_batch_resident_q9<kCil, F>), grd, blk, 0, s, lats, ctrl, steps);
                else
                    hipLaunchKernelGGL((k_batch_resident_q9<kPassive, F>), grd, blk, 0, s, lats, ctrl, steps);
            } else if (model == LBM_MIPS) {
                hipLaunchKernelGGL((k_batch_resident<kMips, ST, F>), grd, blk, 0, s, lats, ctrl, steps);
            } else if (model == LBM_CIL) {
                hipLaunchKernelGGL((k_batch_resident<kCil, ST, F>), grd, blk, 0, s, lats, ctrl, steps);
            } else {
                hipLaunchKernelGGL((k_batch_resident<kPassive, ST, F>), grd, blk, 0, s, lats, ctrl, steps);
            }
            return hipGetLastError();
        });
    });
}

template <int M, int F>
static void launch_q9_two(int ty, int64_t ntiles, const BatchTile *tiles, const LatDesc *lats, const Ctrl *ctrl,
                          int step_off, int launch_off, hipStream_t s)
{
    if (ty == 8)
        hipLaunchKernelGGL((k_batch_q9_step2<M, F, 8, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles, lats, ctrl,
                           step_off, launch_off);
    else
        hipLaunchKernelGGL((k_batch_q9_step2<M, F, 16, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles, lats,
                           ctrl, step_off, launch_off);
}

template <int F>
static hipError_t launch_batch_q9_f(int model, int shape, int64_t ntiles, const BatchTile *tiles, const LatDesc *lats,
                                    const Ctrl *ctrl, int step_off, int launch_off, hipStream_t s)
{
    const Shape &sh = kShapes[shape];
    if (model == kMips && sh.steps == 2 && sh.ty == 8)
        hipLaunchKernelGGL((k_batch_step2_mips<Mips2Q9<kF32>, F, 8, 4>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles,
                           lats, ctrl, step_off, launch_off);
    else if (model == kMips && sh.steps == 2 && sh.ty == 24)
        hipLaunchKernelGGL((k_batch_step2_mips<Mips2Q9<kF32>, F, 24, 8>), dim3((unsigned)ntiles), dim3(512), 0, s, tiles,
                           lats, ctrl, step_off, launch_off);
    else if (model == kMips && sh.steps == 2)
        hipLaunchKernelGGL((k_batch_step2_mips<Mips2Q9<kF32>, F, 16, 8>), dim3((unsigned)ntiles), dim3(512), 0, s, tiles,
                           lats, ctrl, step_off, launch_off);
    else if (model == kMips)
        hipLaunchKernelGGL((k_batch_q9_step_mips<F>), dim3((unsigned)ntiles), dim3(256), 0, s, tiles, lats, ctrl,
                           step_off, launch_off);
    else if (sh.steps == 2 && model == kCil)
        launch_q9_two<kCil, F>(sh.ty, ntiles, tiles, lats, ctrl, step_off, launch_off, s);
    else if (sh.steps == 2)
        launch_q9_two<kPassive, F>(sh.ty, ntiles, tiles, lats, ctrl, step_off, launch_off, s);
    else if (model == kCil)
        hipLaunchKernelGGL((k_batch_q9_step<kCil, F>), dim3((unsigned)ntiles), dim3(sh.tx, sh.ty), 0, s, tiles, lats,
                           ctrl, step_off, launch_off);
    else
        hipLaunchKernelGGL((k_batch_q9_step<kPassive, F>), dim3((unsigned)ntiles), dim3(sh.tx, sh.ty), 0, s, tiles,
                           lats, ctrl, step_off, launch_off);
    return hipGetLastError();
}

// One launch of shape `shape` over a tile list (D2Q9: F32 storage only).
static hipError_t launch_batch_step(int lattice, int model, int storage, int flags, int shape, int64_t ntiles,
                                    const BatchTile *tiles, const LatDesc *lats, const Ctrl *ctrl, int step_off,
                                    int launch_off, hipStream_t s)
{
    return with_flags(flags, [&](auto fl) {
        constexpr int F = decltype(fl)::value;
        if (lattice == LBM_D2Q9)
            return storage == kF32
                       ? launch_batch_q9_f<F>(model, shape, ntiles, tiles, lats, ctrl, step_off, launch_off, s)
                       : hipErrorInvalidValue;
        return with_storage(storage, [&](auto st) {
            constexpr int ST = decltype(st)::value;
            if (model == kMips)
                return launch_batch_mips_f<ST, F>(shape, ntiles, tiles, lats, ctrl, step_off, launch_off, s);
            if (model == kCil)
                return launch_batch_step_mf<kCil, ST, F>(shape, ntiles, tiles, lats, ctrl, step_off, launch_off, s);
            return launch_batch_step_mf<kPassive, ST, F>(shape, ntiles, tiles, lats, ctrl, step_off, launch_off, s);
        });
    });
}

// Tuned tile shape per batch signature (arch + lattice type + multiset of
// lattice sizes + model + flags), kept for the life of the process.
static std::mutex g_tune_mu;
struct Tuned {
    int shape;      // the fastest form
    int split;      // its lattice groups run as two branches
    int direct;     // the form of direct launches: the same shape where it is as fast
    int tile;       // the fastest among the forms that tile_rows names (named_shape)
    bool branches;  // branches were timed too (by a call that runs graphs)
};
static std::map<std::string, Tuned> g_tuned;

static std::string signature(const lbm_params *ps, int n, int flags)
{
    std::map<std::pair<int, int>, int> hist;
    for (int l = 0; l < n; ++l)
        hist[{ps[l].nx, ps[l].ny}]++;
    std::string s = "gfx950/q" + std::to_string(ps[0].lattice == LBM_D2Q9 ? 9 : 7) + "/m" +
                    std::to_string(ps[0].model) + "/s" + std::to_string(ps[0].storage) + "/f" + std::to_string(flags);
    for (auto &h : hist)
        s += "/" + std::to_string(h.first.first) + "x" + std::to_string(h.first.second) + ":" +
             std::to_string(h.second);
    return s;
}

// Instantiated sample-period graphs, least recently used first out.
struct GraphKey {
    int device;
    const void *tiles_main, *tiles_one, *lat, *ctrl, *mt, *part, *colpart, *colmean, *results;
    int lattice, model, storage, flags, shape;
    int64_t ntiles_main, ntiles_one, nmt, n, n_samples, steps;
    int sample, add, rev, split;
    int max_nx;                   // the column means' grid
    int multi_T, multi_tx, multi_ty;  // geometry of the several-steps form
    std::vector<int64_t> groups;  // tile ranges of the lattice groups and branches
    auto tie() const
    {
        return std::tie(device, tiles_main, tiles_one, lat, ctrl, mt, part, colpart, colmean, results, lattice, model,
                        storage, flags, shape, ntiles_main, ntiles_one, nmt, n, n_samples, steps, sample, add, rev, split,
                        max_nx, multi_T, multi_tx, multi_ty, groups);
    }
    bool operator==(const GraphKey &o) const { return tie() == o.tie(); }
};

// An executable graph, destroyed when the last holder lets go (the cache or
// a call still running it).
// An instantiated graph and an event recorded after its latest launch: a
// sweep returns without waiting for its graphs, so an exec evicted from the
// cache (or released at the end of a call) waits for that launch to finish
// before it is destroyed.
struct GraphExec {
    hipGraphExec_t exec = nullptr;
    hipEvent_t done = nullptr;
    hipError_t launched(hipStream_t s)
    {
        if (!done) {
            hipError_t e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
            if (e != hipSuccess) {
                done = nullptr;
                return e;
            }
        }
        return hipEventRecord(done, s);
    }
    ~GraphExec()
    {
        if (done) {
            (void)hipEventSynchronize(done);
            (void)hipEventDestroy(done);
        }
        if (exec)
            (void)hipGraphExecDestroy(exec);
    }
};
using GraphPtr = std::shared_ptr<GraphExec>;

constexpr size_t kGraphCacheSize = 16;
static std::mutex g_graph_mu;
// most recently used last; never destroyed, so no HIP call runs from a static
// destructor after the runtime may have shut down at process exit
static auto &g_graphs = *new std::vector<std::pair<GraphKey, GraphPtr>>();

static GraphPtr graph_cache_get(const GraphKey &k)
{
    std::lock_guard<std::mutex> lk(g_graph_mu);
    for (size_t i = 0; i < g_graphs.size(); ++i)
        if (g_graphs[i].first == k) {
            auto hit = g_graphs[i];
            g_graphs.erase(g_graphs.begin() + (ptrdiff_t)i);
            g_graphs.push_back(hit);
            return hit.second;
        }
    return nullptr;
}

static void graph_cache_put(const GraphKey &k, const GraphPtr &g)
{
    std::lock_guard<std::mutex> lk(g_graph_mu);
    if (g_graphs.size() >= kGraphCacheSize)
        g_graphs.erase(g_graphs.begin());
    g_graphs.emplace_back(k, g);
}

// What this library last wrote into the tables of a workspace (lattice
// descriptors, moments tiles and the tile list held in each of the three list
// regions), per device and workspace address.  A call with keep_tables set
// takes the record at its word (its caller has not written into the
// workspace since) and uploads only the tables that differ, so a repeated
// sweep of the same batch starts its first kernel without host work.
struct WsTables {
    int lattice = -1;
    std::vector<std::pair<int32_t, int32_t>> sizes;  // (nx, ny) of each lattice, in batch order
    std::vector<LatDesc> lat;
    int region[3] = {-1, -1, -1};  // shape whose list is in the one-step / two-step / several-steps region
    // lattice groups in reverse order in the next call: each call starts with
    // the group the previous one ended with, whose state is still in the
    // Infinity Cache
    bool rev_next = false;
};
constexpr size_t kWsRecords = 64;
static std::mutex g_ws_mu;
static auto &g_ws = *new std::map<std::pair<int, const void *>, WsTables>();

// Field-by-field equality (bit patterns: +0 and -0 differ), so padding bytes
// play no part.
#define LBM_SAME(f) (memcmp(&x.f, &y.f, sizeof(x.f)) == 0)
static bool same_args(const StepArgs &x, const StepArgs &y)
{
    return LBM_SAME(nx) && LBM_SAME(ny) && LBM_SAME(pitch) && LBM_SAME(plane) && LBM_SAME(omega) &&
           LBM_SAME(noise_scale) && LBM_SAME(noise_h) && LBM_SAME(A16) && LBM_SAME(B16) && LBM_SAME(C2) && LBM_SAME(rho_star) &&
           LBM_SAME(inv_rho_star) && LBM_SAME(u_max2) && LBM_SAME(wr0) && LBM_SAME(wr1) && LBM_SAME(wr2) &&
           LBM_SAME(key0) && LBM_SAME(key1) && LBM_SAME(noisy);
}
static bool same_desc(const LatDesc &x, const LatDesc &y)
{
    return same_args(x.a, y.a) && LBM_SAME(buf) && LBM_SAME(B) && LBM_SAME(mt_begin) && LBM_SAME(mt_count) &&
           LBM_SAME(nrb) && LBM_SAME(col_off) && LBM_SAME(cm_off) && LBM_SAME(add) && LBM_SAME(stream);
}
#undef LBM_SAME

// Copy a sweep's samples (8 doubles each, lattice-major) to the host after
// the stream's work and turn them into lbm_obs.
static int32_t read_samples(const lbm_params *ps, int n, int64_t n_samples, const double *d_results, hipStream_t s,
                            lbm_obs *out)
{
    const size_t results = (size_t)n * n_samples;
    std::vector<double> res(results * 8);
    HostResult host(results, s);
    LBM_HIP_TRY(host.fetch(d_results, res.data(), results, s));
    bool bad = false;
    for (int l = 0; l < n; ++l)
        for (int64_t k = 0; k < n_samples; ++k) {
            const double *r = &res[((size_t)l * n_samples + k) * 8];
            lbm_obs &ob = out[(size_t)l * n_samples + k];
            finish_obs(ps[l], r, (int64_t)r[7], &ob);
            bad = bad || ob.nonfinite;
        }
    if (bad)
        return fail(LBM_ENONFINITE, "non-finite populations in a batch sample");
    return LBM_OK;
}

}  // namespace lbm

using namespace lbm;

extern "C" {

int32_t lbm_sweep_groups(const lbm_params *ps, int32_t n)
{
    if (!ps || n <= 0)
        return fail(LBM_EINVAL, "null parameters or empty batch");
    return (int32_t)cache_groups(ps, n).size() - 1;
}

int32_t lbm_sweep_tile_rows(const lbm_params *ps, int32_t n)
{
    if (!ps || n <= 0)
        return fail(LBM_EINVAL, "null parameters or empty batch");
    const int flags = sweep_flags(ps, n);
    if (flags < 0)
        return 0;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tuned.find(signature(ps, n, flags));
    if (it == g_tuned.end())
        return 0;
    return it->second.tile == kResident ? LBM_TILE_RESIDENT : kShapes[it->second.tile].ty;
}

// For the tests alone (in no header): the form and branches that a batch of these
// lattices was tuned to, 0 where it was not yet (1: by a call without graphs, which
// times no branches, 2: by one with them); and the same set by hand, as if
// tuned, for a form that such a batch may take (so that each form is reached on
// every machine).  Forms: kShapes, kResident, kMulti.
int32_t lbm_test_tuned(const lbm_params *ps, int32_t n, int32_t *form, int32_t *split)
{
    const int flags = ps && n > 0 ? sweep_flags(ps, n) : -1;
    if (flags < 0 || !form || !split)
        return fail(LBM_EINVAL, "invalid lbm_test_tuned arguments");
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tuned.find(signature(ps, n, flags));
    if (it == g_tuned.end())
        return 0;
    *form = it->second.shape;
    *split = it->second.split;
    return it->second.branches ? 2 : 1;
}

int32_t lbm_test_tune(const lbm_params *ps, int32_t n, int32_t form, int32_t split)
{
    const int flags = ps && n > 0 ? sweep_flags(ps, n) : -1;
    if (flags < 0 || split < 0 || split > 1)
        return fail(LBM_EINVAL, "invalid lbm_test_tune arguments");
    const std::vector<int> shapes = batch_shapes(ps[0]);
    const bool tile = std::count(shapes.begin(), shapes.end(), form) > 0;
    if (!tile && !(form == kResident && resident_fits(ps, n)) && !(form == kMulti && multi_for_batch(ps, n).T))
        return fail(LBM_EINVAL, "a form that this batch may not take");
    if (split && !(tile && kShapes[form].steps == 2 && n > 1))
        return fail(LBM_EINVAL, "branches that this form does not take");
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned[signature(ps, n, flags)] = Tuned{form, split, form, named_shape(form) ? form : shapes[0], true};
    return LBM_OK;
}

size_t lbm_sweep_workspace_bytes(const lbm_params *ps, int32_t n, int64_t n_samples)
{
    if (!ps || n <= 0 || n_samples < 0)
        return 0;
    return layout(ps, n, n_samples).total;
}

int32_t lbm_sweep_batch(const lbm_params *ps, int32_t n, const lbm_sweep_opts *o, void *const *bufs, void *ws,
                        size_t ws_bytes, void *stream, lbm_obs *out)
{
    if (!ps || n <= 0 || !o || !bufs || !ws)
        return fail(LBM_EINVAL, "null argument or empty batch");
    if (o->n_steps < 0 || o->sample_every < 0 || o->step0 < 0)
        return fail(LBM_EINVAL, "negative step counts");
    if (o->use_graph < 0 || o->use_graph > 2)
        return fail(LBM_EINVAL, "use_graph must be 0, 1 or 2");
    if (o->drho)
        for (int l = 0; l < n; ++l)
            if (!isfinite(o->drho[l]))
                return fail(LBM_EINVAL, "drho must be finite");
    for (int l = 0; l < n; ++l) {
        int32_t rc = validate_params(&ps[l], ps[l].nx);
        if (rc)
            return fail(rc, "lattice " + std::to_string(l) + ": " + lbm_last_error());
        if (ps[l].lattice != ps[0].lattice)
            return fail(LBM_EINVAL, "all lattices of a batch must use the same velocity set");
        if (ps[l].storage != ps[0].storage)
            return fail(LBM_EINVAL, "all lattices of a batch must use the same storage");
        if (ps[l].storage != LBM_F32 && ps[l].lattice == LBM_D2Q9)
            return fail(LBM_EUNSUPPORTED, "batched D2Q9 sweeps take F32 storage");
        if (ps[l].model != ps[0].model)
            return fail(LBM_EINVAL, "all lattices of a batch must use the same model");
        if ((uint64_t)ps[l].nx * ps[l].ny * (ps[l].lattice == LBM_D2Q9 ? 9ull : 7ull) >= (1ull << 30))
            return fail(LBM_EINVAL, "batch lattices must hold fewer than 2^30 populations");
        if (!bufs[2 * l] || !bufs[2 * l + 1] || bufs[2 * l] == bufs[2 * l + 1])
            return fail(LBM_EINVAL, "lattice " + std::to_string(l) + ": null or equal buffers");
        if (ps[l].ny > 32760 || ps[l].nx > 64 * 32760)
            return fail(LBM_EINVAL, "batch lattices need ny <= 32760 and nx <= 2096640 (16-bit tile indices)");
    }
    const int flags = sweep_flags(ps, n);
    if (flags < 0)
        return fail(LBM_EINVAL, "all lattices of a batch must agree on tau == 1 and on sigma == 0");
    const int64_t period = o->sample_every > 0 ? o->sample_every : o->n_steps;
    const int64_t n_samples = o->sample_every > 0 ? o->n_steps / o->sample_every : 1;
    if (o->sample_every > 0 && o->n_steps % o->sample_every != 0)
        return fail(LBM_EINVAL, "n_steps must be a multiple of sample_every");
    const Layout Ly = layout(ps, n, n_samples);
    if (ws_bytes < Ly.total)
        return fail(LBM_EINVAL, "workspace smaller than lbm_sweep_workspace_bytes()");
    if (o->surrogate)
        return surrogate_sweep(ps, n, o, bufs, ws, ws_bytes, (hipStream_t)stream, out);
    // tile shape: caller's choice (tile_rows 1, 2, 4: 256x1, 128x2, 64x4
    // sites, one step per launch; 8, 16: 64x8, 64x16 sites, two steps per
    // launch; MIPS 8, 16 and, D2Q7 only, 4 with one step per launch),
    // else the tuned one for
    // this signature, else tuned below: every tuning launch reads the state
    // in the first buffer of each lattice and writes the second (free until
    // the sweep starts), so the state is unchanged.
    int shape = -1, split = 0;
    const bool mips = ps[0].model == LBM_MIPS, q9 = ps[0].lattice == LBM_D2Q9;
    std::vector<int> cands = batch_shapes(ps[0]);
    for (int k : cands)
        if (named_shape(k) && o->tile_rows == kShapes[k].ty)
            shape = k;
    const bool resident_ok = resident_fits(ps, n);
    if (resident_ok)
        cands.push_back(kResident);
    const MultiChoice mc = multi_for_batch(ps, n);
    if (mc.T)
        cands.push_back(kMulti);
    if (o->tile_rows == LBM_TILE_RESIDENT) {
        if (!resident_ok)
            return fail(LBM_EINVAL, "tile_rows LBM_TILE_RESIDENT needs lattices of at most " +
                                        std::to_string(kResidentSites) + " (D2Q7) or " +
                                        std::to_string(kResidentSitesQ9) + " (D2Q9) sites");
        shape = kResident;
    }
    if (shape < 0 && o->tile_rows != 0)
        return fail(LBM_EINVAL, mips ? (q9 ? "D2Q9 MIPS batches take tile_rows 0, 8, 16 or LBM_TILE_RESIDENT"
                                          : "MIPS batches take tile_rows 0, 4, 8, 16 or LBM_TILE_RESIDENT")
                                     : "tile_rows must be 0, 1, 2, 4, 8, 16 or LBM_TILE_RESIDENT");
    const std::string sig = signature(ps, n, flags);
    if (shape < 0) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tuned.find(sig);
        // what a call without graphs has tuned lacks the branches
        if (it != g_tuned.end() && (it->second.branches || !o->use_graph)) {
            shape = o->use_graph ? it->second.shape : it->second.direct;
            split = o->use_graph ? it->second.split : 0;
        }
    }
    hipStream_t s = (hipStream_t)stream;
    char *w = (char *)ws;
    LatDesc *d_lat = (LatDesc *)(w + Ly.lat);
    BatchTile *d_tiles = (BatchTile *)(w + Ly.tiles);
    MomTile *d_mt = (MomTile *)(w + Ly.mtiles);
    Ctrl *d_ctrl = (Ctrl *)(w + Ly.ctrl);
    double *d_part = (double *)(w + Ly.part);
    double *d_colpart = (double *)(w + Ly.colpart);
    double *d_colmean = (double *)(w + Ly.colmean);
    double *d_results = (double *)(w + Ly.results);

    // descriptors (and the moments tiles: per lattice, cx x cy tiles of 256
    // columns x kMomRows rows)
    std::vector<LatDesc> lat(n);
    std::vector<std::pair<int32_t, int32_t>> sizes(n);
    int64_t col_off = 0, cm_off = 0, nmt = 0;
    for (int l = 0; l < n; ++l) {
        LatDesc &D = lat[l];
        D.a = make_step_args(ps[l], ps[l].nx);
        D.buf[0] = bufs[2 * l];
        D.buf[1] = bufs[2 * l + 1];
        D.B = (float)ps[l].B;
        D.add = o->drho ? (float)(o->drho[l] / (ps[l].lattice == LBM_D2Q9 ? 9.0 : 7.0)) : 0.0f;
        D.stream = state_bytes(ps[l]) > kCacheGroupBytes ? 1 : 0;
        const int cx = (ps[l].nx + 255) / 256, cy = (ps[l].ny + kMomRows - 1) / kMomRows;
        D.mt_begin = (int32_t)nmt;
        D.mt_count = cx * cy;
        D.nrb = cy;
        D.col_off = col_off;
        D.cm_off = cm_off;
        nmt += (int64_t)cx * cy;
        col_off += (int64_t)cy * ps[l].nx;
        cm_off += ps[l].nx;
        sizes[l] = {ps[l].nx, ps[l].ny};
    }
    // the workspace's record: a copy, written back once the uploads are enqueued
    int dev = 0;
    LBM_HIP_TRY(hipGetDevice(&dev));
    const std::pair<int, const void *> ws_key{dev, ws};
    WsTables rec;
    if (o->keep_tables) {
        std::lock_guard<std::mutex> lk(g_ws_mu);
        auto it = g_ws.find(ws_key);
        if (it != g_ws.end())
            rec = it->second;
    }
    const bool same_sizes = rec.lattice == ps[0].lattice && rec.sizes == sizes;
    if (!same_sizes)
        rec.region[0] = rec.region[1] = rec.region[2] = -1;
    bool same_lat = same_sizes && rec.lat.size() == lat.size();
    for (int l = 0; l < n && same_lat; ++l)
        same_lat = same_desc(rec.lat[l], lat[l]);
    // host copies of the uploaded tables stay alive until the stream is
    // synchronised at the end of this call
    std::vector<MomTile> mt;
    std::vector<std::vector<BatchTile>> host_lists;
    auto save_record = [&]() {
        std::lock_guard<std::mutex> lk(g_ws_mu);
        if (g_ws.size() >= kWsRecords && !g_ws.count(ws_key))
            g_ws.erase(g_ws.begin());
        g_ws[ws_key] = rec;
    };
    // a failed call leaves the workspace's tables unknown
    auto forget_record = [&]() {
        std::lock_guard<std::mutex> lk(g_ws_mu);
        g_ws.erase(ws_key);
    };

    forget_record();  // until this call has written every table it uses
    const bool uploaded_desc = !same_lat || !same_sizes;
    if (!same_lat)
        LBM_HIP_TRY(hipMemcpyAsync(d_lat, lat.data(), sizeof(LatDesc) * n, hipMemcpyHostToDevice, s));
    if (!same_sizes) {
        mt.reserve((size_t)nmt);
        for (int l = 0; l < n; ++l) {
            const int cx = (ps[l].nx + 255) / 256, cy = (ps[l].ny + kMomRows - 1) / kMomRows;
            for (int j = 0; j < cy; ++j)
                for (int i = 0; i < cx; ++i)
                    mt.push_back(MomTile{l, (int16_t)i, (int16_t)j});
        }
        LBM_HIP_TRY(hipMemcpyAsync(d_mt, mt.data(), sizeof(MomTile) * mt.size(), hipMemcpyHostToDevice, s));
    }
    rec.lattice = ps[0].lattice;
    rec.sizes = sizes;
    rec.lat = lat;
    BatchTile *d_tiles1 = d_tiles, *d_tiles2 = d_tiles + Ly.n_tiles1;
    hipError_t up_err = hipSuccess;
    // the tile list of shape k in its region (one-step shapes in the first, two-step
    // shapes in the second, the several-steps form in the third), uploaded unless the
    // region holds it
    auto upload = [&](int k) -> std::pair<BatchTile *, int64_t> {
        const int r = k == kMulti ? 2 : kShapes[k].steps == 1 ? 0 : 1;
        BatchTile *d = r == 0 ? d_tiles1 : r == 1 ? d_tiles2 : (BatchTile *)(w + Ly.tiles3);
        const int64_t count = k == kMulti ? count_multi_tiles(ps, n, mc) : count_tiles(ps, n, kShapes[k].tx, kShapes[k].ty);
        // the several-steps list also depends on the model (its geometry)
        const int held = k == kMulti ? k | mc.tx << 8 | mc.ty << 16 : k;
        if (rec.region[r] == held)
            return {d, count};
        host_lists.push_back(k == kMulti ? build_multi_tiles(ps, n, mc) : build_tiles(ps, n, kShapes[k].tx, kShapes[k].ty));
        const std::vector<BatchTile> &v = host_lists.back();
        up_err = hipMemcpyAsync(d, v.data(), sizeof(BatchTile) * v.size(), hipMemcpyHostToDevice, s);
        rec.region[r] = up_err == hipSuccess ? held : -1;
        return {up_err == hipSuccess ? d : nullptr, (int64_t)v.size()};
    };
    // one launch of `st` steps of form k over `count` tiles from `tl`
    auto launch_form = [&](int k, int st, const BatchTile *tl, int64_t count, int step_off, int launch_off,
                           hipStream_t on) -> hipError_t {
        if (k == kMulti)
            return launch_batch_multi(ps[0].lattice, ps[0].model, ps[0].storage, flags,
                                      multi_geom(ps[0].model, st, mc.tx, mc.ty), count, tl, d_lat, d_ctrl, step_off,
                                      launch_off, on);
        return launch_batch_step(ps[0].lattice, ps[0].model, ps[0].storage, flags, k, count, tl, d_lat, d_ctrl,
                                 step_off, launch_off, on);
    };
    // Two branches of a captured graph: a lattice group's launches are cut into
    // two halves of its lattices, which need not wait for each other, so one
    // half's launches fill the CUs that the other's last blocks and its next
    // launch's first loads leave idle (whole launches of 35 to 47 us, two to five
    // rounds of blocks, issue vector instructions in 68 to 72% of the cycles, a
    // 4096^2 lattice's in 81%).  Taken where the tuning finds it 3% faster:
    // 48 lattices of 128^2 to 512^2 2.54 -> 2.29 ms per 100 steps, the 50 steps
    // of 64 lattices of 256^2 in a surrogate's judge 1.36 -> 1.18 ms, 20 steps of
    // five lattices of 1024^2 713 -> 697 us; three or four branches are slower.
    // The fork and the join cost about 10 us a graph, so graphs of fewer than
    // kBranchLaunches launches stay on one branch.
    struct Fork {
        hipStream_t side = nullptr;  // the second branch, while capturing
        std::vector<hipEvent_t> events;
        hipError_t after(hipStream_t from, hipStream_t to)  // to's next work waits for from's
        {
            hipEvent_t ev = nullptr;
            hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
            if (e != hipSuccess)
                return e;
            events.push_back(ev);
            e = hipEventRecord(ev, from);
            return e == hipSuccess ? hipStreamWaitEvent(to, ev, 0) : e;
        }
        hipError_t open() { return side ? hipSuccess : hipStreamCreateWithFlags(&side, hipStreamNonBlocking); }
        void close()  // once the capture has ended
        {
            for (hipEvent_t ev : events)
                (void)hipEventDestroy(ev);
            events.clear();
            if (side)
                (void)hipStreamDestroy(side);
            side = nullptr;
        }
        ~Fork() { close(); }
    } fork;
    // run(stream, first, last) for lattices first .. last - 1 of every group gf[g]
    // .. gf[g + 1] - 1 in turn (the last group first where `backwards`).  Where
    // fork is open, as two branches of the capture on s, each taking half of
    // every group: they meet at the end only (a join costs about 9 us).
    auto branches = [&](const std::vector<int> &gf, bool backwards, auto run) -> hipError_t {
        const size_t ng = gf.size() - 1;
        auto half = [&](hipStream_t on, int which) -> hipError_t {
            for (size_t k = 0; k < ng; ++k) {
                const size_t g = backwards ? ng - 1 - k : k;
                const int cut = fork.side ? branch_cut(ps, gf[g], gf[g + 1]) : gf[g + 1];
                const int first = which ? cut : gf[g], last = which ? gf[g + 1] : cut;
                const hipError_t e = first < last ? run(on, first, last) : hipSuccess;
                if (e != hipSuccess)
                    return e;
            }
            return hipSuccess;
        };
        if (!fork.side)
            return half(s, 0);
        hipError_t e = fork.after(s, fork.side);
        if (e != hipSuccess)
            return e;
        e = half(s, 0);
        if (e == hipSuccess)
            e = half(fork.side, 1);
        const hipError_t j = fork.after(fork.side, s);
        return e != hipSuccess ? e : j;
    };
    // first tile of lattice l in the list of form k, and the count up to `last`
    auto tile_range = [&](int k, int l, int last) -> std::pair<int64_t, int64_t> {
        auto count = [&](int a, int b) {
            return k == kMulti ? count_multi_tiles(ps + a, b - a, mc)
                               : count_tiles(ps + a, b - a, kShapes[k].tx, kShapes[k].ty);
        };
        return {count(0, l), count(l, last)};
    };
    if (shape < 0) {
        // each form: ten launches captured in a graph (as the sweep runs them), replayed
        // and timed; the least time per step wins
        struct Form {
            int k, split, steps;  // steps of a launch
            hipGraphExec_t exec = nullptr;
            float replay = 1e30f;  // least ms of a replay
            // Per ten steps.  3% against branches, and against the two-step tiles of eight
            // rows: these issue 8% more vector instructions than those of 16, which bursts
            // as short as a replay show less of than a sweep at the clock that the card
            // then holds (five lattices of 1024^2, 2000 steps: 168 / 176 GLUPS).
            float ms() const
            {
                const bool eight = k < kNumShapes && kShapes[k].steps == 2 && kShapes[k].ty == 8;
                return (k == kResident ? replay * 10.0f : replay) / (float)steps * (split ? 1.03f : 1.0f) *
                       (eight ? 1.03f : 1.0f);
            }
        };
        struct Tuning {  // destroyed on every exit path
            std::vector<Form> forms;
            hipEvent_t a = nullptr, b = nullptr;
            ~Tuning()
            {
                for (Form &f : forms)
                    if (f.exec)
                        (void)hipGraphExecDestroy(f.exec);
                if (a)
                    (void)hipEventDestroy(a);
                if (b)
                    (void)hipEventDestroy(b);
            }
        } tuning;
        LBM_HIP_TRY(hipEventCreate(&tuning.a));
        LBM_HIP_TRY(hipEventCreate(&tuning.b));
        hipLaunchKernelGGL(k_batch_set_ctrl, dim3(1), dim3(64), 0, s, d_ctrl, (int64_t)0);
        const std::vector<int> tfirst = cache_groups(ps, n);
        // the form's list, in its region while the form runs (forms share regions)
        auto list_of = [&](int k) {
            return k == kResident ? std::pair<BatchTile *, int64_t>{d_tiles1, 0} : upload(k);
        };
        auto capture_form = [&](Form &f) -> hipError_t {
            const auto tl = list_of(f.k);
            if (!tl.first)
                return up_err;
            hipError_t e = f.split ? fork.open() : hipSuccess;
            hipStream_t cap = nullptr;
            if (e == hipSuccess)
                e = hipStreamCreateWithFlags(&cap, hipStreamNonBlocking);
            if (e != hipSuccess)
                return e;
            hipGraph_t g = nullptr;
            const hipStream_t saved = s;
            s = cap;
            e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
            if (f.k == kResident && e == hipSuccess)  // first buffer -> second buffer
                e = launch_resident(ps[0].lattice, ps[0].model, ps[0].storage, flags, n, d_lat, d_ctrl, f.steps, s);
            // ten launches per lattice group, group after group, as the sweep runs them
            else if (e == hipSuccess)
                e = branches(tfirst, false, [&](hipStream_t on, int first, int last) -> hipError_t {
                    const auto r = tile_range(f.k, first, last);
                    hipError_t le = hipSuccess;
                    for (int r10 = 0; r10 < 10 && le == hipSuccess; ++r10)
                        le = launch_form(f.k, f.steps, tl.first + r.first, r.second, 0, 0, on);
                    return le;
                });
            s = saved;
            const hipError_t ee = hipStreamEndCapture(cap, &g);
            (void)hipStreamDestroy(cap);
            fork.close();
            if (e == hipSuccess)
                e = ee;
            if (e == hipSuccess)
                e = hipGraphInstantiate(&f.exec, g, nullptr, nullptr, 0);
            if (g)
                (void)hipGraphDestroy(g);
            return e;
        };
        auto time_form = [&](Form &f, int reps) -> hipError_t {
            hipError_t e = list_of(f.k).first ? hipSuccess : up_err;
            for (int rep = 0; rep < reps && e == hipSuccess; ++rep) {
                e = hipEventRecord(tuning.a, s);
                if (e == hipSuccess)
                    e = hipGraphLaunch(f.exec, s);
                if (e == hipSuccess)
                    e = hipEventRecord(tuning.b, s);
                if (e == hipSuccess)
                    e = hipEventSynchronize(tuning.b);
                float m = 0.0f;
                if (e == hipSuccess)
                    e = hipEventElapsedTime(&m, tuning.a, tuning.b);
                f.replay = std::min(f.replay, m);
            }
            return e;
        };
        // captured and timed once, and again where the first replay's own cost (some
        // 50 us) would count
        auto try_form = [&](int k, int with_branches) -> hipError_t {
            Form f;
            f.k = k;
            f.split = with_branches;
            f.steps = k == kResident ? kResidentTuneSteps : k == kMulti ? mc.T : kShapes[k].steps;
            tuning.forms.push_back(f);
            Form &t = tuning.forms.back();
            hipError_t e = capture_form(t);
            if (e == hipSuccess)
                e = time_form(t, 1);
            return e == hipSuccess && t.replay < 0.4f ? time_form(t, 1) : e;
        };
        // these forms once more each, in turn `rounds` times: the card's clock falls while
        // it works, so times taken one form after another favour the first
        auto compare = [&](const std::vector<Form *> &fs, int rounds) -> hipError_t {
            hipError_t e = hipSuccess;
            for (Form *f : fs)
                f->replay = 1e30f;
            for (int r = 0; r < rounds; ++r)
                for (size_t i = 0; i < fs.size() && e == hipSuccess; ++i)
                    e = time_form(*fs[i], 1);
            return e;
        };
        auto best_of = [&](const std::vector<Form *> &fs) {
            return *std::min_element(fs.begin(), fs.end(), [](Form *x, Form *y) { return x->ms() < y->ms(); });
        };
        // Every form once; those near the best against each other; the best against the best
        // two-step shape as two branches.  A batch's first call, ms, with
        // three or six replays of every form and of its branches / so: 48 lattices of 128^2
        // to 512^2 22.1 / 13.0, two of 4096^2 151 / 59, three of 1000x752 D2Q9 MIPS 24 / 9.6.
        tuning.forms.reserve(cands.size() + 1);
        hipError_t e = hipSuccess;
        for (size_t i = 0; i < cands.size() && e == hipSuccess; ++i)
            e = try_form(cands[i], 0);
        if (e != hipSuccess)
            return hip_fail(e, "tile-shape tuning");
        std::vector<Form *> all, near;
        for (Form &f : tuning.forms)
            all.push_back(&f);
        const float limit = 1.12f * best_of(all)->ms();
        for (Form *f : all)
            if (f->ms() <= limit)
                near.push_back(f);
        if (near.size() > 1)
            e = compare(near, 2);
        Form *best = best_of(near);
        auto named_among = [&](std::vector<Form *> fs) -> Form * {
            fs.erase(std::remove_if(fs.begin(), fs.end(), [](Form *f) { return !named_shape(f->k); }), fs.end());
            return fs.empty() ? nullptr : best_of(fs);
        };
        Form *const close = named_among(near), *const named = close ? close : named_among(all);
        Form *const single = best;
        std::vector<Form *> pairs;  // two-step shapes among them
        for (Form *f : near)
            if (f->k < kNumShapes && kShapes[f->k].steps == 2)
                pairs.push_back(f);
        Form *const pair = pairs.empty() ? nullptr : best_of(pairs);
        if (e == hipSuccess && n > 1 && o->use_graph && pair) {
            e = try_form(pair->k, 1);
            Form *two = &tuning.forms.back();
            if (e == hipSuccess && two->ms() <= 1.2f * best->ms())
                e = compare({best, two}, best->replay < 0.7f ? 6 : 3);
            best = best_of({best, two});
        }
        if (e != hipSuccess)
            return hip_fail(e, "tile-shape tuning");
        shape = best->k;
        split = best->split;
        // calls with and without graphs in turn would upload their tile lists each time (45
        // us) if they ran in shapes of their own
        const int direct = split && pair->ms() <= 1.05f * single->ms() ? pair->k : single->k;
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tuned[sig] = Tuned{shape, split, direct, named->k, o->use_graph != 0 || n == 1};
    }
    // the chosen list, and for a two-step shape the list of a one-step shape
    // (256x1; MIPS 64x4, D2Q9 MIPS 64x16) for the single steps that keep the launch count's
    // parity equal to the step count's (so the state ends in
    // bufs[2l + (n_steps & 1)])
    const bool resident = shape == kResident;
    const bool two = !resident && shape != kMulti && kShapes[shape].steps == 2;
    const int one_shape = two ? (mips ? (q9 ? kMipsShape : kMipsShape4) : 0) : shape;
    const int64_t most = resident ? 0 : shape == kMulti ? mc.T : kShapes[shape].steps;  // steps per launch
    std::pair<BatchTile *, int64_t> main_list{d_tiles1, 0};
    if (!resident) {
        main_list = upload(shape);
        if (!main_list.first)
            return hip_fail(up_err, "tile list upload");
    }
    std::pair<BatchTile *, int64_t> one_list = main_list;
    if (two) {
        one_list = upload(one_shape);
        if (!one_list.first)
            return hip_fail(up_err, "tile list upload");
    }
    int max_nx = 0;
    for (int l = 0; l < n; ++l)
        max_nx = std::max(max_nx, ps[l].nx);
    hipLaunchKernelGGL(k_batch_set_ctrl, dim3(1), dim3(64), 0, s, d_ctrl, (int64_t)o->step0);
    LBM_HIP_TRY(hipGetLastError());
    // lattice groups that fit the Infinity Cache (one group when resident)
    const std::vector<int> gfirst = resident ? std::vector<int>{0, n} : cache_groups(ps, n);
    // first moments tile of each lattice (the list is in lattice order)
    std::vector<int> first_mt(n + 1, 0);
    for (int l = 0; l < n; ++l)
        first_mt[l + 1] = first_mt[l] + lat[l].mt_count;
    // rows of a sampling lane by the tiles of an average group (the sums are the same)
    const bool few_tiles = mom_few_tiles(nmt / (int64_t)(cache_groups(ps, n).size() - 1));
    // the graph's launches depend on each group's and branch's tile ranges in the two
    // lists and in the moments tiles (which do not follow from the former: 128 x 512
    // and 256 x 256 sites are as many step tiles and half as many moments tiles)
    std::vector<int64_t> gkey{few_tiles ? 1 : 0};
    for (size_t g = 0; g + 1 < gfirst.size() && !resident; ++g)
        for (int l : {gfirst[g], split ? branch_cut(ps, gfirst[g], gfirst[g + 1]) : gfirst[g + 1]})
            for (int k : {shape, one_shape}) {
                const auto r = tile_range(k, l, gfirst[g + 1]);
                gkey.push_back(r.first);
                gkey.push_back(r.second);
                gkey.push_back(first_mt[l]);
            }

    // the order of the lattice groups in this call, and in the next one
    const bool rev = !resident && gfirst.size() > 2 && rec.rev_next;
    rec.rev_next = o->use_graph == 2 ? rev : (!resident && gfirst.size() > 2 && !rev);
    // the sample's moments of lattices first .. last - 1: right after their last
    // launch, while their state is still in the Infinity Cache
    auto moments = [&](hipStream_t on, int first, int last, int64_t steps) {
        const int base = first_mt[first], cnt = first_mt[last] - base;
        auto go = [&](auto q, auto st, auto rows) {
            constexpr int R = decltype(rows)::value;
            hipLaunchKernelGGL((k_batch_moments<decltype(q)::value, decltype(st)::value, R>), dim3((unsigned)cnt),
                               dim3(mom_lanes(R)), 0, on, d_mt, d_lat, d_ctrl, (int)steps, base, d_part, d_colpart);
        };
        auto rows = [&](auto q, auto st) {
            few_tiles ? go(q, st, IntTag<4>{}) : go(q, st, IntTag<kMomRows>{});
            return hipSuccess;
        };
        if (q9)
            rows(IntTag<9>{}, IntTag<kF32>{});
        else
            (void)with_storage(ps[0].storage, [&](auto st) { return rows(IntTag<7>{}, st); });
    };
    // `steps` steps, then the sample if asked, then the counter update
    auto enqueue = [&](int64_t steps, bool sample) -> hipError_t {
        if (resident && steps > 0) {
            hipError_t e = launch_resident(ps[0].lattice, ps[0].model, ps[0].storage, flags, n, d_lat, d_ctrl, (int)steps, s);
            if (e != hipSuccess)
                return e;
        }
        if (resident && sample)
            moments(s, 0, n, steps);
        // every launch of the chunk for one lattice group, then the next; as few
        // launches as the form allows, an odd number where the steps are (the
        // buffer parity), the steps dealt evenly over them
        if (!resident) {
            int64_t launches = (steps + most - 1) / most;
            launches += (launches ^ steps) & 1;
            hipError_t e = branches(gfirst, rev, [&](hipStream_t on, int first, int last) -> hipError_t {
                const auto r_main = tile_range(shape, first, last);
                const auto r_one = two ? tile_range(one_shape, first, last) : r_main;
                int64_t done = 0;
                for (int64_t i = 0; i < launches; ++i) {
                    const int st = (int)(steps / launches + (i < steps % launches ? 1 : 0));
                    const bool one = two && st == 1;
                    const hipError_t le =
                        launch_form(one ? one_shape : shape, st,
                                    one ? one_list.first + r_one.first : main_list.first + r_main.first,
                                    one ? r_one.second : r_main.second, (int)done, (int)i, on);
                    if (le != hipSuccess)
                        return le;
                    done += st;
                }
                if (sample)
                    moments(on, first, last, steps);
                return hipGetLastError();
            });
            if (e != hipSuccess)
                return e;
        }
        if (sample) {
            const int sto = ps[0].storage;
            hipLaunchKernelGGL(k_batch_colmeans, dim3((unsigned)((max_nx + 255) / 256), (unsigned)n), dim3(256), 0, s,
                               d_lat, d_colpart, d_colmean);
            hipLaunchKernelGGL(k_batch_final, dim3((unsigned)n), dim3(256), 0, s, d_lat, d_ctrl, (int)steps, d_part,
                               d_colmean, d_results, (int)n_samples);
            if (o->drho && q9)
                hipLaunchKernelGGL((k_batch_add_density<9, kF32>), dim3((unsigned)nmt), dim3(256), 0, s, d_mt, d_lat,
                                   d_ctrl, (int)steps);
            else if (o->drho)
                (void)with_storage(sto, [&](auto st) {
                    hipLaunchKernelGGL((k_batch_add_density<7, decltype(st)::value>), dim3((unsigned)nmt), dim3(256),
                                       0, s, d_mt, d_lat, d_ctrl, (int)steps);
                    return hipSuccess;
                });
        }
        hipLaunchKernelGGL(k_batch_advance, dim3(1), dim3(64), 0, s, d_ctrl, steps, sample ? 1 : 0);
        return hipGetLastError();
    };
    // a sample period runs as `reps` chunks of `chunk` steps and a tail of
    // `tail` steps plus the sample; each of the two pieces is captured once
    // (on a private stream: the caller's may be the legacy null stream, which
    // cannot be captured) and replayed on the caller's stream
    const int64_t chunk = std::min<int64_t>(period, kChunk);
    const int64_t reps = o->n_steps == 0 ? 0 : (period - 1) / chunk;
    const int64_t tail = o->n_steps == 0 ? 0 : period - reps * chunk;
    const int64_t n_periods = o->n_steps == 0 ? 1 : o->n_steps / period;
    auto capture = [&](int64_t steps, bool sample, GraphPtr *ge) -> hipError_t {
        // an instantiated graph bakes in the launch shapes and the workspace
        // addresses it reads (descriptors and tile lists are uploaded again by
        // every call before it runs), so it is kept and replayed by later
        // calls with the same key
        const bool two_branches = split && (steps + most - 1) / most >= kBranchLaunches;
        const GraphKey key{dev, (const void *)main_list.first, (const void *)one_list.first, (const void *)d_lat,
                           (const void *)d_ctrl, (const void *)d_mt, (const void *)d_part, (const void *)d_colpart,
                           (const void *)d_colmean, (const void *)d_results, ps[0].lattice, ps[0].model,
                           ps[0].storage, flags,
                           shape,
                           main_list.second, one_list.second, nmt, (int64_t)n, n_samples, steps, sample ? 1 : 0,
                           o->drho ? 1 : 0, rev ? 1 : 0, two_branches ? 1 : 0, max_nx, mc.T, mc.tx, mc.ty, gkey};
        if ((*ge = graph_cache_get(key)))
            return hipSuccess;
        hipGraph_t g;
        hipStream_t cap;
        hipError_t e = two_branches ? fork.open() : hipSuccess;
        if (e == hipSuccess)
            e = hipStreamCreateWithFlags(&cap, hipStreamNonBlocking);
        if (e != hipSuccess)
            return e;
        hipStream_t saved = s;
        s = cap;
        hipError_t be = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
        hipError_t ce = be == hipSuccess ? enqueue(steps, sample) : be;
        hipError_t ee = be == hipSuccess ? hipStreamEndCapture(cap, &g) : be;
        s = saved;
        (void)hipStreamDestroy(cap);
        fork.close();
        if (ce != hipSuccess)
            return ce;
        if (ee != hipSuccess)
            return ee;
        auto holder = std::make_shared<GraphExec>();
        e = hipGraphInstantiate(&holder->exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e == hipSuccess) {
            *ge = holder;
            graph_cache_put(key, holder);
        }
        return e;
    };
    if (o->use_graph) {
        GraphPtr g_chunk, g_tail;
        hipError_t e = reps > 0 ? capture(chunk, false, &g_chunk) : hipSuccess;
        if (e == hipSuccess)
            e = capture(tail, true, &g_tail);
        if (o->use_graph == 2) {  // prepare only: the graphs are cached, nothing runs
            if (e == hipSuccess)
                e = hipStreamSynchronize(s);
            if (e != hipSuccess)
                return hip_fail(e, "lbm_sweep_batch graph");
            save_record();
            return LBM_OK;
        }
        for (int64_t p = 0; p < n_periods && e == hipSuccess; ++p) {
            for (int64_t r = 0; r < reps && e == hipSuccess; ++r)
                e = hipGraphLaunch(g_chunk->exec, s);
            if (e == hipSuccess)
                e = hipGraphLaunch(g_tail->exec, s);
        }
        // no wait here: each exec remembers its latest launch (GraphExec)
        if (e == hipSuccess && g_chunk && reps > 0 && n_periods > 0)
            e = g_chunk->launched(s);
        if (e == hipSuccess)
            e = g_tail->launched(s);
        if (e != hipSuccess)
            return hip_fail(e, "lbm_sweep_batch graph");
    } else {
        for (int64_t p = 0; p < n_periods; ++p) {
            for (int64_t r = 0; r < reps; ++r)
                LBM_HIP_TRY(enqueue(chunk, false));
            LBM_HIP_TRY(enqueue(tail, true));
        }
    }

    const bool uploaded = uploaded_desc || !host_lists.empty();
    if (!out) {
        // enqueue only: the samples stay in the workspace (lbm_sweep_samples);
        // a call that uploaded tables from host vectors waits for those copies
        if (uploaded)
            LBM_HIP_TRY(hipStreamSynchronize(s));
        save_record();
        return LBM_OK;
    }
    int32_t rc = read_samples(ps, n, n_samples, d_results, s, out);
    if (rc != LBM_EHIP)
        save_record();
    return rc;
}

int32_t lbm_sweep_samples(const lbm_params *ps, int32_t n, int64_t n_samples, const void *ws, void *stream,
                          lbm_obs *out)
{
    if (!ps || n <= 0 || n_samples <= 0 || !ws || !out)
        return fail(LBM_EINVAL, "null argument, empty batch or no samples");
    for (int l = 0; l < n; ++l) {
        int32_t rc = validate_params(&ps[l], ps[l].nx);
        if (rc)
            return fail(rc, "lattice " + std::to_string(l) + ": " + lbm_last_error());
    }
    const Layout Ly = layout(ps, n, n_samples);
    return read_samples(ps, n, n_samples, (const double *)((const char *)ws + Ly.results), (hipStream_t)stream,
                        out);
}

}  // extern "C"
