// Fields and FP64 observables of the stored state, taken (like step (ii) of
// the algorithm) on its streamed populations: rho, u (eq.
// D2Q7macroscopic_u_disc), the order parameter phi (eq. phi), the mean speed,
// zeta and the banding measure (standard deviation over x of the y-averaged
// density), section "Regime Categorisation in the phase diagram".
//
// Pass 1 (k_moments): FP64 sums of tiles of 256 columns x 16 rows, one partial
// per tile, and the tiles' column sums of the density in a [row-block][nx] array.
// Pass 2 (k_column_means, left to pass 3 where the columns are few) sums each
// column over the row blocks, and pass 3 (k_moments_final, one block) adds the
// tile partials and the column means.  All in a fixed order, so the result does
// not depend on scheduling.
#include <algorithm>
#include <mutex>

#include "device_q9.h"
#include "internal.h"
#include "moments.h"

namespace lbm {

static int mom_grid_x(const lbm_params &p) { return (p.nx + kMomCols - 1) / kMomCols; }
static int mom_grid_y(const lbm_params &p) { return (p.ny + kMomRows - 1) / kMomRows; }

size_t moments_scratch_doubles(const lbm_params &p)
{
    const size_t blocks = (size_t)mom_grid_x(p) * mom_grid_y(p);
    return blocks * kMomParts + (size_t)mom_grid_y(p) * p.nx + (size_t)p.nx;
}

// The triangular (Q = 7) or the square (Q = 9) lattice, R rows a lane.
template <int S, int Q, int R>
__global__ __launch_bounds__(mom_lanes(R)) void k_moments(const typename Store<S>::T *__restrict__ src, StepArgs a,
                                                       float *__restrict__ rho_out, float *__restrict__ ux_out,
                                                       float *__restrict__ uy_out, double *__restrict__ part,
                                                       double *__restrict__ colpart)
{
    __shared__ MomLds<R> lds;
    const int x0 = blockIdx.x * kMomCols;
    moments_tile<R, Q>(
        lds, a.nx, a.ny, x0, blockIdx.y * kMomRows,
        [&](float *f, int x, int y) {
            if constexpr (Q == 7) {
                const PullSources g = pull_sources(a, x, y);
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    f[i] = Planes<S>::ld(src, g.idx[i], i, a.plane, a);
            } else {
                const Q9Sources g = q9_sources(a, x, y);
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    f[i] = Store<S>::load(src, i * a.plane + g.idx[i], q9_wr(a, i));
            }
        },
        [](const float *f, float &rho, float &jx, float &jy) {
            if constexpr (Q == 7)
                site_moments(f, rho, jx, jy);
            else
                q9_moments(f, rho, jx, jy);
        },
        [&](int x, int y, float rho, float jx, float jy) {
            const int64_t o = (int64_t)y * a.nx + x;
            if (rho_out)
                rho_out[o] = rho;
            if (ux_out)
                ux_out[o] = rho != 0.0f ? jx / rho : 0.0f;
            if (uy_out)
                uy_out[o] = rho != 0.0f ? jy / rho : 0.0f;
        },
        part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kMomParts, colpart + (int64_t)blockIdx.y * a.nx + x0);
}

// Column means rho_y(x): one thread per column, row blocks in order.
__global__ __launch_bounds__(256) void k_column_means(const double *__restrict__ colpart, int nrowblocks,
                                                      double *__restrict__ colmean, int nx, int ny)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= nx)
        return;
    double c = 0.0;
#pragma unroll 16
    for (int r = 0; r < nrowblocks; ++r)
        c += colpart[(int64_t)r * nx + x];
    colmean[x] = c / (double)ny;
}

// One block: totals of the tile partials and of the column means, then the variance
// of the column means over x; with `host`, the result also goes there (host memory
// that the device can write).  OWN: the column means are summed here (nx <=
// kFinLanes, and few enough partials that one CU reads them in the time of a launch,
// kFinOwn).  The order of every sum is that of k_batch_final, 256 lanes: lane t takes
// terms t, t + 256, ..., then lanes of a wave, then waves.  Here each quarter of the
// block takes one of the tiles' first four sums.
constexpr int kFinLanes = 1024, kFinStride = 256;
constexpr int64_t kFinOwn = 1 << 16;

template <bool OWN>
__global__ __launch_bounds__(kFinLanes) void k_moments_final(const double *__restrict__ part, int nblocks,
                                                             const double *__restrict__ col, int nrowblocks, int nx,
                                                             int ny, double *__restrict__ result, double *host)
{
    __shared__ double lds[kMomParts + 2][kFinStride / 64];
    __shared__ double means[OWN ? kFinLanes : 1];
    const int tid = threadIdx.x, t = tid % kFinStride, quarter = tid / kFinStride;
    auto wave_sum = [&](double v, int k) {
        v = mom_wave_sum(v);
        if ((tid & 63) == 0)
            lds[k][t >> 6] = v;
    };
    auto total = [&](int k) { return ((lds[k][0] + lds[k][1]) + lds[k][2]) + lds[k][3]; };
    double own = 0.0;
    if (OWN && tid < nx) {
#pragma unroll 32
        for (int r = 0; r < nrowblocks; ++r)
            own += col[(int64_t)r * nx + tid];
        means[tid] = own / (double)ny;
    }
    double v = 0.0, last = 0.0;
#pragma unroll 4
    for (int b = t; b < nblocks; b += kFinStride)
        v += part[(int64_t)b * kMomParts + quarter];
    wave_sum(v, quarter);
    if (quarter == 1) {
#pragma unroll 4
        for (int b = t; b < nblocks; b += kFinStride)
            last += part[(int64_t)b * kMomParts + 4];
        wave_sum(last, 4);
    }
    if (OWN)
        __syncthreads();
    const double *cm = OWN ? means : col;
    if (quarter == 0) {
        double m = 0.0;
#pragma unroll 8
        for (int x = t; x < nx; x += kFinStride)
            m += cm[x];
        wave_sum(m, kMomParts);
    }
    __syncthreads();
    const double mean = total(kMomParts) / (double)nx;
    if (quarter == 0) {
        double q = 0.0;
#pragma unroll 8
        for (int x = t; x < nx; x += kFinStride) {
            const double d = cm[x] - mean;
            q += d * d;
        }
        wave_sum(q, kMomParts + 1);
    }
    __syncthreads();
    if (tid < 8) {
        const double r = tid < kMomParts ? total(tid)
                         : tid == 5      ? mean
                         : tid == 6      ? total(kMomParts + 1) / (double)nx
                                         : 0.0;
        result[tid] = r;
        if (host)
            host[tid] = r;
    }
}

hipError_t launch_moments(const lbm_params &p, const StepArgs &a, const void *src, float *rho, float *ux,
                          float *uy, double *scratch, double *result, double *host, hipStream_t s)
{
    const int gx = mom_grid_x(p), gy = mom_grid_y(p);
    double *part = scratch;
    double *colpart = part + (size_t)gx * gy * kMomParts;
    double *colmean = colpart + (size_t)gy * p.nx;
    const bool q9 = p.lattice == LBM_D2Q9;
    const hipError_t e = with_storage(p.storage, [&](auto st) {
        constexpr int S = decltype(st)::value;
        using T = typename Store<S>::T;
        auto go = [&](auto rows) {
            constexpr int R = decltype(rows)::value;
            const dim3 grd(gx, gy), blk(mom_lanes(R));
            if (!q9) {
                hipLaunchKernelGGL((k_moments<S, 7, R>), grd, blk, 0, s, (const T *)src, a, rho, ux, uy, part, colpart);
                return hipSuccess;
            }
            if constexpr (S != kBf16R32) {
                hipLaunchKernelGGL((k_moments<S, 9, R>), grd, blk, 0, s, (const T *)src, a, rho, ux, uy, part, colpart);
                return hipSuccess;
            }
            return hipErrorInvalidValue;
        };
        return mom_few_tiles((int64_t)gx * gy) ? go(IntTag<4>{}) : go(IntTag<kMomRows>{});
    });
    if (e != hipSuccess)
        return e;
    if (p.nx <= kFinLanes && (int64_t)gy * p.nx <= kFinOwn) {
        hipLaunchKernelGGL(k_moments_final<true>, dim3(1), dim3(kFinLanes), 0, s, part, gx * gy, colpart, gy, p.nx, p.ny,
                           result, host);
    } else {
        hipLaunchKernelGGL(k_column_means, dim3((p.nx + 255) / 256), dim3(256), 0, s, colpart, gy, colmean, p.nx, p.ny);
        hipLaunchKernelGGL(k_moments_final<false>, dim3(1), dim3(kFinLanes), 0, s, part, gx * gy, colmean, gy, p.nx, p.ny,
                           result, host);
    }
    return hipGetLastError();
}

// Host memory for results that a kernel writes straight to the host: 64 KB of
// slots of eight doubles, pinned on first use and kept; a run of slots belongs
// to one call at a time.  A copy into pageable memory is only enqueued once the
// host has come to it, and then waits for a staging buffer: 15 us at the end of
// a call whose kernels have ended.
constexpr int kHostSlots = 1024;
static std::mutex g_slot_mu;
static double *g_slot_page;
static bool g_slot_failed, g_slot_used[kHostSlots];

HostResult::HostResult(size_t results, hipStream_t s)
{
    // a captured call fails where it waits for its result, with a kernel in the
    // capture that writes to its slots: it gets none
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cs) != hipSuccess)
        (void)hipGetLastError();
    if (results > (size_t)kHostSlots || cs != hipStreamCaptureStatusNone)
        return;
    std::lock_guard<std::mutex> lk(g_slot_mu);
    if (!g_slot_page && !g_slot_failed) {
        // another thread may be capturing a graph: this one's allocation has no
        // part in it
        void *p = nullptr;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        g_slot_failed = hipHostMalloc(&p, kHostSlots * 8 * sizeof(double), hipHostMallocPortable) != hipSuccess;
        if (swapped)
            (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (g_slot_failed)
            (void)hipGetLastError();
        else
            g_slot_page = (double *)p;
    }
    int run = 0;
    for (int k = 0; k < kHostSlots && g_slot_page && !ptr; ++k) {
        run = g_slot_used[k] ? 0 : run + 1;
        if (run < (int)results)
            continue;
        slot = k + 1 - run;
        count = run;
        std::fill_n(g_slot_used + slot, count, true);
        ptr = g_slot_page + 8 * slot;
    }
}

HostResult::~HostResult()
{
    std::lock_guard<std::mutex> lk(g_slot_mu);
    std::fill_n(g_slot_used + slot, count, false);
}

hipError_t HostResult::read(const double *result, double *r, size_t results, hipStream_t s)
{
    const size_t n = 8 * results;
    hipError_t e = ptr ? hipSuccess : hipMemcpyAsync(r, result, n * sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        count = 0;  // a kernel may still write there: not given back
        return e;
    }
    for (size_t k = 0; k < n && ptr; ++k)
        r[k] = ((const volatile double *)ptr)[k];
    return hipSuccess;
}

__global__ void k_results_to_host(const double *__restrict__ result, int n, double *host)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n)
        host[k] = result[k];
}

hipError_t HostResult::fetch(const double *result, double *r, size_t results, hipStream_t s)
{
    if (ptr && results) {
        const int n = 8 * (int)results;
        hipLaunchKernelGGL(k_results_to_host, dim3((n + 255) / 256), dim3(256), 0, s, result, n, ptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return read(result, r, results, s);
}

void finish_obs(const lbm_params &p, const double *r, int64_t step, lbm_obs *o)
{
    o->step = step;
    o->M = r[0];
    o->Jx = r[1];
    o->Jy = r[2];
    o->phi = r[0] != 0.0 ? sqrt(r[1] * r[1] + r[2] * r[2]) / r[0] : 0.0;
    o->mean_speed = r[0] != 0.0 ? r[3] / r[0] : 0.0;
    o->zeta = r[0] != 0.0 ? p.B - r[3] / r[0] : 0.0;
    o->drho = sqrt(r[6]);
    o->nonfinite = (int64_t)r[4];
}

}  // namespace lbm
