// Host-side internals of the library: the context object and the kernel
// launchers that the C ABI layer calls.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <type_traits>

#include "../../include/lbm.h"
#include "../../include/lbm_cnn.h"
#include "device.h"

namespace lbm {

void set_error(const std::string &msg);
int32_t fail(int32_t code, const std::string &msg);
int32_t hip_fail(hipError_t e, const char *what);

#define LBM_HIP_TRY(expr)                                      \
    do {                                                       \
        hipError_t e_ = (expr);                                \
        if (e_ != hipSuccess) return ::lbm::hip_fail(e_, #expr); \
    } while (0)

// Fill the kernel argument block from validated parameters.
StepArgs make_step_args(const lbm_params &p, int64_t pitch);
// Parameter validation shared by lbm_create and lbm_sweep_batch.
int32_t validate_params(const lbm_params *p, int64_t pitch);

// Compile-time variant of the site body for these arguments (kUnitTau, kNoisy).
int step_flags(const StepArgs &a);
// One fused step src -> dst; the step index comes from clock slot `slot`
// and the next index goes to the other slot.
hipError_t launch_step(const lbm_params &p, const StepArgs &a, const void *src, void *dst, StepClock *clk, int slot,
                       hipStream_t s);
// Tile rows (local models 8, 16; MIPS 16, on D2Q9 also 24) of the two-step kernels
// for this lattice, 0 where one step per launch is taken.
int step2_rows(const lbm_params &p, const StepArgs &a);
// Two steps src -> dst in one launch on 64 x rows tiles; the clock advances by
// two.
hipError_t launch_step2(const lbm_params &p, const StepArgs &a, int rows, const void *src, void *dst, StepClock *clk,
                        int slot, hipStream_t s);
hipError_t launch_step2_q9(const lbm_params &p, const StepArgs &a, int rows, const void *src, void *dst, StepClock *clk,
                           int slot, hipStream_t s);
// Grid of ntx x nty tiles in row groups (row_group_tile).
inline dim3 row_group_grid(int ntx, int nty) { return dim3(8u * (unsigned)ntx, (unsigned)((nty + 7) / 8)); }
// Several steps per launch on small tiles (multi.h).  Geometry of one launch: T
// steps on tx x ty tiles; the region a block holds is w x h = (tx + 2 R T) x
// (ty + 2 R T), R = 1 (MIPS 2); mag[k] divides by the width of the box after k
// steps, s / width = (s mag) >> 22 for s < 4096.
constexpr int kMultiMaxT = 8;
struct MultiGeom {
    int32_t T, tx, ty, w, h;
    uint32_t mag[kMultiMaxT + 1];
};
MultiGeom multi_geom(int model, int T, int tx, int ty);
// The geometry for lattices of these sizes launched together: T steps per
// launch (0: none) and its estimated time per step.
struct MultiChoice {
    int T = 0, tx = 0, ty = 0;
    double us = 0.0;
};
struct MultiSize {
    int nx, ny, count;  // count lattices of nx x ny sites
};
// (at most kMultiMaxTiles tiles in all)
constexpr int kMultiMaxTiles = 16 * 256;
MultiChoice multi_choose(int model, const MultiSize *sizes, int n);
// The same for one lattice of lbm_step, T = 0 where another form is faster.
MultiChoice multi_for_lattice(const lbm_params &p, const StepArgs &a);
hipError_t launch_multi(const lbm_params &p, const StepArgs &a, const MultiChoice &c, int steps, const void *src, void *dst,
                        StepClock *clk, int slot, hipStream_t s);
hipError_t launch_multi_q9(const lbm_params &p, const StepArgs &a, const MultiChoice &c, int steps, const void *src,
                           void *dst, StepClock *clk, int slot, hipStream_t s);
// Initial state into dst.
hipError_t launch_init(const lbm_params &p, const lbm_init &in, const StepArgs &a, void *dst, hipStream_t s);
// f_i += drho / 7 in place.
hipError_t launch_add_density(const lbm_params &p, const StepArgs &a, void *buf, double drho, hipStream_t s);
// The same three on the square (D2Q9) lattice (f_i += drho / 9).
hipError_t launch_step_q9(const lbm_params &p, const StepArgs &a, const void *src, void *dst, StepClock *clk,
                          int slot, hipStream_t s);
// Set clock slot `slot` to step index t (enqueued; a kernel, so it may be
// captured into a graph).
hipError_t launch_set_clock(StepClock *clk, int slot, int64_t t, hipStream_t s);
hipError_t launch_init_q9(const lbm_params &p, const lbm_init &in, const StepArgs &a, void *dst, hipStream_t s);
hipError_t launch_add_density_q9(const lbm_params &p, const StepArgs &a, void *buf, double drho, hipStream_t s);

// Moments and FP64 reductions.  scratch: device doubles of
// moments_scratch_doubles(p); result: 8 device doubles
// {M, Jx, Jy, sum |j|, nonfinite, mean_x rho_y, var_x rho_y, unused}, also
// written to host (HostResult::ptr) where it is not null.
size_t moments_scratch_doubles(const lbm_params &p);
hipError_t launch_moments(const lbm_params &p, const StepArgs &a, const void *src, float *rho, float *ux,
                          float *uy, double *scratch, double *result, double *host, hipStream_t s);
// Pinned host memory for `results` results of eight doubles, for one call on
// stream s (ptr null where there is none left, or s is being captured).
struct HostResult {
    double *ptr = nullptr;
    int slot = 0, count = 0;
    HostResult(size_t results, hipStream_t s);
    ~HostResult();
    HostResult(const HostResult &) = delete;
    HostResult &operator=(const HostResult &) = delete;
    // r[8 results] once the stream's work is done: from ptr, to which a kernel
    // has written them, or copied from device memory
    hipError_t read(const double *result, double *r, size_t results, hipStream_t s);
    // the same for results in device memory only
    hipError_t fetch(const double *result, double *r, size_t results, hipStream_t s);
};
// The network's tensors (w1, b1, w2, b2, w3, b3) for an Adam step.
constexpr int kAdamMax = 6;
struct AdamJobs {
    float *theta[kAdamMax], *m[kAdamMax], *v[kAdamMax];
    const float *g[kAdamMax];
    int64_t count[kAdamMax];
    uint16_t *bf16[kAdamMax];  // bf16 copies of theta, or null
};
struct AdamStep {
    float lr, beta1, beta2, eps, bc1, bc2;
};
// Physical fields y [n][cin][h][w] from x (norm: scale, shift, inverse scale
// and inverse shift, cin floats each; at most four channels).
hipError_t cnn_predict(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, const float *norm, float *y,
                       hipStream_t st);
// One Adam step (as lbm_cnn_adam) on samples idx of x and target (idx null:
// the first n).  xn [n][cin][hw], a1, a2 [n][hidden][hw]: scratch; ws:
// lbm_cnn_workspace_bytes.
hipError_t cnn_train(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, const float *target,
                     const int32_t *idx, const float *norm, float *xn, float *a1, float *a2, void *ws,
                     const AdamJobs &adam, float lr, float beta1, float beta2, float eps, int64_t t, float *loss,
                     hipStream_t st);

// The surrogate form of lbm_sweep_batch (opts->surrogate set; arguments
// validated as for a plain sweep).
int32_t surrogate_sweep(const lbm_params *ps, int n, const lbm_sweep_opts *o, void *const *bufs, void *ws,
                        size_t ws_bytes, hipStream_t st, lbm_obs *out);
// Turn the 8 reduced doubles into an lbm_obs (host).
void finish_obs(const lbm_params &p, const double *r, int64_t step, lbm_obs *o);

// Runtime storage and flags to compile-time template arguments.
template <int V>
using IntTag = std::integral_constant<int, V>;

template <class Fn>
inline hipError_t with_storage(int storage, Fn &&fn)
{
    switch (storage) {
    case kF32: return fn(IntTag<kF32>{});
    case kBf16Dev: return fn(IntTag<kBf16Dev>{});
    case kF16Dev: return fn(IntTag<kF16Dev>{});
    case kBf16R32: return fn(IntTag<kBf16R32>{});
    }
    return hipErrorInvalidValue;
}

template <class Fn>
inline hipError_t with_flags(int flags, Fn &&fn)
{
    switch (flags) {
    case 0: return fn(IntTag<0>{});
    case kUnitTau: return fn(IntTag<kUnitTau>{});
    case kNoisy: return fn(IntTag<kNoisy>{});
    default: return fn(IntTag<kUnitTau | kNoisy>{});
    }
}

}  // namespace lbm

struct lbm_ctx {
    lbm_params p;
    lbm::StepArgs args;
    int device;
    hipStream_t stream;
    void *buf[2];
    int cur;
    int64_t pitch;
    int64_t step;
    // in the caller's workspace
    lbm::StepClock *clk;  // device step index (two slots)
    double *d_result;     // 8 doubles
    double *d_scratch;    // reductions
    // graphs of kGraphSteps steps starting from buffer 0 and from buffer 1,
    // captured on first use
    hipGraphExec_t graph[2];
    // how steps are grouped into launches (enqueue_steps)
    lbm::MultiChoice multi;  // several steps per launch on small tiles (T = 0: not)
    int rows;                // else two steps per launch on 64 x rows tiles (0: one)
};
