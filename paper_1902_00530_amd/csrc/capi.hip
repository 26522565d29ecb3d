// C ABI of the library (include/lbm.h): validation, context management and
// the single-lattice entry points.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>

#include "internal.h"

namespace lbm {

static thread_local std::string g_error;

void set_error(const std::string &msg) { g_error = msg; }

int32_t fail(int32_t code, const std::string &msg)
{
    g_error = msg;
    return code;
}

int32_t hip_fail(hipError_t e, const char *what)
{
    g_error = std::string("HIP error in ") + what + ": " + hipGetErrorString(e);
    return LBM_EHIP;
}

static bool finite_nonneg(double v) { return isfinite(v) && v >= 0.0; }

int32_t validate_params(const lbm_params *p, int64_t pitch)
{
    if (!p)
        return fail(LBM_EINVAL, "null parameters");
    if (p->lattice != LBM_D2Q7 && p->lattice != LBM_D2Q9)
        return fail(LBM_EINVAL, "unknown lattice");
    if (p->nx < 2 || p->ny < 2)
        return fail(LBM_EINVAL, "nx and ny must be >= 2");
    if (p->lattice == LBM_D2Q7 && (p->ny & 1))
        return fail(LBM_EINVAL, "ny must be even (offset-row triangular lattice)");
    if (p->ny > 65535)
        return fail(LBM_EINVAL, "ny must be <= 65535 (one grid row of blocks per lattice row)");
    if ((uint64_t)p->nx * (uint64_t)p->ny >= (1ull << 32))
        return fail(LBM_EINVAL, "nx*ny must be < 2^32 (32-bit site counter of the noise)");
    if (pitch < p->nx)
        return fail(LBM_EINVAL, "pitch must be >= nx");
    if (p->model < LBM_PASSIVE || p->model > LBM_CIL)
        return fail(LBM_EINVAL, "unknown model");
    if (p->storage < LBM_F32 || p->storage > LBM_BF16_DEV_R32)
        return fail(LBM_EINVAL, "unknown storage");
    if (p->storage == LBM_BF16_DEV_R32 && p->lattice == LBM_D2Q9)
        return fail(LBM_EUNSUPPORTED, "the float32 rest plane storage takes D2Q7 lattices");
    if (!(p->tau >= 1.0))
        return fail(LBM_EINVAL, "tau must be >= 1 (or +inf for streaming only)");
    if (!finite_nonneg(p->sigma))
        return fail(LBM_EINVAL, "sigma must be finite and >= 0");
    if (!finite_nonneg(p->A) || !finite_nonneg(p->B) || !finite_nonneg(p->C) || !finite_nonneg(p->u_max))
        return fail(LBM_EINVAL, "A, B, C and u_max must be finite and >= 0");
    if (p->model == LBM_MIPS && !(isfinite(p->rho_star) && p->rho_star > 0.0))
        return fail(LBM_EINVAL, "rho_star must be finite and > 0 for MIPS");
    if (p->storage != LBM_F32 && !finite_nonneg(p->rho_ref))
        return fail(LBM_EINVAL, "rho_ref must be finite and >= 0 for deviation storage");
    if (p->lattice == LBM_D2Q9 && (uint64_t)p->ny * (uint64_t)pitch * (p->storage == LBM_F32 ? 4u : 2u) >= (1ull << 32))
        return fail(LBM_EUNSUPPORTED, "D2Q9 population planes must be below 2^32 bytes");
    return LBM_OK;
}

// w rho_ref rounded to the storage format, so that a population of exactly 0
// (what the negative correction leaves) is stored and read back exactly:
// with an unrepresentable reference every corrected zero came back a little
// negative, a mass leak that ran away in disordered states
static float storage_reference(double v, int storage)
{
    float f = (float)v;
    if (storage == LBM_BF16_DEV) {
        uint32_t b;
        memcpy(&b, &f, 4);
        b += 0x7fffu + ((b >> 16) & 1u);  // round to nearest even (finite values)
        b &= 0xffff0000u;
        memcpy(&f, &b, 4);
    } else if (storage == LBM_F16_DEV) {
        f = (float)(_Float16)f;
    }
    return f;
}

StepArgs make_step_args(const lbm_params &p, int64_t pitch)
{
    StepArgs a;
    a.nx = p.nx;
    a.ny = p.ny;
    a.pitch = pitch;
    a.plane = (int64_t)p.ny * pitch;
    a.omega = (float)(1.0 / p.tau);
    const bool q9 = p.lattice == LBM_D2Q9;
    a.noise_scale = (float)(q9 ? p.sigma / 73728.0 : p.sigma / 229376.0);
    a.noise_h = (float)(q9 ? p.sigma / 8192.0 : p.sigma / 32768.0);
    a.A16 = (float)p.A * 65536.0f;
    a.B16 = (float)p.B * 65536.0f;
    a.C2 = 2.0f * (float)p.C;
    a.rho_star = p.model == LBM_MIPS ? (float)p.rho_star : 1.0f;
    a.inv_rho_star = p.model == LBM_MIPS ? (float)(1.0 / p.rho_star) : 1.0f;
    a.u_max2 = 2.0f * (float)p.u_max;
    const double rr = p.storage == LBM_F32 ? 0.0 : p.rho_ref;
    // the float32 rest plane of LBM_BF16_DEV_R32 holds f_0 itself
    const int moving = p.storage == LBM_BF16_DEV_R32 ? LBM_BF16_DEV : p.storage;
    a.wr0 = p.storage == LBM_BF16_DEV_R32 ? 0.0f : storage_reference(q9 ? 4.0 * rr / 9.0 : 0.5 * rr, p.storage);
    a.wr1 = storage_reference(q9 ? rr / 9.0 : rr / 12.0, moving);
    a.wr2 = storage_reference(q9 ? rr / 36.0 : rr / 12.0, moving);
    a.key0 = (uint32_t)(p.seed & 0xffffffffu);
    a.key1 = (uint32_t)(p.seed >> 32);
    a.noisy = p.sigma != 0.0;
    return a;
}

__global__ void k_set_clock(StepClock *clk, int slot, int64_t t)
{
    if ((blockIdx.x | threadIdx.x) == 0)
        clk->t[slot] = t;
}

hipError_t launch_set_clock(StepClock *clk, int slot, int64_t t, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_clock, dim3(1), dim3(64), 0, s, clk, slot, t);
    return hipGetLastError();
}

// A context's workspace: the step clock, the 8 reduced doubles of a sample,
// then the reduction scratch.
constexpr size_t kWsClock = 0, kWsResult = 256, kWsScratch = 512;

static size_t ctx_workspace_bytes(const lbm_params &p)
{
    return kWsScratch + ((moments_scratch_doubles(p) * sizeof(double) + 255) & ~(size_t)255);
}

// Steps per captured graph of lbm_step (even, so a replay leaves the state in
// the buffer it started from).
constexpr int64_t kGraphSteps = 64;
// Steps of the call that first captures it.  Capturing and instantiating takes
// about 0.4 ms and a direct launch about 3 us of the host against 5 us and more
// of the GPU, so a graph only frees the host: shorter runs are launched
// directly (64^2 MIPS, the first 100 steps of a new context: 742 us with one
// launch a step and a graph, 155 us now).  Contexts that take one step per launch
// capture it in the first call that it fits: there the host is the slower one (CIL
// 64^2 with pitch 96, calls of 200 steps: 3.7 us a step launched directly, 2.5 from
// the graph).
constexpr int64_t kGraphFirst = 512;

static int64_t steps_per_launch(const lbm_ctx *c) { return c->multi.T ? c->multi.T : c->rows ? 2 : 1; }

// Where lbm_step takes two steps per launch, and on 64 x 8 or 64 x 16 tiles
// (lattices small enough for multi_for_lattice take more steps per launch).
// Two steps halve the passes over the state and the launches; they cost the
// first step's ring around each tile (a sixteenth to a quarter more site
// bodies; MIPS a fifth to a third) and a longer chain per launch.  Measured in
// us per step, one step per launch against two (64 x 8 / 64 x 16 tiles):
//   CIL F32       180x60 2.49 / 2.49 / 3.21; 256^2 3.09 / 2.61 / 3.32; 1024^2 10.5 / 7.43 / 7.49;
//                 2048^2 34.4 / 21.7 / 21.6; 4096^2 167 / 96.5 / 96.5
//   CIL BF16      256^2 2.75 / 2.83 / 3.92; 512^2 4.34 / 3.58 / 4.12; 4096^2 99 / 94 / 87
//   MIPS F32      256^2 3.48 / 3.55 / 3.63; 512^2 5.62 / 5.21 / 4.22; 4096^2 188 / 135 / 122
//   MIPS BF16     512^2 5.07 / 5.08 / 4.49; 1024^2 10.0 / 11.4 / 10.4; 2048^2 29.6 / 34.2 / 30.9
//   D2Q9 CIL F32  256^2 3.63 / 3.02 / 4.15; 1024^2 13.3 / 9.06 / 9.67; 4096^2 207 / 126 / 125
//   D2Q9 MIPS F32 64^2 5.93 / 3.87 / 3.89; 1024^2 15.3 / 13.1 / 12.0; 4096^2 251 / 171 / 159
//   D2Q9 MIPS F16 512^2 7.22 / 5.83 / 4.87; 1024^2 13.6 / 13.5 / 12.3; 2048^2 36 / 43 / 40
// Below the lines the launch is bound by one block's latency, so the shorter
// one-step chain wins; 16-bit MIPS on large lattices is VALU-bound already, so
// the ring's extra work loses.  Pitched lattices and buffers of 2^30
// populations or more (64-bit offsets) keep one step per launch.
//
// D2Q9 MIPS also has 64 x 24 tiles: their ring costs 24% more collisions in the
// first step against 33% at 16 rows, and two blocks fit a CU either way.  They
// win wherever the last round of 512 blocks is not much emptier: above 2^21
// sites (F32; 16-bit lattices take one step per launch there), and below where
// the rounds times the rows are fewer.  us per step, 16 / 24 rows: F32 512^2 5.0 /
// 5.8; 721x720 9.3 / 8.7; 1024^2 12.3 / 12.7; 1448^2 22.0 / 21.4; 2048^2 46.6 / 44.4;
// 4096^2 161 / 152; BF16 721x720 9.8 / 9.4; 1448x724 14.8 / 13.5.
//
// All that holds for lattices that fill their tiles.  A tile's first step is taken
// on all of its rows and their ring, also past the lattice's edge, where blocks of
// one step have 256 x 1 sites (local models) or rows that leave at once (MIPS); and
// tile rows go to the eight XCDs in turn, so that a lattice of few tile rows uses few
// of them.  Two steps are therefore taken only up to a ratio of the busiest XCD's
// site bodies (step2_work; a lattice that fills its tiles has 1.1 to 1.2): 1.55, for
// F32 local models 2.3, for states beyond the Infinity Cache, which two steps read
// and write half as often, 2.2 at least, for the 16-bit MIPS 1.38 where they gain
// little.  us per step, one / two: CIL F32 100000x18 19.6 / 29.0, 100000x2 7.1 / 22.3,
// 5000x66 5.8 / 4.8; CIL BF16 100000x18 14.9 / 37.1; MIPS F32 400000x6 151 / 260.  16-bit
// local lattices within that cache are bound by vector instructions from about 2^20
// sites on, where only a width that leaves the 256-site blocks half empty pays
// (0.85): CIL BF16 1448^2 13.5 / 14.5, 2896^2 41.5 / 44.8, 300x10000 25.2 / 20.6, and
// 3400^2, beyond the cache, 72.2 / 63.4.  Lattices narrower than half a tile wrap
// several times a load and keep one step: CIL F32 20x60000 16.2 / 19.1.
static double step2_work(const lbm_params &p, int rows)
{
    const bool mips = p.model == LBM_MIPS;
    auto up = [](int64_t n, int64_t d) { return (n + d - 1) / d; };
    const int64_t ntx = up(p.nx, 64), nty = up(p.ny, rows), r = up(nty, 8);  // r: tile rows of the busiest XCD
    const int ring = mips ? 2 : 1;
    const int64_t first = (64 + 2 * ring) * (rows + 2 * ring) * r, second = 64 * std::min<int64_t>(rows * r, p.ny);
    // a tile whose reads wrap around the lattice takes a fifth more
    const int64_t ix = std::max(0, (p.nx - 64 - 2 * ring) / 64), iy = std::max(0, (p.ny - rows - 2 * ring) / rows);
    const double wraps = 1.0 - (double)(ix * iy) / (double)(ntx * nty);
    const double two = 0.5 * (double)(ntx * (first + second)) * (1.0 + 0.2 * wraps);
    double one;
    if (mips) {
        const int one_rows = p.lattice == LBM_D2Q7 && ntx * up(p.ny, 16) < 512 ? 4 : 16;
        one = (double)(ntx * 64 * std::min<int64_t>(one_rows * up(up(p.ny, one_rows), 8), p.ny));
    } else {
        const int64_t bx = p.nx >= 256 ? 256 : 64 * up(p.nx, 64), by = 256 / bx;
        one = (double)(up(p.nx, bx) * bx * by * up(up(p.ny, by), 8));
    }
    return two / one;
}

int step2_rows(const lbm_params &p, const StepArgs &a)
{
    const bool q9 = p.lattice == LBM_D2Q9, f32 = p.storage == LBM_F32, mips = p.model == LBM_MIPS;
    const int64_t sites = (int64_t)p.nx * p.ny;
    if (a.pitch != p.nx || (!q9 && (uint64_t)a.plane * 7ull >= (1ull << 30)) || p.nx < 33)
        return 0;
    const uint64_t state = (uint64_t)sites * (q9 ? 9ull : 7ull) * (f32 ? 4ull : 2ull);
    const bool cached = 2ull * state <= kStreamStateBytes;
    int rows;
    double most;
    if (mips) {
        const int64_t lo = q9 ? 0 : 1 << 17, hi = f32 ? INT64_MAX : q9 ? 3 << 19 : 1 << 19;
        if (sites < lo || sites >= hi)
            return 0;
        auto rounds = [&](int ty) { return (((p.nx + 63) / 64) * (int64_t)((p.ny + ty - 1) / ty) + 511) / 512; };
        rows = q9 && (sites >= 1 << 21 || 24 * rounds(24) < 16 * rounds(16)) ? 24 : 16;
        if (p.ny < rows)
            return 0;
        most = !cached ? 2.2 : !f32 && sites >= (q9 ? 1 << 19 : 3 << 16) ? 1.38 : 1.55;
    } else if (f32) {
        if (sites < 3 << 14)
            return 0;
        rows = sites < 1 << 21 ? 8 : 16;
        most = 2.3;
    } else {
        if (sites < 1 << 17)
            return 0;
        rows = cached ? 8 : 16;
        most = !cached ? 2.2 : sites > (q9 ? 1 << 20 : 5 << 18) ? 0.85 : 1.55;
    }
    return step2_work(p, rows) <= most ? rows : 0;
}

// n steps from buffer `from`, in as few launches as the context's form allows.
// The launches alternate between the buffers and are an odd number where n is,
// so that the state ends where n one-step launches would leave it; the steps
// are dealt evenly over them (a launch of one step takes the one-step kernel).
static hipError_t enqueue_steps(lbm_ctx *c, int from, int64_t n, hipStream_t s)
{
    const bool q9 = c->p.lattice == LBM_D2Q9;
    const int64_t most = steps_per_launch(c);
    int64_t launches = (n + most - 1) / most;
    launches += (launches ^ n) & 1;
    for (int64_t k = 0; k < launches; ++k) {
        const int slot = (from + (int)(k & 1)) & 1;
        const void *src = c->buf[slot];
        void *dst = c->buf[slot ^ 1];
        const int steps = (int)(n / launches + (k < n % launches ? 1 : 0));
        hipError_t e;
        if (steps == 1)
            e = q9 ? launch_step_q9(c->p, c->args, src, dst, c->clk, slot, s)
                   : launch_step(c->p, c->args, src, dst, c->clk, slot, s);
        else if (c->multi.T)
            e = q9 ? launch_multi_q9(c->p, c->args, c->multi, steps, src, dst, c->clk, slot, s)
                   : launch_multi(c->p, c->args, c->multi, steps, src, dst, c->clk, slot, s);
        else
            e = q9 ? launch_step2_q9(c->p, c->args, c->rows, src, dst, c->clk, slot, s)
                   : launch_step2(c->p, c->args, c->rows, src, dst, c->clk, slot, s);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// kGraphSteps steps from buffer `from`, captured on a private stream (the
// caller's may be the legacy null stream, which cannot be captured).
static hipError_t capture_steps(lbm_ctx *c, int from)
{
    hipStream_t cap;
    hipError_t e = hipStreamCreateWithFlags(&cap, hipStreamNonBlocking);
    if (e != hipSuccess)
        return e;
    hipGraph_t g = nullptr;
    e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    hipError_t ce = e == hipSuccess ? enqueue_steps(c, from, kGraphSteps, cap) : e;
    hipError_t ee = e == hipSuccess ? hipStreamEndCapture(cap, &g) : e;
    (void)hipStreamDestroy(cap);
    e = ce != hipSuccess ? ce : ee;
    if (e == hipSuccess)
        e = hipGraphInstantiate(&c->graph[from], g, nullptr, nullptr, 0);
    if (g)
        (void)hipGraphDestroy(g);
    return e;
}

}  // namespace lbm

using namespace lbm;

extern "C" {

const char *lbm_last_error(void) { return g_error.c_str(); }

int32_t lbm_deviation_reference(const lbm_params *p, float *wr)
{
    int32_t rc = validate_params(p, p ? p->nx : 0);
    if (rc)
        return rc;
    if (!wr)
        return fail(LBM_EINVAL, "null output");
    const StepArgs a = make_step_args(*p, p->nx);
    const int q = p->lattice == LBM_D2Q9 ? 9 : 7;
    for (int i = 0; i < q; ++i)
        wr[i] = i == 0 ? a.wr0 : (q == 7 || i <= 4 ? a.wr1 : a.wr2);
    return LBM_OK;
}

size_t lbm_workspace_bytes(const lbm_params *p, int64_t pitch)
{
    if (validate_params(p, pitch) != LBM_OK)
        return 0;
    return ctx_workspace_bytes(*p);
}

int32_t lbm_create(const lbm_params *p, void *f_a, void *f_b, int64_t pitch, const lbm_init *init, void *ws,
                   size_t ws_bytes, void *stream, lbm_ctx **out)
{
    if (!out)
        return fail(LBM_EINVAL, "null output pointer");
    *out = nullptr;
    int32_t rc = validate_params(p, pitch);
    if (rc)
        return rc;
    if (!f_a || !f_b)
        return fail(LBM_EINVAL, "null population buffer");
    if (f_a == f_b)
        return fail(LBM_EINVAL, "f_a and f_b must be distinct buffers");
    if (!ws)
        return fail(LBM_EINVAL, "null workspace");
    if ((uintptr_t)ws % 256 != 0)
        return fail(LBM_EINVAL, "workspace must be 256-byte aligned");
    if (ws_bytes < ctx_workspace_bytes(*p))
        return fail(LBM_EINVAL, "workspace smaller than lbm_workspace_bytes()");
    if (init && (init->mode < LBM_INIT_NONE || init->mode > LBM_INIT_GAUSS_DIR))
        return fail(LBM_EINVAL, "unknown init mode");
    if (init && init->mode != LBM_INIT_NONE &&
        !(isfinite(init->rho_mean) && init->rho_mean >= 0.0 && finite_nonneg(init->rho_spread) &&
          init->rho_spread <= 1.0 && isfinite(init->angle_std) && isfinite(init->u_mag) &&
          isfinite(init->pop_noise)))
        return fail(LBM_EINVAL, "invalid init parameters");
    lbm_ctx *c = new (std::nothrow) lbm_ctx();
    if (!c)
        return fail(LBM_EINVAL, "out of host memory");
    c->p = *p;
    c->pitch = pitch;
    c->args = make_step_args(*p, pitch);
    c->stream = (hipStream_t)stream;
    c->buf[0] = f_a;
    c->buf[1] = f_b;
    c->cur = 0;
    c->step = 0;
    char *w = (char *)ws;
    c->clk = (StepClock *)(w + kWsClock);
    c->d_result = (double *)(w + kWsResult);
    c->d_scratch = (double *)(w + kWsScratch);
    c->graph[0] = c->graph[1] = nullptr;
    c->multi = multi_for_lattice(*p, c->args);
    c->rows = step2_rows(*p, c->args);
    hipError_t e = hipGetDevice(&c->device);
    if (e == hipSuccess)
        e = launch_set_clock(c->clk, 0, 0, c->stream);
    if (e == hipSuccess && init && init->mode != LBM_INIT_NONE)
        e = p->lattice == LBM_D2Q9 ? launch_init_q9(*p, *init, c->args, f_a, c->stream)
                                   : launch_init(*p, *init, c->args, f_a, c->stream);
    if (e != hipSuccess) {
        rc = hip_fail(e, "lbm_create");
        delete c;
        return rc;
    }
    *out = c;
    return LBM_OK;
}

int32_t lbm_step(lbm_ctx *c, int64_t n)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    if (n < 0)
        return fail(LBM_EINVAL, "negative step count");
    // whole graphs of kGraphSteps steps, then direct launches; a stream that
    // the caller is capturing gets direct launches only
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cs) != hipSuccess) {
        (void)hipGetLastError();
        cs = hipStreamCaptureStatusNone;
    }
    int64_t left = n;
    const int64_t first = steps_per_launch(c) > 1 ? kGraphFirst : kGraphSteps;
    if (cs == hipStreamCaptureStatusNone && n >= kGraphSteps && (c->graph[c->cur] || n >= first)) {
        if (!c->graph[c->cur])
            LBM_HIP_TRY(capture_steps(c, c->cur));
        for (; left >= kGraphSteps; left -= kGraphSteps)
            LBM_HIP_TRY(hipGraphLaunch(c->graph[c->cur], c->stream));
    }
    LBM_HIP_TRY(enqueue_steps(c, c->cur, left, c->stream));
    c->cur ^= (int)(n & 1);
    c->step += n;
    return LBM_OK;
}

int32_t lbm_moments(lbm_ctx *c, float *rho, float *ux, float *uy, lbm_obs *obs)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    auto launch = [&](double *host) {
        return launch_moments(c->p, c->args, c->buf[c->cur], rho, ux, uy, c->d_scratch, c->d_result, host, c->stream);
    };
    if (!obs) {
        LBM_HIP_TRY(launch(nullptr));
        return LBM_OK;
    }
    HostResult host(1, c->stream);
    LBM_HIP_TRY(launch(host.ptr));
    double r[8];
    LBM_HIP_TRY(host.read(c->d_result, r, 1, c->stream));
    finish_obs(c->p, r, c->step, obs);
    if (obs->nonfinite)
        return fail(LBM_ENONFINITE, "non-finite populations in the state");
    return LBM_OK;
}

int32_t lbm_current_buffer(const lbm_ctx *c)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    return c->cur;
}

int64_t lbm_get_step(const lbm_ctx *c)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    return c->step;
}

int32_t lbm_set_step(lbm_ctx *c, int64_t step)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    if (step < 0)
        return fail(LBM_EINVAL, "negative step index");
    LBM_HIP_TRY(launch_set_clock(c->clk, c->cur, step, c->stream));
    c->step = step;
    return LBM_OK;
}

int32_t lbm_add_density(lbm_ctx *c, double drho)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    if (!isfinite(drho))
        return fail(LBM_EINVAL, "drho must be finite");
    if (c->p.lattice == LBM_D2Q9)
        LBM_HIP_TRY(launch_add_density_q9(c->p, c->args, c->buf[c->cur], drho, c->stream));
    else
        LBM_HIP_TRY(launch_add_density(c->p, c->args, c->buf[c->cur], drho, c->stream));
    return LBM_OK;
}

int32_t lbm_destroy(lbm_ctx *c)
{
    if (!c)
        return fail(LBM_ESTATE, "null context");
    hipError_t e = hipStreamSynchronize(c->stream);
    for (int k = 0; k < 2; ++k)
        if (c->graph[k])
            (void)hipGraphExecDestroy(c->graph[k]);
    delete c;
    if (e != hipSuccess)
        return hip_fail(e, "lbm_destroy");
    return LBM_OK;
}

}  // extern "C"
