// Several steps of the method on a small tile in one launch, for lattices and
// batches too small to fill the GPU, where a launch costs more than the steps
// it carries.
//
// A block takes the tx x ty sites of its tile and a ring of R T sites around
// it (R = 1; MIPS, whose u* reads neighbour densities, 2) into LDS, once and
// in whole rows, and advances that region T steps in place, its live box
// shrinking by R sites a side per step, until the tile itself is left and is
// written out.  No block waits on another: ring sites are computed again by
// every block that needs them, at their periodic images and with the one-step
// site body on the values a store and a later load of the storage would give,
// so T steps here equal T one-step launches bit for bit.  Buffers have pitch
// nx (an element offset is the noise's site index).
#pragma once

#include "device_q9.h"
#include "internal.h"

namespace lbm {

// Sites of a region (planes of so many floats in LDS: 29 to 42 KB a block) and
// lanes of a block: MIPS, whose steps are the longer chain, one site a lane
// (4 to 9% faster than two on 512 lanes), the local models 512 (the same time,
// and more blocks fit a CU).
constexpr int kMultiSites = 1024;
__host__ __device__ constexpr int multi_lanes(int model) { return model == kMips ? 1024 : 512; }

// Lattice policies: load / store of population i at element e, the value a
// store and a later load give back, and the streamed populations, density and
// target velocity of a region site from LDS (planes of PS floats, row width w).
template <int ST>
struct MultiQ7 {
    static constexpr int Q = 7;
    const StepArgs &a;
    const __amdgpu_buffer_rsrc_t src, dst;
    const uint32_t plane;
    __device__ MultiQ7(const StepArgs &a_, const void *s, void *d)
        : a(a_), src(buffer_rsrc(s, (uint32_t)Planes<ST>::bytes(a_.plane))),
          dst(buffer_rsrc(d, (uint32_t)Planes<ST>::bytes(a_.plane))), plane((uint32_t)a_.plane)
    {
    }
    __device__ float load(uint32_t e, int i) const { return Planes<ST>::load(src, e, 0u, i, plane, a); }
    __device__ void store(uint32_t e, int i, float v) const { Planes<ST>::store(dst, e, 0u, i, plane, v, a); }
    __device__ float round(float v, int i) const { return Planes<ST>::round(v, i, a); }
    template <int PS>
    __device__ static void pull(float *g, const float *st, int c, int w, int p)
    {
        const int u = c + w - 1 + p, d = c - w - 1 + p;  // rows above and below, the left of the two neighbours
        g[0] = st[c];
        g[1] = st[1 * PS + c - 1];
        g[2] = st[2 * PS + d];
        g[3] = st[3 * PS + d + 1];
        g[4] = st[4 * PS + c + 1];
        g[5] = st[5 * PS + u + 1];
        g[6] = st[6 * PS + u];
    }
    __device__ static void moments(const float *g, float &rho, float &jx, float &jy) { site_moments(g, rho, jx, jy); }
    __device__ void ustar(const float *rs, int c, int w, int p, float rho, float &vx, float &vy) const
    {
        const int u = c + w - 1 + p, d = c - w - 1 + p;
        const float nb[7] = {rho, rs[c + 1], rs[u + 1], rs[u], rs[c - 1], rs[d], rs[d + 1]};
        mips_ustar(a, rho, nb, vx, vy);
    }
    __device__ void noise(uint32_t site, uint32_t lo, uint32_t hi, float *nz) const { site_noise(a, site, lo, hi, nz); }
    template <int F>
    __device__ void relax(float *f, float rho, float vx, float vy, const float *nz) const
    {
        site_relax<F, ST>(a, f, rho, vx, vy, nz);
    }
};

template <int ST>
struct MultiQ9 {
    static constexpr int Q = 9;
    using T = typename Store<ST>::T;
    const StepArgs &a;
    const T *const srcp;
    T *const dstp;
    const uint32_t plane;
    __device__ MultiQ9(const StepArgs &a_, const void *s, void *d)
        : a(a_), srcp((const T *)s), dstp((T *)d), plane((uint32_t)a_.plane)
    {
    }
    __device__ float load(uint32_t e, int i) const
    {
        return Store<ST>::widen(BufIO<T>::load(q9_plane_rsrc(srcp, i, plane), e, 0u), q9_wr(a, i));
    }
    __device__ void store(uint32_t e, int i, float v) const
    {
        BufIO<T>::store(q9_plane_rsrc(dstp, i, plane), e, 0u, Store<ST>::narrow(v, q9_wr(a, i)));
    }
    __device__ float round(float v, int i) const { return Store<ST>::round(v, q9_wr(a, i)); }
    template <int PS>
    __device__ static void pull(float *g, const float *st, int c, int w, int)
    {
        const int u = c + w, d = c - w;
        g[0] = st[c];
        g[1] = st[1 * PS + c - 1];
        g[2] = st[2 * PS + d];
        g[3] = st[3 * PS + c + 1];
        g[4] = st[4 * PS + u];
        g[5] = st[5 * PS + d - 1];
        g[6] = st[6 * PS + d + 1];
        g[7] = st[7 * PS + u + 1];
        g[8] = st[8 * PS + u - 1];
    }
    __device__ static void moments(const float *g, float &rho, float &jx, float &jy) { q9_moments(g, rho, jx, jy); }
    __device__ void ustar(const float *rs, int c, int w, int, float rho, float &vx, float &vy) const
    {
        const int u = c + w, d = c - w;
        const float nb[9] = {rho, rs[c + 1], rs[u], rs[c - 1], rs[d], rs[u + 1], rs[u - 1], rs[d - 1], rs[d + 1]};
        q9_mips_ustar(a, rho, nb, vx, vy);
    }
    __device__ void noise(uint32_t site, uint32_t lo, uint32_t hi, float *nz) const { q9_noise(a, site, lo, hi, nz); }
    template <int F>
    __device__ void relax(float *f, float rho, float vx, float vy, const float *nz) const
    {
        q9_relax<F, ST>(a, f, rho, vx, vy, nz);
    }
};

// LDS floats of multi_tile: the planes, the densities (MIPS) and the periodic
// column and row offsets of the region (w, h <= 128).
template <class LP, int M>
constexpr int multi_lds() { return (LP::Q + (M == kMips ? 1 : 0)) * kMultiSites + 256; }

// The tile at (x0, y0), inside the lattice; g.w g.h <= kMultiSites.
template <class LP, int M, int F>
__device__ __forceinline__ void multi_tile(const void *srcp, void *dstp, const StepArgs &a, const MultiGeom &g, int x0,
                                           int y0, uint64_t t, float *lds)
{
    constexpr int Q = LP::Q, R = M == kMips ? 2 : 1;
    constexpr int PS = kMultiSites, NT = multi_lanes(M), K = PS / NT;  // K sites a lane, at most
    float *const st = lds;
    float *const rs = lds + Q * PS;
    int *const xw = (int *)(lds + (Q + (M == kMips ? 1 : 0)) * PS);  // wrapped column of region column x
    int *const yw = xw + 128;                                        // wrapped row of region row y, times nx
    const LP lp(a, srcp, dstp);
    const int tid = threadIdx.x, w = g.w, h = g.h, ring = R * g.T;
    // region coordinates lie in [-ring, n - 1 + tile + ring): one period brings
    // them into the lattice unless it is that small
    const bool once = a.nx >= g.tx + ring && a.ny >= g.ty + ring;
    auto wrap = [&](int c, int n) {
        if (once) {
            c = c < 0 ? c + n : c;
            return c >= n ? c - n : c;
        }
        c %= n;
        return c < 0 ? c + n : c;
    };
    if (tid < w)
        xw[tid] = wrap(x0 - ring + tid, a.nx);
    if (tid >= NT - h)  // the block's last threads, so that both tables are written at once
        yw[tid - (NT - h)] = wrap(y0 - ring + tid - (NT - h), a.ny) * a.nx;

    // the region's stored populations, every load issued before the first use
    float nz[K][Q];
    {
        float f[K][Q];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int s = tid + j * NT;
            if (s < w * h) {
                const int y = (int)(((uint32_t)s * g.mag[0]) >> 22), x = s - y * w;
                const uint32_t e = (uint32_t)(wrap(y0 - ring + y, a.ny) * a.nx + wrap(x0 - ring + x, a.nx));
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    f[j][i] = lp.load(e, i);
            }
        }
        if (F & kNoisy) {
            // meanwhile the first step's noise, which needs no population: twelve
            // 90 x 30 MIPS lattices 2.25 -> 2.14 us a step, fifty 180 x 60 CIL
            // lattices 5.56 -> 5.34
            const int bw = w - 2 * R, n = bw * (h - 2 * R);
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const int s = tid + j * NT;
                if (s < n) {
                    const int y = (int)(((uint32_t)s * g.mag[1]) >> 22), x = s - y * bw;
                    lp.noise((uint32_t)(wrap(y0 - ring + R + y, a.ny) * a.nx + wrap(x0 - ring + R + x, a.nx)),
                             (uint32_t)t, (uint32_t)(t >> 32), nz[j]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int s = tid + j * NT;
            if (s < w * h) {
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    st[i * PS + s] = f[j][i];
            }
        }
    }
    __syncthreads();

    uint32_t mag = g.mag[1];
    for (int k = 1; k <= g.T; ++k) {
        const int m = R * k, bw = w - 2 * m, bh = h - 2 * m, n = bw * bh;
        const uint32_t mag_next = g.mag[k < g.T ? k + 1 : k];  // read a step ahead
        const uint64_t tt = t + (uint64_t)(k - 1);
        const uint32_t lo = (uint32_t)tt, hi = (uint32_t)(tt >> 32);
        float f[K][Q], rho[K], jx[K], jy[K];
        int c[K], x[K], y[K];
        uint32_t site[K];
        // every site of the box: its streamed populations into registers
        // (MIPS: its density into LDS); the noise, which needs no population,
        // is drawn while they arrive
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int s = tid + j * NT;
            if (s < n) {
                y[j] = (int)(((uint32_t)s * mag) >> 22);
                x[j] = s - y[j] * bw;
                c[j] = (y[j] + m) * w + x[j] + m;
                site[j] = (uint32_t)(yw[y[j] + m] + xw[x[j] + m]);
                LP::template pull<PS>(f[j], st, c[j], w, (y0 - ring + y[j] + m) & 1);
                if ((F & kNoisy) && k > 1)
                    lp.noise(site[j], lo, hi, nz[j]);
                LP::moments(f[j], rho[j], jx[j], jy[j]);
                if (M == kMips)
                    rs[c[j]] = rho[j];
            }
        }
        if (M == kMips) {  // and the densities of the ring around it
            for (int e = NT - 1 - tid; e < 2 * (bw + 2) + 2 * bh; e += NT) {
                int rx, ry;  // relative to the box's corner
                if (e < 2 * (bw + 2)) {
                    const bool top = e >= bw + 2;
                    rx = (top ? e - (bw + 2) : e) - 1;
                    ry = top ? bh : -1;
                } else {
                    const int q = e - 2 * (bw + 2);
                    const bool right = q >= bh;
                    rx = right ? bw : -1;
                    ry = right ? q - bh : q;
                }
                const int rc = (ry + m) * w + rx + m;
                float g1[Q], r1, j1, j2;
                LP::template pull<PS>(g1, st, rc, w, (y0 - ring + ry + m) & 1);
                LP::moments(g1, r1, j1, j2);
                rs[rc] = r1;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int s = tid + j * NT;
            if (s < n) {
                float vx, vy;
                if constexpr (M == kMips)
                    lp.ustar(rs, c[j], w, (y0 - ring + y[j] + m) & 1, rho[j], vx, vy);
                else
                    local_ustar<M>(a, rho[j], jx[j], jy[j], vx, vy);
                lp.template relax<F>(f[j], rho[j], vx, vy, nz[j]);
                if (k < g.T) {
#pragma unroll
                    for (int i = 0; i < Q; ++i)
                        st[i * PS + c[j]] = lp.round(f[j][i], i);
                } else if (x0 + x[j] < a.nx && y0 + y[j] < a.ny) {
#pragma unroll
                    for (int i = 0; i < Q; ++i)
                        lp.store(site[j], i, f[j][i]);
                }
            }
        }
        mag = mag_next;
        if (k < g.T)
            __syncthreads();
    }
}

}  // namespace lbm
