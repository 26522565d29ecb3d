// Two steps of the method on one tile in one pass over memory (temporal
// blocking), shared by the single-lattice kernels (twostep.hip) and the batched
// ones (batch.hip).
//
// The state of step t+1 at a site depends on the state of step t at the site
// and its neighbours (one streaming move), so the state of step t+2 on a
// 64 x TY tile needs step t+1 on the tile widened by one site on every side
// (MIPS, whose u* reads neighbour densities: by two), which needs step t
// widened by two (MIPS: four).  The first step's results stay in LDS, the
// second step's are written: one read and one write of the state per two
// updates, for about (66 (TY + 2)) / (64 TY) - 1 extra site bodies.  Every
// site runs the one-step site body on the values a store and a later load of
// the storage would give, so two steps here equal two one-step launches bit
// for bit.  Buffers have pitch nx (an element offset is the noise's site
// index).
#pragma once

#include "device_q9.h"

namespace lbm {

// A tile's population stores at element v + s of each plane: streamed past
// the caches for a lattice whose two buffers exceed the Infinity Cache budget
// (uniform per block), cached otherwise, where the next launch reads them from
// the Infinity Cache.
template <int ST>
__device__ __forceinline__ void store7(bool stream, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, uint32_t plane,
                                       const float f[7], const StepArgs &a)
{
    if (stream) {
#pragma unroll
        for (int i = 0; i < 7; ++i)
            Planes<ST>::template store<kStoreStream>(r, v, s, i, plane, f[i], a);
    } else {
#pragma unroll
        for (int i = 0; i < 7; ++i)
            Planes<ST>::store(r, v, s, i, plane, f[i], a);
    }
}

template <int S>
__device__ __forceinline__ void store9(bool stream, typename Store<S>::T *dst, uint32_t plane, uint32_t v, uint32_t s,
                                       const float f[9], const StepArgs &a)
{
    using T = typename Store<S>::T;
    if (stream) {
#pragma unroll
        for (int i = 0; i < 9; ++i)
            BufIO<T>::template store<kStoreStream>(q9_plane_rsrc(dst, i, plane), v, s, Store<S>::narrow(f[i], q9_wr(a, i)));
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i)
            BufIO<T>::store(q9_plane_rsrc(dst, i, plane), v, s, Store<S>::narrow(f[i], q9_wr(a, i)));
    }
}

// D2Q9, two steps on a 64 x TY tile (the scheme of step2_tile below on the
// square lattice).  The second step reads population i of site
// (lx, ly) from the first step's site (lx - e_ix, ly - e_iy), local
// coordinates (lx, ly) = (x - x0 + 1, y - y0 + 1): every plane keeps TY rows
// of the widened tile's 66 columns, starting one row lower (e_iy = 1: planes
// 2, 5, 6), on the tile's rows (e_iy = 0: 0, 1, 3) or one row higher
// (e_iy = -1: 4, 7, 8).  At TY = 16 that is 38,016 bytes, four blocks per CU.
template <int TY>
struct Q9MidLayout {
    static constexpr int W = 66;
    static constexpr int kSize = 9 * TY * W;
    __host__ __device__ static constexpr int row0(int i)
    {
        return (i == 2 || i == 5 || i == 6) ? 0 : (i == 4 || i == 7 || i == 8) ? 2 : 1;
    }
    __device__ static int at(int i, int lx, int ly) { return (i * TY + ly - row0(i)) * W + lx; }
    __device__ static bool kept(int i, int ly)
    {
        const int r = ly - row0(i);
        return r >= 0 && r < TY;
    }
};

// mid: ML::kSize floats of LDS; stream: stores past the caches.
template <int M, int S, int F, int TY, int NW>
__device__ __forceinline__ void q9_step2_tile(const typename Store<S>::T *src, typename Store<S>::T *dst,
                                              const StepArgs &a, int x0, int y0, uint64_t t, bool stream, float *mid)
{
    using T = typename Store<S>::T;
    using ML = Q9MidLayout<TY>;
    constexpr int W = 66, H = TY + 2;
    static_assert(NW % 2 == 0 && TY % NW == 0 && 2 * (TY + 2) <= 64 * (NW - 2), "rows per wave split evenly; edges fit");
    const uint32_t plane = (uint32_t)a.plane, nx = (uint32_t)a.nx;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform
    const uint32_t ta_lo = (uint32_t)t, ta_hi = (uint32_t)(t >> 32);
    const uint32_t tb_lo = (uint32_t)(t + 1), tb_hi = (uint32_t)((t + 1) >> 32);
    // sources two sites around the tile do not wrap: wave-uniform row bases
    const bool interior = x0 >= 2 && x0 + 66 <= a.nx && y0 >= 2 && y0 + TY + 2 <= a.ny;

    // first step on the widened tile, from HBM into LDS (wave w: rows w,
    // w+NW, ...; waves 2 and up take the two edge columns in their last slot)
    constexpr int NR = (H + NW - 1) / NW;
    float f[NR][9];
    uint32_t site[NR];
    auto load_row = [&](float *g, uint32_t &st, int ly, bool in) {
        if (in) {
            const uint32_t c = (uint32_t)(y0 - 1 + ly) * nx + (uint32_t)x0;  // offset of (x0, y)
            const uint32_t e[9] = {c, c - 1u, c - nx, c + 1u, c + nx, c - nx - 1u, c - nx + 1u, c + nx + 1u,
                                   c + nx - 1u};
#pragma unroll
            for (int i = 0; i < 9; ++i)
                g[i] = Store<S>::widen(BufIO<T>::load(q9_plane_rsrc(src, i, plane), lane, e[i]), q9_wr(a, i));
            st = c + (uint32_t)lane;
        } else {
            const Q9Sources q = q9_sources(a, wrap_coord(x0 + lane, a.nx), wrap_coord(y0 - 1 + ly, a.ny));
#pragma unroll
            for (int i = 0; i < 9; ++i)
                g[i] = Store<S>::widen(BufIO<T>::load(q9_plane_rsrc(src, i, plane), q.idx[i], 0u), q9_wr(a, i));
            st = q.idx[0];  // pitch nx: own offset = site index
        }
    };
    auto compute = [&](float *g, uint32_t st, int lx, int ly) {
        float rho, jx, jy, ux, uy;
        q9_moments(g, rho, jx, jy);
        local_ustar<M>(a, rho, jx, jy, ux, uy);
        q9_collide<F, S>(a, g, rho, ux, uy, st, ta_lo, ta_hi);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (ML::kept(i, ly))
                mid[ML::at(i, lx, ly)] = Store<S>::round(g[i], q9_wr(a, i));  // as a store and a load give it
    };
    if (interior) {
#pragma unroll
        for (int k = 0; k < NR - 1; ++k)
            load_row(f[k], site[k], wv + NW * k, true);
    } else {
#pragma unroll
        for (int k = 0; k < NR - 1; ++k)
            load_row(f[k], site[k], wv + NW * k, false);
    }
    const int e = (wv - 2) * 64 + lane;
    const bool edge = wv >= 2;
    const int elx = edge ? (e < H ? 0 : W - 1) : lane + 1;
    const int ely = edge ? (e < H ? e : e - H) : wv + NW * (NR - 1);
    bool elive = true;
    if (!edge) {
        load_row(f[NR - 1], site[NR - 1], ely, interior);
    } else {
        elive = e < 2 * H;
        if (elive) {
            const Q9Sources q = q9_sources(a, wrap_coord(x0 - 1 + elx, a.nx), wrap_coord(y0 - 1 + ely, a.ny));
#pragma unroll
            for (int i = 0; i < 9; ++i)
                f[NR - 1][i] = Store<S>::widen(BufIO<T>::load(q9_plane_rsrc(src, i, plane), q.idx[i], 0u), q9_wr(a, i));
            site[NR - 1] = q.idx[0];
        }
    }
#pragma unroll
    for (int k = 0; k < NR - 1; ++k)
        compute(f[k], site[k], lane + 1, wv + NW * k);
    if (elive)
        compute(f[NR - 1], site[NR - 1], elx, ely);
    __syncthreads();

    // second step on the tile, from LDS into HBM
    auto second = [&](int r) {
        const int lx = lane + 1, ly = r + 1;
        float g[9];
        g[0] = mid[ML::at(0, lx, ly)];
        g[1] = mid[ML::at(1, lx - 1, ly)];
        g[2] = mid[ML::at(2, lx, ly - 1)];
        g[3] = mid[ML::at(3, lx + 1, ly)];
        g[4] = mid[ML::at(4, lx, ly + 1)];
        g[5] = mid[ML::at(5, lx - 1, ly - 1)];
        g[6] = mid[ML::at(6, lx + 1, ly - 1)];
        g[7] = mid[ML::at(7, lx + 1, ly + 1)];
        g[8] = mid[ML::at(8, lx - 1, ly + 1)];
        float rho, jx, jy, ux, uy;
        q9_moments(g, rho, jx, jy);
        local_ustar<M>(a, rho, jx, jy, ux, uy);
        const uint32_t row = (uint32_t)(y0 + r) * nx + (uint32_t)x0;  // pitch nx
        q9_collide<F, S>(a, g, rho, ux, uy, row + (uint32_t)lane, tb_lo, tb_hi);
        store9<S>(stream, dst, plane, (uint32_t)lane, row, g, a);
    };
    if (interior) {
        for (int r = wv; r < TY; r += NW)
            second(r);
    } else {
        for (int r = wv; r < TY; r += NW)
            if (x0 + lane < a.nx && y0 + r < a.ny)
                second(r);
    }
}

// Step t+1 on the widened tile as the second step reads it, in local
// coordinates (lx, ly) = (x - x0 + 1, y - y0 + 1): population 0 only at the
// tile's own sites (TY rows of 64), 1 and 4 on the tile's rows (ly 1..TY),
// 2 and 3 one row lower (ly 0..TY-1), 5 and 6 one row higher (ly 2..TY+1),
// each TY rows of 66.  At TY = 16 that is 29,440 bytes, so five blocks fit
// in a CU's 160 KB of LDS (all seven planes of all TY+2 rows would not).
template <int TY>
struct MidLayout {
    static constexpr int W = 66;
    static constexpr int kSize = TY * 64 + 6 * TY * W;
    // plane base and first row of plane i
    static constexpr int base(int i)
    {
        return i == 0 ? 0 : TY * 64 + (i == 1 ? 0 : i == 4 ? 1 : i == 2 ? 2 : i == 3 ? 3 : i == 5 ? 4 : 5) * TY * W;
    }
    static constexpr int row0(int i) { return i == 0 || i == 1 || i == 4 ? 1 : (i == 2 || i == 3 ? 0 : 2); }
    __device__ static int at(int i, int lx, int ly)
    {
        return i == 0 ? (ly - 1) * 64 + (lx - 1) : base(i) + (ly - row0(i)) * W + lx;
    }
    // whether the second step reads population i of local site (lx, ly)
    __device__ static bool kept(int i, int lx, int ly)
    {
        const int r = ly - row0(i);
        return r >= 0 && r < TY && (i != 0 || (lx >= 1 && lx <= 64));
    }
};

// Steps t and t+1 on a 64 x TY tile (NW waves: wave w owns rows w, w+NW,
// ...); the first step's results go to LDS in the MidLayout above.
// mid: ML::kSize floats of LDS; stream: stores past the caches.
template <int M, int ST, int F, int TY, int NW>
__device__ __forceinline__ void step2_tile(const void *srcp, void *dstp, const StepArgs &a, int x0, int y0, uint64_t t,
                                           bool stream, float *mid)
{
    using ML = MidLayout<TY>;
    constexpr int W = 66, H = TY + 2;
    static_assert(NW % 2 == 0 && TY % NW == 0 && 2 * (TY + 2) <= 64 * (NW - 2), "rows per wave split evenly; edges fit");
    const uint32_t plane = (uint32_t)a.plane;
    const __amdgpu_buffer_rsrc_t src = buffer_rsrc(srcp, (uint32_t)Planes<ST>::bytes(plane));
    const __amdgpu_buffer_rsrc_t dst = buffer_rsrc(dstp, (uint32_t)Planes<ST>::bytes(plane));
    auto ld = [&](uint32_t elem, uint32_t first, int i) { return Planes<ST>::load(src, elem, first, i, plane, a); };
    const uint32_t nx = (uint32_t)a.nx;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform
    const uint32_t ta_lo = (uint32_t)t, ta_hi = (uint32_t)(t >> 32);
    const uint32_t tb_lo = (uint32_t)(t + 1), tb_hi = (uint32_t)((t + 1) >> 32);
    // A tile whose sources (two sites around it) do not wrap: every offset is
    // a wave-uniform row base plus the lane.
    const bool interior = x0 >= 2 && x0 + 66 <= a.nx && y0 >= 2 && y0 + TY + 2 <= a.ny;

    // First step on the widened tile, from HBM into LDS.  Wave w takes rows
    // w, w+NW, ... of the H rows; waves 2 and up own one row fewer (H = 2 mod
    // NW) and take the two edge columns (2H sites) in that slot instead.  All
    // of a wave's loads are issued before any of its sites is computed.
    constexpr int NR = (H + NW - 1) / NW;
    float f[NR][7];
    uint32_t site[NR];
    auto load_row = [&](float *g, uint32_t &st, int ly, bool in) {
        if (in) {
            const int yg = y0 - 1 + ly;
            const uint32_t p = (uint32_t)yg & 1u;
            const uint32_t c = (uint32_t)yg * nx + (uint32_t)x0;  // offset of (x0, yg)
            g[0] = ld(lane, c, 0);
            g[1] = ld(lane, c - 1u, 1);
            g[2] = ld(lane, c - nx - 1u + p, 2);
            g[3] = ld(lane, c - nx + p, 3);
            g[4] = ld(lane, c + 1u, 4);
            g[5] = ld(lane, c + nx + p, 5);
            g[6] = ld(lane, c + nx - 1u + p, 6);
            st = c + (uint32_t)lane;
        } else {
            const int xg = wrap_coord(x0 + lane, a.nx), yg = wrap_coord(y0 - 1 + ly, a.ny);
            const PullSources32 q = pull_sources32(a, xg, yg);
#pragma unroll
            for (int i = 0; i < 7; ++i)
                g[i] = ld(q.idx[i], 0u, i);
            st = q.idx[0];  // pitch nx: own offset = site index
        }
    };
    auto compute = [&](float *g, uint32_t st, int lx, int ly) {
        float rho, jx, jy, ux, uy;
        site_moments(g, rho, jx, jy);
        local_ustar<M>(a, rho, jx, jy, ux, uy);
        site_collide<F, ST>(a, g, rho, ux, uy, st, ta_lo, ta_hi);
#pragma unroll
        for (int i = 0; i < 7; ++i)
            if (ML::kept(i, lx, ly))  // the value a store and the next step's load would give
                mid[ML::at(i, lx, ly)] = Planes<ST>::round(g[i], i, a);
    };
    // slots 0 .. NR-2: rows of every wave
    if (interior) {
#pragma unroll
        for (int k = 0; k < NR - 1; ++k)
            load_row(f[k], site[k], wv + NW * k, true);
    } else {
#pragma unroll
        for (int k = 0; k < NR - 1; ++k)
            load_row(f[k], site[k], wv + NW * k, false);
    }
    // slot NR-1: last row of waves 0 and 1, edge sites of waves 2 and up
    const int e = (wv - 2) * 64 + lane;
    const bool edge = wv >= 2;
    const int elx = edge ? (e < H ? 0 : W - 1) : lane + 1;
    const int ely = edge ? (e < H ? e : e - H) : wv + NW * (NR - 1);
    bool elive = true;
    if (!edge) {
        load_row(f[NR - 1], site[NR - 1], ely, interior);
    } else {
        elive = e < 2 * H;
        if (elive) {
            const int xg = wrap_coord(x0 - 1 + elx, a.nx), yg = wrap_coord(y0 - 1 + ely, a.ny);
            const PullSources32 q = pull_sources32(a, xg, yg);
#pragma unroll
            for (int i = 0; i < 7; ++i)
                f[NR - 1][i] = ld(q.idx[i], 0u, i);
            site[NR - 1] = q.idx[0];
        }
    }
#pragma unroll
    for (int k = 0; k < NR - 1; ++k)
        compute(f[k], site[k], lane + 1, wv + NW * k);
    if (elive)
        compute(f[NR - 1], site[NR - 1], elx, ely);
    __syncthreads();

    // second step on the tile, from LDS into HBM; y0 is even, so row r has
    // parity r & 1 = wv & 1
    const int p = wv & 1;
    auto second = [&](int r) {
        const int lx = lane + 1, ly = r + 1;
        float f[7];
        f[0] = mid[ML::at(0, lx, ly)];
        f[1] = mid[ML::at(1, lx - 1, ly)];
        f[2] = mid[ML::at(2, lx - 1 + p, ly - 1)];
        f[3] = mid[ML::at(3, lx + p, ly - 1)];
        f[4] = mid[ML::at(4, lx + 1, ly)];
        f[5] = mid[ML::at(5, lx + p, ly + 1)];
        f[6] = mid[ML::at(6, lx - 1 + p, ly + 1)];
        float rho, jx, jy, ux, uy;
        site_moments(f, rho, jx, jy);
        local_ustar<M>(a, rho, jx, jy, ux, uy);
        const uint32_t row = (uint32_t)(y0 + r) * nx + (uint32_t)x0;  // pitch nx
        site_collide<F, ST>(a, f, rho, ux, uy, row + (uint32_t)lane, tb_lo, tb_hi);
        store7<ST>(stream, dst, (uint32_t)lane, row, plane, f, a);
    };
    if (interior) {
        for (int r = wv; r < TY; r += NW)
            second(r);
    } else {
        for (int r = wv; r < TY; r += NW)
            if (x0 + lane < a.nx && y0 + r < a.ny)
                second(r);
    }
}

// ---------------------------------------------------------------------------
// MIPS, steps t and t+1 on a 64 x TY tile, on either lattice.  u* at a site
// needs the streamed density of its neighbours (eq. bu_mips with the
// isotropic stencil: six on the triangular lattice, eight on the square), so
// the second step on the tile reads the first step's populations on a ring of
// two sites around it (region B) and its densities on a ring of one (C), and
// the first step on B reads densities on a ring of three (A), which gather
// from the stored state on a ring of four.  Four phases, a barrier after each
// of the first three:
//  1. every site of A: its streamed populations from HBM and their density
//     into LDS; B's sites come first and keep their populations in
//     registers, the ring A \ B follows in one more slot, so the collisions
//     of phase 2 fill whole waves;
//  2. every site of B: u* from the densities, collision of step t, the
//     populations into LDS as a store and a later load give them back;
//  3. every site of C: the streamed density of step t+1 from LDS;
//  4. every site of the tile: its streamed populations from LDS, u* from the
//     densities of phase 3, collision of step t+1, store.
// Ring sites are computed at their periodic images with the one-step site
// body, so every site gets the values two one-step launches give it, bit for
// bit.  On the triangular lattice row parity follows the global row (y0 and
// ny are even).
// ---------------------------------------------------------------------------
template <int TY>
struct Mips2Layout {
    static constexpr int WA = 70, HA = TY + 6;  // A: x0-3 .. x0+66, y0-3 .. y0+TY+2
    static constexpr int WB = 68, HB = TY + 4;  // B: x0-2 .. x0+65, y0-2 .. y0+TY+1
    static constexpr int WC = 66, HC = TY + 2;  // C: x0-1 .. x0+64, y0-1 .. y0+TY
    static constexpr int NA = WA * HA, NB = WB * HB, NC = WC * HC;
    static constexpr int kRing = NA - NB;           // A outside B: 2 WA + 2 (HA - 2) sites
    static constexpr int kRho = NA > NC ? NA : NC;  // densities on A (phases 1-2), then on C (3-4)
    // A-local position of ring site e (0 <= e < kRing): the row above B, the
    // row below, then the left and the right column between them
    __device__ static void ring(int e, int &ax, int &ay)
    {
        if (e < WA) {
            ax = e;
            ay = 0;
        } else if (e < 2 * WA) {
            ax = e - WA;
            ay = HA - 1;
        } else {
            const int c = e - 2 * WA;
            ax = c < HA - 2 ? 0 : WA - 1;
            ay = 1 + (c < HA - 2 ? c : c - (HA - 2));
        }
    }
};

// Lattice policies of the two-step MIPS kernel: the streamed populations of a
// global site from the stored state (sources inside the lattice, or at the
// periodic images of a wrapped site), the density, u* from the densities
// around position c of an LDS map of row width W, the collision, the value a
// store and a later load give back, the streamed populations of a site of
// the step-t map (nb sites per plane, row width wb), and the store.
template <int ST>
struct Mips2Q7 {  // offset-row triangular lattice, any storage
    static constexpr int Q = 7;
    const StepArgs &a;
    const __amdgpu_buffer_rsrc_t src, dst;
    const uint32_t plane, nx;
    __device__ Mips2Q7(const StepArgs &a_, const void *s, void *d)
        : a(a_), src(buffer_rsrc(s, (uint32_t)Planes<ST>::bytes(a_.plane))),
          dst(buffer_rsrc(d, (uint32_t)Planes<ST>::bytes(a_.plane))), plane((uint32_t)a_.plane), nx((uint32_t)a_.nx)
    {
    }
    __device__ float ld(uint32_t e, int i) const { return Planes<ST>::load(src, e, 0u, i, plane, a); }
    __device__ void gather_in(float *g, uint32_t &own, int x, int y) const
    {
        const uint32_t p = (uint32_t)y & 1u;
        const uint32_t c = (uint32_t)y * nx + (uint32_t)x;
        g[0] = ld(c, 0);
        g[1] = ld(c - 1u, 1);
        g[2] = ld(c - nx - 1u + p, 2);
        g[3] = ld(c - nx + p, 3);
        g[4] = ld(c + 1u, 4);
        g[5] = ld(c + nx + p, 5);
        g[6] = ld(c + nx - 1u + p, 6);
        own = c;
    }
    __device__ void gather_wrapped(float *g, uint32_t &own, int xg, int yg) const
    {
        const PullSources32 q = pull_sources32(a, xg, yg);
#pragma unroll
        for (int i = 0; i < 7; ++i)
            g[i] = ld(q.idx[i], i);
        own = q.idx[0];
    }
    __device__ static float density(const float *g) { return g[0] + ((g[1] + g[4]) + ((g[2] + g[5]) + (g[3] + g[6]))); }
    template <int W>
    __device__ void ustar(const float *rs, int c, int p, float rho, float &ux, float &uy) const
    {
        float nb[7];
        nb[0] = rho;
        nb[1] = rs[c + 1];
        nb[2] = rs[c + W + p];
        nb[3] = rs[c + W - 1 + p];
        nb[4] = rs[c - 1];
        nb[5] = rs[c - W - 1 + p];
        nb[6] = rs[c - W + p];
        mips_ustar(a, rho, nb, ux, uy);
    }
    template <int F>
    __device__ void collide(float *f, float rho, float ux, float uy, uint32_t site, uint32_t lo, uint32_t hi) const
    {
        site_collide<F, ST>(a, f, rho, ux, uy, site, lo, hi);
    }
    __device__ float round(float v, int i) const { return Planes<ST>::round(v, i, a); }
    template <int NB, int WB>
    __device__ static void pull_mid(float *g, const float *mid, int bx, int by, int p)
    {
        const int m = by * WB + bx;
        g[0] = mid[0 * NB + m];
        g[1] = mid[1 * NB + m - 1];
        g[2] = mid[2 * NB + m - WB - 1 + p];
        g[3] = mid[3 * NB + m - WB + p];
        g[4] = mid[4 * NB + m + 1];
        g[5] = mid[5 * NB + m + WB + p];
        g[6] = mid[6 * NB + m + WB - 1 + p];
    }
    __device__ void store(bool stream, uint32_t row, int lane, const float *g) const
    {
        store7<ST>(stream, dst, (uint32_t)lane, row, plane, g, a);
    }
};

template <int ST>
struct Mips2Q9 {  // square lattice, one 16- or 32-bit type per buffer; one buffer resource per plane
    using T = typename Store<ST>::T;
    static constexpr int Q = 9;
    const StepArgs &a;
    const T *const srcp;
    T *const dstp;
    const uint32_t plane, nx;
    __device__ Mips2Q9(const StepArgs &a_, const void *s, void *d)
        : a(a_), srcp((const T *)s), dstp((T *)d), plane((uint32_t)a_.plane), nx((uint32_t)a_.nx)
    {
    }
    __device__ float ld(uint32_t e, int i) const
    {
        return Store<ST>::widen(BufIO<T>::load(q9_plane_rsrc(srcp, i, plane), e, 0u), q9_wr(a, i));
    }
    __device__ void gather_in(float *g, uint32_t &own, int x, int y) const
    {
        const uint32_t c = (uint32_t)y * nx + (uint32_t)x;
        const uint32_t e[9] = {c, c - 1u, c - nx, c + 1u, c + nx, c - nx - 1u, c - nx + 1u, c + nx + 1u, c + nx - 1u};
#pragma unroll
        for (int i = 0; i < 9; ++i)
            g[i] = ld(e[i], i);
        own = c;
    }
    __device__ void gather_wrapped(float *g, uint32_t &own, int xg, int yg) const
    {
        const Q9Sources q = q9_sources(a, xg, yg);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            g[i] = ld(q.idx[i], i);
        own = q.idx[0];
    }
    __device__ static float density(const float *g)
    {
        return g[0] + (((g[1] + g[3]) + (g[2] + g[4])) + ((g[5] + g[7]) + (g[6] + g[8])));
    }
    template <int W>
    __device__ void ustar(const float *rs, int c, int, float rho, float &ux, float &uy) const
    {
        float nb[9];
        nb[0] = rho;
        nb[1] = rs[c + 1];
        nb[2] = rs[c + W];
        nb[3] = rs[c - 1];
        nb[4] = rs[c - W];
        nb[5] = rs[c + W + 1];
        nb[6] = rs[c + W - 1];
        nb[7] = rs[c - W - 1];
        nb[8] = rs[c - W + 1];
        q9_mips_ustar(a, rho, nb, ux, uy);
    }
    template <int F>
    __device__ void collide(float *f, float rho, float ux, float uy, uint32_t site, uint32_t lo, uint32_t hi) const
    {
        q9_collide<F, ST>(a, f, rho, ux, uy, site, lo, hi);
    }
    __device__ float round(float v, int i) const { return Store<ST>::round(v, q9_wr(a, i)); }
    template <int NB, int WB>
    __device__ static void pull_mid(float *g, const float *mid, int bx, int by, int)
    {
        const int m = by * WB + bx;
        g[0] = mid[0 * NB + m];
        g[1] = mid[1 * NB + m - 1];
        g[2] = mid[2 * NB + m - WB];
        g[3] = mid[3 * NB + m + 1];
        g[4] = mid[4 * NB + m + WB];
        g[5] = mid[5 * NB + m - WB - 1];
        g[6] = mid[6 * NB + m - WB + 1];
        g[7] = mid[7 * NB + m + WB + 1];
        g[8] = mid[8 * NB + m + WB - 1];
    }
    __device__ void store(bool stream, uint32_t row, int lane, const float *g) const
    {
        store9<ST>(stream, dstp, plane, (uint32_t)lane, row, g, a);
    }
};

// floats of LDS of step2_mips_tile
template <class LP, int TY>
constexpr int mips2_lds() { return LP::Q * Mips2Layout<TY>::NB + Mips2Layout<TY>::kRho; }

template <class LP, int F, int TY, int NW>
__device__ __forceinline__ void step2_mips_tile(const void *srcp, void *dstp, const StepArgs &a, int x0, int y0,
                                                uint64_t t, bool stream, float *lds)
{
    using ML = Mips2Layout<TY>;
    constexpr int Q = LP::Q, NT = 64 * NW;
    constexpr int KB = (ML::NB + NT - 1) / NT, KR = (ML::kRing + NT - 1) / NT, KC = (ML::NC + NT - 1) / NT;
    static_assert(TY % NW == 0 && TY % 2 == 0, "rows per wave split evenly; tile rows start even");
    float *const mid = lds;               // [Q][HB][WB]
    float *const rs = lds + Q * ML::NB;  // [HA][WA], then [HC][WC]
    const LP lp(a, srcp, dstp);
    const uint32_t nx = (uint32_t)a.nx;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const uint32_t ta_lo = (uint32_t)t, ta_hi = (uint32_t)(t >> 32);
    const uint32_t tb_lo = (uint32_t)(t + 1), tb_hi = (uint32_t)((t + 1) >> 32);
    // sources four sites around the tile inside the lattice: no wrap at all
    const bool interior = x0 >= 4 && x0 + 68 <= a.nx && y0 >= 4 && y0 + TY + 4 <= a.ny;
    // A's coordinates lie in [-3, n + 65] (x) and [-3, n + TY + 1] (y): one
    // period brings them into the lattice unless it is that small
    const bool once = a.nx >= 66 && a.ny >= TY + 2;
    auto wrap = [&](int c, int n) {
        if (once) {
            c = c < 0 ? c + n : c;
            return c >= n ? c - n : c;
        }
        c %= n;
        return c < 0 ? c + n : c;
    };
    // the Q streamed populations of global site (x, y), unwrapped
    // coordinates; `own` its offset (pitch nx: the site index of the noise)
    auto gather = [&](float *g, uint32_t &own, int x, int y) {
        if (interior)
            lp.gather_in(g, own, x, y);
        else
            lp.gather_wrapped(g, own, wrap(x, a.nx), wrap(y, a.ny));
    };

    // phase 1: every load of the block's sites of A is issued first
    float f[KB][Q], fr[KR][Q];
    uint32_t own[KB], ownr[KR];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        const int s = tid + k * NT;
        if ((k + 1) * NT <= ML::NB || s < ML::NB)
            gather(f[k], own[k], x0 - 2 + s % ML::WB, y0 - 2 + s / ML::WB);
    }
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const int e = tid + k * NT;
        if (e < ML::kRing) {
            int ax, ay;
            ML::ring(e, ax, ay);
            gather(fr[k], ownr[k], x0 - 3 + ax, y0 - 3 + ay);
        }
    }
    float rho[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        const int s = tid + k * NT;
        if ((k + 1) * NT <= ML::NB || s < ML::NB) {
            rho[k] = LP::density(f[k]);
            rs[(s / ML::WB + 1) * ML::WA + s % ML::WB + 1] = rho[k];
        }
    }
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const int e = tid + k * NT;
        if (e < ML::kRing) {
            int ax, ay;
            ML::ring(e, ax, ay);
            rs[ay * ML::WA + ax] = LP::density(fr[k]);
        }
    }
    __syncthreads();

    // phase 2: step t on B (row by has parity by & 1: y0 is even)
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        const int s = tid + k * NT;
        if ((k + 1) * NT <= ML::NB || s < ML::NB) {
            const int by = s / ML::WB, ax = s % ML::WB + 1, ay = by + 1;
            float ux, uy;
            lp.template ustar<ML::WA>(rs, ay * ML::WA + ax, by & 1, rho[k], ux, uy);
            lp.template collide<F>(f[k], rho[k], ux, uy, own[k], ta_lo, ta_hi);
#pragma unroll
            for (int i = 0; i < Q; ++i)
                mid[i * ML::NB + s] = lp.round(f[k][i], i);
        }
    }
    __syncthreads();

    // phase 3: densities of step t+1 on C (row cy has parity (cy + 1) & 1)
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int s = tid + k * NT;
        if ((k + 1) * NT <= ML::NC || s < ML::NC) {
            const int cx = s % ML::WC, cy = s / ML::WC;
            float g[Q];
            LP::template pull_mid<ML::NB, ML::WB>(g, mid, cx + 1, cy + 1, (cy + 1) & 1);
            rs[s] = LP::density(g);
        }
    }
    __syncthreads();

    // phase 4: step t+1 on the tile; wave w takes rows w, w + NW, ...
    for (int r = wv; r < TY; r += NW) {
        const int x = x0 + lane, y = y0 + r;
        if (!interior && (x >= a.nx || y >= a.ny))
            continue;
        float g[Q];
        LP::template pull_mid<ML::NB, ML::WB>(g, mid, lane + 2, r + 2, r & 1);
        const float rh = LP::density(g);
        float ux, uy;
        lp.template ustar<ML::WC>(rs, (r + 1) * ML::WC + lane + 1, r & 1, rh, ux, uy);
        const uint32_t row = (uint32_t)y * nx + (uint32_t)x0;  // pitch nx
        lp.template collide<F>(g, rh, ux, uy, row + (uint32_t)lane, tb_lo, tb_hi);
        lp.store(stream, row, lane, g);
    }
}

}  // namespace lbm
