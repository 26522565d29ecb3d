// Surrogate network kernels: a three-layer convolutional net (3x3 kernels,
// circular padding, ReLU, residual on the predicted fields) that advances the
// coarse density and momentum fields of a lattice by k steps, its training
// (mean-squared error, backward pass, Adam) and the maps between populations
// and coarse fields.  Not part of the paper; it is judged by the lattice
// Boltzmann step itself.
//
// Layout: activations NCHW float32; weights stored as bfloat16 (the Adam
// step keeps float32 master copies), so every product is a bf16 x f32 -> f32
// product with float32 accumulation.  Convolutions (bf16 operands: the
// weights, and each activation split into three bf16 parts) and weight
// gradients (FP32 operands) are matrix products on the matrix cores over
// 16 x 8 pixel tiles staged in LDS with their halo.  Reductions (weight
// gradients, loss) use fixed partitions and orders, so results are
// deterministic.
//
// A pass is a few launches: the forward pass one (k_cnn_forward, with the
// normalisation before it and the loss, or the return to physical fields,
// after it), the gradients one (k_cnn_backward), their sums, the loss and Adam
// one (k_cnn_reduce).  The fields
// are small (tens of pixels a side), so a pass of one kernel per layer was
// bound by launches, staging and gaps: 64 samples of 32 x 32 took 36.1 us to
// predict (6 launches; now 15.2 us, 1 launch) and 132.4 us to train on (18
// launches; now 66.7 us, 3 launches).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "../../include/lbm_cnn.h"
#include "internal.h"

namespace lbm {

// ---------------------------------------------------------------------------
// 3x3 convolutions on the matrix cores, bf16 operands with float32
// accumulation (v_mfma_f32_32x32x16_bf16).  The weights are bf16 values
// already; each float32 activation x is split into three bf16 parts, x = h +
// m + l + r with |r| < 2^-24 |x| (h: x with its low 16 bits cleared, m and l
// the same of the exact remainders), and the product of each part with the
// weight is exact, so the three products together give the float32 product
// and only the order of the float32 sums differs from the definition.
//
// A block owns a 16 x 8 pixel tile of one sample.  A layer's output on the
// tile widened by R pixels (16 + 2 R by 8 + 2 R, circular) comes from its input
// on the tile widened by R + 1: consecutive layers run in one block, each on a
// region one pixel narrower than the last, halo pixels computed again by every
// block that needs them (at their periodic images, with the same sums, so
// every block gets the same values), and hidden activations pass through LDS.
//
// Convolution as a matrix product per slab of 32 pixels: D[o][pixel] = sum_k
// A[o][k] B[k][pixel], k = tap * CP + c (tap = 3 ky + kx, c < CP = ci rounded up
// to 16 with zero channels), A the weights, B the input at the pixel shifted
// by the tap, channel-last in LDS.  The input gradient of a convolution with
// weights w[c][o][tap] is the convolution with wt[o][tap][c] = w[c][o][8 - tap].
//
// MFMA 32x32x16 operand layout (per lane l of the wave): A row l mod 32 with
// k = 8 (l / 32) + j, j < 8; B column l mod 32, the same k; result register r
// holds row 8 (r / 4) + 4 (l / 32) + r mod 4 of column l mod 32: a lane has
// one pixel and, per four registers, four consecutive channels, which go to
// LDS in one 8-byte write per part and to memory in rows of 16 pixels.
// ---------------------------------------------------------------------------
constexpr int kTW = 16, kTH = 8;                   // pixel tile
constexpr int kHW_ = kTW + 2, kHH = kTH + 2;       // with a one-pixel halo
constexpr int kHalo = kHW_ * kHH;                  // 180 pixels
constexpr int kMaxC = 32;                          // channels
constexpr int kCnnWaves = 8;                       // waves of a forward / input-gradient block

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// the tile widened by R pixels
template <int R>
struct Region {
    static constexpr int W = kTW + 2 * R, H = kTH + 2 * R, N = W * H;
    static constexpr int kSlabs = 4 + (N - kTW * kTH + 31) / 32;
    // Pixel (ry, rx) of the region that column m of slab s takes: slabs 0..3
    // the tile itself, two image rows of 16 each, the others the ring around
    // it; false past the ring's end (the pixel is then a valid one all the
    // same).
    __device__ static bool pixel(int s, int m, int &ry, int &rx)
    {
        if (R == 0 || s < 4) {
            ry = R + 2 * s + (m >> 4);
            rx = R + (m & 15);
            return true;
        }
        int e = (s - 4) * 32 + m;
        const bool live = e < N - kTW * kTH;
        e = live ? e : 0;
        if (e < 2 * R * W) {  // the rows above and below
            const int row = e / W;
            ry = row < R ? row : H - 2 * R + row;
            rx = e - row * W;
        } else {  // the columns left and right
            constexpr int R2 = R ? 2 * R : 1;
            e -= 2 * R * W;
            const int row = e / R2, c = e - row * R2;
            ry = R + row;
            rx = c < R ? c : W - 2 * R + c;
        }
        return live;
    }
};

// v >= -3 wrapped into [0, n); SMALL: n may be smaller than the widened tile,
// so v may wrap more than once
template <bool SMALL>
__device__ __forceinline__ int wrap_index(int v, int n)
{
    if (SMALL)
        return (v + 3 * n) % n;
    return v < 0 ? v + n : (v >= n ? v - n : v);
}

__device__ __forceinline__ int wrap_index(bool small, int v, int n)
{
    return small ? wrap_index<true>(v, n) : wrap_index<false>(v, n);
}

// the three bf16 parts of x (bit patterns): x = h + m + l + r, |r| < 2^-24 |x|
__device__ __forceinline__ void split3(float x, uint16_t &h, uint16_t &m, uint16_t &l)
{
    const uint32_t hb = __float_as_uint(x) & 0xffff0000u;
    const float r1 = x - __uint_as_float(hb);  // exact: the low 16 bits of x
    const uint32_t mb = __float_as_uint(r1) & 0xffff0000u;
    const float r2 = r1 - __uint_as_float(mb);  // exact
    h = (uint16_t)(hb >> 16);
    m = (uint16_t)(mb >> 16);
    l = (uint16_t)(__float_as_uint(r2) >> 16);
}

// four values split into s (element index e, a multiple of 4) of three parts
// `parts` elements apart
__device__ __forceinline__ void put_split4(uint16_t *s, int e, int parts, const float v[4])
{
    uint16_t h[4], m[4], l[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        split3(v[u], h[u], m[u], l[u]);
    auto pack = [](const uint16_t *q) {
        return make_uint2((uint32_t)q[0] | (uint32_t)q[1] << 16, (uint32_t)q[2] | (uint32_t)q[3] << 16);
    };
    *(uint2 *)(s + e) = pack(h);
    *(uint2 *)(s + parts + e) = pack(m);
    *(uint2 *)(s + 2 * parts + e) = pack(l);
}

__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// LDS layouts.  Inputs: [part][pixel][channel], pixels of CS elements;
// weights: [out][tap][channel], taps of TS elements, rows of WS.  Padded so
// that eight consecutive lanes' 16-byte reads fall in distinct banks (32
// channels: also the 2-byte writes of consecutive taps).  CP = 4: at most
// four channels, held without the zero ones, which lanes 32..63 (and the
// upper half of the others) take as zeros.
template <int CP>
struct ConvLds {
    static constexpr int CS = CP == 4 ? 4 : CP + 8;
    static constexpr int TS = CP == 4 ? 4 : CP == 16 ? 24 : 40;
    static constexpr int WS = 9 * TS + (CP == 4 ? 4 : 8);
};
// The first layer's: with 17 to 32 channels no padding of pixels and taps, so
// that every layer's tiles fit a CU's LDS together.
template <int CP>
struct FirstLds : ConvLds<CP> {};
template <>
struct FirstLds<32> {
    static constexpr int CS = 32, TS = 32, WS = 9 * TS + 8;
};

// One slab: x the LDS input of `parts` elements per part, p the pixel at the
// lane's top-left tap, RW the input region's width; w the lane's weight row.
// A tap's operands are read while the previous tap multiplies: left to the
// compiler, each read was waited on right before its product, and a wave alone
// on its SIMD took 69 cycles a product instead of the 35 it issues in.
template <int CP, int CS, int TS, int RW>
__device__ __forceinline__ f32x16 conv_slab(const uint16_t *x, int parts, int p, const uint16_t *w, int hk)
{
    constexpr int NC = CP <= 16 ? 1 : CP / 16;  // 16-channel steps of a tap
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        acc[r] = 0.0f;
    const uint16_t *px = x + p * CS + (CP == 4 ? 0 : 8 * hk), *pw = w + (CP == 4 ? 0 : 8 * hk);
    using Raw = std::conditional_t<CP == 4, uint2, uint4>;
    Raw fa[2][NC], fb[2][NC][3];
    auto read = [&](int t) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            fa[t & 1][c] = *(const Raw *)(pw + t * TS + 16 * c);
#pragma unroll
            for (int part = 0; part < 3; ++part)
                fb[t & 1][c][part] = *(const Raw *)(px + part * parts + ((t / 3) * RW + t % 3) * CS + 16 * c);
        }
    };
    auto operand = [&](const Raw &v) -> bf16x8 {
        if constexpr (CP == 4)
            return __builtin_bit_cast(bf16x8, make_uint4(hk ? 0u : v.x, hk ? 0u : v.y, 0u, 0u));
        else
            return __builtin_bit_cast(bf16x8, v);
    };
    read(0);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        if (t < 8)
            read(t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int part = 0; part < 3; ++part)
                acc = mfma_bf16(operand(fa[t & 1][c]), operand(fb[t & 1][c][part]), acc);
    }
    return acc;
}

// bf16 weights [rows][9] of `rows` 3x3 kernels (9 rows a multiple of 8), loaded
// eight to a thread (16 bytes where the pointer allows it), then handed to
// put(row, tap, value).  Split in two, so that a block's loads are all in
// flight before its first LDS write.
template <int NT, int ROWS>
struct WeightStage {
    static constexpr int U = (ROWS * 9 / 8 + NT - 1) / NT;
    uint4 v[U];
    __device__ __forceinline__ void load(const uint16_t *__restrict__ w, int rows)
    {
        const int last = rows * 9 / 8 - 1;
        const bool wide = ((uintptr_t)w & 15) == 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = min((int)threadIdx.x + u * NT, last);
            if (wide) {
                v[u] = ((const uint4 *)w)[q];
            } else {
                uint32_t d[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    d[k] = (uint32_t)w[8 * q + 2 * k] | (uint32_t)w[8 * q + 2 * k + 1] << 16;
                v[u] = make_uint4(d[0], d[1], d[2], d[3]);
            }
        }
    }
    template <class Put>
    __device__ __forceinline__ void store(int rows, Put put) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = threadIdx.x + u * NT;
            if (q >= rows * 9 / 8)
                continue;
            const uint32_t d[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            int row = 8 * q / 9, t = 8 * q - 9 * row;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                put(row, t, (uint16_t)(d[k >> 1] >> 16 * (k & 1)));
                if (++t == 9) {
                    t = 0;
                    ++row;
                }
            }
        }
    }
};

__device__ __forceinline__ double cwave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_down(v, off, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Forward pass.  kCnnRaw: x as it is; a1, a2 and y out.  kCnnPredict: x
// normalised on the way in, y the physical fields (channels past the third
// copied from x), nothing else written.  kCnnTrain: samples idx[n], x and the
// target normalised; a1, a2, the normalised x (the weight gradient's input),
// dy = 2 (y - t) / count and each block's float64 sum of (y - t)^2 out.
//
// One block per tile, all three layers: LDS holds the input on 22 x 14 pixels
// (at most four channels: 7 KB), a1 on 20 x 12 and a2 on 18 x 10 (58 and 43
// KB) and the weights (28 KB), so one block of eight waves fits a CU.  The halo
// costs 1.4 times the products, which are a few us in all; what the separate
// layers cost was staging, launches and the normalisation's passes.  A block
// takes every 256th tile, its weights staged once and the next tile's input
// loaded during the last layer.  What bounds it: per tile about 16,000 cycles of
// three phases between barriers with two waves a SIMD, of which the products
// are 6,000; 17 us for 512 tiles against 45 us of kernels before.
// ---------------------------------------------------------------------------
enum CnnMode : int { kCnnRaw = 0, kCnnPredict = 1, kCnnTrain = 2 };

struct CnnForward {
    const float *x;        // [.][cin][H][W]
    const int32_t *idx;    // sample numbers, or null (0, 1, ...)
    const float *norm;     // scale, shift, inverse scale, inverse shift: cin floats each
    const uint16_t *w[3];  // as stored: [out][in][tap]
    const float *b[3];
    float *a1, *a2, *y, *xn, *dy;
    const float *target;  // [.][cin][H][W]
    double *loss;         // one partial per tile
    float dscale;
    int cin, H, W, tiles;
};

template <int CP, int MODE>
__global__ __launch_bounds__(64 * kCnnWaves) void k_cnn_forward(CnnForward q)
{
    constexpr int NT = 64 * kCnnWaves;
    using R3 = Region<3>;
    using R2 = Region<2>;
    using R1 = Region<1>;
    using L1 = FirstLds<CP>;
    using L2 = ConvLds<32>;
    constexpr int XP = R3::N * L1::CS;                            // input: elements per part
    constexpr int CS = L2::CS, P1 = R2::N * CS, P2 = R1::N * CS;  // hidden activations
    __shared__ __attribute__((aligned(16))) uint16_t s_a1[3 * P1];
    __shared__ __attribute__((aligned(16))) uint16_t s_xa[3 * (XP > P2 ? XP : P2)];  // input, then a2
    __shared__ __attribute__((aligned(16))) uint16_t s_w1[32 * L1::WS];
    __shared__ __attribute__((aligned(16))) uint16_t s_w2[32 * L2::WS];
    __shared__ __attribute__((aligned(16))) uint16_t s_w3[4 * L2::WS];  // three outputs and a zero row
    __shared__ float s_b[68];
    __shared__ double s_red[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 31, hk = lane >> 5;
    const int H = q.H, W = q.W, cin = q.cin;
    const size_t HW = (size_t)H * W;
    const int tiles_j = (W + kTW - 1) / kTW, per = tiles_j * ((H + kTH - 1) / kTH);
    constexpr bool kNorm = MODE != kCnnRaw;
    // a thread takes one pixel of the widened tile and every channel: one wrap,
    // loads of consecutive pixels
    static_assert(R3::N <= NT, "a thread per pixel");
    const int xy = tid / R3::W, xx = tid - xy * R3::W;
    const bool small = H < R3::H || W < R3::W;
    int n, i0, j0;     // this tile: sample, origin
    const float *xs;   // its input
    size_t x_at = 0;   // the thread's pixel of its input
    float xv[CP];
    auto load_input = [&](int tile) {
        n = tile / per;
        const int r = tile - n * per, ti = r / tiles_j;
        i0 = ti * kTH;
        j0 = (r - ti * tiles_j) * kTW;
        xs = q.x + (size_t)(q.idx ? q.idx[n] : n) * cin * HW;
        if (tid < R3::N) {
            x_at = (size_t)wrap_index(small, i0 + xy - 3, H) * W + wrap_index(small, j0 + xx - 3, W);
#pragma unroll
            for (int c = 0; c < CP; ++c)
                xv[c] = xs[(size_t)min(c, cin - 1) * HW + x_at];
        }
    };
    auto store_input = [&]() {
        if (tid >= R3::N)
            return;
        const bool own = xy >= 3 && xy < 3 + kTH && xx >= 3 && xx < 3 + kTW && i0 + xy - 3 < H && j0 + xx - 3 < W;
#pragma unroll
        for (int c0 = 0; c0 < CP; c0 += 4) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = min(c0 + u, cin - 1);
                v[u] = kNorm ? fmaf(xv[c0 + u], q.norm[c], q.norm[cin + c]) : xv[c0 + u];
                if (MODE == kCnnTrain && own && c0 + u < cin)
                    q.xn[((size_t)n * cin + c) * HW + x_at] = v[u];
                v[u] = c0 + u < cin ? v[u] : 0.0f;
            }
            put_split4(s_xa, tid * L1::CS + c0, XP, v);
        }
    };
    load_input(blockIdx.x);
    {
        WeightStage<NT, 32 * CP> w1;
        WeightStage<NT, 32 * 32> w2;
        WeightStage<NT, 3 * 32> w3;
        w1.load(q.w[0], 32 * cin);
        w2.load(q.w[1], 32 * 32);
        w3.load(q.w[2], 3 * 32);
        if (CP != 4 || cin < 4) {  // channels past cin
            for (int e = tid; e < 32 * L1::WS; e += NT)
                s_w1[e] = 0;
            __syncthreads();
        }
        for (int e = tid; e < L2::WS; e += NT)
            s_w3[3 * L2::WS + e] = 0;
        if (tid < 67)
            s_b[tid] = tid < 32 ? q.b[0][tid] : tid < 64 ? q.b[1][tid - 32] : q.b[2][tid - 64];
        w1.store(32 * cin, [&](int row, int t, uint16_t v) {
            const int o = row / cin, c = row - o * cin;
            s_w1[o * L1::WS + t * L1::TS + c] = v;
        });
        w2.store(32 * 32, [&](int row, int t, uint16_t v) { s_w2[(row >> 5) * L2::WS + t * L2::TS + (row & 31)] = v; });
        w3.store(3 * 32, [&](int row, int t, uint16_t v) { s_w3[(row >> 5) * L2::WS + t * L2::TS + (row & 31)] = v; });
    }
    store_input();

    // layers 1 and 2: v = relu(acc + b) on region R, into LDS and (the tile's
    // own pixels) memory
    auto hidden = [&](const f32x16 &acc, const float *b, bool live, int s, int pix, uint16_t *lds, int parts,
                      float *out) {
        const int gi = i0 + 2 * s + (m >> 4), gj = j0 + (m & 15);
        float *o = MODE != kCnnPredict && s < 4 && gi < H && gj < W
                       ? out + (size_t)n * 32 * HW + (size_t)gi * W + gj
                       : nullptr;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int ch = 8 * g + 4 * hk;
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v[u] = fmaxf(acc[4 * g + u] + b[ch + u], 0.0f);
            if (live)
                put_split4(lds, pix * CS + ch, parts, v);
            if (o)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    o[(size_t)(ch + u) * HW] = v[u];
        }
    };
    for (int tile = blockIdx.x;;) {
        __syncthreads();
        for (int s = wv; s < R2::kSlabs; s += kCnnWaves) {
            int ry, rx;
            const bool live = R2::pixel(s, m, ry, rx);
            const f32x16 acc =
                conv_slab<CP, L1::CS, L1::TS, R3::W>(s_xa, XP, ry * R3::W + rx, s_w1 + m * L1::WS, hk);
            hidden(acc, s_b, live, s, ry * R2::W + rx, s_a1, P1, q.a1);
        }
        __syncthreads();
        for (int s = wv; s < R1::kSlabs; s += kCnnWaves) {
            int ry, rx;
            const bool live = R1::pixel(s, m, ry, rx);
            const f32x16 acc =
                conv_slab<32, CS, L2::TS, R2::W>(s_a1, P1, ry * R2::W + rx, s_w2 + m * L2::WS, hk);
            hidden(acc, s_b + 32, live, s, ry * R1::W + rx, s_xa, P2, q.a2);
        }
        // layer 3's residual and target, and the next tile's input, arrive
        // while the block waits and multiplies
        const int gi = i0 + 2 * wv + (m >> 4), gj = j0 + (m & 15);
        const bool mine = wv < 4 && hk == 0 && gi < H && gj < W;
        const size_t at = mine ? (size_t)gi * W + gj : 0;
        const int n_this = n, block_this = tile;
        const float *xs_this = xs;
        float xr[CP == 4 ? 4 : 3], tr[3];
        if (wv < 4) {
#pragma unroll
            for (int o = 0; o < (CP == 4 ? 4 : 3); ++o)
                xr[o] = xs_this[(size_t)min(o, cin - 1) * HW + at];
            if (MODE == kCnnTrain)
#pragma unroll
                for (int o = 0; o < 3; ++o)
                    tr[o] = q.target[((size_t)(q.idx ? q.idx[n] : n) * cin + o) * HW + at];
        }
        tile += gridDim.x;
        const bool more = tile < q.tiles;
        if (more)
            load_input(tile);
        __syncthreads();
        double sum = 0.0;
        if (wv < 4) {
            int ry, rx;
            Region<0>::pixel(wv, m, ry, rx);
            const f32x16 acc =
                conv_slab<32, CS, L2::TS, R1::W>(s_xa, P2, ry * R1::W + rx, s_w3 + min(m, 3) * L2::WS, hk);
            if (mine) {
#pragma unroll
                for (int o = 0; o < 3; ++o) {
                    float v = acc[o] + s_b[64 + o];
                    v += kNorm ? fmaf(xr[o], q.norm[o], q.norm[cin + o]) : xr[o];
                    if (MODE == kCnnRaw) {
                        q.y[((size_t)n_this * 3 + o) * HW + at] = v;
                    } else if (MODE == kCnnPredict) {
                        q.y[((size_t)n_this * cin + o) * HW + at] = fmaf(v, q.norm[2 * cin + o], q.norm[3 * cin + o]);
                    } else {
                        const float d = v - fmaf(tr[o], q.norm[o], q.norm[cin + o]);
                        q.dy[((size_t)n_this * 3 + o) * HW + at] = d * q.dscale;
                        sum += (double)d * (double)d;
                    }
                }
                if (MODE == kCnnPredict && cin > 3)
                    q.y[((size_t)n_this * cin + 3) * HW + at] = xr[3];
            }
        }
        if (MODE == kCnnTrain) {
            sum = cwave_sum(sum);
            if (lane == 0 && wv < 4)
                s_red[wv] = sum;
        }
        if (MODE == kCnnTrain || more)
            __syncthreads();
        if (MODE == kCnnTrain && tid == 0)
            q.loss[block_this] = ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];
        if (!more)
            break;
        store_input();
    }
}

// ---------------------------------------------------------------------------
// Backward pass of one tile: the input gradients dz2 = (a2 > 0) conv(dy, w3
// flipped) and dz1 = (a1 > 0) conv(dz2, w2 flipped), and the tile's partial sums
// of the three layers' weight and bias gradients, dw[o,c,tap] = sum_{n,i,j}
// dz[n,o,i,j] x[n,c,i+ky-1,j+kx-1], db[o] = sum dz[n,o,i,j] (dz: dz1, dz2, dy;
// x: the layer's input).  The partials of tile t go to part[k] + t (co ci 9 +
// co); k_cnn_reduce adds the tiles in order in float64.
//
// Weight gradients are matrix products on the matrix cores: D[o][k] = sum_p
// A[o][p] B[p][k], p the tile's 128 pixels, k = c * 9 + tap.  With 32 rows
// v_mfma_f32_16x16x4_f32, groups of four neighbouring pixels (lane group q =
// l / 16 takes pixel 4 s + q of step s): a wave takes 16 columns k at a time for
// both row blocks, so the A operands stay in registers over its columns and
// each B operand read from LDS feeds two products.
// 16x16x4 operand layout (lane l): A row l mod 16, k = l / 16; B column
// l mod 16, k = l / 16; result register r holds row 4 (l / 16) + r of
// column l mod 16.
//
// One block of eight waves a CU (134 KB of LDS), taking every 256th tile; each
// phase's input tile is loaded during the phase before.  Per tile the products
// take 15,000 cycles of a SIMD's matrix core (most of them FP32, 32 cycles each),
// the phases together 34,000, and the first loads and weights 16,000 a block: 42
// us for 512 tiles.  dz1 and dz2 never leave the CU: as kernels of their own,
// input and weight gradients waited 6 to 10 us for their first loads and moved
// 34 MB more, 15 and 34 us.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

// dz rows of kDS floats: lanes (l mod 16, l / 16) read 64 distinct banks
constexpr int kDS = kTW * kTH + 4;

// The 16 columns from 16 cb of row blocks rb0 .. rb0 + NRB - 1 (16 rows each).
template <int NRB>
__device__ __forceinline__ void wgrad_columns(const float *s_x, const float av[][kTW * kTH / 4], int rb0, int K, int cb,
                                              int l16, int q, float *__restrict__ out)
{
    constexpr int NS = kTW * kTH / 4;
    const int col = cb * 16 + l16;  // this lane's B column k
    const int cc = col < K ? col / 9 : 0, t = col < K ? col - cc * 9 : 0, ty = t / 3, tx = t - ty * 3;
    const float *pb = s_x + cc * kHalo + ty * kHW_ + tx + q;
    float bv[NS];
#pragma unroll
    for (int s4 = 0; s4 < NS; ++s4)  // pixel 4 s4 + q: row s4 / 4, column 4 s4 mod 16 + q
        bv[s4] = pb[(s4 >> 2) * kHW_ + ((4 * s4) & 15)];
    __builtin_amdgcn_sched_barrier(0);  // every read in flight before the first product
    f32x4 acc[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
        acc[rb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s4 = 0; s4 < NS; ++s4)
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
            acc[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[rb][s4], bv[s4], acc[rb], 0, 0, 0);
    if (col < K)
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[(size_t)((rb0 + rb) * 16 + 4 * q + r) * K + col] = acc[rb][r];
}

// 32 rows: columns 16 at a time, eight waves' worth of them with both row
// blocks each; of what is left, (column block, row block) pairs, from wave 4 on
// (waves 0..3 have the input gradient's slabs besides).
__device__ __forceinline__ void wgrad_32rows(const float *s_x, const float *s_d, int K, int wv, int l16, int q,
                                             float *__restrict__ out)
{
    constexpr int NS = kTW * kTH / 4, NW = kCnnWaves;
    float av[2][NS];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int s4 = 0; s4 < NS; ++s4)
            av[rb][s4] = s_d[(rb * 16 + l16) * kDS + q + 4 * s4];
    const int ncb = (K + 15) >> 4, whole = ncb / NW * NW;
#pragma unroll 1  // one set of operands in registers
    for (int cb = wv; cb < whole; cb += NW)
        wgrad_columns<2>(s_x, av, 0, K, cb, l16, q, out);
#pragma unroll 1
    for (int i = (wv + 4) % NW; i < 2 * (ncb - whole); i += NW) {
        if (i & 1)
            wgrad_columns<1>(s_x, av + 1, 1, K, whole + (i >> 1), l16, q, out);
        else
            wgrad_columns<1>(s_x, av, 0, K, whole + (i >> 1), l16, q, out);
    }
}

// Three rows (the output layer), the 64 columns from c0:
// v_mfma_f32_4x4x1_16b_f32, a row o = l mod 4 and a column of its own per lane,
// one pixel per product: the sum over pixels runs in the same order, one fma
// each, as in the 16x16x4 products (equal bit for bit), at 4 rows of matrix
// work instead of 16.
// 4x4x1 operand layout (lane l, block l / 4): A row l mod 4; B column l mod 4;
// result register r holds row r of column l mod 4.
__device__ __forceinline__ void wgrad_3rows(const float *s_x, const float *s_d, int K, int c0, int lane,
                                            float *__restrict__ out)
{
    static_assert(kTW == 16, "tile rows of 16 pixels");
    const int col = c0 + lane;
    const int cc = col < K ? col / 9 : 0, t = col < K ? col - cc * 9 : 0, ty = t / 3, tx = t - ty * 3;
    const float *pb = s_x + cc * kHalo + ty * kHW_ + tx, *pa = s_d + (lane & 3) * kDS;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float av[2][16], bv[2][16];  // a tile row of operands, read while the last one multiplies
    auto read = [&](int y) {
#pragma unroll
        for (int x = 0; x < 16; x += 4) {
            const float4 v = *(const float4 *)(pa + 16 * y + x);
            av[y & 1][x] = v.x, av[y & 1][x + 1] = v.y, av[y & 1][x + 2] = v.z, av[y & 1][x + 3] = v.w;
        }
#pragma unroll
        for (int x = 0; x < 16; ++x)
            bv[y & 1][x] = pb[y * kHW_ + x];
    };
    read(0);
#pragma unroll
    for (int y = 0; y < kTH; ++y) {
        if (y + 1 < kTH)
            read(y + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < 16; ++x)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(av[y & 1][x], bv[y & 1][x], acc, 0, 0, 0);
    }
    if (col < K)
#pragma unroll
        for (int o = 0; o < 3; ++o)
            out[(size_t)o * K + col] = acc[o];
}

// Bias sums of rows o < co: wave w takes rows w, w + 8, ... (all at once: one
// chain of lane exchanges); lane l adds pixels l and l + 64, then a fixed
// butterfly over the wave.
__device__ __forceinline__ void bias_sums(const float *s_d, int co, int wv, int lane, float *__restrict__ out)
{
    constexpr int NB = kMaxC / kCnnWaves;
    float v[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int o = min(wv + k * kCnnWaves, co - 1);
        v[k] = s_d[o * kDS + lane] + s_d[o * kDS + lane + 64];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < NB; ++k)
            v[k] += __shfl_xor(v[k], off, 64);
#pragma unroll
    for (int k = 0; k < NB; ++k)
        if (lane == 0 && wv + k * kCnnWaves < co)
            out[wv + k * kCnnWaves] = v[k];
}

struct CnnBackward {
    const float *dy, *x, *a1, *a2;
    const uint16_t *w2, *w3;
    float *part[3];
    int cin, H, W, tiles;
};

// CX: channels of x held (4, or 32 where there are more)
template <int CX>
__global__ __launch_bounds__(64 * kCnnWaves) void k_cnn_backward(CnnBackward q)
{
    constexpr int NT = 64 * kCnnWaves;
    using R2 = Region<2>;
    using R1 = Region<1>;
    using L1 = ConvLds<4>;
    using L2 = ConvLds<32>;
    constexpr int P1 = R2::N * 4, CS = L2::CS, P2 = R1::N * CS;
    __shared__ __attribute__((aligned(16))) uint16_t s_dy[3 * P1];
    __shared__ __attribute__((aligned(16))) uint16_t s_dz[3 * P2];
    __shared__ __attribute__((aligned(16))) uint16_t s_w3[32 * L1::WS];
    __shared__ __attribute__((aligned(16))) uint16_t s_w2[32 * L2::WS];
    __shared__ float s_x[kMaxC * kHalo];  // a2, then a1, then x on the tile with its halo
    // dy, dz2 and dz1 of the tile [o][p] (pixels outside the field zero)
    __shared__ __attribute__((aligned(16))) float s_d3[4 * kDS];
    __shared__ float s_d2[kMaxC * kDS], s_d1[kMaxC * kDS];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 31, hk = lane >> 5;
    const int H = q.H, W = q.W, cin = q.cin;
    const size_t HW = (size_t)H * W;
    const int tiles_j = (W + kTW - 1) / kTW, per = tiles_j * ((H + kTH - 1) / kTH);
    const bool small = H < Region<3>::H || W < Region<3>::W;
    // input tiles: thread (group g, pixel p) takes channels g, g + 2, ... of its
    // pixel; dy on the widened tile R2: a thread per pixel
    static_assert(2 * kHalo <= NT && R2::N <= NT && R1::N == kHalo && R1::kSlabs <= kCnnWaves, "threads and slabs");
    const int hp = tid % kHalo, hg = tid / kHalo, dyy = tid / R2::W, dyx = tid - dyy * R2::W;
    int n = 0, i0 = 0, j0 = 0;
    size_t halo_at = 0, dy_at = 0;
    float hv[kMaxC / 2], dv[4];
    dv[3] = 0.0f;
    auto locate = [&](int tile) {
        n = tile / per;
        const int r = tile - n * per, ti = r / tiles_j;
        i0 = ti * kTH;
        j0 = (r - ti * tiles_j) * kTW;
        halo_at = (size_t)wrap_index(small, i0 + hp / kHW_ - 1, H) * W + wrap_index(small, j0 + hp % kHW_ - 1, W);
        if (tid < R2::N)
            dy_at = (size_t)wrap_index(small, i0 + dyy - 2, H) * W + wrap_index(small, j0 + dyx - 2, W);
    };
    auto load_halo = [&](auto nu, const float *__restrict__ src, int ci) {
        if (hg < 2)
#pragma unroll
            for (int u = 0; u < decltype(nu)::value; ++u)
                hv[u] = src[((size_t)n * ci + min(hg + 2 * u, ci - 1)) * HW + halo_at];
    };
    auto store_halo = [&](auto nu) {
        if (hg < 2)
#pragma unroll
            for (int u = 0; u < decltype(nu)::value; ++u)
                s_x[(hg + 2 * u) * kHalo + hp] = hv[u];
    };
    using All = IntTag<kMaxC / 2>;
    auto load_first = [&]() {
        load_halo(All{}, q.a2, 32);
        if (tid < R2::N)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                dv[c] = q.dy[((size_t)n * 3 + c) * HW + dy_at];
    };
    locate(blockIdx.x);
    load_first();
    {
        WeightStage<NT, 32 * 32> sw2;
        WeightStage<NT, 3 * 32> sw3;
        sw2.load(q.w2, 32 * 32);
        sw3.load(q.w3, 3 * 32);
        for (int e = tid; e < 32 * 9; e += NT)  // the fourth channel's weights
            s_w3[(e / 9) * L1::WS + (e % 9) * 4 + 3] = 0;
        sw2.store(32 * 32, [&](int row, int t, uint16_t v) {  // row = c * 32 + o
            s_w2[(row & 31) * L2::WS + (8 - t) * L2::TS + (row >> 5)] = v;
        });
        sw3.store(3 * 32, [&](int row, int t, uint16_t v) {
            s_w3[(row & 31) * L1::WS + (8 - t) * L1::TS + (row >> 5)] = v;
        });
    }
    // the lane's r-th channel in a result, and its pixel of the tile in slab wv
    auto channel = [&](int r) { return 8 * (r >> 2) + 4 * hk + (r & 3); };
    for (int tile = blockIdx.x;;) {
        store_halo(All{});
        if (tid < R2::N) {
            put_split4(s_dy, tid * 4, P1, dv);
            const int y = dyy - 2, x = dyx - 2;
            if (y >= 0 && y < kTH && x >= 0 && x < kTW)
#pragma unroll
                for (int o = 0; o < 4; ++o)
                    s_d3[o * kDS + y * kTW + x] = i0 + y < H && j0 + x < W ? dv[o] : 0.0f;
        }
        load_halo(All{}, q.a1, 32);
        __syncthreads();
        const bool own = i0 + 2 * wv + (m >> 4) < H && j0 + (m & 15) < W;  // slab wv < 4
        float *out3 = q.part[2] + (size_t)tile * (3 * 288 + 3);
        // dz2 (waves 0..5), the output layer's gradients (waves 6, 7, then 2..4)
        if (wv < R1::kSlabs) {
            int ry, rx;
            const bool live = R1::pixel(wv, m, ry, rx);
            const int pix = ry * R1::W + rx;
            float mask[16];
#pragma unroll
            for (int r = 0; r < 16; ++r)
                mask[r] = s_x[channel(r) * kHalo + pix];
            const f32x16 acc = conv_slab<4, 4, L1::TS, R2::W>(s_dy, P1, ry * R2::W + rx, s_w3 + m * L1::WS, hk);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int ch = channel(4 * g + u);
                    v[u] = mask[4 * g + u] > 0.0f ? acc[4 * g + u] : 0.0f;
                    if (wv < 4)
                        s_d2[ch * kDS + wv * 32 + m] = own ? v[u] : 0.0f;
                }
                if (live)
                    put_split4(s_dz, pix * CS + channel(4 * g), P2, v);
            }
        }
        if (wv >= 6)
            wgrad_3rows(s_x, s_d3, 288, (wv - 6) * 64, lane, out3);
        else if (wv >= 2 && wv < 5)
            wgrad_3rows(s_x, s_d3, 288, wv * 64, lane, out3);
        bias_sums(s_d3, 3, wv, lane, out3 + 3 * 288);
        __syncthreads();
        store_halo(All{});
        load_halo(IntTag<CX / 2>{}, q.x, cin);
        __syncthreads();
        // dz1 (waves 0..3), the second layer's gradients
        float *out2 = q.part[1] + (size_t)tile * (32 * 288 + 32);
        if (wv < 4) {
            int ry, rx;
            Region<0>::pixel(wv, m, ry, rx);
            const int pix = (ry + 1) * R1::W + rx + 1;
            float mask[16];
#pragma unroll
            for (int r = 0; r < 16; ++r)
                mask[r] = s_x[channel(r) * kHalo + pix];
            // before the other waves' products, which keep the matrix cores busy
            // while these wait for LDS: else they ended 10,000 cycles later
            __builtin_amdgcn_s_setprio(3);
            const f32x16 acc =
                conv_slab<32, CS, L2::TS, R1::W>(s_dz, P2, ry * R1::W + rx, s_w2 + m * L2::WS, hk);
            __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                s_d1[channel(r) * kDS + wv * 32 + m] = own && mask[r] > 0.0f ? acc[r] : 0.0f;
        }
        wgrad_32rows(s_x, s_d2, 288, wv, lane & 15, lane >> 4, out2);
        bias_sums(s_d2, 32, wv, lane, out2 + 32 * 288);
        __syncthreads();
        store_halo(IntTag<CX / 2>{});
        float *out1 = q.part[0] + (size_t)tile * (32 * cin * 9 + 32);
        tile += gridDim.x;
        const bool more = tile < q.tiles;
        if (more) {
            locate(tile);
            load_first();
        }
        __syncthreads();
        wgrad_32rows(s_x, s_d1, cin * 9, wv, lane & 15, lane >> 4, out1);
        bias_sums(s_d1, 32, wv, lane, out1 + 32 * cin * 9);
        if (!more)
            break;
        __syncthreads();
    }
}

// Adam (Kingma & Ba, algorithm 1) on element e of tensor q of the jobs, with
// gradient gi.
__device__ __forceinline__ void adam_element(const AdamJobs &j, int q, int64_t e, float gi, const AdamStep &a)
{
    float *theta = j.theta[q], *m = j.m[q], *v = j.v[q];
    const float mi = a.beta1 * m[e] + (1.0f - a.beta1) * gi;
    const float vi = a.beta2 * v[e] + (1.0f - a.beta2) * gi * gi;
    m[e] = mi;
    v[e] = vi;
    const float th = theta[e] - a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
    theta[e] = th;
    if (j.bf16[q])
        j.bf16[q][e] = float_to_bf16_rne(th);
}

// The sums over blocks of the three layers' gradient partials (float64, in
// block order), and of the loss partials.  A block takes kReduceCols entries
// of one layer with kReduceSlices threads each: thread slice s adds blocks s,
// s + slices, ... in order, then the slices are added in order.  Entry e <
// nw of layer k goes to the weight gradient, the others to the bias gradient,
// each written to g[2 k], g[2 k + 1] of the jobs (ADAM: taken straight into
// the Adam step of that tensor instead).  The last block adds the loss
// partials: thread t partials t, t + 256, ... in order, then a fixed tree.
// 32 columns: whole 128-byte lines of the partials, which blocks of 16
// columns on different XCDs fetched twice.
constexpr int kReduceCols = 32, kReduceSlices = 16, kReduceThreads = kReduceCols * kReduceSlices;

struct ReduceJobs {
    const float *part[3];
    int nw[3], nb[3], first[3];  // weights, biases, first block
    float *g[6];
    const double *loss_part;
    int nblocks, nloss;
    int64_t count;  // values under the loss's mean
    float *loss;
};

template <bool ADAM>
__global__ __launch_bounds__(kReduceThreads) void k_cnn_reduce(ReduceJobs r, AdamJobs j, AdamStep a)
{
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ double s_red[4];
        double s = 0.0;
        if (threadIdx.x < 256)
            for (int b = threadIdx.x; b < r.nloss; b += 256)
                s += r.loss_part[b];
        s = cwave_sum(s);
        if ((threadIdx.x & 63) == 0 && threadIdx.x < 256)
            s_red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0)
            *r.loss = (float)((((s_red[0] + s_red[1]) + s_red[2]) + s_red[3]) / (double)r.count);
        return;
    }
    __shared__ double s_sum[kReduceSlices][kReduceCols];
    const int k = (int)blockIdx.x >= r.first[2] ? 2 : (int)blockIdx.x >= r.first[1] ? 1 : 0;
    const int nw = r.nw[k], total = nw + r.nb[k];
    const int col = threadIdx.x % kReduceCols, slice = threadIdx.x / kReduceCols;
    const int e = ((int)blockIdx.x - r.first[k]) * kReduceCols + col;
    double sum = 0.0;
    if (e < total) {
        const float *p = r.part[k] + e;
        int b = slice;
        constexpr int U = 32;  // loads in flight per thread; the additions stay in block order
        for (; b + (U - 1) * kReduceSlices < r.nblocks; b += U * kReduceSlices) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                v[u] = p[(size_t)(b + u * kReduceSlices) * total];
#pragma unroll
            for (int u = 0; u < U; ++u)
                sum += (double)v[u];
        }
        for (; b < r.nblocks; b += kReduceSlices)
            sum += (double)p[(size_t)b * total];
    }
    s_sum[slice][col] = sum;
    __syncthreads();
    if (slice == 0 && e < total) {
        double t = s_sum[0][col];
        for (int i = 1; i < kReduceSlices; ++i)
            t += s_sum[i][col];
        const int q = 2 * k + (e < nw ? 0 : 1), at = e < nw ? e : e - nw;
        if (ADAM)
            adam_element(j, q, at, (float)t, a);
        else
            r.g[q][at] = (float)t;
    }
}

// Mean squared error of given outputs: dy = 2 (y - t) / count, per-block
// float64 partials of sum (y - t)^2, added in order by k_cnn_reduce.
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ y, const float *__restrict__ t, int64_t count,
                                             float *__restrict__ dy, double *__restrict__ part)
{
    __shared__ double s_red[4];
    double acc = 0.0;
    const float scale = (float)(2.0 / (double)count);
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256) {
        const float d = y[e] - t[e];
        dy[e] = d * scale;
        acc += (double)d * (double)d;
    }
    acc = cwave_sum(acc);
    if ((threadIdx.x & 63) == 0)
        s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0)
        part[blockIdx.x] = ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];
}

// Adam on float32 master tensors with given gradients, up to kAdamMax of them
// in one launch (blockIdx.y selects the tensor); writes the bf16 copy where
// one is given.
__global__ void k_adam_many(AdamJobs j, AdamStep a)
{
    const int q = blockIdx.y;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < j.count[q])
        adam_element(j, q, e, j.g[q][e], a);
}

static AdamStep adam_step(float lr, float beta1, float beta2, float eps, int64_t t)
{
    return AdamStep{lr, beta1, beta2, eps, (float)(1.0 - pow((double)beta1, (double)t)),
                    (float)(1.0 - pow((double)beta2, (double)t))};
}

// x[n, c, p] = x[n, c, p] * scale[c] + shift[c] for c < nc (in place).
__global__ void k_channel_affine(float *__restrict__ x, int N, int C, int nc, int64_t HW,
                                 const float *__restrict__ scale, const float *__restrict__ shift)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per = (int64_t)nc * HW;
    if (e >= (int64_t)N * per)
        return;
    const int64_t n = e / per, r = e - n * per;
    const int c = (int)(r / HW);
    float *p = x + (n * C + c) * HW + (r - (int64_t)c * HW);
    *p = *p * scale[c] + shift[c];
}

// Per-sample relative L2 error of the first nc channels: out[s] =
// |a_s - b_s| / |b_s| (float64 sums, one block per sample, fixed order).
__global__ __launch_bounds__(256) void k_field_error(const float *__restrict__ a, const float *__restrict__ b, int C,
                                                     int nc, int64_t hw, double *__restrict__ out)
{
    __shared__ double s_red[2][4];
    const int smp = blockIdx.x;
    double num = 0.0, den = 0.0;
    for (int64_t e = threadIdx.x; e < (int64_t)nc * hw; e += 256) {
        const int64_t o = (int64_t)smp * C * hw + e;
        const double d = (double)a[o] - (double)b[o];
        num += d * d;
        den += (double)b[o] * (double)b[o];
    }
    num = cwave_sum(num);
    den = cwave_sum(den);
    if ((threadIdx.x & 63) == 0) {
        s_red[0][threadIdx.x >> 6] = num;
        s_red[1][threadIdx.x >> 6] = den;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double nn = ((s_red[0][0] + s_red[0][1]) + s_red[0][2]) + s_red[0][3];
        const double dd = ((s_red[1][0] + s_red[1][1]) + s_red[1][2]) + s_red[1][3];
        out[smp] = dd > 0.0 ? sqrt(nn / dd) : (nn > 0.0 ? INFINITY : 0.0);
    }
}

// Per-channel mean and standard deviation over n samples and hw pixels, in
// float64 and in a fixed order: each of kStatBlocks blocks of a channel sums
// its contiguous share of the channel's n * hw values (pass 1: values, pass
// 3: squared deviations from the mean), and one block per channel adds the
// shares in block order (passes 2 and 4).
constexpr int kStatBlocks = 256;

__device__ __forceinline__ double stat_block_sum(double acc)
{
    __shared__ double s_red[4];
    acc = cwave_sum(acc);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    return ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];  // valid in every thread
}

// pass 1 (mean == nullptr) or 3: partial sums of x, or of (x - mean)^2
__global__ __launch_bounds__(256) void k_stat_partial(const float *__restrict__ x, int n, int C, int64_t hw,
                                                      const double *__restrict__ mean, double *__restrict__ part)
{
    const int c = blockIdx.y, b = blockIdx.x;
    const int64_t cnt = (int64_t)n * hw;
    const int64_t lo = cnt * b / kStatBlocks, hi = cnt * (b + 1) / kStatBlocks;
    const double m = mean ? mean[c] : 0.0;
    double acc = 0.0;
    for (int64_t e = lo + threadIdx.x; e < hi; e += 256) {
        const int64_t smp = e / hw, px = e - smp * hw;
        const double v = (double)x[(smp * C + c) * hw + px];
        acc += mean ? (v - m) * (v - m) : v;
    }
    acc = stat_block_sum(acc);
    if (threadIdx.x == 0)
        part[(int64_t)c * kStatBlocks + b] = acc;
}

// pass 2 (mean of the partial sums) or 4 (standard deviation)
__global__ __launch_bounds__(256) void k_stat_final(const double *__restrict__ part, int64_t cnt,
                                                    double *__restrict__ out, int root)
{
    const int c = blockIdx.x;
    double acc = threadIdx.x < kStatBlocks ? part[(int64_t)c * kStatBlocks + threadIdx.x] : 0.0;
    acc = stat_block_sum(acc);
    if (threadIdx.x == 0)
        out[c] = root ? sqrt(acc / (double)cnt) : acc / (double)cnt;
}

// x[s, ch, :] = values[s]
__global__ void k_fill_channel(float *__restrict__ x, int n, int C, int ch, int64_t hw,
                               const float *__restrict__ values)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)n * hw)
        return;
    const int64_t s = e / hw;
    x[(s * C + ch) * hw + (e - s * hw)] = values[s];
}

// ---------------------------------------------------------------------------
// Coarse fields of a lattice: the mean over c x c blocks of sites of rho, jx,
// jy of the streamed populations (the fields step (ii) of the algorithm
// sees), out[3][ny/c][nx/c].  Many lattices of one shape: blockIdx.z selects
// the lattice, whose stored state is bufs[z] (or f alone), and its output
// starts at out + z * out_stride.
//
// A block takes one row of cells, kCoarsenCols columns of sites: its lanes load
// kCoarsenRows rows of sites at a time, neighbours in x on neighbouring lanes,
// and put their rho, jx, jy into LDS, where one lane per cell and field adds
// its cell's sites row by row.  One lane per cell loading its own sites read
// 7 c^2 scattered values in turn: 64 lattices of 256^2 in cells of 8 x 8 (117 MB)
// 61 -> 21 us.  Cells of one site, of two a side (of states that the caches hold) and
// of four on lattices narrower than a wave take a lane each all the same
// (k_coarsen_cells): there its loads are within a line of their neighbours' and LDS and
// barriers cost more.  us, a lane a cell / rows: 4096^2, c = 1 115 / 185, c = 2 110 / 100;
// 1024^2, c = 2 7.5 / 8.4; 64x8192, c = 2 5.5 / 9.4; 256^2, c = 2 3.7 / 4.3, c = 4 5.9 /
// 4.7; 16x30000, c = 4 16.4 / 17.9.  The sums and their order are the same.
// ---------------------------------------------------------------------------
constexpr int kCoarsenCols = 256, kCoarsenRows = 4;

__global__ __launch_bounds__(kCoarsenCols) void k_coarsen_cells(const float *f, const float *const *__restrict__ bufs,
                                                                StepArgs a, int cs, int cw, int chh,
                                                                float *__restrict__ out, int64_t out_stride)
{
    const int cx = blockIdx.x * kCoarsenCols + threadIdx.x, cy = blockIdx.y;
    if (cx >= cw)
        return;
    if (bufs)
        f = bufs[blockIdx.z];
    float sums[3] = {0.0f, 0.0f, 0.0f};
    for (int dy = 0; dy < cs; ++dy)
        for (int dx = 0; dx < cs; ++dx) {
            const PullSources32 g = pull_sources32(a, cx * cs + dx, cy * cs + dy);
            float v[7], m[3];
#pragma unroll
            for (int i = 0; i < 7; ++i)
                v[i] = ld32(f + (size_t)i * (uint32_t)a.plane, g.idx[i]);
            site_moments(v, m[0], m[1], m[2]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                sums[k] += m[k];
        }
    const float inv = 1.0f / (float)(cs * cs);
    float *o = out + (int64_t)blockIdx.z * out_stride + (size_t)cy * cw + cx;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        o[(size_t)k * chh * cw] = sums[k] * inv;
}

__global__ __launch_bounds__(kCoarsenCols) void k_coarsen(const float *f, const float *const *__restrict__ bufs,
                                                          StepArgs a, int cs, int cw, int chh, float *__restrict__ out,
                                                          int64_t out_stride)
{
    // site x of a row at x + x / cs (a cell's row starts in a bank of its own
    // where cs is a power of two); a cell wider than the block comes a row at a
    // time, in turns of the block's columns
    constexpr int W = 2 * kCoarsenCols;
    __shared__ float s[3][kCoarsenRows][W];
    if (bufs)
        f = bufs[blockIdx.z];
    const int per = cs < kCoarsenCols ? kCoarsenCols / cs : 1;  // cells of a block
    const int cx0 = blockIdx.x * per, cells = min(per, cw - cx0);
    const int x0 = cx0 * cs, width = cells * cs;
    const int cell = threadIdx.x / 3, q = threadIdx.x % 3;
    const uint32_t plane = (uint32_t)a.plane;
    float sums[(kCoarsenCols + 84) / 85];  // three lanes a cell: up to four cells of a lane
    constexpr int NS = sizeof(sums) / sizeof(sums[0]);
#pragma unroll
    for (int k = 0; k < NS; ++k)
        sums[k] = 0.0f;
    const int step = cs > kCoarsenCols ? 1 : kCoarsenRows;  // rows at a time
    for (int dy0 = 0; dy0 < cs; dy0 += step)
        for (int xb = 0; xb < width; xb += kCoarsenCols) {
            const int x = xb + (int)threadIdx.x, n = min(kCoarsenCols, width - xb);
            const int rows = min(step, cs - dy0);
            if (x < width) {
                float v[kCoarsenRows][7];
#pragma unroll
                for (int r = 0; r < kCoarsenRows; ++r) {
                    const PullSources32 g = pull_sources32(a, x0 + x, blockIdx.y * cs + dy0 + min(r, rows - 1));
#pragma unroll
                    for (int i = 0; i < 7; ++i)
                        v[r][i] = ld32(f + (size_t)i * plane, g.idx[i]);
                }
                const int at = (int)threadIdx.x + (int)threadIdx.x / cs;
#pragma unroll
                for (int r = 0; r < kCoarsenRows; ++r)
                    site_moments(v[r], s[0][r][at], s[1][r][at], s[2][r][at]);
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const int c = cell + k * 85;
                if (threadIdx.x < 255 && c < cells) {
                    const int m = min(cs, n);
                    const float *row = &s[q][0][c * (cs + 1)];
                    for (int r = 0; r < rows; ++r)
#pragma unroll 8
                        for (int dx = 0; dx < m; ++dx)
                            sums[k] += row[r * W + dx];
                }
            }
            __syncthreads();
        }
    const float inv = 1.0f / (float)(cs * cs);
    float *o = out + (int64_t)blockIdx.z * out_stride + (size_t)blockIdx.y * cw + cx0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const int c = cell + k * 85;
        if (threadIdx.x < 255 && c < cells)
            o[(size_t)q * chh * cw + c] = sums[k] * inv;
    }
}

__global__ __launch_bounds__(256) void k_lift_many(const float *__restrict__ coarse, int64_t in_stride, StepArgs a,
                                                   int cs, int cw, int chh, float *const *__restrict__ bufs)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
    if (x >= a.nx)
        return;
    const float *cf = coarse + (int64_t)blockIdx.z * in_stride;
    float *f = bufs[blockIdx.z];
    const int cx = x / cs, cy = y / cs;
    const size_t cp = (size_t)chh * cw;
    const float rho = fmaxf(cf[(size_t)cy * cw + cx], 0.0f);
    const float jx = cf[cp + (size_t)cy * cw + cx], jy = cf[2 * cp + (size_t)cy * cw + cx];
    const float r = rho > 0.0f ? 2.0f / rho : 0.0f;  // the steady state takes 2 u
    float eq[7];
    site_equilibrium(rho, jx * r, jy * r, eq);
    const uint32_t own = (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
#pragma unroll
    for (int i = 0; i < 7; ++i)
        st32(f + (size_t)i * (uint32_t)a.plane, own, eq[i]);
}

// Populations from coarse fields: every site of a c x c block gets the
// steady state xi(rho, j/rho) of its block (eq. fssD2Q7 with u* = u), as a
// stored state.  rho <= 0 gives empty sites.
__global__ __launch_bounds__(256) void k_lift(const float *__restrict__ coarse, StepArgs a, int cs, int cw, int chh,
                                              float *__restrict__ f)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
    if (x >= a.nx)
        return;
    const int cx = x / cs, cy = y / cs;
    const size_t cp = (size_t)chh * cw;
    const float rho = fmaxf(coarse[(size_t)cy * cw + cx], 0.0f);
    const float jx = coarse[cp + (size_t)cy * cw + cx], jy = coarse[2 * cp + (size_t)cy * cw + cx];
    const float r = rho > 0.0f ? 2.0f / rho : 0.0f;  // the steady state takes 2 u
    float eq[7];
    site_equilibrium(rho, jx * r, jy * r, eq);
    const uint32_t own = (uint32_t)y * (uint32_t)a.pitch + (uint32_t)x;
#pragma unroll
    for (int i = 0; i < 7; ++i)
        st32(f + (size_t)i * (uint32_t)a.plane, own, eq[i]);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static bool shape_ok(const lbm_cnn_shape *s)
{
    return s && s->n > 0 && s->h > 0 && s->w > 0 && s->hidden == 32 && s->cout == 3 && s->cin >= 3 &&
           s->cin <= 32 && (int64_t)s->h * s->w <= (1 << 26) && s->n <= 65535;
}
static int conv_tiles(int H, int W) { return ((H + kTH - 1) / kTH) * ((W + kTW - 1) / kTW); }

static int layer_total(const lbm_cnn_shape *s, int k)  // weights and biases of layer k
{
    return k == 0 ? 32 * s->cin * 9 + 32 : k == 1 ? 32 * 32 * 9 + 32 : 3 * 32 * 9 + 3;
}

struct CnnWs {
    double *part;     // loss partials
    float *gpart[3];  // per-tile gradient partials of each layer
    float *dy;        // dL/dy [n][cout][hw]
    size_t total;
};

static const int kMseBlocks = 1024;

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Workspace of the backward pass: loss and gradient partials, dL/dy.  base == nullptr only measures the size.
static CnnWs cnn_layout(const lbm_cnn_shape *s, char *base)
{
    CnnWs L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align256(off + bytes);
        return base ? base + o : nullptr;
    };
    const int64_t hw = (int64_t)s->h * s->w;
    const size_t tiles = (size_t)s->n * conv_tiles(s->h, s->w);
    L.part = (double *)take(std::max(tiles, (size_t)kMseBlocks) * sizeof(double));
    for (int k = 0; k < 3; ++k)
        L.gpart[k] = (float *)take(tiles * (size_t)layer_total(s, k) * sizeof(float));
    L.dy = (float *)take((size_t)s->n * s->cout * hw * sizeof(float));
    L.total = off;
    return L;
}

// whether a[na] and b[nb] share memory
static bool overlap(const float *a, size_t na, const float *b, size_t nb)
{
    return (uintptr_t)a < (uintptr_t)(b + nb) && (uintptr_t)b < (uintptr_t)(a + na);
}

static void launch_coarsen(const float *f, const float *const *bufs, int n, const StepArgs &a, int c, int cw, int chh,
                           float *out, int64_t out_stride, hipStream_t st)
{
    if (c == 1 || (c == 2 && (int64_t)n * a.nx * a.ny < 1 << 23) || (c == 4 && a.nx < 64)) {
        hipLaunchKernelGGL(k_coarsen_cells, dim3((cw + kCoarsenCols - 1) / kCoarsenCols, chh, n), dim3(kCoarsenCols), 0,
                           st, f, bufs, a, c, cw, chh, out, out_stride);
        return;
    }
    const int per = std::max(1, kCoarsenCols / c);
    hipLaunchKernelGGL(k_coarsen, dim3((cw + per - 1) / per, chh, n), dim3(kCoarsenCols), 0, st, f, bufs, a, c, cw, chh,
                       out, out_stride);
}

template <int MODE>
static hipError_t forward(const lbm_cnn_shape *s, const lbm_cnn_params *p, CnnForward q, hipStream_t st)
{
    for (int k = 0; k < 3; ++k) {
        q.w[k] = p->w[k];
        q.b[k] = p->b[k];
    }
    q.cin = s->cin;
    q.H = s->h;
    q.W = s->w;
    q.tiles = s->n * conv_tiles(s->h, s->w);
    // a block fills a CU's LDS: one per CU, each taking every 256th tile
    const dim3 grd(std::min(q.tiles, 256)), blk(64 * kCnnWaves);
    if (s->cin <= 4)
        hipLaunchKernelGGL((k_cnn_forward<4, MODE>), grd, blk, 0, st, q);
    else if (MODE == kCnnRaw && s->cin <= 16)
        hipLaunchKernelGGL((k_cnn_forward<16, kCnnRaw>), grd, blk, 0, st, q);
    else if (MODE == kCnnRaw)
        hipLaunchKernelGGL((k_cnn_forward<32, kCnnRaw>), grd, blk, 0, st, q);
    else
        return hipErrorInvalidValue;  // the surrogate has three or four channels
    return hipGetLastError();
}

// From dy and the activations to the gradients (adam == nullptr: in g; else
// taken into the Adam step) and the loss (from nloss partials).
static hipError_t backward(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, const float *a1,
                           const float *a2, const CnnWs &L, int nloss, float *loss, const lbm_cnn_grads *g,
                           const AdamJobs *adam, const AdamStep &step, hipStream_t st)
{
    const int co[3] = {32, 32, 3}, ci[3] = {s->cin, 32, 32};
    ReduceJobs r{};
    CnnBackward q{L.dy, x, a1, a2, p->w[1], p->w[2], {}, s->cin, s->h, s->w, s->n * conv_tiles(s->h, s->w)};
    int first = 0;
    for (int i = 0; i < 3; ++i) {
        q.part[i] = L.gpart[i];
        r.part[i] = L.gpart[i];
        r.nw[i] = co[i] * ci[i] * 9;
        r.nb[i] = co[i];
        r.first[i] = first;
        first += (layer_total(s, i) + kReduceCols - 1) / kReduceCols;
        if (g) {
            r.g[2 * i] = g->w[i];
            r.g[2 * i + 1] = g->b[i];
        }
    }
    r.nblocks = q.tiles;
    r.loss_part = L.part;
    r.nloss = nloss;
    r.count = (int64_t)s->n * s->cout * s->h * s->w;
    r.loss = loss;
    const dim3 grd(std::min(q.tiles, 256)), blk(64 * kCnnWaves);
    if (s->cin <= 4)
        hipLaunchKernelGGL(k_cnn_backward<4>, grd, blk, 0, st, q);
    else
        hipLaunchKernelGGL(k_cnn_backward<kMaxC>, grd, blk, 0, st, q);
    if (adam)
        hipLaunchKernelGGL(k_cnn_reduce<true>, dim3(first + 1), dim3(kReduceThreads), 0, st, r, *adam, step);
    else
        hipLaunchKernelGGL(k_cnn_reduce<false>, dim3(first + 1), dim3(kReduceThreads), 0, st, r, AdamJobs{}, step);
    return hipGetLastError();
}

hipError_t cnn_predict(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, const float *norm, float *y,
                       hipStream_t st)
{
    CnnForward q{};
    q.x = x;
    q.norm = norm;
    q.y = y;
    return forward<kCnnPredict>(s, p, q, st);
}

hipError_t cnn_train(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, const float *target,
                     const int32_t *idx, const float *norm, float *xn, float *a1, float *a2, void *ws,
                     const AdamJobs &adam, float lr, float beta1, float beta2, float eps, int64_t t, float *loss,
                     hipStream_t st)
{
    const CnnWs L = cnn_layout(s, (char *)ws);
    CnnForward q{};
    q.x = x;
    q.target = target;
    q.idx = idx;
    q.norm = norm;
    q.xn = xn;
    q.a1 = a1;
    q.a2 = a2;
    q.dy = L.dy;
    q.loss = L.part;
    q.dscale = (float)(2.0 / (double)((int64_t)s->n * s->cout * s->h * s->w));
    hipError_t e = forward<kCnnTrain>(s, p, q, st);
    if (e != hipSuccess)
        return e;
    return backward(s, p, xn, a1, a2, L, s->n * conv_tiles(s->h, s->w), loss, nullptr, &adam,
                    adam_step(lr, beta1, beta2, eps, t), st);
}

}  // namespace lbm

using namespace lbm;

extern "C" {

size_t lbm_cnn_workspace_bytes(const lbm_cnn_shape *s)
{
    if (!shape_ok(s))
        return 0;
    return cnn_layout(s, nullptr).total;
}

int32_t lbm_cnn_forward(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, float *a1, float *a2,
                        float *y, void *ws, size_t ws_bytes, void *stream)
{
    if (!shape_ok(s))
        return fail(LBM_EINVAL, "invalid network shape (hidden must be 32, cout 3, 3 <= cin <= 32)");
    if (!p || !x || !a1 || !a2 || !y || !ws)
        return fail(LBM_EINVAL, "null pointer");
    for (int k = 0; k < 3; ++k)
        if (!p->w[k] || !p->b[k])
            return fail(LBM_EINVAL, "null weight or bias");
    if (ws_bytes < cnn_layout(s, nullptr).total)
        return fail(LBM_EINVAL, "workspace smaller than lbm_cnn_workspace_bytes()");
    const size_t px = (size_t)s->n * s->h * s->w;
    // y in x's or a1's memory: a block writes its tile while others still read x
    // around theirs or write a1, so y comes by way of the workspace
    const bool aside = overlap(y, 3 * px, x, s->cin * px) || overlap(y, 3 * px, a1, 32 * px);
    CnnForward q{};
    q.x = x;
    q.a1 = a1;
    q.a2 = a2;
    q.y = aside ? cnn_layout(s, (char *)ws).dy : y;
    LBM_HIP_TRY(forward<kCnnRaw>(s, p, q, (hipStream_t)stream));
    if (aside)
        LBM_HIP_TRY(hipMemcpyAsync(y, q.y, 3 * px * sizeof(float), hipMemcpyDeviceToDevice, (hipStream_t)stream));
    return LBM_OK;
}

int32_t lbm_cnn_backward(const lbm_cnn_shape *s, const lbm_cnn_params *p, const float *x, const float *a1,
                         const float *a2, const float *y, const float *target, const lbm_cnn_grads *g,
                         float *loss, void *ws, size_t ws_bytes, void *stream)
{
    if (!shape_ok(s))
        return fail(LBM_EINVAL, "invalid network shape (hidden must be 32, cout 3, 3 <= cin <= 32)");
    if (!p || !x || !a1 || !a2 || !y || !target || !g || !loss || !ws)
        return fail(LBM_EINVAL, "null pointer");
    for (int k = 0; k < 3; ++k)
        if (!g->w[k] || !g->b[k])
            return fail(LBM_EINVAL, "null gradient buffer");
    const CnnWs L = cnn_layout(s, (char *)ws);
    if (ws_bytes < L.total)
        return fail(LBM_EINVAL, "workspace smaller than lbm_cnn_workspace_bytes()");
    hipStream_t st = (hipStream_t)stream;
    const int64_t count = (int64_t)s->n * s->cout * s->h * s->w;
    hipLaunchKernelGGL(k_mse, dim3(kMseBlocks), dim3(256), 0, st, y, target, count, L.dy, L.part);
    LBM_HIP_TRY(backward(s, p, x, a1, a2, L, kMseBlocks, loss, g, nullptr, AdamStep{}, st));
    return LBM_OK;
}

int32_t lbm_cnn_adam(float *theta, float *m, float *v, const float *grad, int64_t count, float lr, float beta1,
                     float beta2, float eps, int64_t t, uint16_t *bf16_out, void *stream)
{
    if (!theta || !m || !v || !grad || count < 0 || t < 1)
        return fail(LBM_EINVAL, "invalid Adam arguments");
    if (!(lr >= 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
        return fail(LBM_EINVAL, "invalid Adam hyper-parameters");
    AdamJobs j{};
    j.theta[0] = theta;
    j.m[0] = m;
    j.v[0] = v;
    j.g[0] = grad;
    j.count[0] = count;
    j.bf16[0] = bf16_out;
    if (count > 0)
        hipLaunchKernelGGL(k_adam_many, dim3((unsigned)((count + 255) / 256), 1), dim3(256), 0, (hipStream_t)stream, j,
                           adam_step(lr, beta1, beta2, eps, t));
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

int32_t lbm_channel_affine(float *x, int32_t n, int32_t c, int32_t nc, int64_t hw, const float *scale,
                           const float *shift, void *stream)
{
    if (!x || !scale || !shift || n < 0 || c < 1 || nc < 0 || nc > c || hw < 0)
        return fail(LBM_EINVAL, "invalid channel_affine arguments");
    const int64_t total = (int64_t)n * nc * hw;
    if (total > 0)
        hipLaunchKernelGGL(k_channel_affine, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           x, n, c, nc, hw, scale, shift);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

int32_t lbm_field_error(const float *a, const float *b, int32_t n, int32_t c, int32_t nc, int64_t hw, double *out,
                        void *stream)
{
    if (!a || !b || !out || n < 0 || c < 1 || nc < 1 || nc > c || hw < 1)
        return fail(LBM_EINVAL, "invalid field_error arguments");
    if (n > 0)
        hipLaunchKernelGGL(k_field_error, dim3(n), dim3(256), 0, (hipStream_t)stream, a, b, c, nc, hw, out);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

size_t lbm_channel_stats_workspace_bytes(int32_t c) { return c < 1 ? 0 : (size_t)c * kStatBlocks * sizeof(double); }

int32_t lbm_channel_stats(const float *x, int32_t n, int32_t c, int64_t hw, double *mean, double *stdev, void *ws,
                          size_t ws_bytes, void *stream)
{
    if (!x || !mean || !stdev || !ws || n < 1 || c < 1 || hw < 1)
        return fail(LBM_EINVAL, "invalid channel_stats arguments");
    if (ws_bytes < lbm_channel_stats_workspace_bytes(c))
        return fail(LBM_EINVAL, "workspace smaller than lbm_channel_stats_workspace_bytes()");
    hipStream_t st = (hipStream_t)stream;
    double *part = (double *)ws;
    const int64_t cnt = (int64_t)n * hw;
    hipLaunchKernelGGL(k_stat_partial, dim3(kStatBlocks, c), dim3(256), 0, st, x, n, c, hw, (const double *)nullptr,
                       part);
    hipLaunchKernelGGL(k_stat_final, dim3(c), dim3(256), 0, st, part, cnt, mean, 0);
    hipLaunchKernelGGL(k_stat_partial, dim3(kStatBlocks, c), dim3(256), 0, st, x, n, c, hw, (const double *)mean,
                       part);
    hipLaunchKernelGGL(k_stat_final, dim3(c), dim3(256), 0, st, part, cnt, stdev, 1);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

int32_t lbm_fill_channel(float *x, int32_t n, int32_t c, int32_t ch, int64_t hw, const float *values, void *stream)
{
    if (!x || !values || n < 0 || c < 1 || ch < 0 || ch >= c || hw < 1)
        return fail(LBM_EINVAL, "invalid fill_channel arguments");
    const int64_t total = (int64_t)n * hw;
    if (total > 0)
        hipLaunchKernelGGL(k_fill_channel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           x, n, c, ch, hw, values);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

int32_t lbm_coarsen(const lbm_params *p, const float *f, int32_t c, float *out, void *stream)
{
    int32_t rc = validate_params(p, p ? p->nx : 0);
    if (rc)
        return rc;
    if (!f || !out)
        return fail(LBM_EINVAL, "null pointer");
    if (p->lattice != LBM_D2Q7)
        return fail(LBM_EUNSUPPORTED, "coarse fields take the D2Q7 lattice");
    if (p->storage != LBM_F32)
        return fail(LBM_EUNSUPPORTED, "coarse fields take F32 storage");
    if (c < 1 || p->nx % c || p->ny % c || ((c & 1) && c != 1))
        return fail(LBM_EINVAL, "c must divide nx and ny and be 1 or even");
    if ((uint64_t)p->nx * p->ny * 7ull >= (1ull << 30))
        return fail(LBM_EINVAL, "lattice too large");
    const StepArgs a = make_step_args(*p, p->nx);
    const int cw = p->nx / c, chh = p->ny / c;
    launch_coarsen(f, nullptr, 1, a, c, cw, chh, out, 0, (hipStream_t)stream);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

static int32_t check_fields(const lbm_params *p, int32_t c)
{
    int32_t rc = validate_params(p, p ? p->nx : 0);
    if (rc)
        return rc;
    if (p->lattice != LBM_D2Q7)
        return fail(LBM_EUNSUPPORTED, "coarse fields take the D2Q7 lattice");
    if (p->storage != LBM_F32)
        return fail(LBM_EUNSUPPORTED, "coarse fields take F32 storage");
    if (c < 1 || p->nx % c || p->ny % c || ((c & 1) && c != 1))
        return fail(LBM_EINVAL, "c must divide nx and ny and be 1 or even");
    if ((uint64_t)p->nx * p->ny * 7ull >= (1ull << 30))
        return fail(LBM_EINVAL, "lattice too large");
    return LBM_OK;
}

int32_t lbm_coarsen_many(const lbm_params *p, int32_t n, const float *const *bufs, int32_t c, float *out,
                         int64_t out_stride, void *stream)
{
    int32_t rc = check_fields(p, c);
    if (rc)
        return rc;
    const int cw = p->nx / c, chh = p->ny / c;
    if (!bufs || !out || n < 0 || n > 65535 || out_stride < 3ll * cw * chh)
        return fail(LBM_EINVAL, "invalid coarsen_many arguments");
    const StepArgs a = make_step_args(*p, p->nx);
    if (n > 0)
        launch_coarsen(nullptr, bufs, n, a, c, cw, chh, out, out_stride, (hipStream_t)stream);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

int32_t lbm_lift_many(const lbm_params *p, int32_t n, const float *coarse, int64_t in_stride, int32_t c,
                      float *const *bufs, void *stream)
{
    int32_t rc = check_fields(p, c);
    if (rc)
        return rc;
    const int cw = p->nx / c, chh = p->ny / c;
    if (!bufs || !coarse || n < 0 || n > 65535 || in_stride < 3ll * cw * chh)
        return fail(LBM_EINVAL, "invalid lift_many arguments");
    const StepArgs a = make_step_args(*p, p->nx);
    if (n > 0)
        hipLaunchKernelGGL(k_lift_many, dim3((p->nx + 255) / 256, p->ny, n), dim3(256), 0, (hipStream_t)stream,
                           coarse, in_stride, a, c, cw, chh, bufs);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

int32_t lbm_lift(const lbm_params *p, const float *coarse, int32_t c, float *f, void *stream)
{
    int32_t rc = validate_params(p, p ? p->nx : 0);
    if (rc)
        return rc;
    if (!f || !coarse)
        return fail(LBM_EINVAL, "null pointer");
    if (p->lattice != LBM_D2Q7)
        return fail(LBM_EUNSUPPORTED, "lifting takes the D2Q7 lattice");
    if (p->storage != LBM_F32)
        return fail(LBM_EUNSUPPORTED, "lifting writes F32 storage");
    if (c < 1 || p->nx % c || p->ny % c || ((c & 1) && c != 1))
        return fail(LBM_EINVAL, "c must divide nx and ny and be 1 or even");
    if ((uint64_t)p->nx * p->ny * 7ull >= (1ull << 30))
        return fail(LBM_EINVAL, "lattice too large");
    const StepArgs a = make_step_args(*p, p->nx);
    hipLaunchKernelGGL(k_lift, dim3((p->nx + 255) / 256, p->ny), dim3(256), 0, (hipStream_t)stream, coarse, a, c,
                       p->nx / c, p->ny / c, f);
    LBM_HIP_TRY(hipGetLastError());
    return LBM_OK;
}

}  // extern "C"
