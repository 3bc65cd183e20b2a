// k_cnn.hip -- the learned depth denoiser that can replace APSS in the depth
// block (the paper treats the denoiser as interchangeable: Results,
// "Reconstruction algorithm"; Discussion, other denoisers trade quality for
// speed).  Reading (not in the paper): a four-layer 3x3 convolutional network
// on per-pixel slot maps (features of the first three slots: depth relative
// to the mean of the same-surface neighbours -- points of the 5x5 window
// within 3 sigma_h -- in sigma_h units, log(1 + r), valid flag, neighbour
// count) predicting each slot's depth correction in sigma_h units; pixels
// with four points keep APSS.
//
// Every convolution is an implicit GEMM on the matrix cores:
// v_mfma_f32_16x16x32_f16 (FP16 inputs, FP32 accumulation).  Activations are
// FP16 NHWC with 16 or 32 channels, weights FP16.
//   forward:         Y[p][co]   = b[co] + sum_{tap, ci} X[p + tap][ci] W[tap][ci][co]
//   backward data:   dX[p][ci]  = sum_{tap, co} dY[p + tap][co] W'[tap][co][ci],
//                    W' the tap-flipped transpose, gated by the ReLU of X
//   backward weight: dW[tap][ci][co] = sum_p X[p + tap][ci] dY[p][co],
//                    per-workgroup partials reduced in a fixed order
// Forward and backward data each run as one kernel on 16 x 16 tiles, the
// intermediate maps of a tile (grown by the receptive field of the layers that
// follow) in LDS; a training step stores the hidden activations and gradient
// maps for the weight gradients, which are one launch over all layers, and one
// more kernel reduces them and updates the weights.
#include "rt3d_dev.h"
#include "rt3d_points.h"
#include "rt3d_cnn.h"

#include <hip/hip_fp16.h>

#include <type_traits>

namespace rt3d {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float4_t mfma32(half8_t a, half8_t b, float4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ half4_t to_half4(float4_t v)
{
    return (half4_t){(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

// Features of the first three slots, FP16 [P][16].
// Features of slots k < min(cnt, 3): the neighbours of slot k are the points
// (any slot) of the 5x5 window (same frame, inside the image, itself
// included) within CNN_GATE sigma_h of t_k; channels 4k .. 4k+3 hold
// (t_k - their mean) / sigma_h clipped to [-8, 8], log(1 + r_k), 1 and their
// number / 25.  The other channels are zero.
// Features of 16 x 16 pixel tiles: the tile's depths with a 2-pixel halo (the
// 5 x 5 windows) staged in LDS (slots without a point as no_depth()), a thread
// per point (list_points), which passes the window's 100 slots without a
// branch, a row's reads in flight together; features meet in LDS and leave as
// whole lines.  4 x 256 x 256 pixels of 1.4 points: 21 us (half of it the vector
// ALU), against 29 us for a thread per pixel that followed the counts.
constexpr int PKT = 16, PKS = PKT + 4, PK_THREADS = 512;
__global__ __launch_bounds__(PK_THREADS, 4) void k_cnn_pack(Shape sh, DevState s, float sigma_h,
                                                            __half* __restrict__ x)
{
    constexpr int NS = PKS * PKS;
    __shared__ double tl[KM * NS];
    __shared__ uint4 out[PKT * PKT * 2];              // 16 halves per pixel
    __shared__ uint16_t pl[KM * PKT * PKT];
    __shared__ int wave_points[4];
    const long long S = sh.S;   // slot stride (the whole batch's pixels when sh is one group of it)
    const int tiles_x = (sh.cols + PKT - 1) / PKT, tiles_y = (sh.rows + PKT - 1) / PKT;
    const int tpf = tiles_x * tiles_y;
    const int fr = (int)(blockIdx.x / tpf), tr = (int)(blockIdx.x % tpf);
    const int i0 = (tr / tiles_x) * PKT, j0 = (tr % tiles_x) * PKT;
    const long long fbase = (long long)fr * sh.rows * sh.cols;
    for (int xx = threadIdx.x; xx < NS; xx += PK_THREADS) {
        const int i2 = i0 - 2 + xx / PKS, j2 = j0 - 2 + xx % PKS;
        const bool inside = i2 >= 0 && i2 < sh.rows && j2 >= 0 && j2 < sh.cols;
        const long long pp = fbase + (inside ? (long long)i2 * sh.cols + j2 : 0);
        double t[KM];
        const int c2 = load_cnt(s.cnt, pp);
#pragma unroll
        for (int k = 0; k < KM; ++k) t[k] = s.t[k * S + pp];
#pragma unroll
        for (int k = 0; k < KM; ++k) tl[k * NS + xx] = inside && k < c2 ? t[k] : no_depth();
    }
    out[threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
    int c = 0;
    if (threadIdx.x < PKT * PKT) {
        const int i = i0 + threadIdx.x / PKT, j = j0 + threadIdx.x % PKT;
        if (i < sh.rows && j < sh.cols) c = min(load_cnt(s.cnt, fbase + (long long)i * sh.cols + j), 3);
    }
    const int points = list_points(c, wave_points, pl);         // (its barriers: the tile too)
    const double gate = CNN_GATE * (double)sigma_h;
    for (int q = threadIdx.x; q < points; q += PK_THREADS) {
        const int pk = pl[q], k = pk % KM, px = pk / KM, ty = px / PKT, tx = px % PKT;
        const int xc = (ty + 2) * PKS + tx + 2;
        const float r = s.r[k * S + fbase + (long long)(i0 + ty) * sh.cols + j0 + tx];
        const double tk = tl[k * NS + xc];
        double sum = 0.0;
        int n = 0;
        // the terms in window order: rows, then columns, then slots
#pragma unroll 1
        for (int di = -2; di <= 2; ++di)
#pragma unroll
            for (int dj = -2; dj <= 2; ++dj)
#pragma unroll
                for (int k2 = 0; k2 < KM; ++k2) {
                    const double tm = tl[k2 * NS + xc + di * PKS + dj];
                    const bool in = fabs(tm - tk) <= gate;
                    sum += in ? tm : 0.0;
                    n += in ? 1 : 0;
                }
        const double mean = sum / n;
        const float v0 = fminf(fmaxf((float)((tk - mean) / (double)sigma_h), -8.f), 8.f), v1 = log1pf(r);
        const float v3 = (float)n / 25.f;
        uint2 o;
        o.x = (uint32_t)__half_as_ushort(__float2half(v0)) | ((uint32_t)__half_as_ushort(__float2half(v1)) << 16);
        o.y = (uint32_t)__half_as_ushort(__float2half(1.f)) | ((uint32_t)__half_as_ushort(__float2half(v3)) << 16);
        reinterpret_cast<uint2*>(out)[px * 4 + k] = o;
    }
    __syncthreads();
    const int px = threadIdx.x / 2, i = i0 + px / PKT, j = j0 + px % PKT;
    if (i < sh.rows && j < sh.cols)
        reinterpret_cast<uint4*>(x + (fbase + (long long)i * sh.cols + j) * 16)[threadIdx.x % 2] = out[threadIdx.x];
}
static_assert(PK_THREADS == 2 * PKT * PKT, "a thread per 16 bytes of the tile's features");

// Adam on one FP32 master weight.
__device__ __forceinline__ float adam_step(float* w, float* m, float* v, int idx, float gi, const CnnAdam& o, float c1,
                                           float c2)
{
    const float mi = o.beta1 * m[idx] + (1.f - o.beta1) * gi;
    const float vi = o.beta2 * v[idx] + (1.f - o.beta2) * gi * gi;
    m[idx] = mi;
    v[idx] = vi;
    const float wn = w[idx] - o.lr * (mi / c1) / (sqrtf(vi / c2) + o.eps);
    w[idx] = wn;
    return wn;
}

// The FP16 kernel layouts of master weight idx (flat: per layer [3][3][cin]
// [cout], then bias[cout]) with value v: forward wt[co][tap cis + ci];
// backward data wb[ci][tap' cos + co], tap' = 8 - tap, of layers 1 and 2, and
// wb[ci][4 tap' + co] (rows of 64) of layer 3, whose output gradient has four
// stored channels.  The padding (zero) is the allocation's.
__device__ __forceinline__ void store_weight(const CnnWeights& W, int idx, float v)
{
    int l = 0;
#pragma unroll
    for (int k = 1; k < CNN_LAYERS; ++k) l = idx >= CNN_OFF[k] ? k : l;
    const int off = l == 0 ? CNN_OFF[0] : l == 1 ? CNN_OFF[1] : l == 2 ? CNN_OFF[2] : CNN_OFF[3];
    const int cin = l == 0 ? 16 : 32, cout = l == 3 ? 3 : 32;
    const int p = idx - off;
    __half* wt = l == 0 ? W.wt[0] : l == 1 ? W.wt[1] : l == 2 ? W.wt[2] : W.wt[3];
    float* bias = l == 0 ? W.bias[0] : l == 1 ? W.bias[1] : l == 2 ? W.bias[2] : W.bias[3];
    if (p >= 9 * cin * cout) {
        bias[p - 9 * cin * cout] = v;
        return;
    }
    const int co = p % cout, row = p / cout, ci = row % cin, tap = row / cin;
    const __half h = __float2half(v);
    wt[co * 9 * cin + row] = h;
    if (l == 3) W.wb[3][ci * 64 + (8 - tap) * 4 + co] = h;
    else if (l > 0) (l == 1 ? W.wb[1] : W.wb[2])[ci * 288 + (8 - tap) * 32 + co] = h;
}

__global__ __launch_bounds__(256) void k_cnn_prepare(CnnWeights W)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < CNN_PARAMS) store_weight(W, idx, W.master[idx]);
}

// ---------------------------------------------------------------------------
// Forward and backward data, fused over the layers: one FT x FT output tile in
// one workgroup of FW wavefronts, every intermediate map kept in LDS as
// FP16 (the rounding of a stored activation).  Layer l computes its output
// over the tile grown by the receptive field of the layers after it; outputs
// at positions outside the image are set to zero, which is the next layer's
// zero padding.  The weights are the matrix product's A operand (rows: output
// channels; lane i + 16 g holds row i, k = 8 g .. 8 g + 7) and stay in
// registers for the whole layer; B's columns are 16 pixels, gathered from LDS
// per lane (16-byte chunks of 8 channels of the pixel under the tap), so that
// a lane ends with four consecutive channels (4 g .. 4 g + 3) of pixel i: one
// 8-byte store.  262 k pixels' forward pass: 37.0 us, 65 us with the pixels as
// rows, two-byte LDS stores and a swizzled layout (its matrix products take 9
// us, its LDS reads about as long); bound by the layers' serial chains at two
// wavefronts per SIMD (four of 128 registers, with spilled or single tiles in
// flight: 45 to 63 us).  A training step's forward pass on 131 k pixels: 32 us,
// backward data 19 us (47 and 46 us as a launch per layer).
constexpr int FT = 16;                   // output tile side
constexpr int FR0 = FT + 8;              // side of the staged input features (4-pixel halo)
constexpr int FW = 4;                    // wavefronts
constexpr int FU = 2;                    // 16-pixel tiles a wavefront works on at once
constexpr int FA = 3;                    // chunks read ahead of their products

// Halves from one pixel to the next in LDS: padded by 16 bytes, so that the
// same 16-byte chunk of 8 consecutive pixels lies in 8 distinct bank groups
// and every tap is a constant offset (an instruction's immediate).
template <int C>
constexpr int px_stride() { return C == 4 ? 4 : C + 8; }

// The tile's place.
struct TilePos {
    int Y0, X0, H, W;
    long long fbase;      // first pixel of the frame

    __device__ __forceinline__ TilePos(int tile, int H_, int W_) : H(H_), W(W_)
    {
        const int tx_n = (W + FT - 1) / FT, ty_n = (H + FT - 1) / FT;
        const int f = tile / (tx_n * ty_n), tr = tile % (tx_n * ty_n);
        Y0 = (tr / tx_n) * FT;
        X0 = (tr % tx_n) * FT;
        fbase = (long long)f * H * W;
    }
};

// A layer's weights [16 NT][K] as A operands, and its bias (nullptr: zero),
// loaded where this is written (the pointer is one the compiler cannot see
// through: all layers' weights together do not fit the registers; loading them
// a layer ahead cost more registers than the wait, 42.5 against 37.0 us).
template <int CIN, int NT>
struct LayerWeights {
    static constexpr int K = CIN == 4 ? 64 : 9 * CIN;      // weights per output channel, stored
    static constexpr int KC = (K + 31) / 32;
    half8_t w[KC][NT];
    float4_t b[NT];

    __device__ __forceinline__ LayerWeights(const __half* src, const float* bias)
    {
        auto Wt = (const __attribute__((address_space(1))) _Float16*)src;
        asm volatile("" : "+s"(Wt));
        const int i = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            b[n] = (float4_t){0.f, 0.f, 0.f, 0.f};
            if (bias) b[n] = *reinterpret_cast<const float4_t*>(bias + n * 16 + 4 * g);
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const int k0 = kc * 32 + 8 * g;
                half8_t v = {};
                if (K % 32 == 0 || k0 < K) v = *(const __attribute__((address_space(1))) half8_t*)(Wt + (n * 16 + i) * K + k0);
                w[kc][n] = v;
            }
        }
    }
};

// One layer over the RO x RO output region (the tile grown by HALO = (RO -
// FT) / 2 pixels) whose input region (RO + 2 wide) sits in `in`: CIN channels
// per pixel (4: 8 bytes each, two taps per 16-byte chunk), NT output tiles of 16
// channels, the bias added to the sums.  pre(inside, pix, n) runs before the products of a 16-pixel
// tile and gives what epi(m, oy, ox, inside, pix, n, sums, pre's value) takes
// after them, per tile n of output channels; pix: the pixel's number in the
// batch (where inside the image).  A lane of a region's last, partial tile
// past its end works on pixel 0 and stores nothing; a chunk past the ninth tap
// (zero weights) reads the ninth.
template <int CIN, int NT, int RO, class PRE, class EPI>
__device__ __forceinline__ void fused_layer(const __half* __restrict__ in, const LayerWeights<CIN, NT>& lw,
                                            const TilePos& tp, PRE pre, EPI epi)
{
    constexpr int KC = LayerWeights<CIN, NT>::KC, PS = px_stride<CIN>();
    constexpr int RI = RO + 2, NPX = RO * RO, NMT = (NPX + 15) / 16, HALO = (RO - FT) / 2;
    // (opaque: one layer's addresses in registers at a time)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    auto tap_at = [](int tap) { return tap < 9 ? (tap / 3) * RI + tap % 3 : 2 * RI + 2; };
    for (int mt0 = wv; mt0 < NMT; mt0 += FU * FW) {
        const __half* at[FU];
        int m[FU];
        bool aval[FU], inside[FU];
        long long pix[FU];
        decltype(pre(true, 0ll, 0)) held[FU][NT];
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            m[u] = (mt0 + FW * u) * 16 + i;
            aval[u] = m[u] < NPX;
            const int mm = aval[u] ? m[u] : 0;
            at[u] = in + ((mm / RO) * RI + mm % RO) * PS + (CIN == 32 ? 8 * g : CIN == 16 ? 8 * (g & 1) : 0);
            const int gy = tp.Y0 - HALO + mm / RO, gx = tp.X0 - HALO + mm % RO;
            inside[u] = aval[u] && gy >= 0 && gy < tp.H && gx >= 0 && gx < tp.W;
            pix[u] = tp.fbase + (long long)gy * tp.W + gx;
#pragma unroll
            for (int n = 0; n < NT; ++n) held[u][n] = pre(inside[u], pix[u], n);
        }
        float4_t acc[FU][NT];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
            for (int u = 0; u < FU; ++u) {
                half8_t b;
                if constexpr (CIN == 4) {
                    // the chunk's two taps, 8 kc + 2 g and the next
                    const int t0 = 8 * kc + 2 * g, c0 = min(t0, 8), c1 = min(t0 + 1, 8);
                    const half4_t lo = *reinterpret_cast<const half4_t*>(at[u] + 4 * ((c0 / 3) * RI + c0 % 3));
                    const half4_t hi = *reinterpret_cast<const half4_t*>(at[u] + 4 * ((c1 / 3) * RI + c1 % 3));
                    b = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                } else if constexpr (CIN == 16) {
                    b = *reinterpret_cast<const half8_t*>(at[u] + PS * (g >> 1 ? tap_at(2 * kc + 1) : tap_at(2 * kc)));
                } else {
                    b = *reinterpret_cast<const half8_t*>(at[u] + PS * tap_at(kc));
                }
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[u][n] = mfma32(lw.w[kc][n], b, kc == 0 ? (float4_t){0.f, 0.f, 0.f, 0.f} : acc[u][n]);
            }
        }
        if constexpr (CIN == 32) {
            // the next chunks' reads in flight under the products
            __builtin_amdgcn_sched_group_barrier(0x100, FA * FU, 0);
#pragma unroll
            for (int kc = 0; kc < KC - FA; ++kc) {
                __builtin_amdgcn_sched_group_barrier(0x008, FU * NT, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, FU, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, FA * FU * NT, 0);
        }
#pragma unroll
        for (int u = 0; u < FU; ++u)
            if (aval[u])
#pragma unroll
                for (int n = 0; n < NT; ++n) epi(m[u], m[u] / RO, m[u] % RO, inside[u], pix[u], n, acc[u][n] + lw.b[n],
                        held[u][n]);
    }
}

// Whether position (oy, ox) of a region grown by HALO lies in the tile itself.
template <int HALO>
__device__ __forceinline__ bool in_tile(int oy, int ox)
{
    return (unsigned)(oy - HALO) < (unsigned)FT && (unsigned)(ox - HALO) < (unsigned)FT;
}

// What the network's output is for.
enum class CnnUse { OUTPUT, APPLY, TRAIN };

struct CnnForward {
    CnnWeights w;
    CnnBuffers b;
    int F, H, W;
    // OUTPUT: y [3][P], the corrections in sigma_h units
    float* y;
    // APPLY: slot k < 3 of a pixel with at most three points moves by sigma_h y_k
    DevState s;
    long long S;              // the state's slot stride
    float sigma_h;
    double tmax;
    // TRAIN: true depths [n_surf][P]
    const float* truth;
    int n_surf;
};

// A pixel's points and true depths as the last layer's results meet them.
constexpr int TRUTH_HELD = 4;
struct OutputInputs {
    int c;
    double t[3];
    float tr[TRUTH_HELD];
};

template <CnnUse USE>
__global__ __launch_bounds__(64 * FW, 2) void k_cnn_forward(CnnForward a)
{
    // buf0: the input features (FR0^2 x 16 channels), later layer 2's output
    // ((FT + 4)^2 x 32); buf1: layer 1's output ((FT + 6)^2 x 32), later layer 3's
    __shared__ __align__(16) __half buf0[(FT + 4) * (FT + 4) * px_stride<32>()];
    __shared__ __align__(16) __half buf1[(FT + 6) * (FT + 6) * px_stride<32>()];
    static_assert(FR0 * FR0 * px_stride<16>() <= (FT + 4) * (FT + 4) * px_stride<32>(), "the features fit buf0");
    const int tiles = a.F * ((a.W + FT - 1) / FT) * ((a.H + FT - 1) / FT);
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const long long P = (long long)a.F * a.H * a.W;
    float se = 0.f, num = 0.f;
    // (one tile per workgroup, or a stride of the grid over them in training,
    // where each workgroup leaves one pair of loss sums)
    for (int t = (int)xcd_block(blockIdx.x, gridDim.x); t < tiles; t += gridDim.x) {
        const TilePos tp(t, a.H, a.W);
        if (t >= (int)gridDim.x) __syncthreads();
        for (int v = threadIdx.x; v < FR0 * FR0 * 2; v += blockDim.x) {
            const int p = v >> 1, q = v & 1;
            const int gy = tp.Y0 - 4 + p / FR0, gx = tp.X0 - 4 + p % FR0;
            uint4 val = make_uint4(0, 0, 0, 0);
            if (gy >= 0 && gy < a.H && gx >= 0 && gx < a.W)
                val = reinterpret_cast<const uint4*>(a.b.act[0] + (tp.fbase + (long long)gy * a.W + gx) * 16)[q];
            *reinterpret_cast<uint4*>(buf0 + p * px_stride<16>() + 8 * q) = val;
        }
        __syncthreads();
        auto none = [](bool, long long, int) { return 0; };
        // a hidden layer: bias, ReLU, zero outside the image; into LDS and, in
        // training, the tile's own part to memory
        auto hidden = [&](auto halo, __half* out, __half* act) {
            return [=](int m, int oy, int ox, bool inside, long long pix, int n, float4_t v, int) {
                float4_t r;
#pragma unroll
                for (int c = 0; c < 4; ++c) r[c] = inside ? fmaxf(v[c], 0.f) : 0.f;
                const half4_t h = to_half4(r);
                const int ch = n * 16 + 4 * g;
                *reinterpret_cast<half4_t*>(out + m * px_stride<32>() + ch) = h;
                if (USE == CnnUse::TRAIN && inside && in_tile<decltype(halo)::value>(oy, ox))
                    *reinterpret_cast<half4_t*>(act + pix * 32 + ch) = h;
            };
        };
        const LayerWeights<16, 2> w0(a.w.wt[0], a.w.bias[0]);
        fused_layer<16, 2, FT + 6>(buf0, w0, tp, none,
                                   hidden(std::integral_constant<int, 3>(), buf1, a.b.act[1]));
        __syncthreads();
        const LayerWeights<32, 2> w1(a.w.wt[1], a.w.bias[1]);
        fused_layer<32, 2, FT + 4>(buf1, w1, tp, none,
                                   hidden(std::integral_constant<int, 2>(), buf0, a.b.act[2]));
        __syncthreads();
        const LayerWeights<32, 2> w2(a.w.wt[2], a.w.bias[2]);
        fused_layer<32, 2, FT + 2>(buf0, w2, tp, none,
                                   hidden(std::integral_constant<int, 1>(), buf1, a.b.act[3]));
        __syncthreads();
        const LayerWeights<32, 1> w3(a.w.wt[3], a.w.bias[3]);
        // what the output is used on, loaded ahead of the layer's products
        auto inputs = [&](bool inside, long long pix, int) {
            OutputInputs in{};
            if (USE == CnnUse::OUTPUT || !inside || g != 0) return in;
            in.c = load_cnt(a.s.cnt, pix);
#pragma unroll
            for (int k = 0; k < 3; ++k) in.t[k] = a.s.t[k * a.S + pix];
            if (USE == CnnUse::TRAIN) {
                in.c = min(in.c, 3);
#pragma unroll
                for (int q = 0; q < TRUTH_HELD; ++q)
                    if (q < a.n_surf) in.tr[q] = a.truth[(long long)q * P + pix];
            }
            return in;
        };
        fused_layer<32, 1, FT>(buf1, w3, tp, inputs,
                               [&](int, int, int, bool inside, long long pix, int, float4_t v, const OutputInputs& in) {
            if (!inside || g != 0) return;                 // channels 0 .. 3: slots 0 .. 2
            const half4_t y = to_half4(v);
            if (USE == CnnUse::OUTPUT) {
#pragma unroll
                for (int k = 0; k < 3; ++k) a.y[k * P + pix] = (float)y[k];
            } else if (USE == CnnUse::APPLY) {
                if (in.c > 3) return;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (k < in.c) {
                        double t = in.t[k] + (double)(a.sigma_h * (float)y[k]);
                        t = t < 0.0 ? 0.0 : (t > a.tmax ? a.tmax : t);
                        a.s.t[k * a.S + pix] = t;
                    }
            } else {
                // targets: slot k < min(cnt, 3) takes the nearest true depth of
                // its pixel within 3 sigma_h (first surface on ties; NaN:
                // absent); the loss is the masked squared error, dY its gradient
                // 2 (y - y*) of the sum (1/count is applied to the weight gradients)
                half4_t dy = {};
                double bd[3] = {0.0, 0.0, 0.0};
                float bt[3] = {0.f, 0.f, 0.f};
                bool any[3] = {false, false, false};
                for (int q = 0; q < a.n_surf; ++q) {
                    const float tr = q < TRUTH_HELD ? (q == 0 ? in.tr[0] : q == 1 ? in.tr[1] : q == 2 ? in.tr[2] : in.tr[3])
                                                    : a.truth[(long long)q * P + pix];
                    if (!(tr == tr)) continue;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const double d = fabs((double)tr - in.t[k]);
                        if (!any[k] || d < bd[k]) {
                            any[k] = true;
                            bt[k] = tr;
                            bd[k] = d;
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (k < in.c && any[k] && bd[k] <= 3.0 * (double)a.sigma_h) {
                        const float ty =
                            fminf(fmaxf((float)(((double)bt[k] - in.t[k]) / (double)a.sigma_h), -8.f), 8.f);
                        const float d = (float)y[k] - ty;
                        se += d * d;
                        num += 1.f;
                        dy[k] = (_Float16)(2.f * d);
                    }
                *reinterpret_cast<half4_t*>(a.b.dy4 + pix * 4) = dy;
            }
        });
    }
    if (USE == CnnUse::TRAIN) {
        // the workgroup's sums, in a fixed order (lanes past i hold zeros)
        __shared__ float red[2][FW * 16];
        static_assert(FW * 16 == 64, "a value per lane of the first wavefront");
        if (g == 0) {
            red[0][(threadIdx.x >> 6) * 16 + i] = se;
            red[1][(threadIdx.x >> 6) * 16 + i] = num;
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            float s0 = red[0][threadIdx.x], s1 = red[1][threadIdx.x];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                s0 += __shfl_xor(s0, d, 64);
                s1 += __shfl_xor(s1, d, 64);
            }
            if (threadIdx.x == 0) {
                a.b.lpart[2 * blockIdx.x] = s0;
                a.b.lpart[2 * blockIdx.x + 1] = s1;
            }
        }
    }
}

// Backward data of layers 3, 2 and 1 on a tile: the output gradient (dy4)
// staged with a 3-pixel halo, each layer's result gated by the ReLU of its
// input's activation, kept in LDS for the next layer and written to memory
// (the tile's own part) for the weight gradients.
struct CnnBackward {
    CnnWeights w;
    CnnBuffers b;
    int F, H, W;
};

__global__ __launch_bounds__(64 * FW, 2) void k_cnn_backward(CnnBackward a)
{
    __shared__ __align__(16) __half dyb[(FT + 6) * (FT + 6) * 4];
    __shared__ __align__(16) __half d3[(FT + 4) * (FT + 4) * px_stride<32>()];
    __shared__ __align__(16) __half d2[(FT + 2) * (FT + 2) * px_stride<32>()];
    const int g = (threadIdx.x & 63) >> 4;
    const TilePos tp((int)xcd_block(blockIdx.x, gridDim.x), a.H, a.W);
    const LayerWeights<4, 2> w3(a.w.wb[3], nullptr);
    for (int p = threadIdx.x; p < (FT + 6) * (FT + 6); p += blockDim.x) {
        const int gy = tp.Y0 - 3 + p / (FT + 6), gx = tp.X0 - 3 + p % (FT + 6);
        half4_t v = {};
        if (gy >= 0 && gy < a.H && gx >= 0 && gx < a.W)
            v = *reinterpret_cast<const half4_t*>(a.b.dy4 + (tp.fbase + (long long)gy * a.W + gx) * 4);
        *reinterpret_cast<half4_t*>(dyb + 4 * p) = v;
    }
    __syncthreads();
    // the four activations a lane's results are gated by
    auto gate = [&](const __half* act) {
        return [=](bool inside, long long pix, int n) {
            half4_t v = {};
            if (inside) v = *reinterpret_cast<const half4_t*>(act + pix * 32 + n * 16 + 4 * g);
            return v;
        };
    };
    auto result = [&](auto halo, __half* lds, __half* mem) {
        return [=](int m, int oy, int ox, bool inside, long long pix, int n, float4_t v, half4_t act) {
            float4_t r;
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = (float)act[c] > 0.f ? v[c] : 0.f;     // (zero outside the image)
            const half4_t h = to_half4(r);
            const int ch = n * 16 + 4 * g;
            if (lds) *reinterpret_cast<half4_t*>(lds + m * px_stride<32>() + ch) = h;
            if (inside && in_tile<decltype(halo)::value>(oy, ox)) *reinterpret_cast<half4_t*>(mem + pix * 32 + ch) = h;
        };
    };
    fused_layer<4, 2, FT + 4>(dyb, w3, tp, gate(a.b.act[3]),
                              result(std::integral_constant<int, 2>(), d3, a.b.dact[3]));
    __syncthreads();
    const LayerWeights<32, 2> w2(a.w.wb[2], nullptr);
    fused_layer<32, 2, FT + 2>(d3, w2, tp, gate(a.b.act[2]),
                               result(std::integral_constant<int, 1>(), d2, a.b.dact[2]));
    __syncthreads();
    const LayerWeights<32, 2> w1(a.w.wb[1], nullptr);
    fused_layer<32, 2, FT>(d2, w1, tp, gate(a.b.act[1]),
                           result(std::integral_constant<int, 0>(), (__half*)nullptr, a.b.dact[1]));
}

// ---------------------------------------------------------------------------
// Weight gradients of all four layers (blockIdx.y) in one launch.  A workgroup
// takes units of WG_ROWS image rows x 64 columns, strided by the grid, and
// accumulates dW in registers over all of them: rows (tap, ci), columns co, K
// = pixels.  Both operands lie in LDS as [pixel][channel]; the transposed LDS
// read (ds_read_b64_tr_b16: 16 lanes read a 4 x 16 block of halves and each
// gets a column of four) hands every lane the pixels of its channel.  Input
// rows live in a ring of four, so each is loaded once per unit, the next row's
// loads in flight during two rows' products.  The bias gradient is a product
// with ones.  131 k pixels: 26 us for the four layers (162 us with the operands
// gathered from LDS two bytes at a time, a launch per layer).
constexpr int WG_ROWS = 8;
constexpr int WG_COLS = 64;
constexpr int WG_WAVES = 6;
constexpr int WG_GROUPS = 256;     // workgroups per layer (one per CU): partial sums kept

typedef short short4_t __attribute__((__vector_size__(4 * sizeof(short))));
typedef __attribute__((address_space(3))) short4_t lds_short4;

// Rows p .. p + 7 of LDS [pixel][C] (C halves per pixel, this lane's group of
// four lanes at pixel p + (i >> 2)), channels 16 cb .. 16 cb + 15: lane i of
// the group gets channel 16 cb + i of the eight pixels.
template <int C>
__device__ __forceinline__ int tr_at(int px, int cb, int i)
{
    // (32 channels: the two 32-byte halves of a pixel swap places every four
    // pixels, so that the 16 rows a wavefront reads cover all banks)
    return C == 32 ? px * 32 + 16 * (cb ^ ((px >> 2) & 1)) + 4 * (i & 3) : px * 16 + 4 * (i & 3);
}

template <int C>
__device__ __forceinline__ half8_t tr_read8(const __half* base, int p, int cb, int i)
{
    union {
        short4_t s[2];
        half8_t h;
    } v;
    const int px = p + (i >> 2);
    v.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(base + tr_at<C>(px, cb, i)));
    v.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(base + tr_at<C>(px + 4, cb, i)));
    return v.h;
}

// Offset of 16-byte chunk q of pixel px in the same layout.
template <int C>
__device__ __forceinline__ int row_chunk(int px, int q)
{
    return C == 32 ? px * 32 + 16 * ((q >> 1) ^ ((px >> 2) & 1)) + 8 * (q & 1) : px * 16 + 8 * q;
}

// CIN channels of X; the output gradient has GC stored channels (32, or 4 that
// stand for 16).
template <int CIN, int GC>
__device__ __forceinline__ void wgrad_layer(const __half* __restrict__ X, const __half* __restrict__ dY,
                                            float* __restrict__ part, float* __restrict__ bpart, int F, int H, int W,
                                            __half* xs, __half* ds)
{
    constexpr int CO = GC == 4 ? 16 : 32, NT = CO / 16, CB = CIN / 16;
    constexpr int TILES = 9 * CB * NT, TPW = (TILES + WG_WAVES - 1) / WG_WAVES;
    constexpr int XR = (WG_COLS + 2) * CIN, DR = WG_COLS * CO;      // halves of a row of X, of dY
    constexpr int XV = (WG_COLS + 2) * CIN / 8;                     // 16-byte chunks of a row of X
    static_assert(XV <= 64 * WG_WAVES && WG_COLS * CO / 8 <= 64 * WG_WAVES, "one chunk per thread");
    static_assert(TILES % WG_WAVES == 0, "whole tiles per wavefront");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, i = lane & 15, g = lane >> 4;
    const int segs = (W + WG_COLS - 1) / WG_COLS, rblocks = (H + WG_ROWS - 1) / WG_ROWS, units = F * rblocks * segs;
    float4_t acc[TPW], accb[NT];
#pragma unroll
    for (int t = 0; t < TPW; ++t) acc[t] = (float4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < NT; ++n) accb[n] = (float4_t){0.f, 0.f, 0.f, 0.f};
    half8_t ones;
#pragma unroll
    for (int q = 0; q < 8; ++q) ones[q] = (_Float16)1.f;
    for (int unit = blockIdx.x; unit < units; unit += gridDim.x) {
        const int x0 = (unit % segs) * WG_COLS, y0 = (unit / segs % rblocks) * WG_ROWS, f = unit / (segs * rblocks);
        const int y1 = min(y0 + WG_ROWS, H);
        const long long fbase = (long long)f * H * W;
        auto load_x = [&](int y) {
            uint4 v = make_uint4(0, 0, 0, 0);
            const int px = tid / (CIN / 8), x = x0 + px - 1;
            if (tid < XV && y >= 0 && y < H && x >= 0 && x < W)
                v = reinterpret_cast<const uint4*>(X + (fbase + (long long)y * W + x) * CIN)[tid % (CIN / 8)];
            return v;
        };
        auto store_x = [&](int y, uint4 v) {
            if (tid < XV)
                *reinterpret_cast<uint4*>(xs + ((y + 1) & 3) * XR + row_chunk<CIN>(tid / (CIN / 8), tid % (CIN / 8))) = v;
        };
        auto load_d = [&](int y) {
            uint4 v = make_uint4(0, 0, 0, 0);
            const int px = tid / (CO / 8), q = tid % (CO / 8), x = x0 + px;
            if (tid < WG_COLS * CO / 8 && y < y1 && x < W) {
                const __half* p = dY + (fbase + (long long)y * W + x) * GC;
                if constexpr (GC == 4) {
                    if (q == 0) {
                        const uint2 w = *reinterpret_cast<const uint2*>(p);
                        v = make_uint4(w.x, w.y, 0, 0);
                    }
                } else {
                    v = reinterpret_cast<const uint4*>(p)[q];
                }
            }
            return v;
        };
        auto store_d = [&](int y, uint4 v) {
            if (tid < WG_COLS * CO / 8)
                *reinterpret_cast<uint4*>(ds + (y & 1) * DR + row_chunk<CO>(tid / (CO / 8), tid % (CO / 8))) = v;
        };
        uint4 nx, nd;            // rows y + 2 of X and y + 1 of dY, in flight for two rows' products
        {
            const uint4 a = load_x(y0 - 1), b = load_x(y0), c = load_x(y0 + 1), d = load_d(y0);
            nx = load_x(y0 + 2);
            nd = load_d(y0 + 1);
            store_x(y0 - 1, a);
            store_x(y0, b);
            store_x(y0 + 1, c);
            store_d(y0, d);
        }
        __syncthreads();
        for (int y = y0; y < y1; ++y) {
            const uint4 fx = load_x(y + 3), fd = load_d(y + 2);     // (past the unit: not read)
            const __half* dr = ds + (y & 1) * DR;
#pragma unroll
            for (int s = 0; s < WG_COLS / 32; ++s) {
                const int p0 = 32 * s + 8 * g;
                half8_t b[NT];
#pragma unroll
                for (int n = 0; n < NT; ++n) b[n] = tr_read8<CO>(dr, p0, n, i);
                half8_t a = {};
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    const int tile = wv * TPW + t, mt = tile / NT, nt = tile % NT;
                    const int tap = mt / CB, cb = mt % CB, ky = tap / 3, kx = tap % 3;
                    if (t == 0 || nt == 0) a = tr_read8<CIN>(xs + ((y + ky) & 3) * XR, p0 + kx, cb, i);
                    acc[t] = mfma32(a, NT == 1 || nt == 0 ? b[0] : b[NT - 1], acc[t]);
                }
                if (wv == 0)
#pragma unroll
                    for (int n = 0; n < NT; ++n) accb[n] = mfma32(ones, b[n], accb[n]);
            }
            store_x(y + 2, nx);
            store_d(y + 1, nd);
            nx = fx;
            nd = fd;
            __syncthreads();
        }
    }
    float* out = part + (size_t)blockIdx.x * CNN_PART;
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int tile = wv * TPW + t, mt = tile / NT, nt = tile % NT;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(mt * 16 + 4 * g + r) * CO + nt * 16 + i] = acc[t][r];
    }
    if (wv == 0 && g == 0)
#pragma unroll
        for (int n = 0; n < NT; ++n) bpart[(size_t)blockIdx.x * CNN_PART + n * 16 + i] = accb[n][0];
}

__global__ __launch_bounds__(64 * WG_WAVES) void k_cnn_wgrad(CnnBackward a)
{
    __shared__ __align__(16) __half xs[4 * (WG_COLS + 2) * 32];
    __shared__ __align__(16) __half ds[2 * WG_COLS * 32];
    float* part = a.b.part;
    switch (blockIdx.y) {
    case 0:
        wgrad_layer<16, 32>(a.b.act[0], a.b.dact[1], part + CNN_POFF[0], part + CNN_PBIAS[0], a.F, a.H, a.W, xs, ds);
        break;
    case 1:
        wgrad_layer<32, 32>(a.b.act[1], a.b.dact[2], part + CNN_POFF[1], part + CNN_PBIAS[1], a.F, a.H, a.W, xs, ds);
        break;
    case 2:
        wgrad_layer<32, 32>(a.b.act[2], a.b.dact[3], part + CNN_POFF[2], part + CNN_PBIAS[2], a.F, a.H, a.W, xs, ds);
        break;
    default:
        wgrad_layer<32, 4>(a.b.act[3], a.b.dy4, part + CNN_POFF[3], part + CNN_PBIAS[3], a.F, a.H, a.W, xs, ds);
        break;
    }
}

// The gradient from the partial sums (ng of them), scaled by 1/count, Adam and
// the FP16 layouts, a thread per parameter and sixteen slices of the partials
// each, added in a fixed order; the loss (sums of nl pairs) from workgroup 0.
// 10 us for 28 MB of partials (4 x 76 us as one thread per parameter over all
// of them, a launch per layer, and 36 us for the loss on one lane).
constexpr int UPD_PARAMS = 64, UPD_SLICES = 16;

__global__ __launch_bounds__(UPD_PARAMS * UPD_SLICES) void k_cnn_update(CnnWeights W, CnnBuffers b, int ng, int nl,
                                                                        CnnAdam opt, float c1, float c2, float* loss)
{
    __shared__ double lsum[2][UPD_SLICES];
    __shared__ float red[UPD_SLICES][UPD_PARAMS];
    const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
    // loss sums (of whole numbers below 2^31, and of squared errors): slice by slice
    {
        double se = 0.0, n = 0.0;
        for (int k = slice * 64 + lane; k < nl; k += UPD_SLICES * 64) {
            se += b.lpart[2 * k];
            n += b.lpart[2 * k + 1];
        }
        se = wave_sum(se);
        n = wave_sum(n);
        if (lane == 0) {
            lsum[0][slice] = se;
            lsum[1][slice] = n;
        }
    }
    const int idx = blockIdx.x * UPD_PARAMS + lane;
    float s = 0.f;
    if (idx < CNN_PARAMS) {
        int l = 0;
#pragma unroll
        for (int k = 1; k < CNN_LAYERS; ++k) l = idx >= CNN_OFF[k] ? k : l;
        const int p = idx - (l == 0 ? CNN_OFF[0] : l == 1 ? CNN_OFF[1] : l == 2 ? CNN_OFF[2] : CNN_OFF[3]);
        const int nw = l == 0 ? 9 * 16 * 32 : l == 3 ? 9 * 32 * 3 : 9 * 32 * 32;
        const int po = l == 0 ? CNN_POFF[0] : l == 1 ? CNN_POFF[1] : l == 2 ? CNN_POFF[2] : CNN_POFF[3];
        const int pb = l == 0 ? CNN_PBIAS[0] : l == 1 ? CNN_PBIAS[1] : l == 2 ? CNN_PBIAS[2] : CNN_PBIAS[3];
        const int at = p >= nw ? pb + p - nw : l == 3 ? po + (p / 3) * 16 + p % 3 : po + p;
        const int per = (ng + UPD_SLICES - 1) / UPD_SLICES, g0 = slice * per, g1 = min(g0 + per, ng);
        const float* src = b.part + at;
        int k = g0;
        for (; k + 8 <= g1; k += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(k + u) * CNN_PART];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; k < g1; ++k) s += src[(size_t)k * CNN_PART];
    }
    red[slice][lane] = s;
    __syncthreads();
    if (slice != 0) return;
    double se = 0.0, n = 0.0;
#pragma unroll
    for (int k = 0; k < UPD_SLICES; ++k) {
        se += lsum[0][k];
        n += lsum[1][k];
    }
    if (blockIdx.x == 0 && lane == 0) {
        loss[0] = (float)(se / (n > 1.0 ? n : 1.0));
        loss[1] = (float)n;
    }
    if (idx >= CNN_PARAMS) return;
    s = 0.f;
#pragma unroll
    for (int k = 0; k < UPD_SLICES; ++k) s += red[k][lane];
    const float gi = s * (1.f / fmaxf((float)n, 1.f));
    b.grad[idx] = gi;
    store_weight(W, idx, adam_step(W.master, W.m, W.v, idx, gi, opt, c1, c2));
}

// ---------------------------------------------------------------------------
// launchers

static unsigned tiles_of_frames(const Shape& sh, int t)
{
    return (unsigned)(sh.F * ((sh.rows + t - 1) / t) * ((sh.cols + t - 1) / t));
}

// Units of the weight gradient (a workspace admits shapes of at most as many
// as it was sized for); WG_GROUPS workgroups at most share them.
unsigned cnn_wgrad_groups(const Shape& sh)
{
    return (unsigned)(sh.F * ((sh.rows + WG_ROWS - 1) / WG_ROWS) * ((sh.cols + WG_COLS - 1) / WG_COLS));
}

unsigned cnn_wgrad_partials(unsigned groups) { return groups < (unsigned)WG_GROUPS ? groups : (unsigned)WG_GROUPS; }

hipError_t launch_cnn_prepare(const CnnWeights& w, hipStream_t st)
{
    hipLaunchKernelGGL(k_cnn_prepare, dim3((CNN_PARAMS + 255) / 256), dim3(256), 0, st, w);
    return hipGetLastError();
}

static void launch_pack(const Shape& sh, DevState s, float sigma_h, const CnnBuffers& b, hipStream_t st)
{
    hipLaunchKernelGGL(k_cnn_pack, dim3(tiles_of_frames(sh, PKT)), dim3(PK_THREADS), 0, st, sh, s, sigma_h, b.act[0]);
}

hipError_t launch_cnn_output(const Shape& sh, DevState s, float sigma_h, const CnnWeights& w, const CnnBuffers& b,
                             float* y, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    launch_pack(sh, s, sigma_h, b, st);
    CnnForward a{};
    a.w = w;
    a.b = b;
    a.F = sh.F;
    a.H = sh.rows;
    a.W = sh.cols;
    a.y = y;
    hipLaunchKernelGGL(k_cnn_forward<CnnUse::OUTPUT>, dim3(tiles_of_frames(sh, FT)), dim3(64 * FW), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_cnn_apply(const Shape& sh, DevState s, float sigma_h, const CnnWeights& w, const CnnBuffers& b,
                            double tmax, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    launch_pack(sh, s, sigma_h, b, st);
    CnnForward a{};
    a.w = w;
    a.b = b;
    a.F = sh.F;
    a.H = sh.rows;
    a.W = sh.cols;
    a.s = s;
    a.S = sh.S;
    a.sigma_h = sigma_h;
    a.tmax = tmax;
    hipLaunchKernelGGL(k_cnn_forward<CnnUse::APPLY>, dim3(tiles_of_frames(sh, FT)), dim3(64 * FW), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_cnn_train_step(const Shape& sh, DevState s, float sigma_h, const float* truth, int S,
                                 CnnWeights& w, const CnnBuffers& b, const CnnAdam& opt, float* loss,
                                 hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    launch_pack(sh, s, sigma_h, b, st);
    CnnForward a{};
    a.w = w;
    a.b = b;
    a.F = sh.F;
    a.H = sh.rows;
    a.W = sh.cols;
    a.s = s;
    a.S = sh.S;
    a.sigma_h = sigma_h;
    a.truth = truth;
    a.n_surf = S;
    const unsigned ft = tiles_of_frames(sh, FT);
    const unsigned nl = ft < CNN_LOSS_PARTS ? ft : CNN_LOSS_PARTS;
    hipLaunchKernelGGL(k_cnn_forward<CnnUse::TRAIN>, dim3(nl), dim3(64 * FW), 0, st, a);
    const CnnBackward c{w, b, sh.F, sh.rows, sh.cols};
    hipLaunchKernelGGL(k_cnn_backward, dim3(ft), dim3(64 * FW), 0, st, c);
    const unsigned ng = cnn_wgrad_partials(cnn_wgrad_groups(sh));
    hipLaunchKernelGGL(k_cnn_wgrad, dim3(ng, CNN_LAYERS), dim3(64 * WG_WAVES), 0, st, c);
    ++w.step;
    const float c1 = 1.f - powf(opt.beta1, (float)w.step), c2 = 1.f - powf(opt.beta2, (float)w.step);
    hipLaunchKernelGGL(k_cnn_update, dim3((CNN_PARAMS + UPD_PARAMS - 1) / UPD_PARAMS), dim3(UPD_PARAMS * UPD_SLICES),
                       0, st, w, b, (int)ng, (int)nl, opt, c1, c2, loss);
    return hipGetLastError();
}

}  // namespace rt3d
