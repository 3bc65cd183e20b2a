// k_steps.hip -- the likelihood gradient steps on depth, intensity and
// background (Results, "Reconstruction algorithm": each block update is a
// gradient step on the Poisson negative log-likelihood of the "Observation
// model"), and the raw gradients.
//
// For pixel p with active entries (t, z), points (t_n, r_n), background b and
// gain g, lambda_t = g (sum_n r_n h(t - t_n) + b) and
//   dNLL/dt_n = g r_n [S'(t_n) + sum z h'(t - t_n) / lambda_t]
//   dNLL/dr_n = g     [S(t_n)  - sum z h(t - t_n) / lambda_t]
//   dNLL/db   = g     [T       - sum z / lambda_t]
// Steps (readings of the unstated step sizes):
//   depth:      t_n -= (beta_t / I_h) [S' + sum z h'/lambda], clipped to dmax,
//               clamped to [0, T-1]; I_h is the shift Fisher information of
//               one photon, so g r I_h is the expected curvature (PALM-style
//               1/Lipschitz scaling, damped by beta_t);
//   intensity:  r_n <- max(0, r_n [(1-beta_r) + beta_r sum z h/(lambda S)]);
//   background: b <- max(b_min, b [(1-beta_b) + beta_b sum z/(lambda T)]).
// Within a pixel every point uses lambda from before the step (Jacobi).
//
// Mapping: LPP (4 or 8) lanes per pixel share its active entries (cost linear in
// active bins, as in the paper's Methods; consecutive lanes read consecutive
// entries) and combine their partial sums with wavefront shuffles; every lane
// keeps the pixel's <= 4 points in registers.  Depth is held in FP64 state and
// evaluated in FP32 around an integer anchor, so the IRF lookup error stays
// at FP32 rounding of the local offset whatever T is.
#include "rt3d_steps.h"

namespace rt3d {

// Seven workgroups per CU (at most 72 VGPRs; the few values the compiler then
// keeps in scratch are written before the entry loop and read after it).
template <int LPP, bool TLDS>
__global__ __launch_bounds__(256, 7) void k_depth_step(DevModel m, DevParams p, Shape sh,
                                                    const uint32_t* __restrict__ off,
                                                    const uint32_t* __restrict__ ent,
                                                    const float* __restrict__ gain, DevState s)
{
    __shared__ uint32_t stage[step_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    const long long P = sh.P;
    const Lane L = lane_setup<LPP>(m, s, P, off, gain, true);    // its loads stay in flight across the staging
    const float4* cr = stage_segments<TLDS>(m, crl, stl);
    uint32_t* seg = stage_segment<LPP>(stage);
    float sz, shh[KM], shp[KM];
    accumulate<LPP>(m, cr, L.q, L.live ? s.b[L.pix] : 1.f, L.live ? L.G : 1.f, ent, L.etot, L.e0, L.e1, L.sub, seg, sz, shh, shp);
    reduce_lanes<LPP>(sz, shh, shp);
    // S' after the entries: nothing of it stays live across the entry loop
    float Sv[KM], Spv[KM];
    s_eval_points<LPP>(m, L.q, L.sub, stl, Sv, Spv);
    if (!L.live || L.sub != 0) return;
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (k < L.q.c && L.q.r[k] > 0.f) s.t[k * P + L.pix] = depth_next(m, p, L.q.t[k], Spv[k], shp[k]);
}

// MERGE: the in-pixel merge runs first (the loop's order: merge, then the
// intensity step on the merged points).
template <int LPP, bool MERGE, bool TLDS>
__global__ __launch_bounds__(256, 7) void k_intensity_step(DevModel m, DevParams p, Shape sh,
                                                        const uint32_t* __restrict__ off,
                                                        const uint32_t* __restrict__ ent,
                                                        const float* __restrict__ gain, DevState s)
{
    __shared__ uint32_t stage[step_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    const long long P = sh.P;
    Lane L = lane_setup<LPP>(m, s, P, off, gain, true);          // its loads stay in flight across the staging
    const float4* cr = stage_segments<TLDS>(m, crl, stl);
    uint32_t* seg = stage_segment<LPP>(stage);
    if (MERGE && L.member) merge_lane(s, P, p, L.pix, L.sub, L.q);
    float sz, shh[KM], shp[KM];
    accumulate<LPP>(m, cr, L.q, L.live ? s.b[L.pix] : 1.f, L.live ? L.G : 1.f, ent, L.etot, L.e0, L.e1, L.sub, seg, sz, shh, shp);
    reduce_lanes<LPP>(sz, shh, shp);
    float Sv[KM], Spv[KM];
    s_eval_points<LPP>(m, L.q, L.sub, stl, Sv, Spv);
    if (!L.live || L.sub != 0) return;
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (k < L.q.c && Sv[k] > 0.f) s.r[k * P + L.pix] = intensity_next(p, L.q.r[k], Sv[k], shh[k]);
}

// The background step writes the new b to bdst (the state's own b, or a
// second buffer the background filter reads); dead pixels keep their b.
template <int LPP, bool TLDS>
__global__ __launch_bounds__(256) void k_bg_step(DevModel m, DevParams p, Shape sh,
                                                 const uint32_t* __restrict__ off,
                                                 const uint32_t* __restrict__ ent,
                                                 const float* __restrict__ gain, DevState s, float* bdst)
{
    __shared__ uint32_t stage[step_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    const long long P = sh.P;
    const Lane L = lane_setup<LPP>(m, s, P, off, gain, false);   // its loads stay in flight across the staging
    const float4* cr = stage_segments<TLDS, false>(m, crl, stl);
    uint32_t* seg = stage_segment<LPP>(stage);
    const float braw = L.pix < P ? s.b[L.pix] : 1.f;
    const float bb = L.live ? braw : 1.f;
    float sz, shh[KM], shp[KM];
    accumulate<LPP>(m, cr, L.q, bb, L.live ? L.G : 1.f, ent, L.etot, L.e0, L.e1, L.sub, seg, sz, shh, shp);
    reduce_lanes<LPP>(sz, shh, shp);
    if (!L.member || L.sub != 0) return;
    if (!L.live) {
        bdst[L.pix] = braw;
        return;
    }
    bdst[L.pix] = background_next(m, p, bb, sz);
}

template <int LPP, bool TLDS>
__global__ __launch_bounds__(256) void k_gradients(DevModel m, Shape sh, const uint32_t* __restrict__ off,
                                                   const uint32_t* __restrict__ ent,
                                                   const float* __restrict__ gain, DevState s,
                                                   float* __restrict__ gt, float* __restrict__ gr,
                                                   float* __restrict__ gb)
{
    __shared__ uint32_t stage[step_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    const long long P = sh.P;
    const Lane L = lane_setup<LPP>(m, s, P, off, gain, false);   // its loads stay in flight across the staging
    const float4* cr = stage_segments<TLDS>(m, crl, stl);
    uint32_t* seg = stage_segment<LPP>(stage);
    float sz, shh[KM], shp[KM];
    accumulate<LPP>(m, cr, L.q, L.live ? s.b[L.pix] : 1.f, L.live ? L.G : 1.f, ent, L.etot, L.e0, L.e1, L.sub, seg, sz, shh, shp);
    reduce_lanes<LPP>(sz, shh, shp);
    float Sv[KM], Spv[KM];
    s_eval_points<LPP>(m, L.q, L.sub, stl, Sv, Spv);
    if (!L.member || L.sub != 0) return;
    const float G = L.G;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        float vt = 0.f, vr = 0.f;
        if (k < L.q.c && G > 0.f) {
            vt = G * L.q.r[k] * (Spv[k] + shp[k]);
            vr = G * (Sv[k] - shh[k]);
        }
        gt[k * P + L.pix] = vt;
        gr[k * P + L.pix] = vr;
    }
    gb[L.pix] = G > 0.f ? G * ((float)m.T - sz) : 0.f;
}

static inline unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Per-class pixel lists (per-pixel IRFs).  meta[0 .. n] holds each class's
// first list position (meta[n] = P), meta[RT3D_MAX_IRFS + 1 + k] the class's
// cursor.  Each wavefront takes 64 consecutive pixels and appends the pixels
// of every class in ascending order (a ballot rank), so list chunks stay
// contiguous in memory; chunks follow in the order the wavefronts reach the
// cursor, which no per-pixel step depends on.
constexpr int CLASS_CUR = RT3D_MAX_IRFS + 1;

__device__ __forceinline__ int class_of(const uint8_t* cls, long long pix, long long P, int n)
{
    if (pix >= P) return -1;
    const int k = cls[pix];
    return k < n ? k : 0;
}

__global__ void k_class_zero(uint32_t* meta)
{
    if (threadIdx.x < CLASS_META) meta[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void k_class_count(const uint8_t* __restrict__ cls, long long P, int n,
                                                     uint32_t* meta)
{
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int k = class_of(cls, pix, P, n);
    for (int c = 0; c < n; ++c) {
        const unsigned long long mask = __ballot(k == c);
        if ((threadIdx.x & 63) == 0 && mask) atomicAdd(&meta[CLASS_CUR + c], (uint32_t)__popcll(mask));
    }
}

__global__ void k_class_base(int n, uint32_t* meta)
{
    if (threadIdx.x != 0) return;
    uint32_t acc = 0;
    for (int c = 0; c < n; ++c) {
        const uint32_t cnt = meta[CLASS_CUR + c];
        meta[c] = acc;
        meta[CLASS_CUR + c] = acc;
        acc += cnt;
    }
    meta[n] = acc;
}

__global__ __launch_bounds__(256) void k_class_scatter(const uint8_t* __restrict__ cls, long long P, int n,
                                                       uint32_t* meta, uint32_t* __restrict__ list)
{
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int k = class_of(cls, pix, P, n);
    const int lane = (int)(threadIdx.x & 63);
    const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
    for (int c = 0; c < n; ++c) {
        const unsigned long long mask = __ballot(k == c);
        if (!mask) continue;
        uint32_t b = 0;
        if (lane == 0) b = atomicAdd(&meta[CLASS_CUR + c], (uint32_t)__popcll(mask));
        b = (uint32_t)__shfl((int)b, 0, 64);
        if (k == c) list[b + (uint32_t)__popcll(mask & below)] = (uint32_t)pix;
    }
}

hipError_t launch_class_lists(const uint8_t* cls, long long P, int n, uint32_t* list, uint32_t* meta,
                              hipStream_t st)
{
    if (n < 1 || n > RT3D_MAX_IRFS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_class_zero, dim3(1), dim3(64), 0, st, meta);
    if (P > 0) hipLaunchKernelGGL(k_class_count, dim3(blocks_for(P, 256)), dim3(256), 0, st, cls, P, n, meta);
    hipLaunchKernelGGL(k_class_base, dim3(1), dim3(64), 0, st, n, meta);
    if (P > 0) hipLaunchKernelGGL(k_class_scatter, dim3(blocks_for(P, 256)), dim3(256), 0, st, cls, P, n, meta, list);
    return hipGetLastError();
}

// The kernels for lanes-per-pixel p.lpp (4 or 8) and the segment staging.
template <int LPP>
static hipError_t depth_step_lpp(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                                 const uint32_t* ent, const float* gain, DevState s, hipStream_t st)
{
    const dim3 g(blocks_for(sh.P * LPP, 256)), b(256);
    if (segments_fit(m)) hipLaunchKernelGGL((k_depth_step<LPP, true>), g, b, 0, st, m, p, sh, off, ent, gain, s);
    else hipLaunchKernelGGL((k_depth_step<LPP, false>), g, b, 0, st, m, p, sh, off, ent, gain, s);
    return hipGetLastError();
}

template <int LPP>
static hipError_t intensity_step_lpp(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                                     const uint32_t* ent, const float* gain, DevState s, bool merge, hipStream_t st)
{
    const dim3 g(blocks_for(sh.P * LPP, 256)), b(256);
    const bool tl = segments_fit(m);
    if (merge && tl) hipLaunchKernelGGL((k_intensity_step<LPP, true, true>), g, b, 0, st, m, p, sh, off, ent, gain, s);
    else if (merge) hipLaunchKernelGGL((k_intensity_step<LPP, true, false>), g, b, 0, st, m, p, sh, off, ent, gain, s);
    else if (tl) hipLaunchKernelGGL((k_intensity_step<LPP, false, true>), g, b, 0, st, m, p, sh, off, ent, gain, s);
    else hipLaunchKernelGGL((k_intensity_step<LPP, false, false>), g, b, 0, st, m, p, sh, off, ent, gain, s);
    return hipGetLastError();
}

template <int LPP>
static hipError_t bg_step_lpp(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                              const uint32_t* ent, const float* gain, DevState s, float* dst, hipStream_t st)
{
    const dim3 g(blocks_for(sh.P * LPP, 256)), b(256);
    if (segments_fit(m)) hipLaunchKernelGGL((k_bg_step<LPP, true>), g, b, 0, st, m, p, sh, off, ent, gain, s, dst);
    else hipLaunchKernelGGL((k_bg_step<LPP, false>), g, b, 0, st, m, p, sh, off, ent, gain, s, dst);
    return hipGetLastError();
}

hipError_t launch_depth_step(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                             const uint32_t* ent, const float* gain, DevState s, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    return p.lpp == 8 ? depth_step_lpp<8>(m, p, sh, off, ent, gain, s, st)
                      : depth_step_lpp<4>(m, p, sh, off, ent, gain, s, st);
}

hipError_t launch_intensity_step(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                                 const uint32_t* ent, const float* gain, DevState s, bool merge, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    return p.lpp == 8 ? intensity_step_lpp<8>(m, p, sh, off, ent, gain, s, merge, st)
                      : intensity_step_lpp<4>(m, p, sh, off, ent, gain, s, merge, st);
}

hipError_t launch_bg_step(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                          const uint32_t* ent, const float* gain, DevState s, float* bdst, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    float* dst = bdst ? bdst : s.b;
    return p.lpp == 8 ? bg_step_lpp<8>(m, p, sh, off, ent, gain, s, dst, st)
                      : bg_step_lpp<4>(m, p, sh, off, ent, gain, s, dst, st);
}

hipError_t launch_gradients(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                            const uint32_t* ent, const float* gain, DevState s, float* gt, float* gr, float* gb,
                            hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    const bool tl = segments_fit(m);
    if (p.lpp == 8) {
        const dim3 g(blocks_for(sh.P * 8, 256)), b(256);
        if (tl) hipLaunchKernelGGL((k_gradients<8, true>), g, b, 0, st, m, sh, off, ent, gain, s, gt, gr, gb);
        else hipLaunchKernelGGL((k_gradients<8, false>), g, b, 0, st, m, sh, off, ent, gain, s, gt, gr, gb);
    } else {
        const dim3 g(blocks_for(sh.P * 4, 256)), b(256);
        if (tl) hipLaunchKernelGGL((k_gradients<4, true>), g, b, 0, st, m, sh, off, ent, gain, s, gt, gr, gb);
        else hipLaunchKernelGGL((k_gradients<4, false>), g, b, 0, st, m, sh, off, ent, gain, s, gt, gr, gb);
    }
    return hipGetLastError();
}

}  // namespace rt3d
