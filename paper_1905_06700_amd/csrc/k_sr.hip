// k_sr.hip -- the super-resolved data term (Results, dynamic scenes, and
// Discussion: the map f may undersample).  The point cloud lives on a grid s
// times finer than the lidar pixels; the s x s point-grid pixels
// (i s + u, j s + v) all map to lidar pixel (i, j), whose Poisson intensity
// adds their points:
//   lambda_{p,t} = g_p (sum_{q -> p} sum_{n in q} r_n h(t - t_n) + b_p).
// Gain and background stay per lidar pixel.  Each point's gradient is that of
// the plain model with its lidar pixel's lambda:
//   dNLL/dt_n = g r_n [S'(t_n) + sum z h'(t - t_n)/lambda]
//   dNLL/dr_n = g     [S(t_n)  - sum z h(t - t_n)/lambda]
//   dNLL/db_p = g     [T       - sum z/lambda]
// and the steps are those of k_steps.hip (depth_next, intensity_next,
// background_next), Jacobi over the whole block.
//
// State: point arrays (t, r, n, cnt) on the point grid with slot stride Pf;
// the lidar pixels' background in b[0 .. P - 1] of the same state.
//
// Mapping: sixteen lanes per lidar pixel, four lidar pixels per wavefront.
// Lane u holds the points of the block's point-grid pixel u in registers
// (s <= 4, so s^2 <= 16 lanes); the block's points are also staged in LDS.
// The pixel's entries go through 16 at a time, one per lane: a lane
// evaluates lambda of its entry over the staged points and, when the entry lies
// in some point's support, leaves z/(g lambda) and the bin in LDS; then every
// lane adds the batch's z h'/lambda and z h/lambda to each of its points.  The
// background's sum z/lambda is a sum over the sixteen lanes.
// A frame's lidar pixels fill two wavefronts per SIMD, so the time is the chain
// of reads: segments and the cubic's table in LDS, several points' (entries')
// segments read at once, the next batch of entries on its way.  8 frames of
// 32 x 32 lidar pixels, 3 x 3 point-grid pixels each: 12.3 us the depth step, 11.1
// the intensity step (the merge in it), 6.3 the background step, against 15, 15
// and 10 us and 5 us of merge with the segments read from memory one point, one
// entry after the other.
#include "rt3d_steps.h"

#include <type_traits>

namespace rt3d {

// Lanes per lidar pixel (one per point-grid pixel of its block, s <= 4) and
// lidar pixels per workgroup.
constexpr int SR_GROUP = 16;
constexpr int SR_GROUPS = 16;

// What a launch of k_sr_step computes (SR_MERGE_INTENSITY: the in-pixel merge,
// then the intensity step).
enum SrWork { SR_DEPTH, SR_INTENSITY, SR_MERGE_INTENSITY, SR_BKG, SR_GRADIENTS };

// Orders a wavefront's LDS writes before its reads (and reads before the next writes).
__device__ __forceinline__ void sr_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Point-grid pixel of sub-position u (row-major in the s x s block) of lidar
// pixel p, for frames of rows x cols lidar pixels.
__device__ __forceinline__ long long sr_fine(long long p, int u, int s, int rows, int cols)
{
    // (32-bit divisions: pixels of both grids total below 2^31)
    const uint32_t row = (uint32_t)p / (uint32_t)cols, j = (uint32_t)p - row * (uint32_t)cols;   // f rows + i
    const uint32_t du = (uint32_t)u / (uint32_t)s, dv = (uint32_t)u - du * (uint32_t)s;
    return (long long)(row * (uint32_t)s + du) * ((long long)cols * s) + j * (uint32_t)s + dv;
}

// h and h' at bin tb of a point with anchor a and fraction f, the segment read
// whether or not the bin lies in the support (any place of the table then), so
// that the reads of several points or bins are in flight together.  The values
// of irf_eval_t; returns whether it does.
__device__ __forceinline__ bool sr_irf(const float4* cr, int L, int o, int tb, int a, float f, float& h, float& hp)
{
    const int sh = f > 0.f ? 1 : 0;
    const float s = sh ? 1.f - f : 0.f;
    const int lo = 1 - sh;
    const int idx = tb - a + o + lo;
    const bool in = (unsigned)(idx - lo) <= (unsigned)(L - lo);
    cr_segment(cr[in ? idx : 0], s, h, hp);
    h = in ? h : 0.f;
    hp = in ? hp : 0.f;
    return in;
}

// Inclusive prefix sum over each row of 16 lanes.
__device__ __forceinline__ int sr_scan(int v)
{
    uint32_t x = (uint32_t)v;
    x += dpp_or_zero<0x111>(x);
    x += dpp_or_zero<0x112>(x);
    x += dpp_or_zero<0x114>(x);
    x += dpp_or_zero<0x118>(x);
    return (int)x;
}

template <SrWork WHICH, bool TLDS>
__global__ __launch_bounds__(SR_GROUP * SR_GROUPS) void k_sr_step(DevModel m, DevParams p, Shape lid, int s,
                                                                 long long Pf, const uint32_t* __restrict__ off,
                                                                 const uint32_t* __restrict__ ent,
                                                                 const float* __restrict__ gain, DevState st,
                                                                 float* __restrict__ bdst, float* __restrict__ gt,
                                                                 float* __restrict__ gr, float* __restrict__ gb)
{
    __shared__ float4 s_pt[SR_GROUPS][SR_GROUP * KM];       // anchor (bits), fraction, intensity
    __shared__ float2 s_wt[SR_GROUPS][SR_GROUP];            // z / (g lambda), bin (bits)
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    const int g = (int)(threadIdx.x / SR_GROUP), u = (int)(threadIdx.x % SR_GROUP);
    const long long pix = (long long)blockIdx.x * SR_GROUPS + g;
    const bool valid = pix < lid.P;                 // the whole group
    const long long pq = valid ? pix : 0;
    // lane u: point-grid pixel u of the block, its points in registers
    const bool in_block = valid && u < s * s;
    const long long q = in_block ? sr_fine(pq, u, s, lid.rows, lid.cols) : 0;
    PixPoints pts;
    load_points(st, Pf, q, pts);
    if (!in_block) pts.c = 0;
    if (WHICH == SR_MERGE_INTENSITY && in_block) merge_lane(st, Pf, p, q, 0, pts);
    const uint32_t o0 = off[pq], o1 = off[pq + 1];
    const float G = valid ? gain_at(gain, pq) : 0.f;
    const float bb = st.b[pq];
    const float4* cr = stage_segments<TLDS, WHICH != SR_BKG>(m, crl, stl);
    const bool live = G > 0.f;                      // group-uniform
    // the block's points staged in LDS, lane after lane (prefix of the counts in the group)
    const int upto = sr_scan(pts.c), np = __shfl(upto, (int)(threadIdx.x & ~(SR_GROUP - 1)) + SR_GROUP - 1, 64);
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (k < pts.c)
            s_pt[g][upto - pts.c + k] = make_float4(__int_as_float(pts.a[k]), pts.f[k], pts.r[k], 0.f);
    sr_sync();
    float sh[KM], shp[KM], sz = 0.f;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        sh[k] = 0.f;
        shp[k] = 0.f;
    }
    const uint32_t e0 = live ? o0 : 0u, e1 = live ? o1 : 0u;
    const float invG = live ? 1.f / G : 0.f;
    const int cmax = wave_max_count(pts.c);
    uint32_t next = e0 + (uint32_t)u < e1 ? ent[e0 + (uint32_t)u] : 0u;
    for (uint32_t eb = e0; eb < e1; eb += SR_GROUP) {   // the same trip count on the group's lanes
        const uint32_t x = eb + (uint32_t)u;
        const bool on = x < e1;
        const uint32_t v = next;
        next = x + SR_GROUP < e1 ? ent[x + SR_GROUP] : 0u;
        const int tb = ent_bin(v);
        float lam = bb;
        bool hit = false;
#pragma unroll 4
        for (int n = 0; n < np; ++n) {
            const float4 pt = s_pt[g][n];
            float h, hp;
            hit |= sr_irf(cr, m.L, m.o, tb, __float_as_int(pt.x), pt.y, h, hp);
            lam = fmaf(pt.z, h, lam);
        }
        const float w = on ? (float)ent_cnt(v) * invG * __builtin_amdgcn_rcpf(lam) : 0.f;
        sz += w;
        if (WHICH != SR_BKG) {
            // the entries in some point's support, in order (the others add zeros;
            // a weight that is not finite is kept, to reach the sums)
            hit = on && (hit || !(w <= 3.402823466e38f));
            const unsigned hits = (unsigned)(__builtin_amdgcn_ballot_w64(hit) >> (threadIdx.x & 48)) & 0xffffu;
            if (hit) s_wt[g][__popc(hits & ((1u << u) - 1u))] = make_float2(w, __int_as_float(tb));
            sr_sync();
            const int nb = __popc(hits);
            // slots past a lane's count have an anchor that no bin reaches: they add zeros
            auto add = [&](auto slots) {
#pragma unroll 4
                for (int y = 0; y < nb; ++y) {
                    const float2 wt = s_wt[g][y];
#pragma unroll
                    for (int k = 0; k < decltype(slots)::value; ++k) {
                        float h, hp;
                        sr_irf(cr, m.L, m.o, __float_as_int(wt.y), pts.a[k], pts.f[k], h, hp);
                        sh[k] = fmaf(wt.x, h, sh[k]);
                        shp[k] = fmaf(wt.x, hp, shp[k]);
                    }
                }
            };
            if (cmax == 1) add(std::integral_constant<int, 1>{});
            else if (cmax == 2) add(std::integral_constant<int, 2>{});
            else add(std::integral_constant<int, KM>{});
            sr_sync();                              // reads done before the next batch's writes
        }
    }
    // S and S' of a point (the cubic's table in LDS where it fits)
    auto s_of = [&](double t, float& S, float& Sp) {
        if (!s_whole(m, t)) s_direct(m, t, S, Sp, 0, 1);
        else if (stab_staged(m)) s_cubic(m, stl, t, S, Sp);
        else s_cubic(m, m.s_tab, t, S, Sp);
    };
    if (WHICH == SR_BKG || WHICH == SR_GRADIENTS) {
#pragma unroll
        for (int d = SR_GROUP / 2; d >= 1; d >>= 1) sz += __shfl_xor(sz, d, 64);
    }
    if (WHICH == SR_DEPTH) {
        if (live)
#pragma unroll
            for (int k = 0; k < KM; ++k)
                if (k < pts.c && pts.r[k] > 0.f) {
                    float S, Sp;
                    s_of(pts.t[k], S, Sp);
                    st.t[(long long)k * Pf + q] = depth_next(m, p, pts.t[k], Sp, shp[k]);
                }
    } else if (WHICH == SR_INTENSITY || WHICH == SR_MERGE_INTENSITY) {
        if (live)
#pragma unroll
            for (int k = 0; k < KM; ++k)
                if (k < pts.c) {
                    float S, Sp;
                    s_of(pts.t[k], S, Sp);
                    if (S > 0.f) st.r[(long long)k * Pf + q] = intensity_next(p, pts.r[k], S, sh[k]);
                }
    } else if (WHICH == SR_BKG) {
        if (valid && u == 0) bdst[pix] = live ? background_next(m, p, bb, sz) : bb;
    } else {   // raw gradients: every slot of the block's point-grid pixels, and gb
        if (in_block)
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                float vt = 0.f, vr = 0.f;
                if (live && k < pts.c) {
                    float S, Sp;
                    s_of(pts.t[k], S, Sp);
                    vt = G * pts.r[k] * (Sp + shp[k]);
                    vr = G * (S - sh[k]);
                }
                gt[(long long)k * Pf + q] = vt;
                gr[(long long)k * Pf + q] = vr;
            }
        if (valid && u == 0) gb[pix] = live ? G * ((float)m.T - sz) : 0.f;
    }
}

// The lidar-grid initialisation (lid: stride lid.P) spread over the point
// grid (out: stride Pf): every point-grid pixel takes its lidar pixel's
// points with 1/s^2 of the intensity (lambda unchanged), normals facing the
// sensor until they are fitted; the lidar background goes to out.b[0 .. P-1].
__global__ __launch_bounds__(256) void k_sr_expand(Shape lsh, int s, long long Pf, DevState lid, DevState out)
{
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= Pf) return;
    const long long R = (long long)lsh.rows * s, C = (long long)lsh.cols * s;
    const long long f = q / (R * C);
    const long long rem = q - f * R * C;
    const long long fi = rem / C, fj = rem - fi * C;
    const long long P = lsh.P;
    const long long pix = (f * lsh.rows + fi / s) * lsh.cols + fj / s;
    const int c = load_cnt(lid.cnt, pix);
    const float share = 1.f / (float)(s * s);
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        const bool on = k < c;
        out.t[(long long)k * Pf + q] = on ? lid.t[(long long)k * P + pix] : 0.0;
        out.r[(long long)k * Pf + q] = on ? lid.r[(long long)k * P + pix] * share : 0.f;
        out.n[(long long)(0 * KM + k) * Pf + q] = 0.f;
        out.n[(long long)(1 * KM + k) * Pf + q] = 0.f;
        out.n[(long long)(2 * KM + k) * Pf + q] = -1.f;
    }
    out.cnt[q] = (uint8_t)c;
    if (q < P) out.b[q] = lid.b[q];
}

template <SrWork WHICH>
static hipError_t sr_launch(const DevModel& m, const DevParams& p, const Shape& lid, int s, long long Pf,
                            const uint32_t* off, const uint32_t* ent, const float* gain, DevState st, float* bdst,
                            float* gt, float* gr, float* gb, hipStream_t stream)
{
    if (lid.P == 0) return hipSuccess;
    const dim3 g((unsigned)((lid.P + SR_GROUPS - 1) / SR_GROUPS)), b(SR_GROUP * SR_GROUPS);
    if (segments_fit(m))
        hipLaunchKernelGGL((k_sr_step<WHICH, true>), g, b, 0, stream, m, p, lid, s, Pf, off, ent, gain, st, bdst, gt,
                           gr, gb);
    else
        hipLaunchKernelGGL((k_sr_step<WHICH, false>), g, b, 0, stream, m, p, lid, s, Pf, off, ent, gain, st, bdst, gt,
                           gr, gb);
    return hipGetLastError();
}

hipError_t launch_sr_step(int step, bool merge, const DevModel& m, const DevParams& p, const Shape& lid, int s, long long Pf,
                          const uint32_t* off, const uint32_t* ent, const float* gain, DevState st, float* bdst,
                          hipStream_t stream)
{
    switch (step) {
    case RT3D_STEP_DEPTH:
        return sr_launch<SR_DEPTH>(m, p, lid, s, Pf, off, ent, gain, st, nullptr, nullptr, nullptr, nullptr, stream);
    case RT3D_STEP_INTENSITY:
        if (merge)
            return sr_launch<SR_MERGE_INTENSITY>(m, p, lid, s, Pf, off, ent, gain, st, nullptr, nullptr, nullptr,
                                                 nullptr, stream);
        return sr_launch<SR_INTENSITY>(m, p, lid, s, Pf, off, ent, gain, st, nullptr, nullptr, nullptr, nullptr,
                                       stream);
    case RT3D_STEP_BKG:
        return sr_launch<SR_BKG>(m, p, lid, s, Pf, off, ent, gain, st, bdst ? bdst : st.b, nullptr, nullptr, nullptr,
                                 stream);
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t launch_sr_gradients(const DevModel& m, const DevParams& p, const Shape& lid, int s, long long Pf,
                               const uint32_t* off, const uint32_t* ent, const float* gain, DevState st, float* gt,
                               float* gr, float* gb, hipStream_t stream)
{
    return sr_launch<SR_GRADIENTS>(m, p, lid, s, Pf, off, ent, gain, st, nullptr, gt, gr, gb, stream);
}

hipError_t launch_sr_expand(const Shape& lsh, int s, long long Pf, DevState lid, DevState out, hipStream_t stream)
{
    if (Pf == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sr_expand, dim3((unsigned)((Pf + 255) / 256)), dim3(256), 0, stream, lsh, s, Pf, lid, out);
    return hipGetLastError();
}

}  // namespace rt3d
