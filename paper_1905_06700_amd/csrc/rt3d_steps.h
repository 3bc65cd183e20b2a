// rt3d_steps.h -- the gradient steps' device code: a pixel's lanes, its staged
// entries and their sums (k_steps.hip has the formulas; k_iter.hip runs the
// same code on tiles).
#pragma once
#include "rt3d_dev.h"

namespace rt3d {

// Lanes per pixel, LPP (a template parameter: 4 or 8): a pixel's active
// entries are split over LPP consecutive lanes (entry e + LPP i), whose
// partial sums meet in a shuffle tree.  Four lanes fill the chip at large
// batches; eight halve the entries each lane walks, which shortens one
// frame's critical path (the autotuner picks per batch shape).
template <int LPP>
constexpr int step_batch() { return 64 / LPP; }   // entries a lane loads at once

// Entries of one batch of a pixel: step_batch per lane, STEP_LIST per pixel.
constexpr int STEP_LIST = 64;

// LDS words per workgroup for the lanes' staged entries.
template <int LPP>
constexpr int step_stage_words() { return 256 * step_batch<LPP>(); }

// A lane's staging segment: slot n of lane l of a wavefront at n * 64 + l, so
// that the wavefront's writes and reads of one slot each fall on distinct banks
// whatever slot each lane is at.
template <int LPP>
__device__ __forceinline__ uint32_t* stage_segment(uint32_t* stage)
{
    return stage + (threadIdx.x / 64) * (64 * step_batch<LPP>()) + (threadIdx.x % 64);
}

// Largest point count over the wavefront (uniform).
__device__ __forceinline__ int wave_max_count(int c)
{
    if (__builtin_amdgcn_ballot_w64(c > 3)) return 4;
    if (__builtin_amdgcn_ballot_w64(c > 2)) return 3;
    if (__builtin_amdgcn_ballot_w64(c > 1)) return 2;
    if (__builtin_amdgcn_ballot_w64(c > 0)) return 1;
    return 0;
}

// Entries the buffer loads address (byte offsets below 2^31, so that an entry
// past a pixel's end can be given an offset past every record).
constexpr uint32_t STEP_BUF_ENTRIES = 1u << 29;

// One batch of SB entries per lane from eb: load, select the entries inside
// some point's support into the lane's LDS segment, evaluate them.  BUF: the
// loads are buffer loads (an entry past the pixel's end reads 0 from an
// out-of-range offset), else global loads under the same condition.
template <int LPP, int NPT, int SB, bool BUF>
__device__ __forceinline__ void step_batch_n(const DevModel& m, const float4* cr, const PixPoints& q, float bb,
                                             float invG, const uint32_t* __restrict__ ent,
                                             __amdgpu_buffer_rsrc_t rsrc, uint32_t eb, uint32_t e1, int sub,
                                             uint32_t* seg, uint32_t& zout, float& sz, float (&sh)[KM],
                                             float (&shp)[KM])
{
    const uint32_t rem = e1 - eb;
    // this lane's entries of the batch: u < nv
    const int nv = (uint32_t)sub < rem ? (int)min((rem - (uint32_t)sub + LPP - 1) / LPP, (uint32_t)SB) : 0;
    uint32_t v[SB];
    if (BUF) {
        const uint32_t b4 = (eb + (uint32_t)sub) * 4u;
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const uint32_t o4 = u < nv ? b4 : 0x80000000u;
            v[u] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rsrc, o4, u * LPP * 4, 0);
        }
    } else {
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const uint32_t x = eb + sub + u * LPP;
            v[u] = x < e1 ? ent[x] : 0u;
        }
    }
    uint32_t* wp = seg;
#pragma unroll
    for (int u = 0; u < SB; ++u) {
        const int tbo = ent_bin(v[u]) + m.o;
        bool in = false;
#pragma unroll
        for (int k = 0; k < NPT; ++k) in = in || (uint32_t)(tbo - q.a[k]) <= (uint32_t)m.L;
        in = in && u < nv;
        *wp = v[u];                                       // kept only when it lies in a support
        wp += in ? 64 : 0;
        zout += in ? 0u : (uint32_t)ent_cnt(v[u]);        // zero where not valid
    }
    if (NPT == 0) return;
    for (const uint32_t* rp = seg; rp < wp; rp += 64) {
        const uint32_t v1 = *rp;
        const int tb = ent_bin(v1);
        const float z = (float)ent_cnt(v1);
        float h[KM], hp[KM];
        float lam = bb;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            irf_eval_t(cr, m.L, m.o, tb, q.a[k], q.f[k], h[k], hp[k]);
            lam = fmaf(q.r[k], h[k], lam);
        }
        const float zl = z * invG * __builtin_amdgcn_rcpf(lam);
        sz += zl;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            sh[k] = fmaf(zl, h[k], sh[k]);
            shp[k] = fmaf(zl, hp[k], shp[k]);
        }
    }
}

// Partial sums over one pixel's entries (e0p .. e1 - 1):
// sz = sum z/lambda, sh[k] = sum z h_k/lambda, shp[k] = sum z h'_k/lambda.
// h_k is zero outside bins floor(t_k) - o .. floor(t_k) - o + L (the
// segments' domain), so an entry in none of these ranges has lambda = g b and
// only adds z / (g b) to sz; those photons are summed as integers and added
// once.  The pixel's LPP lanes load its entries in batches, entry
// eb + sub + LPP u to lane sub: the first STEP_LIST entries form one batch,
// later ones batches of STEP_LIST / 2 (a wavefront's later batches are short,
// and a batch costs its full width on every lane).  Each lane writes the
// entries of its batch that lie in some point's support to its own LDS
// segment and evaluates them itself, so the work of a wavefront is the
// largest count of such entries on one lane, whatever the spread of the
// points of its pixels.  NPT is the largest point count of the wavefront;
// points at or beyond a lane's count have r = 0 and an anchor no entry's bin
// reaches, so they neither select entries nor change lambda, and a lane's
// sums do not depend on the other pixels of its wavefront.  BUF: the entries
// are read through a buffer resource over the whole entry array (etot
// entries; 0x00020000 is the resource word of a raw 32-bit buffer on this
// architecture).
template <int LPP, int NPT, bool BUF>
__device__ __forceinline__ void accumulate_n(const DevModel& m, const float4* cr, const PixPoints& q, float bb,
                                             float invG, const uint32_t* __restrict__ ent, uint32_t etot,
                                             uint32_t e0p, uint32_t e1, int sub, uint32_t* seg, float& sz,
                                             float (&sh)[KM], float (&shp)[KM])
{
    constexpr int SB = step_batch<LPP>();
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)ent, (short)0, BUF ? (int)(etot * 4u) : 0, 0x00020000);
    uint32_t zout = 0;                                    // photons of this lane's entries outside every support
    if (e0p < e1)
        step_batch_n<LPP, NPT, SB, BUF>(m, cr, q, bb, invG, ent, rsrc, e0p, e1, sub, seg, zout, sz, sh, shp);
    for (uint32_t eb = e0p + STEP_LIST; eb < e1; eb += STEP_LIST / 2)
        step_batch_n<LPP, NPT, SB / 2, BUF>(m, cr, q, bb, invG, ent, rsrc, eb, e1, sub, seg, zout, sz, sh, shp);
    sz += (float)zout * invG * __builtin_amdgcn_rcpf(bb);
}

template <int LPP, bool BUF>
__device__ __forceinline__ void accumulate_b(const DevModel& m, const float4* cr, const PixPoints& q, float bb,
                                             float invG, const uint32_t* __restrict__ ent, uint32_t etot,
                                             uint32_t e0p, uint32_t e1, int sub, uint32_t* seg, float& sz,
                                             float (&sh)[KM], float (&shp)[KM])
{
    switch (wave_max_count(q.c)) {
    case 0: accumulate_n<LPP, 0, BUF>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp); break;
    case 1: accumulate_n<LPP, 1, BUF>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp); break;
    case 2: accumulate_n<LPP, 2, BUF>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp); break;
    case 3: accumulate_n<LPP, 3, BUF>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp); break;
    default: accumulate_n<LPP, KM, BUF>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp); break;
    }
}

// etot: the entry count of all pixels (off[P], the same on every lane).
template <int LPP>
__device__ __forceinline__ void accumulate(const DevModel& m, const float4* cr, const PixPoints& q, float bb,
                                           float G, const uint32_t* __restrict__ ent, uint32_t etot, uint32_t e0p,
                                           uint32_t e1, int sub, uint32_t* seg, float& sz, float (&sh)[KM],
                                           float (&shp)[KM])
{
    sz = 0.f;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        sh[k] = 0.f;
        shp[k] = 0.f;
    }
    const float invG = __builtin_amdgcn_rcpf(G);   // 1 / g (exact for g = 1)
    if (etot <= STEP_BUF_ENTRIES)
        accumulate_b<LPP, true>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp);
    else
        accumulate_b<LPP, false>(m, cr, q, bb, invG, ent, etot, e0p, e1, sub, seg, sz, sh, shp);
}

// Sums the partials of the LPP lanes of a pixel (every lane ends with the total).
template <int LPP>
__device__ __forceinline__ float lane_sum(float v)
{
    static_assert(LPP == 4 || LPP == 8, "the lane reductions are sums over 4 or 8 lanes");
    return LPP == 4 ? quad_sum(v) : oct_sum(v);
}

template <int LPP>
__device__ __forceinline__ void reduce_lanes(float& sz, float (&sh)[KM], float (&shp)[KM])
{
    sz = lane_sum<LPP>(sz);
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        sh[k] = lane_sum<LPP>(sh[k]);
        shp[k] = lane_sum<LPP>(shp[k]);
    }
}

// S and S' of the pixel's points: the cubic of slot k by lane k of the pixel's
// LPP lanes, a direct sum split over them (strided segments), combined with
// shuffles; every lane ends with the totals.  (The cubics one slot after the
// other by the pixel's first lane: about 2 us of every step on a small batch.)
// The piecewise cubic's table, staged in LDS by the workgroup when it has at
// most STEP_STAB_PIECES pieces (its reads come at the end of a wavefront's
// work, where nothing else waits with them).
constexpr int STEP_STAB_PIECES = 8;
constexpr int STEP_STAB_LDS = STEP_STAB_PIECES + 1 + 4 * STEP_STAB_PIECES;

__device__ __forceinline__ bool stab_staged(const DevModel& m) { return m.s_np > 0 && m.s_np <= STEP_STAB_PIECES; }

template <int LPP>
__device__ __forceinline__ void s_eval_points(const DevModel& m, const PixPoints& q, int sub, const double* stl,
                                              float (&S)[KM], float (&Sp)[KM])
{
    // lane sub takes slot sub's cubic: the slots side by side, not one after the other
    static_assert(LPP >= KM, "a lane per slot");
    double tm = q.t[0];
#pragma unroll
    for (int k = 1; k < KM; ++k) tm = sub == k ? q.t[k] : tm;
    float Sm = 0.f, Spm = 0.f;
    const bool cubic = sub < q.c && s_whole(m, tm);
    if (cubic) {
        if (stab_staged(m)) s_cubic(m, stl, tm, Sm, Spm);
        else s_cubic(m, m.s_tab, tm, Sm, Spm);
    }
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        S[k] = sub == k ? Sm : 0.f;
        Sp[k] = sub == k ? Spm : 0.f;
        if (k < q.c && !s_whole(m, q.t[k])) s_direct(m, q.t[k], S[k], Sp[k], sub, LPP);
    }
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        S[k] = lane_sum<LPP>(S[k]);
        Sp[k] = lane_sum<LPP>(Sp[k]);
    }
}

// The IRF's Catmull-Rom segments for the entry loop: staged in the
// workgroup's LDS when they fit (TLDS), else read from global memory.
constexpr int STEP_CR_LDS = 256;

// STAB: the kernel evaluates S and S' (the table of the piecewise cubic too).
template <bool TLDS, bool STAB = true>
__device__ __forceinline__ const float4* stage_segments(const DevModel& m, float4* crl, double* stl)
{
    if (STAB && stab_staged(m))
        for (int i = threadIdx.x; i < 5 * m.s_np + 1; i += blockDim.x) stl[i] = m.s_tab[i];
    if (TLDS)
        for (int i = threadIdx.x; i <= m.L; i += blockDim.x) crl[i] = m.cr[i];
    __syncthreads();
    return TLDS ? crl : m.cr;
}

// Common prologue: the pixel of this lane, its points and its entry range.
struct Lane {
    long long pix;
    int sub;
    bool member;       // a pixel of the launch's IRF class (every pixel with one IRF)
    bool live;
    float G;
    PixPoints q;
    uint32_t e0, e1;   // the pixel's entries
    uint32_t etot;     // entries of all pixels (the same on every lane)
};

template <int LPP>
__device__ __forceinline__ Lane lane_setup(const DevModel& m, const DevState& s, long long P,
                                           const uint32_t* __restrict__ off, const float* __restrict__ gain,
                                           bool need_points)
{
    Lane L;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    L.sub = (int)(gid % LPP);
    if (m.lst) {   // the pixels of the launch's IRF class, from its list
        const uint32_t b0 = m.lst_meta[m.cls_id], b1 = m.lst_meta[m.cls_id + 1];
        const long long idx = gid / LPP;
        L.member = idx < (long long)(b1 - b0);
        L.pix = L.member ? (long long)m.lst[b0 + idx] : 0;
    } else {
        L.pix = gid / LPP;
        L.member = L.pix < P && in_class(m, L.pix);
    }
    L.live = L.member;
    const long long pp = L.live ? L.pix : 0;
    const uint32_t e0 = off[pp], e1 = off[pp + 1];
    L.etot = __builtin_amdgcn_readfirstlane(off[P]);
    L.G = L.live ? gain_at(gain, pp) : 0.f;
    load_points(s, P, pp, L.q);
    if (!L.live) L.q.c = 0;
    const bool work = L.live && L.G > 0.f && (!need_points || L.q.c > 0);
    L.e0 = work ? e0 : 0;
    L.e1 = work ? e1 : 0;
    L.live = work;
    return L;
}

// The in-pixel merge ahead of the intensity step: every lane of the pixel
// merges its copy of the points (merge_points); lane 0 writes the merged
// state.  Pixels whose points are in depth order and at least d_merge apart
// (almost all) keep their state untouched.
__device__ __forceinline__ void merge_lane(const DevState& s, long long P, const DevParams& p, long long pix,
                                           int sub, PixPoints& q)
{
    const int c0 = q.c;
    bool need = false;
#pragma unroll
    for (int k = 1; k < KM; ++k)
        if (k < c0 && (q.t[k] < q.t[k - 1] || q.t[k] - q.t[k - 1] < p.d_merge)) need = true;
    if (!need) return;
    double t[KM];
    float r[KM], nx[KM], ny[KM], nz[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        t[k] = q.t[k];
        r[k] = q.r[k];
        nx[k] = s.n[(0 * KM + k) * P + pix];
        ny[k] = s.n[(1 * KM + k) * P + pix];
        nz[k] = s.n[(2 * KM + k) * P + pix];
    }
    int c = c0;
    merge_points(t, r, nx, ny, nz, c, p.d_merge);
    if (sub == 0) store_points(s, P, pix, t, r, nx, ny, nz, c);
    q.c = c;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        const bool on = k < c;
        const double tk = on ? t[k] : 0.0;
        const double fl = floor(tk);
        q.t[k] = tk;
        q.a[k] = on ? (int)fl : PT_ABSENT;
        q.f[k] = (float)(tk - fl);
        q.r[k] = on ? r[k] : 0.f;
    }
}

inline bool segments_fit(const DevModel& m) { return m.L + 1 <= STEP_CR_LDS; }

}  // namespace rt3d
