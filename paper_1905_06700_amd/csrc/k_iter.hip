// k_iter.hip -- one iteration of the reconstruction loop (Results,
// "Reconstruction algorithm") in three launches on tiles of 8 x 4 pixels:
//   k_iter_depth      the background filter of the iteration before, the depth
//                     step;
//   k_iter_intensity  APSS, the in-pixel merge, the intensity step;
//   k_iter_background the intensity filter and threshold, the background step.
// Each launch starts at a step that reads neighbouring pixels (or at the first
// step) and goes on with the steps that read only their own: what the tile's
// pixels just computed stays in LDS.  The same readings, arithmetic and order
// of sums as the steps' own kernels (k_steps.hip, k_apss.hip, k_filter.hip), so the
// result is the same to the bit.
//
// Mapping: LPP lanes per pixel, 32 LPP threads.  Steps on points (APSS, the
// intensity filter) take a thread per slot, thread 4 q + k slot k of tile pixel
// q; the gradient steps the pixel's LPP lanes, which load what does not depend
// on the first part (entries' range, gain, background) ahead of it.
//
// What a step's own launch costs a small batch is its start, its first loads
// and its last wavefronts (about 4 us whatever it does), and its pixels are
// few for tiles of 16 x 16.  An iteration on a frame of 32 x 32 takes 24 us (7 +
// 11 + 6) against 34 us in six launches, on one of 141 x 141 31 us (9 + 14 + 8)
// against 48 us; the host's rule has the sizes where that turns.
#include "rt3d_points.h"
#include "rt3d_steps.h"

namespace rt3d {

constexpr int ITX = 8, ITY = 4;         // tile: columns, rows (16 x 4: the same at 1 k pixels, 3% slower at 20 k)
static_assert(ITX * ITY == ITER_TILE_PIXELS, "the host's rule counts in tiles");
constexpr int IPX = ITX * ITY;          // pixels of a tile
static_assert(KM == 4, "a pixel's slots: a quad of lanes");

template <int LPP>
constexpr int iter_stage_words() { return IPX * LPP * step_batch<LPP>(); }

// Reads a word of every 64 bytes of the kernel's first BYTES of arguments: one
// wait for all of them, where the code would meet each line's miss by itself.
template <int BYTES>
__device__ __forceinline__ void touch_arguments()
{
    typedef __attribute__((address_space(4))) const uint32_t word;
    word* a = (word*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t v[BYTES / 64];
#pragma unroll
    for (int i = 0; i < BYTES / 64; ++i) v[i] = a[16 * i];
#pragma unroll
    for (int i = 0; i < BYTES / 64; ++i) asm volatile("" ::"s"(v[i]));
}
constexpr int ITER_ARGS = sizeof(DevModel) + sizeof(DevParams) + sizeof(Tiles) + 3 * sizeof(void*) + sizeof(DevState);

// The workgroup's tile: its frame's first pixel in the batch, its place.
struct IterTile {
    Shape sh;
    long long fbase;
    int i0, j0;
};

__device__ __forceinline__ IterTile iter_tile(const Tiles& tg)
{
    const int tile0 = (int)xcd_block(blockIdx.x, gridDim.x);
    const int g = tile_group(tg, tile0);
    IterTile t;
    t.sh = group_shape(tg, g);
    const int tile = tile0 - tg.tile0[g];
    const int tx = (t.sh.cols + ITX - 1) / ITX, tpf = tx * ((t.sh.rows + ITY - 1) / ITY);
    const int fr = tile / tpf, tr = tile - fr * tpf;
    t.i0 = (tr / tx) * ITY;
    t.j0 = (tr % tx) * ITX;
    t.fbase = tg.base[g] + (long long)fr * t.sh.rows * t.sh.cols;
    return t;
}

// This lane's pixel; its points come later (q.c = 0, every slot absent).
struct IterLane {
    long long pix;
    int px, sub;
    bool member, live;
    float G, b;
    uint32_t e0, e1, etot;
};

template <int LPP>
__device__ __forceinline__ IterLane iter_lane(const IterTile& t, const DevState& s, long long P,
                                              const uint32_t* __restrict__ off, const float* __restrict__ gain)
{
    IterLane L;
    L.px = threadIdx.x / LPP;
    L.sub = threadIdx.x % LPP;
    const int i = t.i0 + L.px / ITX, j = t.j0 + L.px % ITX;
    L.member = i < t.sh.rows && j < t.sh.cols;
    L.pix = t.fbase + (L.member ? (long long)i * t.sh.cols + j : 0);
    L.e0 = off[L.pix];
    L.e1 = off[L.pix + 1];
    L.etot = __builtin_amdgcn_readfirstlane(off[P]);
    L.G = L.member ? gain_at(gain, L.pix) : 0.f;
    L.b = s.b[L.pix];
    L.live = L.member && L.G > 0.f;
    return L;
}

// The points of a pixel from its slots' values (as load_points).
__device__ __forceinline__ void set_points(const double* t, const float* r, int c, PixPoints& q)
{
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

// The sums over the pixel's entries, on every one of its lanes.
template <int LPP>
__device__ __forceinline__ void iter_sums(const DevModel& m, const float4* cr, const IterLane& L, const PixPoints& q,
                                          bool work, float b, const uint32_t* __restrict__ ent, uint32_t* stage,
                                          float& sz, float (&sh)[KM], float (&shp)[KM])
{
    accumulate<LPP>(m, cr, q, work ? b : 1.f, work ? L.G : 1.f, ent, L.etot, work ? L.e0 : 0, work ? L.e1 : 0, L.sub,
                    stage_segment<LPP>(stage), sz, sh, shp);
    reduce_lanes<LPP>(sz, sh, shp);
}

// Floats of the background filter's region and row pass on a tile.
inline size_t iter_filter_floats(int rb)
{
    const size_t SX = ITX + 2 * (size_t)rb, SY = ITY + 2 * (size_t)rb;
    return SX * SY + SY * ITX + 2 * (size_t)rb + 1;
}

// FILTER: s.b becomes the filtered src floored at b_min first (k_bfilter_tile's
// sums); rb = 0: the floor alone.
template <int LPP, bool TLDS, bool FILTER>
__global__ __launch_bounds__(IPX * LPP, 5) void k_iter_depth(DevModel m, DevParams p, Tiles tg,
                                                             const uint32_t* __restrict__ off,
                                                             const uint32_t* __restrict__ ent,
                                                             const float* __restrict__ gain, DevState s,
                                                             const float* __restrict__ src,
                                                             const float* __restrict__ w, int rb, long long P)
{
    extern __shared__ float bf_lds[];
    __shared__ uint32_t stage[iter_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    __shared__ float bl[IPX];
    constexpr int NT = IPX * LPP;
    touch_arguments<ITER_ARGS>();
    const IterTile t = iter_tile(tg);
    const IterLane L = iter_lane<LPP>(t, s, P, off, gain);
    PixPoints q;
    load_points(s, P, L.pix, q);
    if (FILTER) {
        const int SX = ITX + 2 * rb, SY = ITY + 2 * rb;
        float* reg = bf_lds;              // [SY][SX], circular
        float* tmp = reg + SX * SY;       // [SY][ITX]: row pass
        float* wl = tmp + SY * ITX;       // [2 rb + 1] taps
        for (int k = threadIdx.x; k < 2 * rb + 1; k += NT) wl[k] = rb > 0 ? w[k] : 1.f;
        for (int x = threadIdx.x; x < SX * SY; x += NT) {
            const int r = x / SX, c = x - r * SX;
            int i = t.i0 - rb + r, j = t.j0 - rb + c;
            while (i < 0) i += t.sh.rows;
            while (i >= t.sh.rows) i -= t.sh.rows;
            while (j < 0) j += t.sh.cols;
            while (j >= t.sh.cols) j -= t.sh.cols;
            reg[x] = src[t.fbase + (long long)i * t.sh.cols + j];
        }
        const float4* cr0 = stage_segments<TLDS>(m, crl, stl);   // (its barrier: the region too)
        (void)cr0;
        float* out = rb > 0 ? tmp : reg;
        if (rb > 0) {
            for (int x = threadIdx.x; x < SY * ITX; x += NT) {
                const float* row = reg + (x / ITX) * SX + x % ITX + rb;
                float a = 0.f;
                for (int d = -rb; d <= rb; ++d) a = fmaf(wl[d + rb], row[d], a);
                tmp[x] = a;
            }
            __syncthreads();
        }
        if (threadIdx.x < IPX) {
            float a = 0.f;
            if (rb > 0)
                for (int d = -rb; d <= rb; ++d)
                    a = fmaf(wl[d + rb], out[(threadIdx.x / ITX + rb + d) * ITX + threadIdx.x % ITX], a);
            else
                a = out[threadIdx.x];
            bl[threadIdx.x] = fmaxf(a, (float)p.b_min);
        }
        __syncthreads();
        if (L.member && L.sub == 0) s.b[L.pix] = bl[L.px];
    } else {
        stage_segments<TLDS>(m, crl, stl);
    }
    const float4* cr = TLDS ? crl : m.cr;
    if (!L.member) set_points(nullptr, nullptr, 0, q);
    const bool work = L.live && q.c > 0;
    float sz, shh[KM], shp[KM], Sv[KM], Spv[KM];
    s_eval_points<LPP>(m, q, L.sub, stl, Sv, Spv);
    iter_sums<LPP>(m, cr, L, q, work, FILTER ? bl[L.px] : L.b, ent, stage, sz, shh, shp);
    if (!work || L.sub != 0) return;
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (k < q.c && q.r[k] > 0.f) s.t[k * P + L.pix] = depth_next(m, p, q.t[k], Spv[k], shp[k]);
}

// LDS bytes of the APSS tile with its halo: depths, normals, counts.
inline size_t iter_apss_bytes(int R)
{
    const size_t SX = ITX + 2 * (size_t)R, SY = ITY + 2 * (size_t)R;
    return SX * SY * (KM * sizeof(double) + 3 * KM * sizeof(float) + sizeof(int));
}

// in: the state; out: the same but for its other buffers of the depths, the
// normals and the counts.
template <int LPP, bool TLDS>
__global__ __launch_bounds__(IPX * LPP, 5) void k_iter_intensity(DevModel m, DevParams p, Tiles tg,
                                                                 const uint32_t* __restrict__ off,
                                                                 const uint32_t* __restrict__ ent,
                                                                 const float* __restrict__ gain, DevState in,
                                                                 DevState out, long long P)
{
    extern __shared__ double apss_lds[];
    __shared__ uint32_t stage[iter_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double stl[STEP_STAB_LDS];
    __shared__ double tn_l[IPX * KM];
    constexpr int NT = IPX * LPP;
    const int R = p.apss_Rs, SX = ITX + 2 * R, NS = SX * (ITY + 2 * R);
    double* tl = apss_lds;                                      // [KM][NS] depths
    float* nl = reinterpret_cast<float*>(tl + KM * NS);         // [3][KM][NS] normals
    int* cl = reinterpret_cast<int*>(nl + 3 * KM * NS);         // [NS] counts (0 outside the frame)
    touch_arguments<ITER_ARGS>();
    const IterTile t = iter_tile(tg);
    for (int x = threadIdx.x; x < NS; x += NT) {
        const int r = x / SX, i2 = t.i0 - R + r, j2 = t.j0 - R + x - r * SX;
        int c = 0;
        if (i2 >= 0 && i2 < t.sh.rows && j2 >= 0 && j2 < t.sh.cols) {
            const long long pp = t.fbase + (long long)i2 * t.sh.cols + j2;
            double ts[KM];
            c = load_cnt(in.cnt, pp);
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                ts[k] = in.t[k * P + pp];
#pragma unroll
                for (int a = 0; a < 3; ++a) nl[(a * KM + k) * NS + x] = in.n[(a * KM + k) * P + pp];
            }
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k * NS + x] = k < c ? ts[k] : no_depth();
        } else {
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k * NS + x] = no_depth();
        }
        cl[x] = c;
    }
    const IterLane L = iter_lane<LPP>(t, in, P, off, gain);
    float rq[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) rq[k] = in.r[k * P + L.pix];
    const float4* cr = stage_segments<TLDS>(m, crl, stl);      // (its barrier: the tile too)
    if (threadIdx.x < IPX * KM) {
        const int px = threadIdx.x / KM, k = threadIdx.x % KM;
        const int i = t.i0 + px / ITX, j = t.j0 + px % ITX, xc = (px / ITX + R) * SX + px % ITX + R;
        const long long pix = t.fbase + (long long)i * t.sh.cols + j;
        const int c = cl[xc];                                   // 0 outside the frame
        if (k == 0 && i < t.sh.rows && j < t.sh.cols) out.cnt[pix] = (uint8_t)c;
        if (k < c) {
            const float h = (float)p.h_apss, h2 = h * h;
            const double dz = p.dz, tq = tl[k * NS + xc];
            const Moments v =
                apss_moments(tl, NS, SX, xc, R, h2, (float)p.p_xy, dz, 1.001 * p.h_apss / dz, tq, TileNormals{nl, NS});
            double tn = tq;
            float on[3] = {nl[(0 * KM + k) * NS + xc], nl[(1 * KM + k) * NS + xc], nl[(2 * KM + k) * NS + xc]};
            apss_project(v.nn >= (float)p.m_min, v.W, v.Px, v.Py, v.Pz, v.Nx, v.Ny, v.Nz, v.PN, v.PP, h, h2, dz,
                         (double)(m.T - 1), tn, on);
            tn_l[threadIdx.x] = tn;
            out.t[k * P + pix] = tn;
#pragma unroll
            for (int a = 0; a < 3; ++a) out.n[(a * KM + k) * P + pix] = on[a];
        }
    }
    __syncthreads();
    PixPoints q;
    set_points(tn_l + L.px * KM, rq, cl[(L.px / ITX + R) * SX + L.px % ITX + R], q);
    if (L.member) merge_lane(out, P, p, L.pix, L.sub, q);      // (reads the normals just written)
    const bool work = L.live && q.c > 0;
    float sz, shh[KM], shp[KM], Sv[KM], Spv[KM];
    s_eval_points<LPP>(m, q, L.sub, stl, Sv, Spv);
    iter_sums<LPP>(m, cr, L, q, work, L.b, ent, stage, sz, shh, shp);
    if (!work || L.sub != 0) return;
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (k < q.c && Sv[k] > 0.f) out.r[k * P + L.pix] = intensity_next(p, q.r[k], Sv[k], shh[k]);
}

// in: the state; out: the same but for its other buffers of the depths, the
// intensities and the counts.  The new background goes to bdst.
template <int LPP, bool TLDS>
__global__ __launch_bounds__(IPX * LPP, 5) void k_iter_background(DevModel m, DevParams p, Tiles tg,
                                                                  const uint32_t* __restrict__ off,
                                                                  const uint32_t* __restrict__ ent,
                                                                  const float* __restrict__ gain, DevState in,
                                                                  DevState out, float* __restrict__ bdst, long long P)
{
    constexpr int NT = IPX * LPP, SX = ITX + 2, NS = SX * (ITY + 2);
    __shared__ uint32_t stage[iter_stage_words<LPP>()];
    __shared__ float4 crl[TLDS ? STEP_CR_LDS : 1];
    __shared__ double tl[KM][NS];
    __shared__ float rl[KM][NS];
    __shared__ int cl[NS];
    __shared__ double tn_l[IPX * KM];
    __shared__ float rn_l[IPX * KM];
    __shared__ int cn_l[IPX];
    touch_arguments<ITER_ARGS>();
    const IterTile t = iter_tile(tg);
    for (int x = threadIdx.x; x < NS; x += NT) {
        const int i2 = t.i0 - 1 + x / SX, j2 = t.j0 - 1 + x % SX;
        int c = 0;
        if (i2 >= 0 && i2 < t.sh.rows && j2 >= 0 && j2 < t.sh.cols) {
            const long long pp = t.fbase + (long long)i2 * t.sh.cols + j2;
            double ts[KM];
            c = load_cnt(in.cnt, pp);
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                ts[k] = in.t[k * P + pp];
                rl[k][x] = in.r[k * P + pp];
            }
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k][x] = k < c ? ts[k] : no_depth();
        } else {
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k][x] = no_depth();
        }
        cl[x] = c;
    }
    const IterLane L = iter_lane<LPP>(t, in, P, off, gain);
    const float4* cr = stage_segments<TLDS, false>(m, crl, nullptr);   // (its barrier: the tile too)
    if (threadIdx.x < IPX * KM) {
        const int px = threadIdx.x / KM, k = threadIdx.x % KM;
        const int i = t.i0 + px / ITX, j = t.j0 + px % ITX, xc = (px / ITX + 1) * SX + px % ITX + 1;
        const long long pix = t.fbase + (long long)i * t.sh.cols + j;
        const int c = cl[xc];                                   // 0 outside the frame
        bool keep = false;
        double tq = 0.0;
        float rn = 0.f;
        if (k < c) {
            tq = tl[k][xc];
            rn = ifilter_mean<3>(tl[0], rl[0], NS, SX, xc, (float)(p.h_int * p.h_int), (float)p.p_xy, p.dz, p.ilp_box,
                              ifilter_sides(i, j, t.sh.rows, t.sh.cols), tq, rl[k][xc]);
            keep = !(rn < (float)p.r_min);
        }
        // kept slots move down to the pixel's first places (the quad's ballot);
        // normals in place: all of a wavefront's are read before one is written
        const unsigned kept = (unsigned)(__builtin_amdgcn_ballot_w64(keep) >> (threadIdx.x & 60)) & 15u;
        const int nk = __popc(kept), to = __popc(kept & ((1u << k) - 1u));
        float n[3] = {0.f, 0.f, -1.f};
        if (keep && to != k)
#pragma unroll
            for (int a = 0; a < 3; ++a) n[a] = in.n[(a * KM + k) * P + pix];
        if (keep) {
            out.t[to * P + pix] = tq;
            out.r[to * P + pix] = rn;
            tn_l[px * KM + to] = tq;
            rn_l[px * KM + to] = rn;
        }
        if (k < c && k >= nk) {                                 // cleared: it held a point
            out.t[k * P + pix] = 0.0;
            out.r[k * P + pix] = 0.f;
        }
        __builtin_amdgcn_wave_barrier();
        if (keep && to != k)
#pragma unroll
            for (int a = 0; a < 3; ++a) out.n[(a * KM + to) * P + pix] = n[a];
        if (k < c && k >= nk)
#pragma unroll
            for (int a = 0; a < 3; ++a) out.n[(a * KM + k) * P + pix] = a == 2 ? -1.f : 0.f;
        if (k == 0) {
            cn_l[px] = nk;
            if (i < t.sh.rows && j < t.sh.cols) out.cnt[pix] = (uint8_t)nk;
        }
    }
    __syncthreads();
    PixPoints q;
    set_points(tn_l + L.px * KM, rn_l + L.px * KM, cn_l[L.px], q);
    float sz, shh[KM], shp[KM];
    iter_sums<LPP>(m, cr, L, q, L.live, L.b, ent, stage, sz, shh, shp);
    if (!L.member || L.sub != 0) return;
    bdst[L.pix] = L.live ? background_next(m, p, L.b, sz) : L.b;
}

// Whether the tiles' LDS fits (wide background filters and APSS windows take
// the steps' own kernels).
bool iter_fits(const DevParams& p, int rb)
{
    return iter_filter_floats(rb) * sizeof(float) <= 32768 && p.apss_Rs <= APSS_ROW &&
           iter_apss_bytes(p.apss_Rs) <= 32768;
}

long long iter_tiles(const Shape& sh)
{
    return tile_count(sh, ITX, ITY);
}

bool iter_tiles_add(Tiles& tg, long long base, const Shape& sh) { return tiles_add(tg, base, sh, ITX, ITY); }

template <int LPP, bool TLDS>
static hipError_t iter_launch(const IterArgs& a, const Tiles& tg, int part, hipStream_t st)
{
    const dim3 g((unsigned)tg.tile0[tg.n]), b(IPX * LPP);
    const size_t fl = iter_filter_floats(a.rb) * sizeof(float);
    if (part == 0 && a.filter)
        hipLaunchKernelGGL((k_iter_depth<LPP, TLDS, true>), g, b, fl, st, a.m, a.p, tg, a.off, a.ent, a.gain, a.in,
                           a.btmp, a.w, a.rb, a.P);
    else if (part == 0)
        hipLaunchKernelGGL((k_iter_depth<LPP, TLDS, false>), g, b, 0, st, a.m, a.p, tg, a.off, a.ent, a.gain, a.in,
                           a.btmp, a.w, a.rb, a.P);
    else if (part == 1)
        hipLaunchKernelGGL((k_iter_intensity<LPP, TLDS>), g, b, iter_apss_bytes(a.p.apss_Rs), st, a.m, a.p, tg, a.off,
                           a.ent, a.gain, a.in, a.out, a.P);
    else
        hipLaunchKernelGGL((k_iter_background<LPP, TLDS>), g, b, 0, st, a.m, a.p, tg, a.off, a.ent, a.gain, a.in,
                           a.out, a.btmp, a.P);
    return hipGetLastError();
}

hipError_t launch_iter(const IterArgs& a, const Tiles& tg, int part, hipStream_t st)
{
    if (tg.n == 0 || tg.tile0[tg.n] == 0) return hipSuccess;
    if (a.p.lpp == 8)
        return segments_fit(a.m) ? iter_launch<8, true>(a, tg, part, st) : iter_launch<8, false>(a, tg, part, st);
    return segments_fit(a.m) ? iter_launch<4, true>(a, tg, part, st) : iter_launch<4, false>(a, tg, part, st);
}

}  // namespace rt3d
