// k_apss.hip -- APSS point-cloud denoising of depth (Results, "Reconstruction
// algorithm", depth update: algebraic point set surfaces fit local spheres to
// the points in world coordinates, the kernel size setting the low-pass) and
// the in-pixel merge of coincident points.
//
// Sphere fit (derived from its least-squares definition): with neighbours
// y_m = x_m - x_q closer than h, weights w = (1 - d^2/h^2)^4 and unit normals
// n_m, the sphere s(y) = u0 + ul.y + u4 |y|^2 minimising
// sum w |grad s(y_m) - n_m|^2, then sum w s(y_m)^2 over u0, is
//   u4 = (PN - P.N/W) / (2 (PP - P.P/W)),  ul = (N - 2 u4 P)/W,
//   u0 = -(ul.P + u4 PP)/W,
// W = sum w, P = sum w y, N = sum w n, PN = sum w y.n, PP = sum w y.y.
// Reading: q moves along its line of sight to the sphere's root nearest to it
// (clipped to [-h, h]); its normal becomes grad s there, facing the sensor.
// Jacobi: every query reads the state before the step.
//
// Mapping: a workgroup takes a tile of ATY x ATX pixels of one frame; it stages
// the counts and every slot of the tile with a halo in LDS in one round of
// loads (depths in FP64, normals; a second round for the live slots only,
// after the counts, cost more time than the bytes it saved), then one thread
// per live point, listed by pixel (tiles of many points: one per two slots of a
// pixel), fits and projects it, accumulating the sphere moments over
// the window from LDS in FP32, in coordinates local to the query (depth
// differences formed in FP64); under the orthographic map the halo covers only
// the pixels whose lateral offset stays below h (apss_moments), under the
// pinhole camera see k_apss_pinhole.
// Windows whose staged tile does not fit in 64 KB of LDS take a variant with
// eight lanes per pixel reading the state from global memory, the partial
// moment sets meeting in a fixed wavefront-shuffle tree.
#include "rt3d_points.h"

namespace rt3d {

constexpr int ATX = TILE, ATY = TILE;   // tile of the LDS variant: columns, rows

// LDS bytes of a staged tile with an R-pixel halo: per pixel KM depths (FP64),
// 3 x KM normal components and the count.
inline size_t apss_tile_bytes(int R)
{
    const size_t SX = ATX + 2 * (size_t)R, SY = ATY + 2 * (size_t)R;
    return SX * SY * (KM * sizeof(double) + 3 * KM * sizeof(float) + sizeof(int));
}

// The pinhole kernel's: also the inverse ray length per pixel, and the list of
// the tile's points.
inline size_t pinhole_tile_bytes(int R)
{
    const size_t SX = ATX + 2 * (size_t)R, SY = ATY + 2 * (size_t)R;
    return apss_tile_bytes(R) + SX * SY * sizeof(double) + KM * ATX * ATY * sizeof(uint16_t);
}

size_t apss_lds_bytes(int R) { return apss_tile_bytes(R); }

// Halo the orthographic tile kernel stages: the largest ring r of window
// pixels (Chebyshev distance r) whose nearest pixel, r pixels away along a
// row, lies closer than h -- pixels of farther rings hold no neighbour.  The
// same FP32 arithmetic as the kernel's lateral pre-test.
int apss_staged_halo(double h_apss, double p_xy, int R)
{
    const float h = (float)h_apss, h2 = h * h, pxy = (float)p_xy;
    int r = 0;
    while (r < R) {
        const float x = (float)(r + 1) * pxy;
        if (!(x * x < h2)) break;
        ++r;
    }
    return r;
}

// The orthographic map, staged halo p.apss_Rs.  carry: also copy the count,
// background and intensities to `out` (else `out` receives only the depths and
// normals of the live slots).  A tile of at most APSS_SPARSE points takes a
// thread per point, which leaves no lane to a pixel without points and no slot
// to wait for another; a fuller one, whose list would take a second round of
// threads, takes a thread per two slots of a pixel, past each neighbour at once.
// The sums are the same in either.  Windows of 1 / 2 / 5 rings, us: 636 k pixels of
// 1.4 points 41 / 70 / 163 (the planes read and written at the rate of a copy
// would take 22), of 2.8 points right after the initialisation 57 / 100 / 213, a
// thread per point 76 / 145 / 366; 262 k pixels of 2.8 points 28 / 48 / 98 against
// 36 / 65 / 160; 74 k pixels of 1.5 points 15 / 25 / 55.
// 256 threads with a thread per pixel, its four slots at once, fill 111 registers:
// dense tiles 57 / 101 / 257 us and 26 / 45 / 124, but 43 / 75 / 196 and 17 / 30 / 67
// on the sparse ones, whose points then need two rounds.  The neighbours' loop
// stays rolled: unrolled it takes 112 registers, two workgroups per CU instead of
// three (49 us where this takes 41).
constexpr int APT = 512;
constexpr int APSS_SPARSE = APT;        // points of a tile of 256 pixels
constexpr int APSS_PAIR = 2;            // slots of a pixel a thread takes on the others
static_assert(APT == ATX * ATY * KM / APSS_PAIR, "a thread per pair");

// LDS bytes of the orthographic kernel: depths, normals, counts, the list.
inline size_t apss_staged_bytes(int R)
{
    const size_t NS = (ATX + 2 * (size_t)R) * (ATY + 2 * (size_t)R);
    return NS * (KM * sizeof(double) + 3 * KM * sizeof(float) + sizeof(uint8_t)) + APSS_SPARSE * sizeof(uint16_t);
}

// The moments of n points of a pixel (depths tq) at once, its neighbours in the
// window's order: each neighbour is read once.
__device__ __forceinline__ void apss_moments_slots(const double* tl, const float* nl, const uint8_t* cl, int NS, int SX,
                                                   int xc, int R, float h2, float pxy, double dz,
                                                   const double (&tq)[APSS_PAIR], int n,
                                                   Moments (&s)[APSS_PAIR])
{
    const float inv_h2 = 1.f / h2;
    for (int di = -R; di <= R; ++di) {
        const float yy = (float)di * pxy;
        for (int dj = -R; dj <= R; ++dj) {
            const float yx = (float)dj * pxy;
            const float dl = fmaf(yx, yx, yy * yy);
            if (!(dl < h2)) continue;
            const int x = xc + di * SX + dj;
            const int cc = cl[x];
#pragma unroll 1
            for (int k = 0; k < cc; ++k) {
                const double t2 = tl[k * NS + x];
                const float nx = nl[(0 * KM + k) * NS + x];
                const float ny = nl[(1 * KM + k) * NS + x];
                const float nz = nl[(2 * KM + k) * NS + x];
                const float yn = fmaf(yx, nx, yy * ny);
#pragma unroll
                for (int q = 0; q < APSS_PAIR; ++q) {
                    if (q >= n) break;
                    const float yz = (float)((t2 - tq[q]) * dz);
                    const float d2 = fmaf(yz, yz, dl);
                    if (!(d2 < h2)) continue;
                    float a = 1.f - d2 * inv_h2;
                    a = a * a;
                    const float w = a * a;
                    s[q].W += w;
                    s[q].Px = fmaf(w, yx, s[q].Px);
                    s[q].Py = fmaf(w, yy, s[q].Py);
                    s[q].Pz = fmaf(w, yz, s[q].Pz);
                    s[q].Nx = fmaf(w, nx, s[q].Nx);
                    s[q].Ny = fmaf(w, ny, s[q].Ny);
                    s[q].Nz = fmaf(w, nz, s[q].Nz);
                    s[q].PN = fmaf(w, fmaf(yz, nz, yn), s[q].PN);
                    s[q].PP = fmaf(w, d2, s[q].PP);
                    s[q].nn += 1.f;
                }
            }
        }
    }
}

__global__ __launch_bounds__(APT, 6) void k_apss_tile(DevModel m, DevParams p, Tiles tg, DevState in, DevState out,
                                                      int only_above, int carry)
{
    extern __shared__ double apss_lds[];
    const int R = p.apss_Rs, SX = ATX + 2 * R, NS = SX * (ATY + 2 * R);
    double* tl = apss_lds;                                      // [KM][NS] depths
    float* nl = reinterpret_cast<float*>(tl + KM * NS);         // [3][KM][NS] normals
    uint8_t* cl = reinterpret_cast<uint8_t*>(nl + 3 * KM * NS); // [NS] counts (0 outside the frame)
    const int tile0 = (int)xcd_block(blockIdx.x, gridDim.x);
    const int g = tile_group(tg, tile0);
    const Shape sh = group_shape(tg, g);
    in = state_at(in, tg.base[g]);
    out = state_at(out, tg.base[g]);
    const long long S = sh.S;
    const int tile = tile0 - tg.tile0[g];
    const int tiles_x = (sh.cols + ATX - 1) / ATX, tiles_y = (sh.rows + ATY - 1) / ATY;
    const int tpf = tiles_x * tiles_y;
    const int fr = tile / tpf, tr = tile % tpf;
    const int i0 = (tr / tiles_x) * ATY, j0 = (tr % tiles_x) * ATX;
    const long long fbase = (long long)fr * sh.rows * sh.cols;
    // stage the counts and every slot of the tile and its halo (without
    // waiting for the counts)
    __shared__ int wave_points[ATX * ATY / 64];
    uint16_t* pl = reinterpret_cast<uint16_t*>(cl + NS);        // [APSS_SPARSE] points (NS is even)
    for (int x = threadIdx.x; x < NS; x += APT) {
        const int i2 = i0 - R + x / SX, j2 = j0 - R + x % SX;
        int c = 0;
        if (i2 >= 0 && i2 < sh.rows && j2 >= 0 && j2 < sh.cols) {
            const long long pp = fbase + (long long)i2 * sh.cols + j2;
            double ts[KM];
            c = load_cnt(in.cnt, pp);
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                ts[k] = in.t[k * S + pp];
#pragma unroll
                for (int a = 0; a < 3; ++a) nl[(a * KM + k) * NS + x] = in.n[(a * KM + k) * S + pp];
            }
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k * NS + x] = k < c ? ts[k] : no_depth();
        } else {
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k * NS + x] = no_depth();
        }
        cl[x] = (uint8_t)c;
    }
    __syncthreads();
    const int ty = threadIdx.x / ATX, tx = threadIdx.x % ATX;
    const bool inside = ty < ATY && i0 + ty < sh.rows && j0 + tx < sh.cols;
    const int c = inside ? cl[(ty + R) * SX + tx + R] : 0;
    if (carry && inside) {
        const long long pix = fbase + (long long)(i0 + ty) * sh.cols + j0 + tx;
        out.cnt[pix] = (uint8_t)c;
        out.b[pix] = in.b[pix];
#pragma unroll
        for (int k = 0; k < KM; ++k) out.r[k * S + pix] = in.r[k * S + pix];
    }
    const int points = list_points(c, wave_points, pl, APSS_SPARSE);
    const float h = (float)p.h_apss, h2 = h * h;
    const double dz = p.dz, reach = 1.001 * p.h_apss / dz, tmax = (double)(m.T - 1);
    auto finish = [&](int k, int xc, long long pix, double tq, bool fit, const Moments& v) {
        double tn = tq;
        float on[3] = {nl[(0 * KM + k) * NS + xc], nl[(1 * KM + k) * NS + xc], nl[(2 * KM + k) * NS + xc]};
        apss_project(fit && v.nn >= (float)p.m_min, v.W, v.Px, v.Py, v.Pz, v.Nx, v.Ny, v.Nz, v.PN, v.PP, h, h2, dz,
                     tmax, tn, on);
        out.t[k * S + pix] = tn;
#pragma unroll
        for (int a = 0; a < 3; ++a) out.n[(a * KM + k) * S + pix] = on[a];
    };
    if (points > APSS_SPARSE) {
        const int qy = ty % ATY, xq = (qy + R) * SX + tx + R, k0 = ty / ATY * APSS_PAIR;
        const int cq = i0 + qy < sh.rows && j0 + tx < sh.cols ? cl[xq] : 0;
        if (cq <= k0) return;
        const long long pix = fbase + (long long)(i0 + qy) * sh.cols + j0 + tx;
        const bool fit = !(only_above >= 0 && cq <= only_above);
        double tq[APSS_PAIR];
        Moments v[APSS_PAIR];
#pragma unroll
        for (int q = 0; q < APSS_PAIR; ++q) {
            tq[q] = tl[(k0 + q) * NS + xq];
            v[q] = Moments{};
        }
        if (fit) apss_moments_slots(tl, nl, cl, NS, SX, xq, R, h2, (float)p.p_xy, dz, tq, cq - k0, v);
#pragma unroll
        for (int q = 0; q < APSS_PAIR; ++q) {
            if (k0 + q >= cq) break;
            finish(k0 + q, xq, pix, tq[q], fit, v[q]);
        }
        return;
    }
    for (int q = threadIdx.x; q < points; q += APT) {
        const int pk = pl[q], k = pk % KM, qy = pk / KM / ATX, qx = pk / KM % ATX, xq = (qy + R) * SX + qx + R;
        const double tq = tl[k * NS + xq];
        const bool fit = !(only_above >= 0 && cl[xq] <= only_above);
        Moments v{};
        if (fit) v = apss_moments(tl, NS, SX, xq, R, h2, (float)p.p_xy, dz, reach, tq, TileNormals{nl, NS});
        finish(k, xq, fbase + (long long)(i0 + qy) * sh.cols + j0 + qx, tq, fit, v);
    }
}

// The pinhole camera: a point at depth t lies t dz along its pixel's ray
// (ray_dir), differences formed in FP64, the projection along the query's ray.
// The tile is staged as above with the full halo p.apss_R and each pixel's
// inverse ray length (the ray is its unnormalised form times that); then one
// thread per live point of the tile (listed by pixel in LDS), so that neither
// the pixels without points nor the second and third slots leave lanes idle,
// and the rays' square roots are taken once per staged pixel.  A thread's
// window is cut to the pixels whose rays pass closer than h to the point at
// all: with uq and u2 = uq + a (dj, di, 0) the unnormalised rays, the point at
// range rho lies at least rho |uq x u2| / (|uq| |u2|) away from the ray u2,
// |uq x u2|^2 = a^2 (dj^2 + di^2 + (ux di - uy dj)^2): an ellipse of pixels.
// Points are taken in the order of their ellipses' rows, so that a wavefront's
// lanes walk windows of one size, and every second round of workgroups hands
// the large ones to the SIMDs that have the small ones of the round before.
// Only slots within h in range are looked at closer: mostly one of a pixel's.
// 512 threads: two workgroups' worth of LDS per CU, so sixteen wavefronts.
// 2 x 256 x 256 pixels of 1.7 points, R = 5: 97 us (11 staging, 32 finding the
// slots in range, 54 the moments; half of the issue slots of the vector ALU),
// against 370 us for one thread per pixel that took every slot of all 121
// pixels by itself.
constexpr int PNT = 512;
constexpr int APSS_PINHOLE_R = 5;   // largest halo whose staged tile fits the 64 KB that the host admits
static_assert(KM * ATX * ATY <= 1024, "a listed point: 10 bits for pixel and slot");
static_assert(KM * (2 * APSS_PINHOLE_R + 1) <= 64, "a row's slots: a bit each");

__global__ __launch_bounds__(PNT, 4) void k_apss_pinhole(DevModel m, DevParams p, Tiles tg, DevState in, DevState out,
                                                         int only_above, int carry)
{
    extern __shared__ double apss_lds[];
    __shared__ int by_radius[APSS_PINHOLE_R + 1];
    const int R = p.apss_R, SX = ATX + 2 * R, NS = SX * (ATY + 2 * R);
    double* tl = apss_lds;                                      // [KM][NS] depths
    double* vl = tl + KM * NS;                                  // [NS] inverse ray lengths
    float* nl = reinterpret_cast<float*>(vl + NS);              // [3][KM][NS] normals
    int* cl = reinterpret_cast<int*>(nl + 3 * KM * NS);         // [NS] counts (0 outside the frame)
    uint16_t* pl = reinterpret_cast<uint16_t*>(cl + NS);        // [KM ATX ATY] points: radius, KM (tile pixel) + slot
    if (threadIdx.x <= APSS_PINHOLE_R) by_radius[threadIdx.x] = 0;
    const int tile0 = (int)xcd_block(blockIdx.x, gridDim.x);
    const int g = tile_group(tg, tile0);
    const Shape sh = group_shape(tg, g);
    in = state_at(in, tg.base[g]);
    out = state_at(out, tg.base[g]);
    const long long S = sh.S;
    const int tile = tile0 - tg.tile0[g];
    const int tiles_x = (sh.cols + ATX - 1) / ATX, tiles_y = (sh.rows + ATY - 1) / ATY;
    const int tpf = tiles_x * tiles_y;
    const int fr = tile / tpf, tr = tile % tpf;
    const int i0 = (tr / tiles_x) * ATY, j0 = (tr % tiles_x) * ATX;
    const long long fbase = (long long)fr * sh.rows * sh.cols;
    const float h = (float)p.h_apss, h2 = h * h, inv_h2 = 1.f / h2;
    const double dz = p.dz, persp = p.persp;
    const double tmax = (double)(m.T - 1);
    const double cxd = 0.5 * (sh.cols - 1), cyd = 0.5 * (sh.rows - 1);
    const float pa = (float)persp;
    const double trange = 1.001 * p.h_apss / dz;   // points farther apart in range are farther apart than h
    // the ellipse of a point: A dj^2 - 2 ux uy di dj + (1 + ux^2) di^2 < K, A = 1 + uy^2
    // (0.999: the squared range rounded down; |u2| at its largest over the window)
    struct Ellipse {
        float K, A, uu, xy;
    };
    auto ellipse = [&](int i, int j, double t) {
        const float ux = pa * (float)(j - cxd), uy = pa * (float)(i - cyd), rho = (float)(t * dz);
        const float fx = fabsf(ux) + pa * (float)R, fy = fabsf(uy) + pa * (float)R;
        Ellipse e;
        e.A = fmaf(uy, uy, 1.f);
        e.uu = fmaf(ux, ux, e.A);
        e.xy = ux * uy;
        e.K = h2 * e.uu * fmaf(fx, fx, fmaf(fy, fy, 1.f)) / (0.999f * rho * rho * pa * pa);
        return e;
    };
    const double none = __builtin_nan("");                      // a slot without a point: in range of nothing
    for (int x = threadIdx.x; x < NS; x += PNT) {
        const int i2 = i0 - R + x / SX, j2 = j0 - R + x % SX;
        int c = 0;
        if (i2 >= 0 && i2 < sh.rows && j2 >= 0 && j2 < sh.cols) {
            const long long pp = fbase + (long long)i2 * sh.cols + j2;
            double ts[KM];
            c = load_cnt(in.cnt, pp);
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                ts[k] = in.t[k * S + pp];
#pragma unroll
                for (int a = 0; a < 3; ++a) nl[(a * KM + k) * NS + x] = in.n[(a * KM + k) * S + pp];
            }
            double v[3];
            ray_dir(p.persp, sh.rows, sh.cols, i2, j2, v);
            vl[x] = v[2];
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k * NS + x] = k < c ? ts[k] : none;
        } else {
#pragma unroll
            for (int k = 0; k < KM; ++k) tl[k * NS + x] = none;
        }
        cl[x] = c;
    }
    __syncthreads();
    // the tile's points, by window radius
    int c = 0, rk[KM];
    if (threadIdx.x < ATX * ATY) {
        const int ty = threadIdx.x / ATX, tx = threadIdx.x % ATX, i = i0 + ty, j = j0 + tx;
        const int xc = (ty + R) * SX + tx + R;
        const bool inside = i < sh.rows && j < sh.cols;
        c = inside ? cl[xc] : 0;
        const bool fit = !(only_above >= 0 && c <= only_above);
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            rk[k] = 0;
            if (k >= c) continue;
            if (fit) {
                const Ellipse e = ellipse(i, j, tl[k * NS + xc]);
                rk[k] = (int)fminf((float)R, sqrtf(e.K * e.A / e.uu));
            }
            atomicAdd(&by_radius[rk[k]], 1);
        }
        if (carry && inside) {
            const long long pix = fbase + (long long)i * sh.cols + j;
            out.cnt[pix] = (uint8_t)c;
            out.b[pix] = in.b[pix];
#pragma unroll
            for (int k = 0; k < KM; ++k) out.r[k * S + pix] = in.r[k * S + pix];
        }
    }
    __syncthreads();
    int points = 0;
    for (int r = R; r >= 0; --r) points += by_radius[r];
    __syncthreads();
    if (threadIdx.x == 0) {                     // largest first
        int run = 0;
        for (int r = R; r >= 0; --r) {
            const int n = by_radius[r];
            by_radius[r] = run;
            run += n;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (k < c)
            pl[atomicAdd(&by_radius[rk[k]], 1)] = (uint16_t)((rk[k] << 10) | (threadIdx.x * KM + k));
    __syncthreads();
    for (int q = threadIdx.x ^ ((blockIdx.x >> 8 & 1) << 7); q < points; q += PNT) {
        const int pk = pl[q], k = pk % KM, px = (pk & 1023) / KM, r = pk >> 10;
        const int i = i0 + px / ATX, j = j0 + px % ATX;
        const int xc = (px / ATX + R) * SX + px % ATX + R;
        const long long pix = fbase + (long long)i * sh.cols + j;
        const int cq = cl[xc];
        const bool fit = !(only_above >= 0 && cq <= only_above);
        const double iq = vl[xc];
        const double vq[3] = {persp * (j - cxd) * iq, persp * (i - cyd) * iq, iq};
        const float rq[3] = {(float)vq[0], (float)vq[1], (float)vq[2]};
        const double tq = tl[k * NS + xc];
        float W = 0.f, Px = 0.f, Py = 0.f, Pz = 0.f, Nx = 0.f, Ny = 0.f, Nz = 0.f, PN = 0.f, PP = 0.f, nn = 0.f;
        if (fit) {
            const Ellipse e = ellipse(i, j, tq);
            const float iA = 1.f / e.A, duu = e.uu * iA;
            for (int di = -r; di <= r; ++di) {
                const double wy = persp * (i + di - cyd);
                const float mid = e.xy * (float)di * iA;
                const float half = sqrtf(fmaxf((e.K - (float)(di * di) * duu) * iA, 0.f));
                const int j1 = (int)fminf((float)R, floorf(mid + half));
                const int jl = (int)fmaxf((float)-R, ceilf(mid - half));
                // the row's slots within h in range, KM bits per pixel
                const int row = xc + di * SX;
                uint64_t near = 0;
#pragma unroll 2
                for (int dj = jl; dj <= j1; ++dj) {
                    unsigned bits = 0;
#pragma unroll
                    for (int k2 = 0; k2 < KM; ++k2)
                        bits |= fabs(fabs(tl[k2 * NS + row + dj]) - fabs(tq)) < trange ? 1u << k2 : 0u;
                    near |= (uint64_t)bits << (KM * (dj - jl));
                }
                // each in turn, the next one's values on their way
                int at = 0;
                double t2 = 0.0, iv2 = 0.0;
                float nx = 0.f, ny = 0.f, nz = 0.f;
                auto fetch = [&] {
                    const int bit = __ffsll((unsigned long long)near) - 1, k2 = bit % KM;
                    at = jl + bit / KM;
                    const int x = row + at, y = k2 * NS + x;
                    t2 = tl[y];
                    iv2 = vl[x];
                    nx = nl[y];
                    ny = nl[KM * NS + y];
                    nz = nl[2 * KM * NS + y];
                    near &= near - 1;
                };
                bool more = near != 0;
                if (more) fetch();
                while (more) {
                    const double wx = persp * (j + at - cxd), t = t2, i2 = iv2;
                    const float mx = nx, my = ny, mz = nz;
                    more = near != 0;
                    if (more) fetch();
                    const double v2[3] = {wx * i2, wy * i2, i2};
                    const float yx = (float)((t * v2[0] - tq * vq[0]) * dz);
                    const float yy = (float)((t * v2[1] - tq * vq[1]) * dz);
                    const float yz = (float)((t * v2[2] - tq * vq[2]) * dz);
                    const float d2 = fmaf(yx, yx, fmaf(yy, yy, yz * yz));
                    if (d2 < h2) {
                        float a = 1.f - d2 * inv_h2;
                        a = a * a;
                        const float w = a * a;
                        W += w;
                        Px = fmaf(w, yx, Px);
                        Py = fmaf(w, yy, Py);
                        Pz = fmaf(w, yz, Pz);
                        Nx = fmaf(w, mx, Nx);
                        Ny = fmaf(w, my, Ny);
                        Nz = fmaf(w, mz, Nz);
                        PN = fmaf(w, yx * mx + yy * my + yz * mz, PN);
                        PP = fmaf(w, d2, PP);
                        nn += 1.f;
                    }
                }
            }
        }
        double tn = tq;
        float on[3] = {nl[(0 * KM + k) * NS + xc], nl[(1 * KM + k) * NS + xc], nl[(2 * KM + k) * NS + xc]};
        apss_project(fit && nn >= (float)p.m_min, W, Px, Py, Pz, Nx, Ny, Nz, PN, PP, h, h2, dz, tmax, tn, on, rq);
        out.t[k * S + pix] = tn;
#pragma unroll
        for (int a = 0; a < 3; ++a) out.n[(a * KM + k) * S + pix] = on[a];
    }
}

constexpr int LPA = 8;   // lanes per pixel: the window's pixels are split over them
static_assert(LPA == 8, "the lane sums below are sums over 8 lanes");

__global__ __launch_bounds__(256) void k_apss(DevModel m, DevParams p, Shape sh, DevState in, DevState out,
                                              int only_above)
{
    const long long P = sh.P, S = sh.S;
    const long long gid = (long long)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const long long pix = gid / LPA;
    const int sub = (int)(gid % LPA);
    const bool live = pix < P;
    const long long pq = live ? pix : 0;
    const int c = live ? load_cnt(in.cnt, pq) : 0;
    if (live) {
        if (sub == 0) {
            out.cnt[pix] = (uint8_t)c;
            out.b[pix] = in.b[pix];
        }
        if (sub < KM) out.r[sub * S + pix] = in.r[sub * S + pix];   // depth and normal: lane 0 below
    }
    const bool fit = live && !(only_above >= 0 && c <= only_above);
    const int per_frame = sh.rows * sh.cols;
    const long long fr = pq / per_frame;
    const int i = (int)((pq / sh.cols) % sh.rows), j = (int)(pq % sh.cols);
    const int R = p.apss_R, side = 2 * R + 1;
    const float h = (float)p.h_apss, h2 = h * h, inv_h2 = 1.f / h2;
    const float pxy = (float)p.p_xy;
    const double dz = p.dz;
    const double tmax = (double)(m.T - 1);
    for (int k = 0; k < KM; ++k) {                  // every lane runs the slot (lane sums below)
        const bool act = fit && k < c;
        if (__ballot(live && k < c) == 0ull) break;  // no pixel of the wavefront has slot k
        const double tq = act ? in.t[k * S + pq] : 0.0;
        float W = 0.f, Px = 0.f, Py = 0.f, Pz = 0.f, Nx = 0.f, Ny = 0.f, Nz = 0.f, PN = 0.f, PP = 0.f, nn = 0.f;
        if (act) {
            for (int widx = sub; widx < side * side; widx += LPA) {
                const int i2 = i + widx / side - R, j2 = j + widx % side - R;
                if (i2 < 0 || i2 >= sh.rows || j2 < 0 || j2 >= sh.cols) continue;
                const float yy = (float)(i2 - i) * pxy, yx = (float)(j2 - j) * pxy;
                const float dl = fmaf(yx, yx, yy * yy);
                if (!(dl < h2)) continue;                  // no neighbour in this pixel
                const long long pp = (fr * sh.rows + i2) * sh.cols + j2;
                const int cc = load_cnt(in.cnt, pp);
                for (int k2 = 0; k2 < cc; ++k2) {
                    const float yz = (float)((in.t[k2 * S + pp] - tq) * dz);
                    const float d2 = fmaf(yz, yz, dl);
                    if (!(d2 < h2)) continue;
                    float a = 1.f - d2 * inv_h2;
                    a = a * a;
                    const float w = a * a;
                    const float nx = in.n[(0 * KM + k2) * S + pp];
                    const float ny = in.n[(1 * KM + k2) * S + pp];
                    const float nz = in.n[(2 * KM + k2) * S + pp];
                    W += w;
                    Px = fmaf(w, yx, Px);
                    Py = fmaf(w, yy, Py);
                    Pz = fmaf(w, yz, Pz);
                    Nx = fmaf(w, nx, Nx);
                    Ny = fmaf(w, ny, Ny);
                    Nz = fmaf(w, nz, Nz);
                    PN = fmaf(w, yx * nx + yy * ny + yz * nz, PN);
                    PP = fmaf(w, d2, PP);
                    nn += 1.f;
                }
            }
        }
        // sphere moments of the pixel's LPA lanes
        W = oct_sum(W);
        Px = oct_sum(Px);
        Py = oct_sum(Py);
        Pz = oct_sum(Pz);
        Nx = oct_sum(Nx);
        Ny = oct_sum(Ny);
        Nz = oct_sum(Nz);
        PN = oct_sum(PN);
        PP = oct_sum(PP);
        nn = oct_sum(nn);
        if (!live || sub != 0) continue;
        // lane 0 writes the slot: the projection when the fit succeeds, else the input
        double tn = in.t[k * S + pix];
        float on[3] = {in.n[(0 * KM + k) * S + pix], in.n[(1 * KM + k) * S + pix], in.n[(2 * KM + k) * S + pix]};
        apss_project(act && nn >= (float)p.m_min, W, Px, Py, Pz, Nx, Ny, Nz, PN, PP, h, h2, dz, tmax, tn, on);
        out.t[k * S + pix] = tn;
#pragma unroll
        for (int a = 0; a < 3; ++a) out.n[(a * KM + k) * S + pix] = on[a];
    }
}

// Reading (not in the paper): points of one pixel closer than d_merge bins in
// depth describe one surface; in depth order they merge into the
// intensity-weighted depth, summed intensity and weighted normal
// (merge_points).
// (m: only the pixels of its IRF class; d_merge in p is that class's)
__global__ __launch_bounds__(256) void k_merge(DevModel m, DevParams p, Shape sh, DevState s)
{
    const long long P = sh.P;
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= P || !in_class(m, pix)) return;
    int c = load_cnt(s.cnt, pix);
    if (c < 2) return;
    double t[KM];
    float r[KM], nx[KM], ny[KM], nz[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        if (k < c) {
            t[k] = s.t[k * P + pix];
            r[k] = s.r[k * P + pix];
            nx[k] = s.n[(0 * KM + k) * P + pix];
            ny[k] = s.n[(1 * KM + k) * P + pix];
            nz[k] = s.n[(2 * KM + k) * P + pix];
        }
    }
    merge_points(t, r, nx, ny, nz, c, p.d_merge);
    store_points(s, P, pix, t, r, nx, ny, nz, c);
}

hipError_t launch_apss_tiles(const DevModel& m, const DevParams& p, const Tiles& tg, DevState in, DevState out,
                             int only_above, bool carry, hipStream_t st)
{
    if (tg.n == 0 || tg.tile0[tg.n] == 0) return hipSuccess;
    if (p.persp > 0.0) {   // the host admits the perspective camera only where the tile fits
        const size_t lds = apss_tile_bytes(p.apss_R);
        if (lds > 65536 || p.apss_R > APSS_PINHOLE_R) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_apss_pinhole, dim3((unsigned)tg.tile0[tg.n]), dim3(PNT), pinhole_tile_bytes(p.apss_R),
                           st, m, p, tg, in, out, only_above, (int)carry);
        return hipGetLastError();
    }
    if (p.apss_Rs <= APSS_ROW) {
        hipLaunchKernelGGL(k_apss_tile, dim3((unsigned)tg.tile0[tg.n]), dim3(APT), apss_staged_bytes(p.apss_Rs), st, m, p, tg,
                           in, out, only_above, (int)carry);
        return hipGetLastError();
    }
    for (int g = 0; g < tg.n; ++g) {
        const Shape sh = group_shape(tg, g);
        hipLaunchKernelGGL(k_apss, dim3((unsigned)((sh.P * LPA + 255) / 256)), dim3(256), 0, st, m, p, sh,
                           state_at(in, tg.base[g]), state_at(out, tg.base[g]), only_above);
    }
    return hipGetLastError();
}

hipError_t launch_apss(const DevModel& m, const DevParams& p, const Shape& sh, DevState in, DevState out,
                       int only_above, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    return launch_apss_tiles(m, p, tiles_of(sh), in, out, only_above, true, st);
}

hipError_t launch_merge(const DevModel& m, const DevParams& p, const Shape& sh, DevState s, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_merge, dim3((unsigned)((sh.P + 255) / 256)), dim3(256), 0, st, m, p, sh, s);
    return hipGetLastError();
}

}  // namespace rt3d
