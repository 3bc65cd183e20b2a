// rt3d_points.h -- the denoisers' work on one point, over a tile staged in LDS:
// APSS moments under the orthographic map and the intensity low-pass.
// (k_apss.hip and k_filter.hip have the readings.)
//
// A tile's slot arrays are [KM][NS], a pixel's window SX apart by row; slots
// that hold no point are staged as no_depth(), so that no read waits on a
// count: the slots in reach are found first, all of a row's reads in
// flight together, then the few found are summed one by one in the window's
// order.
#pragma once
#include "rt3d_dev.h"

namespace rt3d {

constexpr int APSS_ROW = 5;   // widest halo: a row's slots, KM bits per pixel, in 64 bits
static_assert(KM * (2 * APSS_ROW + 1) <= 64, "a row's slots: a bit each");

// Lists the points of a tile of 256 pixels by pixel and slot (KM pixel + slot),
// so that a thread can take a point: thread x < 256 gives its pixel's count c,
// the others 0.  Every thread of the workgroup; returns the number of points,
// the list complete (left out when there are more than cap).
__device__ __forceinline__ int list_points(int c, int (&wave_points)[4], uint16_t* pl, int cap = KM * 256)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int place = (int)wave_incl_scan((uint32_t)c);
    if (w < 4 && lane == 63) wave_points[w] = place;
    place -= c;
    __syncthreads();
    int points = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        place += q < w ? wave_points[q] : 0;
        points += wave_points[q];
    }
    if (points > cap) return points;
    for (int k = 0; k < c; ++k) pl[place + k] = (uint16_t)(threadIdx.x * KM + k);
    __syncthreads();
    return points;
}

// The slots of pixels row - R .. row + R closer in depth than reach: bit
// KM (dj + R) + slot.
__device__ __forceinline__ uint64_t near_slots(const double* tl, int NS, int row, int R, double reach, double tq)
{
    uint64_t near = 0;
#pragma unroll 3
    for (int dj = -R; dj <= R; ++dj) {
        unsigned bits = 0;
#pragma unroll
        for (int k = 0; k < KM; ++k) bits |= fabs(tl[k * NS + row + dj] - tq) < reach ? 1u << k : 0u;
        near |= (uint64_t)bits << (KM * (dj + R));
    }
    return near;
}

struct Moments {
    float W, Px, Py, Pz, Nx, Ny, Nz, PN, PP, nn;
};

// A depth in reach of nothing and nearest to nothing.
__device__ __forceinline__ double no_depth() { return __builtin_nan(""); }

// The sphere moments of the point at depth tq of the pixel at xc: neighbours
// closer than h (h2 = h^2), R <= APSS_ROW.  (reach: 1.001 h / dz, an upper
// bound of the depth offset of a neighbour; the exact test follows.)
// normals(slot, di, dj, at, n): the normal of a slot of the window's pixel (di, dj),
// its place `at` in the slot's tile.
template <class Normals>
__device__ __forceinline__ Moments apss_moments(const double* tl, int NS, int SX, int xc, int R, float h2, float pxy,
                                                double dz, double reach, double tq, Normals normals)
{
    Moments s{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const float inv_h2 = 1.f / h2;
    for (int di = -R; di <= R; ++di) {
        const float yy = (float)di * pxy;
        const int row = xc + di * SX;
        uint64_t near = near_slots(tl, NS, row, R, reach, tq);
        int at = 0;
        double t2 = 0.0;
        float n[3] = {0.f, 0.f, 0.f};
        auto fetch = [&] {
            const int bit = __ffsll((unsigned long long)near) - 1, k = bit % KM;
            at = bit / KM - R;
            t2 = tl[k * NS + row + at];
            normals(k, di, at, row + at, n);
            near &= near - 1;
        };
        bool more = near != 0;
        if (more) fetch();
        while (more) {
            const float yx = (float)at * pxy, mx = n[0], my = n[1], mz = n[2];
            const float yz = (float)((t2 - tq) * dz);
            more = near != 0;
            if (more) fetch();
            const float dl = fmaf(yx, yx, yy * yy), d2 = fmaf(yz, yz, dl);
            if (dl < h2 && d2 < h2) {
                float a = 1.f - d2 * inv_h2;
                a = a * a;
                const float w = a * a;
                s.W += w;
                s.Px = fmaf(w, yx, s.Px);
                s.Py = fmaf(w, yy, s.Py);
                s.Pz = fmaf(w, yz, s.Pz);
                s.Nx = fmaf(w, mx, s.Nx);
                s.Ny = fmaf(w, my, s.Ny);
                s.Nz = fmaf(w, mz, s.Nz);
                s.PN = fmaf(w, fmaf(yz, mz, fmaf(yx, mx, yy * my)), s.PN);
                s.PP = fmaf(w, d2, s.PP);
                s.nn += 1.f;
            }
        }
    }
    return s;
}

// Normals staged as [3][KM][NS].
struct TileNormals {
    const float* nl;
    int NS;
    __device__ __forceinline__ void operator()(int k, int, int, int at, float (&n)[3]) const
    {
#pragma unroll
        for (int a = 0; a < 3; ++a) n[a] = nl[(a * KM + k) * NS + at];
    }
};

// The low-passed intensity of the point at depth tq, intensity r of the pixel
// at xc: the 8 surrounding pixels' nearest points (lowest slot on ties) closer
// than hi2 = h_int^2.  nside: surrounding pixels inside the image.
// ROWS: rows whose reads are in flight together.
template <int ROWS>
__device__ __forceinline__ float ifilter_mean(const double* tl, const float* rl, int NS, int SX, int xc, float hi2,
                                              float pxy, double dz, bool box, int nside, double tq, float r)
{
    float sum = r;
    int deg = 0;
#pragma unroll ROWS
    for (int di = -1; di <= 1; ++di) {
        const float dy = (float)di * pxy;
#pragma unroll
        for (int dj = -1; dj <= 1; ++dj) {
            if (di == 0 && dj == 0) continue;
            const float dx = (float)dj * pxy;
            const int x = xc + di * SX + dj;
            int best = 0;
            float bd = 0.f;
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                const float ddz = (float)((tl[k * NS + x] - tq) * dz);
                const float d2 = dx * dx + dy * dy + ddz * ddz;
                if (k == 0 || d2 < bd) {
                    best = k;
                    bd = d2;
                }
            }
            const bool hit = bd < hi2;
            sum += hit ? rl[best * NS + x] : 0.f;
            deg += hit ? 1 : 0;
        }
    }
    return sum / (float)(1 + (box ? nside : deg));
}

// Surrounding pixels of (i, j) inside a rows x cols image.
__device__ __forceinline__ int ifilter_sides(int i, int j, int rows, int cols)
{
    const int ni = 1 + (i > 0) + (i + 1 < rows), nj = 1 + (j > 0) + (j + 1 < cols);
    return ni * nj - 1;
}

}  // namespace rt3d
