// rt3d_init.h -- sizes of the initialisation's dense search, shared by its
// kernels and the host code that builds its weight tables (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace rt3d {

constexpr int INIT_WAVES = 4;       // wavefronts per workgroup (fewer where their LDS areas are large)
constexpr int INIT_OCC = 5;         // workgroups per CU the registers allow
constexpr int INIT_T_MAX = 32768;   // bins the dense search covers (2048 blocks of 16 tau: a bit of 32 in each lane)
static_assert(INIT_T_MAX <= 16 * 64 * 32, "a mark per block");
constexpr int INIT_L_MAX = 3904;    // IRF bins the weight tables cover
constexpr int INIT_E_BITS = 7;      // low digit of e = 2^qshift qc - q (both digits up to 127: qshift up to 14)

// Steps of 64 bins that hold the L + 15 lags of a block of 16 tau.
inline __host__ __device__ int init_ks(int L) { return (L + 15 + 63) / 64; }

// Tiles of 16 blocks of 16 tau, rounded up to an odd number.
inline __host__ __device__ int init_stride(int T) { return ((((T + 15) >> 4) + 15) >> 4) | 1; }

// 16-byte chunks of the dense pool: what the last column's last step reads.
inline __host__ __device__ int init_chunks(int NS, int ks) { return 15 * NS + 4 * ((NS + 3) / 4) + 4 * ks; }

// LDS bytes of one wavefront: the dense pool (in one or two planes) and the
// block bounds (ks = 0: none), or the global-memory search's list ranges and
// block bounds.
inline size_t init_area(int T, int ks, int r_init, int planes)
{
    const size_t side = 2 * (size_t)r_init + 1;
    const size_t lists = 8 * (side * side + (size_t)(T + 63) / 64);
    const int NS = init_stride(T);
    const size_t dense = ks ? 16 * (size_t)planes * init_chunks(NS, ks) + 64 * (size_t)NS : 0;
    return ((lists > dense ? lists : dense) + 15) / 16 * 16;
}

// Bin counts and IRF lengths a context takes (E_UNSUPPORTED otherwise).  The
// interface's limit: long IRFs with many bins, whose weights, two tables of
// window maxima and per-wavefront bounds would pass 64 KB of LDS.
inline bool init_admits(int T, int L, int r_init)
{
    const size_t side = 2 * (size_t)r_init + 1, t = (size_t)T, l = (size_t)L;
    const size_t lists = side * side + (t + 63) / 64;
    const size_t pairs = ((l - 1 + 7) / 8 + 3) / 2;
    const size_t bounds = t <= 8192 ? pairs + (t + l - 2) / 16 + 304 + ((t + 31) / 32 + 3) / 4 : 0;
    const size_t weights = l <= INIT_L_MAX ? (l + 192 + 16 * pairs + 8 + 1) / 2 : 0;
    return 8 * (4 * (lists > bounds ? lists : bounds) + weights) <= 65536;
}

}  // namespace rt3d
