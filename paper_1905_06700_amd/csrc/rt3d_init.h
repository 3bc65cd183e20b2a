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
constexpr int INIT_LIST = 1024;     // pooled entries the list search stages, at most
constexpr int INIT_LONG_LIST = 4096;   // the same in the launch for larger pools
constexpr int LIST_PAD = 255;       // zeros on each side of the padded weights
constexpr int INIT_E_BITS = 7;      // low digit of e = 2^qshift qc - q (both digits up to 127: qshift up to 14)

// Steps of 64 bins that hold the L + 15 lags of a block of 16 tau.
constexpr __host__ __device__ int init_ks(int L) { return (L + 15 + 63) / 64; }

// Tiles of 16 blocks of 16 tau, rounded up to an odd number.
constexpr __host__ __device__ int init_stride(int T) { return ((((T + 15) >> 4) + 15) >> 4) | 1; }

// 16-byte chunks of the dense pool: what the last column's last step reads.
constexpr __host__ __device__ int init_chunks(int NS, int ks) { return 15 * NS + 4 * ((NS + 3) / 4) + 4 * ks; }

// LDS bytes of one wavefront: the dense pool (in one or two planes) and the
// block bounds; the list search's staged entries and block bounds.
constexpr size_t init_dense_area(int T, int ks, int planes)
{
    const int NS = init_stride(T);
    return 16 * (size_t)planes * init_chunks(NS, ks) + 64 * (size_t)NS;
}
constexpr size_t init_list_area(int T, int entries) { return 4 * (size_t)entries + 8 * (size_t)((T + 63) / 64); }

// Bin counts and IRF lengths a context takes (E_UNSUPPORTED otherwise).  A limit
// of the interface, kept as it was published: long IRFs with many bins, whose
// weights, two tables of window maxima and bounds of four wavefronts would pass
// 64 KB.  The launches themselves fit for any bin count and IRF length.
static_assert(init_dense_area(INIT_T_MAX, init_ks(INIT_L_MAX), 1) <= 65536, "a pool in one plane");
static_assert(init_list_area(65535, INIT_LONG_LIST) <= 65536, "a list");
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
