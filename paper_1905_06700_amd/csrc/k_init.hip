// k_init.hip -- per-pixel initialisation (Methods: initialisation processes
// each pixel independently) as a log-matched filter, then initial normals.
//
// Reading of the initialisation: photons of the (2 r_init + 1)^2 window are
// pooled; the score L(tau) = sum z q[t - tau + o], q = log((h + eps)/eps) in
// 16-bit fixed point, is exact integer arithmetic, so its argmax does not
// depend on summation order.  Peaks are taken greedily (largest score,
// smallest tau on ties), each suppressing |tau - tau*| <= w_nms, while the
// window's unclaimed photons exceed the background expectation by kappa
// standard deviations (and n_min); an accepted peak claims the unclaimed bins
// of its window (5%..95% IRF mass) and later scores use unclaimed photons
// only.  Intensity = own photons in the claimed bins minus background over
// the IRF mass there; background = own photons outside the claimed bins.
//
// Mapping: one wavefront per pixel (several consecutive pixels in turn).  The
// window's rows are contiguous ranges of the photon lists (pixel-major CSR);
// their photons are added into a dense histogram of bytes in LDS, so the
// score of every tau is a contraction of that histogram with the weights: a
// Toeplitz product on the integer matrix cores.  With q = 2^k qc - e, qc =
// ceil(q / 2^k) <= 127 and 0 <= e < 2^k,
//   2^k sum z qc            bounds the score of every tau from above, and
//   2^k sum z qc - sum z e  is the score, exactly.
// One pass of the first product over all tau (v_mfma_i32_16x16x64_i8: 16 tau
// of 16 blocks against 64 bins per instruction) leaves the largest bound of
// every block of 16 tau in LDS; the search then takes the block with the
// largest bound, computes the exact scores of the 16 blocks around it (the
// second product, e in two digits), and stops once no remaining bound reaches
// the best score.  The gap between bound and score is about half of 2^k per
// photon in the IRF's support (1% of a peak's score): 1.15 such tiles are
// scored per peak sought on head-shaped scenes.  An accepted peak's bins drop to zero and
// the blocks that see them are bounded again (one tile).
//
// Bound by vector instruction issue (1,138 VALU instructions a pixel, 0.76 of
// the slots; 90 of them on the matrix cores, 57 for the bounds of 4613 bins and
// a 137-bin IRF).  32 head-shaped frames (636 k pixels, pools of 490 entries):
// 1.69 ms, where photon-by-photon bounds in LDS and scores on the vector ALU
// took 4.20 ms; 65 k pixels of 2000 bins with pools of 880 entries: 0.18
// against 1.29 ms.  Five workgroups per CU (96 VGPRs): four 1.89, six (spills)
// 1.77 ms.
//
// Pixels with more than 127 pooled photons in one bin are left to a second
// kernel, which holds the counts as two 7-bit digits in two planes of bytes
// and adds both planes' products.
//
// The dense pool costs the same however few photons it holds.  Sparse pools of
// long histograms or long IRFs (list_mean), and what the digits do not cover
// (IRFs over INIT_L_MAX bins, histograms over INIT_T_MAX bins, more than 16383
// photons in one bin, scores past 32 bits), take the list search: an exact
// branch and bound over the photon list, most of the time one of a dependent
// chain (pick a block, add its few entries' weights, compare).
#include "rt3d_dev.h"
#include "rt3d_init.h"
#include "rt3d_points.h"

namespace rt3d {

typedef int v4i __attribute__((ext_vector_type(4)));

// Accepted peaks of one pixel, held in scalar registers (every index below is
// a compile-time constant after unrolling, so nothing spills to scratch).
// Slots at or past n hold a tau no bin is near.
constexpr int NO_PEAK = -(1 << 28);

struct Peaks {
    int t[KM], w[KM];       // tau; unclaimed bins of its window when it was accepted
    int n;

    __device__ __forceinline__ void clear()
    {
        n = 0;
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            t[k] = NO_PEAK;
            w[k] = 0;
        }
    }

    // whether the window [t - wl, t + wr] of peak j holds bin tb (0 <= tb < T)
    __device__ __forceinline__ bool holds(const DevModel& m, int j, int tb) const
    {
        return (unsigned)(tb - (t[j] - m.wl)) <= (unsigned)(m.wl + m.wr);
    }

    // first accepted peak whose window holds bin tb, or -1
    __device__ __forceinline__ int owner(const DevModel& m, int tb) const
    {
        int ow = -1;
#pragma unroll
        for (int j = KM - 1; j >= 0; --j)
            if (j < n) ow = holds(m, j, tb) ? j : ow;
        return ow;
    }

    __device__ __forceinline__ bool claimed(const DevModel& m, int tb) const
    {
        bool any = false;
#pragma unroll
        for (int j = 0; j < KM; ++j)
            if (j < n) any = any || holds(m, j, tb);
        return any;
    }

    __device__ __forceinline__ bool suppressed(int tau, int wnms) const
    {
        bool any = false;
#pragma unroll
        for (int j = 0; j < KM; ++j)
            if (j < n) any = any || (unsigned)(tau - t[j] + wnms) <= (unsigned)(2 * wnms);
        return any;
    }

    // (wave-uniform values: kept in scalar registers)
    __device__ __forceinline__ void push(int tt, int ww)
    {
        tt = __builtin_amdgcn_readfirstlane(tt);
        ww = __builtin_amdgcn_readfirstlane(ww);
#pragma unroll
        for (int j = 0; j < KM; ++j)
            if (j == n) {
                t[j] = tt;
                w[j] = ww;
            }
        ++n;
    }
};

// A kernel's arguments, read through a pointer the compiler cannot see
// through: what a stage of the kernel needs is loaded (scalar, from the
// constant cache) where it is needed.  Loaded once for the whole kernel, the
// arguments would not fit the scalar registers beside the search's state and
// wait in vector lanes, an instruction per use.
struct InitArgs {
    DevModel m;
    DevParams p;
    Shape sh;
    const uint32_t* off;
    const uint32_t* ent;
    const float* gain;
    DevState s;
    int ppw;            // pixels per wavefront
    int area;           // LDS bytes of one wavefront
    uint32_t mean;      // k_init_lists: pooled entries of an average pixel up to which it takes any,
    uint32_t limit;     // and of the pixels it takes
    uint32_t cap;       // pooled entries the list search's LDS holds
    int left;           // only the pixels that the launch before left
    int wide;           // k_init_rest: two planes of bytes fit the wavefront's LDS
};

__device__ __forceinline__ const InitArgs& init_args()
{
    auto k = (const __attribute__((address_space(4))) InitArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return *(const InitArgs*)k;
}

// Orders LDS traffic between the lanes of one wavefront.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int popc_ballot(bool x) { return __popcll(__ballot(x)); }

__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c)
{
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// Maximum over the four rows of 16 lanes, column by column (every lane ends
// with its column's): the halves swapped, then the rows of each half.
__device__ __forceinline__ uint32_t rows_max(uint32_t v)
{
    auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = max(h[0], h[1]);
    auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return max(r[0], r[1]);
}

// The same for four values at once: row g of the lanes ends with the column
// maxima of v[g].
__device__ __forceinline__ uint32_t rows_max4(const uint32_t (&v)[4])
{
    auto a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    auto b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    auto r = __builtin_amdgcn_permlane16_swap(max(a[0], a[1]), max(b[0], b[1]), false, false);
    return max(r[0], r[1]);
}

__device__ __forceinline__ uint32_t max4(v4i d)
{
    return (uint32_t)max(max(d[0], d[1]), max(d[2], d[3]));
}

// Whole-wavefront sum, maximum and minimum: four moves inside the rows of 16
// lanes that have a source for every lane (quad permutations, half-row and
// row mirrors: one instruction each with the operation), then the rows and
// halves swapped.  Every lane must be active; the result is wave-uniform.
struct OpAdd { static __device__ __forceinline__ uint32_t f(uint32_t a, uint32_t b) { return a + b; } };
struct OpMax { static __device__ __forceinline__ uint32_t f(uint32_t a, uint32_t b) { return a > b ? a : b; } };
struct OpMin { static __device__ __forceinline__ uint32_t f(uint32_t a, uint32_t b) { return a < b ? a : b; } };

template <int CTRL>
__device__ __forceinline__ uint32_t row_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

template <class OP>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v)
{
    v = OP::f(v, row_move<0xB1>(v));
    v = OP::f(v, row_move<0x4E>(v));
    v = OP::f(v, row_move<0x141>(v));
    v = OP::f(v, row_move<0x140>(v));
    auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = OP::f(r[0], r[1]);
    auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)OP::f(h[0], h[1]));
}

constexpr int NO_TAU = 0x7fffffff;

// Scores: 32 bits where the caller has checked that they fit, else 64.
template <bool WIDE> struct ScoreOf { typedef uint32_t T; };
template <> struct ScoreOf<true> { typedef unsigned long long T; };

__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return wave_reduce<OpMax>(v); }
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v)
{
    const uint32_t hi = (uint32_t)(v >> 32), mh = wave_reduce<OpMax>(hi);
    return ((unsigned long long)mh << 32) | wave_reduce<OpMax>(hi == mh ? (uint32_t)v : 0u);
}

// One wavefront's dense pool and the matrix products over it.  KS: steps of
// 64 bins that hold a block's lags (L + 15 of them), or 0: m.ks of them, with
// the weights read from global memory.
//
// Pooled bin t is byte t + o of Z, so that block a (tau 16 a .. 16 a + 15)
// sees bytes 16 a .. 16 a + L + 14: row i of the weights' matrix holds
// q[kk - i] at kk, and lane (column j, group g) reads the 16-byte chunk
// a_j + g + 4 step.  Over all blocks, tile n takes blocks n + NS j (NS odd: 8
// neighbouring lanes then read 8 distinct bank groups), so that the chunks of
// tile n + 4 at one step are those of tile n at the next: each chunk is read
// once, into a rolling window of KS x 4 registers.  WIDE: a second plane
// of bytes, `plane` chunks on, holds the counts' multiples of 128 (KS = 0).
template <int KS, bool WIDE>
struct InitPool {
    static_assert(!WIDE || KS == 0, "two planes are built with the weights in global memory");
    typedef typename ScoreOf<WIDE>::T Score;
    int plane;
    v4i* Z;                 // the pool's bytes
    uint32_t* B;            // [16 NS] one plus the largest bound of each block, in units of 2^k
    const v4i* e;           // the digits of e: [2][KS][64] in LDS (KS > 0)
    const v4i* qa;          // the tables in global memory: [3][ks][64]
    int ks, NS, lane, j, g;
    v4i A[KS ? KS : 1];     // qc

    __device__ __forceinline__ uint8_t* bytes() const { return reinterpret_cast<uint8_t*>(Z); }

    // photons in byte x, and clearing it
    __device__ __forceinline__ uint32_t count(int x) const
    {
        return bytes()[x] + (WIDE ? 128u * bytes()[16 * plane + x] : 0u);
    }
    __device__ __forceinline__ void clear(int x) const
    {
        bytes()[x] = 0;
        if (WIDE) bytes()[16 * plane + x] = 0;
    }

    // d += A-operand a times chunk c (both planes)
    struct Acc {
        v4i lo, hi;
        __device__ __forceinline__ Acc() : lo{0, 0, 0, 0}, hi{0, 0, 0, 0} {}
        __device__ __forceinline__ v4i sum() const { return WIDE ? lo + (hi << 7) : lo; }
    };
    __device__ __forceinline__ void add(Acc& d, v4i a, int c) const
    {
        d.lo = mfma_i8(a, Z[c], d.lo);
        if (WIDE) d.hi = mfma_i8(a, Z[plane + c], d.hi);
    }

    // bounds of every block
    __device__ __forceinline__ void bound_all() const
    {
        const int NG = (NS + 3) >> 2, lb = NS * j + g;
        if constexpr (KS > 0) {
            v4i w[KS][4];
#pragma unroll
            for (int k = 0; k + 1 < KS; ++k)
#pragma unroll
                for (int c = 0; c < 4; ++c) w[k][c] = Z[lb + 4 * k + c];
            for (int b0 = 0; b0 < NG; b0 += KS) {
#pragma unroll
                for (int r = 0; r < KS; ++r) {
                    const int b = b0 + r;
                    if (b >= NG) break;
#pragma unroll
                    for (int c = 0; c < 4; ++c) w[(r + KS - 1) % KS][c] = Z[lb + 4 * (b + KS - 1) + c];
                    uint32_t v[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        v4i d = {0, 0, 0, 0};
#pragma unroll
                        for (int k = 0; k < KS; ++k) d = mfma_i8(A[k], w[(r + k) % KS][c], d);
                        v[c] = max4(d);
                    }
                    store4(b, v);
                }
            }
        } else {
            // (two groups of four tiles per read of the weights, where the registers allow)
            constexpr int G = WIDE ? 1 : 2;
            for (int b0 = 0; b0 < NG; b0 += G) {
                Acc d[G][4];
                int at[G];
#pragma unroll
                for (int u = 0; u < G; ++u) at[u] = lb + 4 * min(b0 + u, NG - 1);
#pragma unroll 2
                for (int k = 0; k < ks; ++k) {
                    const v4i a = qa[k * 64 + lane];
#pragma unroll
                    for (int u = 0; u < G; ++u)
#pragma unroll
                        for (int c = 0; c < 4; ++c) add(d[u][c], a, at[u] + 4 * k + c);
                }
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const uint32_t v[4] = {max4(d[u][0].sum()), max4(d[u][1].sum()), max4(d[u][2].sum()),
                                           max4(d[u][3].sum())};
                    store4(min(b0 + u, NG - 1), v);
                }
            }
        }
    }

    __device__ __forceinline__ void store4(int b, const uint32_t (&v)[4]) const
    {
        const uint32_t u = rows_max4(v);
        const int n = 4 * b + g;
        if (n < NS) B[n + NS * j] = u + 1u;
    }

    // bounds of the blocks a0 .. a0 + 15 again
    __device__ __forceinline__ void bound_tile(int a0) const
    {
        Acc d;
        const int at = a0 + j + g;
        if constexpr (KS > 0) {
#pragma unroll
            for (int k = 0; k < KS; ++k) add(d, A[k], at + 4 * k);
        } else {
            for (int k = 0; k < ks; ++k) add(d, qa[k * 64 + lane], at + 4 * k);
        }
        const uint32_t u = rows_max(max4(d.sum()));
        if (g == 0) B[a0 + j] = u + 1u;
    }

    // exact scores of tau 16 (a0 + j) + 4 g + r, r = 0..3 (one plane: modulo
    // 2^32, the caller has checked that they fit)
    __device__ __forceinline__ void score_tile(int a0, int qshift, Score (&sc)[4]) const
    {
        Acc ac, a1, a2;
        const int at = a0 + j + g;
        if constexpr (KS > 0) {
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                add(ac, A[k], at + 4 * k);
                add(a1, e[k * 64 + lane], at + 4 * k);
                add(a2, e[(KS + k) * 64 + lane], at + 4 * k);
            }
        } else {
            for (int k = 0; k < ks; ++k) {
                add(ac, qa[k * 64 + lane], at + 4 * k);
                add(a1, qa[(ks + k) * 64 + lane], at + 4 * k);
                add(a2, qa[(2 * ks + k) * 64 + lane], at + 4 * k);
            }
        }
        const v4i dc = ac.sum(), d1 = a1.sum(), d0 = a2.sum();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            sc[r] = ((Score)(uint32_t)dc[r] << qshift) - ((Score)(uint32_t)d1[r] << INIT_E_BITS) - (Score)(uint32_t)d0[r];
    }
};

// The window's photons: row r's entries are [rs, re) of lane r.
struct PoolRows {
    uint32_t rs, re;
    int side;
    const uint32_t* ent;
};

// Adds the pooled photons into the dense pool (cleared here); nt gains this
// lane's photons.  Returns whether a byte passed 127: the byte that first does
// so still holds at most 255 (counts go in as at most 128), and the lane that
// adds to it sees that in the value it replaced, so no overflow goes unseen.
// Three rows of four chunks of 64 entries are in flight at a time.
template <int KS>
__device__ __forceinline__ bool fill_pool(const InitPool<KS, false>& P, const PoolRows& W, int T, int o, uint32_t& nt)
{
    const int lane = P.lane;
    const int nz = init_chunks(P.NS, KS ? KS : P.ks);
    for (int x = lane; x < nz; x += 64) P.Z[x] = (v4i){0, 0, 0, 0};
    wave_sync();
    uint32_t* Zw = reinterpret_cast<uint32_t*>(P.Z);
    uint32_t most = 0;
    for (int r0 = 0; r0 < W.side; r0 += 3) {
        uint32_t a[3], n[3], len = 0;
#pragma unroll
        for (int r = 0; r < 3; ++r) {       // (lanes past the rows hold empty ranges)
            a[r] = (uint32_t)__builtin_amdgcn_readlane((int)W.rs, r0 + r);
            n[r] = (uint32_t)__builtin_amdgcn_readlane((int)W.re, r0 + r) - a[r];
            len = max(len, n[r]);
        }
        for (uint32_t c0 = 0; c0 < len; c0 += 256) {
            uint32_t v[3][4];
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    v[r][u] = 0xffff0000u;                             // (a bin past every histogram)
                    if (c0 + 64 * u < n[r]) {                          // (uniform)
                        const uint32_t x = c0 + 64 * u + lane;
                        if (x < n[r]) v[r][u] = W.ent[a[r] + x];
                    }
                }
            uint32_t old[3][4];
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    old[r][u] = 0;
                    if (!(c0 + 64 * u < n[r])) continue;               // (uniform)
                    const int t = ent_bin(v[r][u]);
                    const uint32_t z = (uint32_t)ent_cnt(v[r][u]);
                    if (t >= T) continue;
                    nt += z;
                    const uint32_t zs = min(z, 128u);
                    const int x = t + o;
                    const int sh = (x & 3) << 3;
                    old[r][u] = ((atomicAdd(&Zw[x >> 2], zs << sh) >> sh) & 0xffu) + zs;
                }
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int u = 0; u < 4; ++u) most = max(most, old[r][u]);
        }
    }
    wave_sync();
    return __ballot(most > 127u) != 0ull;
}

// The same into two planes, pixel by pixel of the window (the bins of one
// pixel's list are distinct, so no two lanes meet in a byte and a byte holds at
// most 254 before its 128 moves to the upper plane).  Returns whether a bin
// passed 16383 photons.
__device__ __forceinline__ bool fill_planes(const InitPool<0, true>& P, const PoolRows& W, const uint32_t* off,
                                            long long base, int cols, int i, int j, int rows, int T, int o, uint32_t& nt)
{
    const int lane = P.lane, R = W.side >> 1;
    for (int x = lane; x < 2 * P.plane; x += 64) P.Z[x] = (v4i){0, 0, 0, 0};
    wave_sync();
    uint32_t* lo = reinterpret_cast<uint32_t*>(P.Z);
    uint32_t* hi = reinterpret_cast<uint32_t*>(P.Z + P.plane);
    bool over = false;
    for (int di = max(-R, -i); di <= min(R, rows - 1 - i); ++di)
        for (int dj = max(-R, -j); dj <= min(R, cols - 1 - j); ++dj) {
            const uint32_t* q = off + base + (long long)di * cols + dj;
            const uint32_t e0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)q[0]);
            const uint32_t e1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)q[1]);
            for (uint32_t x0 = e0; x0 < e1; x0 += 64) {
                const uint32_t v = x0 + lane < e1 ? W.ent[x0 + lane] : 0xffff0000u;
                const int t = ent_bin(v);
                const uint32_t z = (uint32_t)ent_cnt(v);
                if (t < T) {
                    nt += z;
                    const int x = t + o, sh = (x & 3) << 3;
                    const uint32_t zl = z & 127u;
                    const bool carry = ((atomicAdd(&lo[x >> 2], zl << sh) >> sh) & 0xffu) + zl > 127u;
                    if (carry) atomicSub(&lo[x >> 2], 128u << sh);
                    const uint32_t zh = min((z >> 7) + (carry ? 1u : 0u), 128u);
                    if (zh) over = over || ((atomicAdd(&hi[x >> 2], zh << sh) >> sh) & 0xffu) + zh > 127u;
                }
            }
            wave_sync();
        }
    return __ballot(over) != 0ull;
}

// The unscored block with the largest bound: the bounds of blocks lane + 64 u
// in registers (u < PICK_REGS; 0: scored or past the last block), reloaded
// every round.
constexpr int PICK_REGS = 8;

struct PickRegs {
    uint32_t v[PICK_REGS];

    __device__ __forceinline__ void load(const uint32_t* B, int nblk, int lane)
    {
#pragma unroll
        for (int u = 0; u < PICK_REGS; ++u) {
            v[u] = 0;
            if (64 * u < nblk) {                         // (uniform)
                const uint32_t x = B[min(lane + 64 * u, nblk - 1)];
                v[u] = lane + 64 * u < nblk ? x : 0u;
            }
        }
    }

    // whether some bound plus one is above thr
    __device__ __forceinline__ bool above(uint32_t thr) const { return __ballot(most() > thr) != 0ull; }

    // the largest bound plus one (0: none is left) and its block
    __device__ __forceinline__ uint32_t pick(int& block) const
    {
        const uint32_t mx = wave_reduce<OpMax>(most());
        block = 0;
#pragma unroll
        for (int u = PICK_REGS - 1; u >= 0; --u) {
            const unsigned long long hit = __ballot(v[u] == mx);
            block = hit ? 64 * u + __builtin_ctzll(hit) : block;
        }
        return mx;
    }

    __device__ __forceinline__ uint32_t most() const
    {
        uint32_t key = 0;
#pragma unroll
        for (int u = 0; u < PICK_REGS; ++u) key = max(key, v[u]);
        return key;
    }

    // blocks d0 .. d0 + n - 1 are scored (n <= 16)
    __device__ __forceinline__ void mark(int d0, int n, int lane)
    {
#pragma unroll
        for (int u = 0; u < PICK_REGS; ++u)
            if (u == d0 >> 6 || u == (d0 + n - 1) >> 6) {  // (uniform)
                if ((unsigned)(lane + 64 * u - d0) < (unsigned)n) v[u] = 0;
            }
    }
};

// The same for any number of blocks, from LDS with a bit per block.
struct PickLoop {
    const uint32_t* B;
    int nblk, lane;
    uint32_t done;          // bit u: block lane + 64 u scored (u < 32: INIT_T_MAX)

    __device__ __forceinline__ void load(const uint32_t* b, int n, int l)
    {
        B = b;
        nblk = n;
        lane = l;
        done = 0;
    }

    __device__ __forceinline__ uint32_t most(int& kb) const
    {
        uint32_t key = 0;
        kb = 0;
        for (int u = 0, b = lane; b < nblk; ++u, b += 64) {
            const uint32_t v = (done >> u) & 1u ? 0u : B[b];
            if (v > key) {
                key = v;
                kb = b;
            }
        }
        return key;
    }

    __device__ __forceinline__ bool above(uint32_t thr) const
    {
        int kb;
        return __ballot(most(kb) > thr) != 0ull;
    }

    __device__ __forceinline__ uint32_t pick(int& block) const
    {
        int kb;
        const uint32_t key = most(kb);
        const uint32_t mx = wave_reduce<OpMax>(key);
        block = __builtin_amdgcn_readlane(kb, __builtin_ctzll(__ballot(key == mx)));
        return mx;
    }

    __device__ __forceinline__ void mark(int d0, int n, int)
    {
        // (a tile's blocks past the last one have no mark: a 33rd with 32768 bins)
        const int d1 = min(d0 + n, nblk) - 1, u = (d1 - lane) >> 6;   // the last block of this lane at or below d1
        if (d1 >= lane && lane + 64 * u >= d0) done |= 1u << u;
    }
};

template <bool REGS> struct PickOf { typedef PickRegs T; };
template <> struct PickOf<false> { typedef PickLoop T; };

// d * d >= k2 * bw and d >= 0 for d = nwin - bw, bw = ntot * win / T, as the
// FP64 expressions decide: first in FP32, whose error is below 1e-6 of the
// terms, and in FP64 where that is too close.
__device__ __forceinline__ bool stands_out(uint32_t nwin, uint32_t ntot, int win, int T, double kappa)
{
    const float bwf = (float)ntot * (float)win * __builtin_amdgcn_rcpf((float)T);
    const float df = (float)nwin - bwf, big = (float)nwin + bwf;
    const float k2f = (float)kappa * (float)kappa;
    const float l = df * df, r = k2f * bwf, tol = 1e-4f * (big * big + r);
    const bool yes = df > 1e-4f * big && l > r + tol, no = df < -1e-4f * big || l < r - tol;
    if (__builtin_amdgcn_readfirstlane((int)(yes || no))) return __builtin_amdgcn_readfirstlane((int)yes) != 0;
    const double bw = (double)ntot * (double)win / (double)T;
    const double d = (double)nwin - bw;
    const double k2 = kappa * kappa;
    return d >= 0.0 && d * d >= k2 * bw;
}

// The search over the dense pool.  The caller has checked that the scores fit
// their type: ntot x the largest weight below 2^32 - 1 with one plane.
template <int KS, bool WIDE>
__device__ __forceinline__ void dense_search(const InitPool<KS, WIDE>& P, uint32_t ntot, Peaks& pk)
{
    const int lane = P.lane;
    P.bound_all();
    wave_sync();
    typename PickOf<(KS > 0)>::T pick;
    for (int it = 0;; ++it) {
        const InitArgs& A = init_args();
        const DevModel& m = A.m;
        const int T = m.T, o = m.o, nblk = (T + 15) >> 4, a0max = 16 * P.NS - 16;
        const int up = m.qshift;
        pick.load(P.B, nblk, lane);
        typedef typename InitPool<KS, WIDE>::Score Score;
        Score best = 0;
        int bestt = NO_TAU;
        int bb = 0;
        while (pick.pick(bb) != 0) {
            // exact scores of the blocks around it (one tile), plus one (0: past
            // the last bin or under a peak's suppression)
            int st = NO_TAU;
            const int d0 = min(max(bb - 8, 0), a0max);
            constexpr Score NONE = ~(Score)0;
            Score sc[4], sk = 0;
            P.score_tile(d0, m.qshift, sc);
            const int t0 = 16 * (d0 + P.j) + 4 * P.g;
            if (16 * d0 + 255 >= T) {
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[r] = t0 + r < T ? sc[r] : NONE;
            }
#pragma unroll
            for (int k = 0; k < KM; ++k)
                if (k < pk.n && (unsigned)(pk.t[k] + m.wnms - 16 * d0) <= (unsigned)(255 + 2 * m.wnms)) {
                    const int x = t0 - pk.t[k] + m.wnms;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        sc[r] = (unsigned)(x + r) <= (unsigned)(2 * m.wnms) ? NONE : sc[r];
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                ++sc[r];
                sk = max(sk, sc[r]);
            }
            pick.mark(d0, 16, lane);
            const Score smx = wave_max(sk);
            if (smx != 0) {
                // the first tau that reaches it
                int tk = NO_TAU;
#pragma unroll
                for (int r = 3; r >= 0; --r) tk = sc[r] == smx ? t0 + r : tk;
                const unsigned long long hit = __ballot(sk == smx);
                st = hit & (hit - 1ull) ? (int)wave_reduce<OpMin>((uint32_t)tk)
                                        : __builtin_amdgcn_readlane(tk, __builtin_ctzll(hit));
            }
            if (smx != 0 && (bestt == NO_TAU || smx - 1 > best || (smx - 1 == best && st < bestt))) {
                best = smx - 1;
                bestt = st;
            }
            // a block whose bound is at least best may still reach (or tie) it:
            // bound 2^up >= best, i.e. bound + 1 > ceil(best / 2^up)
            const uint32_t thr = (uint32_t)(((unsigned long long)best + ((1ull << up) - 1ull)) >> up);
            if (bestt != NO_TAU && !pick.above(thr)) break;
        }
        if (bestt == NO_TAU) break;          // every tau suppressed
        const int a = max(0, bestt - m.wl), c = min(T - 1, bestt + m.wr);
        int win = 0;
        uint32_t nwin = 0;                                      // at most ntot
        for (int t0 = a; t0 <= c; t0 += 64) {
            const int tb = t0 + lane;
            const bool open = tb <= c && !pk.claimed(m, tb);
            win += popc_ballot(open);
            if (open) nwin += P.count(tb + o);
        }
        nwin = wave_reduce<OpAdd>(nwin);
        if (!(win > 0 && (long long)nwin >= A.p.n_min && stands_out(nwin, ntot, win, T, A.p.kappa))) break;
        pk.push(bestt, win);
        if (it + 1 >= A.p.k_init) break;
        // the peak claims the photons of its window, and the blocks that see
        // those bins are bounded afresh
        for (int tb = a + lane; tb <= c; tb += 64) P.clear(tb + o);
        wave_sync();
        const int b0 = max(0, a + o - m.L + 1) >> 4, b1 = min(T - 1, c + o) >> 4;
        for (int x = b0; x <= b1; x += 16) P.bound_tile(min(x, a0max));
        wave_sync();
    }
}

// The search over the photon list: an exact branch and bound over blocks of 64
// tau, one per lane.  The bound of a block, sum z x the largest weight of the 64
// lags a photon's bin can have in it, is added up in LDS; blocks are scored
// exactly in decreasing bound order until no remaining bound can beat (or tie
// at a smaller tau) the best score.  A score takes the entries in reach one by
// one (their lanes from a ballot over 64 entries), each lane's weight one read
// of the padded table.  STAGED: the entries, n of them, are in LDS, and an
// accepted peak's photons leave them and the bounds; else they are read from
// memory, row by row of the window, for every block.  The scores fit the type.
// LIST_BLOCKS blocks are scored at once, LIST_TAKE entries in flight: 10 k
// pixels, pools of 200 entries of 8192 bins, a 2001-bin IRF 287 us against 434
// us for one block and four entries; of 20000 bins, a 19-bin IRF 462 against
// 393 us.
constexpr int LIST_BLOCKS = 4, LIST_TAKE = 2;
static_assert(64 * LIST_BLOCKS - 1 <= LIST_PAD, "the weights' zeros reach over the blocks");

template <class Score, bool STAGED>
__device__ __forceinline__ void list_search(const PoolRows& W, uint32_t* list, uint32_t n, Score* ub, Peaks& pk)
{
    const InitArgs& A = init_args();
    const DevModel& m = A.m;
    const int T = m.T, L = m.L, o = m.o, nb = (T + 63) >> 6, lane = threadIdx.x & 63;
    const int32_t* q = m.q;
    const int32_t* qwin = m.qwin;
    // f(entry, its place), 64 at a time; places past the end hold bin 65535
    auto each = [&](auto f) {
        if constexpr (STAGED) {
            for (uint32_t x = lane; x - lane < n; x += 64) f(x < n ? list[x] : 0xffff0000u, x);
        } else {
            for (int r = 0; r < W.side; ++r) {
                const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)W.rs, r);
                const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)W.re, r);
#pragma unroll 4
                for (uint32_t x = a; x < b; x += 64) f(x + lane < b ? W.ent[x + lane] : 0xffff0000u, 0u);
            }
        }
    };
    // the bins of the staged entries 64 lane .. 64 lane + 63 (a pixel's are in
    // order: most of its chunks are out of a block's reach)
    int first = 0, last = -1;
    if (STAGED)
        each([&](uint32_t v, uint32_t x) {
            const uint32_t t = (uint32_t)ent_bin(v);
            const uint32_t a = wave_reduce<OpMin>(t), b = wave_reduce<OpMax>(t < (uint32_t)T ? t : 0u);
            const bool here = (uint32_t)lane == (x - lane) >> 6;
            first = here ? (int)a : first;
            last = here ? (int)b : last;
        });
    // the same for entries of bins lo .. hi at least
    auto each_in = [&](int lo, int hi, auto f) {
        if constexpr (STAGED) {
            for (unsigned long long c = __ballot(first <= hi && last >= lo); c; c &= c - 1) {
                const uint32_t x = 64u * (uint32_t)__builtin_ctzll(c) + lane;
                f(x < n ? list[x] : 0xffff0000u, x);
            }
        } else {
            each(f);
        }
    };
    // adds an entry's terms to the bounds (or takes them away)
    auto bound = [&](uint32_t v, bool away) {
        const int t = ent_bin(v);
        if (t >= T) return;
        const Score z = (Score)(uint32_t)ent_cnt(v);
        const int b0 = max(0, t + o - L + 1) >> 6, b1 = min(T - 1, t + o) >> 6;
        for (int b = b0; b <= b1; ++b) {
            const Score w = z * (Score)(uint32_t)qwin[t + o - 64 * b];
            atomicAdd(&ub[b], away ? (Score)0 - w : w);
        }
    };
    unsigned long long nt = 0;
    for (int b = lane; b < nb; b += 64) ub[b] = 0;
    wave_sync();
    each([&](uint32_t v, uint32_t) {
        bound(v, false);
        nt += ent_bin(v) < T ? (uint32_t)ent_cnt(v) : 0u;
    });
    const long long ntot = wave_sum((long long)nt);
    wave_sync();
    for (int it = 0; it < A.p.k_init; ++it) {
        Score best = 0;
        int bestt = NO_TAU;
        uint32_t done = 0;                      // bit u: block lane + 64 u scored in this round
        while (true) {
            // the unscored block with the largest bound (the first on ties)
            Score bu = 0;
            int bb = NO_TAU;
            for (int u = 0; lane + 64 * u < nb; ++u) {
                if ((done >> u) & 1u) continue;
                const Score x = ub[lane + 64 * u];
                if (bb == NO_TAU || x > bu) {
                    bu = x;
                    bb = lane + 64 * u;
                }
            }
            const Score mx = wave_max(bu);
            bb = (int)wave_reduce<OpMin>((uint32_t)(bu == mx ? bb : NO_TAU));
            if (bb == NO_TAU) break;
            if (bestt != NO_TAU && (mx < best || (mx == best && (bb << 6) > bestt))) break;
            // exact scores of LIST_BLOCKS blocks around it
            const int s0 = max(0, min(bb - LIST_BLOCKS / 2, nb - LIST_BLOCKS)), lo = 64 * s0 - o;
            const int hi = lo + 64 * LIST_BLOCKS - 1 + L - 1;
            const int32_t* ql = q + LIST_PAD - lo - lane;  // lag t - tau + o of this lane's first tau
            Score sc[LIST_BLOCKS] = {};
            unsigned long long in;
            uint32_t v;
            auto take = [&] {                              // the next few entries' terms
                constexpr int N = LIST_TAKE;
                int tt[N], zz[N], w[N][LIST_BLOCKS];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)v, in ? __builtin_ctzll(in) : 0);
                    tt[u] = in ? ent_bin(e) : lo;
                    zz[u] = in ? ent_cnt(e) : 0;
                    in &= in - 1;
                }
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int k = 0; k < LIST_BLOCKS; ++k) w[u][k] = ql[tt[u] - 64 * k];
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int k = 0; k < LIST_BLOCKS; ++k)
                        sc[k] += sizeof(Score) == 4 ? (Score)__umul24(zz[u], w[u][k])
                                                    : (Score)(uint32_t)zz[u] * (Score)(uint32_t)w[u][k];
            };
            each_in(lo, hi, [&](uint32_t e, uint32_t) {
                const int t = ent_bin(e);
                v = e;
                in = __ballot(t >= lo && t <= hi && t < T && (STAGED || !pk.claimed(m, t)));
                while (in) take();
            });
            Score sk = 0, smx;
            int tk = NO_TAU;
#pragma unroll
            for (int k = 0; k < LIST_BLOCKS; ++k) {
                const int b = s0 + k, tau = 64 * b + lane;
                if (b < nb && lane == (b & 63)) done |= 1u << (b >> 6);
                const Score x = tau < T && !pk.suppressed(tau, m.wnms) ? sc[k] + 1 : 0;      // (0: none)
                tk = x > sk ? tau : tk;
                sk = max(sk, x);
            }
            smx = wave_max(sk);
            const int st = (int)wave_reduce<OpMin>((uint32_t)(sk == smx ? tk : NO_TAU));
            if (smx != 0 && (bestt == NO_TAU || smx - 1 > best || (smx - 1 == best && st < bestt))) {
                best = smx - 1;
                bestt = st;
            }
        }
        if (bestt == NO_TAU) break;             // every tau suppressed
        const int a = max(0, bestt - m.wl), c = min(T - 1, bestt + m.wr);
        int win = 0;
        for (int tb = a + lane; tb <= c; tb += 64) win += !pk.claimed(m, tb);
        win = wave_sum(win);
        unsigned long long nw = 0;
        each_in(a, c, [&](uint32_t v, uint32_t) {
            const int t = ent_bin(v);
            if (t >= a && t <= c && (STAGED || !pk.claimed(m, t))) nw += (uint32_t)ent_cnt(v);
        });
        const long long nwin = wave_sum((long long)nw);
        const double bw = (double)ntot * (double)win / (double)T;
        const double d = (double)nwin - bw;
        const double k2 = A.p.kappa * A.p.kappa;
        if (!(win > 0 && nwin >= A.p.n_min && d >= 0.0 && d * d >= k2 * bw)) break;
        pk.push(bestt, win);
        if (STAGED && it + 1 < A.p.k_init) {
            each_in(a, c, [&](uint32_t v, uint32_t x) {
                const int t = ent_bin(v);
                if (t < a || t > c) return;
                bound(v, true);
                list[x] = 0xffff0000u;
            });
            wave_sync();
        }
    }
}

// The same for a window of n entries, area its LDS.
__device__ __forceinline__ void list_search_any(const PoolRows& W, uint32_t n, v4i* area, Peaks& pk)
{
    const InitArgs& A = init_args();
    unsigned long long* ub = reinterpret_cast<unsigned long long*>(area);
    uint32_t* list = reinterpret_cast<uint32_t*>(ub + ((A.m.T + 63) >> 6));
    if (n > A.cap) {
        list_search<unsigned long long, false>(W, list, n, ub, pk);
        return;
    }
    // the rows side by side, three rows' first entries in flight at a time
    const int lane = threadIdx.x & 63, T = A.m.T;
    const uint32_t len = W.re - W.rs, at = wave_incl_scan(len) - len;
    uint32_t nt = 0;                            // (at most 4096 x 65535)
    for (int r0 = 0; r0 < W.side; r0 += 3) {
        uint32_t a[3], k[3], d[3], v[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            a[r] = (uint32_t)__builtin_amdgcn_readlane((int)W.rs, r0 + r);
            k[r] = (uint32_t)__builtin_amdgcn_readlane((int)len, r0 + r);
            d[r] = (uint32_t)__builtin_amdgcn_readlane((int)at, r0 + r);
            v[r] = (uint32_t)lane < k[r] ? W.ent[a[r] + lane] : 0u;
        }
#pragma unroll
        for (int r = 0; r < 3; ++r)
            for (uint32_t x = lane; x < k[r]; x += 64) {
                if (x >= 64) v[r] = W.ent[a[r] + x];
                list[d[r] + x] = v[r];
                nt += ent_bin(v[r]) < T ? (uint32_t)ent_cnt(v[r]) : 0u;
            }
    }
    wave_sync();
    const uint32_t ntot = wave_reduce<OpAdd>(nt);
    if (A.m.qmax < 1 << 24 && (unsigned long long)ntot * (unsigned long long)A.m.qmax <= 0xfffffffeull)
        list_search<uint32_t, true>(W, list, n, reinterpret_cast<uint32_t*>(ub), pk);
    else
        list_search<unsigned long long, true>(W, list, n, ub, pk);
}

// The peaks of the wavefront's pixels, pixel x's peak k in lane 4 x + k, from
// which finish() makes the initial states of all of them at once (the sixteen
// FP64 divisions and the scattered stores of one pixel would otherwise keep
// four lanes busy).
constexpr int INIT_PPW_MAX = 16;
enum : int { PIX_NONE = 0, PIX_LIVE = 1, PIX_DEAD = 2, PIX_LEFT = 3 };
constexpr uint8_t INIT_LEFT = 255;   // the count of a pixel k_init leaves to k_init_rest

struct InitRecords {
    int t, w, mode;         // tau and window of the lane's peak; the pixel's mode
    uint32_t nown, zp;      // own photons in the peak's window; all own photons
    float G;
    double H;               // IRF mass in the window

    __device__ __forceinline__ void clear()
    {
        t = w = mode = 0;
        nown = zp = 0;
        G = 1.f;
        H = 0.0;
    }

    __device__ __forceinline__ void set_mode(int x, int md)
    {
        if ((int)((threadIdx.x & 63) >> 2) == x) mode = md;
    }

    // pixel x's accepted peaks: v0 the first 64 of its own entries e0 .. e1 - 1
    __device__ __forceinline__ void set(int x, const Peaks& pk, float g, uint32_t v0, uint32_t e0, uint32_t e1,
                                        double hfull)
    {
        const InitArgs& A = init_args();
        const DevModel& m = A.m;
        const int lane = threadIdx.x & 63;
        // own photons: total and per claimed window
        // (a pixel holds at most 65535 entries, each count below 65536: the
        // sums fit 32 bits)
        uint32_t z = 0, n[KM] = {0, 0, 0, 0};
        uint32_t v = e0 + lane < e1 ? v0 : 0u;
        for (uint32_t e = e0;;) {
            const uint32_t zv = (uint32_t)ent_cnt(v);
            z += zv;
            if (pk.n > 0) {
                const int ow = pk.owner(m, ent_bin(v));
#pragma unroll
                for (int k = 0; k < KM; ++k)
                    if (k < pk.n) n[k] += ow == k ? zv : 0u;
            }
            e += 64;
            if (e >= e1) break;
            v = e + lane < e1 ? A.ent[e + lane] : 0u;
        }
        if (__ballot(z >= 1024u) == 0ull) {                    // sums below 65536: two per word
            const uint32_t s0 = wave_reduce<OpAdd>(z | (n[0] << 16));
            z = s0 & 0xffffu;
            n[0] = s0 >> 16;
            if (pk.n > 1) {
                const uint32_t s1 = wave_reduce<OpAdd>(n[1] | (n[2] << 16));
                n[1] = s1 & 0xffffu;
                n[2] = s1 >> 16;
            }
            if (pk.n > 3) n[3] = wave_reduce<OpAdd>(n[3]);
        } else {
            z = wave_reduce<OpAdd>(z);
#pragma unroll
            for (int k = 0; k < KM; ++k)
                if (k < pk.n) n[k] = wave_reduce<OpAdd>(n[k]);
        }
        const bool here = (lane >> 2) == x;
        mode = here ? PIX_LIVE : mode;
        zp = here ? z : zp;
        G = here ? g : G;
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k < pk.n) {
                double h = hfull;
                if (pk.w[k] != m.wl + m.wr + 1) {     // clipped, or bins claimed before it
                    const int a = max(0, pk.t[k] - m.wl), c = min(m.T - 1, pk.t[k] + m.wr);
                    double hs = 0.0;
                    for (int tb = a + lane; tb <= c; tb += 64) {
                        const int idx = tb - pk.t[k] + m.o;
                        if (pk.owner(m, tb) == k && idx >= 0 && idx < m.L) hs += m.hbar[idx];
                    }
                    h = wave_sum(hs);
                }
                const bool me = lane == 4 * x + k;
                t = me ? pk.t[k] : t;
                w = me ? pk.w[k] : w;
                nown = me ? n[k] : nown;
                H = me ? h : H;
            }
    }

    // writes the states of pixels first .. first + 15 as far as they are set
    __device__ __forceinline__ void finish(uint32_t first) const
    {
        const InitArgs& A = init_args();
        const long long S = A.sh.S;
        const int lane = threadIdx.x & 63, k = lane & 3;
        const long long pix = (long long)first + (lane >> 2);
        const long long num = max((long long)zp - (long long)quad_sum_u32(nown), 0ll);
        const int den = A.m.T - (int)quad_sum_u32((uint32_t)w);
        // (all below 2^32: exact as doubles, and so are their products)
        const double fnum = (double)num, fden = (double)den, fw = (double)w, nwk = (double)nown;
        // the kept peaks take the slots in ascending depth (depths are
        // distinct): a peak's slot is the number of kept peaks above it; the
        // other lanes clear the slots past the kept ones
        bool keep = w > 0 && (den > 0 ? (nwk * fden > fnum * fw) : (nwk > 0.0)) && H > 0.0;
        const int kt = keep ? t : 0x7fffffff;
        const uint32_t kept = (uint32_t)(__ballot(keep) >> (lane & ~3)) & 15u;
        int rank = 0;
        rank += __builtin_amdgcn_update_dpp(0, kt, 0x00, 0xF, 0xF, true) < kt ? 1 : 0;
        rank += __builtin_amdgcn_update_dpp(0, kt, 0x55, 0xF, 0xF, true) < kt ? 1 : 0;
        rank += __builtin_amdgcn_update_dpp(0, kt, 0xAA, 0xF, 0xF, true) < kt ? 1 : 0;
        rank += __builtin_amdgcn_update_dpp(0, kt, 0xFF, 0xF, 0xF, true) < kt ? 1 : 0;
        int nkeep = __builtin_popcount(kept);
        if (!keep) rank = nkeep + __builtin_popcount(~kept & ((1u << k) - 1u));
        nkeep = min(nkeep, A.p.k_max);
        keep = keep && rank < nkeep;
        if (mode == PIX_NONE) return;
        if (mode == PIX_LEFT) {
            if (k == 0) A.s.cnt[pix] = INIT_LEFT;
            return;
        }
        const double excess = den > 0 ? nwk - fnum * fw / fden : nwk;
        A.s.t[rank * S + pix] = keep ? (double)kt : 0.0;
        A.s.r[rank * S + pix] = keep ? (float)(excess / ((double)G * H)) : 0.f;
        A.s.n[(0 * KM + rank) * S + pix] = 0.f;
        A.s.n[(1 * KM + rank) * S + pix] = 0.f;
        A.s.n[(2 * KM + rank) * S + pix] = -1.f;
        if (k != 0) return;
        A.s.cnt[pix] = (uint8_t)nkeep;
        const double bown = den > 0 && mode == PIX_LIVE ? fnum / fden : 0.0;
        const double b0 = bown / (double)G;
        A.s.b[pix] = (float)(b0 > A.p.b_min ? b0 : A.p.b_min);
    }
};

// The wavefront's pixel: its place in the frame (32-bit arithmetic: a batch
// holds below 2^31 pixels).
struct InitPixel {
    uint32_t pix;
    int i, j;

    __device__ __forceinline__ void at(uint32_t p, const Shape& sh)
    {
        pix = p;
        const uint32_t row = p / (uint32_t)sh.cols;
        j = (int)(p - row * (uint32_t)sh.cols);
        i = (int)(row % (uint32_t)sh.rows);
    }

    __device__ __forceinline__ void next(const Shape& sh)
    {
        ++pix;
        if (++j == sh.cols) {
            j = 0;
            if (++i == sh.rows) i = 0;
        }
    }

    // lane r < side holds the CSR range of window row i - R + r (the row's
    // pixels are consecutive, so their photons are one range)
    __device__ __forceinline__ PoolRows rows(const Shape& sh, int R, const uint32_t* off, const uint32_t* ent) const
    {
        const int lane = threadIdx.x & 63;
        PoolRows W{0, 0, 2 * R + 1, ent};
        const int i2 = i - R + lane;
        if (lane < W.side && i2 >= 0 && i2 < sh.rows) {
            const long long base = (long long)pix - j + (long long)(i2 - i) * sh.cols;
            W.rs = off[base + max(0, j - R)];
            W.re = off[base + min(sh.cols - 1, j + R) + 1];
        }
        return W;
    }
};

template <int KS, bool WIDE>
__device__ __forceinline__ InitPool<KS, WIDE> init_pool(const DevModel& m, v4i* area)
{
    InitPool<KS, WIDE> P;
    P.Z = area;
    P.ks = KS ? KS : m.ks;
    P.NS = init_stride(m.T);
    P.plane = init_chunks(P.NS, P.ks);
    P.B = reinterpret_cast<uint32_t*>(P.Z + (WIDE ? 2 : 1) * P.plane);
    P.lane = threadIdx.x & 63;
    P.j = P.lane & 15;
    P.g = P.lane >> 4;
    P.qa = reinterpret_cast<const v4i*>(m.qa);
    P.e = nullptr;
    return P;
}

// The IRF mass of a whole peak window (summed as InitRecords::set sums one).
__device__ __forceinline__ double window_mass(const DevModel& m)
{
    double hs = 0.0;
    for (int x = threadIdx.x & 63; x <= m.wl + m.wr; x += 64) {
        const int idx = x - m.wl + m.o;
        if (idx >= 0 && idx < m.L) hs += m.hbar[idx];
    }
    return wave_sum(hs);
}

// Wavefront wv of workgroup b takes the ppw <= 16 consecutive pixels from
// (b W + wv) ppw on.
template <int KS>
__global__ __launch_bounds__(64 * INIT_WAVES, INIT_OCC) void k_init(InitArgs args)
{
    extern __shared__ v4i smem[];
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    InitPool<KS, false> P = init_pool<KS, false>(args.m, smem + (size_t)wv * (args.area / 16));
    if constexpr (KS > 0) {
        v4i* e = smem + (size_t)nw * (args.area / 16);
        P.e = e;
        for (int x = threadIdx.x; x < 2 * KS * 64; x += blockDim.x) e[x] = P.qa[KS * 64 + x];
#pragma unroll
        for (int k = 0; k < KS; ++k) P.A[k] = P.qa[k * 64 + lane];
        __syncthreads();
    }
    const double hfull = window_mass(args.m);
    const int ppw = args.ppw;
    const uint32_t first = (xcd_block(blockIdx.x, gridDim.x) * nw + wv) * ppw;
    InitRecords rec;
    rec.clear();
    InitPixel q;
    q.at(first, args.sh);
    for (int x = 0; x < ppw; ++x) {
        const InitArgs& A = init_args();
        // whole wavefront (pixels of other IRF classes: their own launch); no workgroup barriers here
        if (q.pix >= (uint32_t)A.sh.P) break;
        if (in_class(A.m, q.pix) && !(KS == 0 && A.left && A.s.cnt[q.pix] != INIT_LEFT)) {
            const PoolRows W = q.rows(A.sh, A.p.r_init, A.off, A.ent);
            const uint32_t e0 = A.off[q.pix], e1 = A.off[q.pix + 1];
            const float G = gain_at(A.gain, q.pix);
            if (!(G > 0.f)) {
                rec.set_mode(x, PIX_DEAD);
            } else {
                const uint32_t v0 = e0 + lane < e1 ? A.ent[e0 + lane] : 0u;
                // 65536 entries of at most 65535 photons: their sum fits 32 bits
                bool ok = wave_reduce<OpAdd>(W.re - W.rs) <= 65536u;
                uint32_t ntot = 0;
                if (ok) {
                    uint32_t nt = 0;
                    ok = !fill_pool(P, W, A.m.T, A.m.o, nt);
                    ntot = wave_reduce<OpAdd>(nt);
                    ok = ok && (unsigned long long)ntot * (unsigned long long)A.m.qmax <= 0xfffffffeull;
                }
                if (!ok) {
                    rec.set_mode(x, PIX_LEFT);
                } else {
                    Peaks pk;
                    pk.clear();
                    if (ntot > 0 || A.p.n_min < 1) dense_search(P, ntot, pk);
                    rec.set(x, pk, G, v0, e0, e1, hfull);
                }
            }
        }
        q.next(init_args().sh);
    }
    rec.finish(first);
}

// The same pixels per wavefront, by the list search: those of at most
// args.limit pooled entries, if the launch's pixels have at most args.mean on
// average (the others are left).
__global__ __launch_bounds__(64 * INIT_WAVES) void k_init_lists(InitArgs args)
{
    extern __shared__ v4i smem[];
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    v4i* area = smem + (size_t)wv * (args.area / 16);
    const double hfull = window_mass(args.m);
    const int ppw = args.ppw, side = 2 * args.p.r_init + 1;
    const unsigned long long pooled = (unsigned long long)(args.off[args.sh.P] - args.off[0]) * (unsigned)(side * side);
    const bool any = pooled <= (unsigned long long)args.mean * (unsigned long long)args.sh.P;
    const uint32_t first = (xcd_block(blockIdx.x, gridDim.x) * nw + wv) * ppw;
    InitRecords rec;
    rec.clear();
    InitPixel q;
    q.at(first, args.sh);
    for (int x = 0; x < ppw; ++x) {
        const InitArgs& A = init_args();
        if (q.pix >= (uint32_t)A.sh.P) break;   // (whole wavefront; no workgroup barriers here)
        if (in_class(A.m, q.pix) && !(A.left && A.s.cnt[q.pix] != INIT_LEFT)) {
            const PoolRows W = q.rows(A.sh, A.p.r_init, A.off, A.ent);
            const uint32_t e0 = A.off[q.pix], e1 = A.off[q.pix + 1];
            const float G = gain_at(A.gain, q.pix);
            const uint32_t n = wave_reduce<OpAdd>(W.re - W.rs);
            if (!(G > 0.f)) {
                rec.set_mode(x, PIX_DEAD);
            } else if (!any || n > A.limit) {
                rec.set_mode(x, PIX_LEFT);
            } else {
                Peaks pk;
                pk.clear();
                list_search_any(W, n, area, pk);
                rec.set(x, pk, G, e0 + lane < e1 ? A.ent[e0 + lane] : 0u, e0, e1, hfull);
            }
        }
        q.next(init_args().sh);
    }
    rec.finish(first);
}

// The pixels left over, a wavefront looking through args.ppw <= 64 consecutive
// pixels: pools with over 127 photons in a bin from two planes of bytes
// (args.wide: they fit), the rest from the lists.
__global__ __launch_bounds__(64 * INIT_WAVES, INIT_OCC) void k_init_rest(InitArgs args)
{
    extern __shared__ v4i smem[];
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int chunk = args.ppw;
    const long long first = ((long long)blockIdx.x * nw + wv) * chunk;
    const bool mine = lane < chunk && first + lane < args.sh.P && in_class(args.m, first + lane) &&
                      args.s.cnt[first + lane] == INIT_LEFT;
    unsigned long long todo = __ballot(mine);
    if (!todo) return;                      // (no workgroup barriers here)
    const InitPool<0, true> P = init_pool<0, true>(args.m, smem + (size_t)wv * (args.area / 16));
    const double hfull = window_mass(args.m);
    for (; todo; todo &= todo - 1ull) {
        const InitArgs& A = init_args();
        const DevModel& m = A.m;
        InitPixel q;
        q.at((uint32_t)(first + __builtin_ctzll(todo)), A.sh);
        const PoolRows W = q.rows(A.sh, A.p.r_init, A.off, A.ent);
        const uint32_t e0 = A.off[q.pix], e1 = A.off[q.pix + 1], n = wave_reduce<OpAdd>(W.re - W.rs);
        const float G = gain_at(A.gain, q.pix);
        InitRecords rec;
        rec.clear();
        Peaks pk;
        pk.clear();
        bool dense = A.wide && n <= 65536u;
        if (dense) {
            uint32_t nt = 0;
            dense = !fill_planes(P, W, A.off, q.pix, A.sh.cols, q.i, q.j, A.sh.rows, m.T, m.o, nt);
            const uint32_t ntot = wave_reduce<OpAdd>(nt);
            dense = dense && ntot <= 1u << 24;           // the products' sums stay below 2^31
            if (dense) dense_search(P, ntot, pk);
        }
        if (!dense) list_search_any(W, n, P.Z, pk);
        wave_sync();
        rec.set(0, pk, G, e0 + lane < e1 ? A.ent[e0 + lane] : 0u, e0, e1, hfull);
        rec.finish(q.pix);
    }
}

// Initial normals (reading): weighted least-squares plane Z = a + c1 X + c2 Y
// over the APSS neighbourhood in FP64, local coordinates; n = (c1, c2, -1)/|.|,
// or (0, 0, -1) with fewer than 3 neighbours or a near-singular system.
struct PlaneFit {
    double M00 = 0, M01 = 0, M02 = 0, M11 = 0, M12 = 0, M22 = 0, v0 = 0, v1 = 0, v2 = 0, W = 0;
    int nn = 0;

    // a neighbour at (x, y, z) from the point, closer than h
    __device__ __forceinline__ void add(double x, double y, double z, double h2, double inv_h2)
    {
        const double d2 = x * x + y * y + z * z;
        if (!(d2 < h2)) return;
        double a = 1.0 - d2 * inv_h2;
        a = a * a;
        const double w = a * a;
        M00 += w; M01 += w * x; M02 += w * y;
        M11 += w * x * x; M12 += w * x * y; M22 += w * y * y;
        v0 += w * z; v1 += w * x * z; v2 += w * y * z;
        W += w;
        ++nn;
    }

    // vq: the pixel's line of sight
    __device__ __forceinline__ void normal(double h2, bool persp, const double (&vq)[3], float (&n)[3]) const
    {
        n[0] = n[1] = 0.f;
        n[2] = -1.f;
        if (nn >= 3) {
            const double det = M00 * (M11 * M22 - M12 * M12) - M01 * (M01 * M22 - M12 * M02)
                             + M02 * (M01 * M12 - M11 * M02);
            const double scale = W * W * W * h2 * h2;
            if (det > 1e-9 * scale) {
                const double d1 = M00 * (v1 * M22 - M12 * v2) - v0 * (M01 * M22 - M12 * M02)
                                + M02 * (M01 * v2 - v1 * M02);
                const double d2 = M00 * (M11 * v2 - v1 * M12) - M01 * (M01 * v2 - v1 * M02)
                                + v0 * (M01 * M12 - M11 * M02);
                const double c1 = d1 / det, c2 = d2 / det;
                const double nrm = sqrt(c1 * c1 + c2 * c2 + 1.0);
                // facing the sensor: against the pixel's ray (always so for the
                // orthographic map); a plane containing the pinhole camera's
                // line of sight (within 1e-6) takes n = -v
                const double nv = (c1 * vq[0] + c2 * vq[1] - vq[2]) / nrm;
                if (persp && fabs(nv) <= 1e-6) {
                    n[0] = (float)(-vq[0]);
                    n[1] = (float)(-vq[1]);
                    n[2] = (float)(-vq[2]);
                } else {
                    const double sg = nv > 0.0 ? -1.0 : 1.0;
                    n[0] = (float)(sg * c1 / nrm);
                    n[1] = (float)(sg * c2 / nrm);
                    n[2] = (float)(-sg / nrm);
                }
            }
        }
    }
};

// The orthographic map, windows of at most NORMALS_R rings: the depths of a 16 x 16
// pixel tile and its halo in LDS, a thread per live point (list_points), the
// slots in reach of it found a row at a time, then summed one by one.  What
// took the time was one dependent read after the other: 45 us for 636 k pixels,
// 7.5 us for 1 k, against 159 and 37 us for a thread per pixel on the state in
// memory.
constexpr int NORMALS_R = APSS_ROW, NT_SIDE = TILE, NT_THREADS = 512;

inline size_t normals_tile_bytes(int R)
{
    const size_t SX = NT_SIDE + 2 * (size_t)R;
    return SX * SX * KM * sizeof(double) + KM * NT_SIDE * NT_SIDE * sizeof(uint16_t);
}

__global__ __launch_bounds__(NT_THREADS, 4) void k_init_normals_tile(DevParams p, Shape sh, DevState s, int R)
{
    extern __shared__ double normals_lds[];
    __shared__ int wave_points[4];
    const int SX = NT_SIDE + 2 * R, NS = SX * SX;
    double* tl = normals_lds;                                   // [KM][NS] depths
    uint16_t* pl = reinterpret_cast<uint16_t*>(tl + KM * NS);   // points
    const long long S = sh.S;
    const int tiles_x = (sh.cols + NT_SIDE - 1) / NT_SIDE, tiles_y = (sh.rows + NT_SIDE - 1) / NT_SIDE;
    const int tile = (int)xcd_block(blockIdx.x, gridDim.x), tpf = tiles_x * tiles_y;
    const int fr = tile / tpf, tr = tile - fr * tpf;
    const int i0 = (tr / tiles_x) * NT_SIDE, j0 = (tr % tiles_x) * NT_SIDE;
    const long long fbase = (long long)fr * sh.rows * sh.cols;
    for (int x = threadIdx.x; x < NS; x += NT_THREADS) {
        const int r = x / SX, i2 = i0 - R + r, j2 = j0 - R + x - r * SX;
        const bool inside = i2 >= 0 && i2 < sh.rows && j2 >= 0 && j2 < sh.cols;
        const long long pp = fbase + (inside ? (long long)i2 * sh.cols + j2 : 0);
        double t[KM];
        const int cc = load_cnt(s.cnt, pp);
#pragma unroll
        for (int k = 0; k < KM; ++k) t[k] = s.t[k * S + pp];
#pragma unroll
        for (int k = 0; k < KM; ++k) tl[k * NS + x] = inside && k < cc ? t[k] : no_depth();
    }
    int c = 0;
    if (threadIdx.x < NT_SIDE * NT_SIDE) {
        const int i = i0 + threadIdx.x / NT_SIDE, j = j0 + threadIdx.x % NT_SIDE;
        if (i < sh.rows && j < sh.cols) c = load_cnt(s.cnt, fbase + (long long)i * sh.cols + j);
    }
    const int points = list_points(c, wave_points, pl);         // (its barriers: the tile too)
    const double h2 = p.h_apss * p.h_apss, inv_h2 = 1.0 / h2, reach = 1.001 * p.h_apss / p.dz;
    const double vq[3] = {0.0, 0.0, 1.0};
    for (int q = threadIdx.x; q < points; q += NT_THREADS) {
        const int pk = pl[q], k = pk % KM, px = pk / KM, ty = px / NT_SIDE, tx = px % NT_SIDE;
        const int xc = (ty + R) * SX + tx + R;
        const double tq = tl[k * NS + xc];
        PlaneFit f;
        for (int di = -R; di <= R; ++di) {
            const double y = di * p.p_xy;
            uint64_t near = near_slots(tl, NS, xc + di * SX, R, reach, tq);
            for (; near; near &= near - 1) {
                const int bit = __ffsll((unsigned long long)near) - 1, dj = bit / KM - R;
                f.add(dj * p.p_xy, y, (tl[(bit % KM) * NS + xc + di * SX + dj] - tq) * p.dz, h2, inv_h2);
            }
        }
        float n[3];
        f.normal(h2, false, vq, n);
        const long long pix = fbase + (long long)(i0 + ty) * sh.cols + j0 + tx;
#pragma unroll
        for (int a = 0; a < 3; ++a) s.n[(a * KM + k) * S + pix] = n[a];
    }
}

// The pinhole camera (t dz along each pixel's ray) and wider windows: a thread
// per pixel, the state read from memory.
__global__ __launch_bounds__(256) void k_init_normals(DevParams p, Shape sh, DevState s)
{
    const long long P = sh.P, S = sh.S;
    const long long pix = (long long)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (pix >= P) return;
    const int c = load_cnt(s.cnt, pix);
    const int per_frame = sh.rows * sh.cols;
    const long long fr = pix / per_frame;
    const int i = (int)((pix / sh.cols) % sh.rows), j = (int)(pix % sh.cols);
    const double h2 = p.h_apss * p.h_apss, inv_h2 = 1.0 / h2;
    const int R = p.apss_R;
    const bool persp = p.persp > 0.0;   // pinhole camera: t dz along each pixel's ray
    double vq[3] = {0.0, 0.0, 1.0};
    if (persp) ray_dir(p.persp, sh.rows, sh.cols, i, j, vq);
    for (int k = 0; k < KM; ++k) {
        if (k >= c) break;
        const double tq = s.t[k * S + pix];
        PlaneFit f;
        for (int i2 = i - R; i2 <= i + R; ++i2) {
            if (i2 < 0 || i2 >= sh.rows) continue;
            for (int j2 = j - R; j2 <= j + R; ++j2) {
                if (j2 < 0 || j2 >= sh.cols) continue;
                const long long pp = (fr * sh.rows + i2) * sh.cols + j2;
                const int cc = load_cnt(s.cnt, pp);
                // every slot's depth without waiting for the count
                double tn[KM];
#pragma unroll
                for (int k2 = 0; k2 < KM; ++k2) tn[k2] = s.t[k2 * S + pp];
                double vn[3] = {0.0, 0.0, 1.0};
                if (persp && cc > 0) ray_dir(p.persp, sh.rows, sh.cols, i2, j2, vn);
#pragma unroll
                for (int k2 = 0; k2 < KM; ++k2) {
                    if (k2 >= cc) break;
                    double x = (j2 - j) * p.p_xy, y = (i2 - i) * p.p_xy;
                    double z = (tn[k2] - tq) * p.dz;
                    if (persp) {
                        const double t2 = tn[k2];
                        x = (t2 * vn[0] - tq * vq[0]) * p.dz;
                        y = (t2 * vn[1] - tq * vq[1]) * p.dz;
                        z = (t2 * vn[2] - tq * vq[2]) * p.dz;
                    }
                    f.add(x, y, z, h2, inv_h2);
                }
            }
        }
        float n[3];
        f.normal(h2, persp, vq, n);
#pragma unroll
        for (int a = 0; a < 3; ++a) s.n[(a * KM + k) * S + pix] = n[a];
    }
}

// Wavefronts per workgroup, as many as 64 KB of LDS hold.
static int init_waves(size_t area, size_t tables)
{
    int nw = INIT_WAVES;
    while (nw > 1 && nw * area + tables > 65536) nw >>= 1;
    return nw;
}

// Consecutive pixels per wavefront (at most INIT_PPW_MAX): the workgroup's
// tables (a few loads and a barrier) and the wavefront's output serve all of
// them, but a grid needs enough wavefronts to fill the chip (1024 SIMDs with
// five each).  Measured with 1, 2, 4, 8 and 16 pixels, us: 1,960, 1,778, 1,681,
// 1,642 and 1,647 at 636 k pixels; 212, 197, 197, 213 and 220 at 65 k; 85, 81, 80,
// 111 and 180 at 20 k; 20, 28, 39, 62 and 105 at 1 k.
static int pixels_per_wave(long long P) { return P >= 131072 ? 8 : P >= 32768 ? 4 : P >= 16384 ? 2 : 1; }
static_assert(INIT_PPW_MAX >= 8, "a wavefront's pixels have a lane per peak");

// A launch of one of the kernels over pixels, `area` bytes of LDS per wavefront.
static_assert(init_dense_area(1024 * PICK_REGS, 4, 1) + 2 * 4 * 64 * 16 <= 65536, "a pool beside the weights");
template <class Kernel>
static hipError_t launch_pixels(Kernel kernel, InitArgs a, size_t area, size_t tables, hipStream_t st)
{
    a.area = (int)((area + 15) / 16 * 16);
    const int nw = init_waves(a.area, tables);
    a.ppw = pixels_per_wave(a.sh.P);
    const long long per = (long long)nw * a.ppw;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((a.sh.P + per - 1) / per)), dim3(64 * nw), nw * a.area + tables, st, a);
    return hipGetLastError();
}

// Average pool up to which a launch's pixels take the list search, where the
// weights' steps are not in registers (L > 241 or T > 8192).  The dense search
// costs by bins and steps (and by the tiles it scores: more in sparse pools), the
// list search by entries and a little by bins.  20 k pixels, pools of 30 / 100 /
// 200 / 400 entries, lists against dense, us: 8200 bins, 19-bin IRF 131 / 452 /
// 686 / 1270 against 381 / 230 / 159 / 159, 137-bin IRF 137 / 264 / 463 / 924 against
// 238 / 162 / 168 / 185; 20000 bins 118 / 375 / 795 / 1266 against 1247 / 1197 / 436
// / 422 and 123 / 259 / 370 / 647 against 795 / 420 / 412 / 430; 32768 bins 139 /
// 369 / 905 / 1476 against 3261 / 3578 / 1312 / 1037 and 149 / 330 / 417 / 697
// against 2065 / 1022 / 1023 / 1064; 501-bin IRF, 4613 bins 111 / 172 / 276 / 584
// against 140 / 132 / 133 / 135, 8192 bins 115 / 165 / 237 / 437 against 273 / 255 /
// 255 / 259; 2001-bin IRF, 4613 bins 203 / 363 / 739 / 1417 against 558 / 460 / 437 /
// 497.  Both lines are fitted to where such pairs cross, within 15% of the better
// one over 484 calls; pools of strong peaks cross later (32768 bins, 420 entries, a
// fifth of them signal, a 19-bin IRF: 329 against 835).  One choice
// for the launch: a line drawn pixel by pixel lets pools near it take both kernels'
// time (206 us where the one takes 147 and the other 136).
static uint32_t list_mean(int T, int ks)
{
    if (ks == 1) return (uint32_t)(T / 130);
    return (uint32_t)std::min((double)INIT_LIST, 2.6e-5 * T * sqrt((double)T) * std::min(ks, 16));
}

hipError_t launch_init(const DevModel& m, const DevParams& p, const Shape& sh, const uint32_t* off,
                       const uint32_t* ent, const float* gain, DevState s, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    InitArgs a{m, p, sh, off, ent, gain, s, 1, 0, ~0u, (uint32_t)INIT_LIST, (uint32_t)INIT_LIST, 0, 0};
    const size_t lists = init_list_area(m.T, INIT_LIST), tables = (size_t)2 * m.ks * 64 * 16;
    if (!m.qa) {
        const hipError_t e = launch_pixels(k_init_lists, a, lists, 0, st);
        if (e != hipSuccess) return e;
        // larger pools in fewer wavefronts: 10 k pixels, pools of 1510 entries of
        // 40000 bins 5.6 ms, 11.6 ms read from memory for every block
        a.limit = ~0u;
        a.cap = INIT_LONG_LIST;
        a.left = 1;
        return launch_pixels(k_init_lists, a, init_list_area(m.T, INIT_LONG_LIST), 0, st);
    }
    const size_t pool = init_dense_area(m.T, m.ks, 1);
    hipError_t e = hipSuccess;
    switch (m.T > 1024 * PICK_REGS ? 0 : m.ks) {
    case 1: e = launch_pixels(k_init<1>, a, pool, tables, st); break;
    case 2: e = launch_pixels(k_init<2>, a, pool, tables, st); break;
    case 3: e = launch_pixels(k_init<3>, a, pool, tables, st); break;
    case 4: e = launch_pixels(k_init<4>, a, pool, tables, st); break;
    default:
        a.mean = list_mean(m.T, m.ks);
        if (a.mean >= 32) {                    // (below, hardly a pool: not worth the launch)
            e = launch_pixels(k_init_lists, a, lists, 0, st);
            if (e != hipSuccess) return e;
            a.left = 1;
        }
        e = launch_pixels(k_init<0>, a, pool, 0, st);
    }
    if (e != hipSuccess) return e;
    // the pixels left over: enough wavefronts to fill the chip if that is all
    // of them, at most 64 pixels each (one count per lane)
    const size_t planes = init_dense_area(m.T, m.ks, 2);
    a.wide = planes <= 65536;
    a.area = (int)(((a.wide ? std::max(planes, lists) : lists) + 15) / 16 * 16);
    const int nw = init_waves(a.area, 0);
    a.ppw = (int)std::max(1ll, std::min(64ll, sh.P / 8192));
    const long long per = (long long)nw * a.ppw;
    hipLaunchKernelGGL(k_init_rest, dim3((unsigned)((sh.P + per - 1) / per)), dim3(64 * nw), nw * a.area, st, a);
    return hipGetLastError();
}

hipError_t launch_init_normals(const DevParams& p, const Shape& sh, DevState s, hipStream_t st)
{
    if (sh.P == 0) return hipSuccess;
    // rings that can hold a neighbour
    int R = p.apss_R;
    while (R > 0 && !((R * p.p_xy) * (R * p.p_xy) < p.h_apss * p.h_apss)) --R;
    // Tiles where a frame fills them, or where a grid of them is small (what it
    // costs then is its chain of reads): pixels a tile >= 24, or >= 4 with at most
    // 2048 tiles.  Tiles against pixels, us: 1000 frames of 1 x 1 and more 16 to
    // 200 / 10 to 12, 10000 of 2 x 2 41 / 22, 1 x 131072 34 / 17, 2000 of 3 x 3 15 / 41,
    // 1 x 20000 11 / 15, 10000 of 5 x 5 53 / 68, 2 x 60000 26 to 68 / 29 to 59.
    const Tiles tg = tiles_of(sh);
    const long long tiles = tg.tile0[1];
    const bool full = sh.P >= 24 * tiles || (sh.P >= 4 * tiles && tiles <= 2048);
    if (!(p.persp > 0.0) && R <= NORMALS_R && full) {
        hipLaunchKernelGGL(k_init_normals_tile, dim3((unsigned)tg.tile0[1]), dim3(NT_THREADS), normals_tile_bytes(R),
                           st, p, sh, s, R);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_init_normals, dim3((unsigned)((sh.P + 255) / 256)), dim3(256), 0, st, p, sh, s);
    return hipGetLastError();
}

}  // namespace rt3d
