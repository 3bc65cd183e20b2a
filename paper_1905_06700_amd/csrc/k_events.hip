// k_events.hip -- photon events -> active-bin lists, the same CSR that the
// histogram compaction writes.  A time-tagged detector delivers photons as
// (pixel, bin) events rather than histograms; the method only ever needs each
// pixel's non-zero bins and their counts (Methods: cost linear in the active
// bins), so events are counted straight into those lists.
//
// The events go through buckets of B consecutive pixels (a power of two: at
// most EV_MEAN events each on average, at most EV_BUCKETS of them).  A
// workgroup counts its share of the events per bucket in LDS, so that memory
// sees one atomic per workgroup and bucket instead of one per event: bucket
// totals, their scan, then the scatter of (pixel in the bucket, bin) words, each workgroup's
// events of a bucket side by side.  One workgroup per bucket then orders its
// events by pixel in LDS, sorts each pixel's bins (up to 128 of them in the
// lanes of a wavefront), run-length encodes them and leaves the bucket's
// entries packed; a scan of the buckets' entry counts, and the entries move to
// their place.  Buckets with more than EV_CAP events (a few pixels much
// brighter than the rest, or more than EV_CAP events per pixel) take the
// direct way: events counted and scattered per pixel with memory atomics, each
// pixel sorted by one wavefront (in LDS up to EV_LDS events, in place in the
// scratch buffer beyond).  The result does not depend on the event order.
//
// What bounds it is the events' traffic to memory, one place at a time: 4.4 M
// events of 79.5 k pixels (26 MB) took 575 us by the direct way alone (284 in
// the scatter, 174 in the count: an atomic and a scattered store per event)
// and take 122 us by buckets (47 in the scatter, 13 in the count, 39 in the
// sort, 8 in the copy, the rest launches of a few us; the sort took 54 while
// pixels of 65 to 128 events, a tenth of them, were sorted in LDS).
#include "rt3d_dev.h"

#include <algorithm>

namespace rt3d {

constexpr int EV_WAVES = 4;        // wavefronts per block in the per-pixel kernels
constexpr int EV_LDS = 2048;       // longest segment sorted in LDS (8 KB per wavefront)
constexpr uint32_t EV_INF = 0xffffffffu;
constexpr int EV_THREADS = 1024;   // threads of the kernels over the events
constexpr int EV_EPT = 16;         // events per thread, at most
constexpr int EV_BUCKETS = 16384;  // buckets, at most (64 KB of counters)
constexpr int EV_MEAN = 4096;      // events per bucket, at most on average
constexpr int EV_CAP = 6144;       // events a bucket's workgroup orders in LDS
constexpr int EV_PER = EV_CAP / (64 * EV_WAVES);   // of them per thread
constexpr int EV_BMAX = 1024;      // pixels per bucket, at most (else every bucket goes the direct way)

// The buckets' arrays in the workspace (NB of them, B = 2^lg pixels each).
struct EvBuckets {
    int NB, lg;
    uint32_t cap;          // EV_CAP, or 0: every bucket goes the direct way
    uint32_t* total;       // [NB] events
    uint32_t* start;       // [NB + 1] first event
    uint32_t* cursor;      // [NB] next free place
    uint32_t* entries;     // [NB + 1] entries, then (k_ev_bases) first entry and the total
    uint32_t* direct;      // [1] whether some bucket goes the direct way
};

long long ev_bucket_words(long long P)
{
    const long long nb = P < EV_BUCKETS ? P : EV_BUCKETS;
    return 4 * nb + 64;
}

static EvBuckets ev_buckets(uint32_t* w, uint64_t n, long long P)
{
    EvBuckets b;
    b.lg = 0;
    while (((P - 1) >> b.lg) + 1 > EV_BUCKETS) ++b.lg;
    // four pixels (one per wavefront of the sort), more while that leaves 1024
    // buckets or more to work on
    while ((1 << (b.lg + 1)) <= 256 && (n << (b.lg + 1)) <= (uint64_t)EV_MEAN * P &&
           (b.lg < 2 || (P >> (b.lg + 1)) >= 1024))
        ++b.lg;
    b.NB = (int)(((P - 1) >> b.lg) + 1);
    b.cap = (1 << b.lg) <= EV_BMAX ? EV_CAP : 0;
    b.total = w;
    b.start = b.total + b.NB;
    b.cursor = b.start + b.NB + 1;
    b.entries = b.cursor + b.NB;
    b.direct = b.entries + b.NB + 1;
    return b;
}

__device__ __forceinline__ bool ev_valid(uint32_t p, uint32_t b, long long P, int T)
{
    return (long long)p < P && (int)b < T;
}

// Whether bucket k goes the direct way (its total is final).
__device__ __forceinline__ bool ev_direct(const EvBuckets& b, uint32_t k) { return b.cap == 0 || b.total[k] > b.cap; }

// Clears the buckets' counters and the pixels' (which only the direct way uses:
// cheaper than a launch of its own behind the decision).
__global__ __launch_bounds__(256) void k_ev_zero(EvBuckets b, uint32_t* __restrict__ counts, long long P)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < b.NB) {
        b.total[i] = 0;
        b.entries[i] = 0;
    }
    if (i < P) counts[i] = 0;
    if (i == 0) *b.direct = 0;
}

// Bucket totals: workgroup w counts events [w EPW, (w + 1) EPW), EPW = ept x
// EV_THREADS.
__global__ __launch_bounds__(EV_THREADS) void k_ev_count(EvBuckets b, const uint32_t* __restrict__ pix,
                                                         const uint16_t* __restrict__ bin, uint64_t n, long long P,
                                                         int T, int ept, int32_t* __restrict__ err)
{
    extern __shared__ uint32_t ev_hist[];
    for (int k = threadIdx.x; k < b.NB; k += EV_THREADS) ev_hist[k] = 0;
    __syncthreads();
    const uint64_t i0 = (uint64_t)blockIdx.x * ept * EV_THREADS + threadIdx.x;
    bool bad = false;
#pragma unroll 4
    for (int u = 0; u < ept; ++u) {
        const uint64_t i = i0 + (uint64_t)u * EV_THREADS;
        if (i >= n) break;
        const uint32_t p = pix[i], t = bin[i];
        if (ev_valid(p, t, P, T)) atomicAdd(&ev_hist[p >> b.lg], 1u);
        else bad = true;
    }
    if (bad) *err = RT3D_E_INVALID;
    __syncthreads();
    for (int k = threadIdx.x; k < b.NB; k += EV_THREADS)
        if (ev_hist[k]) atomicAdd(&b.total[k], ev_hist[k]);
}

// Exclusive scan of v[0 .. n - 1] by one workgroup of 1024 threads (contiguous
// runs of values per thread): f(k, value, prefix) for every k; returns the
// total.  (All sums fit 32 bits: below 2^31 events.)
template <class F>
__device__ __forceinline__ uint32_t ev_scan(const uint32_t* v, int n, F f)
{
    __shared__ uint32_t wsum[16];
    const int per = (n + 1023) / 1024, k0 = threadIdx.x * per, k1 = min(k0 + per, n);
    uint32_t s = 0;
    for (int k = k0; k < k1; ++k) s += v[k];
    const uint32_t inc = wave_incl_scan(s);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t run = inc - s, total = 0;
    for (int q = 0; q < 16; ++q) {
        run += q < w ? wsum[q] : 0u;
        total += wsum[q];
    }
    for (int k = k0; k < k1; ++k) {
        const uint32_t x = v[k];
        f(k, x, run);
        run += x;
    }
    return total;
}

// Bucket starts and cursors; notes whether a bucket goes the direct way.
__global__ __launch_bounds__(1024) void k_ev_starts(EvBuckets b)
{
    const uint32_t total = ev_scan(b.total, b.NB, [&](int k, uint32_t x, uint32_t run) {
        b.start[k] = run;
        b.cursor[k] = run;
        if (x > b.cap) *b.direct = 1;
    });
    if (threadIdx.x == 0) {
        b.start[b.NB] = total;
        if (b.cap == 0) *b.direct = 1;
    }
}

// The direct way: per-pixel counts, and the pixels' segments [evoff[p],
// evoff[p] + events); counts then holds their cursors.
__global__ __launch_bounds__(256) void k_ev_direct_count(EvBuckets b, const uint32_t* __restrict__ pix,
                                                         const uint16_t* __restrict__ bin, uint64_t n, long long P,
                                                         int T, uint32_t* __restrict__ counts)
{
    if (!*b.direct) return;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
        const uint32_t p = pix[i];
        if (ev_valid(p, bin[i], P, T) && ev_direct(b, p >> b.lg)) atomicAdd(&counts[p], 1u);
    }
}

__global__ __launch_bounds__(256) void k_ev_direct_offsets(EvBuckets b, uint32_t* __restrict__ counts,
                                                           uint32_t* __restrict__ evoff, long long P)
{
    if (!*b.direct) return;
    const int lane = threadIdx.x & 63;
    for (int k = blockIdx.x * 4 + (threadIdx.x >> 6); k < b.NB; k += gridDim.x * 4) {
        if (!ev_direct(b, k)) continue;
        const long long p0 = (long long)k << b.lg, p1 = min(p0 + (1ll << b.lg), P);
        uint32_t run = b.start[k];
        for (long long p = p0; p < p1; p += 64) {
            const uint32_t c = p + lane < p1 ? counts[p + lane] : 0u;
            const uint32_t inc = wave_incl_scan(c);
            if (p + lane < p1) {
                evoff[p + lane] = run + inc - c;
                counts[p + lane] = run + inc - c;
            }
            run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
    }
}

// The scatter: a workgroup ranks its events within each bucket with LDS
// atomics, reserves each bucket's places with one memory atomic and writes
// (pixel in the bucket, bin) words there; events of buckets on the direct way
// go to their pixel's segment, the bin alone.
__global__ __launch_bounds__(EV_THREADS) void k_ev_scatter(EvBuckets b, const uint32_t* __restrict__ pix,
                                                           const uint16_t* __restrict__ bin, uint64_t n, long long P,
                                                           int T, int ept, uint32_t* __restrict__ counts,
                                                           uint32_t* __restrict__ scratch)
{
    extern __shared__ uint32_t ev_hist[];
    for (int k = threadIdx.x; k < b.NB; k += EV_THREADS) ev_hist[k] = 0;
    __syncthreads();
    const bool direct = *b.direct != 0;
    const uint64_t i0 = (uint64_t)blockIdx.x * ept * EV_THREADS + threadIdx.x;
    uint32_t pv[EV_EPT], tv[EV_EPT], rank[EV_EPT];
#pragma unroll
    for (int u = 0; u < EV_EPT; ++u) {
        const uint64_t i = i0 + (uint64_t)u * EV_THREADS;
        pv[u] = EV_INF;
        tv[u] = 0;
        if (u < ept && i < n) {
            pv[u] = pix[i];
            tv[u] = bin[i];
        }
    }
#pragma unroll
    for (int u = 0; u < EV_EPT; ++u) {
        rank[u] = EV_INF;
        if (!ev_valid(pv[u], tv[u], P, T)) continue;
        const uint32_t k = pv[u] >> b.lg;
        if (direct && ev_direct(b, k)) scratch[atomicAdd(&counts[pv[u]], 1u)] = tv[u];
        else rank[u] = atomicAdd(&ev_hist[k], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < b.NB; k += EV_THREADS)
        if (ev_hist[k]) ev_hist[k] = atomicAdd(&b.cursor[k], ev_hist[k]);
    __syncthreads();
    const uint32_t local = (1u << b.lg) - 1u;
#pragma unroll
    for (int u = 0; u < EV_EPT; ++u)
        if (rank[u] != EV_INF) scratch[ev_hist[pv[u] >> b.lg] + rank[u]] = ((pv[u] & local) << 16) | tv[u];
}

// Orders the wavefront's memory traffic (LDS or global) between network stages.
__device__ __forceinline__ void ev_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <class V>
__device__ __forceinline__ void ev_cswap(V* a, uint32_t i, uint32_t l)
{
    const V x = a[i], y = a[l];
    if (y < x) {
        a[i] = y;
        a[l] = x;
    }
}

// Ascending bitonic sort of a[0..n) by one wavefront, on the next power of two
// N2 >= n with a[n..N2) taken as +infinity.  Every comparator puts the smaller
// value at the lower index, so a comparator whose upper index is >= n would
// leave both places as they are: it is skipped and the padding is never
// stored.
template <class V>
__device__ void ev_bitonic(V* a, uint32_t n)
{
    uint32_t N2 = 1;
    while (N2 < n) N2 <<= 1;
    const uint32_t lane = threadIdx.x & 63, half = N2 >> 1;
    for (uint32_t k = 2; k <= N2; k <<= 1) {
        const uint32_t hk = k >> 1;
        for (uint32_t t = lane; t < half; t += 64) {       // merge step of width k (mirrored pairs)
            const uint32_t o = t & (hk - 1), base = (t - o) << 1;
            const uint32_t i = base + o, l = base + k - 1 - o;
            if (l < n) ev_cswap(a, i, l);
        }
        ev_sync();
        for (uint32_t j = hk >> 1; j > 0; j >>= 1) {         // half-cleaners
            for (uint32_t t = lane; t < half; t += 64) {
                const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i + j;
                if (l < n) ev_cswap(a, i, l);
            }
            ev_sync();
        }
    }
}

// Ascending sort of one value per lane (the mirrored merge network: partners
// lane ^ (k - 1), then lane ^ j), every move on the vector ALU.
template <int CTRL>
__device__ __forceinline__ uint32_t ev_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// PAIR: two 16-bit values per lane, two sorts side by side.
template <bool PAIR>
__device__ __forceinline__ uint32_t ev_min(uint32_t v, uint32_t o)
{
    typedef unsigned short pair __attribute__((ext_vector_type(2)));
    if (!PAIR) return v < o ? v : o;
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(pair, v),
                                                                  __builtin_bit_cast(pair, o)));
}

template <bool PAIR>
__device__ __forceinline__ uint32_t ev_max(uint32_t v, uint32_t o)
{
    typedef unsigned short pair __attribute__((ext_vector_type(2)));
    if (!PAIR) return v < o ? o : v;
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(pair, v),
                                                                  __builtin_bit_cast(pair, o)));
}

template <bool PAIR>
__device__ __forceinline__ uint32_t ev_keep(uint32_t v, uint32_t o, bool upper)
{
    const uint32_t lo = ev_min<PAIR>(v, o), hi = ev_max<PAIR>(v, o);
    return upper ? hi : lo;
}

__device__ __forceinline__ uint32_t ev_xor16(uint32_t v, bool b16)
{
    auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return b16 ? r[0] : r[1];
}

__device__ __forceinline__ uint32_t ev_xor32(uint32_t v, bool b32)
{
    auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b32 ? r[0] : r[1];
}

template <bool PAIR>
__device__ __forceinline__ uint32_t ev_sort64(uint32_t v, int lane)
{
    const bool b1 = lane & 1, b2 = lane & 2, b4 = lane & 4, b8 = lane & 8, b16 = lane & 16, b32 = lane & 32;
    auto x1 = [&] { v = ev_keep<PAIR>(v, ev_move<0xB1>(v), b1); };                       // lane ^ 1
    auto x2 = [&] { v = ev_keep<PAIR>(v, ev_move<0x4E>(v), b2); };                       // ^ 2
    auto x4 = [&] { v = ev_keep<PAIR>(v, ev_move<0x1B>(ev_move<0x141>(v)), b4); };       // ^ 7 ^ 3
    auto x8 = [&] { v = ev_keep<PAIR>(v, ev_move<0x128>(v), b8); };                      // rotated by 8 of 16
    x1();
    v = ev_keep<PAIR>(v, ev_move<0x1B>(v), b2);                                          // ^ 3
    x1();
    v = ev_keep<PAIR>(v, ev_move<0x141>(v), b4);                                         // ^ 7
    x2(), x1();
    v = ev_keep<PAIR>(v, ev_move<0x140>(v), b8);                                         // ^ 15
    x4(), x2(), x1();
    v = ev_keep<PAIR>(v, ev_xor16(ev_move<0x140>(v), b16), b16);                         // ^ 31
    x8(), x4(), x2(), x1();
    v = ev_keep<PAIR>(v, ev_xor32(ev_xor16(ev_move<0x140>(v), b16), b32), b32);          // ^ 63
    v = ev_keep<PAIR>(v, ev_xor16(v, b16), b16);
    x8(), x4(), x2(), x1();
    return v;
}

// Ascending sort of 128 16-bit values, value i in the low half of lane i, value
// 64 + i in the high half: both halves sorted side by side, the mirrored pairs
// between them, then the half-cleaners on both.
__device__ __forceinline__ uint32_t ev_sort128(uint32_t v, int lane)
{
    const bool b1 = lane & 1, b2 = lane & 2, b4 = lane & 4, b8 = lane & 8, b16 = lane & 16, b32 = lane & 32;
    v = ev_sort64<true>(v, lane);
    const uint32_t m = ev_xor32(ev_xor16(ev_move<0x140>(v), b16), b32);            // lane ^ 63
    const uint32_t o = (m >> 16) | (m << 16);
    v = (ev_min<true>(v, o) & 0xffffu) | (ev_max<true>(v, o) & 0xffff0000u);
    v = ev_keep<true>(v, ev_xor32(v, b32), b32);
    v = ev_keep<true>(v, ev_xor16(v, b16), b16);
    v = ev_keep<true>(v, ev_move<0x128>(v), b8);
    v = ev_keep<true>(v, ev_move<0x1B>(ev_move<0x141>(v)), b4);
    v = ev_keep<true>(v, ev_move<0x4E>(v), b2);
    v = ev_keep<true>(v, ev_move<0xB1>(v), b1);
    return v;
}

// Distinct values of the sorted a[0 .. n - 1] (every lane gets the count).
template <class V>
__device__ __forceinline__ uint32_t ev_distinct(const V* a, uint32_t n)
{
    uint32_t heads = 0;
    for (uint32_t i = threadIdx.x & 63; i < n; i += 64) heads += (i == 0 || a[i] != a[i - 1]) ? 1u : 0u;
    return wave_sum(heads);
}

// Run-length encodes the sorted a[0 .. n - 1] into out[0 ..] as (bin, count)
// entries.  Chunks of 64 bins: a run ends at lane i when the next bin differs;
// its start is the last run head at or before i (from the chunk's head ballot,
// or carried from earlier chunks).  Returns whether a count passed 65535 (it
// does not fit the entry's 16 bits and is stored as 65535).  out may be a
// itself (a chunk's entries go at or before its first bin, and its bins are
// read first).
template <class V>
__device__ __forceinline__ bool ev_rle(const V* a, uint32_t n, uint32_t* out)
{
    const int lane = threadIdx.x & 63;
    const uint64_t le = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);   // lanes <= this one
    uint32_t runs = 0, carry = 0, prev = EV_INF;
    bool over = false;
    for (uint32_t c0 = 0; c0 < n; c0 += 64) {                // uniform over the wavefront
        const uint32_t i = c0 + lane;
        const bool in = i < n;
        const uint32_t v = in ? (uint32_t)a[i] : EV_INF;
        const uint32_t nv = i + 1 < n ? (uint32_t)a[i + 1] : EV_INF;
        uint32_t pv = (uint32_t)__shfl_up((int)v, 1, 64);
        if (lane == 0) pv = prev;
        prev = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
        const bool head = in && v != pv;
        const bool last = in && v != nv;
        const uint64_t hm = __ballot(head);
        const uint64_t mh = hm & le;
        if (last) {
            const uint32_t start = mh ? c0 + 63u - (uint32_t)__clzll(mh) : carry;
            const uint32_t cnt = i + 1 - start;
            over = over || cnt > 0xffffu;
            out[runs + (uint32_t)__popcll(mh) - 1u] = (v << 16) | (cnt > 0xffffu ? 0xffffu : cnt);
        }
        if (hm) carry = c0 + 63u - (uint32_t)__clzll(hm);
        runs += (uint32_t)__popcll(hm);
    }
    return over;
}

// One bucket per workgroup: its events by pixel in LDS, each pixel's bins
// sorted, the entries packed at the bucket's start in scratch, off[p] the
// place of pixel p's first entry within the bucket.
__global__ __launch_bounds__(64 * EV_WAVES) void k_ev_sort(EvBuckets b, long long P, uint32_t* __restrict__ scratch,
                                                           uint32_t* __restrict__ off, int32_t* __restrict__ err)
{
    extern __shared__ uint32_t ev_lds[];
    const int k = blockIdx.x, B = 1 << b.lg, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (ev_direct(b, k)) return;
    uint16_t* bins = reinterpret_cast<uint16_t*>(ev_lds);      // [EV_CAP]
    uint32_t* seg = ev_lds + EV_CAP / 2;                       // [B + 1] segment starts
    uint32_t* cur = seg + B + 1;                               // [B] cursors, then entries, then places
    const uint32_t s0 = b.start[k], n = b.start[k + 1] - s0;
    const long long p0 = (long long)k << b.lg;
    const int np = (int)min((long long)B, P - p0);
    for (int x = threadIdx.x; x < B; x += 64 * EV_WAVES) cur[x] = 0;
    __syncthreads();
    // the bucket's events in registers, every read in flight at once; an event's
    // place in its pixel's segment is the counter's value before it
    uint32_t v[EV_PER], rank[EV_PER];
#pragma unroll
    for (int u = 0; u < EV_PER; ++u) {
        const uint32_t x = threadIdx.x + u * 64 * EV_WAVES;
        v[u] = x < n ? scratch[s0 + x] : EV_INF;
    }
#pragma unroll
    for (int u = 0; u < EV_PER; ++u)
        rank[u] = threadIdx.x + u * 64 * EV_WAVES < n ? atomicAdd(&cur[v[u] >> 16], 1u) : 0u;
    __syncthreads();
    auto scan = [&](bool places) {             // wavefront 0: exclusive scan of cur into cur (and seg)
        uint32_t run = 0;
        for (int c = 0; c < B; c += 64) {
            const uint32_t v = c + lane < B ? cur[c + lane] : 0u;
            const uint32_t inc = wave_incl_scan(v);
            if (c + lane < B) {
                cur[c + lane] = run + inc - v;
                if (!places) seg[c + lane] = run + inc - v;
            }
            run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
        return run;
    };
    if (w == 0) {
        const uint32_t run = scan(false);
        if (lane == 0) seg[B] = run;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < EV_PER; ++u)
        if (threadIdx.x + u * 64 * EV_WAVES < n) bins[seg[v[u] >> 16] + rank[u]] = (uint16_t)v[u];
    __syncthreads();
    for (int p = w; p < B; p += EV_WAVES) {
        const uint32_t at = seg[p], m = seg[p + 1] - at;
        uint32_t d;
        if (m <= 64) {
            uint32_t v = (uint32_t)lane < m ? bins[at + lane] : EV_INF;
            v = ev_sort64<false>(v, lane);
            if ((uint32_t)lane < m) bins[at + lane] = (uint16_t)v;
            const uint32_t pv = (uint32_t)__shfl_up((int)v, 1, 64);
            d = (uint32_t)__popcll(__ballot((uint32_t)lane < m && (lane == 0 || v != pv)));
        } else if (m <= 128) {
            const bool in = 64u + lane < m;
            const uint32_t v = ev_sort128(bins[at + lane] | (in ? (uint32_t)bins[at + 64 + lane] << 16 : 0xffff0000u),
                                          lane);
            bins[at + lane] = (uint16_t)v;
            if (in) bins[at + 64 + lane] = (uint16_t)(v >> 16);
            const uint32_t df = v ^ (uint32_t)__shfl_up((int)v, 1, 64);
            const uint32_t mid = (uint32_t)__builtin_amdgcn_readlane((int)v, 63) & 0xffffu;   // value 63
            const bool head = lane == 0 ? (v >> 16) != mid : (df >> 16) != 0;
            d = (uint32_t)(__popcll(__ballot(lane == 0 || (df & 0xffffu))) + __popcll(__ballot(in && head)));
        } else {
            ev_bitonic(bins + at, m);
            d = ev_distinct(bins + at, m);
        }
        if (lane == 0) cur[p] = d;
    }
    __syncthreads();
    if (w == 0) {
        const uint32_t run = scan(true);
        if (lane == 0) b.entries[k] = run;
    }
    __syncthreads();
    bool over = false;
    for (int p = w; p < np; p += EV_WAVES) {
        const uint32_t at = seg[p], m = seg[p + 1] - at, o = cur[p];
        if (lane == 0) off[p0 + p] = o;
        over = ev_rle(bins + at, m, scratch + s0 + o) || over;
    }
    if (over) *err = RT3D_E_INVALID;
}

// The direct way's pixels, a wavefront each: the segment sorted and encoded in
// place; counts[p] = entries, added to the bucket's.
__global__ __launch_bounds__(64 * EV_WAVES) void k_ev_direct_sort(EvBuckets b, long long P,
                                                                  uint32_t* __restrict__ counts,
                                                                  const uint32_t* __restrict__ evoff,
                                                                  uint32_t* __restrict__ scratch,
                                                                  int32_t* __restrict__ err)
{
    __shared__ uint32_t lds[EV_WAVES][EV_LDS];
    if (!*b.direct) return;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (long long p = (long long)blockIdx.x * EV_WAVES + w; p < P; p += (long long)gridDim.x * EV_WAVES) {
        const uint32_t k = (uint32_t)(p >> b.lg);
        if (!ev_direct(b, k)) continue;                         // whole wavefront; no block barrier below
        const uint32_t lo = evoff[p], n = counts[p] - lo;       // (the cursor ended past the segment)
        uint32_t* seg = scratch + lo;
        bool over;
        uint32_t d;
        if (n <= (uint32_t)EV_LDS) {
            for (uint32_t i = lane; i < n; i += 64) lds[w][i] = seg[i];
            ev_sync();
            ev_bitonic(lds[w], n);
            d = ev_distinct(lds[w], n);
            over = ev_rle(lds[w], n, seg);
            ev_sync();
        } else {
            ev_bitonic(seg, n);
            d = ev_distinct(seg, n);
            over = ev_rle(seg, n, seg);
        }
        if (over) *err = RT3D_E_INVALID;
        if (lane == 0) {
            counts[p] = d;
            atomicAdd(&b.entries[k], d);
        }
    }
}

// First entries of the buckets; off[P] = the total, clamped to cap (E_CAPACITY
// beyond).
__global__ __launch_bounds__(1024) void k_ev_bases(EvBuckets b, long long P, uint64_t cap, uint32_t* __restrict__ off,
                                                   int32_t* __restrict__ err)
{
    const uint32_t total = ev_scan(b.entries, b.NB, [&](int k, uint32_t, uint32_t run) { b.entries[k] = run; });
    if (threadIdx.x == 0) {
        b.entries[b.NB] = total;
        off[P] = total < cap ? total : (uint32_t)cap;
        if (total > cap) *err = RT3D_E_CAPACITY;
    }
}

// The entries to their place: a bucket per workgroup, off[p] from places within
// the bucket to the lists' (clamped to cap, as the lists are cut there).
__global__ __launch_bounds__(256) void k_ev_copy(EvBuckets b, long long P, const uint32_t* __restrict__ counts,
                                                 const uint32_t* __restrict__ evoff,
                                                 const uint32_t* __restrict__ scratch, uint32_t* __restrict__ off,
                                                 uint32_t* __restrict__ ent, uint64_t cap)
{
    const int k = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long p0 = (long long)k << b.lg, p1 = min(p0 + (1ll << b.lg), P);
    const uint32_t base = b.entries[k];
    auto place = [&](uint64_t x) { return (uint32_t)(x < cap ? x : cap); };
    if (!ev_direct(b, k)) {
        for (long long p = p0 + threadIdx.x; p < p1; p += 256) off[p] = place((uint64_t)base + off[p]);
        const uint32_t n = b.entries[k + 1] - base;
        const uint32_t* src = scratch + b.start[k];
        for (uint32_t x = threadIdx.x; x < n; x += 256)
            if ((uint64_t)base + x < cap) ent[base + x] = src[x];
        return;
    }
    // the direct way: wavefront w takes every fourth chunk of 64 pixels' lists
    uint64_t run = base;
    for (long long q = p0; q < p1; q += 64) {
        const uint32_t c = q + lane < p1 ? counts[q + lane] : 0u;
        const uint32_t inc = wave_incl_scan(c);
        if (w == 0 && q + lane < p1) off[q + lane] = place(run + inc - c);
        for (int j = w; j < 64 && q + j < p1; j += 4) {
            const uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)c, j);
            const uint64_t at = run + (uint32_t)__builtin_amdgcn_readlane((int)(inc - c), j);
            const uint32_t* src = scratch + evoff[q + j];
            for (uint32_t x = lane; x < m; x += 64)
                if (at + x < cap) ent[at + x] = src[x];
        }
        run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
}

hipError_t launch_compact_events(const uint32_t* pix, const uint16_t* bin, uint64_t n, long long P, int T,
                                 uint32_t* evoff, uint32_t* scratch, uint32_t* off, uint32_t* ent, uint64_t cap,
                                 uint32_t* counts, uint32_t* buckets, int32_t* err, hipStream_t st)
{
    if (P <= 0) return hipSuccess;
    if (cap > 0xffffffffull) cap = 0xffffffffull;   // offsets are 32-bit
    const EvBuckets b = ev_buckets(buckets, n, P);
    // events per thread: as many as keep one workgroup per CU
    const int ept = (int)std::min<uint64_t>(EV_EPT, n / (256ull * EV_THREADS) + 1);
    const unsigned eb = (unsigned)((n + (uint64_t)ept * EV_THREADS - 1) / ((uint64_t)ept * EV_THREADS));
    const size_t hist = sizeof(uint32_t) * b.NB;
    const unsigned db = 1024;                       // the direct way's grids (strided; nothing to do most times)
    hipLaunchKernelGGL(k_ev_zero, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, b, counts, P);
    if (eb) hipLaunchKernelGGL(k_ev_count, dim3(eb), dim3(EV_THREADS), hist, st, b, pix, bin, n, P, T, ept, err);
    hipLaunchKernelGGL(k_ev_starts, dim3(1), dim3(1024), 0, st, b);
    hipLaunchKernelGGL(k_ev_direct_count, dim3(db), dim3(256), 0, st, b, pix, bin, n, P, T, counts);
    hipLaunchKernelGGL(k_ev_direct_offsets, dim3(db), dim3(256), 0, st, b, counts, evoff, P);
    if (eb)
        hipLaunchKernelGGL(k_ev_scatter, dim3(eb), dim3(EV_THREADS), hist, st, b, pix, bin, n, P, T, ept, counts,
                           scratch);
    const size_t lds = sizeof(uint32_t) * (EV_CAP / 2 + 2 * (size_t)(b.cap ? 1 << b.lg : 0) + 1);
    hipLaunchKernelGGL(k_ev_sort, dim3(b.NB), dim3(64 * EV_WAVES), lds, st, b, P, scratch, off, err);
    hipLaunchKernelGGL(k_ev_direct_sort, dim3(db), dim3(64 * EV_WAVES), 0, st, b, P, counts, evoff, scratch,
                       err);
    hipLaunchKernelGGL(k_ev_bases, dim3(1), dim3(1024), 0, st, b, P, cap, off, err);
    hipLaunchKernelGGL(k_ev_copy, dim3(b.NB), dim3(256), 0, st, b, P, counts, evoff, scratch, off, ent, cap);
    return hipGetLastError();
}

}  // namespace rt3d
