// histogram.hip -- reduction(+: hist[0:bins]) over a loop whose iteration i
// does hist[key[i]] += 1: an array-section reduction whose list item is
// chosen by the data.  Each team takes a team-shared copy of (a range of)
// the histogram with team_alloc (in LDS when it fits, else in its slice of
// a global pool), counts its balanced block of keys into it with atomic
// adds, and adds the non-zero bins of its copy into hist.  Past the LDS
// ranges the default is no copy at all: atomic adds on hist.  Counts wrap modulo 2^32; keys
// outside [0, bins) are not counted and set bit 3 (value 4) of the stream's
// workspace status.
#include <math.h>

#include <algorithm>
#include <map>
#include <mutex>

#include "device.h"
#include "runtime.h"
#include "shared_alloc.h"

namespace omprt {

typedef __attribute__((address_space(3))) uint32_t lds_u32;

// The team copy lives in LDS (LdsCopy, ds atomics) or in the team's slice of
// the global pool (GlobalCopy, atomics performed at L2; the team's own loads
// and stores of it also go to L2, bypassing the compute unit's cache).
struct LdsCopy {
    lds_u32* h;
    __device__ __forceinline__ void zero(uint32_t b) { h[b] = 0u; }
    __device__ __forceinline__ void add(uint32_t k, uint32_t n = 1u) {
        __hip_atomic_fetch_add(h + k, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ uint32_t get(uint32_t b) const { return h[b]; }
};
struct GlobalCopy {
    uint32_t* h;
    __device__ __forceinline__ void zero(uint32_t b) {
        __hip_atomic_store(h + b, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void add(uint32_t k, uint32_t n = 1u) {
        __hip_atomic_fetch_add(h + k, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t get(uint32_t b) const {
        return __hip_atomic_load(h + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// The team's bins are [b0, b0 + tb) of [0, bins).
struct BinRange {
    uint32_t bins, b0, tb;
};

template <class C>
__device__ __forceinline__ void count_key(C& c, int32_t k, const BinRange& r, bool& bad) {
    if ((uint32_t)k >= r.bins)
        bad = true;
    else if ((uint32_t)k - r.b0 < r.tb)
        c.add((uint32_t)k - r.b0);
}

// A vector of four keys a lane.  When every key of the wave's vectors is the
// same (constant or sorted inputs) one lane adds their number: same-address
// lanes of an LDS atomic are served one after another (10^8 equal keys into
// 1000 bins: 333 us lane by lane, 65 this way).
using i32x4 = int32_t __attribute__((ext_vector_type(4)));
template <class C>
__device__ __forceinline__ void count_vector(C& c, const i32x4& k, const BinRange& r, bool& bad) {
    const int32_t f = __builtin_amdgcn_readfirstlane(k[0]);
    const bool same = ((k[0] ^ f) | (k[1] ^ f) | (k[2] ^ f) | (k[3] ^ f)) == 0;
    const uint64_t active = __ballot(1);
    if (__ballot(same) == active) {
        if ((uint32_t)f >= r.bins)
            bad = true;
        else if ((uint32_t)f - r.b0 < r.tb && (int)__lane_id() == __ffsll((unsigned long long)active) - 1)
            c.add((uint32_t)f - r.b0, 4u * (uint32_t)__popcll(active));
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) count_key(c, k[q], r, bad);
    }
}

// U vectors a lane, with one comparison for other inputs: only where the lanes'
// first keys are all the same does each vector look (looking at every vector
// cost 2 % of 2 * 10^8 uniform keys).
template <int U, class C>
__device__ __forceinline__ void count_vectors(C& c, const i32x4 (&k)[U], const BinRange& r,
                                              bool& bad) {
    if (__ballot(k[0][0] != __builtin_amdgcn_readfirstlane(k[0][0])) == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) count_vector(c, k[u], r, bad);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) count_key(c, k[u][q], r, bad);
    }
}

// Zero the copy, count the keys of the team's balanced block that fall in
// its bins, add the non-zero bins into hist.  Returns whether a key was
// outside [0, bins).
template <int U, class C>
__device__ __forceinline__ bool team_histogram(C c, const int32_t* __restrict__ keys, int64_t n,
                                               const BinRange& bins, int64_t row, int64_t rows,
                                               int32_t* __restrict__ hist) {
    const int tid = threadIdx.x, P = team_size();
    for (uint32_t b = tid; b < bins.tb; b += P) c.zero(b);
    __syncthreads();
    bool bad = false;
    const Range blk = bal_share(n, rows, row);
    if (blk.lo < blk.hi) {
        const int64_t a = blk.lo, e = blk.hi;
        const uintptr_t mis = reinterpret_cast<uintptr_t>(keys + a) & 15;
        int64_t head = (int64_t)(((16 - mis) & 15) / 4);
        if (head > e - a) head = e - a;
        if (tid < head) count_key(c, keys[a + tid], bins, bad);
        const int64_t p0 = a + head;
        const int64_t nv = (e - p0) / 4;
        const i32x4* __restrict__ vp = reinterpret_cast<const i32x4*>(keys + p0);
        int64_t v = tid;
        for (; v + (int64_t)(U - 1) * P < nv; v += (int64_t)U * P) {
            i32x4 r[U];
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = __builtin_nontemporal_load(vp + v + (int64_t)u * P);
            count_vectors<U>(c, r, bins, bad);
        }
        for (; v < nv; v += P) count_vector(c, __builtin_nontemporal_load(vp + v), bins, bad);
        const int64_t t0 = p0 + nv * 4;
        if (tid < e - t0) count_key(c, keys[t0 + tid], bins, bad);
    }
    __syncthreads();
    for (uint32_t b = tid; b < bins.tb; b += P) {
        const uint32_t v = c.get(b);
        if (v)
            __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(hist) + bins.b0 + b, v,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return bad;
}

// Team k takes bin range k % tiles (tile_bins bins each, the last one
// shorter) and row block k / tiles of the keys.
template <int U>
__global__ __launch_bounds__(1024) void histogram_kernel(const int32_t* __restrict__ keys,
                                                         int64_t n, uint32_t bins,
                                                         uint32_t tiles, uint32_t tile_bins,
                                                         int32_t* __restrict__ hist, char* pool,
                                                         uint64_t pool_per_team,
                                                         uint32_t lds_cap, uint32_t* status) {
    extern __shared__ __align__(16) char arena[];
    __shared__ TeamStack st;
    __shared__ int s_bad;
    const int tid = threadIdx.x;
    team_stack_init(&st, arena, lds_cap, pool ? pool + blockIdx.x * pool_per_team : nullptr,
                    pool_per_team);
    if (tid == 0) s_bad = 0;
    const uint32_t tile = blockIdx.x % tiles;
    BinRange r;
    r.bins = bins;
    r.b0 = tile * tile_bins;
    r.tb = r.b0 >= bins ? 0u : (bins - r.b0 < tile_bins ? bins - r.b0 : tile_bins);
    const int64_t rows = gridDim.x / tiles, row = blockIdx.x / tiles;
    void* h = team_alloc(&st, (uint64_t)r.tb * 4);
    if (!h) {   // the host sizes the pool so that this cannot happen
        if (tid == 0) __hip_atomic_fetch_or(status, 8u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const bool in_lds = static_cast<char*>(h) >= st.lds && static_cast<char*>(h) < st.lds + st.lds_cap;
    const bool bad = in_lds
                         ? team_histogram<U>(LdsCopy{(lds_u32*)h}, keys, n, r, row, rows, hist)
                         : team_histogram<U>(GlobalCopy{static_cast<uint32_t*>(h)}, keys, n, r,
                                             row, rows, hist);
    if (bad) s_bad = 1;
    __syncthreads();
    if (tid == 0 && s_bad) __hip_atomic_fetch_or(status, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    team_free(&st, h, (uint64_t)r.tb * 4);
}

// Without a team copy: every key is an atomic add on hist itself (performed
// at the memory side's atomic units, coherent across the XCDs).  For bins
// far beyond LDS this is the cheaper reduction: no copy to zero and merge,
// and few keys meet on one bin.
template <int U>
__global__ __launch_bounds__(1024) void histogram_direct_kernel(const int32_t* __restrict__ keys,
                                                                int64_t n, uint32_t bins,
                                                                int32_t* __restrict__ hist,
                                                                uint32_t* status) {
    __shared__ int s_bad;
    const int tid = threadIdx.x;
    const int64_t P = team_size();
    if (tid == 0) s_bad = 0;
    __syncthreads();
    uint32_t* h = reinterpret_cast<uint32_t*>(hist);
    bool bad = false;
    auto count = [&](int32_t k) {
        if ((uint32_t)k >= bins)
            bad = true;
        else
            __hip_atomic_fetch_add(h + k, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const Range blk = bal_share(n, gridDim.x, blockIdx.x);
    if (blk.lo < blk.hi) {
        const int64_t a = blk.lo, e = blk.hi;
        const uintptr_t mis = reinterpret_cast<uintptr_t>(keys + a) & 15;
        int64_t head = (int64_t)(((16 - mis) & 15) / 4);
        if (head > e - a) head = e - a;
        if (tid < head) count(keys[a + tid]);
        const int64_t p0 = a + head;
        const int64_t nv = (e - p0) / 4;
        const i32x4* __restrict__ vp = reinterpret_cast<const i32x4*>(keys + p0);
        int64_t v = tid;
        for (; v + (U - 1) * P < nv; v += U * P) {
            i32x4 r[U];
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = __builtin_nontemporal_load(vp + v + u * P);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) count(r[u][q]);
        }
        for (; v < nv; v += P) {
            const i32x4 r = __builtin_nontemporal_load(vp + v);
#pragma unroll
            for (int q = 0; q < 4; ++q) count(r[q]);
        }
        const int64_t t0 = p0 + nv * 4;
        if (tid < e - t0) count(keys[t0 + tid]);
    }
    if (bad) s_bad = 1;
    __syncthreads();
    if (tid == 0 && s_bad) __hip_atomic_fetch_or(status, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- partitioned bins
//
// Bins beyond one team's LDS copy, without reading the keys once per range:
// the keys are first partitioned by range (ranges of kPartBins bins, a
// power of two, so a key's range is key >> kPartLog2 and its place in the
// range key & (kPartBins - 1), kept as 16 bits), then each range's keys are
// counted in an LDS copy of that range alone.  Four kernels and a merge:
//   count    team t counts the valid keys of its balanced block per range
//            (LDS counters) -> cnt[r][t]
//   scan     one workgroup: off[r][t] = exclusive prefix of cnt in (r, t)
//            order, rstart[r] = off[r][0], rstart[R] = valid keys
//   scatter  team t re-reads its block and writes each valid key's 16-bit
//            place to part[off[r][t] + its rank among the team's keys of r]
//            (rank from an LDS cursor per range)
//   range    team (r, s) counts slice s of range r's part (S slices a range)
//            into an LDS copy of the range's bins; with S == 1 it adds the
//            copy into hist (it alone owns those bins), else it stores the
//            copy as partial s of those bins
//   merge    (S > 1) hist[b] += sum over s of partial[s][b]
// Key traffic: read twice, 16-bit places written once and read once (3 x
// the key bytes) against once per range for the range-by-range copies.
constexpr int kPartLog2 = 15;
constexpr uint32_t kPartBins = 1u << kPartLog2;   // 128 KiB of LDS counts
constexpr uint32_t kPartMaxRanges = 256;          // 8 388 608 bins
static_assert(kPartMaxRanges % 64 == 0 && kPartMaxRanges <= 1024, "one workgroup scans the ranges");
constexpr int kPartThreads = 512;

__device__ __forceinline__ void flag_bad(bool bad, int* s_bad, uint32_t* status) {
    if (bad) *s_bad = 1;
    __syncthreads();
    if (threadIdx.x == 0 && *s_bad)
        __hip_atomic_fetch_or(status, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The valid keys of team t's balanced block of n, in order of position, to f
// (16-byte vectors, U in flight per lane); keys outside [0, bins) set bad.
template <int U, class F>
__device__ __forceinline__ void part_keys(const int32_t* __restrict__ keys, int64_t n,
                                          uint32_t bins, F&& f, bool& bad) {
    const int tid = threadIdx.x, P = team_size();
    const Range blk = bal_share(n, gridDim.x, blockIdx.x);
    if (blk.lo >= blk.hi) return;
    auto one = [&](int32_t k) {
        if ((uint32_t)k >= bins)
            bad = true;
        else
            f((uint32_t)k);
    };
    const int64_t a = blk.lo, e = blk.hi;
    const uintptr_t mis = reinterpret_cast<uintptr_t>(keys + a) & 15;
    int64_t head = (int64_t)(((16 - mis) & 15) / 4);
    if (head > e - a) head = e - a;
    if (tid < head) one(keys[a + tid]);
    const int64_t p0 = a + head;
    const int64_t nv = (e - p0) / 4;
    const i32x4* __restrict__ vp = reinterpret_cast<const i32x4*>(keys + p0);
    int64_t v = tid;
    for (; v + (int64_t)(U - 1) * P < nv; v += (int64_t)U * P) {
        i32x4 r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = __builtin_nontemporal_load(vp + v + (int64_t)u * P);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) one(r[u][q]);
    }
    for (; v < nv; v += P) {
        const i32x4 r = __builtin_nontemporal_load(vp + v);
#pragma unroll
        for (int q = 0; q < 4; ++q) one(r[q]);
    }
    const int64_t t0 = p0 + nv * 4;
    if (tid < e - t0) one(keys[t0 + tid]);
}

constexpr int kPartPerThread = 16;
constexpr int kPartTile = kPartThreads * kPartPerThread;

// LDS counters per range are kept in C copies, lane l adding to copy l % C:
// the lanes of a wave that meet on one range then meet on up to C addresses
// instead of one (same-address lanes of an LDS atomic are served one after
// another).  C = kPartCopies for up to 32 ranges, fewer above (R x C <= 256:
// the scatter scans R x C tile counts per tile, and with many ranges few
// lanes meet anyway).
constexpr uint32_t kPartCopies = 8;
__host__ __device__ constexpr uint32_t part_copies(uint32_t R) {
    return R <= 32 ? kPartCopies : R <= 64 ? 4u : R <= 128 ? 2u : 1u;
}

// Team t counts the valid keys of its balanced block per range.
__global__ __launch_bounds__(kPartThreads) void hist_part_count_kernel(
    const int32_t* __restrict__ keys, int64_t n, uint32_t bins, uint32_t R,
    uint32_t* __restrict__ cnt, uint32_t* status) {
    __shared__ uint32_t rc[kPartMaxRanges * kPartCopies];
    __shared__ int s_bad;
    const int tid = threadIdx.x;
    const uint32_t C = part_copies(R);
    const uint32_t copy = (uint32_t)tid % C;
    if (tid == 0) s_bad = 0;
    for (uint32_t r = tid; r < R * C; r += team_size()) rc[r] = 0u;
    __syncthreads();
    bool bad = false;
    part_keys<4>(keys, n, bins,
                 [&](uint32_t k) {
                     __hip_atomic_fetch_add(rc + (k >> kPartLog2) * C + copy, 1u,
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                 },
                 bad);
    __syncthreads();
    for (uint32_t r = tid; r < R; r += team_size()) {
        uint32_t c = 0;
        for (uint32_t q = 0; q < C; ++q) c += rc[r * C + q];
        cnt[(size_t)r * gridDim.x + blockIdx.x] = c;
    }
    flag_bad(bad, &s_bad, status);
}

// Inclusive scan of v over the workgroup (wave shuffles, then the wave totals
// in LDS); returns v's inclusive prefix, *total the workgroup's sum.  Every
// thread of the workgroup calls it; the workgroup is whole waves.
__device__ inline int64_t block_scan_inclusive(int64_t v, int64_t* wsum, int64_t* total) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int nw = (team_size() + kWave - 1) / kWave;
    int64_t inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int64_t o = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += o;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    if (wave == 0) {
        int64_t w = lane < nw ? wsum[lane] : 0;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int64_t o = __shfl_up(w, d, kWave);
            if (lane >= d) w += o;
        }
        if (lane < nw) wsum[lane] = w;   // inclusive totals of waves 0..lane
    }
    __syncthreads();
    const int64_t r = inc + (wave > 0 ? wsum[wave - 1] : 0);
    *total = wsum[nw - 1];
    __syncthreads();   // wsum is reused by the next call
    return r;
}

// Places within each range: workgroup r scans range r's T team counts
// (cnt[r T + t], coalesced, a workgroup-wide piece at a time) into
// off[r T + t] = the keys teams 0..t-1 put in range r, and leaves the
// range's total in rstart[r].
__global__ __launch_bounds__(1024) void hist_part_scan_range_kernel(const uint32_t* __restrict__ cnt,
                                                                    uint32_t T,
                                                                    int64_t* __restrict__ off,
                                                                    int64_t* __restrict__ rstart) {
    __shared__ int64_t wsum[kMaxWaves];
    const size_t r = blockIdx.x;
    int64_t carry = 0;
    for (uint32_t t0 = 0; t0 < T; t0 += team_size()) {
        const uint32_t t = t0 + threadIdx.x;
        const int64_t v = t < T ? cnt[r * T + t] : 0;
        int64_t tot = 0;
        const int64_t inc = block_scan_inclusive(v, wsum, &tot);
        if (t < T) off[r * T + t] = carry + inc - v;
        carry += tot;
    }
    if (threadIdx.x == 0) rstart[r] = carry;
}

// Range starts: rstart[0..R) holds the range totals on entry and their
// exclusive prefix sums on return, rstart[R] the number of valid keys.  One
// workgroup; every total is read before any is written.
__global__ __launch_bounds__(1024) void hist_part_scan_start_kernel(uint32_t R,
                                                                    int64_t* __restrict__ rstart) {
    __shared__ int64_t wsum[kMaxWaves];
    const uint32_t r = threadIdx.x;   // R <= blockDim.x
    const int64_t v = r < R ? rstart[r] : 0;
    int64_t tot = 0;
    const int64_t inc = block_scan_inclusive(v, wsum, &tot);
    if (r < R) rstart[r] = inc - v;
    if (r == 0) rstart[R] = tot;
}

// Scatter, a tile of kPartTile keys at a time: the tile's valid keys are
// ranked within their range (LDS counters), the ranges' tile
// counts scanned, and the 16-bit places sorted by range into an LDS buffer;
// then consecutive lanes store consecutive places of one range to
// consecutive positions of its bucket, so the stores come as contiguous runs
// (not one 2-byte store per key anywhere in memory).  Within its part of a
// range's bucket a team writes its keys tile by tile; the count kernel
// fixed how many there are.
__global__ __launch_bounds__(kPartThreads) void hist_part_scatter_kernel(
    const int32_t* __restrict__ keys, int64_t n, uint32_t bins, uint32_t R,
    const int64_t* __restrict__ off, const int64_t* __restrict__ rstart,
    uint16_t* __restrict__ part) {
    const uint32_t C = part_copies(R);
    __shared__ int64_t base[kPartMaxRanges];
    __shared__ uint32_t tcnt[kPartMaxRanges * kPartCopies];       // [range][copy]
    __shared__ uint32_t toff[kPartMaxRanges * kPartCopies + 1];   // exclusive scan of tcnt
    __shared__ uint16_t buf_place[kPartTile];
    __shared__ uint16_t buf_range[kPartTile];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), P = team_size();
    const uint32_t copy = (uint32_t)tid % C;
    const uint32_t RC = R * C;
    for (uint32_t r = tid; r < R; r += P)
        base[r] = rstart[r] + off[(size_t)r * gridDim.x + blockIdx.x];
    const Range blk = bal_share(n, gridDim.x, blockIdx.x);
    // the next tile's keys are loaded while this one is sorted and stored
    uint32_t kn[kPartPerThread];
    auto load_tile = [&](int64_t t0) {
#pragma unroll
        for (int q = 0; q < kPartPerThread; ++q) {
            const int64_t i = t0 + (int64_t)q * P + tid;
            kn[q] = i < blk.hi ? (uint32_t)__builtin_nontemporal_load(keys + i) : 0xFFFFFFFFu;
        }
    };
    if (blk.lo < blk.hi) load_tile(blk.lo);
    for (int64_t t0 = blk.lo; t0 < blk.hi; t0 += kPartTile) {
        for (uint32_t e = tid; e < RC; e += P) tcnt[e] = 0u;
        uint32_t kr[kPartPerThread], rank[kPartPerThread];
#pragma unroll
        for (int q = 0; q < kPartPerThread; ++q) kr[q] = kn[q];
        if (t0 + kPartTile < blk.hi) load_tile(t0 + kPartTile);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPartPerThread; ++q)
            if (kr[q] < bins)
                rank[q] = __hip_atomic_fetch_add(tcnt + (kr[q] >> kPartLog2) * C + copy, 1u,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        if (tid < kWave) {   // exclusive scan of the tile counts in (range, copy) order, one wave
            uint32_t carry = 0;
            for (uint32_t c0 = 0; c0 < RC; c0 += kWave) {
                const uint32_t e = c0 + lane;
                const uint32_t v = e < RC ? tcnt[e] : 0u;
                uint32_t inc = v;
#pragma unroll
                for (int d = 1; d < kWave; d <<= 1) {
                    const uint32_t o = __shfl_up(inc, d, kWave);
                    if (lane >= d) inc += o;
                }
                if (e < RC) toff[e] = carry + inc - v;
                carry += __shfl(inc, kWave - 1, kWave);
            }
            if (lane == 0) toff[RC] = carry;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPartPerThread; ++q)
            if (kr[q] < bins) {
                const uint32_t r = kr[q] >> kPartLog2;
                const uint32_t at = toff[r * C + copy] + rank[q];
                buf_place[at] = (uint16_t)(kr[q] & (kPartBins - 1));
                buf_range[at] = (uint16_t)r;
            }
        __syncthreads();
        // a range's keys of the tile are buf[toff[r C] .. toff[(r + 1) C])
        const uint32_t total = toff[RC];
        for (uint32_t at = tid; at < total; at += P) {
            const uint32_t r = buf_range[at];
            part[base[r] + (at - toff[r * C])] = buf_place[at];
        }
        __syncthreads();
        for (uint32_t r = tid; r < R; r += P) base[r] += toff[(r + 1) * C] - toff[r * C];
        __syncthreads();
    }
}

// Team (r, s): slice s of S of range r's places.  out is hist (S == 1) or
// the partials, S x bins.
__global__ __launch_bounds__(kPartThreads) void hist_part_range_kernel(
    const uint16_t* __restrict__ part, const int64_t* __restrict__ rstart, uint32_t bins,
    uint32_t S, uint32_t* __restrict__ out) {
    extern __shared__ __align__(16) char arena[];
    lds_u32* h = (lds_u32*)arena;
    const int tid = threadIdx.x, P = team_size();
    const uint32_t r = blockIdx.x / S, s = blockIdx.x % S;
    const uint32_t b0 = r << kPartLog2;
    const uint32_t tb = bins - b0 < kPartBins ? bins - b0 : kPartBins;
    for (uint32_t b = tid; b < tb; b += P) h[b] = 0u;
    __syncthreads();
    const Range sl = bal_share(rstart[r + 1] - rstart[r], S, s);
    const int64_t a = rstart[r] + sl.lo, e = rstart[r] + sl.hi;
    auto add = [&](uint32_t j) {
        __hip_atomic_fetch_add(h + j, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    if (a < e) {
        const uintptr_t mis = reinterpret_cast<uintptr_t>(part + a) & 15;
        int64_t head = (int64_t)(((16 - mis) & 15) / 2);
        if (head > e - a) head = e - a;
        if (tid < head) add(part[a + tid]);
        const int64_t p0 = a + head;
        const int64_t nv = (e - p0) / 8;
        using u32x4v = uint32_t __attribute__((ext_vector_type(4)));
        const u32x4v* __restrict__ vp = reinterpret_cast<const u32x4v*>(part + p0);
        constexpr int U = 4;
        int64_t v = tid;
        for (; v + (int64_t)(U - 1) * P < nv; v += (int64_t)U * P) {
            u32x4v w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = __builtin_nontemporal_load(vp + v + (int64_t)u * P);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    add(w[u][q] & 0xFFFFu);
                    add(w[u][q] >> 16);
                }
        }
        for (; v < nv; v += P) {
            const u32x4v w = __builtin_nontemporal_load(vp + v);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                add(w[q] & 0xFFFFu);
                add(w[q] >> 16);
            }
        }
        const int64_t t0 = p0 + nv * 8;
        if (tid < e - t0) add(part[t0 + tid]);
    }
    __syncthreads();
    if (S == 1) {
        for (uint32_t b = tid; b < tb; b += P) {
            const uint32_t c = h[b];
            if (c) out[b0 + b] += c;
        }
    } else {
        uint32_t* o = out + (size_t)s * bins + b0;
        for (uint32_t b = tid; b < tb; b += P) o[b] = h[b];
    }
}

__global__ void hist_part_merge_kernel(const uint32_t* __restrict__ partial, uint32_t S,
                                       uint32_t bins, uint32_t* __restrict__ hist) {
    const int64_t b = (int64_t)blockIdx.x * team_size() + threadIdx.x;
    if (b >= bins) return;
    uint32_t c = 0;
    for (uint32_t s = 0; s < S; ++s) c += partial[(size_t)s * bins + b];
    if (c) hist[b] += c;
}

// Tile-sorted partition, up to kTsortMaxRanges ranges: every tile of
// kPartTile keys is ranked and sorted by range in LDS and stored whole into a
// slot of its own, kTsortSlot places: range r's run starts on a 16-byte
// boundary (each run is padded with kTsortPad to a multiple of eight places)
// and the runs' starts, in 16-byte vectors, go to tstart[r G + g] (G tiles;
// entry R is the slot's end).  No count pass and no scan across teams: the
// range kernel then reads range r's run of every tile.  Key traffic: read
// once, places written once and read once (2 x the key bytes), against three
// times for the partition above; the runs of a tile are 8192 / R places long
// on average (64 at 128 ranges), and the padding adds at most 8 R places a
// tile (12.5 % at 128 ranges).
//
// How many workgroups count a range follows from how many keys it has (the
// plan kernel): W workgroups are shared out over the ranges in proportion, so
// a skewed input is counted by as many as a uniform one, and a range that
// gets one adds into hist itself, without a partial.
constexpr uint32_t kTsortMaxRanges = 128;
constexpr uint32_t kTsortSlot = kPartTile + 8 * kTsortMaxRanges;   // places, 16-byte multiple
constexpr uint32_t kTsortPad = kPartBins;   // the counter past a range's bins: counted, never read
constexpr uint32_t kTsortCounters = 256;                           // ranges x copies, at most
static_assert(kTsortSlot % 8 == 0 && kTsortSlot / 8 < 65536, "slot of whole 16-byte vectors");

// Tile g of n keys whose first `head` (0..3) lie before a 16-byte boundary:
// the head alone, then kPartTile keys each.
struct TileSplit {
    int64_t n, G;
    int head;
    __host__ __device__ __forceinline__ int64_t lo(int64_t g) const {
        return head ? (g ? head + (g - 1) * (int64_t)kPartTile : 0) : g * (int64_t)kPartTile;
    }
    __host__ __device__ __forceinline__ int64_t hi(int64_t g) const {
        const int64_t h = lo(g + 1);
        return h < n ? h : n;
    }
};

// Team t sorts its balanced share of the tiles and leaves the number of keys it
// put in range r in cnt[t R + r].  Three barriers a tile: after the ranks, after
// the scan (one wave, which also clears the counters and writes the padding),
// after the sort; the copy to memory runs into the next tile's ranks.  Whole
// tiles load 16-byte vectors, and a wave whose keys are all in range skips
// their bounds checks.  2^28 keys over 32 ranges: 291 us (423 with element
// loads, six barriers, three LDS reads a key where one precombined offset
// does).
__global__ __launch_bounds__(kPartThreads, 4) void hist_tsort_scatter_kernel(
    const int32_t* __restrict__ keys, TileSplit ts, BalSplit share, uint32_t bins, uint32_t R,
    uint16_t* __restrict__ part, uint16_t* __restrict__ tstart, uint32_t* __restrict__ cnt,
    uint32_t* status) {
    constexpr int P = kPartThreads, NV = kPartPerThread / 4;
    const uint32_t C = part_copies(R);
    __shared__ __align__(16) uint32_t tcnt[kTsortCounters];   // [range][copy]
    __shared__ __align__(16) uint32_t off[kTsortCounters];    // where that copy's places go
    __shared__ uint32_t s_vectors;                            // 16-byte vectors of the sorted tile
    __shared__ __align__(16) uint16_t buf[kTsortSlot];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t copy = (uint32_t)tid % C;
    if (tid == 0) s_bad = 0;
    if (tid < (int)kTsortCounters) tcnt[tid] = 0u;
    bool bad = false;
    const Range blk = share.share(blockIdx.x);
    using u32x4v = uint32_t __attribute__((ext_vector_type(4)));
    // the next tile's keys are loaded while this one is sorted and stored;
    // positions past a partial tile's end read as 0xFFFFFFFF (not a valid key)
    u32x4v kn[NV];
    auto load_tile = [&](int64_t g) {
        const int64_t lo = ts.lo(g);
        const int count = (int)(ts.hi(g) - lo);
        const uint32_t* __restrict__ p = reinterpret_cast<const uint32_t*>(keys) + lo;
        if (count == kPartTile) {
#pragma unroll
            for (int q = 0; q < NV; ++q)
                kn[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(p) + q * P + tid);
        } else {
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = (q * P + tid) * 4 + u;
                    kn[q][u] = e < count ? p[e] : 0xFFFFFFFFu;
                }
        }
    };
    uint32_t total[kTsortMaxRanges / kWave] = {};   // the first wave: keys of the lane's ranges
    if (blk.lo < blk.hi) load_tile(blk.lo);
    __syncthreads();
    for (int64_t g = blk.lo; g < blk.hi; ++g) {
        u32x4v kr[NV], rank[NV];
        uint32_t mx = 0;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            kr[q] = kn[q];
#pragma unroll
            for (int u = 0; u < 4; ++u) mx = mx > kr[q][u] ? mx : kr[q][u];
        }
        const int count = (int)(ts.hi(g) - ts.lo(g));
        if (g + 1 < blk.hi) load_tile(g + 1);
        const bool all_in = __ballot(mx >= bins) == 0;   // wave-uniform
        auto rank_key = [&](uint32_t k) {
            return __hip_atomic_fetch_add(tcnt + (k >> kPartLog2) * C + copy, 1u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        if (all_in) {
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u) rank[q][u] = rank_key(kr[q][u]);
        } else {
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (kr[q][u] < bins)
                        rank[q][u] = rank_key(kr[q][u]);
                    else if ((q * P + tid) * 4 + u < count)
                        bad = true;
                }
        }
        __syncthreads();
        if (tid < kWave) {
            // lane l takes ranges l and l + 64: the run's padded length, its
            // start by a scan over the ranges, then each copy's part of the run
            uint32_t carry = 0;
#pragma unroll
            for (uint32_t h = 0; h < kTsortMaxRanges / kWave; ++h) {
                if (h * kWave > R) break;
                const uint32_t r = h * kWave + (uint32_t)lane;
                uint32_t c[kPartCopies], len = 0;
#pragma unroll
                for (uint32_t q = 0; q < kPartCopies; ++q) {
                    c[q] = q < C && r < R ? tcnt[r * C + q] : 0u;
                    len += c[q];
                }
                const uint32_t pl = (len + 7u) & ~7u;
                uint32_t inc = pl;
#pragma unroll
                for (int d = 1; d < kWave; d <<= 1) {
                    const uint32_t o = __shfl_up(inc, d, kWave);
                    if (lane >= d) inc += o;
                }
                const uint32_t start = carry + inc - pl;
                if (r < R) {
                    uint32_t at = start;
#pragma unroll
                    for (uint32_t q = 0; q < kPartCopies; ++q)
                        if (q < C) {
                            off[r * C + q] = at;
                            tcnt[r * C + q] = 0u;
                            at += c[q];
                        }
                    for (; at < start + pl; ++at) buf[at] = (uint16_t)kTsortPad;
                    total[h] += len;
                }
                if (r <= R) tstart[(size_t)r * ts.G + g] = (uint16_t)(start / 8);
                if (r == R) s_vectors = start / 8;
                carry += __shfl(inc, kWave - 1, kWave);
            }
            // with a multiple of 64 ranges entry R starts the next group of lanes
            if (R % kWave == 0 && lane == 0) {
                tstart[(size_t)R * ts.G + g] = (uint16_t)(carry / 8);
                s_vectors = carry / 8;
            }
        }
        __syncthreads();
        auto place_key = [&](uint32_t k, uint32_t rk) {
            buf[off[(k >> kPartLog2) * C + copy] + rk] = (uint16_t)(k & (kPartBins - 1));
        };
        if (all_in) {
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u) place_key(kr[q][u], rank[q][u]);
        } else {
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (kr[q][u] < bins) place_key(kr[q][u], rank[q][u]);
        }
        __syncthreads();
        u32x4* __restrict__ slot = reinterpret_cast<u32x4*>(part + (size_t)g * kTsortSlot);
        const u32x4* lb = reinterpret_cast<const u32x4*>(buf);
        for (uint32_t v = tid; v < s_vectors; v += P) slot[v] = lb[v];
        // buf, off and s_vectors are written again only after the next ranks'
        // barrier, which every thread reaches past this copy
    }
    if (tid < kWave)
#pragma unroll
        for (uint32_t h = 0; h < kTsortMaxRanges / kWave; ++h) {
            const uint32_t r = h * kWave + (uint32_t)lane;
            if (r < R) cnt[(size_t)blockIdx.x * R + r] = total[h];
        }
    flag_bad(bad, &s_bad, status);
}

// One workgroup: the keys of every range (cnt[t R + r] over the T teams), then
// first[r], the first of the W workgroups that count range r (first[R]: the
// number in use): one each and the rest in proportion to the keys.
__global__ __launch_bounds__(1024) void hist_tsort_plan_kernel(const uint32_t* __restrict__ cnt,
                                                               uint32_t T, uint32_t R, uint32_t W,
                                                               uint32_t* __restrict__ first) {
    __shared__ uint64_t part_sum[1024];   // [group of teams][range]
    __shared__ uint64_t sum[kTsortMaxRanges];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t rp = R <= 32 ? 32u : R <= 64 ? 64u : kTsortMaxRanges;   // ranges, padded
    const uint32_t r = tid & (rp - 1), groups = 1024 / rp, grp = tid / rp;
    uint64_t a = 0;
    if (r < R)
#pragma unroll 16
        for (uint32_t t = grp; t < T; t += groups) a += cnt[(size_t)t * R + r];
    part_sum[tid] = a;
    __syncthreads();
    if (tid < R) {
        uint64_t q = 0;
        for (uint32_t k = 0; k < groups; ++k) q += part_sum[k * rp + tid];
        sum[tid] = q;
    }
    __syncthreads();
    if (wave != 0) return;
    a = 0;
    for (uint32_t i = lane; i < R; i += kWave) a += sum[i];
    const double all = (double)wave_reduce<Red<DT_I64, OP_SUM>>(a);
    uint32_t carry = 0;
    for (uint32_t r0 = 0; r0 < R; r0 += kWave) {
        const uint32_t i = r0 + lane;
        // (the floor of an exact share or one less: never more than W in all)
        const uint32_t k =
            i < R ? 1u + (all > 0.0 ? (uint32_t)((double)(W - R) * ((double)sum[i] / all)) : 0u) : 0u;
        uint32_t inc = k;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d, kWave);
            if ((int)lane >= d) inc += o;
        }
        if (i < R) first[i] = carry + inc - k;
        carry += __shfl(inc, kWave - 1, kWave);
    }
    if (lane == 0) first[R] = carry;
}

// Workgroup w of range r (first[r] <= w < first[r + 1]): the range's runs in
// its share of the G tile slots, counted in LDS.  Each group of SW lanes takes
// K neighbouring tiles at a time, one 16-byte vector of each in flight per lane
// (the LDS copy of the range allows one workgroup a CU: sixteen waves of it
// keep 256 KiB of loads in flight; 2^28 keys, 32 ranges: 150 us, with eight
// waves 193).  A range with one workgroup adds into hist, else the counts are
// partial w.
constexpr int kRangeThreads = 1024;
template <int SW>
__global__ __launch_bounds__(kRangeThreads) void hist_tsort_range_kernel(
    const uint16_t* __restrict__ part, const uint16_t* __restrict__ tstart, int64_t G, uint32_t R,
    uint32_t bins, const uint32_t* __restrict__ first, uint32_t* __restrict__ partial,
    uint32_t* __restrict__ hist) {
    extern __shared__ __align__(16) char arena[];
    __shared__ uint32_t s_range[3];   // the range, its first workgroup, the next range's
    lds_u32* h = (lds_u32*)arena;
    constexpr int P = kRangeThreads;
    const int tid = threadIdx.x, lane = tid & (SW - 1);
    uint32_t fa = 0, fb = 0;
    if (tid < (int)R) {
        fa = first[tid];
        fb = first[tid + 1];
    }
    if (blockIdx.x >= first[R]) return;
    if (blockIdx.x >= fa && blockIdx.x < fb) {   // one thread
        s_range[0] = (uint32_t)tid;
        s_range[1] = fa;
        s_range[2] = fb;
    }
    for (int b = tid; b < (int)kPartBins / 4; b += P)
        reinterpret_cast<u32x4*>(arena)[b] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    const uint32_t r = s_range[0], s = blockIdx.x - s_range[1], S = s_range[2] - s_range[1];
    const uint32_t b0 = r << kPartLog2;
    const uint32_t tb = bins - b0 < kPartBins ? bins - b0 : kPartBins;
    const Range sl = bal_share(G, S, s);
    auto add = [&](uint32_t j) {
        __hip_atomic_fetch_add(h + j, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    constexpr int K = 8;   // tiles of a group: one lane fetches each
    constexpr int64_t step = (int64_t)K * (P / SW);
    static_assert(K <= SW, "a lane per tile of the group");
    const uint16_t* __restrict__ ta = tstart + (size_t)r * G;
    const uint16_t* __restrict__ tz = ta + G;
    // run starts and lengths of K tiles from g0 on: the next group's are loaded
    // while this group's places stream in (lane k of the group loads tile k's
    // entries; the group shares them)
    const int lane0 = (tid & (kWave - 1)) - lane;   // the group's first lane in the wave
    uint32_t st[K], nv[K];
    auto fetch = [&](int64_t g0) {
        const int64_t g = g0 + lane;
        uint32_t a = 0, b = 0;
        if (lane < K && g < sl.hi) {
            a = ta[g];
            b = tz[g];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            st[k] = (uint32_t)__shfl((int)a, lane0 + k, kWave);
            nv[k] = (uint32_t)__shfl((int)b, lane0 + k, kWave) - st[k];
        }
    };
    int64_t g0 = sl.lo + (int64_t)(tid / SW) * K;
    if (g0 < sl.hi) fetch(g0);
    for (; g0 < sl.hi; g0 += step) {
        uint32_t cst[K], cnv[K], mx = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            cst[k] = st[k];
            cnv[k] = nv[k];
            mx = cnv[k] > mx ? cnv[k] : mx;
        }
        if (g0 + step < sl.hi) fetch(g0 + step);
        for (uint32_t i = lane; i < mx; i += SW) {
            u32x4 w[K];
#pragma unroll
            for (int k = 0; k < K; ++k)
                w[k] = i < cnv[k] ? __builtin_nontemporal_load(
                                        reinterpret_cast<const u32x4*>(part + (g0 + k) * kTsortSlot) +
                                        cst[k] + i)
                                  : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (i < cnv[k])
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        add(w[k][q] & 0xFFFFu);
                        add(w[k][q] >> 16);
                    }
        }
    }
    __syncthreads();
    if (S == 1) {
        constexpr int U = 16;   // the bins' old counts load together
        for (uint32_t b = tid; b < tb; b += U * P) {
            uint32_t c[U], old[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                c[u] = b + u * P < tb ? h[b + u * P] : 0u;
                old[u] = 0u;
                if (c[u]) old[u] = hist[b0 + b + u * P];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c[u]) hist[b0 + b + u * P] = old[u] + c[u];
        }
    } else {
        uint32_t* o = partial + (size_t)blockIdx.x * kPartBins;
        for (uint32_t b = tid; b < tb; b += P) o[b] = h[b];
    }
}

// hist[b] += the partials of b's range, where it has several.
__global__ __launch_bounds__(256) void hist_tsort_merge_kernel(const uint32_t* __restrict__ partial,
                                                               const uint32_t* __restrict__ first,
                                                               uint32_t bins,
                                                               uint32_t* __restrict__ hist) {
    const uint32_t b = blockIdx.x * 256 + threadIdx.x;
    const uint32_t r = b >> kPartLog2;   // the same for the whole workgroup
    if (b >= bins) return;
    const uint32_t w0 = first[r], w1 = first[r + 1];
    if (w1 - w0 == 1) return;
    uint32_t c = 0;
#pragma unroll 8
    for (uint32_t w = w0; w < w1; ++w) c += partial[(size_t)w * kPartBins + (b & (kPartBins - 1))];
    if (c) hist[b] += c;
}

// Global pool of the team copies that do not fit LDS: per (device, stream),
// grown on demand outside capture.
struct Pool {
    void* ptr = nullptr;
    uint64_t bytes = 0;
};
static std::mutex g_hmu;
static std::map<std::pair<int, hipStream_t>, Pool> g_pools;

static omprt_status pool_get(hipStream_t stream, uint64_t bytes, void** out) {
    int dev = 0;
    OMPRT_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_hmu);
    Pool& p = g_pools[{dev, stream}];
    if (p.bytes < bytes) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        OMPRT_HIP(hipStreamIsCapturing(stream, &cs));
        if (cs != hipStreamCaptureStatusNone)
            return fail(OMPRT_ERR_INVALID, "stream is being captured and the histogram pool is "
                                           "too small: make the same call once before capturing");
        void* q = nullptr;
        if (hipMalloc(&q, bytes) != hipSuccess)
            return fail(OMPRT_ERR_NOMEM, "histogram pool of %llu bytes", (unsigned long long)bytes);
        retire_device_memory(dev, p.ptr);   // a captured graph may still name it
        p.ptr = q;
        p.bytes = bytes;
    }
    *out = p.ptr;
    return OMPRT_OK;
}

void histogram_finalize() {
    std::lock_guard<std::mutex> lk(g_hmu);
    for (auto& kv : g_pools) {
        (void)hipSetDevice(kv.first.first);
        (void)hipFree(kv.second.ptr);
    }
    g_pools.clear();
}

// Dynamic LDS a team's copy may take: the device's LDS per workgroup (160 KiB
// on gfx950: 40 704 bins) less 1 KiB of room for the kernel's static LDS.
constexpr uint32_t kHistStaticLds = 1024;
static uint32_t hist_lds_cap() {
    static uint32_t cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 64 * 1024 - kHistStaticLds;
    if (!cached[dev]) {
        int bytes = 0;
        if (hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
                hipSuccess ||
            bytes < 64 * 1024)
            bytes = 64 * 1024;
        cached[dev] = (uint32_t)bytes - kHistStaticLds;
    }
    return cached[dev];
}
// Bin ranges before atomics on hist: a key is read once per range, so ranges
// cost about 1.6 T keys/s / ranges at 2^28 keys (2: 808 G/s, 16: 125 G/s with
// 64 KiB ranges) against about 27 G keys/s for atomics on hist; 32 ranges
// keep a 2x margin.
constexpr uint32_t kMaxBinTiles = 32;
// Ranges the default takes before partitioning the keys: ranges cost one
// read of the keys each, the partition about three plus its passes' fixed
// costs; at 2^28 uniform keys 3 ranges ran at 441 G keys/s against 267 for
// the partition, 7 ranges at 197 against 319.
constexpr uint32_t kDefaultMaxBinTiles = 4;
// LDS ranges the default takes before the tile sort (which reads the keys
// once and moves 2-byte places twice): at 2^28 uniform keys 3 ranges ran at
// 444 G keys/s against 600 for the tile sort, 2 ranges at 813 against 590 (few
// keys take up to kMaxBinTiles ranges, see omprt_histogram).
constexpr uint32_t kDefaultMaxTsortTiles = 2;

// Default shape of the LDS copies.  A team of 1024 threads counts about 8500
// keys a microsecond and adding its copy into hist takes about 3e-6 us a bin
// and team (coalesced atomics) and 6e-3 us a team (teams meeting on the same
// bins), so the time n / (8500 T) + T (3e-6 bins + 6e-3) is least at
// T = sqrt(39 n / (bins + 2000)): one team a CU for 10^8 keys, 30 teams for 10^6
// keys and 40 000 bins (16 us; 512 teams of 512 threads, the earlier default,
// 36), 114 for 10^6 keys and 1000 bins (8.3 against 13).  One team of 1024 a CU
// also beats two of 512 where a copy leaves room for one team only (2^28 keys,
// 40 000 bins: 176 against 274 us); with small copies and 9e7 keys or more, two
// of 1024 are ahead of one (217 bins: 1e8 keys 65.6 against 67.3 us, 2e8 125.9
// against 128.8, 3e8 185 against 193; 5e7 40.0 against 35.5) and of two of 512
// (2e8 137).  The counts above are for keys spread over the bins.  Keys that
// meet on few bins are counted one after another, longer the fewer the teams
// (10^6 keys of 16384 bins: uniform 28.3 -> 8.8 us, skewed 19.5 -> 12.3, but
// sorted 8.0 -> 13.6 and two values 12.8 -> 15.6).
static void hist_shape(int64_t n, uint32_t bins, uint32_t tiles, int cus, int* teams,
                       int* threads) {
    const double best = sqrt(39.0 * (double)n / ((double)bins + 2000.0));
    if (best >= 3.0 * cus && n >= 90000000 && tiles == 1 && bins * 4 <= 64 * 1024) {
        *teams = 2 * cus;
        *threads = 1024;
        return;
    }
    const int64_t rows = std::min<int64_t>(std::max<int64_t>((int64_t)best, 1),
                                           std::max<int64_t>(cus / (int64_t)tiles, 1));
    *teams = (int)(rows * tiles);
    *threads = 1024;
}

// Partitioned bins (count, scan, scatter, range, merge), teams x 512
// threads for the passes over the keys.
static omprt_status histogram_partitioned(const int32_t* d_keys, int64_t n, uint32_t bins,
                                          int32_t* d_hist, int teams, hipStream_t stream) {
    const uint32_t R = (bins + kPartBins - 1) >> kPartLog2;
    if (R > kPartMaxRanges)
        return fail(OMPRT_ERR_INVALID, "partitioned histogram: %u bins above %u", bins,
                    kPartMaxRanges * kPartBins);
    const uint32_t T = (uint32_t)teams;
    uint32_t S = (uint32_t)((2 * device_cus() + R - 1) / R);
    S = std::min<uint32_t>(std::max<uint32_t>(S, 1u), 64u);
    auto up = [](uint64_t b) { return (b + 255) / 256 * 256; };
    const uint64_t b_part = up((uint64_t)n * 2), b_cnt = up((uint64_t)R * T * 4),
                   b_off = up((uint64_t)R * T * 8), b_rs = up((uint64_t)(R + 1) * 8),
                   b_partial = S > 1 ? up((uint64_t)S * bins * 4) : 0;
    void* pool = nullptr;
    if (omprt_status st = pool_get(stream, b_part + b_cnt + b_off + b_rs + b_partial, &pool))
        return st;
    char* p = static_cast<char*>(pool);
    uint16_t* part = reinterpret_cast<uint16_t*>(p);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(p + b_part);
    int64_t* off = reinterpret_cast<int64_t*>(p + b_part + b_cnt);
    int64_t* rstart = reinterpret_cast<int64_t*>(p + b_part + b_cnt + b_off);
    uint32_t* partial = reinterpret_cast<uint32_t*>(p + b_part + b_cnt + b_off + b_rs);
    Workspace* ws = nullptr;
    if (omprt_status st = workspace_get(stream, 1, &ws)) return st;
    uint32_t* hist = reinterpret_cast<uint32_t*>(d_hist);
    hipLaunchKernelGGL(hist_part_count_kernel, dim3(T), dim3(kPartThreads), 0, stream, d_keys, n,
                       bins, R, cnt, ws->status());
    const uint32_t scan_threads = std::min<uint32_t>((T + kWave - 1) / kWave * kWave, 1024u);
    hipLaunchKernelGGL(hist_part_scan_range_kernel, dim3(R), dim3(scan_threads), 0, stream, cnt,
                       T, off, rstart);
    hipLaunchKernelGGL(hist_part_scan_start_kernel, dim3(1), dim3(kPartMaxRanges), 0, stream, R,
                       rstart);
    hipLaunchKernelGGL(hist_part_scatter_kernel, dim3(T), dim3(kPartThreads), 0, stream, d_keys,
                       n, bins, R, off, rstart, part);
    const uint32_t lds = std::min(bins, kPartBins) * 4;
    if (lds > 64 * 1024) {   // past the default dynamic LDS limit: ask for it
        const hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void*>(hist_part_range_kernel),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return fail(OMPRT_ERR_DEVICE, "histogram: %u bytes of LDS: %s", lds,
                        hipGetErrorString(e));
    }
    hipLaunchKernelGGL(hist_part_range_kernel, dim3(R * S), dim3(kPartThreads), lds, stream, part,
                       rstart, bins, S, S > 1 ? partial : hist);
    if (S > 1)
        hipLaunchKernelGGL(hist_part_merge_kernel, dim3((bins + 255) / 256), dim3(256), 0, stream,
                           partial, S, bins, hist);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "histogram launch: %s", hipGetErrorString(e));
    return OMPRT_OK;
}

// Tile-sorted bins (scatter into tile slots, plan, range, merge), up to
// kTsortMaxRanges ranges; teams x 512 threads for the pass over the keys.
static omprt_status histogram_tsorted(const int32_t* d_keys, int64_t n, uint32_t bins,
                                      int32_t* d_hist, int teams, hipStream_t stream) {
    const uint32_t R = (bins + kPartBins - 1) >> kPartLog2;
    if (R > kTsortMaxRanges)
        return fail(OMPRT_ERR_INVALID, "tile-sorted histogram: %u bins above %u", bins,
                    kTsortMaxRanges * kPartBins);
    TileSplit ts{};
    ts.n = n;
    ts.head = (int)std::min<int64_t>((16 - (reinterpret_cast<uintptr_t>(d_keys) & 15)) % 16 / 4, n);
    ts.G = (n - ts.head + kPartTile - 1) / kPartTile + (ts.head ? 1 : 0);
    const uint32_t T = (uint32_t)std::min<int64_t>(teams, ts.G);   // no team without a tile
    // Workgroups of the counting pass: one a range, and more as there are keys
    // to count, up to one a CU, or two with so many ranges that whole shares
    // would leave part of the chip idle.  A further workgroup costs a partial of
    // 128 KiB written and read (about what 32768 keys cost; with many ranges
    // three times that, 10^7 keys over 128 ranges: 82 us at 32768, 69 so).
    const uint32_t cus = (uint32_t)device_cus();
    const uint32_t most = std::max(R <= 64 ? cus : 2 * cus, R);
    const int64_t keys_each = R <= 64 ? 32768 : 98304;
    const uint32_t W = (uint32_t)std::min<int64_t>(most, R + n / keys_each);
    auto up = [](uint64_t b) { return (b + 255) / 256 * 256; };
    // room for the tiles at any alignment of the keys, and for partials that grow
    // with the keys and the ranges, so that a call made once covers a capture with
    // other keys, and with fewer keys or bins
    const uint64_t W_any = (uint64_t)std::min<int64_t>(std::max(2 * cus, R), R + n / 32768);
    const uint64_t G_any = (uint64_t)((n + kPartTile - 1) / kPartTile + 1);
    const uint64_t b_part = up(G_any * kTsortSlot * 2), b_ts = up(G_any * (R + 1) * 2),
                   b_cnt = up((uint64_t)R * std::min<uint64_t>((uint64_t)teams, G_any) * 4),
                   b_first = up((uint64_t)(R + 1) * 4),
                   b_partial = W_any > R ? W_any * kPartBins * 4 : 0;
    void* pool = nullptr;
    if (omprt_status st = pool_get(stream, b_part + b_ts + b_cnt + b_first + b_partial, &pool))
        return st;
    char* p = static_cast<char*>(pool);
    uint16_t* part = reinterpret_cast<uint16_t*>(p);
    uint16_t* tstart = reinterpret_cast<uint16_t*>(p + b_part);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(p + b_part + b_ts);
    uint32_t* first = reinterpret_cast<uint32_t*>(p + b_part + b_ts + b_cnt);
    uint32_t* partial = reinterpret_cast<uint32_t*>(p + b_part + b_ts + b_cnt + b_first);
    Workspace* ws = nullptr;
    if (omprt_status st = workspace_get(stream, 1, &ws)) return st;
    uint32_t* hist = reinterpret_cast<uint32_t*>(d_hist);
    hipLaunchKernelGGL(hist_tsort_scatter_kernel, dim3(T), dim3(kPartThreads), 0, stream, d_keys, ts,
                       bal_split(ts.G, T), bins, R, part, tstart, cnt, ws->status());
    hipLaunchKernelGGL(hist_tsort_plan_kernel, dim3(1), dim3(1024), 0, stream, cnt, T, R, W, first);
    const uint32_t lds = (kPartBins + 4) * 4;   // a range's bins and the padding's counter
    hipError_t attr = hipSuccess;
    auto range = [&](auto kernel) {   // past the default dynamic LDS limit: ask for it
        attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (attr == hipSuccess)
            hipLaunchKernelGGL(kernel, dim3(W), dim3(kRangeThreads), lds, stream, part, tstart, ts.G,
                               R, bins, first, partial, hist);
    };
    // runs average kPartTile / R places: half a wave takes a tile, from 48 ranges
    // on (21 vectors or fewer) a quarter (2^28 keys: 4 ranges 143 us, 228 with
    // whole waves; 32 ranges 150, 177 with quarters; 128 ranges 236, 277 with
    // eighths)
    if (R >= 48)
        range(hist_tsort_range_kernel<16>);
    else
        range(hist_tsort_range_kernel<32>);
    if (attr != hipSuccess)
        return fail(OMPRT_ERR_DEVICE, "histogram: %u bytes of LDS: %s", lds, hipGetErrorString(attr));
    if (W > R)
        hipLaunchKernelGGL(hist_tsort_merge_kernel, dim3((bins + 255) / 256), dim3(256), 0, stream,
                           partial, first, bins, hist);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "histogram launch: %s", hipGetErrorString(e));
    return OMPRT_OK;
}

}  // namespace omprt

using namespace omprt;

extern "C" omprt_status omprt_histogram(const int32_t* d_keys, int64_t n, int32_t bins,
                                        int32_t* d_hist, const omprt_config* cfg,
                                        void* hip_stream) {
    if (n < 0 || n > ((int64_t)1 << 50))
        return fail(OMPRT_ERR_INVALID, "n = %lld outside 0..2^50", (long long)n);
    if (bins < 1 || bins > (1 << 28)) return fail(OMPRT_ERR_INVALID, "bins %d outside 1..2^28", bins);
    if (!d_hist) return fail(OMPRT_ERR_INVALID, "hist is NULL");
    if (n > 0 && !d_keys) return fail(OMPRT_ERR_INVALID, "keys is NULL with n > 0");
    if ((reinterpret_cast<uintptr_t>(d_keys) | reinterpret_cast<uintptr_t>(d_hist)) & 3)
        return fail(OMPRT_ERR_INVALID, "keys / hist not 4-byte aligned");
    const int cus = device_cus();
    int teams = 2 * cus, threads = 512, unroll = 4;
    const bool auto_shape = !cfg || (!cfg->num_teams && !cfg->threads_per_team);
    if (cfg) {
        if (cfg->num_teams < 0 || cfg->num_teams > 65535)
            return fail(OMPRT_ERR_INVALID, "num_teams %d", cfg->num_teams);
        if (cfg->threads_per_team &&
            (cfg->threads_per_team < 64 || cfg->threads_per_team > 1024 || cfg->threads_per_team % 64))
            return fail(OMPRT_ERR_INVALID, "threads_per_team %d", cfg->threads_per_team);
        if (cfg->unroll && cfg->unroll != 1 && cfg->unroll != 2 && cfg->unroll != 4)
            return fail(OMPRT_ERR_INVALID, "unroll %d (1, 2 or 4)", cfg->unroll);
        if (cfg->num_teams) teams = cfg->num_teams;
        if (cfg->threads_per_team) threads = cfg->threads_per_team;
        if (cfg->unroll) unroll = cfg->unroll;
    }
    const uint32_t flags = cfg ? cfg->flags : 0u;
    const uint32_t forced = flags & (OMPRT_CFG_HIST_DIRECT | OMPRT_CFG_HIST_TEAM_COPY |
                                     OMPRT_CFG_HIST_PARTITION | OMPRT_CFG_HIST_RANGES |
                                     OMPRT_CFG_HIST_TILE_SORT);
    if (forced & (forced - 1))
        return fail(OMPRT_ERR_INVALID, "at most one of HIST_DIRECT, HIST_TEAM_COPY, "
                                       "HIST_PARTITION, HIST_RANGES, HIST_TILE_SORT");
    if ((flags & OMPRT_CFG_HIST_PARTITION) && bins > (int64_t)kPartMaxRanges * kPartBins)
        return fail(OMPRT_ERR_INVALID, "HIST_PARTITION takes up to %u bins",
                    kPartMaxRanges * kPartBins);
    if ((flags & OMPRT_CFG_HIST_TILE_SORT) && bins > (int64_t)kTsortMaxRanges * kPartBins)
        return fail(OMPRT_ERR_INVALID, "HIST_TILE_SORT takes up to %u bins",
                    kTsortMaxRanges * kPartBins);
    if (n == 0) return OMPRT_OK;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // Bins that do not fit one team's LDS: up to four ranges of bins, each
    // counted by its own teams (every team reads its block of the keys and
    // counts those in its range); from five ranges on, the keys partitioned by
    // range first: up to kTsortMaxRanges ranges each tile sorted by range into
    // a slot of its own (keys read once, 16-bit places written and read
    // once), then up to kPartMaxRanges x kPartBins bins partitioned across
    // teams (keys read twice), both within 16 GiB of places; past that,
    // atomics on hist.  On request: ranges up to kMaxBinTiles of them, team
    // copies in the global pool (atomics at L2, then a merge), either
    // partition, or atomics on hist for any bin count.
    const uint32_t lds_bins = hist_lds_cap() / 4 / 4 * 4;
    uint32_t tiles = (uint32_t)((bins + lds_bins - 1) / lds_bins);
    uint32_t tile_bins = tiles > 1 ? (uint32_t)((bins + tiles - 1) / tiles + 3) / 4 * 4 : (uint32_t)bins;
    const bool part_fits = bins <= (int64_t)kPartMaxRanges * kPartBins &&
                           (uint64_t)n * 2 <= ((uint64_t)16 << 30);
    const bool tsort_fits = part_fits && bins <= (int64_t)kTsortMaxRanges * kPartBins;
    // few keys: the ranges in one launch (each team reads its block once per
    // range) while they take less than the partitions' four launches, 25 us:
    // 2 sqrt(n / 8500 (3e-6 bins + 6e-3)) + 6 < 24 (hist_shape's time at its best
    // T; 10^5 keys, 2^20 bins: 21 us, 51 before)
    const bool few_keys = !forced && auto_shape && tiles > kDefaultMaxTsortTiles &&
                          tiles <= kMaxBinTiles && (double)n * ((double)bins + 2000.0) < 2.3e11;
    if ((flags & OMPRT_CFG_HIST_TILE_SORT) ||
        (!forced && tiles > kDefaultMaxTsortTiles && tsort_fits && !few_keys))
        return histogram_tsorted(d_keys, n, (uint32_t)bins, d_hist, teams, stream);
    if ((flags & OMPRT_CFG_HIST_PARTITION) ||
        (!forced && tiles > kDefaultMaxBinTiles && part_fits && !few_keys))
        return histogram_partitioned(d_keys, n, (uint32_t)bins, d_hist, teams, stream);
    const bool direct = (flags & OMPRT_CFG_HIST_DIRECT) ||
                        (tiles > kMaxBinTiles && !(flags & OMPRT_CFG_HIST_TEAM_COPY)) ||
                        (!forced && tiles > kDefaultMaxBinTiles && !few_keys);
    if (direct) {
        Workspace* ws = nullptr;
        if (omprt_status st = workspace_get(stream, 1, &ws)) return st;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)teams), dim3(threads), 0, stream, d_keys, n,
                               (uint32_t)bins, d_hist, ws->status());
        };
        switch (unroll) {
            case 1: launch(histogram_direct_kernel<1>); break;
            case 2: launch(histogram_direct_kernel<2>); break;
            default: launch(histogram_direct_kernel<4>); break;
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "histogram launch: %s", hipGetErrorString(e));
        return OMPRT_OK;
    }
    const bool in_lds = tiles <= kMaxBinTiles;
    if (!in_lds) {
        tiles = 1;
        tile_bins = (uint32_t)bins;
    }
    if (auto_shape && in_lds) hist_shape(n, (uint32_t)bins, tiles, cus, &teams, &threads);
    const uint64_t hbytes = ((uint64_t)tile_bins * 4 + kSharedAlign - 1) / kSharedAlign * kSharedAlign;
    const int64_t rows = std::max<int64_t>(1, teams / (int64_t)tiles);
    const int64_t grid = rows * tiles;
    if (grid > INT32_MAX) return fail(OMPRT_ERR_INVALID, "grid too large");
    void* pool = nullptr;
    uint64_t per_team = 0;
    if (!in_lds) {
        per_team = (hbytes + 255) / 256 * 256;
        if (omprt_status st = pool_get(stream, per_team * (uint64_t)grid, &pool)) return st;
    }
    Workspace* ws = nullptr;
    if (omprt_status st = workspace_get(stream, 1, &ws)) return st;
    const uint32_t lds = in_lds ? (uint32_t)hbytes : 0u;
    hipError_t attr = hipSuccess;
    auto launch = [&](auto kernel) {
        if (lds > 64 * 1024)   // past the default dynamic LDS limit: ask for it
            attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (attr != hipSuccess) return;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(threads), lds, stream, d_keys, n,
                           (uint32_t)bins, tiles, tile_bins, d_hist, static_cast<char*>(pool),
                           per_team, lds, ws->status());
    };
    switch (unroll) {
        case 1: launch(histogram_kernel<1>); break;
        case 2: launch(histogram_kernel<2>); break;
        default: launch(histogram_kernel<4>); break;
    }
    if (attr != hipSuccess)
        return fail(OMPRT_ERR_DEVICE, "histogram: %u bytes of LDS: %s", lds, hipGetErrorString(attr));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "histogram launch: %s", hipGetErrorString(e));
    return OMPRT_OK;
}
