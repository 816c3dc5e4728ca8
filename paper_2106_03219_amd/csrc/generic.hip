// generic.hip -- a target region in generic (non-SPMD) mode: each team's
// main thread (thread 0) runs the region's sequential code and hands each
// parallel loop to its team through a work descriptor in team-shared
// memory (the routines a compiled target region calls, paper sec. 2.1).
// The other threads wait at the team barrier for work -- a state machine --
// run their share of the loop and meet the main thread, which works on the
// loop as thread 0 of the team, at the join barrier.  Loops with no sequential
// code between them that needs their results are handed out together.  One
// launch runs the whole region, however many parallel loops it has, so nothing
// returns to the host between them.
//
// The region is a power iteration on a diagonal matrix D = diag(d):
//   repeat iters times:
//     parallel loop:   w = d * v (written over v), s = sum of w^2
//     sequential code: r = 1 / sqrt(s)
//     parallel loop:   v = w * r
//   sequential code:   lambda = sqrt(s)
// s accumulates in compensated fp32 (TwoSum per element, float-float
// through the team tree).
//
// With one team (the mode's own shape) the team owns [0, n).  With T > 1
// co-resident teams the loops are also distributed: team k owns the
// balanced block bal(n, T, k) in both loops, every team runs the
// sequential code on the same values, and the sum reaches all of them by an
// all-gather of team partials: each team publishes its partial as tagged
// slot words (the cross-team slots of the reductions; tag = the launch tag
// of epoch + step), then reads every team's partial in team order, so all
// teams hold bit-identical s.  Steps alternate between two slot sets: a
// team can run at most one step ahead of another (step k + 1's all-gather
// needs everyone's step k + 1 partial), so a set is overwritten only after
// every team has read it.  The normalising loop touches only the team's own
// block, so it needs no cross-team wait.  Inside a team loops take the
// static schedule with chunk 1 (thread t owns lo + t, lo + t + P, ...), so
// a wave's lanes touch neighbouring elements and each thread rewrites in
// the second loop exactly the elements it wrote in the first.
#include <algorithm>

#include "device.h"
#include "runtime.h"
#include "sched.h"

namespace omprt {

// The work descriptor: the loops the team runs next.  The normalising loop of
// one step and the scaling loop of the next have no sequential code between
// them that needs either's result and put every element on the same thread, so
// they are handed out together (two worksharing loops of one parallel region,
// the first nowait): a step then has one hand-off and one join.
enum { WORK_SCALE = 0, WORK_NORMALISE_SCALE = 1, WORK_NORMALISE_EXIT = 2 };

constexpr int kGenericUnroll = 8;   // loads in flight per lane and array
// Teams of the distributed form: each team reads every team's partial once a
// step, so the all-gather grows as teams^2 (512 teams: 4 MiB of reads).
constexpr int kMaxGenericTeams = 512;
constexpr int kGatherWords = 2;     // 64-bit words of a team's partial
// Copies of every partial, each read by every kGatherCopies-th team: all teams
// poll at the same time, and one copy of 256 partials is 4 KiB on a few memory
// channels that would serve every team's reads.
constexpr int kGatherCopies = 8;

__device__ __forceinline__ float scaled_square(float d, float v, ff_t& acc) {
    const float w = d * v;
    comp_add(acc, w * w);
    return w;
}

// The calling thread's iterations lo + t, lo + t + P, ... of both loops, with v
// and d in memory: the loops' pair reads d and v and writes v, 12 bytes an
// element and step.
struct MemoryShare {
    const float* __restrict__ d;
    float* __restrict__ v;
    int64_t i0, hi, P;
    __device__ __forceinline__ MemoryShare(const float* d_, float* v_, const Range& blk)
        : d(d_), v(v_), i0(blk.lo + threadIdx.x), hi(blk.hi), P(team_size()) {}
    // v = w = d * (NORMALISE ? v * r : v), acc += w * w
    template <bool NORMALISE>
    __device__ __forceinline__ void scale(float r, ff_t& acc) {
        constexpr int U = kGenericUnroll;
        int64_t i = i0;
        for (; i + (U - 1) * P < hi; i += U * P) {
            float a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = d[i + u * P];
                b[u] = v[i + u * P];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                v[i + u * P] = scaled_square(a[u], NORMALISE ? b[u] * r : b[u], acc);
        }
        for (; i < hi; i += P) v[i] = scaled_square(d[i], NORMALISE ? v[i] * r : v[i], acc);
    }
    __device__ __forceinline__ void finish(float r) {
        constexpr int U = kGenericUnroll;
        int64_t i = i0;
        for (; i + (U - 1) * P < hi; i += U * P) {
            float b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) b[u] = v[i + u * P];
#pragma unroll
            for (int u = 0; u < U; ++u) v[i + u * P] = b[u] * r;
        }
        for (; i < hi; i += P) v[i] *= r;
    }
};

// The same with the thread's elements (at most E) in registers for the whole
// region: d and v are read once, v is written once, and a step touches no
// memory but the all-gather's slots.  Elements past the share are zeros, which
// add exactly nothing to the sum (an infinite or NaN r makes them NaN, but then
// every real element of the loop is infinite or NaN and the sum NaN as well).
template <int E>
struct RegisterShare {
    float d[E], v[E];
    float* __restrict__ out;   // the block's first element
    int len, P;                // the block has at most E * P elements
    __device__ __forceinline__ RegisterShare(const float* __restrict__ d_, float* __restrict__ v_,
                                             const Range& blk)
        : out(v_ + blk.lo), len((int)(blk.hi - blk.lo)), P(team_size()) {
        const float* __restrict__ in = d_ + blk.lo;
        // an empty block reads its neighbour's element before it (blk.lo <= n)
        const int none = len > 0 ? 0 : -1;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = (int)threadIdx.x + e * P;
            const float a = in[i < len ? i : none], b = out[i < len ? i : none];
            d[e] = i < len ? a : 0.0f;
            v[e] = i < len ? b : 0.0f;
        }
    }
    template <bool NORMALISE>
    __device__ __forceinline__ void scale(float r, ff_t& acc) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            v[e] = scaled_square(d[e], NORMALISE ? v[e] * r : v[e], acc);
            // keeps the products of later elements from being formed (and held
            // in registers) ahead of the sum's chain
            if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ __forceinline__ void finish(float r) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));   // the offsets are formed here, not kept through the region
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = t + e * P;
            if (i < len) out[i] = v[e] * r;
        }
    }
};

// All-gather by one wave: every team's partial of this step, combined in team
// order (lane l takes teams l, l + 64, ..., then the wave's tree).  The words
// of up to kBatch teams load together, again and again until all of them carry
// the tag (a word polled after another would wait out its own latency).
// Bounded like poll_slot_word; every 256 polls it also looks at *status, so
// once one poll of the launch has timed out the others give up at once instead
// of each waiting out its own limit.  Result in every lane.
__device__ __forceinline__ ff_t gather_partials(const uint64_t* set, int T, uint32_t tag,
                                                uint32_t* status) {
    using R = Red<DT_F32, OP_SUM>;
    constexpr int kBatch = 4;
    ff_t c = R::identity();
    for (int t0 = threadIdx.x & (kWave - 1); t0 < T; t0 += kBatch * kWave) {
        uint64_t w[kBatch][kGatherWords];
        for (uint32_t polls = 1;; ++polls) {
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int t = t0 + b * kWave < T ? t0 + b * kWave : t0;
#pragma unroll
                for (int i = 0; i < kGatherWords; ++i)
                    w[b][i] = load_slot_word(set + (size_t)t * kGatherWords + i);
            }
            bool all = true;
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
#pragma unroll
                for (int i = 0; i < kGatherWords; ++i) all = all && (uint32_t)(w[b][i] >> 32) == tag;
            if (all) break;
            if (polls >= kPollLimit) {
                __hip_atomic_fetch_or(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            if ((polls & 255) == 0 &&
                (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u))
                break;
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
            if (t0 + b * kWave < T)
                c = R::combine(c, ff_t{__uint_as_float((uint32_t)w[b][0]),
                                       __uint_as_float((uint32_t)w[b][1])});
    }
    return wave_reduce<R>(c);
}

// Workspace slots (of kSlotWords words) the two sets take per team.
constexpr int kGenericSlots = 2 * kGatherCopies * kGatherWords / kSlotWords;

// SHARE: MemoryShare or RegisterShare<E>; at most MAXP threads a team, at least
// MINW waves a SIMD (8: two teams of 1024 threads a CU, which the documented
// limit of 512 teams needs).
template <bool TEAMS, class SHARE, int MAXP, int MINW>
__global__ __launch_bounds__(MAXP, MINW) void generic_power_kernel(const float* __restrict__ d,
                                                             float* __restrict__ v, int64_t n,
                                                             int iters, float* __restrict__ lambda,
                                                             CrossTeam ct) {
    using R = Red<DT_F32, OP_SUM>;
    __shared__ int s_work;       // the work descriptor: which loops run next
    __shared__ float s_scale;    // and their argument
    __shared__ ff_t s_red[kMaxWaves];
    const int tid = threadIdx.x;
    const int64_t T = gridDim.x;
    const Range blk = TEAMS ? bal_share(n, T, blockIdx.x) : Range{0, n};
    const uint32_t epoch = TEAMS ? read_epoch(ct.epoch) : 0u;
    SHARE share(d, v, blk);
    float s = 0.0f;   // the main thread's sequential state (only thread 0's copy is used)
    for (int k = 0;; ++k) {   // k: steps whose sum is complete
        if (tid == 0) {   // sequential code
            if (k == 0) {
                s_work = WORK_SCALE;
            } else {
                s_scale = 1.0f / sqrtf(s);
                s_work = k == iters ? WORK_NORMALISE_EXIT : WORK_NORMALISE_SCALE;
            }
        }
        __syncthreads();   // the team picks up the work descriptor
        const int work = s_work;
        ff_t acc = R::identity();
        if (work == WORK_NORMALISE_EXIT) {
            share.finish(s_scale);
            break;
        }
        if (work == WORK_SCALE)
            share.template scale<false>(1.0f, acc);
        else
            share.template scale<true>(s_scale, acc);
        // The tree's barrier is the join: every thread has read the descriptor
        // and finished its loops.  Thread 0 has the sum; the slots are written
        // again only after the next hand-off, which thread 0's wave reaches
        // last.
        acc = team_reduce<R>(acc, s_red);
        if constexpr (TEAMS) {
            if (tid < kWave) {
                const uint32_t tag = launch_tag(epoch + (uint32_t)k);
                uint64_t* set = ct.slots + (size_t)(k & 1) * T * (kGatherCopies * kGatherWords);
                acc.hi = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(acc.hi)));
                acc.lo = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(acc.lo)));
                if (tid < kGatherCopies)
                    publish_tagged(acc, set + ((size_t)tid * T + blockIdx.x) * kGatherWords, tag);
                acc = gather_partials(set + (size_t)(blockIdx.x % kGatherCopies) * T * kGatherWords,
                                      (int)T, tag, ct.status);
            }
        }
        if (tid == 0) s = acc.hi + acc.lo;
    }
    if (blockIdx.x == 0 && tid == 0) {
        lambda[0] = sqrtf(s);
        // Every team read the epoch before publishing its first partial, and team
        // 0 has read every team's last partial: the next launch may take new tags.
        if (TEAMS)
            __hip_atomic_store(ct.epoch, epoch + (uint32_t)iters, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The kernel variants: elements a thread holds in registers (0: in memory) and
// the largest team.  32 elements of d and of v leave room for the 16 waves of a
// 1024-thread team a CU (128 registers a lane), 64 for 512 threads, 128 for 256
// (512 registers a lane).
struct GenericVariant {
    int elems, max_threads;
    const void* one;    // one team
    const void* many;   // co-resident teams
};
template <class SHARE, int MAXP, int MINW>
static GenericVariant generic_variant(int elems) {
    return GenericVariant{
        elems, MAXP, reinterpret_cast<const void*>(&generic_power_kernel<false, SHARE, MAXP, MINW>),
        reinterpret_cast<const void*>(&generic_power_kernel<true, SHARE, MAXP, MINW>)};
}
static const GenericVariant* generic_variants(int* count) {
    static const GenericVariant v[] = {
        generic_variant<RegisterShare<4>, 1024, 8>(4),
        generic_variant<RegisterShare<8>, 1024, 8>(8),
        generic_variant<RegisterShare<16>, 1024, 4>(16),
        generic_variant<RegisterShare<32>, 1024, 4>(32),
        generic_variant<RegisterShare<64>, 512, 2>(64),
        generic_variant<RegisterShare<128>, 256, 1>(128),
        generic_variant<MemoryShare, 1024, 8>(0)};
    *count = (int)(sizeof(v) / sizeof(v[0]));
    return v;
}

// Teams of `threads` of the variant that can be resident at once on the
// current device.
static omprt_status coresident_teams(const GenericVariant& v, int threads, int* out) {
    int dev = 0;
    OMPRT_HIP(hipGetDevice(&dev));
    int coop = 0;
    OMPRT_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop) return fail(OMPRT_ERR_UNSUPPORTED, "device %d has no cooperative launch", dev);
    int per_cu = 0;
    OMPRT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, v.many, threads, 0));
    *out = per_cu * device_cus();
    return OMPRT_OK;
}

// The variant for n elements over teams x threads: the smallest that holds a
// thread's share in registers and keeps the teams resident, else the one that
// keeps them in memory (whose residency limits the team count: the registers
// are never why a launch is refused).
static omprt_status pick_variant(int64_t n, int teams, int threads, const GenericVariant** out) {
    int count = 0;
    const GenericVariant* v = generic_variants(&count);
    const int64_t share = ((n + teams - 1) / teams + threads - 1) / threads;
    for (int i = 0; i < count; ++i) {
        *out = &v[i];
        if (v[i].elems == 0) break;   // the last one takes every shape
        if (share > v[i].elems || threads > v[i].max_threads) continue;
        if (teams == 1) break;
        int resident = 0;
        if (omprt_status st = coresident_teams(v[i], threads, &resident)) return st;
        if (teams <= resident) break;
    }
    return OMPRT_OK;
}

}  // namespace omprt

using namespace omprt;

extern "C" omprt_status omprt_generic_power(const float* d_diag, float* d_v, int64_t n,
                                            int32_t iters, int32_t teams, int32_t threads,
                                            float* d_lambda, void* hip_stream) {
    if (n < 1 || n > ((int64_t)1 << 32))
        return fail(OMPRT_ERR_INVALID, "n = %lld outside 1..2^32", (long long)n);
    if (iters < 1) return fail(OMPRT_ERR_INVALID, "iters %d < 1", iters);
    if (teams < 0) return fail(OMPRT_ERR_INVALID, "teams %d < 0", teams);
    // default shape (measured at 2^10..2^24 elements, 100 steps, us a step): one
    // team of 512 threads while its loops are shorter than an all-gather (2^15:
    // 2.12 against 2.41 with 8 teams), else teams of 512 threads with 16
    // elements a thread up to half the CUs (2^16: 2.56 with 8 teams, 2.65 with
    // 64 of 256; 2^20: 3.15 with 128 teams, 3.33 with 256 of 256) and one a CU
    // past that (2^21: 3.47 against 3.67 with 128; 2^23: 4.47 against 17.0,
    // whose share no longer fits the registers), of 256 threads once the loops
    // stream (2^24: 30.8, 30.4 with 512)
    const bool auto_threads = threads == 0;
    const int64_t cus = device_cus();
    if (auto_threads) threads = teams > 1 || (teams == 0 && n > cus * 512 * 64) ? 256 : 512;
    if (threads < 64 || threads > 1024 || threads % 64)
        return fail(OMPRT_ERR_INVALID, "threads %d: 64..1024, a multiple of 64", threads);
    if (!d_diag || !d_v || !d_lambda) return fail(OMPRT_ERR_INVALID, "NULL pointer");
    if ((reinterpret_cast<uintptr_t>(d_diag) | reinterpret_cast<uintptr_t>(d_v) |
         reinterpret_cast<uintptr_t>(d_lambda)) % sizeof(float))
        return fail(OMPRT_ERR_INVALID, "pointer not aligned to 4 bytes");
    const uintptr_t db = reinterpret_cast<uintptr_t>(d_diag), vb = reinterpret_cast<uintptr_t>(d_v),
                    lb = reinterpret_cast<uintptr_t>(d_lambda), nb = (uintptr_t)n * sizeof(float);
    if (db < vb + nb && vb < db + nb) return fail(OMPRT_ERR_INVALID, "diag and v overlap");
    if ((lb >= vb && lb < vb + nb) || (lb >= db && lb < db + nb))
        return fail(OMPRT_ERR_INVALID, "lambda lies inside diag or v");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    int64_t want = teams;
    if (teams == 0) {
        if (auto_threads)
            want = n <= 32768 ? 1 : n / 8192 <= cus / 2 ? n / 8192 : cus;
        else
            want = n / ((int64_t)threads * 8);
    }
    if (want <= 1) {
        teams = 1;
    } else {
        int maxco = 0;
        int count = 0;
        const GenericVariant* memory = generic_variants(&count) + (count - 1);
        if (omprt_status st = coresident_teams(*memory, threads, &maxco)) return st;
        const int limit = std::min(maxco, kMaxGenericTeams);
        if (teams == 0)
            teams = (int)std::max<int64_t>(1, std::min<int64_t>(want, std::min<int64_t>(limit, cus)));
        else if (teams > limit)
            return fail(OMPRT_ERR_INVALID, "teams %d: at most %d teams of %d threads can be resident "
                        "at once here", teams, limit, threads);
    }
    const GenericVariant* var = nullptr;
    if (omprt_status st = pick_variant(n, teams, threads, &var)) return st;
    CrossTeam ct{};
    int it = iters;
    void* args[] = {&d_diag, &d_v, &n, &it, &d_lambda, &ct};
    hipError_t e;
    if (teams == 1) {
        e = hipLaunchKernel(var->one, dim3(1), dim3(threads), args, 0, stream);
    } else {
        Workspace* ws = nullptr;
        if (omprt_status st = workspace_get(stream, kGenericSlots * teams, &ws)) return st;
        const CrossTeamArgs ca = ws->cross();
        ct = CrossTeam{static_cast<uint64_t*>(ca.slots), ca.counter, ca.epoch, ca.status, ca.groups};
        e = hipLaunchCooperativeKernel(var->many, dim3(teams), dim3(threads), args, 0, stream);
    }
    if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "generic launch: %s", hipGetErrorString(e));
    return OMPRT_OK;
}
