// batched.hip -- many independent reductions in one persistent launch.
//
// A plan splits every segment into tiles of a fixed byte size (a segment
// shorter than one tile is one tile).  A grid of one device-wide wave of
// workgroups takes tiles either by an atomic ticket (the wrap-around
// increment again, with bound ntiles - 1, so the ticket returns to 0 when
// every workgroup, which starts with the tile of its own number, has drawn its
// final, out-of-range ticket) or round-robin.  Each tile is streamed and
// team-reduced exactly like a plain reduction's team block; a multi-tile segment's tile partials go to fixed
// slots and the segment's own wrap-increment counter (bound tiles - 1)
// elects the tile that finishes last to combine them in tile order and
// write x.  Slots are tagged with the launch epoch like the plain kernels'
// (device.h); a launch-wide wrap-increment elects the workgroup that ends
// last, which advances the epoch.  Results do not depend on which
// workgroup ran which tile.  A segment of a few KB is not worth a workgroup's
// barriers: one wave reduces it, and a tile is a bundle of as many as the
// workgroup has waves (4096 segments of 1000 elements: 127 -> 9.0 us).  A
// repeat call is one launch of the plan: counters, ticket and epoch maintain
// themselves, so it needs no memset, also when a caller's graph replays it.
#include <string.h>

#include <algorithm>
#include <map>
#include <memory>
#include <mutex>
#include <vector>

#include "device.h"
#include "launch.h"
#include "runtime.h"
#include "stream.h"

namespace omprt {

struct SegDesc {
    const void* in;
    void* x;
    int64_t n;
    int32_t dtype, op;
    int32_t first_tile, ntiles;
};

// Elements [lo, hi) of segment seg; or (seg < 0) entries [lo, hi) of the list
// of short segments, each reduced by one wave.
struct TileDesc {
    int64_t lo, hi;
    int32_t seg, pad;
};

// Device state of one plan: tagged slot per tile, election counter per
// segment, tile ticket, finished-workgroup counter, epoch and status words.
struct BatchState {
    uint64_t* slots;
    uint32_t* seg_counters;
    uint32_t* ticket;
    uint32_t* done;
    uint32_t* epoch;
    uint32_t* status;
    int32_t ntiles;
    int32_t done_groups;   // `done` counts in kElectGroups groups
};

// Reduce one tile, and combine its segment's if it is the last of them.
template <int DT, int OP, int VB, int U>
__device__ __forceinline__ void process_tile(const SegDesc& sd, const TileDesc& td, int tile,
                                             const BatchState& bs, uint32_t tag, void* lds_raw,
                                             int* s_last) {
    using R = Red<DT, OP>;
    using Acc = typename R::Acc;
    Acc acc[R::kNA];
#pragma unroll
    for (int i = 0; i < R::kNA; ++i) acc[i] = R::identity();
    stream_range<DT, OP, VB, U>(static_cast<const typename DType<DT>::S*>(sd.in), td.lo, td.hi,
                                acc);
    Acc t = fold_accs<R>(acc);
    Acc* lds = static_cast<Acc*>(lds_raw);
    t = team_reduce<R>(t, lds);
    typename R::Out* x = static_cast<typename R::Out*>(sd.x);
    if (sd.ntiles == 1) {
        if (threadIdx.x == 0) x[0] = R::finish(t, x[0]);
        return;
    }
    if (!publish_and_elect(t, bs.slots + (size_t)tile * kSlotWords, bs.seg_counters + td.seg,
                           (uint32_t)(sd.ntiles - 1), tag, s_last))
        return;
    const Acc c = combine_slots<R>(bs.slots + (size_t)sd.first_tile * kSlotWords, sd.ntiles, tag,
                                   bs.status, lds);
    if (threadIdx.x == 0) x[0] = R::finish(c, x[0]);
}

// Reduce a short segment by the calling wave alone.
template <int DT, int OP, int VB, int U>
__device__ __forceinline__ void wave_segment(const SegDesc& sd) {
    using R = Red<DT, OP>;
    typename R::Acc acc[R::kNA];
#pragma unroll
    for (int i = 0; i < R::kNA; ++i) acc[i] = R::identity();
    const int lane = threadIdx.x & (kWave - 1);
    stream_range_by<R, DT, VB, U>(static_cast<const typename DType<DT>::S*>(sd.in), 0, sd.n, acc,
                                  lane, kWave);
    const typename R::Acc t = wave_reduce<R>(fold_accs<R>(acc));
    typename R::Out* x = static_cast<typename R::Out*>(sd.x);
    if (lane == 0) x[0] = R::finish(t, x[0]);
}

#define OMPRT_CASES(F)                                                                      \
    F(DT_I32, OP_SUM) F(DT_I32, OP_MAX) F(DT_I32, OP_MIN)                                   \
    F(DT_I64, OP_SUM) F(DT_I64, OP_MAX) F(DT_I64, OP_MIN)                                   \
    F(DT_F32, OP_SUM) F(DT_F32, OP_MAX) F(DT_F32, OP_MIN)                                   \
    F(DT_F64, OP_SUM) F(DT_F64, OP_MAX) F(DT_F64, OP_MIN)                                   \
    F(DT_BF16, OP_SUM) F(DT_BF16, OP_MAX) F(DT_BF16, OP_MIN)

// A workgroup starts with the tile of its own number and draws a ticket for
// each further one, a tile ahead, so that the increment's round trip is over
// when the tile is.  Its one increment of `done` comes at its end: one address
// takes an increment every 13 ns, and with one per ticket and one per segment
// 4096 short segments took 127 us, whatever their length.
template <int VB, int U>
__global__ __launch_bounds__(1024) void batched_kernel(const SegDesc* __restrict__ segs,
                                                       const TileDesc* __restrict__ tiles,
                                                       const int32_t* __restrict__ shorts,
                                                       BatchState bs, int32_t use_ticket) {
    __shared__ Pair<double> lds[kMaxWaves];
    __shared__ int s_tile;
    __shared__ int s_last;
    const uint32_t epoch = read_epoch(bs.epoch);
    const uint32_t tag = launch_tag(epoch);
    int32_t tile = blockIdx.x;
    while (tile < bs.ntiles) {
        const int32_t grid = (int32_t)gridDim.x;
        int32_t next = tile + grid;
        if (use_ticket && threadIdx.x == 0)
            next = grid + (int32_t)__builtin_amdgcn_atomic_inc32(
                              bs.ticket, (uint32_t)(bs.ntiles - 1), __ATOMIC_RELAXED, "agent");
        const TileDesc td = tiles[tile];
        if (td.seg < 0) {   // short segments, one a wave
            const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
            for (int64_t i = td.lo + w; i < td.hi; i += team_size() / kWave) {
                const SegDesc sd = segs[shorts[i]];
                switch (sd.dtype * OP_COUNT + sd.op) {
#define OMPRT_CASE(DT, OP)                   \
    case DT * OP_COUNT + OP:                 \
        wave_segment<DT, OP, VB, U>(sd);     \
        break;
                    OMPRT_CASES(OMPRT_CASE)
#undef OMPRT_CASE
                    default: break;
                }
            }
        } else {
            const SegDesc sd = segs[td.seg];
            switch (sd.dtype * OP_COUNT + sd.op) {
#define OMPRT_CASE(DT, OP)                                                   \
    case DT * OP_COUNT + OP:                                                 \
        process_tile<DT, OP, VB, U>(sd, td, tile, bs, tag, lds, &s_last);    \
        break;
                OMPRT_CASES(OMPRT_CASE)
#undef OMPRT_CASE
                default: break;
            }
        }
        if (use_ticket) {
            if (threadIdx.x == 0) s_tile = next;
            __syncthreads();   // also: LDS from this tile is no longer read
            tile = s_tile;
            __syncthreads();
        } else {
            __syncthreads();
            tile = next;
        }
    }
    // the last workgroup to end advances the epoch (each read it at its start)
    if (threadIdx.x == 0) {
        const uint32_t e = gridDim.x - 1, g = blockIdx.x % kElectGroups;
        const bool last =
            bs.done_groups
                ? last_of(bs.done + (kElectGroupBytes / 4) * (g + 1), (e - g) / kElectGroups) &&
                      last_of(bs.done, kElectGroups - 1)
                : last_of(bs.done, e);
        if (last) advance_epoch(bs.epoch, epoch);
    }
}

using BatchedKernel = void (*)(const SegDesc*, const TileDesc*, const int32_t*, BatchState, int32_t);

static BatchedKernel batched_variant(int vec, int unroll) {
    if (vec == 16) {
        switch (unroll) {
            case 1: return batched_kernel<16, 1>;
            case 2: return batched_kernel<16, 2>;
            case 4: return batched_kernel<16, 4>;
            case 8: return batched_kernel<16, 8>;
        }
    } else if (vec == 8) {
        switch (unroll) {
            case 1: return batched_kernel<8, 1>;
            case 2: return batched_kernel<8, 2>;
            case 4: return batched_kernel<8, 4>;
            case 8: return batched_kernel<8, 8>;
        }
    }
    return nullptr;
}

// ---------------------------------------------------------------- plans

struct Plan {
    int device = 0, cus = 0;
    hipStream_t stream = nullptr;
    std::vector<omprt_segment> segs;
    omprt_config cfg{};
    void* dmem = nullptr;
    int32_t ntiles = 0;
    uint32_t* status = nullptr;
    // the launch
    BatchedKernel kernel = nullptr;
    const SegDesc* segs_dev = nullptr;
    const TileDesc* tiles_dev = nullptr;
    const int32_t* shorts_dev = nullptr;
    BatchState state{};
    int grid = 0;
    int32_t use_ticket = 0;
    // Explicit, never from a destructor: a plan still alive when the process
    // exits is left to the driver (no HIP call runs from static destruction).
    void release() {
        if (dmem) (void)hipFree(dmem);
        dmem = nullptr;
    }
};

static std::mutex g_bmu;
// one cached plan per (device, stream): a repeat call with the same segment
// list and configuration is one launch of it
static std::map<std::pair<int, hipStream_t>, std::unique_ptr<Plan>> g_plans;
// superseded plans: a graph the caller captured around an earlier call may
// still replay their launch, so they live until omprt_finalize
static std::vector<std::unique_ptr<Plan>> g_retired_plans;

// What plans are uploaded with, one per device, used under the lock and idle
// again when the call returns: a stream that holds nothing but the uploads, and
// pinned memory as large as the largest plan's tables so far.
struct Upload {
    hipStream_t stream = nullptr;
    void* host = nullptr;
    size_t cap = 0;
};
static std::map<int, Upload> g_uploads;

static omprt_status upload_get(int dev, size_t bytes, Upload** out) {
    Upload& u = g_uploads[dev];
    if (!u.stream) OMPRT_HIP(hipStreamCreateWithFlags(&u.stream, hipStreamNonBlocking));
    if (u.cap < bytes) {
        if (u.host) (void)hipHostFree(u.host);
        u.host = nullptr;
        u.cap = 0;
        const size_t cap = std::max<size_t>(bytes, (size_t)1 << 18);
        if (hipHostMalloc(&u.host, cap) != hipSuccess)
            return fail(OMPRT_ERR_NOMEM, "pinned allocation of %zu bytes failed", cap);
        u.cap = cap;
    }
    *out = &u;
    return OMPRT_OK;
}

static bool same_plan(const Plan& p, const omprt_segment* s, int32_t count,
                      const omprt_config& cfg) {
    if ((int32_t)p.segs.size() != count) return false;
    if (memcmp(&p.cfg, &cfg, sizeof cfg) != 0) return false;
    return memcmp(p.segs.data(), s, sizeof(omprt_segment) * (size_t)count) == 0;
}

static omprt_status check_segments(const omprt_segment* s, int32_t count) {
    for (int32_t i = 0; i < count; ++i) {
        const omprt_segment& g = s[i];
        if (g.dtype < 0 || g.dtype >= DT_COUNT_ABI || g.op < 0 || g.op > 2)
            return fail(OMPRT_ERR_UNSUPPORTED, "segment %d: dtype %d / op %d", i, g.dtype, g.op);
        if (g.n < 0 || g.n > ((int64_t)1 << 50))
            return fail(OMPRT_ERR_INVALID, "segment %d: n outside 0..2^50", i);
        if (!g.d_x) return fail(OMPRT_ERR_INVALID, "segment %d: x is NULL", i);
        if (g.n > 0 && !g.d_in) return fail(OMPRT_ERR_INVALID, "segment %d: input is NULL", i);
        if (reinterpret_cast<uintptr_t>(g.d_in) % (uintptr_t)dtype_bytes(g.dtype) ||
            reinterpret_cast<uintptr_t>(g.d_x) % (uintptr_t)out_bytes(g.dtype, g.op))
            return fail(OMPRT_ERR_INVALID, "segment %d: misaligned pointer", i);
    }
    return OMPRT_OK;
}

// Defaults of the batched launch: 1024 threads, 16-byte loads, unroll 4,
// 1 MiB tiles (build_plan), at most one workgroup per 1024 threads of device
// capacity (two a CU), ticket.  Over 4096 segments of 10^2..10^7 elements (16 GB) on
// gfx950: 2.34 ms, against 2.54 with 256 threads and 256 KiB tiles, 2.37
// with 1024 threads and 256 KiB, 2.33 with 4 MiB.
static void batched_defaults(const omprt_config* cfg, omprt_config* out, int cus) {
    omprt_config c{};
    if (cfg) c = *cfg;
    if (!c.threads_per_team) c.threads_per_team = 1024;
    if (!c.vec_bytes) c.vec_bytes = 16;
    if (!c.unroll) c.unroll = 4;
    if (!c.num_teams) c.num_teams = cus * (2048 / c.threads_per_team);
    c.flags &= OMPRT_CFG_STATIC_TILES;
    *out = c;
}

// Default tile sizes.
constexpr int64_t kMaxTileBytes = 1 << 20, kMinTileBytes = 64 << 10;

// Segments of up to kShortBytes are reduced by one wave each, in bundles of as
// many as a workgroup has waves; with at least eight a workgroup, up to
// kLongShortBytes (a wave alone needs more round trips, but its workgroup has
// fifteen others): 4096 segments of 4000 elements 65.4 -> 20.4 us.
constexpr int64_t kShortBytes = 8 << 10, kLongShortBytes = 32 << 10;

static omprt_status build_plan(Plan& p) {
    const int32_t count = (int32_t)p.segs.size();
    int64_t tile_bytes = (int64_t)p.cfg.tile_kib * 1024;
    if (!tile_bytes) {
        // 1 MiB, or less where that would be under two tiles a compute unit (or one
        // a workgroup, where the caller asks for fewer of them), but no segment of
        // more than 128 (its tiles meet on one counter).  us, 1 MiB -> now: 16
        // segments of 200000 elements 23.3 -> 10.6, 1000 of 10^2 to 10^5.5 52.9 ->
        // 38.1; one of 240 MB in 480 tiles 39.4 -> 48.3; 300 of 200000 elements
        // over 64 workgroups 58 -> 50 (87 with tiles for every compute unit).
        int64_t total = 0, longest = 0;
        for (const omprt_segment& g : p.segs) {
            const int64_t bytes = std::min<int64_t>(g.n, (int64_t)1 << 40) * dtype_bytes(g.dtype);
            total += bytes;
            longest = std::max(longest, bytes);
        }
        tile_bytes = kMaxTileBytes;
        const int64_t want = p.cfg.num_teams < p.cus ? p.cfg.num_teams : 2 * p.cus;
        while (tile_bytes > kMinTileBytes && total / tile_bytes < want &&
               longest / (tile_bytes / 2) <= 128)
            tile_bytes /= 2;
    }
    std::vector<SegDesc> sd((size_t)count);
    std::vector<TileDesc> td;
    std::vector<uint64_t> keys;   // of the short ones: type, operator, falling length, index
    int64_t under_long = 0;
    for (const omprt_segment& g : p.segs) under_long += g.n * dtype_bytes(g.dtype) <= kLongShortBytes;
    const int64_t short_bytes =
        under_long >= 8 * (int64_t)p.cfg.num_teams ? kLongShortBytes : kShortBytes;
    for (int32_t i = 0; i < count; ++i) {
        const omprt_segment& g = p.segs[i];
        const int eb = dtype_bytes(g.dtype);
        if (g.n > 0 && g.n * eb <= short_bytes) {
            sd[i] = SegDesc{g.d_in, g.d_x, g.n, g.dtype, g.op, 0, 1};
            keys.push_back((uint64_t)(g.dtype * 16 + g.op) << 56 |
                           (uint64_t)(kLongShortBytes - g.n) << 32 | (uint32_t)i);
            continue;
        }
        const int64_t te = std::max<int64_t>(tile_bytes / eb, 1);
        const int64_t nt = g.n == 0 ? 0 : (g.n - 1) / te + 1;
        if ((int64_t)td.size() + nt > INT32_MAX / 2)
            return fail(OMPRT_ERR_INVALID, "batched plan: too many tiles (raise tile_kib)");
        sd[i] = SegDesc{g.d_in, g.d_x, g.n, g.dtype, g.op, (int32_t)td.size(), (int32_t)nt};
        for (int64_t t = 0; t < nt; ++t)
            td.push_back(TileDesc{t * te, std::min(g.n, (t + 1) * te), i, 0});
    }
    // the short ones last, by type and operator (a workgroup's waves then run the
    // same code) and by size (and end together), a segment for each wave
    std::sort(keys.begin(), keys.end());
    const int64_t nshort = (int64_t)keys.size(), each = p.cfg.threads_per_team / kWave;
    for (int64_t j = 0; j < nshort; j += each)
        td.push_back(TileDesc{j, std::min(nshort, j + each), -1, 0});
    p.ntiles = (int32_t)td.size();
    const size_t seg_b = (sizeof(SegDesc) * (size_t)count + 255) / 256 * 256;
    const size_t tile_b = (sizeof(TileDesc) * td.size() + 255) / 256 * 256;
    const size_t slot_b = ((size_t)kSlotBytes * td.size() + 255) / 256 * 256;
    const size_t ctr_b = ((size_t)(count + 4) * 4 + 255) / 256 * 256;
    constexpr size_t done_b = (size_t)kElectGroupBytes * (1 + kElectGroups);
    const size_t short_b = (keys.size() * sizeof(int32_t) + 255) / 256 * 256;
    const size_t tables_b = seg_b + tile_b + short_b;
    if (hipMalloc(&p.dmem, tables_b + slot_b + ctr_b + done_b) != hipSuccess)
        return fail(OMPRT_ERR_NOMEM, "batched plan allocation failed");
    char* base = static_cast<char*>(p.dmem);
    SegDesc* d_seg = reinterpret_cast<SegDesc*>(base);
    TileDesc* d_tile = reinterpret_cast<TileDesc*>(base + seg_b);
    int32_t* d_short = reinterpret_cast<int32_t*>(base + seg_b + tile_b);
    uint32_t* d_ctr = reinterpret_cast<uint32_t*>(base + tables_b + slot_b);
    BatchState bs{reinterpret_cast<uint64_t*>(base + tables_b), d_ctr, d_ctr + count,
                  reinterpret_cast<uint32_t*>(base + tables_b + slot_b + ctr_b),
                  d_ctr + count + 1, d_ctr + count + 2, p.ntiles, 0};
    // The tables in one copy, then zero slots (odd tags never match 0) and zero
    // counters.  The memory is new, so nothing on the caller's stream has to come
    // first, and a stream that holds only this is waited for: the plan is whole
    // when the call returns, whichever stream a graph of its launch is replayed
    // on, and the host waits for no stream's earlier work.  A new list of 2719
    // segments a call takes 99 us, of 94 segments 28; with copies from pageable
    // memory 154 and 33, and waiting for the caller's stream instead 215 and 105.
    Upload* u = nullptr;
    if (omprt_status e = upload_get(p.device, tables_b, &u)) return e;
    char* up = static_cast<char*>(u->host);
    memcpy(up, sd.data(), sizeof(SegDesc) * sd.size());
    if (!td.empty()) memcpy(up + seg_b, td.data(), sizeof(TileDesc) * td.size());
    int32_t* up_short = reinterpret_cast<int32_t*>(up + seg_b + tile_b);
    for (int64_t j = 0; j < nshort; ++j) up_short[j] = (int32_t)(uint32_t)keys[j];
    OMPRT_HIP(hipMemcpyAsync(base, up, tables_b, hipMemcpyHostToDevice, u->stream));
    OMPRT_HIP(hipMemsetAsync(base + tables_b, 0, slot_b + ctr_b + done_b, u->stream));
    OMPRT_HIP(hipStreamSynchronize(u->stream));
    p.status = bs.status;

    p.segs_dev = d_seg;
    p.tiles_dev = d_tile;
    p.shorts_dev = d_short;
    p.state = bs;
    p.kernel = batched_variant(p.cfg.vec_bytes, p.cfg.unroll);
    if (!p.kernel) return fail(OMPRT_ERR_INVALID, "no batched kernel for vec %d unroll %d",
                        p.cfg.vec_bytes, p.cfg.unroll);
    // Tickets: no more workgroups than run at once (a later one would hold the
    // tile of its own number back until an earlier one has run out of tiles:
    // 1000 segments of 1000 elements in 500 workgroups 29 us, in 250 8.8).
    p.use_ticket = (p.cfg.flags & OMPRT_CFG_STATIC_TILES) ? 0 : 1;
    int teams = p.cfg.num_teams, fit = 0;
    if (p.use_ticket) {
        OMPRT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &fit, reinterpret_cast<const void*>(p.kernel), p.cfg.threads_per_team, 0));
        if (fit > 0) teams = std::min(teams, fit * p.cus);
    }
    p.grid = std::max(1, std::min<int>(teams, std::max<int32_t>(p.ntiles, 1)));
    if (p.ntiles <= p.grid) p.use_ticket = 0;   // a tile each: nothing to draw
    p.state.done_groups = p.grid >= 128;
    return OMPRT_OK;
}

void batched_finalize() {
    std::lock_guard<std::mutex> lk(g_bmu);
    for (auto& kv : g_plans)
        if (kv.second) {
            (void)hipSetDevice(kv.second->device);
            kv.second->release();
        }
    for (auto& p : g_retired_plans) {
        (void)hipSetDevice(p->device);
        p->release();
    }
    g_plans.clear();
    g_retired_plans.clear();
    for (auto& kv : g_uploads) {
        (void)hipSetDevice(kv.first);
        if (kv.second.host) (void)hipHostFree(kv.second.host);
        if (kv.second.stream) (void)hipStreamDestroy(kv.second.stream);
    }
    g_uploads.clear();
}

}  // namespace omprt

using namespace omprt;

extern "C" omprt_status omprt_reduce_batched(const omprt_segment* h_segs, int32_t count,
                                             const omprt_config* cfg, void* hip_stream) {
    if (count < 0) return fail(OMPRT_ERR_INVALID, "count < 0");
    if (count > 0 && !h_segs) return fail(OMPRT_ERR_INVALID, "segments pointer is NULL");
    if (count == 0) return OMPRT_OK;
    auto check = [&]() -> omprt_status {
        if (omprt_status st = check_segments(h_segs, count)) return st;
        LaunchCfg dummy;   // field validation only
        return resolve_config(1, OMPRT_F32, OMPRT_SUM, 0, -1, cfg, &dummy, nullptr);
    };
    int dev = 0;
    const hipError_t de = hipGetDevice(&dev);
    if (de != hipSuccess) {   // argument errors come first
        if (omprt_status st = check()) return st;
        OMPRT_HIP(de);
    }
    const int cus = device_cus();
    omprt_config c;
    batched_defaults(cfg, &c, cus);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    std::lock_guard<std::mutex> lk(g_bmu);
    std::unique_ptr<Plan>& slot = g_plans[{dev, stream}];
    if (!slot || !same_plan(*slot, h_segs, count, c)) {
        // (a list and configuration equal to the plan's passed)
        if (omprt_status st = check()) return st;
        hipStreamCaptureStatus cst = hipStreamCaptureStatusNone;
        OMPRT_HIP(hipStreamIsCapturing(stream, &cst));
        if (cst != hipStreamCaptureStatusNone)
            return fail(OMPRT_ERR_INVALID, "omprt_reduce_batched builds its plan outside capture");
        if (slot) g_retired_plans.push_back(std::move(slot));   // replays may still run
        std::unique_ptr<Plan> p(new Plan());
        p->device = dev;
        p->cus = cus;
        p->stream = stream;
        p->segs.assign(h_segs, h_segs + count);
        p->cfg = c;
        if (omprt_status st = build_plan(*p)) {
            p->release();
            return st;
        }
        slot = std::move(p);
    }
    if (slot->ntiles == 0) return OMPRT_OK;
    // The launch itself, not a graph of it: replaying a captured one-node graph
    // took 16 us of host time against 2.5, and 4096 segments of 10^2 to 10^7 2498
    // us against 2468.  A caller's own graph may hold it.
    hipLaunchKernelGGL(slot->kernel, dim3(slot->grid), dim3(slot->cfg.threads_per_team), 0, stream,
                       slot->segs_dev, slot->tiles_dev, slot->shorts_dev, slot->state,
                       slot->use_ticket);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "batched launch: %s", hipGetErrorString(e));
    return OMPRT_OK;
}

extern "C" omprt_status omprt_reduce_each(const omprt_segment* h_segs, int32_t count,
                                          const omprt_config* cfg, void* hip_stream) {
    if (count < 0) return fail(OMPRT_ERR_INVALID, "count < 0");
    if (count > 0 && !h_segs) return fail(OMPRT_ERR_INVALID, "segments pointer is NULL");
    if (omprt_status st = check_segments(h_segs, count)) return st;
    for (int32_t i = 0; i < count; ++i) {
        const omprt_segment& g = h_segs[i];
        if (omprt_status st = omprt_reduce(g.d_in, g.n, g.dtype, g.op, g.d_x, cfg, hip_stream))
            return st;
    }
    return OMPRT_OK;
}

namespace omprt {
// Status word of the stream's cached batched plan (nullptr if none).
uint32_t* batched_status_word(int dev, hipStream_t stream) {
    std::lock_guard<std::mutex> lk(g_bmu);
    auto it = g_plans.find({dev, stream});
    return (it == g_plans.end() || !it->second) ? nullptr : it->second->status;
}
}  // namespace omprt
