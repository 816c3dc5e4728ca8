// array.hip -- array-section reduction, reduction(op: x[0:m]): every list
// item x[j] is a reduction variable of its own; iteration i of the loop
// contributes in[i*m + j] to x[j].
//
// Geometry.  The row-major block is cut into column tiles of W columns
// (W = m, whole rows, when m is small) and each tile into periods of R rows,
// with R * W <= L = threads * E * U elements (E per load, U loads in flight
// per lane).  Within a period, the element at flat offset o (row o / w, column
// o % w of the tile, w its width) belongs to lane slot (u, k) with
// o = (u * P + t) * E + k, so every lane slot keeps a private copy of one list
// item for the whole launch.  Team (c, r) takes tile c and the balanced block
// of its periods; the last row team of a tile also folds the rows left over
// after the whole periods.
//
// Combination.  The private copies go to LDS as an R x w matrix whose rows
// are folded pairwise (R -> ceil(R/2) -> ... -> 1).  With one row team per
// tile the team writes x directly.  Otherwise each team publishes its w
// partials as tagged slot words; the row teams of a tile form election
// groups, sized so that the last team of a group folds the group's rows
// with at most 16 partials per thread, and the wrap-around increment elects
// that last team.  With one group it writes x; otherwise the group results
// are published and the last group of the tile folds them and writes x.
// The last tile to finish advances the launch epoch.
#include <algorithm>
#include <map>
#include <mutex>

#include "array_kernel.h"
#include "runtime.h"

namespace omprt {

static ArrayLauncher array_launcher(int dtype, int op, int loads, int u) {
    switch (dtype) {
        case DT_I32: return array_launcher_i32(op, loads, u);
        case DT_I64: return array_launcher_i64(op, loads, u);
        case DT_F32: return array_launcher_f32(op, loads, u);
        case DT_F64: return array_launcher_f64(op, loads, u);
        case DT_BF16: return array_launcher_bf16(op, loads, u);
    }
    return nullptr;
}

// Bytes of one private copy (the accumulator) per (dtype, op).
static int acc_bytes(int dtype, int op) {
    if (op == OP_LAND || op == OP_LOR) return 4;   // a 0/1 flag
    const bool pair = op == OP_SUM || op == OP_PROD;   // compensated (hi, lo)
    switch (dtype) {
        case DT_I32: return 4;
        case DT_I64: return 8;
        case DT_F32: return pair ? 8 : 4;
        case DT_F64: return pair ? 16 : 8;
        case DT_BF16: return pair ? 8 : 4;
    }
    return 16;
}

// ---------------------------------------------------------------- workspace

// Per (device, stream): a 256-byte header (done counter, epoch, status),
// the election counters (0 between launches) and the tagged slots; zeroed
// once at allocation, grown on demand (never while the stream is captured).
struct ArrayWs {
    void* base = nullptr;
    int64_t counters = 0;   // capacity, words
    int64_t words = 0;      // capacity, 64-bit slot words
    uint32_t* done() const { return static_cast<uint32_t*>(base); }
    uint32_t* epoch() const { return static_cast<uint32_t*>(base) + 16; }
    uint32_t* status() const { return static_cast<uint32_t*>(base) + 32; }
    uint32_t* ctrs() const { return reinterpret_cast<uint32_t*>(static_cast<char*>(base) + 256); }
    uint64_t* slots() const {
        return reinterpret_cast<uint64_t*>(static_cast<char*>(base) + 256 + ctr_bytes(counters));
    }
    static size_t ctr_bytes(int64_t n) { return ((size_t)n * 4 + 255) / 256 * 256; }
};
static std::mutex g_amu;
static std::map<std::pair<int, hipStream_t>, ArrayWs> g_aws;

// The stream's workspace for `counters` and `words`; with room for `room` words
// unless the stream is being captured.
static omprt_status array_ws_get(hipStream_t stream, int64_t counters, int64_t words, int64_t room,
                                 ArrayWs* out) {
    int dev = 0;
    OMPRT_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_amu);
    ArrayWs& ws = g_aws[{dev, stream}];
    const bool too_small = !ws.base || ws.counters < counters || ws.words < words;
    if (too_small || ws.words < room) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        OMPRT_HIP(hipStreamIsCapturing(stream, &cs));
        if (cs != hipStreamCaptureStatusNone) {
            if (too_small)
                return fail(OMPRT_ERR_INVALID,
                            "stream is being captured and its array-reduction workspace is too "
                            "small: make the same call once before capturing");
            *out = ws;
            return OMPRT_OK;
        }
        const int64_t nc = std::max<int64_t>({counters, ws.counters, 1024});
        const int64_t nw = std::max<int64_t>({words, room, ws.words, (int64_t)1 << 16});
        const size_t bytes = 256 + ArrayWs::ctr_bytes(nc) + (size_t)nw * 8;
        void* p = nullptr;
        if (hipMalloc(&p, bytes) != hipSuccess)
            return fail(OMPRT_ERR_NOMEM, "array workspace allocation of %zu bytes failed", bytes);
        retire_device_memory(dev, ws.base);   // a captured graph may still name it
        ws.base = p;
        ws.counters = nc;
        ws.words = nw;
        OMPRT_HIP(hipMemsetAsync(p, 0, bytes, stream));   // tags are odd: zero never matches
    }
    *out = ws;
    return OMPRT_OK;
}

void array_finalize() {
    std::lock_guard<std::mutex> lk(g_amu);
    for (auto& kv : g_aws) {
        if (!kv.second.base) continue;
        (void)hipSetDevice(kv.first.first);
        (void)hipFree(kv.second.base);
    }
    g_aws.clear();
}

uint32_t* array_status_word(int dev, hipStream_t stream) {
    std::lock_guard<std::mutex> lk(g_amu);
    auto it = g_aws.find({dev, stream});
    return (it == g_aws.end() || !it->second.base) ? nullptr : it->second.status();
}

omprt_status array_reset(int dev, hipStream_t stream) {
    std::lock_guard<std::mutex> lk(g_amu);
    auto it = g_aws.find({dev, stream});
    if (it == g_aws.end() || !it->second.base) return OMPRT_OK;
    const ArrayWs& ws = it->second;
    OMPRT_HIP(hipMemsetAsync(ws.done(), 0, 4, stream));
    OMPRT_HIP(hipMemsetAsync(ws.status(), 0, 4, stream));
    OMPRT_HIP(hipMemsetAsync(ws.ctrs(), 0, (size_t)ws.counters * 4, stream));
    return OMPRT_OK;
}

// ---------------------------------------------------------------- planning

constexpr int64_t kTileCols = 256;      // target tile width when rows are wider
constexpr int64_t kFoldItems = 16;     // partials one thread folds per election level
constexpr int kMaxLdsBytes = 64 * 1024 - 256;   // dynamic LDS; the rest is static

static int64_t gcd64(int64_t a, int64_t b) {
    while (b) { const int64_t t = a % b; a = b; b = t; }
    return a;
}

// Column tiles of rows wider than wmax: as few as hold them, or, for blocks
// that fill the chip, a power of two of at least sqrt(m / 32) tiles.  With one
// team a compute unit over them (256 / tiles a tile) one group of teams then
// folds a tile in one level, and a row team's tiles go to one XCD evenly.  us,
// fewest tiles -> this: 65536 x 1001 fp32 47.4 -> 43.6, fp64 94.7 -> 87.7;
// 16000 x 1001 23.2 -> 19.4; 196000 x 333 47.6 -> 44.2; 80000 x 100 20.1 ->
// 15.3; 256000 x 256 fp64 93.9 -> 85.0.  Not for blocks under 16 MiB, whose teams
// have few periods each and wait for the combination (1000 x 1001 10.4 ->
// 11.8), nor past 32 tiles, where the fewest already leave eight teams or fewer
// a tile (3276 x 19999 46.4 -> 48.2).  Past the last-level cache (from 128 MiB)
// 8-byte elements, whose loads bypass it, read the lines that tiles share from
// memory twice: there tiles are wider than four lines (1008246 x 65 fp64, two
// tiles of 264 bytes, 92 -> 112; inside the cache 101265 x 79 28.6 -> 23.1).
static int64_t tile_count(int64_t rows, int64_t m, int64_t wmax, int esize) {
    const int64_t least = (m + wmax - 1) / wmax;
    const int64_t bytes = rows * m * esize;
    if (m <= 64 || least > 32 || bytes < ((int64_t)16 << 20)) return least;
    int64_t t = 1;
    while (t < least || t * t * 32 < m) t *= 2;
    while (esize == 8 && bytes > ((int64_t)128 << 20) && t > least && m * esize <= t * 4 * 128) t /= 2;
    return std::max(t, least);
}

// The most columns of a tile, for L elements a period and E per load.
static int64_t max_tile_width(int E, int64_t L) {
    return std::min<int64_t>(kTileCols, L) / E * E;
}

// Geometry for E elements per load over `tiles` column tiles (of up to
// max_tile_width columns); false if it cannot stream in vectors.
static bool array_geometry(int64_t rows, int64_t m, int E, int64_t L, int64_t tiles,
                           ArrayGeom* g) {
    g->rows = rows;
    g->m = m;
    if (tiles == 1) {   // whole rows; a period's first element must stay 16-byte aligned
        const int64_t step = E / gcd64(m, E);
        g->W = m;
        g->R = (L / m) / step * step;
        g->col_tiles = 1;
        if (g->R < 1) return false;
    } else {           // balanced column tiles; every row start must be aligned
        if (m % E != 0) return false;
        g->W = ((m + tiles - 1) / tiles + E - 1) / E * E;
        g->R = L / g->W;
        const int64_t used = (m + g->W - 1) / g->W;
        if (used > INT32_MAX) return false;
        g->col_tiles = (int32_t)used;
    }
    g->np = rows / g->R;
    return true;
}

// LDS entries a team needs for its private copies: the span of a period,
// or one layer of P * E offsets when the kernel folds the U slots of a lane
// in registers (every slot live, whole rows per layer).  Maximum over the
// full tiles and the last one.
static int64_t lds_entries(const ArrayGeom& g, int64_t layer, int U) {
    const int64_t wl = g.m - (int64_t)(g.col_tiles - 1) * g.W;
    int64_t need = 0;
    for (int64_t wc : {std::min(g.W, g.m), wl}) {
        const int64_t span = g.R * wc;
        const bool fold = U > 1 && span == U * layer && layer % wc == 0;
        need = std::max(need, fold ? layer : span);
    }
    return need;
}

// Geometry for ragged loads of E elements (array_kernel.h): the element loads'
// tiles, a period of U layers of RL rows, one vector a lane and layer.
static bool ragged_geometry(int64_t rows, int64_t m, int E, int P, int U, int ab, ArrayGeom* g) {
    g->rows = rows;
    g->m = m;
    const int64_t wmax = std::min<int64_t>(kTileCols, (int64_t)P * E);
    const int64_t tiles = tile_count(rows, m, wmax, 16 / E);
    g->W = (m + tiles - 1) / tiles;
    if (tiles > INT32_MAX) return false;
    g->col_tiles = (int32_t)((m + g->W - 1) / g->W);
    const int64_t wl = m - (g->col_tiles - 1) * g->W;   // the last tile's width
    if (tiles > 1 && wl < E) return false;
    g->RL = (int32_t)(g->col_tiles == 1 ? (int64_t)P * E / m : P / ((g->W + E - 1) / E));
    g->RL = (int32_t)std::min<int64_t>(g->RL, kMaxLdsBytes / (ab * g->W * U));
    if (g->RL < 1 || g->RL * g->W < E) return false;
    g->R = (int64_t)U * g->RL;
    g->np = rows / g->R;
    return true;
}

struct ArrayPlan {
    ArrayGeom g;
    int loads;   // ArrayLoads
    int threads, unroll;
    size_t lds;
    // The most row teams that the runtime gives a block of this many columns,
    // whatever its rows (0: the caller gave the team count).  Workspaces have room
    // for them: its choice does not grow with the rows, and a call made once has to
    // cover captures of smaller blocks.
    int64_t most;
};

static omprt_status plan_array(int64_t rows, int64_t m, int dtype, int op, const void* in,
                               const omprt_config* cfg, ArrayPlan* out) {
    const int esize = dtype_bytes(dtype);
    const int ab = acc_bytes(dtype, op);
    int P = 512, U = 4, want_teams = 0;
    bool allow_vec = true;
    if (cfg) {
        if (cfg->threads_per_team) {
            if (cfg->threads_per_team < 64 || cfg->threads_per_team > 512 ||
                cfg->threads_per_team % 64)
                return fail(OMPRT_ERR_INVALID, "threads_per_team %d", cfg->threads_per_team);
            P = cfg->threads_per_team;
        }
        if (cfg->unroll) {
            if (cfg->unroll != 1 && cfg->unroll != 2 && cfg->unroll != 4 && cfg->unroll != 8)
                return fail(OMPRT_ERR_INVALID, "unroll %d", cfg->unroll);
            U = cfg->unroll;
        }
        if (cfg->vec_bytes) {
            if (cfg->vec_bytes == esize) allow_vec = false;
            else if (cfg->vec_bytes != 16)
                return fail(OMPRT_ERR_INVALID, "vec_bytes %d (0, 16 or the element size)",
                            cfg->vec_bytes);
        }
        if (cfg->num_teams) {
            if (cfg->num_teams < 1 || cfg->num_teams > 65535)
                return fail(OMPRT_ERR_INVALID, "num_teams %d", cfg->num_teams);
            want_teams = cfg->num_teams;
        }
    }
    const bool explicit_u = cfg && cfg->unroll;
    ArrayPlan pl{};
    pl.threads = P;
    bool found = false;
    // 16-byte loads first, then ragged, then element loads; the default unroll
    // is lowered until the private copies fit LDS, an explicit one is kept or
    // dropped.
    for (int pass = allow_vec ? 0 : 1; pass < 2 && !found; ++pass) {
        const bool vec = pass == 0;
        if (!vec && allow_vec && !explicit_u) {
            const int E = 16 / esize;
            for (int u = 2; u >= 1 && !found; u /= 2) {
                ArrayGeom g{};
                if (!ragged_geometry(rows, m, E, P, u, ab, &g)) continue;
                if (u > 1 && g.np < device_cus() / g.col_tiles) continue;
                pl.g = g;
                pl.loads = kRagged;
                pl.unroll = u;
                pl.lds = (size_t)std::max<int64_t>(g.RL * g.W, P) * ab;
                found = true;
            }
            if (found) break;
        }
        if (vec && (reinterpret_cast<uintptr_t>(in) & 15)) continue;
        const int E = vec ? 16 / esize : 1;
        // element loads: 8 in flight; vectors of column tiles of fp32 pairs, two
        // and two of the next period (65536 x 1000 55.6 -> 53.2 us; bf16 36.4 ->
        // 36.9)
        const bool tiled = m > std::min<int64_t>(kTileCols, (int64_t)P * E * 4);
        const int u0 = explicit_u                                       ? (vec ? std::min(U, 4) : U)
                       : !vec                                           ? 8
                       : tiled && dtype == DT_F32 && ab == 8            ? 2
                                                                        : 4;
        for (int u = u0; u >= 1 && !found; u /= 2) {
            ArrayGeom g{};
            // A given unroll keeps the fewest tiles: it is not lowered until a
            // tile's copies fit, and whole rows of any width stream in vectors
            // where tiles of them would not.  So do element loads, for which more
            // tiles were not measured.
            const int64_t L = (int64_t)P * E * u, wmax = max_tile_width(E, L);
            const int64_t tiles = vec && !explicit_u ? tile_count(rows, m, wmax, esize)
                                                     : (m + wmax - 1) / wmax;
            if (array_geometry(rows, m, E, L, tiles, &g)) {
                // tiles that are not whole lines share them with their neighbours:
                // ragged loads keep the lines in the caches
                if (vec && !explicit_u && g.col_tiles > 1 && (g.W * esize % 128 || m * esize % 128))
                    break;
                // the group fold also needs one entry per thread
                const size_t bytes =
                    (size_t)std::max<int64_t>(lds_entries(g, (int64_t)P * E, u), P) * ab;
                if (bytes <= (size_t)kMaxLdsBytes) {
                    pl.g = g;
                    pl.loads = vec ? kVectors : kElements;
                    pl.unroll = u;
                    pl.lds = bytes;
                    found = true;
                }
            }
            if (explicit_u) break;
        }
    }
    if (!found)
        return fail(OMPRT_ERR_INVALID,
                    "no launch geometry: the private copies of threads %d x unroll %d do not "
                    "fit %d bytes of LDS", P, U, kMaxLdsBytes);
    ArrayGeom& g = pl.g;
    // at most one team per compute unit with vectors, two with element loads
    // (which keep a quarter of the bytes in flight per lane or less)
    const bool choose = !want_teams;
    if (choose) want_teams = device_cus() * (pl.loads == kElements ? 2 : 1);
    int64_t rt = std::max<int64_t>(1, want_teams / g.col_tiles);
    rt = std::min<int64_t>(rt, std::max<int64_t>(1, g.np));
    pl.most = choose ? std::max<int64_t>(1, want_teams / ((m + kTileCols - 1) / kTileCols)) : 0;
    // Election groups: as many teams as the last one can fold with at most
    // kFoldItems partials per thread (fold_group); one group when all fit.
    const int64_t wc_max = std::min(g.W, m);
    const int64_t per_col = wc_max * 2 > P ? 1 : P / wc_max;   // threads per column
    const int64_t rounds = (wc_max + P - 1) / P;               // columns per thread
    const int64_t gs_max = std::max<int64_t>(2, kFoldItems * per_col / rounds);
    if (choose && rt > 1) {
        // Fewer row teams make the combination shorter and the streams longer.
        // Estimated us (fitted on gfx950 over 10^3 to 10^8 elements, 4 to 256
        // teams a tile): a period's latency and its bytes, twice that from 64 MiB
        // on; a level of groups its teams' serial increments, its
        // batches of slot loads and the partials a thread folds in a row.
        const int nw = ab / 4;
        const bool pairs = dtype != DT_I32 && dtype != DT_I64 && (op == OP_SUM || op == OP_PROD);
        const double part = !pairs ? 0.05 : nw == 2 ? 0.2 : 0.4;
        const int64_t batch = nw <= 2 ? 16 : 8;   // fold_tagged
        auto level = [&](int64_t teams) {
            const int64_t parts = (teams + per_col - 1) / per_col * rounds;
            return 0.018 * teams + 1.5 * ((parts + batch - 1) / batch) + part * parts;
        };
        const double kib = (double)g.R * wc_max * esize / 1024.0;
        const double period = (0.1 + 0.25 / 16 * kib) *
                              (rows * m * esize > ((int64_t)64 << 20) ? 2.0 : 1.0);
        auto cost = [&](int64_t r) {
            const int64_t gs = std::min(r, gs_max), ng = (r + gs - 1) / gs;
            return period * ((g.np + r - 1) / r) + (r > 1 ? level(gs) : 0.0) +
                   (ng > 1 ? 2.5 + level(ng) : 0.0);
        };
        int64_t best = rt;
        double least = cost(rt) - 1.0;   // the estimate's own error
        auto consider = [&](int64_t r) {
            if (r < 1 || r > rt) return;
            const double c = cost(r);
            if (c < least) {
                least = c;
                best = r;
            }
        };
        consider(gs_max);
        consider(per_col * batch / rounds);   // one batch
        // by whole numbers of periods a team
        for (int64_t k = (g.np + rt - 1) / rt; k <= g.np; k += std::max<int64_t>(1, k / 4))
            consider((g.np + k - 1) / k);
        rt = best;
    }
    g.rt = (int32_t)rt;
    g.gs = (int32_t)std::min(rt, gs_max);
    g.ng = (int32_t)((rt + g.gs - 1) / g.gs);
    *out = pl;
    return OMPRT_OK;
}

}  // namespace omprt

using namespace omprt;

extern "C" omprt_status omprt_reduce_array(const void* d_in, int64_t rows, int64_t m,
                                           int32_t dtype, int32_t op, void* d_x,
                                           const omprt_config* cfg, void* hip_stream) {
    if (dtype < 0 || dtype >= DT_COUNT_ABI) return fail(OMPRT_ERR_UNSUPPORTED, "dtype %d", dtype);
    if (!op_defined(dtype, op)) return fail(OMPRT_ERR_UNSUPPORTED, "op %d on dtype %d", op, dtype);
    if (rows < 0 || m < 0) return fail(OMPRT_ERR_INVALID, "rows/m negative");
    if (m > 0 && rows > ((int64_t)1 << 50) / m)
        return fail(OMPRT_ERR_INVALID, "rows * m above 2^50");
    if (m > ((int64_t)1 << 40)) return fail(OMPRT_ERR_INVALID, "m above 2^40");
    if (rows == 0 || m == 0) return OMPRT_OK;
    if (!d_in || !d_x) return fail(OMPRT_ERR_INVALID, "in/x is NULL");
    const int esize = dtype_bytes(dtype), xsize = out_bytes(dtype, op);
    if (reinterpret_cast<uintptr_t>(d_in) % esize)
        return fail(OMPRT_ERR_INVALID, "in is not aligned to its element size");
    if (reinterpret_cast<uintptr_t>(d_x) % xsize)
        return fail(OMPRT_ERR_INVALID, "x is not aligned to its element size");
    {
        const char* ib = static_cast<const char*>(d_in);
        const char* xb = static_cast<const char*>(d_x);
        if (xb < ib + rows * m * esize && ib < xb + m * xsize)
            return fail(OMPRT_ERR_INVALID, "x overlaps in");
    }
    ArrayPlan pl;
    if (omprt_status st = plan_array(rows, m, dtype, op, d_in, cfg, &pl)) return st;
    const ArrayGeom& g = pl.g;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    ArrayCross ct{};
    const int nw = acc_bytes(dtype, op) / 4;
    // (groups have at least two teams)
    const int64_t room = pl.most > 1 ? (pl.most + (pl.most + 1) / 2) * m * nw : 0;
    if (g.rt > 1) {
        const int64_t counters = (int64_t)g.col_tiles * g.ng + (g.ng > 1 ? g.col_tiles : 0);
        const int64_t words = ((int64_t)g.rt + (g.ng > 1 ? g.ng : 0)) * m * nw;
        ArrayWs ws;
        if (omprt_status st = array_ws_get(stream, counters, words, room, &ws)) return st;
        ct = ArrayCross{ws.slots(), ws.slots() + (int64_t)g.rt * m * nw, ws.ctrs(), ws.done(),
                        ws.epoch(), ws.status()};
    } else if (room) {
        // a smaller block may take several teams where the estimate gives this one
        // a single one: leave the workspace (this call itself needs none)
        ArrayWs ws;
        if (array_ws_get(stream, 0, 0, room, &ws) != OMPRT_OK) (void)hipGetLastError();
    }
    const ArrayLauncher f = array_launcher(dtype, op, pl.loads, pl.unroll);
    if (!f) return fail(OMPRT_ERR_UNSUPPORTED, "no array kernel for this combination");
    if ((int64_t)g.col_tiles * g.rt > INT32_MAX) return fail(OMPRT_ERR_INVALID, "grid too large");
    f(d_in, d_x, g, ct, pl.threads, pl.lds, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(OMPRT_ERR_DEVICE, "array launch: %s", hipGetErrorString(e));
    return OMPRT_OK;
}

extern "C" omprt_status omprt_reduce_array_plan(int64_t rows, int64_t m, int32_t dtype, int32_t op,
                                         int32_t aligned16, const omprt_config* cfg,
                                         int64_t* h_out8) {
    if (dtype < 0 || dtype >= DT_COUNT_ABI) return fail(OMPRT_ERR_UNSUPPORTED, "dtype %d", dtype);
    if (!op_defined(dtype, op)) return fail(OMPRT_ERR_UNSUPPORTED, "op %d on dtype %d", op, dtype);
    if (rows < 1 || m < 1) return fail(OMPRT_ERR_INVALID, "rows/m must be >= 1");
    if (!h_out8) return fail(OMPRT_ERR_INVALID, "out is NULL");
    ArrayPlan pl;
    const void* fake = reinterpret_cast<const void*>(aligned16 ? (uintptr_t)256 : (uintptr_t)260);
    if (omprt_status st = plan_array(rows, m, dtype, op, fake, cfg, &pl)) return st;
    const int64_t v[8] = {pl.g.W, pl.g.R, pl.g.col_tiles, pl.g.rt, pl.g.ng,
                          pl.loads == kVectors ? 16 : dtype_bytes(dtype), pl.threads,
                          pl.loads == kRagged ? pl.unroll * (16 / dtype_bytes(dtype)) : pl.unroll};
    for (int i = 0; i < 8; ++i) h_out8[i] = v[i];
    return OMPRT_OK;
}
