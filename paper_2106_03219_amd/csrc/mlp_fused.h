// mlp_fused.h -- the picker network's training step in two kernels, for
// networks whose weights fit a compute unit's LDS (every network of the size
// the picker uses; larger ones take the kernels of mlp.hip).
//
// A step of the picker's network is some 10^7 operations on 40 KB of weights:
// what bounds it is the number of launches, each a few microseconds of
// dispatch and cold loads.  mlp_rows_kernel carries a tile of batch rows
// through the forward pass, the softmax cross-entropy and both input
// gradients with every weight in LDS; mlp_grads_kernel forms every weight and
// bias gradient and the mean loss.  (16-64-64-64, 256 rows: loss and gradients
// and Adam 65.6 us with a launch for each matrix, 19.3 us now.)
#pragma once
#include "device.h"
#include "lines.h"

namespace omprt {

// Leading dimension of an LDS matrix whose rows of n floats are read in
// 16-byte blocks: whole blocks, an odd number of them, so that the lanes'
// rows start on different banks.
__host__ __device__ inline int mlp_ld(int n) { return ((n + 3) / 4 | 1) * 4; }

struct MlpShape {
    int F, H1, H2, K;
};

// Floats of LDS the parameters take (biases rounded up to whole 16-byte
// blocks), and mlp_rows_kernel takes for tiles of RT rows.
__host__ __device__ inline int mlp_parts_floats(const MlpShape& s) {
    return s.H1 * mlp_ld(s.F) + s.H2 * mlp_ld(s.H1) + s.K * mlp_ld(s.H2) + mlp_ld(s.H1) +
           mlp_ld(s.H2) + mlp_ld(s.K);
}
__host__ __device__ inline int mlp_rows_lds(const MlpShape& s, int RT) {
    return mlp_parts_floats(s) +
           RT * (mlp_ld(s.F) + 2 * mlp_ld(s.H1) + 2 * mlp_ld(s.H2) + mlp_ld(s.K));
}

constexpr int kRowsThreads = 256;
constexpr int kRowsWaves = kRowsThreads / kWave;

// Where a parameter of the flat buffer lands in LDS: six consecutive parts
// (W1, b1, W2, b2, W3, b3) of rows of n floats, ld floats apart in LDS.
struct MlpPart {
    int end;      // first flat index past the part
    int n, ld;    // row length there and in LDS
    int base;     // float offset in LDS
    float inv;    // 1 / n
};
struct MlpParts {
    MlpPart p[6];
};

inline MlpParts mlp_parts(const MlpShape& s) {
    const int rows[6] = {s.H1, 1, s.H2, 1, s.K, 1};
    const int width[6] = {s.F, s.H1, s.H1, s.H2, s.H2, s.K};
    MlpParts t{};
    int end = 0, base = 0;
    for (int k = 0; k < 6; ++k) {
        end += rows[k] * width[k];
        t.p[k] = MlpPart{end, width[k], mlp_ld(width[k]), base, 1.0f / (float)width[k]};
        base += rows[k] * mlp_ld(width[k]);
    }
    return t;
}

// The flat parameters into their LDS places, V at a time (float4 where every
// row length and the buffer's address allow, else float), all of a network of
// the picker's size in flight at once: 12 loads a thread.
template <class V>
__device__ __forceinline__ void mlp_stage(const float* __restrict__ params, float* lds,
                                          const MlpParts& parts) {
    constexpr int N = sizeof(V) / 4, U = 12;
    const int total = parts.p[5].end / N;
    const V* __restrict__ src = reinterpret_cast<const V*>(params);
    for (int e0 = threadIdx.x; e0 < total; e0 += U * kRowsThreads) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * kRowsThreads;
            v[u] = src[e < total ? e : e0];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * kRowsThreads;
            if (e >= total) break;
            int f = e * N, start = 0, n = parts.p[0].n, ld = parts.p[0].ld, base = parts.p[0].base;
            float inv = parts.p[0].inv;
#pragma unroll
            for (int k = 1; k < 6; ++k) {
                const bool past = f >= parts.p[k - 1].end;
                start = past ? parts.p[k - 1].end : start;
                n = past ? parts.p[k].n : n;
                ld = past ? parts.p[k].ld : ld;
                base = past ? parts.p[k].base : base;
                inv = past ? parts.p[k].inv : inv;
            }
            f -= start;
            // row of f: exact, since (f + 1/2) / n stays 1/(2n) off an integer
            // and a part holds under 2^20 floats
            const int r = (int)(((float)f + 0.5f) * inv);
            *reinterpret_cast<V*>(lds + base + r * ld + (f - r * n)) = v[u];
        }
    }
    if (N == 1)   // rows end inside a 16-byte block: zeros up to its end
#pragma unroll
        for (int k = 0; k < 6; k += 2)
            for (int r = threadIdx.x; r < (parts.p[k].end - (k ? parts.p[k - 1].end : 0)) / parts.p[k].n;
                 r += kRowsThreads)
                for (int c = parts.p[k].n; c < parts.p[k].ld; ++c)
                    lds[parts.p[k].base + r * parts.p[k].ld + c] = 0.0f;
}

// Zeros from a wave's rows' n columns to the end of their last 16-byte block.
template <int RPW>
__device__ __forceinline__ void mlp_pad_rows(float* row, int ld, int n) {
    const int j = n + (threadIdx.x & (kWave - 1));
    if (j < (n + 3) / 4 * 4)
#pragma unroll
        for (int q = 0; q < RPW; ++q) row[q * kRowsWaves * ld + j] = 0.0f;
}

// Wave w's rows w, w + kRowsWaves, ... (RPW of them): y[r][j] = act(b[j] +
// sum_i W[j][i] x[r][i]), lanes over j, four partial sums over i.  The rows
// are padded with zeros to whole 16-byte blocks.
template <int RPW, bool RELU>
__device__ __forceinline__ void mlp_forward_rows(const float* W, int ldw, const float* b,
                                                 const float* x, int ldx, float* y, int ldy, int in,
                                                 int out) {
    constexpr int kBlocks = 4;   // blocks read ahead of their products
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const float* xr = x + wave * ldx;
    float* yr = y + wave * ldy;
    for (int j = lane; j < out; j += kWave) {
        float4 acc[RPW];
#pragma unroll
        for (int q = 0; q < RPW; ++q) acc[q] = float4{0.0f, 0.0f, 0.0f, 0.0f};
        const float4* wv = reinterpret_cast<const float4*>(W + j * ldw);
        const int blocks = (in + 3) / 4;
#pragma unroll kBlocks
        for (int i = 0; i < blocks; ++i) {
            const float4 w = wv[i];
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const float4 v = reinterpret_cast<const float4*>(xr + q * kRowsWaves * ldx)[i];
                acc[q].x = __builtin_fmaf(w.x, v.x, acc[q].x);
                acc[q].y = __builtin_fmaf(w.y, v.y, acc[q].y);
                acc[q].z = __builtin_fmaf(w.z, v.z, acc[q].z);
                acc[q].w = __builtin_fmaf(w.w, v.w, acc[q].w);
            }
        }
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const float s = ((acc[q].x + acc[q].y) + (acc[q].z + acc[q].w)) + b[j];
            yr[q * kRowsWaves * ldy + j] = RELU ? fmaxf(s, 0.0f) : s;
        }
    }
    mlp_pad_rows<RPW>(yr, ldy, out);
}

// The same waves and rows: dp[r][i] = (sum_j d[r][j] W[j][i]) [a[r][i] > 0],
// lanes over i, four partial sums over j (d's padding is zero; W's rows past
// `out` are not read: the last block stops at out).
template <int RPW>
__device__ __forceinline__ void mlp_backward_rows(const float* W, int ldw, const float* d, int ldd,
                                                  const float* a, float* dp, int ldp, int in,
                                                  int out) {
    constexpr int kBlocks = 4;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const float* dr = d + wave * ldd;
    const float* ar = a + wave * ldp;
    float* pr = dp + wave * ldp;
    for (int i = lane; i < in; i += kWave) {
        float4 acc[RPW];
#pragma unroll
        for (int q = 0; q < RPW; ++q) acc[q] = float4{0.0f, 0.0f, 0.0f, 0.0f};
        const float* wc = W + i;
        auto block = [&](int j, int last) {   // rows j .. j + 3, none past `last`
            float w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = wc[(j + u < last ? j + u : last) * ldw];
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const float4 v = reinterpret_cast<const float4*>(dr + q * kRowsWaves * ldd)[j / 4];
                acc[q].x = __builtin_fmaf(v.x, w[0], acc[q].x);
                acc[q].y = __builtin_fmaf(v.y, w[1], acc[q].y);
                acc[q].z = __builtin_fmaf(v.z, w[2], acc[q].z);
                acc[q].w = __builtin_fmaf(v.w, w[3], acc[q].w);
            }
        };
        const int whole = out / 4 * 4;
#pragma unroll kBlocks
        for (int j = 0; j < whole; j += 4) block(j, j + 3);
        if (whole < out) block(whole, out - 1);
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const float s = (acc[q].x + acc[q].y) + (acc[q].z + acc[q].w);
            pr[q * kRowsWaves * ldp + i] = ar[q * kRowsWaves * ldp + i] > 0.0f ? s : 0.0f;
        }
    }
    mlp_pad_rows<RPW>(pr, ldp, in);
}

// Store the wave's rows (columns [0, n) of rows of ld floats) to dst[B][n].
template <int RPW>
__device__ __forceinline__ void mlp_store_rows(const float* src, int ld, float* __restrict__ dst,
                                               int n, int64_t row0, int B) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        const int64_t r = row0 + wave + q * kRowsWaves;
        if (r >= B) break;
        for (int j = lane; j < n; j += kWave) dst[r * n + j] = src[(wave + q * kRowsWaves) * ld + j];
    }
}

// Maximum and plain sum over a wave (softmax).
struct MaxPolicy {
    using Acc = float;
    static __device__ __forceinline__ float combine(float a, float b) { return fmaxf(a, b); }
};
struct AddPolicy {
    using Acc = float;
    static __device__ __forceinline__ float combine(float a, float b) { return a + b; }
};

struct MlpRowsOut {   // [B][..] each; TRAIN writes all but z, else z alone
    float *z, *a1, *a2, *dz, *d2, *d1, *row_loss;
};

// One tile of RT = kRowsWaves * RPW batch rows.  Rows past B run on zeros and
// are not stored.
template <bool TRAIN, int RPW>
__global__ __launch_bounds__(kRowsThreads) void mlp_rows_kernel(
    MlpShape s, MlpParts parts, const float* __restrict__ params, const float* __restrict__ X,
    const int32_t* __restrict__ y, int B, MlpRowsOut o) {
    constexpr int RT = kRowsWaves * RPW;
    extern __shared__ __align__(16) float mlp_lds[];
    const int lF = mlp_ld(s.F), l1 = mlp_ld(s.H1), l2 = mlp_ld(s.H2), lK = mlp_ld(s.K);
    const float* W1 = mlp_lds + parts.p[0].base;
    const float* b1 = mlp_lds + parts.p[1].base;
    const float* W2 = mlp_lds + parts.p[2].base;
    const float* b2 = mlp_lds + parts.p[3].base;
    const float* W3 = mlp_lds + parts.p[4].base;
    const float* b3 = mlp_lds + parts.p[5].base;
    float* x = mlp_lds + mlp_parts_floats(s);
    float* a1 = x + RT * lF;
    float* a2 = a1 + RT * l1;
    float* z = a2 + RT * l2;
    float* d2 = z + RT * lK;
    float* d1 = d2 + RT * l2;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int64_t row0 = (int64_t)blockIdx.x * RT;
    int lab[RPW];   // read with the parameters, used after the forward pass
    if constexpr (TRAIN) {
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const int64_t r = row0 + wave + q * kRowsWaves;
            lab[q] = y[r < B ? r : 0];
        }
    }
    for (int e = tid; e < RT * lF; e += kRowsThreads) {
        const int r = e / lF, c = e - r * lF;
        x[e] = c < s.F && row0 + r < B ? X[(row0 + r) * s.F + c] : 0.0f;
    }
    if (((s.F | s.H1 | s.H2 | s.K) & 3) == 0 && (reinterpret_cast<uintptr_t>(params) & 15) == 0)
        mlp_stage<float4>(params, mlp_lds, parts);
    else
        mlp_stage<float>(params, mlp_lds, parts);
    __syncthreads();
    // a wave works on its own rows from here on: what it reads back it wrote
    // itself, and the LDS runs one wave's accesses in order
    mlp_forward_rows<RPW, true>(W1, lF, b1, x, lF, a1, l1, s.F, s.H1);
    wave_lds_order();
    mlp_forward_rows<RPW, true>(W2, l1, b2, a1, l1, a2, l2, s.H1, s.H2);
    wave_lds_order();
    mlp_forward_rows<RPW, false>(W3, l2, b3, a2, l2, z, lK, s.H2, s.K);
    wave_lds_order();
    if constexpr (!TRAIN) {
        mlp_store_rows<RPW>(z, lK, o.z, s.K, row0, B);
    } else {
        // loss_r = logsumexp(z) - z[y];  dz = (softmax(z) - onehot(y)) / B
        const float inv = 1.0f / (float)B;
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const int64_t r = row0 + wave + q * kRowsWaves;
            float* zr = z + (wave + q * kRowsWaves) * lK;
            float mx = -INFINITY;
            for (int j = lane; j < s.K; j += kWave) mx = fmaxf(mx, zr[j]);
            mx = wave_reduce<MaxPolicy>(mx);
            float den = 0.0f;
            for (int j = lane; j < s.K; j += kWave) den += expf(zr[j] - mx);
            den = wave_reduce<AddPolicy>(den);
            if (lane == 0 && r < B) o.row_loss[r] = logf(den) - (zr[lab[q]] - mx);
            wave_lds_order();   // zr[lab] is read before it is overwritten
            for (int j = lane; j < s.K; j += kWave) {
                const float pj = expf(zr[j] - mx) / den;
                zr[j] = (pj - (j == lab[q] ? 1.0f : 0.0f)) * inv;
            }
        }
        wave_lds_order();
        mlp_backward_rows<RPW>(W3, l2, z, lK, a2, d2, l2, s.H2, s.K);
        wave_lds_order();
        mlp_backward_rows<RPW>(W2, l1, d2, l2, a1, d1, l1, s.H1, s.H2);
        mlp_store_rows<RPW>(a1, l1, o.a1, s.H1, row0, B);
        mlp_store_rows<RPW>(a2, l2, o.a2, s.H2, row0, B);
        mlp_store_rows<RPW>(z, lK, o.dz, s.K, row0, B);
        mlp_store_rows<RPW>(d2, l2, o.d2, s.H2, row0, B);
        wave_lds_order();
        mlp_store_rows<RPW>(d1, l1, o.d1, s.H1, row0, B);
    }
}

// ---------------------------------------------------------------- gradients

// One of the step's three weight matrices: GW[out][in] = D^T A, gb[out] the
// column sums of D, at `grad` floats into the gradients.
struct MlpLayer {
    const float *D, *A;
    int out, in;
    int grad;                 // of W; b's gradient follows it
    int cw;                   // columns of a tile (of one row of W): 16, 32 or 64
    int tiles_i;              // tiles a row
};
struct MlpGradPlan {
    MlpLayer l[3];
    const float* row_loss;
    BalSplit rows;            // the batch rows over the slices
    int B, nparams;
    int first_tile[4];        // first workgroup of each layer's tiles, then of its biases
    int first_bias[4];        // ... [3]: the loss workgroup
};

constexpr int kGradThreads = 1024;
constexpr int kGradWaves = kGradThreads / kWave;

// Join the pairs of the lanes that hold the same columns (lane % Q).
template <int Q>
__device__ __forceinline__ ff_t join_subs(ff_t a) {
    using R = Red<DT_F32, OP_SUM>;
    if constexpr (Q <= 4) a = R::combine(a, dpp_move<kDppRowRor4>(a));
    if constexpr (Q <= 8) a = R::combine(a, dpp_move<kDppRowRor8>(a));
    LanePair<ff_t> p = lane_pair<false>(a);
    a = R::combine(p.lo, p.hi);
    p = lane_pair<true>(a);
    return R::combine(p.lo, p.hi);
}

// The lane's part of sum_r D[r][j] A[r][i0 .. i0 + 3] (columns i0.. of a tile of
// 4 Q columns, rows row0 + sub, in steps of `step`), then the wave's.
template <int Q>
__device__ __forceinline__ void grad_tile(const float* __restrict__ D, const float* __restrict__ A,
                                          int in, int out, int j, int i0, int row0, int hi,
                                          int step, ff_t (&acc)[4]) {
    constexpr int U = 4;   // rows in flight a lane
    for (int r0 = row0; r0 < hi; r0 += U * step) {
        float4 a[U];
        float d[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * step < hi ? r0 + u * step : r0;
            a[u] = *reinterpret_cast<const float4*>(A + (uint32_t)(r * in + i0));
            d[u] = D[(uint32_t)(r * out + j)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u * step >= hi) break;
            comp_add(acc[0], __fmul_rn(d[u], a[u].x));
            comp_add(acc[1], __fmul_rn(d[u], a[u].y));
            comp_add(acc[2], __fmul_rn(d[u], a[u].z));
            comp_add(acc[3], __fmul_rn(d[u], a[u].w));
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = join_subs<Q>(acc[q]);
}

// Workgroup x: one tile of one row of one W's gradient, 64 bias gradients or
// the mean loss; workgroup y: slice y of S of the batch rows.  The 16 waves
// split the slice's rows; every output is a compensated pair (TwoSum of the
// rounded products), and the lanes' and waves' pairs join in a fixed order.
// With S == 1 the gradients are written, else the slice's pairs go to
// partial[y][parameter] (the loss after the parameters).
// VEC (every layer's inputs whole 16-byte blocks): a lane takes four columns
// of one row at a time, so a wave's load of A covers 1 KiB and its load of D
// serves four to sixteen rows; the loads, not the 8 operations a product, are
// what a row costs otherwise (256 rows 5.9 us; one column a lane 7.7, four
// rows of W a lane over a quarter of the workgroups 10.2).
template <bool VEC>
__global__ __launch_bounds__(kGradThreads) void mlp_grads_kernel(MlpGradPlan p,
                                                                 float* __restrict__ grads,
                                                                 float* __restrict__ loss,
                                                                 ff_t* __restrict__ partial) {
    __shared__ __align__(16) ff_t red[kGradWaves][kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int S = gridDim.y;
    const Range slice = p.rows.share(blockIdx.y);
    const int lo = (int)slice.lo, hi = (int)slice.hi;
    const int wg = blockIdx.x;
    int at = 0, cols = 0;   // parameter of the workgroup's first column, columns
    if (wg < p.first_tile[3]) {
        const int li = wg >= p.first_tile[2] ? 2 : wg >= p.first_tile[1] ? 1 : 0;
        const MlpLayer& l = p.l[li];
        const float* __restrict__ A = l.A;
        const float* __restrict__ D = l.D;
        const int in = l.in, out = l.out;   // (under 2^31 elements)
        const int t = wg - p.first_tile[li];
        const int j = t / l.tiles_i, c0 = (t % l.tiles_i) * l.cw;
        at = l.grad + j * in + c0;
        cols = in - c0 < l.cw ? in - c0 : l.cw;
        if constexpr (VEC) {
            const int Q = l.cw / 4, sub = lane / Q, subs = kWave / Q;
            const int q0 = (lane & (Q - 1)) * 4;
            const int i0 = c0 + (q0 < cols ? q0 : 0);
            const int row0 = lo + wave * subs + sub, step = kGradWaves * subs;
            ff_t acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = ff_t{0.0f, 0.0f};
            if (Q == 16)
                grad_tile<16>(D, A, in, out, j, i0, row0, hi, step, acc);
            else if (Q == 8)
                grad_tile<8>(D, A, in, out, j, i0, row0, hi, step, acc);
            else
                grad_tile<4>(D, A, in, out, j, i0, row0, hi, step, acc);
            if (lane < Q) {
#pragma unroll
                for (int q = 0; q < 4; ++q) red[wave][lane * 4 + q] = acc[q];
            }
        } else {
            constexpr int U = 8;
            const int i = c0 + (lane < cols ? lane : 0);
            ff_t acc{0.0f, 0.0f};
            for (int r0 = lo + wave; r0 < hi; r0 += U * kGradWaves) {
                float a[U], d[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = r0 + u * kGradWaves < hi ? r0 + u * kGradWaves : r0;
                    a[u] = A[(uint32_t)(r * in + i)];
                    d[u] = D[(uint32_t)(r * out + j)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (r0 + u * kGradWaves < hi) comp_add(acc, __fmul_rn(d[u], a[u]));
            }
            red[wave][lane] = acc;
        }
    } else {
        const bool is_loss = wg >= p.first_bias[3];
        const int li = is_loss ? 0 : wg >= p.first_bias[2] ? 2 : wg >= p.first_bias[1] ? 1 : 0;
        const MlpLayer& l = p.l[li];
        const float* __restrict__ src = is_loss ? p.row_loss : l.D;
        const int stride = is_loss ? 1 : l.out;
        const int j0 = is_loss ? 0 : (wg - p.first_bias[li]) * kWave;
        at = is_loss ? p.nparams : l.grad + l.out * l.in + j0;
        cols = stride - j0 < kWave ? stride - j0 : kWave;
        const int j = j0 + (lane < cols ? lane : 0);
        constexpr int U = 8;
        ff_t acc{0.0f, 0.0f};
        for (int r0 = lo + wave; r0 < hi; r0 += U * kGradWaves) {
            float d[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = r0 + u * kGradWaves < hi ? r0 + u * kGradWaves : r0;
                d[u] = src[(uint32_t)(r * stride + j)];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (r0 + u * kGradWaves < hi) comp_add(acc, d[u]);
        }
        red[wave][lane] = acc;
    }
    __syncthreads();
    // the first wave joins the waves' pairs, a column a lane
    if (tid >= cols) return;
    ff_t s = red[0][tid];
#pragma unroll
    for (int w = 1; w < kGradWaves; ++w) s = pair_join(s, red[w][tid]);
    const int e = at + tid;
    if (S > 1)
        partial[(size_t)blockIdx.y * (p.nparams + 1) + e] = s;
    else if (e == p.nparams)
        loss[0] = (s.hi + s.lo) / (float)p.B;
    else
        grads[e] = s.hi + s.lo;
}

// The slices' pairs, joined in slice order.
__global__ __launch_bounds__(256) void mlp_grads_merge_kernel(const ff_t* __restrict__ partial,
                                                              int S, int nparams, int B,
                                                              float* __restrict__ grads,
                                                              float* __restrict__ loss) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e > nparams) return;
    ff_t s = partial[e];
    for (int k = 1; k < S; ++k) s = pair_join(s, partial[(size_t)k * (nparams + 1) + e]);
    if (e == nparams)
        loss[0] = (s.hi + s.lo) / (float)B;
    else
        grads[e] = s.hi + s.lo;
}

}  // namespace omprt
