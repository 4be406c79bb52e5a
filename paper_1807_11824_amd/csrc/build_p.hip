// Alg. 1 lines 1-2 of the paper on gfx950: the sparse affinity matrix P.
//
//   row_norms            |x_i|^2 in double, rounded to float
//   split_bf16           every x as bf16 high part + bf16 low part
//   knn_tile_mfma        Sec. III-B, exact reading: all-pairs squared distances
//                        |q|^2 + |x|^2 - 2 q.x, the dot products on the matrix cores
//                        (three v_mfma_f32_32x32x16_bf16 per step on the split values, 256x128 or
//                        128x128 tiles through LDS).  The N x N matrix is never stored: the
//                        epilogue keeps a pair only if it beats the query row's current cut-off
//                        and appends it to that row's candidate buffer.
//   knn_tile_resident    the same for d <= 64 and many query rows: a workgroup keeps 256 query rows
//                        on chip for the whole launch and streams the database rows past them
//   knn_compact          per query row, keeps the best k' = k + margin of the buffer and lowers
//                        the cut-off to the k'-th distance
//   knn_rerank           recomputes the k' candidate distances as sum_t (x_it - x_jt)^2 in double,
//                        orders them by (distance, index), keeps k, and certifies the row: every
//                        discarded pair had a tile distance >= cut-off, so it cannot belong to
//                        the k nearest if cut-off - error bound > exact k-th distance
//   knn_exact_dists / knn_exact_select   rows that fail the certificate: all n distances in
//                        double, radix selection of the k-th smallest, ties by index
//   ivf_probe_tiles / ivf_search_tiles   Eq. (10) and (11) of the approximate search for rows longer than 64
//                        coordinates, on the same tiles, re-rank and certificate (called from ivf.hip)
//   perplexity_search    Eq. (1) on the k neighbours, beta by bracketing, Newton steps and bisection on the entropy
//   sym_count / sym_fill / sym_sort_rows   p_ij = (p_j|i + p_i|j) / 2N as CSR, columns ascending
#include "tsne_internal.h"

#include <algorithm>
#include <functional>

#include <limits.h>
#include <math.h>
#include <stdio.h>
#include <string.h>

namespace {

constexpr size_t ALIGN = 256;
__host__ __device__ inline size_t up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

constexpr int QB = 65536;       // query rows per pass
constexpr int DBC = 2048;       // database rows per launch (bounds what one launch can append per row)
constexpr int MAX_KP = 1920;    // k' limit (the re-rank's LDS arrays: 24 bytes each)
constexpr int SORT_SHORT = 512, SORT_CAP = 4096;  // entries of a row of P that are sorted in LDS at a time (ordinary, long rows)
constexpr int TN = 128;         // database rows per tile
constexpr int KNN_MB = 4;        // 32-row query blocks per wave of the general single-level tile kernel
constexpr int COMPACT_SLACK = 64;  // new candidates per row that trigger a compaction of its buffer
constexpr int COMPACT_EVERY = 2;   // after the resident tile kernel a compaction pass follows every second slab only (a pass
                                   // costs a third of a slab; cut-offs one slab older let a few more pairs through)
constexpr int KFLUSH = 64;      // columns summed on the matrix cores before a flush into the running sum
constexpr int HALF_OWN_MIN_ROWS = 128 * 256, HALF_OWN_MAX_D = 2048;     // where the half-precision tiles go query tile by query tile
constexpr int HIGH_FIRST_MIN_D = 256;   // from this many columns on the exact search always sweeps in half precision first

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t orderable(float f)
{
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unorderable(uint32_t u)
{
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}
__device__ __forceinline__ uint64_t orderable64(double d)
{
    uint64_t u = (uint64_t)__double_as_longlong(d);
    return (u & 0x8000000000000000ull) ? ~u : (u | 0x8000000000000000ull);
}

// Squared distances do not change when every row is moved by the same vector, while the error of
// the candidate search grows with the rows' norms: the search therefore works on X - mu, mu the
// column means (only the split copy and the norms are centred; the re-rank reads the caller's X).
// Any mu gives correct lists; this one is computed in a fixed order so that a build is reproducible, and of MEAN_ROWS to
// 2 MEAN_ROWS rows at most: one of every `step`, at a place in its share that follows no period of the data.  (All rows of
// 1,281,167 x 2048 took 2.7 ms, three times in an approximate build; now 0.11 ms.)
constexpr int MEAN_CHUNKS = 256;     // row chunks of the first stage
constexpr int MEAN_ROWS = 65536;
__global__ __launch_bounds__(256) void col_mean_part(const float *__restrict__ X, int n, int d, int step, int rows, int rows_per_chunk,
                                                     double *__restrict__ part)
{
    __shared__ double acc[4][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), rg = threadIdx.x >> 6;
    const int r0 = blockIdx.y * rows_per_chunk, r1 = min(rows, r0 + rows_per_chunk);
    double s = 0.0;
    if (c < d) {
#pragma unroll 4
        for (int r = r0 + rg; r < r1; r += 4) {
            const int src = min(r * step + (int)((uint32_t)r * 2654435761u >> 16) % step, n - 1);
            s += (double)X[(size_t)src * d + c];
        }
    }
    acc[rg][threadIdx.x & 63] = s;
    __syncthreads();
    if (rg == 0 && c < d) part[(size_t)blockIdx.y * d + c] = ((acc[0][threadIdx.x] + acc[1][threadIdx.x]) + acc[2][threadIdx.x]) + acc[3][threadIdx.x];
}

// MEAN_SEGS threads a column, each a contiguous share of the chunks (one thread a column was a chain of 256 dependent
// reads: 60 of the 382 us of a build of 2000 x 50).
constexpr int MEAN_SEGS = 16;
__global__ __launch_bounds__(256) void col_mean_final(const double *__restrict__ part, int nchunks, int n, int d, int dp,
                                                      float *__restrict__ mu)
{
    __shared__ double sum[MEAN_SEGS][256 / MEAN_SEGS];
    const int cl = (int)threadIdx.x % (256 / MEAN_SEGS), seg = (int)threadIdx.x / (256 / MEAN_SEGS);
    const int c = blockIdx.x * (256 / MEAN_SEGS) + cl, len = (nchunks + MEAN_SEGS - 1) / MEAN_SEGS;
    double s = 0.0;
    if (c < d) {
#pragma unroll 8
        for (int q = seg * len; q < min(nchunks, (seg + 1) * len); ++q) s += part[(size_t)q * d + c];
    }
    sum[seg][cl] = s;
    __syncthreads();
    if (seg != 0 || c >= dp) return;
    for (int k = 1; k < MEAN_SEGS; ++k) s += sum[k][cl];
    mu[c] = c < d ? (float)(s / (double)n) : 0.f;
}
static void launch_col_mean(const float *X, int n, int d, int dp, double *part, float *mu, hipStream_t s)
{
    const int step = std::max(1, n / MEAN_ROWS), rows = (n + step - 1) / step;
    const int rows_per_chunk = (rows + MEAN_CHUNKS - 1) / MEAN_CHUNKS, nchunks = (rows + rows_per_chunk - 1) / rows_per_chunk;
    hipLaunchKernelGGL(col_mean_part, dim3((d + 63) / 64, nchunks), dim3(256), 0, s, X, n, d, step, rows, rows_per_chunk, part);
    hipLaunchKernelGGL(col_mean_final, dim3((dp + 256 / MEAN_SEGS - 1) / (256 / MEAN_SEGS)), dim3(256), 0, s, part, nchunks, rows, d, dp, mu);
}

// |x - mu|^2 of the centred row as the tiles see it (each x_t - mu_t rounded to float)
// (rowmap: row r of the result is row rowmap[r] of the nsrc rows of X; null = the same rows)
__global__ __launch_bounds__(256) void row_norms(const float *__restrict__ X, const float *__restrict__ mu, int n, int d,
                                                 const int *__restrict__ rowmap, int nsrc, float *__restrict__ norms)
{
    const size_t w = global_index() >> 6;
    if (w >= (size_t)n) return;
    const int row = (int)w;
    const float *x = X + (size_t)(rowmap ? min(max(rowmap[row], 0), nsrc - 1) : row) * d;
    double s = 0.0;
#pragma unroll 8
    for (int t = lane_id(); t < d; t += WAVE) { double v = (double)(x[t] - mu[t]); s += v * v; }
    s = wave_sum(s);
    if (lane_id() == 0) norms[row] = (float)s;
}

__global__ void knn_reset(float *__restrict__ tau, int *__restrict__ cnt, int rows, int *__restrict__ ccount)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) { tau[i] = INFINITY; cnt[i] = 0; }
    if (i < 2) ccount[i] = 0;
}

// ---- the distance tiles
// Candidates only have to be found, not ranked (knn_rerank does that in double), so the dot
// products run on the bf16 matrix cores at sixteen times the rate of the fp32 ones: every value
// is split as x = hi + lo + rest, hi = bf16(x), lo = bf16(x - hi), |rest| <= 2^-18 |x|, and
// q.x is taken as sum hi.hi + hi.lo + lo.hi, accumulated in fp32.  What this leaves out, and
// what the accumulation rounds away, is bounded in tile_error_coeff(); knn_rerank certifies
// each row against that bound, so the neighbour lists stay exact.
//
// split_bf16 lays the two parts out for the tile kernel: row-major, the row padded to a multiple
// of SLAB columns, and per SLAB columns the 32 high parts followed by the 32 low parts (128 bytes,
// the piece of a row that one LDS slab holds).
constexpr int SLAB = 32;                  // columns per LDS slab (two matrix-core steps of 16)
constexpr int SLAB_ROW = 4 * SLAB;        // bytes of a row's piece of a slab
constexpr int LDS_ROW = SLAB_ROW + 16;    // padded: 8 consecutive rows' 16-byte reads hit distinct banks

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t bf16_rne(float x)
{
    uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__global__ __launch_bounds__(256) void split_bf16(const float *__restrict__ X, const float *__restrict__ mu, int n, int d,
                                                  int dp, const int *__restrict__ rowmap, int nsrc,
                                                  uint16_t *__restrict__ Xs)
{
    const size_t e = global_index();
    if (e >= (size_t)n * dp) return;
    const size_t row = e / dp;
    const int k = (int)(e % dp);
    const size_t src = rowmap ? (size_t)min(max(rowmap[row], 0), nsrc - 1) : row;
    const float x = k < d ? X[src * d + k] - mu[k] : 0.f;
    const uint32_t hi = bf16_rne(x);
    const uint32_t lo = bf16_rne(x - __uint_as_float(hi << 16));      // the difference is exact in fp32
    uint16_t *o = Xs + row * dp * 2 + (size_t)(k / SLAB) * (2 * SLAB) + (k % SLAB);
    o[0] = (uint16_t)hi;
    o[SLAB] = (uint16_t)lo;
}

// The values in half precision, for the first sweep over long rows: row-major, rows padded to a multiple of 64
// columns, scaled by a power of two (`scale`) that brings the largest magnitude just below 2^15: nothing overflows,
// and what is too small for a normal half is below 2^-28 of the largest magnitude.
// Eight columns a thread: two 16-byte loads where rows are whole 16-byte pieces, one 16-byte store.  (rowmap: as in row_norms.)
__global__ __launch_bounds__(256) void split_high(const float *__restrict__ X, const float *__restrict__ mu, int n, int d,
                                                  int dph, float scale, const int *__restrict__ rowmap, int nsrc,
                                                  uint16_t *__restrict__ Xh)
{
    const size_t e = global_index();
    const int per = dph / 8;
    if (e >= (size_t)n * per) return;
    const size_t row = e / per;
    const int k = (int)(e % per) * 8;
    const float *x = X + (rowmap ? (size_t)min(max(rowmap[row], 0), nsrc - 1) : row) * d;
    float v[8];
    if (d % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0 && k + 8 <= d) {
        const float4 a = *reinterpret_cast<const float4 *>(x + k), b = *reinterpret_cast<const float4 *>(x + k + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] -= mu[k + q];
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = k + q < d ? x[k + q] - mu[k + q] : 0.f;
    }
    halfx8 h;
#pragma unroll
    for (int q = 0; q < 8; ++q) h[q] = (_Float16)(v[q] * scale);       // round to nearest even
    *reinterpret_cast<halfx8 *>(Xh + row * dph + k) = h;
}

// max |x - mu| over all values, as the bits of a non-negative float (they order like the values)
// (a wave a row at a time: with one index over all values its remainder took longer than the loads, 60,000 x 784 128 us
// against 118)
__global__ __launch_bounds__(256) void max_abs_centred(const float *__restrict__ X, const float *__restrict__ mu, int n,
                                                       int d, unsigned int *__restrict__ out)
{
    float v = 0.f;
    for (size_t r = global_index() >> 6; r < (size_t)n; r += (size_t)gridDim.x * (blockDim.x >> 6)) {
        const float *x = X + r * d;
#pragma unroll 8
        for (int t = lane_id(); t < d; t += WAVE) v = fmaxf(v, fabsf(x[t] - mu[t]));
    }
    v = wave_max(v);
    if (lane_id() == 0) atomicMax(out, __float_as_uint(v));
}

// Bound on |computed - exact| of one tile distance, as a multiple of |q|^2 + |x|^2.
//   split: the products left out (lo.lo, rest.x, x.rest) are at most 3 (1 + 2^-18) 2^-18 |q_t x_t| each;
//   accumulation: a sum reaches the result through at most R fp32 additions, R = 3 * (columns per
//     flush) + number of flushes; each is taken to lose up to 2^-23 relative (one unit in the last
//     place, which also covers truncating adders), so the sum is off by R 2^-23 / (1 - R 2^-23)
//     times the sum of |terms| <= (1 + 2^-8)^2 sum |q_t x_t|;
//   sum |q_t x_t| <= (|q|^2 + |x|^2) / 2, and the distance takes -2 times the dot product;
//   norms (each a rounded double sum), their sum and the final fused multiply-add: 8 more roundings
//   of quantities below 2 (|q|^2 + |x|^2);
//   centring: q' = fl(q - mu), x' = fl(x - mu) are off by 2^-24 relative per coordinate, which moves
//   |q' - x'|^2 by at most 2 |q - x| 2^-24 (|q'| + |x'|) <= 4 2^-24 (|q'|^2 + |x'|^2) (and a second-order term).
// 5 % on top for the norms themselves being rounded values.  q, x here are the centred rows.
// high_only: the tiles multiply the values rounded to half precision (one product per coordinate): what is left
// out is then q ex + eq x - eq ex with |eq| <= 2^-11 |q|, |ex| <= 2^-11 |x|, at most (2^-10 + 2^-22) |q_t x_t|
// (values too small for a normal half are covered by an additive term, see high_first_extra()).
__host__ __device__ inline double tile_error_coeff(int d, bool two_level, bool high_only = false)
{
    const int dp = (d + SLAB - 1) / SLAB * SLAB;
    const double per = high_only ? 1.0 : 3.0;      // products per coordinate
    const double R = two_level ? per * KFLUSH + (double)((dp + KFLUSH - 1) / KFLUSH) : per * dp;
    const double u = 1.1920928955078125e-07;   // 2^-23
    const double split = high_only ? 0.0009765625 + 2.384185791015625e-07
                                   : 3.0 * (1.0 + 3.814697265625e-06) * 3.814697265625e-06;
    const double accum = 1.0079 * R * u / (1.0 - R * u);
    return 1.05 * (split + accum + (16.0 + 4.2) * 5.9604644775390625e-08);
}

// Are the k-th and the k'-th neighbour farther apart than half precision can be off?  Asked of a few query rows, a workgroup
// each, spread evenly over X, among an even sample of GAP_SAMPLE rows, where the two have the ranks r1 and r2; counts the
// query rows that say no.  (Of points near a plane, close to their neighbours and far from the mean, hardly a row gets a
// certificate, and without the question both sweeps are paid for.  50 to 90 us, bound by the latency of the sample's rows,
// eight of which a lane has on their way.  33,000 x 100, 50,000 x 100 and 65,000 x 200 near a plane: 9.7 -> 6.0, 16.5 -> 10.3,
// 27.4 -> 17.5 ms; 33,000 x 100 in clusters 4.50 -> 4.56.)
constexpr int GAP_QUERIES = 32, GAP_SAMPLE = 4096;

__global__ __launch_bounds__(1024) void half_gap_sample(const float *__restrict__ X, int n, int d, int m, int r1, int r2,
                                                        const float *__restrict__ norms, float norm_max, double coeff,
                                                        int *__restrict__ narrow)
{
    __shared__ float dist[GAP_SAMPLE];
    __shared__ int below[2][2][16];
    const int i = (int)(((long long)blockIdx.x * n) / gridDim.x), g = threadIdx.x / 16, sub = threadIdx.x % 16;
    const float *x = X + (size_t)i * d;
    for (int c0 = g; c0 < m; c0 += 64 * 8) {
        const float *y[8];
        float a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            y[u] = X + (size_t)(((long long)min(c0 + 64 * u, m - 1) * n) / m) * d;
            a[u] = 0.f;
        }
#pragma unroll 2
        for (int t = sub; t < d; t += 16)
#pragma unroll
            for (int u = 0; u < 8; ++u) { const float df = x[t] - y[u][t]; a[u] = fmaf(df, df, a[u]); }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) a[u] += __shfl_xor(a[u], o, WAVE);
            if (sub == 0 && c0 + 64 * u < m) dist[c0 + 64 * u] = y[u] == x ? INFINITY : a[u];
        }
    }
    __syncthreads();
    // the values of the two ranks, from their leading bits down (squares: the bit patterns are ordered)
    uint32_t v[GAP_SAMPLE / 1024], at[2] = {0u, 0u};
#pragma unroll
    for (int u = 0; u < GAP_SAMPLE / 1024; ++u) {
        const int c = u * 1024 + (int)threadIdx.x;
        v[u] = c < m ? __float_as_uint(dist[c]) : 0xFFFFFFFFu;
    }
    for (int bit = 30; bit >= 0; --bit) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            int here = 0;
#pragma unroll
            for (int u = 0; u < GAP_SAMPLE / 1024; ++u) here += (int)__popcll(__ballot(v[u] < (at[r] | (1u << bit))));
            if (lane_id() == 0) below[bit & 1][r][threadIdx.x >> 6] = here;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            int all = 0;
#pragma unroll
            for (int w = 0; w < 16; ++w) all += below[bit & 1][r][w];
            if (all < (r == 0 ? r1 : r2)) at[r] |= 1u << bit;
        }
    }
    const double gap = (double)__uint_as_float(at[1]) - (double)__uint_as_float(at[0]);
    if (threadIdx.x == 0 && !(gap > coeff * ((double)norms[i] + (double)norm_max))) atomicAdd(narrow, 1);
}

// Scaling of the values for half precision, every one of them below xmax: by a power of two so that all are below 2^15.
// dot_scale undoes it in a product.  A scaled value below 2^-14 may be rounded to a subnormal half or flushed to zero: off
// by at most delta = 2^-14 / scale per value, the dot product by delta (sum |q_t| + sum |x_t|) + D delta^2, the distance by
// twice that (e_add); sum |x_t| <= sqrt(D) |x|.
struct HalfScale {
    float scale, dot_scale;
    double e_add;
};
// Values it is for: dot_scale is a normal float from 2^-49 on (2^-126; the rule was 1e-15, a little less, and gave 2^-128), and
// below 1e15 the squares are far from the largest float.  Not 0 and not a number that is none.
inline bool half_scales(float xmax) { return xmax >= 0x1p-49f && xmax < 1e15f; }
inline HalfScale half_scale(float xmax, int d, double norm_max)
{
    HalfScale h;
    int e = 0;
    (void)frexpf(xmax, &e);                                 // xmax < 2^e
    h.scale = ldexpf(1.0f, 15 - e);
    h.dot_scale = ldexpf(1.0f, 2 * (e - 15));
    const double delta = ldexp(1.0, -14) / (double)h.scale;
    h.e_add = 2.0 * (delta * 2.0 * sqrt((double)d) * sqrt(norm_max) + (double)d * delta * delta);
    return h;
}

// A wave's queue of accepted pairs lives in LDS.
typedef __attribute__((address_space(3))) uint64_t lds_u64;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) float lds_f32;

// A wave appends the `fill` pairs it has queued to their rows' candidate buffers.
__device__ __forceinline__ void append_queue_inline(const lds_u32 *qrow, const lds_u64 *qkey, int fill, int *__restrict__ cnt,
                                                    uint64_t *__restrict__ cand, int cap)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int e = (int)lane_id(); e < fill; e += WAVE) {
        const uint32_t row = qrow[e];
        const int pos = atomicAdd(&cnt[row], 1);
        if (pos < cap) cand[(size_t)row * cap + pos] = qkey[e];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __noinline__ void append_queue(const lds_u32 *qrow, const lds_u64 *qkey, int fill, int *__restrict__ cnt,
                                          uint64_t *__restrict__ cand, int cap)
{
    append_queue_inline(qrow, qkey, fill, cnt, cand, cap);
}

// The rare path of a tile's epilogue (some lane of the wave found a pair under its row's cut-off),
// out of line so that the unrolled test loop stays a handful of instructions per pair.  Called
// with all lanes active; queues the pairs (slots from a ballot) and returns the new fill level.
// ql: the lane's query row within the tile (row qa + ql of X, row qa + ql - q0 of the block).
// A leaf on purpose: a function that calls another one saves its return address through memory.
// qid (or null): the tile's query rows are not consecutive; qid[ql] is the row of the lane's query.
__device__ __noinline__ int queue_pairs(bool near, int j, int ql, int qa, int q0, const lds_f32 *qn, float nj, float dot,
                                        int fill, int qcap, lds_u64 *qkey, lds_u32 *qrow, int *__restrict__ cnt,
                                        uint64_t *__restrict__ cand, int cap, const lds_u32 *qid, int exclude_self,
                                        const int *__restrict__ selfmap)
{
    const int q = qid ? (int)qid[ql] : qa + ql;
    // (selfmap: query q is row selfmap[q] of the database)
    const bool take = near && (!exclude_self || j != (selfmap ? selfmap[q] : q));
    const uint64_t m = __ballot(take);
    if (m == 0) return fill;
    if (fill + WAVE > qcap) { append_queue_inline(qrow, qkey, fill, cnt, cand, cap); fill = 0; }
    if (take) {
        const int slot = fill + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        const float dist = (qn[ql] + nj) - 2.0f * dot;
        qkey[slot] = ((uint64_t)orderable(dist) << 32) | (uint32_t)j;
        qrow[slot] = (uint32_t)(q - q0);
    }
    return fill + __popcll(m);
}

// The first launch of a query block (DENSE): no row has a cut-off yet, so every pair is kept, and its place in the row's
// buffer is its database row's number: no counters, no queue, whole lines.  A pair that no cut-off would take (the row
// itself, a distance that is no finite number) leaves NO_PAIR, which the compaction behind the launch drops; the row's
// count is the launch's width.  (Through the queue every wave of a first slab of 256 rows made 128 trips to memory one
// after the other, each for the answer of an atomic: 1.05 ms of the build of 2000 points, 1.43 -> 0.39 in all;
// 60,000 x 784 21.4 -> 18.7 ms, 512,000 x 50 unchanged, 1,281,167 x 2048 from lists 812 -> 723.)
constexpr uint64_t NO_PAIR = ~0ull;
__device__ __forceinline__ uint64_t dense_pair(float nq, float nj, float dot, bool self, int j)
{
    const bool near = fmaf(-2.0f, dot, nj) < INFINITY && !self;
    return near ? ((uint64_t)orderable((nq + nj) - 2.0f * dot) << 32) | (uint32_t)j : NO_PAIR;
}

// MB x 2 blocks of 32 x 32 per wave, 2 x 2 waves: 64 MB query rows [q0 + 64 MB bx, ..) against 128
// database rows [j0 + 128 by, ..).  MB = 4 (256 x 128) halves the bytes loaded per product, which
// is what bounds the kernel once the matrix cores run at the bf16 rate.
// TWO: two-level accumulation, needed once d exceeds KFLUSH: the matrix cores sum KFLUSH columns
// into `part`, which is then added to `acc` and cleared, so the accumulation error stays that of
// a short sum.  It doubles the accumulator registers, hence MB = 2 there.
// Xb, norms_b: the database rows and their norms (Xs and norms again when the rows are searched among themselves,
// exclude_self = 1: a row is not its own neighbour).
// GATHER: the tiles of an inverted-file search (Eq. (11)) instead of a rectangle of the all-pairs matrix.  The
// rows are in list order (cellptr[L] .. cellptr[L+1] hold list L); the queries of the pass that probe list L at
// the current rank are pairq[pairptr[L] .. pairptr[L+1]) (row numbers, any order); a launch takes the rows
// chunk * DBC .. of every list.  With selfmap query q is row selfmap[q] (a second sweep over some of the rows).  Workgroup t < tptr[nlist] belongs to the list L with tptr[L] <= t < tptr[L+1] and
// is tile (a, b) of its ceil(queries / TQ) x ceil(rows of the chunk / TN) tiles; workgroups past the end leave.
template <int MB, bool TWO, bool GATHER, bool DENSE = false>
__global__ __launch_bounds__(256, 2) void knn_tile_mfma(const uint4 *__restrict__ Xs, int dp, int q0, int qend, int j0,
                                                        int jend, const float *__restrict__ norms,
                                                        const float *__restrict__ tau, int *__restrict__ cnt,
                                                        uint64_t *__restrict__ cand, int cap, int *__restrict__ ccount,
                                                        const uint4 *__restrict__ Xb, const float *__restrict__ norms_b,
                                                        int exclude_self, const int *__restrict__ selfmap,
                                                        const int *__restrict__ tptr, int nlist,
                                                        const int *__restrict__ pairptr, const int *__restrict__ pairq,
                                                        const int *__restrict__ cellptr, int chunk)
{
    static_assert(!TWO || MB == 2, "two-level accumulation has registers for 2 x 2 blocks only");
    constexpr int TQ = 64 * MB;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *ccount = 0;   // for the compaction pass that follows
    __shared__ __align__(16) unsigned char As[TQ * LDS_ROW];
    __shared__ __align__(16) unsigned char Bs[TN * LDS_ROW];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w >> 1, wn = w & 1;
    int qa = q0 + blockIdx.x * TQ, ja = j0 + blockIdx.y * TN;
    int po = 0, nq = TQ;            // GATHER: first entry of pairq and number of queries of this tile
    if (GATHER) {
        const int t = (int)blockIdx.x;
        if (t >= tptr[nlist]) return;
        int lo = 0, hi = nlist;     // tptr[lo] <= t < tptr[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (tptr[mid] <= t) lo = mid; else hi = mid;
        }
        const int nql = pairptr[lo + 1] - pairptr[lo];
        const int rs = min(cellptr[lo] + chunk * DBC, cellptr[lo + 1]), re = min(cellptr[lo + 1], rs + DBC);
        const int tr = max((re - rs + TN - 1) / TN, 1);
        const int a = (t - tptr[lo]) / tr, b = (t - tptr[lo]) % tr;
        po = pairptr[lo] + a * TQ;
        nq = max(min(TQ, nql - a * TQ), 0);
        ja = rs + b * TN;
        jend = min(re, ja + TN);
        qa = 0;
    }
    const int row16 = dp / 4;              // 16-byte pieces per row of Xs
    const int piece = tid & 7, lrow = tid >> 3;
    floatx16 acc[TWO ? MB : 1][TWO ? 2 : 1], part[MB][2];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (TWO) acc[TWO ? a : 0][TWO ? b : 0][i] = 0.f;
                part[a][b][i] = 0.f;
            }
    uint4 ra[2 * MB], rb[4];
    int arow[2 * MB];               // the query rows this thread loads (-1: none)
#pragma unroll
    for (int it = 0; it < 2 * MB; ++it) {
        const int lr = lrow + 32 * it;
        if (GATHER) arow[it] = lr < nq ? (selfmap ? selfmap[max(pairq[po + lr], 0)] : max(pairq[po + lr], 0)) : -1;
        else arow[it] = qa + lr < qend ? qa + lr : -1;
    }
    auto load = [&](int slab) {
#pragma unroll
        for (int it = 0; it < 2 * MB; ++it)
            ra[it] = arow[it] >= 0 ? Xs[(size_t)arow[it] * row16 + slab * 8 + piece] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int r = ja + lrow + 32 * it;
            rb[it] = r < jend ? Xb[(size_t)r * row16 + slab * 8 + piece] : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    load(0);
    const int r32 = lane & 31, h = lane >> 5;
    const int nslab = dp / SLAB;
    for (int slab = 0; slab < nslab; ++slab) {
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 2 * MB; ++it)
            *reinterpret_cast<uint4 *>(As + (lrow + 32 * it) * LDS_ROW + piece * 16) = ra[it];
#pragma unroll
        for (int it = 0; it < 4; ++it)
            *reinterpret_cast<uint4 *>(Bs + (lrow + 32 * it) * LDS_ROW + piece * 16) = rb[it];
        __syncthreads();
        if (slab + 1 < nslab) load(slab + 1);
        // a lane holds 8 consecutive columns of its row for each step of 16: columns 8 h .. 8 h + 7.
        // Both operands use the same assignment, so the products pair up whatever order the
        // hardware sums them in.
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            // low.high, high.high, high.low, in that order so that at most three fragment sets are live
            bf16x8 ah[MB], al[MB], bh[2], bl[2];
            const unsigned char *pa = As + (wm * 32 * MB + r32) * LDS_ROW + ks * 32 + h * 16;
            const unsigned char *pb = Bs + (wn * 64 + r32) * LDS_ROW + ks * 32 + h * 16;
#pragma unroll
            for (int a = 0; a < MB; ++a)
                al[a] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + a * 32 * LDS_ROW + 2 * SLAB));
#pragma unroll
            for (int b = 0; b < 2; ++b)
                bh[b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pb + b * 32 * LDS_ROW));
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    part[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[a], bh[b], part[a][b], 0, 0, 0);
#pragma unroll
            for (int a = 0; a < MB; ++a)
                ah[a] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + a * 32 * LDS_ROW));
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    part[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bh[b], part[a][b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < 2; ++b)
                bl[b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pb + b * 32 * LDS_ROW + 2 * SLAB));
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    part[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bl[b], part[a][b], 0, 0, 0);
        }
        if (TWO && ((slab % (KFLUSH / SLAB)) == (KFLUSH / SLAB) - 1 || slab + 1 == nslab)) {
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        acc[TWO ? a : 0][TWO ? b : 0][i] += part[a][b][i];
                        part[a][b][i] = 0.f;
                    }
        }
    }
    // epilogue: lane holds column (lane % 32) and rows 8 (i / 4) + 4 (lane / 32) + i % 4 of each block.
    // The tile's query norms and cut-offs are staged once in LDS (the slabs are no longer needed).
    // Accepted pairs are few (well under 1 % once the cut-offs have settled), but nearly every wave
    // has some, and an append to a row's buffer is a returning atomic: done where the pair is found,
    // each would stall the wave for a round trip to memory.  So the wave first collects its pairs in
    // an LDS queue (slots from a ballot, no atomics) and appends them all at once, 64 at a time.
    // The test itself is |x|^2 - 2 q.x < cut-off - |q|^2 (one fused multiply-add and one compare per
    // pair); the distance as stored, (|q|^2 + |x|^2) - 2 q.x, is formed for accepted pairs only.
    // Both are within tile_error_coeff() of the exact distance.
    __syncthreads();
    float *qn = reinterpret_cast<float *>(As), *qd = qn + TQ;
    uint32_t *qid = reinterpret_cast<uint32_t *>(qd + TQ);
    for (int t = tid; t < TQ; t += 256) {
        const int q = GATHER ? (t < nq ? max(pairq[po + t], q0) : -1) : (qa + t < qend ? qa + t : -1);
        const float nrm = q >= 0 ? norms[GATHER && selfmap ? selfmap[q] : q] : 0.f;
        qn[t] = nrm;
        qd[t] = q >= 0 ? tau[q - q0] - nrm : -INFINITY;     // rows past the end accept nothing
        if (GATHER) qid[t] = (uint32_t)max(q, 0);
    }
    __syncthreads();
    if (DENSE) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = ja + wn * 64 + b * 32 + r32;
            const float nj = j < jend ? norms_b[j] : INFINITY;
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int ql = wm * 32 * MB + a * 32 + 8 * (i / 4) + 4 * h + i % 4, q = qa + ql;
                    const float dot = TWO ? acc[TWO ? a : 0][TWO ? b : 0][i] : part[a][b][i];
                    if (q < qend && j < jend)
                        cand[(size_t)(q - q0) * cap + (j - j0)] =
                            dense_pair(qn[ql], nj, dot, exclude_self && j == (selfmap ? selfmap[q] : q), j);
                }
        }
        if (blockIdx.y == 0)
            for (int t = tid; t < TQ; t += 256)
                if (qa + t < qend) cnt[qa + t - q0] = jend - j0;
        return;
    }
    constexpr int QCAP = 320;
    static_assert(4 * QCAP * 12 <= TN * LDS_ROW, "the queues live where the database slab was");
    lds_u64 *qkey = (lds_u64 *)(Bs) + w * QCAP;
    lds_u32 *qrow = (lds_u32 *)(Bs + 4 * QCAP * 8) + w * QCAP;
    int fill = 0;       // wave-uniform
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = ja + wn * 64 + b * 32 + r32;
        const float nj = j < jend ? norms_b[j] : INFINITY;    // rows past the end are never closer than any cut-off
#pragma unroll
        for (int a = 0; a < MB; ++a) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const int ql0 = wm * 32 * MB + a * 32 + 8 * i4 + 4 * h;
                const float4 d4 = *reinterpret_cast<const float4 *>(qd + ql0);
                const float dq[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    const int i = 4 * i4 + ii;
                    const float dot = TWO ? acc[TWO ? a : 0][TWO ? b : 0][i] : part[a][b][i];
                    const bool near = fmaf(-2.0f, dot, nj) < dq[ii];
                    if (__ballot(near) != 0)
                        fill = __builtin_amdgcn_readfirstlane(queue_pairs(near, j, ql0 + ii, qa, q0, (const lds_f32 *)qn, nj, dot, fill, QCAP,
                                                                          qkey, qrow, cnt, cand, cap,
                                                                          GATHER ? (const lds_u32 *)qid : (const lds_u32 *)nullptr,
                                                                          exclude_self, selfmap));
                }
            }
        }
    }
    append_queue(qrow, qkey, fill, cnt, cand, cap);
}

// 16-byte piece c of an unpadded 128-byte LDS row r sits at position c ^ swz(r): see knn_tile_resident below
__device__ __forceinline__ int swz(int row) { return ((row >> 1) ^ ((row & 1) << 2)) & 7; }

// ---- the first sweep over long rows: half precision, 256 x 256 tiles
// One product per coordinate makes the operands, not the matrix work, the cost: with 256 x 128 tiles two workgroups
// per compute unit pull 10 TB/s out of the second-level cache.  A 256 x 256 tile needs a third less per product.  One
// workgroup of eight waves per compute unit (a wave owns 128 x 64 outputs, eight 32 x 32 blocks), and the overlap that
// several workgroups would give comes from the kernel itself.  The slabs of 64 columns alternate between two LDS
// buffers, which the loads fill directly (global_load_lds: no registers hold a slab in flight, and no LDS store
// instructions are issued); a wave's instruction brings eight rows of 128 bytes, unpadded, every lane taking the piece
// that the swizzle puts at its position.  There is one barrier per slab, in front of its last step: by then every wave
// has read all it needs of the current buffer, so the loads of the slab after the next go out right behind the barrier
// and have a whole slab's time to arrive, and the first fragments of the next slab are requested while the last
// products of this one run.  Within a step the next step's six fragment reads are placed by hand, one behind each
// of the first six products.  Rows as split_high leaves them (128 bytes per 64 columns); dot_scale undoes their scaling.
// OWN: a workgroup takes all database tiles of the launch for its query tile, one after the other.  With rows of a few
// hundred coordinates a tile is a handful of slabs, and what surrounds them (the first loads, norms, cut-offs, the tests,
// the answers of the appends' atomics), with nothing else on the compute unit, took longer than they did.  Here the next
// tile's first slabs are on their way during the tests of this one, the cut-offs are staged once, and since nobody else
// appends to these rows their fill counts live in LDS, as in knn_tile_resident.  (60,000 x 784: 18.9 -> 14.8 ms for the
// whole build, 400,000 x 300: 252 -> 194.)
// GATHER (knn_tile_half_lists, an OWN kernel): the tiles of an inverted-file search, see knn_tile_mfma.  A workgroup takes up to 256 queries that
// probe one list, and all rows of the chunk of that list; with `dense` set (nobody has a cut-off yet) every pair is kept, at
// the place of its row in the list.  A list that few queries probe leaves the second half of the query tile empty: the
// waves that own it multiply nothing, and the others, which share their SIMDs, go twice as fast.
constexpr int HT = 256;                                 // tile: query rows = database rows
constexpr int HALF_THREADS = 512;
constexpr int HALF_BUF = 2 * HT * 128;                  // one buffer: the tile's query rows, then its database rows
constexpr size_t HALF_TILE_LDS = 2 * (size_t)HALF_BUF;
constexpr size_t HALF_OWN_LDS = HALF_TILE_LDS + 3 * HT * 4;     // and norms, cut-offs and fill counts of the query tile
constexpr size_t HALF_GATHER_LDS = HALF_OWN_LDS + HT * 4;       // and its queries

constexpr int ORD_STEP = DBC / HT;        // tiles a launch takes from a list
static_assert(ORD_STEP == 8, "eight 16-bit numbers are one load");
// The database tiles of every query tile of a block (tile_order_k, tile_rest_k): query tile b has count[b] of them (`all` if
// count is null), tiles[b stride ..], of which the launch takes first .. first + ORD_STEP.  And what the kernel needs to put
// the rows that are due for compaction on the list (the rule of knn_compact_list).
struct TileLists {
    const uint16_t *tiles;
    const int *count;
    int stride, all, first, kp;
    int *clist, *ccount, *ccount_next;
};
// what workgroup b takes of its list: how many tiles, and (tile_numbers) which, two 16-bit numbers a word, wave-uniform
__device__ __forceinline__ int tile_count_of(const TileLists &t, int b)
{
    const int have = t.count ? t.count[b] : t.all;
    return __builtin_amdgcn_readfirstlane(max(min(have - t.first, ORD_STEP), 0));
}
__device__ __forceinline__ uint4 tile_numbers(const TileLists &t, int b)
{
    // (lists start on 16-byte boundaries, `first` is a multiple of eight, and a list has room for whole eights)
    const uint4 v = *reinterpret_cast<const uint4 *>(t.tiles + (size_t)b * t.stride + t.first);
    return make_uint4((uint32_t)__builtin_amdgcn_readfirstlane((int)v.x), (uint32_t)__builtin_amdgcn_readfirstlane((int)v.y),
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)v.z), (uint32_t)__builtin_amdgcn_readfirstlane((int)v.w));
}
// the i-th of them (the last one beyond)
__device__ __forceinline__ int tile_number(uint4 v, int i)
{
    const uint32_t a = i < 4 ? (i < 2 ? v.x : v.y) : (i < 6 ? v.z : v.w);
    return (int)((i & 1) || i >= ORD_STEP ? a >> 16 : a & 0xFFFFu);
}
// a row whose buffer of cap holds c pairs is due for compaction
__device__ __forceinline__ bool compaction_due(int c, float cut, int cap, int kp)
{
    const int cc = min(c, cap);
    return cc >= kp && (!(cut < INFINITY) || cc >= kp + COMPACT_SLACK || cc + COMPACT_EVERY * DBC > cap);
}
// The workgroup puts its rows with `due` on a list whose length is *count, with one atomic operation.  (One a wave: the
// thousand of a launch queue up at the counter: a build of 400,000 x 300 186 -> 181 ms, of 100,000 x 100 16.3 -> 15.9.)
// slot: two ints in LDS that nobody uses any more; all threads call.
__device__ __forceinline__ void list_rows(bool due, int row, int *list, int *count, int *slot)
{
    if (threadIdx.x == 0) slot[0] = 0;
    __syncthreads();
    const int at = due ? atomicAdd(&slot[0], 1) : 0;
    __syncthreads();
    if (threadIdx.x == 0 && slot[0] > 0) slot[1] = atomicAdd(count, slot[0]);
    __syncthreads();
    if (due) list[slot[1] + at] = row;      // any order
}
// where a kernel that has the counts of its rows lists those (their number: the launch's ccount); two lists take turns, `next`
// is the other one's number.  force: also rows with no more than k' and some pairs.  list: null if no pass follows
struct DueRows {
    int *list, *next;
    int kp, force;
};

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void glb_void;

// (No __restrict__ here, the kernels have it: on an inlined function's parameters it makes the compiler wait for the loads
// in flight before every access to LDS that they do not touch.)
template <bool DENSE, bool OWN, bool GATHER, bool SELF>
__device__ __forceinline__ void half_tiles(const uint4 *Xh, int dph, int q0, int qend, int j0, int jend,
                                           const float *norms, const float *tau,
                                           int *cnt, uint64_t *cand, int cap,
                                           int *ccount, float dot_scale, const uint4 *Xb,
                                           const float *norms_b,
                                           const int *tptr, int nlist, const int *pairptr,
                                           const int *pairq, const int *cellptr, int chunk, int dense,
                                           const DueRows &due)
{
    static_assert(!(DENSE && OWN), "a first launch has no counts");
    // SELF: the rows are searched among themselves (known to the compiler: with pointers of their own for the database rows
    // the exact search took 2 % longer)
    static_assert(SELF || !OWN, "the counts of a row");
    const uint4 *Xd = SELF ? Xh : Xb;
    const float *norms_d = SELF ? norms : norms_b;
    static_assert(OWN || !GATHER, "nobody else appends to a gathered query's buffer");
    // for the compaction pass that follows (OWN and not GATHER: for the next launch's, this one's rows are listed here)
    if (blockIdx.x == 0 && threadIdx.x == 0) *(OWN && !GATHER ? due.next : ccount) = 0;
    extern __shared__ __align__(16) unsigned char hsm[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w >> 2, wn = w & 3;
    // Workgroups go to the eight XCDs in turn, and each XCD has a second-level cache of its own.  Workgroup number
    // 8 l + x is XCD x's l-th: XCD x takes a strip of the query tiles and walks it query tile by query tile, all
    // database tiles of one query tile next to each other, so that the 32 workgroups an XCD runs at a time are a few
    // query tiles against all database tiles of the launch and find each other's rows in that cache (taken in plain
    // row-major order, every tile's rows came from memory: 3-4 TB/s of re-reads, which is what bounded the kernel).
    int po = 0, nq = HT;            // GATHER: first entry of pairq and number of queries of this tile
    if (GATHER) {
        const int t = (int)blockIdx.x;
        if (t >= tptr[nlist]) return;
        int lo = 0, hi = nlist;     // tptr[lo] <= t < tptr[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (tptr[mid] <= t) lo = mid; else hi = mid;
        }
        const int a = t - tptr[lo], nql = pairptr[lo + 1] - pairptr[lo];
        j0 = min(cellptr[lo] + chunk * DBC, cellptr[lo + 1]);
        jend = min(cellptr[lo + 1], j0 + DBC);
        po = pairptr[lo] + a * HT;
        nq = min(HT, nql - a * HT);
        if (nq <= 0 || jend <= j0) return;      // (no such tile is counted)
    }
    const int nqt = (qend - q0 + HT - 1) / HT, njt = (jend - j0 + HT - 1) / HT, per = (nqt + 7) / 8;
    const int xcd = (int)(blockIdx.x & 7u), local = (int)(blockIdx.x >> 3);
    // (OWN: workgroup = query tile)
    const int qt = GATHER ? 0 : OWN ? (int)blockIdx.x : xcd * per + local / njt, jt = OWN ? 0 : local % njt;
    if (qt >= nqt || (!OWN && local / njt >= per)) return;     // (the grid is 8 per njt workgroups; the same for all lanes)
    const int qa = q0 + qt * HT;
    int ja = j0 + jt * HT;
    const int total = (OWN ? njt : 1) * (dph / (2 * SLAB));     // slabs of all tiles
    const int row16 = dph / 8;              // 16-byte pieces per row
    const int r32 = lane & 31, h = lane >> 5;
    const int nslab = dph / (2 * SLAB);
    floatx16 acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
    // What this lane loads: wave w brings rows 32 w .. 32 w + 31 of both operands, eight rows an instruction; the
    // lane's row is 8 it + lane / 8 of them and its LDS position lane % 8, so it reads piece (lane % 8) ^ swz(row).
    // A row past the end is read as the last row: its products are finite and the epilogue accepts nothing for it.
    const uint4 *ga[4], *gb[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int lr = 32 * w + 8 * it + (lane >> 3), c = (lane & 7) ^ swz(lr);
        ga[it] = Xh + (size_t)(GATHER ? max(pairq[po + min(lr, nq - 1)], 0) : min(qa + lr, qend - 1)) * row16 + c;
        gb[it] = Xd + (size_t)min(ja + lr, jend - 1) * row16 + c;
    }
    // the slab that is loaded next: number lslab of the tile of database rows at lja
    int lslab = 0, lja = ja;
    auto load_next = [&]() {
        if (++lslab < nslab) return;
        lslab = 0;
        lja += HT;
        if (OWN) {
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int lr = 32 * w + 8 * it + (lane >> 3), c = (lane & 7) ^ swz(lr);
                gb[it] = Xd + (size_t)min(lja + lr, jend - 1) * row16 + c;
            }
        }
    };
#define HALF_LOAD(slab_, buf_)                                                             \
    _Pragma("unroll") for (int it = 0; it < 4; ++it) {                                     \
        unsigned char *d_ = hsm + (size_t)(buf_) * HALF_BUF + (32 * w + 8 * it) * 128;     \
        __builtin_amdgcn_global_load_lds((glb_void *)(ga[it] + (size_t)(slab_) * 8), (lds_void *)d_, 16, 0, 0);              \
        __builtin_amdgcn_global_load_lds((glb_void *)(gb[it] + (size_t)(slab_) * 8), (lds_void *)(d_ + HT * 128), 16, 0, 0); \
    }
    // fragments: lane (r32, h) of block a reads piece 2 ks + h of row 32 a + r32 (swz depends on r32 alone)
    const int sw = swz(r32);
    const int fa_off = (wm * 128 + r32) * 128, fb_off = (HT + wn * 64 + r32) * 128;
    int pk[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) pk[ks] = ((2 * ks + h) ^ sw) * 16;
    halfx8 fa[2][4], fb[2][2];
#define HALF_FRAGS(buf_, ks_, set_)                                                        \
    {                                                                                      \
        const unsigned char *b_ = hsm + (size_t)(buf_) * HALF_BUF + pk[ks_];               \
        _Pragma("unroll") for (int a = 0; a < 4; ++a)                                      \
            fa[set_][a] = __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4 *>(b_ + fa_off + a * 32 * 128)); \
        _Pragma("unroll") for (int b = 0; b < 2; ++b)                                      \
            fb[set_][b] = __builtin_bit_cast(halfx8, *reinterpret_cast<const uint4 *>(b_ + fb_off + b * 32 * 128)); \
    }
#define HALF_PRODUCTS(set_)                                                                \
    _Pragma("unroll") for (int a = 0; a < 4; ++a)                                          \
        _Pragma("unroll") for (int b = 0; b < 2; ++b)                                      \
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[set_][a], fb[set_][b], acc[a][b], 0, 0, 0);
#define HALF_INTERLEAVE()                                                                  \
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);         /* one matrix product */     \
    _Pragma("unroll") for (int i_ = 0; i_ < 6; ++i_) {                                     \
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     /* one LDS read */           \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                 \
    }                                                                                      \
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    float *own_n = reinterpret_cast<float *>(hsm + HALF_TILE_LDS), *own_d = own_n + HT;
    int *own_c = reinterpret_cast<int *>(own_d + HT), *own_q = own_c + HT;
    const bool idle = GATHER && wm * 128 >= nq;
    if (OWN) {
        for (int t = tid; t < HT; t += HALF_THREADS) {
            const bool in = GATHER ? t < nq : qa + t < qend;
            const int q = !in ? -1 : GATHER ? max(pairq[po + t], q0) : qa + t;
            const float nrm = in ? norms[q] : 0.f;
            own_n[t] = nrm;
            own_d[t] = in ? tau[q - q0] - nrm : -INFINITY;     // rows past the end accept nothing
            own_c[t] = in ? cnt[q - q0] : 0;
            if (GATHER) own_q[t] = in ? q - q0 : 0;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    HALF_LOAD(lslab, 0)
    load_next();
    if (total > 1) {
        HALF_LOAD(lslab, 1)
        load_next();
    }
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");     // (the first slab; all of them if there is only one)
    if (total == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (!idle) HALF_FRAGS(0, 0, 0)
    int slab = 0;
    float njn[2] = {0.f, 0.f};
    for (int flat = 0; flat < total; ++flat) {
        const int cur = flat & 1, oth = cur ^ 1;
        if (OWN && slab == 0) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int j = ja + wn * 64 + b * 32 + r32;
                njn[b] = norms_d[min(j, jend - 1)];
            }
        }
        if (!idle) {
            HALF_FRAGS(cur, 1, 1)
            HALF_PRODUCTS(0)
            HALF_INTERLEAVE()
            __builtin_amdgcn_sched_barrier(0);
            HALF_FRAGS(cur, 2, 0)
            HALF_PRODUCTS(1)
            HALF_INTERLEAVE()
            __builtin_amdgcn_sched_barrier(0);
            HALF_FRAGS(cur, 3, 1)
            HALF_PRODUCTS(0)
            HALF_INTERLEAVE()
            __builtin_amdgcn_sched_barrier(0);
        }
        // this wave's part of the next slab has arrived (OWN: so have the norms, which the compiler has to see)
        if (OWN) __builtin_amdgcn_s_waitcnt(0x0F70);
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();        // the other buffer is complete; nobody reads this one any more
        __builtin_amdgcn_sched_barrier(0);
        if (flat + 2 < total) {
            HALF_LOAD(lslab, cur)
            load_next();
        }
        // (past the last slab these fragments are read from a buffer nobody fills any more, and never used)
        if (!idle) {
            HALF_FRAGS(oth, 0, 0)
            HALF_PRODUCTS(1)
            HALF_INTERLEAVE()
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!OWN || ++slab < nslab) continue;
        if (idle) { slab = 0; ja += HT; continue; }
        // (one base per lane, the rest compile-time offsets)
        int lbase = wm * 128 + 4 * h;
        asm volatile("" : "+v"(lbase));
        const float *qd_l = own_d + lbase, *qn_l = own_n + lbase;
        int *qc_l = own_c + lbase;
        const int *qq_l = own_q + lbase;
        if (GATHER && dense) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int j = ja + wn * 64 + b * 32 + r32;
                const float nj = j < jend ? njn[b] : INFINITY;
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int off = a * 32 + 8 * (i / 4) + i % 4, q = qq_l[off];
                        if (lbase + off < nq && j < jend)
                            cand[(size_t)q * cap + (j - j0)] = dense_pair(qn_l[off], nj, acc[a][b][i] * dot_scale, j == q0 + q, j);
                        acc[a][b][i] = 0.f;
                        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);      // (four addresses at a time: there are no registers for 64)
                    }
            }
            slab = 0;
            ja += HT;
            continue;
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = ja + wn * 64 + b * 32 + r32;
            const float nj = j < jend ? njn[b] : INFINITY;      // rows past the end are never closer than any cut-off
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const float4 d4 = *reinterpret_cast<const float4 *>(qd_l + a * 32 + 8 * i4);
                    const float dq[4] = {d4.x, d4.y, d4.z, d4.w};
                    bool near[4];
#pragma unroll
                    for (int ii = 0; ii < 4; ++ii) near[ii] = fmaf(-2.0f * dot_scale, acc[a][b][4 * i4 + ii], nj) < dq[ii];
                    if (__builtin_expect(__ballot(near[0] || near[1] || near[2] || near[3]) != 0, 0)) {
#pragma unroll
                        for (int ii = 0; ii < 4; ++ii) {
                            const int off = a * 32 + 8 * i4 + ii, q = GATHER ? q0 + qq_l[off] : qa + lbase + off;
                            if (near[ii] && (j != q)) {
                                const float dist = (qn_l[off] + nj) - 2.0f * (acc[a][b][4 * i4 + ii] * dot_scale);
                                const int pos = atomicAdd(qc_l + off, 1);
                                if (pos < cap)
                                    cand[(size_t)(q - q0) * cap + pos] = ((uint64_t)orderable(dist) << 32) | (uint32_t)j;
                            }
                        }
                    }
#pragma unroll
                    for (int ii = 0; ii < 4; ++ii) acc[a][b][4 * i4 + ii] = 0.f;
                }
        }
        slab = 0;
        ja += HT;
    }
    __syncthreads();            // (the epilogue reuses the buffers)
    if (OWN) {
        static_assert(HALF_THREADS >= HT, "a thread a row");
        if (GATHER) {
            if (tid < nq) cnt[own_q[tid]] = dense ? jend - j0 : own_c[tid];
        } else {
            // (by the rule of knn_compact_list, whose launch behind every second one this saves)
            const bool in = tid < HT && qa + tid < qend;
            const int c = in ? own_c[tid] : 0;
            if (in) cnt[qa + tid - q0] = c;
            if (due.list)
                list_rows(in && (compaction_due(c, own_d[min(tid, HT - 1)], cap, due.kp) || (due.force && min(c, cap) >= due.kp)),
                          qa + tid - q0, due.list, ccount, reinterpret_cast<int *>(own_n));
        }
        return;
    }
#undef HALF_LOAD
#undef HALF_FRAGS
#undef HALF_PRODUCTS
#undef HALF_INTERLEAVE
    // epilogue, as in knn_tile_mfma: lane holds column (lane % 32) and rows 8 (i / 4) + 4 (lane / 32) + i % 4 of each
    // block; norms and cut-offs of the tile's queries staged in LDS, accepted pairs queued per wave
    float *qn = reinterpret_cast<float *>(hsm), *qd = qn + HT;
    for (int t = tid; t < HT; t += HALF_THREADS) {
        const int q = qa + t < qend ? qa + t : -1;
        const float nrm = q >= 0 ? norms[q] : 0.f;
        qn[t] = nrm;
        qd[t] = q >= 0 ? tau[q - q0] - nrm : -INFINITY;     // rows past the end accept nothing
    }
    __syncthreads();
    if (DENSE) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = ja + wn * 64 + b * 32 + r32;
            const float nj = j < jend ? norms_d[j] : INFINITY;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int ql = wm * 128 + a * 32 + 8 * (i / 4) + 4 * h + i % 4, q = qa + ql;
                    if (q < qend && j < jend)
                        cand[(size_t)(q - q0) * cap + (j - j0)] = dense_pair(qn[ql], nj, acc[a][b][i] * dot_scale, SELF && j == q, j);
                }
        }
        if (jt == 0)
            for (int t = tid; t < HT; t += HALF_THREADS)
                if (qa + t < qend) cnt[qa + t - q0] = jend - j0;
        return;
    }
    constexpr int QCAP = 320;
    unsigned char *qbase = hsm + 4096;
    lds_u64 *qkey = (lds_u64 *)(qbase) + w * QCAP;
    lds_u32 *qrow = (lds_u32 *)(qbase + 8 * QCAP * 8) + w * QCAP;
    int fill = 0;       // wave-uniform
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = ja + wn * 64 + b * 32 + r32;
        const float nj = j < jend ? norms_d[j] : INFINITY;    // rows past the end are never closer than any cut-off
#pragma unroll
        for (int a = 0; a < 4; ++a) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const int ql0 = wm * 128 + a * 32 + 8 * i4 + 4 * h;
                const float4 d4 = *reinterpret_cast<const float4 *>(qd + ql0);
                const float dq[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    const float dot = acc[a][b][4 * i4 + ii] * dot_scale;
                    const bool near = fmaf(-2.0f, dot, nj) < dq[ii];
                    if (__ballot(near) != 0)
                        fill = __builtin_amdgcn_readfirstlane(queue_pairs(near, j, ql0 + ii, qa, q0, (const lds_f32 *)qn, nj, dot, fill, QCAP,
                                                                          qkey, qrow, cnt, cand, cap, (const lds_u32 *)nullptr, SELF ? 1 : 0,
                                                                          (const int *)nullptr));
                }
            }
        }
    }
    append_queue(qrow, qkey, fill, cnt, cand, cap);
}

template <bool DENSE, bool OWN>
__global__ __launch_bounds__(HALF_THREADS, 1) void knn_tile_half(const uint4 *__restrict__ Xh, int dph, int q0, int qend, int j0,
                                                                 int jend, const float *__restrict__ norms,
                                                                 const float *__restrict__ tau, int *__restrict__ cnt,
                                                                 uint64_t *__restrict__ cand, int cap, int *__restrict__ ccount,
                                                                 float dot_scale, DueRows due)
{
    half_tiles<DENSE, OWN, false, true>(Xh, dph, q0, qend, j0, jend, norms, tau, cnt, cand, cap, ccount, dot_scale, nullptr, nullptr,
                                        nullptr, 0, nullptr, nullptr, nullptr, 0, 0, due);
}

// Against other rows (centroids, pivots): Xb, norms_b.
template <bool DENSE>
__global__ __launch_bounds__(HALF_THREADS, 1) void knn_tile_half_other(const uint4 *__restrict__ Xh, int dph, int q0, int qend, int j0,
                                                                       int jend, const float *__restrict__ norms,
                                                                       const float *__restrict__ tau, int *__restrict__ cnt,
                                                                       uint64_t *__restrict__ cand, int cap,
                                                                       int *__restrict__ ccount, float dot_scale,
                                                                       const uint4 *__restrict__ Xb, const float *__restrict__ norms_b)
{
    half_tiles<DENSE, false, false, false>(Xh, dph, q0, qend, j0, jend, norms, tau, cnt, cand, cap, ccount, dot_scale, Xb, norms_b,
                                           nullptr, 0, nullptr, nullptr, nullptr, 0, 0, DueRows{});
}

__global__ __launch_bounds__(HALF_THREADS, 1) void knn_tile_half_lists(const uint4 *__restrict__ Xh, int dph, int q0, int qend,
                                                                       const float *__restrict__ norms,
                                                                       const float *__restrict__ tau, int *__restrict__ cnt,
                                                                       uint64_t *__restrict__ cand, int cap,
                                                                       int *__restrict__ ccount, float dot_scale,
                                                                       const int *__restrict__ tptr, int nlist,
                                                                       const int *__restrict__ pairptr,
                                                                       const int *__restrict__ pairq,
                                                                       const int *__restrict__ cellptr, int chunk, int dense)
{
    half_tiles<false, true, true, true>(Xh, dph, q0, qend, 0, 0, norms, tau, cnt, cand, cap, ccount, dot_scale, nullptr, nullptr, tptr, nlist,
                                  pairptr, pairq, cellptr, chunk, dense, DueRows{});
}

// ---- d <= 64: the query tile stays in LDS
// With two slabs at most, the kernel above spends its time waiting: a workgroup makes five
// dependent round trips to memory (two slabs, norms and cut-offs, the appends) around 2 x 48 matrix
// instructions.  Here a workgroup keeps its 256 query rows on chip for the whole launch (each
// wave holds the fragments of its 64 rows in registers) and walks over the database rows; the
// next rows are in flight (registers) while the current ones are multiplied and tested.  The
// workgroup is the only one that appends to its rows' buffers during the launch, so the fill
// counts live in LDS: an append is an LDS atomic and a store that nobody waits for.
// Eight waves in two groups of four: each group takes every other tile of 128 database rows, in
// two halves of 64; a wave holds 64 x 64 of its group's 256 x 64 products.  Group 0 multiplies a
// half and then tests it, group 1 tests its previous half first and then multiplies the next, so
// that on every SIMD one wave feeds the matrix cores while the other one runs the tests on the
// vector unit.  (Two halves per trip: one half's work is shorter than a load takes to arrive.)
// LDS rows are 128 bytes (32 high parts, 32 low parts), unpadded; the 16-byte piece c of row r sits
// at position c ^ swz(r), chosen so that 16 consecutive rows' reads of one piece fall on 16
// different 16-byte bank groups of a 256-byte LDS line (and 8 consecutive rows on 8 of a
// 128-byte line), while the 8 pieces of a row stay a permutation of the row.
constexpr int RQ = 256;          // query rows per workgroup
constexpr int RT = 128;          // database rows per group and trip, taken in two halves
constexpr int RESIDENT_MIN_ROWS = 64 * RQ;   // fewer query rows than this leave most compute units without a workgroup

constexpr size_t resident_lds_bytes(int ns)
{
    return 2 * (size_t)ns * RT * SLAB_ROW + 3 * RQ * 4;
}


// A workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every global
// store of the wave to complete, which would put the appends' trip to memory on the critical path.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ORDER: not all tiles from j0 to jend but those on the query tile's list, see tile_order_k; a launch takes ORD_STEP of them.
// DENSE is then every pair at the place of its tile in the launch and its row in the tile.
template <int NS, bool DENSE, bool ORDER>
__global__ __launch_bounds__(512, 1) void knn_tile_resident(const uint4 *__restrict__ Xs, int q0, int qend, int j0, int jend,
                                                            const float *__restrict__ norms,
                                                            const float *__restrict__ tau, int *__restrict__ cnt,
                                                            uint64_t *__restrict__ cand, int cap, int kp, int force,
                                                            int *__restrict__ clist, int *__restrict__ ccount,
                                                            int *__restrict__ ccount_next, TileLists lists)
{
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *Bs = smem;                                   // [2 groups][NS][RT] rows
    float *qn = reinterpret_cast<float *>(Bs + 2 * NS * RT * SLAB_ROW), *qd = qn + RQ;
    int *qc = reinterpret_cast<int *>(qd + RQ);                 // candidates in each row's buffer
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int g = w >> 2, wq = w & 3;
    const int r32 = lane & 31, h = lane >> 5, sw = swz(r32);
    const int per = ((qend - q0 + RQ - 1) / RQ + 7) / 8;
    const int qt = ORDER ? (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    if (blockIdx.x == 0 && tid == 0) *ccount_next = 0;   // the list of the next launch (nobody reads it any more)
    uint4 nos = make_uint4(0u, 0u, 0u, 0u);
    int nmine = 0;
    if (ORDER) {
        if ((int)(blockIdx.x >> 3) >= per || q0 + qt * RQ >= qend) return;       // (the grid is 8 per workgroups)
        nmine = tile_count_of(lists, qt);
        if (nmine == 0) return;
        nos = tile_numbers(lists, qt);
    }
    const int qa = q0 + qt * RQ;
    constexpr int row16 = NS * 8;          // 16-byte pieces per row of Xs
    // the wave's query fragments: [block][slab][step] high and low parts, as the matrix cores take them
    bf16x8 afh[2][NS][2], afl[2][NS][2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int r = qa + wq * 64 + a * 32 + r32;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const uint4 z = make_uint4(0u, 0u, 0u, 0u);
                afh[a][sl][ks] = __builtin_bit_cast(bf16x8, r < qend ? Xs[(size_t)r * row16 + sl * 8 + 2 * ks + h] : z);
                afl[a][sl][ks] = __builtin_bit_cast(bf16x8, r < qend ? Xs[(size_t)r * row16 + sl * 8 + 4 + 2 * ks + h] : z);
            }
    }
    for (int t = tid; t < RQ; t += 512) {
        const int q = qa + t;
        const float nq = q < qend ? norms[q] : 0.f;
        qn[t] = nq;
        qd[t] = q < qend ? tau[q - q0] - nq : -INFINITY;     // rows past the end accept nothing
        qc[t] = q < qend ? cnt[q - q0] : 0;
    }
    unsigned char *Bg = Bs + g * NS * RT * SLAB_ROW;
    const int bpiece = tid & 7, blrow = (tid & 255) >> 3;
    const int ntile = (jend - j0 + RT - 1) / RT, npair = ORDER ? nmine : (ntile + 1) / 2;
    // first database row of a trip (ORDER: two of this kernel's tiles are one of the lists')
    auto trip_base = [=](int pair) { return ORDER ? tile_number(nos, pair) * HT : j0 + 2 * pair * RT; };
    uint4 rb[4 * NS];
    float njn[2][2];   // |x|^2 of this lane's two columns of each half of the tile in rb
    auto load_tile = [&](int pair) {
        const int ja = trip_base(pair) + g * RT;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int r = ja + blrow + 32 * it;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl)
                rb[it * NS + sl] = r < jend ? Xs[(size_t)r * row16 + sl * 8 + bpiece] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int j = ja + hf * 64 + b * 32 + r32;
                njn[hf][b] = j < jend ? norms[j] : INFINITY;    // rows past the end are never closer than any cut-off
            }
    };
    floatx16 part[2][2];
    float njc[2] = {INFINITY, INFINITY};   // the same for the half in `part`
    int jac = j0, place = 0;               // first database row of that half, and its place in a dense launch
    auto test_tile = [&]() {
        // one base per lane, the rest compile-time offsets (and no addresses carried around the loop)
        int lbase = wq * 64 + 4 * h;
        asm volatile("" : "+v"(lbase));
        const float *qd_l = qd + lbase, *qn_l = qn + lbase;
        int *qc_l = qc + lbase;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = jac + b * 32 + r32;
            const float nj = njc[b];
            if (DENSE) {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int off = a * 32 + 8 * (i / 4) + i % 4, q = qa + lbase + off;
                        // (ORDER: a row past the end leaves no pair, at its place)
                        if (q < qend && (ORDER || j < jend))
                            cand[(size_t)(q - q0) * cap + (ORDER ? place + b * 32 + r32 : j - j0)] = dense_pair(qn_l[off], nj, part[a][b][i], j == q, j);
                    }
                continue;
            }
#pragma unroll
            for (int a = 0; a < 2; ++a) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const float4 d4 = *reinterpret_cast<const float4 *>(qd_l + a * 32 + 8 * i4);
                    const float dq[4] = {d4.x, d4.y, d4.z, d4.w};
                    // four pairs per branch: a branch on a vector compare waits for the compare, and that
                    // wait, not the arithmetic, is what a test costs (sixteen per branch: slower again,
                    // the rare path is entered too often)
                    bool near[4];
#pragma unroll
                    for (int ii = 0; ii < 4; ++ii) near[ii] = fmaf(-2.0f, part[a][b][4 * i4 + ii], nj) < dq[ii];
                    if (__builtin_expect(__ballot(near[0] || near[1] || near[2] || near[3]) != 0, 0)) {
#pragma unroll
                        for (int ii = 0; ii < 4; ++ii) {
                            if (__ballot(near[ii]) == 0) continue;
                            const float dot = part[a][b][4 * i4 + ii];
                            const int off = a * 32 + 8 * i4 + ii;
                            const int q = qa + lbase + off;
                            if (near[ii] && j != q) {
                                const float dist = (qn_l[off] + nj) - 2.0f * dot;
                                const int pos = atomicAdd(qc_l + off, 1);
                                if (pos < cap)
                                    cand[(size_t)(q - q0) * cap + pos] = ((uint64_t)orderable(dist) << 32) | (uint32_t)j;
                            }
                        }
                    }
                }
            }
        }
    };
    if (npair > 0) load_tile(0);
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bool have = false;      // group 1: `part` holds a half that has not been tested yet
    for (int pair = 0; pair < npair; ++pair) {
        lds_barrier();          // every wave is done with the tiles in LDS (first trip: the query rows are in)
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = blrow + 32 * it;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl)
                *reinterpret_cast<uint4 *>(Bg + (sl * RT + row) * SLAB_ROW + ((bpiece ^ swz(row)) << 4)) = rb[it * NS + sl];
        }
        const float njl[2][2] = {{njn[0][0], njn[0][1]}, {njn[1][0], njn[1][1]}};
        lds_barrier();
        // the next rows are requested after the first tests of this trip: a wait for them (the counter
        // is in order) then never covers stores made by tests, except those of the half in between
        for (int hf = 0; hf < 2; ++hf) {
            if (g == 1 && have) test_tile();
            if (hf == 0 && pair + 1 < npair) load_tile(pair + 1);
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    // low.high, high.low, high.high; piece index = 4 (low part) + 2 ks + h
                    bf16x8 bh[2], bl[2];
                    const unsigned char *pb = Bg + (sl * RT + hf * 64 + r32) * SLAB_ROW;
                    const int ch = ((2 * ks + h) ^ sw) << 4, cl = ((4 + 2 * ks + h) ^ sw) << 4;
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        bh[b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pb + b * 32 * SLAB_ROW + ch));
                        bl[b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pb + b * 32 * SLAB_ROW + cl));
                    }
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            part[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afl[a][sl][ks], bh[b],
                                                                                 (sl == 0 && ks == 0) ? zero16 : part[a][b], 0, 0, 0);
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            part[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afh[a][sl][ks], bl[b], part[a][b], 0, 0, 0);
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
                            part[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afh[a][sl][ks], bh[b], part[a][b], 0, 0, 0);
                }
            }
            njc[0] = njl[hf][0];
            njc[1] = njl[hf][1];
            jac = trip_base(pair) + g * RT + hf * 64;
            place = (2 * pair + g) * RT + hf * 64;
            have = true;
            if (g == 0) test_tile();
        }
    }
    if (g == 1 && have) test_tile();
    lds_barrier();
    // the fill counts go back, and the rows whose buffers are due for compaction go on the list (the
    // rule of knn_compact_list, which this kernel makes unnecessary)
    const int q = qa + tid;
    const bool in = tid < RQ && q < qend;
    const int c = !in ? 0 : DENSE ? (ORDER ? nmine * HT : jend - j0) : qc[tid];
    if (in) cnt[q - q0] = c;
    if (clist)                  // (null: no pass follows)
        list_rows(in && (compaction_due(c, qd[min(tid, RQ - 1)], cap, kp) || (force && min(c, cap) >= kp)), q - q0, clist, ccount,
                  reinterpret_cast<int *>(qn));
}

// Which rows of the query block need their candidates compacted now (one thread per row; the
// compaction itself takes a workgroup per row, and on most slabs only a few rows need it).
__global__ __launch_bounds__(256) void knn_compact_list(const float *__restrict__ tau, const int *__restrict__ cnt,
                                                        int cap, int kp, int rows, int force, int *__restrict__ list,
                                                        int *__restrict__ count)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= rows) return;
    int c = cnt[row];
    if (c > cap) c = cap;
    if (c < kp) return;                 // not yet k' candidates: the cut-off stays +inf
    // sort only when enough new candidates have piled up to matter, when the next slab could
    // overflow the buffer, or at the end (force); in between the cut-off is merely a bit stale
    if (!force && tau[row] < INFINITY && c < kp + COMPACT_SLACK && c + COMPACT_EVERY * DBC <= cap) return;
    list[atomicAdd(count, 1)] = row;    // any order
}

// One wave per listed row: keeps the best k' of the row's candidates (in any order) and lowers the cut-off to the k'-th.
// Nobody needs them sorted, so the k'-th distance is found by halving the range of the keys' 32 distance bits: a lane holds
// R pairs in registers, a step is R compares, and a step that leaves exactly k' pairs below the middle ends the search
// (some ten steps for a few hundred pairs).  No LDS, no barriers: 32 rows in flight per compute unit.  (A bitonic sort of
// the row in LDS by two waves, 45 exchange stages with a barrier each: with it
// tsne_build_P took 329 ms for 400,000 x 300 and 262 ms for 512,000 x 50, without 297 and 224.)
// A longer buffer (the first slabs of a query block) goes through the registers in several rounds, each keeping the best
// k' so far.
template <int R>
__global__ __launch_bounds__(256) void knn_compact(float *__restrict__ tau, int *__restrict__ cnt, uint64_t *__restrict__ cand,
                                                   int cap, int kp, int rows, const int *__restrict__ list,
                                                   const int *__restrict__ count)
{
    const int m = min(*count, rows), lane = (int)lane_id();
    for (int i = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); i < m; i += (int)gridDim.x * 4) {
        const int row = __builtin_amdgcn_readfirstlane(min(max(list[i], 0), rows - 1));
        int c = __builtin_amdgcn_readfirstlane(cnt[row]);
        // (more pairs than the buffer holds cannot arrive between two passes as the launches are sized; should it
        // happen all the same, pairs were dropped: the cut-off goes to -inf for good, which fails the row's certificate)
        const bool lost = c > cap || tau[row] == -INFINITY;
        if (c > cap) c = cap;
        uint64_t *buf = cand + (size_t)row * cap;
        int done = 0, have = 0;         // pairs read so far; survivors in buf[0 .. have)
        uint32_t kth = 0;               // the survivors' largest distance
        constexpr uint32_t NONE = 0xFFFFFFFFu;      // NO_PAIR's distance
        while (done < c) {
            const int take = min(WAVE * R - have, c - done), total = have + take;
            uint64_t v[R];
            uint32_t lo = NONE, hi = 0u;
            int valid = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int e = lane + WAVE * r;
                // (read whatever it is: 32 loads each behind a branch took nearly twice as long)
                const uint64_t got = buf[min(e < have ? e : done + (e - have), c - 1)];
                v[r] = e < total ? got : NO_PAIR;
                const uint32_t d = (uint32_t)(v[r] >> 32);
                valid += (int)__popcll(__ballot(d != NONE));
                lo = min(lo, d);
                if (d != NONE) hi = max(hi, d);
            }
#pragma unroll
            for (int o = WAVE / 2; o > 0; o >>= 1) {
                lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, WAVE));
                hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, WAVE));
            }
            lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
            hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
            done += take;
            // smallest hi with at least k' distances <= hi; `all`: exactly k' are
            bool all = valid <= kp;
            int under = 0, upto = valid;        // how many are below lo, and up to hi
            if (R >= 16 && kp <= WAVE && !all) {
                // few of many: the k'-th smallest of the lanes' smallest is as far as the k'-th of all can be
                uint32_t least = NONE, a = lo, b = hi;
#pragma unroll
                for (int r = 0; r < R; ++r) least = min(least, (uint32_t)(v[r] >> 32));
                while (a < b) {
                    const uint32_t mid = a + ((b - a) >> 1);
                    if ((int)__popcll(__ballot(least <= mid)) >= kp) b = mid; else a = mid + 1;
                }
                hi = b;
                upto = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) upto += (int)__popcll(__ballot((uint32_t)(v[r] >> 32) <= hi));
                all = upto == kp;
            }
            // every other step splits the range where the counts at its ends say, the others halve it
            for (int step = 0; lo < hi && !all; ++step) {
                uint32_t cut = (hi - lo) >> 1;
                if (step % 2 == 0) cut = min((uint32_t)((float)(hi - lo) * ((float)(kp - under) / (float)(upto - under))), hi - lo - 1u);
                const uint32_t mid = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lo + cut));     // (below hi)
                int below = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) below += (int)__popcll(__ballot((uint32_t)(v[r] >> 32) <= mid));
                if (below >= kp) { hi = mid; upto = below; } else { lo = mid + 1; under = below; }
                all = below == kp;
            }
            int ties = kp;              // how many of the distances equal to hi are kept
            if (!all) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    ties -= (int)__popcll(__ballot((uint32_t)(v[r] >> 32) < hi));
            }
            int pos = 0;
            uint32_t top = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t d = (uint32_t)(v[r] >> 32);
                const bool eq = d == hi;            // (hi is a pair's distance or lies between two, below NONE)
                const uint64_t meq = __ballot(eq);
                const bool keep = d < hi ||
                                  (eq && (all || (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(meq >> 32),
                                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)meq, 0u)) < ties));
                if (!all) ties -= (int)__popcll(meq);
                const uint64_t mk = __ballot(keep);
                if (mk == 0) continue;
                if (keep) {
                    buf[pos + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u))] = v[r];
                    top = max(top, d);
                }
                pos += (int)__popcll(mk);
            }
#pragma unroll
            for (int o = WAVE / 2; o > 0; o >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, o, WAVE));
            kth = top;
            have = pos;
            __threadfence_block();      // (the next round reads what other lanes wrote)
        }
        if (lane == 0) {
            cnt[row] = have;
            tau[row] = lost ? -INFINITY : have >= kp ? unorderable(kth) : tau[row];
        }
    }
}

// (beside k' survivors a round takes in 192 new pairs at least: 512 - 320, 1024 - 832, 4096 - 1920; an ordinary pass has
// some COMPACT_SLACK of them, one or two rounds)
// dense: the pairs of a row behind a first launch (at most DBC), 0 behind others
static void launch_compact(float *tau, int *cnt, uint64_t *cand, int cap, int kp, int rows, const int *list, const int *count,
                           int dense, hipStream_t s)
{
    const dim3 grid((unsigned)((rows < 8192 ? rows : 8192) + 3) / 4);
    if (dense > 1536 && kp <= 832)
        hipLaunchKernelGGL(knn_compact<DBC / WAVE>, grid, dim3(256), 0, s, tau, cnt, cand, cap, kp, rows, list, count);
    else if (dense > 1024 && kp <= 832)
        hipLaunchKernelGGL(knn_compact<24>, grid, dim3(256), 0, s, tau, cnt, cand, cap, kp, rows, list, count);
    else if (dense > 0 && kp <= 832)
        hipLaunchKernelGGL(knn_compact<16>, grid, dim3(256), 0, s, tau, cnt, cand, cap, kp, rows, list, count);
    else if (kp <= 320)
        hipLaunchKernelGGL(knn_compact<8>, grid, dim3(256), 0, s, tau, cnt, cand, cap, kp, rows, list, count);
    else if (kp <= 832)
        hipLaunchKernelGGL(knn_compact<16>, grid, dim3(256), 0, s, tau, cnt, cand, cap, kp, rows, list, count);
    else
        hipLaunchKernelGGL(knn_compact<64>, grid, dim3(256), 0, s, tau, cnt, cand, cap, kp, rows, list, count);
}

// Exact distances of the candidates, final order, certificate.  One workgroup per query.
// Query number i = q0 + row is row qmap[i] of X (row i if qmap is null); candidate number j is row cmap[j] of Y
// (row j); distances are taken from those rows, equal distances are ordered by the candidates' row numbers, which
// are also what is written, to row omap[i] (row i) of the result.  n_all: how many candidates a query can have at
// all (one that has them all needs no certificate).  norms_q by query number, norm_max over the database; coeff:
// tile_error_coeff() of the tiles that found the candidates, e_add: what else their distances may be off by.  A query without a certificate is listed as failmap[i] (i).
// What it costs is reading the candidates' rows, so only those that can still be among the k nearest are read: with t the
// k-th smallest tile distance and E the bound of its error, k candidates lie within t + E, and one whose tile distance
// is beyond t + 2 E does not.  Sixteen lanes take a candidate, so a wave has four (vectors of four coordinates: sixteen
// loads in flight), and the LDS is sized by k', not by its limit, which is what lets eight workgroups run per compute
// unit (three before).  The workgroups an XCD runs take consecutive queries, whose candidates (rows in list order, or
// sorted data) its second-level cache then shares.  (Builds of 400,000 x 300 and 512,000 x 50: 295 and 224 -> 283 and 211 ms; of
// 1,281,167 x 2048 from lists: 930 -> 823 ms.)
constexpr int RERANK_LANES = 16;

size_t rerank_lds_bytes(int d, int kp) { return up((size_t)d * 4) + (size_t)kp * 24 + 16; }

__device__ __forceinline__ double sum16(double v)
{
#pragma unroll
    for (int o = RERANK_LANES / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}

__global__ __launch_bounds__(256) void knn_rerank(const float *__restrict__ X, int nx, int d, const int *__restrict__ qmap,
                                                  const float *__restrict__ Y, int ny, const int *__restrict__ cmap,
                                                  const int *__restrict__ omap, const int *__restrict__ failmap, int q0,
                                                  int rows, int k, int kp, int n_all, double coeff, double e_add,
                                                  const float *__restrict__ norms_q, float norm_max,
                                                  const float *__restrict__ tau, const int *__restrict__ cnt,
                                                  const uint64_t *__restrict__ cand, int cap,
                                                  int32_t *__restrict__ knn_idx, double *__restrict__ knn_d2,
                                                  int *__restrict__ fail_count, int *__restrict__ fail_rows,
                                                  const int *__restrict__ sched)
{
    extern __shared__ __align__(16) unsigned char smem[];
    float *xi = reinterpret_cast<float *>(smem);                       // d floats
    double *dd = reinterpret_cast<double *>(smem + up((size_t)d * 4)); // kp each of the following
    uint64_t *key = reinterpret_cast<uint64_t *>(dd + kp);             // tile distances, later the exact ones' order
    int *order = reinterpret_cast<int *>(key + kp);
    int *cid = order + kp;               // the candidates' row numbers in Y
    int *shared = cid + kp;              // candidates left; the k-th smallest tile distance
    // (the grid is 8 x ceil(rows / 8) workgroups, which go to the eight XCDs in turn)
    const int per = (rows + 7) / 8;
    const int turn = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
    if (turn >= rows || (int)(blockIdx.x >> 3) >= per) return;
    const int row = sched ? min(max(sched[turn], 0), rows - 1) : turn;
    const int i = q0 + row;
    const int c_all = min(cnt[row], kp);
    const int iu = min(max(qmap ? qmap[i] : i, 0), nx - 1);
    const float *x = X + (size_t)iu * d;
    for (int t = threadIdx.x; t < d; t += blockDim.x) xi[t] = x[t];
    const uint64_t *buf = cand + (size_t)row * cap;
    for (int a = threadIdx.x; a < c_all; a += blockDim.x) key[a] = buf[a];
    if (threadIdx.x == 0) { shared[0] = 0; shared[1] = -1; }
    __syncthreads();
    // (the additive term covers matrix cores that flush denormal bf16 parts to zero)
    const double E = coeff * ((double)norms_q[i] + (double)norm_max) + 1e-30 * d + e_add;
    if (c_all > k) {
        // the k-th smallest of the (different) words (distance, candidate) by its rank
        for (int a = threadIdx.x; a < c_all; a += blockDim.x) {
            const uint64_t ka = key[a];
            int r = 0;
            for (int b = 0; b < c_all; ++b) r += key[b] < ka;
            if (r == k - 1) shared[1] = a;
        }
        __syncthreads();
    }
    double limit = INFINITY;
    if (shared[1] >= 0) limit = (double)unorderable((uint32_t)(key[shared[1]] >> 32)) + 2.0 * E;
    for (int a = threadIdx.x; a < c_all; a += blockDim.x) {
        // (not "beyond": a distance that is no number stays)
        // (NO_PAIR: from a first launch over fewer rows than k', which nothing compacts)
        if (key[a] == NO_PAIR || (double)unorderable((uint32_t)(key[a] >> 32)) > limit) continue;
        const int j = (int)(uint32_t)key[a];
        cid[atomicAdd(&shared[0], 1)] = min(max(cmap ? cmap[min(j, ny - 1)] : j, 0), ny - 1);
    }
    __syncthreads();
    const int c = shared[0];
    const int g = threadIdx.x / RERANK_LANES, sub = threadIdx.x % RERANK_LANES, ngroups = 256 / RERANK_LANES;
    if (d % 4 == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0) {
        // rows of whole 16-byte pieces: a lane takes four coordinates a load and keeps four partial sums
        const float4 *x4 = reinterpret_cast<const float4 *>(xi);
        const int d4 = d / 4;
        for (int a = g; a < c; a += ngroups) {
            const float4 *y4 = reinterpret_cast<const float4 *>(Y + (size_t)cid[a] * d);
            double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
#pragma unroll 4
            for (int t = sub; t < d4; t += RERANK_LANES) {
                const float4 q = x4[t], u = y4[t];
                double df;
                df = (double)q.x - (double)u.x; a0 += df * df;
                df = (double)q.y - (double)u.y; a1 += df * df;
                df = (double)q.z - (double)u.z; a2 += df * df;
                df = (double)q.w - (double)u.w; a3 += df * df;
            }
            const double s = sum16((a0 + a1) + (a2 + a3));
            if (sub == 0) dd[a] = s;
        }
    } else {
        for (int a = g; a < c; a += ngroups) {
            const float *y = Y + (size_t)cid[a] * d;
            double s = 0.0;
#pragma unroll 4
            for (int t = sub; t < d; t += RERANK_LANES) { double df = (double)xi[t] - (double)y[t]; s += df * df; }
            s = sum16(s);
            if (sub == 0) dd[a] = s;
        }
    }
    __syncthreads();
    // rank by (distance, index): c <= 1920, plain counting rank is enough
    for (int a = threadIdx.x; a < c; a += blockDim.x) key[a] = orderable64(dd[a]);
    __syncthreads();
    for (int a = threadIdx.x; a < c; a += blockDim.x) {
        const uint64_t ka = key[a];
        const int ja = cid[a];
        int r = 0;
        for (int b = 0; b < c; ++b) {
            const uint64_t kb = key[b];
            r += (kb < ka) || (kb == ka && cid[b] < ja);
        }
        order[r] = a;
    }
    __syncthreads();
    const size_t orow = (size_t)(omap ? min(max(omap[i], 0), nx - 1) : i);
    for (int r = threadIdx.x; r < k && r < c; r += blockDim.x) {
        const int a = order[r];
        knn_idx[orow * k + r] = (int32_t)cid[a];
        if (knn_d2) knn_d2[orow * k + r] = dd[a];
    }
    if (threadIdx.x == 0) {
        // pairs never kept had single-precision distance >= tau; the error of that distance is
        // at most E, so they are farther than the exact k-th candidate if tau - E > D_k
        bool ok = c >= k;
        if (ok && c_all < n_all) ok = (double)tau[row] - E > dd[order[k - 1]];
        if (!ok) fail_rows[atomicAdd(fail_count, 1)] = failmap ? failmap[i] : i;
    }
}

// ---- rows that failed the certificate: exact distances to every row, then selection
// A batch of `nb` failed rows rows[0..nb) at a time: okey[f * n + j] = ordered key of the exact distance
// between rows[f] and j.  A wave holds one database row in registers and meets every failed row
// (which come from the second-level cache), so X is read from memory once per batch.
constexpr int EXACT_MAX_D = 4096;
// (queries: rows qmap[rows[f]] of X, or rows[f]; database: the ny rows of Y; exclude_self: X and Y are the same rows)
__global__ __launch_bounds__(256) void knn_exact_dists(const float *__restrict__ X, int nx, const int *__restrict__ qmap,
                                                       const float *__restrict__ Y, int ny, int d,
                                                       const int *__restrict__ rows, int nb, int exclude_self,
                                                       uint64_t *__restrict__ okey)
{
    const size_t w = global_index() >> 6;
    if (w >= (size_t)ny) return;
    const int j = (int)w;
    const float *y = Y + (size_t)j * d;
    float yr[EXACT_MAX_D / WAVE];
#pragma unroll
    for (int q = 0; q < EXACT_MAX_D / WAVE; ++q) {
        const int t = q * WAVE + lane_id();
        yr[q] = (q * WAVE < d && t < d) ? y[t] : 0.f;
    }
    for (int f = 0; f < nb; ++f) {
        int i = rows[f];
        if (qmap) i = qmap[i];
        i = min(max(i, 0), nx - 1);
        const float *x = X + (size_t)i * d;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < EXACT_MAX_D / WAVE; ++q) {
            if (q * WAVE < d) {
                const int t = q * WAVE + lane_id();
                const double df = t < d ? (double)x[t] - (double)yr[q] : 0.0;
                s += df * df;
            }
        }
        s = wave_sum(s);
        if (lane_id() == 0) okey[(size_t)f * ny + j] = (exclude_self && j == i) ? ~0ull : orderable64(s);
    }
}

// One block: 8 radix passes over the ordered 64-bit keys find the k-th smallest distance; then
// the keys below it and the lowest-index ties are put in (distance, index) order.
constexpr int TIE_CAP = 4096;

__device__ __forceinline__ double key_to_double(uint64_t v)
{
    const uint64_t u = (v & 0x8000000000000000ull) ? (v & 0x7FFFFFFFFFFFFFFFull) : ~v;
    return __longlong_as_double((long long)u);
}

// One workgroup per failed row of the batch.  Row f of the batch has its keys at okey_all + f * stride: n of them,
// or counts[f] if counts is given; key j belongs to point j, or to point ids[f * stride + j] if ids is given
// (equal distances are ordered by that number); the list goes to row rows[f] of the output, or rowmap[rows[f]].
__global__ __launch_bounds__(1024) void knn_exact_select(const uint64_t *__restrict__ okey_all, size_t stride, int n,
                                                         const int *__restrict__ counts, const int *__restrict__ ids,
                                                         int k, const int *__restrict__ rows, const int *__restrict__ rowmap,
                                                         int nrows, int32_t *__restrict__ knn_idx, double *__restrict__ knn_d2)
{
    const uint64_t *okey = okey_all + (size_t)blockIdx.x * stride;
    const int *id = ids ? ids + (size_t)blockIdx.x * stride : nullptr;
    if (counts) n = min(counts[blockIdx.x], (int)stride);
    int i = min(max(rows[blockIdx.x], 0), nrows - 1);
    if (rowmap) i = min(max(rowmap[i], 0), nrows - 1);
    __shared__ uint32_t hist[256];
    __shared__ uint64_t prefix_s;
    __shared__ int want_s, nsel, ntie, best;
    __shared__ uint64_t selk[MAX_KP];
    __shared__ int selj[MAX_KP];
    __shared__ uint64_t tie[TIE_CAP];
    uint64_t prefix = 0;
    int want = k;   // rank (1-based) of the target among the keys that match the prefix so far
    for (int pass = 7; pass >= 0; --pass) {
        if (threadIdx.x < 256) hist[threadIdx.x] = 0;
        __syncthreads();
        const int sh = pass * 8;
        const uint64_t mask = pass == 7 ? 0ull : (~0ull << (sh + 8));
        for (int j = threadIdx.x; j < n; j += blockDim.x) {
            const uint64_t v = okey[j];
            if ((v & mask) == prefix) atomicAdd(&hist[(v >> sh) & 0xFF], 1u);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int acc = 0, b = 0;
            for (; b < 255; ++b) {
                if (acc + (int)hist[b] >= want) break;
                acc += (int)hist[b];
            }
            prefix_s = prefix | ((uint64_t)b << sh);
            want_s = want - acc;
        }
        __syncthreads();
        prefix = prefix_s;
        want = want_s;
        __syncthreads();
    }
    // prefix = k-th smallest key; k - want keys lie below it; `want` of its ties are needed
    if (threadIdx.x == 0) { nsel = 0; ntie = 0; }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const uint64_t v = okey[j];
        if (v < prefix) {
            const int p = atomicAdd(&nsel, 1);
            if (p < MAX_KP) { selk[p] = v; selj[p] = id ? id[j] : j; }
        } else if (v == prefix) {
            const int p = atomicAdd(&ntie, 1);
            if (p < TIE_CAP) tie[p] = (uint64_t)(uint32_t)(id ? id[j] : j);
        }
    }
    __syncthreads();
    const int below = min(nsel, k - want);
    for (int a = threadIdx.x; a < below; a += blockDim.x) {
        const uint64_t ka = selk[a];
        const int ja = selj[a];
        int r = 0;
        for (int b = 0; b < below; ++b) r += (selk[b] < ka) || (selk[b] == ka && selj[b] < ja);
        knn_idx[(size_t)i * k + r] = ja;
        if (knn_d2) knn_d2[(size_t)i * k + r] = key_to_double(ka);
    }
    const double dk = key_to_double(prefix);
    if (ntie <= TIE_CAP) {
        int size = 1;
        while (size < ntie) size <<= 1;
        for (int t = threadIdx.x; t < size; t += blockDim.x) if (t >= ntie) tie[t] = ~0ull;
        __syncthreads();
        for (int kk = 2; kk <= size; kk <<= 1)
            for (int jj = kk >> 1; jj > 0; jj >>= 1) {
                for (int t = threadIdx.x; t < size; t += blockDim.x) {
                    const int ixj = t ^ jj;
                    if (ixj > t) {
                        const uint64_t a = tie[t], b = tie[ixj];
                        if ((a > b) == ((t & kk) == 0)) { tie[t] = b; tie[ixj] = a; }
                    }
                }
                __syncthreads();
            }
        for (int t = threadIdx.x; t < want && t < ntie; t += blockDim.x) {
            knn_idx[(size_t)i * k + below + t] = (int32_t)tie[t];
            if (knn_d2) knn_d2[(size_t)i * k + below + t] = dk;
        }
    } else {
        // more equidistant rows than the tie buffer holds: the lowest number above the last one taken, `want` times
        int last = -1;
        for (int out = below; out < k; ++out) {
            __syncthreads();
            if (threadIdx.x == 0) best = 0x7FFFFFFF;
            __syncthreads();
            int mine = 0x7FFFFFFF;
            for (int j = threadIdx.x; j < n; j += blockDim.x)
                if (okey[j] == prefix) {
                    const int v = id ? id[j] : j;
                    if (v > last && v < mine) mine = v;
                }
            if (mine != 0x7FFFFFFF) atomicMin(&best, mine);
            __syncthreads();
            last = best;
            if (last == 0x7FFFFFFF) break;
            if (threadIdx.x == 0) { knn_idx[(size_t)i * k + out] = last; if (knn_d2) knn_d2[(size_t)i * k + out] = dk; }
        }
    }
}

// ---- Eq. (1): conditional probabilities with the entropy fixed at ln(perplexity)
// Sixteen lanes per row: an evaluation of the entropy is k / 16 exponentials a lane and three sums over the lanes
// (which all lanes get with the same bits, so they branch alike).  What bounds it is the number of evaluations, each
// waiting for the one before.  Doubling and halving from beta = 1 brackets the root, and then beta goes to Newton's point,
// dH/dbeta = -beta Var(r), if that lies inside the bracket and the last step has at least halved the miss, and to the
// middle if not.  Where the entropy hardly depends on beta (beta^2 Var(r) small at the end: ties at the target, the target
// at the entropy of equal weights) many beta pass the test, and rows that never pass it end where the halving ends: both are
// done again by doubling and halving alone, whose beta is the defined one.  (One lane per row and bisection,
// some forty evaluations of k exponentials: 0.37 ms of a build of 2000 points, 1.80 -> 1.45 ms in all; 60,000 points
// 0.95 ms, 22.2 -> 21.4.)
constexpr int PERP_LANES = 16, PERP_ROWS = 256 / PERP_LANES;

__global__ __launch_bounds__(256) void perplexity_search(const double *__restrict__ d2, int n, int k, double target,
                                                         double tol, double *__restrict__ cond, double *__restrict__ reach,
                                                         int *__restrict__ unconverged, int staged)
{
    extern __shared__ __align__(16) unsigned char ps_smem[];
    double *sd = reinterpret_cast<double *>(ps_smem);
    const int row0 = blockIdx.x * PERP_ROWS, g = threadIdx.x / PERP_LANES, sub = threadIdx.x % PERP_LANES;
    const int i = row0 + g;
    const double *dd = d2 + (size_t)min(i, n - 1) * k;
    if (staged) {                       // the workgroup's rows of distances fit in LDS
        const size_t total = (size_t)min(PERP_ROWS, n - row0) * k;
        const double *src = d2 + (size_t)row0 * k;
        for (size_t t = threadIdx.x; t < total; t += 256) sd[t] = src[t];
        __syncthreads();
        dd = sd + (size_t)min(g, n - 1 - row0) * k;
    }
    double dmin = INFINITY, dmax = 0.0;
    for (int m = sub; m < k; m += PERP_LANES) {
        dmin = fmin(dmin, dd[m]);
        dmax = dd[m] <= dmax ? dmax : dd[m];            // (a distance that is no number stays)
    }
#pragma unroll
    for (int o = PERP_LANES / 2; o > 0; o >>= 1) {
        dmin = fmin(dmin, __shfl_xor(dmin, o, WAVE));
        const double other = __shfl_xor(dmax, o, WAVE);
        dmax = dmax != dmax || other <= dmax ? dmax : other;
    }
    if (i < n && sub == 0) reach[i] = dmax;
    double beta = 1.0;
    bool ok = false;
    for (int plain = 0; plain < 2; ++plain) {
        double lo = 0.0, hi = INFINITY, miss = INFINITY, slope = 1.0;
        beta = 1.0;
        ok = false;
        for (int it = 0; it < (plain ? 400 : 60); ++it) {
            double S = 0.0, T = 0.0, Q = 0.0;
            for (int m = sub; m < k; m += PERP_LANES) {
                const double r = dd[m] - dmin, e = exp(-beta * r), re = r * e;
                S += e;
                T += re;
                Q += r * re;
            }
            S = sum16(S);
            T = sum16(T);
            Q = sum16(Q);
            const double mean = T / S, f = log(S) + beta * mean - target;
            slope = beta * (Q / S - mean * mean);
            if (fabs(f) <= tol) { ok = true; break; }
            const double newton = beta + f / slope;
            const bool fast = fabs(f) <= 0.5 * miss;
            miss = fabs(f);
            if (f > 0.0) lo = beta; else hi = beta;
            if (isinf(hi)) beta *= 2.0;
            else beta = !plain && fast && newton > lo && newton < hi ? newton : 0.5 * (lo + hi);
            if (!(beta > 0.0) || isinf(beta)) break;
        }
        if (ok && beta * slope >= 0.02) break;
    }
    double S = 0.0;
    for (int m = sub; m < k; m += PERP_LANES) S += exp(-beta * (dd[m] - dmin));
    S = sum16(S);
    if (i >= n) return;
    if (!ok && sub == 0) atomicAdd(unconverged, 1);
    for (int m = sub; m < k; m += PERP_LANES) cond[(size_t)i * k + m] = exp(-beta * (dd[m] - dmin)) / S;
}

// ---- symmetrisation
// extra[j] = number of rows i that list j while j does not list i; slot[e] = where i sits in j's list
// (-1 if it does not), kept for sym_fill (k <= 1280 fits 16 bits).  Sixteen lanes look one edge up: they
// read 64 contiguous bytes of row j at a time, so a row costs its three or four cache lines once.
// About half of the edges have no partner, and nearly all of those are settled without row j: a row that j does not list
// is farther from j than the farthest one j lists (reach[j]; d2 and reach are sums in double, possibly in another order,
// hence the factor).  symmetric = 0: the distance from j to i may be another (product-quantised codes).  (1,281,167 x 2048
// from lists: 16.4 -> 13.8 ms, 512,000 x 50 5.7 -> 4.6.)
__global__ __launch_bounds__(256) void sym_count(const int32_t *__restrict__ idx, int n, int k, int *__restrict__ extra,
                                                 int16_t *__restrict__ slot, const double *__restrict__ d2,
                                                 const double *__restrict__ reach, int symmetric)
{
    const size_t e = global_index() >> 4;
    const int sub = (int)(threadIdx.x & 15u), grp = (int)((threadIdx.x & 63u) >> 4);
    const bool live = e < (size_t)n * k;
    const size_t ee = live ? e : 0;
    const int i = (int)(ee / k), j = idx[ee];
    const int32_t *r = idx + (size_t)j * k;
    const bool far = symmetric && d2[ee] > reach[j] * (1.0 + 1e-9);
    int found = -1;
    for (int a0 = 0; a0 < k; a0 += 16) {
        if (__all(far || found >= 0)) break;
        const int a = a0 + sub;
        const bool hit = !far && a < k && r[a] == i;
        const unsigned m = (unsigned)(__ballot(hit) >> (16 * grp)) & 0xFFFFu;
        if (m != 0u && found < 0) found = a0 + __builtin_ctz(m);
    }
    if (live && sub == 0) {
        slot[e] = (int16_t)found;
        if (found < 0) atomicAdd(&extra[j], 1);
    }
}

// row_ptr[i] = sum_{r<i} (k + extra[r]); single block, n up to 2^30
__global__ __launch_bounds__(1024) void sym_scan(const int *__restrict__ extra, int n, int k, int32_t *__restrict__ row_ptr,
                                                 int *__restrict__ cursor)
{
    __shared__ long long ws[16];
    const int per = (n + 1023) / 1024;
    const int s = threadIdx.x * per, e = min(n, s + per);
    long long a = 0;
    for (int i = s; i < e; ++i) a += k + extra[i];
    long long inc = a;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        long long t = __shfl_up(inc, o, WAVE);
        if (lane_id() >= o) inc += t;
    }
    if (lane_id() == WAVE - 1) ws[threadIdx.x >> 6] = inc;
    __syncthreads();
    long long base = 0;
    for (int q = 0; q < (int)(threadIdx.x >> 6); ++q) base += ws[q];
    long long pre = base + inc - a;
    for (int i = s; i < e; ++i) {
        row_ptr[i] = (int32_t)pre;
        cursor[i] = (int)pre + k;     // extras are appended after the row's own k entries
        pre += k + extra[i];
    }
    if (threadIdx.x == 1023) row_ptr[n] = (int32_t)pre;
}

__global__ __launch_bounds__(256) void sym_fill(const int32_t *__restrict__ idx, const double *__restrict__ cond, int n,
                                                int k, const int32_t *__restrict__ row_ptr, int *__restrict__ cursor,
                                                const int16_t *__restrict__ slots, int32_t *__restrict__ col,
                                                float *__restrict__ val)
{
    const size_t e = global_index();
    if (e >= (size_t)n * k) return;
    const int i = (int)(e / k), a = (int)(e % k), j = idx[e];
    const double pji = cond[e];
    const int slot = slots[e];
    const double pij = slot >= 0 ? cond[(size_t)j * k + slot] : 0.0;
    const float v = (float)((pji + pij) / (2.0 * (double)n));
    col[row_ptr[i] + a] = j;
    val[row_ptr[i] + a] = v;
    if (slot < 0) {
        const int pos = atomicAdd(&cursor[j], 1);
        col[pos] = i;
        val[pos] = v;
    }
}

// Bitonic sort of `size` (power of two) 64-bit keys in LDS by one workgroup.
__device__ __forceinline__ void bitonic_sort(uint64_t *s, int size)
{
    for (int k = 2; k <= size; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < size; t += blockDim.x) {
                int ixj = t ^ j;
                if (ixj > t) {
                    uint64_t a = s[t], b = s[ixj];
                    bool up = (t & k) == 0;
                    if ((a > b) == up) { s[t] = b; s[ixj] = a; }
                }
            }
            __syncthreads();
        }
    }
}

// Sort each row by column.  Two waves per row do it in LDS, SORT_SHORT entries of it, so that sixteen rows are in flight
// per compute unit and hide each other's barriers; a longer row (a point near the middle of a wide cluster is in thousands
// of lists) goes on a list for sym_sort_long.  (60,000 rows 0.65 -> 0.20 ms with the whole 32 KB a row before,
// 1,281,167 rows 10.9 -> 4.2.)
__global__ __launch_bounds__(128) void sym_sort_rows(const int32_t *__restrict__ row_ptr, int n, int32_t *__restrict__ col,
                                                     float *__restrict__ val, int *__restrict__ long_rows,
                                                     int *__restrict__ long_count)
{
    __shared__ uint64_t s[SORT_SHORT];
    if (global_block() >= (size_t)n) return;
    const int row = (int)global_block();
    const int b = row_ptr[row], len = row_ptr[row + 1] - b;
    if (len <= 1) return;
    if (len > SORT_SHORT) {
        if (threadIdx.x == 0) long_rows[atomicAdd(long_count, 1)] = row;
        return;
    }
    int size = 1;
    while (size < len) size <<= 1;
    for (int t = threadIdx.x; t < size; t += blockDim.x)
        s[t] = t < len ? (((uint64_t)(uint32_t)col[b + t] << 32) | __float_as_uint(val[b + t])) : ~0ull;
    __syncthreads();
    bitonic_sort(s, size);
    for (int t = threadIdx.x; t < len; t += blockDim.x) {
        col[b + t] = (int32_t)(s[t] >> 32);
        val[b + t] = __uint_as_float((uint32_t)s[t]);
    }
}

// The rows on the list, a workgroup of 1024 lanes each: runs of SORT_CAP entries are sorted in LDS and left in scratch,
// then an entry's place is its place in its own run plus, by binary search, the number of smaller entries in every other
// run (columns are different, so places are).  (Ranking by one comparison per pair of entries let the longest row of
// 512,000 points in four wide clusters hold the whole launch up: 20.5 of 205 ms, now 193 in all.)
__global__ __launch_bounds__(1024) void sym_sort_long(const int32_t *__restrict__ row_ptr, int n, int32_t *__restrict__ col,
                                                      float *__restrict__ val, uint64_t *__restrict__ scratch,
                                                      const int *__restrict__ long_rows, const int *__restrict__ long_count)
{
    __shared__ uint64_t s[SORT_CAP];
    const int m = min(*long_count, n);
    for (int i = blockIdx.x; i < m; i += gridDim.x) {
        const int row = long_rows[i];
        const int b = row_ptr[row], len = row_ptr[row + 1] - b;
        uint64_t *tmp = scratch + b;
        for (int r0 = 0; r0 < len; r0 += SORT_CAP) {
            const int take = min(SORT_CAP, len - r0);
            int size = 1;
            while (size < take) size <<= 1;
            __syncthreads();            // the previous run (or row) is out of s
            for (int t = threadIdx.x; t < size; t += 1024)
                s[t] = t < take ? (((uint64_t)(uint32_t)col[b + r0 + t] << 32) | __float_as_uint(val[b + r0 + t])) : ~0ull;
            __syncthreads();
            bitonic_sort(s, size);
            for (int t = threadIdx.x; t < take; t += 1024) tmp[r0 + t] = s[t];
        }
        __syncthreads();
        for (int t = threadIdx.x; t < len; t += 1024) {
            const uint64_t me = tmp[t];
            const int own = t / SORT_CAP * SORT_CAP;
            int place = t - own;
            for (int r0 = 0; r0 < len; r0 += SORT_CAP) {
                if (r0 == own) continue;
                int lo = r0, hi = min(r0 + SORT_CAP, len);      // the first entry of the run that is not smaller
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (tmp[mid] < me) lo = mid + 1; else hi = mid;
                }
                place += lo - r0;
            }
            col[b + place] = (int32_t)(me >> 32);
            val[b + place] = __uint_as_float((uint32_t)me);
        }
    }
}

__global__ void max_norm_k(const float *__restrict__ norms, int n, float *__restrict__ out)
{
    __shared__ float ws[16];
    float m = 0.f;
#pragma unroll 8
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = fmaxf(m, norms[i]);
    m = wave_max(m);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < (int)(blockDim.x >> 6); ++q) m = fmaxf(m, ws[q]);
        *out = m;
    }
}

__global__ void d2_to_float(const double *__restrict__ in, float *__restrict__ out, size_t m)
{
    size_t i = global_index();
    if (i < m) out[i] = (float)in[i];
}

// ---- the order in which the rows of a block are re-ranked
// A row's re-rank reads about k' whole rows.  Where X is larger than the second-level caches, rows that are re-ranked at
// the same time should be near each other, so that they find each other's candidates there: they go by the nearest of the
// first SCHED_PIVOTS rows, whose distances the first launch leaves at the first places of every buffer.
// (60,000 x 784: the re-rank 2.63 -> 1.76 ms, the build 13.4 -> 12.5; 100,000 x 784 31.8 -> 30.1.  Rows of 300 coordinates
// gain nothing: 60,000 8.71 -> 8.80 ms, 400,000 179.5 -> 179.7.)
constexpr int SCHED_PIVOTS = WAVE, SCHED_ROWS = 256, SCHED_MIN_D = 512, SCHED_MIN_ROWS = 8192;
constexpr size_t SCHED_MIN_BYTES = 32u << 20;       // (eight caches of 4 MB)
// label[row] = the nearest of these, and how many rows each has; a wave a row
__global__ __launch_bounds__(256) void rerank_label_k(const uint64_t *__restrict__ cand, int cap, int rows, int *__restrict__ label,
                                                      int *__restrict__ total)
{
    __shared__ int hist[SCHED_PIVOTS];
    const int tid = (int)threadIdx.x, r0 = (int)blockIdx.x * SCHED_ROWS;
    if (tid < SCHED_PIVOTS) hist[tid] = 0;
    __syncthreads();
    for (int t = tid >> 6; t < SCHED_ROWS && r0 + t < rows; t += 4) {
        uint64_t best = cand[(size_t)(r0 + t) * cap + lane_id()];
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) best = min(best, (uint64_t)__shfl_xor((unsigned long long)best, o, WAVE));
        if (lane_id() == 0) {
            const int l = (int)((uint32_t)best % SCHED_PIVOTS);         // (NO_PAIR everywhere: the last)
            label[r0 + t] = l;
            atomicAdd(&hist[l], 1);
        }
    }
    __syncthreads();
    if (tid < SCHED_PIVOTS && hist[tid] > 0) atomicAdd(&total[tid], hist[tid]);
}

// sched = the rows by label; taken[label] (zero on entry): how many places workgroups have taken so far
__global__ __launch_bounds__(SCHED_ROWS) void rerank_sched_k(const int *__restrict__ label, int rows, const int *__restrict__ total,
                                                             int *__restrict__ taken, int *__restrict__ sched)
{
    __shared__ int hist[SCHED_PIVOTS], base[SCHED_PIVOTS];
    const int tid = (int)threadIdx.x, row = (int)blockIdx.x * SCHED_ROWS + tid;
    if (tid < SCHED_PIVOTS) hist[tid] = 0;
    __syncthreads();
    const int l = row < rows ? label[row] % SCHED_PIVOTS : 0;
    const int at = row < rows ? atomicAdd(&hist[l], 1) : 0;
    __syncthreads();
    if (tid < SCHED_PIVOTS) {
        int before = 0;
        for (int k = 0; k < tid; ++k) before += total[k];
        base[tid] = before + (hist[tid] > 0 ? atomicAdd(&taken[tid], hist[tid]) : 0);
    }
    __syncthreads();
    if (row < rows) sched[min(base[l] + at, rows - 1)] = row;
}

// ---- the exact search in an order of the rows that keeps neighbours together
// Taken as they come, a query's neighbours turn up anywhere in the sweep: its cut-off settles slowly, and some hundreds of
// pairs beyond the k' it ends with are tested the long way, appended and compacted; and no tile can be left out.  So the rows
// are grouped by the nearest of some evenly spaced rows (the pivots, in an order that puts each next to one near it), the
// search works on copies in that order, and every query tile of 256 rows first meets the ORD_FIRST database tiles whose
// centres are nearest to its own.  That settles the cut-offs.  Of the other tiles it meets, in row order, those that can
// still hold a neighbour: with |c - c'| the distance of the centres and r, r' the tiles' radii, no pair is closer than
// |c - c'| - r - r', and a tile where that is beyond the largest cut-off is left out (its pairs are, as the certificate
// asks of every pair that was not kept, no closer than the cut-off).  Between clusters that are well apart nearly all tiles
// are.  The neighbour lists are what they were: any order of the rows gives them.
// 512,000 rows of 50 coordinates in four blobs: 187 -> 104 ms.  Where no tile can be left out the order only costs (the query tiles
// no longer meet the same database tiles at a time, and 33,000, 60,000 and 200,000 rows in clusters that touch went from 4.6,
// 7.5 and 48.5 to 6.0, 10.2 and 54.9 ms), so it is taken where the pivots say that the rows fall into groups well apart: at
// least half of their pairs farther apart than ORD_APART times what a pivot is from the nearest other one (root mean square).
// A tile's radius and a row's cut-off are about as large as the latter, which makes two radii and a cut-off.  For four blobs
// three quarters of the pairs are, by a factor of ten; for clusters that touch at most a quarter.  And from ORD_MIN_ROWS rows
// on: 100,000 rows in four blobs 17.1 -> 19.1 ms, 140,000 29.6 -> 26.8, 200,000 49 -> 36, 300,000 82 -> 56; with twenty blobs
// in 8 dimensions too many query tiles straddle two, which the first block of query rows finds out in 2 ms.
constexpr int ORD_FIRST = 16;                  // tiles taken nearest first
constexpr int ORD_MIN_ROWS = 196608, ORD_MAX_TILES = 4096;
constexpr int ORD_MAX_PIVOTS = 512;
// What launches take (with the compaction behind them 120, 80 and 40 us): along the lists, over DBC of all rows, and over
// ORD_ALONE_ROWS of all rows for one query tile by itself.
constexpr int ORD_LAUNCH = 3, ORD_PLAIN = 2, ORD_ALONE = 1, ORD_ALONE_ROWS = COMPACT_EVERY * DBC;
constexpr float ORD_APART = 3.f;
static_assert(ORD_FIRST % ORD_STEP == 0 && ORD_MAX_TILES % ORD_STEP == 0 && RQ == HT, "whole launches");

// label[row] = number (in the pivots' own order: prank) of the nearest pivot, from a dense launch against m pivots; a wave a row
__global__ __launch_bounds__(256) void nearest_pivot_k(const uint64_t *__restrict__ cand, int cap, int rows, int m,
                                                       const int *__restrict__ prank, int32_t *__restrict__ label)
{
    const int row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (row >= rows) return;
    uint64_t best = NO_PAIR;
#pragma unroll 4
    for (int j = lane_id(); j < m; j += WAVE) best = min(best, cand[(size_t)row * cap + j]);
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) best = min(best, (uint64_t)__shfl_xor((unsigned long long)best, o, WAVE));
    // (a row without a finite distance: the first pivot)
    if (lane_id() == 0) label[row] = prank[best == NO_PAIR ? 0 : min((int)(uint32_t)best, m - 1)];
}

// apart[0] = pairs of pivots that are farther apart than ORD_APART times a pivot's distance from the nearest other one; one
// workgroup, a thread a pivot.  cand: their squared distances (dense).
__global__ __launch_bounds__(ORD_MAX_PIVOTS) void pivot_apart_k(const uint64_t *__restrict__ cand, int cap, int m, int *__restrict__ apart)
{
    __shared__ double part[ORD_MAX_PIVOTS / WAVE];
    __shared__ int count[ORD_MAX_PIVOTS / WAVE];
    const int tid = (int)threadIdx.x, i = min(tid, m - 1);
    // (column i of the symmetric table: neighbouring threads read neighbouring words; a pair that is none is no number)
    float near = INFINITY;
#pragma unroll 8
    for (int j = 0; j < m; ++j) {
        const float v = unorderable((uint32_t)(cand[(size_t)j * cap + i] >> 32));
        if (j != i && v < near) near = v;
    }
    const double mine = wave_sum(tid < m ? (double)fmaxf(near, 0.f) : 0.0);
    if (lane_id() == 0) part[tid >> 6] = mine;
    __syncthreads();
    double sum = 0.0;
    for (int w = 0; w < ORD_MAX_PIVOTS / WAVE; ++w) sum += part[w];
    const float limit = (float)(sum / m) * (ORD_APART * ORD_APART);
    int far = 0;
#pragma unroll 8
    for (int j = 0; j < m; ++j) far += unorderable((uint32_t)(cand[(size_t)j * cap + i] >> 32)) > limit ? 1 : 0;
    if (tid >= m) far = 0;
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) far += __shfl_xor(far, o, WAVE);
    if (lane_id() == 0) count[tid >> 6] = far;
    __syncthreads();
    if (tid == 0) {
        int all = 0;
        for (int w = 0; w < ORD_MAX_PIVOTS / WAVE; ++w) all += count[w];
        apart[0] = all / 2;
    }
}

// The pivots in an order in which each is followed by the nearest one left; one workgroup.  cand: their distances (dense).
__global__ __launch_bounds__(ORD_MAX_PIVOTS) void pivot_chain_k(const uint64_t *__restrict__ cand, int cap, int m, int *__restrict__ prank)
{
    __shared__ uint64_t best[ORD_MAX_PIVOTS / WAVE];
    const int tid = (int)threadIdx.x;
    bool left = tid < m && tid != 0;
    int cur = 0;
    if (tid == 0) prank[0] = 0;
    for (int i = 1; i < m; ++i) {
        // (a pair that is none, say between copies of values that are no numbers, comes last; ties by number)
        uint64_t key = left ? ((cand[(size_t)cur * cap + tid] >> 32) << 32) | (uint32_t)tid : ~0ull;
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) key = min(key, (uint64_t)__shfl_xor((unsigned long long)key, o, WAVE));
        if (lane_id() == 0) best[tid >> 6] = key;
        __syncthreads();
        key = best[0];
        for (int w = 1; w < ORD_MAX_PIVOTS / WAVE; ++w) key = min(key, best[w]);
        cur = min((int)(uint32_t)key, m - 1);
        if (tid == cur) { left = false; prank[cur] = i; }
        __syncthreads();
    }
}

// Centre (relative to mu) of the rows of every tile of HT rows; a workgroup a tile, a thread a column.
__global__ __launch_bounds__(256) void tile_centre_k(const float *__restrict__ X, const float *__restrict__ mu, int n, int d,
                                                     const int *__restrict__ ord, float *__restrict__ centre)
{
    __shared__ int rows[HT];
    const int r0 = (int)blockIdx.x * HT, m = min(HT, n - r0);
    for (int t = (int)threadIdx.x; t < m; t += 256) rows[t] = min(max(ord[r0 + t], 0), n - 1);
    __syncthreads();
    for (int c = (int)threadIdx.x; c < d; c += 256) {
        float a = 0.f;
#pragma unroll 8
        for (int t = 0; t < m; ++t) a += X[(size_t)rows[t] * d + c] - mu[c];
        centre[(size_t)blockIdx.x * d + c] = a / (float)m;
    }
}

// radius2[tile] = largest squared distance of its rows from its centre (bits of a non-negative float; zero on entry).  Any
// point would do for a centre, as long as the radius is taken around the same one.
__global__ __launch_bounds__(256) void tile_radius_k(const float *__restrict__ X, const float *__restrict__ mu, int n, int d,
                                                     const int *__restrict__ ord, const float *__restrict__ centre,
                                                     unsigned int *__restrict__ radius2)
{
    const int r = (int)(global_index() >> 6);
    if (r >= n) return;
    const float *x = X + (size_t)min(max(ord[r], 0), n - 1) * d, *c = centre + (size_t)(r / HT) * d;
    float a = 0.f;
#pragma unroll 4
    for (int t = lane_id(); t < d; t += WAVE) { const float v = (x[t] - mu[t]) - c[t]; a = fmaf(v, v, a); }
    a = wave_sum(a);
    // (not a number: nothing is left out around it)
    if (lane_id() == 0) atomicMax(radius2 + r / HT, a >= 0.f ? __float_as_uint(a) : 0x7F800000u);
}

// For query tile qt0 + blockIdx.x: near[tile] = what its pairs with every tile are apart at least, and the ORD_FIRST
// tiles with the nearest centres (less their radius, so that a wide tile comes early).  The bound: each of the three
// distances is a float sum of at most 2048 squares and a root, good to 2^-24 (2048 / 64 + 16) < 3e-6 relative, of
// coordinates that are off by 2^-24 |x - mu| each; 1e-4 of the centres' distance and of the radii covers that as long as
// the coordinates' own rounding is small against the distances (and where it is not, the bound of a tile distance, which
// the certificate takes off the cut-off, is far larger).
__global__ __launch_bounds__(1024) void tile_order_k(const float *__restrict__ centre, const float *__restrict__ radius2, int ntiles,
                                                     int d, int qt0, float *__restrict__ near, uint16_t *__restrict__ first)
{
    extern __shared__ __align__(16) unsigned char osm[];
    float *c = reinterpret_cast<float *>(osm);                // the query tile's centre
    float *key = c + d;                                       // of every tile
    __shared__ uint64_t best[16];
    const int tid = (int)threadIdx.x, w = tid >> 6, me = qt0 + (int)blockIdx.x;
    for (int t = tid; t < d; t += 1024) c[t] = centre[(size_t)me * d + t];
    __syncthreads();
    const float r1 = sqrtf(radius2[me]);
    for (int t = w; t < ntiles; t += 16) {
        const float *o = centre + (size_t)t * d;
        float a = 0.f;
#pragma unroll 4
        for (int u = lane_id(); u < d; u += WAVE) { const float v = c[u] - o[u]; a = fmaf(v, v, a); }
        a = wave_sum(a);
        if (lane_id() == 0) {
            const float dist = sqrtf(a), r2 = sqrtf(radius2[t]);
            const float b = dist * (1.f - 1e-4f) - (r1 + r2) * (1.f + 1e-4f);
            near[(size_t)blockIdx.x * ntiles + t] = b > 0.f ? b : 0.f;      // (also where it is no number)
            const float k = t == me ? -INFINITY : dist - r2;
            key[t] = k < INFINITY ? k : 3.0e38f;
        }
    }
    __syncthreads();
    for (int i = 0; i < ORD_FIRST; ++i) {
        uint64_t b = ~0ull;
        for (int t = tid; t < ntiles; t += 1024) b = min(b, ((uint64_t)orderable(key[t]) << 32) | (uint32_t)t);
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) b = min(b, (uint64_t)__shfl_xor((unsigned long long)b, o, WAVE));
        if (lane_id() == 0) best[w] = b;
        __syncthreads();
        b = best[0];
        for (int k = 1; k < 16; ++k) b = min(b, best[k]);
        const int t = (int)(uint32_t)b;
        if (tid == 0 && i < ntiles) { first[(size_t)blockIdx.x * ORD_FIRST + i] = (uint16_t)t; key[min(t, ntiles - 1)] = INFINITY; }
        __syncthreads();
    }
}

// The tiles that query tile blockIdx.x still has to meet, in row order: not among the first ones, and not farther than
// the largest cut-off of its rows.
__global__ __launch_bounds__(256) void tile_rest_k(const float *__restrict__ near, int ntiles, const uint16_t *__restrict__ first,
                                                   const float *__restrict__ tau, int rows, uint16_t *__restrict__ rest,
                                                   int *__restrict__ count)
{
    __shared__ float cuts[4];
    __shared__ int wsum[4];
    __shared__ uint16_t done[ORD_FIRST];
    const int tid = (int)threadIdx.x, b = (int)blockIdx.x, row = b * HT + tid;
    float cut = wave_max(row < rows ? tau[row] : -INFINITY);
    if (lane_id() == 0) cuts[tid >> 6] = cut;
    if (tid < ORD_FIRST) done[tid] = tid < min(ntiles, ORD_FIRST) ? first[(size_t)b * ORD_FIRST + tid] : 0xFFFFu;
    __syncthreads();
    cut = fmaxf(fmaxf(cuts[0], cuts[1]), fmaxf(cuts[2], cuts[3]));
    int have = 0;
    for (int t0 = 0; t0 < ntiles; t0 += 256) {
        const int t = t0 + tid;
        bool take = t < ntiles;
        if (take) {
            const float a = near[(size_t)b * ntiles + t];
            take = !(a * a * (1.f - 1e-6f) >= cut);
            for (int i = 0; i < ORD_FIRST; ++i) take = take && done[i] != (uint16_t)t;
        }
        const uint64_t m = __ballot(take);
        if (lane_id() == 0) wsum[tid >> 6] = (int)__popcll(m);
        __syncthreads();
        int at = have + (int)__popcll(m & lanemask_lt());
        for (int k = 0; k < 4; ++k) { if (k < (tid >> 6)) at += wsum[k]; have += wsum[k]; }
        if (take) rest[(size_t)b * ORD_MAX_TILES + at] = (uint16_t)t;
        __syncthreads();
    }
    if (tid == 0) count[b] = have;
}

// query tiles with more than `limit` tiles left to meet are not for the lists
__global__ void tile_rest_limit_k(int *__restrict__ count, int m, int limit)
{
    const int t = (int)global_index();
    if (t < m && count[t] > limit) count[t] = 0;
}

// ---- Eq. (10)-(11) for long rows on the same tiles: helpers of ivf_search_tiles() below
// the probed lists of every row, rows in list order
__global__ void probe_gather(const int32_t *__restrict__ probe, const int *__restrict__ lorder, int n, int tau, int nlist,
                             int32_t *__restrict__ probe_l)
{
    const size_t e = global_index();
    if (e >= (size_t)n * tau) return;
    const size_t pos = e / tau;
    const int r = (int)(e % tau);
    const int row = min(max(lorder[pos], 0), n - 1);
    probe_l[e] = min(max(probe[(size_t)row * tau + r], 0), nlist - 1);
}

// queries q0 .. q0 + rows of the pass, grouped by the list they probe at rank r
// A counter per list, one addition per query: the queries come in list order, so at the first rank a wave's queries mostly
// probe the same list, and additions to one address follow one another at the memory side.  The lanes that share the first
// live lane's list, then those that share the next one's, add up once; the others, at most a few lists of a wave at the
// later ranks in common, add for themselves.  (With gather_double left out where nobody
// reads its result: 1,281,167 x 2048 from lists, 816 -> 774 ms.)
__device__ __forceinline__ int wave_add(int *__restrict__ counters, int c, bool live)
{
    int mine = 0;
    uint64_t left = __ballot(live);
    for (int round = 0; round < 2 && left != 0; ++round) {
        const int lead = __builtin_ctzll(left), lc = __builtin_amdgcn_readlane(c, lead);
        const uint64_t same = __ballot(live && c == lc) & left;
        int base = 0;
        if ((int)lane_id() == lead) base = atomicAdd(&counters[lc], (int)__popcll(same));
        base = __builtin_amdgcn_readlane(base, lead);
        if ((same >> lane_id()) & 1ull)
            mine = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        left &= ~same;
    }
    if ((left >> lane_id()) & 1ull) mine = atomicAdd(&counters[c], 1);
    return mine;
}

// (qmap: query q is row qmap[q] of the list order; null: row q)
__global__ void rank_hist(const int32_t *__restrict__ probe_l, const int *__restrict__ qmap, int q0, int rows, int tau, int r,
                          int *__restrict__ bcnt)
{
    const size_t i = global_index();
    const bool live = i < (size_t)rows;
    wave_add(bcnt, live ? probe_l[(qmap ? (size_t)qmap[q0 + i] : (size_t)q0 + i) * tau + r] : 0, live);
}

__global__ void rank_scatter(const int32_t *__restrict__ probe_l, const int *__restrict__ qmap, int q0, int rows, int tau, int r,
                             const int *__restrict__ pairptr, int *__restrict__ bcur, int *__restrict__ pairq)
{
    const size_t i = global_index();
    const bool live = i < (size_t)rows;
    const int L = live ? probe_l[(qmap ? (size_t)qmap[q0 + i] : (size_t)q0 + i) * tau + r] : 0;
    const int at = wave_add(bcur, L, live);
    if (live) pairq[pairptr[L] + at] = q0 + (int)i;     // any order inside a list
}

// tiles of list L in the launch that takes rows chunk * DBC .. of every list
// (tr database rows a tile)
__global__ void tile_count(const int *__restrict__ pairptr, const int *__restrict__ cellptr, int nlist, int chunk, int tq, int tr,
                           int *__restrict__ tcnt)
{
    const int L = blockIdx.x * blockDim.x + threadIdx.x;
    if (L >= nlist) return;
    const int nq = pairptr[L + 1] - pairptr[L];
    const int rs = min(cellptr[L] + chunk * DBC, cellptr[L + 1]), re = min(cellptr[L + 1], rs + DBC);
    tcnt[L] = ((nq + tq - 1) / tq) * ((re - rs + tr - 1) / tr);
}

// out[i] = in[0] + .. + in[i-1], i = 0 .. m (one workgroup; the sums stay below 2^31 as the callers size things)
__global__ __launch_bounds__(1024) void excl_scan_k(const int *__restrict__ in, int m, int *__restrict__ out)
{
    __shared__ int ws[16];
    const int per = (m + 1023) / 1024;
    const int b = min((int)threadIdx.x * per, m), e = min(b + per, m);
    int a = 0;
    for (int i = b; i < e; ++i) a += in[i];
    int inc = a;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int t = __shfl_up(inc, o, WAVE);
        if (lane_id() >= o) inc += t;
    }
    if (lane_id() == WAVE - 1) ws[threadIdx.x >> 6] = inc;
    __syncthreads();
    int base = 0;
    for (int q = 0; q < (int)(threadIdx.x >> 6); ++q) base += ws[q];
    int pre = base + inc - a;
    for (int i = b; i < e; ++i) { const int v = in[i]; out[i] = pre; pre += v; }
    if (threadIdx.x == 1023) out[m] = pre;
}

// rows list[0 .. m) of a numbering that maps to X by map (null: itself): their rows in X, and their norms
__global__ void pick_rows_k(const int *__restrict__ list, int m, int n, const int *__restrict__ map,
                            const float *__restrict__ norms, int *__restrict__ xrow, float *__restrict__ norms_out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    const int p = min(max(list[i], 0), n - 1);
    xrow[i] = map ? map[p] : p;
    norms_out[i] = norms[p];
}

// the evenly spaced sample of m of n rows: floor(i n / m)
__global__ void sample_rows_k(int *__restrict__ rows, int n, int m)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) rows[i] = (int)(((long long)i * n) / m);
}

__global__ void fill_int_k(int *__restrict__ a, int v, int m)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) a[i] = v;
}

// Queries without a certificate: exact distances to every row of their tau lists.  One workgroup per failed
// query f (row rows[f] of the list order): key t of its `stride` slots is the ordered distance to the t-th row
// of its lists taken in probe order, ids[t] that row's number in X; counts[f] = how many there are.
__global__ __launch_bounds__(256) void ivf_exact_keys(const float *__restrict__ X, int n, int d, const int *__restrict__ rows,
                                                      const int32_t *__restrict__ probe_l, int tau,
                                                      const int *__restrict__ cellptr, const int *__restrict__ lorder,
                                                      size_t stride, uint64_t *__restrict__ okey, int *__restrict__ ids,
                                                      int *__restrict__ counts)
{
    extern __shared__ __align__(16) unsigned char smem[];
    float *xi = reinterpret_cast<float *>(smem);
    const int f = blockIdx.x;
    const int pos = min(max(rows[f], 0), n - 1);
    const float *x = X + (size_t)min(max(lorder[pos], 0), n - 1) * d;
    for (int t = threadIdx.x; t < d; t += blockDim.x) xi[t] = x[t];
    __syncthreads();
    const int w = threadIdx.x >> 6;
    size_t off = 0;
    for (int r = 0; r < tau; ++r) {
        const int L = probe_l[(size_t)pos * tau + r];
        const int rs = cellptr[L], m = cellptr[L + 1] - rs;
        for (int u = w; u < m; u += 4) {
            if (off + u >= stride) break;
            const int row = min(max(lorder[rs + u], 0), n - 1);
            const float *y = X + (size_t)row * d;
            double sum = 0.0;
            for (int t = lane_id(); t < d; t += WAVE) { const double df = (double)xi[t] - (double)y[t]; sum += df * df; }
            sum = wave_sum(sum);
            if (lane_id() == 0) {
                okey[(size_t)f * stride + off + u] = rs + u == pos ? ~0ull : orderable64(sum);
                ids[(size_t)f * stride + off + u] = row;
            }
        }
        off += (size_t)m;
    }
    if (threadIdx.x == 0) counts[f] = (int)(off < stride ? off : stride);
}


struct Layout {
    float *norms, *norm_max, *tau;
    int *cnt, *fail_count, *fail_rows, *extra, *cursor, *unconv;
    float *mu;               // column means (d rounded up to SLAB)
    double *mu_part;         // their partial sums, MEAN_CHUNKS x d
    uint64_t *cand, *sort_scratch;
    uint16_t *xs;            // the split copy of X
    uint16_t *xh, *xsf;      // long rows: the high parts alone; the split copy of the rows of the second sweep
    float *norms_f;          // their norms
    int *fail2_count, *fail2_rows;
    int *clist, *ccount;     // rows of the current query block that need compaction, and how many (two counters take turns)
    int32_t *knn_idx;
    double *knn_d2, *cond;
    int kp, cap;
    bool high_fits;          // there is room for the half-precision sweep
    // the search in an order of the rows (see ORD_MIN_ROWS); ord is null where n, d and k are not in its range
    int *ord, *prow, *prank, *bcnt, *bcur, *bptr, *rest_count, *rest_most;
    int32_t *label;
    uint16_t *pivots, *first, *rest;
    float *norms_p, *centre, *radius2, *near;
};

int margin_kp(int n, int k)
{
    int kp = k + (k / 2 > 32 ? k / 2 : 32);
    if (kp > n - 1) kp = n - 1;
    return kp;
}

bool ordered_size(int n, int d);
int pivot_count(int n);

size_t carve(Layout *L, int n, int d, int k, char *base)
{
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = base ? base + off : nullptr; off += up(bytes); return (void *)p; };
    const int kp = margin_kp(n, k);
    const int cap = kp + COMPACT_SLACK + COMPACT_EVERY * DBC;
    const size_t qb = (size_t)(n < QB ? n : QB);
    void *q;
    q = take(4 * (size_t)n); if (L) L->norms = (float *)q;
    q = take(4); if (L) L->norm_max = (float *)q;
    q = take(4 * qb); if (L) L->tau = (float *)q;
    q = take(4 * qb); if (L) L->cnt = (int *)q;
    q = take(4 * qb); if (L) L->clist = (int *)q;
    q = take(8); if (L) L->ccount = (int *)q;
    q = take(4); if (L) L->fail_count = (int *)q;
    q = take(4 * (size_t)n); if (L) L->fail_rows = (int *)q;
    q = take(4 * (size_t)n); if (L) L->extra = (int *)q;
    q = take(4 * (size_t)n); if (L) L->cursor = (int *)q;
    q = take(4); if (L) L->unconv = (int *)q;
    q = take(4 * (size_t)((d + SLAB - 1) / SLAB * SLAB)); if (L) L->mu = (float *)q;
    q = take(8 * (size_t)MEAN_CHUNKS * d); if (L) L->mu_part = (double *)q;
    q = take(8 * qb * cap); if (L) L->cand = (uint64_t *)q;
    q = take(8 * (size_t)2 * n * k); if (L) L->sort_scratch = (uint64_t *)q;
    q = take(4 * (size_t)n * k); if (L) L->knn_idx = (int32_t *)q;
    q = take(8 * (size_t)n * k); if (L) L->knn_d2 = (double *)q;
    q = take(8 * (size_t)n * k); if (L) L->cond = (double *)q;
    q = take(4 * (size_t)n * ((d + SLAB - 1) / SLAB * SLAB)); if (L) L->xs = (uint16_t *)q;
    if (d >= HIGH_FIRST_MIN_D) {
        q = take(2 * (size_t)n * ((d + 2 * SLAB - 1) / (2 * SLAB) * (2 * SLAB))); if (L) L->xh = (uint16_t *)q;
        q = take(4 * qb * ((d + SLAB - 1) / SLAB * SLAB)); if (L) L->xsf = (uint16_t *)q;
        q = take(4 * qb); if (L) L->norms_f = (float *)q;
        q = take(4); if (L) L->fail2_count = (int *)q;
        q = take(4 * (size_t)n); if (L) L->fail2_rows = (int *)q;
    }
    if (L) L->ord = nullptr;
    if (L) {
        L->kp = kp;
        L->cap = cap;
        L->high_fits = d >= HIGH_FIRST_MIN_D;
        if (!L->high_fits) {
            // the half-precision sweep of shorter rows lives where the rows of P are sorted later (its last list where
            // their extra entries are counted off), if that is large enough: 2 n dph + 4 min(n, QB) dp bytes in 16 n k
            const size_t dp = (size_t)(d + SLAB - 1) / SLAB * SLAB, dph = (size_t)(d + 2 * SLAB - 1) / (2 * SLAB) * (2 * SLAB);
            char *p = (char *)L->sort_scratch;
            L->xh = (uint16_t *)p; p += up(2 * (size_t)n * dph);
            L->xsf = (uint16_t *)p; p += up(4 * qb * dp);
            L->norms_f = (float *)p; p += up(4 * qb);
            L->high_fits = (size_t)(p - (char *)L->sort_scratch) <= 16 * (size_t)n * k;
            L->fail2_count = L->fail_count + 16;         // (a count has 256 bytes to itself)
            L->fail2_rows = L->cursor;
        }
        if (ordered_size(n, d)) {
            // what the search in an order of the rows needs lives there too, if it fits: some 8 n + 2.2 n + 2 MB (m and the
            // query tiles are bounded) in 16 n k
            const size_t m = (size_t)pivot_count(n), ntiles = ((size_t)n + HT - 1) / HT, qtiles = (qb + HT - 1) / HT;
            const size_t dp = (size_t)(d + SLAB - 1) / SLAB * SLAB;
            char *p = (char *)L->sort_scratch;
            auto put = [&](size_t bytes) { char *at = p; p += up(bytes); return (void *)at; };
            L->ord = (int *)put(4 * (size_t)n);
            L->label = (int32_t *)put(4 * (size_t)n);
            L->prow = (int *)put(4 * m);
            L->prank = (int *)put(4 * m);
            L->norms_p = (float *)put(4 * m);
            L->bcnt = (int *)put(4 * (m + 1));
            L->bcur = (int *)put(4 * (m + 1));
            L->bptr = (int *)put(4 * (m + 1));
            L->pivots = (uint16_t *)put(4 * m * dp);
            L->centre = (float *)put(4 * ntiles * d);
            L->radius2 = (float *)put(4 * ntiles);
            L->near = (float *)put(4 * qtiles * ntiles);
            L->first = (uint16_t *)put(2 * qtiles * ORD_FIRST);
            L->rest = (uint16_t *)put(2 * qtiles * ORD_MAX_TILES);
            L->rest_count = (int *)put(4 * qtiles);
            L->rest_most = (int *)put(4);
            if ((size_t)(p - (char *)L->sort_scratch) > 16 * (size_t)n * k) L->ord = nullptr;
        }
    }
    return off;
}

bool ordered_size(int n, int d) { return d <= 2 * SLAB && n >= ORD_MIN_ROWS && n <= ORD_MAX_TILES * HT; }
int pivot_count(int n) { return std::min(ORD_MAX_PIVOTS, std::max(16, n / 2048)); }

int check_args(int32_t n, int32_t d, int32_t k)
{
    if (n < 2 || d < 1 || k < 1 || k >= n) return TSNE_EINVAL;
    if (k + (k / 2 > 32 ? k / 2 : 32) > MAX_KP || d > 4096) return TSNE_EINVAL;
    if ((int64_t)2 * n * k > 0x7FFFFFFFll) return TSNE_EINVAL;
    return TSNE_OK;
}

}  // namespace

#define HIPCHK(call)                                      \
    do {                                                  \
        hipError_t e_ = (call);                           \
        if (e_ != hipSuccess) {                           \
            fprintf(stderr, "tsne_build_P: %s failed: %s\n", #call, hipGetErrorString(e_)); \
            return TSNE_EHIP;                             \
        }                                                 \
    } while (0)

// ---- Eq. (10)-(11) with a flat second stage, rows longer than the double-precision kernels like
// The k nearest of the points in a query's tau probed lists, found the way tsne_build_P finds neighbours among all
// points: candidates from bf16 matrix-core tiles on the centred rows (here the tiles of (queries probing a list) x
// (rows of the list), queries grouped by list once per probe rank), exact distances in double for the k' best,
// a certificate per query, and an exact pass over its lists for a query without one.  The result is Eq. (11)'s by
// (distance in double, row number).  probe: n x tau list numbers (Eq. (10)), lorder: the rows in list order,
// cellptr: where each list starts in it; max_list and max_cand (longest list, most rows in one query's lists) from the caller.
namespace {
struct TileSearchLayout {
    float *norms, *norm_max, *tau, *mu;
    double *mu_part;
    int *cnt, *clist, *ccount, *fail_count, *fail_rows, *bcnt, *bcur, *pairptr, *tcnt, *tptr, *pairq, *fcnt;
    int *fail2_count, *fail2_rows, *xrow;      // a second sweep: rows it fails, and its queries' rows in X and norms
    float *norms_f;
    int32_t *probe_l;
    uint64_t *cand;
    uint16_t *xs;
    size_t cand_bytes;
};
constexpr int TS_ROWS = 1 << 17;     // queries per pass
// queries without a certificate from which on a second sweep is quicker than exact distances: those read all rows of a
// query's lists for it alone, or compare it with every centroid (4096 queries a launch of some 0.8 ms)
constexpr int SECOND_SWEEP_MIN = 1024, PROBE_SWEEP_MIN = 8192;

size_t ts_carve(TileSearchLayout *L, int n, int d, int k, int nlist, int tau, char *base)
{
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = base ? base + off : nullptr; off += up(bytes); return (void *)p; };
    const int kp = margin_kp(n, k);
    const size_t cap = (size_t)kp + COMPACT_SLACK + COMPACT_EVERY * DBC;
    const size_t qb = (size_t)(n < TS_ROWS ? n : TS_ROWS);
    const size_t dp = ((size_t)d + SLAB - 1) / SLAB * SLAB;
    void *q;
    q = take(4 * (size_t)n); if (L) L->norms = (float *)q;
    q = take(4); if (L) L->norm_max = (float *)q;
    q = take(4 * qb); if (L) L->tau = (float *)q;
    q = take(4 * dp); if (L) L->mu = (float *)q;
    q = take(8 * (size_t)MEAN_CHUNKS * d); if (L) L->mu_part = (double *)q;
    q = take(4 * qb); if (L) L->cnt = (int *)q;
    q = take(4 * qb); if (L) L->clist = (int *)q;
    q = take(8); if (L) L->ccount = (int *)q;
    q = take(4); if (L) L->fail_count = (int *)q;
    q = take(4 * (size_t)n); if (L) L->fail_rows = (int *)q;
    q = take(4); if (L) L->fail2_count = (int *)q;
    q = take(4 * (size_t)n); if (L) L->fail2_rows = (int *)q;
    q = take(4 * (size_t)n); if (L) L->xrow = (int *)q;
    q = take(4 * (size_t)n); if (L) L->norms_f = (float *)q;
    q = take(4 * ((size_t)nlist + 1)); if (L) L->bcnt = (int *)q;
    q = take(4 * ((size_t)nlist + 1)); if (L) L->bcur = (int *)q;
    q = take(4 * ((size_t)nlist + 1)); if (L) L->pairptr = (int *)q;
    q = take(4 * ((size_t)nlist + 1)); if (L) L->tcnt = (int *)q;
    q = take(4 * ((size_t)nlist + 1)); if (L) L->tptr = (int *)q;
    q = take(4 * qb); if (L) L->pairq = (int *)q;
    q = take(4 * (size_t)(2 * k > 1 ? 2 * k : 1)); if (L) L->fcnt = (int *)q;
    q = take(4 * (size_t)n * tau); if (L) L->probe_l = (int32_t *)q;
    q = take(4 * (size_t)n * dp); if (L) L->xs = (uint16_t *)q;
    // candidate buffers; afterwards the keys and row numbers of the exact pass (12 bytes a slot, at least one query's n slots)
    size_t cb = 8 * qb * cap;
    if (cb < 12 * (size_t)n) cb = 12 * (size_t)n;
    q = take(cb); if (L) { L->cand = (uint64_t *)q; L->cand_bytes = cb; }
    return off;
}
}  // namespace

int ivf_search_tiles(const float *X, int n, int d, int k, int nlist, int tau, const int32_t *probe, const int *lorder,
                     const int *cellptr, int max_list, long long max_cand, int32_t *knn_idx, double *knn_d2, void *ws,
                     size_t ws_bytes, hipStream_t s)
{
    if (check_args(n, d, k) != TSNE_OK || nlist < 1 || tau < 1 || max_list < 1 || max_cand < 1) return TSNE_EINVAL;
    if (ws_bytes < ts_carve(nullptr, n, d, k, nlist, tau, nullptr)) return TSNE_ENOSPC;
    TileSearchLayout L;
    ts_carve(&L, n, d, k, nlist, tau, (char *)ws);
    const int kp = margin_kp(n, k), cap = kp + COMPACT_SLACK + COMPACT_EVERY * DBC;
    const int dp = (d + SLAB - 1) / SLAB * SLAB;
    launch_col_mean(X, n, d, dp, L.mu_part, L.mu, s);
    hipLaunchKernelGGL(row_norms, wide_grid((size_t)n * WAVE), dim3(256), 0, s, X, L.mu, n, d, lorder, n, L.norms);
    hipLaunchKernelGGL(max_norm_k, dim3(1), dim3(1024), 0, s, L.norms, n, L.norm_max);
    hipLaunchKernelGGL(probe_gather, wide_grid((size_t)n * tau), dim3(256), 0, s, probe, lorder, n, tau, nlist, L.probe_l);
    HIPCHK(hipMemsetAsync(L.fail_count, 0, 4, s));
    HIPCHK(hipMemsetAsync(L.fail2_count, 0, 4, s));
    float norm_max = 0.f;
    HIPCHK(hipMemcpyAsync(&norm_max, L.norm_max, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const size_t rerank_smem = rerank_lds_bytes(d, kp);
    const int nchunks = (max_list + DBC - 1) / DBC;
    const unsigned lb = (unsigned)((nlist + 1 + 255) / 256);
    // As in tsne_build_P: a first sweep with the values in half precision, whose certificate holds for nearly every query
    // of ordinary data, the three-product tiles for the queries it fails (or for all passes that follow one of which it fails
    // half), exact distances for a few.  The copies take turns in L.xs (2 n dph <= 4 n dp bytes from 33 columns on).
    // (1,281,167 x 2048, four lists a query: tiles of a pass 8.35 -> 1.6 ms, quantizer and lists together 688 -> 360 ms.)
    const int dph = (d + 2 * SLAB - 1) / (2 * SLAB) * (2 * SLAB);
    const float xmax = sqrtf(norm_max) * 1.0001f;      // (no value is larger than its row's norm, whose square is a rounded sum)
    const bool half_first = d > KFLUSH && half_scales(xmax);
    HalfScale hs = {};
    if (half_first) {
        hs = half_scale(xmax, d, norm_max);
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&knn_tile_half_lists),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)HALF_GATHER_LDS));
        hipLaunchKernelGGL(split_high, wide_grid((size_t)n * (dph / 8)), dim3(256), 0, s, X, L.mu, n, d, dph, hs.scale, lorder, n, L.xs);
    }
    auto split = [&]() {
        hipLaunchKernelGGL(split_bf16, wide_grid((size_t)n * dp), dim3(256), 0, s, X, L.mu, n, d, dp, lorder, n, L.xs);
    };
    // queries q0 .. q0 + rows (of qmap, or of the list order) against their lists
    auto pass = [&](bool half, const int *qmap, int q0, int rows, int *fail_count, int *fail_rows) {
        hipLaunchKernelGGL(knn_reset, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, rows, L.ccount);
        // an upper bound of the tiles of one launch: sum over the lists of ceil(queries / 128) x (DBC / TN)
        const int tq = half ? HT : 128, tr = half ? DBC : TN;
        const unsigned bound = (unsigned)(((size_t)rows / tq + (size_t)nlist + 1) * (DBC / tr));
        for (int r = 0; r < tau; ++r) {
            hipLaunchKernelGGL(fill_int_k, dim3(lb), dim3(256), 0, s, L.bcnt, 0, nlist + 1);
            hipLaunchKernelGGL(fill_int_k, dim3(lb), dim3(256), 0, s, L.bcur, 0, nlist + 1);
            hipLaunchKernelGGL(rank_hist, wide_grid((size_t)rows), dim3(256), 0, s, L.probe_l, qmap, q0, rows, tau, r, L.bcnt);
            hipLaunchKernelGGL(excl_scan_k, dim3(1), dim3(1024), 0, s, L.bcnt, nlist, L.pairptr);
            hipLaunchKernelGGL(rank_scatter, wide_grid((size_t)rows), dim3(256), 0, s, L.probe_l, qmap, q0, rows, tau, r, L.pairptr,
                               L.bcur, L.pairq);
            for (int c = 0; c < nchunks; ++c) {
                const bool dense = half && r == 0 && c == 0;
                hipLaunchKernelGGL(tile_count, dim3(lb), dim3(256), 0, s, L.pairptr, cellptr, nlist, c, tq, tr, L.tcnt);
                hipLaunchKernelGGL(excl_scan_k, dim3(1), dim3(1024), 0, s, L.tcnt, nlist, L.tptr);
                if (half)
                    hipLaunchKernelGGL(knn_tile_half_lists, dim3(bound), dim3(HALF_THREADS), HALF_GATHER_LDS, s,
                                       (const uint4 *)L.xs, dph, q0, q0 + rows, L.norms, L.tau, L.cnt, L.cand, cap, L.ccount,
                                       hs.dot_scale, L.tptr, nlist, L.pairptr, L.pairq, cellptr, c, dense ? 1 : 0);
                else
                    hipLaunchKernelGGL((knn_tile_mfma<2, true, true>), dim3(bound), dim3(256), 0, s, (const uint4 *)L.xs, dp, q0,
                                       q0 + rows, 0, 0, L.norms, L.tau, L.cnt, L.cand, cap, L.ccount, (const uint4 *)L.xs, L.norms, 1,
                                       qmap, L.tptr, nlist, L.pairptr, L.pairq, cellptr, c);
                const int force = r == tau - 1 && c == nchunks - 1 ? 1 : 0;
                hipLaunchKernelGGL(knn_compact_list, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, cap, kp, rows, force,
                                   L.clist, L.ccount);
                launch_compact(L.tau, L.cnt, L.cand, cap, kp, rows, L.clist, L.ccount, dense ? std::min(max_list, DBC) : 0, s);
            }
        }
        hipLaunchKernelGGL(knn_rerank, dim3((unsigned)((rows + 7) / 8 * 8)), dim3(256), rerank_smem, s, X, n, d,
                           qmap ? (const int *)L.xrow : lorder, X, n, lorder, qmap ? (const int *)L.xrow : lorder, qmap, q0, rows, k, kp,
                           0x7FFFFFFF, half ? tile_error_coeff(d, false, true) : tile_error_coeff(d, true), half ? hs.e_add : 0.0,
                           qmap ? (const float *)L.norms_f : L.norms, norm_max, L.tau, L.cnt, L.cand, cap, knn_idx, knn_d2, fail_count,
                           fail_rows, (const int *)nullptr);
    };
    bool half = half_first;
    if (!half) split();
    int nfail = 0;
    for (int q0 = 0; q0 < n; q0 += TS_ROWS) {
        const int rows = n - q0 < TS_ROWS ? n - q0 : TS_ROWS;
        // (three products after all: what those cannot certify goes to the exact pass)
        pass(half, nullptr, q0, rows, half == half_first ? L.fail_count : L.fail2_count, half == half_first ? L.fail_rows : L.fail2_rows);
        HIPCHK(hipGetLastError());
        if (half && q0 + rows < n) {        // (behind every pass: the lists of one say little about those of the next)
            const int before = nfail;
            HIPCHK(hipMemcpyAsync(&nfail, L.fail_count, 4, hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            if (nfail - before > rows / 2) { half = false; split(); }
        }
    }
    HIPCHK(hipMemcpyAsync(&nfail, L.fail_count, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const int *exact_rows = L.fail_rows;
    // A second sweep pays from some hundreds of queries on: an exact one reads all rows of its lists by itself.
    if (half != half_first || (half_first && nfail > SECOND_SWEEP_MIN)) {
        if (half) split();
        hipLaunchKernelGGL(pick_rows_k, dim3((nfail + 255) / 256 + 1), dim3(256), 0, s, L.fail_rows, nfail, n, lorder, L.norms, L.xrow,
                           L.norms_f);
        for (int f0 = 0; f0 < nfail; f0 += TS_ROWS)
            pass(false, L.fail_rows, f0, nfail - f0 < TS_ROWS ? nfail - f0 : TS_ROWS, L.fail2_count, L.fail2_rows);
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(&nfail, L.fail2_count, 4, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        exact_rows = L.fail2_rows;
    }
    if (nfail > 0) {
        const size_t stride = (size_t)max_cand;
        size_t nb_max = L.cand_bytes / (12 * stride);
        if (nb_max > (size_t)(2 * k)) nb_max = (size_t)(2 * k);
        if (nb_max < 1) return TSNE_ENOSPC;
        uint64_t *okey = L.cand;
        int *ids = reinterpret_cast<int *>(okey + nb_max * stride);
        for (int f0 = 0; f0 < nfail; f0 += (int)nb_max) {
            const int nb = nfail - f0 < (int)nb_max ? nfail - f0 : (int)nb_max;
            hipLaunchKernelGGL(ivf_exact_keys, dim3(nb), dim3(256), up((size_t)d * 4), s, X, n, d, exact_rows + f0, L.probe_l, tau,
                               cellptr, lorder, stride, okey, ids, L.fcnt);
            hipLaunchKernelGGL(knn_exact_select, dim3(nb), dim3(1024), 0, s, okey, stride, 0, L.fcnt, ids, k, exact_rows + f0,
                               lorder, n, knn_idx, knn_d2);
            HIPCHK(hipGetLastError());
        }
    }
    return TSNE_OK;
}

// ---- Eq. (10) for long rows: the tau nearest centroids of m rows of X (all rows, or the evenly spaced sample
// floor(i n / m) that k-means works on), by (distance in double, centroid number).  The same scheme once more:
// candidates from the tiles (queries against centroids, both centred on X's column means), the tau + 32 best
// re-ranked in double, a certificate, and all centroids in double for a query without one.
namespace {
struct TileProbeLayout {
    float *norms_q, *norms_c, *norm_max, *norms_f, *tau, *mu;      // norm_max: of the centroids, then of the queries
    double *mu_part;
    int *cnt, *clist, *ccount, *fail_count, *fail_rows, *fail2_count, *fail2_rows, *xrow, *qrows;
    uint64_t *cand;
    uint16_t *xs, *cs;
    size_t cand_bytes;
};

// (centroids are far apart against the error of a tile distance: eight spare candidates certify nearly every query)
int probe_kp(int nlist, int tau) { return tau + 8 < nlist ? tau + 8 : nlist; }

size_t tp_carve(TileProbeLayout *L, int n, int d, int nlist, int tau, char *base)
{
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = base ? base + off : nullptr; off += up(bytes); return (void *)p; };
    const size_t cap = (size_t)probe_kp(nlist, tau) + COMPACT_SLACK + COMPACT_EVERY * DBC;
    const size_t qb = (size_t)(n < TS_ROWS ? n : TS_ROWS);
    const size_t dp = ((size_t)d + SLAB - 1) / SLAB * SLAB;
    void *q;
    q = take(4 * (size_t)n); if (L) L->norms_q = (float *)q;
    q = take(4 * (size_t)nlist); if (L) L->norms_c = (float *)q;
    q = take(8); if (L) L->norm_max = (float *)q;
    q = take(4 * (size_t)n); if (L) L->norms_f = (float *)q;
    q = take(4 * qb); if (L) L->tau = (float *)q;
    q = take(4 * dp); if (L) L->mu = (float *)q;
    q = take(8 * (size_t)MEAN_CHUNKS * d); if (L) L->mu_part = (double *)q;
    q = take(4 * qb); if (L) L->cnt = (int *)q;
    q = take(4 * qb); if (L) L->clist = (int *)q;
    q = take(8); if (L) L->ccount = (int *)q;
    q = take(4); if (L) L->fail_count = (int *)q;
    q = take(4 * (size_t)n); if (L) L->fail_rows = (int *)q;
    q = take(4); if (L) L->fail2_count = (int *)q;
    q = take(4 * (size_t)n); if (L) L->fail2_rows = (int *)q;
    q = take(4 * (size_t)n); if (L) L->xrow = (int *)q;
    q = take(4 * (size_t)n); if (L) L->qrows = (int *)q;
    q = take(4 * (size_t)n * dp); if (L) L->xs = (uint16_t *)q;
    q = take(4 * (size_t)nlist * dp); if (L) L->cs = (uint16_t *)q;
    size_t cb = 8 * qb * cap;
    if (cb < 8 * (size_t)nlist) cb = 8 * (size_t)nlist;      // the exact pass: at least one query's keys
    q = take(cb); if (L) { L->cand = (uint64_t *)q; L->cand_bytes = cb; }
    return off;
}
}  // namespace

// workspace of ivf_probe_tiles and, if k > 0, of ivf_search_tiles, which run one after the other (0: not for these sizes)
size_t ivf_tiles_workspace(int n, int d, int k, int nlist, int tau)
{
    if (n < 2 || d < 1 || d > 4096 || nlist < 1 || tau < 1 || tau > nlist) return 0;
    size_t a = tp_carve(nullptr, n, d, nlist, tau, nullptr), b = 0;
    if (k > 0) {
        if (check_args(n, d, k) != TSNE_OK) return 0;
        b = ts_carve(nullptr, n, d, k, nlist, tau, nullptr);
    }
    return a > b ? a : b;
}

// queries: what the workspace holds of the query side (column means, sample rows, norms, copy) from a previous call with
// the same X, n, d and m (the rounds of k-means: only the centroids change); left as what it holds now.
// As in tsne_build_P: the values in half precision first, three products for the queries that leaves without a certificate.
// (131,072 x 1132 x 2048 products: 2.10 -> 0.80 ms.)
int ivf_probe_tiles(const float *X, int n, int d, const float *C, int nlist, int tau, int m, int32_t *probe, void *ws,
                    size_t ws_bytes, hipStream_t s, ProbeQueries *queries)
{
    if (n < 2 || d < 1 || d > 4096 || nlist < 1 || tau < 1 || tau > nlist || m < 1 || m > n) return TSNE_EINVAL;
    if (ws_bytes < tp_carve(nullptr, n, d, nlist, tau, nullptr)) return TSNE_ENOSPC;
    TileProbeLayout L;
    tp_carve(&L, n, d, nlist, tau, (char *)ws);
    const int kp = probe_kp(nlist, tau), cap = kp + COMPACT_SLACK + COMPACT_EVERY * DBC;
    const int dp = (d + SLAB - 1) / SLAB * SLAB, dph = (d + 2 * SLAB - 1) / (2 * SLAB) * (2 * SLAB);
    const int *rowmap = m < n ? L.qrows : nullptr;
    if (queries->copy == ProbeQueries::NONE) {
        launch_col_mean(X, n, d, dp, L.mu_part, L.mu, s);
        if (m < n) hipLaunchKernelGGL(sample_rows_k, dim3((m + 255) / 256), dim3(256), 0, s, L.qrows, n, m);
        hipLaunchKernelGGL(row_norms, wide_grid((size_t)m * WAVE), dim3(256), 0, s, X, L.mu, m, d, rowmap, n, L.norms_q);
        hipLaunchKernelGGL(max_norm_k, dim3(1), dim3(1024), 0, s, L.norms_q, m, L.norm_max + 1);
    }
    hipLaunchKernelGGL(row_norms, wide_grid((size_t)nlist * WAVE), dim3(256), 0, s, C, L.mu, nlist, d, (const int *)nullptr, nlist,
                       L.norms_c);
    hipLaunchKernelGGL(max_norm_k, dim3(1), dim3(1024), 0, s, L.norms_c, nlist, L.norm_max);
    HIPCHK(hipMemsetAsync(L.fail_count, 0, 4, s));
    HIPCHK(hipMemsetAsync(L.fail2_count, 0, 4, s));
    float norm_max2[2] = {0.f, 0.f};
    HIPCHK(hipMemcpyAsync(norm_max2, L.norm_max, 8, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const float norm_max = norm_max2[0];
    auto split_queries = [&]() {
        hipLaunchKernelGGL(split_bf16, wide_grid((size_t)m * dp), dim3(256), 0, s, X, L.mu, m, d, dp, rowmap, n, L.xs);
        queries->copy = ProbeQueries::SPLIT;
    };
    auto split_centroids = [&]() {
        hipLaunchKernelGGL(split_bf16, wide_grid((size_t)nlist * dp), dim3(256), 0, s, C, L.mu, nlist, d, dp, (const int *)nullptr, nlist, L.cs);
    };
    // the scale is the queries' (it has to stay what it was when they were copied); centroids are means of rows, but a
    // caller's may be anything: 2^15 for the queries leaves them a factor of two, and 1e30 keeps everything finite
    HalfScale hs = {};
    const float xmax = sqrtf(norm_max2[1]) * 1.0001f;
    bool half = d > KFLUSH && !queries->no_half && half_scales(xmax);
    if (half) {
        hs = half_scale(xmax, d, std::max(norm_max, norm_max2[1]));
        half = sqrtf(norm_max) * 1.0001f * hs.scale < 60000.f;
    }
    if (half) {
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&knn_tile_half_other<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)HALF_TILE_LDS));
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&knn_tile_half_other<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)HALF_TILE_LDS));
        if (queries->copy != ProbeQueries::HALF) {
            hipLaunchKernelGGL(split_high, wide_grid((size_t)m * (dph / 8)), dim3(256), 0, s, X, L.mu, m, d, dph, hs.scale, rowmap, n, L.xs);
            queries->copy = ProbeQueries::HALF;
        }
        hipLaunchKernelGGL(split_high, wide_grid((size_t)nlist * (dph / 8)), dim3(256), 0, s, C, L.mu, nlist, d, dph, hs.scale,
                           (const int *)nullptr, nlist, L.cs);
    } else {
        if (queries->copy != ProbeQueries::SPLIT) split_queries();
        split_centroids();
    }
    const size_t rerank_smem = rerank_lds_bytes(d, kp);
    // queries q0 .. q0 + rows of the copy in L.xs; qmap, norms: where they are in X, their norms; omap: whose they are
    auto pass = [&](bool half, int q0, int rows, const int *qmap, const float *norms, const int *omap, int *fail_count, int *fail_rows) {
        hipLaunchKernelGGL(knn_reset, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, rows, L.ccount);
        for (int j0 = 0, jend; j0 < nlist; j0 = jend) {
            jend = j0 + DBC < nlist ? j0 + DBC : nlist;
            const int force = jend >= nlist ? 1 : 0;
            auto tiles = [&](auto kernel, int tq) {
                hipLaunchKernelGGL(kernel, dim3((unsigned)((rows + tq - 1) / tq), (unsigned)((jend - j0 + TN - 1) / TN)), dim3(256), 0, s,
                                   (const uint4 *)L.xs, dp, q0, q0 + rows, j0, jend, norms, L.tau, L.cnt, L.cand, cap, L.ccount,
                                   (const uint4 *)L.cs, L.norms_c, 0, (const int *)nullptr, (const int *)nullptr, 0, (const int *)nullptr,
                                   (const int *)nullptr, (const int *)nullptr, 0);
            };
            if (half) {
                const unsigned nqt = (unsigned)((rows + HT - 1) / HT), njt = (unsigned)((jend - j0 + HT - 1) / HT);
                auto half_tiles = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, dim3(8 * ((nqt + 7) / 8) * njt), dim3(HALF_THREADS), HALF_TILE_LDS, s, (const uint4 *)L.xs, dph,
                                       q0, q0 + rows, j0, jend, norms, L.tau, L.cnt, L.cand, cap, L.ccount, hs.dot_scale,
                                       (const uint4 *)L.cs, L.norms_c);
                };
                if (j0 == 0) half_tiles(knn_tile_half_other<true>); else half_tiles(knn_tile_half_other<false>);
            } else if (d > KFLUSH) {
                if (j0 == 0) tiles(knn_tile_mfma<2, true, false, true>, 128);
                else tiles(knn_tile_mfma<2, true, false>, 128);
            } else {
                if (j0 == 0) tiles(knn_tile_mfma<KNN_MB, false, false, true>, 64 * KNN_MB);
                else tiles(knn_tile_mfma<KNN_MB, false, false>, 64 * KNN_MB);
            }
            hipLaunchKernelGGL(knn_compact_list, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, cap, kp, rows, force,
                               L.clist, L.ccount);
            launch_compact(L.tau, L.cnt, L.cand, cap, kp, rows, L.clist, L.ccount, j0 == 0 ? jend : 0, s);
        }
        hipLaunchKernelGGL(knn_rerank, dim3((unsigned)((rows + 7) / 8 * 8)), dim3(256), rerank_smem, s, X, n, d, qmap, C, nlist, (const int *)nullptr,
                           omap, omap, q0, rows, tau, kp, nlist, half ? tile_error_coeff(d, false, true) : tile_error_coeff(d, d > KFLUSH),
                           half ? hs.e_add : 0.0, norms, norm_max, L.tau, L.cnt, L.cand, cap, probe,
                           (double *)nullptr, fail_count, fail_rows, (const int *)nullptr);
    };
    for (int q0 = 0; q0 < m; q0 += TS_ROWS)
        pass(half, q0, m - q0 < TS_ROWS ? m - q0 : TS_ROWS, rowmap, L.norms_q, nullptr, L.fail_count, L.fail_rows);
    HIPCHK(hipGetLastError());
    int nfail = 0;
    HIPCHK(hipMemcpyAsync(&nfail, L.fail_count, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const int *exact_rows = L.fail_rows;
    if (half && nfail > PROBE_SWEEP_MIN) {
        // the queries without a certificate, a pass at a time in the place of the copy that just failed them
        queries->copy = ProbeQueries::NONE;
        if (nfail > m / 4) queries->no_half = true;       // (and no more of it in the rounds to come)
        split_centroids();
        hipLaunchKernelGGL(pick_rows_k, dim3((nfail + 255) / 256), dim3(256), 0, s, L.fail_rows, nfail, m, rowmap, L.norms_q, L.xrow, L.norms_f);
        hipLaunchKernelGGL(split_bf16, wide_grid((size_t)nfail * dp), dim3(256), 0, s, X, L.mu, nfail, d, dp, L.xrow, n, L.xs);
        for (int f0 = 0; f0 < nfail; f0 += TS_ROWS)
            pass(false, f0, nfail - f0 < TS_ROWS ? nfail - f0 : TS_ROWS, L.xrow, L.norms_f, L.fail_rows, L.fail2_count, L.fail2_rows);
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(&nfail, L.fail2_count, 4, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        exact_rows = L.fail2_rows;
    }
    if (nfail > 0) {
        size_t nb_max = L.cand_bytes / (8 * (size_t)nlist);
        if (nb_max > 4096) nb_max = 4096;
        if (nb_max < 1) return TSNE_ENOSPC;
        for (int f0 = 0; f0 < nfail; f0 += (int)nb_max) {
            const int nb = nfail - f0 < (int)nb_max ? nfail - f0 : (int)nb_max;
            hipLaunchKernelGGL(knn_exact_dists, wide_grid((size_t)nlist * WAVE), dim3(256), 0, s, X, n, rowmap, C, nlist, d,
                               exact_rows + f0, nb, 0, L.cand);
            hipLaunchKernelGGL(knn_exact_select, dim3(nb), dim3(1024), 0, s, L.cand, (size_t)nlist, nlist, (const int *)nullptr,
                               (const int *)nullptr, tau, exact_rows + f0, (const int *)nullptr, m, probe, (double *)nullptr);
            HIPCHK(hipGetLastError());
        }
    }
    return TSNE_OK;
}

extern "C" {

int tsne_build_P_workspace_bytes(int32_t n, int32_t d, int32_t k, size_t *bytes)
{
    if (!bytes || check_args(n, d, k) != TSNE_OK) return TSNE_EINVAL;
    *bytes = carve(nullptr, n, d, k, nullptr);
    return TSNE_OK;
}


// Alg. 1 line 2 from finished neighbour lists (L.knn_idx, L.knn_d2): Eq. (1) per row, then the symmetric CSR.
static int finish_P(const Layout &L, int32_t n, int32_t k, float perplexity, int32_t *d_row_ptr, int32_t *d_col,
                    float *d_val, int64_t cap_nnz, int64_t *nnz, int32_t *d_knn_idx, float *d_knn_d2,
                    int32_t *n_unconverged, int symmetric, hipStream_t s)
{
    const size_t nk = (size_t)n * k;
    double *reach = reinterpret_cast<double *>(L.sort_scratch);       // n of its 2 n k words, until the rows are sorted
    const size_t ps_bytes = PERP_ROWS * (size_t)k * 8;
    const int ps_staged = ps_bytes <= 60 * 1024 ? 1 : 0;
    hipLaunchKernelGGL(perplexity_search, dim3((n + PERP_ROWS - 1) / PERP_ROWS), dim3(256), ps_staged ? ps_bytes : 0, s, L.knn_d2, n, k,
                       log((double)perplexity), 1e-10, L.cond, reach, L.unconv, ps_staged);
    // (the candidate buffers are free by now and hold 2 n k bytes with room to spare: 2 n k < 2^31 <= 8 * 65536 * 4160
    // for a full query block, and 2 k < 8 * 4160 for a short one)
    int16_t *slots = reinterpret_cast<int16_t *>(L.cand);
    hipLaunchKernelGGL(sym_count, wide_grid(nk * 16), dim3(256), 0, s, L.knn_idx, n, k, L.extra, slots,
                       L.knn_d2, reach, symmetric);
    hipLaunchKernelGGL(sym_scan, dim3(1), dim3(1024), 0, s, L.extra, n, k, d_row_ptr, L.cursor);
    int32_t total = 0;
    HIPCHK(hipMemcpyAsync(&total, d_row_ptr + n, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if ((int64_t)total > cap_nnz) return TSNE_ENOSPC;
    hipLaunchKernelGGL(sym_fill, wide_grid(nk), dim3(256), 0, s, L.knn_idx, L.cond, n, k, d_row_ptr,
                       L.cursor, slots, d_col, d_val);
    // (the lists of rows without a certificate are done with)
    HIPCHK(hipMemsetAsync(L.fail_count, 0, 4, s));
    hipLaunchKernelGGL(sym_sort_rows, wide_grid((size_t)n * 256), dim3(128), 0, s, d_row_ptr, n, d_col, d_val, L.fail_rows, L.fail_count);
    hipLaunchKernelGGL(sym_sort_long, dim3(2048), dim3(1024), 0, s, d_row_ptr, n, d_col, d_val, L.sort_scratch, L.fail_rows, L.fail_count);
    if (d_knn_idx) HIPCHK(hipMemcpyAsync(d_knn_idx, L.knn_idx, 4 * nk, hipMemcpyDeviceToDevice, s));
    if (d_knn_d2)
        hipLaunchKernelGGL(d2_to_float, wide_grid(nk), dim3(256), 0, s, L.knn_d2, d_knn_d2, nk);
    int unconv = 0;
    HIPCHK(hipMemcpyAsync(&unconv, L.unconv, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    HIPCHK(hipGetLastError());
    *nnz = total;
    if (n_unconverged) *n_unconverged = unconv;
    return TSNE_OK;
}

int tsne_build_P(const float *d_X, int32_t n, int32_t d, float perplexity, int32_t k, int32_t *d_row_ptr,
                 int32_t *d_col, float *d_val, int64_t cap_nnz, int64_t *nnz, int32_t *d_knn_idx, float *d_knn_d2,
                 int32_t *n_unconverged, void *d_workspace, size_t workspace_bytes, void *stream)
{
    if (!d_X || !d_row_ptr || !d_col || !d_val || !nnz || !d_workspace) return TSNE_EINVAL;
    if (check_args(n, d, k) != TSNE_OK) return TSNE_EINVAL;
    if (!(perplexity > 0.0f) || !(perplexity <= (float)k)) return TSNE_EINVAL;
    if (((uintptr_t)d_workspace % ALIGN) != 0) return TSNE_EINVAL;
    if (workspace_bytes < carve(nullptr, n, d, k, nullptr)) return TSNE_ENOSPC;
    hipStream_t s = (hipStream_t)stream;
    Layout L;
    carve(&L, n, d, k, (char *)d_workspace);
    const int kp = L.kp, cap = L.cap;

    const int dp = (d + SLAB - 1) / SLAB * SLAB;
    launch_col_mean(d_X, n, d, dp, L.mu_part, L.mu, s);
    hipLaunchKernelGGL(row_norms, wide_grid((size_t)n * WAVE), dim3(256), 0, s, d_X, L.mu, n, d, (const int *)nullptr, n, L.norms);
    hipLaunchKernelGGL(max_norm_k, dim3(1), dim3(1024), 0, s, L.norms, n, L.norm_max);
    HIPCHK(hipMemsetAsync(L.fail_count, 0, 4, s));
    HIPCHK(hipMemsetAsync(L.unconv, 0, 4, s));
    HIPCHK(hipMemsetAsync(L.extra, 0, 4 * (size_t)n, s));
    float norm_max = 0.f;
    HIPCHK(hipMemcpyAsync(&norm_max, L.norm_max, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));

    // more LDS than a kernel may use by default
    const struct { const void *kernel; size_t bytes; } lds[] = {
        {reinterpret_cast<const void *>(&knn_tile_resident<1, false, false>), resident_lds_bytes(1)},
        {reinterpret_cast<const void *>(&knn_tile_resident<1, true, false>), resident_lds_bytes(1)},
        {reinterpret_cast<const void *>(&knn_tile_resident<2, false, false>), resident_lds_bytes(2)},
        {reinterpret_cast<const void *>(&knn_tile_resident<2, true, false>), resident_lds_bytes(2)},
        {reinterpret_cast<const void *>(&knn_tile_resident<1, false, true>), resident_lds_bytes(1)},
        {reinterpret_cast<const void *>(&knn_tile_resident<1, true, true>), resident_lds_bytes(1)},
        {reinterpret_cast<const void *>(&knn_tile_resident<2, false, true>), resident_lds_bytes(2)},
        {reinterpret_cast<const void *>(&knn_tile_resident<2, true, true>), resident_lds_bytes(2)},
        {reinterpret_cast<const void *>(&knn_tile_half<false, false>), HALF_TILE_LDS},
        {reinterpret_cast<const void *>(&knn_tile_half<true, false>), HALF_TILE_LDS},
        {reinterpret_cast<const void *>(&knn_tile_half<false, true>), HALF_OWN_LDS},
    };
    for (const auto &a : lds) HIPCHK(hipFuncSetAttribute(a.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.bytes));
    const size_t rerank_smem = rerank_lds_bytes(d, kp);
    auto compact = [&](int rows, const int *cc, int dense) {
        launch_compact(L.tau, L.cnt, L.cand, cap, kp, rows, L.clist, cc, dense, s);
    };
    // three-product tiles of query rows q0 .. qend (row fr[q] of X if fr is given) against database rows j0 .. jend
    auto mfma_tiles = [&](const uint16_t *xq, const float *norms_q, int q0, int qend, int j0, int jend, const int *fr, int *cc) {
        auto tiles = [&](auto kernel, int tq) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((qend - q0 + tq - 1) / tq), (unsigned)((jend - j0 + TN - 1) / TN)), dim3(256), 0,
                               s, (const uint4 *)xq, dp, q0, qend, j0, jend, norms_q, L.tau, L.cnt, L.cand, cap, cc,
                               (const uint4 *)L.xs, L.norms, 1, fr, (const int *)nullptr, 0, (const int *)nullptr,
                               (const int *)nullptr, (const int *)nullptr, 0);
        };
        if (d > KFLUSH) {
            if (j0 == 0) tiles(knn_tile_mfma<2, true, false, true>, 128); else tiles(knn_tile_mfma<2, true, false>, 128);
        } else {
            if (j0 == 0) tiles(knn_tile_mfma<KNN_MB, false, false, true>, 64 * KNN_MB);
            else tiles(knn_tile_mfma<KNN_MB, false, false>, 64 * KNN_MB);
        }
    };
    // Long rows: a first sweep with the values rounded to half precision (a third of the matrix work, half the bytes, a
    // coarser bound: 2^-10 of the norms instead of some 2^-15); its certificate still holds wherever the k-th and the k'-th
    // neighbour are farther apart than that, and only the rows it fails go through the three-product tiles.
    // From HIGH_FIRST_MIN_D columns on always.  Shorter rows beyond the resident kernel's take it if three things hold: the
    // tiles go query tile by query tile (k = 90: 50,000 rows of 72 and 200 coordinates 9.3 -> 6.5 and 11.3 -> 7.4 ms, 33,000 of
    // 100: 5.7 -> 4.5; 8000, where they do not: 1.0 -> 1.2); its buffers fit where the rows of P are sorted later, which
    // depends on k (see carve(): up to 65,536 rows that is k >= 0.375 d or so, d rounded up to 64, beyond it falls
    // to 0.125 d); and a sample's neighbours are far enough apart.
    const int nblocks = (n + QB - 1) / QB, block = ((n + nblocks - 1) / nblocks + HT - 1) / HT * HT;   // see the loop below
    bool high_first = d >= HIGH_FIRST_MIN_D || (dp > 2 * SLAB && (n < block ? n : block) >= HALF_OWN_MIN_ROWS && L.high_fits);
    const int dph = (d + 2 * SLAB - 1) / (2 * SLAB) * (2 * SLAB);
    float dot_scale = 1.0f;
    double e_add = 0.0;
    if (high_first) {
        HIPCHK(hipMemsetAsync(L.fail2_count, 0, 8, s));            // (borrowed for the largest magnitude and the sample's vote)
        hipLaunchKernelGGL(max_abs_centred, dim3(2048), dim3(256), 0, s, d_X, L.mu, n, d,
                           reinterpret_cast<unsigned int *>(L.fail2_count));
        if (d < HIGH_FIRST_MIN_D) {
            const int m = n < GAP_SAMPLE ? n : GAP_SAMPLE;
            const int r1 = (int)std::max<int64_t>(1, (int64_t)k * m / n), r2 = std::max(r1 + 1, (int)(((int64_t)kp * m + n - 1) / n));
            hipLaunchKernelGGL(half_gap_sample, dim3(GAP_QUERIES), dim3(1024), 0, s, d_X, n, d, m, r1, r2, L.norms, norm_max,
                               tile_error_coeff(d, false, true), L.fail2_count + 1);
        }
        int found[2] = {0, 0};
        HIPCHK(hipMemcpyAsync(found, L.fail2_count, 8, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        float xmax;
        memcpy(&xmax, &found[0], 4);
        if (!half_scales(xmax) || found[1] > GAP_QUERIES / 2) {
            // all rows equal, values half precision cannot scale, or neighbours it cannot tell apart
            high_first = false;
        } else {
            const HalfScale h = half_scale(xmax, d, norm_max);
            dot_scale = h.dot_scale;
            e_add = h.e_add;
            hipLaunchKernelGGL(split_high, wide_grid((size_t)n * (dph / 8)), dim3(256), 0, s, d_X, L.mu, n, d, dph, h.scale, (const int *)nullptr, n,
                               L.xh);
            HIPCHK(hipMemsetAsync(L.fail2_count, 0, 4, s));
        }
    }
    // the order of the rows that the copies and the norms are in (null: the caller's)
    const int *ord = nullptr;
    // (only where three-product tiles run: not if half precision certifies every row)
    auto split = [&]() {
        hipLaunchKernelGGL(split_bf16, wide_grid((size_t)n * dp), dim3(256), 0, s, d_X, L.mu, n, d, dp, ord, n, L.xs);
    };
    if (!high_first) split();
    const int ntiles = (n + HT - 1) / HT;
    if (L.ord) {
        // the nearest pivot of every row, from dense launches on the copies in the caller's order
        const int m = pivot_count(n);
        hipLaunchKernelGGL(sample_rows_k, dim3((m + 255) / 256), dim3(256), 0, s, L.prow, n, m);
        hipLaunchKernelGGL(row_norms, wide_grid((size_t)m * WAVE), dim3(256), 0, s, d_X, L.mu, m, d, L.prow, n, L.norms_p);
        hipLaunchKernelGGL(split_bf16, wide_grid((size_t)m * dp), dim3(256), 0, s, d_X, L.mu, m, d, dp, L.prow, n, L.pivots);
        auto against_pivots = [&](const uint16_t *xq, const float *norms_q, int q0, int qend) {
            hipLaunchKernelGGL((knn_tile_mfma<KNN_MB, false, false, true>), dim3((unsigned)((qend - q0 + 64 * KNN_MB - 1) / (64 * KNN_MB)), (unsigned)((m + TN - 1) / TN)),
                               dim3(256), 0, s, (const uint4 *)xq, dp, q0, qend, 0, m, norms_q, L.tau, L.cnt, L.cand, cap, L.ccount,
                               (const uint4 *)L.pivots, L.norms_p, 0, (const int *)nullptr, (const int *)nullptr, 0,
                               (const int *)nullptr, (const int *)nullptr, (const int *)nullptr, 0);
        };
        hipLaunchKernelGGL(knn_reset, dim3((QB + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, n < QB ? n : QB, L.ccount);
        against_pivots(L.pivots, L.norms_p, 0, m);
        hipLaunchKernelGGL(pivot_apart_k, dim3(1), dim3(ORD_MAX_PIVOTS), 0, s, L.cand, cap, m, L.rest_most);
        int apart = 0;
        HIPCHK(hipMemcpyAsync(&apart, L.rest_most, 4, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        if (apart >= m * (m - 1) / 4) ord = L.ord;
        if (ord) {
            hipLaunchKernelGGL(pivot_chain_k, dim3(1), dim3(ORD_MAX_PIVOTS), 0, s, L.cand, cap, m, L.prank);
            for (int q0 = 0; q0 < n; q0 += QB) {
                const int rows = n - q0 < QB ? n - q0 : QB;
                against_pivots(L.xs, L.norms, q0, q0 + rows);
                hipLaunchKernelGGL(nearest_pivot_k, dim3((rows + 3) / 4), dim3(256), 0, s, L.cand, cap, rows, m, L.prank, L.label + q0);
            }
            hipLaunchKernelGGL(fill_int_k, dim3((m + 256) / 256), dim3(256), 0, s, L.bcnt, 0, m + 1);
            hipLaunchKernelGGL(fill_int_k, dim3((m + 256) / 256), dim3(256), 0, s, L.bcur, 0, m + 1);
            hipLaunchKernelGGL(rank_hist, wide_grid((size_t)n), dim3(256), 0, s, L.label, (const int *)nullptr, 0, n, 1, 0, L.bcnt);
            hipLaunchKernelGGL(excl_scan_k, dim3(1), dim3(1024), 0, s, L.bcnt, m, L.bptr);
            hipLaunchKernelGGL(rank_scatter, wide_grid((size_t)n), dim3(256), 0, s, L.label, (const int *)nullptr, 0, n, 1, 0, L.bptr, L.bcur, L.ord);
            // the copy and the norms once more, in that order
            hipLaunchKernelGGL(row_norms, wide_grid((size_t)n * WAVE), dim3(256), 0, s, d_X, L.mu, n, d, ord, n, L.norms);
            split();
            hipLaunchKernelGGL(tile_centre_k, dim3(ntiles), dim3(256), 0, s, d_X, L.mu, n, d, ord, L.centre);
            hipLaunchKernelGGL(fill_int_k, dim3((ntiles + 255) / 256), dim3(256), 0, s, (int *)L.radius2, 0, ntiles);
            hipLaunchKernelGGL(tile_radius_k, wide_grid((size_t)n * WAVE), dim3(256), 0, s, d_X, L.mu, n, d, ord, L.centre, (unsigned int *)L.radius2);
            HIPCHK(hipGetLastError());
        }
    }
    // equal blocks of whole tiles (a short last one would leave most compute units idle)
    bool high = high_first;
    // (the order and its counts are where the conditional P goes later, the labels where the re-rank writes a block's distances)
    const bool grouped = high_first && d >= SCHED_MIN_D && 4 * (size_t)n * d > SCHED_MIN_BYTES;
    int *sched_of = (int *)L.cond, *total = sched_of + std::min(n, QB);
    for (int q0 = 0; q0 < n; q0 += block) {
        const int qend = q0 + block < n ? q0 + block : n, rows = qend - q0;
        // (a workgroup per query tile: at least half of the compute units have to get one, 41,000 rows of 300 coordinates
        // 8.9 -> 6.6 ms; and a row must be short, because its tile is read again for every database tile and no longer found
        // in the second-level cache: 100,000 rows of 300, 768, 1536, 2048, 3072 coordinates 30.5 -> 21.7, 40.5 -> 33.2,
        // 58.3 -> 52.7, 70.7 -> 66.2, 96.3 -> 104.7 ms)
        const bool own = dph <= HALF_OWN_MAX_D && rows >= HALF_OWN_MIN_ROWS;
        hipLaunchKernelGGL(knn_reset, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, rows, L.ccount);
        const bool resident = dp <= 2 * SLAB && rows >= RESIDENT_MIN_ROWS;
        const int *sched = nullptr;
        int launch = 0;
        bool listed = ord && resident, known = false;      // known: a sweep over all rows that starts with cut-offs
        if (listed) {
            // (as below: a compaction pass behind every second launch, whose own and the one before's appends it has room for)
            const unsigned nqt = (unsigned)((rows + HT - 1) / HT), grid = 8 * ((nqt + 7) / 8);
            TileLists lists = {L.first, nullptr, ORD_FIRST, std::min(ntiles, ORD_FIRST), 0, kp, L.clist, nullptr, nullptr};
            bool dense = true;
            auto step = [&](bool pass) {
                int *cc = L.ccount + (launch & 1), *cc_next = L.ccount + ((launch + 1) & 1);
                lists.ccount = cc;
                lists.ccount_next = cc_next;
                auto resident_tiles = [&](auto kernel, int ns) {
                    hipLaunchKernelGGL(kernel, dim3(grid), dim3(512), resident_lds_bytes(ns), s, (const uint4 *)L.xs, q0, qend, 0, n, L.norms,
                                       L.tau, L.cnt, L.cand, cap, kp, 0, pass ? L.clist : nullptr, cc, cc_next, lists);
                };
                if (dp == SLAB) { if (dense) resident_tiles(knn_tile_resident<1, true, true>, 1); else resident_tiles(knn_tile_resident<1, false, true>, 1); }
                else { if (dense) resident_tiles(knn_tile_resident<2, true, true>, 2); else resident_tiles(knn_tile_resident<2, false, true>, 2); }
                if (pass) compact(rows, cc, dense ? std::min(n, DBC) : 0);
                dense = false;
                lists.first += ORD_STEP;
                ++launch;
            };
            const int qt0 = q0 / HT;
            hipLaunchKernelGGL(tile_order_k, dim3(nqt), dim3(1024), 4 * ((size_t)d + ntiles), s, L.centre, L.radius2, ntiles, d, qt0, L.near, L.first);
            while (lists.first < lists.all) step(true);
            // every row's cut-off as low as it is by now
            hipLaunchKernelGGL(fill_int_k, dim3(1), dim3(256), 0, s, L.ccount, 0, 2);
            hipLaunchKernelGGL(knn_compact_list, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, cap, kp, rows, 1, L.clist, L.ccount);
            compact(rows, L.ccount, 0);
            hipLaunchKernelGGL(tile_rest_k, dim3(nqt), dim3(256), 0, s, L.near, ntiles, L.first, L.tau, rows, L.rest, L.rest_count);
            hipLaunchKernelGGL(fill_int_k, dim3(1), dim3(256), 0, s, L.ccount, 0, 2);
            int left[QB / HT], down[QB / HT];
            HIPCHK(hipMemcpyAsync(left, L.rest_count, 4 * nqt, hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            // A launch takes as long as one workgroup's ORD_STEP tiles, however few workgroups still have any.  A query tile
            // with rows of two groups can leave out hardly anything, so the few with the longest lists are better swept
            // by themselves, over all rows: as many as make the sum smallest.
            memcpy(down, left, 4 * nqt);
            std::sort(down, down + nqt, std::greater<int>());
            const int plain = (n + DBC - 1) / DBC;
            int alone = 0, limit = 0, best = INT_MAX;
            for (int x = 0; x < (int)nqt; ++x) {
                if (x > 0 && down[x] == down[x - 1]) continue;
                const int cost = ORD_LAUNCH * ((down[x] + ORD_STEP - 1) / ORD_STEP) + ORD_ALONE * x * ((n + ORD_ALONE_ROWS - 1) / ORD_ALONE_ROWS);
                if (cost < best) { best = cost; alone = x; limit = down[x]; }
            }
            if (q0 == 0 && 10 * best > 7 * ORD_PLAIN * plain) {
                // too little is left out: all rows against all, in the caller's order (in this one a query tile finds all its
                // neighbours in the same few launches, which wait for its appends: 150,000 rows of 8 coordinates in twenty
                // blobs 28 ms in the caller's order, 50 in this one)
                ord = nullptr;
                listed = false;
                limit = alone = 0;
                hipLaunchKernelGGL(row_norms, wide_grid((size_t)n * WAVE), dim3(256), 0, s, d_X, L.mu, n, d, ord, n, L.norms);
                split();
                hipLaunchKernelGGL(knn_reset, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, rows, L.ccount);
            } else if (best > ORD_PLAIN * plain) {
                // (the first block of query rows says little about this one: it is a region of its own)  All rows here too, with
                // the cut-offs so far; the pairs so far are dropped, as below.
                listed = false;
                known = true;
                limit = alone = 0;
                hipLaunchKernelGGL(fill_int_k, dim3((rows + 255) / 256), dim3(256), 0, s, L.cnt, 0, rows);
            }
            if (alone > 0) hipLaunchKernelGGL(tile_rest_limit_k, dim3(1), dim3(QB / HT), 0, s, L.rest_count, (int)nqt, limit);
            for (int b = 0; b < (int)nqt && alone > 0; ++b) {
                if (left[b] <= limit) continue;
                const int r0 = b * HT, m = std::min(HT, rows - r0);
                float *tau = L.tau + r0;
                int *cnt = L.cnt + r0;
                uint64_t *cand = L.cand + (size_t)r0 * cap;
                // The pairs so far are dropped, their cut-offs stay: nothing at or beyond them is kept or needed.  (A buffer
                // has room for k' pairs and ORD_ALONE_ROWS more; with four times the rows a launch those of the smaller group
                // overflowed it, and the exact pass took 23 ms.)
                hipLaunchKernelGGL(fill_int_k, dim3(1), dim3(256), 0, s, cnt, 0, m);
                for (int j0 = 0; j0 < n; j0 += ORD_ALONE_ROWS) {
                    const int jend = std::min(n, j0 + ORD_ALONE_ROWS);
                    hipLaunchKernelGGL((knn_tile_mfma<KNN_MB, false, false, false>),
                                       dim3((unsigned)((m + 64 * KNN_MB - 1) / (64 * KNN_MB)), (unsigned)((jend - j0 + TN - 1) / TN)), dim3(256), 0, s,
                                       (const uint4 *)L.xs, dp, q0 + r0, q0 + r0 + m, j0, jend, L.norms, tau, cnt, cand, cap, L.ccount,
                                       (const uint4 *)L.xs, L.norms, 1, (const int *)nullptr, (const int *)nullptr, 0,
                                       (const int *)nullptr, (const int *)nullptr, (const int *)nullptr, 0);
                    hipLaunchKernelGGL(knn_compact_list, dim3(1), dim3(256), 0, s, tau, cnt, cap, kp, m, 1, L.clist, L.ccount);
                    launch_compact(tau, cnt, cand, cap, kp, m, L.clist, L.ccount, 0, s);
                }
            }
            hipLaunchKernelGGL(fill_int_k, dim3(1), dim3(256), 0, s, L.ccount, 0, 2);
            lists.tiles = L.rest;
            lists.count = L.rest_count;
            lists.stride = ORD_MAX_TILES;
            lists.first = 0;
            launch = 0;
            while (lists.first < limit) step(launch % COMPACT_EVERY != 0);
            hipLaunchKernelGGL(fill_int_k, dim3(1), dim3(256), 0, s, L.ccount, 0, 2);
            hipLaunchKernelGGL(knn_compact_list, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, cap, kp, rows, 1, L.clist, L.ccount);
            compact(rows, L.ccount, 0);
            launch = 0;
        }
        for (int j0 = 0, jend; !listed && j0 < n; j0 = jend, ++launch) {
            jend = j0 + DBC < n ? j0 + DBC : n;
            const bool dense = j0 == 0 && !known;
            const int force = jend >= n ? 1 : 0;
            int *cc = L.ccount + (launch & 1), *cc_next = L.ccount + ((launch + 1) & 1);   // two lists take turns
            // (a row that is not listed has room for what two launches can append, so a pass over the rows follows every
            // second launch only: it costs a third of a launch after the resident kernel, and the two small kernels of a
            // pass are 8 % of the time between the half-precision sweep's; the rows stay listed)
            const bool skip = !dense && !force && launch % COMPACT_EVERY != 0;
            if (resident) {
                auto tiles = [&](auto kernel, int ns) {
                    hipLaunchKernelGGL(kernel, dim3((rows + RQ - 1) / RQ), dim3(512), resident_lds_bytes(ns), s, (const uint4 *)L.xs,
                                       q0, qend, j0, jend, L.norms, L.tau, L.cnt, L.cand, cap, kp, force, skip ? nullptr : L.clist, cc, cc_next, TileLists{});
                };
                if (dp == SLAB) {
                    if (dense) tiles(knn_tile_resident<1, true, false>, 1); else tiles(knn_tile_resident<1, false, false>, 1);
                } else {
                    if (dense) tiles(knn_tile_resident<2, true, false>, 2); else tiles(knn_tile_resident<2, false, false>, 2);
                }
                if (skip) continue;
            } else {
                if (high) {
                    const unsigned nqt = (unsigned)((rows + HT - 1) / HT), njt = (unsigned)((jend - j0 + HT - 1) / HT);
                    auto tiles = [&](auto kernel, unsigned grid, size_t lds_bytes) {
                        hipLaunchKernelGGL(kernel, dim3(grid), dim3(HALF_THREADS), lds_bytes, s, (const uint4 *)L.xh, dph, q0, qend,
                                           j0, jend, L.norms, L.tau, L.cnt, L.cand, cap, cc, dot_scale, DueRows{skip ? nullptr : L.clist, cc_next, kp, force});
                    };
                    if (dense) tiles(knn_tile_half<true, false>, 8 * ((nqt + 7) / 8) * njt, HALF_TILE_LDS);
                    else if (own) tiles(knn_tile_half<false, true>, nqt, HALF_OWN_LDS);
                    else tiles(knn_tile_half<false, false>, 8 * ((nqt + 7) / 8) * njt, HALF_TILE_LDS);
                    if (dense && grouped && rows >= SCHED_MIN_ROWS) {
                        const unsigned nb = (unsigned)((rows + SCHED_ROWS - 1) / SCHED_ROWS);
                        int *label = (int *)(L.knn_d2 + (size_t)q0 * k);
                        hipLaunchKernelGGL(fill_int_k, dim3(1), dim3(256), 0, s, total, 0, 2 * SCHED_PIVOTS);
                        hipLaunchKernelGGL(rerank_label_k, dim3(nb), dim3(256), 0, s, L.cand, cap, rows, label, total);
                        hipLaunchKernelGGL(rerank_sched_k, dim3(nb), dim3(SCHED_ROWS), 0, s, label, rows, total, total + SCHED_PIVOTS, sched_of);
                        sched = sched_of;
                    }
                } else {
                    mfma_tiles(L.xs, L.norms, q0, qend, j0, jend, nullptr, cc);
                }
                if (high && skip) continue;
                if (!high || dense || !own)
                    hipLaunchKernelGGL(knn_compact_list, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, cap, kp, rows,
                                       force, L.clist, cc);
            }
            compact(rows, cc, dense ? std::min(n, DBC) : 0);
        }
        hipLaunchKernelGGL(knn_rerank, dim3((unsigned)((rows + 7) / 8 * 8)), dim3(256), rerank_smem, s, d_X, n, d, ord, d_X, n,
                           ord, ord, ord, q0, rows, k, kp, n - 1,
                           high ? tile_error_coeff(d, false, true) : tile_error_coeff(d, d > KFLUSH), high ? e_add : 0.0, L.norms, norm_max,
                           L.tau, L.cnt, L.cand, cap, L.knn_idx, L.knn_d2, high == high_first ? L.fail_count : L.fail2_count,
                           high == high_first ? L.fail_rows : L.fail2_rows, sched);
        HIPCHK(hipGetLastError());
        if (high && q0 == 0 && qend < n) {
            // half precision that certifies less than half of the first block's rows is no use for the others (whose rows
            // without a certificate the second sweep, the same tiles once more, could not help: they go on its list of those)
            int failed = 0;
            HIPCHK(hipMemcpyAsync(&failed, L.fail_count, 4, hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            if (failed > rows / 2) { high = false; split(); }
        }
    }
    int nfail = 0, nfail2 = 0;
    HIPCHK(hipMemcpyAsync(&nfail, L.fail_count, 4, hipMemcpyDeviceToHost, s));
    if (high != high_first) HIPCHK(hipMemcpyAsync(&nfail2, L.fail2_count, 4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const int *exact_rows = L.fail_rows;
    if (high_first && nfail + nfail2 > 0) {
        // second sweep: the rows the first one could not certify, QB at a time, as queries of their own (a split
        // copy of just these rows) against all rows
        if (high && nfail > 0) split();
        for (int f0 = 0; f0 < nfail; f0 += QB) {
            const int rows = nfail - f0 < QB ? nfail - f0 : QB;
            const int *fr = L.fail_rows + f0;
            hipLaunchKernelGGL(row_norms, wide_grid((size_t)rows * WAVE), dim3(256), 0, s, d_X, L.mu, rows, d, fr, n, L.norms_f);
            hipLaunchKernelGGL(split_bf16, wide_grid((size_t)rows * dp), dim3(256), 0, s, d_X, L.mu, rows, d, dp, fr, n, L.xsf);
            hipLaunchKernelGGL(knn_reset, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, rows, L.ccount);
            for (int j0 = 0, jend; j0 < n; j0 = jend) {
                jend = j0 + DBC < n ? j0 + DBC : n;
                const int force = jend >= n ? 1 : 0;
                mfma_tiles(L.xsf, L.norms_f, 0, rows, j0, jend, fr, L.ccount);
                hipLaunchKernelGGL(knn_compact_list, dim3((rows + 255) / 256), dim3(256), 0, s, L.tau, L.cnt, cap, kp, rows, force,
                                   L.clist, L.ccount);
                compact(rows, L.ccount, j0 == 0 ? jend : 0);
            }
            hipLaunchKernelGGL(knn_rerank, dim3((unsigned)((rows + 7) / 8 * 8)), dim3(256), rerank_smem, s, d_X, n, d, fr, d_X, n, (const int *)nullptr, fr, fr,
                               0, rows, k, kp, n - 1, tile_error_coeff(d, true), 0.0, L.norms_f, norm_max, L.tau, L.cnt, L.cand, cap,
                               L.knn_idx, L.knn_d2, L.fail2_count, L.fail2_rows, (const int *)nullptr);
            HIPCHK(hipGetLastError());
        }
        HIPCHK(hipMemcpyAsync(&nfail, L.fail2_count, 4, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        exact_rows = L.fail2_rows;
    }
    // Rows without a certificate (ties at the k-th distance, duplicates): exact distances to every row, 2k failed
    // rows a launch (their n keys each fit the space the symmetrisation sorts in later, 2 n k words).
    for (int f0 = 0; f0 < nfail; f0 += 2 * k) {
        const int nb = nfail - f0 < 2 * k ? nfail - f0 : 2 * k;
        hipLaunchKernelGGL(knn_exact_dists, wide_grid((size_t)n * WAVE), dim3(256), 0, s, d_X, n, (const int *)nullptr, d_X, n, d,
                           exact_rows + f0, nb, 1, L.sort_scratch);
        hipLaunchKernelGGL(knn_exact_select, dim3(nb), dim3(1024), 0, s, L.sort_scratch, (size_t)n, n, (const int *)nullptr,
                           (const int *)nullptr, k, exact_rows + f0, (const int *)nullptr, n, L.knn_idx, L.knn_d2);
        HIPCHK(hipGetLastError());
    }
    return finish_P(L, n, k, perplexity, d_row_ptr, d_col, d_val, cap_nnz, nnz, d_knn_idx, d_knn_d2, n_unconverged, 1, s);
}

static int approx_lists(int32_t n, int32_t nlist)
{
    if (nlist > 0) return nlist;
    int v = (int)llround(sqrt((double)n));     // Sec. III-B: |C| = sqrt(N)
    if (v < 1) v = 1;
    if (v > 65536) v = 65536;
    return v;
}

constexpr int PQ_KSUB = 256;     // centroids per sub-quantiser: one code byte per sub-vector

int tsne_build_P_approx_workspace_bytes(int32_t n, int32_t d, int32_t k, int32_t nlist, int32_t tau, int32_t pq_m,
                                        size_t *bytes)
{
    if (!bytes || check_args(n, d, k) != TSNE_OK || pq_m < 0) return TSNE_EINVAL;
    nlist = approx_lists(n, nlist);
    const int tau_max = nlist < 32 ? nlist : 32;
    size_t ivf = 0, ivf_max = 0;
    // (room for the search to be repeated with more lists, see tsne_build_P_approx)
    if (pq_m > 0) {
        const int ksub = n < PQ_KSUB ? n : PQ_KSUB;
        if (tsne_ivfpq_workspace_bytes(n, d, k, nlist, tau, pq_m, ksub, &ivf) != TSNE_OK) return TSNE_EINVAL;
        if (tsne_ivfpq_workspace_bytes(n, d, k, nlist, tau_max, pq_m, ksub, &ivf_max) != TSNE_OK) return TSNE_EINVAL;
        const size_t coarse = ivf_workspace(n, d, 0, nlist, 1);       // training the coarse centroids comes first
        if (coarse > ivf) ivf = coarse;
    } else {
        if (tsne_ivf_workspace_bytes(n, d, k, nlist, tau, &ivf) != TSNE_OK) return TSNE_EINVAL;
        if (tsne_ivf_workspace_bytes(n, d, k, nlist, tau_max, &ivf_max) != TSNE_OK) return TSNE_EINVAL;
    }
    *bytes = carve(nullptr, n, d, k, nullptr) + up(4 * (size_t)nlist * d) + up(4 * (size_t)PQ_KSUB * d) +
             (ivf_max > ivf ? ivf_max : ivf);
    return TSNE_OK;
}

int tsne_build_P_approx(const float *d_X, int32_t n, int32_t d, float perplexity, int32_t k, int32_t nlist, int32_t tau,
                        int32_t kmeans_iters, int32_t pq_m, int32_t *d_row_ptr, int32_t *d_col, float *d_val, int64_t cap_nnz,
                        int64_t *nnz, int32_t *d_knn_idx, float *d_knn_d2, int32_t *n_unconverged, int32_t *tau_used,
                        void *d_workspace, size_t workspace_bytes, void *stream)
{
    if (!d_X || !d_row_ptr || !d_col || !d_val || !nnz || !d_workspace || kmeans_iters < 0) return TSNE_EINVAL;
    if (check_args(n, d, k) != TSNE_OK) return TSNE_EINVAL;
    if (!(perplexity > 0.0f) || !(perplexity <= (float)k)) return TSNE_EINVAL;
    if (((uintptr_t)d_workspace % ALIGN) != 0) return TSNE_EINVAL;
    nlist = approx_lists(n, nlist);
    size_t need = 0;
    if (tsne_build_P_approx_workspace_bytes(n, d, k, nlist, tau, pq_m, &need) != TSNE_OK) return TSNE_EINVAL;
    if (workspace_bytes < need) return TSNE_ENOSPC;
    hipStream_t s = (hipStream_t)stream;
    Layout L;
    size_t off = carve(&L, n, d, k, (char *)d_workspace);
    float *centroids = (float *)((char *)d_workspace + off);
    off += up(4 * (size_t)nlist * d);
    float *codebooks = (float *)((char *)d_workspace + off);
    off += up(4 * (size_t)PQ_KSUB * d);
    const int ksub = n < PQ_KSUB ? n : PQ_KSUB;
    void *ivf_ws = (char *)d_workspace + off;
    const size_t ivf_bytes = workspace_bytes - off;
    HIPCHK(hipMemsetAsync(L.unconv, 0, 4, s));
    HIPCHK(hipMemsetAsync(L.extra, 0, 4 * (size_t)n, s));
    int rc = ivf_train_device(d_X, n, d, nlist, kmeans_iters, centroids, ivf_ws, ivf_bytes, s);
    if (rc != TSNE_OK) return rc;
    if (pq_m > 0) {     // Eq. (8): the second-stage codebooks, one code byte per sub-vector
        rc = tsne_ivfpq_train(d_X, n, d, centroids, nlist, pq_m, ksub, kmeans_iters, codebooks, ivf_ws, ivf_bytes, s);
        if (rc != TSNE_OK) return rc;
    }
    // a row that finds fewer than k other points in its tau lists: twice the lists for everybody, and again
    const int tau_max = nlist < 32 ? nlist : 32;
    for (;;) {
        rc = pq_m > 0 ? tsne_ivfpq_knn(d_X, n, d, centroids, nlist, codebooks, pq_m, ksub, tau, k, L.knn_idx, L.knn_d2, ivf_ws,
                                       ivf_bytes, s)
                      : ivf_knn_device(d_X, n, d, centroids, nlist, tau, k, L.knn_idx, L.knn_d2, ivf_ws, ivf_bytes, s);
        if (rc != TSNE_ENUM || tau >= tau_max) break;
        tau = 2 * tau < tau_max ? 2 * tau : tau_max;
    }
    if (rc != TSNE_OK) return rc;
    if (tau_used) *tau_used = tau;
    return finish_P(L, n, k, perplexity, d_row_ptr, d_col, d_val, cap_nnz, nnz, d_knn_idx, d_knn_d2, n_unconverged, pq_m == 0, s);
}

}  // extern "C"
