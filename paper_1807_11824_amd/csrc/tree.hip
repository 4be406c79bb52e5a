// Sec. III-C steps 1-4 of the paper on gfx950: bounding box, grid keys, spatial sort,
// quad tree and cell summaries.  Nothing here walks pointers or inserts points one by one:
// the tree is read off the sorted keys.
//
//   bbox_partial / bbox_final   step 1   min/max reduction -> root square (power-of-two side)
//   morton_encode_hist          step 2a  grid coordinates (up to 24 bits per axis), bit-interleaved key
//   radix_hist / _scan / _scatter  step 4  stable LSD radix sort, 11 bits a pass
//   rank_tiles / _samples / _merge  steps 1, 2a, 4 by counting smaller keys, for up to 131,072 points (122,880 not renumbered)
//   gather_levels               step 2b  which cells start at each sorted position
//   downsweep                   step 3   prefix sums: cell numbering and running coordinate sums
//   write_cells                 steps 2c+3  cell records: members, count, centre of mass, children
//   small_tree                  steps 2b, 2c, 3 in one launch of one workgroup, for up to 4096 points
//
// The sort works on one 64-bit word per point, (key << key_shift) | slot with key_shift = 64 - 2 bits:
// the order of the words is the order by (key, slot), which is the stable order the tree is defined
// on, and no index array travels through the passes.
//
// A cell at depth t is the run of sorted positions sharing the top 2t key bits.  A position p
// opens cells at depths tmin(p).. where tmin is fixed by the first digit in which key[p] differs
// from key[p-1]; the chain stops at the first depth whose parent holds <= leaf_cap points.
// Numbering cells by (position, depth) is exactly depth-first pre-order, so one scalar prefix
// sum over "cells opened at p" numbers the whole tree, and the centre of mass of any cell is a
// difference of two entries of the double-precision running sum of the sorted coordinates.
#include "tsne_internal.h"

#include <algorithm>

#include <math.h>

// ------------------------------------------------------------------ bounding box
// Also brings the caller's Y (original point order) into the library's slot order:
// Yi[s] = Y[orig[s]].
__global__ __launch_bounds__(256) void bbox_partial(const float2 *__restrict__ Y, const uint32_t *__restrict__ orig,
                                                    float2 *__restrict__ Yi, int n, float4 *__restrict__ part,
                                                    uint32_t *status)
{
    float mnx = INFINITY, mny = INFINITY, mxx = -INFINITY, mxy = -INFINITY;
    bool bad = false;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        float2 y = Y[min(orig[i], (uint32_t)n - 1u)];
        Yi[i] = y;
        bad |= !(isfinite(y.x) && isfinite(y.y));
        mnx = fminf(mnx, y.x); mxx = fmaxf(mxx, y.x);
        mny = fminf(mny, y.y); mxy = fmaxf(mxy, y.y);
    }
    mnx = wave_min(mnx); mny = wave_min(mny); mxx = wave_max(mxx); mxy = wave_max(mxy);
    __shared__ float4 smn[4], smx[4];
    int w = threadIdx.x >> 6;
    if (lane_id() == 0) { smn[w] = make_float4(mnx, mny, 0, 0); smx[w] = make_float4(mxx, mxy, 0, 0); }
    if (__any(bad) && lane_id() == 0) atomicOr(status, TSNE_STATUS_NONFINITE);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k) {
            mnx = fminf(mnx, smn[k].x); mny = fminf(mny, smn[k].y);
            mxx = fmaxf(mxx, smx[k].x); mxy = fmaxf(mxy, smx[k].y);
        }
        part[2 * blockIdx.x] = make_float4(mnx, mny, 0, 0);
        part[2 * blockIdx.x + 1] = make_float4(mxx, mxy, 0, 0);
    }
}

// Root square: lower corner (min x, min y); side = smallest power of two >= the larger extent,
// at least 2^-40; scale S = 2^bits / side (an exact power of two).
__device__ __forceinline__ float4 root_square(float mnx, float mny, float mxx, float mxy, int bits, uint32_t *status)
{
    float ex = mxx - mnx, ey = mxy - mny;
    float e = fmaxf(ex, ey);
    float W = ldexpf(1.0f, -40);
    if (!isfinite(e) || !isfinite(mnx) || !isfinite(mny)) {
        atomicOr(status, TSNE_STATUS_NONFINITE);
        mnx = 0.0f; mny = 0.0f; W = 1.0f;
    } else if (e > W) {
        int ex2;
        float m = frexpf(e, &ex2);          // e = m 2^ex2, m in [0.5, 1)
        W = (m == 0.5f) ? e : ldexpf(1.0f, ex2);
    }
    float S = ldexpf(1.0f, bits) / W;
    return make_float4(mnx, mny, W, S);
}

__global__ __launch_bounds__(1024) void bbox_final(const float4 *__restrict__ part, int nparts, int bits,
                                                   float4 *__restrict__ root, uint32_t *status)
{
    float mnx = INFINITY, mny = INFINITY, mxx = -INFINITY, mxy = -INFINITY;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) {
        float4 a = part[2 * i], b = part[2 * i + 1];
        mnx = fminf(mnx, a.x); mny = fminf(mny, a.y);
        mxx = fmaxf(mxx, b.x); mxy = fmaxf(mxy, b.y);
    }
    mnx = wave_min(mnx); mny = wave_min(mny); mxx = wave_max(mxx); mxy = wave_max(mxy);
    __shared__ float4 smn[16], smx[16];
    const int w = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
    if (lane_id() == 0) { smn[w] = make_float4(mnx, mny, 0, 0); smx[w] = make_float4(mxx, mxy, 0, 0); }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < nw; ++k) {
            mnx = fminf(mnx, smn[k].x); mny = fminf(mny, smn[k].y);
            mxx = fmaxf(mxx, smx[k].x); mxy = fmaxf(mxy, smx[k].y);
        }
        *root = root_square(mnx, mny, mxx, mxy, bits, status);
    }
}

// ------------------------------------------------------------------ grid keys
// bits of v (up to 24) to the even positions
__device__ __forceinline__ uint64_t spread24(uint32_t q)
{
    uint64_t v = q & 0xFFFFFFu;
    v = (v | (v << 16)) & 0x0000FFFF0000FFFFull;
    v = (v | (v << 8)) & 0x00FF00FF00FF00FFull;
    v = (v | (v << 4)) & 0x0F0F0F0F0F0F0F0Full;
    v = (v | (v << 2)) & 0x3333333333333333ull;
    v = (v | (v << 1)) & 0x5555555555555555ull;
    return v;
}

// One rounding per operation: the subtraction rounds, the product with a power of two is exact.
__device__ __forceinline__ uint32_t grid_coord(float v, float origin, float S, uint32_t qmax)
{
#pragma clang fp contract(off)
    float r = v - origin;
    float s = r * S;
    float f = floorf(s);
    return f >= (float)qmax ? qmax : (f > 0.0f ? (uint32_t)f : 0u);
}

__device__ __forceinline__ uint64_t grid_key(float2 y, float4 r, uint32_t qmax)
{
    return spread24(grid_coord(y.x, r.x, r.w, qmax)) | (spread24(grid_coord(y.y, r.y, r.w, qmax)) << 1);
}

// ------------------------------------------------------------------ few points: order by counting
// Up to RANK_MAX points the radix passes would be a dozen launches that are far too short to fill the chip.  The words
// are all different, so a word's place is the number of smaller words, and counting is what an idle chip has room for:
//
//   rank_tiles     root square, keys and the order inside tiles of RANK_TILE points (n <= SMALL_SORT_MAX: all points are
//                  one tile, and this is the whole sort).  A workgroup holds its tile's words in LDS and counts for
//                  `points` of them; a thread compares one word with one segment of the tile.
//   rank_samples   every RANK_GAP-th word of the sorted tiles, in order, by the same count
//   rank_merge     a bucket of the sorted samples per workgroup: finds the piece of every tile that falls into it,
//                  collects the pieces, counts again, and writes its stretch of the order.  The number of words below
//                  the bucket is the sum of the pieces' starts, so no bucket waits for another.
//
// A tile's words between two of its samples are at most RANK_GAP - 1, so a bucket of s samples holds at most
// RANK_GAP s + (RANK_GAP - 1) tiles words, whatever the embedding looks like.  Where the samples of a tile start
// differs from tile to tile (rank_offset): with equal starts tiles of the same distribution would all have their
// samples at the same quantiles and nothing in between, and a few buckets would hold most of the words.
// Same root, keys and order as bbox_final + morton_encode_hist + the radix passes.  25 iterations of a run: 60,000 points
// 4.28 -> 3.46 ms, 30,011 4.25 -> 3.35, 100,000 4.35 -> 3.85 (three launches where there were fourteen); 2000 points 2.42
// -> 2.27 (before, one workgroup sorted up to 8192 words in LDS).  Beyond RANK_MAX there are more tiles than a wave scans, the counting grows with the
// number of tiles, and the radix passes have enough to do.  In the caller's numbering, which says nothing about where the
// points are, every tile has words in every bucket: rank_merge of 131,072 points then takes 52 us instead of 24, and the
// limit is lower (25 iterations, radix passes / counting: 106,496 points 5.41 / 5.17 ms, 114,688 5.56 / 5.36, 122,880 5.71 /
// 5.64, 131,072 5.91 / 6.01; renumbered 131,072 4.61 / 4.21).
constexpr int RANK_THREADS = 512, RANK_TILE = 1024, RANK_GAP = 64, RANK_PER_TILE = RANK_TILE / RANK_GAP;
constexpr int RANK_BUCKETS = 256;              // most workgroups of rank_merge: about one per compute unit
constexpr int RANK_MAX = RANK_SORT_MAX, RANK_MAX_CALLER = 122880;
static_assert(RANK_MAX <= 2 * WAVE * RANK_TILE, "rank_merge scans two tiles a lane of one wave");

__host__ __device__ inline int rank_offset(int tile) { return (tile * 39) & (RANK_GAP - 1); }   // (64 / golden ratio, odd)

// words[seg * len .. + len) below `own`; len is even, the words are 16-byte aligned
__device__ __forceinline__ uint32_t count_below(const uint64_t *words, int len, uint64_t own)
{
    uint32_t below = 0;
#pragma unroll 8
    for (int j = 0; j < len; j += 2) {
        const ulonglong2 w = *reinterpret_cast<const ulonglong2 *>(words + j);
        below += w.x < own ? 1u : 0u;
        below += w.y < own ? 1u : 0u;
    }
    return below;
}

// Length of one of `segs` equal, even segments that cover len words (the array is padded to segs times this).
__host__ __device__ inline int rank_segment(int len, int segs) { return ((len + segs - 1) / segs + 1) & ~1; }

// The workgroup's words are in LDS at `words`, padded with all-ones to whole segments; writes those numbered
// p0 .. p0 + points - 1 to out[their rank].  rk: `points` counters.
__device__ __forceinline__ void rank_and_write(const uint64_t *words, int len, uint32_t *rk, int p0, int points,
                                               uint64_t *__restrict__ out)
{
    const int tid = (int)threadIdx.x, segs = RANK_THREADS / points, seg = tid / points, p = tid % points;
    const int slen = rank_segment(len, segs);
    if (tid < points) rk[tid] = 0u;
    __syncthreads();
    const uint64_t own = words[min(p0 + p, len - 1)];
    atomicAdd(&rk[p], count_below(words + seg * slen, slen, own));
    __syncthreads();
    if (tid < points && p0 + tid < len) out[min(rk[tid], (uint32_t)len - 1u)] = own;     // (seg 0: own is word p0 + tid)
}

__global__ __launch_bounds__(RANK_THREADS) void rank_tiles(const float2 *__restrict__ Y, int n, int tile, int points,
                                                           const float4 *__restrict__ part, int nparts, int bits, int ks,
                                                           float4 *__restrict__ root, uint64_t *__restrict__ out,
                                                           uint32_t *status)
{
    extern __shared__ __align__(16) uint64_t rank_words[];
    __shared__ float4 smm[RANK_THREADS / WAVE];
    __shared__ float4 sroot;
    __shared__ uint32_t rk[RANK_THREADS];
    const int tid = (int)threadIdx.x;
    const int pieces = (tile + points - 1) / points, t = (int)blockIdx.x / pieces, p0 = ((int)blockIdx.x % pieces) * points;
    const int tile0 = t * tile, len = min(tile, n - tile0);
    if (p0 >= len) return;                       // the same for every thread of the workgroup
    if (nparts > 0) {
        float mnx = INFINITY, mny = INFINITY, mxx = -INFINITY, mxy = -INFINITY;
        for (int i = tid; i < nparts; i += RANK_THREADS) {
            const float4 a = part[2 * i], b = part[2 * i + 1];
            mnx = fminf(mnx, a.x); mny = fminf(mny, a.y);
            mxx = fmaxf(mxx, b.x); mxy = fmaxf(mxy, b.y);
        }
        mnx = wave_min(mnx); mny = wave_min(mny); mxx = wave_max(mxx); mxy = wave_max(mxy);
        if (lane_id() == 0) smm[tid >> 6] = make_float4(mnx, mny, mxx, mxy);
        __syncthreads();
        if (tid == 0) {
            for (int k = 1; k < RANK_THREADS / WAVE; ++k) {
                mnx = fminf(mnx, smm[k].x); mny = fminf(mny, smm[k].y);
                mxx = fmaxf(mxx, smm[k].z); mxy = fmaxf(mxy, smm[k].w);
            }
            sroot = root_square(mnx, mny, mxx, mxy, bits, status);
            if (blockIdx.x == 0) *root = sroot;
        }
    } else if (tid == 0) {
        sroot = *root;                           // already in place
    }
    __syncthreads();
    const float4 r = sroot;
    const uint32_t qmax = (1u << bits) - 1u;
    const int segs = RANK_THREADS / points, padded = segs * rank_segment(len, segs);
    for (int i = tid; i < padded; i += RANK_THREADS)
        rank_words[i] = i < len ? (grid_key(Y[tile0 + i], r, qmax) << ks) | (uint32_t)(tile0 + i) : ~0ull;
    rank_and_write(rank_words, len, rk, p0, points, out + tile0);
}

// number of samples of n words in tiles
static int rank_sample_count(int n)
{
    const int last = (n - 1) / RANK_TILE, left = n - last * RANK_TILE - rank_offset(last);
    return last * RANK_PER_TILE + (left > 0 ? (left + RANK_GAP - 1) / RANK_GAP : 0);
}

__global__ __launch_bounds__(RANK_THREADS) void rank_samples(const uint64_t *__restrict__ tiles, int n, int count, int points,
                                                             uint64_t *__restrict__ out)
{
    extern __shared__ __align__(16) uint64_t rank_words[];
    __shared__ uint32_t rk[RANK_THREADS];
    const int segs = RANK_THREADS / points, padded = segs * rank_segment(count, segs);
    for (int i = (int)threadIdx.x; i < padded; i += RANK_THREADS) {
        const int t = i / RANK_PER_TILE, at = t * RANK_TILE + (i % RANK_PER_TILE) * RANK_GAP + rank_offset(t);
        rank_words[i] = i < count && at < n ? tiles[at] : ~0ull;
    }
    rank_and_write(rank_words, count, rk, (int)blockIdx.x * points, points, out);
}

// Most words of one of nb buckets (see above).
static int rank_bucket_cap(int n, int nb)
{
    const int m = (n + RANK_TILE - 1) / RANK_TILE, q = rank_sample_count(n);
    return RANK_GAP * ((q + nb - 1) / nb) + (RANK_GAP - 1) * m;
}

// cap: words that fit the LDS arrays (rank_bucket_cap), padded to whole segments of eight waves.
__global__ __launch_bounds__(RANK_THREADS) void rank_merge(const uint64_t *__restrict__ tiles, int n,
                                                           const uint64_t *__restrict__ samples, int count, int cap,
                                                           uint64_t *__restrict__ out)
{
    constexpr int NW = RANK_THREADS / WAVE;
    extern __shared__ __align__(16) uint64_t rank_words[];
    uint32_t *rk = reinterpret_cast<uint32_t *>(rank_words + cap);
    __shared__ int lb[2][RANK_MAX / RANK_TILE];     // first word of the bucket in every tile, first word behind it
    __shared__ int off[RANK_MAX / RANK_TILE + 1];   // where the tile's piece starts in the bucket
    __shared__ uint32_t sbase;
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6, m = (n + RANK_TILE - 1) / RANK_TILE;
    const int b = (int)blockIdx.x, nb = (int)gridDim.x;
    const int s0 = (int)((long long)b * count / nb), s1 = (int)((long long)(b + 1) * count / nb);
    const uint64_t lo = b == 0 ? 0ull : samples[s0], hi = b + 1 == nb ? ~0ull : samples[s1];
    // Sixteen lanes a search, in three rounds: every 64th, every 4th, every word.  (The last bucket takes what is left,
    // by its side and not by a comparison: a word may be all-ones.)
    for (int g = tid >> 4; g < 2 * m; g += RANK_THREADS / 16) {
        const int t = g >> 1, sub = lane & 15, len = min(RANK_TILE, n - t * RANK_TILE);
        const uint64_t *words = tiles + (size_t)t * RANK_TILE;
        const uint64_t want = (g & 1) ? hi : lo;
        const bool rest = (g & 1) && b + 1 == nb;
        int at = 0;
#pragma unroll
        for (int step = 64; step > 0; step = step == 64 ? 4 : step == 4 ? 1 : 0) {
            const int q = at + (sub + 1) * step - 1;
            const bool below = q < len && (step > 1 || sub < 4) && (rest || words[q] < want);
            at += step * __popcll((__ballot(below) >> (lane & 48)) & 0xFFFFull);
        }
        if (sub == 0) lb[g & 1][t] = min(at, len);
    }
    __syncthreads();
    if (w == 0) {
        int v[2], base = 0;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int t = 2 * lane + k;
            v[k] = t < m ? max(lb[1][t] - lb[0][t], 0) : 0;
            base += t < m ? lb[0][t] : 0;
        }
        int total;
        const int ex = wave_excl_scan(v[0] + v[1], &total);
        base = wave_sum(base);
        if (2 * lane < m) off[2 * lane] = ex;
        if (2 * lane + 1 < m) off[2 * lane + 1] = ex + v[0];
        if (lane == 0) { off[m] = total; sbase = (uint32_t)base; }
    }
    __syncthreads();
    const int c = min(off[m], cap), slen = rank_segment(c, NW), padded = min(NW * slen, cap);
    for (int i = tid; i < padded; i += RANK_THREADS) {
        uint64_t v = ~0ull;
        if (i < c) {
            int t0 = 0, t1 = m;                    // off[t0] <= i < off[t1]
            while (t1 - t0 > 1) {
                const int mid = (t0 + t1) >> 1;
                if (off[mid] <= i) t0 = mid; else t1 = mid;
            }
            v = tiles[min(t0 * RANK_TILE + min(lb[0][t0] + (i - off[t0]), RANK_TILE - 1), n - 1)];
        }
        rank_words[i] = v;
        rk[i] = 0u;
    }
    __syncthreads();
    for (int e = 0; e < c; e += WAVE) {
        const uint64_t own = rank_words[min(e + lane, c - 1)];
        const uint32_t below = count_below(rank_words + w * slen, slen, own);
        if (e + lane < c) atomicAdd(&rk[e + lane], below);
    }
    __syncthreads();
    for (int i = tid; i < c; i += RANK_THREADS) out[min(sbase + rk[i], (uint32_t)n - 1u)] = rank_words[i];
}

static size_t rank_lds(int len, int points) { const int segs = RANK_THREADS / points; return 8 * (size_t)(segs * rank_segment(len, segs)); }
static int rank_merge_cap(int n, int nb) { return 8 * rank_segment(rank_bucket_cap(n, nb), 8); }
// Points a workgroup counts for: a sixteenth of its threads' where all points are one tile, so that a few thousand of
// them reach most of the chip; a quarter in tiles, where every workgroup of a tile works all its keys out again.
constexpr int RANK_POINTS_ONE = 32, RANK_POINTS_TILED = 128;

hipError_t rank_sort_prepare()
{
    hipError_t e;
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void *>(&rank_tiles), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)rank_lds(SMALL_SORT_MAX, RANK_POINTS_ONE))) != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&rank_merge), hipFuncAttributeMaxDynamicSharedMemorySize,
                               12 * rank_merge_cap(RANK_MAX, RANK_BUCKETS));
}

// The order of the points of c->Yi in c->words[c->sorted_buf], for n <= RANK_MAX (root_fresh: the root square is in place).
static hipError_t launch_rank_sort(tsne_ctx *c, hipStream_t s)
{
    const int n = c->p.n, B = c->p.morton_bits, ks = c->key_shift, nparts = c->root_fresh ? 0 : c->bbox_nparts;
    c->root_fresh = 0;
    if (n <= SMALL_SORT_MAX) {
        hipLaunchKernelGGL(rank_tiles, dim3((n + RANK_POINTS_ONE - 1) / RANK_POINTS_ONE), dim3(RANK_THREADS),
                           rank_lds(n, RANK_POINTS_ONE), s, c->Yi, n, n, RANK_POINTS_ONE, c->bbox_part, nparts, B, ks, c->root,
                           c->words[0], c->status);
        c->sorted_buf = 0;
        return hipGetLastError();
    }
    const int m = (n + RANK_TILE - 1) / RANK_TILE, q = rank_sample_count(n);
    const int nb = std::min(RANK_BUCKETS, (n + 127) / 128), cap = rank_merge_cap(n, nb);
    uint64_t *samples = reinterpret_cast<uint64_t *>(c->hist);
    hipLaunchKernelGGL(rank_tiles, dim3(m * (RANK_TILE / RANK_POINTS_TILED)), dim3(RANK_THREADS),
                       rank_lds(RANK_TILE, RANK_POINTS_TILED), s, c->Yi, n, RANK_TILE, RANK_POINTS_TILED, c->bbox_part, nparts, B,
                       ks, c->root, c->words[0], c->status);
    hipLaunchKernelGGL(rank_samples, dim3((q + RANK_POINTS_ONE - 1) / RANK_POINTS_ONE), dim3(RANK_THREADS),
                       rank_lds(q, RANK_POINTS_ONE), s, c->words[0], n, q, RANK_POINTS_ONE, samples);
    hipLaunchKernelGGL(rank_merge, dim3(nb), dim3(RANK_THREADS), 12 * (size_t)cap, s, c->words[0], n, samples, q, cap, c->words[1]);
    c->sorted_buf = 1;
    return hipGetLastError();
}

// ------------------------------------------------------------------ radix sort (stable, LSD, 11 bits a pass)
// Three kernels a pass: digit counts per tile (hist[tile][digit]; the first pass gets them from
// the kernel that wrote the words), their prefix over the tiles, and the scatter.
__device__ __forceinline__ uint32_t digit_of(uint64_t w, int lo, uint32_t mask) { return (uint32_t)(w >> lo) & mask; }

// Root square (already reduced), grid key and word of every point, and the digit counts of the
// first radix pass.
// (ITEMS words per thread: the tile size is chosen per context, see sort_items())
template <int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void morton_encode_hist(const float2 *__restrict__ Y, int n,
                                                                   const float4 *__restrict__ root, int bits, int ks,
                                                                   uint32_t mask, uint64_t *__restrict__ words,
                                                                   uint32_t *__restrict__ hist, int nblk)
{
    __shared__ uint32_t h[RADIX];
    for (int d = threadIdx.x; d < RADIX; d += SORT_THREADS) h[d] = 0u;
    __syncthreads();
    const float4 r = *root;
    const uint32_t qmax = (1u << bits) - 1u;
    const int base = blockIdx.x * (SORT_THREADS * ITEMS);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int e = base + k * SORT_THREADS + (int)threadIdx.x;
        if (e < n) {
            const uint64_t w = (grid_key(Y[e], r, qmax) << ks) | (uint32_t)e;
            words[e] = w;
            atomicAdd(&h[digit_of(w, ks, mask)], 1u);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < RADIX; d += SORT_THREADS) hist[(size_t)blockIdx.x * RADIX + d] = h[d];
}

template <int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void radix_hist(const uint64_t *__restrict__ words, int n, int lo, uint32_t mask,
                                                           uint32_t *__restrict__ hist, int nblk)
{
    __shared__ uint32_t h[RADIX];
    for (int d = threadIdx.x; d < RADIX; d += SORT_THREADS) h[d] = 0u;
    __syncthreads();
    const int base = blockIdx.x * (SORT_THREADS * ITEMS);
    uint64_t w[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {          // all loads in flight before the first count
        const int e = base + k * SORT_THREADS + (int)threadIdx.x;
        w[k] = e < n ? words[e] : 0ull;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if (base + k * SORT_THREADS + (int)threadIdx.x < n) atomicAdd(&h[digit_of(w[k], lo, mask)], 1u);
    __syncthreads();
    for (int d = threadIdx.x; d < RADIX; d += SORT_THREADS) hist[(size_t)blockIdx.x * RADIX + d] = h[d];
}

// hist[t][d] becomes the number of words with digit d in tiles before t; dtot[d] the digit's total.
// A workgroup takes SCAN_DIGITS neighbouring digits; SCAN_SEGS threads share a digit, each a segment of
// the tiles, whose counts it loads in batches (so that its loads are in flight together).
constexpr int SCAN_DIGITS = 16, SCAN_SEGS = 64, SCAN_BATCH = 8;
__global__ __launch_bounds__(SCAN_DIGITS * SCAN_SEGS) void radix_scan(uint32_t *__restrict__ hist, int nblk,
                                                                      uint32_t *__restrict__ dtot)
{
    __shared__ uint32_t ssum[SCAN_SEGS][SCAN_DIGITS];
    const int dl = (int)threadIdx.x % SCAN_DIGITS, sg = (int)threadIdx.x / SCAN_DIGITS;
    const int d = blockIdx.x * SCAN_DIGITS + dl;
    const int len = (nblk + SCAN_SEGS - 1) / SCAN_SEGS;
    const int t0 = min(nblk, sg * len), t1 = min(nblk, t0 + len);
    uint32_t sum = 0;
    for (int tb = t0; tb < t1; tb += SCAN_BATCH) {
        uint32_t v[SCAN_BATCH];
#pragma unroll
        for (int k = 0; k < SCAN_BATCH; ++k) v[k] = tb + k < t1 ? hist[(size_t)(tb + k) * RADIX + d] : 0u;
#pragma unroll
        for (int k = 0; k < SCAN_BATCH; ++k) sum += v[k];
    }
    ssum[sg][dl] = sum;
    __syncthreads();
    uint32_t run = 0, all = 0;
    for (int k = 0; k < SCAN_SEGS; ++k) {
        const uint32_t v = ssum[k][dl];
        run += k < sg ? v : 0u;
        all += v;
    }
    if (sg == 0) dtot[d] = all;
    for (int tb = t0; tb < t1; tb += SCAN_BATCH) {
        uint32_t v[SCAN_BATCH];
#pragma unroll
        for (int k = 0; k < SCAN_BATCH; ++k) v[k] = tb + k < t1 ? hist[(size_t)(tb + k) * RADIX + d] : 0u;
#pragma unroll
        for (int k = 0; k < SCAN_BATCH; ++k) {
            if (tb + k < t1) hist[(size_t)(tb + k) * RADIX + d] = run;
            run += v[k];
        }
    }
}

// Exclusive prefix over the workgroup of one value per thread (SORT_THREADS threads); all threads call.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *wsum /* SORT_THREADS / 64 */)
{
    int tot;
    const int ex = wave_excl_scan((int)v, &tot);
    const int w = (int)threadIdx.x >> 6;
    __syncthreads();
    if (lane_id() == 0) wsum[w] = (uint32_t)tot;
    __syncthreads();
    uint32_t wb = 0;
    for (int k = 0; k < w; ++k) wb += wsum[k];
    return wb + (uint32_t)ex;
}

// Workgroups reach the eight XCDs in turn.  Tile numbers are dealt so that each XCD works on a
// contiguous range of tiles: the pieces of one digit's output run that neighbouring tiles write
// are adjacent in memory, and this way they meet in one second-level cache and leave it as whole lines.
__device__ __forceinline__ int scatter_tile(int block, int nblk)
{
    const int per = (nblk + 7) / 8;
    return (block % 8) * per + block / 8;
}

template <int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void radix_scatter(const uint64_t *__restrict__ in, uint64_t *__restrict__ out,
                                                              int n, int lo, uint32_t mask,
                                                              const uint32_t *__restrict__ hist,
                                                              const uint32_t *__restrict__ dtot, int nblk)
{
    constexpr int NW = SORT_THREADS / WAVE, DPT = RADIX / SORT_THREADS;   // digits per thread
    constexpr int TILE = SORT_THREADS * ITEMS;
    // per-wave running digit counts, later per-wave starts; once every word knows its place in the
    // locally sorted tile the same memory holds that tile
    constexpr size_t OVERLAY = sizeof(uint16_t) * NW * RADIX > (size_t)TILE * 8 ? sizeof(uint16_t) * NW * RADIX
                                                                                   : (size_t)TILE * 8;
    __shared__ __align__(16) unsigned char overlay[OVERLAY];
    uint16_t (*whist)[RADIX] = reinterpret_cast<uint16_t (*)[RADIX]>(overlay);
    uint64_t *sorted = reinterpret_cast<uint64_t *>(overlay);
    __shared__ uint32_t gbase[RADIX];       // global start of (digit, this tile)
    __shared__ uint16_t lstart[RADIX];      // start of the digit inside the locally sorted tile
    __shared__ uint32_t wsum[NW];
    const int tile = scatter_tile((int)blockIdx.x, nblk);
    if (tile >= nblk) return;               // the same for every thread of the workgroup
    const int tid = (int)threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int tile0 = tile * TILE;
    const int base = tile0 + w * (WAVE * ITEMS);
    uint64_t word[ITEMS];
    uint32_t rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {       // requested first: they arrive while the offsets below are worked out
        const int e = base + r * WAVE + lane;
        word[r] = e < n ? in[e] : 0ull;
    }
    {
        uint32_t *z = reinterpret_cast<uint32_t *>(overlay);
        for (int i = tid; i < NW * RADIX / 2; i += SORT_THREADS) z[i] = 0u;
    }
    // where every digit's run starts in the output: digits before it, then tiles before this one
    {
        uint32_t t[DPT], before[DPT], sum = 0;
#pragma unroll
        for (int j = 0; j < DPT; ++j) {
            t[j] = dtot[tid * DPT + j];
            before[j] = hist[(size_t)tile * RADIX + tid * DPT + j];
            sum += t[j];
        }
        uint32_t run = block_excl_scan(sum, wsum);      // (its barriers also cover the zeroing above)
#pragma unroll
        for (int j = 0; j < DPT; ++j) {
            gbase[tid * DPT + j] = run + before[j];
            run += t[j];
        }
    }
    // Rank inside the wave's share, one item of every lane at a time: lanes with the same digit are
    // found with one ballot per digit bit.  whist[w] is touched by wave w alone, whose LDS
    // instructions execute in program order, so the rounds need no barrier between them.
    volatile uint16_t *mine = whist[w];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = base + r * WAVE + lane < n;
        const uint32_t d = digit_of(word[r], lo, mask);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < RADIX_BITS; ++b) {
            const uint64_t bal = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? bal : ~bal;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t pre = mine[d];
        rank[r] = pre + before;
        if (valid && before == 0) mine[d] = (uint16_t)(pre + (uint32_t)__popcll(peers));
    }
    __syncthreads();
    // per digit: where each wave's share starts inside the tile's run, and where the run starts
    // inside the locally sorted tile
    {
        uint32_t tot[DPT], sum = 0;
#pragma unroll
        for (int j = 0; j < DPT; ++j) {
            uint32_t acc = 0;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                const uint32_t c = whist[k][tid * DPT + j];
                whist[k][tid * DPT + j] = (uint16_t)acc;
                acc += c;
            }
            tot[j] = acc;
            sum += acc;
        }
        uint32_t run = block_excl_scan(sum, wsum);
#pragma unroll
        for (int j = 0; j < DPT; ++j) { lstart[tid * DPT + j] = (uint16_t)run; run += tot[j]; }
    }
    __syncthreads();
    // stable local sort through LDS ...
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = digit_of(word[r], lo, mask);
        rank[r] += (uint32_t)lstart[d] + (uint32_t)whist[w][d];
    }
    __syncthreads();      // the counts are no longer needed: their memory becomes the sorted tile
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if (base + r * WAVE + lane < n) sorted[min(rank[r], (uint32_t)TILE - 1u)] = word[r];
    __syncthreads();
    // ... so that consecutive threads write consecutive addresses within each digit's run
    const int cnt = min(TILE, n - tile0);
    for (int j = tid; j < cnt; j += SORT_THREADS) {
        const uint64_t v = sorted[j];
        const uint32_t d = digit_of(v, lo, mask);
        const uint32_t pos = gbase[d] + ((uint32_t)j - (uint32_t)lstart[d]);
        if (pos < (uint32_t)n) out[pos] = v;
    }
}

// the low 32 bits of every word
__global__ __launch_bounds__(256) void unpack_perm_k(const uint64_t *__restrict__ words, int n, uint32_t *__restrict__ perm)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) perm[p] = (uint32_t)words[p];
}

// ------------------------------------------------------------------ cells opened at each position
// The searches below are chains of dependent reads of the sorted keys, almost always within a
// few dozen positions of where they start.  Each workgroup therefore keeps the keys of its own
// positions plus a halo on both sides in LDS; reads outside that window go to memory.
constexpr int KEY_HALO = 256;

struct KeyWindow {
    const uint64_t *__restrict__ words;  // sorted words in memory (key << ks | slot)
    const uint64_t *lds;                 // keys of positions [lo, lo + len)
    uint32_t lo, len;
    int ks;
    __device__ __forceinline__ uint64_t operator[](uint32_t q) const
    {
        const uint32_t off = q - lo;
        return off < len ? lds[off] : words[q] >> ks;
    }
};

// Keys of positions [lo, ...) in LDS, for searches that are known to stay inside.
struct LdsKeys {
    const uint64_t *lds;
    uint32_t lo;
    __device__ __forceinline__ uint64_t operator[](uint32_t q) const { return lds[q - lo]; }
};

// Cooperative fill; the caller synchronises the workgroup afterwards.
__device__ __forceinline__ KeyWindow key_window_fill(const uint64_t *__restrict__ words, int ks, uint32_t n, uint32_t first,
                                                     uint32_t count, uint64_t *lds)
{
    KeyWindow w;
    w.words = words;
    w.lds = lds;
    w.ks = ks;
    w.lo = first > (uint32_t)KEY_HALO ? first - KEY_HALO : 0u;
    const uint32_t hi = min(n, first + count + KEY_HALO);
    w.len = hi > w.lo ? hi - w.lo : 0u;
    for (uint32_t t = threadIdx.x; t < w.len; t += blockDim.x) lds[t] = words[w.lo + t] >> ks;
    return w;
}

// Sorted keys: the positions whose key shifted right by sh equals pre form one contiguous run.
template <class Keys>
__device__ __forceinline__ uint32_t run_end(const Keys &keys, uint32_t n, uint32_t p, int sh, uint64_t pre)
{
    uint32_t lo = p, hi, step = 1;
    for (;;) {
        uint64_t cand = (uint64_t)p + step;
        if (cand >= n) { hi = n; break; }
        if ((keys[cand] >> sh) != pre) { hi = (uint32_t)cand; break; }
        lo = (uint32_t)cand;
        step <<= 1;
    }
    while (hi - lo > 1) {
        uint32_t mid = lo + ((hi - lo) >> 1);
        if ((keys[mid] >> sh) != pre) hi = mid; else lo = mid;
    }
    return hi;
}

__device__ __forceinline__ uint32_t run_begin(const KeyWindow &keys, uint32_t p, int sh, uint64_t pre)
{
    int64_t lo, hi = p, step = 1;
    for (;;) {
        int64_t cand = (int64_t)p - step;
        if (cand < 0) { lo = -1; break; }
        if ((keys[cand] >> sh) != pre) { lo = cand; break; }
        hi = cand;
        step <<= 1;
    }
    while (hi - lo > 1) {
        int64_t mid = lo + ((hi - lo) >> 1);
        if ((keys[mid] >> sh) != pre) lo = mid; else hi = mid;
    }
    return (uint32_t)hi;
}

// Depths [tmin, tend) of the cells that start at sorted position p.
__device__ __forceinline__ void levels_at(const KeyWindow &keys, uint32_t n, uint32_t p, int B,
                                          uint32_t C, int *tmin_out, int *tend_out)
{
    uint64_t key = keys[p];
    int tmin;
    if (p == 0) tmin = 0;
    else {
        uint64_t x = key ^ keys[p - 1];
        tmin = x ? B - ((63 - __clzll((long long)x)) >> 1) : B + 1;
    }
    int tend = tmin;
    if (tmin <= B) {
        uint32_t pc;   // number of points in the parent of the candidate cell
        if (tmin == 0) pc = 0xFFFFFFFFu;
        else if (tmin == 1) pc = n;
        else {
            int sh = 2 * (B - (tmin - 1));
            uint64_t pre = key >> sh;
            pc = run_end(keys, n, p, sh, pre) - run_begin(keys, p, sh, pre);
        }
        int t = tmin;
        while (t <= B && pc > C) {
            tend = t + 1;
            if (t == 0) pc = n;
            else {
                int sh = 2 * (B - t);
                pc = run_end(keys, n, p, sh, key >> sh) - p;
            }
            ++t;
        }
    }
    *tmin_out = tmin;
    *tend_out = tend;
}

// The same answer without any search when leaf_cap is small: the cell of depth s around p holds
// more than C points iff at least C of the 2C nearest positions (C on either side) share p's
// top s digits (L[j], R[j]: number of leading digits p shares with positions p-j, p+j).
constexpr int LEVELS_WINDOW_MAXC = 16;

__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b, int B)
{
    const uint64_t x = a ^ b;
    return x ? B - 1 - ((63 - __clzll((long long)x)) >> 1) : B;
}

// The keys are sorted, so the digits p shares with p+j are the fewest shared by any two
// neighbours in between: with adj[q] = digits shared by positions q and q+1 (-1 beyond either end
// of the array), R[j] = min(adj[p], .., adj[p+j-1]) and L[j] = min(adj[p-1], .., adj[p-j]).  Every
// workgroup works adj out once for its positions and a margin (one 64-bit comparison per position),
// after which a position needs 2C byte reads and minima.
// CT > 0: leaf_cap known at compile time (all indices static, no bisection); CT = 0: any
// leaf_cap <= LEVELS_WINDOW_MAXC at run time.  adj points at the entry of position p.
template <int CT>
__device__ __forceinline__ void levels_window(const signed char *adj, int B, int C, int *tmin_out, int *tend_out)
{
    const int prev = adj[-1];
    const int tmin = prev == B ? B + 1 : prev + 1;       // (position 0: adj[-1] = -1, depth 0)
    int smax;
    if (CT > 0) {
        // C-th largest of the two non-increasing lists: max over k of min(L[k], R[CT - k]), with
        // L[0] = R[0] = B standing for "no neighbour needed on that side"
        int L[CT + 1], R[CT + 1];
        L[0] = R[0] = B;
#pragma unroll
        for (int j = 1; j <= CT; ++j) {
            L[j] = min(L[j - 1], (int)adj[-j]);
            R[j] = min(R[j - 1], (int)adj[j - 1]);
        }
        smax = -1;
#pragma unroll
        for (int k = 0; k <= CT; ++k) smax = max(smax, min(L[k], R[CT - k]));
    } else {
        int L[LEVELS_WINDOW_MAXC], R[LEVELS_WINDOW_MAXC];
        int l = B, r = B;
#pragma unroll
        for (int j = 1; j <= LEVELS_WINDOW_MAXC; ++j) {
            l = min(l, (int)adj[-j]);
            r = min(r, (int)adj[j - 1]);
            L[j - 1] = j <= C ? l : -1;
            R[j - 1] = j <= C ? r : -1;
        }
        // deepest s in [0, B] with at least C of the 2C neighbours sharing s digits (-1 if none):
        // the count is non-increasing in s, so bisect
        int lo = -1, hi = B + 1;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            int cnt = 0;
#pragma unroll
            for (int j = 0; j < LEVELS_WINDOW_MAXC; ++j) cnt += (L[j] >= mid) + (R[j] >= mid);
            if (cnt >= C) lo = mid; else hi = mid;
        }
        smax = lo;
    }
    // cell (t, p) exists iff t == 0 or the depth t-1 cell around p holds more than C points
    int tend = min(B, smax + 1) + 1;
    if (tend < tmin) tend = tmin;
    *tmin_out = tmin;
    *tend_out = tend;
}

// Also moves the points into spatial order (step 4), writes the order itself (position -> slot)
// and reduces each tile's (cells, sum x, sum y).  CT < 0: any leaf_cap, by searching the keys.
template <int CT>
__global__ __launch_bounds__(LEVEL_THREADS) void gather_levels(const float2 *__restrict__ Y,
                                                               const uint64_t *__restrict__ words, int ks, int n, int B,
                                                               int C, float2 *__restrict__ Ys,
                                                               uint32_t *__restrict__ perm, uint16_t *__restrict__ lev,
                                                               ScanPart *__restrict__ part,
                                                               uint32_t *__restrict__ counters)
{
    __shared__ double sx[4], sy[4];
    __shared__ uint32_t sc[4];
    constexpr int MARGIN = LEVELS_WINDOW_MAXC + 1;
    __shared__ uint64_t kwin[CT < 0 ? LEVEL_TILE + 2 * KEY_HALO : 1];
    __shared__ signed char adjw[CT < 0 ? 1 : LEVEL_TILE + 2 * MARGIN];
    // the list of large cells (write_cells) and the work counters of the walk start at zero
    if (blockIdx.x == 0 && threadIdx.x < 1 + WALK_COUNTERS) counters[threadIdx.x] = 0u;
    const int first = blockIdx.x * LEVEL_TILE;
    KeyWindow kw;
    if (CT < 0) {
        kw = key_window_fill(words, ks, (uint32_t)n, (uint32_t)first, LEVEL_TILE, kwin);
    } else {
        // adjw[i]: digits shared by positions q = first - MARGIN + i and q + 1
        for (int i = threadIdx.x; i < LEVEL_TILE + 2 * MARGIN; i += LEVEL_THREADS) {
            const int q = first - MARGIN + i;
            adjw[i] = (q < 0 || q + 1 >= n) ? (signed char)-1
                                            : (signed char)common_digits(words[q] >> ks, words[q + 1] >> ks, B);
        }
    }
    double ax = 0.0, ay = 0.0;
    uint32_t ac = 0;
    float2 y[LEVEL_ITEMS];
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) {
        const int p = first + k * LEVEL_THREADS + threadIdx.x;
        y[k] = make_float2(0.f, 0.f);
        if (p < n) {
            const uint32_t slot = min((uint32_t)(words[p] & ((1ull << ks) - 1ull)), (uint32_t)n - 1u);
            perm[p] = slot;
            y[k] = Y[slot];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) {
        const int p = first + k * LEVEL_THREADS + threadIdx.x;
        if (p < n) {
            Ys[p] = y[k];
            ax += (double)y[k].x; ay += (double)y[k].y;
            int tmin, tend;
            if constexpr (CT < 0) levels_at(kw, (uint32_t)n, (uint32_t)p, B, (uint32_t)C, &tmin, &tend);
            else levels_window<CT>(adjw + MARGIN + (p - first), B, C, &tmin, &tend);
            lev[p] = (uint16_t)(tmin | (tend << 8));
            ac += (uint32_t)(tend - tmin);
        }
    }
    ax = wave_sum(ax); ay = wave_sum(ay); ac = wave_sum(ac);
    int w = threadIdx.x >> 6;
    if (lane_id() == 0) { sx[w] = ax; sy[w] = ay; sc[w] = ac; }
    __syncthreads();
    if (threadIdx.x == 0) {
        ScanPart q;
        q.sx = ((sx[0] + sx[1]) + sx[2]) + sx[3];
        q.sy = ((sy[0] + sy[1]) + sy[2]) + sy[3];
        q.cnt = sc[0] + sc[1] + sc[2] + sc[3];
        q.pad = 0;
        part[blockIdx.x] = q;
    }
}

// Per position: index of the first cell opened there, and the running sums of the sorted
// coordinates (ps[p] = sum of Ys[0..p), ps[n] = total).  Every workgroup first adds up the tile
// sums before its own tile (in a fixed order, so a run is reproducible; a few KB from the
// second-level cache instead of one more kernel); the last one also knows the number of cells.
__global__ __launch_bounds__(LEVEL_THREADS) void downsweep(const float2 *__restrict__ Ys,
                                                           const uint16_t *__restrict__ lev, int n,
                                                           const ScanPart *__restrict__ part,
                                                           uint32_t *__restrict__ cellseq, double2 *__restrict__ ps,
                                                           uint32_t *__restrict__ cell_p, uint8_t *__restrict__ cell_t,
                                                           uint32_t cap_cells, uint32_t *__restrict__ ncells,
                                                           uint32_t *status)
{
    __shared__ double wx[4], wy[4];
    __shared__ uint32_t wc[4];
    __shared__ double bx[4], by[4];
    __shared__ uint32_t bc[4];
    const int tid = threadIdx.x, w = tid >> 6;
    // tiles before this one
    double qx = 0.0, qy = 0.0;
    uint32_t qc = 0;
    for (int i = tid; i < (int)blockIdx.x; i += LEVEL_THREADS) {
        const ScanPart q = part[i];
        qx += q.sx; qy += q.sy; qc += q.cnt;
    }
    qx = wave_sum(qx); qy = wave_sum(qy); qc = wave_sum(qc);
    if (lane_id() == 0) { bx[w] = qx; by[w] = qy; bc[w] = qc; }
    int p0 = blockIdx.x * LEVEL_TILE + tid * LEVEL_ITEMS;
    float2 y[LEVEL_ITEMS];
    uint32_t c[LEVEL_ITEMS], t0[LEVEL_ITEMS];
    double ax = 0.0, ay = 0.0;
    uint32_t ac = 0;
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) {
        int p = p0 + k;
        if (p < n) {
            y[k] = Ys[p];
            uint32_t l = lev[p];
            c[k] = (l >> 8) - (l & 0xFFu);
            t0[k] = l & 0xFFu;
        } else { y[k] = make_float2(0.f, 0.f); c[k] = 0; t0[k] = 0; }
        ax += (double)y[k].x; ay += (double)y[k].y; ac += c[k];
    }
    double ix = ax, iy = ay;
    uint32_t icn = ac;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        double tx = __shfl_up(ix, o, WAVE), ty = __shfl_up(iy, o, WAVE);
        uint32_t tc = __shfl_up(icn, o, WAVE);
        if (lane_id() >= o) { ix += tx; iy += ty; icn += tc; }
    }
    if (lane_id() == WAVE - 1) { wx[w] = ix; wy[w] = iy; wc[w] = icn; }
    __syncthreads();
    double px = ((bx[0] + bx[1]) + bx[2]) + bx[3], py = ((by[0] + by[1]) + by[2]) + by[3];
    uint32_t pc = bc[0] + bc[1] + bc[2] + bc[3];
    for (int k = 0; k < w; ++k) { px += wx[k]; py += wy[k]; pc += wc[k]; }
    px += ix - ax; py += iy - ay; pc += icn - ac;
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) {
        int p = p0 + k;
        if (p < n) {
            cellseq[p] = pc;
            ps[p] = make_double2(px, py);
            for (uint32_t q = 0; q < c[k]; ++q)
                if (pc + q < cap_cells) { cell_p[pc + q] = (uint32_t)p; cell_t[pc + q] = (uint8_t)(t0[k] + q); }
            px += (double)y[k].x; py += (double)y[k].y; pc += c[k];
            if (p == n - 1) {
                cellseq[n] = pc;
                ps[n] = make_double2(px, py);
                *ncells = pc;
                if (pc > cap_cells) atomicOr(status, TSNE_STATUS_CELL_OVERFLOW);
            }
        }
    }
}

// First position in [s, e) whose digit (2 bits at sh) is >= q; e if none.
template <class Keys>
__device__ __forceinline__ uint32_t digit_lower_bound(const Keys &keys, uint32_t s, uint32_t e,
                                                      int sh, uint32_t q)
{
    while (s < e) {
        uint32_t mid = s + ((e - s) >> 1);
        if (((uint32_t)(keys[mid] >> sh) & 3u) < q) s = mid + 1; else e = mid;
    }
    return s;
}

// One lane per cell (cells are numbered in pre-order, so the cells of a workgroup start at
// non-decreasing positions and the keys they search sit in one stretch of CELL_WINDOW positions,
// staged in LDS).  A cell whose run of positions ends inside that stretch is finished on the spot,
// by searches that never leave LDS.  The large cells near the top of the tree would each be a
// chain of dozens of dependent memory reads in a single lane; they (and any cell that starts past
// the stretch) are put on a list instead and finished by write_big_cells, one wave per search.
constexpr int CELL_WINDOW = 2048;

// End of the cell (p, t) and the first positions of its children after the first; returns their number.
template <class Keys>
__device__ __forceinline__ int cell_extent(const Keys &keys, uint32_t lim, uint32_t n, uint32_t p, int t, int B, int C,
                                           uint64_t key, uint32_t *e_out, bool *leaf_out, uint32_t kid_pos[3])
{
    const uint32_t e = (t == 0) ? n : run_end(keys, lim, p, 2 * (B - t), key >> (2 * (B - t)));
    const bool leaf = e - p <= (uint32_t)C || t == B;
    int nk = 0;
    if (!leaf) {
        const int sh = 2 * (B - t - 1);
        uint32_t s = p;
        const uint32_t qfirst = (uint32_t)(key >> sh) & 3u;
        for (uint32_t q = qfirst + 1; q < 4; ++q) {
            const uint32_t b = digit_lower_bound(keys, s, e, sh, q);
            if (b < e && ((uint32_t)(keys[b] >> sh) & 3u) == q) kid_pos[nk++] = b;
            s = b;
        }
    }
    *e_out = e;
    *leaf_out = leaf;
    return nk;
}

__global__ __launch_bounds__(256) void write_cells(const uint64_t *__restrict__ words, int ks,
                                                   const uint32_t *__restrict__ cellseq,
                                                   const double2 *__restrict__ ps,
                                                   const uint32_t *__restrict__ cell_p, const uint8_t *__restrict__ cell_t,
                                                   const uint32_t *__restrict__ ncells, int n, int B, int C,
                                                   Cell *__restrict__ cells, uint32_t cap_cells,
                                                   uint32_t *__restrict__ big_count, uint2 *__restrict__ big_list,
                                                   uint32_t big_cap)
{
    __shared__ uint64_t kwin[CELL_WINDOW];
    const uint32_t m = min(*ncells, cap_cells);
    for (uint32_t base = blockIdx.x * 256u; base < m; base += gridDim.x * 256u) {
        const uint32_t id = base + threadIdx.x;
        const bool live = id < m;
        const uint32_t p_first = min(cell_p[base], (uint32_t)n - 1u);
        const uint32_t wlen = min((uint32_t)n - p_first, (uint32_t)CELL_WINDOW), wend = p_first + wlen;
        // the cell of this lane and the running sum at its first position: requested before the
        // window so that they travel together with it
        uint32_t p = 0;
        int t = 0;
        double2 s0 = make_double2(0.0, 0.0);
        if (live) { p = min(cell_p[id], (uint32_t)n - 1u); t = min((int)cell_t[id], B); s0 = ps[p]; }
        __syncthreads();                    // previous round's readers are done with the window
        for (uint32_t q = threadIdx.x; q < wlen; q += 256u) kwin[q] = words[p_first + q] >> ks;
        __syncthreads();
        if (!live) continue;
        const bool inside = p >= p_first && p < wend;
        const uint64_t key = inside ? kwin[p - p_first] : words[p] >> ks;
        // large: starts past the window, or shares its prefix with the window's last position
        // while the array goes on (the root, t = 0, shares it with every position)
        const bool big = !inside || (wend < (uint32_t)n &&
                                     (t == 0 || (kwin[wlen - 1] >> (2 * (B - t))) == (key >> (2 * (B - t)))));
        uint32_t e, kid_pos[3];
        bool leaf;
        int nk;
        if (big) {
            const uint32_t slot = atomicAdd(big_count, 1u);
            if (slot < big_cap) { big_list[slot] = make_uint2(p, (uint32_t)t); continue; }
            // list full (cannot happen for capacity n/8 + 1024 unless most cells are large): finish it here,
            // reading keys from memory wherever the window does not hold them
            KeyWindow kw;
            kw.words = words; kw.lds = kwin; kw.ks = ks; kw.lo = p_first; kw.len = wlen;
            nk = cell_extent(kw, (uint32_t)n, (uint32_t)n, p, t, B, C, key, &e, &leaf, kid_pos);
        } else {
            // the run ends before the window's last position (which is not part of it), or at n: no probe leaves LDS
            LdsKeys lk;
            lk.lds = kwin; lk.lo = p_first;
            nk = cell_extent(lk, wend < (uint32_t)n ? wend - 1u : (uint32_t)n, (uint32_t)n, p, t, B, C, key, &e, &leaf, kid_pos);
        }
        // the reads from memory that the searches lead to, together
        const double2 s1 = ps[e];
        const uint32_t cnt = e - p;
        Cell c;
        c.c1 = nk > 0 ? cellseq[kid_pos[0]] : TSNE_NONE;
        c.c2 = nk > 1 ? cellseq[kid_pos[1]] : TSNE_NONE;
        c.c3 = nk > 2 ? cellseq[kid_pos[2]] : TSNE_NONE;
        c.cx = (float)((s1.x - s0.x) / (double)cnt);
        c.cy = (float)((s1.y - s0.y) / (double)cnt);
        c.cnt = cnt;
        c.meta = (uint32_t)t | (leaf ? 0x100u : 0u);
        c.lo = p;
        cells[id] = c;
    }
}

// ---- few points: levels, prefix sums and cells in one launch of one workgroup, everything the searches need in LDS.
// (Four launches of a few microseconds each otherwise, all of them waiting for the one before: an iteration of 2000
// points 91 -> 71 us.  Beyond SMALL_TREE_MAX points the arrays outgrow a compute unit's LDS.)  Coordinates are added up in the order
// of gather_levels and downsweep, tile by tile, so that the centres of mass are the same to the bit.
constexpr int SMALL_TREE_MAX = 4096, SMALL_TREE_THREADS = 1024, SMALL_TREE_MARGIN = LEVELS_WINDOW_MAXC + 1;
static_assert(SMALL_TREE_MAX == SMALL_TREE_THREADS * LEVEL_ITEMS && SMALL_TREE_MAX == 4 * LEVEL_TILE, "four tiles");

__host__ __device__ inline size_t small_tree_lds(int n)
{
    return 16 * (size_t)(n + 1) + 8 * (size_t)n + 4 * (size_t)(n + 1) + (size_t)(n + 2 * SMALL_TREE_MARGIN) + (size_t)n;
}

template <int CT>
__global__ __launch_bounds__(SMALL_TREE_THREADS) void small_tree(const float2 *__restrict__ Y, const uint64_t *__restrict__ words,
                                                                 int ks, int n, int B, int C, float2 *__restrict__ Ys,
                                                                 uint32_t *__restrict__ perm, Cell *__restrict__ cells,
                                                                 uint32_t cap_cells, uint32_t *__restrict__ ncells,
                                                                 uint32_t *__restrict__ counters, uint32_t *status)
{
    constexpr int MARGIN = SMALL_TREE_MARGIN, NW = SMALL_TREE_THREADS / WAVE;
    extern __shared__ __align__(16) unsigned char tree_lds[];
    double2 *ps = reinterpret_cast<double2 *>(tree_lds);                     // running sums of the coordinates
    uint64_t *keys = reinterpret_cast<uint64_t *>(ps + n + 1);
    uint32_t *seq = reinterpret_cast<uint32_t *>(keys + n);                  // first cell of every position
    signed char *adj = reinterpret_cast<signed char *>(seq + n + 1);         // digits shared by neighbours (levels_window)
    unsigned char *first_depth = reinterpret_cast<unsigned char *>(adj + n + 2 * MARGIN);
    float2 *ysort = reinterpret_cast<float2 *>(ps);      // sorted points, until the running sums take their place
    __shared__ double wx[NW], wy[NW], tx[NW], ty[NW];
    __shared__ uint32_t wc[NW];
    const int tid = (int)threadIdx.x, w = tid >> 6, tile = tid / LEVEL_THREADS, tt = tid % LEVEL_THREADS;
    const int p0 = tid * LEVEL_ITEMS;
    if (tid < 1 + WALK_COUNTERS) counters[tid] = 0u;     // as gather_levels does: a resident walk counts from zero
    {
        double gx = 0.0, gy = 0.0;
#pragma unroll
        for (int k = 0; k < LEVEL_ITEMS; ++k) {
            const int p = tile * LEVEL_TILE + k * LEVEL_THREADS + tt;
            if (p < n) {
                const uint64_t word = words[p];
                const uint32_t slot = min((uint32_t)(word & ((1ull << ks) - 1ull)), (uint32_t)n - 1u);
                const float2 v = Y[slot];
                keys[p] = word >> ks;
                perm[p] = slot;
                Ys[p] = v;
                ysort[p] = v;
                gx += (double)v.x; gy += (double)v.y;
            }
        }
        gx = wave_sum(gx); gy = wave_sum(gy);
        if (lane_id() == 0) { tx[w] = gx; ty[w] = gy; }
    }
    __syncthreads();
    float2 y[LEVEL_ITEMS];
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) y[k] = p0 + k < n ? ysort[p0 + k] : make_float2(0.f, 0.f);
    for (int i = tid; i < n + 2 * MARGIN; i += SMALL_TREE_THREADS) {
        const int q = i - MARGIN;
        adj[i] = q < 0 || q + 1 >= n ? (signed char)-1 : (signed char)common_digits(keys[q], keys[q + 1], B);
    }
    __syncthreads();
    uint32_t c[LEVEL_ITEMS];
    double ax = 0.0, ay = 0.0;
    uint32_t ac = 0;
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) {
        const int p = p0 + k;
        c[k] = 0;
        if (p < n) {
            int tmin, tend;
            levels_window<CT>(adj + MARGIN + p, B, C, &tmin, &tend);
            first_depth[p] = (unsigned char)tmin;
            c[k] = (uint32_t)(tend - tmin);
        }
        ax += (double)y[k].x; ay += (double)y[k].y; ac += c[k];
    }
    double ix = ax, iy = ay;
    uint32_t icn = ac;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const double ux = __shfl_up(ix, o, WAVE), uy = __shfl_up(iy, o, WAVE);
        const uint32_t uc = __shfl_up(icn, o, WAVE);
        if (lane_id() >= o) { ix += ux; iy += uy; icn += uc; }
    }
    if (lane_id() == WAVE - 1) { wx[w] = ix; wy[w] = iy; wc[w] = icn; }
    __syncthreads();
    // the tiles before this one, as downsweep's first wave adds them (lanes 0 and 2, then 1 and 3)
    auto before = [&](const double *v) {
        auto of = [&](int b) { return ((v[4 * b] + v[4 * b + 1]) + v[4 * b + 2]) + v[4 * b + 3]; };
        return tile == 0 ? 0.0 : tile == 1 ? of(0) : tile == 2 ? of(0) + of(1) : (of(0) + of(2)) + of(1);
    };
    double px = before(tx), py = before(ty);
    uint32_t pc = 0, m = 0;
    for (int k = 0; k < NW; ++k) {
        if (k < w && k >= 4 * tile) { px += wx[k]; py += wy[k]; }
        if (k < w) pc += wc[k];
        m += wc[k];
    }
    px += ix - ax; py += iy - ay; pc += icn - ac;
#pragma unroll
    for (int k = 0; k < LEVEL_ITEMS; ++k) {
        const int p = p0 + k;
        if (p < n) {
            seq[p] = pc;
            ps[p] = make_double2(px, py);
            px += (double)y[k].x; py += (double)y[k].y; pc += c[k];
            if (p == n - 1) { seq[n] = pc; ps[n] = make_double2(px, py); }
        }
    }
    if (tid == 0) {
        *ncells = m;
        if (m > cap_cells) atomicOr(status, TSNE_STATUS_CELL_OVERFLOW);
    }
    __syncthreads();
    LdsKeys lk;
    lk.lds = keys; lk.lo = 0u;
    const uint32_t live = min(m, cap_cells);
    for (uint32_t id = (uint32_t)tid; id < live; id += SMALL_TREE_THREADS) {
        uint32_t lo = 0, hi = (uint32_t)n;      // the position that opens the cell: seq[lo] <= id < seq[lo + 1]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (seq[mid] <= id) lo = mid; else hi = mid;
        }
        const uint32_t p = lo;
        const int t = min((int)first_depth[p] + (int)(id - seq[p]), B);
        uint32_t e, kid_pos[3];
        bool leaf;
        const int nk = cell_extent(lk, (uint32_t)n, (uint32_t)n, p, t, B, C, keys[p], &e, &leaf, kid_pos);
        const double2 s0 = ps[p], s1 = ps[e];
        const uint32_t cnt = e - p;
        Cell q;
        q.c1 = nk > 0 ? seq[kid_pos[0]] : TSNE_NONE;
        q.c2 = nk > 1 ? seq[kid_pos[1]] : TSNE_NONE;
        q.c3 = nk > 2 ? seq[kid_pos[2]] : TSNE_NONE;
        q.cx = (float)((s1.x - s0.x) / (double)cnt);
        q.cy = (float)((s1.y - s0.y) / (double)cnt);
        q.cnt = cnt;
        q.meta = (uint32_t)t | (leaf ? 0x100u : 0u);
        q.lo = p;
        cells[id] = q;
    }
}

hipError_t small_tree_prepare()
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&small_tree<8>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)small_tree_lds(SMALL_TREE_MAX));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&small_tree<0>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)small_tree_lds(SMALL_TREE_MAX));
}

// First position i in [lo, n) with (key[i] >> sh) >= target (n if there is none), found by the
// whole wave: every round the 64 lanes probe 64 evenly spaced positions of the remaining range,
// which shrinks 64-fold, so five rounds cover any n.  All lanes must call with the same
// arguments; every probed index lies inside [lo, n) whatever the keys hold.
__device__ __forceinline__ uint32_t wave_shifted_lower_bound(const uint64_t *__restrict__ words, int ks, uint32_t lo,
                                                             uint32_t n, int sh, uint64_t target)
{
    uint32_t hi = n;
    const uint32_t lane = (uint32_t)lane_id();
    while (lo < hi) {
        const uint32_t step = (hi - lo + 63u) >> 6;
        const uint64_t probe = (uint64_t)lo + (uint64_t)(lane + 1u) * step - 1ull;
        bool below = false;
        if (probe < (uint64_t)hi) below = ((words[probe] >> ks) >> sh) < target;
        const uint32_t c = (uint32_t)__popcll(__ballot(below));   // the keys are sorted: lanes 0..c-1
        const uint64_t top = (uint64_t)lo + (uint64_t)(c + 1u) * step - 1ull;
        lo += c * step;
        hi = top < (uint64_t)hi ? (uint32_t)top : hi;
    }
    return lo;
}

// One workgroup per listed cell, one wave per search: wave 0 finds the end of the cell, waves
// 1-3 the first position of quadrants 1-3 among its points (all four are lower bounds in the
// globally sorted keys).
__global__ __launch_bounds__(256) void write_big_cells(const uint64_t *__restrict__ words, int ks,
                                                       const uint16_t *__restrict__ lev,
                                                       const uint32_t *__restrict__ cellseq,
                                                       const double2 *__restrict__ ps, int n, int B, int C,
                                                       Cell *__restrict__ cells, uint32_t cap_cells,
                                                       const uint32_t *__restrict__ big_count,
                                                       const uint2 *__restrict__ big_list, uint32_t big_cap)
{
    __shared__ uint32_t found_s[4];
    const int role = (int)(threadIdx.x >> 6);
    const uint32_t m = min(*big_count, big_cap);
    for (uint32_t item = blockIdx.x; item < m; item += gridDim.x) {
        const uint2 it = big_list[item];
        const uint32_t p = min(it.x, (uint32_t)n - 1u);
        const int t = min((int)it.y, B);
        const uint64_t key = words[p] >> ks;
        uint32_t found = (uint32_t)n;
        if (role == 0) {
            if (t > 0) {
                const int sh = 2 * (B - t);
                found = wave_shifted_lower_bound(words, ks, p, (uint32_t)n, sh, (key >> sh) + 1ull);
            }
        } else if (t < B) {
            const int sh = 2 * (B - t - 1);
            const uint64_t parent = t > 0 ? (key >> (2 * (B - t))) : 0ull;
            found = wave_shifted_lower_bound(words, ks, p, (uint32_t)n, sh, (parent << 2) + (uint64_t)role);
        }
        if (lane_id() == 0) found_s[role] = found;
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t e = found_s[0];
            const uint32_t b1 = min(found_s[1], e), b2 = min(found_s[2], e), b3 = min(found_s[3], e);
            const uint32_t l = lev[p];
            const uint32_t id = cellseq[p] + (uint32_t)(t - (int)(l & 0xFFu));
            if (id < cap_cells) {
                const uint32_t cnt = e - p;
                const double2 s0 = ps[p], s1 = ps[e];
                Cell c;
                c.cx = (float)((s1.x - s0.x) / (double)cnt);
                c.cy = (float)((s1.y - s0.y) / (double)cnt);
                c.cnt = cnt;
                const bool leaf = cnt <= (uint32_t)C || t == B;
                c.meta = (uint32_t)t | (leaf ? 0x100u : 0u);
                c.lo = p;
                c.c1 = c.c2 = c.c3 = TSNE_NONE;
                if (!leaf) {
                    // quadrant q > first quadrant exists iff its first position precedes the next boundary
                    const uint32_t qfirst = (uint32_t)(key >> (2 * (B - t - 1))) & 3u;
                    const uint32_t bnd[5] = {p, b1, b2, b3, e};
                    uint32_t kids[3];
                    int nk = 0;
                    for (uint32_t q = qfirst + 1; q < 4; ++q)
                        if (bnd[q] < bnd[q + 1]) kids[nk++] = cellseq[bnd[q]];
                    if (nk > 0) c.c1 = kids[0];
                    if (nk > 1) c.c2 = kids[1];
                    if (nk > 2) c.c3 = kids[2];
                }
                cells[id] = c;
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ export (tests only)
__global__ void export_cells_k(const Cell *__restrict__ cells, const uint32_t *__restrict__ ncells, int cap,
                               int32_t *depth, int32_t *lo, int32_t *hi, int32_t *leaf, float *com)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    int m = (int)min(*ncells, (uint32_t)cap);
    if (i >= m) return;
    Cell c = cells[i];
    if (depth) depth[i] = (int32_t)(c.meta & 0xFFu);
    if (lo) lo[i] = (int32_t)c.lo;
    if (hi) hi[i] = (int32_t)(c.lo + c.cnt);
    if (leaf) leaf[i] = (int32_t)((c.meta >> 8) & 1u);
    if (com) { com[2 * i] = c.cx; com[2 * i + 1] = c.cy; }
}

hipError_t launch_export_cells(tsne_ctx *c, int32_t cap, int32_t *depth, int32_t *lo, int32_t *hi, int32_t *leaf,
                               float *com, hipStream_t s)
{
    if (cap <= 0) return hipSuccess;
    int m = cap < c->cap_cells ? cap : c->cap_cells;
    hipLaunchKernelGGL(export_cells_k, dim3((m + 255) / 256), dim3(256), 0, s, c->cells, c->ncells, m, depth, lo, hi,
                       leaf, com);
    return hipGetLastError();
}

// keys and spatial order in the caller's numbering
__global__ __launch_bounds__(256) void export_order_k(const uint64_t *__restrict__ words, int ks,
                                                      const uint32_t *__restrict__ orig, int n, uint64_t *__restrict__ keys_out,
                                                      int32_t *__restrict__ perm_out)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint64_t w = words[p];
    const uint32_t o = orig[min((uint32_t)(w & ((1ull << ks) - 1ull)), (uint32_t)n - 1u)];
    if (keys_out) keys_out[min(o, (uint32_t)n - 1u)] = w >> ks;
    if (perm_out) perm_out[p] = (int32_t)o;
}

hipError_t launch_export_order(tsne_ctx *c, uint64_t *d_keys, int32_t *d_perm, hipStream_t s)
{
    const int n = c->p.n;
    hipLaunchKernelGGL(export_order_k, dim3((n + 255) / 256), dim3(256), 0, s, c->words[c->sorted_buf], c->key_shift,
                       c->orig[c->cur_state], n, d_keys, d_perm);
    return hipGetLastError();
}

// ------------------------------------------------------------------ host: enqueue the whole build
static int bbox_blocks(int n)
{
    int nb = (n + 255) / 256;
    return nb < BBOX_MAX_BLOCKS ? nb : BBOX_MAX_BLOCKS;
}

// Words per thread of the sort's tiles: a tile is a workgroup, and a launch is as long as its busiest compute unit,
// so the tile size is taken (from 8, 10 or 12 words a thread) to make the number of tiles per compute unit, rounded
// up, times the tile size smallest: 1,281,167 words are 313 tiles of 4096, which leaves 57 units with two, or 251
// tiles of 5120, one each.  Where tiles of two or four words a thread still are no more than one per unit they are taken:
// 60,000 words are 15 tiles of 4096, or 59 of 1024 on as many units.  (25 iterations of a run: 60,000 points 4.66
// -> 4.26 ms, 30,011 4.68 -> 4.25, 512,000 13.53 -> 13.23.)
int sort_items(int n, int num_cu)
{
    const int cu = num_cu > 0 ? num_cu : 256, fine = cu < SORT_FINE_TILES ? cu : SORT_FINE_TILES;
    for (int items = 2; items <= 4; items += 2)
        if (((long long)n + SORT_THREADS * items - 1) / (SORT_THREADS * items) <= fine) return items;
    int best = 8;
    long long best_cost = -1;
    for (int items = 8; items <= 12; items += 2) {
        const long long nblk = ((long long)n + SORT_THREADS * items - 1) / (SORT_THREADS * items);
        const long long cost = ((nblk + cu - 1) / cu) * items;
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = items; }
    }
    return best;
}

template <int ITEMS>
static void sort_passes(tsne_ctx *c, int lo, int nbits, bool hist0, hipStream_t s)
{
    const int n = c->p.n;
    const int nblk = (n + SORT_THREADS * ITEMS - 1) / (SORT_THREADS * ITEMS);
    const int grid = 8 * ((nblk + 7) / 8);       // scatter_tile() deals the tiles to the XCDs
    int cur = 0;
    for (int plo = lo; plo < lo + nbits; plo += RADIX_BITS) {
        const int width = lo + nbits - plo < RADIX_BITS ? lo + nbits - plo : RADIX_BITS;
        const uint32_t mask = (1u << width) - 1u;
        if (!(hist0 && plo == lo))
            hipLaunchKernelGGL(radix_hist<ITEMS>, dim3(nblk), dim3(SORT_THREADS), 0, s, c->words[cur], n, plo, mask, c->hist,
                               nblk);
        hipLaunchKernelGGL(radix_scan, dim3(RADIX / SCAN_DIGITS), dim3(SCAN_DIGITS * SCAN_SEGS), 0, s, c->hist, nblk,
                           c->dtot);
        hipLaunchKernelGGL(radix_scatter<ITEMS>, dim3(grid), dim3(SORT_THREADS), 0, s, c->words[cur], c->words[cur ^ 1], n,
                           plo, mask, c->hist, c->dtot, nblk);
        cur ^= 1;
    }
    c->sorted_buf = cur;
}

// Stable LSD radix sort of words[0] on bits [lo, lo + nbits), RADIX_BITS a pass.
hipError_t launch_sort(tsne_ctx *c, int lo, int nbits, bool hist0, hipStream_t s)
{
    switch (c->sort_items) {
    case 2: sort_passes<2>(c, lo, nbits, hist0, s); break;
    case 4: sort_passes<4>(c, lo, nbits, hist0, s); break;
    case 10: sort_passes<10>(c, lo, nbits, hist0, s); break;
    case 12: sort_passes<12>(c, lo, nbits, hist0, s); break;
    default: sort_passes<8>(c, lo, nbits, hist0, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_unpack_perm(tsne_ctx *c, hipStream_t s)
{
    const int n = c->p.n;
    hipLaunchKernelGGL(unpack_perm_k, dim3((n + 255) / 256), dim3(256), 0, s, c->words[c->sorted_buf], n, c->perm);
    return hipGetLastError();
}

// Step 1, first half: the caller's Y into slot order plus per-block bounding boxes.
hipError_t launch_gather_bbox(tsne_ctx *c, const float *d_Y, hipStream_t s)
{
    const int n = c->p.n;
    hipLaunchKernelGGL(bbox_partial, dim3(bbox_blocks(n)), dim3(256), 0, s, (const float2 *)d_Y,
                       c->orig[c->cur_state], c->Yi, n, c->bbox_part, c->status);
    c->bbox_nparts = bbox_blocks(n);
    return hipGetLastError();
}

// Step 1 second half on its own, for a step whose attraction wants the root square before the sort is enqueued.
hipError_t launch_tree_root(tsne_ctx *c, hipStream_t s)
{
    if (c->p.n <= SMALL_SORT_MAX) return hipSuccess;      // (there the root comes out of the one launch that also sorts)
    hipLaunchKernelGGL(bbox_final, dim3(1), dim3(c->bbox_nparts > 1024 ? 1024 : 256), 0, s, c->bbox_part, c->bbox_nparts,
                       c->p.morton_bits, c->root, c->status);
    c->root_fresh = 1;
    return hipGetLastError();
}

// Step 1 second half, step 2a and step 4: root square, keys, spatial sort.
hipError_t launch_tree_sort(tsne_ctx *c, hipStream_t s)
{
    const int n = c->p.n, B = c->p.morton_bits, ks = c->key_shift;
    const float2 *Y = c->Yi;
    if (n <= (c->identity ? RANK_MAX_CALLER : RANK_MAX)) return launch_rank_sort(c, s);
    if (!c->root_fresh)
        hipLaunchKernelGGL(bbox_final, dim3(1), dim3(c->bbox_nparts > 1024 ? 1024 : 256), 0, s, c->bbox_part, c->bbox_nparts, B,
                           c->root, c->status);
    c->root_fresh = 0;
    const int items = c->sort_items, nblk = (n + SORT_THREADS * items - 1) / (SORT_THREADS * items);
    const int width0 = 2 * B < RADIX_BITS ? 2 * B : RADIX_BITS;
    auto encode = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblk), dim3(SORT_THREADS), 0, s, Y, n, c->root, B, ks, (1u << width0) - 1u, c->words[0],
                           c->hist, nblk);
    };
    switch (items) {
    case 2: encode(morton_encode_hist<2>); break;
    case 4: encode(morton_encode_hist<4>); break;
    case 10: encode(morton_encode_hist<10>); break;
    case 12: encode(morton_encode_hist<12>); break;
    default: encode(morton_encode_hist<8>); break;
    }
    return launch_sort(c, ks, 2 * B, true, s);
}

// Steps 2b, 2c and 3: cells, counts, centres of mass from the sorted keys.
hipError_t launch_tree_cells(tsne_ctx *c, hipStream_t s)
{
    const int n = c->p.n, B = c->p.morton_bits, C = c->p.leaf_cap, ks = c->key_shift;
    const float2 *Y = c->Yi;
    const int nb = (n + 255) / 256;
    const uint64_t *words = c->words[c->sorted_buf];
    if (n <= SMALL_TREE_MAX && C <= LEVELS_WINDOW_MAXC) {
        hipLaunchKernelGGL(C == 8 ? small_tree<8> : small_tree<0>, dim3(1), dim3(SMALL_TREE_THREADS), small_tree_lds(n), s, Y,
                           words, ks, n, B, C, c->Ys, c->perm, c->cells, (uint32_t)c->cap_cells, c->ncells, c->big_count, c->status);
        return hipGetLastError();
    }
    int nl = (n + LEVEL_TILE - 1) / LEVEL_TILE;
    if (C == 8)
        hipLaunchKernelGGL(gather_levels<8>, dim3(nl), dim3(LEVEL_THREADS), 0, s, Y, words, ks, n, B, C, c->Ys, c->perm,
                           c->lev, c->part, c->big_count);
    else if (C <= LEVELS_WINDOW_MAXC)
        hipLaunchKernelGGL(gather_levels<0>, dim3(nl), dim3(LEVEL_THREADS), 0, s, Y, words, ks, n, B, C, c->Ys, c->perm,
                           c->lev, c->part, c->big_count);
    else
        hipLaunchKernelGGL(gather_levels<-1>, dim3(nl), dim3(LEVEL_THREADS), 0, s, Y, words, ks, n, B, C, c->Ys, c->perm,
                           c->lev, c->part, c->big_count);
    hipLaunchKernelGGL(downsweep, dim3(nl), dim3(LEVEL_THREADS), 0, s, c->Ys, c->lev, n, c->part, c->cellseq, c->ps,
                       c->cell_p, c->cell_t, (uint32_t)c->cap_cells, c->ncells, c->status);
    // grid sized for n / 2 cells (a typical tree has about n / 3); the kernel strides if there are more
    hipLaunchKernelGGL(write_cells, dim3((nb + 1) / 2), dim3(256), 0, s, words, ks, c->cellseq, c->ps, c->cell_p, c->cell_t,
                       c->ncells, n, B, C, c->cells, (uint32_t)c->cap_cells, c->big_count, c->big_list,
                       (uint32_t)c->big_cap);
    hipLaunchKernelGGL(write_big_cells, dim3(4096), dim3(256), 0, s, words, ks, c->lev,
                       c->cellseq, c->ps, n, B, C, c->cells, (uint32_t)c->cap_cells, c->big_count, c->big_list,
                       (uint32_t)c->big_cap);
    return hipGetLastError();
}
