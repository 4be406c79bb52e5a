// Renumbering of the points.
//
// The paper names the attractive forces as the bottleneck because the sparsity pattern of P is
// disorganised (Sec. IV-D): row i gathers y_j from all over memory.  The library therefore keeps
// its own numbering of the points ("slots", `orig` maps them back to the caller's indices) in
// which neighbours in P get nearby numbers -- from the structure of P (below) or from the
// spatial order of the embedding, which the tree build computes anyway (Sec. III-C step 4).
// In that numbering almost all of P lies in a band around the diagonal.  The private copy of
// P is stored split: the near part (|column - row| <= ATTRACT_BAND), which the attraction
// kernel serves from a sliding window of Y in LDS, and the far remainder.  Values and the
// order of the entries inside each part of a row are those of the caller's P.
#include "tsne_internal.h"

#include <algorithm>

// position p of the new order takes over old slot s = perm[p]
__global__ __launch_bounds__(256) void reorder_state_k(const uint32_t *__restrict__ perm, int n,
                                                       const uint32_t *__restrict__ orig_in, uint32_t *__restrict__ orig_out,
                                                       const float2 *__restrict__ u_in, float2 *__restrict__ u_out,
                                                       const float2 *__restrict__ g_in, float2 *__restrict__ g_out,
                                                       uint32_t *__restrict__ inv)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t s = min(perm[p], (uint32_t)n - 1u);
    const uint32_t o = min(orig_in[s], (uint32_t)n - 1u);
    orig_out[p] = o;
    u_out[p] = u_in[s];
    g_out[p] = g_in[s];
    inv[o] = (uint32_t)p;
}

__global__ void zero_word_k(uint32_t *w) { *w = 0u; }

__device__ __forceinline__ bool in_band(uint32_t col_slot, int row_slot)
{
    const int d = (int)col_slot - row_slot;
    return d <= ATTRACT_BAND && d >= -ATTRACT_BAND;
}

// 16 lanes per slot p: how many entries of the caller's row orig[p] fall in the band
__global__ __launch_bounds__(256) void split_count_k(const uint32_t *__restrict__ orig, const uint32_t *__restrict__ inv,
                                                     int n, const int32_t *__restrict__ urp,
                                                     const int32_t *__restrict__ ucol, int32_t *__restrict__ len_near,
                                                     int32_t *__restrict__ len_far, uint32_t *__restrict__ far_rows,
                                                     uint32_t *__restrict__ far_count)
{
    const int p = (int)((blockIdx.x * 256u + threadIdx.x) / 16);
    const int sub = (int)(threadIdx.x % 16);
    int near = 0, len = 0;
    if (p < n) {
        const uint32_t u = min(orig[p], (uint32_t)n - 1u);
        const int src = urp[u];
        len = urp[u + 1] - src;
        for (int e = sub; e < len; e += 16)
            near += in_band(inv[min((uint32_t)ucol[src + e], (uint32_t)n - 1u)], p) ? 1 : 0;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) near += __shfl_xor(near, o, WAVE);
    if (p < n && sub == 0) {
        len_near[p] = (near + ATTRACT_CHUNK - 1) / ATTRACT_CHUNK * ATTRACT_CHUNK;     // padded to whole chunks
        len_far[p] = len - near;
        if (len > near) far_rows[atomicAdd(far_count, 1u)] = (uint32_t)p;   // any order will do
    }
}

// rp_out = base + exclusive prefix sum of len, in two launches: sums of SCAN_TILE numbers, then every workgroup adds up
// the sums before its own (8 bytes per 8192 numbers) and scans its tile.  (One workgroup doing all of it took 2.9 ms for
// 1,281,167 rows, each thread walking its own stretch of memory; the two launches take 0.02.)
constexpr int SCAN_ITEMS = 8, SCAN_TILE = 1024 * SCAN_ITEMS;

// sum over the workgroup of 1024; every thread gets it
__device__ __forceinline__ long long block_sum_1024(long long v, long long *ws)
{
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    long long t = 0;
    for (int q = 0; q < 16; ++q) t += ws[q];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(1024) void scan_sums_k(const int32_t *__restrict__ len, int n, long long *__restrict__ sums)
{
    __shared__ long long ws[16];
    const int64_t i0 = (int64_t)blockIdx.x * SCAN_TILE;
    long long a = 0;
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS; ++q) {
        const int64_t i = i0 + q * 1024 + threadIdx.x;
        if (i < n) a += len[i];
    }
    a = block_sum_1024(a, ws);
    if (threadIdx.x == 0) sums[blockIdx.x] = a;
}

__global__ __launch_bounds__(1024) void scan_apply_k(const int32_t *__restrict__ len, int n, const long long *__restrict__ sums,
                                                     const int32_t *__restrict__ base, int32_t *__restrict__ rp_out)
{
    __shared__ long long ws[16];
    long long before = 0;
    for (unsigned b = threadIdx.x; b < blockIdx.x; b += 1024) before += sums[b];
    before = block_sum_1024(before, ws);
    const int64_t i0 = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int v[SCAN_ITEMS];
    long long a = 0;
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS; ++q) { v[q] = i0 + q < n ? len[i0 + q] : 0; a += v[q]; }
    long long inc = a;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        long long t = __shfl_up(inc, o, WAVE);
        if (lane_id() >= o) inc += t;
    }
    if (lane_id() == WAVE - 1) ws[threadIdx.x >> 6] = inc;
    __syncthreads();
    long long pre = before + inc - a + (base ? (long long)*base : 0ll);
    for (int q = 0; q < (int)(threadIdx.x >> 6); ++q) pre += ws[q];
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS; ++q) {
        if (i0 + q < n) { rp_out[i0 + q] = (int32_t)pre; pre += v[q]; }
        if (i0 + q == n - 1) rp_out[n] = (int32_t)pre;
    }
}

// sums: room for 8 bytes per SCAN_TILE numbers (the sort's digit counts, 2 bytes a point and more, are free here)
void launch_scan(const int32_t *len, int n, const int32_t *base, int32_t *rp_out, void *sums, hipStream_t s)
{
    const unsigned blocks = (unsigned)(((int64_t)n + SCAN_TILE - 1) / SCAN_TILE);
    hipLaunchKernelGGL(scan_sums_k, dim3(blocks), dim3(1024), 0, s, len, n, (long long *)sums);
    hipLaunchKernelGGL(scan_apply_k, dim3(blocks), dim3(1024), 0, s, len, n, (const long long *)sums, base, rp_out);
}

// 16 lanes copy one row: columns are relabelled, the entries go to the near or the far part in
// their original order, and the near part is filled up to whole chunks with (own slot, 0)
__global__ __launch_bounds__(256) void split_fill_k(const uint32_t *__restrict__ orig, const uint32_t *__restrict__ inv,
                                                    int n, const int32_t *__restrict__ urp,
                                                    const int32_t *__restrict__ ucol, const float *__restrict__ uval,
                                                    const int32_t *__restrict__ rp_near, const int32_t *__restrict__ rp_far,
                                                    uint16_t *__restrict__ col_near, int32_t *__restrict__ col_far,
                                                    float *__restrict__ val_s)
{
    const int p = (int)((blockIdx.x * 256u + threadIdx.x) / 16);
    const int sub = (int)(threadIdx.x % 16);
    if (p >= n) return;
    const int shift = (int)(lane_id() & 48);          // first lane of this 16-lane group
    const uint32_t below = (1u << sub) - 1u;
    const uint32_t u = min(orig[p], (uint32_t)n - 1u);
    const int src = urp[u], len = urp[u + 1] - src;
    int dn = rp_near[p], df = rp_far[p];
    const int far0 = rp_far[0];
    const int end_near = rp_near[p + 1];
    for (int e0 = 0; e0 < len; e0 += 16) {
        const int e = e0 + sub;
        const bool in = e < len;
        uint32_t cs = 0u;
        float v = 0.f;
        if (in) {
            cs = inv[min((uint32_t)ucol[src + e], (uint32_t)n - 1u)];
            v = uval[src + e];
        }
        const bool near = in && in_band(cs, p);
        const uint32_t mn = (uint32_t)(__ballot(near) >> shift) & 0xFFFFu;
        const uint32_t mf = (uint32_t)(__ballot(in && !near) >> shift) & 0xFFFFu;
        if (near) {   // near columns are stored as the byte offset of the point in the ring of Y
            const int d = dn + __popc(mn & below);
            col_near[d] = (uint16_t)((cs % (uint32_t)ATTRACT_RING) * 8u);
            val_s[d] = v;
        } else if (in) {
            const int d = df + __popc(mf & below);
            col_far[d - far0] = (int32_t)cs;
            val_s[d] = v;
        }
        dn += __popc(mn);
        df += __popc(mf);
    }
    for (int d = dn + sub; d < end_near; d += 16) {       // padding: own point, weight 0
        col_near[d] = (uint16_t)((p % ATTRACT_RING) * 8);
        val_s[d] = 0.f;
    }
}


// ---- the far part once more, bucketed by tiles (for attract_far_tiled)
// meta: [0] tiles in use, [1] largest value of P (bits of a non-negative float), [2] longest far row.
__global__ void ft_begin_k(uint32_t *meta) { meta[0] = 0u; meta[1] = 0u; meta[2] = 0u; }

__global__ __launch_bounds__(256) void ft_stats_k(const float *__restrict__ uval, int64_t nnz,
                                                  const int32_t *__restrict__ len_far, int n, uint32_t *meta)
{
    uint32_t pm = 0u, lm = 0u;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nnz; e += stride) {
        const float v = uval[e];
        if (v > 0.f) pm = max(pm, __float_as_uint(v));
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) lm = max(lm, (uint32_t)len_far[i]);
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        pm = max(pm, (uint32_t)__shfl_xor((int)pm, o, WAVE));
        lm = max(lm, (uint32_t)__shfl_xor((int)lm, o, WAVE));
    }
    if (lane_id() == 0) {
        if (pm) atomicMax(meta + 1, pm);
        if (lm) atomicMax(meta + 2, lm);
    }
}

// mode: 0 = tiles if the far part is at least half of the entries and there are at least FT_MIN_POINTS points
// (measured on four 50-dimensional blobs: 0.23 against 0.30 ms per iteration row by row at 128,000 points, 0.57
// against 0.47 at 256,000: below the limit all of Y stays in the second-level cache; a far part
// that is a minority -- clusters a little wider than the band -- is quicker row by row beside the tree
// build: measured on the 400,000-point, 200-cluster workload), 1 = never, 2 = always
__global__ void ft_decide_k(const int32_t *__restrict__ rp_far, int n, int64_t nnz, int mode, uint32_t *meta)
{
    const int64_t far_total = (int64_t)rp_far[n] - rp_far[0];
    meta[0] = far_total > 0 && (mode == 2 || (mode == 0 && far_total * 2 >= nnz && n >= FT_MIN_POINTS)) ? 1u : 0u;
    meta[4] = (uint32_t)far_total;      // for the host: how many workgroups the tile kernel is worth
}

__global__ __launch_bounds__(256) void ft_zero_k(uint32_t *__restrict__ cnt, int64_t tiles, const uint32_t *meta)
{
    if (!meta[0]) return;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < tiles; t += stride) cnt[t] = 0u;
}

// FILL: place the entries (the counts run down to 0 as positions are handed out).  A workgroup takes FT_SC_ROWS rows of
// one row tile, 16 lanes a row, counts its entries per column tile in LDS (FT_SC_TILES column tiles at a time) and
// asks for a range of each tile once: an atomic in device memory per entry took 12.5 ms to count and 20.6 ms to place
// the 80 M far entries of 512,000 points (their counters sit in eight second-level caches), the pair now takes 2.2 ms.
constexpr int FT_SC_ROWS = 384, FT_SC_TILES = 8192;
static_assert(FT_ROWS % FT_SC_ROWS == 0, "a workgroup's rows are in one row tile");
template <bool FILL>
__global__ __launch_bounds__(512) void ft_scatter_k(const int32_t *__restrict__ rp_far, const int32_t *__restrict__ col_far,
                                                    const float *__restrict__ val_s, int n, int nct,
                                                    uint32_t *__restrict__ cnt, const int32_t *__restrict__ ptr,
                                                    int32_t *__restrict__ tcol, uint16_t *__restrict__ trow,
                                                    float *__restrict__ tval, const uint32_t *meta)
{
    if (!meta[0]) return;
    __shared__ uint32_t h[FT_SC_TILES];
    const int row0 = (int)blockIdx.x * FT_SC_ROWS, row1 = min(n, row0 + FT_SC_ROWS);
    const int grp = (int)(threadIdx.x / 16), sub = (int)(threadIdx.x % 16);
    const int far0 = rp_far[0];
    const int64_t tile0 = (int64_t)(row0 / FT_ROWS) * nct;
    for (int c0 = 0; c0 < nct; c0 += FT_SC_TILES) {
        const int m = min(FT_SC_TILES, nct - c0);
        __syncthreads();
        for (int t = (int)threadIdx.x; t < m; t += 512) h[t] = 0u;
        __syncthreads();
        for (int p = row0 + grp; p < row1; p += 32)
            for (int e = rp_far[p] + sub; e < rp_far[p + 1]; e += 16) {
                const int t = (int)(min((uint32_t)col_far[e - far0], (uint32_t)n - 1u) / FT_COLS) - c0;
                if (t >= 0 && t < m) atomicAdd(&h[t], 1u);
            }
        __syncthreads();
        for (int t = (int)threadIdx.x; t < m; t += 512) {
            const uint32_t k = h[t];
            if (k == 0u) continue;
            if (!FILL) atomicAdd(cnt + tile0 + c0 + t, k);
            else h[t] = (uint32_t)ptr[tile0 + c0 + t] + atomicSub(cnt + tile0 + c0 + t, k) - k;   // any order inside the tile
        }
        if (!FILL) continue;
        __syncthreads();
        for (int p = row0 + grp; p < row1; p += 32)
            for (int e = rp_far[p] + sub; e < rp_far[p + 1]; e += 16) {
                const uint32_t cs = min((uint32_t)col_far[e - far0], (uint32_t)n - 1u);
                const int t = (int)(cs / FT_COLS) - c0;
                if (t < 0 || t >= m) continue;
                const uint32_t pos = atomicAdd(&h[t], 1u);
                tcol[pos] = (int32_t)cs;
                trow[pos] = (uint16_t)(p % FT_ROWS);
                tval[pos] = val_s[e];
            }
    }
}

// The entries of every tile, placed in any order, into the order of their columns, FT_SORT_PIECE entries
// at a time (a counting sort in LDS over the tile's FT_COLS columns).  A gather instruction pays per cache
// line of Y that its 64 lanes touch: 64 consecutive entries of a sorted piece of m entries span about
// 64 / m of the tile's 128 lines instead of some 50 of them.  The row sums do not depend on the order.
constexpr int FT_SORT_PIECE = 4096;
__global__ __launch_bounds__(256) void ft_sort_k(const int32_t *__restrict__ ptr, int64_t tiles, int nct,
                                                 int32_t *__restrict__ tcol, uint16_t *__restrict__ trow,
                                                 float *__restrict__ tval, const uint32_t *meta)
{
    if (!meta[0]) return;
    __shared__ int32_t scol[FT_SORT_PIECE];
    __shared__ float sval[FT_SORT_PIECE];
    __shared__ uint16_t srow[FT_SORT_PIECE];
    __shared__ uint32_t bin[FT_COLS];
    __shared__ uint32_t wsum[4];
    static_assert(FT_COLS % 256 == 0, "columns per thread");
    constexpr int BPT = FT_COLS / 256;
    const int tid = (int)threadIdx.x, w = tid >> 6;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int b0 = ptr[t], b1 = ptr[t + 1];
        const uint32_t c0 = (uint32_t)(t % nct) * (uint32_t)FT_COLS;
        for (int s0 = b0; s0 < b1; s0 += FT_SORT_PIECE) {     // (b0, b1: the same for every thread)
            const int m = min(FT_SORT_PIECE, b1 - s0);
            __syncthreads();                                  // the previous piece is written out
            for (int i = tid; i < FT_COLS; i += 256) bin[i] = 0u;
            __syncthreads();
            for (int i = tid; i < m; i += 256) {
                const int32_t cj = tcol[s0 + i];
                scol[i] = cj;
                srow[i] = trow[s0 + i];
                sval[i] = tval[s0 + i];
                atomicAdd(&bin[min((uint32_t)cj - c0, (uint32_t)FT_COLS - 1u)], 1u);
            }
            __syncthreads();
            uint32_t loc[BPT], sum = 0;
#pragma unroll
            for (int k = 0; k < BPT; ++k) { loc[k] = bin[tid * BPT + k]; sum += loc[k]; }
            int tot;
            const int ex = wave_excl_scan((int)sum, &tot);
            if (lane_id() == 0) wsum[w] = (uint32_t)tot;
            __syncthreads();
            uint32_t run = (uint32_t)ex;
            for (int k = 0; k < w; ++k) run += wsum[k];
#pragma unroll
            for (int k = 0; k < BPT; ++k) { bin[tid * BPT + k] = run; run += loc[k]; }
            __syncthreads();
            for (int i = tid; i < m; i += 256) {
                const int32_t cj = scol[i];
                const uint32_t pos = min(atomicAdd(&bin[min((uint32_t)cj - c0, (uint32_t)FT_COLS - 1u)], 1u), (uint32_t)m - 1u);
                tcol[s0 + pos] = cj;
                trow[s0 + pos] = srow[i];
                tval[s0 + pos] = sval[i];
            }
        }
    }
}

hipError_t launch_reorder(tsne_ctx *c, hipStream_t s, int tiles_mode)
{
    const int n = c->p.n;
    const uint32_t *perm = c->perm;
    const int a = c->cur_state, b = a ^ 1;
    hipLaunchKernelGGL(reorder_state_k, dim3((n + 255) / 256), dim3(256), 0, s, perm, n, c->orig[a], c->orig[b],
                       c->uYb[a], c->uYb[b], c->gainsb[a], c->gainsb[b], c->inv);
    const unsigned blocks = (unsigned)(((int64_t)n * 16 + 255) / 256);
    hipLaunchKernelGGL(zero_word_k, dim3(1), dim3(1), 0, s, c->far_count);
    hipLaunchKernelGGL(split_count_k, dim3(blocks), dim3(256), 0, s, c->orig[b], c->inv, n, c->user_row_ptr, c->user_col,
                       c->len_near, c->len_far, c->far_rows, c->far_count);
    launch_scan(c->len_near, n, nullptr, c->rp_near, c->hist, s);
    launch_scan(c->len_far, n, c->rp_near + n, c->rp_far, c->hist, s);
    hipLaunchKernelGGL(split_fill_k, dim3(blocks), dim3(256), 0, s, c->orig[b], c->inv, n, c->user_row_ptr, c->user_col,
                       c->user_val, c->rp_near, c->rp_far, c->col_near, c->col_far, c->val_s);
    if (c->ft_tiles > 0) {
        const unsigned sblocks = (unsigned)std::min<int64_t>(4096, (std::max<int64_t>(c->nnz, n) + 255) / 256);
        const unsigned scblocks = (unsigned)((n + FT_SC_ROWS - 1) / FT_SC_ROWS);
        const unsigned zblocks = (unsigned)std::min<int64_t>(4096, (c->ft_tiles + 255) / 256);
        hipLaunchKernelGGL(ft_begin_k, dim3(1), dim3(1), 0, s, c->ft_meta);
        hipLaunchKernelGGL(ft_stats_k, dim3(sblocks), dim3(256), 0, s, c->user_val, c->nnz, c->len_far, n, c->ft_meta);
        hipLaunchKernelGGL(ft_decide_k, dim3(1), dim3(1), 0, s, c->rp_far, n, c->nnz, tiles_mode, c->ft_meta);
        hipLaunchKernelGGL(ft_zero_k, dim3(zblocks), dim3(256), 0, s, c->ft_cnt, c->ft_tiles, c->ft_meta);
        hipLaunchKernelGGL(ft_scatter_k<false>, dim3(scblocks), dim3(512), 0, s, c->rp_far, c->col_far, c->val_s, n, c->ft_nct,
                           c->ft_cnt, c->ft_ptr, c->ft_col, c->ft_row, c->ft_val, c->ft_meta);
        launch_scan((const int32_t *)c->ft_cnt, (int)c->ft_tiles, nullptr, c->ft_ptr, c->hist, s);
        hipLaunchKernelGGL(ft_scatter_k<true>, dim3(scblocks), dim3(512), 0, s, c->rp_far, c->col_far, c->val_s, n, c->ft_nct,
                           c->ft_cnt, c->ft_ptr, c->ft_col, c->ft_row, c->ft_val, c->ft_meta);
        hipLaunchKernelGGL(ft_sort_k, dim3((unsigned)std::min<int64_t>(c->ft_tiles, 1 << 20)), dim3(256), 0, s, c->ft_ptr,
                           c->ft_tiles, c->ft_nct, c->ft_col, c->ft_row, c->ft_val, c->ft_meta);
    }
    c->cur_state = b;
    c->arow_valid = 0;
    c->identity = 0;
    return hipGetLastError();
}

// ---- ordering of the points by the structure of P alone
// x_i starts as a hash of i in [0,1) and is replaced T times by the p-weighted mean of x over
// row i of P.  Values inside a well-connected neighbourhood converge to a common value long
// before different neighbourhoods mix, so sorting by x groups the points the way P links them.
__device__ __forceinline__ uint32_t mix32(uint32_t v)
{
    v ^= v >> 16; v *= 0x7feb352du; v ^= v >> 15; v *= 0x846ca68bu; v ^= v >> 16;
    return v;
}

__global__ __launch_bounds__(256) void graph_seed_k(float *__restrict__ x, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = (float)(mix32((uint32_t)i + 0x9e3779b9u) >> 8) * (1.0f / 16777216.0f);
}

// What graph_sample_k and graph_relabel_k find out about a copy (words of SmoothSeen::count).
enum { SEEN_OUTSIDE, SEEN_ALL, SEEN_CLOSE, SEEN_REACH, SEEN_WORDS };
constexpr int SMOOTH_CLOSE = 256;
// Whether the passes on a copy go by windows (graph_smooth_window_k): of the entries of a sample of its rows, up to `outside`
// percent may lie outside, and up to `close` percent within SMOOTH_CLOSE places of the row, where gathers touch few lines.  The
// kernel that is not to run is launched all the same, and leaves.
struct SmoothSeen {
    uint32_t *count;      // null: no such choice, the kernel that is launched runs
    uint32_t outside, close;
};
__device__ __forceinline__ bool smooth_by_window(const SmoothSeen &s)
{
    const uint64_t all = s.count[SEEN_ALL];
    return (uint64_t)s.count[SEEN_OUTSIDE] * 100u <= all * s.outside && (uint64_t)s.count[SEEN_CLOSE] * 100u <= all * s.close;
}

// 16 U entries of a row from j on, U of them a lane's.  (Past its end: weight 0, and x of the row itself, which is near.  One
// value for all would be a cache line that the whole chip asks for: a pass over 200,000 points in four blobs 52 -> 76 us.)
template <int U>
__device__ __forceinline__ void smooth_gather(const int32_t *col, const float *val, const float *x, int n, int row, int j, int e, int sub,
                                              float &a, float &w)
{
    float v[U], xv[U];
    uint32_t c[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int i = j + sub + 16 * q;
        v[q] = i < e ? val[i] : 0.f;
        c[q] = i < e ? (uint32_t)col[i] : (uint32_t)row;
    }
#pragma unroll
    for (int q = 0; q < U; ++q) xv[q] = x[min(c[q], (uint32_t)n - 1u)];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        a = fmaf(v[q], xv[q], a);
        w += v[q];
    }
}

// a row: U entries a lane on their way, or four where the rest of it is no more and U is larger than six
template <int U>
__device__ __forceinline__ void smooth_gather_row(const int32_t *col, const float *val, const float *x, int n, int row, int j, int e, int sub,
                                                  float &a, float &w)
{
    if (U <= 6) {
        for (; j < e; j += 16 * U) smooth_gather<U>(col, val, x, n, row, j, e, sub, a, w);
    } else {
        for (; e - j > 64; j += 16 * U) smooth_gather<U>(col, val, x, n, row, j, e, sub, a, w);
        if (j < e) smooth_gather<4>(col, val, x, n, row, j, e, sub, a, w);
    }
}

template <int U>
__global__ __launch_bounds__(256) void graph_smooth_k(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                                      const float *__restrict__ val, const float *__restrict__ x, int n,
                                                      float *__restrict__ xo, SmoothSeen seen)
{
    const int row = (int)((blockIdx.x * 256u + threadIdx.x) / 16), r = min(row, n - 1);
    const int sub = (int)(threadIdx.x % 16);
    const int begin = row_ptr[r], end = row_ptr[r + 1];         // (on their way with the counts, not behind them)
    if (seen.count && smooth_by_window(seen)) return;
    float a = 0.f, w = 0.f;
    if (row < n) smooth_gather_row<U>(col, val, x, n, row, begin, end, sub, a, w);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) { a += __shfl_xor(a, o, WAVE); w += __shfl_xor(w, o, WAVE); }
    if (row < n && sub == 0) xo[row] = w > 0.f ? a / w : x[row];
}

// ---- the same passes on a copy of P in the order of the values so far
// There a row's entries point near the row, but every gather still pays per cache line that its 64 lanes touch, some forty
// cycles a load and twice what the entries take to arrive.  So a workgroup takes a contiguous share of the rows, with x of
// its rows and of as many rows on either side as its LDS holds, and reads x from there; columns are stored a second time as
// 16-bit places in that window (SMOOTH_OUTSIDE: outside, the 32-bit column says where), so that an entry is 6 bytes.  Sixteen
// lanes a row, every lane's entries in the order of graph_smooth_k and the same operations on them: the same values to the
// bit, whichever of the two takes a pass.  1,281,167 points, 187 M entries: a pass 0.55 -> 0.35 ms (3.3 TB/s).
constexpr int SMOOTH_WINDOW_MAX = 38912, SMOOTH_WINDOW = 20000, SMOOTH_ROWS_MAX = 8192, SMOOTH_THREADS = 1024;
constexpr uint32_t SMOOTH_OUTSIDE = 0xFFFFu;
static_assert(SMOOTH_WINDOW_MAX < (int)SMOOTH_OUTSIDE && SMOOTH_WINDOW_MAX * 4 <= 160 * 1024 - 1024 && SMOOTH_WINDOW * 4 <= 80 * 1024,
              "places are 16 bits, and LDS is 160 KB");

// Rows of a workgroup's share and length of its window; start(row): the first row of the window of the share that holds it.
struct SmoothShape {
    int share, window;
    __device__ __forceinline__ int start(int row) const { return row / share * share - (window - share) / 2; }
};
static SmoothShape smooth_shape(int n, int num_cu, int window)
{
    const int groups = window > SMOOTH_WINDOW ? num_cu : 2 * num_cu, by_cu = (n + groups - 1) / groups;
    return {by_cu < SMOOTH_ROWS_MAX ? by_cu : SMOOTH_ROWS_MAX, window};
}

// The same as smooth_gather from the window in LDS (own: the place of the row itself).
template <int U>
__device__ __forceinline__ void smooth_windowed(const float *win, const uint16_t *place, const int32_t *col, const float *val, const float *x, int n,
                                                int window, int own, int j, int e, int sub, float &a, float &w)
{
    float v[U], xv[U];
    uint32_t c[U];
    bool far = false;
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int i = j + sub + 16 * q;
        v[q] = i < e ? val[i] : 0.f;
        c[q] = i < e ? (uint32_t)place[i] : (uint32_t)own;      // (a place that is filled: 0 times what LDS held before may be no number)
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
        xv[q] = win[min(c[q], (uint32_t)window - 1u)];
        far |= c[q] == SMOOTH_OUTSIDE;
    }
    if (far) {          // (all columns, then all values: one after the other they are 2 U round trips to memory)
        uint32_t at[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            at[q] = 0u;
            if (c[q] == SMOOTH_OUTSIDE) at[q] = (uint32_t)col[j + sub + 16 * q];
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (c[q] == SMOOTH_OUTSIDE) xv[q] = x[min(at[q], (uint32_t)n - 1u)];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
        a = fmaf(v[q], xv[q], a);
        w += v[q];
    }
}

template <int U>
__global__ __launch_bounds__(SMOOTH_THREADS, 8) void graph_smooth_window_k(const int32_t *__restrict__ row_ptr,
                                                                         const uint16_t *__restrict__ place,
                                                                         const int32_t *__restrict__ col,
                                                                         const float *__restrict__ val, const float *__restrict__ x,
                                                                         int n, SmoothShape shape, float *__restrict__ xo,
                                                                         SmoothSeen seen, const uint32_t *__restrict__ reach)
{
    extern __shared__ float win[];
    const int sub = (int)(threadIdx.x % 16);
    if (seen.count && !smooth_by_window(seen)) return;
    const int r0 = (int)blockIdx.x * shape.share, r1 = min(n, r0 + shape.share), base = shape.start(r0);
    // (no entry that has a place lies farther from its row than this)
    const int far = (int)min(*reach, (uint32_t)shape.window), first = max(r0 - base - far, 0), last = min(r1 - base + far, shape.window);
#pragma unroll 8
    for (int i = first + (int)threadIdx.x; i < last; i += SMOOTH_THREADS) win[i] = x[min(max(base + i, 0), n - 1)];
    __syncthreads();
    for (int row = r0 + (int)threadIdx.x / 16; row < r1; row += SMOOTH_THREADS / 16) {
        const int e = row_ptr[row + 1];
        float a = 0.f, w = 0.f;
        for (int j = row_ptr[row]; j < e; j += 16 * U) smooth_windowed<U>(win, place, col, val, x, n, shape.window, row - base, j, e, sub, a, w);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) { a += __shfl_xor(a, o, WAVE); w += __shfl_xor(w, o, WAVE); }
        if (sub == 0) xo[row] = w > 0.f ? a / w : win[row - base];
    }
}

hipError_t graph_smooth_prepare()
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&graph_smooth_window_k<4>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMOOTH_WINDOW_MAX * 4);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&graph_smooth_window_k<10>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               SMOOTH_WINDOW_MAX * 4);
}

// (who: which point x[p] belongs to; null: point p.  Words go to the places of their points, so that the stable sort
// leaves points with equal x in the order of their numbers whatever order they come in.)
__global__ __launch_bounds__(256) void graph_keys_k(const float *__restrict__ x, int n, const uint32_t *__restrict__ who,
                                                    uint64_t *__restrict__ words)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint32_t u = __float_as_uint(x[p]);     // x >= 0: the bit pattern is already ordered
    const uint32_t i = who ? min(who[p], (uint32_t)n - 1u) : (uint32_t)p;
    words[i] = ((uint64_t)u << 32) | i;
}

// Position p of the order of x so far: its point, that point's value and row length, and where the point is now.
__global__ __launch_bounds__(256) void graph_place_k(const uint64_t *__restrict__ words, int n, const int32_t *__restrict__ row_ptr,
                                                     uint32_t *__restrict__ who, uint32_t *__restrict__ place,
                                                     float *__restrict__ x, int32_t *__restrict__ len, uint32_t *__restrict__ seen)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < SEEN_WORDS) seen[p] = 0u;
    if (p >= n) return;
    const uint64_t w = words[p];
    const uint32_t i = min((uint32_t)w, (uint32_t)n - 1u);
    who[p] = i;
    place[i] = (uint32_t)p;
    x[p] = __uint_as_float((uint32_t)(w >> 32));
    len[p] = row_ptr[i + 1] - row_ptr[i];
}

// Entries of every 64th sixteen rows of the copy: outside the window of their row, close to it, all.
constexpr int SMOOTH_SAMPLE = 64;
__global__ __launch_bounds__(256) void graph_sample_k(const uint32_t *__restrict__ who, const uint32_t *__restrict__ place, int n,
                                                      const int32_t *__restrict__ urp, const int32_t *__restrict__ ucol, SmoothShape shape,
                                                      uint32_t *__restrict__ seen)
{
    const int p = (int)blockIdx.x * 16 * SMOOTH_SAMPLE + (int)(threadIdx.x / 16);
    uint32_t outside = 0, close = 0, all = 0;
    if (p < n) {
        const uint32_t u = min(who[p], (uint32_t)n - 1u);
        const int base = shape.start(p), e = urp[u + 1];
#pragma unroll 4
        for (int j = urp[u] + (int)(threadIdx.x % 16); j < e; j += 16) {
            const int c = (int)place[min((uint32_t)ucol[j], (uint32_t)n - 1u)];
            outside += c < base || c - base >= shape.window ? 1u : 0u;
            close += abs(c - p) <= SMOOTH_CLOSE ? 1u : 0u;
            all += 1u;
        }
    }
    outside = wave_sum(outside);
    close = wave_sum(close);
    all = wave_sum(all);
    if (lane_id() == 0) {
        atomicAdd(seen + SEEN_OUTSIDE, outside);
        atomicAdd(seen + SEEN_CLOSE, close);
        atomicAdd(seen + SEEN_ALL, all);
    }
}

// 16 lanes copy the row of the point at position p, columns as positions, entries in the caller's order
__global__ __launch_bounds__(256) void graph_relabel_k(const uint32_t *__restrict__ who, const uint32_t *__restrict__ place, int n,
                                                       const int32_t *__restrict__ urp, const int32_t *__restrict__ ucol,
                                                       const float *__restrict__ uval, const int32_t *__restrict__ rp, SmoothShape shape,
                                                       int32_t *__restrict__ col, uint16_t *__restrict__ in_window,
                                                       float *__restrict__ val, SmoothSeen seen, uint32_t *reach)
{
    const int p = (int)((blockIdx.x * 256u + threadIdx.x) / 16);
    const int sub = (int)(threadIdx.x % 16);
    const bool by_window = seen.count ? smooth_by_window(seen) : in_window != nullptr;
    uint32_t far = 0u;
    if (p < n) {
        const uint32_t u = min(who[p], (uint32_t)n - 1u);
        const int src = urp[u], dst = rp[p], len = rp[p + 1] - dst;
        const int base = shape.start(p);
        for (int e = sub; e < len; e += 16) {
            const int c = (int)place[min((uint32_t)ucol[src + e], (uint32_t)n - 1u)];
            col[dst + e] = c;
            if (by_window) {
                const bool in = c >= base && c - base < shape.window;
                in_window[dst + e] = (uint16_t)(in ? (uint32_t)(c - base) : SMOOTH_OUTSIDE);
                if (in) far = max(far, (uint32_t)abs(c - p));
            }
            val[dst + e] = uval[src + e];
        }
    }
    if (!by_window) return;
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) far = max(far, (uint32_t)__shfl_xor((int)far, o, WAVE));
    // (a look first, which may be late: hardly any wave has to add to the queue at the one address)
    if (lane_id() == 0 && far > __hip_atomic_load(reach, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(reach, far);
}

// In the caller's numbering a pass is bound by its gathers of x: every entry is a cache line of its own (1.35 ms for
// 187 M entries at 1,281,167 points, where reading the entries is 0.3).  Once the values tell the neighbourhoods apart,
// P is copied in the order of the values so far, columns as positions: neighbouring rows then gather the same lines.
// A row's entries keep their order, so every value, and with it the final order, is to the bit what it would be
// without the copies.  They are written where the split copy of P goes afterwards and take no memory of their own.
// Measured for all of set_P and one step, all passes by gathers, at 1,281,167 / 400,000 / 60,000 points in clusters (ms): no copy 96 / - / 4.03;
// one copy after 8 passes 75 / - / 3.48, after 16: 57 / 22.9 / 3.41, after 20: 57 / 22.6 / 3.47, after 24: 58 / 22.0 / 3.42;
// copies after 8 and 20 passes 53 / 22.3 / 3.34, after 10 and 24 52 / 21.2 / 3.24.  A copy costs about three late passes;
// at 20,000 points, where x fits the first-level caches, it gains nothing.  P without a band (512,000 points in four
// blobs) takes as long with copies as without.
constexpr int GRAPH_RELABEL_AFTER[2] = {10, 24};
constexpr int GRAPH_RELABEL_LEFT = 8;        // passes that must still follow a copy
constexpr int GRAPH_RELABEL_MIN = 32768;     // points

// How the passes on a copy go.  Windows pay where rows are long or x is large, wider ones where P reaches farther; a few entries
// outside are enough to lose that where some rows are much longer than others (100,000 points in four blobs, k = 90, with up to
// 5 % instead of 2: 6.2 -> 7.4 ms), and the launch that leaves costs 4 us a pass.  All of set_P and a step, by gathers only / by
// these rules (ms; clusters of 2000 points where nothing else is said):
//   up to 64 entries a row (k = 30): up to SMOOTH_ALL points gathers only (by windows 100,000 2.18 -> 2.47, 140,000 2.74 -> 2.85);
//   beyond, windows of 20,000 values, two workgroups a compute unit, with up to a quarter outside: 400,000 6.5 / 6.3, 1,281,167
//   24.8 / 22.2;
//   longer rows (k = 90): windows of 38,912.  Up to SMOOTH_FEW points whatever is outside, which cannot be much: 60,000 2.85 /
//   2.46, in four blobs 4.37 / 3.39, with all columns random 3.27 / 2.77; up to SMOOTH_ALL with up to 2 % outside: 100,000 3.84 /
//   3.57, in four blobs (gathers) 6.4 / 6.2, in five clusters 5.7 / 4.5, 200,000 7.2 / 6.1, unless most entries are close: 100,000 in
//   clusters of 230 2.61 by gathers, 2.84 by windows; beyond with up to a quarter: 400,000 17.3 / 13.0, in 25 clusters of 20,000
//   500,000 36.0 / 24.8, 1,281,167 52.3 / 42, 512,000 in four blobs (gathers) 44.1 / 38.8.
constexpr int SMOOTH_FEW = 65536, SMOOTH_ALL = 262144;

hipError_t launch_graph_order(tsne_ctx *c, hipStream_t s)
{
    const int n = c->p.n, iters = c->p.graph_order_iters;
    float *xa = (float *)c->Yi, *xb = xa + n;      // Yi (2n floats) is free between steps
    const unsigned pblocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(graph_seed_k, dim3(pblocks), dim3(256), 0, s, xa, n);
    const unsigned blocks = (unsigned)(((int64_t)n * 16 + 255) / 256);
    const int32_t *rp = c->user_row_ptr, *col = c->user_col;
    const float *val = c->user_val;
    const uint32_t *who = nullptr;
    const bool short_rows = c->nnz <= 64 * (int64_t)n, windows = !short_rows || n > SMOOTH_ALL, choose = windows && n > SMOOTH_FEW;
    const SmoothShape shape = smooth_shape(n, c->num_cu, short_rows ? SMOOTH_WINDOW : SMOOTH_WINDOW_MAX);
    // (counts in the sort's totals, free between two sorts)
    const SmoothSeen always = {nullptr, 0u, 0u}, seen = {choose ? c->dtot : nullptr, n <= SMOOTH_ALL ? 2u : 25u, n <= SMOOTH_ALL ? 60u : 100u};
    const int wblocks = (n + shape.share - 1) / shape.share;
    hipError_t e;
    for (int t = 0; t < iters; ++t) {
        if ((t == GRAPH_RELABEL_AFTER[0] || t == GRAPH_RELABEL_AFTER[1]) && iters - t >= GRAPH_RELABEL_LEFT && n >= GRAPH_RELABEL_MIN) {
            hipLaunchKernelGGL(graph_keys_k, dim3(pblocks), dim3(256), 0, s, xa, n, who, c->words[0]);
            if ((e = launch_sort(c, 32, 32, false, s)) != hipSuccess) return e;
            hipLaunchKernelGGL(graph_place_k, dim3(pblocks), dim3(256), 0, s, c->words[c->sorted_buf], n, c->user_row_ptr,
                               c->perm, c->inv, xa, c->len_near, c->dtot);
            launch_scan(c->len_near, n, nullptr, c->rp_near, c->hist, s);
            if (choose)
                hipLaunchKernelGGL(graph_sample_k, dim3((unsigned)((n + 16 * SMOOTH_SAMPLE - 1) / (16 * SMOOTH_SAMPLE))), dim3(256), 0, s,
                                   c->perm, c->inv, n, c->user_row_ptr, c->user_col, shape, c->dtot);
            hipLaunchKernelGGL(graph_relabel_k, dim3(blocks), dim3(256), 0, s, c->perm, c->inv, n, c->user_row_ptr, c->user_col,
                               c->user_val, c->rp_near, shape, c->col_far, windows ? c->col_near : (uint16_t *)nullptr, c->val_s, seen, c->dtot + SEEN_REACH);
            rp = c->rp_near; col = c->col_far; val = c->val_s; who = c->perm;
        }
        if (who && windows)
            hipLaunchKernelGGL(short_rows ? graph_smooth_window_k<4> : graph_smooth_window_k<10>, dim3((unsigned)wblocks), dim3(SMOOTH_THREADS),
                               shape.window * 4, s, rp, c->col_near, col, val, xa, n, shape, xb, seen, c->dtot + SEEN_REACH);
        if (!who || !windows || choose)
            hipLaunchKernelGGL(short_rows ? graph_smooth_k<6> : graph_smooth_k<10>, dim3(blocks), dim3(256), 0, s, rp, col, val, xa, n, xb,
                               who && choose ? seen : always);
        std::swap(xa, xb);
    }
    hipLaunchKernelGGL(graph_keys_k, dim3(pblocks), dim3(256), 0, s, xa, n, who, c->words[0]);
    e = launch_sort(c, 32, 32, false, s);
    return e != hipSuccess ? e : launch_unpack_perm(c, s);
}

// out[orig[s]] = in[s] and its inverse (copies between slot order and the caller's order)
__global__ __launch_bounds__(256) void scatter2_k(const float2 *__restrict__ in, const uint32_t *__restrict__ orig,
                                                  float2 *__restrict__ out, int n)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < n) out[min(orig[s], (uint32_t)n - 1u)] = in[s];
}

__global__ __launch_bounds__(256) void gather2_k(const float2 *__restrict__ in, const uint32_t *__restrict__ orig,
                                                 float2 *__restrict__ out, int n)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < n) out[s] = in[min(orig[s], (uint32_t)n - 1u)];
}

hipError_t launch_scatter2(const float2 *in, const uint32_t *orig, float2 *out, int n, hipStream_t s)
{
    hipLaunchKernelGGL(scatter2_k, dim3((n + 255) / 256), dim3(256), 0, s, in, orig, out, n);
    return hipGetLastError();
}

hipError_t launch_gather2(const float2 *in, const uint32_t *orig, float2 *out, int n, hipStream_t s)
{
    hipLaunchKernelGGL(gather2_k, dim3((n + 255) / 256), dim3(256), 0, s, in, orig, out, n);
    return hipGetLastError();
}
