// The walk of few points, a wave a group, with the rows of the attraction in the same launch.  (A file of its own: beside a
// second kernel with the same walk the compiler gives bh_walk other registers, and an iteration of 1,281,167 points 1 % more.)
#include "walk_group.h"

// Attraction of one row (Eq. (5)) by sixteen lanes, y_j gathered from the caches, where all of Y is when there are few
// points.  From the caller's P, or from the renumbered copy, whose near columns say by how much they differ from the row
// (modulo the length of the ring they index).  The operations and their order are those of attract_csr, or of
// attract_far and attract_near (a near chunk is four lanes' work, eight entries each), so the sums are the same to the bit.
__device__ __forceinline__ void attract_row(const AttractRows &P, const int row, const int n, const int sub)
{
    const bool live = row < n;
    const float2 yi = P.Y[live ? row : 0];
    auto add = [&](float2 yj, float p, float &ax, float &ay) {
        const float dx = yi.x - yj.x, dy = yi.y - yj.y;
        const float w = __builtin_amdgcn_rcpf(fmaf(dy, dy, fmaf(dx, dx, 1.0f)));
        const float pw = p * w;
        ax = fmaf(pw, dx, ax);
        ay = fmaf(pw, dy, ay);
    };
    const int first = P.rp_near ? P.rp[0] : 0;       // (far values sit behind the near ones, far columns start at 0)
    const int begin = live ? P.rp[row] : 0, end = live ? P.rp[row + 1] : 0;
    float fx = 0.f, fy = 0.f;
    for (int j0 = begin + sub; j0 < end; j0 += 64) {
        int c[4];
        float v[4];
        float2 yj[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = j0 + 16 * q;
            const bool in = j < end;
            c[q] = in ? P.col[j - first] : row;      // padding: own point, weight 0
            v[q] = in ? P.val[j] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) yj[q] = P.Y[min((uint32_t)c[q], (uint32_t)n - 1u)];
#pragma unroll
        for (int q = 0; q < 4; ++q) add(yj[q], v[q], fx, fy);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        fx += __shfl_xor(fx, o, WAVE);
        fy += __shfl_xor(fy, o, WAVE);
    }
    if (P.rp_near) {
        float ax = 0.f, ay = 0.f;
        if (live && sub < 4)
            for (int j = P.rp_near[row] + 8 * sub; j < P.rp_near[row + 1]; j += ATTRACT_CHUNK) {
                const uint4 c = *reinterpret_cast<const uint4 *>(P.col_near + j);
                const float4 v0 = *reinterpret_cast<const float4 *>(P.val + j), v1 = *reinterpret_cast<const float4 *>(P.val + j + 4);
                const uint32_t o[8] = {c.x & 0xFFFFu, c.x >> 16, c.y & 0xFFFFu, c.y >> 16, c.z & 0xFFFFu, c.z >> 16, c.w & 0xFFFFu, c.w >> 16};
                const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
                float2 yj[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    int d = (int)(o[q] >> 3) - row % ATTRACT_RING;
                    d += d > ATTRACT_RING / 2 ? -ATTRACT_RING : d < -ATTRACT_RING / 2 ? ATTRACT_RING : 0;
                    yj[q] = P.Y[min(max(row + d, 0), n - 1)];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) add(yj[q], v[q], ax, ay);
            }
        ax = sum4(ax);
        ay = sum4(ay);
        if (end > begin) { ax += fx; ay += fy; }
        fx = ax;
        fy = ay;
    }
    if (live && sub == 0) P.A[row] = make_float2(fx, fy);
}

// A workgroup a group without a counter, and behind the last group workgroups that take four rows of the attraction each.
__global__ __attribute__((amdgpu_waves_per_eu(5))) __launch_bounds__(WAVE) void bh_walk_rows(const Cell *__restrict__ cells, const float2 *__restrict__ Ys,
                                                const uint32_t *__restrict__ perm, int n,
                                                const float4 *__restrict__ root, float theta2,
                                                const uint32_t *__restrict__ ncells, uint32_t cap_cells,
                                                float2 *__restrict__ R, double *__restrict__ zpart,
                                                uint32_t *status, AttractRows rows)
{
    const int ngroups = (n + WAVE - 1) / WAVE;
    if ((int)blockIdx.x >= ngroups) {
        attract_row(rows, ((int)blockIdx.x - ngroups) * (WAVE / 16) + (int)threadIdx.x / 16, n, (int)threadIdx.x % 16);
        return;
    }
    __shared__ uint32_t stack[WALK_STACK];
    __shared__ uint32_t pend[WALK_PEND];
    __shared__ float2 pts[WAVE];
    __shared__ float4 clist[WALK_CLIST];
    __shared__ float2 plist[WALK_PLIST];
    walk_group((int)blockIdx.x, stack, pend, pts, clist, plist, cells, Ys, perm, n, root, theta2, ncells, cap_cells, R, zpart, status);
}

hipError_t launch_walk_rows(tsne_ctx *c, hipStream_t s)
{
    const int n = c->p.n, ngroups = (n + WAVE - 1) / WAVE;
    const bool split = c->reorder_on && !c->identity;
    AttractRows rows;
    rows.rp = split ? c->rp_far : c->user_row_ptr;
    rows.col = split ? c->col_far : c->user_col;
    rows.val = split ? c->val_s : c->user_val;
    rows.rp_near = split ? c->rp_near : nullptr;
    rows.col_near = c->col_near;
    rows.Y = c->Yi;
    rows.A = c->A;
    hipLaunchKernelGGL(bh_walk_rows, dim3(ngroups + (n + WAVE / 16 - 1) / (WAVE / 16)), dim3(WAVE), 0, s, c->cells, c->Ys,
                       c->perm, n, c->root, c->p.theta * c->p.theta, c->ncells, (uint32_t)c->cap_cells, c->R, c->zpart, c->status, rows);
    return hipGetLastError();
}
