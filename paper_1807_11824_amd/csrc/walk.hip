// Sec. III-C step 5: the walk as resident waves or a wave a group (the walk itself is in walk_group.h), and Z.
#include "walk_group.h"

// One wave per workgroup.  With a work counter the grid is a fixed number of resident waves that
// take groups from the counter until none is left (every wave ends when the counter has passed
// the number of groups); without one, workgroup g walks group g.
__global__ __attribute__((amdgpu_waves_per_eu(5))) __launch_bounds__(WAVE) void bh_walk(const Cell *__restrict__ cells, const float2 *__restrict__ Ys,
                                                const uint32_t *__restrict__ perm, int n,
                                                const float4 *__restrict__ root, float theta2,
                                                const uint32_t *__restrict__ ncells, uint32_t cap_cells,
                                                float2 *__restrict__ R, double *__restrict__ zpart,
                                                uint32_t *status, uint32_t *counter)
{
    __shared__ uint32_t stack[WALK_STACK];
    __shared__ uint32_t pend[WALK_PEND];
    __shared__ float2 pts[WAVE];
    __shared__ float4 clist[WALK_CLIST];
    __shared__ float2 plist[WALK_PLIST];
    const int ngroups = (n + WAVE - 1) / WAVE;
    if (!counter) {
        walk_group((int)blockIdx.x, stack, pend, pts, clist, plist, cells, Ys, perm, n, root, theta2, ncells, cap_cells, R,
                   zpart, status);
        return;
    }
    // The first group of a wave is its workgroup number; further groups come from counters.
    // (All waves start together: if each began with a draw, thousands of atomics on one address
    // would queue up and the last wave would start tens of microseconds late.)  Same-address
    // atomics are served one after the other, about one every 20 ns, which 20 000 draws in a
    // third of a millisecond would saturate: the groups are dealt into WALK_COUNTERS classes
    // (group mod WALK_COUNTERS), each with its own counter and its own share of the waves.
    // The grid is a multiple of WALK_COUNTERS, so every class has grid / WALK_COUNTERS waves.
    __shared__ uint32_t next_group;
    const uint32_t cls = blockIdx.x % WALK_COUNTERS, dealt = gridDim.x / WALK_COUNTERS;
    uint32_t g = blockIdx.x;
    while (g < (uint32_t)ngroups) {
        walk_group((int)g, stack, pend, pts, clist, plist, cells, Ys, perm, n, root, theta2, ncells, cap_cells, R, zpart,
                   status);
        // lane 0 draws the next group of the class; every lane reads the number back from LDS
        __syncthreads();
        if (threadIdx.x == 0) next_group = cls + WALK_COUNTERS * (dealt + atomicAdd(counter + cls, 1u));
        __syncthreads();
        g = (uint32_t)__builtin_amdgcn_readfirstlane((int)next_group);
    }
}

// Z = sum of the per-group partial sums, in a fixed order (thread t takes groups t, t + 1024, ...,
// eight running sums so that eight loads are in flight, combined pairwise).
__global__ __launch_bounds__(1024) void z_final(const double *__restrict__ zpart, int ngroups, double *__restrict__ Z)
{
    __shared__ double ws[16];
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i = (int)threadIdx.x; i < ngroups; i += 8 * 1024) {
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += i + 1024 * k < ngroups ? zpart[i + 1024 * k] : 0.0;
    }
    double a = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    a = wave_sum(a);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < 16; ++k) t += ws[k];
        *Z = t;
    }
}

// Few points: an iteration is bound by the number of calls the host makes for it (5 us each) and by the chain of its
// launches, and the walk, a wave a group, leaves most of the chip idle.  The attraction then takes part in the walk's
// launch, on one stream: two launches, three events and three waits less.  500 points 67 -> 46 us an iteration, 2000 71 ->
// 59, 8192 105 -> 89, 30,011 131 -> 112, 60,000 136 -> 120; 100,000 153 -> 164: there the walk fills the chip, and the
// gathers of the rows, which on a stream of their own start beside the tree build, come on top.
constexpr int WALK_ROWS_MAX = 65536;

bool walk_takes_attraction(const tsne_ctx *c)
{
    return c->p.n <= WALK_ROWS_MAX && !(c->ft_active && c->reorder_on && !c->identity);
}

hipError_t launch_walk(tsne_ctx *c, hipStream_t s, bool attraction, bool sum_z)
{
    const int n = c->p.n;
    const int ngroups = (n + WAVE - 1) / WAVE;
    const float theta2 = c->p.theta * c->p.theta;
    if (attraction) {
        const hipError_t e = launch_walk_rows(c, s);
        if (e != hipSuccess) return e;
    } else {
        // walk_resident > 0: that many resident waves per compute unit share the groups through a
        // counter (zeroed by the tree build), which leaves a known part of every unit to the attraction
        const bool resident = c->p.walk_resident > 0 && ngroups > c->p.walk_resident * c->num_cu &&
                              c->p.walk_resident * c->num_cu >= WALK_COUNTERS;
        const int grid = resident ? c->p.walk_resident * c->num_cu / WALK_COUNTERS * WALK_COUNTERS : ngroups;
        hipLaunchKernelGGL(bh_walk, dim3(grid), dim3(WAVE), 0, s, c->cells, c->Ys, c->perm, n, c->root,
                           theta2, c->ncells, (uint32_t)c->cap_cells, c->R, c->zpart, c->status,
                           resident ? c->walk_counter : (uint32_t *)nullptr);
    }
    if (sum_z) hipLaunchKernelGGL(z_final, dim3(1), dim3(1024), 0, s, c->zpart, ngroups, c->Z);
    return hipGetLastError();
}
