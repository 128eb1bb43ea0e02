// The carve engine over many images: the batched launch and the step-wise launch of a serving loop.
#include "sc_carver.h"

namespace sc {

// Batched carve: block b is member blk[b].y of team blk[b].x; team t carves the images
// team_imgs[teams[t].x .. teams[t].x + teams[t].y) one after another.
template <int CPL, int KR, int NT>
__global__ __launch_bounds__(NT, 4) void carve_batch_kernel(const Img* __restrict__ imgs, const int2* __restrict__ blk,
                                                         const int2* __restrict__ teams,
                                                         const int* __restrict__ team_imgs) {
    using CV = Carver<CPL, KR, NT>;
    __shared__ typename CV::Smem sm;
    const int2 me = blk[blockIdx.x];
    if (me.x < 0) return;
    const int2 tr = teams[me.x];
    for (int i = 0; i < tr.y; ++i) {
        const CAS Img* gd = (const CAS Img*)(imgs + team_imgs[tr.x + i]);
        CV::carve_image(gd, me.y, gd->G, team_word(gd), sm, 0);
        __syncthreads();
    }
}

// Step-wise carve (serving): each image of the slot table advances by at most max_seams seams and
// reports how many seams it has removed in total (-1 on a device error, -2 for an empty slot).
// Without a plan block b carves slot b alone; with one, block b is member plan[b].y & 0xFFFF of the team
// of plan[b].y >> 16 workgroups that carves slot plan[b].x (-1: no work), the members of a team on one
// XCD, 8 blocks apart.  The plan comes anew with every step, and with it, in the second half of the
// entry of a team's member 0, the word by which the team forms.
// The table is a device array of descriptors written by slot_write_kernel.
template <int CPL, int KR, int NT>
__global__ __launch_bounds__(NT, 4) void carve_steps_kernel(const Img* __restrict__ table, int n, int max_seams,
                                                            unsigned long long budget_ticks,
                                                            int* __restrict__ progress, int4* plan) {
    using CV = Carver<CPL, KR, NT>;
    __shared__ typename CV::Smem sm;
    int slot = (int)blockIdx.x, rank = 0, G = 1;
    GAS unsigned long long* join = nullptr;
    if (plan) {
        slot = __builtin_amdgcn_readfirstlane(plan[blockIdx.x].x);
        const int place = __builtin_amdgcn_readfirstlane(plan[blockIdx.x].y);
        rank = place & 0xFFFF;
        G = place >> 16;
        join = gp(reinterpret_cast<unsigned long long*>(plan + blockIdx.x - 8 * rank) + 1);
    }
    if (slot < 0 || slot >= n) return;
    const CAS Img* gd = (const CAS Img*)(table + slot);
    if (gd->H == 0) {
        if (rank == 0 && threadIdx.x == 0 && progress) progress[slot] = -2;
        return;
    }
    // a time budget (device wall clock ticks) ends the image's share after the seam that crosses
    // it, so a step's workgroups stay busy for about the same time
    CV::carve_image(gd, rank, G, join, sm, max_seams, budget_ticks ? wall_clock64() + budget_ticks : 0ull);
    __syncthreads();
    if (CV::first_member(sm, G) && progress) {
        const GAS Ctl* ctl = gp(reinterpret_cast<const Ctl*>(gd->bar));
        progress[slot] = (ctl->status & (kStatusTimeout | kStatusPlacement)) ? -1 : (int)ctl->done;
    }
}

hipError_t launch_carve_batch(const Img* imgs, const int2* blk, const int2* teams, const int* ti, int nb, int v,
                              hipStream_t st) {
    switch (v) {
#define X(id, c, k, t) \
    case id: hipLaunchKernelGGL((carve_batch_kernel<c, k, t>), dim3(nb), dim3(t), 0, st, imgs, blk, teams, ti); break;
        SC_VARIANTS(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_carve_steps(const Img* table, int n, int v, int max_seams, unsigned long long budget_ticks,
                              int* progress, const int4* plan, int nblocks, hipStream_t st) {
    const int nb = plan ? nblocks : n;
    switch (v) {
#define X(id, c, k, t)                                                                                        \
    case id:                                                                                                  \
        hipLaunchKernelGGL((carve_steps_kernel<c, k, t>), dim3(nb), dim3(t), 0, st, table, n, max_seams, budget_ticks, \
                           progress, const_cast<int4*>(plan));                                                                        \
        break;
        SC_VARIANTS(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int carve_blocks_per_cu(int v) {
    int nb = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (v) {
#define X(id, c, k, t) \
    case id: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, carve_batch_kernel<c, k, t>, t, 0); break;
        SC_VARIANTS(X)
#undef X
        default: break;
    }
    return e == hipSuccess ? nb : 0;
}

}  // namespace sc
