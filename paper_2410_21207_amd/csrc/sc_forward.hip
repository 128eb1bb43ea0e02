// Forward-energy carve (sec. "Forward Energy Calculation", the standard definition with no per-pixel
// term; readings R17-R19): the DP cost of a pixel is the difference of the pixel pairs its removal
// makes neighbours, CU = D(left, right), plus D(up, left) for the upper-left parent or D(up, right)
// for the upper-right one, D = the channel sum of absolute differences, neighbour indices clamped to
// the row.  The costs come from the current pixels, so there is no energy plane and no band update.
//
// The working copy keeps one dword per pixel (channels in the low C bytes, zeros above), so D is one
// v_sad_u8.  The carve engine sweeps it as it sweeps energies, from both ends of the image: the row
// formula read upward is the same one, an edge's cost depends on its two pixels alone, and the two
// middle rows are joined with the cost of the edge between them.  The tie rules hold as they do there:
// of two paths that cross, the uncrossed pair runs straight down, which costs nothing more.
//
// What bounds it: the chain of rows, 22 instructions for 256 columns (three v_sad_u8 and a v_min3
// per column, six wave shifts and moves).  A sweep with directions from the top alone, its teams
// exchanging keys every 112 rows, took 202 us per seam of 1920 x 1080 by 32 workgroups and takes 66 us so;
// 64 images up to 2000 x 2000 went from 247 to 73 ms.
#include "sc_carver.h"

namespace sc {

using FwdCarver = Carver<4, kFwdKR, kFwdThreads, kForward>;

// Batched forward carve: block b is member blk[b].y of the team of image blk[b].x (-1: no work).
// Single image: the team's members are blocks xcd, xcd + 8, ... (the others exit at once).
__global__ __launch_bounds__(kFwdThreads, 4) void fwt_carve_kernel(const Img* __restrict__ imgs,
                                                                   const int2* __restrict__ blk, int xcd) {
    __shared__ FwdCarver::Smem sm;
    int2 me;
    if (blk) {
        me = blk[blockIdx.x];
    } else {
        if ((int)(blockIdx.x & 7) != xcd) return;
        me = make_int2(0, (int)(blockIdx.x >> 3));
    }
    if (me.x < 0) return;
    const CAS Img* pd = (const CAS Img*)(imgs + me.x);
    if (me.y >= pd->G) return;
    FwdCarver::carve_image(pd, me.y, pd->G, team_word(pd), sm, 0);
}

// Copy-in for the forward carve: every pixel of src (or img) as one dword of wk (channels in the
// low bytes), control words reset, rows started, published keys and seam words cleared of tags, the
// row of zeros below the last one, and src copied to img when nothing is carved.  Grid: (workgroups per image, images).
template <int C>
__device__ void fwt_prepare_rows(const Img& d, const uint8_t* srcimg, int row0, int rstep) {
    const int W = d.W;
    const bool identity = d.src && d.target_w == d.W;
    for (int y = row0; y < d.H; y += rstep) {
        uint32_t* wr = reinterpret_cast<uint32_t*>(d.wk + (long long)y * d.wp);
        for (int x0 = 4 * (int)threadIdx.x; x0 < W; x0 += 4 * (int)blockDim.x) {
            SrcRow<C> r;
            r.load(srcimg, d.pitch, W, y, x0);
            if (x0 + 3 < W) {
                *gp(reinterpret_cast<v4u*>(wr + x0)) = v4u{r.px(0), r.px(1), r.px(2), r.px(3)};
            } else {
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (x0 + p < W) *gp(wr + x0 + p) = r.px(p);
            }
            if (identity) {
                uint8_t* o = d.img + (long long)y * d.pitch + (long long)x0 * C;
#pragma unroll
                for (int b = 0; b < 4 * C; ++b)
                    if (x0 * C + b < W * C) *gp(o + b) = (uint8_t)(r.r[1 + (b >> 2)] >> (8 * (b & 3)));
            }
        }
    }
}

__global__ __launch_bounds__(256) void fwt_prepare_kernel(const Img* __restrict__ imgs, int n) {
    const int i = blockIdx.y;
    if (i >= n) return;
    const Img d = imgs[i];
    const int t = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
    if (t == 0) reset_ctl(d);
    for (int x = t; x < d.H; x += nt) *gp(d.ro + x) = *gp(d.seam + x) = 0;
    for (int x = t; x < d.P * d.xw; x += nt) *gp(d.xq + x) = 0u;
    for (int x = t; x < d.wp / 4; x += nt) *gp(reinterpret_cast<uint32_t*>(d.wk + (long long)d.H * d.wp) + x) = 0u;
    const uint8_t* srcimg = d.src ? d.src : d.img;
    switch (d.C) {
        case 1: fwt_prepare_rows<1>(d, srcimg, blockIdx.x, gridDim.x); break;
        case 2: fwt_prepare_rows<2>(d, srcimg, blockIdx.x, gridDim.x); break;
        case 3: fwt_prepare_rows<3>(d, srcimg, blockIdx.x, gridDim.x); break;
        default: fwt_prepare_rows<4>(d, srcimg, blockIdx.x, gridDim.x); break;
    }
}

hipError_t launch_fwt_prepare(const Img* imgs, int n, int max_rows, hipStream_t st) {
    const int per = max_rows < 256 ? max_rows : 256;
    hipLaunchKernelGGL(fwt_prepare_kernel, dim3(per, n), dim3(256), 0, st, imgs, n);
    return hipGetLastError();
}

hipError_t launch_fwt_carve(const Img* imgs, const int2* blk, int nblocks, int xcd, hipStream_t st) {
    hipLaunchKernelGGL(fwt_carve_kernel, dim3(nblocks), dim3(kFwdThreads), 0, st, imgs, blk, xcd & 7);
    return hipGetLastError();
}

int fwt_blocks_per_cu() {
    int nb = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fwt_carve_kernel, kFwdThreads, 0) == hipSuccess ? nb : 0;
}

}  // namespace sc
