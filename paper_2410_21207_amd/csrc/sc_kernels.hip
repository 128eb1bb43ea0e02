// HIP kernels of the seam-carving hot path for gfx950 (CDNA4): the energy passes, single-step calls,
// the carve of one image, seam insertion and the allocation-free carve's scratch.  The carve
// engine is in sc_carver.h, its batched and step-wise kernels in sc_batch.hip.
#include <mutex>

#include "sc_carver.h"

namespace sc {

// Standalone energy map (int32, dense): a thread takes 4 pixels of kEnergyRows rows from whole dwords
// (SrcRow) and keeps the rows above and below in registers.  What bounds it: its loads' latency.  (A
// byte load per channel and neighbour: 8 passes of energy, seam and removal at 1920 x 1080 took 886 us
// with it and take 846 us so.)
constexpr int kEnergyRows = 4;
template <int C>
__device__ void energy_rows(const uint8_t* img, int H, int W, long long pitch, int32_t* out, int y0, int x0) {
    typedef uint32_t v4u_row __attribute__((ext_vector_type(4), aligned(4)));  // a row starts at any dword
    SrcRow<C> row[kEnergyRows + 2];
#pragma unroll
    for (int i = 0; i < kEnergyRows + 2; ++i) row[i].load(img, pitch, W, min(max(y0 + i - 1, 0), H - 1), x0);
    if (x0 >= W) return;
#pragma unroll
    for (int i = 0; i < kEnergyRows; ++i) {
        if (y0 + i >= H) break;
        const SrcRow<C>&up = row[i], &cur = row[i + 1], &dn = row[i + 2];
        uint32_t e[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t l = x0 + p > 0 ? cur.px(p - 1) : cur.px(p);
            const uint32_t r = x0 + p + 1 < W ? cur.px(p + 1) : cur.px(p);
            e[p] = __builtin_amdgcn_sad_u8(up.px(p), dn.px(p), __builtin_amdgcn_sad_u8(l, r, 0u));
        }
        int32_t* o = out + (long long)(y0 + i) * W + x0;
        if (x0 + 3 < W) {
            *gp(reinterpret_cast<v4u_row*>(o)) = v4u_row{e[0], e[1], e[2], e[3]};
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if (x0 + p < W) *gp(o + p) = (int32_t)e[p];
        }
    }
}

__global__ __launch_bounds__(256) void energy_i32_kernel(const uint8_t* __restrict__ img, int H, int W, int C,
                                                         long long pitch, int32_t* __restrict__ out) {
    const int y0 = blockIdx.y * kEnergyRows, x0 = 4 * (int)(blockIdx.x * blockDim.x + threadIdx.x);
    switch (C) {
        case 1: energy_rows<1>(img, H, W, pitch, out, y0, x0); break;
        case 2: energy_rows<2>(img, H, W, pitch, out, y0, x0); break;
        case 3: energy_rows<3>(img, H, W, pitch, out, y0, x0); break;
        default: energy_rows<4>(img, H, W, pitch, out, y0, x0); break;
    }
}

// A single-image workspace starts with a header: magic, image count, then the descriptor itself
// (read by the step-wise carve kernel), then the image's Ctl block.
__device__ __forceinline__ void write_single_header(const Img& d) {
    char* h = reinterpret_cast<char*>(d.bar) - kWsHeadBytes;
    reinterpret_cast<uint32_t*>(h)[0] = kWsMagic;
    reinterpret_cast<uint32_t*>(h)[1] = 1u;
    *reinterpret_cast<Img*>(h + kWsImgOffset) = d;
}

// Per-image preparation: reset the control words, optionally copy src -> img, fill the energy plane,
// and zero the rows of published keys (row y of the d.P rows of ck, which are never more than the
// image's rows): a published key carries its seam's tag (never 0), so nothing a previous launch left
// there can pass for a key of this one.

// The energy pass (a1) and the copy into the working image.  The carve works on the copy in wk;
// img receives the result at the end (a carve that removes nothing copies src into img here).
//
// A workgroup sweeps one tile: a strip of 1024 columns (4 per thread) down kTileRows rows.  Each
// source row is read once per tile, as the aligned dwords covering the thread's 4 pixels and one
// pixel on each side, realigned to the row start with v_alignbyte (rows may start anywhere); the
// rows above and below stay in registers as the tile moves down.  The energy goes out as one
// 8-byte store of 4 uint16 per thread, the pixels as C dword stores into the rows of
// wk, which start at multiples of 16 bytes.
constexpr int kTileRows = 32;
constexpr int kTileCols = 1024;  // 256 threads x 4 pixels

template <int C>
__device__ void prepare_tile(const Img& d, const uint8_t* srcimg, int y0, int y1, int xs) {
    const int t = threadIdx.x, x0 = xs + 4 * t, H = d.H, W = d.W;
    const bool act = x0 < W;
    const bool identity = d.src && d.target_w == d.W;
    SrcRow<C> up, cur, dn;
    up.load(srcimg, d.pitch, W, max(y0 - 1, 0), x0);
    cur.load(srcimg, d.pitch, W, y0, x0);
    dn.load(srcimg, d.pitch, W, min(y0 + 1, H - 1), x0);
#pragma unroll 1
    for (int y = y0; y < y1; ++y) {
        SrcRow<C> nx;
        if (y + 1 < y1) nx.load(srcimg, d.pitch, W, min(y + 2, H - 1), x0);
        if (act) {
            if (d.e) {
                if (y == H - 1) *gp(reinterpret_cast<v2u*>(d.e + (long long)H * d.ep + x0)) = v2u{0u, 0u};  // row of zeros
                uint32_t e[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int x = x0 + p;
                    const uint32_t l = x > 0 ? cur.px(p - 1) : cur.px(p);
                    const uint32_t rr = x + 1 < W ? cur.px(p + 1) : cur.px(p);
                    e[p] = __builtin_amdgcn_sad_u8(up.px(p), dn.px(p), __builtin_amdgcn_sad_u8(l, rr, 0u));
                }
                uint16_t* er = d.e + (long long)y * d.ep + x0;
                if (x0 + 3 < W) {
                    *gp(reinterpret_cast<v2u*>(er)) = v2u{e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
                } else {
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        if (x0 + p < W) *gp(er + p) = (uint16_t)e[p];
                }
            }
            if (y < d.P) *gp(reinterpret_cast<v4u*>(d.xq + (size_t)y * d.xw + x0)) = v4u{0u, 0u, 0u, 0u};
            uint32_t* wr = reinterpret_cast<uint32_t*>(d.wk + (long long)y * d.wp + (long long)x0 * C);
#pragma unroll
            for (int m = 0; m < C; ++m)
                if (x0 * C + 4 * m < W * C) *gp(wr + m) = cur.r[m + 1];
            if (identity) {
                uint8_t* o = d.img + (long long)y * d.pitch + (long long)x0 * C;
#pragma unroll
                for (int b = 0; b < 4 * C; ++b)
                    if (x0 * C + b < W * C) *gp(o + b) = (uint8_t)(cur.r[1 + (b >> 2)] >> (8 * (b & 3)));
            }
        }
        up = cur;
        cur = dn;
        dn = nx;
    }
}

// Tiles tile0, tile0 + tstep, ... of one image (tiles numbered strip-major within row chunks);
// tile 0 also resets the control words.
__device__ void prepare_image(const Img& d, int tile0, int tstep) {
    const uint8_t* srcimg = d.src ? d.src : d.img;
    if (tile0 == 0 && threadIdx.x == 0) reset_ctl(d);
    const int ns = (d.W + kTileCols - 1) / kTileCols, nc = (d.H + kTileRows - 1) / kTileRows;
    for (int tile = tile0; tile < ns * nc; tile += tstep) {
        const int strip = tile % ns, chunk = tile / ns;
        const int y0 = chunk * kTileRows, y1 = min(d.H, y0 + kTileRows);
        if (strip == 0 && (int)threadIdx.x < y1 - y0) {
            *gp(d.ro + y0 + threadIdx.x) = 0;
            *gp(d.seam + y0 + threadIdx.x) = 0;  // no seam's tag
        }
        switch (d.C) {
            case 1: prepare_tile<1>(d, srcimg, y0, y1, strip * kTileCols); break;
            case 2: prepare_tile<2>(d, srcimg, y0, y1, strip * kTileCols); break;
            case 3: prepare_tile<3>(d, srcimg, y0, y1, strip * kTileCols); break;
            default: prepare_tile<4>(d, srcimg, y0, y1, strip * kTileCols); break;
        }
    }
}

__global__ __launch_bounds__(256) void prepare_single_kernel(Img d) {
    if (blockIdx.x == 0 && threadIdx.x == 0) write_single_header(d);
    prepare_image(d, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void prepare_batch_kernel(const Img* __restrict__ imgs, int n) {
    const int i = blockIdx.y;
    if (i < n) {
        const Img d = imgs[i];
        prepare_image(d, blockIdx.x, gridDim.x);
    }
}

// Energy plane from a caller's int32 energy map (sc_dp_seam).
__global__ void prepare_from_i32_kernel(Img d, const int32_t* __restrict__ e) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        write_single_header(d);
        reset_ctl(d);
    }
    const int y = blockIdx.y;
    if (blockIdx.x == 0 && threadIdx.x == 0) *gp(d.ro + y) = 0;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < d.W; x += gridDim.x * blockDim.x) {
        *gp(d.e + (long long)y * d.ep + x) = (uint16_t)*gp(e + (long long)y * d.W + x);
        if (y < d.P) *gp(d.xq + (size_t)y * d.xw + x) = 0u;
        if (y == d.H - 1) *gp(d.e + (long long)d.H * d.ep + x) = 0;  // the plane's row of zeros
    }
}

// ----------------------------------------------------------------------------------------------
// In-place left shift of a row segment by one pixel, one wave: the bytes of [lo, hi) take the values sh
// (1..4) bytes to their right.  The work is cut into 16-byte slots aligned to absolute addresses; a pass
// gives each lane U slots and issues every load of the pass before any store.  A slot's store writes
// only inside the slot, and the bytes it needs beyond its end belong to the next slot, loaded in the
// same pass or a later one, so the in-place update is hazard free.
template <int U>
__device__ __forceinline__ void shift_segment_wave(uint8_t* lo_p, uint8_t* hi_p, int sh, int lane) {
    const int lo = (int)((uintptr_t)lo_p & 15);
    uint8_t* const base = lo_p - lo;  // 16-byte aligned (wave-uniform)
    const int hi = hi_p > lo_p ? lo + (int)(hi_p - lo_p) : lo;
    const int n = hi > lo ? ((hi - 1) >> 4) + 1 : 0;  // slots covering the segment
#pragma unroll 1
    for (int fb = 0; fb < n; fb += 64 * U) {
        uint32_t D[U][5];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = fb + u * 64 + lane;
#pragma unroll
            for (int i = 0; i < 5; ++i) D[u][i] = 0;
            if (f < n) {
                const uint32_t so = (uint32_t)f << 4;  // slot offset from the uniform base
                const uint64_t* q = reinterpret_cast<const uint64_t*>(base + so);
                const uint64_t v0 = *gp(q), v1 = *gp(q + 1);
                D[u][0] = (uint32_t)v0; D[u][1] = (uint32_t)(v0 >> 32);
                D[u][2] = (uint32_t)v1; D[u][3] = (uint32_t)(v1 >> 32);
                if ((int)so + 16 - sh < hi) D[u][4] = *gp(reinterpret_cast<const uint32_t*>(base + so + 16));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = fb + u * 64 + lane;
            if (f >= n) continue;
            const int so = f << 4;
            uint8_t* sp = base + so;
            uint32_t o[4];
            if (sh == 4) {
                o[0] = D[u][1]; o[1] = D[u][2]; o[2] = D[u][3]; o[3] = D[u][4];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_alignbyte(D[u][i + 1], D[u][i], (uint32_t)sh);
            }
            if (so >= lo && so + 16 <= hi) {
                *gp(reinterpret_cast<u32x4*>(sp)) = u32x4{o[0], o[1], o[2], o[3]};
            } else {
                // a slot at the segment's edge: store only the bytes inside the segment, one predicated
                // byte store per position (static offsets and register indices)
                const int k0 = so > lo ? 0 : lo - so;
                const int k1 = so + 16 < hi ? 16 : hi - so;
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (k >= k0 && k < k1) *gp(sp + k) = (uint8_t)(o[k >> 2] >> ((k & 3) * 8));
            }
        }
    }
}

// Standalone seam removal: one wave per row.
__global__ void remove_seam_kernel(uint8_t* __restrict__ img, int H, int W, int C, long long pitch,
                                   const int32_t* __restrict__ seam) {
    const int lane = threadIdx.x & 63;
    const int wv = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nw = (gridDim.x * blockDim.x) >> 6;
    for (int y = wv; y < H; y += nw) {
        const int s = *gp(seam + y);
        if (s < 0 || s >= W) continue;
        uint8_t* row = img + (long long)y * pitch;
        shift_segment_wave<4>(row + (long long)s * C, row + (long long)(W - 1) * C, C, lane);
    }
}

// ----------------------------------------------------------------------------------------------
// Transpose J(x,y,c) = I(y,x,c) through a 64x64-pixel LDS tile.
template <int C>
__global__ void transpose_kernel(const uint8_t* __restrict__ src, int H, int W, long long sp,
                                 uint8_t* __restrict__ dst, long long dp) {
    __shared__ uint8_t tile[64][64 * C + 4];
    const int bx = blockIdx.x * 64, by = blockIdx.y * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 256 threads: 4 rows per pass
    for (int r = ty; r < 64; r += 4) {
        const int y = by + r, x = bx + tx;
        if (y < H && x < W)
            for (int c = 0; c < C; ++c) tile[r][tx * C + c] = *gp(src + (long long)y * sp + (long long)x * C + c);
    }
    __syncthreads();
    for (int r = ty; r < 64; r += 4) {
        const int x = bx + r, y = by + tx;  // output row x, column y
        if (y < H && x < W)
            for (int c = 0; c < C; ++c) *gp(dst + (long long)x * dp + (long long)y * C + c) = tile[tx][r * C + c];
    }
}

template <int CPL, int KR, int NT>
__global__ __launch_bounds__(NT, 4) void carve_single_kernel(Img d, int xcd) {
    using CV = Carver<CPL, KR, NT>;
    __shared__ typename CV::Smem sm;
    // Team members are blocks xcd, xcd + 8, xcd + 16, ...: workgroups are dispatched to the 8 XCDs
    // round-robin by block index, so they share XCD `xcd`'s L2; the other blocks exit at once.
    if ((int)(blockIdx.x & 7) != xcd) return;
    const CAS Img* gd = (const CAS Img*)__builtin_amdgcn_kernarg_segment_ptr();  // d, the first argument
    CV::template carve_image<true>(gd, blockIdx.x >> 3, d.G, team_word(gd), sm, 0);
}

// Slot management: write (or clear) one descriptor of the slot table.
__global__ void slot_write_kernel(Img* table, int slot, Img d) { table[slot] = d; }

// ----------------------------------------------------------------------------------------------
// Seam insertion (image enlargement).
//
// Original columns of seams recorded during removal.  Seam j's column x is one of the row without
// seams 0 .. j-1; putting them back, last first, moves it by one wherever x is not left of seam i:
// x += (x >= s_i).  One wave per row, seam 64 b + l in lane l: a block's 64 columns are read once and
// handed out by v_readlane, so a pair of seams costs three instructions for 64 lanes.
// What bounds it: those instructions, k * k / 128 triples per row.  (A Fenwick tree per row, a thread
// each, waits for 2 log W memory accesses one behind the other for every seam: 0.76 ms for 201 seams of
// 1080 rows, and 1920 x 1080 widened by 480 took 26.5 ms with it and takes 25.0 ms so.)
__global__ __launch_bounds__(256) void seam_origins_kernel(const int32_t* __restrict__ seams, int k, int H, int W,
                                                           int32_t* __restrict__ orig) {
    const int lane = threadIdx.x & 63;
    const int r = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    if (r >= H) return;
    auto column = [&](int b) {
        const int j = 64 * b + lane;
        return j < k ? min(max(*gp(seams + (size_t)j * H + r), 0), W - 1 - j) : 0;
    };
    for (int b = 0; 64 * b < k; ++b) {
        int y = column(b), x = y;
        static_for<63>([&](auto I) {
            constexpr int i = 62 - decltype(I)::value;
            x += lane > i && x >= __builtin_amdgcn_readlane(y, i);
        });
        y = b > 0 ? column(b - 1) : 0;
        for (int q = b - 1; q >= 0; --q) {
            const int next = q > 0 ? column(q - 1) : 0;
            static_for<64>([&](auto I) { x += x >= __builtin_amdgcn_readlane(y, 63 - decltype(I)::value); });
            y = next;
        }
        if (64 * b + lane < k) *gp(orig + (size_t)(64 * b + lane) * H + r) = x;
    }
}

// Widened rows: one workgroup per row marks the seams' original columns in an LDS bitmap, counts
// the marks per thread chunk, scans the counts, and writes every pixel at its column plus the
// number of marks left of it, followed by the new pixel ((a + b + 1) >> 1 with the right
// neighbour; the pixel itself at the last column) where a column is marked.
constexpr int kInsertThreads = 256;
constexpr int kInsertMaxW = kInsertMaxWidth;  // the row bitmap lives in LDS
__global__ __launch_bounds__(kInsertThreads) void insert_seams_kernel(const uint8_t* __restrict__ img, int W, int C,
                                                                    long long pitch, int H, int k,
                                                                    const int32_t* __restrict__ orig,
                                                                    uint8_t* __restrict__ out, long long out_pitch) {
    __shared__ uint32_t bm[kInsertMaxW / 32];
    __shared__ int part[kInsertThreads];
    const int r = blockIdx.x, t = threadIdx.x;
    const int nwords = (W + 31) >> 5;
    for (int i = t; i < nwords; i += kInsertThreads) bm[i] = 0u;
    __syncthreads();
    for (int j = t; j < k; j += kInsertThreads) {
        const int c = min(max(*gp(orig + (size_t)j * H + r), 0), W - 1);
        atomicOr(&bm[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    const int wpt = (nwords + kInsertThreads - 1) / kInsertThreads;  // bitmap words per thread
    const int w0 = min(t * wpt, nwords), w1 = min(w0 + wpt, nwords);
    int cnt = 0;
    for (int i = w0; i < w1; ++i) cnt += __popc(bm[i]);
    part[t] = cnt;
    __syncthreads();
    if (t == 0) {
        int acc = 0;
        for (int i = 0; i < kInsertThreads; ++i) {
            const int v = part[i];
            part[i] = acc;
            acc += v;
        }
    }
    __syncthreads();
    int before = part[t];  // marks left of this thread's first column
    const uint8_t* row = img + (long long)r * pitch;
    uint8_t* o = out + (long long)r * out_pitch;
    for (int c = w0 * 32; c < min(w1 * 32, W); ++c) {
        const int pos = c + before;
        for (int ch = 0; ch < C; ++ch) *gp(o + (long long)pos * C + ch) = *gp(row + (long long)c * C + ch);
        if ((bm[c >> 5] >> (c & 31)) & 1u) {
            const int cr = c + 1 < W ? c + 1 : c;
            for (int ch = 0; ch < C; ++ch) {
                const int a = *gp(row + (long long)c * C + ch), b = *gp(row + (long long)cr * C + ch);
                *gp(o + (long long)(pos + 1) * C + ch) = (uint8_t)((a + b + 1) >> 1);
            }
            ++before;
        }
    }
}

// Launchers of the carve kernel variants (the table of shapes: SC_VARIANTS in sc_internal.h).
hipError_t launch_carve_single(const Img& d, int v, int G, int xcd, hipStream_t st) {
    switch (v) {
#define X(id, c, k, t) \
    case id: hipLaunchKernelGGL((carve_single_kernel<c, k, t>), dim3(8 * G), dim3(t), 0, st, d, xcd & 7); break;
        SC_VARIANTS(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_slot_write(Img* table, int slot, const Img& d, hipStream_t st) {
    hipLaunchKernelGGL(slot_write_kernel, dim3(1), dim3(1), 0, st, table, slot, d);
    return hipGetLastError();
}

hipError_t launch_seam_origins(const int32_t* seams, int k, int H, int W, int32_t*, int32_t* orig, hipStream_t st) {
    hipLaunchKernelGGL(seam_origins_kernel, dim3((H + 3) / 4), dim3(256), 0, st, seams, k, H, W, orig);
    return hipGetLastError();
}

hipError_t launch_insert_seams(const uint8_t* img, int H, int W, int C, long long pitch, int k, const int32_t* orig,
                               uint8_t* out, long long out_pitch, hipStream_t st) {
    if (W > kInsertMaxW) return hipErrorInvalidValue;
    hipLaunchKernelGGL(insert_seams_kernel, dim3(H), dim3(kInsertThreads), 0, st, img, W, C, pitch, H, k, orig, out,
                       out_pitch);
    return hipGetLastError();
}

hipError_t launch_energy_i32(const uint8_t* img, int H, int W, int C, long long pitch, int32_t* out, hipStream_t st) {
    dim3 grid((W + 1023) / 1024, (H + kEnergyRows - 1) / kEnergyRows);
    hipLaunchKernelGGL(energy_i32_kernel, grid, dim3(256), 0, st, img, H, W, C, pitch, out);
    return hipGetLastError();
}

hipError_t launch_prepare_single(const Img& d, hipStream_t st) {
    const int tiles = ((d.W + kTileCols - 1) / kTileCols) * ((d.H + kTileRows - 1) / kTileRows);
    const int blocks = tiles < 4096 ? tiles : 4096;
    hipLaunchKernelGGL(prepare_single_kernel, dim3(blocks), dim3(256), 0, st, d);
    return hipGetLastError();
}

hipError_t launch_prepare_from_i32(const Img& d, const int32_t* e, hipStream_t st) {
    dim3 grid((d.W + 255) / 256, d.H);
    hipLaunchKernelGGL(prepare_from_i32_kernel, grid, dim3(256), 0, st, d, e);
    return hipGetLastError();
}

hipError_t launch_prepare_batch(const Img* imgs, int n, int max_rows, hipStream_t st) {
    // workgroups per image: enough for the tiles of a tall image (each takes every per-th tile)
    const int chunks = (max_rows + kTileRows - 1) / kTileRows;
    const int per = chunks < 64 ? chunks : 64;
    hipLaunchKernelGGL(prepare_batch_kernel, dim3(per, n), dim3(256), 0, st, imgs, n);
    return hipGetLastError();
}

hipError_t launch_remove_seam(uint8_t* img, int H, int W, int C, long long pitch, const int32_t* seam,
                              hipStream_t st) {
    const int waves = H < 4096 ? H : 4096;
    hipLaunchKernelGGL(remove_seam_kernel, dim3((waves + 3) / 4), dim3(256), 0, st, img, H, W, C, pitch, seam);
    return hipGetLastError();
}

hipError_t launch_transpose(const uint8_t* src, int H, int W, int C, long long sp, uint8_t* dst, long long dp,
                            hipStream_t st) {
    dim3 grid((W + 63) / 64, (H + 63) / 64);
    switch (C) {
        case 1: hipLaunchKernelGGL(transpose_kernel<1>, grid, dim3(256), 0, st, src, H, W, sp, dst, dp); break;
        case 2: hipLaunchKernelGGL(transpose_kernel<2>, grid, dim3(256), 0, st, src, H, W, sp, dst, dp); break;
        case 3: hipLaunchKernelGGL(transpose_kernel<3>, grid, dim3(256), 0, st, src, H, W, sp, dst, dp); break;
        case 4: hipLaunchKernelGGL(transpose_kernel<4>, grid, dim3(256), 0, st, src, H, W, sp, dst, dp); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------------------
// Fixed scratch of the allocation-free carve (sc_carve_noalloc): a file-scope device array, one
// copy per GPU, held until the process ends.  In host code the array's name is only a host-side
// stand-in for it; the device address of each GPU's copy is looked up once per device with that
// device current and kept, and only that address is ever handed to kernels or copies.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

hipError_t noalloc_scratch(void** ptr) {
    static std::mutex mu;
    static void* addr[kNoAllocMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

__global__ void copy_status_kernel(const unsigned* __restrict__ src, uint32_t* __restrict__ dst) { *dst = *src; }

hipError_t launch_copy_status(const unsigned* src, uint32_t* dst, hipStream_t st) {
    hipLaunchKernelGGL(copy_status_kernel, dim3(1), dim3(1), 0, st, src, dst);
    return hipGetLastError();
}

}  // namespace sc
