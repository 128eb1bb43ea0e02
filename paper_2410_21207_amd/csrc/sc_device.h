// Device helpers shared by the kernels of libseamcarve (gfx950): global-address-space casts,
// raw buffer descriptors, the in-place row shifters, packed-pixel row loads and small VALU
// idioms.  Included by the .hip sources only.
#pragma once
#include <type_traits>
#include <utility>

#include "sc_internal.h"

namespace sc {

#define GAS __attribute__((address_space(1)))
// Every pointer reaches the kernels inside a descriptor, i.e. as a generic pointer; casting it to
// the global address space lets the compiler emit global_* instead of flat_* memory instructions.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ GAS T* gp(T* p) {
    return (GAS T*)p;
}

// A descriptor in constant memory (a kernel argument, or a table an earlier launch wrote).  fetch()
// reads it anew through scalar loads: each stage of a long loop takes its own copy, so that the
// compiler does not keep every stage's buffer descriptors and strides alive in scalar registers
// through all the others (hundreds of them, spilled to vector registers otherwise).
#ifdef __HIP_DEVICE_COMPILE__
#define CAS __attribute__((address_space(4)))
#else
#define CAS  // the host pass only parses the kernels
#endif
template <class T>
__device__ __forceinline__ T fetch(const CAS T* p) {
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(p));
#endif
    return *p;
}

// Words that a team shares, for the steps of sc_team.h.
struct DevMem {
    template <class W>
    static __device__ __forceinline__ W load(GAS W* p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    template <class W>
    static __device__ __forceinline__ void store(GAS W* p, W v) {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    template <class W>
    static __device__ __forceinline__ W add(GAS W* p, W v) {
        return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    template <class W>
    static __device__ __forceinline__ bool swap(GAS W* p, W& seen, W v) {
        return __hip_atomic_compare_exchange_strong(p, &seen, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};
struct DevClock {
    static __device__ __forceinline__ unsigned long long now() { return wall_clock64(); }
    static __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(1); }
};

// Raw buffer descriptors (gfx9 word 3).  A raw buffer access adds a wave-uniform byte offset
// (scalar register) to a per-lane byte offset (vector register); only the per-lane part is
// range checked, and an access whose per-lane offset is >= the descriptor's size is dropped
// (loads return 0, stores write nothing).
constexpr int kBufWord3 = 0x00020000;
constexpr uint32_t kBufDrop = 0x80000000u;  // a per-lane offset beyond any descriptor used here
typedef unsigned int v2u __attribute__((__vector_size__(8)));
typedef unsigned int v4u __attribute__((__vector_size__(16)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, kBufWord3);
}

// A dword at a lane's byte offset into a buffer.  COH, for data that another workgroup of the same team
// may have written since this compute unit last read it, sets the sc1 bit: the load skips the unit's L1 and
// reads the XCD's L2, where the other workgroup's stores have landed (a team always runs on one XCD).
// It is a plain load and leaves the compiler's memory-counter waits for later loads exact, where an
// atomic load in flight makes it wait for every outstanding access.
template <bool COH>
__device__ __forceinline__ uint32_t buf_ld32(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, 0, COH ? 16 : 0);
}

template <bool COH>
__device__ __forceinline__ uint8_t buf_ld8(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    return __builtin_amdgcn_raw_buffer_load_b8(r, (int)voff, 0, COH ? 16 : 0);
}

// A 16-byte store, with no scalar offset: with one, the compiler may overwrite the data registers in
// the very next instruction, and stores on gfx950 have been seen to take the new value (the first
// dword of a lane's 16 bytes), where without one it keeps the registers for the cycles they need.
__device__ __forceinline__ void buf_st128(__amdgpu_buffer_rsrc_t r, v4u v, uint32_t voff) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)voff, 0, 0);
}

__device__ __forceinline__ uint32_t xcc_id() {
    uint32_t v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return v;
}

// Calls f(std::integral_constant<int, 0>{}) ... f(std::integral_constant<int, N-1>{}) in order.
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// One-pixel shifts inside rows, in place, one wave.  Row i of a plane closes the gap of its seam
// pixel s: the pixels right of it move one column left (right = false), or the pixels left of it one
// column right (right = true; the row then starts one column later).  A row's pixels start at column
// o of the plane and w of them are in use.
//
// The work is the row's aligned 16-byte slots in ascending order, one per lane.  A lane loads 16 bytes
// from its slot (right: from a dword below it) and takes the dword above them from the next lane; its
// new bytes are then one v_perm per dword, whichever the direction.  The seam's slot, where the bytes on
// the far side of the seam pixel are kept, is left to lane l for row l, with selectors of its own: it
// is loaded before anything is stored and no other slot reads it.  At the other end the last slot runs
// over bytes of the row that are not in use.  A pass stores 63 slots: its last lane only lends its
// dword.  Moving right, a pass reads bytes that the pass before it writes, so a pass must load before
// the pass before it stores.
//
// What bounds it: accesses and their latency.  Every access is dword aligned: one that is not costs 64
// cycles of the compute unit's address path instead of 16 (measured, 16 bytes per lane), which a
// workgroup moving its rows with unaligned slots ran into (1200 x 1200 by one workgroup: 108 us per
// seam so, 86 us aligned; 3840 x 2160 by 16: 42 us and 30 us).  NR rows of NP planes are one item, and
// the next item's loads go out before this item's stores, so a wait for loads never covers a store (one
// counter for both, drained in order); nothing branches between them, or the counter's state would be
// lost.  Handing the seam slot's selectors to its lane in every pass cost four readlanes per row and plane, a third of
// the instructions: 1200 x 1200 by one workgroup 141 us of walk and removal so, 127 us with the
// seams' slots apart; 1920 x 1080 by 32 24.5 and 22 us.  Three rows to an item: four spill (512 thumbnails 2.98 ms
// against 2.75), two are as fast.
struct ShiftPlane {
    __amdgpu_buffer_rsrc_t r;  // from 16 bytes below the first row to 64 past the last
    uint32_t pitch;            // bytes per row, a multiple of 16
    int px;                    // bytes per pixel, 1..4
};

// n rows (at most 64) of a plane; there are 16 bytes of the workspace below them and 64 above.
__device__ __forceinline__ ShiftPlane shift_plane(void* row0, int n, uint32_t pitch, int px) {
    return {make_rsrc(static_cast<uint8_t*>(row0) - 16, 16u + (uint32_t)n * pitch + 64u), pitch, px};
}

// The n rows of the planes; lane l holds row l's seam s, start o and side.  LPR lanes work on a row
// (64 / LPR rows share an access; every row then fits LPR - 1 slots).
template <int LPR, int NR, int NP>
__device__ __forceinline__ void shift_rows_lpr(const ShiftPlane (&p)[NP], int n, int w, int s, int o, bool right, int lane) {
    constexpr int RPA = 64 / LPR;  // rows per access
    // per row and plane: the load offset of slot 0, the slots, the seam's slot with its selectors
    int at[NP], cnt[NP];
    uint32_t sel[NP][4], seam_off[NP], seam_up[NP];
    v4u seam_v[NP];
#pragma unroll
    for (int x = 0; x < NP; ++x) {
        const int px = p[x].px;
        const int lo = (right ? o + 1 : o + s) * px, hi = (right ? o + s + 1 : o + w - 1) * px;
        at[x] = lane * (int)p[x].pitch + 16 + (lo & ~15) - (right ? 4 : 0);
        cnt[x] = lane < n && hi > lo ? ((hi - 1) >> 4) - (lo >> 4) + 1 : 0;
        const int z = right ? ((hi - 1) & 15) + 1 : lo & 15;  // kept: the bytes below z, or from z on
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = z - 4 * i;
            const uint32_t low = c >= 4 ? ~0u : c <= 0 ? 0u : (1u << (8 * c)) - 1u;
            const uint32_t move = (uint32_t)px * 0x01010101u;
            // a moved byte of dword i is byte px (right: 4 - px) further on in dwords i, i + 1
            sel[x][i] = 0x03020100u + (right ? 0x04040404u - (move & low) : move & ~low);
        }
        seam_off[x] = cnt[x] > 0 ? (uint32_t)(at[x] + (right ? 16 * (cnt[x] - 1) : 0)) : kBufDrop;
        seam_v[x] = __builtin_amdgcn_raw_buffer_load_b128(p[x].r, (int)seam_off[x], 0, 0);
        seam_up[x] = __builtin_amdgcn_raw_buffer_load_b32(p[x].r, (int)(cnt[x] > 0 ? seam_off[x] + 16u : kBufDrop), 0, 0);
    }
    auto store_seams = [&]() {
#pragma unroll
        for (int x = 0; x < NP; ++x) {
            const uint32_t y[5] = {seam_v[x][0], seam_v[x][1], seam_v[x][2], seam_v[x][3], seam_up[x]};
            v4u out;
#pragma unroll
            for (int i = 0; i < 4; ++i) out[i] = __builtin_amdgcn_perm(y[i + 1], y[i], sel[x][i]);
            buf_st128(p[x].r, out, seam_off[x] + (right ? 4u : 0u));
        }
    };
    const int sub = lane / LPR, f0 = lane % LPR;
    auto row_of = [&](int v, int i) {  // row i's value, in the lanes that work on it
        if constexpr (LPR == 64) return __builtin_amdgcn_readlane(v, i);
        else return __shfl(v, i + sub, 64);
    };
    const int side = right;
    struct Slot {
        v4u v;
        uint32_t vo;
        int sd;
    };
    auto load = [&](Slot (&b)[NR][NP], int i, int fb) {  // rows i .. i + NR * RPA - 1, from slot fb of each
        int most = 0;
#pragma unroll
        for (int a = 0; a < NR; ++a) {
            const int li = min(i + a * RPA, 64 - RPA);  // rows past n have no slots
            const bool live = i + a * RPA < n;
            const int sd = row_of(side, li);
#pragma unroll
            for (int x = 0; x < NP; ++x) {
                const int base = row_of(at[x], li), c = live ? row_of(cnt[x], li) : 0;
                const int f = fb + f0;
                const uint32_t off = (uint32_t)(base + 16 * f);
                Slot& q = b[a][x];
                q.v = __builtin_amdgcn_raw_buffer_load_b128(p[x].r, (int)(f <= c && c > 0 ? off : kBufDrop), 0, 0);
                q.vo = f < c && f != (sd ? c - 1 : 0) && f0 < LPR - 1 ? off + (sd ? 4u : 0u) : kBufDrop;
                q.sd = sd;
                if constexpr (LPR == 64) most = max(most, c);
            }
        }
        return most;
    };
    auto store = [&](const Slot (&b)[NR][NP]) {
#pragma unroll
        for (int a = 0; a < NR; ++a)
#pragma unroll
            for (int x = 0; x < NP; ++x) {
                const Slot& q = b[a][x];
                const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q.v[0], 0x130, 0xf, 0xf, true);
                const uint32_t y[5] = {q.v[0], q.v[1], q.v[2], q.v[3], up};
                const uint32_t all = 0x03020100u + (uint32_t)(q.sd ? 4 - p[x].px : p[x].px) * 0x01010101u;
                v4u out;
#pragma unroll
                for (int i = 0; i < 4; ++i) out[i] = __builtin_amdgcn_perm(y[i + 1], y[i], all);
                buf_st128(p[x].r, out, q.vo);
            }
    };
    int i = 0, fb = 0;
    auto step = [&](int most) {  // the next pass of these rows, or the next rows
        const bool again = LPR == 64 && fb + 63 < most;
        i = again ? i : i + NR * RPA;
        fb = again ? fb + 63 : 0;
    };
    Slot A[NR][NP], B[NR][NP];
    step(load(A, i, fb));
    bool mb = i < n;
    step(load(B, i, fb));
    store_seams();
    for (;;) {
        store(A);
        if (!mb) break;
        const bool ma = i < n;
        step(load(A, i, fb));
        store(B);
        if (!ma) break;
        mb = i < n;
        step(load(B, i, fb));
    }
}

// `most`: the bytes that the widest row may have to move.  Rows of narrow images share accesses.
template <int NR, int NP>
__device__ __forceinline__ void shift_rows(const ShiftPlane (&p)[NP], int n, int w, int s, int o, bool right, int most,
                                           int lane) {
    if (most <= 208) shift_rows_lpr<16, 2, NP>(p, n, w, s, o, right, lane);
    else shift_rows_lpr<64, NR, NP>(p, n, w, s, o, right, lane);
}

// dst bytes [dst, dst + n) take the bytes of [src, src + n), one wave; the buffers do not overlap.
// Dword-granular on the destination; bytes of a destination dword outside [dst, dst + n) are not
// written (they may belong to a neighbouring row).  Source dwords may be read a few bytes beyond
// either end of the source range.
__device__ __forceinline__ void copy_bytes_wave(uint8_t* dst, const uint8_t* src, int n, int lane) {
    if (n <= 0) return;
    const int off = (int)((uintptr_t)dst & 3);
    uint8_t* const base = dst - off;  // dword-aligned; destination dword j covers base + 4j
    const int nd = ((off + n - 1) >> 2) + 1;
    const uintptr_t s0 = (uintptr_t)src - (uintptr_t)off;  // source byte of base + x is s0 + x
#pragma unroll 1
    for (int jb = 0; jb < nd; jb += 64 * 4) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = jb + u * 64 + lane;
            v[u] = 0;
            if (j < nd) {
                const uintptr_t sa = s0 + 4 * (uintptr_t)j;
                const uint32_t* sp = reinterpret_cast<const uint32_t*>(sa & ~(uintptr_t)3);
                const uint32_t lo = *gp(sp);
                const uint32_t hi = (sa & 3) ? *gp(sp + 1) : 0u;
                v[u] = __builtin_amdgcn_alignbyte(hi, lo, (uint32_t)(sa & 3));
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = jb + u * 64 + lane;
            if (j >= nd) continue;
            uint8_t* dp = base + 4 * j;
            if (dp >= dst && dp + 4 <= dst + n) {
                *gp(reinterpret_cast<uint32_t*>(dp)) = v[u];
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (dp + k >= dst && dp + k < dst + n) *gp(dp + k) = (uint8_t)(v[u] >> (8 * k));
            }
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Helpers of the single-workgroup DP (object removal on tall frames).

// v_min3_u32: the smallest of three tagged keys (ties go to the smallest tag, i.e. the leftmost).
__device__ __forceinline__ uint32_t min3u(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t o;
    asm("v_min3_u32 %0, %1, %2, %3" : "=v"(o) : "v"(a), "v"(b), "v"(c));
    return o;
}

// kk + (cu << 9) - 127 * tag - 1 with tag = bits 7-8 of kk: drops the tag, adds CU to M and moves
// the ancestor offset by tag - 1.
__device__ __forceinline__ uint32_t next_state(uint32_t kk, uint32_t cu) {
    const uint32_t tag = (kk >> 7) & 3u;
    uint32_t o;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(o) : "v"(tag), "s"(-127), "v"(kk + (cu << 9) - 1u));
    return o;
}

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The pixels a thread needs from one row of a working image: CPL columns j0 .. j0+CPL-1 and one
// neighbour on each side, as packed channels.
template <int C, int CPL>
struct PixRow {
    // A thread reads the dwords covering columns j0-1 .. j0+CPL of a row: they start at byte
    // j0*C - 4 (j0*C is a multiple of 4 because CPL is), where column j0-1 sits at byte LEAD.
    static constexpr int LEAD = (4 - C % 4) % 4;
    static constexpr int NDW = (LEAD + (CPL + 2) * C + 3) / 4;
    static constexpr uint32_t PMASK = C == 4 ? 0xFFFFFFFFu : (1u << (8 * C)) - 1u;
    static_assert(CPL % 4 == 0, "a thread's directions fill whole bytes");

    // vl: byte offset of the dword left of column j0 (it holds only column j0-1); v0: of column j0.
    // Either is kBufDrop where nothing may be read (the load then returns 0).
    static __device__ __forceinline__ void load_row(uint32_t (&v)[NDW], __amdgpu_buffer_rsrc_t r, uint32_t vl,
                                                    uint32_t v0, uint32_t soff) {
        v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)vl, (int)soff, 0);
#pragma unroll
        for (int q = 1; q < NDW; ++q) v[q] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(v0 + 4u * (q - 1)), (int)soff, 0);
    }

    // pixel k (column j0-1+k) of a loaded row, channels packed in the low bytes
    static __device__ __forceinline__ void pixels(const uint32_t (&v)[NDW], uint32_t (&p)[CPL + 2]) {
#pragma unroll
        for (int k = 0; k < CPL + 2; ++k) {
            const int o = LEAD + C * k, q = o >> 2, r = o & 3;
            uint32_t x;
            if (r == 0) x = v[q];
            else if (r + C <= 4) x = v[q] >> (8 * r);
            else x = __builtin_amdgcn_alignbyte(v[q + 1], v[q], (uint32_t)r);
            p[k] = x & PMASK;
        }
    }

};

// ----------------------------------------------------------------------------------------------
// Team barrier.  One workgroup: a workgroup barrier.  A team of G workgroups on one XCD: each
// thread waits for its own stores to reach the L2 (vmcnt), then one thread per workgroup bumps
// the image's counter with a device-scope atomic and polls it with device-scope loads until all
// G have arrived; readers then fetch shared data with sc1 loads (see buf_ld32).  The wait is
// bounded: after ~10 s it flags the image and every member gives up on it.
template <bool TEAM>
__device__ __forceinline__ bool team_sync(const CAS Img* gd, unsigned& epoch, int G, int* flag) {
    if constexpr (!TEAM) {
        __syncthreads();
        return true;
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) {
            const Img d = fetch(gd);
            epoch += (unsigned)G;
            __hip_atomic_fetch_add(gp(d.bar), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long t0 = wall_clock64();
            int ab = 0;
            while (__hip_atomic_load(gp(d.bar), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch) {
                __builtin_amdgcn_s_sleep(1);
                if (__hip_atomic_load(gp(d.status), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
                    (kStatusTimeout | kStatusPlacement)) {
                    ab = 1;
                    break;
                }
                if (wall_clock64() - t0 > 1000000000ull) {  // 10 s at the 100 MHz constant clock
                    __hip_atomic_fetch_or(gp(d.status), kStatusTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ab = 1;
                    break;
                }
            }
            *flag = ab;
        }
        __syncthreads();
        return *flag == 0;
    }
}

// Reset the control words of one image (every carve launch starts from them).
__device__ __forceinline__ void reset_ctl(const Img& d) {
    GAS Ctl* c = gp(reinterpret_cast<Ctl*>(d.bar));
    c->bar = 0;
    c->status = 0;
    c->t_begin = c->t_end = 0;
    c->join = 0;
    c->done = 0;
    c->t_stage[0] = c->t_stage[1] = c->t_stage[2] = 0;
    c->ebase = 0;
    c->stop = 0;
    c->left = 0;
}

// One source row as seen by a thread owning 4 pixels from column x0: the aligned dwords covering
// the pixels and one neighbour on each side, realigned to the row's start with v_alignbyte (a
// caller's rows may start at any byte).
template <int C>
struct SrcRow {
    static constexpr int ND = C + 3;   // dwords loaded per thread
    static constexpr uint32_t PMASK = C == 4 ? 0xFFFFFFFFu : (1u << (8 * C)) - 1u;
    uint32_t r[C + 2];                 // row bytes [x0*C - 4, x0*C + 4*C + 4), dword aligned to the row

    // Row y of the image (pitch bytes per row, W*C bytes used): the thread's pixels start at x0.
    __device__ __forceinline__ void load(const uint8_t* img, long long pitch, int W, int y, int x0) {
        const uint8_t* row = img + (long long)y * pitch;
        const uint32_t sh = (uint32_t)((uintptr_t)row & 3u);
        // the descriptor covers the whole dwords holding the row's bytes (a dword-aligned dword that
        // holds an image byte lies inside the image's allocation); dwords outside are dropped (read
        // as 0), and only clamped neighbours would use them
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(row - sh, (sh + (uint32_t)(W * C) + 3u) & ~3u);
        // per-lane offsets never wrap: the dword left of column x0 has an offset of its own (dropped
        // at x0 = 0), the others count up from column x0 (an immediate offset may be folded in)
        const uint32_t v0 = x0 < W ? (uint32_t)(x0 * C) : kBufDrop;
        const uint32_t vl = x0 < W && x0 > 0 ? (uint32_t)(x0 * C - 4) : kBufDrop;
        uint32_t d[ND];
        d[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)vl, 0, 0);
#pragma unroll
        for (int m = 1; m < ND; ++m) d[m] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(v0 + 4u * (m - 1)), 0, 0);
#pragma unroll
        for (int m = 0; m < C + 2; ++m) r[m] = __builtin_amdgcn_alignbyte(d[m + 1], d[m], sh);
    }
    // pixel p of the thread (p = -1 .. 4), channels packed in the low bytes
    __device__ __forceinline__ uint32_t px(int p) const {
        const int o = 4 + p * C, q = o >> 2, b = o & 3;
        const uint32_t v = b == 0 ? r[q] : __builtin_amdgcn_alignbyte(r[q + 1], r[q], (uint32_t)b);
        return v & PMASK;
    }
};

}  // namespace sc
