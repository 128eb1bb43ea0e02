// The carve engine of the seam-carving hot path for gfx950 (CDNA4), included by the .hip sources.
//
// Steps (arXiv 2410.21207): e1 energy (sec. "Energy Mapping"), the DP table
// M(i,j) = e(i,j) + min(M(i-1,j-1..j+1)) (DP section, Alg. 3), the bottom-row
// argmin, the backtrack (Alg. 3) and the removal of the seam (sec. "Removal of
// Seams"), repeated once per seam on the current image (flowchart loop).
//
// Design (nothing here is a contraction, so no MFMA; every step is integer):
//  * The cost table is swept from both ends of the image at once, costs only: a row is a v_min3 and an
//    add per column and two DPP wave shifts, and the chain of dependent rows is half the image.
//  * A wave owns a strip of columns and computes KR ghost columns on each side, so it runs KR rows
//    without its neighbours ("ghost zone" tiling).  Every R rows the exact costs go out to memory
//    with the seam's tag; whoever needs them (the neighbours at the next phase, the middle, the
//    backtrack) loads until the tag shows, so a team's waves wait for data and not for each other.
//  * The cheapest pair of neighbouring cells in the two middle rows gives the seam's cost and its two
//    middle columns.
//  * The backtrack computes the directions again, in blocks of R rows, all at once and only for 256
//    columns around the path: keys M << 9 | u << 2 | tag carry the direction tag (0/1/2: left, up, right, so
//    one minimum picks the value AND the leftmost tie, reading R5) and the ancestor's offset; the path
//    then hops from block to block and is walked from registers.  No direction map goes to memory.
//  * Removal shifts the shorter side of each row one pixel toward the seam (the right side only when
//    min-side removal is off); the energy is then recomputed only at the two new columns {s-1, s} of each
//    row (the only cells whose stencil changed).
//
// Three kinds of image share the engine (Kind below): energies, forward energy and masked energies.
//
// What bounds it (1920 x 1080 by 32 workgroups on MI355X, us per seam, in all 53, 122 before the sweep
// from both ends): sweep and middle 28 (issue: a wave starts an instruction every 5.3 cycles, 14 of them
// per row, and waits about a microsecond for its neighbours at each of nine phases), backtrack and
// removal 20 (when they took 23: trace 4.4, barrier and hops 7.7, walk 0.8, removal 10.3), barrier and
// new energies 4.  The workspace's address is worth 5 %: the same carve takes 51.5 to 54 at offsets of 0 to
// 100 MB, the removal and the energies 3 of them.
#pragma once
#include "sc_device.h"
#include "sc_team.h"

namespace sc {

constexpr uint32_t QINF = 0xFFFFFF00u;  // "+infinity" key: larger than any real key, +10 cannot wrap

// r + 512 * (low or high 16 bits of `pair`): one v_mad_u32_u16 adds e(i,j) << 9 to a backtrack key
// straight from the packed uint16 energy pair, with no separate unpack.
__device__ __forceinline__ uint32_t mad_lo16(uint32_t pair, uint32_t r) {
    uint32_t o;
    asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(o) : "v"(pair), "s"(512u), "v"(r));
    return o;
}
__device__ __forceinline__ uint32_t mad_hi16(uint32_t pair, uint32_t r) {
    uint32_t o;
    asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(o) : "v"(pair), "s"(512u), "v"(r));
    return o;
}

// ----------------------------------------------------------------------------------------------
// e1 energy at logical column x of a row from a buffer: the row starts at byte offset br of the
// descriptor's memory, the rows above and below at bu and bd (min-side removal keeps every row at
// its own offset).  The channel loop runs to 4 with dropped offsets past C, so the loads carry no
// branches and go out together; a column outside [0, w) is clamped like the pixels of any other
// (callers do not store its value).
template <bool COH>
__device__ __forceinline__ uint32_t energy_buf(__amdgpu_buffer_rsrc_t rb, uint32_t br, uint32_t bu, uint32_t bd, int w,
                                               int C, int x) {
    x = min(max(x, 0), w - 1);
    const int xl = x > 0 ? x - 1 : 0, xr = x + 1 < w ? x + 1 : w - 1;
    uint32_t s = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const bool ok = c < C;
        const int a = (int)buf_ld8<COH>(rb, ok ? br + (uint32_t)(xr * C + c) : kBufDrop);
        const int b = (int)buf_ld8<COH>(rb, ok ? br + (uint32_t)(xl * C + c) : kBufDrop);
        const int dn = (int)buf_ld8<COH>(rb, ok ? bd + (uint32_t)(x * C + c) : kBufDrop);
        const int up = (int)buf_ld8<COH>(rb, ok ? bu + (uint32_t)(x * C + c) : kBufDrop);
        s += (uint32_t)abs(a - b) + (uint32_t)abs(dn - up);
    }
    return s;
}

// ----------------------------------------------------------------------------------------------
// Energies at the lane's byte offset `off` of the row starting `soff` bytes into the plane
// (wave-uniform: row base plus the row's start offset).  COH sets the sc1 bit.
template <bool COH, int N>
__device__ __forceinline__ void load_ev(uint64_t (&e)[(N + 3) / 4], __amdgpu_buffer_rsrc_t re, uint32_t soff,
                                               uint32_t off) {
    if constexpr (N == 2) {
        e[0] = __builtin_amdgcn_raw_buffer_load_b32(re, (int)off, (int)soff, COH ? 16 : 0);
    } else if constexpr (N == 4) {
        const v2u v = __builtin_amdgcn_raw_buffer_load_b64(re, (int)off, (int)soff, COH ? 16 : 0);
        e[0] = ((uint64_t)v[1] << 32) | v[0];
    } else {
        const v4u v = __builtin_amdgcn_raw_buffer_load_b128(re, (int)off, (int)soff, COH ? 16 : 0);
        e[0] = ((uint64_t)v[1] << 32) | v[0];
        e[1] = ((uint64_t)v[3] << 32) | v[2];
        if constexpr (N == 16) {
            const v4u u = __builtin_amdgcn_raw_buffer_load_b128(re, (int)(off + 16u), (int)soff, COH ? 16 : 0);
            e[2] = ((uint64_t)u[1] << 32) | u[0];
            e[3] = ((uint64_t)u[3] << 32) | u[2];
        }
    }
}

// One wait for the loads up to this one, in place of one at the first use of each.
template <int N>
__device__ __forceinline__ void arrived(const uint64_t (&e)[N]) {
    asm volatile("" ::"v"(e[N - 1]));
}

// A team's waves wait for each other's data, not for each other: what a seam publishes carries its
// tag, and a reader loads again until it shows.  Bounded: `late` says when to give up (10 s at the
// 100 MHz constant clock, or at once when the image has failed) and flags the image.
struct Wait {
    unsigned long long t0 = 0;
    int n = 0;
    __device__ __forceinline__ bool late(const Img& d) {
        __builtin_amdgcn_s_sleep(1);
        if ((n++ & 63) != 63) return false;
        const unsigned long long now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 <= 1000000000ull &&
            !(__hip_atomic_load(gp(d.status), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
              (kStatusTimeout | kStatusPlacement)))
            return false;
        __hip_atomic_fetch_or(gp(d.status), kStatusTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
};

// The word by which an image's team forms; the image's first pass of every launch clears it.
__device__ __forceinline__ GAS unsigned long long* team_word(const CAS Img* gd) {
    return &gp(reinterpret_cast<Ctl*>(gd->bar))->join;
}

// Tag of a row's seam column (16 bits, columns below 65535), in the upper half of its word: never 0.
__device__ __forceinline__ uint32_t seam_word(int k) { return ((uint32_t)k + 1u) << 16; }

// What the sweep and the backtrack read: the plane of 16-bit energies; the current pixels, a dword
// each (forward energy); or energies of 32 bits, those of pixels outside the mask raised by
// masked_bias (object removal).
enum Kind { kEnergy, kForward, kMasked };
// Tag of the keys a seam publishes, never the 0 of a cleared row.  Every row of ck is written once
// per seam, so a reader only has to tell a seam from the one before it: 1..511 in nine bits, or one
// bit under the 31-bit costs of a masked image.
template <Kind KD>
__device__ __forceinline__ uint32_t seam_tag(int k) {
    return KD == kMasked ? ~(uint32_t)k & 1u : 1u + (uint32_t)k % 511u;
}

template <int R, Kind KD>
struct Rows {
    static constexpr bool FWD = KD == kForward, MSK = KD == kMasked;
    static constexpr uint32_t CB = KD == kEnergy ? 2 : 4;  // bytes per column
    static constexpr int SH = MSK ? 1 : 9;                 // bits of a published key's tag
    static constexpr uint32_t TAG = (1u << SH) - 1;
    // The rows of one half (h = 0: from the top down to the split row, 1: from the bottom up).
    // Virtual row v of a half is image row v - pad counted from the half's border; the rows below
    // pad do not exist and read the plane's row of zeros (row H), so that the half is a whole number
    // of blocks and its first real row costs its own energy.
    struct Half {
        int n, B, pad;  // rows, blocks, missing rows
    };
    static __device__ __forceinline__ Half half_of(int H, int mode, int h) {
        const int m = split_row(H, mode);
        Half x;
        x.n = h ? H - m : m;
        x.B = (x.n + R - 1) / R;
        x.pad = x.B * R - x.n;
        return x;
    }

    // Byte offset in the energy plane of virtual row v (its base plus its start offset) of half h,
    // rows past the half clamped to its last one.
    template <bool COH>
    static __device__ __forceinline__ uint32_t row_off(const Img& d, const Half& x, int h, int v,
                                                       __amdgpu_buffer_rsrc_t rro) {
        const int i = min(v - x.pad, x.n - 1);
        const int r = i < 0 ? d.H : h ? d.H - 1 - i : i;
        return (uint32_t)r * (uint32_t)d.ep * 2u + CB * buf_ld32<COH>(rro, i < 0 ? kBufDrop : (uint32_t)r * 4u);
    }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t energy_rsrc(const Img& d) {
        return make_rsrc(d.e, (uint32_t)(d.H + 1) * (uint32_t)d.ep * 2u);
    }

};

// ---- the cost sweep (a3): costs only, no directions; published as M << SH | tag.
//
// A seam's cost table is swept from both ends of the image at once, T from the top row down to
// the split row and B from the bottom row up, and the cheapest pair of adjacent cells in the two
// middle rows gives the seam's cost and its two middle columns.  The tie rules survive: among
// the cheapest seams the backtrack wants the smallest (s[H-1], ..., s[0]), paths chosen by
// "leftmost minimum" from neighbouring cells never cross, so in the lower half the leftmost
// child leads to the leftmost end, and the leftmost middle column to the leftmost path of all.
//
// What bounds it: a chain of rows, each one wave's instructions.  Without directions and
// ancestor offsets a row is a v_min3 and an add per column and two wave shifts (15 instructions for
// 256 columns), and the two ends halve the chain.  Rows are loaded a block ahead, one wait per eight
// rows.  1920 x 1080 by 32 workgroups: 27 us per seam where the one-ended sweep with directions took 106.
template <int CPL, int KR, int R, Kind KD>
struct Sweep : Rows<R, KD> {
    using Half = typename Rows<R, KD>::Half;
    using Rows<R, KD>::half_of;
    using Rows<R, KD>::energy_rsrc;
    using Rows<R, KD>::CB;
    using Rows<R, KD>::FWD;
    using Rows<R, KD>::MSK;
    using Rows<R, KD>::SH;
    using Rows<R, KD>::TAG;
    static constexpr int ND = CB == 4 ? CPL / 2 : (CPL + 3) / 4;  // 64-bit words of a lane's columns
    // FWD needs the row above too, so a row's registers are loaded anew only after the next row.
    static constexpr int LATE = FWD ? 1 : 0;
    // The cost of a missing parent, more than any real one; FWD adds to it and must not wrap.
    static constexpr uint32_t INF = FWD ? 0x40000000u : 0xFFFFFFFFu;
    static constexpr int WIN = 64 * CPL;    // columns a wave computes
    static constexpr int S = WIN - 2 * KR;  // columns a strip adds: KR ghost columns on each side
    static constexpr int PF = R == 32 ? (CB == 4 ? 64 : 128) / CPL : R;  // rows prefetched ahead
    static_assert(CPL == 2 || CPL == 4 || CPL == 8, "one energy load per lane and row");
    static_assert(KR % R == 0 && R % PF == 0 && PF % 8 == 0 && KR <= 64 && R <= 63 && KR % CPL == 0 && S > 0, "phase shape");

    // Eight columns per lane: rows are loaded from the dword at or below the lane's first energy and
    // moved by half a dword where the row starts at an odd column (an access off the dword grid costs
    // four times as much, and strips this wide run several to a compute unit).  A lane takes the dword
    // after its own from the next lane; lane 63 has none, so it is ghost columns, or past the image:
    // the last strip's window runs eight columns past w, and the first of them stays all ones.
    static constexpr bool GRID = CPL == 8 && CB == 2;  // (dwords start on the grid)
    static constexpr int WINR = GRID ? WIN - CPL : WIN;  // columns of the last strip's window in the image

    static __device__ __forceinline__ int strips(int w) { return w <= WINR ? 1 : (w - WINR + S - 1) / S + 1; }

    struct Item {
        int p, j;      // phase, the wave's item in it
        int h, t;      // half, strip
        int v0, v1;    // virtual rows
        uint32_t off;  // byte offset of the lane's first column in an energy row
        int col0;      // the lane's first column
        int base;      // the strip's first column
        int ns;
    };
    static __device__ __forceinline__ Item make_item(const Half (&hf)[2], int w, int ns, int tw, int TW, int p, int j,
                                                     int lane) {
        Item it;
        it.p = p;
        it.j = j;
        it.ns = ns;
        const int q = __builtin_amdgcn_readfirstlane(tw + j * TW);
        const bool two = hf[1].n > 0;
        it.h = two ? q & 1 : 0;
        it.t = two ? q >> 1 : q;
        const Half x = it.h ? hf[1] : hf[0];
        it.v0 = p ? p * KR : x.pad - x.pad % PF;
        it.v1 = min(x.B * R, p * KR + KR);
        const int base = it.t == ns - 1 ? max(0, w - WINR) : it.t * S;
        it.base = __builtin_amdgcn_readfirstlane(base);
        it.v0 = __builtin_amdgcn_readfirstlane(it.v0);
        it.v1 = __builtin_amdgcn_readfirstlane(it.v1);
        it.col0 = base + lane * CPL;
        it.off = GRID ? (uint32_t)lane * (2u * CPL) : (uint32_t)(it.col0 < w ? it.col0 : 0) * CB;
        return it;
    }

    // EDGE: the one strip of an image narrower than a window (columns from w on are kept all ones).
    template <bool EDGE>
    static __device__ __forceinline__ void cost_step(uint32_t (&Q)[CPL], uint32_t& left, uint32_t& right,
                                                     const uint64_t (&raw)[ND], uint32_t odd, const uint32_t (&em)[CPL]) {
        // Neighbours of the lane's first and last column come from lanes -1 and +1.  Lane 0's left and
        // lane 63's right keep all ones: a window's side is either the image's edge, where that is the
        // missing parent, or ghost columns, where a wrong value moves one column inward per row and
        // never reaches an owned column within a phase.
        left = (uint32_t)__builtin_amdgcn_update_dpp((int)left, (int)Q[CPL - 1], 0x138, 0xf, 0xf, false);
        right = (uint32_t)__builtin_amdgcn_update_dpp((int)right, (int)Q[0], 0x130, 0xf, 0xf, false);
        // (three-operand minima by hand: the compiler would share two-operand ones between columns,
        // one instruction more per pair) first and last column first, for the next row's wave shifts
        uint32_t pair[CPL / 2];  // energies of columns 2j, 2j + 1
#pragma unroll
        for (int j = 0; j < CPL / 2; ++j) pair[j] = MSK ? 0u : (uint32_t)(raw[j >> 1] >> ((j & 1) * 32));
        if constexpr (GRID) {  // odd: 0 or 16
            const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)pair[0], 0x130, 0xf, 0xf, true);
#pragma unroll
            for (int j = 0; j < CPL / 2; ++j)
                pair[j] = __builtin_amdgcn_alignbit(j + 1 < CPL / 2 ? pair[j + 1] : up, pair[j], odd);
        }
        uint32_t n[CPL];
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            const int k = i == 0 ? 0 : i == 1 ? CPL - 1 : i - 1;
            n[k] = min3u(k ? Q[k - 1] : left, Q[k], k + 1 < CPL ? Q[k + 1] : right);
        }
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            const int k = i == 0 ? 0 : i == 1 ? CPL - 1 : i - 1;
            if constexpr (MSK) Q[k] = n[k] + (uint32_t)(raw[k >> 1] >> ((k & 1) * 32));
            else Q[k] = n[k] + ((k & 1) ? pair[k >> 1] >> 16 : pair[k >> 1] & 0xFFFFu);
            if (EDGE || (GRID && k == 0)) Q[k] |= em[k];
        }
    }

    // The same row of the forward energy: the parents' keys cost the pairs of pixels that become
    // neighbours (D = one v_sad_u8 on packed channels, which adds the key too).  The row formula
    // is the same upward: the child at the left costs D(left pixel, pixel below), the one at the right
    // D(right pixel, pixel below).  A pixel missing at a window's side is the lane's own: at the image's
    // edge that is the clamp, elsewhere the side is ghost columns.  last: columns whose right neighbour
    // is past the image (EDGE).
    template <bool EDGE>
    static __device__ __forceinline__ void forward_step(uint32_t (&Q)[CPL], uint32_t& left, uint32_t& right,
                                                        const uint64_t (&above)[ND], const uint64_t (&raw)[ND],
                                                        const uint32_t (&em)[CPL], const bool (&last)[CPL]) {
        uint32_t p[CPL], P[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            p[c] = (uint32_t)(raw[c >> 1] >> ((c & 1) * 32));
            P[c] = (uint32_t)(above[c >> 1] >> ((c & 1) * 32));
        }
        left = (uint32_t)__builtin_amdgcn_update_dpp((int)left, (int)Q[CPL - 1], 0x138, 0xf, 0xf, false);
        right = (uint32_t)__builtin_amdgcn_update_dpp((int)right, (int)Q[0], 0x130, 0xf, 0xf, false);
        const uint32_t pl = (uint32_t)__builtin_amdgcn_update_dpp((int)p[0], (int)p[CPL - 1], 0x138, 0xf, 0xf, false);
        const uint32_t pr = (uint32_t)__builtin_amdgcn_update_dpp((int)p[CPL - 1], (int)p[0], 0x130, 0xf, 0xf, false);
        uint32_t n[CPL];
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            const int k = i == 0 ? 0 : i == 1 ? CPL - 1 : i - 1;
            const uint32_t l = k ? p[k - 1] : pl;
            uint32_t r = k + 1 < CPL ? p[k + 1] : pr;
            if (EDGE) r = last[k] ? p[k] : r;
            const uint32_t a = __builtin_amdgcn_sad_u8(P[k], l, k ? Q[k - 1] : left);
            const uint32_t b = __builtin_amdgcn_sad_u8(P[k], r, k + 1 < CPL ? Q[k + 1] : right);
            n[k] = __builtin_amdgcn_sad_u8(l, r, min3u(a, Q[k], b));
            if (EDGE) n[k] |= em[k];
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c) Q[c] = n[c];
    }

    // Returns false when the wait for a neighbour's keys timed out (the image's status says so).
    template <bool EDGE, bool TEAM>
    static __device__ __forceinline__ bool cost_sweep(const Img& d, int w, int k, int tw, int TW, int lane) {
        const Half hf[2] = {half_of(d.H, d.mode, 0), half_of(d.H, d.mode, 1)};
        const int ns = strips(w), items = hf[1].n > 0 ? 2 * ns : ns;
        if (tw >= items) return true;
        const int nsw = (items - tw + TW - 1) / TW;
        const int P0 = (hf[0].B * R + KR - 1) / KR, P1 = (hf[1].B * R + KR - 1) / KR;
        const uint32_t tag = seam_tag<KD>(k);
        const __amdgpu_buffer_rsrc_t re = energy_rsrc(d);
        const __amdgpu_buffer_rsrc_t rro = make_rsrc(d.ro, (uint32_t)d.H * 4u);
        const uint32_t ckrow = (uint32_t)d.xw * 4u;
        const __amdgpu_buffer_rsrc_t rck = make_rsrc(d.xq, (uint32_t)d.P * ckrow);
        constexpr uint32_t kGrid = GRID ? ~3u : ~0u;

        Item it = make_item(hf, w, ns, tw, TW, 0, 0, lane);
        uint32_t roff = Rows<R, KD>::template row_off<TEAM>(d, it.h ? hf[1] : hf[0], it.h, it.v0 + lane, rro) + (GRID ? 2u * (uint32_t)it.base : 0u);
        uint64_t ring[PF][ND];
#pragma unroll
        for (int i = 0; i + LATE < PF; ++i)
            load_ev<TEAM, (int)CB * CPL / 2>(ring[i], re, (uint32_t)__builtin_amdgcn_readlane(roff, i) & kGrid, it.off);
        uint32_t Q[CPL], em[CPL];  // em: all ones in columns past the image
        auto set_em = [&]() {
#pragma unroll
            for (int c = 0; c < CPL; ++c) em[c] = (EDGE || GRID) && it.col0 + c >= w ? INF : 0u;
        };
        set_em();
#pragma unroll
        for (int c = 0; c < CPL; ++c) Q[c] = em[c];
        bool last[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) last[c] = FWD && EDGE && it.col0 + c + 1 >= w;
        // in lane l: half a dword if row l of the item starts off the dword grid
        auto odd_of = [&](uint32_t r) { return GRID ? (r & 2u) << 3 : 0u; };
        uint32_t odd = odd_of(roff);
        uint32_t left = INF, right = INF;
        for (;;) {
            // the wave's next item: its row offsets now, its first rows during this item's last block
            int pn = it.p, jn = it.j;
            do {
                if (++jn == nsw) jn = 0, ++pn;
            } while (pn < P0 && hf[1].n > 0 && pn >= P1 && ((tw + jn * TW) & 1));
            const bool more = pn < P0;
            const Item nx = more ? make_item(hf, w, ns, tw, TW, pn, jn, lane) : it;
            const uint32_t roffn = Rows<R, KD>::template row_off<TEAM>(d, nx.h ? hf[1] : hf[0], nx.h, nx.v0 + lane, rro) + (GRID ? 2u * (uint32_t)nx.base : 0u);
            // lanes from rg on are ghost columns: KR of them left of the window's right side, or (GRID: the
            // last strip but one may reach past the image) of the image's
            const int rg = it.t == ns - 1 ? 64 : GRID ? min(64 - KR / CPL, (w - it.base - KR) / CPL) : 64 - KR / CPL;
            // keys of the row above: the ghost columns, or every column when the wave has several items
            if (it.p == 0) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) Q[c] = em[c];
                if constexpr (FWD) {
#pragma unroll
                    for (int c = 0; c < ND; ++c) ring[PF - 1][c] = 0;
                }
            } else if (ns > 1) {
                if (FWD && nsw > 1)  // the wave comes from another strip
                    load_ev<TEAM, (int)CB * CPL / 2>(ring[PF - 1], re, (uint32_t)__builtin_amdgcn_readfirstlane(Rows<R, KD>::template row_off<TEAM>(
                                                                           d, it.h ? hf[1] : hf[0], it.h, it.v0 - 1, rro)), it.off);
                const bool need = nsw > 1 || (it.t > 0 && lane < KR / CPL) || lane >= rg;
                const uint32_t krow = (uint32_t)((it.h ? hf[0].B : 0) + it.v0 / R - 1) * ckrow;
                const uint32_t ko = need ? (uint32_t)it.col0 * 4u : kBufDrop;
                Wait wait;
                for (;;) {
                    uint32_t x[CPL];
                    if constexpr (CPL == 2) {
                        const v2u v = __builtin_amdgcn_raw_buffer_load_b64(rck, (int)ko, (int)krow, 16);
                        x[0] = v[0], x[1] = v[1];
                    } else {
#pragma unroll
                        for (int c = 0; c < CPL; c += 4) {
                            const v4u v = __builtin_amdgcn_raw_buffer_load_b128(rck, (int)(ko + 4u * c), (int)krow, 16);
                            x[c] = v[0], x[c + 1] = v[1], x[c + 2] = v[2], x[c + 3] = v[3];
                        }
                    }
                    bool ok = true;
#pragma unroll
                    for (int c = 0; c < CPL; ++c) ok = ok && ((x[c] & TAG) == tag || (GRID && em[c]));
                    if (__all(ok || !need)) {
#pragma unroll
                        for (int c = 0; c < CPL; ++c) Q[c] = need ? x[c] >> SH | (GRID ? em[c] : 0u) : Q[c];
                        break;
                    }
                    if (wait.late(d)) return false;
                }
            }
            // exact columns go out with the seam's tag at every block's last row (whole lanes: a
            // window's side is ghost columns or the image's edge); the next phase's neighbours and
            // the backtrack blocks start from them.  Columns two strips share are stored twice with
            // the same value.
            const bool pub = (it.t == 0 || lane >= KR / CPL) && lane < rg && it.col0 < w;
            auto publish = [&](int v) {  // v: the row just done is v - 1
                const uint32_t krow = (uint32_t)((it.h ? hf[0].B : 0) + v / R - 1) * ckrow;
                if constexpr (EDGE) {
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        __builtin_amdgcn_raw_buffer_store_b32((Q[c] << SH) | tag, rck, (int)(em[c] ? kBufDrop : (uint32_t)(it.col0 + c) * 4u),
                                                              (int)krow, 0);
                } else {
                    const uint32_t ko = pub ? (uint32_t)it.col0 * 4u : kBufDrop;
                    if constexpr (CPL == 2) {
                        __builtin_amdgcn_raw_buffer_store_b64((v2u){(Q[0] << SH) | tag, (Q[1] << SH) | tag}, rck, (int)ko, (int)krow, 0);
                    } else {
#pragma unroll
                        for (int c = 0; c < CPL; c += 4)
                            buf_st128(rck, (v4u){(Q[c] << SH) | tag, (Q[c + 1] << SH) | tag, (Q[c + 2] << SH) | tag, (Q[c + 3] << SH) | tag},
                                      krow + ko + 4u * c);
                    }
                }
            };
            int v = __builtin_amdgcn_readfirstlane(it.v0);
            const int v1 = __builtin_amdgcn_readfirstlane(it.v1), v0 = v;
#pragma unroll 1
            while (v < v1) {
                // the next rows' scalar offsets first: a scalar written by the vector unit may not be
                // used as a buffer offset for some cycles
                const bool cross = v + PF >= v1;
                const uint32_t ro = cross ? roffn : roff;
                const uint32_t eo = cross ? nx.off : it.off;
                const int l0 = __builtin_amdgcn_readfirstlane(cross ? 0 : v + PF - it.v0);
#pragma unroll
                for (int g = 0; g < PF; g += 8) {
                    uint32_t so[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const bool own = LATE && g + i == 0;  // the current block's last row
                        so[i] = (uint32_t)__builtin_amdgcn_readlane(own ? roff : ro, own ? v - v0 + PF - 1 : l0 + g + i - LATE) & kGrid;
                    }
                    uint32_t sh[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) sh[i] = GRID ? (uint32_t)__builtin_amdgcn_readlane(odd, v - v0 + g + i) : 0u;
                    arrived(ring[g + 7 - LATE]);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int r = (g + i + PF - LATE) % PF;  // FWD: the row above's slot
                        if constexpr (FWD) forward_step<EDGE>(Q, left, right, ring[r], ring[g + i], em, last);
                        else cost_step<EDGE>(Q, left, right, ring[g + i], sh[i], em);
                        load_ev<TEAM, (int)CB * CPL / 2>(ring[r], re, so[i], LATE && g + i == 0 ? it.off : eo);
                        __builtin_amdgcn_sched_barrier(0);  // keep the prefetch PF rows ahead of its use
                    }
                }
                v += PF;
                if (v % R == 0) publish(v);
            }
            if (!more) return true;
            it = nx;
            roff = roffn;
            if constexpr (GRID) {
                odd = odd_of(roff);
                set_em();
            }
        }
    }
};

// ----------------------------------------------------------------------------------------------
// The carve engine: one image, carved by a team of G workgroups of NT threads.
template <int CPL, int KR, int NT, Kind KD = kEnergy>
struct Carver : Rows<block_rows(KR), KD> {
    static constexpr int R = block_rows(KR);  // rows of a backtrack block
    using Half = typename Rows<R, KD>::Half;
    using Rows<R, KD>::half_of;
    using Rows<R, KD>::energy_rsrc;
    using Rows<R, KD>::CB;
    using Rows<R, KD>::FWD;
    using Rows<R, KD>::MSK;
    using Rows<R, KD>::SH;
    using Rows<R, KD>::TAG;
    using Narrow = Sweep<CPL, KR, R, KD>;
    static constexpr bool HAS_WIDE = CPL == 4 && R == 32;
    using Wide = std::conditional_t<HAS_WIDE, Sweep<8, 32, 32, KD>, Narrow>;  // of the same blocks
    static constexpr int NW = NT / 64;      // waves per workgroup
    static constexpr int PB = CB == 4 ? R / 2 : R;   // rows of a backtrack block prefetched ahead
    static constexpr int BCPL = 4;            // columns per lane of a backtrack window
    static constexpr int BW = 64 * BCPL;      // columns of a backtrack window
    static constexpr int BS = BW - 2 * R;     // of which exact at the block's last row
    static constexpr int NG = R / 4;          // 4-row direction groups of a block
    static constexpr int BMAX = (kMaxRows / 2 + 4) / R + 2;  // blocks of half the tallest image
    static constexpr int CH = 496 / R + 1;    // hops per memory round trip: h * R + 15 < 512 for h < CH
    static_assert((PB == R || 2 * PB == R) && PB % 8 == 0, "whole prefetch groups");

    struct Smem {
        int jend[2 * BMAX];            // seam column at the last row of block b of half h at [h * BMAX + b]
        int2 pos[2];                   // per half: the block the backtrack has reached (-1: done), its column
        uint32_t cw[2][CH * 256];      // windows of ancestor offsets, 1024 bytes per hop
        uint32_t al[NW][64];           // ancestor offsets of the waves' windows (a lone workgroup's round)
        unsigned long long red[NW];
        int flag;
        int stop;                      // step mode: the time budget is spent
        Member me;                     // this workgroup's place in its team
        unsigned long long spent[3];   // the stage clocks of this call (its first member's first thread)
    };

    // ---- the middle (a4): the cheapest pair of T's and B's last rows, leftmost lower column, then
    // leftmost upper one (an image of one half: the leftmost minimum of T's last row).  Every
    // workgroup of a team finds it by itself.  Key: M << KC | lower column << 2 | (upper - lower + 1).
    static constexpr int KC = 18;
    template <bool TEAM>
    static __device__ __forceinline__ unsigned long long middle(const Img& d, Smem& sm, int w, int k) {
        constexpr int kC = TEAM ? 16 : 0;
        const Half h0 = half_of(d.H, d.mode, 0), h1 = half_of(d.H, d.mode, 1);
        const uint32_t ckrow = (uint32_t)d.xw * 4u;
        const __amdgpu_buffer_rsrc_t rck = make_rsrc(d.xq, (uint32_t)d.P * ckrow);
        const uint32_t t0 = (uint32_t)(h0.B - 1) * ckrow;
        // one half: row t0 stands in for the missing lower one, and counts nothing
        const uint32_t b0 = h1.n ? (uint32_t)(h0.B + h1.B - 1) * ckrow : t0, bm = h1.n ? ~0u : 0u;
        const uint32_t tag = seam_tag<KD>(k);
        unsigned long long best = ~0ull;
        for (int c0 = 4 * (int)threadIdx.x; c0 < w; c0 += 4 * NT) {
            uint32_t x[6], y[4];
            // FWD: what the lower column's diagonal parents add
            uint32_t dl[4] = {}, dr[4] = {};
            if constexpr (FWD) {
                if (bm) {
                    const __amdgpu_buffer_rsrc_t re = energy_rsrc(d), rro = make_rsrc(d.ro, (uint32_t)d.H * 4u);
                    const uint32_t ou = (uint32_t)__builtin_amdgcn_readfirstlane(Rows<R, KD>::template row_off<TEAM>(d, h0, 0, h0.B * R - 1, rro));
                    const uint32_t od = (uint32_t)__builtin_amdgcn_readfirstlane(Rows<R, KD>::template row_off<TEAM>(d, h1, 1, h1.B * R - 1, rro));
                    const v4u u = __builtin_amdgcn_raw_buffer_load_b128(re, c0 * 4, (int)ou, kC);
                    const v4u v = __builtin_amdgcn_raw_buffer_load_b128(re, c0 * 4, (int)od, kC);
                    const uint32_t vl = __builtin_amdgcn_raw_buffer_load_b32(re, c0 > 0 ? c0 * 4 - 4 : (int)kBufDrop, (int)od, kC);
                    const uint32_t vr = __builtin_amdgcn_raw_buffer_load_b32(re, c0 * 4 + 16, (int)od, kC);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        dl[c] = __builtin_amdgcn_sad_u8(u[c], c ? v[c - 1] : vl, 0u);
                        dr[c] = __builtin_amdgcn_sad_u8(u[c], c < 3 ? v[c + 1] : vr, 0u);
                    }
                }
            }
            Wait wait;
            for (;;) {
                const v4u T = __builtin_amdgcn_raw_buffer_load_b128(rck, c0 * 4, (int)t0, kC);
                const v4u B = __builtin_amdgcn_raw_buffer_load_b128(rck, c0 * 4, (int)b0, kC);
                x[0] = __builtin_amdgcn_raw_buffer_load_b32(rck, c0 > 0 ? c0 * 4 - 4 : (int)kBufDrop, (int)t0, kC);
                x[5] = __builtin_amdgcn_raw_buffer_load_b32(rck, c0 + 4 < w ? c0 * 4 + 16 : (int)kBufDrop, (int)t0, kC);
                bool ok = (c0 == 0 || (x[0] & TAG) == tag) && (c0 + 4 >= w || (x[5] & TAG) == tag);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    x[c + 1] = T[c];
                    y[c] = B[c];
                    ok = ok && (c0 + c >= w || ((T[c] & TAG) == tag && (B[c] & TAG) == tag));
                }
                if (!TEAM || ok || wait.late(d)) break;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (c0 + c >= w) continue;
                uint32_t m = x[c + 1] >> SH, dir = 1;
                if (bm) {
                    const uint32_t ml = (x[c] >> SH) + dl[c], mr = (x[c + 2] >> SH) + dr[c];
                    if (c0 + c > 0 && ml <= m) m = ml, dir = 0;
                    if (c0 + c + 1 < w && mr < m) m = mr, dir = 2;
                }
                best = min(best, (((unsigned long long)m + ((y[c] & bm) >> SH)) << KC) | (unsigned)((c0 + c) << 2) | dir);
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) best = min(best, (unsigned long long)__shfl_xor((long long)best, o, 64));
        if ((threadIdx.x & 63) == 0) sm.red[threadIdx.x >> 6] = best;
        __syncthreads();
        best = sm.red[0];
#pragma unroll
        for (int i = 1; i < NW; ++i) best = min(best, sm.red[i]);
        return best;
    }

    // ---- the backtrack (a5).  The cost sweep leaves the keys of every block's last row in ck; a
    // block's directions are computed again, for a window of columns, with keys M << 9 | u << 2 | tag:
    // the candidates get tags 0 / 1 / 2 (left, middle, right) and move u by the same, so one v_min3
    // picks the minimum, the leftmost tie and the ancestor's offset.  On return pk[g] holds the
    // directions of the block's rows 4g .. 4g+3 (a byte per row, 2 bits per column) and Q the keys of
    // its last row.  All blocks run at once, one wave each, where the path can still be.
    template <bool EDGE, bool COH>
    static __device__ __forceinline__ void trace_block(const Img& d, const Half& x, int h, int blk, int ckbase, int w,
                                                       int k, int base, int lane, uint32_t (&pk)[NG], uint32_t (&Q)[BCPL]) {
        const __amdgpu_buffer_rsrc_t re = energy_rsrc(d);
        const __amdgpu_buffer_rsrc_t rro = make_rsrc(d.ro, (uint32_t)d.H * 4u);
        const uint32_t ckrow = (uint32_t)d.xw * 4u;
        const __amdgpu_buffer_rsrc_t rck = make_rsrc(d.xq, (uint32_t)d.P * ckrow);
        const int col0 = base + lane * BCPL;
        // lane l < R: row l; the others: the row before the block (of zeros before the first one)
        const uint32_t roff = Rows<R, KD>::template row_off<COH>(d, x, h, blk * R + (lane < R ? lane : -1), rro);
        auto load_keys = [&]() {
            return __builtin_amdgcn_raw_buffer_load_b128(rck, blk > 0 && col0 < w ? col0 * 4 : (int)kBufDrop,
                                                         (int)((uint32_t)(ckbase + max(blk, 1) - 1) * ckrow), COH ? 16 : 0);
        };
        v4u kv = load_keys();
        const uint32_t eo = (uint32_t)(col0 < w ? col0 : 0) * CB;
        // Rows are passed over by as many as stay whole prefetches: eight where the ring holds the block, else
        // PB.  None for FWD: with the branch its 128 registers spill, and with a loop over the halves 1920 x 1080
        // takes 4 % longer (and 16 x 900 19 % less).
        constexpr int SKIP = PB == R ? 8 : FWD ? R : PB;
        const int none = __builtin_amdgcn_readfirstlane(blk == 0 ? x.pad : 0);
        const int first = SKIP == PB && none >= PB ? PB : 0;  // the ring's first row
        uint64_t ring[PB][CB == 4 ? 2 : 1];
#pragma unroll
        for (int i = 0; i < PB; ++i)
            load_ev<COH, (int)CB * BCPL / 2>(ring[i], re, (uint32_t)__builtin_amdgcn_readlane(roff, first + i), eo);
        uint32_t P[BCPL] = {};  // FWD: the pixels of the row above
        if constexpr (FWD) {
            uint64_t a[2];
            load_ev<COH, (int)CB * BCPL / 2>(a, re, (uint32_t)__builtin_amdgcn_readlane(roff, R), eo);
#pragma unroll
            for (int c = 0; c < BCPL; ++c) P[c] = (uint32_t)(a[c >> 1] >> ((c & 1) * 32));
        }
        // FWD adds to the keys of missing parents, so those are all ones only after that
        const uint32_t noL = lane == 0 ? ~0u : 0u;
        uint32_t noR[BCPL];
#pragma unroll
        for (int c = 0; c < BCPL; ++c) noR[c] = (EDGE && col0 + c + 1 >= w) || (lane == 63 && c == BCPL - 1) ? ~0u : 0u;
        bool valid[BCPL];
#pragma unroll
        for (int c = 0; c < BCPL; ++c) valid[c] = !EDGE || col0 + c < w;
        if (COH && blk > 0) {  // the strips' stores may still be on their way
            Wait wait;
            for (;;) {
                bool ok = true;
#pragma unroll
                for (int c = 0; c < BCPL; ++c) ok = ok && (!valid[c] || (kv[c] & TAG) == seam_tag<KD>(k));
                if (__all(ok) || wait.late(d)) break;
                kv = load_keys();
            }
        }
#pragma unroll
        for (int c = 0; c < BCPL; ++c) {
            Q[c] = valid[c] ? kv[c] & ~0x1FFu : QINF;
        }
        // masked: costs of 31 bits in words of their own, Q holds only offset and tag
        uint32_t M[BCPL], ml = ~0u, mr = ~0u;
        if constexpr (MSK) {
#pragma unroll
            for (int c = 0; c < BCPL; ++c) M[c] = valid[c] ? kv[c] >> SH : ~0u, Q[c] = 0;
        }
        uint32_t left = QINF, right = QINF, p = 0;
        auto row = [&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i % 8 == 0) arrived(ring[(i + 7) % PB]);
            uint32_t t[BCPL];
#pragma unroll
            for (int c = 0; c < BCPL; ++c) t[c] = Q[c] & ~3u;
            left = (uint32_t)__builtin_amdgcn_update_dpp((int)left, (int)t[BCPL - 1], 0x138, 0xf, 0xf, false);
            right = (uint32_t)__builtin_amdgcn_update_dpp((int)right, (int)(t[0] + 10u), 0x130, 0xf, 0xf, false);
            uint32_t acc = 0;
            if constexpr (FWD) {
                uint32_t px[BCPL];
#pragma unroll
                for (int c = 0; c < BCPL; ++c) px[c] = (uint32_t)(ring[i % PB][c >> 1] >> ((c & 1) * 32));
                const uint32_t pl = (uint32_t)__builtin_amdgcn_update_dpp((int)px[0], (int)px[BCPL - 1], 0x138, 0xf, 0xf, false);
                const uint32_t pr = (uint32_t)__builtin_amdgcn_update_dpp((int)px[BCPL - 1], (int)px[0], 0x130, 0xf, 0xf, false);
#pragma unroll
                for (int c = 0; c < BCPL; ++c) {
                    const uint32_t l = c ? px[c - 1] : pl;
                    uint32_t r = c + 1 < BCPL ? px[c + 1] : pr;
                    if (EDGE) r = noR[c] ? px[c] : r;
                    uint32_t a = (__builtin_amdgcn_sad_u8(P[c], l, 0u) << 9) + (c ? t[c - 1] : left);
                    uint32_t b = (__builtin_amdgcn_sad_u8(P[c], r, 0u) << 9) + (c + 1 < BCPL ? t[c + 1] + 10u : right);
                    if (c == 0) a |= noL;
                    if (EDGE || c == BCPL - 1) b |= noR[c];
                    const uint32_t m = min3u(a, t[c] + 5u, b);
                    Q[c] = (__builtin_amdgcn_sad_u8(l, r, 0u) << 9) + m;
                    if (EDGE) Q[c] = valid[c] ? Q[c] : QINF;
                    acc = __builtin_amdgcn_alignbit(m, acc, 2u);
                }
#pragma unroll
                for (int c = 0; c < BCPL; ++c) P[c] = px[c];
            } else if constexpr (MSK) {
                ml = (uint32_t)__builtin_amdgcn_update_dpp((int)ml, (int)M[BCPL - 1], 0x138, 0xf, 0xf, false);
                mr = (uint32_t)__builtin_amdgcn_update_dpp((int)mr, (int)M[0], 0x130, 0xf, 0xf, false);
                uint32_t n[BCPL];
#pragma unroll
                for (int c = 0; c < BCPL; ++c) {
                    const uint32_t a = c ? M[c - 1] : ml, b = c + 1 < BCPL ? M[c + 1] : mr;
                    const uint32_t m = min3u(a, M[c], b);
                    uint32_t q = M[c] == m ? t[c] + 5u : (c + 1 < BCPL ? t[c + 1] + 10u : right);
                    q = a == m ? (c ? t[c - 1] : left) : q;
                    n[c] = m + (uint32_t)(ring[i % PB][c >> 1] >> ((c & 1) * 32));
                    if (EDGE) n[c] = valid[c] ? n[c] : ~0u;
                    Q[c] = q;
                    acc = __builtin_amdgcn_alignbit(q, acc, 2u);
                }
#pragma unroll
                for (int c = 0; c < BCPL; ++c) M[c] = n[c];
            } else {
#pragma unroll
                for (int c = 0; c < BCPL; ++c) {
                    const uint32_t m = min(min(c ? t[c - 1] : left, t[c] + 5u), c + 1 < BCPL ? t[c + 1] + 10u : right);
                    const uint32_t pair = (uint32_t)(ring[i % PB][0] >> ((c >> 1) * 32));
                    Q[c] = (c & 1) ? mad_hi16(pair, m) : mad_lo16(pair, m);
                    if (EDGE) Q[c] = valid[c] ? Q[c] : QINF;
                    acc = __builtin_amdgcn_alignbit(m, acc, 2u);
                }
            }
            p = __builtin_amdgcn_perm(acc, p, 0x07030201u);  // this row's byte on top
            if constexpr (i % 4 == 3) pk[i / 4] = p;
            if constexpr (i + PB < R)
                load_ev<COH, (int)CB * BCPL / 2>(ring[i % PB], re, (uint32_t)__builtin_amdgcn_readlane(roff, i + PB), eo);
            __builtin_amdgcn_sched_barrier(0);
        };
        // Rows that do not exist (none of them) cost nothing and leave the keys at 0.
        static_for<R / SKIP>([&](auto Q) {
            constexpr int g = SKIP * decltype(Q)::value;
            if (SKIP < R && g + SKIP <= none) {
                static_for<SKIP / 4>([&](auto I) { pk[g / 4 + decltype(I)::value] = 0x55555555u; });  // (straight up)
            } else {
                static_for<SKIP>([&](auto I) { row(std::integral_constant<int, g + decltype(I)::value>{}); });
            }
        });
    }

    // Every direction of the map as bytes (one half, mode 2): windows dealt to the waves of the team.
    template <bool COH>
    static __device__ __forceinline__ void write_map(const Img& d, int w, int tw, int TW, int lane) {
        const Half x = half_of(d.H, d.mode, 0);
        const int nw = w <= BW ? 1 : (w - 2 * R + BS - 1) / BS;
        const __amdgpu_buffer_rsrc_t ro = make_rsrc(d.img, (uint32_t)d.H * (uint32_t)w);
        for (int q = tw; q < x.B * nw; q += TW) {
            const int blk = q / nw, j = q % nw, base = j * BS, col0 = base + lane * BCPL;
            uint32_t pk[NG], Q[BCPL];
            trace_block<true, COH>(d, x, 0, blk, 0, w, 0, base, lane, pk, Q);
            const bool own = (j == 0 || lane >= R / BCPL) && (j == nw - 1 || lane < 64 - R / BCPL);
            for (int i = 0; i < R; ++i) {
                const int y = blk * R + i - x.pad;
                if (y < 0) continue;
                uint32_t v = 0;
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    if (g == i / 4) v = pk[g];
                v = y ? v >> (8 * (i & 3)) : 0x55u;  // row 0 has no parent: 1
#pragma unroll
                for (int c = 0; c < BCPL; ++c)
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)((v >> (2 * c)) & 3u), ro,
                                                         (int)(own && col0 + c < w ? (uint32_t)(col0 + c) : kBufDrop),
                                                         (int)((uint32_t)y * (uint32_t)w), 0);
            }
        }
    }

    // The seam from its middle columns outward, written to d.seam (and seams_out).  Rounds: the
    // waves of the team are split over the halves still open and, in each, over the blocks from the
    // one the path has reached toward the border, with as many windows per block as there are
    // waves for, centred at the path's column; then every workgroup hops through the blocks' ancestor
    // offsets as far as the path stays inside the windows' exact columns, and the waves that hold a
    // block of the path walk it from their registers.  One round is enough unless the path drifts
    // out or the team has fewer waves than blocks.
    template <bool TEAM>
    static __device__ __forceinline__ bool backtrack(const Img& d, const CAS Img* gd, Smem& sm, int w, int k, int tw, int TW, int lane,
                                                     int G, unsigned& epoch, unsigned long long key) {
        const Half hf[2] = {half_of(d.H, d.mode, 0), half_of(d.H, d.mode, 1)};
        const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const __amdgpu_buffer_rsrc_t ranc = make_rsrc(d.anc, (uint32_t)d.P * (uint32_t)d.xw);
        int cB = min(max((int)((key & ((1ull << KC) - 1)) >> 2), 0), w - 1);
        int b[2], c[2];
        b[0] = hf[0].B - 1;
        b[1] = hf[1].B - 1;  // -1 when there is no lower half
        c[1] = cB;
        c[0] = min(max(cB + (int)(key & 3u) - 1, 0), w - 1);
        while (b[0] >= 0 || b[1] >= 0) {
            // the round's plan (the same in every wave of the team)
            const int nopen = (b[0] >= 0) + (b[1] >= 0);
            const int NWH = max(1, TW / nopen);
            int nblk[2], nwin[2], X0[2], ulo[2], uhi[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                nblk[h] = min(b[h] + 1, NWH);
                const int all = w <= BW ? 1 : (w - 2 * R + BS - 1) / BS;
                nwin[h] = nblk[h] > 0 ? min(all, NWH / nblk[h]) : 1;
                const int span = nwin[h] * BS + 2 * R;
                X0[h] = max(0, min(c[h] - span / 2, w - span));
                const int end = min(X0[h] + span, max(w, BW));
                ulo[h] = X0[h] == 0 ? 0 : X0[h] + R;
                uhi[h] = end >= w ? w : end - R;
            }
            const int h = nopen == 2 ? tw & 1 : (b[0] >= 0 ? 0 : 1);
            const int idx = nopen == 2 ? tw >> 1 : tw;
            const Half x = h ? hf[1] : hf[0];
            const int nw = h ? nwin[1] : nwin[0];
            const bool act = idx < (h ? nblk[1] : nblk[0]) * nw;
            const int blk = (h ? b[1] : b[0]) - idx / nw;
            const int base = min((h ? X0[1] : X0[0]) + (idx % nw) * BS, max(0, w - BW));
            const int elo = base == 0 ? 0 : base + R, ehi = base + BW >= w ? w : base + BW - R;
            uint32_t pk[NG];
            if (act) {
                uint32_t Q[BCPL];
                const int ckb = h ? hf[0].B : 0;
                if (base + BW > w) trace_block<true, TEAM>(d, x, h, blk, ckb, w, k, base, lane, pk, Q);
                else trace_block<false, TEAM>(d, x, h, blk, ckb, w, k, base, lane, pk, Q);
                // ancestor offsets of the exact columns (whole lanes; a lane past w - 1 writes into
                // the row's slack)
                const int col0 = base + lane * BCPL;
                const bool own = (base == 0 || lane >= R / BCPL) && (base + BW >= w || lane < 64 - R / BCPL) && col0 < w;
                uint32_t a = 0;
#pragma unroll
                for (int q = 0; q < BCPL; ++q) a |= (((Q[q] >> 2) & 127u) & 0xFFu) << (8 * q);
                if constexpr (TEAM)
                    __builtin_amdgcn_raw_buffer_store_b32(a, ranc, (int)(own ? (uint32_t)col0 : kBufDrop),
                                                          (int)((uint32_t)(ckb + blk) * (uint32_t)d.xw), 0);
                else
                    sm.al[wv][lane] = a;
            }
            if (!team_sync<TEAM>(gd, epoch, G, &sm.flag)) return false;
            // wave h hops through half h: a block's path column at its last row is within R columns of
            // the next block's, so a round trip loads the offsets of CH blocks at once (1 KB of
            // each row around the current column) and takes CH hops from LDS
            const int hh = wv & 1;
            if (wv < 2 && (hh ? b[1] : b[0]) >= 0) {
                const int ckb = hh ? hf[0].B : 0, lo = hh ? ulo[1] : ulo[0], hi = hh ? uhi[1] : uhi[0];
                uint32_t* cw = sm.cw[hh];
                int p = hh ? b[1] : b[0], j = hh ? c[1] : c[0];
                const int low = p - (hh ? nblk[1] : nblk[0]) + 1;
                if (lane == 0) sm.jend[hh * BMAX + p] = j;
                if constexpr (!TEAM) {
                    // the round's offsets are in LDS: block p's window j is wave (p0 - p) * nw + j of this half
                    const int p0 = p, X = hh ? X0[1] : X0[0], nwh = hh ? nwin[1] : nwin[0];
                    while (p > 0) {
                        const int win = min(max((j - X - R) / BS, 0), nwh - 1);
                        const int idx = (p0 - p) * nwh + win, wo = nopen == 2 ? 2 * idx + hh : idx;
                        const int bs = min(X + win * BS, max(0, w - BW));
                        const int a = reinterpret_cast<const uint8_t*>(sm.al[wo])[min(max(j - bs, 0), BW - 1)];
                        j = __builtin_amdgcn_readfirstlane(min(max(j + a - R, 0), w - 1));
                        --p;
                        if (p < low || j < lo || j >= hi) break;
                        if (lane == 0) sm.jend[hh * BMAX + p] = j;
                    }
                    if (p == 0 && p >= low && j >= lo && j < hi) p = -1;
                }
                for (bool run = TEAM; run;) {
                    const int j0 = j, p0 = p, m = min(CH, p - max(low, 1) + 1);
                    v4u v[CH];
                    // byte window [o, o + 1024) of every block's row, from a multiple of 16 at or below
                    // j0 - 512; what lies before the array is dropped
                    const int w0 = (j0 - 512) & ~15;
#pragma unroll
                    for (int i = 0; i < CH; ++i) {
                        const int bo = (ckb + p0 - i) * d.xw + w0 + 16 * lane;
                        v[i] = __builtin_amdgcn_raw_buffer_load_b128(ranc, (int)(i < m && bo >= 0 ? (uint32_t)bo : kBufDrop), 0, 16);
                    }
#pragma unroll
                    for (int i = 0; i < CH; ++i) *reinterpret_cast<v4u*>(cw + i * 256 + 4 * lane) = v[i];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    const uint8_t* cb = reinterpret_cast<const uint8_t*>(cw);
                    for (int i = 0; i < m; ++i) {
                        const int a = (int)(int8_t)cb[i * 1024 + min(max(j - w0, 0), 1023)];
                        j = __builtin_amdgcn_readfirstlane(min(max(j + a - R, 0), w - 1));
                        --p;
                        if (p < low || j < lo || j >= hi) {
                            run = false;
                            break;
                        }
                        if (lane == 0) sm.jend[hh * BMAX + p] = j;
                    }
                    if (run && p == 0) {
                        run = false;
                        p = -1;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
                if (lane == 0) sm.pos[hh] = make_int2(p, j);
            }
            __syncthreads();
            const int nb0 = b[0] >= 0 ? sm.pos[0].x : -1, nb1 = b[1] >= 0 ? sm.pos[1].x : -1;
            if (act && blk > (h ? nb1 : nb0)) {
                const int je = __builtin_amdgcn_readfirstlane(sm.jend[h * BMAX + blk]);
                if (je >= elo && je < ehi) {
                    int s = je - base, mys = 0;
                    static_for<R>([&](auto I) {
                        constexpr int i = R - 1 - decltype(I)::value;
                        mys = lane == i ? s : mys;
                        if constexpr (i > 0) {
                            const uint32_t wd = (uint32_t)__builtin_amdgcn_readlane((int)pk[i / 4], s >> 2);
                            s += (int)((wd >> ((i & 3) * 8 + (s & 3) * 2)) & 3u) - 1;
                        }
                    });
                    const int y = blk * R + lane - x.pad;
                    if (lane < R && y >= 0) {
                        const int r = h ? d.H - 1 - y : y;
                        const int col = min(max(base + mys, 0), w - 1);
                        *gp(d.seam + r) = (int32_t)((uint32_t)col | seam_word(k));
                        if (d.seams_out) *gp(d.seams_out + (size_t)k * d.H + r) = col;
                    }
                }
            }
            if (b[0] >= 0) b[0] = nb0, c[0] = sm.pos[0].y;
            if (b[1] >= 0) b[1] = nb1, c[1] = sm.pos[1].y;
        }
        return true;
    }

    // ---- removal (a6) of rows [ra, rb): the shorter side of a row moves (pixels right of the seam one
    // column left, or pixels left of it one column right with the row's start offset advanced by one;
    // without min-side removal always the right side).  A row is only ever written by the wave owning
    // it, so plain loads see its current bytes even in a team.
    template <bool TEAM>
    static __device__ __forceinline__ void remove_rows(const Img& d, int w, int k, int ra, int rb, int lane) {
        const __amdgpu_buffer_rsrc_t rsm = make_rsrc(d.seam, (uint32_t)d.H * 4u);
        const __amdgpu_buffer_rsrc_t rro = make_rsrc(d.ro, (uint32_t)d.H * 4u);
        for (int row = ra; row < rb; row += 64) {
            // no branch on a lane's row here: the compiler would carry the row through it in vector
            // registers, take the planes' descriptors for lane dependent and loop over the lanes at every access
            const int rc = __builtin_amdgcn_readfirstlane(row);
            const int n = __builtin_amdgcn_readfirstlane(min(64, rb - row));
            const uint32_t mine = lane < n ? (uint32_t)(rc + lane) * 4u : kBufDrop;
            const int o = (int)buf_ld32<false>(rro, mine);
            uint32_t word;
            Wait wait;
            for (;;) {  // the rows' walkers may still be at it
                word = buf_ld32<TEAM>(rsm, mine);
                if (!TEAM || __all(lane >= n || (word & 0xFFFF0000u) == seam_word(k)) || wait.late(d)) break;
            }
            const int s = min((int)(word & 0xFFFFu), w - 1);
            const bool right = d.minside && s < w - 1 - s;
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(o + 1), rro, (int)(right ? mine : kBufDrop), 0, 0);
            if constexpr (FWD) {
                const ShiftPlane planes[1] = {shift_plane(d.wk + (size_t)rc * d.wp, n, (uint32_t)d.wp, 4)};
                shift_rows<4, 1>(planes, n, w, s, o, right, (d.minside ? w / 2 : w) * 4, lane);
            } else {
                const ShiftPlane planes[2] = {shift_plane(d.wk + (size_t)rc * d.wp, n, (uint32_t)d.wp, d.C),
                                              shift_plane(d.e + (size_t)rc * d.ep, n, (uint32_t)d.ep * 2u, (int)CB)};
                shift_rows<3, 2>(planes, n, w, s, o, right, (d.minside ? w / 2 : w) * max(d.C, (int)CB), lane);
            }
        }
    }

    // Seams k_begin .. k_end-1 of one image (the image has W - k_begin columns on entry).  With a
    // deadline (device wall clock) it stops after the first seam that ends past it.  Returns the
    // number of seams removed in total (k_begin + the seams of this call).
    template <bool TEAM, bool MAP>
    static __device__ __forceinline__ int carve_seams(const CAS Img* gd, int rank, int G, Smem& sm, int k_begin, int k_end,
                                                      unsigned& epoch, unsigned long long deadline) {
        const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        // waves are numbered across the team first, so a phase's strips land on different compute
        // units (one DP wave per SIMD) before any workgroup takes a second one
        const int TW = G * NW, tw = wv * G + rank;
        const int H = gd->H, W = gd->W, mode = gd->mode;
        const int rpw = (H + TW - 1) / TW;
        const int ra = min(H, tw * rpw), rb = min(H, ra + rpw);  // rows this wave owns
        GAS Ctl* ctl = gp(reinterpret_cast<Ctl*>(gd->bar));
        const bool timer = rank == 0 && threadIdx.x == 0;  // one clock reader per image
        // The stage clocks run in LDS: in registers they would be alive through the stages they measure
        // (512 thumbnails up to 250 x 250: 2.61 ms with them there, 2.50 so).  A stage gets the time it ends
        // added and the time it begins taken away, so nothing is read either (forward energy, 1920 x 1080:
        // 65.9 us per seam with the last stamp read back, 65.7 so).
        const auto stamp = [&](int stage) {  // `stage` ends and the next one begins
            if (!timer) return;
            const unsigned long long now = wall_clock64();
            if (stage >= 0) __hip_atomic_fetch_add(&sm.spent[stage], now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (stage < 2) __hip_atomic_fetch_add(&sm.spent[stage + 1], 0ull - now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        if (timer) sm.spent[0] = sm.spent[1] = sm.spent[2] = 0;
        // masked pixels left in the image (kMasked: the carve ends with the last of them)
        int left = 0;
        if constexpr (MSK) left = (int)__hip_atomic_load(&ctl->left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned bias = masked_bias(H, gd->C);
        for (int k = k_begin; k < k_end; ++k) {
            if (MSK && left <= 0) {
                k_end = k;
                break;
            }
            const int w = W - k;
            stamp(-1);
            {
                const Img d = fetch(gd);
                // (a wave that gives up waiting flags the image; the others then give up at once)
                // Wide strips (eight columns per lane) where the waves are too few for one narrow strip
                // each: their ghost columns are a sixteenth of the window on each side against a quarter.
                // The 256-image batch by one workgroup per image takes 426 ms so and 515 ms with narrow
                // strips alone; with a wave for every narrow strip those are faster (1920 x 1080 by 32
                // workgroups: 27 us per sweep against 50).
                if (w < Narrow::WIN && Narrow::strips(w) == 1) Narrow::template cost_sweep<true, TEAM>(d, w, k, tw, TW, lane);
                else if (!HAS_WIDE || 2 * Narrow::strips(w) <= TW || w <= Wide::WINR) Narrow::template cost_sweep<false, TEAM>(d, w, k, tw, TW, lane);
                else Wide::template cost_sweep<false, TEAM>(d, w, k, tw, TW, lane);
            }
            if (MSK) stamp(0);
            // (a team's waves go on to wait for the tags of what they need)
            if constexpr (!TEAM) __syncthreads();
            {
                const Img d = fetch(gd);
                const unsigned long long key = middle<TEAM>(d, sm, w, k);
                long long cost = (long long)(key >> KC);
                if constexpr (MSK) {  // the pixels outside the mask pay the bias here, those inside get it
                    const int out = (int)(cost / bias);
                    left -= H - out;
                    cost -= (long long)H * bias;
                }
                if (rank == 0 && threadIdx.x == 0 && d.costs_out) *gp(d.costs_out + k) = cost;
                if (!MSK) stamp(0);
                if constexpr (MAP) {
                    if (mode == 2) write_map<TEAM>(d, w, tw, TW, lane);
                }
                if (!backtrack<TEAM>(d, gd, sm, w, k, tw, TW, lane, G, epoch, key)) return k;
            }
            if (mode) break;
            if constexpr (!TEAM) __syncthreads();
            if (MSK) stamp(1);
            remove_rows<TEAM>(fetch(gd), w, k, ra, rb, lane);
            if (!team_sync<TEAM>(gd, epoch, G, &sm.flag)) return k;
            if (!MSK) stamp(1);
            if constexpr (!FWD) {
                const Img d = fetch(gd);
                // ---- band energy (a2): only the new columns s-1 and s of each row changed.  Buffer
                // loads (sc1 in a team: the rows above and below were shifted by other workgroups) at
                // 32-bit offsets; a lane past the wave's rows reads row ra and stores nothing.
                const int w2 = w - 1;
                const __amdgpu_buffer_rsrc_t rwk = make_rsrc(d.wk, (uint32_t)H * (uint32_t)d.wp);
                const __amdgpu_buffer_rsrc_t rsm = make_rsrc(d.seam, (uint32_t)H * 4u);
                const __amdgpu_buffer_rsrc_t rof = make_rsrc(d.ro, (uint32_t)H * 4u);
                for (int rc = ra; rc < rb; rc += 64) {
                    const int r = rc + lane < rb ? rc + lane : ra;
                    const int ru = r > 0 ? r - 1 : 0, rd = r + 1 < H ? r + 1 : H - 1;
                    const int s = min((int)(buf_ld32<TEAM>(rsm, (uint32_t)r * 4u) & 0xFFFFu), w - 1);
                    const int o = (int)buf_ld32<TEAM>(rof, (uint32_t)r * 4u);
                    const uint32_t br = (uint32_t)r * (uint32_t)d.wp + (uint32_t)(o * d.C);
                    const uint32_t bu = (uint32_t)ru * (uint32_t)d.wp + buf_ld32<TEAM>(rof, (uint32_t)ru * 4u) * (uint32_t)d.C;
                    const uint32_t bd = (uint32_t)rd * (uint32_t)d.wp + buf_ld32<TEAM>(rof, (uint32_t)rd * 4u) * (uint32_t)d.C;
                    const uint32_t e0 = energy_buf<TEAM>(rwk, br, bu, bd, w2, d.C, s - 1);
                    const uint32_t e1 = energy_buf<TEAM>(rwk, br, bu, bd, w2, d.C, s);
                    if (rc + lane < rb) {
                        if constexpr (MSK) {
                            uint32_t* er = reinterpret_cast<uint32_t*>(d.e + (size_t)r * d.ep) + o;
                            if (s - 1 >= 0 && s - 1 < w2) *gp(er + s - 1) = e0 + (*gp(er + s - 1) >= bias ? bias : 0u);
                            if (s < w2) *gp(er + s) = e1 + (*gp(er + s) >= bias ? bias : 0u);
                        } else {
                            uint16_t* er = d.e + (size_t)r * d.ep + o;
                            if (s - 1 >= 0 && s - 1 < w2) *gp(er + s - 1) = (uint16_t)e0;
                            if (s < w2) *gp(er + s) = (uint16_t)e1;
                        }
                    }
                }
            }
            // a team's time budget: its first member decides before the seam's last barrier, every
            // member reads the decision after it
            const bool timed = deadline && G > 1 && k + 1 < k_end;
            if (timed && rank == 0 && threadIdx.x == 0 && wall_clock64() >= deadline) stop_after<DevMem>(&ctl->stop, k);
            if (!FWD && !team_sync<TEAM>(gd, epoch, G, &sm.flag)) return k;
            if (timed && stops_after<DevMem>(&ctl->stop, k)) k_end = k + 1;
            stamp(2);
            if (deadline && G == 1 && k + 1 < k_end) {  // one decision for the whole workgroup
                if (threadIdx.x == 0) sm.stop = wall_clock64() >= deadline;
                __syncthreads();
                const int stop = sm.stop;
                __syncthreads();
                if (stop) k_end = k + 1;
            }
        }
        // ---- after the last seam, the carved rows go from wk (each from its start offset) to img
        const Img d = fetch(gd);
        if (!mode && (MSK || k_end == W - d.target_w) && k_end > k_begin) {
            const int nb = (W - k_end) * d.C;
            for (int rc = ra; rc < rb; rc += 64) {
                const int n = min(64, rb - rc);
                const int rof = lane < n ? *gp(d.ro + rc + lane) : 0;
#pragma unroll 1
                for (int i = 0; i < n; ++i) {
                    const int o = __builtin_amdgcn_readlane(rof, i);
                    if constexpr (FWD) {  // the low C bytes of each pixel's dword
                        const uint32_t* src = reinterpret_cast<const uint32_t*>(d.wk + (long long)(rc + i) * d.wp) + o;
                        uint8_t* dst = d.img + (long long)(rc + i) * d.pitch;
                        // (eight loads in flight; one by one they are most of a carve of a single seam: 16447 x 8192
                        // 14.9 ms, 5.7 so)
                        for (int x0 = 0; x0 < d.target_w; x0 += 512) {
                            uint32_t px[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) px[u] = *gp(src + min(x0 + 64 * u + lane, d.target_w - 1));
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                const int x = x0 + 64 * u + lane;
                                if (x >= d.target_w) continue;
                                for (int c = 0; c < d.C; ++c) *gp(dst + (long long)x * d.C + c) = (uint8_t)(px[u] >> (8 * c));
                            }
                        }
                        continue;
                    }
                    copy_bytes_wave(d.img + (long long)(rc + i) * d.pitch, d.wk + (long long)(rc + i) * d.wp + (long long)o * d.C,
                                    nb, lane);
                }
            }
            team_sync<TEAM>(gd, epoch, G, &sm.flag);
        }
        if (MSK && rank == 0 && threadIdx.x == 0) ctl->left = (unsigned)left;
        return k_end;
    }

    // Carve one image, or (max_seams > 0) continue it by at most max_seams seams.  rank, G: this
    // workgroup's place in the team that the launch means; join: the word by which those that come form
    // one (0 at the launch; used with G > 1 only).  sm.me keeps the place taken (first_member).
    template <bool MAP = false>
    static __device__ __forceinline__ void carve_image(const CAS Img* gd, int rank, int G, GAS unsigned long long* join, Smem& sm,
                                                       int max_seams, unsigned long long deadline = 0) {
        const Img d = fetch(gd);
        GAS Ctl* ctl = gp(reinterpret_cast<Ctl*>(d.bar));
        const int nseams = d.mode ? 1 : d.W - d.target_w;
        if (G > 1) {  // (first: a workgroup that comes late must not read what its team is changing)
            if (threadIdx.x == 0) {
                const unsigned long long now = wall_clock64();
                sm.me = join_team<DevMem, DevClock>(join, (int)xcc_id(), G,
                                                    team_patience(max_seams > 0 ? min(nseams, max_seams) : nseams,
                                                                  deadline > now ? deadline - now : 0ull));
            }
            __syncthreads();
            rank = __builtin_amdgcn_readfirstlane(sm.me.rank);
            G = __builtin_amdgcn_readfirstlane(sm.me.size);
            if (rank < 0) return;
            // a team spread over several XCDs would not see each other's stores through sc1 loads, so
            // such an image is flagged instead of carved
            if (__builtin_amdgcn_readfirstlane((int)sm.me.apart)) {
                if (rank == 0 && threadIdx.x == 0)
                    __hip_atomic_fetch_or(gp(d.status), kStatusPlacement, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
        }
        const int k0 = max_seams > 0 ? (int)ctl->done : 0;
        const int k1 = max_seams > 0 ? min(nseams, k0 + max_seams) : nseams;
        if (k0 >= k1) return;
        if (rank == 0 && threadIdx.x == 0 && k0 == 0) ctl->t_begin = wall_clock64();
        // a call that continues a carve (step mode) starts from the barrier count the previous
        // calls left behind, so a team's barrier counter never has to be reset between launches
        unsigned epoch = max_seams > 0 ? __hip_atomic_load(&ctl->ebase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        const int kd = G > 1 ? carve_seams<true, MAP>(gd, rank, G, sm, k0, k1, epoch, deadline)
                             : carve_seams<false, MAP>(gd, 0, 1, sm, k0, k1, epoch, deadline);  // seams removed in total
        __syncthreads();
        if (rank == 0 && threadIdx.x == 0) {
            if (MSK || kd == nseams) ctl->t_end = wall_clock64();
            if (!d.mode && !ctl->status)  // (else a stage has begun and not ended)
                for (int i = 0; i < 3; ++i) ctl->t_stage[i] += sm.spent[i];
            if (max_seams > 0) leave_call(ctl, kd, epoch);  // every member ended this call at the same barrier count
            else ctl->done = (unsigned)kd;
        }
    }

    // After carve_image with the same G: whether this thread speaks for the team.
    static __device__ __forceinline__ bool first_member(const Smem& sm, int G) {
        return threadIdx.x == 0 && (G == 1 || sm.me.rank == 0);
    }
};

}  // namespace sc
