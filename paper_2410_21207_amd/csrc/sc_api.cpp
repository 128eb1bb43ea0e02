// C ABI of libseamcarve: argument validation, workspace layout, batch planning, launches.
// Declarations and the meaning of every argument: include/sc.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <numeric>
#include <vector>

#include "../../include/sc.h"
#include "sc_internal.h"

namespace {

thread_local char g_err[512] = "";

sc_status fail(sc_status code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

sc_status ok() {
    g_err[0] = 0;
    return SC_OK;
}

sc_status hip_fail(hipError_t e, const char* what) {
    return fail(SC_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// Workspace header: the first 256 bytes of every workspace, then one Ctl per image.
struct WsHead {
    uint32_t magic;
    int32_t n;
    uint32_t pad[62];
};
constexpr uint32_t kMagic = sc::kWsMagic;
static_assert(sizeof(WsHead) == sc::kWsHeadBytes, "header size");
static_assert(sizeof(sc::Ctl) == 128, "ctl size");
static_assert(sc::kWsImgOffset + sizeof(sc::Img) <= sc::kWsHeadBytes, "a single image's descriptor fits the header");

constexpr int kMaxCostBound = 8388000;  // H*510*C: the column cost must fit 23 bits
constexpr int kMaxTeamSingle = 16;      // largest team a single image gets without a tuned one
static_assert(sc::kObjMaxTeam >= kMaxTeamSingle, "the object kernel's grid holds every team");
constexpr int kDefaultTeamBatch = 16;   // largest team for one image of a batch

sc_status check_image(int H, int W, int C, int pitch) {
    if (H < 1 || W < 1) return fail(SC_EINVAL, "H=%d W=%d must be >= 1", H, W);
    if (C < 1 || C > 4) return fail(SC_EINVAL, "C=%d must be in 1..4", C);
    if ((long long)pitch < (long long)W * C) return fail(SC_EINVAL, "pitch=%d < W*C=%lld", pitch, (long long)W * C);
    if (W > 65535) return fail(SC_EUNSUPPORTED, "W=%d > 65535", W);
    if ((long long)H * 510 * C > kMaxCostBound)
        return fail(SC_EUNSUPPORTED, "H*510*C=%lld exceeds %d (23-bit cumulative cost)", (long long)H * 510 * C,
                    kMaxCostBound);
    return SC_OK;
}

size_t ctl_region(int n) { return sc::align_up(sizeof(WsHead) + (size_t)n * sizeof(sc::Ctl), sc::kAlign); }

// Fill the device descriptor of one image whose scratch starts at `base` and whose Ctl is `ctl`.
sc::Img make_img(const uint8_t* src, uint8_t* img, int H, int W, int C, long long pitch, int target_w,
                 int32_t* seams_out, int64_t* costs_out, char* base, sc::Ctl* ctl, int kr, int G, int mode) {
    const sc::Layout L = sc::layout_for(H, W, C);
    sc::Img d;
    memset(&d, 0, sizeof(d));
    d.src = src;
    d.img = img;
    d.pitch = pitch;
    d.H = H;
    d.W = W;
    d.C = C;
    d.target_w = target_w;
    d.seams_out = seams_out;
    d.costs_out = reinterpret_cast<long long*>(costs_out);
    d.e = reinterpret_cast<uint16_t*>(base + L.e);
    d.P = sc::key_rows(H, kr, mode);
    d.xw = sc::key_pitch(W);
    d.anc = reinterpret_cast<int8_t*>(base + L.scratch);
    d.xq = reinterpret_cast<uint32_t*>(base + L.scratch + sc::align_up((size_t)d.P * d.xw, sc::kAlign));
    d.seam = reinterpret_cast<int32_t*>(base + L.seam);
    d.ro = reinterpret_cast<int32_t*>(base + L.ro);
    d.wk = reinterpret_cast<uint8_t*>(base + L.wk);
    d.wp = L.wp;
    d.minside = 1;
    d.bar = &ctl->bar;
    d.status = &ctl->status;
    d.ep = L.ep;
    d.G = G;
    d.mode = mode;
    return d;
}

int resolve_variant(const sc_tune* t) {
    if (t && t->variant >= 0) return t->variant < sc::variant_count() ? t->variant : -1;
    return sc::default_variant();
}

// Microseconds one seam of an H x w image takes a team of G workgroups of nw waves: the sweep from
// both ends (by strips of 128 columns, or of 448 where those are more than the waves), the walk
// back over blocks of rows, the removal and the band of new energies.  Fitted to 25 sizes from 64 x 64 to
// 2100 x 2100 with six team sizes each on an idle MI355X; the team it ranks first is within 6 % of
// the fastest there, and within 10 % for flat images of 1 to 33 rows and up to 8000 columns.  Forward
// energy takes up to a third more or less and ranks the teams the same way.
double seam_us(int H, int w, int G, int nw) {
    const int tw = G * nw;
    const auto strips = [](int cols, int win, int step) { return cols <= win ? 1 : (cols - win + step - 1) / step + 1; };
    const bool flat = H <= sc::kFlatRows;  // swept as one block
    const double rows = flat ? sc::kFlatRows : H / 2 + 16;
    const int n4 = (flat ? 1 : 2) * strips(w, 256, 128), n8 = (flat ? 1 : 2) * strips(w, 504, 448);
    const double sweep = n4 <= tw || w <= 504
                             ? rows * (0.047 + (n4 > 2 ? 0.0085 * std::max(0.0, (double)n4 / G - 2) : 0.0))
                             : rows * (0.045 + 0.0175 * n8 / G);
    const int each = (H + tw - 1) / tw, blocks = 2 * ((H + 63) / 64);
    const double back = 4.5 + 4.8 * ((blocks + tw - 1) / tw - 1);
    const double remove = 2.5 + each * (0.085 + (w <= 138 ? 0.2 : 0.45 + std::max(0, w - 600) * 0.00037));
    return sweep + back + remove + (G > 1 ? 5.5 + 0.0012 * H + 0.002 * std::min(w, 2100) : std::min(3.5, 0.006 * w));
}

constexpr int kTeamSizes[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};

// The team of a single image: the smallest that seam_us puts within 3 % of the fastest one, at most 16
// (forward energy at 1920 x 1080: 67.0 us per seam, 66.4 with 32; 3840 x 2160 and its transpose: 121 ms,
// 101 with 32).  Single images all go to one XCD unless the caller names another, and it holds 64 workgroups: four streams
// find room for a whole team of 16 each.  A team that does not find it carves with the workgroups that
// came (join_team).
int single_team(int H, int w, int nw) {
    double best = 1e30;
    for (int g : kTeamSizes)
        if (g <= kMaxTeamSingle) best = std::min(best, seam_us(H, w, g, nw));
    for (int g : kTeamSizes)
        if (seam_us(H, w, g, nw) <= 1.03 * best) return g;
    return 1;
}

// A launch plan of a batch: the workgroups of every image and the order of the blocks.
struct BatchPlan {
    std::vector<int> team;               // workgroups per job
    std::vector<int2> blk, teams;        // block -> (team, member), team -> (first of team_imgs, count)
    std::vector<int> team_imgs;
    double us = 0;                       // the time the plan should take
};

// The plan in which image i has a team of kTeamSizes[pick[i]], which carves it in t[i * nsizes + pick[i]]
// microseconds.  Teams come first, largest first and each on the XCD with the most free
// workgroups, so that all of them are resident at once; the images of one workgroup follow, longest
// first, each on the XCD (block index mod 8) that is free earliest.
//
// Teams may take every slot that the occupancy query reports.  That many are resident: over 17,920 teams of
// batches that fill 384 to 512 of the 512 slots, e1 and forward, none was short of a member and all of a launch
// began within 11 us (forward; 72 us e1).  A team that is short, with other streams' work on the device,
// carves with those that came.  Keeping a third free took 256 forward images from 196 to 204 ms.
BatchPlan place_batch(const std::vector<double>& t, const std::vector<int>& pick, int n, int per_xcd) {
    constexpr int ns = sizeof(kTeamSizes) / sizeof(kTeamSizes[0]);
    BatchPlan p;
    p.team.resize(n);
    std::vector<double> us(n);
    std::vector<int> order(n);
    std::iota(order.begin(), order.end(), 0);
    for (int i = 0; i < n; ++i) {
        p.team[i] = kTeamSizes[pick[i]];
        us[i] = t[i * ns + pick[i]];
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return p.team[a] != p.team[b] ? p.team[a] > p.team[b] : us[a] > us[b];
    });
    std::vector<int2> col[8];             // the blocks of each XCD
    std::vector<double> busy[8];          // when each of its workgroup slots is free: min-heaps
    size_t first_single = 0;
    for (; first_single < (size_t)n && p.team[order[first_single]] > 1; ++first_single) {
        const int i = order[first_single];
        int x = 0;
        for (int c = 1; c < 8; ++c)
            if (col[c].size() < col[x].size()) x = c;
        if ((int)col[x].size() + p.team[i] > per_xcd) {  // no room for a resident team
            p.team[i] = 1;
            us[i] = t[i * ns];
            continue;
        }
        for (int r = 0; r < p.team[i]; ++r) {
            col[x].push_back(make_int2((int)p.teams.size(), r));
            busy[x].push_back(us[i]);
        }
        p.teams.push_back(make_int2((int)p.team_imgs.size(), 1));
        p.team_imgs.push_back(i);
        p.us = std::max(p.us, us[i]);
    }
    order.erase(std::remove_if(order.begin(), order.end(), [&](int i) { return p.team[i] > 1; }), order.end());
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return us[a] > us[b]; });
    for (auto& h : busy) {
        h.resize(per_xcd, 0.0);
        std::make_heap(h.begin(), h.end(), std::greater<double>());
    }
    for (int i : order) {
        int x = 0;
        for (int c = 1; c < 8; ++c)
            if (busy[c][0] < busy[x][0] || (busy[c][0] == busy[x][0] && col[c].size() < col[x].size())) x = c;
        std::pop_heap(busy[x].begin(), busy[x].end(), std::greater<double>());
        busy[x].back() += us[i];
        p.us = std::max(p.us, busy[x].back());
        std::push_heap(busy[x].begin(), busy[x].end(), std::greater<double>());
        col[x].push_back(make_int2((int)p.teams.size(), 0));
        p.teams.push_back(make_int2((int)p.team_imgs.size(), 1));
        p.team_imgs.push_back(i);
    }
    size_t rows = 0;
    for (const auto& c : col) rows = std::max(rows, c.size());
    for (size_t r = 0; r < rows; ++r)
        for (const auto& c : col) p.blk.push_back(r < c.size() ? c[r] : make_int2(-1, -1));
    while (!p.blk.empty() && p.blk.back().x < 0) p.blk.pop_back();
    return p;
}

// The plan whose limit gives the shortest estimated time.  max_team bounds the teams; the image with
// the longest chain alone may have twice that.  Teams sized by an image's share of the pixels instead fill
// every slot, and the images of one workgroup only begin when the teams end: 256 images up to
// 2000 x 2000 took 204 ms that way and take 170 ms here, 512 thumbnails up to 250 x 250 took 3.3 ms and take 2.7.
// (All the images at once wait for memory, so they take 2 to 3 times the estimate; the order of the
// plans holds: limits of 0.8, 1.1, 1.6 and 2 times the chosen one took 205, 185, 185 and 203 ms.)
BatchPlan plan_batch(const sc_job* jobs, int n, int max_team, int per_xcd, int nw) {
    constexpr int ns = sizeof(kTeamSizes) / sizeof(kTeamSizes[0]);
    std::vector<double> t((size_t)n * ns);
    std::vector<int> cap(n, std::min(max_team, per_xcd));
    double longest = 0, shortest = 0;
    int crit = 0;
    const auto time = [&](int i, int g) {
        const int k = jobs[i].W - jobs[i].target_w;
        t[i * ns + g] = k * seam_us(jobs[i].H, jobs[i].W - k / 2, kTeamSizes[g], nw);
    };
    for (int i = 0; i < n; ++i) {
        double best = 1e30;
        for (int g = 0; g < ns && kTeamSizes[g] <= cap[i]; ++g) {
            time(i, g);
            best = std::min(best, t[i * ns + g]);
        }
        if (t[i * ns] > longest) longest = t[i * ns], crit = i;
        shortest = std::max(shortest, best);
    }
    if (max_team > 1 && n > 1) cap[crit] = std::min(std::min(2 * max_team, 32), per_xcd);
    for (int g = 0; g < ns && kTeamSizes[g] <= cap[crit]; ++g) time(crit, g);
    // Every image gets the smallest team that carves it within the limit, or the one that carves it
    // fastest.  A plan takes as long as its longest image, and as its work spread over all slots: limits
    // are tried in the order of that bound (of equal plans the larger limit's) up to the best plan's time, and one that
    // changes no team is dropped.  With every limit placed, 256 images of 240 to 2160 took 0.62 ms to plan and take
    // 0.30; 2000 of 16 to 60, 2.1 and 0.77.
    struct Try {
        double bound;
        std::vector<int> pick;
    };
    std::vector<Try> tries;
    for (double limit = longest; tries.empty() || limit > 0.3 * shortest; limit *= 0.85) {
        Try next{0, std::vector<int>(n)};
        double work = 0;
        for (int i = 0; i < n; ++i) {
            int p = 0;
            for (int g = 0; g < ns && kTeamSizes[g] <= cap[i]; ++g) {
                if (t[i * ns + g] < t[i * ns + p]) p = g;
                if (t[i * ns + p] <= limit) break;
            }
            next.pick[i] = p;
            next.bound = std::max(next.bound, t[i * ns + p]);
            work += kTeamSizes[p] * t[i * ns + p];
        }
        next.bound = std::max(next.bound, work / (8 * per_xcd));
        if (tries.empty() || next.pick != tries.back().pick) tries.push_back(std::move(next));
    }
    std::vector<int> order(tries.size());
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return tries[a].bound < tries[b].bound; });
    BatchPlan best;
    int from = -1;
    for (int i : order) {
        if (from >= 0 && tries[i].bound > best.us) break;
        BatchPlan p = place_batch(t, tries[i].pick, n, per_xcd);
        if (from < 0 || p.us < best.us || (p.us == best.us && i < from)) best = std::move(p), from = i;
    }
    return best;
}

}  // namespace

namespace sc {

Layout layout_for(int H, int W, int C) {
    Layout L;
    L.ep = (int)align_up((size_t)W + 8, 64);
    size_t off = 64;  // the row shifter may write up to 16 bytes below a plane
    L.ctl = 0;
    L.e = off;
    off = align_up(off + (size_t)(H + 1) * L.ep * 2, kAlign);  // and a row of zeros
    // the backtrack's scratch: ancestor offsets and published keys, 5 * key_rows * key_pitch bytes
    L.scratch = off;
    const size_t rows = std::max(key_rows(H, 48, 0), key_rows(H, 48, 2));  // of 24, the smallest blocks
    off = align_up(off + rows * key_pitch(W), kAlign);
    off = align_up(off + rows * key_pitch(W) * 4, kAlign);
    L.seam = off;
    off = align_up(off + (size_t)H * 4, kAlign);
    L.ro = off;
    off = align_up(off + (size_t)H * 4, kAlign);
    // working image: 16 bytes between rows and below the first one (the row shifter's last slot may
    // run over a row's end)
    L.wp = (int)align_up((size_t)W * C + 16, 16);
    L.wk = off + 64;
    off += 64;
    off = align_up(off + (size_t)H * L.wp, kAlign);
    L.total = off + kAlign;  // slack: row copies read a few bytes past the last row
    return L;
}

}  // namespace sc

extern "C" {

const char* sc_last_error(void) { return g_err; }

const char* sc_version(void) { return "seamcarve-mi355x 0.1 (gfx950)"; }

int sc_variant_count(void) { return sc::variant_count(); }

const char* sc_variant_name(int v) {
    if (v < 0 || v >= sc::variant_count()) return "";
    return sc::variant(v).name;
}

size_t sc_workspace_bytes(int H, int W, int C) {
    if (H < 1 || W < 1 || C < 1 || C > 4) return 0;
    return ctl_region(1) + sc::layout_for(H, W, C).total;
}

sc_status sc_energy(const uint8_t* img, int H, int W, int C, int pitch, int32_t* energy, void* stream) {
    sc_status s = check_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    if (!img || !energy) return fail(SC_EINVAL, "null pointer");
    hipError_t e = sc::launch_energy_i32(img, H, W, C, pitch, energy, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "energy launch");
    return ok();
}

sc_status sc_dp_seam(const int32_t* energy, int H, int W, int32_t* seam, int64_t* cost, void* ws, size_t ws_bytes,
                     void* stream, uint8_t* dirs_out) {
    sc_status s = check_image(H, W, 1, W);
    if (s != SC_OK) return s;
    if (!energy || !seam || !cost || !ws) return fail(SC_EINVAL, "null pointer");
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    const size_t need = sc_workspace_bytes(H, W, 1);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);
    const int v = sc::default_variant();
    const int G = single_team(H, W, sc::variant(v).threads / 64);
    char* base = static_cast<char*>(ws);
    sc::Ctl* ctl = reinterpret_cast<sc::Ctl*>(base + sizeof(WsHead));
    // with dirs_out the sweep runs down over all rows (mode 2) and writes the map itself
    sc::Img d = make_img(nullptr, dirs_out, H, W, 1, W, W > 1 ? W - 1 : 1, seam, cost, base + ctl_region(1), ctl,
                         sc::variant(v).kr, G, dirs_out ? 2 : 1);
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = sc::launch_prepare_from_i32(d, energy, st);
    if (e == hipSuccess) e = sc::launch_carve_single(d, v, G, 0, st);
    if (e != hipSuccess) return hip_fail(e, "dp launch");
    return ok();
}

sc_status sc_remove_seam(uint8_t* img, int H, int W, int C, int pitch, const int32_t* seam, void* stream) {
    sc_status s = check_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    if (!img || !seam) return fail(SC_EINVAL, "null pointer");
    hipError_t e = sc::launch_remove_seam(img, H, W, C, pitch, seam, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "remove launch");
    return ok();
}

sc_status sc_transpose_u8(const uint8_t* src, int H, int W, int C, int src_pitch, uint8_t* dst, int dst_pitch,
                          void* stream) {
    if (H < 1 || W < 1 || C < 1 || C > 4) return fail(SC_EINVAL, "bad shape H=%d W=%d C=%d", H, W, C);
    if ((long long)src_pitch < (long long)W * C || (long long)dst_pitch < (long long)H * C)
        return fail(SC_EINVAL, "pitch too small");
    if (!src || !dst) return fail(SC_EINVAL, "null pointer");
    const uintptr_t s0 = (uintptr_t)src, s1 = s0 + (size_t)(H - 1) * src_pitch + (size_t)W * C;
    const uintptr_t d0 = (uintptr_t)dst, d1 = d0 + (size_t)(W - 1) * dst_pitch + (size_t)H * C;
    if (s0 < d1 && d0 < s1) return fail(SC_EINVAL, "src and dst overlap");
    hipError_t e = sc::launch_transpose(src, H, W, C, src_pitch, dst, dst_pitch, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "transpose launch");
    return ok();
}

sc_status sc_carve(uint8_t* img, int H, int W, int C, int target_w, int pitch, int32_t* seams_out, int64_t* costs_out,
                   void* ws, size_t ws_bytes, void* stream, const uint8_t* src, const sc_tune* tune) {
    sc_status s = check_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    if (!img || !ws) return fail(SC_EINVAL, "null pointer");
    if (target_w < 1 || target_w > W) return fail(SC_EINVAL, "target_w=%d not in [1, W=%d]", target_w, W);
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    const size_t need = sc_workspace_bytes(H, W, C);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);
    const int v = resolve_variant(tune);
    if (v < 0) return fail(SC_EINVAL, "unknown kernel variant %d", tune->variant);
    const int G = tune && tune->team > 0 ? tune->team : single_team(H, W - (W - target_w) / 2, sc::variant(v).threads / 64);
    if (G > 32) return fail(SC_EUNSUPPORTED, "team of %d workgroups > 32", G);
    char* base = static_cast<char*>(ws);
    sc::Ctl* ctl = reinterpret_cast<sc::Ctl*>(base + sizeof(WsHead));
    sc::Img d = make_img(src, img, H, W, C, pitch, target_w, seams_out, costs_out, base + ctl_region(1), ctl,
                         sc::variant(v).kr, G, 0);
    if (tune && (tune->flags & SC_TUNE_NO_MINSIDE)) d.minside = 0;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = sc::launch_prepare_single(d, st);
    const int xcd = tune ? (tune->flags >> SC_TUNE_XCD_SHIFT) & 7 : 0;
    if (e == hipSuccess && target_w < W) e = sc::launch_carve_single(d, v, G, xcd, st);
    if (e != hipSuccess) return hip_fail(e, "carve launch");
    return ok();
}

// sc_carve with its scratch in the library's fixed per-GPU device array instead of a caller's
// workspace: same validation, same kernels, no allocation of any kind.
sc_status sc_carve_noalloc(uint8_t* img, int H, int W, int C, int target_w, int pitch, int32_t* seams_out,
                           int64_t* costs_out, uint32_t* status_out, void* stream, const uint8_t* src,
                           const sc_tune* tune) {
    static_assert(sc::kNoAllocScratchBytes == (size_t)SC_NOALLOC_SCRATCH_BYTES, "scratch size");
    sc_status s = check_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    const size_t need = sc_workspace_bytes(H, W, C);
    if (need > sc::kNoAllocScratchBytes)
        return fail(SC_ENOMEM, "a %dx%dx%d image needs %zu bytes of scratch; the fixed scratch holds %zu", H, W, C,
                    need, sc::kNoAllocScratchBytes);
    if (!img) return fail(SC_EINVAL, "null pointer");
    if (target_w < 1 || target_w > W) return fail(SC_EINVAL, "target_w=%d not in [1, W=%d]", target_w, W);
    void* ws = nullptr;
    hipError_t e = sc::noalloc_scratch(&ws);
    if (e != hipSuccess) return hip_fail(e, "scratch address");
    s = sc_carve(img, H, W, C, target_w, pitch, seams_out, costs_out, ws, sc::kNoAllocScratchBytes, stream, src,
                 tune);
    if (s != SC_OK) return s;
    if (status_out) {
        const sc::Ctl* ctl = reinterpret_cast<const sc::Ctl*>(static_cast<const char*>(ws) + sizeof(WsHead));
        e = sc::launch_copy_status(&ctl->status, status_out, (hipStream_t)stream);
        if (e != hipSuccess) return hip_fail(e, "status copy");
    }
    return ok();
}

namespace {
// Workspace of sc_insert_seams: the carve's own workspace, a scratch image the carve writes, the
// seams in removal coordinates and in original columns.
struct InsertLayout {
    size_t carve, scratch, cur, orig, total;
};

InsertLayout insert_layout(int H, int W, int C, int pitch, int k) {
    InsertLayout L;
    size_t off = 0;
    L.carve = off;
    off = sc::align_up(off + sc_workspace_bytes(H, W, C), sc::kAlign);
    L.scratch = off;
    off = sc::align_up(off + (size_t)H * pitch, sc::kAlign);
    L.cur = off;
    off = sc::align_up(off + (size_t)std::max(k, 1) * H * 4, sc::kAlign);
    L.orig = off;
    off = sc::align_up(off + (size_t)std::max(k, 1) * H * 4, sc::kAlign);
    L.total = off;
    return L;
}
}  // namespace

size_t sc_insert_workspace_bytes(int H, int W, int C, int pitch, int k) {
    if (H < 1 || W < 1 || C < 1 || C > 4 || pitch < W * C || k < 0 || k >= W) return 0;
    return insert_layout(H, W, C, pitch, k).total;
}

sc_status sc_insert_seams(const uint8_t* img, int H, int W, int C, int pitch, int k, uint8_t* out, int out_pitch,
                          int32_t* seams_out, const sc_tune* tune, void* ws, size_t ws_bytes, void* stream) {
    sc_status s = check_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    if (!img || !out || !ws) return fail(SC_EINVAL, "null pointer");
    if (k < 0 || k >= W) return fail(SC_EINVAL, "k=%d not in [0, W=%d)", k, W);
    if (W > sc::kInsertMaxWidth) return fail(SC_EUNSUPPORTED, "W=%d > %d", W, sc::kInsertMaxWidth);
    if ((long long)out_pitch < (long long)(W + k) * C)
        return fail(SC_EINVAL, "out_pitch=%d < (W + k) * C = %lld", out_pitch, (long long)(W + k) * C);
    const uintptr_t a0 = (uintptr_t)img, a1 = a0 + (size_t)(H - 1) * pitch + (size_t)W * C;
    const uintptr_t b0 = (uintptr_t)out, b1 = b0 + (size_t)(H - 1) * out_pitch + (size_t)(W + k) * C;
    if (a0 < b1 && b0 < a1) return fail(SC_EINVAL, "out overlaps img");
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    const InsertLayout L = insert_layout(H, W, C, pitch, k);
    if (ws_bytes < L.total) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, L.total);
    char* base = static_cast<char*>(ws);
    int32_t* orig = seams_out ? seams_out : reinterpret_cast<int32_t*>(base + L.orig);
    hipStream_t st = (hipStream_t)stream;
    if (k > 0) {
        // the seams: carve a copy (img is the source and stays unmodified), recording each seam
        s = sc_carve(reinterpret_cast<uint8_t*>(base + L.scratch), H, W, C, W - k, pitch,
                     reinterpret_cast<int32_t*>(base + L.cur), nullptr, base + L.carve, sc_workspace_bytes(H, W, C),
                     stream, img, tune);
        if (s != SC_OK) return s;
        hipError_t e = sc::launch_seam_origins(reinterpret_cast<const int32_t*>(base + L.cur), k, H, W,
                                               nullptr, orig, st);
        if (e != hipSuccess) return hip_fail(e, "seam origins launch");
    }
    hipError_t e = sc::launch_insert_seams(img, H, W, C, pitch, k, orig, out, out_pitch, st);
    if (e != hipSuccess) return hip_fail(e, "insert launch");
    return ok();
}

size_t sc_batch_workspace_bytes(const sc_job* jobs, int n) {
    if (!jobs || n < 1) return 0;
    size_t total = ctl_region(n);
    total += sc::align_up((size_t)n * sizeof(sc::Img), sc::kAlign);
    // plan arrays: blocks (<= 8 * n * 32 int2), teams (n int2), team images (n int)
    total += sc::align_up((size_t)8 * 32 * n * sizeof(int2), sc::kAlign);
    total += sc::align_up((size_t)n * sizeof(int2), sc::kAlign);
    total += sc::align_up((size_t)n * sizeof(int), sc::kAlign);
    for (int i = 0; i < n; ++i) {
        if (jobs[i].H < 1 || jobs[i].W < 1) return 0;
        total += sc::layout_for(jobs[i].H, jobs[i].W, jobs[i].C).total;
    }
    return total;
}

sc_status sc_batch_prepare(const sc_job* jobs, int n, const sc_tune* tune, void* ws, size_t ws_bytes,
                           sc_batch_info* info) {
    if (!jobs || n < 1 || !ws || !info) return fail(SC_EINVAL, "null pointer or n < 1");
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    for (int i = 0; i < n; ++i) {
        const sc_job& j = jobs[i];
        sc_status s = check_image(j.H, j.W, j.C, j.pitch);
        if (s != SC_OK) return fail(s, "job %d: %s", i, g_err);
        if (!j.img) return fail(SC_EINVAL, "job %d: null image", i);
        if (j.target_w < 1 || j.target_w > j.W) return fail(SC_EINVAL, "job %d: target_w=%d not in [1, %d]", i,
                                                            j.target_w, j.W);
    }
    const size_t need = sc_batch_workspace_bytes(jobs, n);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);
    const int v = resolve_variant(tune);
    if (v < 0) return fail(SC_EINVAL, "unknown kernel variant %d", tune->variant);
    int G = tune && tune->team > 0 ? tune->team : kDefaultTeamBatch;
    if (G > 32) return fail(SC_EUNSUPPORTED, "team of %d workgroups > 32", G);

    int dev = 0, ncu = 0;
    hipError_t he = hipGetDevice(&dev);
    if (he == hipSuccess) he = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (he != hipSuccess) return hip_fail(he, "device query");
    const int per_xcd = std::max(1, sc::carve_blocks_per_cu(v) * ncu / 8);
    const BatchPlan plan = plan_batch(jobs, n, G, per_xcd, sc::variant(v).threads / 64);
    const std::vector<int>& gsz = plan.team;
    const std::vector<int2>&blk = plan.blk, &teams = plan.teams;
    const std::vector<int>& team_imgs = plan.team_imgs;

    // host image of the plan region
    const size_t off_imgs = ctl_region(n);
    const size_t off_blk = off_imgs + sc::align_up((size_t)n * sizeof(sc::Img), sc::kAlign);
    const size_t off_teams = off_blk + sc::align_up((size_t)8 * 32 * n * sizeof(int2), sc::kAlign);
    const size_t off_ti = off_teams + sc::align_up((size_t)n * sizeof(int2), sc::kAlign);
    size_t off_data = off_ti + sc::align_up((size_t)n * sizeof(int), sc::kAlign);
    if (blk.size() > (size_t)8 * 32 * n) return fail(SC_EUNSUPPORTED, "plan too large");
    int teams_used = 0;
    for (int i = 0; i < n; ++i) teams_used += gsz[i] > 1;
    std::vector<char> host(off_data, 0);
    WsHead* h = reinterpret_cast<WsHead*>(host.data());
    h->magic = kMagic;
    h->n = n;
    char* base = static_cast<char*>(ws);
    sc::Img* imgs = reinterpret_cast<sc::Img*>(host.data() + off_imgs);
    int max_rows = 1;
    for (int i = 0; i < n; ++i) {
        const sc_job& j = jobs[i];
        sc::Ctl* ctl = reinterpret_cast<sc::Ctl*>(base + sizeof(WsHead)) + i;
        imgs[i] = make_img(j.src, j.img, j.H, j.W, j.C, j.pitch, j.target_w, j.seams_out, j.costs_out,
                           base + off_data, ctl, sc::variant(v).kr, gsz[i], 0);
        if (tune && (tune->flags & SC_TUNE_NO_MINSIDE)) imgs[i].minside = 0;
        off_data += sc::layout_for(j.H, j.W, j.C).total;
        max_rows = std::max(max_rows, j.H);
    }
    memcpy(host.data() + off_blk, blk.data(), blk.size() * sizeof(int2));
    memcpy(host.data() + off_teams, teams.data(), teams.size() * sizeof(int2));
    memcpy(host.data() + off_ti, team_imgs.data(), team_imgs.size() * sizeof(int));
    hipError_t e = hipMemcpy(ws, host.data(), host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "plan upload");

    memset(info, 0, sizeof(*info));
    info->n = n;
    info->nblocks = (int)blk.size();
    info->variant = v;
    info->max_rows = max_rows;
    info->team = G;
    info->teams_used = teams_used;
    info->off_imgs = off_imgs;
    info->off_blk = off_blk;
    info->off_teams = off_teams;
    info->off_team_imgs = off_ti;
    return ok();
}

static sc_status batch_pass(const sc_batch_info* info, void* ws, void* stream, bool energy, bool carve) {
    if (!info || !ws || info->n < 1 || info->nblocks < 1 || info->team < 1) return fail(SC_EINVAL, "bad batch info");
    char* base = static_cast<char*>(ws);
    hipStream_t st = (hipStream_t)stream;
    const sc::Img* imgs = reinterpret_cast<const sc::Img*>(base + info->off_imgs);
    hipError_t e = hipSuccess;
    if (energy) e = sc::launch_prepare_batch(imgs, info->n, info->max_rows, st);
    if (e == hipSuccess && carve)
        e = sc::launch_carve_batch(imgs, reinterpret_cast<const int2*>(base + info->off_blk),
                                   reinterpret_cast<const int2*>(base + info->off_teams),
                                   reinterpret_cast<const int*>(base + info->off_team_imgs), info->nblocks,
                                   info->variant, st);
    if (e != hipSuccess) return hip_fail(e, "batch launch");
    return ok();
}

sc_status sc_batch_launch(const sc_batch_info* info, void* ws, void* stream) {
    return batch_pass(info, ws, stream, true, true);
}

sc_status sc_batch_launch_energy(const sc_batch_info* info, void* ws, void* stream) {
    return batch_pass(info, ws, stream, true, false);
}

sc_status sc_batch_launch_carve(const sc_batch_info* info, void* ws, void* stream) {
    return batch_pass(info, ws, stream, false, true);
}

sc_status sc_carve_batch(const sc_job* jobs, int n, const sc_tune* tune, void* ws, size_t ws_bytes, void* stream) {
    sc_batch_info info;
    sc_status s = sc_batch_prepare(jobs, n, tune, ws, ws_bytes, &info);
    if (s != SC_OK) return s;
    return sc_batch_launch(&info, ws, stream);
}

int sc_read_status(const void* ws, uint32_t* flags, int max_n) {
    if (!ws || !flags || max_n < 1) {
        fail(SC_EINVAL, "bad arguments");
        return -1;
    }
    if (hipDeviceSynchronize() != hipSuccess) {
        fail(SC_EHIP, "device synchronize failed");
        return -1;
    }
    // the head and the first image's flags in one copy: all of them for a single image
    struct {
        WsHead h;
        sc::Ctl c;
    } first;
    static_assert(sizeof(first) == sizeof(WsHead) + sizeof(sc::Ctl), "no gap");
    if (hipMemcpy(&first, ws, sizeof(first), hipMemcpyDeviceToHost) != hipSuccess || first.h.magic != kMagic ||
        first.h.n < 1) {
        fail(SC_EINVAL, "not a prepared workspace");
        return -1;
    }
    const int n = std::min(first.h.n, max_n);
    flags[0] = first.c.status;
    std::vector<sc::Ctl> c(n - 1);
    if (n > 1 && hipMemcpy(c.data(), static_cast<const char*>(ws) + sizeof(first), (n - 1) * sizeof(sc::Ctl),
                           hipMemcpyDeviceToHost) != hipSuccess) {
        fail(SC_EHIP, "status copy failed");
        return -1;
    }
    for (int i = 1; i < n; ++i) flags[i] = c[i - 1].status;
    ok();
    return n;
}

}  // extern "C"

extern "C" int sc_read_times(const void* ws, uint64_t* t_begin, uint64_t* t_end, int max_n, double* hz) {
    if (!ws || !t_begin || !t_end || max_n < 1) {
        fail(SC_EINVAL, "bad arguments");
        return -1;
    }
    if (hipDeviceSynchronize() != hipSuccess) {
        fail(SC_EHIP, "device synchronize failed");
        return -1;
    }
    WsHead h;
    if (hipMemcpy(&h, ws, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess || h.magic != kMagic || h.n < 1) {
        fail(SC_EINVAL, "not a prepared workspace");
        return -1;
    }
    const int n = std::min(h.n, max_n);
    std::vector<sc::Ctl> c(n);
    if (hipMemcpy(c.data(), static_cast<const char*>(ws) + sizeof(WsHead), n * sizeof(sc::Ctl),
                  hipMemcpyDeviceToHost) != hipSuccess) {
        fail(SC_EHIP, "times copy failed");
        return -1;
    }
    for (int i = 0; i < n; ++i) {
        t_begin[i] = c[i].t_begin;
        t_end[i] = c[i].t_end;
    }
    if (hz) {
        int dev = 0, khz = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) == hipSuccess && khz > 0)
            *hz = khz * 1000.0;
        else
            *hz = 100e6;
    }
    ok();
    return n;
}

extern "C" int sc_read_stages(const void* ws, uint64_t* stages, int max_n) {
    if (!ws || !stages || max_n < 1) {
        fail(SC_EINVAL, "bad arguments");
        return -1;
    }
    if (hipDeviceSynchronize() != hipSuccess) {
        fail(SC_EHIP, "device synchronize failed");
        return -1;
    }
    WsHead h;
    if (hipMemcpy(&h, ws, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess || h.magic != kMagic || h.n < 1) {
        fail(SC_EINVAL, "not a prepared workspace");
        return -1;
    }
    const int n = std::min(h.n, max_n);
    std::vector<sc::Ctl> c(n);
    if (hipMemcpy(c.data(), static_cast<const char*>(ws) + sizeof(WsHead), n * sizeof(sc::Ctl),
                  hipMemcpyDeviceToHost) != hipSuccess) {
        fail(SC_EHIP, "stages copy failed");
        return -1;
    }
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < 3; ++j) stages[3 * i + j] = c[i].t_stage[j];
    ok();
    return n;
}

// ---------------------------------------------------------------------------------- serving slots
constexpr size_t kSlotBytes = sizeof(sc::Img);  // the table is a device array of descriptors
constexpr int kMaxSlotTeam = 32;                // workgroups of one slot's team in a step

// The table: the slots' descriptors, then room for the block plan of a step with teams (teams
// laid out per XCD, then one block per slot).
size_t slot_plan_offset(int n_slots) { return sc::align_up((size_t)n_slots * kSlotBytes, sc::kAlign); }
size_t slot_plan_capacity(int n_slots) { return (size_t)8 * kMaxSlotTeam * n_slots + n_slots; }

extern "C" size_t sc_slot_table_bytes(int n_slots) {
    if (n_slots < 1) return 0;
    return slot_plan_offset(n_slots) + sc::align_up(slot_plan_capacity(n_slots) * sizeof(int4), sc::kAlign);
}

extern "C" sc_status sc_slot_start(const sc_job* job, void* ws, size_t ws_bytes, void* table, int n_slots, int slot,
                                   void* stream) {
    if (!job || !ws || !table) return fail(SC_EINVAL, "null pointer");
    if (n_slots < 1 || slot < 0 || slot >= n_slots) return fail(SC_EINVAL, "slot %d not in [0, %d)", slot, n_slots);
    sc_status s = check_image(job->H, job->W, job->C, job->pitch);
    if (s != SC_OK) return s;
    if (!job->img) return fail(SC_EINVAL, "null image");
    if (job->target_w < 1 || job->target_w > job->W)
        return fail(SC_EINVAL, "target_w=%d not in [1, W=%d]", job->target_w, job->W);
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    const size_t need = sc_workspace_bytes(job->H, job->W, job->C);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);
    const int v = sc::default_variant();
    char* base = static_cast<char*>(ws);
    sc::Ctl* ctl = reinterpret_cast<sc::Ctl*>(base + sizeof(WsHead));
    sc::Img d = make_img(job->src, job->img, job->H, job->W, job->C, job->pitch, job->target_w, job->seams_out,
                         job->costs_out, base + ctl_region(1), ctl, sc::variant(v).kr, 1, 0);
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = sc::launch_prepare_single(d, st);
    if (e == hipSuccess) e = sc::launch_slot_write(static_cast<sc::Img*>(table), slot, d, st);
    if (e != hipSuccess) return hip_fail(e, "slot start");
    return ok();
}

extern "C" sc_status sc_slot_clear(void* table, int n_slots, int slot, void* stream) {
    if (!table) return fail(SC_EINVAL, "null table");
    if (n_slots < 1 || slot < 0 || slot >= n_slots) return fail(SC_EINVAL, "slot %d not in [0, %d)", slot, n_slots);
    sc::Img d;
    memset(&d, 0, sizeof(d));
    hipError_t e = sc::launch_slot_write(static_cast<sc::Img*>(table), slot, d, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "slot clear");
    return ok();
}

extern "C" sc_status sc_slots_step(const void* table, int n_slots, int max_seams, int32_t* progress, void* stream) {
    return sc_slots_step_timed(table, n_slots, max_seams, 0, progress, stream);
}

extern "C" sc_status sc_slots_step_timed(const void* table, int n_slots, int max_seams, long long budget_us,
                                         int32_t* progress, void* stream) {
    if (!table || n_slots < 1 || max_seams < 1 || budget_us < 0) return fail(SC_EINVAL, "bad slot step arguments");
    // the device wall clock runs at 100 MHz: 100 ticks per microsecond
    hipError_t e = sc::launch_carve_steps(static_cast<const sc::Img*>(table), n_slots, sc::default_variant(),
                                          max_seams, (unsigned long long)budget_us * 100ull, progress, nullptr, 0,
                                          (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "slot step");
    return ok();
}

extern "C" sc_status sc_slots_step_teams(const void* table, int table_slots, int n_slots, const int32_t* team,
                                         int max_seams, long long budget_us, int32_t* progress, void* stream) {
    if (!table || !team || n_slots < 1 || max_seams < 1 || budget_us < 0)
        return fail(SC_EINVAL, "bad slot step arguments");
    if (table_slots < n_slots) return fail(SC_EINVAL, "n_slots=%d > table_slots=%d", n_slots, table_slots);
    const int v = sc::default_variant();
    int dev = 0, ncu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, "device query");
    // Teams first in the grid, each on one XCD, with room for all of them at once (a team goes without
    // the members that come late); a team that finds no room carves with one workgroup.  Then one
    // block per remaining slot (those need no company and may wait for a free slot of the device).
    const int per_xcd = std::max(1, sc::carve_blocks_per_cu(v) * ncu / 8 * 3 / 4);
    std::vector<int> order;
    for (int s = 0; s < n_slots; ++s)
        if (team[s] > 1) order.push_back(s);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return team[a] > team[b]; });
    int used[8] = {0};
    std::vector<int4> plan;
    std::vector<char> single(n_slots, 1);
    for (int s : order) {
        const int G = std::min(team[s], kMaxSlotTeam);
        int x = 0;
        for (int c = 1; c < 8; ++c)
            if (used[c] < used[x]) x = c;
        if (used[x] + G > per_xcd) continue;
        for (int r = 0; r < G; ++r) {
            const size_t b = (size_t)x + 8 * (size_t)(used[x] + r);
            if (plan.size() <= b) plan.resize(b + 1, make_int4(-1, 0, 0, 0));
            plan[b] = make_int4(s, r | G << 16, 0, 0);
        }
        used[x] += G;
        single[s] = 0;
    }
    for (int s = 0; s < n_slots; ++s)
        if (single[s]) plan.push_back(make_int4(s, 1 << 16, 0, 0));
    if (plan.size() > slot_plan_capacity(table_slots)) return fail(SC_EUNSUPPORTED, "step plan too large");
    hipStream_t st = (hipStream_t)stream;
    char* base = static_cast<char*>(const_cast<void*>(table));
    // the plan goes after the descriptors of every slot of the table, so no descriptor is touched
    int4* dplan = reinterpret_cast<int4*>(base + slot_plan_offset(table_slots));
    e = hipMemcpyAsync(dplan, plan.data(), plan.size() * sizeof(int4), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = sc::launch_carve_steps(static_cast<const sc::Img*>(table), n_slots, v, max_seams,
                                   (unsigned long long)budget_us * 100ull, progress, dplan, (int)plan.size(), st);
    if (e != hipSuccess) return hip_fail(e, "slot step");
    return ok();
}

// ---------------------------------------------------------------------------------------------
// Forward energy (sec. "Forward Energy Calculation"): the carve engine on a dword per working pixel,
// no energy plane.
namespace {

struct FwdLayout {
    size_t anc, xq, seam, ro, wk, total;
    int wp, xw, P;
};

FwdLayout fwd_layout(int H, int W, int C) {
    (void)C;
    FwdLayout L;
    L.P = sc::key_rows(H, sc::kFwdKR, 0);
    L.wp = (int)sc::align_up((size_t)W * 4 + 16, 16);  // 16 bytes between rows: the row shifter's last slot
    L.xw = sc::key_pitch(W);
    size_t off = 0;
    L.anc = off;
    off = sc::align_up(off + (size_t)L.P * L.xw, sc::kAlign);
    L.xq = off;
    off = sc::align_up(off + (size_t)L.P * L.xw * 4, sc::kAlign);
    L.seam = off;
    off = sc::align_up(off + (size_t)H * 4, sc::kAlign);
    L.ro = off;
    off = sc::align_up(off + (size_t)H * 4, sc::kAlign);
    L.wk = off + 64;  // the row shifter may write up to 16 bytes below a plane
    off = sc::align_up(L.wk + (size_t)(H + 1) * L.wp + 64, sc::kAlign);  // and a row of zeros
    L.total = off;
    return L;
}

sc_status check_fwd_image(int H, int W, int C, int pitch) {
    sc_status s = check_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    if (W > sc::kFwdMaxW) return fail(SC_EUNSUPPORTED, "W=%d > %d (forward energy)", W, sc::kFwdMaxW);
    if (H > sc::kFwdMaxH) return fail(SC_EUNSUPPORTED, "H=%d > %d (forward energy)", H, sc::kFwdMaxH);
    if ((long long)H * (long long)sc::align_up((size_t)W * 4, 64) + (long long)sc::kFwdSlack >= (1ll << 31))
        return fail(SC_EUNSUPPORTED, "image of %lld pixels too large for the forward-energy path", (long long)H * W);
    return SC_OK;
}

int fwd_units(int W) { return W <= sc::kFwdUnitFirst ? 1 : (W + sc::kFwdUnitCols - 1) / sc::kFwdUnitCols; }

sc::Img make_fwd_img(const uint8_t* src, uint8_t* img, int H, int W, int C, long long pitch, int target_w,
                     int32_t* seams_out, int64_t* costs_out, char* base, sc::Ctl* ctl, int G) {
    const FwdLayout L = fwd_layout(H, W, C);
    sc::Img d;
    memset(&d, 0, sizeof(d));
    d.src = src;
    d.img = img;
    d.pitch = pitch;
    d.H = H;
    d.W = W;
    d.C = C;
    d.target_w = target_w;
    d.seams_out = seams_out;
    d.costs_out = reinterpret_cast<long long*>(costs_out);
    d.anc = reinterpret_cast<int8_t*>(base + L.anc);
    d.xq = reinterpret_cast<uint32_t*>(base + L.xq);
    d.xw = L.xw;
    d.seam = reinterpret_cast<int32_t*>(base + L.seam);
    d.ro = reinterpret_cast<int32_t*>(base + L.ro);
    d.wk = reinterpret_cast<uint8_t*>(base + L.wk);
    d.wp = L.wp;
    d.e = reinterpret_cast<uint16_t*>(d.wk);
    d.ep = L.wp / 2;
    d.minside = 1;
    d.P = L.P;
    d.bar = &ctl->bar;
    d.status = &ctl->status;
    d.G = G;
    return d;
}

}  // namespace

extern "C" size_t sc_forward_workspace_bytes(int H, int W, int C) {
    if (H < 1 || W < 1 || C < 1 || C > 4) return 0;
    return ctl_region(1) + sc::align_up(sizeof(sc::Img), sc::kAlign) + fwd_layout(H, W, C).total;
}

extern "C" sc_status sc_carve_forward(uint8_t* img, int H, int W, int C, int target_w, int pitch, int32_t* seams_out,
                                      int64_t* costs_out, void* ws, size_t ws_bytes, void* stream, const uint8_t* src) {
    sc_status s = check_fwd_image(H, W, C, pitch);
    if (s != SC_OK) return s;
    if (!img || !ws) return fail(SC_EINVAL, "null pointer");
    if (target_w < 1 || target_w > W) return fail(SC_EINVAL, "target_w=%d not in [1, W=%d]", target_w, W);
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    const size_t need = sc_forward_workspace_bytes(H, W, C);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);
    char* base = static_cast<char*>(ws);
    sc::Ctl* ctl = reinterpret_cast<sc::Ctl*>(base + sizeof(WsHead));
    const size_t off_img = ctl_region(1);
    const int G = single_team(H, W - (W - target_w) / 2, sc::kFwdThreads / 64);
    const sc::Img d = make_fwd_img(src, img, H, W, C, pitch, target_w, seams_out, costs_out,
                                   base + off_img + sc::align_up(sizeof(sc::Img), sc::kAlign), ctl, G);
    // header (magic, one image) and the descriptor, which the kernels read from the workspace
    WsHead h;
    memset(&h, 0, sizeof(h));
    h.magic = kMagic;
    h.n = 1;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(base, &h, sizeof(h), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(base + off_img, &d, sizeof(d), hipMemcpyHostToDevice, st);
    const sc::Img* dd = reinterpret_cast<const sc::Img*>(base + off_img);
    if (e == hipSuccess) e = sc::launch_fwt_prepare(dd, 1, H, st);
    if (e == hipSuccess && target_w < W) e = sc::launch_fwt_carve(dd, nullptr, 8 * G, 0, st);
    if (e != hipSuccess) return hip_fail(e, "forward carve launch");
    return ok();
}

extern "C" size_t sc_forward_batch_workspace_bytes(const sc_job* jobs, int n) {
    if (!jobs || n < 1) return 0;
    size_t total = ctl_region(n);
    total += sc::align_up((size_t)n * sizeof(sc::Img), sc::kAlign);
    total += sc::align_up((size_t)8 * 32 * n * sizeof(int2), sc::kAlign);
    for (int i = 0; i < n; ++i) {
        if (jobs[i].H < 1 || jobs[i].W < 1 || jobs[i].C < 1 || jobs[i].C > 4) return 0;
        total += fwd_layout(jobs[i].H, jobs[i].W, jobs[i].C).total;
    }
    return total;
}

extern "C" sc_status sc_forward_batch_prepare(const sc_job* jobs, int n, void* ws, size_t ws_bytes,
                                              sc_batch_info* info) {
    if (!jobs || n < 1 || !ws || !info) return fail(SC_EINVAL, "null pointer or n < 1");
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    int max_rows = 1;
    for (int i = 0; i < n; ++i) {
        const sc_job& j = jobs[i];
        sc_status s = check_fwd_image(j.H, j.W, j.C, j.pitch);
        if (s != SC_OK) return fail(s, "job %d: %s", i, g_err);
        if (!j.img) return fail(SC_EINVAL, "job %d: null image", i);
        if (j.target_w < 1 || j.target_w > j.W)
            return fail(SC_EINVAL, "job %d: target_w=%d not in [1, %d]", i, j.target_w, j.W);
        max_rows = std::max(max_rows, j.H);
    }
    const size_t need = sc_forward_batch_workspace_bytes(jobs, n);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);

    int dev = 0, ncu = 0;
    hipError_t he = hipGetDevice(&dev);
    if (he == hipSuccess) he = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (he != hipSuccess) return hip_fail(he, "device query");
    long long units = 0;
    for (int i = 0; i < n; ++i) units += fwd_units(jobs[i].W);
    if (units > sc::kFwdBatchUnits)
        return fail(SC_EUNSUPPORTED, "%lld units of %d columns exceed the %d of a forward batch; split the batch", units,
                    sc::kFwdUnitCols, sc::kFwdBatchUnits);
    const int per_xcd = std::max(1, sc::fwt_blocks_per_cu() * ncu / 8);
    const BatchPlan plan = plan_batch(jobs, n, kDefaultTeamBatch, per_xcd, sc::kFwdThreads / 64);
    const std::vector<int>& gsz = plan.team;
    std::vector<int2> blk(plan.blk);
    for (int2& b : blk)
        if (b.x >= 0) b.x = plan.team_imgs[plan.teams[b.x].x];
    if (blk.size() > (size_t)8 * 32 * n) return fail(SC_EUNSUPPORTED, "plan too large");
    const size_t off_imgs = ctl_region(n);
    const size_t off_blk = off_imgs + sc::align_up((size_t)n * sizeof(sc::Img), sc::kAlign);
    size_t off_data = off_blk + sc::align_up((size_t)8 * 32 * n * sizeof(int2), sc::kAlign);
    std::vector<char> host(off_data, 0);
    WsHead* h = reinterpret_cast<WsHead*>(host.data());
    h->magic = kMagic;
    h->n = n;
    char* base = static_cast<char*>(ws);
    sc::Img* imgs = reinterpret_cast<sc::Img*>(host.data() + off_imgs);
    for (int i = 0; i < n; ++i) {
        const sc_job& j = jobs[i];
        sc::Ctl* ctl = reinterpret_cast<sc::Ctl*>(base + sizeof(WsHead)) + i;
        imgs[i] = make_fwd_img(j.src, j.img, j.H, j.W, j.C, j.pitch, j.target_w, j.seams_out, j.costs_out,
                               base + off_data, ctl, gsz[i]);
        off_data += fwd_layout(j.H, j.W, j.C).total;
    }
    memcpy(host.data() + off_blk, blk.data(), blk.size() * sizeof(int2));
    hipError_t e = hipMemcpy(ws, host.data(), host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "forward batch upload");
    int teams = 0;
    for (int i = 0; i < n; ++i) teams += gsz[i] > 1;
    memset(info, 0, sizeof(*info));
    info->n = n;
    info->nblocks = (int)blk.size();
    info->variant = -1;     // the forward kernel has one shape
    info->max_rows = max_rows;
    info->team = 0;         // marks a forward-energy batch
    info->teams_used = teams;
    info->off_imgs = off_imgs;
    info->off_blk = off_blk;
    return ok();
}

static sc_status fwd_batch_pass(const sc_batch_info* info, void* ws, void* stream, bool copy, bool carve) {
    if (!info || !ws || info->n < 1 || info->nblocks < 1 || info->team != 0 || info->variant != -1)
        return fail(SC_EINVAL, "not a forward-energy batch");
    char* base = static_cast<char*>(ws);
    const sc::Img* imgs = reinterpret_cast<const sc::Img*>(base + info->off_imgs);
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipSuccess;
    if (copy) e = sc::launch_fwt_prepare(imgs, info->n, info->max_rows, st);
    if (e == hipSuccess && carve)
        e = sc::launch_fwt_carve(imgs, reinterpret_cast<const int2*>(base + info->off_blk), info->nblocks, 0, st);
    if (e != hipSuccess) return hip_fail(e, "forward batch launch");
    return ok();
}

extern "C" sc_status sc_forward_batch_launch(const sc_batch_info* info, void* ws, void* stream) {
    return fwd_batch_pass(info, ws, stream, true, true);
}

extern "C" sc_status sc_forward_batch_launch_copy(const sc_batch_info* info, void* ws, void* stream) {
    return fwd_batch_pass(info, ws, stream, true, false);
}

extern "C" sc_status sc_forward_batch_launch_carve(const sc_batch_info* info, void* ws, void* stream) {
    return fwd_batch_pass(info, ws, stream, false, true);
}

// ---------------------------------------------------------------------------------------------
// Object removal with a mask (sec. "Object Removal"): direction from the mask's extent, masked
// carve of the frame (the image, or its transpose for horizontal seams), optional restore by
// seam insertion, then the result back in the caller's orientation.
namespace {

struct ObjLayout {
    size_t ctl, desc, tctl, wk, mk, dirs, anc, seam, buf_a, buf_b, ins, ins_bytes, total;
    size_t e, canc, xq, ro;  // by teams
    int wp, mp, db, ep, P, xw;
};

// Workspace of one carved frame of h rows by w0 columns.
ObjLayout obj_layout(int h, int w0, int C, bool restore) {
    ObjLayout L;
    memset(&L, 0, sizeof(L));
    const int P = (h + sc::kFwdPhaseRows - 1) / sc::kFwdPhaseRows;
    L.wp = (int)sc::align_up((size_t)w0 * C + 16, 64);  // 16 bytes between rows: the row shifter's last slot
    L.mp = (int)sc::align_up((size_t)w0 + 16, 64);
    L.db = (int)sc::align_up((size_t)(w0 + 3) / 4, 16);
    size_t off = 0;
    L.ctl = off;
    off = sc::align_up(off + sizeof(sc::ObjCtl), sc::kAlign);
    L.desc = off;
    off = sc::align_up(off + sizeof(sc::ObjImg), sc::kAlign);
    L.tctl = off;
    off = sc::align_up(off + sizeof(sc::Ctl), sc::kAlign);
    L.wk = off + 64;  // the row shifter may write up to 16 bytes below a plane
    off = sc::align_up(L.wk + (size_t)h * L.wp + sc::kFwdSlack, sc::kAlign);
    L.mk = off;
    off = sc::align_up(off + (size_t)h * L.mp + sc::kFwdSlack, sc::kAlign);
    L.dirs = off;
    off = sc::align_up(off + (size_t)((h + 3) / 4) * L.db * 4, sc::kAlign);
    L.anc = off;
    off = sc::align_up(off + (size_t)P * w0, sc::kAlign);
    L.seam = off;
    off = sc::align_up(off + (size_t)h * 4, sc::kAlign);
    if (sc::masked_by_teams(h, C)) {
        L.P = sc::key_rows(h, sc::kObjKR, 0);
        L.xw = sc::key_pitch(w0);
        L.ep = (int)sc::align_up((size_t)w0 * 4 + 16, 16) / 2;
        L.e = off + 64;
        off = sc::align_up(L.e + (size_t)(h + 1) * L.ep * 2 + 64, sc::kAlign);
        L.canc = off;
        off = sc::align_up(off + (size_t)L.P * L.xw, sc::kAlign);
        L.xq = off;
        off = sc::align_up(off + (size_t)L.P * L.xw * 4, sc::kAlign);
        L.ro = off;
        off = sc::align_up(off + (size_t)h * 4, sc::kAlign);
    }
    L.buf_a = L.buf_b = L.ins = L.ins_bytes = 0;
    if (restore && w0 >= 2) {
        L.buf_a = off;
        off = sc::align_up(off + (size_t)h * L.wp, sc::kAlign);
        L.buf_b = off;
        off = sc::align_up(off + (size_t)h * L.wp, sc::kAlign);
        L.ins = off;
        L.ins_bytes = sc_insert_workspace_bytes(h, w0, C, std::max(L.wp, 2 * L.ep), w0 - 1);  // the largest round
        off = sc::align_up(off + L.ins_bytes, sc::kAlign);
    }
    L.total = off;
    return L;
}

sc_status check_obj_frame(int h, int w0, int C) {
    if (w0 > sc::kFwdMaxW) return fail(SC_EUNSUPPORTED, "%d columns to carve > %d", w0, sc::kFwdMaxW);
    if (h > sc::kFwdMaxH) return fail(SC_EUNSUPPORTED, "%d rows to carve > %d", h, sc::kFwdMaxH);
    if ((long long)h * 510 * C > kMaxCostBound)
        return fail(SC_EUNSUPPORTED, "rows*510*C=%lld exceeds %d (23-bit seam energy)", (long long)h * 510 * C,
                    kMaxCostBound);
    if ((long long)h * (long long)sc::align_up((size_t)w0 * C, 64) + (long long)sc::kFwdSlack >= (1ll << 31))
        return fail(SC_EUNSUPPORTED, "frame of %lld bytes too large", (long long)h * w0 * C);
    return SC_OK;
}

bool ranges_overlap(const void* a, size_t a_len, const void* b, size_t b_len) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + b_len && b0 < a0 + a_len;
}

}  // namespace

extern "C" size_t sc_object_workspace_bytes(int H, int W, int C, int restore) {
    if (H < 1 || W < 1 || C < 1 || C > 4) return 0;
    return std::max(obj_layout(H, W, C, restore != 0).total, obj_layout(W, H, C, restore != 0).total);
}

extern "C" sc_status sc_remove_object(const uint8_t* img, const uint8_t* mask, int H, int W, int C, int pitch,
                                      int mpitch, int direction, int restore, uint8_t* out, int out_pitch,
                                      sc_object_info* info, int32_t* seams_out, int64_t* costs_out, void* ws,
                                      size_t ws_bytes, void* stream) {
    if (H < 1 || W < 1) return fail(SC_EINVAL, "H=%d W=%d must be >= 1", H, W);
    if (C < 1 || C > 4) return fail(SC_EINVAL, "C=%d must be in 1..4", C);
    if ((long long)pitch < (long long)W * C) return fail(SC_EINVAL, "pitch=%d < W*C=%lld", pitch, (long long)W * C);
    if (mpitch < W) return fail(SC_EINVAL, "mpitch=%d < W=%d", mpitch, W);
    if ((long long)out_pitch < (long long)W * C)
        return fail(SC_EINVAL, "out_pitch=%d < W*C=%lld", out_pitch, (long long)W * C);
    if (direction < SC_OBJ_AUTO || direction > SC_OBJ_HORIZONTAL)
        return fail(SC_EINVAL, "direction=%d not in {-1, 0, 1}", direction);
    if (restore != 0 && restore != 1) return fail(SC_EINVAL, "restore=%d not 0 or 1", restore);
    if (!img || !mask || !out || !info || !ws) return fail(SC_EINVAL, "null pointer");
    const size_t img_len = (size_t)(H - 1) * pitch + (size_t)W * C;
    const size_t out_len = (size_t)(H - 1) * out_pitch + (size_t)W * C;
    if (ranges_overlap(out, out_len, img, img_len) || ranges_overlap(out, out_len, mask, (size_t)(H - 1) * mpitch + W))
        return fail(SC_EINVAL, "out overlaps img or mask");
    if ((uintptr_t)ws % sc::kAlign) return fail(SC_EINVAL, "workspace must be %zu-byte aligned", sc::kAlign);
    const size_t need = sc_object_workspace_bytes(H, W, C, restore);
    if (ws_bytes < need) return fail(SC_ENOMEM, "workspace %zu < %zu bytes", ws_bytes, need);
    hipStream_t st = (hipStream_t)stream;
    char* base = static_cast<char*>(ws);
    sc::ObjCtl* ctl = reinterpret_cast<sc::ObjCtl*>(base);  // the control block sits first in both layouts
    sc::ObjCtl hc;
    hipError_t e = sc::launch_obj_reset(ctl, 1, st);
    if (e != hipSuccess) return hip_fail(e, "object reset");

    // the direction (synchronous: the frame to carve depends on it)
    int dir = direction;
    if (dir == SC_OBJ_AUTO) {
        e = sc::launch_mask_bbox(mask, H, W, mpitch, ctl->bbox, st);
        if (e == hipSuccess) e = hipMemcpyAsync(&hc, ctl, sizeof(hc), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return hip_fail(e, "mask extent");
        const int r0 = hc.bbox[0], r1 = hc.bbox[1], c0 = hc.bbox[2], c1 = hc.bbox[3];
        dir = (r1 < 0 || (c1 - c0 + 1) <= (r1 - r0 + 1)) ? SC_OBJ_VERTICAL : SC_OBJ_HORIZONTAL;
    }
    const bool vert = dir == SC_OBJ_VERTICAL;
    const int h = vert ? H : W, w0 = vert ? W : H;
    sc_status s = check_obj_frame(h, w0, C);
    if (s != SC_OK) return s;
    const ObjLayout L = obj_layout(h, w0, C, restore != 0);
    uint8_t* wk = reinterpret_cast<uint8_t*>(base + L.wk);
    uint8_t* mk = reinterpret_cast<uint8_t*>(base + L.mk);

    // the frame: image and mask, copied or transposed into the working buffers
    if (vert) {
        e = sc::launch_copy_rows(img, pitch, wk, L.wp, H, W * C, st);
        if (e == hipSuccess) e = sc::launch_copy_rows(mask, mpitch, mk, L.mp, H, W, st);
    } else {
        e = sc::launch_transpose(img, H, W, C, pitch, wk, L.wp, st);
        if (e == hipSuccess) e = sc::launch_transpose(mask, H, W, 1, mpitch, mk, L.mp, st);
    }
    if (e != hipSuccess) return hip_fail(e, "object frame");

    // the masked carve: seams until the mask is gone (or one column is left)
    sc::ObjImg d;
    memset(&d, 0, sizeof(d));
    d.wk = wk;
    d.mk = mk;
    d.dirs = reinterpret_cast<uint8_t*>(base + L.dirs);
    d.anc = reinterpret_cast<int8_t*>(base + L.anc);
    d.seam = reinterpret_cast<int32_t*>(base + L.seam);
    d.seams_out = seams_out;
    d.costs_out = reinterpret_cast<long long*>(costs_out);
    d.ctl = ctl;
    d.out = nullptr;
    d.H = h;
    d.W = w0;
    d.C = C;
    d.wp = L.wp;
    d.mp = L.mp;
    d.db = L.db;
    d.max_seams = w0 - 1;
    const bool teams = sc::masked_by_teams(h, C);
    if (teams) {
        sc::Ctl* tc = reinterpret_cast<sc::Ctl*>(base + L.tctl);
        d.c.img = reinterpret_cast<uint8_t*>(base + L.e);  // the carved rows, once the energies have served
        d.c.pitch = 2ll * L.ep;
        d.c.H = h;
        d.c.W = w0;
        d.c.C = C;
        d.c.target_w = 1;
        d.c.seams_out = seams_out;
        d.c.costs_out = reinterpret_cast<long long*>(costs_out);
        d.c.e = reinterpret_cast<uint16_t*>(base + L.e);
        d.c.ep = L.ep;
        d.c.anc = reinterpret_cast<int8_t*>(base + L.canc);
        d.c.xq = reinterpret_cast<uint32_t*>(base + L.xq);
        d.c.P = L.P;
        d.c.xw = L.xw;
        d.c.seam = d.seam;
        d.c.ro = reinterpret_cast<int32_t*>(base + L.ro);
        d.c.wk = wk;
        d.c.wp = L.wp;
        d.c.bar = &tc->bar;
        d.c.status = &tc->status;
        d.c.minside = 1;
        d.c.G = single_team(h, w0, sc::kObjThreads / 64);
    }
    sc::ObjImg* desc = reinterpret_cast<sc::ObjImg*>(base + L.desc);
    e = hipMemcpyAsync(desc, &d, sizeof(d), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = sc::launch_obj_carve(desc, 1, teams ? 0 : w0, st);
    if (e == hipSuccess) e = hipMemcpyAsync(&hc, ctl, sizeof(hc), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "object carve");
    const int k = hc.k, left = hc.left;
    int rw = hc.w;
    if (k < 0 || k > w0 - 1 || rw != w0 - k) return fail(SC_EHIP, "object carve returned k=%d w=%d", k, rw);

    // restore the size by seam insertion, in rounds of at most (current width - 1) seams
    const uint8_t* cur = teams && k > 0 ? d.c.img : wk;
    int curp = teams && k > 0 ? 2 * L.ep : L.wp;
    if (restore && k > 0) {
        if (rw < 2) return fail(SC_EINVAL, "the carve left one column: nothing to insert seams into");
        uint8_t* bufs[2] = {reinterpret_cast<uint8_t*>(base + L.buf_a), reinterpret_cast<uint8_t*>(base + L.buf_b)};
        int nb = 0;
        while (rw < w0) {
            const int n = std::min(w0 - rw, rw - 1);
            s = sc_insert_seams(cur, h, rw, C, curp, n, bufs[nb], L.wp, nullptr, nullptr, base + L.ins, L.ins_bytes,
                                stream);
            if (s != SC_OK) return s;
            cur = bufs[nb];
            curp = L.wp;
            nb ^= 1;
            rw += n;
        }
    }

    // the result in the caller's orientation
    if (vert) e = sc::launch_copy_rows(cur, curp, out, out_pitch, h, rw * C, st);
    else e = sc::launch_transpose(cur, h, rw, C, curp, out, out_pitch, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "object output");
    int dev = 0, khz = 0;
    double tick_ms = 0.0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) == hipSuccess && khz > 0)
        tick_ms = 1.0 / khz;
    memset(info, 0, sizeof(*info));
    info->direction = dir;
    info->k = k;
    info->rows = vert ? h : rw;
    info->cols = vert ? rw : h;
    info->left = left;
    info->carve_ms = (double)(hc.t_end - hc.t_begin) * tick_ms;
    for (int i = 0; i < 3; ++i) info->stage_ms[i] = (double)hc.t_stage[i] * tick_ms;
    return ok();
}
