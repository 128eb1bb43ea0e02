// The batch planner (sc_api.cpp), run on the host through sc_batch_prepare and sc_forward_batch_prepare:
// the HIP runtime is replaced by the few functions below (a device of 256 compute units, whose memory is
// host memory), the kernel launchers by kernel_stubs.cpp.  Every plan is taken apart.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <memory>
#include <vector>

#include "sc.h"
#include "sc_internal.h"

namespace {
int bad = 0;
#define EXPECT(cond, i)                                                                         \
    do {                                                                                        \
        if (!(cond)) std::fprintf(stderr, "line %d, batch %d: %s\n", __LINE__, (int)(i), #cond), ++bad; \
    } while (0)
std::vector<char> uploaded;  // the plan region, as the last hipMemcpy wrote it
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
    return hipSuccess;
}
hipError_t hipMemcpy(void*, const void* src, size_t n, hipMemcpyKind) {
    uploaded.assign(static_cast<const char*>(src), static_cast<const char*>(src) + n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "none"; }
}

static void check(const std::vector<sc_job>& jobs, int max_team, bool forward, int id) {
    const int n = (int)jobs.size();
    alignas(256) static char ws[256];  // never touched: uploads are caught above
    sc_batch_info info;
    sc_tune tune = {max_team, -1, 0};
    const size_t need = forward ? sc_forward_batch_workspace_bytes(jobs.data(), n) : sc_batch_workspace_bytes(jobs.data(), n);
    const sc_status s = forward ? sc_forward_batch_prepare(jobs.data(), n, ws, need, &info)
                                : sc_batch_prepare(jobs.data(), n, &tune, ws, need, &info);
    EXPECT(s == SC_OK, id);
    if (s != SC_OK) return;
    const int per_cu = forward ? sc::fwt_blocks_per_cu() : sc::carve_blocks_per_cu(sc::default_variant());
    const int per_xcd = per_cu * 256 / 8;
    const int most = max_team ? max_team : 16;
    EXPECT(uploaded.size() <= need && info.nblocks <= 8 * 32 * n, id);
    const sc::Img* imgs = reinterpret_cast<const sc::Img*>(uploaded.data() + info.off_imgs);
    const int2* blk = reinterpret_cast<const int2*>(uploaded.data() + info.off_blk);
    const int2* teams = reinterpret_cast<const int2*>(uploaded.data() + info.off_teams);
    const int* ti = reinterpret_cast<const int*>(uploaded.data() + info.off_team_imgs);
    std::vector<std::vector<int>> members(n);  // per image: the block of each member
    int in_teams[8] = {}, larger = 0, singles_seen[8] = {}, used = 0;
    for (int b = 0; b < info.nblocks; ++b) {
        if (blk[b].x < 0) continue;
        EXPECT(forward || teams[blk[b].x].y == 1, id);
        const int i = forward ? blk[b].x : ti[teams[blk[b].x].x];
        if (i < 0 || i >= n) {
            EXPECT(!"an image that is not there", id);
            return;
        }
        EXPECT(blk[b].y == (int)members[i].size(), id);  // members in order
        EXPECT(members[i].empty() || b == members[i].back() + 8, id);  // 8 blocks apart: on one XCD
        members[i].push_back(b);
        if (imgs[i].G > 1) {
            ++in_teams[b % 8];
            EXPECT(!singles_seen[b % 8], id);  // teams first: nothing that may queue lies before them
        } else {
            singles_seen[b % 8] = 1;
        }
    }
    for (int i = 0; i < n; ++i) {
        EXPECT((int)members[i].size() == imgs[i].G, id);
        larger += imgs[i].G > most;
        EXPECT(imgs[i].G <= std::min(2 * most, 32) && (most > 1 || imgs[i].G == 1), id);
        used += imgs[i].G > 1;
    }
    EXPECT(larger <= 1 && used == info.teams_used, id);  // the longest image alone may have twice the largest team
    for (int x = 0; x < 8; ++x) EXPECT(in_teams[x] <= per_xcd, id);
}

int main() {
    static uint8_t pixels[16];
    uint64_t x = 88172645463325252ull;
    auto rnd = [&](int lo, int hi) {
        x ^= x << 13, x ^= x >> 7, x ^= x << 17;
        return lo + (int)(x % (uint64_t)(hi - lo + 1));
    };
    auto batch = [&](int n, int lo, int hi, int keep) {
        std::vector<sc_job> jobs(n);
        for (auto& j : jobs) {
            j = sc_job{};
            j.img = pixels;
            j.H = rnd(lo, hi);
            j.W = rnd(lo, hi);
            j.C = rnd(1, 3);
            j.pitch = j.W * j.C;
            j.target_w = std::max(1, j.W - rnd(0, std::max(1, j.W * keep / 100)));
        }
        return jobs;
    };
    int id = 0;
    for (int n : {1, 2, 3, 8, 9, 31, 64, 65, 200, 256, 512, 700, 3000})
        for (int hi : {1, 40, 260, 2160}) {
            const auto jobs = batch(n, hi == 1 ? 1 : 16, hi, 40);
            for (int team : {0, 1, 2, 5, 16, 32}) check(jobs, team, false, ++id);
            if (n <= 150 || (hi < 900 && n <= 512)) check(jobs, 0, true, ++id);
        }
    check(std::vector<sc_job>(64, batch(1, 1500, 1500, 40)[0]), 32, false, ++id);  // all alike
    check(std::vector<sc_job>(64, batch(1, 1500, 1500, 40)[0]), 0, true, ++id);
    auto still = batch(40, 100, 900, 30);  // nothing to remove but in one
    for (int i = 1; i < 40; ++i) still[i].target_w = still[i].W;
    check(still, 0, false, ++id);
    check(still, 0, true, ++id);
    check(batch(5, 5000, 5400, 10), 0, false, ++id);
    check(batch(5, 5000, 5400, 10), 0, true, ++id);
    if (!bad) std::printf("all plans hold\n");
    return bad != 0;
}
