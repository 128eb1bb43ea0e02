// How a team forms (join_team of sc_team.h), on host memory and threads that stand for workgroups.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <mutex>
#include <condition_variable>
#include <random>
#include <thread>
#include <vector>

#include "sc_team.h"

struct HostMem {
    template <class W>
    static W load(W* p) {
        return __atomic_load_n(p, __ATOMIC_RELAXED);
    }
    template <class W>
    static W add(W* p, W v) {
        return __atomic_fetch_add(p, v, __ATOMIC_RELAXED);
    }
    template <class W>
    static bool swap(W* p, W& seen, W v) {
        return __atomic_compare_exchange_n(p, &seen, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED);
    }
};
struct HostClock {  // ticks of 10 ns
    static unsigned long long now() {
        return (unsigned long long)std::chrono::duration_cast<std::chrono::nanoseconds>(
                   std::chrono::steady_clock::now().time_since_epoch()).count() / 10;
    }
    static void pause() { std::this_thread::yield(); }
};

static std::atomic<int> bad{0};
static void expect(bool ok, const char* what) {
    if (!ok) std::fprintf(stderr, "%s\n", what), ++bad;
}
static sc::Member join(unsigned long long* w, int xcd, int G, unsigned long long patience) {
    return sc::join_team<HostMem, HostClock>(w, xcd, G, patience);
}

// Members agree on the size and hold the ranks below it, once each; the others were told so.
static void check(const std::vector<sc::Member>& m, int least, bool apart) {
    int size = 0, members = 0;
    for (const auto& x : m)
        if (x.rank >= 0) size = x.size, ++members;
    std::vector<int> seen(m.size() + 1, 0);
    for (const auto& x : m) {
        if (x.rank < 0) continue;
        expect(x.size == size && x.rank < size, "members disagree on the size");
        expect(x.apart == apart, "members disagree on where they sit");
        expect(++seen[x.rank] == 1, "a rank taken twice");
    }
    expect(members == size && size >= least, "not as many members as the team says");
}

int main() {
    std::mt19937 rng(7);
    // everybody comes: the whole team, whatever the order
    for (int i = 0; i < 300; ++i) {
        const int G = 2 + (int)(rng() % 31), odd = i % 10 == 9 ? 1 : 0;
        unsigned long long w = 0;
        std::vector<sc::Member> m(G);
        std::vector<std::thread> t;
        for (int g = 0; g < G; ++g)
            t.emplace_back([&, g] { m[g] = join(&w, odd && g == G - 1 ? 3 : 5, G, 100000000000ull); });
        for (auto& x : t) x.join();
        check(m, G, odd != 0);
    }
    // some come while the team is being closed, or after
    for (int i = 0; i < 2000; ++i) {
        const int G = 2 + (int)(rng() % 7);
        unsigned long long w = 0;
        std::vector<sc::Member> m(G);
        std::vector<std::thread> t;
        const unsigned long long patience = rng() % 3 ? rng() % 4000 : 0;
        for (int g = 0; g < G; ++g) t.emplace_back([&, g] { m[g] = join(&w, 2, G, patience); });
        for (auto& x : t) x.join();
        check(m, 1, false);
    }
    // nobody else comes in time
    unsigned long long w = 0;
    const sc::Member alone = join(&w, 0, 32, 1000), late = join(&w, 0, 32, 1000);
    expect(alone.rank == 0 && alone.size == 1 && late.rank == -1, "a lone first member");
    // three teams of four on five slots, dealt in turn: no two whole teams fit, and each waits at
    // barriers of its own; all of them end
    for (int i = 0; i < 50; ++i) {
        constexpr int T = 3, G = 4, SLOTS = 5;
        unsigned long long words[T] = {};
        std::atomic<int> next{0}, arrived[T] = {}, done[T] = {};
        std::vector<std::thread> slots;
        for (int s = 0; s < SLOTS; ++s)
            slots.emplace_back([&] {
                for (int b; (b = next++) < T * G;) {
                    const int team = b % T;
                    const sc::Member me = join(&words[team], 1, G, 20000);
                    if (me.rank < 0) continue;
                    for (int round = 1; round <= 5; ++round) {
                        ++arrived[team];
                        while (arrived[team].load() < round * me.size) std::this_thread::yield();
                    }
                    if (me.rank == 0) ++done[team];
                }
            });
        for (auto& x : slots) x.join();
        for (int t = 0; t < T; ++t) expect(done[t].load() == 1, "a team that did not end once");
    }
    expect(sc::team_patience(1, 0) >= 20000 && sc::team_patience(1 << 30, 0) <= 5000000 && sc::team_patience(900, 2000) == 500,
           "patience out of range");
    if (!bad) std::printf("all teams formed\n");
    return bad != 0;
}
