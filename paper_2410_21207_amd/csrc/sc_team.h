// What the workgroups of a team agree on through words of memory that all of them see, with no barrier
// at hand.  The steps are written over Mem (relaxed accesses of the team's scope), so that the same
// code runs in the kernels and, on host memory and threads, in the CPU tests.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define TEAM_FN __host__ __device__ __forceinline__
#else
#define TEAM_FN inline
#endif

namespace sc {

// Joining a team.  The workgroups that a launch means to work together need not all be resident: other
// streams' kernels may hold the slots of their XCD, and two teams that each hold some of them would
// wait for each other for ever.  So a team is whoever has come when its first member closes it: at
// once when all G are there (a few microseconds after the first), else when its patience ends.  A
// workgroup that comes later is told so and leaves.  From then on members wait only for members, which
// are all running, and any number of them carves the same seams.
//
// The word, 0 at the launch: six bits per XCD with the number of workgroups that came from it, and
// from bit 48 on the size of the closed team, with bit 54 where its members sit on several XCDs.
struct Member {
    int rank, size;  // rank -1: the team went without this workgroup
    bool apart;      // on several XCDs: members do not see each other's stores
};
constexpr int kTeamClosed = 48;
TEAM_FN int team_count(unsigned long long word) {
    int n = 0;
    for (int x = 0; x < 8; ++x) n += (int)(word >> (6 * x)) & 63;
    return n;
}
TEAM_FN unsigned long long team_close(unsigned long long word) {  // the word of the team as it stands
    int xcds = 0;
    for (int x = 0; x < 8; ++x) xcds += ((word >> (6 * x)) & 63) != 0;
    return word | (unsigned long long)(team_count(word) | (xcds > 1 ? 64 : 0)) << kTeamClosed;
}
template <class Mem, class Clock, class Word>
TEAM_FN Member join_team(Word* word, int xcd, int G, unsigned long long patience) {
    const unsigned long long before = Mem::add(word, 1ull << (6 * (xcd & 7)));
    if (before >> kTeamClosed) return {-1, 0, false};
    const int rank = team_count(before);
    unsigned long long w = Mem::load(word);
    if (rank == 0) {
        for (const unsigned long long t0 = Clock::now(); team_count(w) < G && Clock::now() - t0 <= patience; w = Mem::load(word))
            Clock::pause();
        while (!Mem::swap(word, w, team_close(w))) {}  // (a failed swap loads w anew)
        w = team_close(w);
    } else {
        for (; !(w >> kTeamClosed); w = Mem::load(word)) Clock::pause();  // the first member is running and will close it
    }
    const int size = (int)(w >> kTeamClosed);
    return {rank, size & 63, (size & 64) != 0};
}
// Ticks of the 100 MHz clock that a team of `seams` seams waits for its missing workgroups: 0.2 ms, many
// times what a dispatch takes, and about as long as the whole team then takes for its seams, 50 us each
// (1003 x 701 takes 38 us by 16 workgroups and 110 by one), at most 50 ms; a quarter of the time
// budget where there is one.  A wait in vain so at most doubles the time, and what a team that went without its
// members loses is more: 256 images launched with a 25 ms carve that held slots of their XCD took 269 ms
// with 20 us per seam and a cap of 10 ms, which closed the longest image's team early, and take 177 to 197 (175 alone).
TEAM_FN unsigned long long team_patience(int seams, unsigned long long budget) {
    const unsigned long long p = seams < 996 ? 20000ull + 5000ull * (unsigned)seams : 5000000ull;
    return budget && budget / 4 < p ? budget / 4 : p;
}

// The end of a call by its time budget (step-wise carving).  The team's first member decides before
// a seam's last barrier and every member reads the decision after it, some of them late: the first
// member may have left the call by then.  So the word names the seam after which the call ends, and
// nothing takes that back: a later seam's number is another, and a new image clears the word before
// its first launch.  (A flag that the first member cleared on its way out let a late reader go on alone.)
template <class Mem, class Word>
TEAM_FN void stop_after(Word* word, int k) {
    Mem::store(word, (unsigned)k + 1u);
}
template <class Mem, class Word>
TEAM_FN bool stops_after(Word* word, int k) {
    return Mem::load(word) == (unsigned)k + 1u;
}

// What the first member leaves behind for the next call (seams removed, barrier count), written when
// its own workgroup is through; other members may still be on their way out and read the word above.
template <class Control>
TEAM_FN void leave_call(Control* ctl, int done, unsigned epoch) {
    ctl->done = (unsigned)done;
    ctl->ebase = epoch;
}

}  // namespace sc
