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
    ctl->xmask = 0;
}

}  // namespace sc
