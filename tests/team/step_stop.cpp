// The time-budget decision of a team (sc_team.h) on host memory, with a member that reads it at every
// point from the decision to the end of the next call's first seam.
#include <cstdio>

#include "sc_internal.h"
#include "sc_team.h"

struct HostMem {
    template <class W>
    static W load(W* p) {
        return __atomic_load_n(p, __ATOMIC_RELAXED);
    }
    template <class W>
    static void store(W* p, W v) {
        __atomic_store_n(p, v, __ATOMIC_RELAXED);
    }
};

static int bad = 0;
static void expect(bool ok, const char* what, int k) {
    if (!ok) std::fprintf(stderr, "seam %d: %s\n", k, what), ++bad;
}

int main() {
    using namespace sc;
    Ctl c{};  // as a new image's first pass leaves it
    // calls of 1, 2, 5, ... seams, each ended by its budget
    int k = 0;
    unsigned epoch = 0;
    for (int len : {1, 2, 5, 1, 1, 40}) {
        for (int i = 0; i < len; ++i, ++k) {
            const bool last = i + 1 == len;
            expect(!stops_after<HostMem>(&c.stop, k), "stops before the decision", k);
            if (last) stop_after<HostMem>(&c.stop, k);
            epoch += 3;
            // the last barrier of seam k: the first member reads at once, another whenever it gets there
            expect(stops_after<HostMem>(&c.stop, k) == last, "the first member reads another decision", k);
            if (!last) continue;
            expect(stops_after<HostMem>(&c.stop, k), "a member still in the barrier goes on alone", k);
            leave_call(&c, k + 1, epoch);
            expect(stops_after<HostMem>(&c.stop, k), "a member goes on alone after the first has left the call", k);
            expect(c.done == (unsigned)k + 1 && c.ebase == epoch, "what the call leaves", k);
        }
    }
    if (!bad) std::printf("all members agreed\n");
    return bad != 0;
}
