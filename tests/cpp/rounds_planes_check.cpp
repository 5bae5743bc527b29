// Host-side check of how lc_kmeans_rounds_kernel keeps the centroid of a cluster that has lost its members (csrc/lc_rounds_planes.h):
// the wavefronts of two workgroups that come to it, one piece of the row at a time and in drawn orders, a helper among them wherever a
// look leaves pieces open.  No word but the standing centroid's may ever be posted, and every workgroup ends up comparing with it.
// The same orders are played with one plane number to a cluster, set by the first piece seen, which has to show as a fault.
// Prints "ok <orders> <faults of the one number>" or the first violation.
#include <cstdio>
#include <random>
#include "lc_rounds_planes.h"

namespace {

constexpr int PIECES = 4, PLANES = 8, UNPOSTED = -1, NOT_A_NUMBER = -2;

struct OneNumber {
    int at[1];
    void start(int) { at[0] = 0; }
    void enter(int, int, bool) {}
    void seen(int it, int piece) { if (piece == 0) at[0] = it; }
    int now(int, int) const { return at[0]; }
    int before(int, int) const { return at[0]; }
};
struct TwoNumbers : LcPlanes<1> {
    void seen(int, int) {}
};

template <typename Planes>
struct Play {
    int posts[PLANES][PIECES];
    int expect;                              // the standing centroid: 10 + the iteration that made it
    Planes planes[2];
    int open[2];                             // pieces of the row that the workgroup's looking wavefront has not seen
    bool bad = false;

    // one wavefront's own steps, in turn
    struct Wave {
        int group;
        bool looks;                          // the one that looks for the row (and helps); otherwise the cluster's own
        int step = 0, piece = 0, from = 0, value[PIECES];
        bool done = false, helping = false;
    };

    void post(int it, int piece, int v) {
        if (v == UNPOSTED) v = NOT_A_NUMBER;
        if (v != expect) bad = true;
        posts[it][piece] = v;
    }
    // pieces read one by one, then posted one by one
    bool work_out(Wave& w, int it) {
        if (w.step == 0) { w.from = planes[w.group].before(it, 0); w.step = 1; w.piece = 0; return false; }
        if (w.step == 1) {
            w.value[w.piece] = posts[w.from][w.piece];
            if (++w.piece == PIECES) { w.step = 2; w.piece = 0; }
            return false;
        }
        post(it, w.piece, w.value[w.piece]);
        return ++w.piece == PIECES;
    }
    void advance(Wave& w, int it, bool impatient) {
        if (!w.looks || w.helping) {
            if (!work_out(w, it)) return;
            if (w.looks) { w.helping = false; w.step = 0; w.piece = 0; }
            else w.done = true;
            return;
        }
        const int p = w.piece;               // (a look is not one moment for all pieces)
        if ((open[w.group] >> p & 1) && posts[it][p] != UNPOSTED) {
            open[w.group] &= ~(1 << p);
            planes[w.group].seen(it, p);
        }
        w.piece = (p + 1) % PIECES;
        if (open[w.group] == 0) w.done = true;
        else if (w.piece == 0 && impatient) { w.helping = true; w.step = 0; }
    }

    // an iteration leaves the cluster alone, makes its centroid from members, or touches it and keeps its centroid
    bool run(std::mt19937& r) {
        for (auto& plane : posts) for (int& w : plane) w = UNPOSTED;
        for (int& w : posts[0]) w = 10;
        expect = 10;
        for (auto& p : planes) p.start(0);
        for (int it = 0; it < PLANES; ++it) {
            const bool touched = it == 0 || r() % 3 != 0, members = it > 0 && touched && r() % 2 == 0;
            for (auto& p : planes) p.enter(it, 0, touched);
            if (members) expect = 10 + it;
            if (it == 0 || members) {        // (made from its members: the same bits by whoever)
                for (int& w : posts[it]) w = expect;
                for (auto& p : planes) for (int i = 0; i < PIECES; ++i) p.seen(it, i);
            } else if (touched) {
                Wave waves[3] = {{0, false}, {0, true}, {1, true}};
                open[0] = open[1] = (1 << PIECES) - 1;
                const unsigned late = r() % 3;                       // the owner starts at once, late, or hardly at all
                for (int steps = 0; !(waves[0].done && waves[1].done && waves[2].done); ++steps) {
                    if (steps > 100000) return false;
                    Wave& w = waves[r() % 3];
                    if (w.done || (&w == &waves[0] && late && r() % (late == 1 ? 8 : 64))) continue;
                    advance(w, it, r() % 2 == 0);
                }
            }
            for (auto& p : planes)           // behind the barrier
                for (int i = 0; i < PIECES; ++i)
                    if (posts[p.now(it, 0)][i] != expect) bad = true;
            if (bad) return false;
        }
        return true;
    }
};

}  // namespace

int main() {
    constexpr int ORDERS = 20000;
    int faults = 0;
    for (int seed = 0; seed < ORDERS; ++seed) {
        std::mt19937 r(seed), same(seed);
        Play<TwoNumbers> play;
        if (!play.run(r)) { std::printf("FAIL order %d\n", seed); return 1; }
        Play<OneNumber> one;
        faults += !one.run(same);
    }
    std::printf("ok %d %d\n", ORDERS, faults);
    return 0;
}
