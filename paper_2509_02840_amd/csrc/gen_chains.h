// gen_chains.h -- how the threads of the in-LDS generation kernel go through
// the chains of a phase: thread l of nt runs chains l, l + nt, ... and takes
// the next one at a step boundary.  The kernel (gen.hip) runs this code with a
// Wave that is one lane voting with its wavefront, the host tests with a Wave
// of 64 lanes.
#pragma once
#include "schedule.h"

namespace bdu {

template <typename Chain>
struct GenCursor {
    int ci, nt, nch;  // chain in flight, threads, chains of the phase
    Chain cur, nxt;   // chain ci, and ci + nt if `more`
    bool more;
    int q0;           // rotation of chain ci at the step's first tick
};

// The lane's chain at tick tb, where a part of the pass starts.
template <typename Chain, typename Load>
BDU_HD void gen_first_chain(GenCursor<Chain> &l, int tb, Load load)
{
    l.cur = load(l.ci);
    while (l.ci + l.nt < l.nch && l.cur.tau + l.cur.len <= tb) {
        l.ci += l.nt;
        l.cur = load(l.ci);
    }
    l.more = l.ci + l.nt < l.nch;
    l.nxt = load(l.ci + l.nt);
}

// At the start of a step: a lane whose chain has ended takes its next one.
// The fetch of the chains after those waits for memory, so a wavefront makes
// one once all its lanes have used theirs, well before the next is due.  But
// the lanes of a resumed part may be a chain apart: a lane that is due and
// holds none, while others do, is not kept waiting for them (it would pass its
// chain's first rotation).
template <typename Wave>
BDU_HD void gen_next_chain(Wave &w)
{
    auto due = [](const auto &l) { return l.q0 >= l.cur.len && l.ci + l.nt < l.nch; };
    auto holds = [](const auto &l) { return l.more; };
    if (!w.any(due)) return;
    if (w.any([&](const auto &l) { return due(l) && !holds(l); })) w.fetch();
    w.each(due, [&](auto &l) {
        l.ci += l.nt;
        l.cur = l.nxt;
        l.more = false;
        w.place(l);
    });
    if (!w.any(holds)) w.fetch();
}

}  // namespace bdu
