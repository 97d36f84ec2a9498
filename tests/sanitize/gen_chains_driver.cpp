// Replays, wavefront by wavefront, how the in-LDS generation kernel's threads
// go through the chains of a plan (gen_chains.h, the code that the kernel
// runs), for the whole pass, its two parts and its segments: at every step, the
// chain that has rotations in it has to be the one its thread holds.
//   gen_chains_driver n_first n_last stride [K0 NW]
// Prints each shape and tiling that loses a chain; exit status 0 if none does.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <vector>

#include "../../paper_2509_02840_amd/csrc/gen_chains.h"
#include "../../paper_2509_02840_amd/csrc/plan.h"

namespace {

using namespace bdu;

struct Chain {
    int len, tau;
};
const Chain kNone = {0, 1 << 30};

struct Wave {
    std::vector<GenCursor<Chain>> lane;
    const std::vector<Chain> &chains;
    int t = 0;  // first tick of the step
    Chain load(int c) const { return c < (int)chains.size() ? chains[(size_t)c] : kNone; }
    template <typename F>
    bool any(F f) const
    {
        return std::any_of(lane.begin(), lane.end(), f);
    }
    template <typename F, typename G>
    void each(F f, G g)
    {
        for (auto &l : lane)
            if (f(l)) g(l);
    }
    void place(GenCursor<Chain> &l) { l.q0 = t - l.cur.tau; }
    void fetch()
    {
        for (auto &l : lane) {
            l.more = l.ci + l.nt < l.nch;
            l.nxt = load(l.ci + l.nt);
        }
    }
};

// Chains (by index in their phase) that are not held in a step in which they
// have rotations, ticks [tb, te) with nt threads.
int lost(const std::vector<Chain> &chains, int nt, int tb, int te)
{
    int bad = 0;
    for (int w0 = 0; w0 < nt; w0 += kGenChunk) {
        Wave w{{}, chains};
        std::vector<int> expect;  // the chain each lane should be on, or a later one
        for (int l = 0; l < kGenChunk; ++l) {
            GenCursor<Chain> g{};
            g.ci = w0 + l;
            g.nt = nt;
            g.nch = (int)chains.size();
            gen_first_chain(g, tb, [&](int c) { return w.load(c); });
            w.lane.push_back(g);
            expect.push_back(w0 + l);
        }
        w.t = tb;
        for (auto &l : w.lane) w.place(l);
        for (int t = tb; t < te; t += kGenStep) {
            w.t = t;
            gen_next_chain(w);
            for (int l = 0; l < kGenChunk; ++l) {
                int &c = expect[(size_t)l];
                auto ended = [&](int x) { return x < (int)chains.size() && w.load(x).tau + w.load(x).len <= t; };
                while (ended(c)) c += nt;
                const Chain x = w.load(c);
                if (x.len > 0 && x.tau < t + kGenStep && w.lane[(size_t)l].ci != c) ++bad;
                w.lane[(size_t)l].q0 += kGenStep;
            }
        }
    }
    return bad;
}

int check(int64_t m, int64_t n, int k0, int nw)
{
    const auto P = build_plan(m, n, k0, nw, kGenThreads);
    std::vector<Chain> ph[2];
    for (const GenChain &g : P->chains) {
        if (g.type == CH_FOLD) continue;
        auto &v = ph[chain_phase(g.type) - 1];
        v.resize((size_t)chain_in_phase(g.type, g.param), kNone);  // an index without a chain stays empty
        v.push_back(Chain{g.len, g.tau0});
    }
    const int split = (int)P->split, ticks = (int)P->ticks;
    const int t2 = (split + kGenStep - 1) / kGenStep * kGenStep;
    int bad = 0;
    auto part = [&](int t0, int t1) {  // as gen_lds_kernel runs it
        if (t0 < split - 1) bad += lost(ph[0], P->L, t0, std::min(t1, split - 1));
        if (t1 > t2) bad += lost(ph[1], P->L, std::max(t0, t2), t1);
    };
    part(0, ticks);
    part(0, split);
    part(split, ticks);
    for (int k = 0; k < P->nseg; ++k) part(k == 0 ? 0 : P->tcut[k - 1], P->tcut[k]);
    if (bad) printf("m %ld n %ld K0 %d NW %d: %d lane steps on the wrong chain\n", (long)m, (long)n, k0, nw, bad);
    return bad;
}

}  // namespace

int main(int argc, char **argv)
{
    if (argc != 4 && argc != 6) return 2;
    const int tilings[][2] = {{12, 3}, {12, 7}, {12, 15}, {18, 3}, {18, 5}, {18, 7}, {6, 1}, {6, 2},
                              {6, 4},  {6, 8},  {12, 1},  {12, 2}, {12, 4}, {12, 8}};
    int shapes = 0, bad = 0;
    for (int n = atoi(argv[1]); n <= atoi(argv[2]); n += atoi(argv[3]))
        for (auto &t : tilings) {
            if (argc == 6 && (t[0] != atoi(argv[4]) || t[1] != atoi(argv[5]))) continue;
            bad += check(n, n, t[0], t[1]) > 0;
            if (n < (int)kMaxGenLdsRows) bad += check(n + 9, n, t[0], t[1]) > 0;
            shapes += 1 + (n < (int)kMaxGenLdsRows);
        }
    printf("gen chains: %d of %d plans lose a chain\n", bad, shapes);
    return bad != 0;
}
