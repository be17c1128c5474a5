// Host simulation of the key groups' rings of the attention kernel (GroupRing in csrc/lds_plan.h, attn_stream16.hip:
// s16_segment with G > 1 and s16_group_idle).  The eight waves of a workgroup run the kernel's sequence of direct-to-LDS
// loads, LDS reads, waits and barriers under random interleavings; loads land at random later times unless a wait
// forces them.  Violations: a read of a fragment that has not landed or holds another kblock, a load issued to a fragment
// that some wave still has a read of in flight, waves that leave with unequal numbers of barriers behind them (the
// barrier is the workgroup's: all groups run the same number of steps).  Waves that bring kblocks into L2 ahead (GroupRing::TOUCHES)
// issue such a load, which nobody reads, in front of some hand-overs, whose wait leaves it in flight.  Exit status 0 = no violation
// in any run.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <vector>

#include "../paper_2509_22622_amd/csrc/lds_plan.h"

enum Kind { LOAD, TOUCH, WAIT_LOADS, WAIT_BUT_TOUCH, BARRIER, READ, READ_DONE };
struct Op { Kind kind; int is_v, rel, frag; };           // rel: kblock relative to the share's first

// what one wave of a group issues
template <int D, int G>
struct Program {
    using Plan = ll::LdsPlan16<D>;
    using Ring = ll::GroupRing<D, G>;
    static constexpr int KS = Plan::KS, NV = Plan::NV, NF = KS + NV, NW = 8 / G, LPW = Ring::PERIOD * NF / NW;
    std::vector<Op> ops;
    int wave, share;                                     // among the waves of the ring; kblocks of the share
    int every = 0, touch_in = 0;                         // S16Touch: one touch every so many periods (0: none); periods to the next

    void load(int first, int l) {                        // as issue_group: V of the period's kblocks, K two kblocks on
        const int j = NW * l / NF, part = NW * l % NF;
        const int is_v = part >= KS;
        ops.push_back({LOAD, is_v, first + j + (is_v ? 0 : 2), (is_v ? part - KS : part) + wave});
    }
    void handover(bool touches) {
        if (touches && every > 0 && --touch_in < 0) {
            ops.push_back({TOUCH, 0, 0, 0});
            touch_in += every;
            ops.push_back({WAIT_BUT_TOUCH, 0, 0, 0});
        } else {
            ops.push_back({WAIT_LOADS, 0, 0, 0});
        }
        if (NW > 1) ops.push_back({BARRIER, 0, 0, 0});
    }
    void works(int n_steps) {
        for (int l = 0; l < LPW; ++l) load(0, l);
        for (int t = touch_in; every > 0 && t < Ring::TOUCH_AHEAD; t += every) ops.push_back({TOUCH, 0, 0, 0});
        handover(false);
        std::vector<int> k_pending(KS, -1);              // K reads in flight from the step before: their kblock
        for (int r = 0; r < n_steps; ++r) {
            for (int slot = 0; slot < NF; ++slot) {
                if (slot < KS && k_pending[slot] >= 0) {
                    ops.push_back({READ_DONE, 0, k_pending[slot], slot});
                    k_pending[slot] = -1;
                }
                for (int f = 0; f < NV; ++f)
                    if (Plan::first_use_v(f) == slot) ops.push_back({READ_DONE, 1, r, f});
                if (r % Ring::PERIOD == 0)
                    for (int l = 0; l < LPW; ++l)
                        if (Ring::dma_slot(l, LPW, NF) == slot) load(r + Ring::PERIOD, l);
                for (int f = 0; f < NV; ++f)
                    if (Plan::vslot(f) == slot) ops.push_back({READ, 1, r, f});
                for (int f = 0; f < KS; ++f)
                    if (Plan::kslot(f) == slot) {
                        ops.push_back({READ, 0, r + 2, f});
                        k_pending[f] = r + 2;
                    }
            }
            if (r % Ring::PERIOD == Ring::PERIOD - 1) {
                for (int f = 0; f < KS; ++f) {
                    ops.push_back({READ_DONE, 0, k_pending[f], f});
                    k_pending[f] = -1;
                }
                handover(true);
            }
        }
    }
    void idles(int n_steps) {                            // as s16_group_idle: no rows, or (share 0) no kblocks
        if (NW == 1) return;
        for (int r = -Ring::PERIOD; r + Ring::PERIOD <= n_steps; r += Ring::PERIOD) {
            if (share > 0)
                for (int l = 0; l < LPW; ++l) load(r + Ring::PERIOD, l);
            handover(false);
        }
        if (n_steps % Ring::PERIOD != 0 && share > 0)
            for (int l = 0; l < LPW; ++l) load(n_steps / Ring::PERIOD * Ring::PERIOD + Ring::PERIOD, l);
    }
};

struct Fragment { int kblock = -1, owner = -1, seq = -1, readers = 0; };

// T kblocks; the first `with_rows` of a group's waves have query rows, which touch every `every` periods from the `first` on
template <int D, int G>
static int simulate(int T, int with_rows, unsigned seed, int every, int first) {
    using P = Program<D, G>;
    constexpr int DEPTH = P::Ring::DEPTH;
    std::srand(seed);
    const int lag = seed % 2 ? 4 : 256;                  // how late loads land that nothing waits for
    const int n_steps = (T + G - 1) / G;
    std::vector<P> prog(8);
    int barriers[8];
    for (int w = 0; w < 8; ++w) {
        const int group = w / P::NW;
        prog[w].wave = w % P::NW;
        prog[w].every = every;
        prog[w].touch_in = first;
        prog[w].share = T * (group + 1) / G - T * group / G;
        if (prog[w].share > 0 && prog[w].wave < with_rows) prog[w].works(n_steps);
        else prog[w].idles(n_steps);
        barriers[w] = 0;
        for (const Op& op : prog[w].ops) barriers[w] += op.kind == BARRIER;
        if (barriers[w] != barriers[0]) {
            std::printf("D %d G %d T %d: wave %d meets %d barriers, wave 0 %d\n", D, G, T, w, barriers[w], barriers[0]);
            return 1;
        }
    }
    std::vector<Fragment> lds(G * 2 * DEPTH * P::KS);
    auto at = [&](int group, const Op& op) -> Fragment& {
        return lds[((size_t(group) * 2 + op.is_v) * DEPTH + (op.rel & (DEPTH - 1))) * P::KS + op.frag];
    };
    std::vector<size_t> pc(8, 0);
    int issued[8] = {}, landed[8] = {}, waiting[8] = {};             // loads of a wave land in order
    for (;;) {
        bool all_done = true, all_waiting = true;
        for (int w = 0; w < 8; ++w)
            if (pc[w] < prog[w].ops.size()) {
                all_done = false;
                if (!waiting[w]) all_waiting = false;
            }
        if (all_done) return 0;
        if (all_waiting) {
            for (int w = 0; w < 8; ++w)
                if (pc[w] < prog[w].ops.size()) { waiting[w] = 0; ++pc[w]; }
            continue;
        }
        const int w = std::rand() % 8, group = w / P::NW;
        if (pc[w] >= prog[w].ops.size() || waiting[w]) continue;
        for (int o = 0; o < 8; ++o)
            if (landed[o] < issued[o] && std::rand() % lag == 0) ++landed[o];
        const Op op = prog[w].ops[pc[w]];
        Fragment& f = at(group, op);
        const int kblock = op.rel < prog[w].share - 1 ? op.rel : prog[w].share - 1;      // past the end the last one again
        const char* what = op.is_v ? "V" : "K";
        if (op.kind == BARRIER) { waiting[w] = 1; continue; }
        if (op.kind == TOUCH) ++issued[w];
        if (op.kind == WAIT_LOADS) landed[w] = issued[w];
        if (op.kind == WAIT_BUT_TOUCH && landed[w] < issued[w] - P::Ring::TOUCH_LOADS) landed[w] = issued[w] - P::Ring::TOUCH_LOADS;
        if (op.kind == LOAD) {
            if (f.readers > 0) {
                std::printf("D %d G %d T %d: wave %d loads %s %d over a fragment being read\n", D, G, T, w, what, op.rel);
                return 1;
            }
            const int readers = f.readers;
            f = Fragment{kblock, w, ++issued[w], readers};
        }
        if (op.kind == READ) {
            if (f.owner < 0 || landed[f.owner] < f.seq || f.kblock != kblock) {
                std::printf("D %d G %d T %d: wave %d reads %s %d (kblock %d), the fragment holds %s kblock %d\n", D, G, T, w, what, op.rel,
                            kblock, f.owner < 0 ? "no" : landed[f.owner] < f.seq ? "in-flight" : "landed", f.kblock);
                return 1;
            }
            ++f.readers;
        }
        if (op.kind == READ_DONE) --f.readers;
        ++pc[w];
    }
}

template <int D, int G>
static int check() {
    for (int T : {1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 64, 83})
        for (int with_rows = 1; with_rows <= 8 / G; ++with_rows)
            for (unsigned seed = 1; seed <= 25; ++seed) {
                if (simulate<D, G>(T, with_rows, seed * 7919u + T, 0, 0)) return 1;
                for (int every = 1; every <= 8 && ll::GroupRing<D, G>::TOUCHES; every *= 2)
                    if (simulate<D, G>(T, with_rows, seed * 7919u + T, every, int(seed) % every)) return 1;
            }
    return 0;
}

int main() {
    if (check<64, 2>() || check<64, 4>() || check<64, 8>() || check<128, 2>() || check<128, 4>()) return 1;
    std::printf("group rings ok\n");
    return 0;
}
