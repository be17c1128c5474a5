// Host simulation of the rings of the 8-bit attention kernel's key groups (Fp8GroupRing in csrc/lds_plan.h, attn_fp8.hip:
// f8_segment_sp with G > 1 and f8_group_idle).  The eight waves of a workgroup run the kernel's sequence of direct-to-LDS loads, LDS
// reads, waits and barriers under random interleavings; loads land at random later times unless a wait forces them.  Violations:
// a read of a piece (1 KB) that has not landed or holds another kblock, a load issued to a piece that some wave still has a
// read of in flight, waves that leave with unequal numbers of barriers behind them.  Exit status 0 = no violation in any run.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2509_22622_amd/csrc/lds_plan.h"

enum Kind { LOAD, WAIT_LOADS, BARRIER, READ, READ_DONE };
struct Op { Kind kind; int half, piece, kblock; };       // half stage; kblock of the tile, values + VALUES
constexpr int VALUES = 1 << 20;

template <int D, int G>
struct Program {
    using Plan = ll::Fp8LdsPlan<D>;
    using Ring = ll::Fp8GroupRing<D, G>;
    static constexpr int NW = 8 / G, PIECES = Ring::KB_BYTES / 1024, LPW = 2 * PIECES / NW;      // of a kblock's keys; loads a wave and step
    std::vector<Op> ops;
    int wave, vb, ve;                                    // among the waves of the ring; the share

    void first_keys() {                                  // of the tile
        for (int l = 0; l < PIECES / NW; ++l) ops.push_back({LOAD, Ring::FIRST_HALF, wave + NW * l, 0});
    }
    void load(int rel, int l) {                          // as issue_group: K first, then V
        const bool is_k = l < LPW / 2;
        const int ahead = rel + (is_k ? Ring::K_AHEAD : Ring::V_AHEAD), v = vb + ahead < ve - 1 ? vb + ahead : ve - 1;
        ops.push_back({LOAD, is_k ? Ring::k_half(ahead) : Ring::v_half(ahead), wave + NW * (is_k ? l : l - LPW / 2), is_k ? v : v + VALUES});
    }
    void wait_loads() { ops.push_back({WAIT_LOADS, 0, 0, 0}); }
    void barrier() { ops.push_back({BARRIER, 0, 0, 0}); }
    void scores(int half, int kblock) {                  // all of a kblock's keys, read by the compiler
        for (Kind kind : {READ, READ_DONE})
            for (int piece = 0; piece < PIECES; ++piece) ops.push_back({kind, half, piece, kblock});
    }
    void fragment(Kind kind, int rel, int slot) {        // slot's two pieces: K of the kblock after this step's, V of this step's
        const int next = vb + rel + 1 < ve - 1 ? vb + rel + 1 : ve - 1, own = vb + rel < ve - 1 ? vb + rel : ve - 1;
        for (int piece = 0; piece < 2; ++piece) {
            if (slot < Plan::NK) ops.push_back({kind, Ring::k_half(rel + 1), 2 * slot + piece, next});
            else ops.push_back({kind, Ring::v_half(rel), 2 * (slot - Plan::NK) + piece, own + VALUES});
        }
    }
    void works(int n_steps) {
        first_keys();
        for (int l = 0; l < LPW / 2; ++l) load(-Ring::K_AHEAD, l);
        for (int l = 0; l < LPW; ++l) load(-1, l);
        wait_loads();
        barrier();
        scores(Ring::FIRST_HALF, 0);
        scores(Ring::k_half(0), vb);
        barrier();                                       // behind the first reads
        for (int rel = 0; rel < n_steps; ++rel) {
            for (int slot = 0; slot < Plan::AHEAD_SLOTS; ++slot) fragment(READ, rel, slot);
            for (int slot = 0; slot < Plan::NSLOT; ++slot) {
                fragment(READ_DONE, rel, slot);
                for (int l = 0; l < LPW; ++l)
                    if (Ring::dma_slot(l, LPW, Plan::NSLOT) == slot) load(rel, l);
                if (slot + Plan::AHEAD_SLOTS < Plan::NSLOT) fragment(READ, rel, slot + Plan::AHEAD_SLOTS);
            }
            wait_loads();                                // behind a step
            barrier();
        }
    }
    void idles(int n_steps) {                            // as f8_group_idle: no rows, or no kblocks
        const bool loads = ve > vb;
        if (loads) {
            first_keys();
            for (int l = 0; l < LPW / 2; ++l) load(-Ring::K_AHEAD, l);
        }
        for (int rel = -1; rel < n_steps; ++rel) {
            for (int l = 0; loads && l < LPW; ++l) load(rel, l);
            wait_loads();
            barrier();
            if (rel < 0) barrier();                      // the idle wave's
        }
    }
};

struct Piece { int kblock = -1, owner = -1, seq = -1, readers = 0; };

// T kblocks; the first `with_rows` of a group's waves have query rows
template <int D, int G>
static int simulate(int T, int with_rows, unsigned seed) {
    using P = Program<D, G>;
    std::srand(seed);
    const int lag = seed % 2 ? 4 : 256;                  // how late loads land that nothing waits for
    const int n_steps = (T + G - 1) / G;
    std::vector<P> prog(8);
    int barriers[8];
    for (int w = 0; w < 8; ++w) {
        const int group = w / P::NW;
        prog[w].wave = w % P::NW;
        prog[w].vb = T * group / G;
        prog[w].ve = T * (group + 1) / G;
        if (prog[w].ve > prog[w].vb && prog[w].wave < with_rows) prog[w].works(n_steps);
        else prog[w].idles(n_steps);
        barriers[w] = 0;
        for (const Op& op : prog[w].ops) barriers[w] += op.kind == BARRIER;
        if (barriers[w] != barriers[0]) {
            std::printf("D %d G %d T %d: wave %d meets %d barriers, wave 0 %d\n", D, G, T, w, barriers[w], barriers[0]);
            return 1;
        }
    }
    constexpr int HALVES = P::Ring::BYTES / P::Ring::KB_BYTES;
    std::vector<Piece> lds(G * HALVES * P::PIECES);
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
        const int w = std::rand() % 8;
        if (pc[w] >= prog[w].ops.size() || waiting[w]) continue;
        for (int o = 0; o < 8; ++o)
            if (landed[o] < issued[o] && std::rand() % lag == 0) ++landed[o];
        const Op op = prog[w].ops[pc[w]];
        if (op.half < 0 || op.half >= HALVES || op.piece < 0 || op.piece >= P::PIECES) {
            std::printf("D %d G %d T %d: wave %d leaves its ring (half stage %d, piece %d)\n", D, G, T, w, op.half, op.piece);
            return 1;
        }
        Piece& f = lds[(size_t(w / P::NW) * HALVES + op.half) * P::PIECES + op.piece];
        if (op.kind == BARRIER) { waiting[w] = 1; continue; }
        if (op.kind == WAIT_LOADS) landed[w] = issued[w];
        if (op.kind == LOAD) {
            if (f.readers > 0) {
                std::printf("D %d G %d T %d: wave %d loads kblock %d over a piece being read\n", D, G, T, w, op.kblock);
                return 1;
            }
            f = Piece{op.kblock, w, ++issued[w], 0};
        }
        if (op.kind == READ) {
            if (f.owner < 0 || landed[f.owner] < f.seq || f.kblock != op.kblock) {
                std::printf("D %d G %d T %d: wave %d reads kblock %d, the piece holds %s kblock %d\n", D, G, T, w, op.kblock,
                            f.owner < 0 ? "no" : landed[f.owner] < f.seq ? "in-flight" : "landed", f.kblock);
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
    std::vector<int> lengths = {15, 16, 17, 31, 47, 64};
    for (int T = 1; T <= 9; ++T) lengths.push_back(T);
    for (int T : lengths)
        for (int with_rows = 1; with_rows <= 8 / G; ++with_rows)
            for (unsigned seed = 1; seed <= 30; ++seed)
                if (simulate<D, G>(T, with_rows, seed * 7919u + T)) return 1;
    return 0;
}

int main() {
    if (check<64, 4>() || check<128, 4>()) return 1;
    std::printf("fp8 group rings ok\n");
    return 0;
}
