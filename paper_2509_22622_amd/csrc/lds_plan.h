// Issue plan of the LDS fragment reads of one kblock step of the streaming attention kernel, and the
// s_waitcnt counts that go with it.  Plain constexpr C++ so that a host test can replay the plan.
//
// A step has KS + NV slots (KS = D/16 MFMAs of S^T = K Q^T for the next kblock, then NV = D/16 MFMAs of
// O^T += V^T P^T for this one).  Each slot issues its MFMA first, then its reads, V^T reads before K reads, each
// kind in fragment order.  The LDS returns data in issue order, so "at most N reads outstanding" means that every
// read but the N youngest has arrived.
#pragma once

namespace ll {

template <int D>
struct LdsPlan {
    static constexpr int KS = D / 16;    // K fragments per kblock = slots of the first MFMA group
    static constexpr int NV = D / 16;    // V^T fragments per kblock = slots of the second MFMA group
    // V^T fragment f of this step's kblock is read in slot f / 2: before slot KS + f needs it, after the step
    // before has used the register (its slot KS + f).
    static constexpr int vslot(int f) { return f / 2; }
    // K fragment f of the next kblock is read in slot KS + f / 2: after slot f of this step has used the register.
    static constexpr int kslot(int f) { return KS + f / 2; }
    // Reads issued after V^T fragment g when slot KS + g starts (its MFMA consumes the fragment): the later V^T
    // reads and the K reads of earlier slots.
    static constexpr int wait_v(int g) {
        int c = 0;
        for (int f = 0; f < NV; ++f) c += vslot(f) > vslot(g) || (vslot(f) == vslot(g) && f > g);
        for (int f = 0; f < KS; ++f) c += kslot(f) < KS + g;
        return c;
    }
    // Reads issued after K fragment ks (read in the step before) when slot ks starts: the later K reads of that
    // step and the V^T reads of this step's earlier slots.
    static constexpr int wait_k(int ks) {
        int c = 0;
        for (int f = 0; f < KS; ++f) c += kslot(f) > kslot(ks) || (kslot(f) == kslot(ks) && f > ks);
        for (int f = 0; f < NV; ++f) c += vslot(f) < ks;
        return c;
    }
};

// The plan of the same kernel built on 16x16x32 MFMAs (attn_stream16.hip).  A step has the same KS + NV slots, each
// now opened by the two MFMAs that share a fragment: slot k < KS takes K fragment k; the O^T slots run over the
// V^T fragments twice, slot KS + j taking fragments 2 j and 2 j + 1 for the first query block (j < NV / 2) and slot
// KS + NV / 2 + j the same two for the second.  Reads are issued as above (V^T fragment f in slot f / 2, K fragment
// f of the next kblock in slot KS + f / 2, after the slot's MFMAs, V^T before K, in fragment order).  A fragment is
// waited for at its first use only; the younger of a slot's two V^T fragments carries the wait for both.
// SPREAD: one read per slot instead (V^T fragment f in slot f, K fragment f in slot KS + f).
template <int D, bool SPREAD = false>
struct LdsPlan16 {
    static constexpr int KS = D / 16;
    static constexpr int NV = D / 16;
    static constexpr int vslot(int f) { return SPREAD ? f : f / 2; }
    static constexpr int kslot(int f) { return SPREAD ? KS + f : KS + f / 2; }
    static constexpr int first_use_v(int f) { return KS + f / 2; }            // slot of the first query block
    static constexpr int last_use_v(int f) { return KS + NV / 2 + f / 2; }    // slot of the second query block
    // Reads issued after V^T fragment 2 j + 1 when slot KS + j starts.
    static constexpr int wait_v(int j) {
        const int g = 2 * j + 1;
        int c = 0;
        for (int f = 0; f < NV; ++f) c += vslot(f) > vslot(g) || (vslot(f) == vslot(g) && f > g);
        for (int f = 0; f < KS; ++f) c += kslot(f) < KS + j;
        return c;
    }
    // Reads issued after K fragment k (read in the step before) when slot k starts.
    static constexpr int wait_k(int k) {
        int c = 0;
        for (int f = 0; f < KS; ++f) c += kslot(f) > kslot(k) || (kslot(f) == kslot(k) && f > k);
        for (int f = 0; f < NV; ++f) c += vslot(f) < k;
        return c;
    }
};

// The same for the kernel of the 8-bit cache.  A step has NK = 2 * D/64 slots of S^T MFMAs (for the next kblock)
// and DB = D/32 slots of O^T MFMAs (for this one); every MFMA consumes one operand fragment, read with two 16-byte
// LDS reads.  Slot k issues its MFMA first and then the two reads of the fragment that slot k + AHEAD_SLOTS needs
// (slots past the end of the step are the first slots of the next step), into register buffer
// (k + AHEAD_SLOTS) % BUFFERS.  So exactly (AHEAD_SLOTS - 1) fragments are issued between a fragment's reads and
// its use, and one wait count serves every slot.  A buffer is rewritten BUFFERS - AHEAD_SLOTS slots after the MFMA
// that used it was issued: two slots, i.e. after one more MFMA of the same wave has entered the matrix pipe behind it.
template <int D>
struct Fp8LdsPlan {
    static constexpr int NK = 2 * (D / 64);
    static constexpr int DB = D / 32;
    static constexpr int NSLOT = NK + DB;
    static constexpr int AHEAD_SLOTS = 2;
    static constexpr int BUFFERS = 4;
    static constexpr int READS_PER_FRAGMENT = 2;
    static constexpr int buffer(int slot) { return slot % BUFFERS; }
    // reads issued after a fragment's own when its slot starts
    static constexpr int wait() { return (AHEAD_SLOTS - 1) * READS_PER_FRAGMENT; }
    static_assert(NSLOT % BUFFERS == 0, "the buffer of a slot must not depend on the step");
    static_assert(AHEAD_SLOTS < BUFFERS, "a fragment would be read into a buffer still in use");
};

// The rings of a workgroup of the 8-bit kernel whose waves are dealt into G key groups (attn_fp8.hip, G = 4): a group's walk their
// share of the kblocks through two half stages of keys and two of values.  The step for kblock i reads V of i and K of i + 1 and
// issues the loads of V of i + 1 and K of i + 2, over the half stages that the step before has read; behind it a wave waits for
// all it has issued and meets the others at a barrier.  Nothing is read ahead across that.  The prologue loads K of a share's first two
// kblocks and V of the first, and the keys of the tile's first kblock to where V of the share's second will be; it reads those and the
// share's first keys between two barriers.
template <int D, int G>
struct Fp8GroupRing {
    static constexpr int KB_BYTES = 64 * D, BYTES = 4 * KB_BYTES;
    static_assert(G * BYTES <= 128 * 1024, "the rings of a workgroup");
    static constexpr int K_AHEAD = 2, V_AHEAD = 1;               // kblocks from a step to those it loads
    static constexpr int k_half(int rel) { return rel & 1; }     // half stage of a share's rel-th kblock
    static constexpr int v_half(int rel) { return 2 + (rel & 1); }
    static constexpr int FIRST_HALF = v_half(1);
    static constexpr int dma_slot(int l, int n, int slots) { return l * slots / n / 2; }         // in the step's first half
};

// The ring of K/V stages in LDS and its hand-over between the waves of a workgroup.
//   Kblock v lives in stage v % STAGES.  The prologue issues the loads of the first AHEAD kblocks; step i issues
//   those of kblock i + AHEAD, and reads kblock i (V^T) and kblock i + 2 (K for the scores of the step after next;
//   the prologue reads kblocks 0 and 1).  Every wave loads its own fragments of a stage.  Before each barrier a wave
//   waits until all but its youngest (AHEAD - LANDED) kblocks of loads have arrived; barriers stand after the
//   prologue's loads and after every step with an odd index.
struct RingPlan {
    static constexpr int STAGES = 8;   // a power of two
    static constexpr int AHEAD = 6;    // kblocks the loads run ahead of the step that issues them
    static constexpr int LANDED = 4;   // kblocks, counted from the next step, that have arrived at a barrier
    static constexpr bool barrier_after(int step) { return step & 1; }
};

// The rings of a workgroup whose waves are dealt into G key groups (G = 2, 4, 8; attn_stream16.hip): a group's 8 / G
// waves walk their own share of the kblocks through a ring of their own, 128 KB / G at most.  Keys and values have
// separate rings of DEPTH half stages (kblock v in half stage v % DEPTH), because the step for kblock i reads V^T of i
// but K of i + 2.  Loads, waits and barriers come in periods of PERIOD steps: in its first step a period issues the
// loads of the next one (V of its kblocks, K two kblocks further on), at its end a wave waits for all it has issued,
// LDS reads included, and meets the group's other waves at a barrier.  The K of a share's first two kblocks goes straight
// to registers, so the ring starts with the third.
template <int D, int G>
struct GroupRing {
    static constexpr int PERIOD = G * D <= 256 ? 2 : 1;
    static constexpr int DEPTH = 2 * PERIOD;
    static constexpr int BYTES_KBLOCK = 32 * D * 2, BYTES = 2 * DEPTH * BYTES_KBLOCK;
    static_assert(G * BYTES <= 128 * 1024, "the rings of a workgroup");
    // slot of a period's first step behind whose MFMAs load l of n is issued: spread over the step, or, where that step
    // is the whole period, over its first half (they have to land within it)
    static constexpr int dma_slot(int l, int n, int slots) { return l * slots / n / (PERIOD == 1 ? 2 : 1); }
    // Keys that come from memory.  Where a period is one step its loads have half of it to land: enough for L2, not for memory, and
    // the LDS has no room for longer rings.  So one 4-byte load a lane, 128 bytes apart, brings the kblocks of the period
    // TOUCH_AHEAD periods on into L2 (and into LDS_TOUCH bytes a wave that nobody reads).  A head's tiles on an XCD take turns,
    // since a wave's next wait is for the touch too.  Periods of two steps gain less and lose more where the keys are in the
    // last-level cache (G = 4 at head_dim 64: 39 -> 33 us from memory, but 40 -> 43 from there; G = 2 75.1 -> 74.5 and 67 -> 69), and
    // launches with eight groups are too short (5 us of 25 at 300 rows x 24 heads x 64, but 0.2 of 8 lost at 180 x 4).
    static constexpr bool TOUCHES = G == 4 && PERIOD == 1;
    // TOUCH_LOADS of a wave, its last in front of a hand-over, may still be in flight behind it.
    static constexpr int TOUCH_AHEAD = 4, TOUCH_LOADS = 1, TOUCH_LANES = PERIOD * 2 * BYTES_KBLOCK / 128, LDS_TOUCH = 64 * 4;
    static_assert(!TOUCHES || TOUCH_LANES == 64 * (8 / G), "one load a wave");
};

// Whether the resident-key attention kernel (attn_resident.hip: one workgroup per CU, which first brings a head's keys and
// values in) has its workgroups fill the chip, or the streaming kernels, whose rows split finer, are to take a launch.
// Up to 128 heads each gets several workgroups, and the kernel was faster at 12 to 128 heads x 300 to 4680 rows (2 % slower
// at 86 heads x 4680 x 400 keys x 64).  Above, a head is one workgroup and the last of the rounds may be nearly empty; us, streaming
// and resident at 400 keys x 64: 129 heads x 4680 rows 109 and 145, 257 x 1170 64 and 87, but 200 x 4680 165 and 152,
// 1000 x 4680 854 and 652.  At few rows the streaming kernels' latency counts more (129 x 300 25 and 16), and at two kblocks of
// keys, as far as measured, what they do around them (129 x 4680 x 64 keys x 128 114 and 72, 257 heads 187 and 161).
constexpr bool resident_fills_chip(int heads, int rows, int n_kblocks) {
    if (heads <= 128 || n_kblocks <= 2) return true;
    if (heads <= 256 && rows <= 512) return true;
    return 4 * heads >= 3 * ((heads + 255) / 256 * 256);         // three quarters of the CUs over the rounds
}

}  // namespace ll
