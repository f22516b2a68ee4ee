// Launch rules and index maps of the attention kernels' workgroup schedule: plain C++,
// for host and device.
#pragma once

#include <stdint.h>

#ifdef __HIP__
#define ACP_HD __host__ __device__ __forceinline__
#else
#define ACP_HD inline
#endif

namespace acp {

// ---- which (head, 128-row block) a workgroup takes -------------------------------------
// Blocks per head from which heads are placed in parts.
constexpr int kLongBlocks = 32;
constexpr int kHeadsMax = 64;          // heads that are placed
constexpr int kPlaceMax = 256;         // parts that are dealt

// log2 of the parts s per head: enough that the parts make whole rounds over the
// XCDs, 8 (then every XCD has the same share of every head) for at most 16 heads, and
// otherwise no more than 64 parts: a head spread further costs L2 reuse.  A head's
// kept share runs from nearly none to all, so with one or two heads per XCD the
// heaviest XCD decides the time.  Measured, forward: 8 heads of 32768 tokens (d = 128)
// 1956 us undivided, 1200 in 8 parts; 12 heads of 8128 tokens 198 us in bh order, 162
// in 4 parts, 135 in 8.  (48 heads of 16384 dealt back and forth instead of to the least
// loaded XCD: every kernel 2% slower.)  Training step at 4 x 16 heads of 8192 tokens: 1.73 ms
// undivided, 1.77 in 2 parts, 1.83 in 4; 2 x 16 heads of 16384 (d = 128): 5.12 ms in 2
// parts, 5.18 in 4, 5.30 in 8.
// (33 to 63 heads that are no multiple of 8 would make more than 64 parts: in bh order.)
ACP_HD constexpr int schedule_log_parts(int BH, int nb) {
    if (nb < kLongBlocks) return 0;
    int s = 0;
    while (s < 3 && (BH <= 16 || ((BH << s) & 7) != 0 || (BH << (s + 1)) <= kHeadsMax)) ++s;
    return BH << s <= kHeadsMax ? s : BH <= kHeadsMax / 2 ? 3 : 0;
}

// How the parts (1 << lp per head) are placed: 8 to a head, one to each XCD; by load; or not
// at all (bh order).
enum class Placing { kDealt, kByLoad, kNone };
ACP_HD Placing schedule_placing(int BH, int lp) {
    const int NP = BH << lp;
    if (lp == 3 && BH <= kHeadsMax / 2) return Placing::kDealt;   // (NP a multiple of 8, <= kPlaceMax)
    return NP % 8 == 0 && NP <= kHeadsMax ? Placing::kByLoad : Placing::kNone;
}

// Slot of part p (0..7) of the head of that rank, dealt: a slot range of BH per XCD.
ACP_HD int deal_slot(int part, int rank, int BH) { return BH * part + rank; }

// Blocks of part p of a head: every (1 << lp)-th from block p on.
ACP_HD int part_blocks(int p, int lp, int nb) { return (nb >> lp) + (p < (nb & ((1 << lp) - 1)) ? 1 : 0); }

// The slot that holds logical id lid, of NP slots that start at first[0] = 0, first[1], ...
ACP_HD int slot_of(const int* first, int NP, int lid) {
    int slot = 0;
    for (int step = kPlaceMax / 2; step >= 1; step >>= 1)
        if (slot + step < NP && first[slot + step] <= lid) slot += step;
    return slot;
}

// Index, in the head's unsorted order, of block `nth` of a part (placed: bh << lp | part).
ACP_HD int part_index(int placed, int lp, int nth) { return (placed & ((1 << lp) - 1)) + (nth << lp); }

// The range of logical ids of XCD x (workgroups are dealt round-robin to the 8 XCDs)
ACP_HD void schedule_range(int nblocks, int x, int& lo, int& hi) {
    const int q = nblocks >> 3, r = nblocks & 7;
    lo = x * q + (x < r ? x : r);
    hi = lo + q + (x < r ? 1 : 0);
}

// Workgroup i of a forward without the tables (forward_direct): block nb - 1 - i / BH of head
// i % BH + i / BH (mod BH), so that every head's longest blocks start first and its blocks
// are spread over the XCDs (workgroup i runs on XCD i % 8).
ACP_HD int direct_item(int i, int BH, int nb) {
    const int blk = i / BH;
    int bh = i - blk * BH + blk % BH;
    bh -= bh >= BH ? BH : 0;
    return bh * nb + nb - 1 - blk;
}

// ---- launch rules ------------------------------------------------------------------------
// Whether the forward takes its blocks in a fixed order (direct_item) and fills the
// schedule's tables itself, instead of reading its blocks from them: a launch less between
// stage 1 and the forward (4 us and the gap), against the tables' order by kept count and
// their keeping of a head on one XCD.  The line is a measured number of blocks.  (With one
// group of waves per workgroup it is also what the CUs hold at once, 1024 blocks at d = 64
// and 512 at 128; with two groups, fwd_groups, they hold half of that and with four a
// quarter, and the blocks beyond wait their turn.)
// Measured, us for the whole forward, tables first -> direct: 48 heads of 1024 tokens 43
// -> 32, 100 of 640 37 -> 34; more blocks, forward kernel alone: 192 of 1024 (1536
// blocks) 43 -> 47, 128 of 2048 (2048) 77 -> 92; d = 128, 32 of 3072 (768) 82 -> 92.
// Long sequences: d = 64, 16 heads of 4096 72 -> 68, 5 of 5184 65 -> 60, 32 of 4096 98 ->
// 91, 24 of 5120 106 -> 104, 12 of 8128 132 -> 130; d = 128, 8 of 8192 155 -> 168, so there
// short sequences only.
inline bool forward_direct(int d, int nblocks, int nb) {
    return d == 64 ? nblocks <= 1024 : nblocks <= 512 && nb < kLongBlocks;
}

// Key groups (query groups in the dK/dV pass) per workgroup of the bf16 attention
// kernels: G groups of 4 waves share a 128-row block, each taking every G-th tile of
// the other operand, so that a block's serial chain of up to 2 nb tiles gets G times
// shorter when the blocks (nblocks of them, nb per head) are too few to fill the chip.
// The price is that a CU's waves meet at one barrier per step instead of running as
// independent workgroups, so one group stays the better form as soon as there are
// blocks enough.  Measured on heads of unequal length, us with one group -> with G:
//   forward, d = 64 (4 workgroups per CU), G = 2: 512 blocks of nb = 32 66 -> 55, 768 of
//     64 137 -> 116, 1024 of 64 170 -> 145, of 128 312 -> 254; but 768 of 8 27 -> 32, 1024 of
//     32 107 -> 113 (unpruned), 1280 of 32 92 -> 97, 1344 of 56 152 -> 157.  G = 4: 205 of 41
//     73 -> 51 (G = 2: 57), 256 of 128 151 (173); but 512 of 32 56 (55), 768 of 64 126 (116).
//   forward, d = 128 (2 per CU), G = 2: 512 of 32 105 -> 82, 512 of 64 193 -> 139; but 768
//     of 32 111 -> 111, 1024 of 32 127 -> 143.
//   dQ, d = 64 (3 per CU), G = 3: 96 of 8 25 -> 24, 192 of 16 42 -> 35, 512 of 32 82 -> 71,
//     768 of 64 158 -> 143; but 384 of 8 30 -> 33, 1024 of 32 101 -> 121.
//   dQ, d = 128, G = 2: 256 of 8 40 -> 35, 512 of 32 131 -> 106, 512 of 64 244 -> 175; but
//     768 of 32 142 -> 141, 1024 of 32 175 -> 196.
//   dK/dV, d = 64, G = 3: 96 of 8 30 -> 25, 192 of 16 52 -> 38, 512 of 32 102 -> 80, 768 of
//     64 207 -> 160; but 1024 of 32 130 -> 135, 1344 of 56 233 -> 253.  (At d = 128 its
//     LDS holds one group of 8 waves.)
// Below 8 blocks per head the prologue and the merge outweigh the shorter chain.
// Beyond 256 blocks the forms with one workgroup of G groups per CU (the backward's, and
// the d = 128 forward's) run in rounds, which pays only where the longest block sets the
// time: with equal heads of a short window, backward at d = 64, 512 blocks of 32, 33 us with
// one group, 50 with 3, 768 of 64 45 and 73; forward at d = 128, 384 of 32 34 and 42.  There
// both forms are launched and the schedule's `chain` says which one works (`by_plan`); an
// empty launch costs 2 to 3 us.  (The direct forward has no schedule before it: its G = 2
// costs equal heads of a window 640 to 1024 blocks up to 7%.)
struct Groups {
    int groups;
    bool by_plan;   // that many if the launch is bound by its longest block, else one
};
inline Groups fwd_groups(int d, int nblocks, int nb, bool direct) {
    if (nb < 8) return {1, false};
    if (d == 128) return nblocks <= 512 ? Groups{2, !direct && nblocks > 256} : Groups{1, false};
    if (!direct) return {1, false};   // (d = 64: several groups in the direct form only)
    if (nblocks <= 256 && nb >= 16) return {4, false};
    return {nblocks <= 1024 && nblocks <= (nblocks <= 512 ? 32 : 24) * nb ? 2 : 1, false};
}
inline Groups bwd_groups(int d, int nblocks, int nb) {
    if (nb < 8) return {1, false};
    if (d == 128) return nblocks <= 512 ? Groups{2, nblocks > 256} : Groups{1, false};
    return nblocks <= 768 && nblocks <= 16 * nb ? Groups{3, nblocks > 256} : Groups{1, false};
}

}  // namespace acp
