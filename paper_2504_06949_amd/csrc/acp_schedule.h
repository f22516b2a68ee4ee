// Workgroup schedule of the attention kernels: which (head, 128-row block) each
// logical workgroup id takes.
#pragma once

#include "acp_device.h"
#include "acp_internal.h"

namespace acp {

// The attention kernels' workgroups each take 128 query rows (forward, dQ) or
// 128 keys (dK/dV) of one head.  Workgroup ids are dealt round-robin to the 8
// XCDs; xcd_logical_id turns that into a contiguous range of logical ids per XCD,
// and the tables say, per XCD range, which (head, block) each logical id takes, so
// that
//   - a head's workgroups run on one XCD (its K and V stay in one L2), or, when
//     there are few long heads of unequal work, on as few as a balanced load allows;
//   - at most kHeadsMax heads whose number is a multiple of 8 are placed by kept-block
//     count, largest first, each on the least loaded XCD that still has room (the same
//     number per XCD).
//     (With more heads an XCD has several of them, and reading the counts first
//     costs this kernel 3 us: 96 heads of 4096 tokens 6.4 -> 9.3, the forward 187
//     either way.)
//   - long heads (32 or more of the 128-row blocks) are placed in parts, every s-th of a
//     head's blocks (schedule_log_parts), unless whole heads already load the XCDs
//     evenly (schedule_even); 8 parts per head are simply dealt out, one to each XCD;
//   - otherwise (other numbers of heads) they stay in bh order;
//   - inside each XCD range the workgroups run largest first (a counting sort
//     on their kept-tile counts), so that the range ends on small ones.
// Entry = bh * nb + block.  Equal counts keep no particular order.

// Heads of equal work gain nothing from parts and pay for them in L2: unpruned, 16 heads of
// 16384 tokens (d = 128) forward 1034 us in whole heads, 1161 in parts, backward 3169 and
// 3472; 32 of 8192 549 and 590; 20 of 8192 (d = 64), each pruned to 3 tiles per row, 44 and 51.
// So they are divided only if the heaviest XCD would carry more than this over the average.
// 100 mixes of heads, in parts against whole: in 2 or 4 parts up to 1.06 over the average 0 to 12%
// slower, from 1.10 on 0 to 6% faster (20 unpruned heads); in 8 parts, where every XCD reads
// every head, up to 1.10 0 to 16% slower (14 heads of 8192 with a window, d = 128, forward 272
// and 228 us), from 1.15 on even or up to 10% faster.
__device__ __forceinline__ float schedule_even_load(int log_parts) { return log_parts == 3 ? 1.105f : 1.08f; }

// Whether the longest block, not the sum of all, sets the time of a launch whose blocks are
// all resident with one group of waves each: from the longest last row against the mean
// over all rows, in tiles, on.  Heads of one window have a ratio of 1 to 1.5, unpruned ones
// 2, heads of unequal length more.
constexpr float kChainBound = 1.6f;

struct ScheduleSmem {
    int sorted[kHeadsMax];                           // kept counts, largest first
    int load[8];                                     // kept tiles per XCD
    int place[kPlaceMax];                            // part of each slot: bh * parts + part
    int first[kPlaceMax + 1];                        // first logical id of each slot
    __attribute__((aligned(16))) int kept[kPlaceMax];
    int more[kPlaceMax / 64];
    int hist[2 * kMaxBlocks + 2];                    // a block's count is at most 2M <= 4096
    int wave[16];
};

// Kept tiles of a 128-row block in table 0 (queries) or 1 (keys)
__device__ __forceinline__ int schedule_work(const ScheduleArgs& a, int table, int bh, int blk) {
    int work = 0;
    for (int u = 0; u < 2; ++u) {
        const int m = 2 * blk + u;
        if (m < a.M) {
            work += table == 0 ? m - a.row_start[(size_t)bh * a.M + m] + 1
                               : a.col_end[(size_t)bh * a.M + m] - m + 1;
        }
    }
    return work;
}

// Whether whole heads load the XCDs evenly: BH a multiple of 8, sorted by count and dealt
// back and forth (placing them by load does no worse); else the ranges of the bh order,
// summed block by block.  sm.kept holds the counts; the answer is uniform and the same in
// every workgroup of the table.
template <int THREADS, typename Rank>
__device__ __forceinline__ bool schedule_even(ScheduleSmem& sm, const ScheduleArgs& a, int table,
                                              float most_load, Rank rank_of) {
    const int t = threadIdx.x, lane = t & 63, BH = a.BH;
    if (BH % 8 == 0) {
        if (t < BH) sm.sorted[rank_of(t)] = sm.kept[t];
        __syncthreads();
        if (t < 8) {
            int sum = 0;
            for (int j = 0; 8 * j < BH; ++j) sum += sm.sorted[8 * j + (j & 1 ? 7 - t : t)];
            sm.load[t] = sum;
        }
    } else {
        for (int x = t >> 6; x < 8; x += THREADS / 64) {
            int lo, hi, sum = 0;
            schedule_range(BH * a.nb, x, lo, hi);
            for (int lid = lo + lane; lid < hi; lid += 64) {
                const int idx = lid % a.nb;
                sum += schedule_work(a, table, lid / a.nb, table == 0 ? a.nb - 1 - idx : idx);
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == 0) sm.load[x] = sum;
        }
    }
    __syncthreads();
    int most = 0;
    float total = 0.f;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        most = max(most, sm.load[x]);
        total += (float)sm.load[x];
    }
    return 8.f * (float)most <= most_load * total;
}

// Table 0 (query blocks) or 1 (key blocks) for XCD x, by a workgroup of THREADS.
template <int THREADS>
__device__ __forceinline__ void schedule_table(ScheduleSmem& sm, const ScheduleArgs& a, int x, int table) {
    const int t = threadIdx.x, BH = a.BH, M = a.M, nb = a.nb;
    const long long* kept = a.kept;
    // the head's rank by kept count (largest first, ties by index)
    auto rank_of = [&](int bh) {
        const int mine = sm.kept[bh];
        int rank = 0;
        for (int j = 0; j < BH; j += 4) {   // (padded with -1)
            const int4 k = *reinterpret_cast<const int4*>(&sm.kept[j]);
            rank += (k.x > mine || (k.x == mine && j < bh)) ? 1 : 0;
            rank += (k.y > mine || (k.y == mine && j + 1 < bh)) ? 1 : 0;
            rank += (k.z > mine || (k.z == mine && j + 2 < bh)) ? 1 : 0;
            rank += (k.w > mine || (k.w == mine && j + 3 < bh)) ? 1 : 0;
        }
        return rank;
    };
    static_assert(THREADS >= kPlaceMax, "a thread per part");
    if (a.chain != nullptr && x == 0 && table == 0 && t >= THREADS - 64) {   // (the last wave)
        int longest = 0;
        float total = 0.f;
        for (int h = t & 63; h < BH; h += 64) {
            longest = max(longest, M - a.row_start[(size_t)h * M + M - 1]);
            total += (float)kept[h];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            longest = max(longest, __shfl_xor(longest, off));
            total += __shfl_xor(total, off);
        }
        if ((t & 63) == 0) *a.chain = (float)longest * (float)BH * (float)M >= kChainBound * total ? 1 : 0;
    }
    if (BH <= kHeadsMax && (BH % 8 == 0 || schedule_log_parts(BH, nb) > 0) && t < kPlaceMax)
        sm.kept[t] = t < BH ? (int)min(max(kept[t], 0ll), 1ll << 22) : -1;
    __syncthreads();
    int lp = schedule_log_parts(BH, nb);                 // (0 beyond kHeadsMax heads)
    if (lp > 0 && schedule_even<THREADS>(sm, a, table, schedule_even_load(lp), rank_of)) lp = 0;
    const int parts = 1 << lp, NP = BH << lp;
    const Placing placing = schedule_placing(BH, lp);
    const bool deal = placing == Placing::kDealt, greedy = placing == Placing::kByLoad;
    if (deal) {
        // slot (NP / 8) j + i: part j of the head of rank i
        if (t < NP) sm.place[deal_slot(t & 7, rank_of(t >> 3), BH)] = t;
    } else if (greedy && t < 64) {
        // Wave 0 alone.  Lane j of 0-7 holds XCD j as the key load << 3 | j; each step
        // the key that equals the minimum over the 8 lanes (the least loaded XCD with
        // room, lowest index on ties) takes the part, and its lane writes the slot.  A
        // head keeps at most M (M + 1) / 2 < 2^22 blocks and an XCD holds at most 8
        // parts, so the key fits 32 bits.
        if (t < NP) sm.first[(rank_of(t >> lp) << lp) + (t & (parts - 1))] = t;
        // (a single wave's LDS accesses complete in order: no barrier)
        const int hd_l = t < NP ? sm.first[t] : 0;
        const int k_l = t < NP ? sm.kept[hd_l >> lp] << 3 : 0;
        asm volatile("" : : "v"(hd_l), "v"(k_l));   // (waits for the LDS reads here, not in the loop)
        const int per = NP / 8;
        if (t < 8) {
            unsigned key = (unsigned)t;
            int pos = per * t;
            const int end = pos + per;
            for (int i = 0; i < NP; ++i) {
                const unsigned k_i = (unsigned)__builtin_amdgcn_readlane(k_l, i);
                const int hd_i = __builtin_amdgcn_readlane(hd_l, i);
                // minimum over the 8 lanes: swap neighbours, pairs, quads
                unsigned mn = min(key, (unsigned)__builtin_amdgcn_mov_dpp((int)key, 0xB1, 0xF, 0xF, false));
                mn = min(mn, (unsigned)__builtin_amdgcn_mov_dpp((int)mn, 0x4E, 0xF, 0xF, false));
                mn = min(mn, (unsigned)__builtin_amdgcn_mov_dpp((int)mn, 0x141, 0xF, 0xF, false));
                const bool mine = key == mn;
                // (the others write a spare word)
                (mine ? &sm.place[pos] : &sm.kept[kPlaceMax - 1])[0] = hd_i;
                pos += mine ? 1 : 0;
                key = pos == end ? 0xffffffffu : key + (mine ? k_i : 0u);
            }
        }
    }
    if (lp > 0 && (deal || greedy)) {
        // first logical id of slot t: t parts of nb >> lp blocks, and one more for those
        // before it that have the extra block
        __syncthreads();
        const bool more = t < NP && part_blocks(sm.place[t] & (parts - 1), lp, nb) > (nb >> lp);
        const unsigned long long bal = __ballot(more);
        if (t < kPlaceMax && (t & 63) == 0) sm.more[t >> 6] = __popcll(bal);
        __syncthreads();
        if (t < NP) {
            int first = t * (nb >> lp) + __popcll(bal & ((1ull << (t & 63)) - 1ull));
            for (int w = 0; w < (t >> 6); ++w) first += sm.more[w];
            sm.first[t] = first;
        }
    }
    const int nbins = 2 * M + 2;
    for (int i = t; i < nbins; i += THREADS) sm.hist[i] = 0;
    __syncthreads();

    int lo, hi;   // this XCD's range of logical ids
    schedule_range(BH * nb, x, lo, hi);
    int* out = table == 0 ? a.sched_q : a.sched_k;
    // the item of a logical id in the unsorted order and its kept-tile count
    auto item = [&](int lid, int& work) {
        int bh, idx;
        if (lp > 0 && (deal || greedy)) {
            const int slot = slot_of(sm.first, NP, lid);
            bh = sm.place[slot] >> lp;
            idx = part_index(sm.place[slot], lp, lid - sm.first[slot]);
        } else {
            const int slot = lid / nb;
            bh = deal || greedy ? sm.place[slot] : slot;
            idx = lid % nb;
        }
        const int blk = table == 0 ? nb - 1 - idx : idx;   // longest rows / first keys first
        work = schedule_work(a, table, bh, blk);
        return bh * nb + blk;
    };
    for (int lid = lo + t; lid < hi; lid += THREADS) {
        int work;
        item(lid, work);
        atomicAdd(&sm.hist[work], 1);
    }
    __syncthreads();
    // Start of each count's run, largest count first: the bins in descending order,
    // thread t owning positions [per t, per t + per) of that order.
    {
        const int per = (nbins + THREADS - 1) / THREADS;
        const int e0 = min(per * t, nbins), e1 = min(e0 + per, nbins);
        int tot = 0;
        for (int e = e0; e < e1; ++e) tot += sm.hist[nbins - 1 - e];
        int incl = tot;   // over the wave, then the waves before
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if ((t & 63) >= off) incl += v;
        }
        if ((t & 63) == 63) sm.wave[t >> 6] = incl;
        __syncthreads();
        int run = lo + incl - tot;
        for (int w = 0; w < (t >> 6); ++w) run += sm.wave[w];
        for (int e = e0; e < e1; ++e) {
            const int cnt = sm.hist[nbins - 1 - e];
            sm.hist[nbins - 1 - e] = run;
            run += cnt;
        }
    }
    __syncthreads();
    for (int lid = lo + t; lid < hi; lid += THREADS) {
        int work;
        const int it = item(lid, work);
        out[atomicAdd(&sm.hist[work], 1)] = it;
    }
}

// In the kernels whose workgroups hold several groups of waves (fwd_groups, bwd_groups): a
// block of up to this many tiles is taken by one group, without the merge: with 2 to 3 tiles
// per row, d = 64, 128 blocks backward 28 -> 24 us, forward 20.1 -> 20.0, 256 34 -> 30 and 25 ->
// 24; 9 tiles instead of 6 are no better (2 groups 21.3 us, one 22.4).
constexpr int kSoloTiles = 6;

}  // namespace acp
