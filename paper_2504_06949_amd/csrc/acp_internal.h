// Host-side interface between the C ABI layer and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "acp.h"

namespace acp {

// Per-block statistics of the gate producer (one entry per 64 gates of a head)
// that stage 1's checks need in place of its own pass over log f.
struct GateStats {
    double abs_sum;           // sum of |log f| as a double-double pair (abs_sum, abs_lo)
    double abs_lo;
    int min_lsb;              // smallest float32 ulp exponent of a nonzero gate
    int flags;                // bit 1: a non-finite gate; bit 5: the chained scan timed out
};

struct PlanArgs {
    const void* Q;
    const void* K;
    const float* log_f;
    bool bf16;
    int B, H, L, d;
    int nchunk;               // norm partials per (head, tensor)
    double log_l_over_eps;    // log L - log eps, +inf for eps = 0
    const float* gamma_q;     // [H] QK-norm scale bounds, or null: U from the row norms
    const float* gamma_k;     // [H]
    bool norms_ready;         // part already holds the chunk maxima (the projection's epilogue)
    const GateStats* gate;    // non-null: c is already in place (the gate producer's
                              // epilogue) and these are its per-head statistics
    double* part;             // [B*H, 2, nchunk]
    float* c;                 // [B*H, L]
    double* u;                // [B*H]
    double* delta;            // [B*H]
    int* row_start;           // [B*H, M]
    int* col_end;             // [B*H, M]
    long long* kept;          // [B*H]
    int* flags;               // [B*H]
};

struct GateArgs {
    const void* X;            // [B*L, Dm] bf16 layer inputs
    const void* W;            // [Dm, H] bf16 gate weights
    const float* bias;        // [H]
    int B, L, Dm, H;
    float* log_f;             // [B*H, L]
    float* c;                 // [B*H, L]
    unsigned long long* agg;  // [B*H, L/64, 2] block totals (float64 bits of hi, lo)
    unsigned long long* incl; // [B*H, L/64, 2] inclusive prefixes (float64 bits of hi, lo)
    GateStats* stats;         // [B*H, L/64]
    void* wt;                 // [H, Dm] bf16: the weights transposed
};

// Tables of B*H*nb entries bh * nb + block, nb = ceil(L / 128): per XCD, heads placed by
// kept count when there are few, blocks largest first.
struct ScheduleArgs {
    const long long* kept;    // [BH]
    const int* row_start;     // [BH, M]
    const int* col_end;       // [BH, M]
    int BH, M, nb;
    int* sched_q;             // query blocks (forward, dQ pass)
    int* sched_k;             // key blocks (dK/dV pass)
    int* chain;               // if not null, gets 1 or 0: whether the launch is bound by its
                              // longest block (kChainBound)
};
// Blocks per head from which heads are placed in parts.
constexpr int kLongBlocks = 32;
// Whether the forward takes its blocks without the tables and fills them itself: as many
// blocks as the CUs hold at once (4 per CU at d = 64, 2 at 128), and at d = 128, whose
// blocks take twice as long, short sequences only.  Beyond that the
// tables' order and their keeping of a head on one XCD are worth their kernel.
// Measured, us for the whole forward, tables first -> direct: 48 heads of 1024 tokens 43
// -> 32, 100 of 640 37 -> 34; more blocks, forward kernel alone: 192 of 1024 (1536
// blocks) 43 -> 47, 128 of 2048 (2048) 77 -> 92; d = 128, 32 of 3072 (768) 82 -> 92.
// Long sequences: d = 64, 16 heads of 4096 72 -> 68, 5 of 5184 65 -> 60, 32 of 4096 98 ->
// 91, 24 of 5120 106 -> 104, 12 of 8128 132 -> 130; d = 128, 8 of 8192 155 -> 168.
inline bool forward_direct(int d, int nblocks, int nb) {
    return d == 64 ? nblocks <= 1024 : nblocks <= 512 && nb < kLongBlocks;
}

struct FwdArgs {
    const void* Q;
    const void* K;
    const void* V;
    bool bf16;
    int B, H, L, d;
    const float* c;
    const int* row_start;
    const double* u;          // [B*H] logit bound U
    ScheduleArgs sched;       // the tables
    bool direct;              // the forward fills them itself
    void* O;
    float* lse;
    float* lse2;
};

struct BwdArgs {
    const void* Q;
    const void* K;
    const void* V;
    const void* O;            // the forward's output
    const void* dO;
    bool bf16;
    int B, H, L, d;
    const float* c;
    const int* row_start;
    const int* col_end;
    const float* lse2;
    const int* chain;         // of the schedule, where bwd_groups goes by the plan
    const int* sched_q;       // query-block schedule (dQ pass)
    const int* sched_k;       // key-block schedule (dK/dV pass)
    float* dsum;              // Delta' from the dQ pass
    float* rowsum;
    float* colsum;
    void* dQ;
    void* dK;
    void* dV;
    float* dlog_f;
};

struct ProjectArgs {
    const void* X;            // [B*L, Dm] bf16
    const void* Wq;           // [Dm, H*d] bf16
    const void* Wk;
    int B, L, Dm, H, d;
    void* Q;                  // [B, H, L, d] bf16
    void* K;
    double* part;             // [B*H, 2, nchunk] chunk maxima of the squared row norms
    int nchunk;
};

struct DecodeInitArgs {
    const void* K;            // [B*H, L0, d] prompt keys
    const void* V;
    const float* log_f;       // [B*H, L0]
    const float* gamma_q;     // [H]
    const float* gamma_k;     // [H]
    bool bf16;
    int B, H, L0, C, d;
    double log_lmax_over_eps; // log L_max - log eps, +inf for eps = 0
    void* Kc;                 // [B*H, C, d] ring caches, position j in slot j mod C
    void* Vc;
    float* cc;                // [B*H, C] c of the cached positions
    double* cs;               // [2][B*H][2] running sum of log f, (hi, lo) (copy p mod 2
                              // holds the value after position p)
    int* ptr;                 // [2][B*H] first kept block of query p, likewise
    double* delta;            // [B*H]
    int* flags;               // [B*H]
};

struct DecodeArgs {
    const void* q;            // [B*H, d] the new token
    const void* k;
    const void* v;
    const float* log_f;       // [B*H]
    bool bf16;
    int B, H, t, C, d;        // t: position of the new token
    void* Kc;
    void* Vc;
    float* cc;
    double* cs;
    int* ptr;
    const double* delta;
    int* flags;
    float* part;              // split partials: [B*H, nsplit, 2] (max, sum), then
                              // [B*H, nsplit, d] (unnormalised O)
    void* O;                  // [B*H, d]
    float* lse;               // [B*H]
};

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

// Records the message that acp_last_error() returns and passes the status on.
acp_status set_error(acp_status s, const char* fmt, ...);

// Tracing hooks: no-ops unless acp_timing_enable(1) was called.
void trace_begin(int kernel, hipStream_t s);
void trace_end(int kernel, hipStream_t s);

int norm_chunks(int L);
hipError_t launch_schedule(const ScheduleArgs& a, hipStream_t s);
hipError_t launch_plan(const PlanArgs& a, hipStream_t s);
hipError_t launch_gate(const GateArgs& a, hipStream_t s);
hipError_t launch_fwd(const FwdArgs& a, hipStream_t s);
hipError_t launch_bwd(const BwdArgs& a, hipStream_t s);
hipError_t launch_dq_bf16(const BwdArgs& a, hipStream_t s);
hipError_t launch_dkdv_bf16(const BwdArgs& a, hipStream_t s);
hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t s);
hipError_t launch_dq_f32(const BwdArgs& a, hipStream_t s);
hipError_t launch_dkdv_f32(const BwdArgs& a, hipStream_t s);
hipError_t launch_qk_project(const ProjectArgs& a, hipStream_t s);
size_t decode_partials_floats(int BH, int C, int d);
hipError_t launch_decode_init(const DecodeInitArgs& a, hipStream_t s);
hipError_t launch_decode(const DecodeArgs& a, hipStream_t s);

}  // namespace acp
