// Forget-gate producer with the cumulative gates in its epilogue (Sec. 2: each
// head's gate is f_t = sigmoid(w_f^T x_t + b_f) of the layer input, and the
// FlashAttention form of Forgetting Attention needs c = cumsum(log f); Sec. 3,
// "Two-stage implementation": stage 1 then only has to read c).
//
// gate_kernel: one workgroup per (sequence b, 64-token block).
//   * Gate logits a = w_f^T x + b_f: every (token, head) sums its products in
//     float32 in ascending feature order (a product of two bfloat16 values is exact
//     in float32, so every step rounds once), the bias added last.  Token rows and
//     weights (transposed by the set-up kernel) stream through LDS.
//     log f = -softplus(-a) in float64, rounded once.
//   * c: a scan of the block's 64 gates per head (float64 while they span under
//     53 bits, else double-double), then a double-double chained scan across
//     the blocks of the sequence (decoupled look-back): each wave
//     first publishes its block total, then walks back over earlier blocks,
//     adding their totals until it meets one whose inclusive prefix is
//     published, and publishes its own.  The whole wave walks: 64 earlier
//     blocks per round.  Whenever the partial sums span at most 105 bits every
//     double-double sum here is exact, so c, the float32 rounding of the pair,
//     is that of the exact prefix sum whatever the association (the span is
//     checked from the statistics below, as stage 1 does).
//   * Per-block statistics for stage 1's checks: the sum of |log f| (a pair),
//     the smallest float32 ulp exponent, and flags (a non-finite gate, a
//     time-out below), written by each block to a slot of its own (stage 1
//     reduces them; same-address atomics from every block of a sequence would
//     serialise).
// A descriptor is a pair of words holding the raw float64 bits of hi and lo; a
// signalling-NaN pattern that no arithmetic produces marks a word "not
// published yet" (gate_init_kernel sets it before every call).  Each word is
// published by an agent-scope 64-bit store and read by an agent-scope load, and
// a reader takes a descriptor only once both words are published, so no fence
// is needed (the values are the message).  Blocks of one sequence wait
// only on blocks with lower workgroup ids, which were dispatched before them;
// the wait is bounded all the same, and on a time-out the wave sets flag bit 5
// and goes on, so every wave ends.
#include "acp_device.h"
#include "acp_internal.h"
#include "acp_scan.h"

namespace acp {

constexpr unsigned long long kUnpublished = 0x7FF4ACB0DEAD0001ull;   // a signalling NaN
constexpr int kGateSpinLimit = 1 << 22;

// Set-up before every call: descriptor words unpublished, and the weights transposed
// to [head][feature], so that the producer's loads of a tile are whole 16-byte pieces.
__global__ __launch_bounds__(256) void gate_init_kernel(unsigned long long* __restrict__ agg,
                                                        unsigned long long* __restrict__ incl,
                                                        int nwords,
                                                        const unsigned short* __restrict__ W,
                                                        unsigned short* __restrict__ wt, int Dm,
                                                        int H) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < H * Dm) wt[(size_t)(i % H) * Dm + i / H] = W[i];
    if (i < nwords) {
        agg[i] = kUnpublished;
        incl[i] = kUnpublished;
    }
}

__device__ __forceinline__ void publish(unsigned long long* w, DD v) {
    __hip_atomic_store(w, (unsigned long long)__double_as_longlong(v.hi), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, (unsigned long long)__double_as_longlong(v.lo), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const unsigned long long* w) {
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double bits_f64(unsigned long long b) {
    return __longlong_as_double((long long)b);
}

// A workgroup of 4 waves takes one (sequence b, 64-token block) for every head; wave
// w forms the logits of tokens 16 w .. + 15.  The block's token rows and the weights
// stream through LDS 64 features at a time (double-buffered, each tile loaded once,
// coalesced, by the whole workgroup, two tiles ahead in named registers: an indexed
// array of them was placed in scratch memory).
//
// The logits' reduction order is fixed (ascending features, every step rounded once),
// so each (token, head) is one chain of d_model dependent multiply-adds, and the kernel
// is bound by how few instructions and cycles a feature takes:
//   * up to 20 heads, on the VALU: lane l takes token 16 w + l / 4 and the N heads
//     l % 4 + 4 q, with the weights as float32 in LDS: one conversion and N multiply-adds
//     per feature, all operands per lane (no broadcast).
//   * more heads, on the matrix cores, one feature at a time:
//     v_mfma_f32_4x4x1_16b_f32, whose 16 independent 4 x 4 blocks are one rounded
//     multiply-add per element (checked against fmaf bit for bit over cancelling,
//     subnormal and mixed magnitudes).  Block 4 i + j takes tokens 4 i .. + 3 of the wave
//     and heads 4 j .. + 3 of a group of 16: lane l holds the features of token
//     4 (l / 16) + l % 4 and the weights of head l % 16, and ends with the logits of tokens
//     4 (l / 16) + (0..3), head l % 16.  A dependent one takes about 44 cycles, whatever the
//     number of heads in its group of 16, which is why fewer go to the VALU: 4096 tokens
//     of d_model 4096, 20 heads 112 us there, 21 to 32 on the matrix cores 143.  Only groups
//     that hold heads are formed: 48 heads 186 us in 3 groups, 258 in 4.
//
// Measured with the set-up kernel (event timing, us) against the earlier form (a lane per
// token and 4 heads per wave, weights broadcast from LDS, one look-back after the other):
// 32768 tokens of d_model 768: 4 heads 33.7 -> 24.0, 8 38.6 -> 29.3, 12 41.9 -> 36.0, 16
// 44.4 -> 41.8, 20 59 -> 46, 33 81 -> 77, 48 97 -> 87 (the last three by graph replay); 1088 tokens of 1088, 24 heads 62.2 -> 54.0.  12 heads on
// the matrix cores: 38.5.  X alone is 50 MB, 10 us at the copy rate; 20 of the 36 us are the
// two launches, log f and the look-back (measured at d_model 64).
constexpr int kGateThreads = 256;
constexpr int kGateTile = 64;          // features per tile (d_model % 64 == 0)
constexpr int kGateRow = 72;           // bf16 per LDS row (144 bytes: 16 rows cover all banks)
constexpr int kGateWRow = 68;          // floats per LDS row of VALU weights (272 bytes: 4 rows
                                       // in 4 different bank groups)
constexpr int kGateLogitRow = 68;      // floats per head of the staged logits

// the exact float32 of the low / high bfloat16 of a word
__device__ __forceinline__ float bf16_lo(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(unsigned x) { return __uint_as_float(x & 0xffff0000u); }

// N: heads per lane (VALU), or groups of 16 heads (kMfma)
template <int N, bool kMfma>
__global__ __launch_bounds__(kGateThreads) void gate_kernel(
    const __bf16* __restrict__ X, const __bf16* __restrict__ wt_g,
    const float* __restrict__ bias, int L, int Dm, int H, int nblk,
    float* __restrict__ log_f, float* __restrict__ c, unsigned long long* __restrict__ agg,
    unsigned long long* __restrict__ incl, GateStats* __restrict__ st) {
    constexpr int kWRows = (kMfma ? 16 : 4) * N;           // weight rows of a tile (heads past H zero)
    constexpr int kWPer = (kWRows * 8 + kGateThreads - 1) / kGateThreads;   // 16-byte pieces per thread
    constexpr int kXBytes = 64 * kGateRow * 2;
    constexpr int kWBytes = kWRows * (kMfma ? kGateRow * 2 : kGateWRow * 4);
    __shared__ __attribute__((aligned(16))) unsigned char gsm[2 * (kXBytes + kWBytes)];
    static_assert(sizeof(gsm) >= kWRows * kGateLogitRow * sizeof(float), "staged logits");
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x % nblk, b = blockIdx.x / nblk;
    const int tok = 64 * blk + lane;
    const int ntile = Dm / kGateTile;
    const __bf16* xsrc = X + ((size_t)b * L + 64 * blk) * Dm;   // the block's 64 rows

    // Tile t: 512 pieces of 16 bytes of X (row p / 8, part p % 8) and 8 H of the weights;
    // thread tid takes pieces tid, tid + 256, ...
    struct Pieces {
        uint4 x0, x1, w0, w1;
    };
    auto fetch = [&](int t) __attribute__((always_inline)) {
        Pieces r;
        const int row = tid >> 3, part = 8 * (tid & 7) + kGateTile * t;
        r.x0 = *reinterpret_cast<const uint4*>(xsrc + (size_t)row * Dm + part);
        r.x1 = *reinterpret_cast<const uint4*>(xsrc + (size_t)(row + 32) * Dm + part);
        r.w0 = make_uint4(0u, 0u, 0u, 0u);
        r.w1 = r.w0;
        if (row < H) r.w0 = *reinterpret_cast<const uint4*>(wt_g + (size_t)row * Dm + part);
        if (kWPer > 1 && row + 32 < H)
            r.w1 = *reinterpret_cast<const uint4*>(wt_g + (size_t)(row + 32) * Dm + part);
        return r;
    };
    auto stash = [&](const Pieces& r, int buf) __attribute__((always_inline)) {
        const int row = tid >> 3, part = 16 * (tid & 7);
        unsigned char* xb = gsm + buf * kXBytes;
        unsigned char* wb = gsm + 2 * kXBytes + buf * kWBytes;
        *reinterpret_cast<uint4*>(xb + row * kGateRow * 2 + part) = r.x0;
        *reinterpret_cast<uint4*>(xb + (row + 32) * kGateRow * 2 + part) = r.x1;
        if constexpr (kMfma) {
            if (row < kWRows) *reinterpret_cast<uint4*>(wb + row * kGateRow * 2 + part) = r.w0;
            if (kWPer > 1 && row + 32 < kWRows)
                *reinterpret_cast<uint4*>(wb + (row + 32) * kGateRow * 2 + part) = r.w1;
        } else if (row < kWRows) {
            float* f = reinterpret_cast<float*>(wb) + row * kGateWRow + 8 * (tid & 7);
            *reinterpret_cast<float4*>(f) = make_float4(bf16_lo(r.w0.x), bf16_hi(r.w0.x), bf16_lo(r.w0.y), bf16_hi(r.w0.y));
            *reinterpret_cast<float4*>(f + 4) = make_float4(bf16_lo(r.w0.z), bf16_hi(r.w0.z), bf16_lo(r.w0.w), bf16_hi(r.w0.w));
        }
    };

    // ---- logits: float32, ascending feature order -----------------------------
    f32x4 acc[N];   // (VALU: element 0 alone)
#pragma unroll
    for (int g = 0; g < N; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the lane's token of the wave's 16 and its head of 16 (of 4 on the VALU)
    const int ltok = kMfma ? 4 * (lane >> 4) + (lane & 3) : lane >> 2;
    const int lhead = kMfma ? lane & 15 : lane & 3;
    auto products = [&](int buf) __attribute__((always_inline)) {
        const unsigned char* xrow = gsm + buf * kXBytes + (16 * w + ltok) * kGateRow * 2;
        const unsigned char* wb = gsm + 2 * kXBytes + buf * kWBytes;
        if constexpr (kMfma) {
            const unsigned char* wrow = wb + lhead * kGateRow * 2;
#pragma unroll
            for (int k = 0; k < kGateTile / 8; ++k) {
                const uint4 xv = *reinterpret_cast<const uint4*>(xrow + 16 * k);
                const unsigned xw[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
                for (int g = 0; g < N; ++g) {
                    const uint4 wv = *reinterpret_cast<const uint4*>(wrow + 16 * g * kGateRow * 2 + 16 * k);
                    const unsigned ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(bf16_lo(xw[e]), bf16_lo(ww[e]), acc[g], 0, 0, 0);
                        acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(bf16_hi(xw[e]), bf16_hi(ww[e]), acc[g], 0, 0, 0);
                    }
                }
            }
        } else {
            // (two steps of 8 features at a time: with the whole tile unrolled the reads of
            // 3 or 4 heads per lane took every register, and 48.7 us instead of 35.8)
            const float* wrow = reinterpret_cast<const float*>(wb) + lhead * kGateWRow;
#pragma unroll 2
            for (int k = 0; k < kGateTile / 8; ++k) {
                const uint4 xv = *reinterpret_cast<const uint4*>(xrow + 16 * k);
                const unsigned xw[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    float4 wv[N];
#pragma unroll
                    for (int g = 0; g < N; ++g)
                        wv[g] = *reinterpret_cast<const float4*>(wrow + 4 * g * kGateWRow + 8 * k + 4 * hf);
                    const float x0 = bf16_lo(xw[2 * hf]), x1 = bf16_hi(xw[2 * hf]),
                                x2 = bf16_lo(xw[2 * hf + 1]), x3 = bf16_hi(xw[2 * hf + 1]);
#pragma unroll
                    for (int g = 0; g < N; ++g) {
                        float a = acc[g][0];
                        a = __builtin_fmaf(x0, wv[g].x, a);
                        a = __builtin_fmaf(x1, wv[g].y, a);
                        a = __builtin_fmaf(x2, wv[g].z, a);
                        acc[g][0] = __builtin_fmaf(x3, wv[g].w, a);
                    }
                }
            }
        }
    };
    Pieces pa = fetch(0), pb = pa;
    stash(pa, 0);
    if (ntile > 1) pa = fetch(1);
    __syncthreads();
    // tile t in LDS, tile t + 1 in registers, tile t + 2 requested
    for (int t = 0; t < ntile; t += 2) {
        if (t + 2 < ntile) pb = fetch(t + 2);
        products(0);
        if (t + 1 < ntile) stash(pa, 1);
        lds_barrier();
        if (t + 1 >= ntile) break;
        if (t + 3 < ntile) pa = fetch(t + 3);
        products(1);
        if (t + 2 < ntile) stash(pb, 0);
        lds_barrier();
    }
    // the logits to [head][token], over the tiles (the last barrier ended their reads)
    float* lg = reinterpret_cast<float*>(gsm);
#pragma unroll
    for (int g = 0; g < N; ++g) {
        if constexpr (kMfma)
            *reinterpret_cast<f32x4*>(lg + (16 * g + lhead) * kGateLogitRow + 16 * w + 4 * (lane >> 4)) = acc[g];
        else
            lg[(4 * g + lhead) * kGateLogitRow + 16 * w + ltok] = acc[g][0];
    }
    lds_barrier();

    // ---- per head: log f, statistics, the block scan, the chained prefix, c.  Wave w
    // takes heads w, w + 4, ..., up to four at a time: lane = token of the block, and
    // lane j keeps the results of the round's head j ----------------------------------
#pragma unroll 1
    for (int r = w; r < H; r += 16) {
        auto head = [&](int j) { return r + 4 * j; };
        const int nh = min(4, (H - r + 3) / 4);
        float a4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) a4[j] = j < nh ? lg[head(j) * kGateLogitRow + lane] : 0.f;
        DD excl_mine{0.0, 0.0};   // lane j < nh: exclusive prefix of head j
        DD abs_mine{0.0, 0.0};    // lane j < nh: the block's statistics of head j
        int lsb_mine = 1 << 30, flags_mine = 0;
        DD scan[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            scan[j] = DD{0.0, 0.0};
            if (j >= nh) continue;
            const double a = (double)(a4[j] + bias[head(j)]);
            const double sp = fmax(-a, 0.0) + log1p(exp(-fabs(a)));   // softplus(-a)
            const float lf32 = (float)(-sp);
            const size_t bh = (size_t)b * H + head(j);
            log_f[bh * L + tok] = lf32;
            // statistics for stage 1's checks, and the block's scan: in float64
            // while the block's own 64 gates span under 53 bits (then every float64
            // sum is exact; the read is stage 1's), else in double-double
            const bool bad = !__builtin_isfinite(lf32);
            const double gv = bad ? 0.0 : (double)lf32;
            const int lsb = bad || lf32 == 0.f ? (1 << 30) : lsb_exp(lf32);
            const double ra = row16_reduce(__builtin_fabs(gv), [](double x, double y) { return x + y; });
            const double sabs_f = ((readlane_f64(ra, 0) + readlane_f64(ra, 16)) + readlane_f64(ra, 32)) +
                                  readlane_f64(ra, 48);
            const int rl = row16_reduce(lsb, [](int x, int y) { return min(x, y); });
            const int slsb = min(min(__builtin_amdgcn_readlane(rl, 0), __builtin_amdgcn_readlane(rl, 16)),
                                 min(__builtin_amdgcn_readlane(rl, 32), __builtin_amdgcn_readlane(rl, 48)));
            const int biased = (int)((__double_as_longlong(sabs_f) >> 52) & 0x7ff);
            const bool bwide = __builtin_amdgcn_readfirstlane(
                sabs_f > 0.0 && (biased > 0 ? biased : 1) - 1023 + 1 - slsb >= 53);
            DD sabs{sabs_f, 0.0};
            if (bwide) {
                sabs = wave_sum_dd(DD{__builtin_fabs(gv), 0.0});
                scan[j] = wave_inclusive_scan_dd(DD{gv, 0.0});
            } else {
                scan[j] = DD{wave_inclusive_scan_f64(gv), 0.0};
            }
            const bool anybad = __ballot(bad) != 0ull;
            if (lane == j) {
                abs_mine = sabs;
                lsb_mine = slsb;
                flags_mine = anybad ? 2 : 0;
            }
        }
        // block totals (lane j holds head j's), published before the look-back
        DD total{0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const DD tj = readlane_dd(scan[j], 63);
            if (lane == j) total = tj;
        }
        if (lane < nh) {
            const size_t d = ((size_t)b * H + head(lane)) * nblk + blk;
            publish((blk == 0 ? incl : agg) + 2 * d, total);
        }
        // Look-back, the whole wave on every head of the round, whose descriptors are
        // requested together (one head after the other, each round trip to memory came
        // on top of the last): lane l reads block i0 - l's, 64 blocks per round.  The
        // nearest block with its inclusive prefix published ends a head's walk if every
        // block after it has its total published; otherwise the round is read again.  A
        // round with no prefix but all 64 totals adds them and moves 64 blocks back.
        DD run[4];
        int i0[4];
        unsigned open = blk == 0 ? 0u : (1u << nh) - 1u;   // heads still walking (uniform)
        int spins = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            run[j] = DD{0.0, 0.0};
            i0[j] = blk - 1;
        }
        while (open != 0u) {
            unsigned long long p[4], pl[4], qq[4], ql[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                p[j] = pl[j] = qq[j] = ql[j] = kUnpublished;
                const int i = i0[j] - lane;
                if ((open >> j & 1u) && i >= 0) {
                    const size_t w2 = 2 * (((size_t)b * H + head(j)) * nblk + i);
                    p[j] = peek(&incl[w2]);
                    pl[j] = peek(&incl[w2 + 1]);
                    qq[j] = peek(&agg[w2]);
                    ql[j] = peek(&agg[w2 + 1]);
                }
            }
            bool moved = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!(open >> j & 1u)) continue;
                const int i = i0[j] - lane;
                // lanes whose block lies before the sequence count as published zeros
                const bool has_p = i >= 0 && p[j] != kUnpublished && pl[j] != kUnpublished;
                const bool has_q = i < 0 || (qq[j] != kUnpublished && ql[j] != kUnpublished) || has_p;
                const unsigned long long pm = __ballot(has_p);
                const int stop = pm ? __builtin_ctzll(pm) : 64;      // nearest prefix
                const unsigned long long need = stop == 64 ? ~0ull : ((1ull << stop) - 1ull);
                const unsigned long long qm = __ballot(has_q);
                if ((qm & need) != need) continue;
                moved = true;
                if (stop == 0) {   // the previous block's prefix alone: no reduction
                    run[j] = dd_add(run[j], DD{readlane_f64(bits_f64(p[j]), 0), readlane_f64(bits_f64(pl[j]), 0)});
                } else {
                    DD v{0.0, 0.0};
                    if (lane < stop && i >= 0) v = DD{bits_f64(qq[j]), bits_f64(ql[j])};
                    if (lane == stop) v = DD{bits_f64(p[j]), bits_f64(pl[j])};
                    double sum;
                    run[j] = dd_add(run[j], wave_sum_f64_if_exact(v, sum) ? DD{sum, 0.0} : wave_sum_dd(v));
                }
                i0[j] -= 64;
                if (stop < 64 || i0[j] < 0) {
                    open &= ~(1u << j);
                    if (lane == j) {
                        excl_mine = run[j];
                        publish(&incl[2 * (((size_t)b * H + head(j)) * nblk + blk)], dd_add(run[j], total));
                    }
                }
            }
            if (moved) {
                spins = 0;
            } else if (++spins > kGateSpinLimit) {
                // time-out: the heads still open go on with what they have
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((open >> j & 1u) && lane == j) {
                        excl_mine = run[j];
                        flags_mine |= 32;
                        publish(&incl[2 * (((size_t)b * H + head(j)) * nblk + blk)], dd_add(run[j], total));
                    }
                open = 0u;
            } else {
                __builtin_amdgcn_s_sleep(1);
            }
        }
        if (lane < nh) {
            GateStats g;
            g.abs_sum = abs_mine.hi;
            g.abs_lo = abs_mine.lo;
            g.min_lsb = lsb_mine;
            g.flags = flags_mine;
            st[((size_t)b * H + head(lane)) * nblk + blk] = g;
        }
        // c of the block: exclusive prefix + the in-block inclusive scan
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= nh) continue;
            const DD ex = readlane_dd(excl_mine, j);
            c[((size_t)b * H + head(j)) * L + tok] = dd_to_f32(dd_add(ex, scan[j]));
        }
    }
}

template <int N, bool kMfma>
static void gate_t(const GateArgs& a, hipStream_t s) {
    const int nblk = a.L / 64;
    hipLaunchKernelGGL((gate_kernel<N, kMfma>), dim3(a.B * nblk), dim3(kGateThreads), 0, s,
                       (const __bf16*)a.X, (const __bf16*)a.wt, a.bias, a.L, a.Dm, a.H, nblk,
                       a.log_f, a.c, a.agg, a.incl, a.stats);
}

hipError_t launch_gate(const GateArgs& a, hipStream_t s) {
    const int ndesc = a.B * a.H * (a.L / 64);
    trace_begin(ACP_K_GATE, s);
    const int ninit = max(2 * ndesc, a.H * a.Dm);
    hipLaunchKernelGGL(gate_init_kernel, dim3((ninit + 255) / 256), dim3(256), 0, s,
                       a.agg, a.incl, 2 * ndesc, (const unsigned short*)a.W,
                       (unsigned short*)a.wt, a.Dm, a.H);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.H <= 4) gate_t<1, false>(a, s);
    else if (a.H <= 8) gate_t<2, false>(a, s);
    else if (a.H <= 12) gate_t<3, false>(a, s);
    else if (a.H <= 16) gate_t<4, false>(a, s);
    else if (a.H <= 20) gate_t<5, false>(a, s);
    else if (a.H <= 32) gate_t<2, true>(a, s);
    else if (a.H <= 48) gate_t<3, true>(a, s);
    else gate_t<4, true>(a, s);
    e = hipGetLastError();
    trace_end(ACP_K_GATE, s);
    return e;
}

}  // namespace acp
