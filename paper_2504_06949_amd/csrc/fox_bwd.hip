// Backward of Forgetting Attention over the blocks kept by ACP.
//
// The paper states only that the backward pass is built like the forward
// (Sec. 2, FlashAttention paragraph).  With x_ij = q_i.k_j/sqrt(d) + c_i - c_j,
// P = softmax_row(x) on the kept, causal entries, and the pruning mask held
// constant, the chain rule through eq. 2 and c gives
//   dV = P^T dO,  dP = dO V^T,  Delta_i = dO_i . O_i,  dS = P o (dP - Delta),
//   dQ = dS K / sqrt(d),  dK = dS^T Q / sqrt(d),
//   dc_i = sum_j dS_ij - sum_j dS_ji,  dlog f_l = sum_{i >= l} dc_i.
//
// Three launches (bf16: fox_bwd_mfma.hip; fp32: fox_f32.hip; the last: below):
//   dq kernel     per query block, loops over kept key blocks: Delta from the rows
//                 of O and dO it holds, dQ, then Delta'_i = sum_j P_ij dP_ij and
//                 the row sums of dS
//   dkdv kernel   per key block, loops over the query blocks that keep it: dK,
//                 dV and the column sums of dS
//   dlogf_kernel  reverse cumulative sum of (row sum - column sum)
// dQ is produced by its own pass (recomputing S and dP) rather than by atomic
// accumulation from the key-block pass, so every output is written once.
#include "acp_device.h"
#include "acp_internal.h"
#include "acp_scan.h"

namespace acp {

// ---------------------------------------------------------------------------
// dlog f_l = sum_{i >= l} (rowsum_i - colsum_i), accumulated in float64.  Each
// thread owns a contiguous run of whole float4s, kept in registers up to kHeld values,
// else read again in batches of that many, from the end; one round through LDS carries
// the waves' totals for the suffix sums.  kHeld = 4 is a whole run up to 4096 positions, and
// two workgroups then fit a CU (kRunHeld takes 84
// VGPRs): 4096 heads of 64 positions 28 -> 14 us, 96 of 4096 6.7 -> 6.5.
// ---------------------------------------------------------------------------
constexpr int kScanThreads = kPlanThreads;

template <int kHeld>
__global__ __launch_bounds__(kScanThreads) void dlogf_kernel(const float* __restrict__ rowsum,
                                                             const float* __restrict__ colsum,
                                                             float* __restrict__ dlog_f, int L) {
    constexpr int kWaves = kScanThreads / 64;
    __shared__ double s_tot[kWaves];
    const int bh = blockIdx.x, t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const size_t head = (size_t)bh * L;
    const int per = run_length(L);
    const int beg = min(t * per, L), n = min(beg + per, L) - beg;   // multiples of 4
    const float* rs = rowsum + head + beg;
    const float* cs = colsum + head + beg;
    double dv[kHeld];
    auto load = [&](int b) __attribute__((always_inline)) {
        float r[kHeld], c[kHeld];
        load_run(rs, b, n, true, r);
        load_run(cs, b, n, true, c);
#pragma unroll
        for (int i = 0; i < kHeld; ++i) dv[i] = (double)r[i] - (double)c[i];
    };
    double local = 0.0;
    const int last = n > 0 ? (n - 1) / kHeld * kHeld : 0;   // the run's last batch
    for (int b = 0; b <= last; b += kHeld) {
        load(b);
#pragma unroll
        for (int i = 0; i < kHeld; ++i) local += dv[i];
    }
    // inclusive suffix sums over the lanes of the wave: within each row of 16 by
    // zero-filled shifts toward lower lanes, then the totals of the later rows
    // (lane 16 r holds row r's)
    double suf = local;
    suf += dpp_f64_or_zero<0x101>(suf);   // row_shl:1
    suf += dpp_f64_or_zero<0x102>(suf);   // row_shl:2
    suf += dpp_f64_or_zero<0x104>(suf);   // row_shl:4
    suf += dpp_f64_or_zero<0x108>(suf);   // row_shl:8
    {
        const double t1 = readlane_f64(suf, 16), t2 = readlane_f64(suf, 32), t3 = readlane_f64(suf, 48);
        const int row = lane >> 4;
        suf += row == 0 ? (t1 + t2) + t3 : row == 1 ? t2 + t3 : row == 2 ? t3 : 0.0;
    }
    if (lane == 0) s_tot[wid] = suf;
    __syncthreads();
    // the waves after this one: lane l < 16 takes wave l's total, summed over the row
    double after;
    {
        const double v = lane < kWaves && lane > wid ? s_tot[lane] : 0.0;
        after = readlane_f64(row16_reduce(v, [](double x, double y) { return x + y; }), 0);
    }
    double run = after + (suf - local);   // sum over the threads after this one
    for (int b = last; b >= 0; b -= kHeld) {
        if (b != last) load(b);   // (the last batch is still in registers)
#pragma unroll
        for (int i = kHeld - 4; i >= 0; i -= 4) {
            if (b + i < n) {
                float4 o;
                run += dv[i + 3]; o.w = (float)run;
                run += dv[i + 2]; o.z = (float)run;
                run += dv[i + 1]; o.y = (float)run;
                run += dv[i];     o.x = (float)run;
                *reinterpret_cast<float4*>(dlog_f + head + beg + b + i) = o;
            }
        }
    }
}

// ---------------------------------------------------------------------------
hipError_t launch_bwd(const BwdArgs& a, hipStream_t s) {
    hipError_t e;
    trace_begin(ACP_K_DQ, s);
    e = a.bf16 ? launch_dq_bf16(a, s) : launch_dq_f32(a, s);
    if (e != hipSuccess) return e;
    trace_end(ACP_K_DQ, s);

    trace_begin(ACP_K_DKDV, s);
    e = a.bf16 ? launch_dkdv_bf16(a, s) : launch_dkdv_f32(a, s);
    if (e != hipSuccess) return e;
    trace_end(ACP_K_DKDV, s);

    trace_begin(ACP_K_DLOGF, s);
    hipLaunchKernelGGL((a.L <= 4 * kScanThreads ? dlogf_kernel<4> : dlogf_kernel<kRunHeld>),
                       dim3(a.B * a.H), dim3(kScanThreads), 0, s, a.rowsum, a.colsum, a.dlog_f, a.L);
    e = hipGetLastError();
    trace_end(ACP_K_DLOGF, s);
    return e;
}

}  // namespace acp
