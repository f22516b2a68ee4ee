// float32 forward and backward of Forgetting Attention over the blocks kept by
// ACP, on the float32 matrix instruction v_mfma_f32_16x16x4_f32 (float32
// products and sums throughout).  Formulas and decay splitting are those of the
// bfloat16 kernels (fox_fwd.hip, fox_bwd_mfma.hip).
//
// What bounds them: the matrix cores at 154 TFLOP/s (a large float32 torch
// product on the same card); each product of a 16 x 16 tile costs 8 d cycles of MFMA, so
// a tile 16 d in the forward, 24 d in the dQ and 32 d in the dK/dV pass, against about 40
// of exp, and nothing else needs hiding but memory latency.
//
// Split: a workgroup owns 16 T rows (queries in the forward and the dQ pass, keys
// in the dK/dV pass) and its 4 waves share out the other operand in 16-row
// subtiles, wave w taking every fourth.  No two waves read the same rows, so the
// subtiles go from memory straight into registers (no LDS, no barrier in the
// loop), and the other waves on the SIMD (two to four) cover the loads; only the 4
// partial results meet in LDS at the end.  T shrinks when a call has few rows, so
// that short sequences still spread over the chip (pick_rows).
//
// Measured against the earlier form (one thread per row, VALU products, tiles in
// LDS; B = 2, H = 12, L = 1984, d = 64): forward 1566 -> 140 us, dQ 2042 -> 212,
// dK/dV 2676 -> 261, i.e. 76, 75 and 81 TFLOP/s of products; B = 1, H = 2, L = 512:
// 298 -> 12, 448 -> 17, 615 -> 20 us.  Holding the next subtile's rows in
// registers (loaded a step ahead) costs a wave per SIMD in the backward: dQ 220 and
// dK/dV 279 us there.
//
// Operand layouts (lane = 16 g + r).  The contraction of an MFMA may run over its
// indices in any order, so each lane reads whole float4s and element e of a
// lane's vectors forms the e-th MFMA:
//   row operand (contraction over features): X[row r][16 s + 4 g + (0..3)];
//   column operand (contraction over the 16 rows of a subtile): step t takes rows
//     4 g + t, X[4 g + t][64 h + 4 r + (0..3)], output tile (h, e) holding the
//     features 64 h + 4 i + e.  The logits' D layout (column r, rows 4 g + t) is
//     then the B operand of step t as it stands, and a lane ends with 16
//     consecutive features 64 h + 16 g + 4 t + e of its row.
#include "acp_device.h"
#include "acp_internal.h"

namespace acp {

constexpr int kF32Threads = 256;
constexpr int kF32Waves = 4;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// row operand of 16 rows from x (row-major, D columns)
template <int D>
struct RowOp {
    f32x4 v[D / 16];
    __device__ __forceinline__ void load(const float* __restrict__ x, int g, int r) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) v[s] = ld4(x + r * D + 16 * s + 4 * g);
    }
};

// column operand of 16 rows
template <int D>
struct ColOp {
    f32x4 v[D / 64][4];
    __device__ __forceinline__ void load(const float* __restrict__ x, int g, int r) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int h = 0; h < D / 64; ++h) v[h][t] = ld4(x + (4 * g + t) * D + 64 * h + 4 * r);
    }
    // Replaces infinities and NaNs by 0; returns whether any lane of the wave had one.
    __device__ __forceinline__ bool take_nonfinite() {
        bool bad = false;
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool f = __builtin_isfinite(v[h][t][e]);
                    bad = bad || !f;
                    v[h][t][e] = f ? v[h][t][e] : 0.f;
                }
        return __ballot(bad) != 0ull;
    }
};

// Whether a logit of the lane is infinite or NaN: in every column of a subtile whose row
// (of K in the dQ pass, of Q in the dK/dV pass) is, so that the rows themselves need a
// look only where this says so.
__device__ __forceinline__ bool any_nonfinite(const f32x4& s) {
    return !__builtin_isfinite(s[0]) || !__builtin_isfinite(s[1]) || !__builtin_isfinite(s[2]) ||
           !__builtin_isfinite(s[3]);
}

template <int D>
__device__ __forceinline__ f32x4 row_product(const RowOp<D>& a, const RowOp<D>& b) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) s = mfma4(a.v[i][e], b.v[i][e], s);
    return s;
}

// acc (+)= X^T p with the subtile X as column operand and p[t] of rows 4 g + t
template <int D>
__device__ __forceinline__ void col_product(const ColOp<D>& x, const f32x4& p, f32x4* acc) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * h + e] = mfma4(x.v[h][t][e], p[t], acc[4 * h + e]);
}

// The products of a diagonal tile with the non-finite entries of X that
// take_nonfinite() set to 0: a masked weight must not meet them (0 * inf), so
// they are added per entry for the weights that are not masked.  Rare; x is the
// subtile in memory, keep(row) tells whether the lane's column keeps that row.
template <int D, typename Keep>
__device__ __forceinline__ void add_nonfinite(const float* __restrict__ x, const f32x4& p, f32x4* acc,
                                              int g, int r, Keep keep) {
#pragma unroll 1
    for (int row = 0; row < 16; ++row) {
        const int src = 16 * (row >> 2) + r;
        float pr = __shfl(p[0], src);
        const float p1 = __shfl(p[1], src), p2 = __shfl(p[2], src), p3 = __shfl(p[3], src);
        pr = (row & 3) == 1 ? p1 : (row & 3) == 2 ? p2 : (row & 3) == 3 ? p3 : pr;
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float xv = x[row * D + 64 * h + 16 * g + 4 * t + e];
                    if (!__builtin_isfinite(xv) && keep(row)) acc[4 * h + e][t] += pr * xv;
                }
    }
}

// acc of T tiles of 16 rows to LDS as [row][feature], rows padded by 16 bytes
// (16 lanes of a store then cover all banks)
template <int D, int T>
__device__ __forceinline__ void put_acc(float* s, const f32x4 (&acc)[T][D / 16], int g, int r) {
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                *reinterpret_cast<f32x4*>(s + (16 * i + r) * (D + 4) + 64 * h + 16 * g + 4 * t) =
                    f32x4{acc[i][4 * h][t], acc[i][4 * h + 1][t], acc[i][4 * h + 2][t], acc[i][4 * h + 3][t]};
}

__device__ __forceinline__ float sum_over_g(float x) {
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    return x;
}

// (head, block of 16 T rows) of a workgroup: a head's blocks on one XCD
__device__ __forceinline__ int f32_item(int nblocks) { return xcd_logical_id(blockIdx.x, nblocks); }

// ---------------------------------------------------------------------------
// Forward: one workgroup per 16 T queries, online maximum per wave.
// ---------------------------------------------------------------------------
template <int D, int T>
__global__ __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(2)))
void fwd_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ cg, const int* __restrict__ row_start, float* __restrict__ O,
    float* __restrict__ lse, float* __restrict__ lse2, int L, int M, int nb, int nblocks,
    float kscale) {
    __shared__ __attribute__((aligned(16))) float s_acc[kF32Waves][16 * T * (D + 4)];
    __shared__ float s_m[kF32Waves][16 * T], s_l[kF32Waves][16 * T];
    const int item = f32_item(nblocks);
    const int bh = item / nb, qb = nb - 1 - item % nb;   // longest rows first
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t head = (size_t)bh * L;
    const int q0 = 16 * T * qb, m = q0 / kBlock;
    const float* Kh = K + head * D;
    const float* Vh = V + head * D;
    const float* ch = cg + head;

    RowOp<D> qf[T];
    f32x4 acc[T][D / 16];
    float ci[T], row[T], mrun[T], lrun[T];
    const float rref = ch[kBlock * m];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        qf[i].load(Q + (head + q0 + 16 * i) * D, g, r);
        ci[i] = ch[q0 + 16 * i + r];
        row[i] = (ci[i] - rref) * kLog2e;
        mrun[i] = -INFINITY;
        lrun[i] = 0.f;
#pragma unroll
        for (int a = 0; a < D / 16; ++a) acc[i][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // softmax of one subtile: y[t] of key 4 g + t; returns the weights
    auto soften = [&](int i, f32x4 y) __attribute__((always_inline)) {
        float mx = fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mnew = fmaxf(mrun[i], mx);
        const float alpha = fast_exp2(mrun[i] - mnew);
        f32x4 p;
#pragma unroll
        for (int t = 0; t < 4; ++t) p[t] = fast_exp2(y[t] - mnew);
        lrun[i] = lrun[i] * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
        if (__ballot(mnew != mrun[i]) != 0ull) {
#pragma unroll
            for (int a = 0; a < D / 16; ++a) acc[i][a] *= alpha;
        }
        mrun[i] = mnew;
        return p;
    };

    // subtiles of earlier blocks, then of the diagonal block up to the last query
    const int kt0 = 4 * row_start[(size_t)bh * M + m] + w, kd = 4 * m, kend = q0 / 16 + T;
    RowOp<D> kf;
    ColOp<D> vf;
    int kt = kt0;
    kf.load(Kh + (size_t)16 * min(kt, kend - 1) * D, g, r);
    for (; kt < kd; kt += kF32Waves) {
        vf.load(Vh + (size_t)16 * kt * D, g, r);
        const f32x4 cj = ld4(ch + 16 * kt + 4 * g);
        f32x4 y[T];
#pragma unroll
        for (int i = 0; i < T; ++i) y[i] = row_product<D>(kf, qf[i]);
        kf.load(Kh + (size_t)16 * min(kt + kF32Waves, kend - 1) * D, g, r);
#pragma unroll
        for (int i = 0; i < T; ++i) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                y[i][t] = __builtin_fmaf(y[i][t], kscale, (rref - cj[t]) * kLog2e) + row[i];
            const f32x4 p = soften(i, y[i]);
            col_product<D>(vf, p, acc[i]);
        }
    }
    for (; kt < kend; kt += kF32Waves) {
        vf.load(Vh + (size_t)16 * kt * D, g, r);
        const f32x4 cj = ld4(ch + 16 * kt + 4 * g);
        const bool bad = vf.take_nonfinite();
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int qt = q0 / 16 + i;
            if (kt <= qt) {   // uniform
                f32x4 y = row_product<D>(kf, qf[i]);
                const int last = kt < qt ? 16 : r;   // last key of the subtile that the query keeps
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    y[t] = __builtin_fmaf(y[t], kscale, (ci[i] - cj[t]) * kLog2e);
                    if (4 * g + t > last) y[t] = -INFINITY;
                }
                const f32x4 p = soften(i, y);
                col_product<D>(vf, p, acc[i]);
                if (bad)
                    add_nonfinite<D>(Vh + (size_t)16 * kt * D, p, acc[i], g, r,
                                     [&](int key) { return key <= last; });
            }
        }
        kf.load(Kh + (size_t)16 * min(kt + kF32Waves, kend - 1) * D, g, r);
    }

    // the 4 waves' sums, brought to one maximum per query
    put_acc<D, T>(s_acc[w], acc, g, r);
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const float l = sum_over_g(lrun[i]);
        if (g == 0) {
            s_m[w][16 * i + r] = mrun[i];
            s_l[w][16 * i + r] = l;
        }
    }
    __syncthreads();
    constexpr int kPer = D / 4;   // float4s per row
    for (int x = tid; x < 16 * T * kPer; x += kF32Threads) {
        const int q = x / kPer, col = 4 * (x % kPer);
        float mw[kF32Waves], mm = -INFINITY;
#pragma unroll
        for (int v = 0; v < kF32Waves; ++v) {
            mw[v] = s_m[v][q];
            mm = fmaxf(mm, mw[v]);
        }
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < kF32Waves; ++v) {
            // (a wave without a key of this query holds nothing: selected away)
            if (mw[v] != -INFINITY || mm == -INFINITY) {
                const float e = fast_exp2(mw[v] - mm);
                l = __builtin_fmaf(s_l[v][q], e, l);
                o += ld4(&s_acc[v][q * (D + 4) + col]) * e;
            }
        }
        *reinterpret_cast<f32x4*>(O + (head + q0 + q) * D + col) = o * (1.0f / l);
        if (col == 0) {
            const float l2 = mm + fast_log2(l);
            lse2[head + q0 + q] = l2;
            lse[head + q0 + q] = l2 * kLn2;
        }
    }
}

// ---------------------------------------------------------------------------
// dQ pass: one workgroup per 16 T queries.  Delta = rowdot(dO, O) is formed from
// the rows it holds; Delta' and the row sums of dS as in the bfloat16 pass.
// ---------------------------------------------------------------------------
template <int D, int T>
__global__ __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(2)))
void dq_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ O, const float* __restrict__ dO, const float* __restrict__ cg,
    const int* __restrict__ row_start, const float* __restrict__ lse2,
    float* __restrict__ dsum, float* __restrict__ dQ, float* __restrict__ rowsum,
    int L, int M, int nb, int nblocks, float kscale, float qscale) {
    __shared__ __attribute__((aligned(16))) float s_acc[kF32Waves][16 * T * (D + 4)];
    __shared__ float s_dp[kF32Waves][16 * T], s_p[kF32Waves][16 * T];
    const int item = f32_item(nblocks);
    const int bh = item / nb, qb = nb - 1 - item % nb;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t head = (size_t)bh * L;
    const int q0 = 16 * T * qb, m = q0 / kBlock;
    const float* Kh = K + head * D;
    const float* Vh = V + head * D;
    const float* ch = cg + head;

    RowOp<D> qf[T], gf[T];
    f32x4 acc[T][D / 16];
    float ci[T], l2[T], l2d[T], dl[T], pdp[T], psum[T];
    const float rref = ch[kBlock * m];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const size_t q = head + q0 + 16 * i;
        qf[i].load(Q + q * D, g, r);
        gf[i].load(dO + q * D, g, r);
        RowOp<D> of;
        of.load(O + q * D, g, r);
        float dd = 0.f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) dd = __builtin_fmaf(gf[i].v[s][e], of.v[s][e], dd);
        dl[i] = sum_over_g(dd);
        ci[i] = cg[q + r];
        l2d[i] = -lse2[q + r];
        l2[i] = (ci[i] - rref) * kLog2e + l2d[i];
        pdp[i] = 0.f;
        psum[i] = 0.f;
#pragma unroll
        for (int a = 0; a < D / 16; ++a) acc[i][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // dS of one subtile from the exponents and dP; keep(t): not masked
    auto ds_of = [&](int i, const f32x4& p, const f32x4& dp, auto keep) __attribute__((always_inline)) {
        f32x4 ds;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool k = keep(t);
            const float pt = k ? p[t] : 0.f;
            ds[t] = k ? pt * (dp[t] - dl[i]) : 0.f;
            pdp[i] = k ? __builtin_fmaf(pt, dp[t], pdp[i]) : pdp[i];
            psum[i] += pt;
        }
        return ds;
    };

    const int kt0 = 4 * row_start[(size_t)bh * M + m] + w, kd = 4 * m, kend = q0 / 16 + T;
    RowOp<D> kf, vf;
    ColOp<D> kc;
    int kt = kt0;
    auto rows_of = [&](int k) __attribute__((always_inline)) {
        kf.load(Kh + (size_t)16 * k * D, g, r);
        vf.load(Vh + (size_t)16 * k * D, g, r);
    };
    for (; kt < kd; kt += kF32Waves) {
        rows_of(kt);
        kc.load(Kh + (size_t)16 * kt * D, g, r);
        const f32x4 cj = ld4(ch + 16 * kt + 4 * g);
        f32x4 s[T], dp[T];
#pragma unroll
        for (int i = 0; i < T; ++i) s[i] = row_product<D>(kf, qf[i]);
#pragma unroll
        for (int i = 0; i < T; ++i) dp[i] = row_product<D>(vf, gf[i]);
#pragma unroll
        for (int i = 0; i < T; ++i) {
            f32x4 p;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                p[t] = fast_exp2(__builtin_fmaf(s[i][t], kscale, (rref - cj[t]) * kLog2e) + l2[i]);
            const f32x4 ds = ds_of(i, p, dp[i], [](int) { return true; });
            col_product<D>(kc, ds, acc[i]);
        }
    }
    for (; kt < kend; kt += kF32Waves) {
        rows_of(kt);
        // (at d = 128 loaded last: next to the other operands it would cost a wave per SIMD)
        if constexpr (D == 64) kc.load(Kh + (size_t)16 * kt * D, g, r);
        const f32x4 cj = ld4(ch + 16 * kt + 4 * g);
        f32x4 ds[T];
        bool odd = false;
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int qt = q0 / 16 + i;
            if (kt <= qt) {
                const f32x4 s = row_product<D>(kf, qf[i]);
                odd = odd || any_nonfinite(s);
                const f32x4 dp = row_product<D>(vf, gf[i]);
                const int last = kt < qt ? 16 : r;
                f32x4 p;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    p[t] = fast_exp2(__builtin_fmaf(s[t], kscale, (ci[i] - cj[t]) * kLog2e) + l2d[i]);
                ds[i] = ds_of(i, p, dp, [&](int t) { return 4 * g + t <= last; });
            }
        }
        if constexpr (D == 128) kc.load(Kh + (size_t)16 * kt * D, g, r);
        const bool bad = __ballot(odd) != 0ull && kc.take_nonfinite();
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int qt = q0 / 16 + i;
            if (kt <= qt) {
                col_product<D>(kc, ds[i], acc[i]);
                const int last = kt < qt ? 16 : r;
                if (bad)
                    add_nonfinite<D>(Kh + (size_t)16 * kt * D, ds[i], acc[i], g, r,
                                     [&](int key) { return key <= last; });
            }
        }
    }

    put_acc<D, T>(s_acc[w], acc, g, r);
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const float a = sum_over_g(pdp[i]), b = sum_over_g(psum[i]);
        if (g == 0) {
            s_dp[w][16 * i + r] = a;
            s_p[w][16 * i + r] = b;
        }
    }
    __syncthreads();
    constexpr int kPer = D / 4;
    for (int x = tid; x < 16 * T * kPer; x += kF32Threads) {
        const int q = x / kPer, col = 4 * (x % kPer);
        f32x4 o = ld4(&s_acc[0][q * (D + 4) + col]);
#pragma unroll
        for (int v = 1; v < kF32Waves; ++v) o += ld4(&s_acc[v][q * (D + 4) + col]);
        *reinterpret_cast<f32x4*>(dQ + (head + q0 + q) * D + col) = o * qscale;
        if (col == 0) {
            const float a = (s_dp[0][q] + s_dp[1][q]) + (s_dp[2][q] + s_dp[3][q]);
            const float b = (s_p[0][q] + s_p[1][q]) + (s_p[2][q] + s_p[3][q]);
            dsum[head + q0 + q] = a;
            rowsum[head + q0 + q] = a - a * b;
        }
    }
}

// ---------------------------------------------------------------------------
// dK/dV pass: one workgroup per 16 T keys, its waves sharing out the query
// subtiles of the blocks that keep them.
// ---------------------------------------------------------------------------
template <int D, int T>
__global__ __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(2)))
void dkdv_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ dO, const float* __restrict__ cg,
    const int* __restrict__ col_end, const float* __restrict__ lse2,
    const float* __restrict__ dsum, float* __restrict__ dK, float* __restrict__ dV,
    float* __restrict__ colsum, int L, int M, int nb, int nblocks, float kscale, float qscale) {
    __shared__ __attribute__((aligned(16))) float s_acc[kF32Waves][16 * T * (D + 4)];
    __shared__ float s_cs[kF32Waves][16 * T];
    const int item = f32_item(nblocks);
    const int bh = item / nb, kb = item % nb;            // first keys (longest columns) first
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t head = (size_t)bh * L;
    const int k0 = 16 * T * kb, n = k0 / kBlock;
    const float* Qh = Q + head * D;
    const float* Gh = dO + head * D;
    const float* ch = cg + head;
    const float* lh = lse2 + head;
    const float* dh = dsum + head;

    RowOp<D> kf[T], vf[T];
    f32x4 ak[T][D / 16], av[T][D / 16];
    float cj[T], nk[T], cs[T];
    const float rref = ch[kBlock * n + kBlock - 1];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const size_t k = head + k0 + 16 * i;
        kf[i].load(K + k * D, g, r);
        vf[i].load(V + k * D, g, r);
        cj[i] = cg[k + r];
        nk[i] = (rref - cj[i]) * kLog2e;
        cs[i] = 0.f;
#pragma unroll
        for (int a = 0; a < D / 16; ++a) {
            ak[i][a] = f32x4{0.f, 0.f, 0.f, 0.f};
            av[i][a] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }

    const int qd = 4 * (n + 1), qend = 4 * (col_end[(size_t)bh * M + n] + 1);
    int qt = k0 / 16 + w;   // (qend - 1 >= the wave's first subtile - 3)
    RowOp<D> qr, gr;
    ColOp<D> oc;
    auto rows_of = [&](int q) __attribute__((always_inline)) {
        qr.load(Qh + (size_t)16 * q * D, g, r);
        gr.load(Gh + (size_t)16 * q * D, g, r);
    };
    for (; qt < min(qd, qend); qt += kF32Waves) {         // the diagonal block
        rows_of(qt);
        const f32x4 c4 = ld4(ch + 16 * qt + 4 * g), l4 = ld4(lh + 16 * qt + 4 * g),
                    d4 = ld4(dh + 16 * qt + 4 * g);
        f32x4 p[T], ds[T];
        bool odd = false;
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int kt = k0 / 16 + i;
            p[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            ds[i] = p[i];
            if (qt >= kt) {
                const f32x4 s = row_product<D>(qr, kf[i]);
                odd = odd || any_nonfinite(s);
                const f32x4 dp = row_product<D>(gr, vf[i]);
                const int first = qt > kt ? 0 : r;        // first query that keeps the lane's key
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const bool keep = 4 * g + t >= first;
                    const float e = fast_exp2(__builtin_fmaf(s[t], kscale, (c4[t] - cj[i]) * kLog2e) - l4[t]);
                    p[i][t] = keep ? e : 0.f;
                    ds[i][t] = keep ? e * (dp[t] - d4[t]) : 0.f;
                    cs[i] += ds[i][t];
                }
            }
        }
        oc.load(Gh + (size_t)16 * qt * D, g, r);
        const bool bad = oc.take_nonfinite();
#pragma unroll
        for (int i = 0; i < T; ++i)
            if (qt >= k0 / 16 + i) {
                col_product<D>(oc, p[i], av[i]);
                const int first = qt > k0 / 16 + i ? 0 : r;
                if (bad)
                    add_nonfinite<D>(Gh + (size_t)16 * qt * D, p[i], av[i], g, r,
                                     [&](int q) { return q >= first; });
            }
        oc.load(Qh + (size_t)16 * qt * D, g, r);
        const bool bad_q = __ballot(odd) != 0ull && oc.take_nonfinite();
#pragma unroll
        for (int i = 0; i < T; ++i)
            if (qt >= k0 / 16 + i) {
                col_product<D>(oc, ds[i], ak[i]);
                const int first = qt > k0 / 16 + i ? 0 : r;
                if (bad_q)
                    add_nonfinite<D>(Qh + (size_t)16 * qt * D, ds[i], ak[i], g, r,
                                     [&](int q) { return q >= first; });
            }
    }
    for (; qt < qend; qt += kF32Waves) {
        rows_of(qt);
        oc.load(Gh + (size_t)16 * qt * D, g, r);
        const f32x4 c4 = ld4(ch + 16 * qt + 4 * g), l4 = ld4(lh + 16 * qt + 4 * g),
                    d4 = ld4(dh + 16 * qt + 4 * g);
        f32x4 p[T], ds[T];
#pragma unroll
        for (int i = 0; i < T; ++i) p[i] = row_product<D>(qr, kf[i]);
#pragma unroll
        for (int i = 0; i < T; ++i) ds[i] = row_product<D>(gr, vf[i]);
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float ls = (c4[t] - rref) * kLog2e - l4[t];
                p[i][t] = fast_exp2(__builtin_fmaf(p[i][t], kscale, nk[i]) + ls);
                ds[i][t] = p[i][t] * (ds[i][t] - d4[t]);
                cs[i] += ds[i][t];
            }
#pragma unroll
        for (int i = 0; i < T; ++i) col_product<D>(oc, p[i], av[i]);
        oc.load(Qh + (size_t)16 * qt * D, g, r);
#pragma unroll
        for (int i = 0; i < T; ++i) col_product<D>(oc, ds[i], ak[i]);
    }

    // the 4 waves' sums, dK then dV through the same LDS
    constexpr int kPer = D / 4;
    auto merge = [&](float* __restrict__ out, float scale) __attribute__((always_inline)) {
        for (int x = tid; x < 16 * T * kPer; x += kF32Threads) {
            const int k = x / kPer, col = 4 * (x % kPer);
            f32x4 o = ld4(&s_acc[0][k * (D + 4) + col]);
#pragma unroll
            for (int v = 1; v < kF32Waves; ++v) o += ld4(&s_acc[v][k * (D + 4) + col]);
            *reinterpret_cast<f32x4*>(out + (head + k0 + k) * D + col) = o * scale;
        }
    };
    put_acc<D, T>(s_acc[w], ak, g, r);
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const float a = sum_over_g(cs[i]);
        if (g == 0) s_cs[w][16 * i + r] = a;
    }
    __syncthreads();
    merge(dK, qscale);
    if (tid < 16 * T)
        colsum[head + k0 + tid] = (s_cs[0][tid] + s_cs[1][tid]) + (s_cs[2][tid] + s_cs[3][tid]);
    lds_barrier();
    put_acc<D, T>(s_acc[w], av, g, r);
    lds_barrier();
    merge(dV, 1.0f);
}

// ---------------------------------------------------------------------------
// Row tiles per workgroup: as many as the registers hold (each operand read then
// feeds more MFMAs), halved while fewer than `least` workgroups would remain, where
// an uneven last round costs more than the reads saved.  Measured (us, d = 64):
// forward at 47616 rows T = 4 (744 workgroups) 150, T = 2 140; dK/dV at 16384 rows
// T = 2 (512) 81, T = 1 75, at 47616 rows T = 2 (1488) 261, T = 1 294; dQ likewise 70
// against 68 and 222 against 268.  d = 128, forward at 23808 rows: T = 2 (744) 175,
// T = 1 206.
static int pick_rows(size_t rows, int most, size_t least) {
    int t = most;
    while (t > 1 && rows / (16 * (size_t)t) < least) t /= 2;
    return t;
}

template <int D, int T>
static void fwd_t(const FwdArgs& a, hipStream_t s) {
    const int nb = a.L / (16 * T), nblocks = a.B * a.H * nb;
    hipLaunchKernelGGL((fwd_f32_kernel<D, T>), dim3(nblocks), dim3(kF32Threads), 0, s,
                       (const float*)a.Q, (const float*)a.K, (const float*)a.V, a.c, a.row_start,
                       (float*)a.O, a.lse, a.lse2, a.L, a.L / kBlock, nb, nblocks,
                       kLog2e / sqrtf((float)D));
}

hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t s) {
    const size_t rows = (size_t)a.B * a.H * a.L;
    if (a.d == 64) {
        const int t = pick_rows(rows, 4, 1024);
        if (t == 4) fwd_t<64, 4>(a, s);
        else if (t == 2) fwd_t<64, 2>(a, s);
        else fwd_t<64, 1>(a, s);
    } else {
        if (pick_rows(rows, 2, 512) == 2) fwd_t<128, 2>(a, s);
        else fwd_t<128, 1>(a, s);
    }
    return hipGetLastError();
}

template <int D, int T>
static void dq_t(const BwdArgs& a, hipStream_t s) {
    const int nb = a.L / (16 * T), nblocks = a.B * a.H * nb;
    hipLaunchKernelGGL((dq_f32_kernel<D, T>), dim3(nblocks), dim3(kF32Threads), 0, s,
                       (const float*)a.Q, (const float*)a.K, (const float*)a.V, (const float*)a.O,
                       (const float*)a.dO, a.c, a.row_start, a.lse2, a.dsum, (float*)a.dQ, a.rowsum,
                       a.L, a.L / kBlock, nb, nblocks, kLog2e / sqrtf((float)D),
                       1.0f / sqrtf((float)D));
}

hipError_t launch_dq_f32(const BwdArgs& a, hipStream_t s) {
    const size_t rows = (size_t)a.B * a.H * a.L;
    if (a.d == 64) {
        if (pick_rows(rows, 2, 1024) == 2) dq_t<64, 2>(a, s);
        else dq_t<64, 1>(a, s);
    } else {
        dq_t<128, 1>(a, s);
    }
    return hipGetLastError();
}

template <int D, int T>
static void dkdv_t(const BwdArgs& a, hipStream_t s) {
    const int nb = a.L / (16 * T), nblocks = a.B * a.H * nb;
    hipLaunchKernelGGL((dkdv_f32_kernel<D, T>), dim3(nblocks), dim3(kF32Threads), 0, s,
                       (const float*)a.Q, (const float*)a.K, (const float*)a.V, (const float*)a.dO,
                       a.c, a.col_end, a.lse2, a.dsum, (float*)a.dK, (float*)a.dV, a.colsum, a.L,
                       a.L / kBlock, nb, nblocks, kLog2e / sqrtf((float)D), 1.0f / sqrtf((float)D));
}

hipError_t launch_dkdv_f32(const BwdArgs& a, hipStream_t s) {
    const size_t rows = (size_t)a.B * a.H * a.L;
    if (a.d == 64) {
        if (pick_rows(rows, 2, 1024) == 2) dkdv_t<64, 2>(a, s);
        else dkdv_t<64, 1>(a, s);
    } else {
        dkdv_t<128, 1>(a, s);
    }
    return hipGetLastError();
}

}  // namespace acp
