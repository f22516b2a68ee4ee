// Q and K projections with the row-norm maxima of stage 1 in their epilogue
// (the fusion of the bound's norm pass into the upstream producer that the
// paper's two-stage design allows: U needs only the largest row norms of the
// stored Q and K, Sec. 3).
//
//   [Q | K] = X [Wq | Wk]     X [B*L, Dm], Wq and Wk [Dm, H*d] (row-major, bf16)
//
// One workgroup computes a 128 x 128 tile of the product (256 threads), or 256 x 256
// (512; project_big), with bf16 MFMA (float32 accumulation), K-blocks of 64 staged
// through LDS by DMA and double-buffered.  Its epilogue rounds the tile to bfloat16, writes every row
// straight into the head-split [B, H, L, d] layout, and forms, per head in the
// tile, the largest float64 sum of squares of the stored row (ascending feature
// order), which is the 128-row chunk maximum that rownorm_max_kernel would
// produce for the same Q and K.
#include "acp_device.h"
#include "acp_internal.h"

namespace acp {

constexpr int kPrjCols = 128;   // columns of a block (one of Wq or of Wk)
constexpr int kPrjK = 64;       // depth of one K-block

// DMA of a 64 x 64*P bf16 block of a row-major matrix with row stride ld
// (elements) into an LDS tile laid out as tile_off describes (P column panels).
// Instruction i of the 8 P per block fills LDS bytes [1024 i, 1024 i + 1024).
template <int P, int NWAVES>
struct StridedDma {
    static constexpr int kInst = 8 * P;
    static constexpr int kPer = kInst / NWAVES;
    unsigned off[kPer];
    __device__ __forceinline__ void init(int wave, int lane, int ld) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = wave + NWAVES * k;
            const int row = 8 * (i & 7) + (lane >> 3);
            const int chunk = (lane & 7) ^ tile_swz(row);
            off[k] = (unsigned)(2 * (row * ld + ((i >> 3) << 6) + 8 * chunk));
        }
    }
    __device__ __forceinline__ void issue(unsigned char* tile, const __bf16* src, int wave) const {
        typedef __attribute__((address_space(3))) unsigned char lds_u8;
        const unsigned long long p = reinterpret_cast<unsigned long long>(src);
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
        const unsigned long long base = ((unsigned long long)hi << 32) | lo;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = wave + NWAVES * k;
            const unsigned lds = __builtin_amdgcn_readfirstlane(
                (unsigned)(unsigned long long)(const lds_u8*)(tile + 1024 * i));
            // One wait state between the SALU write of M0 and the LDS DMA that
            // reads it (a gfx9-family hazard that the compiler's hazard check
            // cannot see inside this statement).  Nothing in these kernels keeps
            // a value in M0 across it (DS instructions do not read M0 on gfx9 and
            // later), so the clobber costs nothing.
            asm volatile(
                "s_mov_b32 m0, %0\n\t"
                "s_nop 0\n\t"
                "global_load_lds_dwordx4 %1, %2"
                :
                : "s"(lds), "v"(off[k]), "s"(base)
                : "memory", "m0");
        }
    }
};

// A workgroup's tile is MB blocks of 64 rows by NB blocks of 128 columns, its 4 NB waves
// each taking 32 MB rows by 64 columns.
template <int MB, int NB>
struct PrjSmem {
    static constexpr int kRows = 64 * MB, kCols = kPrjCols * NB;
    union {
        struct {
            unsigned char a[2][MB][64 * 128];   // X: 64-row blocks of 64 columns
            unsigned char b[2][NB][64 * 256];   // W: 64 rows x 128 columns (two panels)
        } in;
        __bf16 out[kRows][kCols + 8];           // the rounded tile, padded rows
    };
    double rmax[2 * NB][MB];                    // per head of the tile and 64-row block
};

template <int D, int MB, int NB>
__global__ __launch_bounds__(256 * NB) void qk_project_kernel(
    const __bf16* __restrict__ X, const __bf16* __restrict__ Wq, const __bf16* __restrict__ Wk,
    int M, int L, int Dm, int H, __bf16* __restrict__ Qo, __bf16* __restrict__ Ko,
    double* __restrict__ part, int nchunk) {
    constexpr int kRows = PrjSmem<MB, NB>::kRows, kCols = PrjSmem<MB, NB>::kCols;
    constexpr int kThreads = 256 * NB, kWaves = 4 * NB, kI = 2 * MB;
    __shared__ PrjSmem<MB, NB> sm;
    const int HD = H * D;
    // All column tiles of a row block of X run on one XCD (a contiguous range of
    // logical ids per XCD), so that the block is fetched into one L2 only.
    const int ntn = 2 * HD / kCols;
    const int lid = xcd_logical_id(blockIdx.x, gridDim.x);
    const int tn = lid % ntn, tm = lid / ntn;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / (2 * NB), wn = w % (2 * NB);   // the wave's half of the rows, its 64 columns
    const int g = lane >> 4, r16 = lane & 15;
    const int m0 = tm * kRows;
    // Column block j of the tile: 128 columns of [Q | K], of Wq or of Wk (H d is a
    // multiple of 128, so a block never straddles)
    auto which_of = [&](int j) { return tn * kCols + kPrjCols * j >= HD ? 1 : 0; };
    auto col_of = [&](int j) { return tn * kCols + kPrjCols * j - which_of(j) * HD; };

    StridedDma<1, kWaves> dma_a;
    StridedDma<2, kWaves> dma_b;
    dma_a.init(w, lane, Dm);
    dma_b.init(w, lane, HD);
    auto issue = [&](int kb, int buf) __attribute__((always_inline)) {
        const int k0 = kb * kPrjK;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            // (a block past the last row reads the first again; M is a multiple of 128)
            const int row = i < 2 || m0 + 64 * i < M ? m0 + 64 * i : m0;
            dma_a.issue(sm.in.a[buf][i], X + (size_t)row * Dm + k0, w);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)
            dma_b.issue(sm.in.b[buf][j], (which_of(j) == 0 ? Wq : Wk) + (size_t)k0 * HD + col_of(j), w);
    };

    f32x4 acc[kI][4];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The product is formed transposed, C^T = W^T X^T (W columns as the A operand,
    // X rows as the B operand), so that each lane ends with four consecutive
    // columns of one row of C: lane (g, r) holds C[16 i + r][16 j + 4 g + u].
    // (Spreading the next K-block's DMA over this block's MFMAs measured slower.)
    const int nkb = Dm / kPrjK;
    issue(0, 0);
    for (int kb = 0; kb < nkb; ++kb) {
        const int buf = kb & 1;
        wait_vmcnt0();
        __syncthreads();                          // block kb landed; block kb - 1 read
        const bool more = kb + 1 < nkb;
        if (more) issue(kb + 1, buf ^ 1);
        const unsigned char* bt = sm.in.b[buf][wn >> 1];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 af[kI], bfr[4];
#pragma unroll
            for (int i = 0; i < kI; ++i)
                af[i] = tile_row8(sm.in.a[buf][(MB / 2) * wm + (i >> 2)], 16 * (i & 3) + r16, 32 * ks + 8 * g);
#pragma unroll
            for (int j = 0; j < 4; ++j) bfr[j] = tile_col8(bt, 32 * ks + 8 * g, 64 * (wn & 1) + 16 * j, r16);
#pragma unroll
            for (int i = 0; i < kI; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = mfma16(bfr[j], af[i], acc[i][j]);
        }
    }

    // ---- epilogue: the rounded tile through LDS ----------------------------------
    __syncthreads();                              // every wave is done with the inputs
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bf16x4 v;
            v[0] = (__bf16)acc[i][j][0]; v[1] = (__bf16)acc[i][j][1];
            v[2] = (__bf16)acc[i][j][2]; v[3] = (__bf16)acc[i][j][3];
            *reinterpret_cast<bf16x4*>(&sm.out[32 * MB * wm + 16 * i + r16][64 * wn + 16 * j + 4 * g]) = v;
        }
    __syncthreads();

    // Largest sum of squares per head of the tile and 64-row block: a thread per (row,
    // head), a wave per 64 rows of one head
    constexpr int kPerBlock = kPrjCols / D, kHeads = NB * kPerBlock;   // (D = 64: two heads per block)
#pragma unroll
    for (int k = 0; k < (kRows * kHeads + kThreads - 1) / kThreads; ++k) {
        const int i = tid + kThreads * k, row = i % kRows, hh = i / kRows;
        double ss = 0.0;
        if (hh < kHeads) {
#pragma unroll 2
            for (int e8 = 0; e8 < D; e8 += 8) {
                const bf16x8 v = *reinterpret_cast<const bf16x8*>(&sm.out[row][D * hh + e8]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const double x = (double)(float)v[e];
                    ss = __builtin_fma(x, x, ss);
                }
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) ss = nan_max(ss, __shfl_xor(ss, off));
        if (lane == 0 && hh < kHeads) sm.rmax[hh][row >> 6] = ss;
    }
    __syncthreads();
    // The tile in blocks of 128 rows by 128 columns, each of one sequence (L and M are
    // multiples of 128) and of Q or K: everything but the row and piece is uniform.
#pragma unroll
    for (int c = 0; c < MB / 2; ++c) {
        const int mc = m0 + 128 * c;
        if (mc >= M) break;
        const int b = mc / L, l0 = mc - b * L;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int which = which_of(j), col0 = col_of(j), h0 = col0 / D;
            if (tid < kPerBlock) {
                const int hh = kPerBlock * j + tid;
                part[((size_t)(b * H + h0 + tid) * 2 + which) * nchunk + l0 / 128] =
                    nan_max(sm.rmax[hh][2 * c], sm.rmax[hh][2 * c + 1]);
            }
            // rows into [B, H, L, d]: 16-byte pieces, consecutive lanes along a row
            __bf16* out = (which == 0 ? Qo : Ko) + (((size_t)b * H + h0) * L + l0) * D;
            constexpr int kPieces = kPrjCols / 8;
#pragma unroll
            for (int k = 0; k < 128 * kPieces / kThreads; ++k) {
                const int i = tid + kThreads * k, row = i / kPieces, col = 8 * (i % kPieces);
                const uint4 v = *reinterpret_cast<const uint4*>(&sm.out[128 * c + row][kPrjCols * j + col]);
                *reinterpret_cast<uint4*>(out + ((size_t)(col / D) * L + row) * D + col % D) = v;
            }
        }
    }
}

template <int D, int MB, int NB>
static void project_t(const ProjectArgs& a, hipStream_t s) {
    const int M = a.B * a.L, HD = a.H * a.d;
    const int tiles = (2 * HD / (kPrjCols * NB)) * ((M + 64 * MB - 1) / (64 * MB));
    hipLaunchKernelGGL((qk_project_kernel<D, MB, NB>), dim3(tiles), dim3(256 * NB), 0, s,
                       (const __bf16*)a.X, (const __bf16*)a.Wq, (const __bf16*)a.Wk, M, a.L, a.Dm,
                       a.H, (__bf16*)a.Q, (__bf16*)a.K, a.part, a.nchunk);
}

// The 256 x 256 tile or the 128 x 128 one.  The large tile reads half as much through L2
// per product (the small one's loop is bound by that: 0.9 PFLOP/s), but a CU holds one
// workgroup, whose prologue and epilogue nothing overlaps.  Measured over 400 shapes
// (d_model 512 to 2048, 60 to 1500 large tiles), a round of large tiles (256 at once), which
// does the work of two of the small ones (512 at once), takes 1.6 + 165 / d_model of one, and a
// last round of at most 256 small tiles, one to a CU, 0.6.  With that the tile taken is the
// slower one by more than 3% in 12 of them (at most 9%).  us, small -> large: 32768 x 1536 x
// 768 104 -> 98, 32768 x 2048 x 1024 153 -> 139, 32768 x 3072 x 1536 346 -> 303, 16384 x 2048 x
// 1024 (d = 128) 80 -> 68; against the rule: 8192 x 2560 x 1280 (320 large tiles) 61 -> 78, 4096 x
// 1536 x 768 (96) 20 -> 29, 28672 x 2048 x 512 (896) 72.8 -> 79.3, 8192 x 1536 x 512 (192) 21 -> 24.
static bool project_big(int M, int N, int Dm) {
    const int small = (M / 128) * (N / 128), large = ((M + 255) / 256) * (N / 256);
    const int rest = small % 512;
    const double rounds = small / 512 + (rest == 0 ? 0.0 : rest <= 256 ? 0.6 : 1.0);
    return Dm >= 512 && (1.6 + 165.0 / Dm) * ((large + 255) / 256) <= rounds;
}

hipError_t launch_qk_project(const ProjectArgs& a, hipStream_t s) {
    trace_begin(ACP_K_PROJECT, s);
    const bool big = project_big(a.B * a.L, 2 * a.H * a.d, a.Dm);
    if (a.d == 64) {
        if (big) project_t<64, 4, 2>(a, s);
        else project_t<64, 2, 1>(a, s);
    } else {
        if (big) project_t<128, 4, 2>(a, s);
        else project_t<128, 2, 1>(a, s);
    }
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) trace_end(ACP_K_PROJECT, s);
    return e;
}

}  // namespace acp
