// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation, one fused multiply-add per
// product, so nothing is rounded that a plain FMA loop would not round).
//
// The bound is the fp32 matrix rate (157 TFLOP/s nominal, 139 for the vendor's product of 4096^3): a 16x16x4 MFMA takes
// 32 cycles of its SIMD and its two operand fragments are one float per lane each, so LDS and L2 feed it easily and no
// direct-to-LDS machinery is needed; what the shapes of this path (a few thousand rows, 128 .. 512 columns) lack is
// work-groups.  Hence small tiles: 4 wavefronts stacked along M, each 16 RB x 64, i.e. 64 x 64 (RB = 1) or 128 x 64
// (RB = 2) per work-group, 32-deep K tiles staged global -> registers -> LDS in two stages (37 / 55 KB: four / two
// work-groups per CU cover each other's waits).  RB = 2 halves the B traffic per product; it is taken when the 128-row
// tiles alone give every CU two work-groups.  Where not even the 64 x 64 tiles do, KW = 2: eight wavefronts per
// work-group, the second four taking the second half of every K tile into accumulators of their own (added at the end
// through LDS), so that every SIMD still has two wavefronts (weight gradients of the d = 256 stage: 56 -> 42 us).
//
// Measured per launch, averaged over the stage of d = 256, d_ff = 1024 at 7 684 tokens, against the scalar FMA kernel of
// gemm.hip (which keeps what float4 cannot read): forward and input-gradient products 33 / 58 us (d / d_ff columns)
// against 103 / 121; weight gradients 42 us against 1536 (16 to 64 work-groups, nothing split over the tokens).
//
// Orders of the operands in LDS.  A contraction step of the MFMA takes 4 k values, one per 16-lane group g; step (u, j)
// of a tile uses k = 16 u + 4 g + j for every operand.  An operand with contiguous k is stored [row][36] and read as
// float4 (j = 0..3 of one u); an operand with k as its row is stored [k][cols + 4] and read as single floats (4 k rows
// 4 apart land 16 banks apart).  B columns are stored in the order (n/32, (n/4)%2, (n/8)%4, n%4), so that the accumulator
// blocks 2p, 2p+1 of a lane hold 8 CONSECUTIVE columns 32 p + 8 g .. + 7 of its row: the epilogue works on them in
// registers, 128 contiguous bytes per row and group of 4 lanes, without going through LDS again.
#include "gemm_epilogue.hpp"

namespace {

constexpr int F_BK = 32, F_BN = 64;
constexpr int F_LDK = F_BK + 4;                      // row stride (floats) of a k-contiguous tile: 16 rows hit 64 banks

__device__ __forceinline__ int col_slot(int n) { return (n & ~31) | ((n & 4) << 2) | ((n & 24) >> 1) | (n & 3); }

// One operand's tile: ROWS rows (m or n) x 32 k, KC: k contiguous in memory.  PERM: rows are output columns (see above).
// NT threads.  Held in registers between the global read and the LDS write.
template <int ROWS, bool KC, bool PERM, int NT> struct TileF32 {
    static constexpr int NV = ROWS * F_BK / 4 / NT;                   // float4 per thread
    static constexpr int LD = KC ? F_LDK : ROWS + 4;
    static constexpr int FLOATS = KC ? ROWS * F_LDK : F_BK * (ROWS + 4);
    float4 v[NV];
    // src: first element of the operand; ld: its row stride; r0, k0: corner; limits: rows, k (exclusive)
    __device__ __forceinline__ void load(const float* __restrict__ src, long long ld, int r0, int rows, int k0, int k_end, int t) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int u = t + NT * i;
            v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (KC) {                                       // (k ranges are multiples of 4)
                const int r = r0 + (u >> 3), k = k0 + (u & 7) * 4;
                if (r < rows && k < k_end) v[i] = *reinterpret_cast<const float4*>(src + (long long)r * ld + k);
            } else {                                                  // (row counts are multiples of 4)
                constexpr int Q = ROWS / 4;
                const int k = k0 + u / Q, r = r0 + (u % Q) * 4;
                if (k < k_end && r < rows) v[i] = *reinterpret_cast<const float4*>(src + (long long)k * ld + r);
            }
        }
    }
    __device__ __forceinline__ void store(float* tile, int t) const {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int u = t + NT * i;
            if constexpr (KC) {
                const int r = u >> 3;
                *reinterpret_cast<float4*>(tile + (PERM ? col_slot(r) : r) * F_LDK + (u & 7) * 4) = v[i];
            } else {
                constexpr int Q = ROWS / 4;
                const int r = (u % Q) * 4;
                *reinterpret_cast<float4*>(tile + (u / Q) * LD + (PERM ? col_slot(r) : r)) = v[i];
            }
        }
    }
    // fragment of 16-row block at `row` (in LDS order) for the 4 contraction steps of 16-deep group u
    __device__ static __forceinline__ void frag(const float* tile, int row, int u, int lane, float (&f)[4]) {
        const int r = row + (lane & 15), g = lane >> 4;
        if constexpr (KC) {
            const float4 x = *reinterpret_cast<const float4*>(tile + r * F_LDK + 16 * u + 4 * g);
            f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = tile[(16 * u + 4 * g + j) * LD + r];
        }
    }
};

// C[M,N] = A * B with A(m,k) = A[m*lda + k] (AKC) or A[k*lda + m], B(k,n) = B[n*ldb + k] (BKC) or B[k*ldb + n].
// gridDim = (N tiles, M tiles, K splits); with more than one split the partial sums go to split_ws as [split][M][N].
template <int EPI, bool AKC, bool BKC, int RB, int KW>
__global__ __launch_bounds__(256 * KW) void gemm_f32_mfma_kernel(int M, int N, int K, const float* __restrict__ A, long long lda,
                                                            const float* __restrict__ B, long long ldb, float* __restrict__ C,
                                                            int k_per_split, float* __restrict__ split_ws, GemmEpi p) {
    constexpr int BM = 64 * RB;
    typedef TileF32<BM, AKC, false, 256 * KW> TA;
    typedef TileF32<F_BN, BKC, true, 256 * KW> TB;
    __shared__ __attribute__((aligned(16))) float smem[2][TA::FLOATS + TB::FLOATS];
    const int t = threadIdx.x, lane = t & 63, wave = (t >> 6) & 3, kw = t >> 8;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * F_BN;
    const int k_begin = blockIdx.z * k_per_split;
    const int k_end = (k_begin + k_per_split) < K ? k_begin + k_per_split : K;
    f32x4_t acc[RB][4];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

    TA ta;
    TB tb;
    ta.load(A, lda, m0, M, k_begin, k_end, t);
    tb.load(B, ldb, n0, N, k_begin, k_end, t);
    ta.store(smem[0], t);
    tb.store(smem[0] + TA::FLOATS, t);
    __syncthreads();
    int cur = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += F_BK, cur ^= 1) {
        const bool more = k0 + F_BK < k_end;
        if (more) {                                                   // in flight while this tile is multiplied
            ta.load(A, lda, m0, M, k0 + F_BK, k_end, t);
            tb.load(B, ldb, n0, N, k0 + F_BK, k_end, t);
        }
        const float* sa = smem[cur];
        const float* sb = sa + TA::FLOATS;
#pragma unroll
        for (int u0 = 0; u0 < F_BK / 16; u0 += KW) {
            const int u = u0 + kw;
            float fa[RB][4], fb[4][4];
#pragma unroll
            for (int i = 0; i < RB; ++i) TA::frag(sa, (wave * RB + i) * 16, u, lane, fa[i]);
#pragma unroll
            for (int j = 0; j < 4; ++j) TB::frag(sb, j * 16, u, lane, fb[j]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][s], fa[i][s], acc[i][j], 0, 0, 0);
        }
        if (more) {                                                   // the other stage was last read before the previous barrier
            ta.store(smem[cur ^ 1], t);
            tb.store(smem[cur ^ 1] + TA::FLOATS, t);
            __syncthreads();
        }
    }
    if constexpr (KW == 2) {                                          // add the two halves of the contraction
        static_assert(F_BK / 16 == 2, "one 16-deep group per half");
        f32x4_t* part = reinterpret_cast<f32x4_t*>(&smem[0][0]);      // [RB * 4][256]
        static_assert(RB * 4 * 256 * 16 <= sizeof(smem), "the partial accumulators fit in the operand stages");
        __syncthreads();
        if (kw == 1) {
#pragma unroll
            for (int i = 0; i < RB * 4; ++i) part[i * 256 + (t & 255)] = acc[i >> 2][i & 3];
        }
        __syncthreads();
        if (kw == 1) return;
#pragma unroll
        for (int i = 0; i < RB * 4; ++i) acc[i >> 2][i & 3] += part[i * 256 + t];
    }
    const int g = lane >> 4;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int m = m0 + (wave * RB + i) * 16 + (lane & 15);
        if (m >= M) continue;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int n = n0 + 32 * q + 8 * g;
            if (n >= N) continue;                                     // (N is a multiple of 8)
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = acc[i][2 * q][e]; v[4 + e] = acc[i][2 * q + 1][e]; }
            if (gridDim.z > 1) Vec8<float>::store(split_ws + ((size_t)blockIdx.z * M + m) * N + n, v);
            else epilogue8<float, EPI>(m, n, N, v, C, p);
        }
    }
}

template <int EPI, bool AKC, bool BKC>
ds_status launch_form(int M, int N, int K, const float* A, const float* B, float* C, const GemmEpi& p, float* split_ws,
                      size_t split_ws_floats, hipStream_t st) {
    const int n_cu = gemm_cu_count();
    const int gn = (N + F_BN - 1) / F_BN, gm64 = (M + 63) / 64, gm128 = (M + 127) / 128;
    const long long lda = AKC ? K : M, ldb = BKC ? K : N;
    const bool big = (long long)gn * gm128 >= 2 * n_cu;
    // A contraction far longer than the output is wide (weight gradients: every token of the batch) is cut into K ranges
    // until about two work-groups per CU run, each range at least 4 tiles deep; the partial sums stay within the workspace.
    int splits = 1;
    if (split_ws && !big) {
        const int tiles = gn * gm64;
        splits = (2 * n_cu + tiles - 1) / tiles;
        const int by_k = K / (4 * F_BK);
        if (splits > by_k) splits = by_k;
        const size_t by_ws = split_ws_floats / ((size_t)M * N);
        if ((size_t)splits > by_ws) splits = (int)by_ws;
        if (splits < 1) splits = 1;
    }
    int per = (K + splits - 1) / splits;
    per = (per + F_BK - 1) / F_BK * F_BK;
    splits = (K + per - 1) / per;
    if (big)
        hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI, AKC, BKC, 2, 1>), dim3(gn, gm128, splits), dim3(256), 0, st, M, N, K, A, lda, B,
                           ldb, C, per, split_ws, p);
    else if ((long long)gn * gm64 * splits >= 2 * n_cu)
        hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI, AKC, BKC, 1, 1>), dim3(gn, gm64, splits), dim3(256), 0, st, M, N, K, A, lda, B,
                           ldb, C, per, split_ws, p);
    else
        hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI, AKC, BKC, 1, 2>), dim3(gn, gm64, splits), dim3(512), 0, st, M, N, K, A, lda, B,
                           ldb, C, per, split_ws, p);
    DS_LAUNCH_CHECK();
    if (splits > 1) return launch_splitk_finish<float, EPI>(M, N, splits, split_ws, C, p, st);
    return DS_OK;
}

template <int EPI>
ds_status launch_epi(int ta, int tb, int M, int N, int K, const float* A, const float* B, float* C, const GemmEpi& p,
                     float* split_ws, size_t split_ws_floats, hipStream_t st) {
    if (ta) return launch_form<EPI, false, false>(M, N, K, A, B, C, p, split_ws, split_ws_floats, st);
    if (tb) return launch_form<EPI, true, true>(M, N, K, A, B, C, p, split_ws, split_ws_floats, st);
    return launch_form<EPI, true, false>(M, N, K, A, B, C, p, split_ws, split_ws_floats, st);
}

}  // namespace

// What the kernel's float4 reads need: 16-byte aligned operands and, per operand, a contiguous extent that is a multiple
// of 4 (N always is).  Row counts and the K of the weight-gradient form are arbitrary; both operands transposed is left
// to the generic kernel (nothing in the stage needs it).  The grid's second and third extents must fit in 16 bits.
bool gemm_f32_mfma_supported(int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B) {
    if (ta && tb) return false;
    if (ta ? M % 4 != 0 : K % 4 != 0) return false;
    return N % 8 == 0 && (M + 63) / 64 <= 65535 && ((uintptr_t)A & 15) == 0 && ((uintptr_t)B & 15) == 0;
}

ds_status launch_gemm_f32_mfma(int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B, void* C,
                               int32_t epilogue, const GemmEpi& p, float* split_ws, size_t split_ws_floats, hipStream_t st) {
    const float *a = (const float*)A, *b = (const float*)B;
    float* c = (float*)C;
    switch (epilogue) {
    case DS_EPI_NONE: return launch_epi<DS_EPI_NONE>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_GELU: return launch_epi<DS_EPI_GELU>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_RESID: return launch_epi<DS_EPI_RESID>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_DGELU: return launch_epi<DS_EPI_DGELU>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_ACC32: return launch_epi<DS_EPI_ACC32>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_GATE: return launch_epi<DS_EPI_GATE>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_DGATE: return launch_epi<DS_EPI_DGATE>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_GELU_D: return launch_epi<DS_EPI_GELU_D>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    case DS_EPI_MULR: return launch_epi<DS_EPI_MULR>(ta, tb, M, N, K, a, b, c, p, split_ws, split_ws_floats, st);
    }
    return DS_EINVAL;
}
