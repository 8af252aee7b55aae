// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation, one fused multiply-add per
// product, so nothing is rounded that a plain FMA loop would not round).
//
// The bound is the fp32 matrix rate (157 TFLOP/s nominal, 139 for the vendor's product of 4096^3): a 16x16x4 MFMA takes
// 32 cycles of its SIMD and its two operand fragments are one float per lane each, so LDS and L2 feed it easily and no
// direct-to-LDS machinery is needed; what the shapes of this path (a few thousand rows, 128 .. 512 columns) lack is
// work-groups.  Hence 64 x 64 tiles: 4 wavefronts stacked along M, each 16 x 64, 32-deep K tiles staged global ->
// registers -> LDS in two stages (37 KB: four work-groups per CU cover each other's waits), the tile after the next
// requested while one is multiplied (one tile ahead: 1477 us for the stage below, two: 1450).  128-row tiles are
// mixed: at 4096^3 NT 117 TFLOP/s against 111, NN 112 against 109, TN 110 against 116; NT 12 288 x 512 x 2048 87 against 105,
// NN 7684 x 768 x 256 82 against 87.  A stage's widths here are the latter kind, so they are left out; 64-deep K tiles are
// mixed too (4096^3: NN 99 against 110, NT 111 against 111).
// Where the tiles do not give every CU two work-groups, KW = 2: eight wavefronts per work-group, the second four taking
// the second half of every K tile into accumulators of their own (added at the end through LDS), so that every SIMD still
// has two wavefronts (weight gradients of the d = 256 stage: 56 -> 42 us).
//
// Measured per launch, averaged over the stage of d = 256, d_ff = 1024 at 7 684 tokens, against the scalar FMA kernel of
// gemm.hip (which keeps what float4 cannot read): forward and input-gradient products 32 / 51 us (d / d_ff columns)
// against 103 / 121; weight gradients 41 us against 1536 (16 to 64 work-groups, nothing split over the tokens).
//
// Orders of the operands in LDS.  A contraction step of the MFMA takes 4 k values, one per 16-lane group g; step (u, j)
// of a tile uses k = 16 u + 4 g + j for every operand.  An operand with contiguous k is stored [row][36] and read as
// float4 (j = 0..3 of one u); an operand with k as its row is stored [k][cols + 4] and read as single floats (4 k rows
// 4 apart land 16 banks apart).  B columns are stored in the order (n/32, (n/4)%2, (n/8)%4, n%4), so that the accumulator
// blocks 2p, 2p+1 of a lane hold 8 CONSECUTIVE columns 32 p + 8 g .. + 7 of its row: the epilogue works on them in
// registers, 128 contiguous bytes per row and group of 4 lanes, without going through LDS again.
#include "gemm_epilogue.hpp"

namespace {

constexpr int F_BK = 32, F_BM = 64, F_BN = 64;
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
                const int r = r0 + (u / (F_BK / 4)), k = k0 + (u % (F_BK / 4)) * 4;
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
                const int r = u / (F_BK / 4);
                *reinterpret_cast<float4*>(tile + (PERM ? col_slot(r) : r) * F_LDK + (u % (F_BK / 4)) * 4) = v[i];
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
template <int EPI, bool AKC, bool BKC, int KW>
__global__ __launch_bounds__(256 * KW) void gemm_f32_mfma_kernel(int M, int N, int K, const float* __restrict__ A, long long lda,
                                                            const float* __restrict__ B, long long ldb, float* __restrict__ C,
                                                            int k_per_split, float* __restrict__ split_ws, GemmEpi p) {
    typedef TileF32<F_BM, AKC, false, 256 * KW> TA;
    typedef TileF32<F_BN, BKC, true, 256 * KW> TB;
    __shared__ __attribute__((aligned(16))) float smem[2][TA::FLOATS + TB::FLOATS];
    const int t = threadIdx.x, lane = t & 63, wave = (t >> 6) & 3, kw = t >> 8;
    const int m0 = blockIdx.y * F_BM, n0 = blockIdx.x * F_BN;
    const int k_begin = blockIdx.z * k_per_split;
    const int k_end = (k_begin + k_per_split) < K ? k_begin + k_per_split : K;
    f32x4_t acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0.f;

    // two tiles ahead: while tile i is multiplied, tile i + 1 is in registers or on its way there and tile i + 2 is requested
    TA ta[2];
    TB tb[2];
    auto load = [&](int set, int k0) {
        if (k0 >= k_end) return;
        ta[set].load(A, lda, m0, M, k0, k_end, t);
        tb[set].load(B, ldb, n0, N, k0, k_end, t);
    };
    auto store = [&](int set) {
        ta[set].store(smem[set], t);
        tb[set].store(smem[set] + TA::FLOATS, t);
    };
    auto multiply = [&](int set) {
        const float* sa = smem[set];
        const float* sb = sa + TA::FLOATS;
#pragma unroll
        for (int u0 = 0; u0 < F_BK / 16; u0 += KW) {
            const int u = u0 + kw;
            float fa[4], fb[4][4];
            TA::frag(sa, wave * 16, u, lane, fa);
#pragma unroll
            for (int j = 0; j < 4; ++j) TB::frag(sb, j * 16, u, lane, fb[j]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][s], fa[s], acc[j], 0, 0, 0);
        }
    };
    load(0, k_begin);
    load(1, k_begin + F_BK);
    store(0);
    __syncthreads();
    auto step = [&](int set, int k0) {                                // tile at k0 lies in stage `set`
        load(set, k0 + 2 * F_BK);
        multiply(set);
        if (k0 + F_BK < k_end) {                                      // the other stage was last read before the previous barrier
            store(set ^ 1);
            __syncthreads();
        }
    };
    for (int k0 = k_begin; k0 < k_end; k0 += 2 * F_BK) {
        step(0, k0);
        if (k0 + F_BK < k_end) step(1, k0 + F_BK);
    }
    if constexpr (KW == 2) {                                          // add the two halves of the contraction
        static_assert(F_BK / 16 % KW == 0, "whole 16-deep groups per half");
        f32x4_t* part = reinterpret_cast<f32x4_t*>(&smem[0][0]);      // [4][256]
        static_assert(4 * 256 * 16 <= sizeof(smem), "the partial accumulators fit in the operand stages");
        __syncthreads();
        if (kw == 1) {
#pragma unroll
            for (int j = 0; j < 4; ++j) part[j * 256 + (t & 255)] = acc[j];
        }
        __syncthreads();
        if (kw == 1) return;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += part[j * 256 + t];
    }
    const int m = m0 + wave * 16 + (lane & 15);
    if (m >= M) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int n = n0 + 32 * q + 8 * (lane >> 4);
        if (n >= N) continue;                                         // (N is a multiple of 8)
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = acc[2 * q][e]; v[4 + e] = acc[2 * q + 1][e]; }
        if (gridDim.z > 1) Vec8<float>::store(split_ws + ((size_t)blockIdx.z * M + m) * N + n, v);
        else epilogue8<float, EPI>(m, n, N, v, C, p);
    }
}

template <int EPI, bool AKC, bool BKC>
ds_status launch_form(int M, int N, int K, const float* A, const float* B, float* C, const GemmEpi& p, float* split_ws,
                      size_t split_ws_floats, hipStream_t st) {
    const int n_cu = gemm_cu_count();
    const int gn = (N + F_BN - 1) / F_BN, gm = (M + F_BM - 1) / F_BM;
    const long long lda = AKC ? K : M, ldb = BKC ? K : N, tiles = (long long)gn * gm;
    // A contraction far longer than the output is wide (weight gradients: every token of the batch) is cut into K ranges
    // until about two work-groups per CU run, each range at least 4 tiles deep; the partial sums stay within the workspace.
    int splits = 1;
    if (split_ws && tiles < 2 * n_cu) {
        splits = (int)((2 * n_cu + tiles - 1) / tiles);
        const int by_k = K / (4 * F_BK);
        if (splits > by_k) splits = by_k;
        const size_t by_ws = split_ws_floats / ((size_t)M * N);
        if ((size_t)splits > by_ws) splits = (int)by_ws;
        if (splits < 1) splits = 1;
    }
    int per = (K + splits - 1) / splits;
    per = (per + F_BK - 1) / F_BK * F_BK;
    splits = (K + per - 1) / per;
    if (tiles * splits >= 2 * n_cu)
        hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI, AKC, BKC, 1>), dim3(gn, gm, splits), dim3(256), 0, st, M, N, K, A, lda, B,
                           ldb, C, per, split_ws, p);
    else
        hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI, AKC, BKC, 2>), dim3(gn, gm, splits), dim3(512), 0, st, M, N, K, A, lda, B,
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
