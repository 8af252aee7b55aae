// fp32 GEMM on the matrix cores, two kernels:
//   gemm_f32_split_kernel  eight bf16 products per fp32 one, where there are work-groups for it, and all weight gradients of a
//                          layer in one launch; described where it is defined
//   gemm_f32_mfma_kernel   v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation, one fused multiply-add per product, so nothing
//                          is rounded that a plain FMA loop would not round; the rest, described here
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
// Measured per launch at d = 256, d_ff = 1024, 7 684 tokens, against the scalar FMA kernel of gemm.hip (which keeps what float4
// cannot read): weight gradients 41 us against 1536 (16 to 64 work-groups, nothing split over the tokens).
//
// Orders of the operands in LDS.  A contraction step of the MFMA takes 4 k values, one per 16-lane group g; step (u, j)
// of a tile uses k = 16 u + 4 g + j for every operand.  An operand with contiguous k is stored [row][36] and read as
// float4 (j = 0..3 of one u); an operand with k as its row is stored [k][cols + 4] and read as single floats (4 k rows
// 4 apart land 16 banks apart).  B columns are stored in the order (n/32, (n/4)%2, (n/8)%4, n%4), so that the accumulator
// blocks 2p, 2p+1 of a lane hold 8 CONSECUTIVE columns 32 p + 8 g .. + 7 of its row: the epilogue works on them in
// registers, 128 contiguous bytes per row and group of 4 lanes, without going through LDS again.
#include "gemm_epilogue.hpp"

#include <type_traits>
#include <utility>

namespace {

constexpr int F_BK = 32, F_BM = 64, F_BN = 64;
constexpr int G_BM = 64, G_BN = 128;                   // the larger tile of the bf16 form
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

// ---------------------------------------------------------------------------- fp32 products on the bf16 matrix cores
// x = hi + mid + lo exactly, each a bf16 (8 significant bits of what the one before left; three parts of bf16 for one fp32 value are
// described by Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations",
// 2019), and
//   a b = hi hi + (hi mid + mid hi) + (hi lo + mid mid + lo hi) + (mid lo + lo mid) + less than 2^-30 |a b|
// so eight bf16 products give an fp32 one, at 2.5 PFLOP/s / 8 instead of the 157 TFLOP/s of the fp32 matrix instructions.  A
// product of two bf16 is exact in fp32.  The leading products and the seven small ones have accumulators of their own, added at the
// end, so that the small ones are not rounded at the size of the sum, and an MFMA adds 16 products at a time: against 64 bits
// the results are 1.5 to 3 times closer than those of an fp32 multiply-add per product (N(0, 1) x N(0, 0.02), K = 36 .. 1024:
// 0.4e-7 .. 1.9e-7 against 1.0e-7 .. 5.7e-7), and where a result is one product as close (largest error 5.99e-8 and 5.96e-8, root
// mean square 2.53e-8 both).  With the first six products only that was 1.6e-7 and 2.9e-8, and the stage below took 1 077 us
// instead of 1 137.
// hi is rounded (half away from zero, so that mid has either sign), mid and lo are truncations of the rest: integer and plain
// fp32 operations.
//
// What bounds it is the splitting beside the products: an element costs 6.5 vector instructions per work-group that reads it, and the
// vector unit and the matrix unit hardly work at the same time (2 wavefronts per SIMD, clocks per MFMA: 16x16x32 18 alone, 27 with
// four v_and_b32 beside it; 32x32x16 33 alone, 34.6 with four, 43 with eight: hence the latter).  The splitting of the next tile is
// spread between the MFMAs of the current one, pinned there.  4096^3, operands from memory: 955 us against 1 350 - 1 410 (with six
// products 838; timing builds with six: 495 without the splitting, 700 without the stores of the planes).  Loads go through buffers
// that end with the operand, without a test per lane.
//   Operands from memory, us, fp32 MFMA -> this: 7 684 rows, N = 768, K = 256 44 -> 38; N = 256, K = 1024 58 -> 44; N = 1024, K = 256
//   50 -> 44; N = K = 256 25 -> 17; 12 288 rows, N = 2048, K = 512 257 -> 195.  Two layers of d = 256, d_ff = 1024 over 7 684 tokens,
//   weight gradients in one launch: 1 449 -> 1 137.
__device__ __forceinline__ float maximum3_abs(float a, float b, float c) {       // NaN if one is NaN
    float r;
    asm("v_maximum3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// f(0), f(1), .. f(N - 1) with constant arguments
template <class F, int... I> __device__ __forceinline__ void unroll_list(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void unroll(F&& f) { unroll_list(f, std::make_integer_sequence<int, N>{}); }

// one element: bits of hi, mid, lo in the upper halves (what lies below is not part of them)
__device__ __forceinline__ void split_one(float x, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = __float_as_uint(x) + 0x8000u;
    const float r = x - __uint_as_float(h & 0xffff0000u);
    m = __float_as_uint(r);
    l = __float_as_uint(r - __uint_as_float(m & 0xffff0000u));
    asm volatile("" : "+v"(h), "+v"(m), "+v"(l));                     // here, between the MFMAs, not where the planes are stored
}
__device__ __forceinline__ uint32_t upper_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302); }

// One operand's K tile, ROWS rows (m or n) x 32 k, KC: k contiguous in memory.  In LDS three planes (hi, mid, lo) of
//   KC:   [row][64 bytes], 16-byte chunk c = 2 s + g (k = 16 s + 4 g .. + 3 and 16 s + 8 + 4 g .. + 3) at slot c ^ (row / 4) % 4
//   else: [k][2 ROWS bytes], 32-byte unit u of a k row at unit u ^ f(k), read through the LDS transpose read
// both of which give lane half g of MFMA s the same k order.  PERM: rows are output columns, bits 2 and 3 of their number
// swapped, which leaves 8 consecutive columns in accumulator registers 8 h .. 8 h + 7 of a lane.
template <int ROWS, bool KC, bool PERM> struct SplitTile {
    static constexpr int NC = ROWS * 4 / 256, PLANE = ROWS * 64;
    static constexpr int CPR = ROWS / 8;                              // not KC: chunks per k row
    f32x4_t v[2][NC][2];                                              // [tile parity][chunk][half]: on the way from memory
    uint32_t off[NC];                                                 // byte offset of a chunk within the tile in memory ...
    uint32_t lds[NC];                                                 // ... and in a plane
    const float* base;                                                // the tile at k = 0
    long long ld;
    int rows;                                                         // KC: rows that exist from there on; else: elements before the first
    __device__ __forceinline__ static int unit_swz(int k) { return ROWS == 128 ? (k & 3) * 2 : (k & 2); }
    __device__ __forceinline__ static int place(int r) { return PERM ? (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1) : r; }
    __device__ __forceinline__ void setup(const float* src, long long ld_, int r0, int rows_, int t) {
        ld = ld_;
        base = src + (KC ? (long long)r0 * ld_ : (long long)r0);
        rows = KC ? rows_ - r0 : r0;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int u = t + 256 * i;
            if constexpr (KC) {
                const int r = u >> 2, c = u & 3, at = place(r);
                off[i] = (uint32_t)((r * (int)ld_ + (c >> 1) * 16 + (c & 1) * 4) * 4);
                lds[i] = at * 64 + ((c ^ ((at >> 2) & 3)) << 4);
            } else {
                const int k = u / CPR, c = u % CPR;
                off[i] = (uint32_t)((k * (int)ld_ + c * 8) * 4);
                lds[i] = k * (ROWS * 2) + (((c >> 1) ^ unit_swz(k)) << 5) + (c & 1) * (PERM ? 8 : 16);    // PERM: the second half 16 on
            }
        }
    }
    // The tile at k0, through a buffer that ends where the operand does: rows (KC) or k rows past the end read as zeros, without a
    // test per lane.  What else lies outside: k beyond k_end in the last tile of KC operands is replaced by zeros, columns
    // beyond the operand's (not KC) belong to outputs that are not stored.  The buffer's length stays below 2^31, beyond every offset
    // within a tile and below that of the replaced ones, however long the operand is.
    __device__ __forceinline__ void load(int set, int k0, int k_end, int t) {
        const int left = k_end - k0;
        const long long end = KC ? (long long)rows * ld - k0 : (long long)left * ld - rows;
        const uint32_t bytes = left <= 0 || end <= 0 ? 0u : (uint32_t)(end < 0x1fffffff ? end * 4 : 0x7ffffffc);
        __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + (KC ? (long long)k0 : (long long)k0 * ld)), 0,
                                                                       (int)bytes, 0x00020000);
        constexpr int second = KC ? 32 : 16;                          // bytes from the first half of a chunk to the second
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint32_t o0 = off[i], o1 = off[i] + second;
            if (KC && left < F_BK) {
                const int k = ((t >> 1) & 1) * 16 + (t & 1) * 4;
                if (k >= left) o0 = 0xfffffff0u;
                if (k + 8 >= left) o1 = 0xfffffff0u;
            }
            v[set][i][0] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(buf, o0, 0, 0));
            v[set][i][1] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(buf, o1, 0, 0));
        }
    }
    // Splitting and storing a tile goes in steps of 3 to 8 vector instructions, handed out between MFMAs: 13 per chunk (an element,
    // an element, their dword of each plane, four times; then the stores).
    static constexpr int STEPS = 13 * NC;
    uint32_t h[2], m[2], l[2], o[3][4];
    template <int STEP> __device__ __forceinline__ void store_step(int set, char* tile, uint32_t& lost) {
        constexpr int i = STEP / 13, q = STEP % 13, pair = q / 3;
        if constexpr (q < 12 && q % 3 < 2) {
            split_one(v[set][i][pair >> 1][(pair & 1) * 2 + q % 3], h[q % 3], m[q % 3], l[q % 3]);
        } else if constexpr (q < 12) {
            o[0][pair] = upper_halves(h[0], h[1]);
            o[1][pair] = upper_halves(m[0], m[1]);
            o[2][pair] = upper_halves(l[0], l[1]);
            lost |= l[0] | l[1];
            asm volatile("" : "+v"(o[0][pair]), "+v"(o[1][pair]), "+v"(o[2][pair]), "+v"(lost));
        } else {
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                char* d = tile + p * PLANE + lds[i];
                if constexpr (KC || !PERM) {
                    *reinterpret_cast<uint4*>(d) = make_uint4(o[p][0], o[p][1], o[p][2], o[p][3]);
                } else {
                    *reinterpret_cast<uint2*>(d) = make_uint2(o[p][0], o[p][1]);
                    *reinterpret_cast<uint2*>(d + 16) = make_uint2(o[p][2], o[p][3]);
                }
            }
        }
    }
    // fragment (32 rows x 16 k) of the 32-row block `block` of a plane, MFMA s of the tile
    __device__ static __forceinline__ bf16x8_t frag(const char* tile, int plane, int block, int s, int lane) {
        if constexpr (KC) {
            const int row = block * 32 + (lane & 31);
            return *reinterpret_cast<const bf16x8_t*>(tile + plane * PLANE + row * 64 + (((2 * s + (lane >> 5)) ^ ((row >> 2) & 3)) << 4));
        } else {
            typedef short s16x4_t __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) s16x4_t* lds4_t;
            const int k = 4 * (lane >> 5) + ((lane & 15) >> 2), unit = block * 2 + ((lane >> 4) & 1);
            const char* q = tile + plane * PLANE + (16 * s + k) * (ROWS * 2) + ((unit ^ unit_swz(k)) << 5) + (lane & 3) * 8;
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)q);
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(q + 8 * ROWS * 2));
            return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    }
};

// C[M,N] = A * B with the orders of gemm_f32_mfma_kernel.  Grid: (N tiles, M tiles) with k_per_split = K, or, GRP, the work-groups of
// several weight gradients in a row.  4 wavefronts of (BM / 2) x (BN / 2).
template <int EPI, bool AKC, bool BKC, int BM, int BN, bool GRP>
__global__ __launch_bounds__(256, 2) void gemm_f32_split_kernel(int M, int N, int K, const float* __restrict__ A, long long lda,
                                                                const float* __restrict__ B, long long ldb, float* __restrict__ C,
                                                                int k_per_split, GemmEpi p,
                                                                std::conditional_t<GRP, TnGroup, NoGroup> grp) {
    typedef SplitTile<BM, AKC, false> TA;
    typedef SplitTile<BN, BKC, true> TB;
    constexpr int STAGE = 3 * (TA::PLANE + TB::PLANE);
    constexpr int NA = BM / 64, NB = BN / 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN, split = 0;
    float* partial = nullptr;
    if constexpr (GRP) {
        int l = xcd_contiguous(blockIdx.x, gridDim.x);
        const int i = tn_group_problem(grp, l);
        M = grp.p[i].M;
        N = grp.p[i].N;
        A = reinterpret_cast<const float*>(grp.p[i].A);
        B = reinterpret_cast<const float*>(grp.p[i].B);
        C = reinterpret_cast<float*>(grp.p[i].C);
        lda = M;
        ldb = N;
        // one block of the workspace per (split, tile): the problem's first one + split * its tiles + tile
        if (grp.splits > 1) partial = grp.block(grp.first[i] + l);
        const int tn = (N + BN - 1) / BN, tiles = (M + BM - 1) / BM * tn;
        split = l / tiles;
        l -= split * tiles;
        m0 = l / tn * BM;
        n0 = l % tn * BN;
    }
    const int k_begin = split * k_per_split;
    const int k_end = k_begin + k_per_split < K ? k_begin + k_per_split : K;
    f32x16_t acc[NA][NB], small[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = small[i][j][e] = 0.f;
    uint32_t lost = 0;

    TA ta;
    TB tb;
    ta.setup(A, lda, m0, M, t);
    tb.setup(B, ldb, n0, N, t);
    auto load = [&](int set, int k0) {
        ta.load(set, k0, k_end, t);
        tb.load(set, k0, k_end, t);
    };
    constexpr int STEPS = TA::STEPS + TB::STEPS, MFMAS = 16 * NA * NB;
    auto store_step = [&](auto set, auto k) {
        if constexpr (k < TA::STEPS) ta.template store_step<k>(set, smem + set * STAGE, lost);
        else tb.template store_step<k - TA::STEPS>(set, smem + set * STAGE + 3 * TA::PLANE, lost);
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;
    load(0, k_begin);
    load(1, k_begin + F_BK);
    unroll<STEPS>([&](auto k) { store_step(set0, k); });
    __syncthreads();
    // The tile at k0 lies in stage `set`: it is multiplied, and meanwhile the next one (in registers) split into the other stage, which
    // was last read before the previous barrier (past the last tile: zeros that nothing reads).
    auto step = [&](auto set, auto other, int k0) {
        load(set, k0 + 2 * F_BK);
        const char* sa = smem + set * STAGE;
        const char* sb = sa + 3 * TA::PLANE;
        bf16x8_t fa[2][NA][3], fb[2][NB][3];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int i = 0; i < NA; ++i) fa[ks][i][q] = TA::frag(sa, q, wm * NA + i, ks, lane);
#pragma unroll
                for (int j = 0; j < NB; ++j) fb[ks][j][q] = TB::frag(sb, q, wn * NB + j, ks, lane);
            }
        unroll<MFMAS>([&](auto n) {
            constexpr int qa[8] = {0, 1, 0, 1, 2, 0, 2, 1}, qb[8] = {0, 0, 1, 1, 0, 2, 1, 2};
            constexpr int ks = n / (8 * NA * NB), q = n / (NA * NB) % 8, i = n / NB % NA, j = n % NB;
            if constexpr (q == 0) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j][0], fa[ks][i][0], acc[i][j], 0, 0, 0);
            else small[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j][qb[q]], fa[ks][i][qa[q]], small[i][j], 0, 0, 0);
            constexpr int from = n * STEPS / MFMAS, to = (n + 1) * STEPS / MFMAS;
            __builtin_amdgcn_sched_barrier(0);
            unroll<to - from>([&](auto k) { store_step(other, std::integral_constant<int, from + k>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    };
    for (int k0 = k_begin; k0 < k_end; k0 += 2 * F_BK) {
        step(set0, set1, k0);
        if (k0 + F_BK < k_end) step(set1, set0, k0 + F_BK);
    }
    // Where an element has bits that its three parts do not hold, or a result is not finite (an operand that is not, a part that
    // is not, products next to the largest float): the tile again with fp32 products.
    bool again = (lost & 0xffff) != 0;
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            float largest[2] = {0.f, 0.f};                            // per 8 columns
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] += small[i][j][e];
#pragma unroll
            for (int e = 0; e < 16; e += 2) largest[e >> 3] = maximum3_abs(largest[e >> 3], acc[i][j][e], acc[i][j][e + 1]);
            const int m = m0 + wm * (BM / 2) + i * 32 + (lane & 31);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int n = n0 + wn * (BN / 2) + 32 * j + 16 * h + 8 * (lane >> 5);
                again |= m < M && n < N && !(largest[h] < __builtin_inff());
            }
        }
    again = __syncthreads_or(again);
    if (again) {
        const float* pa[NA];
        const float* pb[NB];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int m = min(m0 + wm * (BM / 2) + i * 32 + (lane & 31), M - 1);
            pa[i] = A + (AKC ? (long long)m * lda : (long long)m);
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int n = min(n0 + wn * (BN / 2) + 32 * j + TB::place(lane & 31), N - 1);
            pb[j] = B + (BKC ? (long long)n * ldb : (long long)n);
        }
        for (int k0 = k_begin; k0 < k_end; k0 += 8) {                 // the operands of four steps in flight
            float fa[4][NA], fb[4][NB];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 2 * u + (lane >> 5);
#pragma unroll
                for (int i = 0; i < NA; ++i) fa[u][i] = k < k_end ? pa[i][AKC ? (long long)k : (long long)k * lda] : 0.f;
#pragma unroll
                for (int j = 0; j < NB; ++j) fb[u][j] = k < k_end ? pb[j][BKC ? (long long)k : (long long)k * ldb] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[u][j], fa[u][i], acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int mt = wm * (BM / 2) + i * 32 + (lane & 31), m = m0 + mt;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int nt = wn * (BN / 2) + 32 * j + 16 * h + 8 * (lane >> 5), n = n0 + nt;
                if (n >= N) continue;                                 // (N is a multiple of 8)
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = acc[i][j][8 * h + e];
                if (GRP && partial) Vec8<float>::store(partial + mt * BN + nt, v);
                else epilogue8<float, EPI>(m, n, N, v, C, p);
            }
    }
}

template <int EPI, bool AKC, bool BKC, int BM, int BN, bool GRP>
ds_status launch_split(dim3 grid, int M, int N, int K, const float* A, const float* B, float* C, int k_per_split, const GemmEpi& p,
                       const std::conditional_t<GRP, TnGroup, NoGroup>& grp, hipStream_t st) {
    constexpr int smem = 2 * 3 * 64 * (BM + BN);
    auto kern = gemm_f32_split_kernel<EPI, AKC, BKC, BM, BN, GRP>;
    static bool attr_set = false;
    if (!attr_set) {
        DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(256), smem, st, M, N, K, A, (long long)(AKC ? K : M), B, (long long)(BKC ? K : N), C, k_per_split, p, grp);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

// adds up the partial sums of a group's 64 x 128 tiles; kFinishParts work-groups per tile, tiles counted over the whole group
constexpr int kFinishParts = 4;
__global__ __launch_bounds__(256) void tn_group_f32_finish_kernel(TnGroup g) {
    int at = blockIdx.x / kFinishParts * g.splits;
    const int i = tn_group_problem(g, at);
    const int M = g.p[i].M, N = g.p[i].N, tiles_n = (N + G_BN - 1) / G_BN, tiles = (M + G_BM - 1) / G_BM * tiles_n, tile = at / g.splits;
    const int m0 = tile / tiles_n * G_BM, n0 = tile % tiles_n * G_BN;
    float* C = reinterpret_cast<float*>(g.p[i].C);
    GemmEpi p{};
    p.accumulate = g.accumulate;
    for (int e = blockIdx.x % kFinishParts * blockDim.x + threadIdx.x; e < G_BM * (G_BN / 8); e += kFinishParts * blockDim.x) {
        const int r = e / (G_BN / 8), c8 = (e % (G_BN / 8)) * 8;
        if (m0 + r >= M || n0 + c8 >= N) continue;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = 0.f;
#pragma unroll 4
        for (int sp = 0; sp < g.splits; ++sp) {
            float w[8];
            Vec8<float>::load(g.block(g.first[i] + sp * tiles + tile) + r * G_BN + c8, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] += w[j];
        }
        epilogue8<float, DS_EPI_ACC32>(m0 + r, n0 + c8, N, v, C, p);
    }
}

template <int EPI, bool AKC, bool BKC>
ds_status launch_form(int M, int N, int K, const float* A, const float* B, float* C, const GemmEpi& p, float* split_ws,
                      size_t split_ws_floats, hipStream_t st) {
    const int n_cu = gemm_cu_count();
    const int gn = (N + F_BN - 1) / F_BN, gm = (M + F_BM - 1) / F_BM;
    const long long lda = AKC ? K : M, ldb = BKC ? K : N, tiles = (long long)gn * gm;
    // Enough tiles for the CUs: the bf16 form, with 64 x 128 tiles where every CU gets two, the K loop is long enough to pay for
    // their longer prologue (12 288 rows of d = 512: stage call 5.27 -> 4.87 ms; K = 256: 1.31 -> 1.33) and they add at most an eighth
    // of columns that do not exist (N = 264, 11 535 rows, K = 1536: 136 us, 111 with 64 x 64 tiles, 125 in the fp32 form), else 64 x 64.  Long loops of
    // few tiles stay, cut over K (1800 x 512 x 2048, 232 tiles: 53 us, 58 with the other), and so do short ones, whose prologue and
    // splitting nothing covers (fp32 form -> this, geometric mean and worst of 30 to 40 shapes with tiles enough, operands from memory:
    // K = 32 1.16 and 1.45, 64 1.08 and 1.34, 96 1.03 and 1.22, 128 0.98 and 1.25, 160 0.95 and 1.10, 192 0.92 and 1.08, 224 0.91 and
    // 1.04, 256 0.82 and 0.98).
    if constexpr (AKC) {
        const bool fits = K >= 192 && lda <= (1 << 22) && ldb <= (BKC ? 1 << 22 : 1 << 24);       // byte offsets within a tile: 31 bits
        const int gn2 = (N + G_BN - 1) / G_BN;
        if (fits && (long long)gn2 * gm >= 2 * n_cu && K >= 512 && 2 * gn2 - gn <= gn / 8)
            return launch_split<EPI, AKC, BKC, G_BM, G_BN, false>(dim3(gn2, gm), M, N, K, A, B, C, K, p, NoGroup{}, st);
        if (fits && (tiles >= n_cu * 5 / 4 || (tiles >= n_cu * 7 / 8 && K <= 1024))) return launch_split<EPI, AKC, BKC, 64, 64, false>(dim3(gn, gm), M, N, K, A, B, C, K, p, NoGroup{}, st);
    }
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

// K loops per tile: as many as give the fewest K tiles, one after another, at two work-groups per CU (0.84 us per K tile of the
// two, 8 around a loop), 5 for the launch that adds up the partial sums and their round trip at 4 TB/s; at least 8 K tiles each.
// Always one launch: a stage call with it takes 0.57 to 0.96 of the time with one launch per gradient at all of 51 sizes (d = 128 ..
// 1024, 256 to 40 000 tokens), 0.85 in the mean.
TnPick pick_tn_group_f32(const TnGroup& g) {
    const int steps = (g.K + F_BK - 1) / F_BK, slots = 2 * gemm_cu_count();
    long long tiles = 0;
    for (int i = 0; i < g.n; ++i) tiles += (long long)((g.p[i].M + G_BM - 1) / G_BM) * ((g.p[i].N + G_BN - 1) / G_BN);
    TnPick best{kTnF32, 1};
    double best_cost = 0;
    for (int sp = 1; sp <= 64; ++sp) {
        const int len = (steps + sp - 1) / sp;
        if (sp > 1 && (len < 8 || tiles * sp > g.slab_end[TnGroup::kSlabs - 1])) break;
        if ((steps + len - 1) / len != sp) continue;
        const double rounds = (double)((tiles * sp + slots - 1) / slots);
        const double c = rounds * (len * 0.84 + 8) + (sp > 1 ? 5 + 2e-6 * sp * tiles * (G_BM * G_BN) : 0);
        if (sp == 1 || c < best_cost) {
            best.splits = sp;
            best_cost = c;
        }
    }
    return best;
}

ds_status launch_tn_group_f32(TnGroup& g, hipStream_t st) {
    const int steps = (g.K + F_BK - 1) / F_BK;
    long long blocks = 0;
    for (int i = 0; i < g.n; ++i) {
        g.first[i] = (int32_t)blocks;
        blocks += (long long)((g.p[i].M + G_BM - 1) / G_BM) * ((g.p[i].N + G_BN - 1) / G_BN) * g.splits;
        if (blocks > (1 << 23)) return DS_EOVERFLOW;        // work-items of a grid: 32 bits (2^36 outputs)
    }
    GemmEpi p{};
    p.accumulate = g.accumulate;
    const ds_status r = launch_split<DS_EPI_ACC32, false, false, G_BM, G_BN, true>(dim3((unsigned)blocks), 0, 0, g.K, nullptr, nullptr, nullptr,
                                                                               (steps + g.splits - 1) / g.splits * F_BK, p, g, st);
    if (r != DS_OK || g.splits == 1) return r;
    hipLaunchKernelGGL(tn_group_f32_finish_kernel, dim3((unsigned)(blocks / g.splits * kFinishParts)), dim3(256), 0, st, g);
    DS_LAUNCH_CHECK();
    return DS_OK;
}
