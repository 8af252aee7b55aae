// bf16 GEMMs with smaller macro tiles than the 256 x 256 kernel of gemm.hip, for launches that would not fill the chip with
// those: the micro-batches of a stage that runs them one after another, the decoder side of an encoder-decoder stage, small
// models.  There the large tile has to cut K loops into many pieces to occupy the compute units, and writing and reading
// back 256 KB of partial sums per piece costs more than the products (M = 756, N = K = 2048: 36 us, of which the
// products are 6).
//
// Three tiles, all direct-to-LDS with the operand layouts of the large kernel, 64-deep K tiles in a ring of stages:
//   0: 128 x 128, 8 wavefronts, 4 stages (128 KB: one work-group per CU).  8 of 64 x 32 or, for long loops, four of 64 x 64 twice, each
//      four taking one of the two 32-deep steps of every K tile (KS = 2); the halves of the contraction meet in LDS at the end
//   3: 128 x 128, 8 wavefronts of 64 x 32, 2 stages (64 KB: two per CU)
//   1: 128 x  64, 8 wavefronts of 32 x 32, 3 stages ( 72 KB: two per CU)
//   2:  64 x  64, 4 wavefronts of 32 x 32, 3 stages ( 48 KB: three per CU)
// What bounds them is what one work-group can do between two barriers: more stages change nothing (3, 4 and 5 within 2 %),
// a second work-group on the CU does.  With one tile per CU the deep ring is the better one (M = 1757, N = K = 2048: 19.8 us,
// two stages 22.1), with more the shallow one (M = 756, N = 6144, K = 2048: 27.9 against 39.7).  Time per K tile of a CU:
// 0.49 us for kind 0, 0.32 and 0.20 for 1 and 2, for kind 3 0.39 while the chip is not full and 0.55 - 0.62 per tile when every CU
// works on two.  Four wavefronts of 64 x 64 alone on the 128 x 128 tile are slower at every shape tried (N = 2048, K = 8192,
// M = 1757: 89 us and, with 32-deep tiles and two work-groups per CU, 73, against 60); eight of them, two to a SIMD, with half the
// K steps each read a third less from LDS than eight of 64 x 32 and have one burst of 16 MFMAs per barrier: 4096 x 1024 TN over
// 4173 tokens, operands warm, 50.4 -> 44.4 us, from memory as before (53.3): there the transfers are the limit (timing build without
// the products 52).  At 128 x 64 the same changes nothing.
//
// Which one: the tile and split count with the smallest estimate (pick_gemm_tile), compared with the same kind of
// estimate for the large kernel.  Measured, 256 x 256 kernel (as it was with eight wavefronts) -> this, us (M, N, K; ds_gemm_ws on
// an idle card):
//   NT 256, 768, 256: 10.2 -> 4.8    756, 2048, 2048: 36 -> 13      756, 8192, 2048: 43 -> 29    756, 2048, 8192: 50 -> 40
//      1757, 2048, 2048: 37 -> 20    1757, 6144, 2048: 43 (50 with these: stays)    756, 6144, 2048: 42 -> 28
//   TN 256, 1024, 250: 17 -> 5       2048, 2048, 756: 47 -> 18       2048, 2048, 1757: 43 -> 26  1024, 4096, 4173: 58 -> 47
//      2048, 6144, 756: 34 (stays)   2048, 6144, 1757: 53 (56: stays)
// with the operands warm in the caches (each from memory: 2 to 12 us more in the NT form, 1 to 2 in the TN form).
#include "gemm_epilogue.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

constexpr int T_KD = 64;                             // depth of a K tile

// One operand's K tile: ROWS rows (m or n) x 64 k in LDS.
//   k contiguous (KC): [row][128 bytes], 16-byte chunk c of a row at chunk slot c ^ ((row / 2) % 8); rows past the end of the
//     tensor are clamped (read, never stored).
//   k as the row: [64 k][ROWS * 2 bytes], 32-byte unit u of a k row at unit u ^ f(k) with f(k) = k % 8 (ROWS = 128) or
//     (k / 2) % 4 (ROWS = 64); k rows past the end read zeros through the bounds check of the buffer descriptor.
// Both swizzles are applied by choosing which global chunk a lane fetches.
template <int ROWS, bool KC, int NW> struct OperandTile {
    static constexpr int BYTES = ROWS * T_KD * 2;
    static constexpr int LP = BYTES / 1024 / NW;                      // transfers per wavefront and tile
    const char* base;                                                 // KC: tensor at (r0, k = 0); else at (k = 0, r0)
    long long ld2;                                                    // row stride in bytes
    int K;
    uint32_t off[LP];
    uint32_t lds_wave;                                                // this wavefront's part of a tile
    __device__ __forceinline__ void setup(const bf16_t* src, long long ld, int r0, int rows, int K_, int wave, int lane) {
        ld2 = ld * 2;
        K = K_;
        lds_wave = (uint32_t)__builtin_amdgcn_readfirstlane(wave) * (LP * 1024);
        base = reinterpret_cast<const char*>(src) + (KC ? (long long)r0 * ld2 : (long long)r0 * 2);
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            const int u = (wave * LP + i) * 64 + lane;                // 16-byte slot of the tile
            uint32_t want;
            if constexpr (KC) {
                const int row = u / (T_KD / 8), chunk = (u % (T_KD / 8)) ^ chunk_swz(row);
                const int rc = r0 + row < rows ? row : rows - 1 - r0;
                want = (uint32_t)(rc * ld2 + chunk * 16);
            } else {
                constexpr int CPR = ROWS / 8;                         // chunks per k row
                const int k = u / CPR, pos = u % CPR;
                const int unit = (pos >> 1) ^ unit_swz(k);
                want = (uint32_t)(k * ld2 + (unit * 2 + (pos & 1)) * 16);
            }
            off[i] = dma_lane_offset<LP>(want, i);
        }
    }
    __device__ __forceinline__ static int chunk_swz(int row) { return (row >> 1) & 7; }
    __device__ __forceinline__ static int unit_swz(int k) { return ROWS == 128 ? (k & 7) : ((k >> 1) & 3); }
    __device__ __forceinline__ void issue(int tile, uint32_t lds) const {
        if constexpr (KC) {
            lds_dma16_group<LP>(dma_group_base<LP>(base + (long long)tile * (T_KD * 2)), off, lds + lds_wave);
        } else {
            const int left = K - tile * T_KD;
            const uint32_t bytes = (uint32_t)((left < T_KD ? left : T_KD) - 1) * (uint32_t)ld2 + ROWS * 2;     // to the end of this tile's columns
            const i32x4_t buf = make_raw_buffer(base + (long long)tile * T_KD * ld2 - 1024 * (LP - 1), bytes + 1024u * (LP - 1));
            lds_dma16_buffer_group<LP>(buf, off, lds + lds_wave);
        }
    }
    // MFMA fragment (16 rows x 32 k) of 16-row unit `unit`, k step ks of a tile; both operands list k in the same order
    __device__ static __forceinline__ bf16x8_t frag(const char* tile, int unit, int ks, int lane) {
        if constexpr (KC) {
            const int row = unit * 16 + (lane & 15), chunk = ks * 4 + (lane >> 4);
            return *reinterpret_cast<const bf16x8_t*>(tile + row * (T_KD * 2) + ((chunk ^ chunk_swz(row)) << 4));
        } else {
            typedef short s16x4_t __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) s16x4_t* lds4_t;
            const int k = ks * 32 + 4 * (lane >> 4) + ((lane & 15) >> 2);
            const char* q = tile + k * (ROWS * 2) + ((unit ^ unit_swz(k)) << 5) + (lane & 3) * 8;
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)q);
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(q + 16 * ROWS * 2));
            return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    }
};

// C[M,N] = A B^T (NT: both k-contiguous, K % 64 == 0, N % BN == 0) or A^T B (TN: k rows, M % BM == 0, N % BN == 0, K any).
// WM x WN wavefronts; gridDim.x = tiles x splits, numbered so that each XCD gets a contiguous run, 8 tile rows to a group;
// with more than one split the partial sums go to split_ws as [split][M][N].
// Ring of NS stages, 64-deep K tiles: a tile's transfers are issued NS - 1 tiles ahead, right after the barrier that
// frees their stage; the fragments of the next 32-deep step are read while the current one is multiplied, across the
// tile boundary too.  Transfers past the last tile are clamped so that the wait counts never change.
// KS = 2: WM x WN wavefronts twice, each half takes one of the two 32-deep steps of every K tile.
// GRP (TN form): the work-groups of several weight gradients over the same K rows (grp), problem after problem.
template <int EPI, bool TNF, int BM, int BN, int WM, int WN, int NS, int KS, bool GRP = false>
__global__ __launch_bounds__(WM * WN * KS * 64) void gemm_bf16_tile_kernel(int M, int N, int K, const bf16_t* __restrict__ A,
                                                                      const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
                                                                      int tiles_m, int tiles_n, int splits, int tiles_per_split,
                                                                      float* __restrict__ split_ws, GemmEpi p,
                                                                      std::conditional_t<GRP, TnGroup, NoGroup> grp) {
    static_assert(!GRP || (TNF && EPI == DS_EPI_ACC32), "groups are of weight gradients");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int NW = WM * WN * KS;
    typedef OperandTile<BM, !TNF, NW> TA;
    typedef OperandTile<BN, !TNF, NW> TB;
    constexpr int STAGE = TA::BYTES + TB::BYTES;
    constexpr int WR = BM / WM, WC = BN / WN;                         // a wavefront's rows and columns
    constexpr int NA = WR / 16, NB = WC / 16;
    constexpr int L = TA::LP + TB::LP;
    static_assert(WR % 32 == 0 && WC % 32 == 0, "the epilogue stages 32 rows of at least 32 columns");
    static_assert((NS - 1) * L < 64, "vmcnt has 6 bits");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave / WN % WM, wn = wave % WN, kq = wave / (WM * WN);         // KS = 2: kq = the 32-deep step of a tile it takes

    int tile_m, tile_n, split;
    {
        int logical = xcd_contiguous(blockIdx.x, gridDim.x);
        if constexpr (GRP) {
            const int i = tn_group_problem(grp, logical);
            M = grp.p[i].M;
            N = grp.p[i].N;
            A = reinterpret_cast<const bf16_t*>(grp.p[i].A);
            B = reinterpret_cast<const bf16_t*>(grp.p[i].B);
            C = reinterpret_cast<bf16_t*>(grp.p[i].C);
            tiles_m = M / BM;
            tiles_n = N / BN;
        }
        const int n_tiles = tiles_m * tiles_n;
        split = logical / n_tiles;
        logical -= split * n_tiles;
        constexpr int GROUP = 8;
        const int group = logical / (GROUP * tiles_n), first = group * GROUP;
        const int gs = tiles_m - first < GROUP ? tiles_m - first : GROUP;
        const int in = logical - group * GROUP * tiles_n;
        tile_m = first + in % gs;
        tile_n = in / gs;
    }
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int nt = (K + T_KD - 1) / T_KD;
    const int t_begin = split * tiles_per_split;
    const int t_end = t_begin + tiles_per_split < nt ? t_begin + tiles_per_split : nt;

    TA ta;
    TB tb;
    ta.setup(A, TNF ? M : K, m0, M, K, wave, lane);
    tb.setup(B, TNF ? N : K, n0, N, K, wave, lane);
    const uint32_t lds0 = lds_address(smem);
    auto issue = [&](int tl) {
        const uint32_t dst = lds0 + (uint32_t)((tl - t_begin) % NS) * STAGE;
        const int tc = tl < t_end ? tl : t_end - 1;
        ta.issue(tc, dst);
        tb.issue(tc, dst + TA::BYTES);
    };
    f32x4_t acc[NA][NB];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

    bf16x8_t ax[NA], bx[NB], ay[NA], by[NB];
    auto read = [&](int stage, int ks, bf16x8_t (&fa)[NA], bf16x8_t (&fb)[NB]) {
        const char* a = smem + stage * STAGE;
#pragma unroll
        for (int j = 0; j < NB; ++j) fb[j] = TB::frag(a + TA::BYTES, wn * NB + j, ks, lane);
#pragma unroll
        for (int i = 0; i < NA; ++i) fa[i] = TA::frag(a, wm * NA + i, ks, lane);
    };
    auto mma = [&](const bf16x8_t (&fa)[NA], const bf16x8_t (&fb)[NB]) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int jj = 0; jj < NB; ++jj) {
                const int j = (i & 1) ? NB - 1 - jj : jj;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
            }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) issue(t_begin + s);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 1) * L));              // the first tile: this wavefront's part ...
    __builtin_amdgcn_s_barrier();                                     // ... and everyone's
    read(0, KS == 1 ? 0 : kq, ax, bx);
    if constexpr (KS == 1) {
        int stage = 0;
        for (int tl = t_begin; tl < t_end; ++tl) {
            const int next = stage + 1 == NS ? 0 : stage + 1;
            read(stage, 1, ay, by);
            __builtin_amdgcn_sched_barrier(0);
            mma(ax, bx);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * L) & 0xF0FF); // tile tl + 1 has landed; lgkmcnt(0): reads of tile tl are done
            __builtin_amdgcn_s_barrier();
            issue(tl + NS);                                               // into the stage of tile tl
            read(next, 0, ax, bx);                                        // (past the last tile: a reloaded copy of it, unused)
            __builtin_amdgcn_sched_barrier(0);
            mma(ay, by);
            __builtin_amdgcn_sched_barrier(0);
            stage = next;
        }
    } else {
        int stage = 0;
        auto tile = [&](int tl, bf16x8_t (&fa)[NA], bf16x8_t (&fb)[NB], bf16x8_t (&ga)[NA], bf16x8_t (&gb)[NB]) {
            const int next = stage + 1 == NS ? 0 : stage + 1;
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS - 2) * L) & 0xF0FF); // tile tl + 1 has landed; lgkmcnt(0): reads of tile tl are done
            __builtin_amdgcn_s_barrier();
            issue(tl + NS);                                               // into the stage of tile tl
            read(next, kq, ga, gb);                                       // (past the last tile: a reloaded copy of it, unused)
            __builtin_amdgcn_sched_barrier(0);
            mma(fa, fb);
            __builtin_amdgcn_sched_barrier(0);
            stage = next;
        };
        int tl = t_begin;
        for (; tl + 1 < t_end; tl += 2) {
            tile(tl, ax, bx, ay, by);
            tile(tl + 1, ay, by, ax, bx);
        }
        if (tl < t_end) tile(tl, ax, bx, ay, by);
    }
    __builtin_amdgcn_s_waitcnt(0x0070);                               // no transfer may still be writing the LDS the epilogue uses
    __builtin_amdgcn_s_barrier();
    if constexpr (KS == 2) {
        // the two halves of the contraction meet: a wavefront hands the blocks of half its rows to its partner and finishes the others
        static_assert(NA % 4 == 0, "whole 32-row passes per half");
        f32x4_t* x = reinterpret_cast<f32x4_t*>(smem) + (wave * (NA / 2) * NB) * 64 + lane;
#pragma unroll
        for (int i = 0; i < NA / 2; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) x[(i * NB + j) * 64] = kq ? acc[i][j] : acc[NA / 2 + i][j];
        __syncthreads();
        const f32x4_t* y = reinterpret_cast<const f32x4_t*>(smem) + ((wave ^ (WM * WN)) * (NA / 2) * NB) * 64 + lane;
#pragma unroll
        for (int i = 0; i < NA / 2; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = (kq ? acc[NA / 2 + i][j] : acc[i][j]) + y[(i * NB + j) * 64];
        __syncthreads();
    }
    constexpr int WE = WR / KS;                                       // rows this wavefront finishes, from row m1 on
    const int m1 = m0 + wm * WR + (KS == 2 ? kq * WE : 0);

    // epilogue: 32 rows at a time through a block of LDS that is private to the wavefront
    constexpr int LDC = WC + 4, LPR = WC / 8, RPP = 64 / LPR, NP = 32 / RPP;
    float* stg = reinterpret_cast<float*>(smem) + wave * (32 * LDC);
    const int rd_row = lane / LPR, rd_col = (lane % LPR) * 8;
    const int n = n0 + wn * WC + rd_col;
    const bool direct = splits == 1;
    EpiPre<bf16_t> pre[WE / 32][NP];
    if (epilogue_reads<EPI>() && direct) {
#pragma unroll
        for (int i = 0; i < WE / 32; ++i)
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const int m = m1 + i * 32 + q * RPP + rd_row;
                if (m < M) epilogue_prefetch<bf16_t, EPI>(m, n, N, p, pre[i][q]);
            }
    }
    float csum[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) csum[j] = 0.f;
#pragma unroll
    for (int i = 0; i < WE / 32; ++i) {
        wave_lds_sync();
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const f32x4_t a4 = acc[2 * i + i2][j];
                *reinterpret_cast<float4*>(stg + (i2 * 16 + (lane & 15)) * LDC + j * 16 + 4 * (lane >> 4)) = make_float4(a4[0], a4[1], a4[2], a4[3]);
            }
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int row = q * RPP + rd_row, m = m1 + i * 32 + row;
            if (m >= M) continue;
            float v[8];
            Vec8<float>::load(stg + row * LDC + rd_col, v);
            if (!direct) {
                Vec8<float>::store(split_ws + ((size_t)split * M + m) * N + n, v);
            } else {
                epilogue8<bf16_t, EPI>(m, n, N, v, C, p, epilogue_reads<EPI>() ? &pre[i][q] : nullptr);
                if constexpr (EPI == DS_EPI_DGELU || EPI == DS_EPI_MULR) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) csum[j] += v[j];
                }
            }
        }
    }
    if constexpr ((EPI == DS_EPI_DGELU || EPI == DS_EPI_MULR) && BM == 128) {
        // one row of partial column sums per tile row: the wavefronts of a column add theirs in LDS
        if (p.colsum) {
#pragma unroll
            for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
                for (int j = 0; j < 8; ++j) csum[j] += __shfl_xor(csum[j], o, 64);
            __syncthreads();
            float* red = reinterpret_cast<float*>(smem);              // [WM KS][BN]
            if (lane < LPR) Vec8<float>::store(red + (wm * KS + kq) * BN + wn * WC + rd_col, csum);
            __syncthreads();
            if (t < BN) {
                float s = red[t];
#pragma unroll
                for (int w = 1; w < WM * KS; ++w) s += red[w * BN + t];
                p.colsum[(size_t)tile_m * N + n0 + t] = s;
                // gemm_colsum_rows() counts two rows per 256: the last one may have no tile
                if (tile_m + 1 == tiles_m && (tiles_m & 1)) p.colsum[(size_t)(tile_m + 1) * N + n0 + t] = 0.f;
            }
        }
    }
}

struct TileShape { int bm, bn, waves, stages; double step, fixed; };
// step: microseconds per K tile of a CU that has one tile; fixed: around the K loop
constexpr int kKinds = 4;
constexpr TileShape kShapes[kKinds] = {{128, 128, 8, 4, 0.49, 3.0}, {128, 64, 8, 3, 0.32, 2.5}, {64, 64, 4, 3, 0.20, 2.5}, {128, 128, 8, 2, 0.39, 3.0}};
constexpr double kBusyStep3 = 0.62;                  // kind 3, per tile, when every CU works on two (0.55 on operands that are warm in L2)
constexpr double kBusyStep0 = 0.64;                  // kind 0, per tile, several of them one after the other
constexpr double kLoneStep1 = 0.36, kLoneStep2 = 0.24;                // TN form, one tile per CU: nothing covers its waits
constexpr double kColdStep0Nt = 0.51, kColdStep0Tn = 0.55;           // kind 0, operands from memory

// Kind 0 with two groups of wavefronts (KS = 2) where every work-group has at least 32 K tiles.  Meeting in LDS at the end costs about a
// microsecond, which shorter loops do not earn: two groups / one, geometric means of 10 to 21 NT shapes that go to this tile, operands
// from memory and warm, K = 256 1.10 and 1.04, 512 1.05 and 0.99, 768 1.05 and 1.01, 1024 1.04 and 1.00, 1536 1.03 and 0.97, 2048
// 1.02 and 0.95, 3072 1.02 and 0.93, 4096 1.01 and 0.92, 8192 1.01 and 0.92.
bool two_step_groups(int K, int splits) { return ((K + T_KD - 1) / T_KD + splits - 1) / splits >= 32; }

template <int EPI, bool TNF, int KIND, int WM, int WN, int KS = 1>
ds_status launch_kind(int splits, int M, int N, int K, const void* A, const void* B, void* C, const GemmEpi& p, float* split_ws,
                      hipStream_t st) {
    constexpr TileShape s = kShapes[KIND];
    constexpr int ring = s.stages * (s.bm + s.bn) * T_KD * 2, staging = s.waves * 32 * (s.bn / WN + 4) * 4;
    constexpr int smem = ring > staging ? ring : staging;
    static_assert(WM * WN * KS == s.waves, "wavefront grid");
    static bool attr_set = false;
    auto kern = gemm_bf16_tile_kernel<EPI, TNF, s.bm, s.bn, WM, WN, s.stages, KS>;
    if (!attr_set) {
        DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
        attr_set = true;
    }
    const int tiles_m = (M + s.bm - 1) / s.bm, tiles_n = N / s.bn;
    const int nt = (K + T_KD - 1) / T_KD, per = (nt + splits - 1) / splits;      // (the pick leaves no split empty)
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n * splits)), dim3(s.waves * 64), smem, st, M, N, K, (const bf16_t*)A,
                       (const bf16_t*)B, (bf16_t*)C, tiles_m, tiles_n, splits, per, split_ws, p, NoGroup{});
    DS_LAUNCH_CHECK();
    if (splits > 1) return launch_splitk_finish<bf16_t, EPI>(M, N, splits, split_ws, C, p, st);
    return DS_OK;
}

template <int KIND, int WM, int WN, int KS = 1>
ds_status launch_group_kind(const TnGroup& g, int blocks, hipStream_t st) {
    constexpr TileShape s = kShapes[KIND];
    constexpr int ring = s.stages * (s.bm + s.bn) * T_KD * 2, staging = s.waves * 32 * (s.bn / WN + 4) * 4;
    constexpr int smem = ring > staging ? ring : staging;
    static bool attr_set = false;
    auto kern = gemm_bf16_tile_kernel<DS_EPI_ACC32, true, s.bm, s.bn, WM, WN, s.stages, KS, true>;
    if (!attr_set) {
        DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
        attr_set = true;
    }
    GemmEpi p{};
    p.accumulate = g.accumulate;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(s.waves * 64), smem, st, 0, 0, g.K, (const bf16_t*)nullptr,
                       (const bf16_t*)nullptr, (bf16_t*)nullptr, 0, 0, 1, (g.K + T_KD - 1) / T_KD, (float*)nullptr, p, g);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

template <int EPI, bool TNF>
ds_status launch_form(const TilePick& k, int M, int N, int K, const void* A, const void* B, void* C, const GemmEpi& p, float* split_ws,
                      hipStream_t st) {
    if (k.kind == 0 && two_step_groups(K, k.splits)) return launch_kind<EPI, TNF, 0, 2, 2, 2>(k.splits, M, N, K, A, B, C, p, split_ws, st);
    if (k.kind == 0) return launch_kind<EPI, TNF, 0, 2, 4>(k.splits, M, N, K, A, B, C, p, split_ws, st);
    if (k.kind == 3) return launch_kind<EPI, TNF, 3, 2, 4>(k.splits, M, N, K, A, B, C, p, split_ws, st);
    if (k.kind == 1) return launch_kind<EPI, TNF, 1, 4, 2>(k.splits, M, N, K, A, B, C, p, split_ws, st);
    return launch_kind<EPI, TNF, 2, 2, 2>(k.splits, M, N, K, A, B, C, p, split_ws, st);
}

}  // namespace

int gemm_cu_count() {
    static const int n_cu = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
        return v;
    }();
    return n_cu;
}

// The caller has established what the operands of the 256 x 256 kernel need (N, and M in the TN form, a multiple of 256;
// K a multiple of 64 in the NT form; 16-byte alignment), which covers every tile here.
//   estimate = rounds over the CUs x K tiles per split x step + fixed + what of out_us is not hidden; several splits add the
//   round trip of the partial sums at 4 TB/s and 5 us for the launch that adds them.
// out_us: moving an fp32 output (see gemm_output_us); half of it is hidden where a CU has other tiles to work on meanwhile.
// colsum: the epilogue's column sums are wanted, which takes 128-row tiles and whole K loops.
// versus_large differs in two places that matter only against the other kernel, whose constants hold for operands from memory:
// kind 0 counts its step from memory, and of the output only the reading (out_read: half of out_us) is hidden, by half;
// writing goes at the rate of the memory either way (2048 x 8192 over 126 tokens: 30.9 us on 128 x 64 tiles, 24.5 on
// 256 x 256 ones).  Against that kernel with eight wavefronts, of 1 500 random shapes of stages with d = 256 .. 2048 (96 to 16 000 rows, operands from memory) 12 take
// over 3 % longer than on the large kernel, at most 12 %; with the rates of warm operands throughout it was 40 of 1 100, up to
// 21 %.  (Against the one with four: big_cost.)
TilePick pick_gemm_tile(bool tn, int32_t M, int32_t N, int32_t K, size_t split_ws_floats, bool colsum, double out_us, bool out_read) {
    TilePick best{-1, 1, 0.0, 0.0};
    if (tn && (M > (1 << 25) || N > (1 << 25))) return best;          // a K tile is addressed through a 32-bit buffer length
    const int n_cu = gemm_cu_count(), nt = (K + T_KD - 1) / T_KD;
    for (int k = 0; k < kKinds; ++k) {
        const TileShape& s = kShapes[k];
        if (colsum && s.bm != 128) continue;
        const double tiles = std::ceil((double)M / s.bm) * (N / s.bn);
        for (int sp = 1; sp <= 32; ++sp) {
            if (sp > 1 && (colsum || sp > nt / 4 || (size_t)sp * M * N > split_ws_floats)) break;
            const int per = (nt + sp - 1) / sp;
            if ((nt + per - 1) / per != sp || tiles * sp > 1e9) continue;         // every split owns at least one K tile
            const double rounds = std::ceil(tiles * sp / n_cu);
            if (k == 3 && rounds < 2) continue;                       // kind 0 is the better one
            double loop = rounds * per * s.step;
            if (k == 0 && rounds > 1) loop = rounds * per * kBusyStep0;
            if (tn && rounds == 1 && (k == 1 || k == 2)) loop = per * (k == 1 ? kLoneStep1 : kLoneStep2);
            if (k == 3) loop = std::max(loop, tiles * sp / n_cu * per * kBusyStep3);
            const double around = s.fixed + (sp > 1 ? 2e-6 * sp * (double)M * N + 5 : 0.0);
            const bool hides = k != 0 && rounds > 2;
            const double cost = loop + around + (hides ? 0.5 * out_us : out_us);
            if (best.kind < 0 || cost < best.cost)
                best = TilePick{k, sp, cost, (k == 0 ? rounds * per * (tn ? kColdStep0Tn : kColdStep0Nt) : loop) + around + (hides && out_read ? 0.75 * out_us : out_us)};
        }
    }
    return best;
}

ds_status launch_gemm_tile(const TilePick& pick, bool tn, int32_t M, int32_t N, int32_t K, const void* A, const void* B, void* C,
                           int32_t epilogue, const GemmEpi& p, float* split_ws, hipStream_t st) {
    if (tn) return epilogue == DS_EPI_ACC32 ? launch_form<DS_EPI_ACC32, true>(pick, M, N, K, A, B, C, p, split_ws, st) : DS_EINVAL;
    switch (epilogue) {
    case DS_EPI_NONE: return launch_form<DS_EPI_NONE, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_GELU: return launch_form<DS_EPI_GELU, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_RESID: return launch_form<DS_EPI_RESID, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_DGELU: return launch_form<DS_EPI_DGELU, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_ACC32: return launch_form<DS_EPI_ACC32, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_GATE: return launch_form<DS_EPI_GATE, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_DGATE: return launch_form<DS_EPI_DGATE, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_GELU_D: return launch_form<DS_EPI_GELU_D, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    case DS_EPI_MULR: return launch_form<DS_EPI_MULR, false>(pick, M, N, K, A, B, C, p, split_ws, st);
    }
    return DS_EINVAL;
}

// Weight gradients over `per` 64-deep K tiles with mn output elements in one launch: the kind and split count with the
// smallest estimate, in microseconds:
//   6 + rounds over the CUs x K tiles x step + the fp32 output at 4 TB/s (+ 5 and the round trip of the partial sums)
// with the step a CU takes for a K tile, operands from memory, when it has one tile / several:
//   128 x 128 0.85 / 0.85, 128 x 64 0.60 / 0.50, 64 x 64 0.45 / 0.36, 128 x 128 two per CU 0.85 / 0.75, 256 x 256 1.60.
// Splits only with 256 x 256 tiles (smaller ones have enough work-groups), as far as the blocks for partial sums go.
// (256 x 256: of the kernel with eight wavefronts.  That with four takes 1.43 to 1.46 on long contractions; with 1.40 here 18 stages took the same time within
// 0.4 %, with 1.20 three of d = 768 3 to 4 % longer.)
// Estimate / measured (d, d_ff, tokens; the four gradients of a layer; the first two and the fourth on 256 x 256 tiles of eight
// wavefronts): 2048, 8192, 16384: 1335 / 1334; 1024, 4096, 16384 (4
// splits) 443 / 408; 768, 3072, 1500 (128 x 128, two per CU) 43 / 51; 512, 2048, 9000 (5 splits) 95 / 97; 256, 1024, 228 (64 x 64)
// 9 / 10.
static double tn_cost(double mn, int per, double out_us, int blocks, TnPick& best) {
    struct Rate { double lone, busy; };
    constexpr Rate rate[kKinds + 1] = {{0.85, 0.85}, {0.60, 0.50}, {0.45, 0.36}, {0.85, 0.75}, {1.60, 1.60}};
    best = TnPick{-1, 1};
    double best_cost = 0;
    for (int k = 0; k <= kTnBig; ++k) {
        const double tiles = mn / (k == kTnBig ? 65536.0 : (double)kShapes[k].bm * kShapes[k].bn);
        for (int sp = 1; sp <= (k == kTnBig ? 16 : 1); ++sp) {
            const int len = (per + sp - 1) / sp;
            if (sp > 1 && (len < 4 || tiles * sp > blocks)) break;
            if ((per + len - 1) / len != sp) continue;                            // every split owns at least one K tile
            const double load = tiles * sp / gemm_cu_count();
            const double rounds = k == 3 ? std::max(load, 1.0) : std::ceil(load);     // (kind 3: two work-groups per CU even it out)
            const double c = 6 + rounds * len * (load <= 1 ? rate[k].lone : rate[k].busy) + out_us + (sp > 1 ? 5 + 2e-6 * sp * mn : 0);
            if (best.kind < 0 || c < best_cost) {
                best = TnPick{k, sp};
                best_cost = c;
            }
        }
    }
    return best_cost;
}

// One launch for the group, unless the launches of the problems one by one are estimated within 5 % of it: over very long
// contractions of many tiles (d = 4096 and 32 768 tokens: 9471 us one by one, 9903 together) the work-groups of a launch drift
// apart along K and share less in L2, and launch boundaries bring them together again.
TnPick pick_tn_group(const TnGroup& g) {
    if (g.f32) return pick_tn_group_f32(g);
    const int per = (g.K + T_KD - 1) / T_KD;
    double mn = 0, separate = 0;
    TnPick pick;
    for (int i = 0; i < g.n; ++i) {
        const double q = (double)g.p[i].M * g.p[i].N;
        mn += q;
        separate += tn_cost(q, per, (g.accumulate ? 2e-6 : 1e-6) * q, g.slab_end[0], pick);
    }
    const double together = tn_cost(mn, per, (g.accumulate ? 2e-6 : 1e-6) * mn, g.slab_end[TnGroup::kSlabs - 1], pick);
    return together < 0.95 * separate ? pick : TnPick{-1, 1};
}

ds_status launch_tn_group(const TnPick& pick, TnGroup& g, hipStream_t st) {
    if (pick.kind < 0 || pick.kind > kTnF32) return DS_EINVAL;
    g.splits = pick.kind >= kTnBig ? pick.splits : 1;
    if (pick.kind == kTnF32) return launch_tn_group_f32(g, st);
    const int bm = pick.kind == kTnBig ? 256 : kShapes[pick.kind].bm, bn = pick.kind == kTnBig ? 256 : kShapes[pick.kind].bn;
    long long blocks = 0;
    for (int i = 0; i < g.n; ++i) {
        g.first[i] = (int32_t)blocks;
        blocks += (long long)(g.p[i].M / bm) * (g.p[i].N / bn) * g.splits;
        if (blocks > (1 << 22)) return DS_EOVERFLOW;        // work-items of a grid: 32 bits (2^34 outputs of the smallest tile)
    }
    switch (pick.kind) {
    case 0:
        if (two_step_groups(g.K, 1)) return launch_group_kind<0, 2, 2, 2>(g, (int)blocks, st);
        return launch_group_kind<0, 2, 4>(g, (int)blocks, st);
    case 1: return launch_group_kind<1, 4, 2>(g, (int)blocks, st);
    case 2: return launch_group_kind<2, 2, 2>(g, (int)blocks, st);
    case 3: return launch_group_kind<3, 2, 4>(g, (int)blocks, st);
    case kTnBig: return launch_tn_group_big(g, (int)blocks, st);
    }
    return DS_EINVAL;
}
