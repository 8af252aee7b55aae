// GEMMs of the stage: projections forward (NN), input gradients (NT) and weight gradients (TN,
// the contraction running over every token of every micro-batch, which is the gradient
// accumulation across micro-batches).
//
// Two kernels:
//   * gemm_bf16_nt_kernel — the one the stage runs on: bf16 in, fp32 accumulate on the CDNA4 matrix cores
//     (v_mfma_f32_16x16x32_bf16), operands straight from global memory into LDS, NT form (forward with [N][K]
//     weight copies, input gradients) and TN form (weight gradients); described where it is defined.
//   * gemm_generic_kernel — any dtype / shape / stride, plain FMA: the fallback for the bf16 operand forms and shapes the
//     matrix-core kernel does not take (NN; TN with an epilogue other than fp32 accumulation; N not a multiple of 256)
//     and for fp32 operands that the fp32 matrix-core kernel (gemm_f32.hip) cannot read 16 bytes at a time.
// Epilogues go back through LDS so that global stores (and the residual / activation reads) are 16 bytes per lane
// and row-contiguous.  Work-group ids are remapped so that each XCD (own L2) gets a contiguous run of tiles.
#include "gemm_epilogue.hpp"

#include <atomic>
#include <cmath>
#include <mutex>
#include <type_traits>

namespace {

// ---------------------------------------------------------------------------- generic kernel
// 64x64 tile, 256 threads, 4x4 outputs per thread, K step 16.  A(m,k) = A[m*sam + k*sak].
// Requires N % 8 == 0 (8-wide epilogue); M, K arbitrary.
template <class T, int EPI>
__global__ __launch_bounds__(256) void gemm_generic_kernel(int M, int N, int K, const T* __restrict__ A, long long sam,
                                                           long long sak, const T* __restrict__ B, long long sbk,
                                                           long long sbn, T* __restrict__ C, GemmEpi p) {
    __shared__ float As[16][68];
    __shared__ float Bs[16][68];
    const int t = threadIdx.x;
    const int tx = t & 7, ty = t >> 3;            // tx: 8 column groups of 8, ty: 32 row pairs
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    float acc[2][8];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
    for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int idx = t + 256 * i;
            {
                const int mm = sak == 1 ? idx >> 4 : idx & 63;
                const int kk = sak == 1 ? idx & 15 : idx >> 6;
                const int m = m0 + mm, k = k0 + kk;
                As[kk][mm] = (m < M && k < K) ? to_f32(A[m * sam + k * sak]) : 0.f;
            }
            {
                const int nn = sbk == 1 ? idx >> 4 : idx & 63;
                const int kk = sbk == 1 ? idx & 15 : idx >> 6;
                const int n = n0 + nn, k = k0 + kk;
                Bs[kk][nn] = (n < N && k < K) ? to_f32(B[k * sbk + n * sbn]) : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const float a0 = As[kk][ty * 2], a1 = As[kk][ty * 2 + 1];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float b = Bs[kk][tx * 8 + j];
                acc[0][j] += a0 * b;
                acc[1][j] += a1 * b;
            }
        }
        __syncthreads();
    }
    const int n = n0 + tx * 8;
    if (n < N) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int m = m0 + ty * 2 + i;
            if (m < M) epilogue8<T, EPI>(m, n, N, acc[i], C, p);
        }
    }
}

// macro tile of the matrix-core kernel
constexpr int BM = 256, BN = 256, BK = 64;

// ---------------------------------------------------------------------------- NT / TN kernel, direct to LDS
// NT form: C[M,N] = A[M,K] * B[N,K]^T, both operands k-contiguous (K % 64 == 0, N % 256 == 0).
// TN form: C[M,N] = A[K,M]^T * B[K,N], both operands with the contraction index as the row (weight gradients).
//
// 256x256 macro tile, 4 wavefronts (one per SIMD) in a 2x2 arrangement, each owning a 128x128 accumulator block: 8 x 8
// blocks of v_mfma_f32_16x16x32_bf16, 256 accumulator registers of the 512 a lone wavefront has.  Operands go global ->
// LDS directly (no staging registers, no LDS write instructions): a wavefront instruction deposits 64 x 16 bytes at
// consecutive LDS addresses, and the XOR swizzle that makes the fragment reads conflict-free is obtained by choosing
// WHICH global chunk each lane fetches.  K tiles are 64 deep; an operand's part of one is a unit of 32 KB.
//
// LDS holds a ring of five units (160 KB): while tile t is multiplied (units A(t), B(t)), A(t+1), B(t+1) and A(t+2) have
// landed or are on their way.  A tile is two steps of 64 MFMAs, the fragments of a step read during the one before it;
// the one barrier of a tile stands between its steps, where every fragment of it is in registers, so that its two units
// are free for B(t+2) and A(t+3).  Between its MFMAs a wavefront issues one fragment read every three and, singly, the
// eight transfers of B at every fourth and those of A at every eighth, over both steps.
//
// What it is bound by: the power limit on long launches (without transfers and reads the same loop reaches 1 850 to 1 970
// TFLOP/s on random operands), short K loops by what stands around them.  Why this shape: with eight wavefronts of 128 x 64
// in a ring of two 64 KB stages (the kernel before this one) every K tile took 192 KB of fragment reads from LDS, here 128,
// and a transfer had three quarters of a tile to arrive, here one to two and a half tiles.  Before -> after, us, operands from memory:
// NT 4096 x 4096 x 4096 114 -> 98, 65 582 x 2048 x 8192 with a residual 1 642 -> 1 541, 32 768 x 4096 x 16 384 3 182 -> 2 923, 65 580 x 1024 x
// 1024 142 -> 137; TN 8192 x 2048 x 65 582 1 633 -> 1 476, 4096 x 16 384 x 32 768 3 246 -> 3 001, 2048 x 6144 x 65 582 1 327 -> 1 206.  The price is
// one wavefront per SIMD in the epilogue, where vector instructions issue every 5.3 clocks instead of every 2.7 to 4.2: 65 629 x 2816 x 1024
// with the gated GELU 474 -> 475, with its derivative 555 -> 526, 65 580 x 8192 x 2048 with GELU and derivative 1 946 -> 1 877.  Of 14 large outputs each,
// geometric means by epilogue: K = 256 0.94 to 1.01, K = 512 0.90 to 1.00, K = 1024 0.92 to 0.99, K = 2048 0.91 to 0.95.
// Tried: two 64 KB stages with this wavefront shape (4096 x 4096 x 16 384 519 us, ring 378); all transfers right behind the
// barrier, one every two MFMAs (5 to 8 % slower); 32x32x16 instructions (5 to 9 % slower); 256 x 128 tiles, two work-groups
// of four wavefronts to a CU (15 to 20 % slower: half as many transfers again).
//
// NT launches of at most one round have two lower tiles besides, 192 x 256 and 128 x 256 (NUA = 6, 4: wavefronts of 96 x 128 and
// 64 x 128, the units of A only partly filled); choose_kernel has the rule and what they measured.
constexpr int UNIT = 256 * BK * 2, RING = 5 * UNIT;      // one operand's K tile in LDS; the whole ring
constexpr int NT_WM = 2;                        // rows of wavefronts in a work-group
template <int NUA> struct Issue {               // where in its steps a wavefront issues what
    static constexpr int STEP = NUA * 8;                            // MFMAs of a step
    static constexpr int RD = NUA == 8 ? 3 : 2;                     // a fragment read every RD,
    static constexpr int DB = NUA / 2, DA = NUA == 4 ? 4 : NUA;     // a transfer of B every DB, of A every DA MFMAs
    static constexpr int ALL = (STEP - 8 * DB - 2) / DA + 1, A1 = ALL < NUA ? ALL : NUA;    // transfers of A in a tile's second step; the rest go in the next step
};
// tile number -> tile coordinates: groups of NT_GROUP tile rows, column-major inside a group
constexpr int NT_GROUP = 4;
__host__ __device__ __forceinline__ void nt_tile_coords(int logical, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    const int group_sz = NT_GROUP * tiles_n;
    const int group = logical / group_sz;
    const int first_m = group * NT_GROUP;
    const int gs = (tiles_m - first_m) < NT_GROUP ? (tiles_m - first_m) : NT_GROUP;
    const int in_group = logical - group * group_sz;
    tile_m = first_m + in_group % gs;
    tile_n = in_group / gs;
}

// TN form (weight gradients): a K tile is 64 rows of 512 contiguous bytes per operand, fetched as whole rows, and the
// MFMA fragments (8 consecutive k for one m or n per lane) come out of LDS through the transpose read
// ds_read_b64_tr_b16, 4 k-rows per read; both operands use the same k order, so the contraction is unchanged.  K may be
// ragged: rows past the end read zeros.  This form needs no transposed copies of the activations.
//
// PS (persistent form, NT only, no uniform split-K): the first ps_wgs work-groups, one per compute unit, stay resident
// and take the n_main unsplit tiles one after another; the tail pieces are ordinary work-groups behind them.  The
// tiles keep their XCD-contiguous numbering: work-group w serves the run of XCD w % 8, starts with tile w / 8 of that
// run and draws every further one from that XCD's counter (ps_ctr[xcd], one atomic per tile, issued a whole main
// loop before its result is needed), so a faster compute unit takes more tiles, as under the hardware dispatcher.
// What persistence buys: the first two K tiles of the NEXT tile are requested before the epilogue of the current one
// starts (into units 0 to 3, while the epilogue stages through unit 4), so neither the latency of that first fetch
// nor the end of one work-group and the start of the next leaves the matrix cores idle.  The last work-group to
// finish puts the counters back to zero (ps_ctr[8] counts the finished ones).
//
// GRP (TN form): the work-groups of several weight gradients over the same K rows (grp), problem after problem.
template <int EPI, bool TNF, bool PS, bool GRP = false, int NUA = 8>
__global__ __launch_bounds__(256, 1) void gemm_bf16_nt_kernel(int M, int N, int K, const bf16_t* __restrict__ A,
                                                              const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
                                                              int tiles_m, int tiles_n, int splits,
                                                              int n_main, int tail_splits,
                                                              float* __restrict__ split_ws, GemmEpi p,
                                                              int ps_wgs, int* __restrict__ ps_ctr,
                                                              std::conditional_t<GRP, TnGroup, NoGroup> grp) {
    static_assert(!(PS && TNF), "the persistent form exists for the NT kernel only");
    static_assert(!GRP || (TNF && EPI == DS_EPI_ACC32), "groups are of weight gradients");
    static_assert(NUA == 8 || !(TNF || PS), "lower tiles: NT, one round");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    typedef Issue<NUA> Z;
    constexpr int WA = NUA * 16, TA = 2 * WA;       // rows of a wavefront, of a tile
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 1, wn = wave & 1;

    // ---- work-group id -> (tile, split).  Two regimes share the kernel:
    //  * uniform split-K (weight gradients): every tile is cut into `splits` K ranges, partial sums go to split_ws
    //    as [split][M][N];
    //  * tail split-K (everything else): the first n_main tiles, a whole number of rounds over the compute units,
    //    run unsplit; each of the remaining tiles is cut into tail_splits K ranges so that the last, partly filled
    //    round costs 1/tail_splits of a round; their partial sums go to split_ws as [tail tile][split][256][256].
    // Tiles are numbered so that each XCD works on contiguous runs, in groups of 4 tile rows (L2 reuse).
    int logical, split, nsplit;
    if constexpr (GRP) {
        logical = xcd_contiguous(blockIdx.x, gridDim.x);
        const int i = tn_group_problem(grp, logical);
        M = grp.p[i].M;
        N = grp.p[i].N;
        A = reinterpret_cast<const bf16_t*>(grp.p[i].A);
        B = reinterpret_cast<const bf16_t*>(grp.p[i].B);
        C = reinterpret_cast<bf16_t*>(grp.p[i].C);
        // one block of the workspace per (split, tile): the problem's first one + split * its tiles + tile
        if (splits > 1) split_ws = grp.block(grp.first[i] + logical);
        tiles_m = M / BM;
        tiles_n = N / BN;
    }
    const int n_tiles = tiles_m * tiles_n;
    bool tail = false;
    const bool persistent = PS && (int)blockIdx.x < ps_wgs;
    int run_start = 0, run_cnt = 0;                 // persistent: this XCD's run of unsplit tiles
    if (persistent) {
        const int xcd = blockIdx.x & 7;
        const int per = n_main >> 3, rem = n_main & 7;
        run_start = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
        run_cnt = per + (xcd < rem ? 1 : 0);
        logical = run_start + (blockIdx.x >> 3);    // (the host launches this form only with n_main >= 2 ps_wgs)
        split = 0;
        nsplit = 1;
    } else if constexpr (GRP) {
        split = logical / n_tiles;
        logical -= split * n_tiles;
        nsplit = splits;
    } else {
        const int pid = PS ? (int)blockIdx.x - ps_wgs + n_main : (int)blockIdx.x;
        const int total = splits > 1 ? n_tiles * splits : n_main;
        if (pid < total) {
            logical = xcd_contiguous(pid, total);
            split = logical / n_tiles;
            logical -= split * n_tiles;
            nsplit = splits;
        } else {
            const int r = pid - total;
            logical = n_main + r / tail_splits;
            split = r % tail_splits;
            nsplit = tail_splits;
            tail = true;
        }
    }

    // This work-group's part of the contraction: NT whole K tiles; TN whole 32-row steps (a product's depth), k_len rows from row k_first on,
    // counted in K tiles from there.  (Divisions go through vector registers: what steers the K loop comes back to scalar ones.)
    constexpr int DEPTH = TNF ? BK / 2 : BK;
    const int steps = TNF ? (K + DEPTH - 1) / DEPTH : K / DEPTH, per_split = (steps + nsplit - 1) / nsplit;
    const int s_begin = split * per_split, s_end = s_begin + per_split < steps ? s_begin + per_split : steps;
    const int k_first = __builtin_amdgcn_readfirstlane(s_begin * DEPTH);
    const int k_len = __builtin_amdgcn_readfirstlane((s_end * DEPTH < K ? s_end * DEPTH : K) - s_begin * DEPTH);
    const int t_begin = TNF ? 0 : __builtin_amdgcn_readfirstlane(s_begin);
    const int t_end = TNF ? (k_len + BK - 1) / BK : __builtin_amdgcn_readfirstlane(s_end);
    // What the transfers of a tile need: its corner and the operand bases there (set_tile), and per-lane offsets that are the same for every
    // tile.  An operand's K tile is 32 transfers, eight per wavefront (of A, NUA): NT 8 rows of 128 bytes each, TN 2 k-rows of 512.
    int tile_m = 0, tile_n = 0, m0 = 0, n0 = 0;
    const char* pa = nullptr;
    const char* pb = nullptr;
    uint32_t len_a = 0;                             // NT: length of A's rows from m0 on
    auto set_tile = [&](int lg) {
        nt_tile_coords(lg, tiles_m, tiles_n, tile_m, tile_n);
        tile_m = __builtin_amdgcn_readfirstlane(tile_m);
        tile_n = __builtin_amdgcn_readfirstlane(tile_n);
        m0 = tile_m * TA;
        n0 = tile_n * BN;
        const uint64_t bytes = (uint64_t)(uint32_t)(M - m0 < TA ? M - m0 : TA) * (uint32_t)K * 2u;
        len_a = bytes > 0xFFFFFFFFu ? 0xFFFFFFFFu : (uint32_t)bytes;
        pa = reinterpret_cast<const char*>(A) + (TNF ? ((long long)k_first * M + m0) * 2 : (long long)m0 * K * 2);
        pb = reinterpret_cast<const char*>(B) + (TNF ? ((long long)k_first * N + n0) * 2 : (long long)n0 * K * 2);
    };
    set_tile(logical);
    uint32_t offA[NUA], offB[8];
    auto lane_offset = [&](int first, uint32_t ld) {
        const int u = first * 64 + lane;                            // 16-byte unit of the tile
        const int row = TNF ? u >> 5 : u >> 3, pos = TNF ? u & 31 : u & 7;
        const int chunk = TNF ? (((pos >> 1) ^ (row & 7)) << 1) | (pos & 1) : pos ^ ((row >> 1) & 7);
        return ((uint32_t)row * ld + chunk * 8) * 2;
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        offB[i] = lane_offset(wave * 8 + i, (uint32_t)(TNF ? N : K));
        if (i < NUA) offA[i] = TNF || NUA != 8 ? lane_offset(wave * NUA + i, (uint32_t)(TNF ? M : K)) : offB[i];
    }
    const uint32_t lds0 = lds_address(smem);
    // The A (part 0) or B (1) part of K tile `tile` as a raw buffer, and its transfer i into ring unit `unit`.  Tiles past the
    // end are buffers of length zero: they fetch nothing, but the wait counts are the same at every step.  TN: the buffer ends
    // behind this tile's columns of the last k-row, so that rows past a ragged K arrive as zeros; NT: at the last row of A.
    auto part = [&](int which, int tile) {
        const uint32_t inside = (uint32_t)((tile - t_end) >> 31);   // all ones before the end
        if constexpr (TNF) {
            const uint32_t ld2 = (uint32_t)(which ? N : M) * 2u;
            const int left = k_len - tile * BK;
            return make_raw_buffer((which ? pb : pa) + (long long)tile * BK * ld2, ((uint32_t)((left < BK ? left : BK) - 1) * ld2 + 512u) & inside);
        } else {
            return make_raw_buffer((which ? pb : pa) + (long long)tile * (BK * 2), (which ? 0xFFFFFFFFu : len_a) & inside);
        }
    };
    const uint32_t lds_a = lds0 + (uint32_t)wave * (NUA * 1024), lds_b = lds0 + (uint32_t)wave * 8192;
    auto transfer_a = [&](i32x4_t buf, int unit, int i) { lds_dma16_buffer(buf, offA[i], lds_a + (uint32_t)unit * UNIT + i * 1024); };
    auto transfer_b = [&](i32x4_t buf, int unit, int i) { lds_dma16_buffer(buf, offB[i], lds_b + (uint32_t)unit * UNIT + i * 1024); };
    auto first_transfer = [&](int tile, int h, int i) {             // transfer i (0 .. NUA + 7) of the first (h = 0) or second K tile: units 0 to 3
        if (i < NUA) transfer_a(part(0, tile), 2 * h, i);
        else transfer_b(part(1, tile), 2 * h + 1, i - NUA);
    };
    // fragments: fb[s] / fa[s] = the 8 column / NUA row units of this wavefront, 32-deep step s of a tile.
    // NT: 128-byte rows: 16 consecutive rows at one chunk index must hit 16 different 16-byte units of a 256-byte
    // window: rows 2q and 2q+1 differ by 128 bytes, the XOR with (row/2)%8 separates the 8 row pairs.
    // TN: 512-byte k-rows.  One fragment (16 features x 32 k) is two transpose reads, each 16 k-rows x 32 bytes: lane
    // (i = lane%16, g = lane/16) addresses k-row 4g + i/4 (+16 for the second read) at features (i%4)*4 of the
    // 16-feature unit and receives feature i at k-rows 4g..4g+3.  The 32 lanes served together touch 8 k-rows, so the
    // 32-byte unit index is XORed with row%8.
    bf16x8_t fa[2][NUA], fb[2][8];
    const int fr = lane & 15, fg = lane >> 4;
    const int nt_lane[2] = {fr * 128 + ((fg ^ ((fr >> 1) & 7)) << 4), fr * 128 + (((4 + fg) ^ ((fr >> 1) & 7)) << 4)};
    const int tr_row = 4 * fg + (fr >> 2), tr_lane = tr_row * 512 + (lane & 3) * 8;
    auto fragment = [&](int unit, int part, int rows, int s, int x) -> bf16x8_t {     // part: this wavefront's row or column in the 2 x 2 grid
        if constexpr (TNF) {
            typedef short s16x4_t __attribute__((ext_vector_type(4)));
            typedef short s16x8_t __attribute__((ext_vector_type(8)));
            typedef __attribute__((address_space(3))) s16x4_t* lds4_t;
            const char* q = smem + unit * UNIT + part * 256 + tr_lane + ((x ^ (tr_row & 7)) << 5) + s * (32 * 512);
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)q);
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(q + 16 * 512));
            const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8_t, v);
        } else {
            return *reinterpret_cast<const bf16x8_t*>(smem + unit * UNIT + part * (rows * 128) + nt_lane[s] + x * 2048);
        }
    };
    auto read = [&](int ua, int ub, int s, int r) {                 // read r (0 .. NUA + 7) of a step: the column units first
        if (r < 8) fb[s][r] = fragment(ub, wn, 128, s, r);
        else fa[s][r - 8] = fragment(ua, wm, WA, s, r - 8);
    };
    f32x4_t acc[NUA][8];
    // One step: NUA x 8 MFMAs on the fragments of 32-deep step s, the reads of the next step (from units ua, ub) and what tr(q) issues
    // between them, in exactly this order.  Operands swapped on purpose: the accumulator block is C^T (rows = n, columns =
    // m), so a lane holds 4 CONSECUTIVE n per block and the epilogue stages with 16-byte writes.  Boustrophedon order:
    // consecutive MFMAs share one operand and the other changes to its neighbour (about 2 % more sustained MFMA rate at the
    // power limit than row-major order).  first: the step that starts the accumulators; last: nothing left to read.
    auto step = [&](auto first_t, auto last_t, int s, int ua, int ub, auto&& tr) {
#pragma unroll
        for (int i = 0; i < NUA; ++i)
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                const int j = (i & 1) ? 7 - jj : jj, q = i * 8 + jj;
                if (!decltype(last_t)::value && q % Z::RD == 0 && q / Z::RD < NUA + 8) read(ua, ub, s ^ 1, q / Z::RD);
                tr(q);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[s][j], fa[s][i], decltype(first_t)::value ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    auto wrap = [](int u) { return u >= 5 ? u - 5 : u; };
    const bool direct = !tail && splits == 1;      // this work-group applies the epilogue itself
    // The bias is the last term of every sum, as in the kernels with smaller tiles and for split contractions: a row does not depend on
    // the tile that takes it.  (It can't be the first: 1 + 2^24 - 2^24.)
    constexpr bool BIAS = EPI == DS_EPI_NONE || EPI == DS_EPI_GELU || EPI == DS_EPI_RESID || EPI == DS_EPI_GELU_D;
    bf16x8_t bias[2];                               // of the columns this lane finishes in the epilogue; none: zeros
    auto load_bias = [&]() {
        const auto b = make_buffer(reinterpret_cast<const bf16_t*>(p.bias) + n0 + wn * 128, direct && p.bias ? 256u : 0u);
#pragma unroll
        for (int h = 0; h < 2; ++h) buffer_load16(b, (uint32_t)(lane & 7) * 16 + h * 128, bias[h]);
    };
    if constexpr (BIAS) load_bias();
    bool primed = false;                            // persistent: the first two K tiles of this tile are already on their way
    for (;;) {
        int next_local = 0x7fffffff;
        if (!primed) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < NUA + 8; ++i) first_transfer(t_begin + h, h, i);
            }
        }
        if constexpr (PS) {
            // the tile after this one: drawn now, needed after the main loop (first tiles of a run: one per work-group)
            if (persistent && t == 0)
                next_local = (ps_wgs >> 3) + __hip_atomic_fetch_add(ps_ctr + (blockIdx.x & 7), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // the first K tile is there: behind its transfers came those of the second one and, persistent, at least the previous tile's stores
        constexpr int BEHIND = 16 + 32 * (epilogue_second<EPI>() || EPI == DS_EPI_ACC32 ? 2 : 1);
        if (PS && primed) __builtin_amdgcn_s_waitcnt(vmcnt_imm(BEHIND < 63 ? BEHIND : 63));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(NUA + 8));
        __builtin_amdgcn_s_barrier();
        // A(tl + 2) is issued in part in the second step of tile tl - 1, the rest in the first step of tile tl
        i32x4_t a2 = part(0, t_begin + 2);
#pragma unroll
        for (int i = 0; i < Z::A1; ++i) transfer_a(a2, 4, i);
#pragma unroll
        for (int r = 0; r < NUA + 8; ++r) read(0, 1, 0, r);
        int tl = t_begin, ua = 0;                   // ua: unit of A(tl); those of B(tl), A(tl+1), B(tl+1), A(tl+2) follow it in the ring
        auto rest_of_a = [&](int q) {
            const int x = q + Z::STEP - 8 * Z::DB - 1;
            if (x % Z::DA == 0 && x / Z::DA >= Z::A1 && x / Z::DA < NUA) transfer_a(a2, wrap(ua + 4), x / Z::DA);
        };
        const std::true_type yes;
        const std::false_type no;
        step(yes, no, 0, 0, 1, rest_of_a);
        while (tl + 1 < t_end) {
            const int na = wrap(ua + 2), nb = wrap(ua + 3), ub = wrap(ua + 1);
            const i32x4_t b2 = part(1, tl + 2);
            a2 = part(0, tl + 3);
            // tile tl+1 has landed for this wavefront (A(tl+2) may be outstanding), its reads of tile tl are done, then everybody's:
            // the units of tile tl are free
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(NUA) & 0xF0FF);
            __builtin_amdgcn_s_barrier();
            step(no, no, 1, na, nb, [&](int q) {
                const int x = q - 8 * Z::DB - 1;
                if (q % Z::DB == 1 && q / Z::DB < 8) transfer_b(b2, ua, q / Z::DB);
                if (x >= 0 && x % Z::DA == 0 && x / Z::DA < Z::A1) transfer_a(a2, ub, x / Z::DA);
            });
            ua = na;
            ++tl;
            step(no, no, 0, ua, nb, rest_of_a);
        }

        // ---- epilogue, 16 rows x 64 columns (a pass) at a time through a block of LDS that is private to the wavefront: two times 16 rows of 64
        // floats, 16-byte chunk c of row r at c ^ r.  Pass s takes columns 64 (s % 2) .. of rows 16 (s / 2) ..; a lane finishes rows
        // lane / 8 and lane / 8 + 8 of it (g = 0, 1), 8 columns each.
        constexpr int NP = 2 * NUA;                     // passes
        const int em0 = m0 + wm * WA, en0 = n0 + wn * 128, etile_m = tile_m, elogical = logical;
        int elane = lane;                              // (opaque, so that no address of the epilogue is kept in registers over the K loop)
        asm volatile("" : "+v"(elane));
        const int rd_row = elane >> 3, rd_col = (elane & 7) * 8, wr_row = elane & 15, wr_col = elane >> 4;
        // The wavefront's rows of a tensor of M x N elements of es bytes as a raw buffer that ends behind the last one which exists, so
        // that every access is made, without a branch: rows past M are read as zeros and not written.  (With branches around the rows
        // the compiler cannot count what is in flight and waits for everything, its own last store included, in front of every row:
        // 65 582 x 2048 x 2048 with a residual 487 -> 572 us.)  on = false: an empty buffer
        const int row_cnt = M - em0 < 0 ? 0 : M - em0 < WA ? M - em0 : WA;
        auto rows = [&](const void* tensor, int es, bool on) {
            return make_buffer(reinterpret_cast<const char*>(tensor) + ((size_t)em0 * N + en0) * es, on ? (uint32_t)row_cnt * (uint32_t)N * es : 0u);
        };
        const uint32_t lane_off = (uint32_t)rd_row * (uint32_t)N + rd_col;       // elements
        auto at = [&](int s, int g, int es) { return (lane_off + (uint32_t)((s >> 1) * 16 + g * 8) * (uint32_t)N + (s & 1) * 64) * es; };
        // What the epilogue reads from memory: PRE passes ahead, the first ones before the next tile's transfers
        constexpr bool READS = epilogue_reads<EPI>(), READS2 = EPI == DS_EPI_DGATE, OLD = EPI == DS_EPI_ACC32;
        constexpr int PRE = READS2 || OLD ? 4 : 8;
        EpiPre<bf16_t> pre[PRE][2];
        f32x4_t old[PRE][2][2];                       // accumulation: what is added to
        const buffer_t in_r = rows(READS ? p.R : C, 2, READS && direct), in_r2 = rows(READS2 ? p.R2 : C, 2, READS2 && direct);
        const buffer_t in_valid = make_buffer(p.row_valid + em0, EPI == DS_EPI_RESID && direct && p.row_valid ? row_cnt * 4u : 0u);
        const buffer_t in_old = rows(C, 4, OLD && direct && p.accumulate);
        auto prefetch_pass = [&](int s) {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                EpiPre<bf16_t>& e = pre[s % PRE][g];
                if constexpr (READS) buffer_load16(in_r, at(s, g, 2), e.r);
                if constexpr (READS2) buffer_load16(in_r2, at(s, g, 2), e.r2);
                e.valid = 0;
                if constexpr (EPI == DS_EPI_RESID) e.valid = buffer_load4(in_valid, (uint32_t)((s >> 1) * 16 + g * 8 + rd_row) * 4);
                if constexpr (OLD) {
                    buffer_load16(in_old, at(s, g, 4), old[s % PRE][g][0]);
                    buffer_load16(in_old, at(s, g, 4) + 16, old[s % PRE][g][1]);
                }
            }
        };
        // The last tile's second step: all its fragments are in registers, so the ring is free once everybody has got here (and nothing is
        // on its way into it: explicit, the compiler does not see the transfers).  In front of its products go the first reads of the
        // epilogue, between them the transfers of the next tile's first K tile; those of the second one follow between the passes.
        __builtin_amdgcn_s_waitcnt(0x0070);
        float column[2][8];                             // the bias
        if constexpr (BIAS) {
#pragma unroll
            for (int j = 0; j < 8; ++j) column[0][j] = (float)bias[0][j], column[1][j] = (float)bias[1][j];
        }
        char* stg = smem + 4 * UNIT + wave * 8192;
        int next_logical = -1;
        __builtin_amdgcn_s_barrier();
        if constexpr (PS) {
            // the number of the next tile reaches the other wavefronts through a word of each one's own block (behind the barrier: the
            // unit may have held this tile)
            if (persistent && t == 0) {
#pragma unroll
                for (int w = 0; w < 4; ++w) *reinterpret_cast<volatile int*>(smem + 4 * UNIT + w * 8192) = next_local;
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
        }
        if constexpr (PS) {
            if (persistent) {
                const int nl = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(stg));
                if (nl < run_cnt) {
                    next_logical = run_start + nl;
                    set_tile(next_logical);
                    if constexpr (BIAS) load_bias();
                    primed = true;
                }
            }
        }
        if constexpr (READS) {
#pragma unroll
            for (int s = 0; s < PRE; ++s) prefetch_pass(s);
        }
        if (OLD && p.accumulate) {
#pragma unroll
            for (int s = 0; s < PRE; ++s) prefetch_pass(s);
        }
        const int next_begin = next_logical < 0 ? t_end : t_begin;      // (no next tile: buffers of length zero, drained behind the loop)
        __builtin_amdgcn_sched_barrier(0);
        step(no, yes, 1, 0, 0, [&](int q) {
            if (PS && q % 4 == 1) first_transfer(next_begin, 0, q / 4);
        });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!BIAS && EPI != DS_EPI_ACC32) {
            // a bias where the interface names none: one product of it (columns x k, all but k = 0 zero) with ones adds it to a block
            if (direct && p.bias) {
                const auto b = make_buffer(reinterpret_cast<const bf16_t*>(p.bias) + en0, 256u);
                const float ones = lane < 16 ? 1.f : 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float v = __builtin_bit_cast(float, (uint32_t)buffer_load2(b, lane < 16 ? (uint32_t)(j * 16 + lane) * 2 : 256u) << 16);
#pragma unroll
                    for (int i = 0; i < NUA; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, ones, acc[i][j], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const i32x4_t next_a = part(0, next_begin + 1), next_b = part(1, next_begin + 1);
        // put: the accumulators of pass s into its half of the staging block; get: the 2 x 8 columns of this lane back from it.  A pass is put
        // and read while the one before it is finished.
        struct Pass { float4 x[2][2]; };
        auto put = [&](int s) {
            char* blk = stg + (s & 1) * 4096 + wr_row * 256;
#pragma unroll
            for (int j = 0; j < 4; ++j)         // lane = row m (lane%16); its 4 registers = columns 4*(lane/16) + 0..3 of a block
                *reinterpret_cast<f32x4_t*>(blk + (((4 * j + wr_col) ^ wr_row) << 4)) = acc[s >> 1][(s & 1) * 4 + j];
        };
        auto get = [&](int s) {
            Pass v;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int row = g * 8 + rd_row;
                const char* r = stg + (s & 1) * 4096 + row * 256;
                v.x[g][0] = *reinterpret_cast<const float4*>(r + (((rd_col >> 2) ^ row) << 4));
                v.x[g][1] = *reinterpret_cast<const float4*>(r + ((((rd_col >> 2) + 1) ^ row) << 4));
            }
            return v;
        };
        // every pass: out(s, g, v) gets the 8 columns of row g of this lane; after(s) follows.  rolled: g in a loop, for what is long per row
        // (unrolled over all 32 rows of a lane such kernels come to 45 to 64 KB of code, which a launch fetches from memory)
        auto passes = [&](auto rolled, auto&& out, auto&& after) {
            wave_lds_sync();            // the staging block is private to the wavefront: no work-group barrier (which would
                                        // also wait for the global stores of the previous pass to be acknowledged)
            put(0);
            wave_lds_sync();
            Pass cur = get(0);
#pragma unroll
            for (int s = 0; s < NP; ++s) {
                Pass next = cur;
                if (s + 1 < NP) {
                    put(s + 1);
                    wave_lds_sync();
                    next = get(s + 1);
                }
                auto row_of = [&](int g) {
                    const float4 x0 = g ? cur.x[1][0] : cur.x[0][0], x1 = g ? cur.x[1][1] : cur.x[0][1];
                    float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
                    out(s, g, v);
                };
                if constexpr (decltype(rolled)::value) {
#pragma unroll 1
                    for (int g = 0; g < 2; ++g) row_of(g);
                } else {
                    row_of(0);
                    row_of(1);
                }
                after(s);
                if constexpr (PS) {
                    if (s < 8) transfer_a(next_a, 2, s);
                    else transfer_b(next_b, 3, s - 8);
                }
                cur = next;
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // column sums of what this lane writes (DGELU: the bias gradient of the layer below comes out of this kernel
        // instead of a pass over the stored tensor); every lane finishes 2 NUA rows of the same 16 columns
        constexpr bool SUMS = EPI == DS_EPI_DGELU || EPI == DS_EPI_MULR;
        float csum[2][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) csum[0][j] = csum[1][j] = 0.f;
        if (!direct || (OLD && !p.accumulate)) {
            // an output that is not added to (with the reads and additions of the other form, of nothing, gradients over a few hundred tokens took 3 %
            // longer), or partial sums: [split][M][N], or blocks of a whole tile (rows past M are never read there)
            const bool block = (GRP || tail) && !direct;
            float* dst = direct ? reinterpret_cast<float*>(C)
                       : GRP ? split_ws
                       : tail ? split_ws + (size_t)((elogical - n_main) * tail_splits + split) * (BM * BN) : split_ws + (size_t)split * M * N;
            const buffer_t out = block ? make_buffer(dst + (size_t)(wm * 128) * BN + wn * 128, 128 * BN * 4) : rows(dst, 4, true);
            const uint32_t ld = block ? BN : N, off = ((uint32_t)rd_row * ld + rd_col) * 4;
            passes(no, [&](int s, int g, float (&v)[8]) {
                const uint32_t o = off + ((s >> 1) * 16 + g * 8) * ld * 4 + (s & 1) * 256;
                buffer_store16(f32x4_t{v[0], v[1], v[2], v[3]}, out, o);
                buffer_store16(f32x4_t{v[4], v[5], v[6], v[7]}, out, o + 16);
            }, [](int) {});
        } else {
            constexpr bool LONG = EPI == DS_EPI_GELU || EPI == DS_EPI_GELU_D || EPI == DS_EPI_DGELU || EPI == DS_EPI_GATE || EPI == DS_EPI_DGATE;
            const buffer_t out = rows(C, OLD ? 4 : 2, true), out2 = rows(epilogue_second<EPI>() ? p.C2 : C, 2, epilogue_second<EPI>());
            passes(std::integral_constant<bool, LONG>{}, [&](int s, int g, float (&v)[8]) {
                if constexpr (OLD) {
                    buffer_store16(f32x4_t{v[0], v[1], v[2], v[3]} + old[s % PRE][g][0], out, at(s, g, 4));
                    buffer_store16(f32x4_t{v[4], v[5], v[6], v[7]} + old[s % PRE][g][1], out, at(s, g, 4) + 16);
                } else {
                    if constexpr (BIAS) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) v[j] += column[s & 1][j];
                    }
                    bf16x8_t one, two;
                    EpiPre<bf16_t> e = pre[s % PRE][0];
                    if constexpr (READS) {
                        if (g) e = pre[s % PRE][1];
                    }
                    epilogue_values<bf16_t, EPI>(v, e, one, two);
                    buffer_store16_nt(one, out, at(s, g, 2));
                    if constexpr (epilogue_second<EPI>()) buffer_store16_nt(two, out2, at(s, g, 2));
                    if constexpr (SUMS) {
                        const bool exists = (s >> 1) * 16 + g * 8 + rd_row < row_cnt;
#pragma unroll
                        for (int j = 0; j < 8; ++j) csum[s & 1][j] = exists ? csum[s & 1][j] + v[j] : csum[s & 1][j];    // (one fused multiply-add per term)
                    }
                }
            }, [&](int s) {
                if ((READS || OLD) && s + PRE < NP) prefetch_pass(s + PRE);
            });
        }
        if constexpr (SUMS) {
            if (direct && p.colsum) {
                // lanes l, l + 8, l + 16, ... hold the same columns: fold them, then one row of partial sums per
                // (tile row, wavefront row), written whether or not the wavefront had a valid row
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int o = 8; o < 64; o <<= 1)
#pragma unroll
                        for (int j = 0; j < 8; ++j) csum[h][j] += __shfl_xor(csum[h][j], o, 64);
                    if (NUA == 8 && lane < 8) Vec8<float>::store(p.colsum + (size_t)(etile_m * NT_WM + wm) * N + en0 + h * 64 + rd_col, csum[h]);
                }
                if constexpr (NUA == 4) {
                    // one row per tile row: the two wavefronts of a column add theirs in LDS.  Two rows are counted per 256
                    // (gemm_colsum_rows): the last one may have no tile
                    float* red = reinterpret_cast<float*>(smem);
                    if (lane < 8) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) Vec8<float>::store(red + wm * BN + wn * 128 + h * 64 + rd_col, csum[h]);
                    }
                    __syncthreads();
                    p.colsum[(size_t)etile_m * N + n0 + t] = red[t] + red[BN + t];
                    if (etile_m + 1 == tiles_m && (tiles_m & 1)) p.colsum[(size_t)(etile_m + 1) * N + n0 + t] = 0.f;
                }
            }
        }
        // (not persistent: one tile.  The compiler is kept from knowing, because without the loop around the tile it moves accumulators between
        // the two halves of the register file inside the K loop, hundreds of copies a tile)
        if constexpr (!PS) asm volatile("" : "+s"(next_logical));
        if (next_logical < 0) break;
        logical = next_logical;
        if constexpr (!PS) set_tile(logical);
    }   // for (;;): persistent work-groups go on with their next tile
    if constexpr (PS) {
        __builtin_amdgcn_s_waitcnt(0x0F70);         // no transfer may still be writing LDS when the work-group ends
        if (persistent && t == 0) {
            // every persistent work-group ends with a draw beyond its run; the last one to finish clears the counters
            const int done = __hip_atomic_fetch_add(ps_ctr + 8, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (done == ps_wgs - 1) {
#pragma unroll
                for (int i = 0; i < 9; ++i) ps_ctr[i] = 0;
            }
        }
    }
}

// sum the tail tiles' split-K partials ([tile][split][256][256]) and apply the epilogue; one thread per 8 columns
template <int EPI>
__global__ __launch_bounds__(256) void tail_finish_kernel(int M, int N, int tiles_m, int tiles_n, int n_main, int tail_splits,
                                                          const float* __restrict__ ws, bf16_t* __restrict__ C, GemmEpi p) {
    const int tile = blockIdx.y;
    int tile_m, tile_n;
    nt_tile_coords(n_main + tile, tiles_m, tiles_n, tile_m, tile_n);
    const float* base = ws + (size_t)tile * tail_splits * (BM * BN);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < BM * (BN / 8); i += gridDim.x * blockDim.x) {
        const int r = i / (BN / 8), c8 = (i % (BN / 8)) * 8;
        const int m = tile_m * BM + r, n = tile_n * BN + c8;
        if (m >= M) continue;
        float v[8];
        Vec8<float>::load(base + (size_t)r * BN + c8, v);
        for (int sp = 1; sp < tail_splits; ++sp) {
            float w[8];
            Vec8<float>::load(base + ((size_t)sp * BM + r) * BN + c8, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] += w[j];
        }
        epilogue8<bf16_t, EPI>(m, n, N, v, C, p);
    }
}

// The same with the column sums of the output (p.colsum): one block of 1024 threads per 128-row half of a tile, which
// writes the row of p.colsum the main kernel's work-groups would have written had they finished the tile themselves.
template <int EPI>
__global__ __launch_bounds__(1024) void tail_finish_sums_kernel(int M, int N, int tiles_m, int tiles_n, int n_main, int tail_splits,
                                                                const float* __restrict__ ws, bf16_t* __restrict__ C, GemmEpi p) {
    __shared__ float red[32][BN];
    const int tile = blockIdx.y;
    int tile_m, tile_n;
    nt_tile_coords(n_main + tile, tiles_m, tiles_n, tile_m, tile_n);
    const float* base = ws + (size_t)tile * tail_splits * (BM * BN);
    const int c8 = (threadIdx.x & 31) * 8, n = tile_n * BN + c8;
    float csum[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) csum[j] = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {                   // 4 x 32 rows; independent iterations, their loads in flight together
        const int r = blockIdx.x * 128 + k * 32 + (threadIdx.x >> 5);
        const int m = tile_m * BM + r;
        if (m >= M) continue;
        float v[8];
        Vec8<float>::load(base + (size_t)r * BN + c8, v);
        for (int sp = 1; sp < tail_splits; ++sp) {
            float w[8];
            Vec8<float>::load(base + ((size_t)sp * BM + r) * BN + c8, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] += w[j];
        }
        epilogue8<bf16_t, EPI>(m, n, N, v, C, p);
#pragma unroll
        for (int j = 0; j < 8; ++j) csum[j] += v[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[threadIdx.x >> 5][c8 + j] = csum[j];
    __syncthreads();
    if (threadIdx.x < BN) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 32; ++k) t += red[k][threadIdx.x];
        p.colsum[(size_t)(tile_m * 2 + blockIdx.x) * N + tile_n * BN + threadIdx.x] = t;
    }
}

template <class T, int EPI>
ds_status launch_generic(int ta, int tb, int M, int N, int K, const void* A, const void* B, void* C, const GemmEpi& p,
                         hipStream_t st) {
    const long long sam = ta ? 1 : K, sak = ta ? M : 1;
    const long long sbk = tb ? 1 : N, sbn = tb ? K : 1;
    dim3 grid((N + 63) / 64, (M + 63) / 64);
    hipLaunchKernelGGL((gemm_generic_kernel<T, EPI>), grid, dim3(256), 0, st, M, N, K, (const T*)A, sam, sak, (const T*)B,
                       sbk, sbn, (T*)C, p);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

// number of K splits of a product with fp32 output: the fewest that bring the work-group count closest to a whole
// number of rounds over the compute units (time ~ rounds x split length), of 512 rows or more for a weight gradient, 1 024 for an NT product
static int choose_splits(int tiles, int nt, int M, int N, size_t split_ws_floats) {
    const int n_cu = gemm_cu_count();
    int best = 1;
    double best_cost = 1e30;
    for (int sp = 1; sp <= 16; ++sp) {
        if (sp > 1 && (sp > nt / 16 || (size_t)sp * M * N > split_ws_floats)) break;
        const int per = (nt + sp - 1) / sp;
        if ((nt + per - 1) / per != sp) continue;               // every split must own at least one K tile
        const double rounds = (double)(((long long)tiles * sp + n_cu - 1) / n_cu);
        const double cost = rounds * per * (1.0 + 0.01 * sp);    // slight preference for fewer partial sums
        if (cost < best_cost - 1e-9) { best_cost = cost; best = sp; }
    }
    return best;
}

// How a launch of the 256 x 256 kernel divides its tiles: uniform splits (weight gradients), or whole tiles and a tail
// whose K loops are cut into tail_splits pieces.
struct BigPlan {
    int tiles_m, tiles_n, nt;      // nt: what the contraction is cut in, NT 64-deep K tiles, TN 32-deep steps
    int splits, n_main, tail_splits;
};
static BigPlan plan_big(bool tnf, int epi, int M, int N, int K, size_t split_ws_floats) {
    BigPlan b;
    b.tiles_m = (M + BM - 1) / BM;
    b.tiles_n = N / BN;
    b.nt = tnf ? (K + BK / 2 - 1) / (BK / 2) : K / BK;
    const int tiles = b.tiles_m * b.tiles_n;
    b.splits = epi == DS_EPI_ACC32 && split_ws_floats ? choose_splits(tiles, b.nt, M, N, split_ws_floats) : 1;
    // tail split-K: the tiles beyond the last whole round over the compute units share that round; a launch with
    // fewer tiles than compute units (small micro-batches) is all tail, so that the K loop is spread over the chip
    b.n_main = tiles;
    b.tail_splits = 1;
    if (b.splits == 1 && split_ws_floats) {
        const int n_cu = gemm_cu_count();
        const int rem = tiles % n_cu;
        if (rem > 0) {
            int ts = n_cu / rem;
            if (ts > 32) ts = 32;
            if (ts > b.nt / 4) ts = b.nt / 4;
            while (ts > 1 && (size_t)rem * ts * (BM * BN) > split_ws_floats) --ts;
            if (ts > 1) {
                const int per = (b.nt + ts - 1) / ts;
                ts = (b.nt + per - 1) / per;                    // every split owns at least one K tile
            }
            if (ts > 1) { b.n_main = tiles - rem; b.tail_splits = ts; }
        }
    }
    return b;
}

// Estimated time of that plan in microseconds (see gemm_tile.hip for the other side of the comparison and the fit): 1.15
// (TN) or 1.25 (NT, operands from memory; 1.15 warm) per 64-deep K tile of a 256 x 256 tile and 4 around it, per round over
// the compute units; 0.1 per piece of partial sums (256 KB written and read back) and 4 for the launch that adds them.
// The rates were fitted to the kernel with eight wavefronts.  The choices hold with four: of 400 random NT products (six epilogues, K = 256 .. 8192, up
// to 46 000 rows) and 300 weight gradients (64 to 46 000 tokens) for which they decide something, what is taken takes 0.5 % and 0.9 % longer than the best of
// itself, no smaller tiles and only smaller tiles (mean of operands from memory and warm); 13 and 21 of them over 3 %, 1 and 8 over 10 %, at worst 18 % (weight gradients of
// 70 to 200 tokens, where 128 x 64 tiles are estimated too low).
static double big_cost(const BigPlan& b, bool tnf, int M, int N) {
    const int n_cu = gemm_cu_count(), tiles = b.tiles_m * b.tiles_n;
    const double steps = tnf ? 0.5 * b.nt : b.nt, step = tnf ? 1.15 : 1.25;
    auto rounds = [&](double work_groups) { return std::ceil(work_groups / n_cu); };
    if (b.splits > 1)
        return rounds((double)tiles * b.splits) * (steps / b.splits * step + 4) + 2e-6 * (double)b.splits * M * N + 4;
    double t = b.n_main ? rounds(b.n_main) * (steps * step + 4) : 0;
    const int tail = tiles - b.n_main;
    if (tail) t += steps / b.tail_splits * step + 4 + 0.1 * tail * b.tail_splits + 4;
    return t;
}

// persistent form: one resident work-group per compute unit for the unsplit tiles, when each has several to do
static bool nt_persistent(const BigPlan& b) {
    const int n_cu = gemm_cu_count();
    return b.splits == 1 && n_cu % 8 == 0 && b.n_main >= 2 * n_cu;
}

// Tile counters of the persistent form: 64 slots of [8 per-XCD counters, 1 count of finished work-groups], all zero
// between launches (the last work-group of a launch clears its slot).  Launches take the slots in turn, so two
// launches can only share one if more than 64 are in flight on a device at the same time.
constexpr int PS_SLOTS = 64;
__device__ int g_ps_ctr[PS_SLOTS][16];
static int* ps_counters() {
    static std::mutex mu;
    static int* base[64] = {};
    static std::atomic<unsigned> next{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!base[dev]) {
            void* ptr = nullptr;
            if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_ps_ctr)) != hipSuccess) return nullptr;
            base[dev] = static_cast<int*>(ptr);
        }
    }
    return base[dev] + 16 * (next.fetch_add(1) % PS_SLOTS);
}

template <int EPI, bool TNF>
ds_status launch_nt(int M, int N, int K, const void* A, const void* B, void* C, const GemmEpi& p, float* split_ws,
                    size_t split_ws_floats, hipStream_t st) {
    static bool attr_set = false;
    auto kern = gemm_bf16_nt_kernel<EPI, TNF, false>;
    if (!attr_set) {
        DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, RING));
        attr_set = true;
    }
    const BigPlan plan = plan_big(TNF, EPI, M, N, K, split_ws ? split_ws_floats : 0);
    const int tiles_m = plan.tiles_m, tiles_n = plan.tiles_n, tiles = tiles_m * tiles_n;
    const int splits = plan.splits, n_main = plan.n_main, tail_splits = plan.tail_splits;
    const int total = splits > 1 ? tiles * splits : n_main + (tiles - n_main) * tail_splits;
    bool launched = false;
    if constexpr (!TNF) {
        const int n_cu = gemm_cu_count();
        if (nt_persistent(plan)) {
            static bool ps_attr_set = false;
            auto kern_ps = gemm_bf16_nt_kernel<EPI, false, true>;
            if (!ps_attr_set) {
                DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern_ps), hipFuncAttributeMaxDynamicSharedMemorySize, RING));
                ps_attr_set = true;
            }
            int* ctr = ps_counters();
            if (ctr) {
                hipLaunchKernelGGL(kern_ps, dim3(n_cu + (tiles - n_main) * tail_splits), dim3(256), RING, st, M, N, K,
                                   (const bf16_t*)A, (const bf16_t*)B, (bf16_t*)C, tiles_m, tiles_n, splits, n_main, tail_splits,
                                   split_ws, p, n_cu, ctr, NoGroup{});
                launched = true;
            }
        }
    }
    if (!launched)
        hipLaunchKernelGGL(kern, dim3(total), dim3(256), RING, st, M, N, K, (const bf16_t*)A, (const bf16_t*)B, (bf16_t*)C,
                           tiles_m, tiles_n, splits, n_main, tail_splits, split_ws, p, 0, (int*)nullptr, NoGroup{});
    DS_LAUNCH_CHECK();
    if (splits > 1) {
        return launch_splitk_finish<bf16_t, EPI>(M, N, splits, split_ws, C, p, st);
    } else if (tail_splits > 1) {
        bool with_sums = false;
        if constexpr (EPI == DS_EPI_DGELU || EPI == DS_EPI_MULR) {
            if (p.colsum) {
                with_sums = true;
                hipLaunchKernelGGL(tail_finish_sums_kernel<EPI>, dim3(2, tiles - n_main), dim3(1024), 0, st, M, N, tiles_m, tiles_n,
                                   n_main, tail_splits, split_ws, (bf16_t*)C, p);
            }
        }
        if (!with_sums)
            hipLaunchKernelGGL(tail_finish_kernel<EPI>, dim3(8, tiles - n_main), dim3(256), 0, st, M, N, tiles_m, tiles_n,
                               n_main, tail_splits, split_ws, (bf16_t*)C, p);
        DS_LAUNCH_CHECK();
    }
    return DS_OK;
}

// NT, every tile unsplit, tiles of 32 NUA rows
template <int EPI, int NUA>
ds_status launch_nt_lower(int M, int N, int K, const void* A, const void* B, void* C, const GemmEpi& p, hipStream_t st) {
    static bool attr_set = false;
    auto kern = gemm_bf16_nt_kernel<EPI, false, false, false, NUA>;
    if (!attr_set) {
        DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, RING));
        attr_set = true;
    }
    const int tiles_m = (M + 32 * NUA - 1) / (32 * NUA), tiles_n = N / BN, tiles = tiles_m * tiles_n;
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(256), RING, st, M, N, K, (const bf16_t*)A, (const bf16_t*)B, (bf16_t*)C, tiles_m,
                       tiles_n, 1, tiles, 1, (float*)nullptr, p, 0, (int*)nullptr, NoGroup{});
    DS_LAUNCH_CHECK();
    return DS_OK;
}

// Which matrix-core kernel an NT launch (tn: a weight gradient) goes to and what it is expected to take: pick.kind -1 = 256 x 256
// tiles, kLower192 and kLower128 = 192 x 256 and 128 x 256.
//
// The lower tiles are for launches that leave CUs idle with 256 x 256 tiles and still fit into one round with these: the K loop of a
// CU is shorter by what its tile is lower, less what a transfer, a fragment read and a wait cost per MFMA.  Measured per K tile
// and around them, microseconds, operands from memory / warm: 256 rows 1.25 / 1.15 and 4 (big_cost); 192 rows 1.07 / 0.85, 128 rows 0.99 / 0.65.
// Of 110 shapes whose launch is one round (N = 256 .. 8192, K = 64 .. 8192, plain and residual outputs), with these against without,
// geometric means: from memory 0.97, warm 0.95; below K = 512 on at least two thirds of the CUs 0.83 and 0.93, on fewer 1.11 and 1.05 (not
// taken: where a launch is mostly its ends, small tiles on all CUs are better).  Of the rest 2 lose more than 3 % of the mean of both, at
// worst 6 %.  (Estimates of 1.05 and 0.85, closer to the warm rates: 0.99 and 0.95.)
// Of another 60 shapes that go to them from each epilogue, from memory and warm: 192 rows 0.86 to 0.94 and 0.83 to 0.89, 128 rows 0.88 to 0.97 and
// 0.88 to 0.98, at worst 5 % over in the mean of both (128 rows of K = 2816 from memory alone 1.03, warm 0.87), but for the derivative of the GELU
// on 128 rows, 1.05 and 1.04, at worst 1.11: these go on without (11 operations an element with one wavefront per SIMD).
constexpr int kLower192 = 100, kLower128 = 101;
constexpr double kStep192 = 1.10, kStep128 = 1.05;
struct NtChoice {
    TilePick pick;
    double cost;
};
static NtChoice choose_kernel(bool tn, int epi, int M, int N, int K, size_t wsf, bool colsum, int accumulate) {
    const BigPlan plan = plan_big(tn, epi, M, N, K, wsf);
    const double out_us = gemm_output_us(epi, M, N, accumulate);
    const bool fits = gemm_big_width(epi, N);
    const NtChoice big{TilePick{-1, 1, 0.0, 0.0}, fits ? big_cost(plan, tn, M, N) + out_us : 1e30};
    NtChoice c = big;
    if (!tn && fits)
        for (const int rows : {192, 128}) {
            const long long work_groups = ((long long)M + rows - 1) / rows * (N / BN);
            if (work_groups > gemm_cu_count() || (colsum && rows != 128) || (K < 512 && 3 * work_groups < 2 * gemm_cu_count())) continue;
            const double cost = plan.nt * (rows == 192 ? kStep192 : kStep128) + 4 * rows / 256.0 + out_us;
            if (cost < c.cost) c = NtChoice{TilePick{rows == 192 ? kLower192 : kLower128, 1, cost, cost}, cost};
        }
    if (epi == DS_EPI_DGELU && c.pick.kind == kLower128) c = big;
    if (!fits || (long long)plan.tiles_m * plan.tiles_n <= 2 * gemm_cu_count()) {
        // launches that do not fill the chip with 256 x 256 tiles: smaller ones, where the estimates say so (ties go to the large tile);
        // outputs too wide for these
        const TilePick pick = pick_gemm_tile(tn, M, N, K, wsf, colsum, out_us, accumulate != 0);
        if (pick.kind >= 0 && pick.versus_large < 0.95 * c.cost) c = NtChoice{pick, pick.versus_large};
    }
    return c;
}

// NT launches whose last rows open another round over the CUs (4 173 x 4 096 outputs: 256 tiles of 256 x 256 and 16 more for 77 rows,
// whose K loops are then cut into pieces and added up by a launch of their own) go out as two: the rows of the whole rounds
// first, the rest with the tiles that suit it, where the estimates with 1 us between them are 3 % below that of one.  0: one launch.
// 4 173 x 4 096 x 1 024: 51 -> 45 us, 4 173 x 4 352 x 1 024: 54 -> 46.
// Below K = 512 one launch cuts no K loop, and from two rounds on its tiles are drawn, so that the last ones run beside others; what
// a second launch costs then is not in the estimates.  Of 292 shapes (N = 256 .. 8192, 1 to 8 rounds, operands from memory, plain and
// residual outputs) for which they say two, two launches / one, geometric mean and worst: K = 64 and 128, 1.06 and 1.41; K = 256 .. 448
// two rounds 0.95 and 1.04 (the exception below), one round 0.98 and 1.08, more 1.03 and 1.25; K = 512 and more 0.91 and 1.05.
// (All with the kernel of eight wavefronts.  With four, 300 random products that go out as two against one launch: 0.94 from memory and 0.91 warm, 3 of
// them over 3 % longer, at worst 6 %.)
// Behind one round, rows that fill more than a tenth of another are not worth it either below K = 1536: half a launch more of tiles that
// read and write as much as they multiply.  Of another 220 (all of K >= 512, remainders of any size, epilogues with up to two more
// operands and results), 46 such, from memory and warm: 0.97 and 0.98, worst 1.13 and 1.11; the rest 0.93 and 0.90, worst 1.08 and 1.00.
static int rows_of_whole_rounds(int epi, int M, int N, int K, size_t wsf, bool colsum, int accumulate, double one) {
    const int n_cu = gemm_cu_count(), tiles_n = N / BN;
    const long long rounds = (long long)((M + BM - 1) / BM) * tiles_n / n_cu;
    const long long rows = rounds * n_cu / tiles_n * BM;
    if (rounds < 1 || rows <= 0 || rows >= M) return 0;
    if (K < 512 && (rounds != 2 || K < 256)) return 0;
    const long long behind = (long long)((M + BM - 1) / BM) * tiles_n - rows / BM * tiles_n;
    if (rounds == 1 && K < 1536 && 10 * behind > n_cu) return 0;
    const double two = choose_kernel(false, epi, (int)rows, N, K, wsf, colsum, accumulate).cost + 1 +
                       choose_kernel(false, epi, M - (int)rows, N, K, wsf, colsum, accumulate).cost;
    return two < 0.97 * one ? (int)rows : 0;
}

// Whether a bf16 product goes to the matrix cores: NT, or TN with fp32 output (a K tile of each operand there is addressed through a 32-bit
// buffer length)
static bool matrix_cores_take(int ta, int tb, int epi, int M, int N, int K, const void* A, const void* B, const void* C) {
    if (M < 1 || K < 1 || N % BN || (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) & 15)) return false;
    if (!ta && tb) return K % BK == 0;
    return ta && !tb && epi == DS_EPI_ACC32 && M % BM == 0 && M <= (1 << 25) && N <= (1 << 25);
}

// The launches of a product that matrix_cores_take: one, or the rows of the whole rounds and the rows behind them
struct Launches {
    int n, rows[2];
    NtChoice c[2];
};
static Launches choose_launches(bool tn, int epi, int M, int N, int K, size_t wsf, bool colsum, int accumulate) {
    Launches l{1, {M, 0}, {choose_kernel(tn, epi, M, N, K, wsf, colsum, accumulate), {}}};
    const int rows = tn || !gemm_big_width(epi, N) ? 0 : rows_of_whole_rounds(epi, M, N, K, wsf, colsum, accumulate, l.c[0].cost);
    if (rows > 0) {
        l = Launches{2, {rows, M - rows}, {}};
        for (int i = 0; i < 2; ++i) l.c[i] = choose_kernel(tn, epi, l.rows[i], N, K, wsf, colsum, accumulate);
    }
    return l;
}

template <int EPI>
ds_status dispatch_epi(int dtype, int ta, int tb, int M, int N, int K, const void* A, const void* B, void* C,
                       const GemmEpi& p, bool force_generic, float* split_ws, size_t split_ws_floats, hipStream_t st) {
    if (dtype == DS_DTYPE_BF16 && !force_generic && matrix_cores_take(ta, tb, EPI, M, N, K, A, B, C)) {
        const bool tn = ta;
        const Launches l = choose_launches(tn, EPI, M, N, K, split_ws ? split_ws_floats : 0, p.colsum != nullptr, p.accumulate);
        GemmEpi q = p;
        size_t row = 0;
        for (int i = 0; i < l.n; ++i) {
            const TilePick& pick = l.c[i].pick;
            const int m = l.rows[i];
            const void* a = (const bf16_t*)A + row * K;
            void* out = EPI == DS_EPI_ACC32 ? (void*)((float*)C + row * N) : (void*)((bf16_t*)C + row * N);
            ds_status r;
            if (pick.kind >= 0 && pick.kind < kLower192) r = launch_gemm_tile(pick, tn, m, N, K, a, B, out, EPI, q, split_ws, st);
            else if (pick.kind == kLower192) r = launch_nt_lower<EPI, 6>(m, N, K, a, B, out, q, st);
            else if (pick.kind == kLower128) {
                if constexpr (EPI == DS_EPI_DGELU) r = DS_EINVAL;       // (choose_kernel keeps it off these)
                else r = launch_nt_lower<EPI, 4>(m, N, K, a, B, out, q, st);
            } else if (!tn) r = launch_nt<EPI, false>(m, N, K, a, B, out, q, split_ws, split_ws_floats, st);
            else if constexpr (EPI == DS_EPI_ACC32) r = launch_nt<EPI, true>(m, N, K, a, B, out, q, split_ws, split_ws_floats, st);
            else r = DS_EINVAL;
            if (r != DS_OK || i + 1 == l.n) return r;
            row = (size_t)m;
            auto behind = [&](const void* x) -> const void* { return x ? (const bf16_t*)x + row * N : nullptr; };
            q.R = behind(p.R);
            q.R2 = behind(p.R2);
            q.C2 = const_cast<void*>(behind(p.C2));
            if (p.row_valid) q.row_valid = p.row_valid + row;
            if (p.colsum) q.colsum = p.colsum + gemm_colsum_rows(m) * N;
        }
    }
    if (dtype == DS_DTYPE_BF16) return launch_generic<bf16_t, EPI>(ta, tb, M, N, K, A, B, C, p, st);
    if (!force_generic && gemm_f32_mfma_supported(ta, tb, M, N, K, A, B))
        return launch_gemm_f32_mfma(ta, tb, M, N, K, A, B, C, EPI, p, split_ws, split_ws_floats, st);
    return launch_generic<float, EPI>(ta, tb, M, N, K, A, B, C, p, st);
}

}  // namespace

bool gemm_colsum_fused(int32_t dtype, int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B,
                       const void* C, int32_t epilogue) {
    // every matrix-core kernel of an NT product fills p.colsum: two rows of partial column sums per tile row of 256, one per 128 rows of the
    // 128 x 256 tile and the 128-row tiles of gemm_tile.hip (the only other ones that choose_kernel takes when p.colsum is set)
    static_assert(NT_WM == 2, "two rows of partial column sums per tile row");
    return (epilogue == DS_EPI_DGELU || epilogue == DS_EPI_MULR) && dtype == DS_DTYPE_BF16 && !ta && tb &&
           matrix_cores_take(ta, tb, epilogue, M, N, K, A, B, C);
}

// What ds_gemm_ws does with a bf16 product of 16-byte aligned operands, for the tests, which want each kernel at its edges: the number
// of launches (0: the plain FMA kernel), and of each its rows, tile (TilePick::kind), splits of the contraction, whole tiles, pieces of
// every other tile, whether it is persistent.  colsum: with the stage's column sums.
extern "C" int32_t ds_gemm_launches(int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, int32_t epilogue, int64_t workspace_floats,
                                    int32_t colsum, int32_t accumulate, int32_t (*out)[6]) {
    if (!matrix_cores_take(ta, tb, epilogue, M, N, K, nullptr, nullptr, nullptr)) return 0;
    if (colsum && !gemm_colsum_fused(DS_DTYPE_BF16, ta, tb, M, N, K, nullptr, nullptr, nullptr, epilogue)) return 0;
    const size_t wsf = (size_t)workspace_floats;
    const Launches l = choose_launches(ta != 0, epilogue, M, N, K, wsf, colsum != 0, accumulate);
    for (int i = 0; i < l.n; ++i) {
        const TilePick& k = l.c[i].pick;
        const BigPlan b = plan_big(ta != 0, epilogue, l.rows[i], N, K, wsf);
        const bool big = k.kind < 0;
        const int32_t v[6] = {l.rows[i], k.kind, big ? b.splits : k.splits, big ? b.n_main : 0, big ? b.tail_splits : 0, big && !ta && nt_persistent(b)};
        for (int e = 0; e < 6; ++e) out[i][e] = v[e];
    }
    return l.n;
}

// Shared with the stage driver.
ds_status launch_gemm(int32_t dtype, int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B,
                      void* C, int32_t epilogue, const GemmEpi& p, bool force_generic, float* split_ws,
                      size_t split_ws_floats, hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0 || !A || !B || !C) return DS_EINVAL;
    if (N % 8) return DS_EINVAL;
    if (dtype != DS_DTYPE_F32 && dtype != DS_DTYPE_BF16) return DS_EINVAL;
    switch (epilogue) {
    case DS_EPI_NONE: return dispatch_epi<DS_EPI_NONE>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_GELU:
        if (!p.C2) return DS_EINVAL;
        return dispatch_epi<DS_EPI_GELU>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_RESID:
        if (!p.R) return DS_EINVAL;
        return dispatch_epi<DS_EPI_RESID>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_GELU_D:
        if (!p.C2) return DS_EINVAL;
        return dispatch_epi<DS_EPI_GELU_D>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_MULR:
        if (!p.R) return DS_EINVAL;
        return dispatch_epi<DS_EPI_MULR>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_DGELU:
        if (!p.R) return DS_EINVAL;
        return dispatch_epi<DS_EPI_DGELU>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_ACC32: return dispatch_epi<DS_EPI_ACC32>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_GATE:
        if (!p.R || !p.C2) return DS_EINVAL;
        return dispatch_epi<DS_EPI_GATE>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    case DS_EPI_DGATE:
        if (!p.R || !p.R2 || !p.C2) return DS_EINVAL;
        return dispatch_epi<DS_EPI_DGATE>(dtype, ta, tb, M, N, K, A, B, C, p, force_generic, split_ws, split_ws_floats, st);
    }
    return DS_EINVAL;
}

// adds up the partial sums of a group's tiles; kFinishParts work-groups per tile, tiles counted over the whole group
constexpr int kFinishParts = 8;
__global__ __launch_bounds__(256) void tn_group_finish_kernel(TnGroup g) {
    int at = blockIdx.x / kFinishParts * g.splits;                                   // work-group number of the tile's first split, were they in turn
    const int i = tn_group_problem(g, at);
    const int N = g.p[i].N, tiles_m = g.p[i].M / BM, tiles_n = N / BN, tile = at / g.splits;
    int tile_m, tile_n;
    nt_tile_coords(tile, tiles_m, tiles_n, tile_m, tile_n);
    float* C = reinterpret_cast<float*>(g.p[i].C);
    GemmEpi p{};
    p.accumulate = g.accumulate;
    for (int e = blockIdx.x % kFinishParts * blockDim.x + threadIdx.x; e < BM * (BN / 8); e += kFinishParts * blockDim.x) {
        const int r = e / (BN / 8), c8 = (e % (BN / 8)) * 8;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = 0.f;
#pragma unroll 4
        for (int sp = 0; sp < g.splits; ++sp) {
            float w[8];
            Vec8<float>::load(g.block(g.first[i] + sp * tiles_m * tiles_n + tile) + (size_t)r * BN + c8, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] += w[j];
        }
        epilogue8<float, DS_EPI_ACC32>(tile_m * BM + r, tile_n * BN + c8, N, v, C, p);
    }
}

ds_status launch_tn_group_big(TnGroup& g, int blocks, hipStream_t st) {
    auto kern = gemm_bf16_nt_kernel<DS_EPI_ACC32, true, false, true>;
    static bool attr_set = false;
    if (!attr_set) {
        DS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, RING));
        attr_set = true;
    }
    GemmEpi p{};
    p.accumulate = g.accumulate;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), RING, st, 0, 0, g.K, (const bf16_t*)nullptr,
                       (const bf16_t*)nullptr, (bf16_t*)nullptr, 0, 0, g.splits, 0, 1, (float*)nullptr, p, 0, (int*)nullptr, g);
    DS_LAUNCH_CHECK();
    if (g.splits > 1) {
        hipLaunchKernelGGL(tn_group_finish_kernel, dim3((unsigned)(blocks / g.splits * kFinishParts)), dim3(256), 0, st, g);
        DS_LAUNCH_CHECK();
    }
    return DS_OK;
}

extern "C" ds_status ds_gemm(int32_t dtype, int32_t trans_a, int32_t trans_b, int32_t M, int32_t N, int32_t K,
                             const void* A, const void* B, void* C, int32_t epilogue, const void* bias, const void* R,
                             const void* R2, void* C2, const int32_t* row_valid, int32_t accumulate,
                             int32_t force_generic, void* hip_stream) {
    GemmEpi p{bias, R, R2, C2, row_valid, accumulate};
    return launch_gemm(dtype, trans_a, trans_b, M, N, K, A, B, C, epilogue, p, force_generic != 0, nullptr, 0,
                       (hipStream_t)hip_stream);
}

extern "C" ds_status ds_gemm_ws(int32_t dtype, int32_t trans_a, int32_t trans_b, int32_t M, int32_t N, int32_t K,
                                const void* A, const void* B, void* C, int32_t epilogue, const void* bias, const void* R,
                                const void* R2, void* C2, const int32_t* row_valid, int32_t accumulate,
                                int32_t force_generic, float* workspace, int64_t workspace_floats, void* hip_stream) {
    if (workspace_floats < 0 || (workspace_floats > 0 && (!workspace || ((uintptr_t)workspace & 15)))) return DS_EINVAL;
    GemmEpi p{bias, R, R2, C2, row_valid, accumulate};
    return launch_gemm(dtype, trans_a, trans_b, M, N, K, A, B, C, epilogue, p, force_generic != 0,
                       workspace_floats > 0 ? workspace : nullptr, (size_t)workspace_floats, (hipStream_t)hip_stream);
}
