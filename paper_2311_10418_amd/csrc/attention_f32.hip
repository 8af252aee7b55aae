// fp32 variable-length attention on the matrix cores (v_mfma_f32_16x16x4_f32), any head size up to 128, causal or
// unmasked, forward and backward.  fp32 operands, products and sums throughout: the probabilities are not rounded.
//
// A wavefront owns 16 "column" items (queries in forward and dQ, keys in dK/dV) and computes TRANSPOSED score blocks: 16
// rows of the other side x its 16 columns, lane = (column lane % 16, rows 4 g + e with g = lane / 16, e = 0..3).  What is
// per column (running maximum and sum, log-sum-exp, delta) is then a per-lane scalar, and register e of a block is, as it
// stands, the B operand of the second product for the contraction step over rows {4 g + e}: probabilities never move.
// Both products read the other side's tile from LDS, token-major, rows of HD + 4 floats: the first product 4 consecutive
// features per lane (float4; 16 rows 4 banks apart cover the 64 banks), the second one float per step (4 rows that lie 4
// rows apart start 16 banks apart).  HD is the head size rounded up to 32, 64, 96 or 128; features beyond it are zeros.
//
// The bound is the fp32 matrix rate: per 16 x 16 block HD/4 MFMAs of 32 cycles for each product (two forward, three in
// dQ, four in dK/dV) against 4 exponentials per lane.  Tiles go global -> registers -> LDS, the next tile's reads in
// flight during the current tile's products; 4 wavefronts per work-group (64 columns), 19 - 54 KB of LDS, so several
// work-groups per CU cover each other's two barriers per tile.  Which work-group does what: see `column_block`.  Measured at
// 7 684 tokens in 64 sequences (up to 512), 4 heads of 64, causal: forward 40 us, dQ with delta 51, dK/dV 56, against 508, 435 and
// 581 for one wavefront per query / key row with shuffled probabilities (attention_generic.hip, which keeps the operands
// that float4 cannot read): those read every row of the other side once per row of this one.
#include "attention_rows.hpp"

namespace {

constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;

__device__ __forceinline__ f32x4_t mfma4(float a, float b, f32x4_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4_t zero4() { f32x4_t z = {0.f, 0.f, 0.f, 0.f}; return z; }

template <int HD, int NT = 256> struct F32Tile {                     // NT threads
    static constexpr int ROWS = HD <= 96 ? 64 : 32;                   // rows of the other side per tile
    static constexpr int LD = HD + 4;
    static constexpr int FLOATS = ROWS * LD;
    static constexpr int NV = ROWS * HD / 4 / NT;                     // float4 per thread
    static_assert(ROWS * HD / 4 % NT == 0, "whole float4s per thread");
    float4 v[NV];
    __device__ __forceinline__ bool not_finite() const {              // any of this thread's values
        float zero = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i)
            zero = __builtin_fmaf(v[i].x, 0.f, __builtin_fmaf(v[i].y, 0.f, __builtin_fmaf(v[i].z, 0.f, __builtin_fmaf(v[i].w, 0.f, zero))));
        return !(zero == 0.f);
    }
    // rows r0 .. r0 + ROWS - 1 of a [n_rows][hd] block with row stride ld; beyond either extent: zeros
    __device__ __forceinline__ void load(const float* __restrict__ src, long long ld, int r0, int n_rows, int hd, int t) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int u = t + NT * i, r = r0 + u / (HD / 4), d = (u % (HD / 4)) * 4;
            v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r < n_rows && d < hd) v[i] = *reinterpret_cast<const float4*>(src + (long long)r * ld + d);
        }
    }
    __device__ __forceinline__ void store(float* tile, int t) const {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int u = t + NT * i;
            *reinterpret_cast<float4*>(tile + (u / (HD / 4)) * LD + (u % (HD / 4)) * 4) = v[i];
        }
    }
};

// this lane's column item: features 16 s + 4 g .. + 3 of `row`
template <int HD>
__device__ __forceinline__ void load_column(const float* __restrict__ row, int hd, int g, float4 (&f)[HD / 16]) {
#pragma unroll
    for (int s = 0; s < HD / 16; ++s) {
        const int d = 16 * s + 4 * g;
        f[s] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (d < hd) f[s] = *reinterpret_cast<const float4*>(row + d);
    }
}

// rows rb .. rb+15 of a tile times this lane's column item, contracted over the features
template <int HD>
__device__ __forceinline__ f32x4_t first_product(const float* tile, int rb, int lane, const float4 (&f)[HD / 16]) {
    const float* p = tile + (rb + (lane & 15)) * F32Tile<HD>::LD + 4 * (lane >> 4);
    f32x4_t acc = zero4();
#pragma unroll
    for (int s = 0; s < HD / 16; ++s) {
        const float4 x = *reinterpret_cast<const float4*>(p + 16 * s);
        acc = mfma4(x.x, f[s].x, acc);
        acc = mfma4(x.y, f[s].y, acc);
        acc = mfma4(x.z, f[s].z, acc);
        acc = mfma4(x.w, f[s].w, acc);
    }
    return acc;
}

// out^T[feature][column] += tile[rows rb .. rb+15]^T * w, w = a 16 x 16 block in score layout
template <int HD>
__device__ __forceinline__ void second_product(const float* tile, int rb, int lane, const f32x4_t& w, f32x4_t (&out)[HD / 16]) {
    const float* p = tile + (rb + 4 * (lane >> 4)) * F32Tile<HD>::LD + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int dt = 0; dt < HD / 16; ++dt) out[dt] = mfma4(p[e * F32Tile<HD>::LD + 16 * dt], w[e], out[dt]);
}

template <int HD>
__device__ __forceinline__ void store_column(const f32x4_t (&acc)[HD / 16], float mul, float* __restrict__ row, int hd, int g) {
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) {
        const int d = 16 * dt + 4 * g;
        if (d < hd) *reinterpret_cast<float4*>(row + d) = make_float4(acc[dt][0] * mul, acc[dt][1] * mul, acc[dt][2] * mul, acc[dt][3] * mul);
    }
}

// largest / sum over the four 16-lane groups, which hold different rows of the same columns
__device__ __forceinline__ float groups_max(float v) { v = fmaxf(v, __shfl_xor(v, 16, 64)); return fmaxf(v, __shfl_xor(v, 32, 64)); }
__device__ __forceinline__ float groups_sum(float v) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); }

// A work-group's 64 columns.  The kernel lasts as long as the compute unit with the longest chains of tiles.  Sequences are taken
// last to first (a plan lists them by ascending length), blocks are the fastest grid dimension, and work-groups go to the eight
// XCDs in turn.
//   dK/dV: the first block of every sequence has the longest chain and goes first, and the number of blocks per grid row is odd: with
//   8 (512 tokens) all of those were on the same XCD.  Backward pass, us, causal: 8 heads of 64, 5 168 tokens in 46 sequences 216 -> 123;
//   4 heads of 32, 14 575 tokens in 133 (16 blocks) 279 -> 120; 2 heads of 128, 7 254 tokens in 40 214 -> 159.
//   Forward and dQ: a causal sequence's last block has the longest chain.  From 640 blocks on (2.5 per CU) they go last to first, in an
//   odd number per grid row as well: forward, us, 8 heads of 64, 15 799 tokens (16 blocks) 176 -> 124; 4 heads of 128 unmasked, 10 673
//   tokens 162 -> 99; 4 heads of 32, 14 575 tokens 62 -> 48.  Below that every block is resident at once, and it counts which other one a
//   long chain shares its CU with: in ascending order the XCD with the last blocks has few others (2 heads of 96, 8 sequences of up to
//   1024: 85 us, 120 last to first in an odd number; 8 heads of 32, 4 sequences of up to 1024: 40 and 48).
//   Over 210 batches (2 to 8 heads, 500 to 16 700 tokens in any order) this takes 0.99 of the time of ascending, even rows forward (9
//   more than 3 % longer, worst 15 %; without the line at 640 36, worst 40 %), and 0.88 backward, delta in the dQ kernel included.
// A stage's sequences come by length: two layers of d = 256, 64 sequences, the same with and without the line (1 115 us).
struct ColumnBlock { int s, h, first; };                              // first < 0: nothing to do

__device__ __forceinline__ ColumnBlock column_block(const AttnArgs& a, const int32_t* __restrict__ len, bool last_first) {
    ColumnBlock c = {a.n_seq - 1 - (int)blockIdx.z, (int)blockIdx.y, -1};
    const int n = (len[c.s] + 63) / 64, b = blockIdx.x;
    if (b < n) c.first = 64 * (last_first ? n - 1 - b : b);
    return c;
}
constexpr int kManyBlocks = 640;
bool many_blocks(const AttnArgs& a) { return (long long)a.n_heads * (a.q_total_rows / 64 + a.n_seq / 2) >= kManyBlocks; }
dim3 column_grid(const AttnArgs& a, int max_len, bool odd) { return dim3((max_len + 63) / 64 | (odd ? 1 : 0), a.n_heads, a.n_seq); }

// Causal masks and values that are not finite.  A score that a column does not see is replaced whatever it is; but the second
// product contracts over whole blocks, with weight 0 for the rows a column does not see, and 0 x Inf would reach it.  So a
// work-group looks at the operand of its second product as it stores the tiles on its diagonal (the positions of its own
// 64 columns; tiles beyond them it does not visit), and if anything there is not finite every wavefront computes its
// columns one at a time in the end (attention_rows.hpp).

// ---------------------------------------------------------------- forward
template <int HD>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(AttnArgs a) {
    typedef F32Tile<HD> Tile;
    constexpr int KT = Tile::ROWS, NB = KT / 16;
    __shared__ __attribute__((aligned(16))) float sK[Tile::FLOATS];
    __shared__ __attribute__((aligned(16))) float sV[Tile::FLOATS];
    __shared__ float s_row[4][HD];
    __shared__ int s_by_rows;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), g = lane >> 4;
    const ColumnBlock cb = column_block(a, a.q_len, a.last_first);
    if (cb.first < 0) return;
    const int s = cb.s, h = cb.h, q0 = cb.first;
    const int ql = a.q_len[s], kl = a.k_len[s], hd = a.head_dim;
    const long long qrow0 = a.q_row[s], krow0 = a.k_row[s];
    const float* K = (const float*)a.k + krow0 * a.ldk + h * hd;
    const float* V = (const float*)a.v + krow0 * a.ldv + h * hd;
    const int qw0 = q0 + wave * 16, qi = qw0 + (lane & 15), qi_c = qi < ql ? qi : ql - 1;
    float4 qf[HD / 16];
    load_column<HD>((const float*)a.q + (qrow0 + qi_c) * a.ldq + h * hd, hd, g, qf);
    f32x4_t oacc[HD / 16];
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) oacc[dt] = zero4();
    const float c = a.scale * kLog2eF;
    float m = -INFINITY, lsum = 0.f;                                  // running maximum (exp2 domain), this lane's part of the sum
    const int kv_end = a.mask ? min(kl, q0 + 64) : kl;
    const int wave_last = a.mask ? min(kl - 1, qw0 + 15) : kl - 1;    // last key this wavefront can see
    if (t == 0) s_by_rows = 0;
    Tile tk, tv;
    if (kv_end > 0) {
        tk.load(K, a.ldk, 0, kl, hd, t);
        tv.load(V, a.ldv, 0, kl, hd, t);
    }
    for (int k0 = 0; k0 < kv_end; k0 += KT) {
        __syncthreads();                                              // the previous tile has been read by everybody
        tk.store(sK, t);
        tv.store(sV, t);
        if (a.mask && k0 >= q0 && tv.not_finite()) s_by_rows = 1;
        __syncthreads();
        if (k0 + KT < kv_end) {
            tk.load(K, a.ldk, k0 + KT, kl, hd, t);
            tv.load(V, a.ldv, k0 + KT, kl, hd, t);
        }
        if (k0 > wave_last || qw0 >= ql) continue;
        f32x4_t sc[NB];
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < NB; ++kt) {
            sc[kt] = first_product<HD>(sK, 16 * kt, lane, qf);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = k0 + 16 * kt + 4 * g + e;
                if (key >= kl || (a.mask && key > qi)) sc[kt][e] = -INFINITY;
                mx = fmaxf(mx, sc[kt][e]);
            }
        }
        const float m_new = fmaxf(m, groups_max(mx) * c);             // finite: every column sees a key of every tile it visits
        const float m_use = m_new == -INFINITY ? 0.f : m_new;         // (a clamped column past the end may see none)
        const float alpha = __builtin_amdgcn_exp2f(m - m_use);
        float rs = 0.f;
#pragma unroll
        for (int kt = 0; kt < NB; ++kt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[kt][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kt][e], c, -m_use));
                rs += sc[kt][e];
            }
        lsum = lsum * alpha + rs;
#pragma unroll
        for (int dt = 0; dt < HD / 16; ++dt)
#pragma unroll
            for (int e = 0; e < 4; ++e) oacc[dt][e] *= alpha;
        m = m_new;
#pragma unroll
        for (int kt = 0; kt < NB; ++kt) second_product<HD>(sV, 16 * kt, lane, sc[kt], oacc);
    }
    if (a.mask && kv_end > 0 && s_by_rows) {
        for (int q = qw0; q < min(qw0 + 16, ql); ++q) {
            wave_lds_sync();
            stage_row(s_row[wave], (const float*)a.q + (qrow0 + q) * a.ldq + h * hd, hd, a.scale, lane);
            wave_lds_sync();
            attn_fwd_row<float>(a, s, h, q, s_row[wave], lane);
        }
        return;
    }
    if (qi >= ql) return;
    const float l = groups_sum(lsum);
    const long long row = qrow0 + qi;
    // (no keys: zero output; every score -Inf: l = 0 and NaN, like the quotient)
    store_column<HD>(oacc, kl > 0 ? 1.0f / l : 0.f, (float*)a.o + row * a.ldo + h * hd, hd, g);
    if (g == 0) a.lse[(size_t)h * a.lse_stride + row] = (m + log2f(l)) * kLn2F;
}

// ---------------------------------------------------------------- backward: dQ
template <int HD>
__global__ __launch_bounds__(256) void attn_bwd_dq_f32_kernel(AttnArgs a) {
    typedef F32Tile<HD> Tile;
    constexpr int KT = Tile::ROWS;
    __shared__ __attribute__((aligned(16))) float sK[Tile::FLOATS];
    __shared__ __attribute__((aligned(16))) float sV[Tile::FLOATS];
    __shared__ float s_row[4][2][HD];
    __shared__ int s_by_rows;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), g = lane >> 4;
    const ColumnBlock cb = column_block(a, a.q_len, a.last_first);
    if (cb.first < 0) return;
    const int s = cb.s, h = cb.h, q0 = cb.first;
    const int ql = a.q_len[s], kl = a.k_len[s], hd = a.head_dim;
    const long long qrow0 = a.q_row[s], krow0 = a.k_row[s];
    const float* K = (const float*)a.k + krow0 * a.ldk + h * hd;
    const float* V = (const float*)a.v + krow0 * a.ldv + h * hd;
    const int qw0 = q0 + wave * 16, qi = qw0 + (lane & 15), qi_c = qi < ql ? qi : ql - 1;
    float4 qf[HD / 16], dof[HD / 16];
    load_column<HD>((const float*)a.q + (qrow0 + qi_c) * a.ldq + h * hd, hd, g, qf);
    load_column<HD>((const float*)a.d_o + (qrow0 + qi_c) * a.ldo + h * hd, hd, g, dof);
    const float lse2 = a.lse[(size_t)h * a.lse_stride + qrow0 + qi_c] * kLog2eF;
    // delta = rowsum(dO * O), for this kernel and, through memory, the dK / dV kernel (a launch of its own took 11.5 us: one wavefront
    // per row and head of the longest sequence for every sequence)
    float delta = 0.f;
    {
        float4 of[HD / 16];
        load_column<HD>((const float*)a.o + (qrow0 + qi_c) * a.ldo + h * hd, hd, g, of);
#pragma unroll
        for (int dt = 0; dt < HD / 16; ++dt)
            delta += (of[dt].x * dof[dt].x + of[dt].y * dof[dt].y) + (of[dt].z * dof[dt].z + of[dt].w * dof[dt].w);
        delta = groups_sum(delta);
        if (g == 0 && qi < ql) a.delta[(size_t)h * a.lse_stride + qrow0 + qi] = delta;
    }
    const float c = a.scale * kLog2eF;
    f32x4_t gacc[HD / 16];
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) gacc[dt] = zero4();
    const int kv_end = a.mask ? min(kl, q0 + 64) : kl;
    const int wave_last = a.mask ? min(kl - 1, qw0 + 15) : kl - 1;
    if (t == 0) s_by_rows = 0;
    Tile tk, tv;
    if (kv_end > 0) {
        tk.load(K, a.ldk, 0, kl, hd, t);
        tv.load(V, a.ldv, 0, kl, hd, t);
    }
    for (int k0 = 0; k0 < kv_end; k0 += KT) {
        __syncthreads();
        tk.store(sK, t);
        tv.store(sV, t);
        if (a.mask && k0 >= q0 && tk.not_finite()) s_by_rows = 1;
        __syncthreads();
        if (k0 + KT < kv_end) {
            tk.load(K, a.ldk, k0 + KT, kl, hd, t);
            tv.load(V, a.ldv, k0 + KT, kl, hd, t);
        }
        if (qw0 >= ql) continue;
#pragma unroll
        for (int kt = 0; kt < KT / 16; ++kt) {
            if (k0 + 16 * kt > wave_last) break;
            f32x4_t ds = first_product<HD>(sK, 16 * kt, lane, qf);
            const f32x4_t dp = first_product<HD>(sV, 16 * kt, lane, dof);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = k0 + 16 * kt + 4 * g + e;
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(ds[e], c, -lse2));
                ds[e] = (key >= kl || (a.mask && key > qi)) ? 0.f : p * (dp[e] - delta);
            }
            second_product<HD>(sK, 16 * kt, lane, ds, gacc);
        }
    }
    if (a.mask && kv_end > 0 && s_by_rows) {
        __threadfence_block();                          // (delta, read back by other lanes)
        for (int q = qw0; q < min(qw0 + 16, ql); ++q) {
            wave_lds_sync();
            stage_row(s_row[wave][0], (const float*)a.q + (qrow0 + q) * a.ldq + h * hd, hd, a.scale, lane);
            stage_row(s_row[wave][1], (const float*)a.d_o + (qrow0 + q) * a.ldo + h * hd, hd, 1.0f, lane);
            wave_lds_sync();
            attn_bwd_dq_row<float>(a, s, h, q, s_row[wave][0], s_row[wave][1], lane);
        }
        return;
    }
    if (qi < ql) store_column<HD>(gacc, a.scale, (float*)a.dq + (qrow0 + qi) * a.ldq + h * hd, hd, g);
}

// ---------------------------------------------------------------- backward: dK, dV
// Eight wavefronts: the first key blocks of a long causal sequence meet every query, and their work-groups set the
// kernel's length.  Wavefronts w and w + 4 own the same 16 keys and take alternate 16-query blocks of every tile; their
// accumulators are added through LDS at the end.  116 us with four wavefronts, 107 with eight, 86 with at most 128
// registers (head size up to 64: two work-groups per CU), all three with eight blocks to a grid row.  At head size 64 it takes 127;
// the other two kernels need 20 to 35 more than 128 there and lose with that limit (dQ 53 us instead of 42).
template <int HD>
__global__ __launch_bounds__(512, HD <= 64 ? 4 : 2) void attn_bwd_dkv_f32_kernel(AttnArgs a) {
    typedef F32Tile<HD, 512> Tile;
    constexpr int QT = Tile::ROWS;
    __shared__ __attribute__((aligned(16))) float smem[2 * Tile::FLOATS];
    static_assert(2 * Tile::FLOATS >= HD / 16 * 4 * 256, "one set of accumulators fits in the tiles");
    float* sQ = smem;
    float* sO = smem + Tile::FLOATS;
    __shared__ __attribute__((aligned(16))) float s_lse[QT], s_delta[QT];
    __shared__ float s_row[4][2][HD];
    __shared__ int s_by_rows;
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6) & 3, half = __builtin_amdgcn_readfirstlane(t >> 8);
    const ColumnBlock cb = column_block(a, a.k_len, false);
    if (cb.first < 0) return;
    const int s = cb.s, h = cb.h, k0 = cb.first;
    const int ql = a.q_len[s], kl = a.k_len[s], hd = a.head_dim;
    const long long qrow0 = a.q_row[s], krow0 = a.k_row[s];
    const float* Q = (const float*)a.q + qrow0 * a.ldq + h * hd;
    const float* dO = (const float*)a.d_o + qrow0 * a.ldo + h * hd;
    const float* lse = a.lse + (size_t)h * a.lse_stride + qrow0;
    const float* delta = a.delta + (size_t)h * a.lse_stride + qrow0;
    const int kw0 = k0 + wave * 16, ki = kw0 + (lane & 15), ki_c = ki < kl ? ki : kl - 1;
    float4 kf[HD / 16], vf[HD / 16];
    load_column<HD>((const float*)a.k + (krow0 + ki_c) * a.ldk + h * hd, hd, g, kf);
    load_column<HD>((const float*)a.v + (krow0 + ki_c) * a.ldv + h * hd, hd, g, vf);
    const float c = a.scale * kLog2eF;
    f32x4_t dkacc[HD / 16], dvacc[HD / 16];
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt) { dkacc[dt] = zero4(); dvacc[dt] = zero4(); }
    const int q_begin = a.mask ? k0 : 0;                              // causal: only queries at or after the key see it
    if (t == 0) s_by_rows = 0;
    Tile tq, to;
    float lse_r = 0.f, delta_r = 0.f;
    auto fetch = [&](int q0) {
        tq.load(Q, a.ldq, q0, ql, hd, t);
        to.load(dO, a.ldo, q0, ql, hd, t);
        const bool in = t < QT && q0 + t < ql;
        lse_r = in ? lse[q0 + t] * kLog2eF : 0.f;
        delta_r = in ? delta[q0 + t] : 0.f;
    };
    if (q_begin < ql) fetch(q_begin);
    for (int q0 = q_begin; q0 < ql; q0 += QT) {
        __syncthreads();
        tq.store(sQ, t);
        to.store(sO, t);
        if (a.mask && q0 < k0 + 64 && (tq.not_finite() || to.not_finite())) s_by_rows = 1;
        if (t < QT) { s_lse[t] = lse_r; s_delta[t] = delta_r; }
        __syncthreads();
        if (q0 + QT < ql) fetch(q0 + QT);
        if (kw0 >= kl) continue;
#pragma unroll
        for (int qt2 = 0; qt2 < QT / 32; ++qt2) {
            const int qt = 2 * qt2 + half;
            const int qb = q0 + 16 * qt;
            if (qb >= ql || (a.mask && qb + 15 < kw0)) continue;      // no visible query
            f32x4_t p = first_product<HD>(sQ, 16 * qt, lane, kf);
            f32x4_t ds = first_product<HD>(sO, 16 * qt, lane, vf);
            const float4 l4 = *reinterpret_cast<const float4*>(s_lse + 16 * qt + 4 * g);
            const float4 d4 = *reinterpret_cast<const float4*>(s_delta + 16 * qt + 4 * g);
            const float lq[4] = {l4.x, l4.y, l4.z, l4.w}, dq[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int q = qb + 4 * g + e;
                const bool out = q >= ql || (a.mask && q < ki);
                p[e] = out ? 0.f : __builtin_amdgcn_exp2f(__builtin_fmaf(p[e], c, -lq[e]));
                ds[e] = out ? 0.f : p[e] * (ds[e] - dq[e]);
            }
            second_product<HD>(sO, 16 * qt, lane, p, dvacc);
            second_product<HD>(sQ, 16 * qt, lane, ds, dkacc);
        }
    }
    f32x4_t* part = reinterpret_cast<f32x4_t*>(smem);                 // [HD / 16][256], dK then dV
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        f32x4_t (&acc)[HD / 16] = pass ? dvacc : dkacc;
        __syncthreads();
        if (half == 1) {
#pragma unroll
            for (int dt = 0; dt < HD / 16; ++dt) part[dt * 256 + (t & 255)] = acc[dt];
        }
        __syncthreads();
        if (half == 0) {
#pragma unroll
            for (int dt = 0; dt < HD / 16; ++dt) acc[dt] += part[dt * 256 + t];
        }
    }
    if (half == 1) return;
    if (s_by_rows) {
        for (int k = kw0; k < min(kw0 + 16, kl); ++k) {
            wave_lds_sync();
            stage_row(s_row[wave][0], (const float*)a.k + (krow0 + k) * a.ldk + h * hd, hd, a.scale, lane);
            stage_row(s_row[wave][1], (const float*)a.v + (krow0 + k) * a.ldv + h * hd, hd, 1.0f, lane);
            wave_lds_sync();
            attn_bwd_dkv_row<float>(a, s, h, k, s_row[wave][0], s_row[wave][1], lane);
        }
        return;
    }
    if (ki >= kl) return;
    store_column<HD>(dkacc, a.scale, (float*)a.dk + (krow0 + ki) * a.ldk + h * hd, hd, g);
    store_column<HD>(dvacc, 1.0f, (float*)a.dv + (krow0 + ki) * a.ldv + h * hd, hd, g);
}

template <int HD>
ds_status bwd_f32(AttnArgs a, hipStream_t st) {
    const bool many = many_blocks(a);
    a.last_first = a.mask && many;
    hipLaunchKernelGGL(attn_bwd_dq_f32_kernel<HD>, column_grid(a, a.max_q_len, many), dim3(256), 0, st, a);
    DS_LAUNCH_CHECK();
    hipLaunchKernelGGL(attn_bwd_dkv_f32_kernel<HD>, column_grid(a, a.max_k_len, true), dim3(512), 0, st, a);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

}  // namespace

// What the float4 accesses need; everything else (strides not a multiple of 4, unaligned tensors) keeps the generic kernels.
bool attn_f32_mfma_supported(const AttnArgs& a) {
    if (a.dtype != DS_DTYPE_F32) return false;
    if (a.ldq % 4 || a.ldk % 4 || a.ldv % 4 || a.ldo % 4) return false;
    auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
    if (!al(a.q) || !al(a.k) || !al(a.v) || !al(a.o)) return false;
    return !a.d_o || (al(a.d_o) && al(a.dq) && al(a.dk) && al(a.dv));
}

ds_status attn_fwd_f32_mfma(const AttnArgs& args, hipStream_t st) {
    AttnArgs a = args;
    const bool many = many_blocks(a);
    a.last_first = a.mask && many;
    const dim3 grid = column_grid(a, a.max_q_len, many);
    if (a.head_dim <= 32) hipLaunchKernelGGL(attn_fwd_f32_kernel<32>, grid, dim3(256), 0, st, a);
    else if (a.head_dim <= 64) hipLaunchKernelGGL(attn_fwd_f32_kernel<64>, grid, dim3(256), 0, st, a);
    else if (a.head_dim <= 96) hipLaunchKernelGGL(attn_fwd_f32_kernel<96>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(attn_fwd_f32_kernel<128>, grid, dim3(256), 0, st, a);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status attn_bwd_f32_mfma(const AttnArgs& a, hipStream_t st) {
    if (a.head_dim <= 32) return bwd_f32<32>(a, st);
    if (a.head_dim <= 64) return bwd_f32<64>(a, st);
    if (a.head_dim <= 96) return bwd_f32<96>(a, st);
    return bwd_f32<128>(a, st);
}
