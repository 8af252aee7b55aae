// HBM-bound kernels of the stage: row masking / gathering, LayerNorm and RMSNorm forward and
// backward, column sums (bias gradients).  One 64-lane wavefront owns one row; row reductions
// use wavefront shuffles; every global access is a 16-byte (bf16) or 32-byte (fp32) vector
// per lane, consecutive lanes touching consecutive addresses.
#include "common.hpp"

#include <algorithm>
#include <mutex>

namespace {

constexpr int kPartialRows = 2048;   // upper bound on partial-sum rows written by column reductions

// Partial column sums of ds_colsum_static: 4 MiB of device memory per GPU for the life of the process.  In host code
// this name is only a handle for hipGetSymbolAddress; kernels get the per-device address it returns.
constexpr int kStaticFloats = 1 << 20;
constexpr int kStaticMaxCols = 65536;
constexpr int kMaxDevices = 64;
__device__ __align__(256) float g_colsum_scratch[kStaticFloats];
float* g_colsum_scratch_ptr[kMaxDevices];        // device address of the array on each GPU; null until first used there
std::mutex g_colsum_scratch_mutex;

// ------------------------------------------------------------------ row copy kernels
// blockIdx.y = tensor
template <class T>
__global__ __launch_bounds__(256) void mask_rows_kernel(MaskBatch b, int d8) {
    const int k = blockIdx.y;
    const T* __restrict__ in = reinterpret_cast<const T*>(b.in[k]);
    T* __restrict__ out = reinterpret_cast<T*>(b.out[k]);
    const int32_t* __restrict__ row_valid = b.row_valid[k];
    const long long total = (long long)b.rows[k] * d8;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        float v[8];
        if (row_valid[(int)(i / d8)] >= 0) {
            Vec8<T>::load(in + i * 8, v);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = 0.f;
        }
        Vec8<T>::store(out + i * 8, v);
    }
}

// blockIdx.y = buffer; one wavefront per row; only padding rows are written
__global__ __launch_bounds__(256) void zero_pad_rows_kernel(ZeroPadBatch b, int rows, const int32_t* __restrict__ row_valid) {
    const int w = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
    const int nw = (gridDim.x * blockDim.x) >> 6;
    const int row16 = b.row_bytes[blockIdx.y] / 16;
    uint4* buf = static_cast<uint4*>(b.buf[blockIdx.y]);
    for (int r = w; r < rows; r += nw) {
        if (row_valid[r] >= 0) continue;
        uint4* p = buf + (size_t)r * row16;
        for (int c = lane; c < row16; c += 64) p[c] = make_uint4(0u, 0u, 0u, 0u);
    }
}

// Rows of a padded stream <-> sequences back to back.  The segments (a sequence's rows, then padding up to the next one) are
// kernel arguments, so that nothing is allocated or uploaded; each wavefront moves one stream row with 16-byte accesses,
// four in flight.  Bound by memory: pack and unpack of 65 536 tokens, d = 2048, bf16: 237 us for 1.07 GB (with a row map
// built on the host, allocated, uploaded and freed per call: 253); 16 rows per work-group instead of 4: 246 (a last round
// of work-groups that leaves most of the chip idle).
constexpr int kMoveRows = 4;
template <bool TO_STREAM>
__global__ __launch_bounds__(256) void move_rows_kernel(RowSegments b, int row16, const uint4* __restrict__ in, uint4* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = b.row[0] + (int)blockIdx.x * kMoveRows;
    int lo = 0, hi = b.n;                               // the last segment that starts at or before r0
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (b.row[mid] <= r0) lo = mid;
        else hi = mid;
    }
    const int r = r0 + wave;
    if (r < b.end) {
        while (lo + 1 < b.n && b.row[lo + 1] <= r) ++lo;
        const int at = r - b.row[lo];
        if (at < b.len[lo]) {
            const size_t s = (size_t)r * row16, c = ((size_t)b.canon[lo] + at) * row16;
            const uint4* src = in + (TO_STREAM ? c : s);
            uint4* dst = out + (TO_STREAM ? s : c);
            int i = lane;
            for (; i + 192 < row16; i += 256) {         // four accesses in flight
                const uint4 x0 = src[i], x1 = src[i + 64], x2 = src[i + 128], x3 = src[i + 192];
                dst[i] = x0;
                dst[i + 64] = x1;
                dst[i + 128] = x2;
                dst[i + 192] = x3;
            }
            for (; i < row16; i += 64) dst[i] = src[i];
        } else if (TO_STREAM) {
            for (int i = lane; i < row16; i += 64) out[(size_t)r * row16 + i] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
}

// The same with the row map in memory, for streams of many sequences: a thread moves one 16-byte piece (1024 pieces per
// work-group, four in flight per thread, take 6 % longer at d = 1024), so that short rows leave no lane idle.
template <bool TO_STREAM>
__global__ __launch_bounds__(256) void move_rows_map_kernel(int rows, const int32_t* __restrict__ map, int row16,
                                                            const uint4* __restrict__ in, uint4* __restrict__ out) {
    const size_t s = (size_t)blockIdx.x * 256 + threadIdx.x, r = s / (unsigned)row16;
    if (r >= (size_t)rows) return;
    const int32_t m = map[r];
    const size_t c = (size_t)m * row16 + (s - r * row16);
    if (TO_STREAM) out[s] = m >= 0 ? in[c] : make_uint4(0u, 0u, 0u, 0u);
    else if (m >= 0) out[c] = in[s];
}

// ------------------------------------------------------------------ bf16 transpose
// out[c][r] = in[r][c] for up to kTransposeBatch matrices in one launch (the weight copies of a stage: one launch of a few
// microseconds per matrix is mostly launch).  One wavefront per 64x64 tile as 8x8 blocks of 8x8 elements: each lane loads
// 8 rows of 16 bytes, transposes them in registers (v_perm_b32) and stores 8 rows of 16 bytes; lanes are arranged 8x8 so
// that both the loads and the stores form 128-byte contiguous segments.  No LDS.
__global__ __launch_bounds__(256) void transpose_bf16_kernel(TransposeBatch b) {
    int i = 0;
    while (i + 1 < b.n && (int)blockIdx.x >= b.first_block[i + 1]) ++i;
    const bf16_t* in = static_cast<const bf16_t*>(b.in[i]);
    bf16_t* out = static_cast<bf16_t*>(b.out[i]);
    const int rows = b.rows[i], cols = b.cols[i];
    const int block = blockIdx.x - b.first_block[i], gx = (cols + 63) / 64;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int bx = lane & 7, by = lane >> 3;
    const int c0 = (block % gx) * 64 + bx * 8;
    const int r0 = ((block / gx) * 4 + wave) * 64 + by * 8;
    if (r0 >= rows || c0 >= cols) return;
    uint32_t v[8][4];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint4 x = *reinterpret_cast<const uint4*>(in + (size_t)(r0 + k) * cols + c0);
        v[k][0] = x.x; v[k][1] = x.y; v[k][2] = x.z; v[k][3] = x.w;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {          // output row c0+k gathers element k of the 8 loaded rows
        const uint32_t sel = (k & 1) ? 0x07060302u : 0x05040100u;
        const int w = k >> 1;
        uint4 o;
        o.x = __builtin_amdgcn_perm(v[1][w], v[0][w], sel);
        o.y = __builtin_amdgcn_perm(v[3][w], v[2][w], sel);
        o.z = __builtin_amdgcn_perm(v[5][w], v[4][w], sel);
        o.w = __builtin_amdgcn_perm(v[7][w], v[6][w], sel);
        *reinterpret_cast<uint4*>(out + (size_t)(c0 + k) * rows + r0) = o;
    }
}

inline int grid_for(long long work_items, int block) {
    long long g = (work_items + block - 1) / block;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

// ------------------------------------------------------------------ norm forward
// stats[0..rows) = mean (LayerNorm) or unused (RMS); stats[rows..2rows) = rstd.
template <class T, bool RMS, int NI>
__global__ __launch_bounds__(256) void norm_fwd_kernel(int rows, int d, const T* __restrict__ x, const T* __restrict__ g,
                                                       const T* __restrict__ b, T* __restrict__ y, float* __restrict__ stats) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const T* xr = x + (size_t)row * d;
    float v[NI][8];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = (lane + 64 * i) * 8;
        if (col < d) {
            Vec8<T>::load(xr + col, v[i]);
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[i][j];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[i][j] = 0.f;
        }
    }
    const float inv_d = 1.0f / (float)d;
    const float mean = RMS ? 0.f : wave_sum(s) * inv_d;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = (lane + 64 * i) * 8;
        if (col < d) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float t = v[i][j] - mean;
                q += t * t;
            }
        }
    }
    q = wave_sum(q) * inv_d;
    const float rstd = 1.0f / sqrtf(q + (RMS ? kRmsEps : kLnEps));
    T* yr = y + (size_t)row * d;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = (lane + 64 * i) * 8;
        if (col < d) {
            float gg[8], bb[8], o[8];
            Vec8<T>::load(g + col, gg);
            if (!RMS) Vec8<T>::load(b + col, bb);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float xh = (v[i][j] - mean) * rstd;
                o[j] = RMS ? xh * gg[j] : xh * gg[j] + bb[j];
            }
            Vec8<T>::store(yr + col, o);
        }
    }
    if (lane == 0) {
        stats[row] = mean;
        stats[rows + row] = rstd;
    }
}

// Wide rows (2048 < d <= 4096): one row per work-group of NW wavefronts, each owning d / NW of the columns.  With one
// wavefront per row a lane holds 64 values and the kernel runs at 4.4 TB/s (LayerNorm, d = 4096); at 32 values per
// lane twice as many wavefronts fit and the loads of more rows are in flight: 5.2 TB/s, RMSNorm 5.8.  The two row
// sums (mean, then centred variance: the same two-pass arithmetic as above) are exchanged through LDS (double-buffered
// by row parity should a work-group take more than one row: two barriers per row).
template <class T, bool RMS, int NI, int NW>
__global__ __launch_bounds__(64 * NW) void norm_fwd_multi_kernel(int rows, int d, const T* __restrict__ x, const T* __restrict__ g,
                                                                 const T* __restrict__ b, T* __restrict__ y, float* __restrict__ stats) {
    __shared__ float red_s[2][NW], red_q[2][NW];
    const int part = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int hd = d / NW, c0 = part * hd;
    const float inv_d = 1.0f / (float)d;
    int par = 0;
    for (int row = blockIdx.x; row < rows; row += gridDim.x, par ^= 1) {      // all wavefronts: the same rows
        const T* xr = x + (size_t)row * d + c0;
        float v[NI][8];
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < hd) {
                Vec8<T>::load(xr + col, v[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) s += v[i][j];
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[i][j] = 0.f;
            }
        }
        float mean = 0.f;
        if (!RMS) {
            s = wave_sum(s);
            if (lane == 0) red_s[par][part] = s;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) mean += red_s[par][w];                // the same order in every wavefront
            mean *= inv_d;
        }
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < hd) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float t = v[i][j] - mean;
                    q += t * t;
                }
            }
        }
        q = wave_sum(q);
        if (lane == 0) red_q[par][part] = q;
        __syncthreads();
        q = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) q += red_q[par][w];
        q *= inv_d;
        const float rstd = 1.0f / sqrtf(q + (RMS ? kRmsEps : kLnEps));
        T* yr = y + (size_t)row * d + c0;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < hd) {
                float gg[8], bb[8], o[8];
                Vec8<T>::load(g + c0 + col, gg);
                if (!RMS) Vec8<T>::load(b + c0 + col, bb);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float xh = (v[i][j] - mean) * rstd;
                    o[j] = RMS ? xh * gg[j] : xh * gg[j] + bb[j];
                }
                Vec8<T>::store(yr + col, o);
            }
        }
        if (threadIdx.x == 0) {
            stats[row] = mean;
            stats[rows + row] = rstd;
        }
    }
}

// ------------------------------------------------------------------ norm backward
// dx = resid + rstd * (dy*g - mean(dy*g) - xhat * mean(dy*g*xhat))    (RMS: no mean(dy*g) term)
// partial[b][0][:] = sum over the rows work-group b handled of dy*xhat, partial[b][1][:] = sum of dy.
template <class T, bool RMS, int NI>
__global__ __launch_bounds__(256) void norm_bwd_kernel(int rows, int d, const T* __restrict__ dy, const T* __restrict__ x,
                                                       const T* __restrict__ g, const float* __restrict__ stats,
                                                       const T* __restrict__ resid, T* __restrict__ dx,
                                                       float* __restrict__ partial) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int gw = blockIdx.x * 4 + wave;
    const int nw = gridDim.x * 4;
    float gg[NI][8], dg[NI][8], db[NI][8];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = (lane + 64 * i) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) { dg[i][j] = 0.f; db[i][j] = 0.f; gg[i][j] = 0.f; }
        if (col < d) Vec8<T>::load(g + col, gg[i]);
    }
    const float inv_d = 1.0f / (float)d;
    for (int row = gw; row < rows; row += nw) {
        const float mean = RMS ? 0.f : stats[row];
        const float rstd = stats[rows + row];
        const T* dyr = dy + (size_t)row * d;
        const T* xr = x + (size_t)row * d;
        float a[NI][8], xh[NI][8];
        float c1 = 0.f, c2 = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < d) {
                Vec8<T>::load(dyr + col, a[i]);
                Vec8<T>::load(xr + col, xh[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    xh[i][j] = (xh[i][j] - mean) * rstd;
                    dg[i][j] += a[i][j] * xh[i][j];
                    db[i][j] += a[i][j];
                    a[i][j] *= gg[i][j];
                    c1 += a[i][j];
                    c2 += a[i][j] * xh[i][j];
                }
            }
        }
        c1 = RMS ? 0.f : wave_sum(c1) * inv_d;
        c2 = wave_sum(c2) * inv_d;
        T* dxr = dx + (size_t)row * d;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < d) {
                float o[8];
                if (resid) {
                    Vec8<T>::load(resid + (size_t)row * d + col, o);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) o[j] = 0.f;
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] += rstd * (a[i][j] - c1 - xh[i][j] * c2);
                Vec8<T>::store(dxr + col, o);
            }
        }
    }
    // the four wavefronts' sums are added here, so that one partial row per work-group is left to the second kernel
    __shared__ __attribute__((aligned(16))) float red[4][64 * 8];
    float* p0 = partial + (size_t)blockIdx.x * 2 * d;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int k = 0; k < (RMS ? 1 : 2); ++k) {
            Vec8<float>::store(&red[wave][lane * 8], k ? db[i] : dg[i]);
            __syncthreads();
            const int c = threadIdx.x * 2, col = 64 * 8 * i + c;
            if (col < d) {
                float2 v = *reinterpret_cast<const float2*>(&red[0][c]);
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float2 x = *reinterpret_cast<const float2*>(&red[w][c]);
                    v.x += x.x;
                    v.y += x.y;
                }
                *reinterpret_cast<float2*>(p0 + (size_t)k * d + col) = v;
            }
            __syncthreads();
        }
}

// Wide rows (d > 1024): one row per group of NW = 2 or 4 wavefronts (one work-group), each owning d / NW of the
// columns, so that the per-lane state (gain, dgamma / dbeta sums, dy * g, xhat: 5 x 8 x NI floats) leaves room for
// four wavefronts per SIMD; with one wavefront per row of 4096 columns it needs more than 256 registers and the
// kernel runs at half the memory rate.  The partial row sums are exchanged through LDS (double-buffered by row
// parity: one barrier per row).  partial[group][0][:] / [1][:] as above; a group writes all slices of its partial row.
template <class T, bool RMS, int NI, int NW>
__global__ __launch_bounds__(64 * NW) void norm_bwd_multi_kernel(int rows, int d, const T* __restrict__ dy, const T* __restrict__ x,
                                                                 const T* __restrict__ g, const float* __restrict__ stats,
                                                                 const T* __restrict__ resid, T* __restrict__ dx,
                                                                 float* __restrict__ partial) {
    __shared__ float red[2][NW][2];
    const int part = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int hd = d / NW, c0 = part * hd;
    float gg[NI][8], dg[NI][8], db[NI][8];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = (lane + 64 * i) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) { dg[i][j] = 0.f; db[i][j] = 0.f; gg[i][j] = 0.f; }
        if (col < hd) Vec8<T>::load(g + c0 + col, gg[i]);
    }
    const float inv_d = 1.0f / (float)d;
    int par = 0;
    for (int row = blockIdx.x; row < rows; row += gridDim.x, par ^= 1) {      // all wavefronts: the same rows
        const float mean = RMS ? 0.f : stats[row];
        const float rstd = stats[rows + row];
        const T* dyr = dy + (size_t)row * d + c0;
        const T* xr = x + (size_t)row * d + c0;
        float a[NI][8], xh[NI][8];
        float c1 = 0.f, c2 = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < hd) {
                Vec8<T>::load(dyr + col, a[i]);
                Vec8<T>::load(xr + col, xh[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    xh[i][j] = (xh[i][j] - mean) * rstd;
                    dg[i][j] += a[i][j] * xh[i][j];
                    db[i][j] += a[i][j];
                    a[i][j] *= gg[i][j];
                    c1 += a[i][j];
                    c2 += a[i][j] * xh[i][j];
                }
            }
        }
        c1 = wave_sum(c1);
        c2 = wave_sum(c2);
        if (lane == 0) { red[par][part][0] = c1; red[par][part][1] = c2; }
        __syncthreads();
        c1 = 0.f;
        c2 = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) { c1 += red[par][w][0]; c2 += red[par][w][1]; }    // the same order in every wavefront
        c1 = RMS ? 0.f : c1 * inv_d;
        c2 *= inv_d;
        T* dxr = dx + (size_t)row * d + c0;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int col = (lane + 64 * i) * 8;
            if (col < hd) {
                float o[8];
                if (resid) {
                    Vec8<T>::load(resid + (size_t)row * d + c0 + col, o);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) o[j] = 0.f;
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] += rstd * (a[i][j] - c1 - xh[i][j] * c2);
                Vec8<T>::store(dxr + col, o);
            }
        }
    }
    float* p0 = partial + (size_t)blockIdx.x * 2 * d + c0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int col = (lane + 64 * i) * 8;
        if (col < hd) {
            Vec8<float>::store(p0 + col, dg[i]);
            if (!RMS) Vec8<float>::store(p0 + d + col, db[i]);
        }
    }
}

// out[c] = (accumulate ? out[c] : 0) + sum_p partial[p * stride + c].  A work-group owns 32 columns: 8 lanes of float4 (one
// 128-byte line per partial row) by NT / 8 row lanes, four rows in flight per lane; a wavefront folds its 8 row lanes
// with shuffles, the wavefronts meet in LDS.  Fixed order of additions for a given (n_partial, n).
// blockIdx.y = 1 (when launched with two rows of blocks) reduces a second set of partials into out2.
// What bounds it is the latency of the chain of loads, not the bytes: with 8 row lanes of single floats, as before, a sum
// of 2048 rows of 256 columns (512 loads one after another, on 8 work-groups) took 22 us.
template <int NT>
__global__ __launch_bounds__(NT) void reduce_partials_kernel(int n_partial, int n, size_t stride,
                                                             const float* __restrict__ partial,
                                                             float* __restrict__ out, int accumulate,
                                                             const float* __restrict__ partial2, float* __restrict__ out2) {
    constexpr int RL = NT / 8;
    __shared__ float red[NT / 64][32];
    if (blockIdx.y == 1) {
        partial = partial2;
        out = out2;
    }
    const int cx = threadIdx.x & 7, ry = threadIdx.x >> 3;
    const int col = blockIdx.x * 32 + cx * 4;                         // n is a multiple of 8
    f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0, s2 = s0, s3 = s0;
    if (col < n) {
        const float* src = partial + col;
        int p = ry;
        for (; p + 3 * RL < n_partial; p += 4 * RL) {
            s0 += *reinterpret_cast<const f32x4_t*>(src + (size_t)p * stride);
            s1 += *reinterpret_cast<const f32x4_t*>(src + (size_t)(p + RL) * stride);
            s2 += *reinterpret_cast<const f32x4_t*>(src + (size_t)(p + 2 * RL) * stride);
            s3 += *reinterpret_cast<const f32x4_t*>(src + (size_t)(p + 3 * RL) * stride);
        }
        for (; p < n_partial; p += RL) s0 += *reinterpret_cast<const f32x4_t*>(src + (size_t)p * stride);
    }
    s0 = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int o = 8; o < 64; o <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) s0[e] += __shfl_xor(s0[e], o, 64);
    if ((threadIdx.x & 63) < 8) *reinterpret_cast<f32x4_t*>(&red[threadIdx.x >> 6][cx * 4]) = s0;
    __syncthreads();
    const int c = blockIdx.x * 32 + threadIdx.x;
    if (threadIdx.x < 32 && c < n) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) s += red[k][threadIdx.x];
        out[c] = accumulate ? out[c] + s : s;
    }
}

// out2 != nullptr: a second set of partials (same count and stride) is reduced into it by the same launch.
// wide: work-groups of 1024 threads for long sums.  Not for column sums, which may run beside a GEMM on another stream: a
// resident GEMM work-group leaves registers for one small wavefront per SIMD, not for four, and a wide work-group would
// wait for it to end (380 us instead of 15 at 65 536 tokens).
ds_status reduce_launch(int n_partial, int n, size_t stride, const float* partial, float* out, int accumulate,
                        const float* partial2, float* out2, bool wide, hipStream_t st) {
    const dim3 grid((n + 31) / 32, out2 ? 2 : 1);
    if (wide && n_partial > 256)
        hipLaunchKernelGGL(reduce_partials_kernel<1024>, grid, dim3(1024), 0, st, n_partial, n, stride, partial, out, accumulate, partial2, out2);
    else
        hipLaunchKernelGGL(reduce_partials_kernel<256>, grid, dim3(256), 0, st, n_partial, n, stride, partial, out, accumulate, partial2, out2);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

// ------------------------------------------------------------------ column sums
// block (64, 4): thread (tx, ty) owns 8 columns, rows blockIdx.y*4+ty, stepping gridDim.y*4.
template <class T>
__global__ __launch_bounds__(256) void colsum_kernel(int rows, int n, const T* __restrict__ x, float* __restrict__ partial) {
    __shared__ float red[4][64][9];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int col = (blockIdx.x * 64 + tx) * 8;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    if (col < n) {
        // four rows in flight per wavefront
        const int step = gridDim.y * 4;
        int r = blockIdx.y * 4 + ty;
        for (; r < rows - 3 * step; r += 4 * step) {
            float v[4][8];
#pragma unroll
            for (int k = 0; k < 4; ++k) Vec8<T>::load(x + (size_t)(r + k * step) * n + col, v[k]);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (v[0][j] + v[1][j]) + (v[2][j] + v[3][j]);
        }
        for (; r < rows; r += step) {
            float v[8];
            Vec8<T>::load(x + (size_t)r * n + col, v);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += v[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[ty][tx][j] = acc[j];
    __syncthreads();
    if (ty == 0 && col < n) {
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = red[0][tx][j] + red[1][tx][j] + red[2][tx][j] + red[3][tx][j];
        Vec8<float>::store(partial + (size_t)blockIdx.y * n + col, o);
    }
}

// Few rows: one launch.  A work-group owns 32 columns (4 lanes of 8) and all rows, 64 row lanes.
template <class T>
__global__ __launch_bounds__(256) void colsum_small_kernel(int rows, int n, const T* __restrict__ x, float* __restrict__ out, int accumulate) {
    __shared__ float red[4][32];
    const int cx = threadIdx.x & 3, ry = threadIdx.x >> 2;
    const int col = blockIdx.x * 32 + cx * 8;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    if (col < n)
        for (int r = ry; r < rows; r += 64) {
            float v[8];
            Vec8<T>::load(x + (size_t)r * n + col, v);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += v[j];
        }
#pragma unroll
    for (int o = 4; o < 64; o <<= 1)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += __shfl_xor(acc[j], o, 64);
    if ((threadIdx.x & 63) < 4) {
#pragma unroll
        for (int j = 0; j < 8; ++j) red[threadIdx.x >> 6][cx * 8 + j] = acc[j];
    }
    __syncthreads();
    const int c = blockIdx.x * 32 + threadIdx.x;
    if (threadIdx.x < 32 && c < n) {
        const float s = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
        out[c] = accumulate ? out[c] + s : s;
    }
}

template <class T, bool RMS>
ds_status norm_fwd_dispatch(int rows, int d, const T* x, const T* g, const T* b, T* y, float* stats, hipStream_t st) {
    const int ni = (d + 511) / 512;
    if (ni > 4 && d % 16 == 0) {                 // wide rows: two wavefronts per row (see norm_fwd_multi_kernel)
        // one work-group per row: measured best (a grid striding over the rows with 16 K or 4 K work-groups is 6 - 30 % slower)
        hipLaunchKernelGGL((norm_fwd_multi_kernel<T, RMS, 4, 2>), dim3(rows), dim3(128), 0, st, rows, d, x, g, b, y, stats);
        DS_LAUNCH_CHECK();
        return DS_OK;
    }
    dim3 grid((rows + 3) / 4), block(256);
    if (ni <= 1) hipLaunchKernelGGL((norm_fwd_kernel<T, RMS, 1>), grid, block, 0, st, rows, d, x, g, b, y, stats);
    else if (ni <= 2) hipLaunchKernelGGL((norm_fwd_kernel<T, RMS, 2>), grid, block, 0, st, rows, d, x, g, b, y, stats);
    else if (ni <= 4) hipLaunchKernelGGL((norm_fwd_kernel<T, RMS, 4>), grid, block, 0, st, rows, d, x, g, b, y, stats);
    else hipLaunchKernelGGL((norm_fwd_kernel<T, RMS, 8>), grid, block, 0, st, rows, d, x, g, b, y, stats);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

// Work-groups of the norm backward kernels, each of which leaves one partial row of 2 d floats.
int norm_bwd_groups(int rows, int d) {
    if (d > 1024 && d % 32 == 0) {
        // a group's partial row (8 d bytes) is as much traffic as a bf16 row of all four tensors: beyond 1024 groups (four
        // per CU) each takes at least four rows
        const int np = rows / 4 > 1024 ? rows / 4 : (rows < 1024 ? rows : 1024);
        return np > kPartialRows ? kPartialRows : np;
    }
    const int nblk = (rows + 3) / 4;
    return nblk > kPartialRows / 4 ? kPartialRows / 4 : nblk;
}
template <class T, bool RMS>
ds_status norm_bwd_partials(int rows, int d, const T* dy, const T* x, const T* g, const float* stats, const T* resid, T* dx,
                            float* partial, hipStream_t st) {
    const int ni = (d + 511) / 512;
    const dim3 grid(norm_bwd_groups(rows, d));
    if (ni > 2 && d % 32 == 0) {                 // wide rows: two or four wavefronts per row (see norm_bwd_multi_kernel)
        if (ni > 4) hipLaunchKernelGGL((norm_bwd_multi_kernel<T, RMS, 2, 4>), grid, dim3(256), 0, st, rows, d, dy, x, g, stats, resid, dx, partial);
        else hipLaunchKernelGGL((norm_bwd_multi_kernel<T, RMS, 2, 2>), grid, dim3(128), 0, st, rows, d, dy, x, g, stats, resid, dx, partial);
    } else {
        const dim3 block(256);
        if (ni <= 1) hipLaunchKernelGGL((norm_bwd_kernel<T, RMS, 1>), grid, block, 0, st, rows, d, dy, x, g, stats, resid, dx, partial);
        else if (ni <= 2) hipLaunchKernelGGL((norm_bwd_kernel<T, RMS, 2>), grid, block, 0, st, rows, d, dy, x, g, stats, resid, dx, partial);
        else if (ni <= 4) hipLaunchKernelGGL((norm_bwd_kernel<T, RMS, 4>), grid, block, 0, st, rows, d, dy, x, g, stats, resid, dx, partial);
        else hipLaunchKernelGGL((norm_bwd_kernel<T, RMS, 8>), grid, block, 0, st, rows, d, dy, x, g, stats, resid, dx, partial);
    }
    DS_LAUNCH_CHECK();
    return DS_OK;
}

// ------------------------------------------------------------------ the sums of a layer together
__device__ __forceinline__ int sum_group_item(const SumGroup& g, int& block) {
    int i = 0;
    while (i + 1 < g.n && block >= g.first[i + 1]) ++i;
    block -= g.first[i];
    return i;
}

// First stage of long sums: a work-group (64 lanes of 8 columns, 4 row lanes) adds up one chunk of an item's rows; chunk c of
// item i leaves row c of the [chunks][n] floats that end up as the item's source.
template <class T>
__global__ __launch_bounds__(256) void sum_group_chunks_kernel(SumGroup g, float* __restrict__ partial) {
    __shared__ float red[4][64][9];
    int block = blockIdx.x, off = 0;
    const int i = sum_group_item(g, block);
    for (int k = 0; k < i; ++k) off += g.chunks[k] * g.it[k].n;
    const int rows = g.it[i].rows, n = g.it[i].n, stride = g.it[i].stride, chunks = g.chunks[i];
    const T* x = reinterpret_cast<const T*>(g.it[i].src);
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6, chunk = block % chunks;
    const int col = (block / chunks * 64 + tx) * 8;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    if (col < n) {
        const int step = chunks * 4;
        int r = chunk * 4 + ty;
        for (; r < rows - 3 * step; r += 4 * step) {                  // four rows in flight per wavefront
            float v[4][8];
#pragma unroll
            for (int k = 0; k < 4; ++k) Vec8<T>::load(x + (size_t)(r + k * step) * stride + col, v[k]);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (v[0][j] + v[1][j]) + (v[2][j] + v[3][j]);
        }
        for (; r < rows; r += step) {
            float v[8];
            Vec8<T>::load(x + (size_t)r * stride + col, v);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += v[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[ty][tx][j] = acc[j];
    __syncthreads();
    if (ty == 0 && col < n) {
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (red[0][tx][j] + red[1][tx][j]) + (red[2][tx][j] + red[3][tx][j]);
        Vec8<float>::store(partial + off + (size_t)chunk * n + col, o);
    }
}

// Sums whose rows one work-group can walk: 32 columns per work-group of 512 threads, in 16-byte lanes (8 of float32, 4 of bf16), four
// rows in flight per lane, added up in a fixed order.  One launch for everything a layer's backward pass leaves to be summed (bias
// gradients, norm gradients): what these sums cost is their launches, 5 us each whatever they add up to a few thousand rows.
template <class T>
__global__ __launch_bounds__(512) void sum_group_kernel(SumGroup g) {
    constexpr int NW = 512 / 64;
    __shared__ float red[NW][32];
    int block = blockIdx.x;
    const int i = sum_group_item(g, block);
    const int rows = g.it[i].rows, n = g.it[i].n;
    const size_t stride = g.it[i].stride;
    float* out = g.it[i].out;
    const int c0 = block * 32, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (sizeof(T) == 2 && g.it[i].typed) {
        constexpr int RL = 512 / 4;
        const int cx = threadIdx.x & 3, col = c0 + cx * 8;
        const T* x = reinterpret_cast<const T*>(g.it[i].src) + col;
        float a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = 0.f;
        if (col < n) {
            int r = threadIdx.x >> 2;
            for (; r + 3 * RL < rows; r += 4 * RL) {
                float v[4][8];
#pragma unroll
                for (int k = 0; k < 4; ++k) Vec8<T>::load(x + (size_t)(r + k * RL) * stride, v[k]);
#pragma unroll
                for (int j = 0; j < 8; ++j) a[j] += (v[0][j] + v[1][j]) + (v[2][j] + v[3][j]);
            }
            for (; r < rows; r += RL) {
                float v[8];
                Vec8<T>::load(x + (size_t)r * stride, v);
#pragma unroll
                for (int j = 0; j < 8; ++j) a[j] += v[j];
            }
        }
#pragma unroll
        for (int o = 4; o < 64; o <<= 1)
#pragma unroll
            for (int j = 0; j < 8; ++j) a[j] += __shfl_xor(a[j], o, 64);
        if (lane < 4) Vec8<float>::store(&red[wave][cx * 8], a);
    } else {
        constexpr int RL = 512 / 8;
        const int cx = threadIdx.x & 7, col = c0 + cx * 4;
        const float* x = reinterpret_cast<const float*>(g.it[i].src) + col;
        f32x4_t a = {0.f, 0.f, 0.f, 0.f};
        if (col < n) {
            int r = threadIdx.x >> 3;
            for (; r + 3 * RL < rows; r += 4 * RL) {
                f32x4_t v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const f32x4_t*>(x + (size_t)(r + k * RL) * stride);
                a += (v[0] + v[1]) + (v[2] + v[3]);
            }
            for (; r < rows; r += RL) a += *reinterpret_cast<const f32x4_t*>(x + (size_t)r * stride);
        }
#pragma unroll
        for (int o = 8; o < 64; o <<= 1)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] += __shfl_xor(a[e], o, 64);
        if (lane < 8) *reinterpret_cast<f32x4_t*>(&red[wave][cx * 4]) = a;
    }
    __syncthreads();
    const int c = c0 + threadIdx.x;
    if (threadIdx.x < 32 && c < n) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) s += red[k][threadIdx.x];
        out[c] = g.accumulate ? out[c] + s : s;
    }
}

template <class T>
ds_status sum_group_run(SumGroup& g, float* partial, size_t partial_floats, hipStream_t st, int* launches) {
    // Tensors of more than kColsumSmallRows rows go through a first stage, cut into chunks of at least 32 rows (as many as there is
    // room for); the items of that stage and of the last one are listed by the same struct.
    SumGroup c;
    c.accumulate = 0;
    size_t cols = 0;
    for (int i = 0; i < g.n; ++i)
        if (g.it[i].typed && g.it[i].rows > kColsumSmallRows) cols += (size_t)g.it[i].n;
    int blocks = 0;
    size_t off = 0;
    for (int i = 0; i < g.n; ++i) {
        SumItem& q = g.it[i];
        if (!q.typed || q.rows <= kColsumSmallRows) continue;
        int chunks = (q.rows + 31) / 32;
        const size_t room = partial_floats / cols;
        if ((size_t)chunks > room) chunks = (int)room;
        if (chunks > 512) chunks = 512;
        if (chunks < 1) return DS_EINVAL;
        c.it[c.n] = q;
        c.first[c.n] = blocks;
        c.chunks[c.n++] = chunks;
        blocks += chunks * ((q.n / 8 + 63) / 64);
        q.src = partial + off;
        q.rows = chunks;
        q.stride = q.n;
        q.typed = 0;
        off += (size_t)chunks * q.n;
    }
    if (blocks) {
        hipLaunchKernelGGL(sum_group_chunks_kernel<T>, dim3(blocks), dim3(256), 0, st, c, partial);
        DS_LAUNCH_CHECK();
    }
    *launches = blocks ? 2 : 1;
    blocks = 0;
    for (int i = 0; i < g.n; ++i) {
        g.first[i] = blocks;
        blocks += (g.it[i].n + 31) / 32;
    }
    hipLaunchKernelGGL(sum_group_kernel<T>, dim3(blocks), dim3(512), 0, st, g);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

}  // namespace

ds_status launch_mask_rows(int32_t dtype, const MaskBatch& b, int32_t d, hipStream_t st) {
    if (d % 8) return DS_EINVAL;
    long long items = 0;
    for (int k = 0; k < b.n; ++k) items = std::max(items, (long long)b.rows[k] * (d / 8));
    if (items <= 0) return DS_OK;
    const dim3 grid(grid_for(items, 256), b.n);
    if (dtype == DS_DTYPE_BF16) hipLaunchKernelGGL(mask_rows_kernel<bf16_t>, grid, dim3(256), 0, st, b, d / 8);
    else hipLaunchKernelGGL(mask_rows_kernel<float>, grid, dim3(256), 0, st, b, d / 8);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status launch_zero_pad_rows(const ZeroPadBatch& b, int32_t rows, const int32_t* row_valid, hipStream_t st) {
    if (rows <= 0 || b.n <= 0) return DS_OK;
    int blocks = (rows + 3) / 4;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(zero_pad_rows_kernel, dim3(blocks, b.n), dim3(256), 0, st, b, rows, row_valid);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status launch_move_rows(const RowSegments& b, int32_t row_bytes, const void* in, void* out, bool to_stream, hipStream_t st) {
    if (b.n <= 0 || b.end <= b.row[0]) return DS_OK;
    const dim3 grid((unsigned)((b.end - b.row[0] + kMoveRows - 1) / kMoveRows));
    if (to_stream)
        hipLaunchKernelGGL(move_rows_kernel<true>, grid, dim3(256), 0, st, b, row_bytes / 16, (const uint4*)in, (uint4*)out);
    else
        hipLaunchKernelGGL(move_rows_kernel<false>, grid, dim3(256), 0, st, b, row_bytes / 16, (const uint4*)in, (uint4*)out);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status launch_move_rows_map(int32_t rows, const int32_t* map, int32_t row_bytes, const void* in, void* out, bool to_stream, hipStream_t st) {
    if (rows <= 0) return DS_OK;
    const size_t blocks = ((size_t)rows * (row_bytes / 16) + 255) / 256;
    if (blocks > 0x7fffffff) return DS_EOVERFLOW;
    const dim3 grid((unsigned)blocks);
    if (to_stream)
        hipLaunchKernelGGL(move_rows_map_kernel<true>, grid, dim3(256), 0, st, rows, map, row_bytes / 16, (const uint4*)in, (uint4*)out);
    else
        hipLaunchKernelGGL(move_rows_map_kernel<false>, grid, dim3(256), 0, st, rows, map, row_bytes / 16, (const uint4*)in, (uint4*)out);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status launch_transpose_bf16(TransposeBatch& b, hipStream_t st) {
    int blocks = 0;
    for (int i = 0; i < b.n; ++i) {
        if (b.rows[i] <= 0 || b.cols[i] <= 0 || b.rows[i] % 8 || b.cols[i] % 8 || !b.in[i] || !b.out[i]) return DS_EINVAL;
        b.first_block[i] = blocks;
        blocks += ((b.cols[i] + 63) / 64) * ((b.rows[i] + 255) / 256);
    }
    if (blocks == 0) return DS_OK;
    hipLaunchKernelGGL(transpose_bf16_kernel, dim3(blocks), dim3(256), 0, st, b);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

extern "C" int64_t ds_norm_bwd_scratch_floats(int32_t rows, int32_t d) {
    (void)rows;
    return (int64_t)kPartialRows * 2 * (d > 0 ? d : 0);
}

extern "C" ds_status ds_norm_fwd(int32_t dtype, int32_t rms, int32_t rows, int32_t d, const void* x, const void* g,
                                 const void* b, void* y, float* stats, void* hip_stream) {
    if (rows < 0 || d <= 0 || d % 8 || d > 4096 || !x || !g || !y || !stats || (!rms && !b)) return DS_EINVAL;
    if (dtype != DS_DTYPE_F32 && dtype != DS_DTYPE_BF16) return DS_EINVAL;
    if (rows == 0) return DS_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    if (dtype == DS_DTYPE_BF16) {
        if (rms) return norm_fwd_dispatch<bf16_t, true>(rows, d, (const bf16_t*)x, (const bf16_t*)g, (const bf16_t*)b, (bf16_t*)y, stats, st);
        return norm_fwd_dispatch<bf16_t, false>(rows, d, (const bf16_t*)x, (const bf16_t*)g, (const bf16_t*)b, (bf16_t*)y, stats, st);
    }
    if (rms) return norm_fwd_dispatch<float, true>(rows, d, (const float*)x, (const float*)g, (const float*)b, (float*)y, stats, st);
    return norm_fwd_dispatch<float, false>(rows, d, (const float*)x, (const float*)g, (const float*)b, (float*)y, stats, st);
}

int norm_bwd_partial_rows(int32_t rows, int32_t d) { return norm_bwd_groups(rows, d); }
ds_status launch_norm_bwd_partials(int32_t dtype, int32_t rms, int32_t rows, int32_t d, const void* dy, const void* x, const void* g,
                                   const float* stats, const void* resid, void* dx, float* partial, hipStream_t st) {
    if (dtype == DS_DTYPE_BF16) {
        if (rms) return norm_bwd_partials<bf16_t, true>(rows, d, (const bf16_t*)dy, (const bf16_t*)x, (const bf16_t*)g, stats, (const bf16_t*)resid, (bf16_t*)dx, partial, st);
        return norm_bwd_partials<bf16_t, false>(rows, d, (const bf16_t*)dy, (const bf16_t*)x, (const bf16_t*)g, stats, (const bf16_t*)resid, (bf16_t*)dx, partial, st);
    }
    if (rms) return norm_bwd_partials<float, true>(rows, d, (const float*)dy, (const float*)x, (const float*)g, stats, (const float*)resid, (float*)dx, partial, st);
    return norm_bwd_partials<float, false>(rows, d, (const float*)dy, (const float*)x, (const float*)g, stats, (const float*)resid, (float*)dx, partial, st);
}

ds_status launch_sum_group(int32_t dtype, SumGroup& g, float* partial, size_t partial_floats, hipStream_t st, int* launches) {
    *launches = 0;
    if (g.n <= 0) return DS_OK;
    for (int i = 0; i < g.n; ++i)
        if (!g.it[i].src || !g.it[i].out || g.it[i].rows <= 0 || g.it[i].n <= 0 || g.it[i].n % 8) return DS_EINVAL;
    if (dtype == DS_DTYPE_BF16) return sum_group_run<bf16_t>(g, partial, partial_floats, st, launches);
    return sum_group_run<float>(g, partial, partial_floats, st, launches);
}

extern "C" ds_status ds_norm_bwd(int32_t dtype, int32_t rms, int32_t rows, int32_t d, const void* dy, const void* x,
                                 const void* g, const float* stats, const void* resid, void* dx, float* dg, float* db,
                                 float* partial, int32_t accumulate, void* hip_stream) {
    if (rows <= 0 || d <= 0 || d % 8 || d > 4096 || !dy || !x || !g || !stats || !dx || !dg || !partial || (!rms && !db))
        return DS_EINVAL;
    if (dtype != DS_DTYPE_F32 && dtype != DS_DTYPE_BF16) return DS_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    const ds_status r = launch_norm_bwd_partials(dtype, rms, rows, d, dy, x, g, stats, resid, dx, partial, st);
    if (r != DS_OK) return r;
    // dgamma and, for LayerNorm, dbeta in one launch
    return reduce_launch(norm_bwd_groups(rows, d), d, (size_t)2 * d, partial, dg, accumulate, partial + d, rms ? nullptr : db, true, st);
}

ds_status launch_reduce_partials(int32_t n_partial, int32_t n, const float* partial, float* out, int32_t accumulate,
                                 hipStream_t st) {
    if (n_partial <= 0 || n <= 0 || !partial || !out) return DS_EINVAL;
    return reduce_launch(n_partial, n, (size_t)n, partial, out, accumulate, nullptr, nullptr, false, st);
}

// Column sums: one kernel for few rows (eight rows per lane: the second launch costs more than they do); otherwise two,
// gy partial rows of n floats each (gy <= max_partial_rows), then their sum in a fixed order.
static ds_status colsum_launch(int32_t dtype, int32_t rows, int32_t n, const void* x, float* out, float* partial,
                               int max_partial_rows, int32_t accumulate, hipStream_t st) {
    if (rows <= kColsumSmallRows) {
        const dim3 grid((n + 31) / 32);
        if (dtype == DS_DTYPE_BF16) hipLaunchKernelGGL(colsum_small_kernel<bf16_t>, grid, dim3(256), 0, st, rows, n, (const bf16_t*)x, out, accumulate);
        else hipLaunchKernelGGL(colsum_small_kernel<float>, grid, dim3(256), 0, st, rows, n, (const float*)x, out, accumulate);
        DS_LAUNCH_CHECK();
        return DS_OK;
    }
    const int gx = (n / 8 + 63) / 64;
    int gy = (rows + 31) / 32;                      // 32 rows per work-group: fewer partial rows than data by as much
    int cap = kPartialRows / gx > 0 ? kPartialRows / gx : 1;
    if (cap > max_partial_rows) cap = max_partial_rows;
    if (gy > cap) gy = cap;
    if (dtype == DS_DTYPE_BF16)
        hipLaunchKernelGGL(colsum_kernel<bf16_t>, dim3(gx, gy), dim3(256), 0, st, rows, n, (const bf16_t*)x, partial);
    else
        hipLaunchKernelGGL(colsum_kernel<float>, dim3(gx, gy), dim3(256), 0, st, rows, n, (const float*)x, partial);
    DS_LAUNCH_CHECK();
    return reduce_launch(gy, n, (size_t)n, partial, out, accumulate, nullptr, nullptr, false, st);
}

extern "C" ds_status ds_colsum(int32_t dtype, int32_t rows, int32_t n, const void* x, float* out, float* partial,
                               int32_t accumulate, void* hip_stream) {
    if (rows <= 0 || n <= 0 || n % 8 || !x || !out || !partial) return DS_EINVAL;
    if (dtype != DS_DTYPE_F32 && dtype != DS_DTYPE_BF16) return DS_EINVAL;
    return colsum_launch(dtype, rows, n, x, out, partial, kPartialRows, accumulate, (hipStream_t)hip_stream);
}

extern "C" ds_status ds_colsum_static(int32_t dtype, int32_t rows, int32_t n, const void* x, float* out, int32_t accumulate,
                                      void* hip_stream) {
    if (rows <= 0 || n <= 0 || n % 8 || !x || !out) return DS_EINVAL;
    if (dtype != DS_DTYPE_F32 && dtype != DS_DTYPE_BF16) return DS_EINVAL;
    if (n > kStaticMaxCols) return DS_ELIMIT;
    int dev = -1;
    DS_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return DS_ELIMIT;
    float* scratch = nullptr;
    {
        // once per device, with that device current: every GPU holds its own copy of the array at its own address
        std::lock_guard<std::mutex> lock(g_colsum_scratch_mutex);
        if (!g_colsum_scratch_ptr[dev]) {
            void* p = nullptr;
            DS_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(g_colsum_scratch)));
            if (!p) return DS_EHIP;
            g_colsum_scratch_ptr[dev] = (float*)p;
        }
        scratch = g_colsum_scratch_ptr[dev];
    }
    // every partial row the second kernel reads is written in full by the first: nothing needs clearing between calls
    return colsum_launch(dtype, rows, n, x, out, scratch, kStaticFloats / n, accumulate, (hipStream_t)hip_stream);
}
