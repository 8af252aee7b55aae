// Variable-length attention, generic kernels (any dtype, head_dim <= 128, multiple of 8): the
// fallback for the shapes and alignments the matrix-core kernels (bf16 and fp32) do not take.  One 64-lane wavefront
// per query row (forward, dQ) or per key row (dK/dV); no work is spent on padding because the
// kernels walk the sequence table, never the padded tensor.
#include "attention_rows.hpp"

namespace {

// ---------------------------------------------------------------- forward
template <class T>
__global__ __launch_bounds__(256) void attn_fwd_generic_kernel(AttnArgs a) {
    __shared__ float sq[4][128];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int qi = blockIdx.x * 4 + w, h = blockIdx.y, s = blockIdx.z, hd = a.head_dim;
    const bool active = qi < a.q_len[s];
    if (active) stage_row(sq[w], (const T*)a.q + ((long long)a.q_row[s] + qi) * a.ldq + h * hd, hd, a.scale, lane);
    __syncthreads();
    if (active) attn_fwd_row<T>(a, s, h, qi, sq[w], lane);
}

// ---------------------------------------------------------------- delta = rowsum(dO * O)
template <class T>
__global__ __launch_bounds__(256) void attn_delta_kernel(AttnArgs a) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int qi = blockIdx.x * 4 + w, h = blockIdx.y, s = blockIdx.z;
    if (qi >= a.q_len[s]) return;
    const int hd = a.head_dim;
    const long long qr = (long long)a.q_row[s] + qi;
    const T* o = (const T*)a.o + qr * a.ldo + h * hd;
    const T* d_o = (const T*)a.d_o + qr * a.ldo + h * hd;
    float acc = 0.f;
    for (int d = lane; d < hd; d += 64) acc += to_f32(o[d]) * to_f32(d_o[d]);
    acc = wave_sum(acc);
    if (lane == 0) a.delta[(size_t)h * a.lse_stride + qr] = acc;
}

// ---------------------------------------------------------------- dQ: one wavefront per query row
template <class T>
__global__ __launch_bounds__(256) void attn_bwd_dq_generic_kernel(AttnArgs a) {
    __shared__ float sq[4][128];
    __shared__ float sdo[4][128];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int qi = blockIdx.x * 4 + w, h = blockIdx.y, s = blockIdx.z, hd = a.head_dim;
    const long long qr = (long long)a.q_row[s] + qi;
    const bool active = qi < a.q_len[s];
    if (active) {
        stage_row(sq[w], (const T*)a.q + qr * a.ldq + h * hd, hd, a.scale, lane);
        stage_row(sdo[w], (const T*)a.d_o + qr * a.ldo + h * hd, hd, 1.0f, lane);
    }
    __syncthreads();
    if (active) attn_bwd_dq_row<T>(a, s, h, qi, sq[w], sdo[w], lane);
}

// ---------------------------------------------------------------- dK, dV: one wavefront per key row
template <class T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_generic_kernel(AttnArgs a) {
    __shared__ float sk[4][128];
    __shared__ float sv[4][128];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int kj = blockIdx.x * 4 + w, h = blockIdx.y, s = blockIdx.z, hd = a.head_dim;
    const long long kr = (long long)a.k_row[s] + kj;
    const bool active = kj < a.k_len[s];
    if (active) {
        stage_row(sk[w], (const T*)a.k + kr * a.ldk + h * hd, hd, a.scale, lane);
        stage_row(sv[w], (const T*)a.v + kr * a.ldv + h * hd, hd, 1.0f, lane);
    }
    __syncthreads();
    if (active) attn_bwd_dkv_row<T>(a, s, h, kj, sk[w], sv[w], lane);
}

}  // namespace

template <class T>
static ds_status fwd_generic_t(const AttnArgs& a, hipStream_t st) {
    dim3 grid((a.max_q_len + 3) / 4, a.n_heads, a.n_seq);
    hipLaunchKernelGGL(attn_fwd_generic_kernel<T>, grid, dim3(256), 0, st, a);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status attn_fwd_generic(const AttnArgs& a, hipStream_t st) {
    return a.dtype == DS_DTYPE_BF16 ? fwd_generic_t<bf16_t>(a, st) : fwd_generic_t<float>(a, st);
}

ds_status attn_delta(const AttnArgs& a, hipStream_t st) {
    dim3 grid((a.max_q_len + 3) / 4, a.n_heads, a.n_seq);
    if (a.dtype == DS_DTYPE_BF16)
        hipLaunchKernelGGL(attn_delta_kernel<bf16_t>, grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(attn_delta_kernel<float>, grid, dim3(256), 0, st, a);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

template <class T>
static ds_status bwd_generic_t(const AttnArgs& a, hipStream_t st) {
    dim3 gq((a.max_q_len + 3) / 4, a.n_heads, a.n_seq);
    hipLaunchKernelGGL(attn_bwd_dq_generic_kernel<T>, gq, dim3(256), 0, st, a);
    DS_LAUNCH_CHECK();
    dim3 gk((a.max_k_len + 3) / 4, a.n_heads, a.n_seq);
    hipLaunchKernelGGL(attn_bwd_dkv_generic_kernel<T>, gk, dim3(256), 0, st, a);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

ds_status attn_bwd_generic(const AttnArgs& a, hipStream_t st) {
    return a.dtype == DS_DTYPE_BF16 ? bwd_generic_t<bf16_t>(a, st) : bwd_generic_t<float>(a, st);
}
