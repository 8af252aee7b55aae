// Epilogues of the GEMM kernels: what happens to 8 consecutive columns of an output row after the contraction.
#pragma once
#include "gemm.hpp"

namespace {

// ---------------------------------------------------------------------------- work-group ids
// Work-group id -> logical number such that each XCD (ids are dealt to the XCDs in turn) gets a contiguous run.
__device__ __forceinline__ int xcd_contiguous(int pid, int total) {
    const int xcd = pid & 7, per = total >> 3, rem = total & 7;
    return (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + (pid >> 3);
}
// kernel argument of the forms that run one problem
struct NoGroup {};
// the problem of a group that logical work-group `l` belongs to; l becomes its number within that problem
__device__ __forceinline__ int tn_group_problem(const TnGroup& g, int& l) {
    int i = 0;
    while (i + 1 < g.n && l >= g.first[i + 1]) ++i;
    l -= g.first[i];
    return i;
}

// ---------------------------------------------------------------------------- epilogues
// Applied to 8 consecutive columns n..n+7 of row m; acc holds the fp32 accumulators.
// What an epilogue reads besides the accumulators, fetched ahead of time (8 elements of R, of R2, the row's entry of row_valid),
// so that a caller can issue these loads for several rows at once instead of one dependent round trip per row.
// Kept in storage precision (16 bytes per operand for bf16) so that a whole tile's worth fits in registers.
template <class T> struct EpiPre {
    T r[8], r2[8];
    int valid;
};
template <class T>
__device__ __forceinline__ void load8_raw(const T* src, T (&dst)[8]) {
    if (sizeof(T) == 2) {
        const uint4 v = *reinterpret_cast<const uint4*>(src);
        __builtin_memcpy(dst, &v, 16);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) dst[j] = src[j];
    }
}
template <class T, int EPI>
__device__ __forceinline__ void epilogue_prefetch(int m, int n, int N, const GemmEpi& p, EpiPre<T>& q) {
    const size_t off = (size_t)m * N + n;
    q.valid = 1;
    if (EPI == DS_EPI_RESID) {
        if (p.row_valid) q.valid = p.row_valid[m];
        load8_raw(reinterpret_cast<const T*>(p.R) + off, q.r);
    } else if (EPI == DS_EPI_DGELU || EPI == DS_EPI_GATE || EPI == DS_EPI_MULR) {
        load8_raw(reinterpret_cast<const T*>(p.R) + off, q.r);
    } else if (EPI == DS_EPI_DGATE) {
        load8_raw(reinterpret_cast<const T*>(p.R) + off, q.r);
        load8_raw(reinterpret_cast<const T*>(p.R2) + off, q.r2);
    }
}
template <int EPI> constexpr bool epilogue_reads() {
    return EPI == DS_EPI_RESID || EPI == DS_EPI_DGELU || EPI == DS_EPI_GATE || EPI == DS_EPI_DGATE || EPI == DS_EPI_MULR;
}

// whether there is a second output
template <int EPI> constexpr bool epilogue_second() {
    return EPI == DS_EPI_GELU || EPI == DS_EPI_GELU_D || EPI == DS_EPI_GATE || EPI == DS_EPI_DGATE;
}
// 8 floats as they are stored
template <class T> struct Pack8 { typedef T type __attribute__((ext_vector_type(8))); };
template <class T> __device__ __forceinline__ typename Pack8<T>::type pack8(const float (&v)[8]) {
    typename Pack8<T>::type a;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = from_f32<T>(v[i]);
    return a;
}
// Ordinary stores: the kernels that end here (tiles smaller than 256 x 256, fp32, sums of split contractions) write outputs that the next
// launch reads back from the caches.  With streaming stores, which the 256 x 256 kernel uses for its far larger ones: a call of five short
// sequences through two layers of d = 256 191 -> 199 us, d = 768 micro-batches one by one (2 050 tokens, two layers) 1 597 -> 1 693,
// encoder-decoder d = 512 over 1 138 tokens 380 -> 402, d = 256 fp32 over 40 000 4 374 -> 4 475.  A launch that nothing follows is
// the slower for them, because its end waits for the caches to be written back: 957 x 2816 x 1024 with GELU 17.9 -> 18.9 us, 2 280 x 2048 x 512
// with a bias 15.1 -> 15.8, fp32 with short contractions most, 9 381 x 1536 x 128 46.8 -> 48.6.
template <class T> __device__ __forceinline__ void store8(T* p, const typename Pack8<T>::type& v) {
    __builtin_memcpy(__builtin_assume_aligned(p, 16), &v, sizeof v);
}
// Streaming ones for what the forward pass leaves to the backward pass (the pre-activation or derivative of a GELU, the ungated product):
// nothing reads it soon, and it only makes that wait longer: with ordinary stores for both outputs 1 274 x 3072 x 1024 with GELU 19.4 -> 20.1 us (one
// launch after another 14.5 -> 15.4), fp32 42 095 x 2048 x 64 218 -> 227; whole calls take the same time either way.
template <int EPI> constexpr bool epilogue_keeps_first() { return EPI == DS_EPI_GELU || EPI == DS_EPI_GELU_D || EPI == DS_EPI_GATE; }
template <class T> __device__ __forceinline__ void store8_streaming(T* p, const typename Pack8<T>::type& v) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 part[sizeof v / 16];
    __builtin_memcpy(part, &v, sizeof v);
#pragma unroll
    for (int i = 0; i < (int)(sizeof v / 16); ++i) __builtin_nontemporal_store(part[i], reinterpret_cast<u32x4*>(p) + i);
}
// The epilogue proper (all but ACC32), after the bias: acc becomes what is stored to C, one and two the stored forms of it and of the
// second output
template <class T, int EPI>
__device__ __forceinline__ void epilogue_values(float (&acc)[8], const EpiPre<T>& q, typename Pack8<T>::type& one, typename Pack8<T>::type& two) {
    float b[8];
    if (EPI == DS_EPI_GELU) {
        // round the pre-activation to storage precision first, so that forward and backward see the same z
#pragma unroll
        for (int j = 0; j < 8; ++j) b[j] = gelu_f(to_f32(from_f32<T>(acc[j])));
    } else if (EPI == DS_EPI_GELU_D) {
        // what the layer's backward needs of the pre-activation is GELU'(z) alone: it is computed here, where the
        // logistic term is at hand anyway, and stored in place of z; the backward epilogue is then one multiplication
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float z = acc[j];
            gelu_and_grad_f(z, b[j], acc[j]);
        }
    } else if (EPI == DS_EPI_MULR) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= to_f32(q.r[j]);
    } else if (EPI == DS_EPI_RESID) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = q.valid >= 0 ? acc[j] + to_f32(q.r[j]) : 0.f;
    } else if (EPI == DS_EPI_DGELU) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= gelu_grad_f(to_f32(q.r[j]));
    } else if (EPI == DS_EPI_GATE) {
        // acc = u Wu (stored); second output = GELU(R) * acc with R = u Wg
#pragma unroll
        for (int j = 0; j < 8; ++j) b[j] = gelu_f(to_f32(q.r[j])) * to_f32(from_f32<T>(acc[j]));
    } else if (EPI == DS_EPI_DGATE) {
        // acc = da; R = zg, R2 = zu; outputs dzg = da * zu * GELU'(zg) and dzu = da * GELU(zg)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float zg = to_f32(q.r[j]);
            b[j] = acc[j] * gelu_f(zg);
            acc[j] = acc[j] * to_f32(q.r2[j]) * gelu_grad_f(zg);
        }
    }
    one = pack8<T>(acc);
    if (epilogue_second<EPI>()) two = pack8<T>(b);
}
template <class T, int EPI>
__device__ __forceinline__ void epilogue8(int m, int n, int N, float (&acc)[8], T* __restrict__ C, const GemmEpi& p,
                                          const EpiPre<T>* pre = nullptr) {
    const size_t off = (size_t)m * N + n;
    if (EPI == DS_EPI_ACC32) {
        float* c = reinterpret_cast<float*>(C) + off;
        if (p.accumulate) {
            float old[8];
            Vec8<float>::load(c, old);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += old[j];
        }
        Vec8<float>::store(c, acc);
        return;
    }
    if (p.bias) {
        float b[8];
        Vec8<T>::load(reinterpret_cast<const T*>(p.bias) + n, b);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += b[j];
    }
    EpiPre<T> own;
    if (epilogue_reads<EPI>() && !pre) {
        epilogue_prefetch<T, EPI>(m, n, N, p, own);
        pre = &own;
    }
    typename Pack8<T>::type one, two;
    epilogue_values<T, EPI>(acc, epilogue_reads<EPI>() ? *pre : own, one, two);
    if (epilogue_keeps_first<EPI>()) store8_streaming(C + off, one);
    else store8(C + off, one);
    if (epilogue_second<EPI>()) store8(reinterpret_cast<T*>(p.C2) + off, two);
}

// sum the split-K partials ([split][M][N]) in split order and apply the epilogue; one thread per 8 columns
template <class T, int EPI>
__global__ __launch_bounds__(256) void splitk_finish_kernel(int M, int N, int splits, const float* __restrict__ ws,
                                                            T* __restrict__ C, GemmEpi p) {
    const int n8 = N / 8;
    const long long total = (long long)M * n8;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        const int m = (int)(i / n8);
        const int n = (int)(i - (long long)m * n8) * 8;
        float v[8];
        Vec8<float>::load(ws + (size_t)m * N + n, v);
        for (int s = 1; s < splits; ++s) {
            float w[8];
            Vec8<float>::load(ws + ((size_t)s * M + m) * N + n, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] += w[j];
        }
        epilogue8<T, EPI>(m, n, N, v, C, p);
    }
}

template <class T, int EPI>
ds_status launch_splitk_finish(int M, int N, int splits, const float* ws, void* C, const GemmEpi& p, hipStream_t st) {
    long long blocks = ((long long)M * (N / 8) + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL((splitk_finish_kernel<T, EPI>), dim3((unsigned)blocks), dim3(256), 0, st, M, N, splits, ws, (T*)C, p);
    DS_LAUNCH_CHECK();
    return DS_OK;
}

}  // namespace
