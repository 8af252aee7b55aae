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
// What an epilogue reads besides the accumulators, fetched ahead of time (8 elements of R, of R2, the row flag),
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
        if (p.row_valid) q.valid = p.row_valid[m] >= 0;
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
    if (EPI == DS_EPI_NONE) {
        Vec8<T>::store_nt(C + off, acc);
    } else if (EPI == DS_EPI_GELU) {
        // round the pre-activation to storage precision first, so that forward and backward see the same z
        float z[8], a[8];
        Vec8<T>::store_nt(C + off, acc);
#pragma unroll
        for (int j = 0; j < 8; ++j) { z[j] = to_f32(from_f32<T>(acc[j])); a[j] = gelu_f(z[j]); }
        Vec8<T>::store_nt(reinterpret_cast<T*>(p.C2) + off, a);
    } else if (EPI == DS_EPI_GELU_D) {
        // what the layer's backward needs of the pre-activation is GELU'(z) alone: it is computed here, where the
        // logistic term is at hand anyway, and stored in place of z; the backward epilogue is then one multiplication
        float dz[8], a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) gelu_and_grad_f(acc[j], a[j], dz[j]);
        Vec8<T>::store_nt(C + off, dz);
        Vec8<T>::store_nt(reinterpret_cast<T*>(p.C2) + off, a);
    } else if (EPI == DS_EPI_MULR) {
        float r[8];
        if (pre) {
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = to_f32(pre->r[j]);
        } else {
            Vec8<T>::load(reinterpret_cast<const T*>(p.R) + off, r);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= r[j];
        Vec8<T>::store_nt(C + off, acc);
    } else if (EPI == DS_EPI_RESID) {
        if (pre) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = pre->valid ? acc[j] + to_f32(pre->r[j]) : 0.f;
        } else if (p.row_valid && p.row_valid[m] < 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.f;
        } else {
            float r[8];
            Vec8<T>::load(reinterpret_cast<const T*>(p.R) + off, r);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += r[j];
        }
        Vec8<T>::store_nt(C + off, acc);
    } else if (EPI == DS_EPI_DGELU) {
        float z[8];
        if (pre) {
#pragma unroll
            for (int j = 0; j < 8; ++j) z[j] = to_f32(pre->r[j]);
        } else {
            Vec8<T>::load(reinterpret_cast<const T*>(p.R) + off, z);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= gelu_grad_f(z[j]);
        Vec8<T>::store_nt(C + off, acc);
    } else if (EPI == DS_EPI_GATE) {
        // acc = u Wu (stored); C2 = GELU(R) * acc with R = u Wg
        float zg[8], a[8];
        Vec8<T>::store_nt(C + off, acc);
        if (pre) {
#pragma unroll
            for (int j = 0; j < 8; ++j) zg[j] = to_f32(pre->r[j]);
        } else {
            Vec8<T>::load(reinterpret_cast<const T*>(p.R) + off, zg);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = gelu_f(zg[j]) * to_f32(from_f32<T>(acc[j]));
        Vec8<T>::store_nt(reinterpret_cast<T*>(p.C2) + off, a);
    } else if (EPI == DS_EPI_DGATE) {
        // acc = da; R = zg, R2 = zu; C = dzg = da * zu * GELU'(zg); C2 = dzu = da * GELU(zg)
        float zg[8], zu[8], o1[8], o2[8];
        if (pre) {
#pragma unroll
            for (int j = 0; j < 8; ++j) { zg[j] = to_f32(pre->r[j]); zu[j] = to_f32(pre->r2[j]); }
        } else {
            Vec8<T>::load(reinterpret_cast<const T*>(p.R) + off, zg);
            Vec8<T>::load(reinterpret_cast<const T*>(p.R2) + off, zu);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            o1[j] = acc[j] * zu[j] * gelu_grad_f(zg[j]);
            o2[j] = acc[j] * gelu_f(zg[j]);
        }
        Vec8<T>::store_nt(C + off, o1);
        Vec8<T>::store(reinterpret_cast<T*>(p.C2) + off, o2);
    }
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
