// GEMM launcher shared by the C-ABI entry point and the stage driver.
#pragma once
#include "common.hpp"

struct GemmEpi {
    const void* bias;          // [N] or NULL
    const void* R;             // residual / saved pre-activation, [M,N]
    const void* R2;            // second saved tensor (gated MLP backward)
    void* C2;                  // second output
    const int32_t* row_valid;  // rows with a negative entry are written as zeros (RESID epilogue)
    int accumulate;            // ACC32: add to C instead of overwriting
    // DGELU and MULR epilogues of the bf16 NT kernels (gemm_colsum_fused says when; tiles of 256 rows or of 128): partial
    // column sums of the OUTPUT (before its rounding to bf16), float32 [gemm_colsum_rows(M)][N], every entry written;
    // NULL = not wanted
    float* colsum;
};

// true if launch_gemm with these arguments and p.colsum set fills p.colsum (otherwise it ignores the field)
bool gemm_colsum_fused(int32_t dtype, int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B,
                       const void* C, int32_t epilogue);
// 256 x 256 tiles and the lower ones of that kernel: a wavefront's 128 rows of every tensor of the output's shape have to fit into a
// 32-bit buffer length.  Wider outputs go to the smaller tiles.
inline bool gemm_big_width(int32_t epilogue, int32_t N) { return (uint64_t)N * 128 * (epilogue == DS_EPI_ACC32 ? 4 : 2) <= 0xFFFFFFFFu; }
inline size_t gemm_colsum_rows(int32_t M) { return (size_t)((M + 255) / 256) * 2; }

ds_status launch_gemm(int32_t dtype, int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B,
                      void* C, int32_t epilogue, const GemmEpi& p, bool force_generic, float* split_ws,
                      size_t split_ws_floats, hipStream_t st);

// fp32 on the matrix cores (gemm_f32.hip): whether it takes the operands, and its launcher (checked arguments)
bool gemm_f32_mfma_supported(int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B);
ds_status launch_gemm_f32_mfma(int32_t ta, int32_t tb, int32_t M, int32_t N, int32_t K, const void* A, const void* B, void* C,
                               int32_t epilogue, const GemmEpi& p, float* split_ws, size_t split_ws_floats, hipStream_t st);

// bf16 with smaller macro tiles (gemm_tile.hip).  kind: which tile, -1 = none fits; cost: estimated microseconds, what the
// kinds are ranked by; versus_large: the estimate to compare with that of the 256 x 256 kernel.
struct TilePick {
    int kind, splits;
    double cost, versus_large;
};
TilePick pick_gemm_tile(bool tn, int32_t M, int32_t N, int32_t K, size_t split_ws_floats, bool colsum, double out_us, bool out_read);
// microseconds (4 TB/s) to write an fp32 output and, when it is added to, to read it first: weight gradients of few tokens
// take about as long for this as for the products
inline double gemm_output_us(int epilogue, int32_t M, int32_t N, int accumulate) {
    return epilogue == DS_EPI_ACC32 ? 1e-6 * (accumulate ? 2.0 : 1.0) * M * N : 0.0;
}
ds_status launch_gemm_tile(const TilePick& pick, bool tn, int32_t M, int32_t N, int32_t K, const void* A, const void* B, void* C,
                           int32_t epilogue, const GemmEpi& p, float* split_ws, hipStream_t st);

// Weight gradients that contract over the same K token rows (those of one layer), as one launch:
// C[M,N] (+)= A[K,M]^T B[K,N], fp32 result, pointers 16-byte aligned; bf16 operands: M and N multiples of 256; fp32: M of 4, N of 8.
constexpr int kTnGroup = 8;
struct TnProblem {
    const void* A;
    const void* B;
    void* C;
    int32_t M, N;
};
struct TnGroup {
    int32_t n = 0, K = 0, accumulate = 0, f32 = 0;
    TnProblem p[kTnGroup];
    // Room for partial sums, in blocks of one tile (256 x 256 floats, fp32 operands 64 x 128): block u lies in the first slab i with
    // u < slab_end[i]
    __host__ __device__ int block_log2() const { return f32 ? 13 : 16; }
    static constexpr int kSlabs = 3;
    float* slab[kSlabs];
    int32_t slab_end[kSlabs];
    // filled in by launch_tn_group: K loops per tile, and the first work-group of each problem
    int32_t splits = 1;
    int32_t first[kTnGroup];
    __host__ __device__ float* block(int u) const {
        const int i = u < slab_end[0] ? 0 : u < slab_end[1] ? 1 : 2;
        return slab[i] + ((size_t)(u - (i ? slab_end[i - 1] : 0)) << block_log2());
    }
};
// which tile (a kind of gemm_tile.hip, kTnBig = the 256 x 256 kernel, kTnF32 = the fp32 one, -1: one launch each instead) and how
// many splits
constexpr int kTnBig = 4, kTnF32 = 5;
struct TnPick {
    int kind, splits;
};
TnPick pick_tn_group(const TnGroup& g);
ds_status launch_tn_group(const TnPick& pick, TnGroup& g, hipStream_t st);
ds_status launch_tn_group_big(TnGroup& g, int blocks, hipStream_t st);     // gemm.hip's and gemm_f32.hip's parts of them
TnPick pick_tn_group_f32(const TnGroup& g);
ds_status launch_tn_group_f32(TnGroup& g, hipStream_t st);
inline bool tn_group_takes(const TnProblem& q, int32_t K, bool f32) {
    return q.M > 0 && q.N > 0 && K > 0 && q.M % (f32 ? 4 : 256) == 0 && q.N % (f32 ? 8 : 256) == 0 && q.M <= (1 << 24) && q.N <= (1 << 24) &&
           (f32 || gemm_big_width(DS_EPI_ACC32, q.N)) && (((uintptr_t)q.A | (uintptr_t)q.B | (uintptr_t)q.C) & 15) == 0;
}

// compute units of the current device (256 where it cannot be asked)
int gemm_cu_count();
