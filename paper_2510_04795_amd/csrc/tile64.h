// 64 x 64 x 64 FP64 products of two LDS tiles on the FP64 matrix cores
// (v_mfma_f64_16x16x4_f64), for the kernels that work on 64 x 64 blocks of a
// matrix: 256 threads = 2 x 2 waves of 32 x 32 outputs, each 2 x 2 blocks of
// 16 x 16.  Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator register r of lane l holds C[4 r + l / 16][l % 16].
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace oz {
namespace t64 {

typedef double v4d __attribute__((ext_vector_type(4)));

// Row strides (doubles) of the LDS tiles.  A wave reads 16 rows x 4
// consecutive k of an operand stored along k: a stride of 4 mod 32 doubles
// spreads them evenly over the 64 banks; an operand stored across k (4 rows x
// 16 consecutive columns) needs 16 mod 32.
constexpr int kLdK = 68;   // operand read along its rows (k contiguous)
constexpr int kLdN = 80;   // right operand stored k-major (columns contiguous)

struct Acc {
    v4d c[2][2];
    __device__ void zero() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) c[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    }
};

__device__ __forceinline__ int wave_row() { return (threadIdx.x >> 7) * 32; }
__device__ __forceinline__ int wave_col() { return ((threadIdx.x >> 6) & 1) * 32; }

// s[r][c] (row stride lds) = g[r * ld + c], r, c < 64; g 16-byte aligned, ld even.
__device__ __forceinline__ void load(double *s, int lds, const double *__restrict__ g, int64_t ld) {
    const int r0 = threadIdx.x >> 5, c = (threadIdx.x & 31) * 2;
    double2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const double2 *>(g + (r0 + 8 * q) * ld + c);
#pragma unroll
    for (int q = 0; q < 8; ++q) *reinterpret_cast<double2 *>(s + (r0 + 8 * q) * lds + c) = v[q];
}

// acc += A B^T, A and B row-major along k (stride kLdK)
__device__ __forceinline__ void mul_nt(Acc &acc, const double *sA, const double *sB) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const double *a = sA + (wave_row() + l16) * kLdK + lq;
    const double *b = sB + (wave_col() + l16) * kLdK + lq;
#pragma unroll
    for (int kk = 0; kk < 64; kk += 4) {
        const double a0 = a[kk], a1 = a[16 * kLdK + kk], b0 = b[kk], b1 = b[16 * kLdK + kk];
        acc.c[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc.c[0][0], 0, 0, 0);
        acc.c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc.c[0][1], 0, 0, 0);
        acc.c[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc.c[1][0], 0, 0, 0);
        acc.c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc.c[1][1], 0, 0, 0);
    }
}

// acc += A B, A row-major along k (stride kLdK), B k-major (stride kLdN)
__device__ __forceinline__ void mul_nn(Acc &acc, const double *sA, const double *sB) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const double *a = sA + (wave_row() + l16) * kLdK + lq;
    const double *b = sB + lq * kLdN + wave_col() + l16;
#pragma unroll
    for (int kk = 0; kk < 64; kk += 4) {
        const double a0 = a[kk], a1 = a[16 * kLdK + kk], b0 = b[kk * kLdN], b1 = b[kk * kLdN + 16];
        acc.c[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc.c[0][0], 0, 0, 0);
        acc.c[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc.c[0][1], 0, 0, 0);
        acc.c[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc.c[1][0], 0, 0, 0);
        acc.c[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc.c[1][1], 0, 0, 0);
    }
}

// f(row, column, value) for this lane's 16 elements of the 64 x 64 result
template <typename F>
__device__ __forceinline__ void each(const Acc &acc, F f) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(wave_row() + 16 * i + 4 * r + lq, wave_col() + 16 * j + l16, acc.c[i][j][r]);
}

}  // namespace t64
}  // namespace oz
