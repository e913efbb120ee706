// Where the direct loads of an FP64 GEMM tile read (dgemm.hip): host and device
// code, so that the address ranges can be checked without a GPU.
//
// One operand of a tile: E rows of op(A) or columns of op(B), kBK inner
// elements a step, 16-byte chunks (two doubles).  ALONG: element (i, k) at
// X[i * ld + k], a chunk holds k and k + 1 of a row; else at X[k * ld + i], a
// chunk holds rows i and i + 1 of a k.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define OZ_BOTH __host__ __device__ __forceinline__
#else
#define OZ_BOTH inline
#endif

namespace oz {

constexpr int kBK = 16;

template <int E, bool ALONG>
struct OperandMap {
    static constexpr int PR = kBK / 2;              // pairs of k per row
    static constexpr int CHUNKS = E * kBK / 2;      // of a step

    // Row of the tile and k of the step whose elements chunk c of the LDS
    // stage holds (the swizzle of dgemm.hip's layout).
    static OZ_BOTH void place(int c, int &row, int &k) {
        if (ALONG) {
            row = c / PR;
            k = 2 * ((c % PR) ^ ((row >> 1) & 7));
        } else {
            k = c / (E / 2);
            row = 2 * ((c % (E / 2)) ^ (8 * ((k >> 1) & 1)));
        }
    }

    // Element offset of a step's base, and of its chunk at (row, k) from there;
    // rows past the operand's `n` are clamped to its last (pair of) row.
    static OZ_BOTH int64_t base(int64_t ld, int r0, int step) {
        return ALONG ? static_cast<int64_t>(r0) * ld + step * kBK : static_cast<int64_t>(step) * kBK * ld + r0;
    }
    static OZ_BOTH int clamp(int row, int n, int r0) {
        const int last = ALONG ? n - 1 : (n - 1) & ~1;
        return r0 + row < (ALONG ? n : last) ? row : last - r0;
    }
    static OZ_BOTH int64_t offset(int row, int k, int n, int64_t ld, int r0) {
        const int r = clamp(row, n, r0);
        return ALONG ? r * ld + k : k * ld + r;
    }
    // the same in bytes, where near() holds
    static OZ_BOTH int byte_offset(int row, int k, int n, int64_t ld, int r0) {
        const int r = clamp(row, n, r0);
        return ALONG ? static_cast<int>(r * ld * 8) + k * 8 : static_cast<int>(k * ld * 8) + r * 8;
    }

    // Whether every byte offset within a step fits the buffer loads' 31 bits.
    static OZ_BOTH bool near(int64_t ld) { return ld <= ((int64_t(1) << 31) - 4096) / 8 / (ALONG ? E : kBK); }

    // Steps that direct loads can take: whole ones, but not the one that holds
    // the last row of k when the rows across K are odd in number (their last
    // pair would run past the stored matrix).
    static OZ_BOTH int direct_steps(int n, int K) {
        return (ALONG || (n & 1) == 0) ? K / kBK : (K > 0 ? (K - 1) / kBK : 0);
    }
};

}  // namespace oz
