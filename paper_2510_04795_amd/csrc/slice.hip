// Steps 1 and 2 of the emulated GEMM ("Theory of emulated FP64 arithmetic"):
// one power-of-two exponent per row of A / column of B, then S balanced
// int8 slices per element, written in the packed layout of internal.h.
//
// Large operands are HBM-bound: the exponent pass reads X once (8 B per
// element); the slice pass reads it again and writes S bytes per element.
// Small ones are bound by their launches, so a call's two operands share a
// launch per pass (k_exponents2, k_slice2; one launch for both passes up to K =
// 256, k_slice_groups2), and maxima travel as exponent codes that the slice
// pass turns into exponents.
#include <algorithm>

#include "internal.h"

namespace oz {
namespace {

// |x| for a finite x, NaN for NaN or +-Inf (marks the group as non-finite).
__device__ inline double abs_or_nan(double x) {
    if (!(fabs(x) <= 1.79769313486231570815e308)) return __longlong_as_double(0x7ff8000000000000ll);
    return fabs(x);
}

// Maximum that propagates NaN from either side.
__device__ inline double combine_max(double a, double b) {
    if (a != a || b != b) return __longlong_as_double(0x7ff8000000000000ll);
    return a > b ? a : b;
}

__device__ inline int32_t finish_exponent(double mu, uint32_t *flag) {
    if (mu != mu) {
        atomicOr(flag, 1u);
        return kExpBad;
    }
    return shared_exponent(mu);
}

// One wave per row; 4 rows per 256-thread block.
__global__ __launch_bounds__(256) void k_row_exponents(const double *__restrict__ X, int64_t ld,
                                                        int64_t R, int64_t K,
                                                        int32_t *__restrict__ e,
                                                        uint32_t *flag) {
    const int lane = threadIdx.x & 63;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (r >= R) return;
    const double *row = X + r * ld;
    // four loads in flight per lane; the maximum does not depend on the order
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0;
    int64_t k = lane;
    for (; k + 192 < K; k += 256) {
        const double a = row[k], b = row[k + 64], c = row[k + 128], d = row[k + 192];
        m0 = combine_max(m0, abs_or_nan(a));
        m1 = combine_max(m1, abs_or_nan(b));
        m2 = combine_max(m2, abs_or_nan(c));
        m3 = combine_max(m3, abs_or_nan(d));
    }
    for (; k < K; k += 64) m0 = combine_max(m0, abs_or_nan(row[k]));
    double mu = combine_max(combine_max(m0, m1), combine_max(m2, m3));
    for (int off = 32; off >= 1; off >>= 1) mu = combine_max(mu, __shfl_xor(mu, off, 64));
    if (lane == 0) e[r] = finish_exponent(mu, flag);
}

// Column maxima of X (K x R): block (column strip of 256, row chunk of 256).
constexpr int kColChunk = 256;

__global__ __launch_bounds__(256) void k_col_partial(const double *__restrict__ X, int64_t ld,
                                                      int64_t K, int64_t R,
                                                      double *__restrict__ part) {
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (c >= R) return;
    const int64_t k0 = static_cast<int64_t>(blockIdx.y) * kColChunk;
    const int64_t k1 = k0 + kColChunk < K ? k0 + kColChunk : K;
    // eight loads in flight per lane; the maximum does not depend on the order
    double m[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int64_t k = k0;
    for (; k + 8 <= k1; k += 8) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = X[(k + q) * ld + c];
#pragma unroll
        for (int q = 0; q < 8; ++q) m[q] = combine_max(m[q], abs_or_nan(v[q]));
    }
    for (; k < k1; ++k) m[0] = combine_max(m[0], abs_or_nan(X[k * ld + c]));
    double mu = m[0];
#pragma unroll
    for (int q = 1; q < 8; ++q) mu = combine_max(mu, m[q]);
    part[static_cast<int64_t>(blockIdx.y) * R + c] = mu;
}

__global__ __launch_bounds__(256) void k_col_final(const double *__restrict__ part, int64_t nchunk,
                                                    int64_t R, int32_t *__restrict__ e,
                                                    uint32_t *flag) {
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (c >= R) return;
    double mu = 0.0;
    for (int64_t q = 0; q < nchunk; ++q) mu = combine_max(mu, part[q * R + c]);
    e[c] = finish_exponent(mu, flag);
}

// Sums of squares per group (statistics of the automatic slice count).
// Rows: one wave per row, lanes stride the row, fixed shuffle tree.
__global__ __launch_bounds__(256) void k_row_sumsq(const double *__restrict__ X, int64_t ld, int64_t R,
                                                    int64_t K, double *__restrict__ ss) {
    const int lane = threadIdx.x & 63;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (r >= R) return;
    const double *row = X + r * ld;
    double acc = 0.0;
    for (int64_t k = lane; k < K; k += 64) acc = fma(row[k], row[k], acc);
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) ss[r] = acc;
}

// Columns of X (K x R): partial sums over row chunks, then the chunks in order.
__global__ __launch_bounds__(256) void k_col_sumsq_partial(const double *__restrict__ X, int64_t ld,
                                                            int64_t K, int64_t R, double *__restrict__ part) {
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (c >= R) return;
    const int64_t k0 = static_cast<int64_t>(blockIdx.y) * kColChunk;
    const int64_t k1 = k0 + kColChunk < K ? k0 + kColChunk : K;
    double acc = 0.0;
    for (int64_t k = k0; k < k1; ++k) {
        const double x = X[k * ld + c];
        acc = fma(x, x, acc);
    }
    part[static_cast<int64_t>(blockIdx.y) * R + c] = acc;
}

__global__ __launch_bounds__(256) void k_col_sumsq_final(const double *__restrict__ part, int64_t nchunk,
                                                          int64_t R, double *__restrict__ ss) {
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (c >= R) return;
    double acc = 0.0;
    for (int64_t q = 0; q < nchunk; ++q) acc += part[q * R + c];
    ss[c] = acc;
}

// Balanced base-256 digits of X = RNE(x 2^(8S-1-e)): byte S - 1 - t of the
// result is digit t.  Adding 128 to every digit but the leading one makes all
// of them unsigned without borrows between the bytes (digit + 128 is in [0,
// 255]), so one addition and one exclusive or replace S - 1 rounds of 64-bit
// extraction: slicing is then bound by memory, not by the vector units
// (32 groups of 512, S = 7, in one
// workgroup: 16.3 -> 12.4 us).
template <int S>
__device__ inline uint64_t digit_bytes(double x, int32_t e) {
    const double y = rint(ldexp(x, 8 * S - 1 - e));
    if constexpr (S <= 4) {
        constexpr uint32_t c = 0x80808080u >> (32 - 8 * (S - 1));
        return (static_cast<uint32_t>(static_cast<int32_t>(y)) + c) ^ c;
    } else {
        constexpr uint64_t c = 0x8080808080808080ull >> (64 - 8 * (S - 1));
        return (static_cast<uint64_t>(static_cast<int64_t>(y)) + c) ^ c;
    }
}

// Words of bytes [z0.b, z1.b] pairs: byte b of two values in the low half and
// byte b + 1 in the high half of pair[b / 2].
template <int S>
__device__ inline void byte_pairs(uint64_t z0, uint64_t z1, uint32_t (&pair)[(S + 1) / 2]) {
    const uint32_t l0 = static_cast<uint32_t>(z0), l1 = static_cast<uint32_t>(z1);
    const uint32_t h0 = static_cast<uint32_t>(z0 >> 32), h1 = static_cast<uint32_t>(z1 >> 32);
#pragma unroll
    for (int j = 0; j < (S + 1) / 2; ++j)
        pair[j] = __builtin_amdgcn_perm(j < 2 ? l1 : h1, j < 2 ? l0 : h0, (j & 1) ? 0x07030602u : 0x05010400u);
}

// Digits of four consecutive elements of a group, one word per slice.
template <int S>
__device__ inline void slice4(const double (&x)[4], int32_t e, uint32_t (&w)[S]) {
    uint64_t z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = e == kExpBad ? 0 : digit_bytes<S>(x[q], e);
    uint32_t p01[(S + 1) / 2], p23[(S + 1) / 2];
    byte_pairs<S>(z[0], z[1], p01);
    byte_pairs<S>(z[2], z[3], p23);
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int b = S - 1 - s;
        w[s] = __builtin_amdgcn_perm(p23[b >> 1], p01[b >> 1], (b & 1) ? 0x07060302u : 0x05040100u);
    }
}

// Digits of two consecutive elements of a row per lane, lanes 2 i and 2 i + 1
// holding four elements in a row: their words go into the LDS tile, byte b of
// even b from the even lane, of odd b from the odd lane.
template <int S>
__device__ inline void slice2_store(uint4 (*tile)[32], double x0, double x1, int32_t e, int c, int row, int word) {
    const uint64_t z0 = e == kExpBad ? 0 : digit_bytes<S>(x0, e), z1 = e == kExpBad ? 0 : digit_bytes<S>(x1, e);
    uint32_t own[(S + 1) / 2];
    byte_pairs<S>(z0, z1, own);
    const bool odd = threadIdx.x & 1;
#pragma unroll
    for (int j = 0; j < (S + 1) / 2; ++j) {
        // the neighbour's pair (lanes 1, 0, 3, 2 of each four)
        const uint32_t other = static_cast<uint32_t>(
            __builtin_amdgcn_mov_dpp(static_cast<int>(own[j]), 0xb1, 0xf, 0xf, true));
        const uint32_t lo = odd ? other : own[j], hi = odd ? own[j] : other;
        const uint32_t w = __builtin_amdgcn_perm(hi, lo, odd ? 0x07060302u : 0x05040100u);
        const int s = S - 1 - (2 * j + (odd ? 1 : 0));
        if (s >= 0) reinterpret_cast<uint32_t *>(&tile[s * 2 + c][row])[word] = w;
    }
}

// Slicing of 32 groups (from r0) x 32 inner elements (block kb) by 256
// threads (t), in three steps: four elements per thread into registers, their
// digits into an LDS tile, the tile into the packed planes.  TRANS = false: X
// is R x K and a group is a row (16 lanes per row, two consecutive elements
// each, rows r and r + 16); TRANS = true: X is K x R and a group is a column
// (lanes take consecutive groups, so every load is coalesced).
template <bool TRANS>
__device__ inline void slice_load(double (&x)[4], const double *__restrict__ X, int64_t ld, int64_t R, int64_t K,
                                  int64_t r0, int64_t kb, int t) {
    const int64_t k0 = kb * 32;
    if (TRANS) {
        const int r = t & 31, kq = t >> 5;
        const int64_t gr = r0 + r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t k = k0 + kq * 4 + q;
            x[q] = (gr < R && k < K) ? X[k * ld + gr] : 0.0;
        }
    } else {
        // one 16-byte load when the block is whole and aligned
        const int64_t k = k0 + 2 * (t & 15);
        const bool full = r0 + 32 <= R && k0 + 32 <= K && (ld & 1) == 0 &&
                          (reinterpret_cast<uintptr_t>(X) & 15) == 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t gr = r0 + (t >> 4) + 16 * h;
            double x0 = 0.0, x1 = 0.0;
            if (full) {
                const double2 v = *reinterpret_cast<const double2 *>(X + gr * ld + k);
                x0 = v.x;
                x1 = v.y;
            } else if (gr < R) {
                if (k < K) x0 = X[gr * ld + k];
                if (k + 1 < K) x1 = X[gr * ld + k + 1];
            }
            x[2 * h] = x0;
            x[2 * h + 1] = x1;
        }
    }
}

// e0, e1: exponents of the thread's group (TRANS: e0 only), of rows r and r + 16
template <int S, bool TRANS>
__device__ inline void slice_digits(uint4 (*tile)[32], const double (&x)[4], int32_t e0, int32_t e1, int t) {
    if (TRANS) {
        const int r = t & 31, kq = t >> 5;
        uint32_t w[S];
        slice4<S>(x, e0, w);
        const int c = kq >> 2, word = kq & 3;
#pragma unroll
        for (int s = 0; s < S; ++s) reinterpret_cast<uint32_t *>(&tile[s * 2 + c][r])[word] = w[s];
    } else {
        const int kq = (t & 15) >> 1;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            slice2_store<S>(tile, x[2 * h], x[2 * h + 1], h ? e1 : e0, kq >> 2, (t >> 4) + 16 * h, kq & 3);
    }
}

// 2S runs of 32 rows x 16 bytes
template <int S>
__device__ inline void slice_store(const uint4 (*tile)[32], int8_t *__restrict__ packed, int64_t Rp, int64_t r0,
                                   int64_t kb, int t) {
    uint4 *out = reinterpret_cast<uint4 *>(packed);
    for (int q = t; q < S * 2 * 32; q += 256) {
        const int sc = q >> 5;
        const int rr = q & 31;
        out[(kb * S * 2 + sc) * Rp + r0 + rr] = tile[sc][rr];
    }
}

// The three steps by a workgroup of 256, the groups' exponents at e.
template <int S, bool TRANS>
__device__ inline void slice_tile(uint4 (*tile)[32], const double *__restrict__ X, int64_t ld, int64_t R, int64_t K,
                                  const int32_t *e, int8_t *__restrict__ packed, int64_t Rp, int64_t r0, int64_t kb) {
    const int t = threadIdx.x;
    const int r = TRANS ? t & 31 : t >> 4;
    double x[4];
    slice_load<TRANS>(x, X, ld, R, K, r0, kb, t);
    const int32_t e0 = r0 + r < R ? e[r] : 0, e1 = !TRANS && r0 + r + 16 < R ? e[r + 16] : 0;
    slice_digits<S, TRANS>(tile, x, e0, e1, t);
    __syncthreads();
    slice_store<S>(tile, packed, Rp, r0, kb, t);
}

template <int S, bool TRANS>
__global__ __launch_bounds__(256) void k_slice(const double *__restrict__ X, int64_t ld, int64_t R,
                                                int64_t K, const int32_t *__restrict__ e,
                                                int8_t *__restrict__ packed, int64_t Rp) {
    __shared__ uint4 tile[S * 2][32];
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * 32;
    slice_tile<S, TRANS>(tile, X, ld, R, K, e + r0, packed, Rp, r0, blockIdx.y);
}

// ---- both operands of one product, two launches ---------------------------
// Exponents then slices of op(A) and op(B), each pass one launch over the
// blocks of A followed by those of B (1021 x 2777 times 2777 x 1531, S = 7:
// 38 us against 68 for six launches, whose column maxima ran on 44
// workgroups; 2048^3: 38 against 54; 8192^3: 604 against 619, bound by
// memory).  Groups stored as rows get their
// exponents from the first pass.  Groups stored as columns get one exponent
// code per chunk of rows there (a code is monotone in the magnitude, so the
// largest code is the code of the largest magnitude); every slice block takes
// the maximum of its 32 groups' codes itself, and the blocks of the first K
// block write the exponents the pair kernel reads.

// Maximum over one row by `nl` lanes of which this is lane `l`, eight loads
// in flight (the order does not matter).
__device__ inline double row_max(const double *__restrict__ row, int64_t K, int l, int nl) {
    double m[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int64_t k = l;
    for (; k + 7 * nl < K; k += 8 * nl) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = row[k + q * nl];
#pragma unroll
        for (int q = 0; q < 8; ++q) m[q] = combine_max(m[q], abs_or_nan(v[q]));
    }
    for (; k < K; k += nl) m[0] = combine_max(m[0], abs_or_nan(row[k]));
#pragma unroll
    for (int q = 1; q < 8; ++q) m[0] = combine_max(m[0], m[q]);
    return m[0];
}

__global__ __launch_bounds__(256) void k_exponents2(OperandTask a, OperandTask b, uint32_t *flag) {
    __shared__ double part[4][64];
    const bool first = blockIdx.x < static_cast<unsigned>(a.eblocks);
    const OperandTask o = first ? a : b;
    const int blk = static_cast<int>(blockIdx.x) - (first ? 0 : a.eblocks);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (!o.trans) {
        if (o.wide) {  // one row per block: few rows, many columns
            const double m = row_max(o.X + blk * o.ld, o.K, threadIdx.x, 256);
            part[wave][lane] = m;
            __syncthreads();
            if (wave) return;
            double mu = combine_max(combine_max(part[0][lane], part[1][lane]), combine_max(part[2][lane], part[3][lane]));
            for (int off = 32; off >= 1; off >>= 1) mu = combine_max(mu, __shfl_xor(mu, off, 64));
            if (lane == 0) o.e[blk] = finish_exponent(mu, flag);
        } else {
            const int64_t r = static_cast<int64_t>(blk) * 4 + wave;
            if (r >= o.R) return;
            double mu = row_max(o.X + r * o.ld, o.K, lane, 64);
            for (int off = 32; off >= 1; off >>= 1) mu = combine_max(mu, __shfl_xor(mu, off, 64));
            if (lane == 0) o.e[r] = finish_exponent(mu, flag);
        }
        return;
    }
    const int strips = static_cast<int>((o.R + 63) / 64);
    const int chunk = blk / strips;
    const int64_t c = static_cast<int64_t>(blk - chunk * strips) * 64 + lane;
    const int64_t k0 = static_cast<int64_t>(chunk) * o.chunk;
    const int64_t k1 = k0 + o.chunk < o.K ? k0 + o.chunk : o.K;
    const double *col = o.X + (c < o.R ? c : o.R - 1);
    // the waves take every fourth row, sixteen loads in flight per lane
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t k = k0 + wave;
    for (; k + 60 < k1; k += 64) {
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = col[(k + 4 * q) * o.ld];
#pragma unroll
        for (int q = 0; q < 16; ++q) m[q & 3] = combine_max(m[q & 3], abs_or_nan(v[q]));
    }
    {
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = k + 4 * q < k1 ? col[(k + 4 * q) * o.ld] : 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) m[q & 3] = combine_max(m[q & 3], abs_or_nan(v[q]));
    }
    part[wave][lane] = combine_max(combine_max(m[0], m[1]), combine_max(m[2], m[3]));
    __syncthreads();
    if (wave || c >= o.R) return;
    const double mu = combine_max(combine_max(part[0][lane], part[1][lane]), combine_max(part[2][lane], part[3][lane]));
    o.codes[static_cast<int64_t>(chunk) * o.R + c] = mu != mu ? kEmaxNaN : mu == 0.0 ? kEmaxZero : shared_exponent(mu);
}

// Exponents of the groups stored as columns from their codes, for a long K:
// with more than kMaxCodeChunks codes per group every slice block's own
// reduction costs more than this launch.
constexpr int kMaxCodeChunks = 16;

// The exponent of a group's code: the code itself, 0 for an all-zero group,
// kExpBad for a non-finite one.
__device__ inline int32_t code_exponent(int32_t code) {
    return code == kEmaxNaN ? kExpBad : code == kEmaxZero ? 0 : code;
}

__global__ __launch_bounds__(256) void k_codes_final(OperandTask a, OperandTask b, uint32_t *flag) {
    const OperandTask &o = blockIdx.y ? b : a;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (!o.trans || r >= o.R) return;
    int32_t best = kEmaxZero;
    for (int q = 0; q < o.nchunk; ++q) best = max(best, o.codes[static_cast<int64_t>(q) * o.R + r]);
    const int32_t e = code_exponent(best);
    o.e[r] = e;
    if (e == kExpBad) atomicOr(flag, 1u);
}

template <int S>
__global__ __launch_bounds__(256) void k_slice2(OperandTask a, OperandTask b, uint32_t *flag) {
    __shared__ uint4 tile[S * 2][32];
    const bool first = blockIdx.x < static_cast<unsigned>(a.sblocks);
    const OperandTask o = first ? a : b;
    const int blk = static_cast<int>(blockIdx.x) - (first ? 0 : a.sblocks);
    const int gx = static_cast<int>(o.Rp / 32);
    const int64_t kb = blk / gx, r0 = static_cast<int64_t>(blk - kb * gx) * 32;
    if (!o.trans) {
        slice_tile<S, false>(tile, o.X, o.ld, o.R, o.K, o.e + r0, o.packed, o.Rp, r0, kb);
        return;
    }
    if (o.nchunk > kMaxCodeChunks) {
        slice_tile<S, true>(tile, o.X, o.ld, o.R, o.K, o.e + r0, o.packed, o.Rp, r0, kb);
        return;
    }
    // exponents of the 32 groups: eight threads share a group's chunks
    __shared__ int32_t code[8][32];
    __shared__ int32_t ex[32];
    const int r = threadIdx.x & 31, kq = threadIdx.x >> 5;
    int32_t best = kEmaxZero;
    if (r0 + r < o.R)
        for (int q = kq; q < o.nchunk; q += 8) best = max(best, o.codes[static_cast<int64_t>(q) * o.R + r0 + r]);
    code[kq][r] = best;
    __syncthreads();
    if (kq == 0) {
#pragma unroll
        for (int q = 1; q < 8; ++q) best = max(best, code[q][r]);
        const int32_t e = code_exponent(best);
        ex[r] = e;
        if (kb == 0 && r0 + r < o.R) {
            o.e[r0 + r] = e;
            if (e == kExpBad) atomicOr(flag, 1u);
        }
    }
    __syncthreads();
    slice_tile<S, true>(tile, o.X, o.ld, o.R, o.K, ex, o.packed, o.Rp, r0, kb);
}

// Both passes in one launch for short groups: a workgroup of four teams of 256
// threads takes 32 whole groups, its elements stay in registers between the
// maximum and the digits (K <= 128 NQ: NQ blocks of 32 per team), so X is
// read once.
template <int S, int NQ, bool TRANS>
__device__ inline void slice_groups(uint4 (*tile)[32], double (*part)[33], int32_t *ex, const OperandTask &o, int64_t r0,
                                    uint32_t *flag) {
    const int team = threadIdx.x >> 8, t = threadIdx.x & 255;
    const int nkb = static_cast<int>((o.K + kKB - 1) / kKB);
    double x[NQ][4];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (team + 4 * q < nkb) slice_load<TRANS>(x[q], o.X, o.ld, o.R, o.K, r0, team + 4 * q, t);
    double m0 = 0.0, m1 = 0.0;  // TRANS: m0 only; else rows r and r + 16
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (team + 4 * q >= nkb) continue;
        const double a = combine_max(abs_or_nan(x[q][0]), abs_or_nan(x[q][1]));
        const double b = combine_max(abs_or_nan(x[q][2]), abs_or_nan(x[q][3]));
        m0 = combine_max(m0, TRANS ? combine_max(a, b) : a);
        m1 = combine_max(m1, b);
    }
    if (TRANS) {
        part[threadIdx.x >> 5][t & 31] = m0;
    } else {
        for (int off = 8; off >= 1; off >>= 1) {
            m0 = combine_max(m0, __shfl_xor(m0, off, 64));
            m1 = combine_max(m1, __shfl_xor(m1, off, 64));
        }
        if ((t & 15) == 0) {
            part[team][t >> 4] = m0;
            part[team][(t >> 4) + 16] = m1;
        }
    }
    __syncthreads();
    if (threadIdx.x < 32) {
        const int r = threadIdx.x;
        double mu = 0.0;
        for (int q = 0; q < (TRANS ? 32 : 4); ++q) mu = combine_max(mu, part[q][r]);
        const int32_t e = r0 + r < o.R ? finish_exponent(mu, flag) : 0;
        ex[r] = e;
        if (r0 + r < o.R) o.e[r0 + r] = e;
    }
    __syncthreads();
    const int r = TRANS ? t & 31 : t >> 4;
    const int32_t e0 = ex[r], e1 = TRANS ? 0 : ex[r + 16];
    // every team runs the same barriers
    for (int q = 0; q < NQ; ++q) {
        if (4 * q >= nkb) break;
        const bool on = team + 4 * q < nkb;
        if (q) __syncthreads();
        double y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            y[i] = x[0][i];
#pragma unroll
            for (int p = 1; p < NQ; ++p) y[i] = q == p ? x[p][i] : y[i];
        }
        if (on) slice_digits<S, TRANS>(tile + team * S * 2, y, e0, e1, t);
        __syncthreads();
        if (on) slice_store<S>(tile + team * S * 2, o.packed, o.Rp, r0, team + 4 * q, t);
    }
}

template <int S, int NQ>
__global__ __launch_bounds__(1024) void k_slice_groups2(OperandTask a, OperandTask b, uint32_t *flag) {
    __shared__ uint4 tile[4 * S * 2][32];
    __shared__ double part[32][33];
    __shared__ int32_t ex[32];
    const int na = static_cast<int>(a.Rp / 32);
    const bool first = static_cast<int>(blockIdx.x) < na;
    const OperandTask o = first ? a : b;
    const int64_t r0 = static_cast<int64_t>(static_cast<int>(blockIdx.x) - (first ? 0 : na)) * 32;
    if (o.trans)
        slice_groups<S, NQ, true>(tile, part, ex, o, r0, flag);
    else
        slice_groups<S, NQ, false>(tile, part, ex, o, r0, flag);
}

// Longest group of the one-launch form.  96 x 160 x 200, S = 6: 6.3 us in one
// launch against 4.8 + 4.1 in two; at K = 512 the one form takes 12.4 us (16
// K blocks by one workgroup) against 5.1 + 6.2 over the whole chip.
constexpr int64_t kOnePassK = 256;

template <int S>
hipError_t slice_groups_s(const OperandTask &a, const OperandTask &b, uint32_t *flag, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>((a.Rp + b.Rp) / 32));
    hipLaunchKernelGGL((k_slice_groups2<S, 2>), grid, dim3(1024), 0, s, a, b, flag);
    return hipGetLastError();
}

template <int S>
hipError_t slice_s(bool trans, const double *X, int64_t ld, int64_t R, int64_t K,
                   const int32_t *e, int8_t *packed, int64_t Rp, hipStream_t s) {
    dim3 grid(static_cast<unsigned>(Rp / 32), static_cast<unsigned>(ceil_div(K, kKB)));
    if (trans)
        hipLaunchKernelGGL((k_slice<S, true>), grid, dim3(256), 0, s, X, ld, R, K, e, packed, Rp);
    else
        hipLaunchKernelGGL((k_slice<S, false>), grid, dim3(256), 0, s, X, ld, R, K, e, packed, Rp);
    return hipGetLastError();
}

// ---- grouped versions: one launch for a list of blocks -------------------
// Row groups (trans = 0): 16 rows per task, four per wave, the loads of the
// four rows interleaved so each lane keeps several in flight.
// Column groups (trans = 1): 64 columns per task, one per lane; the four
// waves take every fourth row of the block, eight loads in flight per lane,
// and combine their maxima through LDS.  The maximum is order independent
// (NaN wins), so the split does not change the exponents.

__global__ __launch_bounds__(256) void k_exponents_grouped(const SliceBlock *__restrict__ blocks,
                                                            const SliceTask *__restrict__ tasks,
                                                            const double *__restrict__ x_base,
                                                            int32_t *__restrict__ e_base,
                                                            uint32_t *flag, int32_t *emax_base) {
    __shared__ double part[4][kExpTaskCols];
    const SliceTask tk = tasks[blockIdx.x];
    const SliceBlock bl = blocks[tk.block];
    const double *X = x_base + bl.x_off;
    int32_t *e = e_base + bl.e_off;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (bl.trans == 0) {
        const int r0 = tk.a + wave * 4;
        double mu[4] = {0.0, 0.0, 0.0, 0.0};
        const double *row[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) row[j] = X + static_cast<int64_t>(r0 + j < bl.R ? r0 + j : 0) * bl.ld;
        // two elements of each of the 4 rows per iteration: 8 loads in flight per lane
        int k = lane;
        for (; k + 64 < bl.K; k += 128) {
            double v[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = r0 + j < bl.R;
                v[j][0] = ok ? row[j][k] : 0.0;
                v[j][1] = ok ? row[j][k + 64] : 0.0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mu[j] = combine_max(mu[j], combine_max(abs_or_nan(v[j][0]), abs_or_nan(v[j][1])));
        }
        if (k < bl.K) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (r0 + j < bl.R) mu[j] = combine_max(mu[j], abs_or_nan(row[j][k]));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double m = mu[j];
            for (int off = 32; off >= 1; off >>= 1) m = combine_max(m, __shfl_xor(m, off, 64));
            if (lane == 0 && r0 + j < bl.R) {
                if (!emax_base)
                    e[r0 + j] = finish_exponent(m, flag);
                else if (m != 0.0)
                    atomicMax(emax_base + bl.e_off + r0 + j, m != m ? kEmaxNaN : shared_exponent(m));
            }
        }
    } else {
        const int c = tk.a + lane;
        const bool cok = c < bl.R;
        const double *col = X + (cok ? c : 0);  // lanes past the edge load column 0 and drop it
        // rows [k0, k1): all of them, or one chunk of a split column task
        const int k0 = tk.b;
        const int k1 = tk.rows ? min(bl.K, k0 + tk.rows) : bl.K;
        double m8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) m8[u] = 0.0;
        // eight loads in flight; past the chunk its last row again
        for (int k = k0 + wave; k < k1; k += 32) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = col[static_cast<int64_t>(min(k + 4 * u, k1 - 1)) * bl.ld];
#pragma unroll
            for (int u = 0; u < 8; ++u) m8[u] = combine_max(m8[u], abs_or_nan(v[u]));
        }
        double mu = m8[0];
#pragma unroll
        for (int u = 1; u < 8; ++u) mu = combine_max(mu, m8[u]);
        part[wave][lane] = mu;
        __syncthreads();
        if (wave == 0) {
            mu = combine_max(combine_max(part[0][lane], part[1][lane]), combine_max(part[2][lane], part[3][lane]));
            if (cok) {
                if (!emax_base) {
                    e[c] = finish_exponent(mu, flag);
                } else if (mu != 0.0) {
                    // the code is monotone in the magnitude: the chunks' largest code is the column's
                    atomicMax(emax_base + bl.e_off + c, mu != mu ? kEmaxNaN : shared_exponent(mu));
                }
            }
        }
    }
}

// Exponents from the maxima a producing GEMM left in emax (one code per
// group, combined with atomic max), the flag for a non-finite group.  emax is
// reset to kEmaxZero for the next product.  Only the plans of several chunks
// need it: elsewhere the slice pass reads the codes itself (SliceCodes).
__global__ __launch_bounds__(256) void k_emax_finish(int32_t *__restrict__ emax, int32_t *__restrict__ e,
                                                      int64_t n, uint32_t *flag) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const int32_t x = code_exponent(emax[i]);
        if (x == kExpBad) atomicOr(flag, 1u);
        e[i] = x;
        emax[i] = kEmaxZero;
    }
}

// One task: 32 groups x up to kSliceTaskKB consecutive 32-wide K blocks; the
// elements of the next K block are loaded while the current one is sliced.

template <int S>
__global__ __launch_bounds__(256) void k_slice_grouped(const SliceBlock *__restrict__ blocks,
                                                        const SliceTask *__restrict__ tasks,
                                                        const double *__restrict__ x_base,
                                                        int32_t *__restrict__ e_base,
                                                        int8_t *__restrict__ p_base, SliceCodes codes) {
    __shared__ uint4 tile[S * 2][32];
    const SliceTask tk = tasks[blockIdx.x];
    const SliceBlock bl = blocks[tk.block];
    const double *X = x_base + bl.x_off;
    int32_t *e = e_base + bl.e_off;
    const int t = threadIdx.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + t; i < codes.n_reset; i += static_cast<int64_t>(gridDim.x) * 256)
        codes.reset[i] = kEmaxZero;
    // exponent of group g of the task's 32, also past the block's last group;
    // from a code it is stored by one lane (`owner`) of the first K blocks' task
    auto exponent = [&](int64_t g, bool owner) -> int32_t {
        if (!codes.emax) return g < bl.R ? e[g] : 0;
        const int32_t x = code_exponent(codes.emax[bl.e_off + g]);
        if (owner && tk.b == 0) {
            e[g] = x;
            if (x == kExpBad) atomicOr(codes.flag, 1u);
        }
        return x;
    };
    const int64_t r0 = tk.a;
    const int nkb = (bl.K + kKB - 1) / kKB;
    const int kb_end = tk.b + kSliceTaskKB < nkb ? tk.b + kSliceTaskKB : nkb;
    uint4 *out = reinterpret_cast<uint4 *>(p_base + bl.p_off);
    auto flush = [&](int kb) {
        __syncthreads();
        for (int q = t; q < S * 2 * 32; q += 256) {
            const int sc = q >> 5;
            const int rr = q & 31;
            out[(static_cast<int64_t>(kb) * S * 2 + sc) * bl.Rp + r0 + rr] = tile[sc][rr];
        }
        __syncthreads();
    };
    if (bl.trans) {
        // lanes take consecutive groups (columns): every load is coalesced
        const int r = t & 31, kq = t >> 5;
        const int64_t gr = r0 + r;
        const int32_t ee = exponent(gr, kq == 0);
        auto load = [&](int kb, double (&x)[4]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t k = static_cast<int64_t>(kb) * 32 + kq * 4 + q;
                x[q] = (gr < bl.R && k < bl.K) ? X[k * bl.ld + gr] : 0.0;
            }
        };
        double x[4], nx[4];
        load(tk.b, x);
        const int c = kq >> 2, word = kq & 3;
        for (int kb = tk.b; kb < kb_end; ++kb) {
            if (kb + 1 < kb_end) load(kb + 1, nx);
            uint32_t w[S];
            slice4<S>(x, ee, w);
#pragma unroll
            for (int s = 0; s < S; ++s) reinterpret_cast<uint32_t *>(&tile[s * 2 + c][r])[word] = w[s];
            flush(kb);
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = nx[q];
        }
        return;
    }
    // row groups: 16 lanes per row, two consecutive elements each (one
    // 16-byte load when aligned and inside the block), rows r and r + 16;
    // the two bytes per slice of a lane pair make one word of the tile
    const int kp = t & 15;
    const int rA = t >> 4;
    const bool aligned = (bl.ld & 1) == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
    int32_t ee[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) ee[h] = exponent(r0 + rA + 16 * h, kp == 0);
    auto load = [&](int kb, double (&x)[4]) {
        const int64_t k = static_cast<int64_t>(kb) * 32 + 2 * kp;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t gr = r0 + rA + 16 * h;
            x[2 * h] = 0.0;
            x[2 * h + 1] = 0.0;
            if (gr < bl.R) {
                if (aligned && k + 1 < bl.K) {
                    const double2 v = *reinterpret_cast<const double2 *>(X + gr * bl.ld + k);
                    x[2 * h] = v.x;
                    x[2 * h + 1] = v.y;
                } else {
                    if (k < bl.K) x[2 * h] = X[gr * bl.ld + k];
                    if (k + 1 < bl.K) x[2 * h + 1] = X[gr * bl.ld + k + 1];
                }
            }
        }
    };
    double x[4], nx[4];
    load(tk.b, x);
    const int kq = kp >> 1, c = kq >> 2, word = kq & 3;
    for (int kb = tk.b; kb < kb_end; ++kb) {
        if (kb + 1 < kb_end) load(kb + 1, nx);
#pragma unroll
        for (int h = 0; h < 2; ++h) slice2_store<S>(tile, x[2 * h], x[2 * h + 1], ee[h], c, rA + 16 * h, word);
        flush(kb);
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = nx[q];
    }
}

// Debug layout conversions, one byte per thread.
__global__ void k_pack(int S, const int8_t *__restrict__ canon, int64_t R, int64_t K,
                       int8_t *__restrict__ packed, int64_t Rp, int64_t Kp) {
    const int64_t total = static_cast<int64_t>(S) * Rp * Kp;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t s = i / (Rp * Kp);
        const int64_t r = (i / Kp) % Rp;
        const int64_t k = i % Kp;
        const int8_t v = (r < R && k < K) ? canon[(s * R + r) * K + k] : int8_t(0);
        packed[((k / 32 * S + s) * 2 + (k / 16) % 2) * Rp * 16 + r * 16 + k % 16] = v;
    }
}

__global__ void k_unpack(int S, const int8_t *__restrict__ packed, int64_t Rp, int64_t R,
                         int64_t K, int8_t *__restrict__ canon) {
    const int64_t total = static_cast<int64_t>(S) * R * K;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t s = i / (R * K);
        const int64_t r = (i / K) % R;
        const int64_t k = i % K;
        canon[i] = packed[((k / 32 * S + s) * 2 + (k / 16) % 2) * Rp * 16 + r * 16 + k % 16];
    }
}

__global__ void k_diag_axpy(const double *__restrict__ diag, const double *__restrict__ psi,
                            double *__restrict__ sigma, int64_t n) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const double p = diag[i] * psi[i];
        sigma[i] = sigma[i] + p;
    }
}

unsigned grid_for(int64_t n, int64_t per_block, unsigned cap) {
    const int64_t g = ceil_div(n, per_block);
    return static_cast<unsigned>(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

hipError_t launch_row_exponents(const double *X, int64_t ld, int64_t R, int64_t K, int32_t *e,
                                uint32_t *flag, hipStream_t s) {
    if (R == 0) return hipSuccess;
    hipLaunchKernelGGL(k_row_exponents, dim3(static_cast<unsigned>(ceil_div(R, 4))), dim3(256), 0,
                       s, X, ld, R, K, e, flag);
    return hipGetLastError();
}

size_t col_exponent_scratch(int64_t K, int64_t R) {
    const int64_t nchunk = ceil_div(K, kColChunk) < 1 ? 1 : ceil_div(K, kColChunk);
    return static_cast<size_t>(nchunk * R) * sizeof(double);
}

hipError_t launch_col_exponents(const double *X, int64_t ld, int64_t K, int64_t R, int32_t *e,
                                double *part, uint32_t *flag, hipStream_t s) {
    if (R == 0) return hipSuccess;
    const int64_t nchunk = ceil_div(K, kColChunk);
    if (nchunk > 0) {
        hipLaunchKernelGGL(k_col_partial,
                           dim3(static_cast<unsigned>(ceil_div(R, 256)), static_cast<unsigned>(nchunk)),
                           dim3(256), 0, s, X, ld, K, R, part);
    }
    hipLaunchKernelGGL(k_col_final, dim3(static_cast<unsigned>(ceil_div(R, 256))), dim3(256), 0, s,
                       part, nchunk, R, e, flag);
    return hipGetLastError();
}

hipError_t launch_group_sumsq(bool by_rows, const double *X, int64_t ld, int64_t R, int64_t K, double *ss,
                              double *part, hipStream_t s) {
    if (R == 0) return hipSuccess;
    if (by_rows) {
        hipLaunchKernelGGL(k_row_sumsq, dim3(static_cast<unsigned>(ceil_div(R, 4))), dim3(256), 0, s, X, ld, R, K, ss);
        return hipGetLastError();
    }
    const int64_t nchunk = ceil_div(K, kColChunk);
    if (nchunk > 0)
        hipLaunchKernelGGL(k_col_sumsq_partial,
                           dim3(static_cast<unsigned>(ceil_div(R, 256)), static_cast<unsigned>(nchunk)), dim3(256), 0, s,
                           X, ld, K, R, part);
    hipLaunchKernelGGL(k_col_sumsq_final, dim3(static_cast<unsigned>(ceil_div(R, 256))), dim3(256), 0, s, part, nchunk,
                       R, ss);
    return hipGetLastError();
}

hipError_t launch_slice(int S, bool trans, const double *X, int64_t ld, int64_t R, int64_t K,
                        const int32_t *e, int8_t *packed, int64_t Rp, hipStream_t s) {
    if (Rp == 0 || K == 0) return hipSuccess;
    switch (S) {
        case 2: return slice_s<2>(trans, X, ld, R, K, e, packed, Rp, s);
        case 3: return slice_s<3>(trans, X, ld, R, K, e, packed, Rp, s);
        case 4: return slice_s<4>(trans, X, ld, R, K, e, packed, Rp, s);
        case 5: return slice_s<5>(trans, X, ld, R, K, e, packed, Rp, s);
        case 6: return slice_s<6>(trans, X, ld, R, K, e, packed, Rp, s);
        case 7: return slice_s<7>(trans, X, ld, R, K, e, packed, Rp, s);
        case 8: return slice_s<8>(trans, X, ld, R, K, e, packed, Rp, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_slice_operands(int S, OperandTask a, OperandTask b, int32_t *codes, int num_cu, uint32_t *flag,
                                 hipStream_t s) {
    if (a.K <= kOnePassK) {
        switch (S) {
            case 2: return slice_groups_s<2>(a, b, flag, s);
            case 3: return slice_groups_s<3>(a, b, flag, s);
            case 4: return slice_groups_s<4>(a, b, flag, s);
            case 5: return slice_groups_s<5>(a, b, flag, s);
            case 6: return slice_groups_s<6>(a, b, flag, s);
            case 7: return slice_groups_s<7>(a, b, flag, s);
            case 8: return slice_groups_s<8>(a, b, flag, s);
            default: return hipErrorInvalidValue;
        }
    }
    // rows of a column chunk: 256 when both operands need codes (their scratch
    // holds ceil(K / 256) codes for each of the larger one's groups twice),
    // 128 when one does; more for a long K, at most 32 chunks.  Every slice
    // block reduces up to kMaxCodeChunks codes itself: K <= 2048 with one
    // operand in codes, K <= 4096 with both; past that k_codes_final does
    const int64_t base = a.trans && b.trans ? 256 : 128;
    int64_t at = 0;
    for (OperandTask *o : {&a, &b}) {
        if (o->trans) {
            o->chunk = static_cast<int32_t>(std::max(base, round_up(ceil_div(o->K, 32), base)));
            o->nchunk = static_cast<int32_t>(ceil_div(o->K, o->chunk));
            o->codes = codes + at;
            at += static_cast<int64_t>(o->nchunk) * o->R;
            o->eblocks = static_cast<int32_t>(ceil_div(o->R, 64)) * o->nchunk;
        } else {
            // a block per row while a wave per row would not give every
            // compute unit four blocks and the rows are long enough to share
            o->wide = o->R < 16 * static_cast<int64_t>(num_cu) && o->K >= 1024;
            o->eblocks = static_cast<int32_t>(o->wide ? o->R : ceil_div(o->R, 4));
        }
        o->sblocks = static_cast<int32_t>(o->Rp / 32 * ceil_div(o->K, kKB));
    }
    hipLaunchKernelGGL(k_exponents2, dim3(a.eblocks + b.eblocks), dim3(256), 0, s, a, b, flag);
    if (std::max(a.nchunk, b.nchunk) > kMaxCodeChunks)
        hipLaunchKernelGGL(k_codes_final, dim3(static_cast<unsigned>(ceil_div(std::max(a.R, b.R), 256)), 2), dim3(256),
                           0, s, a, b, flag);
    const dim3 grid(a.sblocks + b.sblocks);
    switch (S) {
        case 2: hipLaunchKernelGGL(k_slice2<2>, grid, dim3(256), 0, s, a, b, flag); break;
        case 3: hipLaunchKernelGGL(k_slice2<3>, grid, dim3(256), 0, s, a, b, flag); break;
        case 4: hipLaunchKernelGGL(k_slice2<4>, grid, dim3(256), 0, s, a, b, flag); break;
        case 5: hipLaunchKernelGGL(k_slice2<5>, grid, dim3(256), 0, s, a, b, flag); break;
        case 6: hipLaunchKernelGGL(k_slice2<6>, grid, dim3(256), 0, s, a, b, flag); break;
        case 7: hipLaunchKernelGGL(k_slice2<7>, grid, dim3(256), 0, s, a, b, flag); break;
        case 8: hipLaunchKernelGGL(k_slice2<8>, grid, dim3(256), 0, s, a, b, flag); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_exponents_grouped(const SliceBlock *blocks, const SliceTask *tasks, int ntasks,
                                    const double *x_base, int32_t *e_base, uint32_t *flag,
                                    hipStream_t s, int32_t *emax_base) {
    if (ntasks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_exponents_grouped, dim3(ntasks), dim3(256), 0, s, blocks, tasks, x_base,
                       e_base, flag, emax_base);
    return hipGetLastError();
}

hipError_t launch_emax_finish(int32_t *emax, int32_t *e, int64_t n, uint32_t *flag, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_emax_finish, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, emax, e, n, flag);
    return hipGetLastError();
}

hipError_t launch_slice_grouped(int S, const SliceBlock *blocks, const SliceTask *tasks, int ntasks,
                                const double *x_base, int32_t *e_base, int8_t *p_base,
                                hipStream_t s, const SliceCodes &codes) {
    if (ntasks == 0) return hipSuccess;
#define OZ_SG(S_)                                                                                \
    case S_:                                                                                     \
        hipLaunchKernelGGL(k_slice_grouped<S_>, dim3(ntasks), dim3(256), 0, s, blocks, tasks,    \
                           x_base, e_base, p_base, codes);                                      \
        break;
    switch (S) {
        OZ_SG(2) OZ_SG(3) OZ_SG(4) OZ_SG(5) OZ_SG(6) OZ_SG(7) OZ_SG(8)
        default: return hipErrorInvalidValue;
    }
#undef OZ_SG
    return hipGetLastError();
}

hipError_t launch_pack(int S, const int8_t *canon, int64_t R, int64_t K, int8_t *packed,
                       int64_t Rp, hipStream_t s) {
    const int64_t Kp = round_up(K, kKB);
    const int64_t total = static_cast<int64_t>(S) * Rp * Kp;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack, dim3(grid_for(total, 256, 65535)), dim3(256), 0, s, S, canon, R, K,
                       packed, Rp, Kp);
    return hipGetLastError();
}

hipError_t launch_unpack(int S, const int8_t *packed, int64_t Rp, int64_t R, int64_t K,
                         int8_t *canon, hipStream_t s) {
    const int64_t total = static_cast<int64_t>(S) * R * K;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpack, dim3(grid_for(total, 256, 65535)), dim3(256), 0, s, S, packed, Rp,
                       R, K, canon);
    return hipGetLastError();
}

hipError_t launch_diag_axpy(const double *diag, const double *psi, double *sigma, int64_t n,
                            hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_diag_axpy, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, diag, psi,
                       sigma, n);
    return hipGetLastError();
}

}  // namespace oz
