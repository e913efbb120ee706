// Orthonormal factor of a square FP64 matrix by Cholesky QR: the
// preconditioner of the block-Jacobi eigensolver (rdm.hip) is one step of QR
// iteration, M -> Q^T M Q with Q R = M + mu I, and only Q is needed.
//
// One pass takes X (np x np) and its Gram matrix G = X^T X = L L^T and
// returns Q = X L^-T.  G and X are eliminated together, 64 columns at a time,
// as one tall matrix [G; X] (right-looking): the Cholesky factor's panel and
// Q's panel are the same product with the inverse of the diagonal block, and
// one trailing update serves both.  A second pass on Q restores the
// orthogonality that forming G lost (about cond(X)^2 u after the first, a few
// u after the second).
//
// Per 64 columns: the Cholesky factor and inverse of the 64 x 64 diagonal block
// (one workgroup, a chain of 64 dependent steps), k_cq_panel and k_cq_update
// (64 x 64 tiles on the FP64 matrix cores), the next diagonal block beside the
// update.  Bound: the chain of the diagonal block and two dependent launches
// per 64 columns, not arithmetic (4/3 n^3 flop a pass).
#include "internal.h"
#include "tile64.h"

namespace oz {
namespace {

// 1 / w to one rounding error: the hardware's estimate (about 2^-23) with one
// third-order correction.
__device__ __forceinline__ double reciprocal(double w) {
    const double y = __builtin_amdgcn_rcp(w);
    const double e = fma(-w, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

constexpr int kDiagLds = 5 * 64;  // doubles

// Cholesky of a 64 x 64 block, element (r, c) = at(r, c), the inverse of its
// factor into Linv (64 x 64 row-major).  Symmetric elimination of [G | I]:
// thread (ti, tj) holds rows ti + 16 a and columns tj + 16 b of both halves
// in registers; a step broadcasts column k of G and row k of the other half
// through LDS (double-buffered, one barrier a step).  A pivot outside
// (lo, hi) sets *bad and is replaced by 1, so every step stays finite.  Bound:
// the chain of 64 steps (broadcast, reciprocal, update), so the pivots' square
// roots wait for the end (32 us with them and an exact division inside,
// 30 without).
template <typename At>
__device__ __forceinline__ void cq_diag(At at, double *__restrict__ Linv, int *__restrict__ bad, double lo, double hi,
                                        double *lds) {
    double (*col)[64] = reinterpret_cast<double (*)[64]>(lds), (*vrow)[64] = col + 2, *piv = lds + 256;
    const int ti = threadIdx.x >> 4, tj = threadIdx.x & 15;
    double g[4][4], v[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int r = ti + 16 * a, c = tj + 16 * b;
            g[a][b] = at(r, c);
            v[a][b] = r == c ? 1.0 : 0.0;
        }
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) {
#pragma unroll 1
        for (int kr = 0; kr < 16; ++kr) {
            const int k = 16 * kq + kr, p = k & 1;
            if (tj == kr) {
#pragma unroll
                for (int a = 0; a < 4; ++a) col[p][ti + 16 * a] = g[a][kq];
            }
            if (ti == kr) {
#pragma unroll
                for (int b = 0; b < 4; ++b) vrow[p][tj + 16 * b] = v[kq][b];
            }
            __syncthreads();
            double w = col[p][k];
            if (!(w > lo && w < hi)) {
                if (threadIdx.x == 0) atomicOr(bad, 1);
                w = 1.0;
            }
            if (threadIdx.x == 0) piv[k] = w;
            const double inv = reciprocal(w);
            double f[4], gc[4], vc[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) f[a] = ti + 16 * a > k ? col[p][ti + 16 * a] * inv : 0.0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                gc[b] = col[p][tj + 16 * b];
                vc[b] = vrow[p][tj + 16 * b];
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    g[a][b] = fma(-f[a], gc[b], g[a][b]);
                    v[a][b] = fma(-f[a], vc[b], v[a][b]);
                }
        }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const double dinv = 1.0 / sqrt(piv[ti + 16 * a]);
#pragma unroll
        for (int b = 0; b < 4; ++b) Linv[(ti + 16 * a) * 64 + tj + 16 * b] = v[a][b] * dinv;
    }
}

// The first diagonal block (the others follow their update).
__global__ __launch_bounds__(256) void k_cq_diag(const double *__restrict__ G, int64_t ld, double *__restrict__ Linv,
                                                 int *__restrict__ bad, double lo, double hi) {
    __shared__ double lds[kDiagLds];
    cq_diag([&](int r, int c) { return G[r * ld + c]; }, Linv, bad, lo, hi, lds);
}

// Column block k of the factor: rows of G below the diagonal block into P
// (64 x 64 tiles, one after the other), rows of X into Q, each times Linv^T.
__global__ __launch_bounds__(256) void k_cq_panel(const double *__restrict__ G, const double *__restrict__ X,
                                                  double *__restrict__ Q, double *__restrict__ P,
                                                  const double *__restrict__ Linv, int64_t np, int k) {
    __shared__ double sA[64 * t64::kLdK], sB[64 * t64::kLdK];
    const int below = static_cast<int>(np / 64) - k - 1;
    const int i = blockIdx.x;
    const bool top = i < below;
    const int64_t row = static_cast<int64_t>(top ? k + 1 + i : i - below) * 64;
    t64::load(sA, t64::kLdK, (top ? G : X) + row * np + static_cast<int64_t>(k) * 64, np);
    t64::load(sB, t64::kLdK, Linv, 64);
    __syncthreads();
    t64::Acc acc;
    acc.zero();
    t64::mul_nt(acc, sA, sB);
    double *out = top ? P + static_cast<int64_t>(i) * 4096 : Q + row * np + static_cast<int64_t>(k) * 64;
    const int64_t ldo = top ? 64 : np;
    t64::each(acc, [&](int r, int c, double x) { out[r * ldo + c] = x; });
}

// Trailing update: tile (i, j) of [G; X] right of column block k loses
// P_i P_j^T (rows of Q in the place of P_i for X's rows).  Tiles of G above
// the diagonal are never read and are left alone.  The first workgroup's tile
// is the next diagonal block: it goes on to factorise it beside the others'
// tiles, a chain that would otherwise leave the chip idle between this launch
// and the next panel's.
__global__ __launch_bounds__(256) void k_cq_update(double *__restrict__ G, double *__restrict__ X,
                                                   const double *__restrict__ Q, const double *__restrict__ P,
                                                   int64_t np, int k, double *__restrict__ Linv, int *__restrict__ bad,
                                                   double lo, double hi) {
    __shared__ double sA[64 * t64::kLdK], sB[64 * t64::kLdK];
    const int below = static_cast<int>(np / 64) - k - 1;
    const int j = blockIdx.x, i = blockIdx.y;
    const bool top = i < below;
    if (top && i < j) return;
    const bool next = i == 0 && j == 0;  // (top: this launch has below > 0)
    const int64_t row = static_cast<int64_t>(top ? k + 1 + i : i - below) * 64;
    if (top)
        t64::load(sA, t64::kLdK, P + static_cast<int64_t>(i) * 4096, 64);
    else
        t64::load(sA, t64::kLdK, Q + row * np + static_cast<int64_t>(k) * 64, np);
    t64::load(sB, t64::kLdK, P + static_cast<int64_t>(j) * 4096, 64);
    double *c = (top ? G : X) + row * np + static_cast<int64_t>(k + 1 + j) * 64;
    __syncthreads();
    t64::Acc acc;
    acc.zero();
    t64::mul_nt(acc, sA, sB);
    if (!next) {
        t64::each(acc, [&](int r, int cc, double x) { c[r * np + cc] -= x; });
        return;
    }
    __syncthreads();
    t64::each(acc, [&](int r, int cc, double x) { sA[r * t64::kLdK + cc] = c[r * np + cc] - x; });  // nothing else reads it
    __syncthreads();
    cq_diag([&](int r, int cc) { return sA[r * t64::kLdK + cc]; }, Linv, bad, lo, hi, sB);
}

// B = A + mu I in the leading n x n part, `unit` on the padded diagonal, 0 elsewhere
__global__ __launch_bounds__(256) void k_cq_shift(const double *__restrict__ A, int64_t lda, int64_t n, int64_t np,
                                                  double mu, double unit, double *__restrict__ B) {
    const int64_t r = blockIdx.y;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; c < np;
         c += static_cast<int64_t>(gridDim.x) * 256) {
        double x = 0.0;
        if (r < n && c < n)
            x = A[r * lda + c] + (r == c ? mu : 0.0);
        else if (r == c)
            x = unit;
        B[r * np + c] = x;
    }
}

}  // namespace

hipError_t launch_shifted_copy(const double *A, int64_t lda, int64_t n, int64_t np, double mu, double unit, double *B,
                               hipStream_t s) {
    const unsigned gx = static_cast<unsigned>(ceil_div(np, 256));
    hipLaunchKernelGGL(k_cq_shift, dim3(gx, static_cast<unsigned>(np)), dim3(256), 0, s, A, lda, n, np, mu, unit, B);
    return hipGetLastError();
}

hipError_t launch_cholqr_pass(double *G, double *X, double *Q, double *P, double *Linv, int64_t np, int *bad,
                              double lo, double hi, int num_cu, hipStream_t s) {
    Dgemm64Args a{};
    a.term = Term64{X, X, np, np, static_cast<int32_t>(np), 0, 1.0};
    a.out = OutDesc{G, np, static_cast<int32_t>(np), static_cast<int32_t>(np)};
    a.mode = kModeGemm;
    hipError_t e = launch_dgemm_single(true, false, a, num_cu, s);  // G = X^T X
    if (e != hipSuccess) return e;
    const int nb = static_cast<int>(np / 64);
    hipLaunchKernelGGL(k_cq_diag, dim3(1), dim3(256), 0, s, G, np, Linv, bad, lo, hi);
    for (int k = 0; k < nb; ++k) {
        const int below = nb - k - 1;
        hipLaunchKernelGGL(k_cq_panel, dim3(below + nb), dim3(256), 0, s, G, X, Q, P, Linv, np, k);
        if (below > 0)
            hipLaunchKernelGGL(k_cq_update, dim3(below, below + nb), dim3(256), 0, s, G, X, Q, P, np, k, Linv, bad,
                               lo, hi);
    }
    return hipGetLastError();
}

}  // namespace oz
