// Davidson iteration for the lowest eigenpair of H_eff (the Krylov solver of
// the second DMRG subroutine, "Theory of TNS/DMRG"; stopped on the residual
// norm as in "Numerical procedure").  The matvec is heff_apply (emulated or
// native); everything else runs in FP64 on the device:
//
//   Rayleigh-Ritz   one-workgroup cyclic Jacobi (round-robin ordering, all
//                   disjoint rotations of a round applied together) on the
//                   m x m projected matrix, m <= 64;
//   Ritz vector     x = V^T y, Hx = W^T y, r = Hx - theta x, rho = |r|;
//   correction      t = r / (diag(H) - theta), |den| >= 1e-8;
//   orthogonalise   classical Gram-Schmidt twice against V, fall back to r
//                   when |t| < 1e-10, normalise;
//   expand          W[m] = H V[m] and the new column of V^T W.
//
// All reductions use a fixed partition and a fixed tree, so a run is
// bit-reproducible.  The host reads (theta, rho) once per step.
//
// A step's vector work is bound by reading V three times and W once (0.15 ms
// of memory traffic at m = 13, n = 2^20) and, for small bases, by one launch
// of 4 to 5 us after another.  So a reduction ends in its consumer: blocks
// write partials, and the kernel that needs the sum adds the 512 partials
// itself (k_project, k_normalise, k_jacobi, k_publish) instead of waiting for
// a one-block launch, and copies ride in passes that hold the values anyway.
// At n = 2^20, m = 13: k_jacobi 91 -> 77 us (groups of lanes sized to a row;
// with one wave per pair 107), dot products 36 -> 19 us, projections 17 + 5 ->
// 25 us including the norm, Ritz vectors 103 -> 62 us (4.3 TB/s, eight loads in
// flight); a Davidson step of 0.3 ms besides its matvec loses 8 launches and a
// copy, a Lanczos solve at n = 9216 goes from 1.25 to 1.04 ms.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "rotation.h"
#include "runtime.h"

using namespace oz;

namespace {

constexpr int kDotThreads = 256;

int dot_blocks(int64_t n) {
    const int64_t b = ceil_div(n, kDotThreads * 4);
    return static_cast<int>(b < 1 ? 1 : (b > 512 ? 512 : b));
}

__device__ inline double block_sum(double v, double *sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (t < s) sh[t] += sh[t + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Basis size of a launch: a host value, or (dev set) the device's, so that one
// captured Davidson step serves every basis size.  A full basis (full set)
// counts as one vector: the step that finds it full starts by collapsing it
// to the Ritz pair.
struct BasisSize {
    int m;
    const int *dev;
    int full;
    __device__ int get() const {
        const int k = dev ? *dev : m;
        return full && k == full ? 1 : k;
    }
};

// partial[row][blk] = sum over this block's share of A[row][i] * v[i], rows
// below the basis size + add (the grid covers the largest count).  With copy
// set, the blocks of row 0 also store v as row `basis size` of copy.
__global__ __launch_bounds__(kDotThreads) void k_dots_partial(const double *__restrict__ A, int64_t lda, const double *__restrict__ v,
                                                              int64_t n, double *__restrict__ partial, const int *gate,
                                                              BasisSize size, int add, double *__restrict__ copy) {
    if (gate && *gate == 0) return;
    const int m = size.get();
    if (static_cast<int>(blockIdx.y) >= m + add) return;
    __shared__ double sh[kDotThreads];
    const int row = blockIdx.y;
    const double *a = A + row * lda;
    double *c = copy && row == 0 ? copy + m * n : nullptr;
    const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
    double acc = 0.0;
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    // four elements of each vector in flight, summed in order
    for (; i + 3 * step < n; i += 4 * step) {
        double x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[q] = a[i + q * step];
            y[q] = v[i + q * step];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc = fma(x[q], y[q], acc);
            if (c) c[i + q * step] = y[q];
        }
    }
    for (; i < n; i += step) {
        acc = fma(a[i], v[i], acc);
        if (c) c[i] = v[i];
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[static_cast<int64_t>(row) * gridDim.x + blockIdx.x] = s;
}

// Sum of one row's partials (nblk <= 512) by one wave, in the order of
// block_sum over 256 threads that each add partials t and t + 256.  All lanes
// get it.
__device__ inline double partials_sum(const double *__restrict__ p, int nblk) {
    const int l = threadIdx.x & 63;
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int t = l + 64 * q;
        double acc = 0.0;
        if (t < nblk) acc += p[t];
        if (t + 256 < nblk) acc += p[t + 256];
        v[q] = acc;
    }
    double s = (v[0] + v[2]) + (v[1] + v[3]);
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_down(s, o, 64);
    return __shfl(s, 0, 64);
}

// out[row] = sum of the row's partials (start vectors; the steps' consumers
// sum the partials themselves)
__global__ __launch_bounds__(64) void k_dots_final(const double *__restrict__ partial, int nblk, double *out) {
    const double s = partials_sum(partial + static_cast<int64_t>(blockIdx.x) * nblk, nblk);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// The new row and column of G from the partials of V[i] . W[m], i <= m, then
// the lowest eigenpair of the (m + 1) x (m + 1) matrix G (leading dimension
// ldg) by cyclic Jacobi with the round-robin pairing; writes theta, y (largest
// |y_i| made positive) and the new basis size.  With nblk = 0 G is complete
// and of size m.  One workgroup of 256 threads, m + 1 <= 64.
// Groups of 16, 32 or 64 lanes (the smallest that holds a row) share a round's
// pairs: a group computes its pairs' rotations, sweeps the columns of rows p,
// q (no other group touches those rows) and, after a barrier, the rows of
// columns p, q.  Bound: the chain of rounds (a rotation, two passes through
// LDS, two barriers).
__global__ __launch_bounds__(256) void k_jacobi(double *__restrict__ G, int ldg, BasisSize size, int *m_dev,
                                                const double *__restrict__ partial, int nblk, double *__restrict__ y,
                                                double *__restrict__ theta_out) {
    __shared__ double A[64][65];
    __shared__ double Vv[64][65];
    __shared__ double red[256];
    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63;
    const int old = size.get();
    const int m = old + (nblk ? 1 : 0);
    for (int r = wave; r < m; r += 4)
        if (lane < m) {
            if (!nblk || (r < old && lane < old)) A[r][lane] = G[r * ldg + lane];
            Vv[r][lane] = r == lane ? 1.0 : 0.0;
        }
    if (nblk) {
        for (int r = wave; r < m; r += 4) {
            const double s = partials_sum(partial + static_cast<int64_t>(r) * nblk, nblk);
            if (lane == 0) {
                A[r][old] = s;
                A[old][r] = s;
                G[r * ldg + old] = s;
                G[old * ldg + r] = s;
            }
        }
        __syncthreads();  // every thread has read the old basis size
        if (t == 0) *m_dev = m;
    }
    __syncthreads();
    const int me = (m + 1) & ~1;  // even number of players (one dummy when m is odd)
    const int gs = m <= 16 ? 16 : m <= 32 ? 32 : 64, ngrp = 256 / gs, grp = t / gs, sub = t % gs;
    for (int sweep = 0; sweep < 30 && m > 1; ++sweep) {
        // convergence test: off(A) <= 1e-14 ||A||_F
        double off = 0.0, tot = 0.0;
        for (int r = wave; r < m; r += 4)
            if (lane < m) {
                const double v = A[r][lane] * A[r][lane];
                tot += v;
                if (r != lane) off += v;
            }
        for (int o = 32; o >= 1; o >>= 1) {
            off += __shfl_xor(off, o, 64);
            tot += __shfl_xor(tot, o, 64);
        }
        if (lane == 0) {
            red[wave] = off;
            red[4 + wave] = tot;
        }
        __syncthreads();
        off = (red[0] + red[1]) + (red[2] + red[3]);
        tot = (red[4] + red[5]) + (red[6] + red[7]);
        __syncthreads();
        if (sqrt(off) <= 1e-14 * sqrt(tot)) break;
        for (int round = 0; round < me - 1; ++round) {
            // round-robin: player me-1 fixed, the others rotate; pair k of the
            // round is (p, q), idle when q is the dummy
            auto pair = [&](int k, int *p, int *q) {
                int a = me - 1, b = round;
                if (k > 0) {
                    a = round + k;
                    a = a >= me - 1 ? a - (me - 1) : a;
                    b = round - k;
                    b = b < 0 ? b + me - 1 : b;
                }
                *p = a < b ? a : b;
                *q = a < b ? b : a;
            };
            double cl = 1.0, sl = 0.0;
            {
                const int k = grp + ngrp * (sub & 7);
                int p, q;
                pair(k, &p, &q);
                if (k < me / 2 && q < m) schur_rotation(A[p][p], A[q][q], A[p][q], &cl, &sl);
            }
            for (int i = 0, k = grp; i * ngrp < me / 2; ++i, k += ngrp) {  // rows: A <- J^T A
                int p, q;
                pair(k, &p, &q);
                const double c = __shfl(cl, lane - sub + i, 64), s = __shfl(sl, lane - sub + i, 64);
                if (k >= me / 2 || q >= m || sub >= m) continue;
                const double ap = A[p][sub], aq = A[q][sub];
                A[p][sub] = c * ap - s * aq;
                A[q][sub] = s * ap + c * aq;
            }
            __syncthreads();
            for (int i = 0, k = grp; i * ngrp < me / 2; ++i, k += ngrp) {  // columns: A <- A J, V <- V J
                int p, q;
                pair(k, &p, &q);
                const double c = __shfl(cl, lane - sub + i, 64), s = __shfl(sl, lane - sub + i, 64);
                if (k >= me / 2 || q >= m || sub >= m) continue;
                const double ap = A[sub][p], aq = A[sub][q];
                const double vp = Vv[sub][p], vq = Vv[sub][q];
                A[sub][p] = c * ap - s * aq;
                A[sub][q] = s * ap + c * aq;
                Vv[sub][p] = c * vp - s * vq;
                Vv[sub][q] = s * vp + c * vq;
            }
            __syncthreads();
        }
    }
    if (t == 0) {
        int best = 0;
        for (int i = 1; i < m; ++i)
            if (A[i][i] < A[best][best]) best = i;
        int big = 0;
        for (int i = 1; i < m; ++i)
            if (fabs(Vv[i][best]) > fabs(Vv[big][best])) big = i;
        const double sgn = Vv[big][best] < 0 ? -1.0 : 1.0;
        for (int i = 0; i < m; ++i) y[i] = sgn * Vv[i][best];
        *theta_out = A[best][best];
    }
}

// x = V^T y, hx = W^T y, r = hx - theta x, partial sums of r^2.
__global__ __launch_bounds__(kDotThreads) void k_ritz(const double *__restrict__ V, const double *__restrict__ W, int64_t n,
                                                      const int *m_dev, const double *__restrict__ y, const double *__restrict__ theta,
                                                      double *__restrict__ x, double *__restrict__ hx, double *__restrict__ r,
                                                      double *__restrict__ partial) {
    const int m = *m_dev;
    __shared__ double sh[kDotThreads];
    const double th = *theta;
    double acc = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        double xi = 0.0, hi = 0.0;
        int j = 0;
        for (; j + 4 <= m; j += 4) {  // eight loads in flight, summed in order
            double a[4], b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[q] = V[(j + q) * n + i];
                b[q] = W[(j + q) * n + i];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                xi = fma(y[j + q], a[q], xi);
                hi = fma(y[j + q], b[q], hi);
            }
        }
        for (; j < m; ++j) {
            xi = fma(y[j], V[j * n + i], xi);
            hi = fma(y[j], W[j * n + i], hi);
        }
        const double ri = hi - th * xi;
        x[i] = xi;
        hx[i] = hi;
        r[i] = ri;
        acc = fma(ri, ri, acc);
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The start of a continuing step: t = r / (diag(H) - theta), |den| >= 1e-8.
// A full basis (*m_dev == full) collapses to the Ritz pair: V[0] = x, W[0] =
// hx, G = [theta] and zero elsewhere; the size stays `full` until k_jacobi
// sets the new one, and the kernels between count it as one (BasisSize).
__global__ __launch_bounds__(256) void k_begin(const double *__restrict__ r, const double *__restrict__ hdiag,
                                               const double *__restrict__ theta, double *__restrict__ t, int64_t n,
                                               const int *m_dev, int full, const double *__restrict__ x,
                                               const double *__restrict__ hx, double *__restrict__ V,
                                               double *__restrict__ W, double *__restrict__ G, int ldg) {
    const double th = *theta;
    const bool collapse = *m_dev == full;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        double den = hdiag[i] - th;
        if (fabs(den) < 1e-8) den = copysign(1e-8, den);
        t[i] = r[i] / den;
        if (collapse) {
            V[i] = x[i];
            W[i] = hx[i];
        }
    }
    if (collapse && blockIdx.x == 0)
        for (int i = threadIdx.x; i < full * full; i += blockDim.x) G[(i / full) * ldg + i % full] = i == 0 ? th : 0.0;
}

// t -= V^T c with c_j the sums of the partials of V[j] . t (every block sums
// them itself); *last (nullable, host-visible) = the last one.  With norm set,
// norm[blk] = the block's partial of |t|^2 afterwards, with k_dots_partial's
// grid and order: thread t < 256 of its blocks adds elements 256 b + t, then
// every 256 gridDim-th.  Here four threads share such a chain's projections
// and the first of them adds the squares from LDS.
constexpr int kProjThreads = 4 * kDotThreads;
__global__ __launch_bounds__(kProjThreads) void k_project(const double *__restrict__ V, int64_t n, BasisSize size,
                                                          const double *__restrict__ partial, double *__restrict__ t,
                                                          const int *gate, double *last, double *__restrict__ norm) {
    if (gate && *gate == 0) return;
    __shared__ double sh[kProjThreads];
    __shared__ double c[64];
    const int m = size.get();
    const int nblk = gridDim.x;
    for (int j = threadIdx.x >> 6; j < m; j += kProjThreads / 64) {
        const double s = partials_sum(partial + static_cast<int64_t>(j) * nblk, nblk);
        if ((threadIdx.x & 63) == 0) c[j] = s;
    }
    __syncthreads();
    if (last && blockIdx.x == 0 && threadIdx.x == 0) *last = c[m - 1];
    const int lane = threadIdx.x % kDotThreads, quarter = threadIdx.x / kDotThreads;
    const int64_t step = static_cast<int64_t>(gridDim.x) * kDotThreads;
    double acc = 0.0;
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * kDotThreads + lane; i0 - lane < n; i0 += 4 * step) {
        const int64_t i = i0 + quarter * step;
        double ti = 0.0;
        if (i < n) {
            double s = 0.0;
            int j = 0;
            for (; j + 8 <= m; j += 8) {  // eight loads in flight, summed in order
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = V[(j + q) * n + i];
#pragma unroll
                for (int q = 0; q < 8; ++q) s = fma(c[j + q], v[q], s);
            }
            for (; j < m; ++j) s = fma(c[j], V[j * n + i], s);
            ti = t[i] - s;
            t[i] = ti;
        }
        if (!norm) continue;
        sh[threadIdx.x] = ti;
        __syncthreads();
        if (quarter == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (i0 + q * step < n) acc = fma(sh[q * kDotThreads + lane], sh[q * kDotThreads + lane], acc);
        __syncthreads();
    }
    if (!norm) return;
    if (quarter == 0) sh[lane] = acc;
    __syncthreads();
    for (int w = kDotThreads / 2; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) norm[blockIdx.x] = sh[0];
}

// when |t|^2 (the sum of the partials) < 1e-20 replace t by r and raise the
// gate for a second pass
__global__ __launch_bounds__(256) void k_fallback(const double *__restrict__ norm, int nblk, const double *__restrict__ r,
                                                  double *__restrict__ t, int64_t n, int *gate) {
    const bool fb = partials_sum(norm, nblk) < 1e-20;
    if (blockIdx.x == 0 && threadIdx.x == 0) *gate = fb ? 1 : 0;
    if (!fb) return;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        t[i] = r[i];
}

// row `basis size` of out = t / |t| with |t|^2 the sum of the partials; the
// same values into out2 when it is set, |t|^2 into *nrm2 (host-visible) when
// that is.  out may be NULL: only the norm.
__global__ __launch_bounds__(256) void k_normalise(const double *__restrict__ t, const double *__restrict__ norm, int nblk,
                                                   double *__restrict__ out, int64_t n, BasisSize size,
                                                   double *__restrict__ out2, double *nrm2) {
    const double sum = partials_sum(norm, nblk);
    if (nrm2 && blockIdx.x == 0 && threadIdx.x == 0) *nrm2 = sum;
    if (!out) return;
    const double inv = 1.0 / sqrt(sum);
    double *o = out + size.get() * n;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const double v = t[i] * inv;
        o[i] = v;
        if (out2) out2[i] = v;
    }
}

// (theta, rho^2) into the pinned host buffer the step reads after its sync,
// rho^2 the sum of the partials
__global__ __launch_bounds__(64) void k_publish(double *__restrict__ scal, const double *__restrict__ partial, int nblk,
                                                double *host) {
    const double s = partials_sum(partial, nblk);
    if (threadIdx.x == 0) {
        scal[1] = s;
        host[0] = scal[0];
        host[1] = s;
    }
}

unsigned grid_n(int64_t n) {
    const int64_t g = ceil_div(n, 256);
    return static_cast<unsigned>(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

// Blocks of the kernels that first sum the norm's partials: four per compute
// unit, so the sum is not repeated more often than it overlaps.
unsigned grid_norm(int64_t n) { return std::min(grid_n(n), 1024u); }

}  // namespace

struct davidson_s {
    ozaki_ctx ctx = nullptr;
    heff_plan H = nullptr;
    int64_t n = 0;
    int m_max = 0, max_iter = 0;
    double tol = 0;
    std::vector<void *> allocs;
    double *V = nullptr, *W = nullptr, *G = nullptr, *hdiag = nullptr;
    // Ritz vectors of two consecutive Rayleigh-Ritz solves: xs[cur] is the
    // latest, xs[rep] the one whose theta the last step reported
    double *xs[2] = {nullptr, nullptr};
    int cur = 0, rep = 0;
    double *hx = nullptr, *r = nullptr, *t = nullptr;
    double *mv_in = nullptr, *mv_out = nullptr;  // the matvec's fixed input and output
    double *y = nullptr, *partial = nullptr, *norm = nullptr, *scal = nullptr;  // scal: theta, rho2, nrm2
    int *gate = nullptr;
    int *m_dev = nullptr;  // the basis size on the device (the host keeps m too)
    double *host = nullptr;  // pinned: theta, rho2 of the latest Rayleigh-Ritz solve
    int m = 0, iter = 0, status = OZ_OK;
    std::vector<double> hist;
    // Replay: the launches that follow a step's decision (correction, basis
    // update, matvec, next Rayleigh-Ritz) read the basis size from the
    // device and use fixed matvec buffers, so they depend only on which Ritz
    // buffer is current: two graphs serve every step.
    bool use_graphs = true;
    hipStream_t cap = nullptr;
    hipGraphExec_t graphs[2] = {nullptr, nullptr};  // per current Ritz buffer
};

namespace {

int dalloc(davidson d, size_t bytes, void **p) {
    hipError_t e = hipMalloc(p, bytes < 8 ? 8 : bytes);
    if (e != hipSuccess) return fail(OZ_ERR_NOMEM, "davidson_create: %zu bytes: %s", bytes, hipGetErrorString(e));
    d->allocs.push_back(*p);
    return OZ_OK;
}

void dfree(davidson d) {
    for (auto g : d->graphs)
        if (g) hipGraphExecDestroy(g);
    if (d->cap) hipStreamDestroy(d->cap);
    for (void *p : d->allocs) hipFree(p);
    if (d->host) hipHostFree(d->host);
    delete d;
}

// |v|^2 into out, through d->norm
hipError_t norm2(double *partial, const double *v, int64_t n, double *out, hipStream_t s) {
    const int nb = dot_blocks(n);
    hipLaunchKernelGGL(k_dots_partial, dim3(nb, 1), dim3(kDotThreads), 0, s, v, n, v, n, partial, nullptr,
                       BasisSize{1, nullptr, 0}, 0, nullptr);
    if (out) hipLaunchKernelGGL(k_dots_final, dim3(1), dim3(64), 0, s, partial, nb, out);
    return hipGetLastError();
}

// Two classical Gram-Schmidt passes of t against the basis; the partials of
// |t|^2 afterwards in `norm`, the first pass's last coefficient in *last.
hipError_t gram_schmidt(const double *V, int64_t n, int rows, BasisSize size, double *t, double *partial, double *norm,
                        const int *gate, double *last, hipStream_t s) {
    const int nb = dot_blocks(n);
    for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(k_dots_partial, dim3(nb, rows), dim3(kDotThreads), 0, s, V, n, t, n, partial, gate, size, 0,
                           nullptr);
        hipLaunchKernelGGL(k_project, dim3(nb), dim3(kProjThreads), 0, s, V, n, size, partial, t, gate,
                           pass == 0 ? last : nullptr, pass == 1 ? norm : nullptr);
    }
    return hipGetLastError();
}

// Rayleigh-Ritz on the device's basis (with grow set, after taking in the new
// vector's column of G from d->partial), the Ritz pair into x_out (and hx, r),
// and (theta, rho^2) published to the pinned host buffer.
int rayleigh_ritz(davidson d, double *x_out, bool grow, hipStream_t s) {
    const int64_t n = d->n;
    const int nb = dot_blocks(n);
    double *theta = d->scal;
    hipLaunchKernelGGL(k_jacobi, dim3(1), dim3(256), 0, s, d->G, d->m_max, BasisSize{0, d->m_dev, grow ? d->m_max : 0},
                       d->m_dev, d->partial, grow ? nb : 0, d->y, theta);
    hipLaunchKernelGGL(k_ritz, dim3(nb), dim3(kDotThreads), 0, s, d->V, d->W, n, d->m_dev, d->y, theta, x_out, d->hx,
                       d->r, d->partial);
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, d->scal, d->partial, nb, d->host);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? OZ_OK : hip_fail(e, "davidson: Rayleigh-Ritz");
}

// Everything a continuing step does after its decision, with current Ritz
// buffer c: correction (and collapse when the basis is full),
// orthogonalisation and matvec, then the next Rayleigh-Ritz into xs[c ^ 1].
int step_tail(davidson d, int c, hipStream_t s) {
    hipError_t e;
    const int64_t n = d->n;
    const int nb = dot_blocks(n);
    const BasisSize size{0, d->m_dev, d->m_max};
    hipLaunchKernelGGL(k_begin, dim3(grid_n(n)), dim3(256), 0, s, d->r, d->hdiag, d->scal, d->t, n, d->m_dev, d->m_max,
                       d->xs[c], d->hx, d->V, d->W, d->G, d->m_max);
    if ((e = gram_schmidt(d->V, n, d->m_max, size, d->t, d->partial, d->norm, nullptr, nullptr, s)) != hipSuccess)
        return hip_fail(e, "davidson: projection");
    hipLaunchKernelGGL(k_fallback, dim3(grid_norm(n)), dim3(256), 0, s, d->norm, nb, d->r, d->t, n, d->gate);
    if ((e = gram_schmidt(d->V, n, d->m_max, size, d->t, d->partial, d->norm, d->gate, nullptr, s)) != hipSuccess)
        return hip_fail(e, "davidson: projection");
    // V[m] and the matvec's input get the same values
    hipLaunchKernelGGL(k_normalise, dim3(grid_norm(n)), dim3(256), 0, s, d->t, d->norm, nb, d->V, n, size, d->mv_in, nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "davidson: orthogonalisation");
    int rc = heff_apply(d->H, d->mv_in, d->mv_out, s);
    if (rc != OZ_OK) return rc;
    // V[i] . W[m], i <= m, and W[m] itself
    hipLaunchKernelGGL(k_dots_partial, dim3(nb, d->m_max + 1), dim3(kDotThreads), 0, s, d->V, n, d->mv_out, n, d->partial,
                       nullptr, size, 1, d->W);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "davidson: projected column");
    return rayleigh_ritz(d, d->xs[c ^ 1], true, s);
}

// step_tail from a captured graph (captured the first time c is seen), or
// issued directly when phases are being timed or graphs are off.
int run_tail(davidson d, int c, hipStream_t s) {
    hipError_t e;
    if (!d->use_graphs || d->ctx->timing) return step_tail(d, c, s);
    hipGraphExec_t &g = d->graphs[c];
    if (!g) {
        if (!d->cap && (e = hipStreamCreateWithFlags(&d->cap, hipStreamNonBlocking)) != hipSuccess)
            return hip_fail(e, "davidson: capture stream");
        if ((e = hipStreamBeginCapture(d->cap, hipStreamCaptureModeThreadLocal)) != hipSuccess)
            return hip_fail(e, "davidson: begin capture");
        const int rc = step_tail(d, c, d->cap);
        hipGraph_t graph = nullptr;
        e = hipStreamEndCapture(d->cap, &graph);
        if (rc != OZ_OK) {
            if (graph) hipGraphDestroy(graph);
            return rc;
        }
        if (e != hipSuccess) return hip_fail(e, "davidson: end capture");
        e = hipGraphInstantiate(&g, graph, nullptr, nullptr, 0);
        hipGraphDestroy(graph);
        if (e != hipSuccess) {
            g = nullptr;
            return hip_fail(e, "davidson: instantiate");
        }
    }
    if ((e = hipGraphLaunch(g, s)) != hipSuccess) return hip_fail(e, "davidson: graph launch");
    return OZ_OK;
}

}  // namespace

extern "C" {

int davidson_create(ozaki_ctx ctx, davidson *out, heff_plan H, const double *hdiag, const double *x0,
                    int m_max, double tol, int max_iter, void *stream) {
    if (!out) return fail(OZ_ERR_ARG, "davidson_create: out is NULL");
    *out = nullptr;
    if (!ctx || !H || !hdiag || !x0) return fail(OZ_ERR_ARG, "davidson_create: NULL argument");
    if (m_max < 2 || m_max > 64) return fail(OZ_ERR_ARG, "davidson_create: m_max = %d (2..64)", m_max);
    if (!(tol >= 0) || max_iter < 1) return fail(OZ_ERR_ARG, "davidson_create: tol / max_iter");
    const int64_t n = heff_vector_length(H);
    if (n < 1) return fail(OZ_ERR_ARG, "davidson_create: empty operator");
    hipError_t e;
    if ((e = hipSetDevice(ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
    hipStream_t s = static_cast<hipStream_t>(stream);
    davidson d = new davidson_s();
    d->ctx = ctx;
    d->H = H;
    d->n = n;
    d->m_max = m_max;
    d->tol = tol;
    d->max_iter = max_iter;
    int rc;
    void *p;
#define OZ_DA(field, bytes) \
    if ((rc = dalloc(d, (bytes), &p)) != OZ_OK) { dfree(d); return rc; } \
    d->field = static_cast<std::remove_reference_t<decltype(d->field)>>(p);
    OZ_DA(V, sizeof(double) * m_max * n)
    OZ_DA(W, sizeof(double) * m_max * n)
    OZ_DA(G, sizeof(double) * m_max * m_max)
    OZ_DA(hdiag, sizeof(double) * n)
    OZ_DA(xs[0], sizeof(double) * n)
    OZ_DA(xs[1], sizeof(double) * n)
    OZ_DA(hx, sizeof(double) * n)
    OZ_DA(mv_in, sizeof(double) * n)
    OZ_DA(mv_out, sizeof(double) * n)
    OZ_DA(m_dev, sizeof(int) * 4)
    OZ_DA(r, sizeof(double) * n)
    OZ_DA(t, sizeof(double) * n)
    OZ_DA(y, sizeof(double) * 64)
    OZ_DA(partial, sizeof(double) * 65 * 512)
    OZ_DA(norm, sizeof(double) * 512)
    OZ_DA(scal, sizeof(double) * 8)
    OZ_DA(gate, sizeof(int) * 4)
#undef OZ_DA
    if ((e = hipHostMalloc(reinterpret_cast<void **>(&d->host), sizeof(double) * 4, 0)) != hipSuccess) {
        d->host = nullptr;
        dfree(d);
        return hip_fail(e, "davidson_create: pinned buffer");
    }
    if ((e = hipMemcpyAsync(d->hdiag, hdiag, sizeof(double) * n, hipMemcpyDeviceToDevice, s)) != hipSuccess ||
        (e = hipMemsetAsync(d->G, 0, sizeof(double) * m_max * m_max, s)) != hipSuccess) {
        dfree(d);
        return hip_fail(e, "davidson_create: copies");
    }
    // v0 = x0 / |x0|, W0 = H v0, G00 = v0 . W0
    double *nrm2 = d->scal + 2;
    if ((e = norm2(d->norm, x0, n, nrm2, s)) != hipSuccess ||
        (e = hipMemcpyAsync(d->host, nrm2, sizeof(double), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess) {
        dfree(d);
        return hip_fail(e, "davidson_create: start vector");
    }
    if (!(d->host[0] > 0) || !std::isfinite(d->host[0])) {
        dfree(d);
        return fail(OZ_ERR_ARG, "davidson_create: start vector is zero or not finite");
    }
    const int nb = dot_blocks(n);
    hipLaunchKernelGGL(k_normalise, dim3(grid_norm(n)), dim3(256), 0, s, x0, d->norm, nb, d->V, n, BasisSize{0, nullptr, 0},
                       nullptr, nullptr);
    if ((rc = heff_apply(H, d->V, d->W, s)) != OZ_OK) { dfree(d); return rc; }
    hipLaunchKernelGGL(k_dots_partial, dim3(nb, 1), dim3(kDotThreads), 0, s, d->V, n, d->W, n, d->partial, nullptr,
                       BasisSize{1, nullptr, 0}, 0, nullptr);
    hipLaunchKernelGGL(k_dots_final, dim3(1), dim3(64), 0, s, d->partial, nb, d->G);
    const int one = 1;
    if ((e = hipMemcpyAsync(d->m_dev, &one, sizeof(int), hipMemcpyHostToDevice, s)) != hipSuccess) {
        dfree(d);
        return hip_fail(e, "davidson_create: basis size");
    }
    // the first step's Rayleigh-Ritz solve (every later one ends the step before)
    if ((rc = rayleigh_ritz(d, d->xs[0], false, s)) != OZ_OK) { dfree(d); return rc; }
    if ((e = hipStreamSynchronize(s)) != hipSuccess) { dfree(d); return hip_fail(e, "davidson_create: sync"); }
    d->m = 1;
    *out = d;
    return OZ_OK;
}

int davidson_step(davidson d, davidson_info *info, void *stream) {
    if (!d) return fail(OZ_ERR_ARG, "davidson_step: NULL solver");
    if (d->status != OZ_OK) {
        if (info) *info = davidson_info{d->host[0], std::sqrt(d->host[1]), d->iter, d->m, d->status};
        return fail(OZ_ERR_STATE, "davidson_step: the iteration has already ended (%s)", ozaki_status_string(d->status));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if ((e = hipSetDevice(d->ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
    // the Rayleigh-Ritz solve on the current basis ended the previous step
    // (or davidson_create): its theta and rho^2 are in the pinned buffer
    d->iter += 1;
    const double theta = d->host[0];
    const double rho = std::sqrt(d->host[1]);
    d->hist.push_back(rho);
    d->rep = d->cur;
    int status = OZ_OK;
    const size_t w = 20;
    if (rho <= d->tol) {
        status = OZ_CONVERGED;
    } else if (d->hist.size() > w) {
        // stagnated: the last w residuals never got below half the best before them
        const size_t first_recent = d->hist.size() - w;
        double recent = INFINITY, before = INFINITY;
        for (size_t i = 0; i < d->hist.size(); ++i) {
            if (i >= first_recent)
                recent = std::min(recent, d->hist[i]);
            else
                before = std::min(before, d->hist[i]);
        }
        if (recent > 0.5 * before) status = OZ_STAGNATED;
    }
    if (status == OZ_OK && d->iter >= d->max_iter) status = OZ_MAX_ITER;
    if (status == OZ_OK) {
        // correction, basis update, matvec and the next Rayleigh-Ritz solve:
        // one graph replay and one synchronisation per step
        const int m = d->m;
        int rc = run_tail(d, d->cur, s);
        if (rc != OZ_OK) return rc;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "davidson_step: sync");
        d->m = (m == d->m_max ? 1 : m) + 1;
        d->cur ^= 1;
    }
    d->status = status;
    if (info) *info = davidson_info{theta, rho, d->iter, d->m, status};
    return status;
}

int davidson_set_graphs(davidson d, int enable) {
    if (!d) return fail(OZ_ERR_ARG, "davidson_set_graphs: NULL solver");
    d->use_graphs = enable != 0;
    return OZ_OK;
}

int davidson_graph_count(davidson d) {
    if (!d) return fail(OZ_ERR_ARG, "davidson_graph_count: NULL solver");
    int k = 0;
    for (auto g : d->graphs) k += g != nullptr;
    return k;
}

int davidson_get_vector(davidson d, double *x_out, void *stream) {
    if (!d || !x_out) return fail(OZ_ERR_ARG, "davidson_get_vector: NULL argument");
    if (d->iter == 0) return fail(OZ_ERR_STATE, "davidson_get_vector: no step taken yet");
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(x_out, d->xs[d->rep], sizeof(double) * d->n, hipMemcpyDeviceToDevice, s);
    return e == hipSuccess ? OZ_OK : hip_fail(e, "davidson_get_vector");
}

int davidson_destroy(davidson d) {
    if (!d) return OZ_OK;
    hipSetDevice(d->ctx->device);
    hipDeviceSynchronize();
    dfree(d);
    return OZ_OK;
}

}  // extern "C"

// ---- Lanczos with full reorthogonalisation and explicit restart -------------

namespace {

// x = Q^T y over the first m basis vectors.
__global__ void k_combine(const double *__restrict__ Q, int64_t n, int m, const double *__restrict__ y,
                          double *__restrict__ x) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        double s = 0.0;
        for (int j = 0; j < m; ++j) s = fma(y[j], Q[j * n + i], s);
        x[i] = s;
    }
}

// Lowest eigenpair of the symmetric m x m matrix a (row-major), cyclic
// Jacobi on the host; y normalised with its largest-magnitude entry positive.
double host_lowest_eigenpair(std::vector<double> a, int m, std::vector<double> *y) {
    std::vector<double> v(static_cast<size_t>(m) * m, 0.0);
    for (int i = 0; i < m; ++i) v[static_cast<size_t>(i) * m + i] = 1.0;
    for (int sweep = 0; sweep < 60; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int i = 0; i < m; ++i)
            for (int j = 0; j < m; ++j) {
                const double x = a[static_cast<size_t>(i) * m + j] * a[static_cast<size_t>(i) * m + j];
                tot += x;
                if (i != j) off += x;
            }
        if (std::sqrt(off) <= 1e-15 * std::sqrt(tot)) break;
        for (int p = 0; p < m - 1; ++p)
            for (int q = p + 1; q < m; ++q) {
                const double apq = a[static_cast<size_t>(p) * m + q];
                if (apq == 0.0) continue;
                const double th = (a[static_cast<size_t>(q) * m + q] - a[static_cast<size_t>(p) * m + p]) / (2.0 * apq);
                const double t = (th >= 0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(th * th + 1.0));
                const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < m; ++k) {  // rows p, q
                    const double ap = a[static_cast<size_t>(p) * m + k], aq = a[static_cast<size_t>(q) * m + k];
                    a[static_cast<size_t>(p) * m + k] = c * ap - s * aq;
                    a[static_cast<size_t>(q) * m + k] = s * ap + c * aq;
                }
                for (int k = 0; k < m; ++k) {  // columns p, q and the eigenvectors
                    const double ap = a[static_cast<size_t>(k) * m + p], aq = a[static_cast<size_t>(k) * m + q];
                    a[static_cast<size_t>(k) * m + p] = c * ap - s * aq;
                    a[static_cast<size_t>(k) * m + q] = s * ap + c * aq;
                    const double vp = v[static_cast<size_t>(k) * m + p], vq = v[static_cast<size_t>(k) * m + q];
                    v[static_cast<size_t>(k) * m + p] = c * vp - s * vq;
                    v[static_cast<size_t>(k) * m + q] = s * vp + c * vq;
                }
            }
    }
    int best = 0;
    for (int i = 1; i < m; ++i)
        if (a[static_cast<size_t>(i) * m + i] < a[static_cast<size_t>(best) * m + best]) best = i;
    int big = 0;
    for (int i = 1; i < m; ++i)
        if (std::fabs(v[static_cast<size_t>(i) * m + best]) > std::fabs(v[static_cast<size_t>(big) * m + best])) big = i;
    const double sgn = v[static_cast<size_t>(big) * m + best] < 0 ? -1.0 : 1.0;
    y->resize(m);
    for (int i = 0; i < m; ++i) (*y)[i] = sgn * v[static_cast<size_t>(i) * m + best];
    return a[static_cast<size_t>(best) * m + best];
}

}  // namespace

struct lanczos_s {
    ozaki_ctx ctx = nullptr;
    heff_plan H = nullptr;
    int64_t n = 0;
    int m_max = 0, max_iter = 0;
    double tol = 0;
    std::vector<void *> allocs;
    double *Q = nullptr, *w = nullptr, *norm = nullptr, *partial = nullptr, *scal = nullptr, *y_dev = nullptr;
    double *host = nullptr;  // pinned: the last step's alpha and |w|^2
    std::vector<double> alpha, beta, y;
    int m = 0, iter = 0, status = OZ_OK;
    double theta = 0, rho = 0;
    std::vector<double> hist;
};

namespace {

int lalloc(lanczos l, size_t bytes, void **p) {
    hipError_t e = hipMalloc(p, bytes < 8 ? 8 : bytes);
    if (e != hipSuccess) return fail(OZ_ERR_NOMEM, "lanczos_create: %zu bytes: %s", bytes, hipGetErrorString(e));
    l->allocs.push_back(*p);
    return OZ_OK;
}

void lfree(lanczos l) {
    for (void *p : l->allocs) hipFree(p);
    if (l->host) hipHostFree(l->host);
    delete l;
}

// q_0 = x / |x| into the basis; resets T
int lanczos_reset(lanczos l, const double *x, hipStream_t s) {
    hipError_t e;
    if ((e = norm2(l->norm, x, l->n, nullptr, s)) != hipSuccess) return hip_fail(e, "lanczos: norm");
    hipLaunchKernelGGL(k_normalise, dim3(grid_norm(l->n)), dim3(256), 0, s, x, l->norm, dot_blocks(l->n), l->Q, l->n,
                       BasisSize{0, nullptr, 0}, nullptr, nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "lanczos: normalise");
    l->m = 1;
    l->alpha.clear();
    l->beta.clear();
    return OZ_OK;
}

}  // namespace

extern "C" {

int lanczos_create(ozaki_ctx ctx, lanczos *out, heff_plan H, const double *x0, int m_max, double tol, int max_iter,
                   void *stream) {
    if (!out) return fail(OZ_ERR_ARG, "lanczos_create: out is NULL");
    *out = nullptr;
    if (!ctx || !H || !x0) return fail(OZ_ERR_ARG, "lanczos_create: NULL argument");
    if (m_max < 2 || m_max > 64) return fail(OZ_ERR_ARG, "lanczos_create: m_max = %d (2..64)", m_max);
    if (!(tol >= 0) || max_iter < 1) return fail(OZ_ERR_ARG, "lanczos_create: tol / max_iter");
    const int64_t n = heff_vector_length(H);
    if (n < 1) return fail(OZ_ERR_ARG, "lanczos_create: empty operator");
    hipError_t e;
    if ((e = hipSetDevice(ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
    hipStream_t s = static_cast<hipStream_t>(stream);
    lanczos l = new lanczos_s();
    l->ctx = ctx;
    l->H = H;
    l->n = n;
    l->m_max = m_max;
    l->tol = tol;
    l->max_iter = max_iter;
    int rc;
    void *p;
#define OZ_LA(field, bytes) \
    if ((rc = lalloc(l, (bytes), &p)) != OZ_OK) { lfree(l); return rc; } \
    l->field = static_cast<decltype(l->field)>(p);
    OZ_LA(Q, sizeof(double) * (m_max + 1) * n)
    OZ_LA(w, sizeof(double) * n)
    OZ_LA(norm, sizeof(double) * 512)
    OZ_LA(partial, sizeof(double) * 66 * 512)
    OZ_LA(scal, sizeof(double) * 8)
    OZ_LA(y_dev, sizeof(double) * 72)
#undef OZ_LA
    if ((e = hipHostMalloc(reinterpret_cast<void **>(&l->host), sizeof(double) * 72, 0)) != hipSuccess) {
        l->host = nullptr;
        lfree(l);
        return hip_fail(e, "lanczos_create: pinned buffer");
    }
    // start vector: |x0| must be positive and finite
    if ((e = norm2(l->norm, x0, n, l->scal, s)) != hipSuccess ||
        (e = hipMemcpyAsync(l->host, l->scal, sizeof(double), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess) {
        lfree(l);
        return hip_fail(e, "lanczos_create: start vector");
    }
    if (!(l->host[0] > 0) || !std::isfinite(l->host[0])) {
        lfree(l);
        return fail(OZ_ERR_ARG, "lanczos_create: start vector is zero or not finite");
    }
    if ((rc = lanczos_reset(l, x0, s)) != OZ_OK) { lfree(l); return rc; }
    if ((e = hipStreamSynchronize(s)) != hipSuccess) { lfree(l); return hip_fail(e, "lanczos_create: sync"); }
    *out = l;
    return OZ_OK;
}

int lanczos_step(lanczos l, davidson_info *info, void *stream) {
    if (!l) return fail(OZ_ERR_ARG, "lanczos_step: NULL solver");
    if (l->status != OZ_OK) {
        if (info) *info = davidson_info{l->theta, l->rho, l->iter, l->m, l->status};
        return fail(OZ_ERR_STATE, "lanczos_step: the iteration has already ended (%s)", ozaki_status_string(l->status));
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if ((e = hipSetDevice(l->ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
    const int64_t n = l->n;
    const int m = l->m;  // basis q_0 .. q_{m-1}; this step expands from q_{m-1}
    double *qj = l->Q + static_cast<int64_t>(m - 1) * n;
    int rc = heff_apply(l->H, qj, l->w, s);
    if (rc != OZ_OK) return rc;
    // two classical Gram-Schmidt passes against the whole basis; alpha (the
    // first pass's coefficient of q_{m-1}) and |w|^2 go straight to the host's
    // buffer, and q_m = w / |w| is written before the decision (unused when
    // the step ends the iteration; a full basis restarts instead)
    const BasisSize size{m, nullptr, 0};
    if ((e = gram_schmidt(l->Q, n, m, size, l->w, l->partial, l->norm, nullptr, l->host, s)) != hipSuccess)
        return hip_fail(e, "lanczos: projection");
    hipLaunchKernelGGL(k_normalise, dim3(grid_norm(n)), dim3(256), 0, s, l->w, l->norm, dot_blocks(n),
                       m < l->m_max ? l->Q : nullptr, n, size, nullptr, l->host + 1);
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess)
        return hip_fail(e, "lanczos: step");
    l->iter += 1;
    const double a = l->host[0];
    const double b = std::sqrt(l->host[1] > 0 ? l->host[1] : 0.0);
    l->alpha.push_back(a);
    // Ritz pair of T_m
    std::vector<double> T(static_cast<size_t>(m) * m, 0.0);
    for (int i = 0; i < m; ++i) {
        T[static_cast<size_t>(i) * m + i] = l->alpha[i];
        if (i + 1 < m) T[static_cast<size_t>(i) * m + i + 1] = T[static_cast<size_t>(i + 1) * m + i] = l->beta[i];
    }
    l->theta = host_lowest_eigenpair(T, m, &l->y);
    l->rho = b * std::fabs(l->y[m - 1]);
    l->hist.push_back(l->rho);
    int status = OZ_OK;
    const bool invariant = !(b > 1e-14 * (std::fabs(a) + (m > 1 ? l->beta[m - 2] : 0.0)));
    if (l->rho <= l->tol || invariant) {
        status = OZ_CONVERGED;
    } else if (l->hist.size() > 20) {
        const size_t first_recent = l->hist.size() - 20;
        double recent = INFINITY, before = INFINITY;
        for (size_t i = 0; i < l->hist.size(); ++i) {
            if (i >= first_recent) recent = std::min(recent, l->hist[i]);
            else before = std::min(before, l->hist[i]);
        }
        if (recent > 0.5 * before) status = OZ_STAGNATED;
    }
    if (status == OZ_OK && l->iter >= l->max_iter) status = OZ_MAX_ITER;
    if (status == OZ_OK) {
        if (m == l->m_max) {
            // restart from the Ritz vector x = Q y (written to w, then normalised into q_0)
            if ((e = hipMemcpyAsync(l->y_dev, l->y.data(), sizeof(double) * m, hipMemcpyHostToDevice, s)) != hipSuccess)
                return hip_fail(e, "lanczos: Ritz coefficients");
            hipLaunchKernelGGL(k_combine, dim3(grid_n(n)), dim3(256), 0, s, l->Q, n, m, l->y_dev, l->w);
            if ((rc = lanczos_reset(l, l->w, s)) != OZ_OK) return rc;
        } else {
            l->beta.push_back(b);
            l->m = m + 1;
        }
    } else {
        // keep the Ritz coefficients of the final basis for lanczos_get_vector
        l->m = m;
    }
    l->status = status;
    if (info) *info = davidson_info{l->theta, l->rho, l->iter, l->m, status};
    return status;
}

int lanczos_get_vector(lanczos l, double *x_out, void *stream) {
    if (!l || !x_out) return fail(OZ_ERR_ARG, "lanczos_get_vector: NULL argument");
    if (l->iter == 0 || l->y.empty()) return fail(OZ_ERR_STATE, "lanczos_get_vector: no step taken yet");
    if (l->status == OZ_OK && l->m == 1 && l->alpha.empty()) {
        // just restarted: q_0 is the Ritz vector
        hipError_t e = hipMemcpyAsync(x_out, l->Q, sizeof(double) * l->n, hipMemcpyDeviceToDevice,
                                      static_cast<hipStream_t>(stream));
        return e == hipSuccess ? OZ_OK : hip_fail(e, "lanczos_get_vector");
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int m = static_cast<int>(l->y.size());
    hipError_t e = hipMemcpyAsync(l->y_dev, l->y.data(), sizeof(double) * m, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "lanczos_get_vector: coefficients");
    hipLaunchKernelGGL(k_combine, dim3(grid_n(l->n)), dim3(256), 0, s, l->Q, l->n, m, l->y_dev, x_out);
    e = hipStreamSynchronize(s);  // y_dev is reused by the next step
    return e == hipSuccess ? OZ_OK : hip_fail(e, "lanczos_get_vector");
}

int lanczos_destroy(lanczos l) {
    if (!l) return OZ_OK;
    hipSetDevice(l->ctx->device);
    hipDeviceSynchronize();
    lfree(l);
    return OZ_OK;
}

}  // extern "C"
