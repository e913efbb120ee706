// The two DMRG steps next to the H_eff diagonalisation: the eigenvalue
// decomposition of the reduced density matrix (truncation to the dominant
// eigenvectors) and the renormalisation of block operators into the kept
// basis.  The paper (numerical-stability discussion) runs both with native
// and with emulated FP64 linear algebra and finds the eigensolver's
// arithmetic decisive at low slice counts; both here take (slices, ndiag)
// like ozaki_dgemm, slices = 0 meaning native FP64.
//
// rdm_eig: two-sided block Jacobi on a symmetric A.  M = W A W^T with W
// orthogonal (W = I at the start; rows are the basis vectors).  The n rows
// (padded to np, a multiple of 64, with zero rows and columns) form np/32
// blocks of 32; a sweep pairs every block with every other once (round-robin
// "circle" schedule, np/32 - 1 rounds).  In a round the paired blocks sit
// next to each other, so pair k owns rows and columns [64k, 64k + 64):
//   1. one sweep of cyclic Jacobi on each pair's diagonal 64 x 64 block of M
//      (one workgroup per pair; nothing when the block is already
//      diagonal): all its rotations in a sweep's first round, the 1024 that
//      couple its two blocks in the others, accumulated from the identity, in
//      that order: Q_k^T (sorting them by eigenvalue would make the block
//      rotation a near-permutation between the two blocks, and block Jacobi
//      then stalls);
//   2. R = Q^T M (rows of each pair);
//   3. M' = Q^T R^T (= Q^T M Q, M symmetric);
//   4. W <- Q^T W;
//   5. rows and columns move to the next round's slots.
// In native FP64 steps 2, 3 and 5 of M are one kernel, and step 4 with its
// move runs beside the next round's step 1; emulated, each of 2-4 is a
// grouped GEMM of inner length 64 and step 5 a copy.
// Before the sweeps up to two steps of shifted QR iteration, M <- Q^T M Q with
// Q R = M + mu I (mu = 3e-7 |A|_F, then 3e-12 |A|_F), gather the weight near
// the diagonal in decreasing order (precondition below); W starts as Q^T.
// The GEMMs of steps 2-4 run in the plan's arithmetic; step 1 and the QR
// iteration in FP64.  The
// largest off-diagonal |M_rc| met in step 1 over a sweep measures
// convergence against tol |A|_F (absolute accuracy, as a tridiagonal-based
// solver gives).  The eigenvectors are then the rows of W and the eigenvalues
// M_cc / |w_c|^2 when emulated, the quotients w_c A w_c^T / |w_c|^2 in native
// FP64 (k_rayleigh).  Padding rows and columns stay exactly zero (a
// zero entry gives an exact identity rotation), so the padding basis vectors
// are recognised by their zero restriction to the first n coordinates.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <utility>
#include <vector>

#include "rotation.h"
#include "runtime.h"
#include "tile64.h"

using namespace oz;

namespace {

constexpr int kBlk = 32;    // rows per Jacobi block
constexpr int kPair = 64;   // rows per pair of blocks
constexpr int kLdE = 65;    // LDS row stride of the 64 x 64 pair problems
constexpr int64_t kMaxEigN = 8192;
constexpr int kScanBlocks = 1024;

// Round-robin schedule of the 64 rows of a pair problem: row 63 fixed, the
// others rotate; step `step` pairs (63, step) and (step + t, step - t) mod 63.
__device__ __forceinline__ void circle_pair(int step, int t, int *p, int *q) {
    int a, b;
    if (t == 0) {
        a = 63;
        b = step;
    } else {
        a = (step + t) % 63;
        b = (step + 63 - t) % 63;
    }
    *p = a < b ? a : b;
    *q = a < b ? b : a;
}

// Block sum of v over the 256 threads, returned to all of them.
__device__ double block_sum(double v, double *red) {
    const int tid = threadIdx.x;
    red[tid] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// Off-diagonal entries a_rc, r != c.  An entry is "exempt" when both
// diagonal entries are below theta (rows outside the wanted part of the
// spectrum).  Returns the largest |a_rc| of the other entries to all
// threads; with sums set also the sum of squares of the counted entries
// (sums[0]) and of the exempt ones (sums[1]).
__device__ double offdiag(const double *a, double *red, double theta, double *sums) {
    const int tid = threadIdx.x;
    double m = 0.0, q = 0.0, qx = 0.0;
    for (int idx = tid; idx < kPair * kPair; idx += 256) {
        const int r = idx >> 6, c = idx & 63;
        if (r == c) continue;
        const double x = fabs(a[r * kLdE + c]);
        if (a[r * kLdE + r] < theta && a[c * kLdE + c] < theta) {
            qx = fma(x, x, qx);
        } else {
            m = fmax(m, x);
            q = fma(x, x, q);
        }
    }
    red[tid] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    sums[0] = block_sum(q, red);
    sums[1] = block_sum(qx, red);
    return r;
}

__device__ __forceinline__ double lane_value(double x, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

// A pair's own rotated tile, element (r, c) = f(r, c) of 64 x 64, in the next
// round's slots: whole when its two 32 x 32 blocks stay together, else its
// diagonal blocks and the block between them on the upper side.  Threads (ty,
// tx) of an 8 x 32 grid, rows 4 ty + m and columns tx of each block.
template <typename F>
__device__ __forceinline__ void store_pair_tile(double *__restrict__ M2, int64_t np, int d0, int d1, F f) {
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int d[2] = {d0, d1};
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            if ((d[rb] >> 1) > (d[cb] >> 1)) continue;
            double *o = M2 + static_cast<int64_t>(d[rb]) * kBlk * np + static_cast<int64_t>(d[cb]) * kBlk + tx;
#pragma unroll
            for (int m = 0; m < 4; ++m) o[(4 * ty + m) * np] = f(rb, cb, m);
        }
}

// Step 1: one workgroup per pair k.  The pair's diagonal block of M (upper
// triangle, mirrored) goes through one sweep of cyclic Jacobi over all its
// rotations, unless its largest off-diagonal entry is <= inner_tol and its
// exempt entries' sum of squares <= exempt_tol2; Qt rows [64k, 64k + 64) receive the accumulated rotations (row t: column t of
// their product); off_out[3k .. 3k + 2]: the block's largest counted
// off-diagonal |entry| and the sums of squares of the counted and of the
// exempt entries (both diagonals below theta) before the rotations.
// Each of the 4 waves owns 8 of a step's 32 disjoint rotations (t = wave +
// 4 i): lane i < 8 computes rotation i, readlane hands it to the wave, the
// lanes then sweep the 64 columns (row pass) and the 64 rows (column pass).
__global__ __launch_bounds__(256) void k_pair_eig(const double *__restrict__ M, int64_t ldm,
                                                  double *__restrict__ Qt, double *__restrict__ off_out,
                                                  double inner_tol, double exempt_tol2, double theta,
                                                  double *__restrict__ M2, const int *__restrict__ dst,
                                                  int *__restrict__ act) {
    __shared__ double a[kPair * kLdE];
    __shared__ double vt[kPair * kPair];  // transposed rotations: row t is column t of the product
    __shared__ double red[256];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int k = blockIdx.x;
    const double *g = M + static_cast<int64_t>(kPair) * k * ldm + static_cast<int64_t>(kPair) * k;
    for (int idx = tid; idx < kPair * kPair; idx += 256) {
        const int r = idx >> 6, c = idx & 63;
        a[r * kLdE + c] = r <= c ? g[r * ldm + c] : g[c * ldm + r];
        vt[r * kPair + c] = r == c ? 1.0 : 0.0;
    }
    __syncthreads();
    double sums[2];
    const double off = offdiag(a, red, theta, sums);
    if (tid == 0) {
        off_out[3 * k] = off;
        off_out[3 * k + 1] = sums[0];
        off_out[3 * k + 2] = sums[1];
        if (act) act[k] = off > inner_tol || sums[1] > exempt_tol2;
    }
    if (off > inner_tol || sums[1] > exempt_tol2) {
        for (int step = 0; step < 63; ++step) {
            double hl = 0.0, sl = 0.0;  // tan(a / 2) and sin(a)
            {
                // rotation wave + 4 (lane & 7): rows other waves leave alone in the row pass
                int p, q;
                circle_pair(step, wave + 4 * (lane & 7), &p, &q);
                const double apq = a[p * kLdE + q];
                if (apq != 0.0) {
                    // symmetric Schur rotation zeroing a_pq (smaller root of t^2 + 2 th t - 1 = 0)
                    const double th = (a[q * kLdE + q] - a[p * kLdE + p]) / (2.0 * apq);
                    const double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                    const double c = 1.0 / sqrt(t * t + 1.0);
                    sl = t * c;
                    hl = sl / (1.0 + c);
                }
            }
            double hs[8], ss[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                hs[i] = lane_value(hl, i);
                ss[i] = lane_value(sl, i);
            }
            // the 8 rotations touch disjoint rows (columns): all loads of a
            // pass first, then all stores, so their latencies overlap
            int pp[8], qq[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) circle_pair(step, wave + 4 * i, &pp[i], &qq[i]);
            double x[8], y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {  // rows p, q; lane = column
                x[i] = a[pp[i] * kLdE + lane];
                y[i] = a[qq[i] * kLdE + lane];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                rotate(ss[i], hs[i], x[i], y[i]);
                a[pp[i] * kLdE + lane] = x[i];
                a[qq[i] * kLdE + lane] = y[i];
            }
            __syncthreads();
            double u[8], v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {  // columns p, q and rotations p, q; lane = row
                x[i] = a[lane * kLdE + pp[i]];
                y[i] = a[lane * kLdE + qq[i]];
                u[i] = vt[pp[i] * kPair + lane];
                v[i] = vt[qq[i] * kPair + lane];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                rotate(ss[i], hs[i], x[i], y[i]);
                rotate(ss[i], hs[i], u[i], v[i]);
                a[lane * kLdE + pp[i]] = x[i];
                a[lane * kLdE + qq[i]] = y[i];
                vt[pp[i] * kPair + lane] = u[i];
                vt[qq[i] * kPair + lane] = v[i];
            }
            __syncthreads();
        }
    }
    double *qt = Qt + static_cast<int64_t>(kPair) * k * kPair;
    for (int idx = tid; idx < kPair * kPair; idx += 256) qt[idx] = vt[idx];
    if (M2)
        store_pair_tile(M2, ldm, dst[2 * k], dst[2 * k + 1], [&](int rb, int cb, int m) {
            return a[(32 * rb + 4 * (tid >> 5) + m) * kLdE + 32 * cb + (tid & 31)];
        });
}

__device__ __forceinline__ double lane_shift(double x, int addr) {
    const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(x));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(x));
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_max(double v) {
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

constexpr int kRotLds = 64 * t64::kLdK + 64 * t64::kLdN;  // doubles: one tile read along k, one across

// Step 1 in the rounds after a sweep's first: only the 1024 rotations that
// couple the pair's two blocks (the first round rotates inside the blocks
// too, so a sweep still meets every pair of rows once).  32 steps; step t
// rotates the disjoint pairs (i, 32 + (i + t) % 32).
//
// Everything stays in registers: thread (ty, tx) holds, for the pairs i = 4
// ty + m (m < 4) and j = tx, the 2 x 2 block of rows (p_i, q_i) and columns
// (p_j, q_j), and the entries of columns tx and tx + 32 of rows p_i, q_i of
// the accumulated rotations.  A rotation is then local once its (c, s) pairs
// are known, and moving on to the next step's pairing shifts the q rows and
// columns by one: within the thread, to the next lane, or (one row in four)
// through LDS, along with the three elements each of the next rotations needs,
// so that every half wave computes all of them and one barrier a step is
// enough.  The finished tile is the pair's part of the next M.  Bound: the
// chain of 32 steps (rotation, broadcast, update, shift) of about 1.1 us: 37 us
// a round at n = 2048 where k_pair_eig, whose 63 steps each move 200 KB
// through LDS, takes 110.
__device__ void pair_cross(const double *__restrict__ g, int64_t ldm, double *__restrict__ qt,
                           double *__restrict__ off_out, double inner_tol, double exempt_tol2, double theta,
                           double *lds, double *__restrict__ M2, int d0, int d1, int *__restrict__ act) {
    double *a = lds;                       // 64 x kLdE staging
    double *red = lds + kPair * kLdE;      // 4 x 3
    double *next = red + 12;               // 2 x (8 x 4 x 32 shifted values, 3 x 32 of the next pairs)
    const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
    for (int idx = tid; idx < kPair * kPair; idx += 256) {
        const int r = idx >> 6, c = idx & 63;
        if (r <= c) {
            const double x = g[r * ldm + c];
            a[r * kLdE + c] = x;
            a[c * kLdE + r] = x;
        }
    }
    __syncthreads();
    double pp[4], pq[4], qp[4], qq[4], vp[4][2], vq[4][2];
    double mx = 0.0, sq = 0.0, sx = 0.0;
    const double dj[2] = {a[tx * kLdE + tx], a[(32 + tx) * kLdE + 32 + tx]};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int i = 4 * ty + m;
        pp[m] = a[i * kLdE + tx];
        pq[m] = a[i * kLdE + 32 + tx];
        qp[m] = a[(32 + i) * kLdE + tx];
        qq[m] = a[(32 + i) * kLdE + 32 + tx];
        const double di[2] = {a[i * kLdE + i], a[(32 + i) * kLdE + 32 + i]};
        const double v[2][2] = {{pp[m], pq[m]}, {qp[m], qq[m]}};
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (r == c && i == tx) continue;
                const double x = fabs(v[r][c]);
                if (di[r] < theta && dj[c] < theta) {
                    sx = fma(x, x, sx);
                } else {
                    mx = fmax(mx, x);
                    sq = fma(x, x, sq);
                }
            }
        vp[m][0] = i == tx ? 1.0 : 0.0;
        vp[m][1] = 0.0;
        vq[m][0] = 0.0;
        vq[m][1] = i == tx ? 1.0 : 0.0;
    }
    mx = wave_max(mx);
    sq = wave_sum(sq);
    sx = wave_sum(sx);
    if ((tid & 63) == 0) {
        red[(tid >> 6) * 3] = mx;
        red[(tid >> 6) * 3 + 1] = sq;
        red[(tid >> 6) * 3 + 2] = sx;
    }
    __syncthreads();
    mx = fmax(fmax(red[0], red[3]), fmax(red[6], red[9]));
    sq = (red[1] + red[4]) + (red[7] + red[10]);
    sx = (red[2] + red[5]) + (red[8] + red[11]);
    if (tid == 0) {
        off_out[0] = mx;
        off_out[1] = sq;
        off_out[2] = sx;
        if (act) *act = mx > inner_tol || sx > exempt_tol2;
    }
    if (mx > inner_tol || sx > exempt_tol2) {
        const int up = (tx + 1) & 31, down = (tx + 31) & 31;
        const int up_lane = 4 * ((tid & 32) + up);  // lane tx + 1 of the same half wave
        const int mi = tx - 4 * ty;                 // 0 <= mi < 4: this thread holds the elements of p_tx, q_tx alone
        const int md = down - 4 * ty;               // and 0 <= md < 4: of rows p_down, column q_tx
        double app = a[tx * kLdE + tx], apq = a[tx * kLdE + 32 + tx], aqq = a[(32 + tx) * kLdE + 32 + tx];
        for (int t = 0; t < 32; ++t) {
            // every half wave computes all 32 rotations, lane tx pair tx's,
            // and takes those of its rows from its lanes
            double c, s;
            schur_rotation(app, aqq, apq, &c, &s);
            const double h = half_tangent(c, s);
            double rh[4], rs[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int lane = 4 * ((tid & 32) + 4 * ty + m);
                rh[m] = lane_shift(h, lane);
                rs[m] = lane_shift(s, lane);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                rotate(rs[m], rh[m], pp[m], qp[m]);
                rotate(rs[m], rh[m], pq[m], qq[m]);
                rotate(s, h, pp[m], pq[m]);
                rotate(s, h, qp[m], qq[m]);
            }
            // next pairing: q_i <- q_{i+1}, q_j <- q_{j+1}; its rotations come
            // from p_i p_i, p_i q_{i+1} and q_{i+1} q_{i+1}
            double *sh = next + ((t + 1) & 1) * 1120, *el = sh + 1024;
            double *mine = sh + ty * 128 + tx;
            mine[0] = qp[0];
            mine[32] = qq[0];
            double dpp = pp[0], dqq = qq[0], dpq = pq[0];
#pragma unroll
            for (int m = 1; m < 4; ++m) {
                dpp = mi == m ? pp[m] : dpp;
                dqq = mi == m ? qq[m] : dqq;
                dpq = md == m ? pq[m] : dpq;
            }
            if (mi >= 0 && mi < 4) {
                el[tx] = dpp;
                el[64 + down] = dqq;
            }
            if (md >= 0 && md < 4) el[32 + down] = dpq;
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int g = 0; g < 2; ++g) rotate(rs[m], rh[m], vp[m][g], vq[m][g]);
            mine[64] = vq[0][0];
            mine[96] = vq[0][1];
            __syncthreads();
            app = el[tx];
            apq = el[32 + tx];
            aqq = el[64 + tx];
            const double *other = sh + ((ty + 1) & 7) * 128;
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                qp[m] = qp[m + 1];
                qq[m] = lane_shift(qq[m + 1], up_lane);
                vq[m][0] = vq[m + 1][0];
                vq[m][1] = vq[m + 1][1];
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) pq[m] = lane_shift(pq[m], up_lane);
            qp[3] = other[tx];
            qq[3] = other[32 + up];
            vq[3][0] = other[64 + tx];
            vq[3][1] = other[96 + tx];
        }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            qt[(4 * ty + m) * kPair + tx + 32 * h] = vp[m][h];
            qt[(32 + 4 * ty + m) * kPair + tx + 32 * h] = vq[m][h];
        }
    if (M2)
        store_pair_tile(M2, ldm, d0, d1, [&](int rb, int cb, int m) {
            return rb ? (cb ? qq[m] : qp[m]) : (cb ? pq[m] : pp[m]);
        });
}

// W' rows of pair i, columns [64 c, 64 c + 64) = Q_i^T W: block 2i + h of 32
// rows goes to slot dst[2i + h].  A pair that rotated nothing only moves.
__device__ void rotate_w(const double *__restrict__ qt, const double *__restrict__ W, double *__restrict__ W2,
                         const int *__restrict__ dst, const int *__restrict__ act, int64_t np, int tile, double *lds) {
    const int tiles = static_cast<int>(np / 64);
    const int i = tile / tiles, c = tile % tiles;
    if (!act[i]) {
        const int r0 = threadIdx.x >> 5, x = (threadIdx.x & 31) * 2;
        const double *w = W + static_cast<int64_t>(i) * 64 * np + c * 64 + x;
        double2 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const double2 *>(w + (r0 + 8 * q) * np);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            *reinterpret_cast<double2 *>(W2 + (static_cast<int64_t>(dst[2 * i + (q >> 2)]) * kBlk + r0 + 8 * (q & 3)) * np +
                                         c * 64 + x) = v[q];
        return;
    }
    double *sA = lds, *sB = lds + 64 * t64::kLdK;
    t64::load(sA, t64::kLdK, qt + static_cast<int64_t>(i) * 4096, 64);
    t64::load(sB, t64::kLdN, W + static_cast<int64_t>(i) * 64 * np + c * 64, np);
    __syncthreads();
    t64::Acc acc;
    acc.zero();
    t64::mul_nn(acc, sA, sB);
    double *o0 = W2 + static_cast<int64_t>(dst[2 * i]) * kBlk * np + c * 64;
    double *o1 = W2 + static_cast<int64_t>(dst[2 * i + 1]) * kBlk * np + c * 64;
    t64::each(acc, [&](int r, int col, double x) { (r < 32 ? o0 : o1)[(r & 31) * np + col] = x; });
}

// A round's step 1 (the first npairs workgroups; none in the sweep's first
// round, which is k_pair_eig's) and step 4 of the round before (the others):
// nothing in a round waits for W, and step 1 leaves most of the chip idle.
__global__ __launch_bounds__(256) void k_pair_cross(const double *__restrict__ M, int64_t np, double *__restrict__ Qt,
                                                    double *__restrict__ off_out, double inner_tol,
                                                    double exempt_tol2, double theta, int npairs,
                                                    const double *__restrict__ Qt_prev, const double *__restrict__ W,
                                                    double *__restrict__ W2, const int *__restrict__ dst_prev,
                                                    const int *__restrict__ act_prev, double *__restrict__ M2,
                                                    const int *__restrict__ dst, int *__restrict__ act) {
    __shared__ __align__(16) double lds[kRotLds];
    const int b = blockIdx.x;
    if (b < npairs) {
        __builtin_amdgcn_s_setprio(3);  // the round waits for this chain, not for W's tiles beside it
        pair_cross(M + (static_cast<int64_t>(kPair) * np + kPair) * b, np, Qt + static_cast<int64_t>(b) * 4096,
                   off_out + 3 * b, inner_tol, exempt_tol2, theta, lds, M2, M2 ? dst[2 * b] : 0, M2 ? dst[2 * b + 1] : 0,
                   act ? act + b : nullptr);
        return;
    }
    rotate_w(Qt_prev, W, W2, dst_prev, act_prev, np, b - npairs, lds);
}

// Steps 2, 3 and 5 of M in one pass: tile (i, j), i < j, of pairs becomes
// Q_i^T M_ij Q_j and goes to the next round's slots (the tiles (i, i) are step
// 1's own result).  Of M only the tiles on and above the diagonal are kept
// (whole 64 x 64 tiles on it): a 32 x 32 block that lands below is stored
// transposed.  Reads half of M and writes half of it where separate products
// and the permutation moved it four times, and at n = 2048 the 496 tiles run
// at once, two on a compute unit, where the 32 diagonal ones made a second,
// almost empty wave.  A pair that rotated nothing takes no product: from the
// second sweep half of the pairs of a truncation are outside the wanted part
// and most of the last sweeps' are done (measured a round: 82 us for the three
// products and the permutation of M and W, 23 us here with the diagonal, 16.5
// without, 6 when no pair rotated; W hidden behind step 1).
__global__ __launch_bounds__(256) void k_rotate_m(const double *__restrict__ M, double *__restrict__ M2,
                                                  const double *__restrict__ Qt, const int *__restrict__ dst,
                                                  const int *__restrict__ act, int64_t np) {
    __shared__ __align__(16) double lds[kRotLds];
    // triangular index: blockIdx.x = j (j - 1) / 2 + i, i < j
    const int b = blockIdx.x;
    int j = static_cast<int>((sqrtf(8.0f * b + 1.0f) + 1.0f) * 0.5f);
    while (j * (j - 1) / 2 > b) --j;
    while (j * (j + 1) / 2 <= b) ++j;
    const int i = b - j * (j - 1) / 2;
    double *sA = lds, *sB = lds + 64 * t64::kLdK;
    const double *tile = M + static_cast<int64_t>(i) * 64 * np + static_cast<int64_t>(j) * 64;
    const bool ai = act[i] != 0, aj = act[j] != 0;  // otherwise Q_i, Q_j is the identity
    if (!ai && !aj) {
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = tile[((threadIdx.x >> 6) + 4 * q) * np + (threadIdx.x & 63)];
#pragma unroll
        for (int q = 0; q < 16; ++q) lds[((threadIdx.x >> 6) + 4 * q) * kLdE + (threadIdx.x & 63)] = v[q];
    } else {
        t64::Acc acc;
        acc.zero();
        if (aj) {
            t64::load(sB, t64::kLdK, tile, np);
            t64::load(sA, t64::kLdK, Qt + static_cast<int64_t>(j) * 4096, 64);
            __syncthreads();
            t64::mul_nt(acc, sB, sA);  // U = M_ij Q_j
            __syncthreads();
        } else {
            t64::load(sB, t64::kLdN, tile, np);  // U = M_ij
        }
        if (ai) {
            t64::load(sA, t64::kLdK, Qt + static_cast<int64_t>(i) * 4096, 64);
            if (aj) t64::each(acc, [&](int r, int c, double x) { sB[r * t64::kLdN + c] = x; });
            __syncthreads();
            acc.zero();
            t64::mul_nn(acc, sA, sB);  // Q_i^T U
            __syncthreads();
        }
        t64::each(acc, [&](int r, int c, double x) { lds[r * kLdE + c] = x; });
    }
    __syncthreads();
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int rb = q >> 1, cb = q & 1;
        const int dr = dst[2 * i + rb], dc = dst[2 * j + cb];
        const double *src = lds + rb * 32 * kLdE + cb * 32;
        if ((dr >> 1) <= (dc >> 1)) {
            double *o = M2 + static_cast<int64_t>(dr) * kBlk * np + static_cast<int64_t>(dc) * kBlk;
#pragma unroll
            for (int r = 0; r < 32; r += 8) o[(r + y) * np + x] = src[(r + y) * kLdE + x];
        }
        if ((dr >> 1) >= (dc >> 1)) {
            double *o = M2 + static_cast<int64_t>(dc) * kBlk * np + static_cast<int64_t>(dr) * kBlk;
#pragma unroll
            for (int r = 0; r < 32; r += 8) o[(r + y) * np + x] = src[x * kLdE + r + y];
        }
    }
}

// Round-0 layout: slot s holds block slot_block[s]: M = P A P^T (zero
// outside n x n), W = the same rows of the identity, or of W0 (of its
// transpose when wtrans is set).
__global__ void k_jac_init(const double *__restrict__ A, int64_t lda, int64_t n, int64_t np,
                           const int *__restrict__ slot_block, double *__restrict__ M, double *__restrict__ W,
                           const double *__restrict__ W0, int wtrans) {
    const int slot = blockIdx.y;
    const int64_t src0 = static_cast<int64_t>(slot_block[slot]) * kBlk;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; c < np;
         c += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t sc = static_cast<int64_t>(slot_block[c / kBlk]) * kBlk + c % kBlk;
        for (int r = 0; r < kBlk; ++r) {
            const int64_t src = src0 + r;
            const int64_t dst = (static_cast<int64_t>(slot) * kBlk + r) * np + c;
            M[dst] = (src < n && sc < n) ? A[src * lda + sc] : 0.0;
            W[dst] = !W0 ? (src == c ? 1.0 : 0.0) : wtrans ? W0[c * np + src] : W0[src * np + c];
        }
    }
}

// Step 5: dst = P src P^T (slot s of dst holds slot src_slot[s] of src, rows
// and columns) for blockIdx.z = 0; Wdst = P Wsrc (rows) for blockIdx.z = 1.
__global__ void k_jac_permute(const double *__restrict__ src, double *__restrict__ dst,
                              const double *__restrict__ Wsrc, double *__restrict__ Wdst,
                              const int *__restrict__ src_slot, int64_t np) {
    const int slot = blockIdx.y;
    const bool sym = blockIdx.z == 0;
    const double *from = (sym ? src : Wsrc) + static_cast<int64_t>(src_slot[slot]) * kBlk * np;
    double *to = (sym ? dst : Wdst) + static_cast<int64_t>(slot) * kBlk * np;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; c < np;
         c += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t sc = sym ? static_cast<int64_t>(src_slot[c / kBlk]) * kBlk + c % kBlk : c;
        for (int r = 0; r < kBlk; ++r) to[r * np + c] = from[r * np + sc];
    }
}

// lam[c] = M_cc; nrm[c] = |w_c restricted to the first n coordinates|^2
__global__ __launch_bounds__(256) void k_jac_diag(const double *__restrict__ M, const double *__restrict__ W,
                                                  int64_t n, int64_t np, double *__restrict__ lam,
                                                  double *__restrict__ nrm) {
    __shared__ double r2[256];
    const int64_t row = blockIdx.x;
    const double *w = W + row * np;
    double t = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) t = fma(w[i], w[i], t);
    r2[threadIdx.x] = t;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (static_cast<int>(threadIdx.x) < k) r2[threadIdx.x] += r2[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        lam[row] = M[row * np + row];
        nrm[row] = r2[0];
    }
}

// lam[c] = t_c . w_c with T = W A, nrm[c] = |w_c|^2 (first n coordinates): the
// native path's final eigenvalues.  Its M is not W A W^T to rounding: a tile on
// the diagonal goes through 32 rotations a round one after another, and a
// rotation by a small angle (s^2 below u / 2, as between rows of nearly equal
// eigenvalues) lengthens its row of W by s^2 while M's entry rounds that away,
// always in the same direction.  On four clusters of 256 at n = 1024 the
// diagonal drifts by up to 680 u, the quotients are within 24 u.  One
// product of n_p x n x n: 0.29 ms of a truncation of 32 at n = 2048.
__global__ __launch_bounds__(256) void k_rayleigh(const double *__restrict__ T, const double *__restrict__ W,
                                                  int64_t n, int64_t np, double *__restrict__ lam,
                                                  double *__restrict__ nrm) {
    __shared__ double red[256];
    const int64_t row = blockIdx.x;
    const double *w = W + row * np, *t = T + row * np;
    double q = 0.0, s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        q = fma(t[i], w[i], q);
        s = fma(w[i], w[i], s);
    }
    q = block_sum(q, red);
    s = block_sum(s, red);
    if (threadIdx.x == 0) {
        lam[row] = q;
        nrm[row] = s;
    }
}

// Z[i][j] = scale[j] W[rows[j]][i], i < n, j < nev (through a 32 x 32 LDS tile)
__global__ void k_jac_gather(const double *__restrict__ W, int64_t np, const int *__restrict__ rows,
                             const double *__restrict__ scale, int64_t n, int64_t nev, double *__restrict__ Z,
                             int64_t ldz) {
    __shared__ double tile[32][33];
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * 32, j0 = static_cast<int64_t>(blockIdx.y) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
    for (int r = ty; r < 32; r += 8) {
        const int64_t j = j0 + r, i = i0 + tx;
        tile[r][tx] = (j < nev && i < n) ? scale[j] * W[static_cast<int64_t>(rows[j]) * np + i] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int64_t i = i0 + r, j = j0 + tx;
        if (i < n && j < nev) Z[i * ldz + j] = tile[tx][r];
    }
}

// What a block's rows of M hold above the diagonal: out[3 blk ..] = the largest
// counted magnitude, the counted and the exempt sum of squares (offdiag).
__global__ __launch_bounds__(256) void k_offdiag(const double *__restrict__ M, int64_t np, double theta,
                                                 double *__restrict__ out) {
    __shared__ double red[256];
    double m = 0.0, q = 0.0, qx = 0.0;
    for (int64_t r = blockIdx.x; r < np; r += gridDim.x) {
        const double *row = M + r * np;
        const bool low = row[r] < theta;
        for (int64_t c = r + 1 + threadIdx.x; c < np; c += 256) {
            const double x = fabs(row[c]);
            if (low && M[c * np + c] < theta) {
                qx = fma(x, x, qx);
            } else {
                m = fmax(m, x);
                q = fma(x, x, q);
            }
        }
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    m = red[0];
    __syncthreads();
    q = block_sum(q, red);
    qx = block_sum(qx, red);
    if (threadIdx.x == 0) {
        out[3 * blockIdx.x] = m;
        out[3 * blockIdx.x + 1] = q;
        out[3 * blockIdx.x + 2] = qx;
    }
}

// bad <- 1 if A has a NaN or Inf; part[block] = sum of squares of the block's
// entries, part[gridDim.x + block] of those off the diagonal
__global__ __launch_bounds__(256) void k_scan(const double *__restrict__ A, int64_t lda, int64_t n,
                                              int *__restrict__ bad, double *__restrict__ part) {
    __shared__ double r[256];
    int found = 0;
    double ss = 0.0, so = 0.0;
    for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < n * n;
         idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const double x = A[(idx / n) * lda + idx % n];
        if (!(fabs(x) <= 1.79769313486231570e308)) found = 1;
        else {
            ss = fma(x, x, ss);
            if (idx / n != idx % n) so = fma(x, x, so);
        }
    }
    if (found) atomicOr(bad, 1);
    const double t = block_sum(ss, r), to = block_sum(so, r);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = t;
        part[gridDim.x + blockIdx.x] = to;
    }
}

}  // namespace

struct rdm_eig_s {
    ozaki_ctx ctx = nullptr;
    int64_t n = 0, np = 0;
    int S = 0, G = 0, nb = 0, npairs = 0, rounds = 0;
    std::vector<void *> allocs;
    double *X = nullptr, *Y = nullptr;    // M and its ping-pong partner, np x np
    double *W = nullptr, *W2 = nullptr;   // basis rows and their rotation, np x np
    double *V = nullptr;                  // QR iteration: Q of the first pass, then the new M, np x np
    double *P = nullptr, *Linv = nullptr; // its panel and diagonal block
    double *Qt = nullptr, *off = nullptr, *lam = nullptr, *nrm = nullptr, *part = nullptr, *scale = nullptr;
    int *slot0 = nullptr, *maps = nullptr, *dst = nullptr, *rows = nullptr, *bad = nullptr;
    unsigned cross_lds = 0;               // bytes of LDS on top of k_pair_cross's own
    int *act = nullptr;                   // pairs that rotated, of this round and the one before
    int start_steps = 0;                  // steps of QR iteration the last solve's sweeps started from
    int ntiles = 0;  // pairs x 64-column tiles
    TileDesc *tiles = nullptr;
    OutDesc *outs = nullptr;
    // emulated: Qt slices, pair panels by columns (trans) and by rows
    int32_t *eQ = nullptr, *eR = nullptr, *eC = nullptr;
    int8_t *pQ = nullptr, *pR = nullptr, *pC = nullptr;
    SliceBlock *bR = nullptr, *bC = nullptr;
    SliceTask *eR_t = nullptr, *sR_t = nullptr, *eC_t = nullptr, *sC_t = nullptr;
    int n_eR = 0, n_sR = 0, n_eC = 0, n_sC = 0;
    TermDesc *e_rows = nullptr, *e_cols = nullptr;
    std::vector<double> host_off;
};

namespace {

int ralloc(rdm_eig h, size_t bytes, void **p) {
    hipError_t e = hipMalloc(p, bytes < 256 ? 256 : bytes);
    if (e != hipSuccess) return fail(OZ_ERR_NOMEM, "rdm_eig_create: %zu bytes: %s", bytes, hipGetErrorString(e));
    h->allocs.push_back(*p);
    return OZ_OK;
}

template <typename T>
int rupload(rdm_eig h, const std::vector<T> &v, T **out) {
    void *p;
    int rc = ralloc(h, sizeof(T) * std::max<size_t>(v.size(), 1), &p);
    if (rc) return rc;
    hipError_t e = hipMemcpy(p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "rdm_eig_create: descriptor upload");
    *out = static_cast<T *>(p);
    return OZ_OK;
}

void rfree(rdm_eig h) {
    for (void *p : h->allocs) hipFree(p);
    delete h;
}

// C rows of each pair <- Q_k^T times the pair's rows of `src` (cols = false)
// or the transpose of its columns (cols = true), emulated.
int rotate(rdm_eig h, const double *src, double *C, bool cols, hipStream_t s) {
    hipError_t e;
    if (cols) {
        if ((e = launch_exponents_grouped(h->bC, h->eC_t, h->n_eC, src, h->eC, h->ctx->d_flags, s)) != hipSuccess ||
            (e = launch_slice_grouped(h->S, h->bC, h->sC_t, h->n_sC, src, h->eC, h->pC, s)) != hipSuccess)
            return hip_fail(e, "rdm_eig: slicing columns");
    } else {
        if ((e = launch_exponents_grouped(h->bR, h->eR_t, h->n_eR, src, h->eR, h->ctx->d_flags, s)) != hipSuccess ||
            (e = launch_slice_grouped(h->S, h->bR, h->sR_t, h->n_sR, src, h->eR, h->pR, s)) != hipSuccess)
            return hip_fail(e, "rdm_eig: slicing rows");
    }
    PairArgs a{};
    a.tiles = h->tiles;
    a.terms = cols ? h->e_cols : h->e_rows;
    a.outs = h->outs;
    a.ntiles = h->ntiles;
    a.mode = kModeGemm;
    a.out_base = C;
    e = launch_pair_grouped(h->S, h->G, 0, a, s);
    return e == hipSuccess ? OZ_OK : hip_fail(e, "rdm_eig: rotation");
}

// Where the sweeps start from: M (n x n, ldm), the basis rows W0 (nullptr:
// the identity; wtrans: its transpose) and the buffers the sweeps use.
struct JacStart {
    const double *M;
    int64_t ldm;
    const double *W0;
    int wtrans;
    double *X, *Y, *W, *W2;  // M and its ping-pong partner, the basis rows and theirs
};

// Step 1 of round r: every rotation of the pairs' blocks in a sweep's first
// round, the ones that couple the two blocks in the others; with W set also
// step 4 of round r - 1 (W -> W2), with M2 set the pairs' own tiles into it.
int pair_step(rdm_eig h, int r, const double *M, double *Qt, double inner_tol, double exempt_tol2, double theta,
              const double *Qt_prev, const double *W, double *W2, double *M2, hipStream_t s) {
    const int64_t np = h->np;
    const int *dst = h->dst + static_cast<int64_t>(r) * h->nb;
    int *act = M2 ? h->act + (r & 1) * h->npairs : nullptr;
    double *off = h->off + static_cast<int64_t>(r) * h->npairs * 3;
    if (r == 0)
        hipLaunchKernelGGL(k_pair_eig, dim3(h->npairs), dim3(256), 0, s, M, np, Qt, off, inner_tol, exempt_tol2, theta,
                           M2, dst, act);
    else
        hipLaunchKernelGGL(k_pair_cross, dim3(h->npairs + (W ? h->ntiles : 0)), dim3(256), W ? h->cross_lds : 0, s, M, np,
                           Qt, off, inner_tol, exempt_tol2, theta, h->npairs, Qt_prev, W, W2,
                           W ? dst - h->nb : nullptr, W ? h->act + ((r + 1) & 1) * h->npairs : nullptr, M2, dst, act);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? OZ_OK : hip_fail(e, "rdm_eig: pair eigensolver");
}

// The first `rounds` rounds of a sweep in native FP64: two launches a round, W
// one round behind M.
int sweep_native(rdm_eig h, JacStart *st, int rounds, double inner_tol, double exempt_tol2, double theta, hipStream_t s) {
    const int64_t np = h->np;
    const int tri = h->npairs * (h->npairs - 1) / 2;
    hipError_t e;
    for (int r = 0; r < rounds; ++r) {
        double *Qt = h->Qt + (r & 1) * np * kPair, *prev = h->Qt + ((r + 1) & 1) * np * kPair;
        const int rc = pair_step(h, r, st->X, Qt, inner_tol, exempt_tol2, theta, prev, st->W, st->W2, st->Y, s);
        if (rc != OZ_OK) return rc;
        if (r > 0) std::swap(st->W, st->W2);
        if (tri > 0)
            hipLaunchKernelGGL(k_rotate_m, dim3(tri), dim3(256), 0, s, st->X, st->Y, Qt,
                               h->dst + static_cast<int64_t>(r) * h->nb, h->act + (r & 1) * h->npairs, np);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "rdm_eig: rotation");
        std::swap(st->X, st->Y);
    }
    const int last = rounds - 1;
    hipLaunchKernelGGL(k_pair_cross, dim3(h->ntiles), dim3(256), 0, s, nullptr, np, nullptr, nullptr, 0.0, 0.0, 0.0, 0,
                       h->Qt + (last & 1) * np * kPair, st->W, st->W2, h->dst + static_cast<int64_t>(last) * h->nb,
                       h->act + (last & 1) * h->npairs, nullptr, nullptr, nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "rdm_eig: basis rotation");
    std::swap(st->W, st->W2);
    return OZ_OK;
}

// One round (steps 1-5) in emulated arithmetic: M in src on entry, in dst on exit.
int enqueue_round(rdm_eig h, int r, const double *src_c, double *dst, double *W, double *W2, double inner_tol,
                  double exempt_tol2, double theta, hipStream_t s) {
    const int64_t np = h->np;
    double *src = const_cast<double *>(src_c);
    hipError_t e;
    int rc;
    if ((rc = pair_step(h, r, src, h->Qt, inner_tol, exempt_tol2, theta, nullptr, nullptr, nullptr, nullptr, s)) != OZ_OK)
        return rc;
    if ((e = launch_row_exponents(h->Qt, kPair, np, kPair, h->eQ, h->ctx->d_flags, s)) != hipSuccess ||
        (e = launch_slice(h->S, false, h->Qt, kPair, np, kPair, h->eQ, h->pQ, np, s)) != hipSuccess)
        return hip_fail(e, "rdm_eig: slicing Q");
    if ((rc = rotate(h, src, dst, false, s)) != OZ_OK) return rc;    // R = Q^T M
    if ((rc = rotate(h, dst, src, true, s)) != OZ_OK) return rc;     // M' = Q^T R^T
    if ((rc = rotate(h, W, W2, false, s)) != OZ_OK) return rc;       // W <- Q^T W
    const unsigned cx = static_cast<unsigned>(std::min<int64_t>(ceil_div(np, 256), 16));
    hipLaunchKernelGGL(k_jac_permute, dim3(cx, h->nb, 2), dim3(256), 0, s, src, dst, W2, W,
                       h->maps + static_cast<int64_t>(r) * h->nb, np);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "rdm_eig: permute");
    return OZ_OK;
}

// One step of QR iteration: Q R = M + mu I (M: n x n, ldm), Mout = Q^T M Q
// with zero padding, all np x np.  Scratch: G and T (may be one buffer), B
// (may be Q) and Q1 (may be Mout).
int qr_step(rdm_eig h, const double *M, int64_t ldm, double mu, double unit, double *B, double *G, double *Q1,
            double *Q, double *T, double *Mout, int *bad, hipStream_t s) {
    const int64_t n = h->n, np = h->np;
    const int cu = h->ctx->num_cu;
    hipError_t e;
    if ((e = launch_shifted_copy(M, ldm, n, np, mu, unit, B, s)) != hipSuccess ||
        (e = launch_cholqr_pass(G, B, Q1, h->P, h->Linv, np, bad, 0.0, INFINITY, cu, s)) != hipSuccess ||
        (e = launch_cholqr_pass(G, Q1, Q, h->P, h->Linv, np, bad, 0.5, 2.0, cu, s)) != hipSuccess)
        return hip_fail(e, "rdm_eig: Cholesky QR");
    Dgemm64Args a{};
    a.mode = kModeGemm;
    a.term = Term64{M, Q, ldm, np, static_cast<int32_t>(n), 0, 1.0};
    a.out = OutDesc{T, np, static_cast<int32_t>(n), static_cast<int32_t>(n)};
    if ((e = launch_dgemm_single(false, false, a, cu, s)) != hipSuccess) return hip_fail(e, "rdm_eig: M Q");
    if ((e = hipMemsetAsync(Mout, 0, sizeof(double) * np * np, s)) != hipSuccess) return hip_fail(e, "rdm_eig: clear");
    a.term = Term64{Q, T, np, np, static_cast<int32_t>(n), 0, 1.0};
    a.out = OutDesc{Mout, np, static_cast<int32_t>(n), static_cast<int32_t>(n)};
    if ((e = launch_dgemm_single(true, false, a, cu, s)) != hipSuccess) return hip_fail(e, "rdm_eig: Q^T M Q");
    return OZ_OK;
}

// QR iteration orders the diagonal by decreasing eigenvalue magnitude and
// shrinks the couplings by the ratio of the eigenvalues, which is what cyclic
// Jacobi is slow at on the graded spectra of density matrices: at n = 2048 on
// a spectrum e^(-i/32) the sweeps go from 28 to 7 and the truncation from 363
// to 108 ms (FP64).  The shift keeps the
// condition number of M + mu I (about 3e6 for a positive semidefinite A)
// inside what Cholesky QR can take; the second step, on an M already graded,
// gets by with a far smaller one, since the factorisation is invariant to the
// scaling of its columns.  A step whose factorisation breaks down (a nearly
// singular M + mu I of an indefinite A) is left out.
int precondition(rdm_eig h, const double *A, int64_t lda, double fro, JacStart *st, hipStream_t s) {
    const int64_t np = h->np;
    hipError_t e;
    int bad[2] = {0, 0};
    int rc;
    if ((e = hipMemsetAsync(h->bad, 0, 2 * sizeof(int), s)) != hipSuccess) return hip_fail(e, "rdm_eig: flags");
    // step 1: Q1 in W2, M1 in Y; step 2: Q2 in X, M2 in V
    if ((rc = qr_step(h, A, lda, 3e-7 * fro, fro, h->W2, h->W, h->V, h->W2, h->W, h->Y, h->bad, s)) != OZ_OK ||
        (rc = qr_step(h, h->Y, np, 3e-12 * fro, fro, h->X, h->W, h->V, h->X, h->W, h->V, h->bad + 1, s)) != OZ_OK)
        return rc;
    // basis rows (Q1 Q2)^T
    Dgemm64Args a{};
    a.mode = kModeGemm;
    a.term = Term64{h->X, h->W2, np, np, static_cast<int32_t>(np), 0, 1.0};
    a.out = OutDesc{h->W, np, static_cast<int32_t>(np), static_cast<int32_t>(np)};
    if ((e = launch_dgemm_single(true, true, a, h->ctx->num_cu, s)) != hipSuccess) return hip_fail(e, "rdm_eig: basis");
    if ((e = hipMemcpyAsync(bad, h->bad, sizeof(bad), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return hip_fail(e, "rdm_eig: QR flags");
    h->start_steps = bad[0] ? 0 : bad[1] ? 1 : 2;
    if (bad[0]) return OZ_OK;
    if (bad[1])
        *st = JacStart{h->Y, np, h->W2, 1, h->X, h->V, h->W, h->W2};
    else
        *st = JacStart{h->V, np, h->W, 0, h->X, h->Y, h->W2, h->W};
    return OZ_OK;
}

}  // namespace

extern "C" {

int rdm_eig_create(ozaki_ctx ctx, rdm_eig *out, int64_t n, int slices, int ndiag) {
    if (!out) return fail(OZ_ERR_ARG, "rdm_eig_create: out is NULL");
    *out = nullptr;
    if (!ctx) return fail(OZ_ERR_ARG, "rdm_eig_create: ctx is NULL");
    if (n < 1 || n > kMaxEigN) return fail(OZ_ERR_ARG, "rdm_eig_create: n = %lld (1..%lld)", (long long)n,
                                           (long long)kMaxEigN);
    if (slices != 0 && (slices < 2 || slices > 8)) return fail(OZ_ERR_ARG, "rdm_eig_create: slices = %d", slices);
    const int G = slices ? resolve_ndiag(slices, ndiag) : 0;
    if (slices && !valid_sg(slices, G))
        return fail(OZ_ERR_ARG, "rdm_eig_create: ndiag = %d for slices = %d (use S, S+1 or 2S-1)", ndiag, slices);
    const int64_t np = round_up(n, kPair);
    hipError_t e;
    if ((e = hipSetDevice(ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
    rdm_eig h = new rdm_eig_s();
    h->ctx = ctx;
    h->n = n;
    h->np = np;
    h->S = slices;
    h->G = G;
    h->nb = static_cast<int>(np / kBlk);
    h->npairs = h->nb / 2;
    h->rounds = h->nb - 1;
    int rc;
    void *p;
    const size_t mat = sizeof(double) * static_cast<size_t>(np) * np;
#define OZ_RA(field, bytes) \
    if ((rc = ralloc(h, (bytes), &p)) != OZ_OK) { rfree(h); return rc; } \
    h->field = static_cast<decltype(h->field)>(p);
    OZ_RA(X, mat)
    OZ_RA(Y, mat)
    OZ_RA(W, mat)
    OZ_RA(W2, mat)
    OZ_RA(V, mat)
    OZ_RA(P, sizeof(double) * np * kPair)
    OZ_RA(Linv, sizeof(double) * kPair * kPair)
    OZ_RA(Qt, 2 * sizeof(double) * np * kPair)
    OZ_RA(off, sizeof(double) * h->rounds * h->npairs * 3)
    OZ_RA(lam, sizeof(double) * np)
    OZ_RA(nrm, sizeof(double) * np)
    OZ_RA(scale, sizeof(double) * np)
    OZ_RA(rows, sizeof(int) * np)
    OZ_RA(bad, sizeof(int) * 4)
    OZ_RA(act, sizeof(int) * 2 * h->npairs)
    OZ_RA(part, sizeof(double) * 2 * kScanBlocks)
#undef OZ_RA
    // A workgroup of step 1 slows down when a tile of W shares its compute
    // unit (45 us against 38 at n = 2048).  While W's tiles go round the other
    // compute units one at a time within step 1's time (8 us each, so up to
    // five rounds), every workgroup of the launch takes more than
    // half of a compute unit's 160 KiB; with more tiles two at a time are
    // faster.
    if (static_cast<int64_t>(h->npairs) * (np / 64) <= 5 * static_cast<int64_t>(ctx->num_cu - h->npairs))
        h->cross_lds = 84 * 1024 - sizeof(double) * kRotLds;
    // circle schedule over the nb blocks
    std::vector<int> a(h->nb);
    std::iota(a.begin(), a.end(), 0);
    std::vector<std::vector<int>> slot_block(h->rounds, std::vector<int>(h->nb));
    for (int r = 0; r < h->rounds; ++r) {
        for (int k = 0; k < h->npairs; ++k) {
            slot_block[r][2 * k] = a[k];
            slot_block[r][2 * k + 1] = a[h->nb - 1 - k];
        }
        std::rotate(a.begin() + 1, a.end() - 1, a.end());
    }
    // maps: the slot a slot's rows come from after round r; dst: the slot its rows go to
    std::vector<int> maps(static_cast<size_t>(h->rounds) * h->nb), dst(maps.size());
    for (int r = 0; r < h->rounds; ++r) {
        const std::vector<int> &cur = slot_block[r], &nxt = slot_block[(r + 1) % h->rounds];
        std::vector<int> slot_of(h->nb);
        for (int sl = 0; sl < h->nb; ++sl) slot_of[cur[sl]] = sl;
        for (int sl = 0; sl < h->nb; ++sl) {
            const int from = slot_of[nxt[sl]];
            maps[static_cast<size_t>(r) * h->nb + sl] = from;
            dst[static_cast<size_t>(r) * h->nb + from] = sl;
        }
    }
    if ((rc = rupload(h, slot_block[0], &h->slot0)) || (rc = rupload(h, maps, &h->maps)) ||
        (rc = rupload(h, dst, &h->dst))) {
        rfree(h);
        return rc;
    }
    // tiles: pair k x 64-column tile c, row offset 64k into Qt and the output
    const int ctiles = static_cast<int>(np / 64);
    std::vector<TileDesc> tiles;
    for (int k = 0; k < h->npairs; ++k)
        for (int c = 0; c < ctiles; ++c) tiles.push_back(TileDesc{k, k + 1, kPair * k, 64 * c, 0, 0});
    h->ntiles = static_cast<int>(tiles.size());
    // outputs and B operands are element offsets from the buffers passed at launch
    const std::vector<OutDesc> outs{OutDesc{nullptr, np, static_cast<int32_t>(np), static_cast<int32_t>(np)}};
    if ((rc = rupload(h, tiles, &h->tiles)) || (rc = rupload(h, outs, &h->outs))) {
        rfree(h);
        return rc;
    }
    if (slices) {
        if ((rc = ralloc(h, sizeof(int32_t) * np, &p)) != OZ_OK) { rfree(h); return rc; }
        h->eQ = static_cast<int32_t *>(p);
        if ((rc = ralloc(h, static_cast<size_t>(slices) * np * kPair, &p)) != OZ_OK) { rfree(h); return rc; }
        h->pQ = static_cast<int8_t *>(p);
        // B operands: the pair's 64 rows grouped by columns (R = Q^T M, W), or
        // the pair's 64 columns grouped by rows (Q^T R^T)
        SliceSet setR, setC;
        std::vector<int64_t> eoR, poR, eoC, poC;
        for (int k = 0; k < h->npairs; ++k) {
            int64_t eo, po;
            setR.add(static_cast<int64_t>(kPair) * k * np, np, np, kPair, true, slices, &eo, &po);
            eoR.push_back(eo);
            poR.push_back(po);
            setC.add(static_cast<int64_t>(kPair) * k, np, np, kPair, false, slices, &eo, &po);
            eoC.push_back(eo);
            poC.push_back(po);
        }
        if ((rc = rupload(h, setR.blocks, &h->bR)) || (rc = rupload(h, setR.etasks, &h->eR_t)) ||
            (rc = rupload(h, setR.stasks, &h->sR_t)) || (rc = rupload(h, setC.blocks, &h->bC)) ||
            (rc = rupload(h, setC.etasks, &h->eC_t)) || (rc = rupload(h, setC.stasks, &h->sC_t))) {
            rfree(h);
            return rc;
        }
        h->n_eR = static_cast<int>(setR.etasks.size());
        h->n_sR = static_cast<int>(setR.stasks.size());
        h->n_eC = static_cast<int>(setC.etasks.size());
        h->n_sC = static_cast<int>(setC.stasks.size());
        if ((rc = ralloc(h, sizeof(int32_t) * setR.e_total, &p)) != OZ_OK) { rfree(h); return rc; }
        h->eR = static_cast<int32_t *>(p);
        if ((rc = ralloc(h, setR.p_total, &p)) != OZ_OK) { rfree(h); return rc; }
        h->pR = static_cast<int8_t *>(p);
        if ((rc = ralloc(h, sizeof(int32_t) * setC.e_total, &p)) != OZ_OK) { rfree(h); return rc; }
        h->eC = static_cast<int32_t *>(p);
        if ((rc = ralloc(h, setC.p_total, &p)) != OZ_OK) { rfree(h); return rc; }
        h->pC = static_cast<int8_t *>(p);
        std::vector<TermDesc> tr, tc;
        for (int k = 0; k < h->npairs; ++k) {
            tr.push_back(TermDesc{h->pQ, h->eQ, h->pR + poR[k], h->eR + eoR[k], np, np, kPair / kKB, 0, 1.0});
            tc.push_back(TermDesc{h->pQ, h->eQ, h->pC + poC[k], h->eC + eoC[k], np, np, kPair / kKB, 0, 1.0});
        }
        if ((rc = rupload(h, tr, &h->e_rows)) || (rc = rupload(h, tc, &h->e_cols))) {
            rfree(h);
            return rc;
        }
    }
    *out = h;
    return OZ_OK;
}

int rdm_eig_solve(rdm_eig h, const double *A, int64_t lda, int64_t nev, double *evals, double *Z, int64_t ldz,
                  double tol, int max_sweeps, rdm_eig_info *info, void *stream) {
    if (!h) return fail(OZ_ERR_ARG, "rdm_eig_solve: NULL solver");
    const int64_t n = h->n, np = h->np;
    if (!A || lda < n) return fail(OZ_ERR_ARG, "rdm_eig_solve: A is NULL or lda < n");
    if (nev < 0 || nev > n) return fail(OZ_ERR_ARG, "rdm_eig_solve: nev = %lld (0..%lld)", (long long)nev,
                                        (long long)n);
    if (nev > 0 && (!evals || !Z || ldz < nev)) return fail(OZ_ERR_ARG, "rdm_eig_solve: evals / Z / ldz");
    if (max_sweeps < 1) return fail(OZ_ERR_ARG, "rdm_eig_solve: max_sweeps = %d", max_sweeps);
    if (!(tol >= 0.0)) return fail(OZ_ERR_ARG, "rdm_eig_solve: tol");
    // unit roundoff of the arithmetic in use: FP64, or the emulation's 8S - 1 bits
    const double u_eff = h->S ? std::max(0x1p-53, std::ldexp(1.0, 1 - 8 * h->S)) : 0x1p-53;
    if (tol == 0.0) tol = 4.0 * std::sqrt(static_cast<double>(np)) * u_eff;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if ((e = hipSetDevice(h->ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
    int hb[1] = {0};
    if ((e = hipMemcpyAsync(h->bad, hb, sizeof(int), hipMemcpyHostToDevice, s)) != hipSuccess)
        return hip_fail(e, "rdm_eig_solve: flag");
    const unsigned scan_blocks = static_cast<unsigned>(std::min<int64_t>(ceil_div(n * n, 256), kScanBlocks));
    hipLaunchKernelGGL(k_scan, dim3(scan_blocks), dim3(256), 0, s, A, lda, n, h->bad, h->part);
    std::vector<double> part(2 * scan_blocks);
    if ((e = hipMemcpyAsync(hb, h->bad, sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipMemcpyAsync(part.data(), h->part, sizeof(double) * part.size(), hipMemcpyDeviceToHost, s)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return hip_fail(e, "rdm_eig_solve: finiteness check");
    if (hb[0]) return fail(OZ_ERR_ARG, "rdm_eig_solve: A has NaN or Inf entries");
    double fro2 = 0.0, off2 = 0.0;
    for (unsigned i = 0; i < scan_blocks; ++i) {
        fro2 += part[i];
        off2 += part[scan_blocks + i];
    }
    const double fro = std::sqrt(fro2);
    const double abs_tol = tol * fro;
    JacStart st{A, lda, nullptr, 0, h->X, h->Y, h->W, h->W2};
    h->start_steps = 0;
    // QR iteration first, unless A is nearly diagonal already (the sweeps
    // then converge at once and leave an exactly diagonal A exact), a single
    // pair of blocks (one round a sweep), or |A|_F^2 is near the range's ends
    if (np > kPair && off2 > 1e-6 * fro2 && fro > 1e-120 && fro < 1e120) {
        const int rc = precondition(h, A, lda, fro, &st, s);
        if (rc != OZ_OK) return rc;
    }
    hipLaunchKernelGGL(k_jac_init, dim3(static_cast<unsigned>(std::min<int64_t>(ceil_div(np, 256), 16)), h->nb),
                       dim3(256), 0, s, st.M, st.ldm, n, np, h->slot0, st.X, st.W, st.W0, st.wtrans);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "rdm_eig_solve: init");
    int status = OZ_MAX_ITER, sweeps = 0, no_progress = 0;
    double best = INFINITY, last = INFINITY;
    h->host_off.resize(static_cast<size_t>(h->rounds) * h->npairs * 3);
    std::vector<double> lam(np), nrm(np);
    // Diagonal of M over the squared basis norms (with `quotients`, w A w^T
    // over them) and the basis rows inside the first n coordinates (the others
    // are padding).
    auto diagonal = [&](std::vector<int> *rows, bool quotients) -> int {
        if (quotients) {
            Dgemm64Args a{};
            a.mode = kModeGemm;
            a.term = Term64{st.W, A, np, lda, static_cast<int32_t>(n), 0, 1.0};
            a.out = OutDesc{st.Y, np, static_cast<int32_t>(np), static_cast<int32_t>(n)};
            if ((e = launch_dgemm_single(false, false, a, h->ctx->num_cu, s)) != hipSuccess)
                return hip_fail(e, "rdm_eig_solve: W A");
            hipLaunchKernelGGL(k_rayleigh, dim3(static_cast<unsigned>(np)), dim3(256), 0, s, st.Y, st.W, n, np, h->lam,
                               h->nrm);
        } else {
            hipLaunchKernelGGL(k_jac_diag, dim3(static_cast<unsigned>(np)), dim3(256), 0, s, st.X, st.W, n, np, h->lam,
                               h->nrm);
        }
        if ((e = hipMemcpyAsync(lam.data(), h->lam, sizeof(double) * np, hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipMemcpyAsync(nrm.data(), h->nrm, sizeof(double) * np, hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return hip_fail(e, "rdm_eig_solve: eigenvalues");
        rows->clear();
        for (int64_t c = 0; c < np; ++c)
            if (nrm[c] > 0.5) rows->push_back(static_cast<int>(c));
        if (static_cast<int64_t>(rows->size()) != n)
            return fail(OZ_ERR_HIP, "rdm_eig_solve: %zu basis rows inside the first %lld coordinates (expected %lld)",
                        rows->size(), (long long)n, (long long)n);
        // the emulated rotations are orthogonal only to the emulation's precision
        for (int c : *rows) lam[c] /= nrm[c];
        std::stable_sort(rows->begin(), rows->end(), [&](int x, int y) { return lam[x] > lam[y]; });
        return OZ_OK;
    };
    std::vector<int> rows;
    // Rows whose diagonal is below theta are outside the wanted part: their
    // mutual couplings are exempt from tol (nev = n: none is).  theta is the
    // midpoint of the gap at the nev-th value of the previous sweep.
    // Exempt couplings are rotated away only while a round's block holds more
    // than its share (exempt_tol2) of the mass that Weyl's bound allows.
    double theta = -INFINITY, exempt_tol2 = 0.0;
    bool met = false;  // native: an earlier sweep met nothing above tol
    for (int sw = 0; sw < max_sweeps && fro > 0.0; ++sw) {
        int rc = OZ_OK;
        if (h->S == 0) {
            rc = sweep_native(h, &st, h->rounds, 0.1 * abs_tol, exempt_tol2, theta, s);
        } else {
            for (int r = 0; r < h->rounds && rc == OZ_OK; ++r) {
                rc = enqueue_round(h, r, st.X, st.Y, st.W, st.W2, 0.1 * abs_tol, exempt_tol2, theta, s);
                std::swap(st.X, st.Y);
            }
        }
        if (rc != OZ_OK) return rc;
        sweeps = sw + 1;
        if ((e = hipMemcpyAsync(h->host_off.data(), h->off, sizeof(double) * h->host_off.size(),
                                hipMemcpyDeviceToHost, s)) != hipSuccess)
            return hip_fail(e, "rdm_eig_solve: sweep");
        if ((rc = diagonal(&rows, false)) != OZ_OK) return rc;
        double sum = 0.0, exempt = 0.0;
        last = 0.0;
        for (size_t i = 0; i < h->host_off.size(); i += 3) {
            last = std::max(last, h->host_off[i]);
            sum += h->host_off[i + 1];
            exempt += h->host_off[i + 2];
        }
        last /= fro;
        // the wanted rows are decoupled to tol, and by Weyl's bound the
        // exempt couplings cannot lift an unwanted eigenvalue above them
        bool separated = true;
        double lo = 0.0, hi = 0.0;
        if (nev < n) {
            lo = lam[rows[nev - 1 < 0 ? 0 : nev - 1]];
            hi = lam[rows[nev]];
            separated = nev == 0 || (hi < theta && theta <= lo && hi + std::sqrt(exempt) < lo);
            theta = nev == 0 ? INFINITY : 0.5 * (lo + hi);
            exempt_tol2 = nev == 0 ? INFINITY : 0.25 * (lo - hi) * (lo - hi) / (static_cast<double>(h->npairs) * h->rounds);
        }
        bool done = last <= tol && separated;
        if (h->S == 0) {
            // the sweep's figures are those met on the way; what it left
            // behind is one read of M, where a sweep that only finds the same
            // takes 63 rounds at n = 2048
            const int blocks = static_cast<int>(std::min<int64_t>({np, 1024, static_cast<int64_t>(h->rounds) * h->npairs}));
            double now = 0.0;
            bool clean = false;
            auto left_behind = [&]() -> int {
                hipLaunchKernelGGL(k_offdiag, dim3(blocks), dim3(256), 0, s, st.X, np, theta, h->off);
                if ((e = hipMemcpyAsync(h->host_off.data(), h->off, sizeof(double) * 3 * blocks, hipMemcpyDeviceToHost,
                                        s)) != hipSuccess ||
                    (e = hipStreamSynchronize(s)) != hipSuccess)
                    return hip_fail(e, "rdm_eig_solve: off-diagonal");
                double left = 0.0;
                now = 0.0;
                for (int i = 0; i < 3 * blocks; i += 3) {
                    now = std::max(now, h->host_off[i]);
                    left += h->host_off[i + 2];
                }
                now /= fro;
                clean = now <= 0.1 * tol &&
                        (nev == 0 || nev == n || (hi < theta && theta <= lo && hi + std::sqrt(2.0 * left) < lo));
                return OZ_OK;
            };
            if ((rc = left_behind()) != OZ_OK) return rc;
            if (!clean && (done || now <= tol)) {
                // Nothing above tol met or left, yet more than the tenth of it
                // that a sweep leaves unrotated: where that is what the later
                // rounds moved into the 32 x 32 diagonal blocks, which only a
                // first round rotates, one such round takes it away; else one
                // more sweep does, or the arithmetic's floor is reached.
                if ((rc = sweep_native(h, &st, 1, 0.1 * abs_tol, exempt_tol2, theta, s)) != OZ_OK ||
                    (rc = left_behind()) != OZ_OK)
                    return rc;
            }
            if (clean && !done) last = now;
            const bool again = done && !clean && !met && sweeps < max_sweeps;
            met = met || done;
            done = clean || (done && !again);
        }
        if (done) {
            status = OZ_CONVERGED;
            break;
        }
        // three sweeps in a row without halving the best off-diagonal mass: the arithmetic's floor
        no_progress = sum > 0.5 * best ? no_progress + 1 : 0;
        best = std::min(best, sum);
        if (no_progress >= 3) {
            status = OZ_STAGNATED;
            break;
        }
    }
    if (fro == 0.0) {
        status = OZ_CONVERGED;
        last = 0.0;
    }
    {
        const int rc = diagonal(&rows, h->S == 0);
        if (rc != OZ_OK) return rc;
    }
    double trace = 0.0;
    for (int c : rows) trace += lam[c];
    if (nev > 0) {
        std::vector<double> ev(nev), scale(nev);
        for (int64_t j = 0; j < nev; ++j) {
            ev[j] = lam[rows[j]];
            scale[j] = 1.0 / std::sqrt(nrm[rows[j]]);
        }
        if ((e = hipMemcpyAsync(h->rows, rows.data(), sizeof(int) * nev, hipMemcpyHostToDevice, s)) != hipSuccess ||
            (e = hipMemcpyAsync(h->scale, scale.data(), sizeof(double) * nev, hipMemcpyHostToDevice, s)) !=
                hipSuccess ||
            (e = hipMemcpyAsync(evals, ev.data(), sizeof(double) * nev, hipMemcpyHostToDevice, s)) != hipSuccess)
            return hip_fail(e, "rdm_eig_solve: output");
        hipLaunchKernelGGL(k_jac_gather, dim3(static_cast<unsigned>(ceil_div(n, 32)), static_cast<unsigned>(ceil_div(nev, 32))),
                           dim3(256), 0, s, st.W, np, h->rows, h->scale, n, nev, Z, ldz);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "rdm_eig_solve: gather");
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "rdm_eig_solve: gather");
    }
    if (info) *info = rdm_eig_info{sweeps, status, last, trace};
    return OZ_OK;
}

int rdm_eig_start_steps(rdm_eig h) {
    if (!h) return fail(OZ_ERR_ARG, "rdm_eig_start_steps: NULL solver");
    return h->start_steps;
}

int rdm_eig_destroy(rdm_eig h) {
    if (!h) return OZ_OK;
    hipSetDevice(h->ctx->device);
    hipDeviceSynchronize();
    rfree(h);
    return OZ_OK;
}

}  // extern "C"

namespace {

// Renormalisation of several operators at once: U is sliced once for the
// whole call (its columns are the right operand's groups of O_k U and the
// left one's of U^T T), and operators go through each step nb at a time, so
// that the D x D products fill the chip (16 operators, n = 2048, D = 512:
// S = 7 1.84 -> 1.36 ms, native 2.09 -> 1.34).  The results are those of the
// two ozaki_dgemm calls per operator.
//
// Workspace: U's slices and exponents and the code scratch, then one slot per
// operator of a batch: O_k's slices (T_k's take their place once T_k is
// there), their exponents and T_k.  One slot more than the per-operator
// workspace holds is what another operator in the batch costs.
struct RenormLayout {
    size_t u_dig, u_e, part, slots, slot, dig, e, T;  // slot: size; dig, e, T: offsets in a slot
};

RenormLayout renorm_layout(int64_t n, int64_t D, int S) {
    const int64_t Np = round_up(n, kRowQ), Dp = round_up(D, kRowQ), Kp = round_up(n, kKB);
    RenormLayout w{};
    size_t off = 0;
    w.u_dig = off; off += align256(static_cast<size_t>(S) * Dp * Kp);
    w.u_e = off; off += align256(sizeof(int32_t) * Dp);
    w.part = off; off += align256(col_exponent_scratch(n, n));
    w.slots = off;
    off = 0;
    w.dig = off; off += align256(static_cast<size_t>(S) * Np * Kp);
    w.e = off; off += align256(sizeof(int32_t) * Np);
    w.T = off; off += align256(sizeof(double) * static_cast<size_t>(n) * D);
    w.slot = off;
    return w;
}

size_t renorm_slot(int64_t n, int64_t D, int S) {
    return S ? renorm_layout(n, D, S).slot : align256(sizeof(double) * static_cast<size_t>(n) * D);
}

// Operators per batch: enough for the D x D products to give each of 256
// compute units two 64 x 64 tiles, and not more than a launch can take.
int renorm_batch(int64_t n, int64_t D, int count, int slices, int ndiag) {
    if (slices && n > max_exact_k(slices, resolve_ndiag(slices, ndiag))) return 1;
    const int64_t tiles = ceil_div(D, 64) * ceil_div(D, 64);
    return static_cast<int>(std::min<int64_t>({ceil_div(512, tiles), kMaxBatch, std::max(count, 1)}));
}

// What ozaki_renormalize_batch_bytes asks for beyond the per-operator
// workspace, at most.  A slot grows with S n^2 while a large n fills the chip
// by itself (16 operators, S = 7; ms with batches of one, of what this allows
// and of all): n = 4096, D = 256 3.59, 2.94, 2.94; n = 8192, D = 64 9.9, 8.2,
// 7.7 (7.1 GB more); D = 512 18.1, 18.0, 18.0.
constexpr size_t kRenormMoreBytes = size_t(2) << 30;

// Whether the call takes the batched form: everything ozaki_dgemm would
// refuse is left to it, and so are inner lengths above the exact int32 range
// (int64 carries) and sizes whose slice passes do not fit one grid.
bool renorm_batched(int64_t n, const double *U, int slices, int ndiag) {
    if (!U || n > INT32_MAX / 2) return false;
    if (slices == 0) return true;
    if (slices < 2 || slices > 8) return false;
    const int G = resolve_ndiag(slices, ndiag);
    if (!valid_sg(slices, G) || n > max_exact_k(slices, G)) return false;
    return 2 * (round_up(n, kRowQ) / kRowQ) * ceil_div(n, kKB) <= (1 << 23);
}

// Whether an output overlaps an input or another output (as when D = n and
// an operator is renormalised in place): the operators then go one by one in
// order.
bool renorm_overlaps(int64_t n, int64_t D, const double *U, int64_t ldu, int count, const double *const *ops, int64_t ldo,
                     double *const *outs, int64_t ldout) {
    typedef std::pair<uintptr_t, uintptr_t> Range;
    auto range = [](const double *p, int64_t rows, int64_t cols, int64_t ld) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p);
        return Range{a, a + sizeof(double) * static_cast<uintptr_t>((rows - 1) * ld + cols)};
    };
    std::vector<Range> o;
    for (int k = 0; k < count; ++k) o.push_back(range(outs[k], D, D, ldout));
    std::sort(o.begin(), o.end());
    for (size_t k = 1; k < o.size(); ++k)
        if (o[k].first < o[k - 1].second) return true;
    auto hit = [&](const Range &r) {
        auto it = std::lower_bound(o.begin(), o.end(), Range{r.second, 0});  // first output that starts past r
        return it != o.begin() && (it - 1)->second > r.first;
    };
    if (hit(range(U, n, D, ldu))) return true;
    for (int k = 0; k < count; ++k)
        if (hit(range(ops[k], n, n, ldo))) return true;
    return false;
}

hipError_t renorm_emulated(ozaki_ctx ctx, int64_t n, int64_t D, const double *U, int64_t ldu, int count,
                           const double *const *ops, int64_t ldo, double *const *outs, int64_t ldout, int S, int G,
                           char *ws, int nb, hipStream_t s) {
    const RenormLayout w = renorm_layout(n, D, S);
    const int64_t Np = round_up(n, kRowQ), Dp = round_up(D, kRowQ), Kp = round_up(n, kKB);
    auto at = [&](int k, size_t off) { return ws + w.slots + static_cast<size_t>(k) * w.slot + off; };
    int8_t *ud = reinterpret_cast<int8_t *>(ws + w.u_dig);
    int32_t *ue = reinterpret_cast<int32_t *>(ws + w.u_e);
    int32_t *codes = reinterpret_cast<int32_t *>(ws + w.part);
    // one phase record per pass over a batch
    hipEvent_t t = mark(ctx, s);
    auto done = [&](int id) {
        const hipEvent_t now = mark(ctx, s);
        phase(ctx, id, t, now);
        t = now;
    };
    // slices of up to two operands per pair of launches
    auto slice = [&](OperandTask a, OperandTask b) {
        return launch_slice_operands(S, a, b, codes, ctx->num_cu, ctx->d_flags, s);
    };
    const OperandTask none{nullptr, 1, 0, n, 0, 0, nullptr, nullptr, 0};
    hipError_t e = slice(OperandTask{U, ldu, D, n, 1, 0, ue, ud, Dp}, none);
    if (e != hipSuccess) return e;
    done(OZ_PHASE_SLICE);
    auto product = [&](int64_t M, const PairArgs &base, int nk) {
        PairArgs a = base;
        const int v = gemm_variant(ctx, S, G, M, D, n, nk);
        const PairShape sh = pair_shape(S, G, v);
        a.tiles_n = static_cast<int32_t>(ceil_div(D, sh.bn));
        a.mode = kModeGemm;
        a.nbatch = nk;
        return launch_pair_single(S, G, v, a, static_cast<int>(ceil_div(M, sh.bm)), s);
    };
    for (int k0 = 0; k0 < count; k0 += nb) {
        const int nk = std::min(nb, count - k0);
        auto o_task = [&](int k) {
            return OperandTask{ops[k0 + k], ldo, n, n, 0, 0, reinterpret_cast<int32_t *>(at(k, w.e)),
                               reinterpret_cast<int8_t *>(at(k, w.dig)), Np};
        };
        auto t_task = [&](int k) {
            return OperandTask{reinterpret_cast<double *>(at(k, w.T)), D, D, n, 1, 0,
                               reinterpret_cast<int32_t *>(at(k, w.e)), reinterpret_cast<int8_t *>(at(k, w.dig)), Dp};
        };
        for (int k = 0; k < nk; k += 2)
            if ((e = slice(o_task(k), k + 1 < nk ? o_task(k + 1) : none)) != hipSuccess) return e;
        done(OZ_PHASE_SLICE);
        // T_k = O_k U
        PairArgs a{};
        int8_t *dig = reinterpret_cast<int8_t *>(at(0, w.dig));
        int32_t *ex = reinterpret_cast<int32_t *>(at(0, w.e));
        a.term = TermDesc{dig, ex, ud, ue, Np, Dp, static_cast<int32_t>(Kp / kKB), 0, 1.0};
        a.out = OutDesc{reinterpret_cast<double *>(at(0, w.T)), D, static_cast<int32_t>(n), static_cast<int32_t>(D)};
        a.batch_A = static_cast<int64_t>(w.slot);
        a.batch_e = static_cast<int64_t>(w.slot / sizeof(int32_t));
        for (int k = 0; k < nk; ++k) a.batch_C[k] = reinterpret_cast<double *>(at(k, w.T));
        if ((e = product(n, a, nk)) != hipSuccess) return e;
        done(OZ_PHASE_PAIR);
        for (int k = 0; k < nk; k += 2)
            if ((e = slice(t_task(k), k + 1 < nk ? t_task(k + 1) : none)) != hipSuccess) return e;
        done(OZ_PHASE_SLICE);
        // O'_k = U^T T_k
        a.term = TermDesc{ud, ue, dig, ex, Dp, Dp, static_cast<int32_t>(Kp / kKB), 0, 1.0};
        a.out = OutDesc{outs[k0], ldout, static_cast<int32_t>(D), static_cast<int32_t>(D)};
        a.batch_B = a.batch_A;
        a.batch_f = a.batch_e;
        a.batch_A = a.batch_e = 0;
        for (int k = 0; k < nk; ++k) a.batch_C[k] = outs[k0 + k];
        if ((e = product(D, a, nk)) != hipSuccess) return e;
        done(OZ_PHASE_PAIR);
    }
    return hipSuccess;
}

hipError_t renorm_native(ozaki_ctx ctx, int64_t n, int64_t D, const double *U, int64_t ldu, int count,
                         const double *const *ops, int64_t ldo, double *const *outs, int64_t ldout, double *T, int nb,
                         hipStream_t s) {
    const size_t stride = renorm_slot(n, D, 0) / sizeof(double);
    hipError_t e;
    for (int k0 = 0; k0 < count; k0 += nb) {
        Dgemm64Args a{};
        a.mode = kModeGemm;
        a.nbatch = std::min(nb, count - k0);
        a.term = Term64{ops[k0], U, ldo, ldu, static_cast<int32_t>(n), 0, 1.0};
        a.out = OutDesc{T, D, static_cast<int32_t>(n), static_cast<int32_t>(D)};
        for (int k = 0; k < a.nbatch; ++k) {
            a.batch_A[k] = ops[k0 + k];
            a.batch_B[k] = U;
            a.batch_C[k] = T + k * stride;
        }
        const hipEvent_t t0 = mark(ctx, s);
        if ((e = launch_dgemm_single(false, false, a, ctx->num_cu, s)) != hipSuccess) return e;
        const hipEvent_t t1 = mark(ctx, s);
        phase(ctx, OZ_PHASE_FP64, t0, t1);
        a.term = Term64{U, T, ldu, D, static_cast<int32_t>(n), 0, 1.0};
        a.out = OutDesc{outs[k0], ldout, static_cast<int32_t>(D), static_cast<int32_t>(D)};
        for (int k = 0; k < a.nbatch; ++k) {
            a.batch_A[k] = U;
            a.batch_B[k] = T + k * stride;
            a.batch_C[k] = outs[k0 + k];
        }
        if ((e = launch_dgemm_single(true, false, a, ctx->num_cu, s)) != hipSuccess) return e;
        phase(ctx, OZ_PHASE_FP64, t1, mark(ctx, s));
    }
    return hipSuccess;
}

}  // namespace

extern "C" {

size_t ozaki_renormalize_workspace_bytes(int64_t n, int64_t D, int slices, int ndiag) {
    if (n < 0 || D < 0) return 0;
    size_t t = align256(sizeof(double) * static_cast<size_t>(n) * D);
    if (slices == 0) return t;
    const size_t w1 = ozaki_dgemm_workspace_bytes(n, D, n, slices, ndiag);
    const size_t w2 = ozaki_dgemm_workspace_bytes(D, D, n, slices, ndiag);
    return t + std::max(w1, w2);
}

size_t ozaki_renormalize_batch_bytes(int64_t n, int64_t D, int count, int slices, int ndiag) {
    const size_t one = ozaki_renormalize_workspace_bytes(n, D, slices, ndiag);
    if (n <= 0 || D <= 0 || count < 1 || slices < 0 || slices == 1 || slices > 8) return one;
    const size_t slot = renorm_slot(n, D, slices);
    const size_t more = std::min<size_t>(renorm_batch(n, D, count, slices, ndiag) - 1, kRenormMoreBytes / slot);
    return one + more * slot;
}

int ozaki_renormalize(ozaki_ctx ctx, int64_t n, int64_t D, const double *U, int64_t ldu, int count,
                      const double *const *ops, int64_t ldo, double *const *outs, int64_t ldout, int slices,
                      int ndiag, void *workspace, size_t workspace_bytes, void *stream) {
    if (!ctx) return fail(OZ_ERR_ARG, "ozaki_renormalize: ctx is NULL");
    if (n < 0 || D < 0 || D > n || count < 0) return fail(OZ_ERR_ARG, "ozaki_renormalize: sizes");
    if (count > 0 && (!ops || !outs)) return fail(OZ_ERR_ARG, "ozaki_renormalize: ops / outs is NULL");
    if (ldu < (D > 1 ? D : 1) || ldo < (n > 1 ? n : 1) || ldout < (D > 1 ? D : 1))
        return fail(OZ_ERR_ARG, "ozaki_renormalize: leading dimension");
    if (n == 0 || D == 0 || count == 0) return OZ_OK;
    const size_t need = ozaki_renormalize_workspace_bytes(n, D, slices, ndiag);
    if (!workspace || workspace_bytes < need)
        return fail(OZ_ERR_WORKSPACE, "ozaki_renormalize: workspace %zu bytes, need %zu", workspace_bytes, need);
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return fail(OZ_ERR_WORKSPACE, "ozaki_renormalize: workspace not 256-byte aligned");
    for (int k = 0; k < count; ++k)
        if (!ops[k] || !outs[k]) return fail(OZ_ERR_ARG, "ozaki_renormalize: operator %d is NULL", k);
    if (renorm_batched(n, U, slices, ndiag) && !renorm_overlaps(n, D, U, ldu, count, ops, ldo, outs, ldout)) {
        const int most = renorm_batch(n, D, count, slices, ndiag);
        const size_t more = (workspace_bytes - need) / renorm_slot(n, D, slices);
        const int nb = more < static_cast<size_t>(most - 1) ? static_cast<int>(more) + 1 : most;
        hipStream_t s = static_cast<hipStream_t>(stream);
        hipError_t e;
        if ((e = hipSetDevice(ctx->device)) != hipSuccess) return hip_fail(e, "hipSetDevice");
        e = slices ? renorm_emulated(ctx, n, D, U, ldu, count, ops, ldo, outs, ldout, slices,
                                     resolve_ndiag(slices, ndiag), static_cast<char *>(workspace), nb, s)
                   : renorm_native(ctx, n, D, U, ldu, count, ops, ldo, outs, ldout, static_cast<double *>(workspace), nb, s);
        return e == hipSuccess ? OZ_OK : hip_fail(e, "ozaki_renormalize");
    }
    double *T = static_cast<double *>(workspace);
    const size_t tb = align256(sizeof(double) * static_cast<size_t>(n) * D);
    void *gw = slices ? static_cast<char *>(workspace) + tb : nullptr;
    const size_t gwb = slices ? workspace_bytes - tb : 0;
    for (int k = 0; k < count; ++k) {
        // T = O_k U (n x D), then O'_k = U^T T (D x D)
        int rc = ozaki_dgemm(ctx, 'N', 'N', n, D, n, 1.0, ops[k], ldo, U, ldu, 0.0, T, D, slices, ndiag, gw, gwb,
                             stream);
        if (rc != OZ_OK) return rc;
        rc = ozaki_dgemm(ctx, 'T', 'N', D, D, n, 1.0, U, ldu, T, D, 0.0, outs[k], ldout, slices, ndiag, gw, gwb,
                         stream);
        if (rc != OZ_OK) return rc;
    }
    return OZ_OK;
}

}  // extern "C"
