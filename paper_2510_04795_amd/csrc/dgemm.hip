// Native FP64 GEMM on the FP64 matrix cores (v_mfma_f64_16x16x4_f64): the
// comparator for the emulated path and the slices = 0 mode of every entry
// point.  Any summation order is a valid FP64 GEMM, so this path is checked
// against the textbook gamma_K |A||B| bound, not bit for bit.
//
// Operand layout of the 16x16x4 instruction (measured): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator register r of lane l
// holds C[4 r + l / 16][l % 16].
//
// Tile: 256 threads = 2 x 2 waves of BM/2 x BM/2 outputs in blocks of 16 x 16;
// BM = 128 (each wave 4 x 4 blocks, 64 FP64 accumulators per lane) or 64, as
// dgemm_tile_for says.  K advances 16 at a time through two LDS stages filled
// by direct global->LDS 16-byte loads (two doubles per lane, no staging
// registers, one barrier a step), and the matrix cores run from fragments in
// registers: at BM = 64 those of the next step are read behind the products
// of this one (two sets, four workgroups per compute unit), at 128 after the
// step's barrier (one set, two workgroups).  Bound: the matrix cores, 16
// products of 64 cycles per wave and step at BM = 64 (8192^3: 72 TFLOP/s
// against 64 with staging registers and strided 32-byte loads; 2048^3, B
// transposed: 258 us against 288; the FP64 block-sparse H_eff of 40 sectors
// 3.5 ms against 4.7).  Products of few tiles take k_dgemm_split below.
//
// Order of k.  Both operands hand lane (l16, lq) the elements k = 8 g + 2 lq
// + s in the s-th product of group g, so an operand stored along K is read
// two elements (16 bytes) at a time.
//
// LDS layout (OperandMap), in 16-byte chunks (where a chunk lands is the loading lane's
// place, what it holds is the lane's choice of address):
//   stored along K (op(A) = A, op(B) = B^T): eight chunks per row, the pair of
//     k at place pair ^ ((row / 2) % 8), so the 16 rows a read takes fall in
//     16 different places modulo 256 bytes;
//   stored across K (op(A) = A^T, op(B) = B): BM / 2 chunks per k, the pair of
//     rows at place pair ^ 8 ((k / 2) % 2), so the two k a half wave reads
//     fall in different halves of the banks.
// A workgroup of eight lanes (along) or of BM / 2 lanes (across) loads whole
// 128-byte lines.  Rows past the operand are clamped to its last row (they
// only feed outputs that are never stored); a last step that K does not fill,
// or whose last pair would run past the end of the stored matrix, goes
// through registers element by element.
#include <type_traits>

#include "dgemm_operand.h"
#include "internal.h"

namespace oz {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(1))) const void global_void;
typedef __attribute__((address_space(3))) void lds_void;
constexpr int kBufferDword3 = 0x00020000;  // raw buffer, 32-bit data format

// One operand of a tile: `rows` rows (or columns) from r0, inner length K.
// ALONG: element (i, k) at X[i * ld + k]; else at X[k * ld + i].  FAR: 64-bit
// addresses, for leading dimensions whose steps do not fit 32-bit offsets (the
// single launch picks it; the grouped one, whose blocks never get there, falls
// back to element copies).
template <int BM, bool ALONG, bool FAR = false>
struct Operand {
    using Map = OperandMap<BM, ALONG>;
    static constexpr int CH = Map::CHUNKS / 256;  // 16-byte chunks per thread and step
    const double *X;
    int64_t ld;
    int rows, K, r0;
    int voff[FAR ? 1 : CH];  // byte offset of the thread's chunks from the step's base
    int nfast;               // steps that take the direct loads

    __device__ __forceinline__ void place(int i, int &row, int &k) const { Map::place(i * 256 + threadIdx.x, row, k); }

    __device__ __forceinline__ void init(const double *x, int64_t l, int n, int kk, int first) {
        X = x;
        ld = l;
        rows = n;
        K = kk;
        r0 = first;
        nfast = FAR || Map::near(ld) ? Map::direct_steps(rows, K) : 0;
        if (FAR) return;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            int row, k;
            place(i, row, k);
            voff[i] = Map::byte_offset(row, k, rows, ld, r0);
        }
    }

    __device__ __forceinline__ void issue(double *stage, int step) const {
        const double *base = X + Map::base(ld, r0, step);
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if constexpr (FAR) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                int row, k;
                place(i, row, k);
                __builtin_amdgcn_global_load_lds((global_void *)(base + Map::offset(row, k, rows, ld, r0)),
                                                 (lds_void *)(stage + (i * 256 + wave * 64) * 2), 16, 0, 0);
            }
        } else {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(base), 0, 0x7fffffff, kBufferDword3);
#pragma unroll
            for (int i = 0; i < CH; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(stage + (i * 256 + wave * 64) * 2), 16,
                                                         voff[i], 0, 0, 0);
        }
    }

    // The same step element by element, zero past K and past the rows.
    __device__ __forceinline__ void copy(double *stage, int step) const {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            int row, k;
            place(i, row, k);
            k += step * kBK;
            row += r0;
            double2 v{0.0, 0.0};
            if (ALONG) {
                const double *p = X + static_cast<int64_t>(row) * ld + k;
                if (row < rows && k < K) v.x = p[0];
                if (row < rows && k + 1 < K) v.y = p[1];
            } else {
                const double *p = X + static_cast<int64_t>(k) * ld + row;
                if (k < K && row < rows) v.x = p[0];
                if (k < K && row + 1 < rows) v.y = p[1];
            }
            *reinterpret_cast<double2 *>(stage + (i * 256 + threadIdx.x) * 2) = v;
        }
    }
};

// This wave's fragments of one stage: [group of eight k][block], elements s = 0, 1.
template <int E, bool ALONG>
__device__ __forceinline__ void read_frags(double2 (&f)[2][E / 32], const double *stage, int wbase) {
    constexpr int NB = E / 32, PR = kBK / 2;
    const int lane = threadIdx.x & 63, lq = lane >> 4, l16 = lane & 15;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (ALONG) {
                const int row = wbase + b * 16 + l16;
                f[g][b] = *reinterpret_cast<const double2 *>(
                    stage + (row * PR + ((4 * g + lq) ^ ((l16 >> 1) & 7))) * 2);
            } else {
                const int pair = wbase / 2 + 8 * (b ^ (lq & 1)) + (l16 >> 1);
                const double *p = stage + ((8 * g + 2 * lq) * (E / 2) + pair) * 2 + (l16 & 1);
                f[g][b].x = p[0];
                f[g][b].y = p[E];
            }
        }
}

template <int BM, int BN, bool TA, bool TB, int MODE, bool FAR = false, typename GetTerm>
__device__ __forceinline__ void dgemm_tile(const Dgemm64Args &a, GetTerm get_term, int tb, int te,
                                           const OutDesc &out, int m0, int n0, double *lds) {
    constexpr int MB = BM / 32, NB = BN / 32, OPA = BM * kBK, STAGE = OPA + BN * kBK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1;
    const int wn = wave & 1;
    const int lq = lane >> 4;   // 0..3
    const int l16 = lane & 15;

    // Accumulating mode: the tile's output elements hold the running sum,
    // sigma = fma(alpha_t, c_t, sigma) after every term in list order (the
    // block owns its tile, each thread re-reads only what it wrote), so the
    // FP64 rounding is that of separately summed terms without keeping a
    // second register tile.  The sum starts from +0, or from the stored value
    // when the output continues a term list split over launches (out.cont).
    const int tend = (MODE == kModeAccum) ? te : tb + 1;
    if (MODE == kModeAccum && tb == te) {
        if (out.cont) return;  // nothing to add to the stored sum
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = m0 + wm * (BM / 2) + mb * 16 + 4 * r + lq;
                    const int j = n0 + wn * (BN / 2) + nb * 16 + l16;
                    if (i < out.M && j < out.N) out.C[static_cast<int64_t>(i) * out.ldc + j] = 0.0;
                }
        return;
    }
    for (int ti = tb; ti < tend; ++ti) {
        const Term64 T = get_term(ti);
        v4d acc[MB][NB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = v4d{0.0, 0.0, 0.0, 0.0};
        const int nk = (T.K + kBK - 1) / kBK;
        Operand<BM, !TA, FAR> oa;
        Operand<BN, TB, FAR> ob;
        oa.init(T.A, T.lda, out.M, T.K, m0);
        ob.init(T.B, T.ldb, out.N, T.K, n0);
        auto load = [&](int step) {
            double *stage = lds + (step & 1) * STAGE;
            if (step < oa.nfast) oa.issue(stage, step);
            else oa.copy(stage, step);
            if (step < ob.nfast) ob.issue(stage + OPA, step);
            else ob.copy(stage + OPA, step);
        };
        // PRE: two sets of fragments, read a step ahead of their products; the
        // 128 x 128 tile has registers for one, read after its step's barrier.
        constexpr bool PRE = MB * NB <= 4;
        double2 fa[PRE ? 2 : 1][2][MB], fb[PRE ? 2 : 1][2][NB];
        auto read = [&](auto F, int step) {
            constexpr int f = decltype(F)::value;
            const double *stage = lds + (step & 1) * STAGE;
            read_frags<BM, !TA>(fa[f], stage, wm * (BM / 2));
            read_frags<BN, TB>(fb[f], stage + OPA, wn * (BN / 2));
        };
        // Step ks with its fragments in set F.  PRE: once step ks + 1 has landed
        // in every wave, its fragments go to the other set and the loads of step
        // ks + 2 start into the stage step ks came from (in registers since the
        // step before); else once step ks has landed, its own fragments are
        // read and the loads of step ks + 1 start.  Both run behind the products.
        auto step = [&](auto F, int ks) {
            constexpr int f = decltype(F)::value;
            if (!PRE || ks + 1 < nk) {
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                if constexpr (PRE) read(std::integral_constant<int, 1 - f>{}, ks + 1);
                else read(F, ks);
                if (ks + (PRE ? 2 : 1) < nk) load(ks + (PRE ? 2 : 1));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                s ? fa[f][g][mb].y : fa[f][g][mb].x, s ? fb[f][g][nb].y : fb[f][g][nb].x, acc[mb][nb],
                                0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        if (nk > 0) {
            __syncthreads();  // the previous term / tile may still read LDS
            load(0);
            if constexpr (PRE) {
                if (nk > 1) load(1);
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                read(std::integral_constant<int, 0>{}, 0);
            }
        }
        constexpr std::integral_constant<int, 0> set0{};
        constexpr std::integral_constant<int, PRE ? 1 : 0> set1{};
        int ks = 0;
        for (; ks + 2 <= nk; ks += 2) {
            step(set0, ks);
            step(set1, ks + 1);
        }
        if (ks < nk) step(set0, ks);
        // the output base is opaque to the optimiser here, so the 16 NB^2
        // element addresses are formed per term instead of being hoisted out
        // of the term loop (where they would not fit in registers)
        double *cbase = out.C;
        asm volatile("" : "+s"(cbase));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // one element's read-modify-write at a time in registers
                    __builtin_amdgcn_sched_barrier(0);
                    const int i = m0 + wm * (BM / 2) + mb * 16 + 4 * r + lq;
                    const int j = n0 + wn * (BN / 2) + nb * 16 + l16;
                    if (i >= out.M || j >= out.N) continue;
                    const double c = acc[mb][nb][r];
                    double *p = cbase + static_cast<int64_t>(i) * out.ldc + j;
                    if (MODE == kModeGemm)
                        *p = (a.beta == 0.0) ? T.alpha * c : fma(T.alpha, c, a.beta * *p);
                    else
                        *p = fma(T.alpha, c, (ti == tb && !out.cont) ? 0.0 : *p);
                }
    }
}

// XCD-aware tile order (blocks are dispatched to the 8 XCDs round robin).
__device__ __forceinline__ void tile_order(int b, int tiles_m, int tiles_n, int nbatch, int &k, int &tm, int &tn) {
    const int T = tiles_m * tiles_n, all = nbatch > 1 ? T * nbatch : T;
    const int q = all / 8, rem = all - q * 8;
    const int x = b % 8, idx = b / 8;
    const int at = x * q + (x < rem ? x : rem) + idx;
    k = nbatch > 1 ? at / T : 0;
    const int lin = at - k * T;
    const int per_group = 4 * tiles_n;
    const int gid = lin / per_group;
    const int first = gid * 4;
    const int rows = tiles_m - first < 4 ? tiles_m - first : 4;
    const int w = lin - gid * per_group;
    tm = first + w % rows;
    tn = w / rows;
}

// Product k of a batched single launch.
__device__ __forceinline__ void batch_product(const Dgemm64Args &a, int k, Term64 &term, OutDesc &out) {
    term = a.term;
    out = a.out;
    if (a.nbatch > 1) {
        term.A = a.batch_A[k];
        term.B = a.batch_B[k];
        out.C = a.batch_C[k];
    }
}

// Workgroups per compute unit the registers are kept for: four of the 64 x 64
// tiles (128 registers a wave; with three, a product of exactly four tiles per
// compute unit runs them in two rounds: 2048^3 in 358 us instead of 250), two
// of the 128 x 128 and of the accumulating mode, whose term loop keeps more
// live (with 128 registers it spills: a small block-sparse H_eff 208 us
// against 175).
constexpr int tile_waves(int bm) { return bm == 64 ? 4 : 2; }

template <int BM, int BN, bool TA, bool TB, bool FAR>
__global__ __launch_bounds__(256, tile_waves(BM)) void k_dgemm_single(Dgemm64Args a, int tiles_m) {
    __shared__ __align__(16) double lds[2 * (BM + BN) * kBK];
    int k, tm, tn;
    tile_order(blockIdx.x, tiles_m, a.tiles_n, a.nbatch, k, tm, tn);
    Term64 term;
    OutDesc out;
    batch_product(a, k, term, out);
    dgemm_tile<BM, BN, TA, TB, kModeGemm, FAR>(a, [&](int) { return term; }, 0, 1, out, tm * BM, tn * BN, lds);
}

template <int BM, bool TB, int MODE>
__global__ __launch_bounds__(256, MODE == kModeAccum ? 2 : tile_waves(BM)) void k_dgemm_grouped(Dgemm64Args a) {
    __shared__ __align__(16) double lds[2 * 2 * BM * kBK];
    const TileDesc td = a.tiles[blockIdx.x];
    if (td.out < 0) return;  // padding of the XCD order
    OutDesc od = a.outs[td.out];
    if (a.out_base) od.C = a.out_base + reinterpret_cast<intptr_t>(od.C);
    const Term64 *terms = a.terms;
    const double *b_base = a.b_base;
    dgemm_tile<BM, BM, false, TB, MODE>(a,
                                            [&](int i) {
                                                Term64 tm = terms[i];
                                                if (b_base) tm.B = b_base + reinterpret_cast<intptr_t>(tm.B);
                                                return tm;
                                            },
                                            td.term_begin, td.term_end, od, td.m0, td.n0, lds);
}

// ---- split kernel for products of few tiles --------------------------------
// One 32 x 32 output block per workgroup; the four waves take every fourth
// group of eight k each and add their sums through LDS at the end, so a
// product with few tiles still gives every SIMD work and a wave's chain is a
// quarter as long.  Fragments come straight from memory into registers
// (along K: 16 bytes per lane, the four waves' groups side by side; across K:
// 16 consecutive elements of four rows), kDepth groups ahead of the matrix
// cores (512^3: 14.3 us with four groups ahead, 11.0 with eight).  Bound:
// latency; measured against the tiles in split_pays.
constexpr int kDepth = 8;

template <bool ALONG>
struct SplitOperand {
    const double *p[2];  // this lane's element of k = 2 lq in each block of 16 rows / columns
    int64_t ld;
    __device__ __forceinline__ void init(const double *X, int64_t l, int rows, int r0) {
        const int lane = threadIdx.x & 63, lq = lane >> 4, l16 = lane & 15;
        ld = l;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int r = r0 + 16 * b + l16;
            const int64_t rc = r < rows ? r : rows - 1;
            p[b] = ALONG ? X + rc * ld + 2 * lq : X + 2 * lq * ld + rc;
        }
    }
    // elements s = 0, 1 of whole group g
    __device__ __forceinline__ void load(double2 (&v)[2], int g) const {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (ALONG) {
                __builtin_memcpy(&v[b], p[b] + 8 * g, sizeof(double2));
            } else {
                const double *q = p[b] + static_cast<int64_t>(8 * g) * ld;
                v[b].x = q[0];
                v[b].y = q[ld];
            }
        }
    }
    // the last group, of which `left` elements exist
    __device__ __forceinline__ void load_tail(double2 (&v)[2], int g, int left) const {
        const int k = 2 * ((threadIdx.x & 63) >> 4);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const double *q = p[b] + (ALONG ? 8 * g : static_cast<int64_t>(8 * g) * ld);
            v[b].x = k < left ? q[0] : 0.0;
            v[b].y = k + 1 < left ? q[ALONG ? 1 : ld] : 0.0;
        }
    }
};

template <bool TA, bool TB>
__global__ __launch_bounds__(256) void k_dgemm_split(Dgemm64Args a, int tiles_m) {
    __shared__ double red[4][3][4][64];  // [block][other wave][register][lane]
    int k, tm, tn;
    tile_order(blockIdx.x, tiles_m, a.tiles_n, a.nbatch, k, tm, tn);
    Term64 T;
    OutDesc out;
    batch_product(a, k, T, out);
    const int m0 = tm * 32, n0 = tn * 32;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, lq = lane >> 4, l16 = lane & 15;
    v4d acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    SplitOperand<!TA> oa;
    SplitOperand<TB> ob;
    oa.init(T.A, T.lda, out.M, m0);
    ob.init(T.B, T.ldb, out.N, n0);
    double2 fa[kDepth][2], fb[kDepth][2];
    // groups of this wave: wave, wave + 4, ... below `full`; the rest of K
    // (fewer than eight) is the next wave's in turn
    const int full = T.K / 8;
    const int n = (full - wave + 3) / 4;
    auto load = [&](int d, int i) {
        oa.load(fa[d], wave + 4 * i);
        ob.load(fb[d], wave + 4 * i);
    };
    auto mul = [&](int d) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(s ? fa[d][i].y : fa[d][i].x,
                                                                     s ? fb[d][j].y : fb[d][j].x, acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < kDepth; ++d)
        if (d < n) load(d, d);
    int at = 0;
    // no branches while every slot has a successor, so the waits stay exact
    for (; at + 2 * kDepth <= n; at += kDepth) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            mul(d);
            load(d, at + kDepth + d);
        }
    }
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
        if (at + d >= n) break;
        mul(d);
        if (at + kDepth + d < n) load(d, at + kDepth + d);
    }
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
        if (at + kDepth + d >= n) break;
        mul(d);
    }
    if (T.K % 8 && full % 4 == wave) {
        oa.load_tail(fa[0], full, T.K % 8);
        ob.load_tail(fb[0], full, T.K % 8);
        mul(0);
    }
    // block b is finished by wave b: the sums of waves 0..3 in that order
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (wave == b) continue;
        const int slot = wave < b ? wave : wave - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) red[b][slot][r][lane] = acc[b >> 1][b & 1][r];
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (wave != b) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = m0 + (b >> 1) * 16 + 4 * r + lq, j = n0 + (b & 1) * 16 + l16;
            if (i >= out.M || j >= out.N) continue;
            const double own = acc[b >> 1][b & 1][r];
            double c = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const double x = w == b ? own : red[b][w < b ? w : w - 1][r][lane];
                c = w ? c + x : x;
            }
            double *p = out.C + static_cast<int64_t>(i) * out.ldc + j;
            *p = (a.beta == 0.0) ? T.alpha * c : fma(T.alpha, c, a.beta * *p);
        }
    }
}

void launch_split(bool ta, bool tb, Dgemm64Args a, hipStream_t s) {
    const int tiles_m = static_cast<int>(ceil_div(a.out.M, 32));
    a.tiles_n = static_cast<int32_t>(ceil_div(a.out.N, 32));
    const unsigned grid = static_cast<unsigned>(tiles_m) * static_cast<unsigned>(a.tiles_n) * (a.nbatch > 1 ? a.nbatch : 1);
    if (!ta && !tb) hipLaunchKernelGGL((k_dgemm_split<false, false>), dim3(grid), dim3(256), 0, s, a, tiles_m);
    if (!ta && tb) hipLaunchKernelGGL((k_dgemm_split<false, true>), dim3(grid), dim3(256), 0, s, a, tiles_m);
    if (ta && !tb) hipLaunchKernelGGL((k_dgemm_split<true, false>), dim3(grid), dim3(256), 0, s, a, tiles_m);
    if (ta && tb) hipLaunchKernelGGL((k_dgemm_split<true, true>), dim3(grid), dim3(256), 0, s, a, tiles_m);
}

template <int BM, int BN, bool FAR>
void launch_single_tile(bool ta, bool tb, Dgemm64Args a, hipStream_t s) {
    const int tiles_m = static_cast<int>(ceil_div(a.out.M, BM));
    a.tiles_n = static_cast<int32_t>(ceil_div(a.out.N, BN));
    const unsigned grid = static_cast<unsigned>(tiles_m) * static_cast<unsigned>(a.tiles_n) * (a.nbatch > 1 ? a.nbatch : 1);
    if (!ta && !tb) hipLaunchKernelGGL((k_dgemm_single<BM, BN, false, false, FAR>), dim3(grid), dim3(256), 0, s, a, tiles_m);
    if (!ta && tb) hipLaunchKernelGGL((k_dgemm_single<BM, BN, false, true, FAR>), dim3(grid), dim3(256), 0, s, a, tiles_m);
    if (ta && !tb) hipLaunchKernelGGL((k_dgemm_single<BM, BN, true, false, FAR>), dim3(grid), dim3(256), 0, s, a, tiles_m);
    if (ta && tb) hipLaunchKernelGGL((k_dgemm_single<BM, BN, true, true, FAR>), dim3(grid), dim3(256), 0, s, a, tiles_m);
}

// 64-bit addresses where a step of either operand does not fit 32-bit offsets
// (a leading dimension from 2^24 elements across K, from 2^22 along it with 64
// rows).  1024 x 1024 x 512, both operands past that, 64-bit against element
// copies: NT 28 us / 54, NN 42 / 55, TT 34 / 58, TN 43 / 61 (26 within the
// 32-bit offsets).
template <int E>
void launch_tile_edge(bool ta, bool tb, const Dgemm64Args &a, hipStream_t s) {
    auto near = [](bool along, int64_t ld) { return along ? OperandMap<E, true>::near(ld) : OperandMap<E, false>::near(ld); };
    if (near(!ta, a.term.lda) && near(tb, a.term.ldb))
        launch_single_tile<E, E, false>(ta, tb, a, s);
    else
        launch_single_tile<E, E, true>(ta, tb, a, s);
}

}  // namespace

// 128 where its tiles still go round every compute unit four times (two at
// once, so a last round that is half empty costs little) and leave no more
// than a twentieth of their area outside the outputs; 64 otherwise.
// Measured: 8192^3 15.2 ms against 16.3, 4096^3 1.92 against 1.96, but 3000^3
// (576 tiles of 128) 1.19 against 0.86, 2048^3 (256) 0.27 against 0.25, and a
// block-sparse H_eff of 40 sectors, where 128 tiles hang over the blocks'
// edges, 4.5 ms against 3.5.
int dgemm_tile_for(int64_t tiles64, int64_t tiles128, int num_cu) {
    return tiles128 >= 4 * static_cast<int64_t>(num_cu) && 80 * tiles128 <= 21 * tiles64 ? 128 : 64;
}

// The split kernel: up to two 32 x 32 blocks per compute unit.  Measured (us,
// against 64 x 64 tiles): 512^3 11.0 / 22.9, 640^3 (100 tiles of 64) 20.6 /
// 28.1, 512 x 512 x 2048 28 / 83, 128 x 128 x 8192 116 / 309; equal at 768^3
// (144 tiles, 33), and 52 / 43 at 1024^3.
static bool split_pays(int64_t tiles64, int num_cu) { return 2 * tiles64 <= num_cu; }

hipError_t launch_dgemm_single(bool ta, bool tb, const Dgemm64Args &a, int num_cu, hipStream_t s) {
    if (a.out.M <= 0 || a.out.N <= 0) return hipSuccess;
    const int64_t nb = a.nbatch > 1 ? a.nbatch : 1;
    const int64_t tiles64 = ceil_div(a.out.M, 64) * ceil_div(a.out.N, 64) * nb;
    if (split_pays(tiles64, num_cu))
        launch_split(ta, tb, a, s);
    else if (dgemm_tile_for(tiles64, ceil_div(a.out.M, 128) * ceil_div(a.out.N, 128) * nb, num_cu) == 64)
        launch_tile_edge<64>(ta, tb, a, s);
    else
        launch_tile_edge<128>(ta, tb, a, s);
    return hipGetLastError();
}

template <int BM>
void launch_grouped_bm(bool tb, const Dgemm64Args &a, hipStream_t s) {
    const bool acc = a.mode == kModeAccum;
    if (tb && acc) hipLaunchKernelGGL((k_dgemm_grouped<BM, true, kModeAccum>), dim3(a.ntiles), dim3(256), 0, s, a);
    if (tb && !acc) hipLaunchKernelGGL((k_dgemm_grouped<BM, true, kModeGemm>), dim3(a.ntiles), dim3(256), 0, s, a);
    if (!tb && acc) hipLaunchKernelGGL((k_dgemm_grouped<BM, false, kModeAccum>), dim3(a.ntiles), dim3(256), 0, s, a);
    if (!tb && !acc) hipLaunchKernelGGL((k_dgemm_grouped<BM, false, kModeGemm>), dim3(a.ntiles), dim3(256), 0, s, a);
}

hipError_t launch_dgemm_grouped(bool tb, const Dgemm64Args &a, hipStream_t s) {
    if (a.ntiles == 0) return hipSuccess;
    if (a.tile == 64)
        launch_grouped_bm<64>(tb, a, s);
    else if (a.tile == 128)
        launch_grouped_bm<128>(tb, a, s);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace oz
