// Dispatch of the pair-GEMM kernels over the slice count and tile variant.
#include "pairgemm_impl.h"

namespace oz {

bool pair_supported(int S, int G) {
    if (S < 2 || S > 8) return false;
    return G == S || G == S + 1 || G == 2 * S - 1;
}

int pair_num_variants() { return pair::kNumVariants; }

bool pair_variant_ok(int G, int v) { return v >= 0 && v < pair::kNumVariants && pair::variant_fits(G, v); }

int pair_default_variant(int G) { return pair::default_variant(G); }

// Each 32 x 32 block on a compute unit of its own, and more K blocks than
// two.  Measured (us, split against 64 x 64 tiles, S = 6 / S = 7 with G = 8):
// 512 x 512 x 2048 (64 tiles of 64) 36 / 43 against 49 / 63, 128 x 128 x 8192
// 72 / 87 against 134 / 186; but 640^3 (100 tiles) 29 / 38 against 29 / 34 and
// 1024^3 (256 tiles) 52 / 75 against 41 / 49, where the larger tile's reuse of
// its operands counts for more.
bool pair_split_pays(int64_t M, int64_t N, int64_t K, int nbatch, int num_cu) {
    return ceil_div(M, 64) * ceil_div(N, 64) * nbatch * 4 <= num_cu && K > 64;
}

// Up to two blocks per compute unit.  Whole H_eff matvecs measured (us, split
// against the better of one workgroup per 64 x 64 tile and paired terms, both
// S = 6): D = 96, 8 terms (9 blocks) 40 against 61; D = 256, 24 terms (64) 103
// against 194; D = 512, 24 terms (256) 194 against 322, 2 terms 77 against 80;
// D = 640, 24 terms (400) 384 against 437; but D = 736, 24 terms (529) 613
// against 564, where the third block of a compute unit and the 64 x 64 tiles'
// reuse of their operands count for more.
bool pair_accum_split_pays(int64_t blocks, int num_cu) { return blocks <= 2 * num_cu; }

PairShape pair_shape(int S, int G, int v) {
    (void)S;
    if (v == kSplitVariant) return PairShape{32, 32};
    if (v < 0) v = pair::default_variant(G);
    return PairShape{pair::variant_bm(v), pair::variant_bn(v)};
}

hipError_t launch_pair_single(int S, int G, int v, const PairArgs &a, int tiles_m, hipStream_t s) {
    if (v < 0) v = pair::default_variant(G);
    switch (S) {
        case 2: return pair_single_s2(G, v, a, tiles_m, s);
        case 3: return pair_single_s3(G, v, a, tiles_m, s);
        case 4: return pair_single_s4(G, v, a, tiles_m, s);
        case 5: return pair_single_s5(G, v, a, tiles_m, s);
        case 6: return pair_single_s6(G, v, a, tiles_m, s);
        case 7: return pair_single_s7(G, v, a, tiles_m, s);
        case 8: return pair_single_s8(G, v, a, tiles_m, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pair_grouped(int S, int G, int v, const PairArgs &a, hipStream_t s) {
    if (v < 0) v = pair::default_variant(G);
    switch (S) {
        case 2: return pair_grouped_s2(G, v, a, s);
        case 3: return pair_grouped_s3(G, v, a, s);
        case 4: return pair_grouped_s4(G, v, a, s);
        case 5: return pair_grouped_s5(G, v, a, s);
        case 6: return pair_grouped_s6(G, v, a, s);
        case 7: return pair_grouped_s7(G, v, a, s);
        case 8: return pair_grouped_s8(G, v, a, s);
        default: return hipErrorInvalidValue;
    }
}

int pair_resident_per_cu(int S, int G, int v) {
    if (v < 0) v = pair::default_variant(G);
    switch (S) {
        case 2: return pair_resident_s2(G, v);
        case 3: return pair_resident_s3(G, v);
        case 4: return pair_resident_s4(G, v);
        case 5: return pair_resident_s5(G, v);
        case 6: return pair_resident_s6(G, v);
        case 7: return pair_resident_s7(G, v);
        case 8: return pair_resident_s8(G, v);
        default: return 0;
    }
}

bool pair_terms2_ok(int S, int G, int v) {
    if (v != 0 || !pair_supported(S, G)) return false;
    switch (S) {
        case 2: return pair_terms2_s2(G);
        case 3: return pair_terms2_s3(G);
        case 4: return pair_terms2_s4(G);
        case 5: return pair_terms2_s5(G);
        case 6: return pair_terms2_s6(G);
        case 7: return pair_terms2_s7(G);
        case 8: return pair_terms2_s8(G);
        default: return false;
    }
}

}  // namespace oz
