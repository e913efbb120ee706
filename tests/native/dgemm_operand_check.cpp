// Address ranges of the FP64 GEMM tiles' direct loads (dgemm_operand.h), over
// rows, inner lengths, tile edges and leading dimensions: every 16-byte load
// lies inside the stored matrix, chunks cover the stage once and hold the
// elements they stand for, and near() leaves room for 31-bit byte offsets.
#include <cstdio>
#include <vector>

#include "dgemm_operand.h"

static long checked = 0;

static int bad(const char *what, int E, bool along, int n, int K, int64_t ld, int r0, int step, int c) {
    std::printf("%s: E %d along %d n %d K %d ld %lld r0 %d step %d chunk %d\n", what, E, along, n, K,
                static_cast<long long>(ld), r0, step, c);
    return 1;
}

template <int E, bool ALONG>
int check(int n, int K, int odd) {
    using Map = oz::OperandMap<E, ALONG>;
    const int64_t cols = ALONG ? K : n, stored = ALONG ? n : K, ld = cols + odd;
    const int64_t end = (stored - 1) * ld + cols;  // elements of the stored matrix
    for (int r0 = 0; r0 < n; r0 += E)
        for (int step = 0; step < Map::direct_steps(n, K); ++step) {
            std::vector<int> seen(E * oz::kBK, 0);
            for (int c = 0; c < Map::CHUNKS; ++c) {
                int row, k;
                Map::place(c, row, k);
                if (row < 0 || row >= E || k < 0 || k >= oz::kBK) return bad("place", E, ALONG, n, K, ld, r0, step, c);
                ++seen[row * oz::kBK + k];
                ++seen[(ALONG ? row : row + 1) * oz::kBK + (ALONG ? k + 1 : k)];
                const int64_t rel = Map::offset(row, k, n, ld, r0), at = Map::base(ld, r0, step) + rel;
                if (at < 0 || at + 1 >= end) return bad("range", E, ALONG, n, K, ld, r0, step, c);
                if (Map::byte_offset(row, k, n, ld, r0) != rel * 8) return bad("bytes", E, ALONG, n, K, ld, r0, step, c);
                const int i = r0 + row, kk = step * oz::kBK + k;
                // a row inside the operand is where it belongs (the odd last one across K: its own pair)
                if (i < n && at != (ALONG ? i * ld + kk : kk * ld + i)) return bad("element", E, ALONG, n, K, ld, r0, step, c);
                if (kk + (ALONG ? 1 : 0) >= K) return bad("past K", E, ALONG, n, K, ld, r0, step, c);
                ++checked;
            }
            for (int x : seen)
                if (x != 1) return bad("cover", E, ALONG, n, K, ld, r0, step, -1);
        }
    return 0;
}

template <int E, bool ALONG>
int limits() {
    using Map = oz::OperandMap<E, ALONG>;
    int64_t ld = 1;
    while (Map::near(2 * ld)) ld *= 2;
    for (int64_t d = ld; d > 0; d /= 2)
        while (Map::near(ld + d)) ld += d;
    for (int c = 0; c < Map::CHUNKS; ++c) {
        int row, k;
        Map::place(c, row, k);
        const int64_t b = Map::offset(row, k, 1 << 20, ld, 0) * 8;
        if (b < 0 || b + 16 > 0x7fffffff || Map::byte_offset(row, k, 1 << 20, ld, 0) != b)
            return bad("near", E, ALONG, 1 << 20, oz::kBK, ld, 0, 0, c);
    }
    return 0;
}

template <int E, bool ALONG>
int all() {
    for (int n : {1, 2, 3, 15, 16, 17, 31, 62, 63, 64, 65, 66, 127, 128, 129, 130, 191, 193, 257})
        for (int K = 1; K <= 67; ++K)
            for (int odd : {0, 1, 2, 7})
                if (check<E, ALONG>(n, K, odd)) return 1;
    return limits<E, ALONG>();
}

int main() {
    if (all<64, true>() || all<64, false>() || all<128, true>() || all<128, false>()) return 1;
    std::printf("ok %ld\n", checked);
    return 0;
}
