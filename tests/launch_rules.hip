// Prints the launch rules of pga_internal.hpp that tests/test_launch_rules.py checks; host code only.
#include "../paper_1403_4099_amd/csrc/pga_internal.hpp"

#include <cstdio>
#include <cstring>

using namespace pga;

// per launch size and largest N: the LDS a breed launch asks for, and the most that an instance of 1 .. N stocks uses
static void breed_lds() {
    for (int inds : {1, 4095, 4096, 16383, 16384, 65535, 65536, 1 << 20}) {
        const BreedShape b = breed_shape(inds);
        size_t used = 0;
        for (int n = 1; n <= PGA_N_MAX; ++n) {
            const size_t x = sizeof(uint32_t) * (size_t)breed_split(n, b).chr * (3 + 4 * (size_t)((n + 127) / 128));
            used = x > used ? x : used;
            printf("%d %d %zu %zu\n", inds, n, breed_lds_bytes(n, b), used);
        }
    }
}

// per N: the entries of C that the FP64 pair-sum's walk loads, and those among them that are outside C or, for a row
// above the lane's column (the ones whose value counts), not the row's own
static void fp64_rows() {
    for (int N = 1; N <= PGA_N_MAX; ++N) {
        const int n_jb = (N + kFp64Cols - 1) / kFp64Cols;
        long loads = 0, outside = 0, other = 0;
        for (int jb = 0; jb < n_jb; ++jb) {
            const int col = (jb + 1) * kFp64Cols <= N ? (jb + 1) * kFp64Cols - 1 : N - 1;   // last stock
            auto load = [&](int i, bool clamped) {
                const long long row = fp64_row(i, N, clamped);
                ++loads;
                if (row < 0 || 8 * (row * N + col) + 8 > 8ll * N * N) ++outside;
                if (i < col && row != i) ++other;
            };
            for (int q = 0; q < kFp64Ahead; ++q) load(q, true);
            for (int ch = 0; ch <= jb; ++ch)
                for (int r = 0; r < 64; r += kFp64Ahead)
                    for (int q = 0; q < kFp64Ahead; ++q) load(64 * ch + r + kFp64Ahead + q, fp64_clamps(ch == jb, r));
        }
        printf("%d %ld %ld %ld\n", N, loads, outside, other);
    }
}

int main(int argc, char **argv) {
    if (argc == 2 && !strcmp(argv[1], "breed_lds")) breed_lds();
    else if (argc == 2 && !strcmp(argv[1], "fp64_rows")) fp64_rows();
    else return 1;
    return 0;
}
