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

int main(int argc, char **argv) {
    if (argc == 2 && !strcmp(argv[1], "breed_lds")) breed_lds();
    else return 1;
    return 0;
}
