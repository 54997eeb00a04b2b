// Prints where a two-launch LoRA call's kernels put the intermediate z: the end, in bytes behind the start of the z
// area, of the last piece that a batch of `blocks` 16-row blocks writes.  Host code only; see test_z_area.py.
#include "../paper_2605_14217_amd/csrc/common.hpp"

#include <cstdio>
#include <cstdlib>

int main(int argc, char **argv)
{
    for (int i = 1; i + 2 < argc; i += 3) {
        const long long blocks = std::atoll(argv[i]);
        const int rank = std::atoi(argv[i + 1]), n = std::atoi(argv[i + 2]), nb = preft::z_rank_blocks(rank);
        std::printf("%lld\n", (long long)(preft::z_piece(blocks - 1, n, n - 1, nb, nb - 1) + 64) * 16);
    }
    return 0;
}
