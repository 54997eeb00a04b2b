// Answers questions about the layouts and rules that the kernels and their launches share, one per line of standard
// input.  Host code only (tests/test_host_rules.py, tests/test_z_area.py):
//   z BLOCKS RANK OUTPUTS      end, in bytes behind the start of the z area, of the last piece that a two-launch LoRA call
//                              writes for that many 16-row blocks
//   piece COLUMNS MOST RANK    last_factor_piece
#include "../paper_2605_14217_amd/csrc/common.hpp"

#include <cstdio>
#include <cstring>

int main()
{
    char what[16];
    while (std::scanf("%15s", what) == 1) {
        long long a[3];
        if (std::scanf("%lld %lld %lld", &a[0], &a[1], &a[2]) != 3) return 1;
        if (!std::strcmp(what, "z")) {
            const int rank = (int)a[1], n = (int)a[2], nb = preft::z_rank_blocks(rank);
            std::printf("%lld\n", (long long)(preft::z_piece(a[0] - 1, n, n - 1, nb, nb - 1) + 64) * 16);
        } else if (!std::strcmp(what, "piece")) {
            std::printf("%d\n", preft::last_factor_piece((int)a[0], (int)a[1], (int)a[2]));
        } else {
            return 1;
        }
    }
    return 0;
}
