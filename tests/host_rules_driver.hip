// Answers questions about the layouts and rules that the kernels and their launches share, one per line of standard
// input.  Host code only (tests/test_host_rules.py, tests/test_z_area.py):
//   z BLOCKS RANK OUTPUTS      end, in bytes behind the start of the z area, of the last piece that a two-launch LoRA call
//                              writes for that many 16-row blocks
//   piece COLUMNS MOST RANK    last_factor_piece
//   small T S N ALL RANK D_IN D0 D1 D2   whether a LoRA call with these outputs (0: none) takes the small-batch kernel, and as what:
//                              units of a share, deep, wavefronts, units of the launch
//   in_place T S N ALL RANK D  whether an in-place call takes the small-batch kernel, and whether with quarter tiles (decode rows alone)
//   route T S RANK D_IN D_OUT DIREFT   what takes a bf16 call above 1024 rows: whether the matrix-core kernels do; whether the column-split kernel
//                              then takes the chunks of a rank above 16 that is no multiple of 4; and whether it fits
#include "../paper_2605_14217_amd/csrc/dispatch.hpp"

#include <cstdio>
#include <cstring>

int main()
{
    char what[16];
    while (std::scanf("%15s", what) == 1) {
        long long a[9];
        if (!std::strcmp(what, "small")) {
            for (long long &v : a)
                if (std::scanf("%lld", &v) != 1) return 1;
            preft::ApplyArgs p = {};
            p.T = (int)a[0]; p.N = (int)a[2]; p.all_tokens = (int)a[3]; p.rank = (int)a[4]; p.d_in = (int)a[5];
            p.d_out = (int)a[6]; p.more[0].d_out = (int)a[7]; p.more[1].d_out = (int)a[8]; p.n_layers = 1; p.col_split = 1;
            const int n = a[8] ? 3 : a[7] ? 2 : 1;
            int widest = 0;
            for (int i = 6; i < 9; ++i) widest = a[i] > widest ? (int)a[i] : widest;
            const preft::Knobs k = {};
            const preft::SmallShape s = preft::small_shape(p, a[1], n, k);
            std::printf("%d %d %d %d %u\n", preft::takes_small(p, a[1], widest, false, k), s.units, s.deep, s.waves, preft::likely_units(p, a[1]));
            continue;
        }
        if (!std::strcmp(what, "in_place")) {
            for (int i = 0; i < 6; ++i)
                if (std::scanf("%lld", &a[i]) != 1) return 1;
            preft::ApplyArgs p = {};
            p.T = (int)a[0]; p.N = (int)a[2]; p.all_tokens = (int)a[3]; p.rank = (int)a[4]; p.d_in = p.d_out = (int)a[5]; p.n_layers = 1;
            std::printf("%d %d\n", preft::takes_small(p, a[1], p.d_in, true, preft::Knobs{}), preft::small_in_place_few(p, a[1]));
            continue;
        }
        if (!std::strcmp(what, "route")) {
            for (int i = 0; i < 6; ++i)
                if (std::scanf("%lld", &a[i]) != 1) return 1;
            preft::ApplyArgs p = {};
            p.T = (int)a[0]; p.rank = (int)a[2]; p.d_in = (int)a[3]; p.d_out = (int)a[4];
            const preft::Knobs k = {};
            std::printf("%d %d %d\n", preft::mfma_takes(p, k), preft::odd_streams(p, a[1], a[5] != 0, k), preft::column_split_fits(p));
            continue;
        }
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
