// Answers what the dispatch does with a call, one per line of standard input: T S N ALL RANK D_IN WIDTH BYTES (of an element), for a call of one output of WIDTH
// columns, and for one in place on rows of D_IN columns.  Host code only (tests/test_dispatch_lines.py).  Answers: takes_small, small_in_two and activations_stay of the
// LoRA call, takes_small, small_in_two, h_stays and
// keeps_units of the one in place, and expand_ids_fit of the LoRA call.
#include "../paper_2605_14217_amd/csrc/dispatch.hpp"

#include <cstdio>

int main()
{
    long long a[8];
    while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7) == 8) {
        preft::ApplyArgs p = {};
        p.T = (int)a[0]; p.N = (int)a[2]; p.all_tokens = (int)a[3]; p.rank = (int)a[4]; p.d_in = (int)a[5]; p.d_out = (int)a[6]; p.n_layers = 1; p.col_split = 1;
        const preft::Knobs k = {};
        const int ids = preft::expand_ids_fit(p, a[1], 1);
        const int lora[3] = {preft::takes_small(p, a[1], p.d_out, p.d_out, false, k), preft::small_in_two(p, a[1], p.d_out, false, k), preft::activations_stay(p, a[1], p.d_out, (int)a[7], a[7] == 4 ? preft::STAY_F32 : preft::STAY_BF16)};
        p.d_out = p.d_in;
        std::printf("%d %d %d %d %d %d %d %d\n", lora[0], lora[1], lora[2], preft::takes_small(p, a[1], p.d_in, p.d_in, true, k), preft::small_in_two(p, a[1], p.d_in, true, k), preft::h_stays(p),
                    preft::keeps_units(p, a[1]), ids);
    }
    return 0;
}
