"""fp32 on the matrix cores: rank blocks and their remainders, widths that are no multiple of a 64-column unit, tiles of
1..16 rows, gathered rows, shared tiles (colsplit) and many layers, against the oracle.  Bar of parity_util: row-wise
1e-5 for fp32 storage."""
import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _table(N):
    lens = np.array([1, 5, 16, 17, 0, 33, 128, 130] + [1] * 21)
    return wl.from_lengths(lens, np.arange(len(lens)) % (N + 1) - (np.arange(len(lens)) % 7 == 3),
                           np.where(np.arange(len(lens)) < 8, np.maximum(lens - (lens > 100), 0), 0))


@pytest.mark.parametrize("colsplit", [0, 3])
@pytest.mark.parametrize("rank,d_in,d_out", [(1, 68, 4), (4, 512, 512), (5, 1004, 700), (16, 4, 516), (17, 324, 64), (33, 512, 132),
                                             (64, 196, 1000), (65, 128, 260), (127, 576, 68), (128, 64, 2052),
                                             (7, 264, 1028), (15, 72, 260), (31, 132, 4100)])
def test_lora(rank, d_in, d_out, colsplit):
    from parity_util import run_lora_case
    N = 4
    tab = _table(N)
    pool = wl.lora_pool(N, rank, d_in, d_out, "f32", device="cuda", seed=rank)
    x = wl.activations(tab.T, d_in, "f32", device="cuda", seed=1)
    y0 = wl.activations(tab.T, d_out, "f32", device="cuda", seed=2)
    prev = preft.set_test_flags(preft.test_flags(colsplit=colsplit))
    try:
        for all_tokens in (False, True):
            run_lora_case(tab, pool, x, y0, "f32", 2.0, all_tokens, pad_cols=4, perm=[2, 0, 3, 1])
    finally:
        preft.set_test_flags(prev)


@pytest.mark.parametrize("rank,d", [(3, 68), (8, 4096), (16, 516), (31, 1004), (48, 512), (63, 132), (100, 260)])
def test_direft_and_layers(rank, d):
    from parity_util import run_direft_case, run_direft_layers_case
    N = 4
    tab = _table(N)
    pools = [wl.direft_pool(N, rank, d, "f32", device="cuda", seed=rank + l) for l in range(2)]
    hs = [wl.activations(tab.T, d, "f32", device="cuda", seed=5 + l) for l in range(2)]
    for all_tokens in (False, True):
        run_direft_case(tab, pools[0], hs[0], "f32", 0.5, all_tokens, pad_cols=4, null_bias=(1,))
        run_direft_layers_case(tab, pools, hs, "f32", 0.5, all_tokens, [True, False], pad_cols=8)


@pytest.mark.parametrize("rank,d_out", [(1, 516), (7, 1028), (13, 260), (18, 4100), (31, 2052)])
def test_both_forms_of_the_expand_give_the_same_bits(rank, d_out):
    """Ranks up to 32 that are no multiple of 4: factors through LDS where a workgroup has units enough, lane by lane where many share a tile."""
    from parity_util import bits, dev_tables, lora_pools_to_device
    tab = _table(4)
    pool = wl.lora_pool(4, rank, 196, d_out, "f32", device="cuda", seed=rank)
    A, B, keep = lora_pools_to_device(pool)
    x, y0 = (wl.activations(tab.T, n, "f32", device="cuda", seed=n) for n in (196, d_out))
    got = []
    for colsplit in (1, 8):
        y = y0.clone()
        prev = preft.set_test_flags(preft.test_flags(colsplit=colsplit))
        try:
            preft.preft_lora_apply(y, x, *dev_tables(tab), A, B, rank, 2.0, preft.PREFT_ALL_TOKENS, preft.new_workspace(tab.T, tab.S))
        finally:
            preft.set_test_flags(prev)
        got.append(y)
    assert torch.equal(bits(got[0]), bits(got[1])) and not torch.equal(bits(got[0]), bits(y0))
