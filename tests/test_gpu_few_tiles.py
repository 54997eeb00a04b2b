"""Batches of a few short prompts, whose tiles the small-batch and fp32 kernels spread over the XCDs: chunks that are mostly
empty beside gathered rows, and chunks that are full, each row exactly once (against the oracle, inactive rows bit for bit)."""
import numpy as np
import pytest

from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu

LENGTHS = {"short": [10, 14, 11, 13] + [1] * 14, "one": [5], "nine": [17] * 9, "full": [128, 128, 256, 120], "edge": [96, 95, 97] + [2] * 5,
           "many": [6] * 70 + [1] * 30, "thousand": [100] * 10}


@pytest.mark.parametrize("dtype,rank", [("bf16", 5), ("bf16", 16), ("bf16", 64), ("f32", 7), ("f32", 16)])
@pytest.mark.parametrize("lens", LENGTHS.values(), ids=LENGTHS.keys())
def test_every_row_once(lens, dtype, rank):
    from parity_util import run_direft_case, run_lora_case
    N = 6
    rng = np.random.Generator(np.random.PCG64(len(lens)))
    tab = wl.from_lengths(np.array(lens), rng.integers(-1, N, size=len(lens)), np.array(lens))
    x = wl.activations(tab.T, 264, dtype, device="cuda", seed=1)
    y0 = wl.activations(tab.T, 1048, dtype, device="cuda", seed=2)
    pool = wl.lora_pool(N, rank, 264, 1048, dtype, device="cuda", seed=3)
    edit = wl.direft_pool(N, rank, 264, dtype, device="cuda", seed=4)
    for all_tokens in (False, True):
        run_lora_case(tab, pool, x, y0, dtype, 2.0, all_tokens, pad_cols=8)
        run_direft_case(tab, edit, x, dtype, 0.5, all_tokens, pad_cols=8)
