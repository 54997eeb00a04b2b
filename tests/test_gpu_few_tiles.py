"""Batches of a few short prompts, whose tiles the small-batch and fp32 kernels spread over the XCDs: chunks that are mostly
empty beside gathered rows, and chunks that are full, each row exactly once (against the oracle, inactive rows bit for bit)."""
import numpy as np
import pytest

from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu

LENGTHS = {"short": [10, 14, 11, 13] + [1] * 14, "one": [5], "nine": [17] * 9, "full": [128, 128, 256, 120], "edge": [96, 95, 97] + [2] * 5,
           "many": [6] * 70 + [1] * 30, "thousand": [100] * 10,
           # empty segments hide the prompt rows from the host's estimate: the launches are too small and stride over their tiles
           "empty": [0] * 500 + [200, 90, 33] + [0] * 400 + [3, 129, 1, 1]}


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


@pytest.mark.parametrize("rank", [3, 7, 16, 32, 40, 64])
@pytest.mark.parametrize("lens", [[1] * 1100, [0] * 2000 + [700, 500, 2, 1], [1] * 1100 + [90]], ids=["decode", "hidden", "one-prompt"])
def test_batches_with_next_to_no_prompt(lens, rank):
    """Above 1024 rows: a step of decode rows alone, prompts hidden from the host's estimate by empty segments, and one prompt beside
    decode rows; with a workspace that has room for two launches, chosen by the library and forced."""
    import paper_2605_14217_amd as preft
    from parity_util import run_lora_case
    N = 6
    rng = np.random.Generator(np.random.PCG64(len(lens)))
    lens = np.array(lens)
    tab = wl.from_lengths(lens, rng.integers(-1, N, size=len(lens)), np.where(lens > 1, lens, 0))
    x = wl.activations(tab.T, 256, "bf16", device="cuda", seed=1)
    y0 = wl.activations(tab.T, 1152, "bf16", device="cuda", seed=2)
    pool = wl.lora_pool(N, rank, 256, 1152, "bf16", device="cuda", seed=3)
    for flags in (0, preft.test_flags(resident=1)):
        prev = preft.set_test_flags(flags)
        try:
            for all_tokens in (False, True):
                run_lora_case(tab, pool, x, y0, "bf16", 2.0, all_tokens, pad_cols=8, z_room=True)
        finally:
            preft.set_test_flags(prev)


@pytest.mark.parametrize("dtype,rank,d,rows", [("bf16", 32, 1024, 1000), ("bf16", 16, 1000, 900), ("bf16", 7, 264, 700), ("f32", 4, 2048, 600),
                                               ("f32", 1, 1536, 700), ("f32", 3, 4096, 150)])
def test_many_layers_give_the_bits_of_one(dtype, rank, d, rows):
    """A layer of a many-layer call is its one-layer call, bit for bit: which kernel runs does not hang on the number of layers."""
    from parity_util import run_direft_layers_case
    N, L = 3, 4
    tab = wl.from_lengths(np.array([rows // 2, rows - rows // 2 - 40] + [1] * 40), np.arange(42) % N, np.array([rows // 2, rows - rows // 2 - 40] + [1] * 40))
    if rows == 150:
        tab = wl.from_lengths(np.ones(rows, int), np.arange(rows) % N, np.ones(rows, int))
    pools = [wl.direft_pool(N, rank, d, dtype, device="cuda", seed=l) for l in range(L)]
    hs = [wl.activations(tab.T, d, dtype, device="cuda", seed=9 + l) for l in range(L)]
    for all_tokens in (False, True):
        run_direft_layers_case(tab, pools, hs, dtype, 0.5, all_tokens, [True] * L, pad_cols=8)
