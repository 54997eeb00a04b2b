"""fp32 calls on both sides of the rule that chooses between the per-row and the tile kernel, and of the one that chooses
how many workgroups share a tile: every combination gives the oracle's result (row-wise 1e-5, parity_util's bar), in place and
out of place, whichever kernel the automatic choice takes."""
import numpy as np
import pytest

from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [1, 3, 4, 5, 7, 8, 9])
@pytest.mark.parametrize("kind", ["decode", "many-adapters", "prompts", "mixed"])
def test_automatic_choice(rank, kind):
    from parity_util import run_direft_case, run_lora_case
    N = 64 if kind == "many-adapters" else 5
    rng = np.random.Generator(np.random.PCG64(rank))
    lens = {"decode": np.ones(70, int), "many-adapters": np.ones(150, int), "prompts": np.array([20, 300, 5]),
            "mixed": np.concatenate([np.array([90, 0, 33]), np.ones(40, int)])}[kind]
    tab = wl.from_lengths(lens, rng.integers(0, N, size=len(lens)), lens)
    for d_in, d_outs in ((132, (260,)), (1540, (1540, 100)), (4100, (132,))):
        x = wl.activations(tab.T, d_in, "f32", device="cuda", seed=1)
        for d_out in d_outs:
            y0 = wl.activations(tab.T, d_out, "f32", device="cuda", seed=2)
            pool = wl.lora_pool(N, rank, d_in, d_out, "f32", device="cuda", seed=3)
            run_lora_case(tab, pool, x, y0, "f32", 2.0, True, pad_cols=4)
        pool = wl.direft_pool(N, rank, d_in, "f32", device="cuda", seed=4)
        run_direft_case(tab, pool, x, "f32", 0.5, True, pad_cols=4)
