"""Infinities and NaN reach exactly the results the definition sends them to: a padded rank or column of a kernel's
tile must not turn an infinite factor, activation or intermediate into NaN elsewhere.  The expected values are the
definition's in float64, where sums and products of infinities do not depend on the order; finite results are compared within
the usual bars."""
import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _same(got, want, dtype):
    got, want = got.double().cpu(), want.cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want)), "NaN where the definition has none, or none where it has"
    assert torch.equal(torch.isposinf(got), torch.isposinf(want)) and torch.equal(torch.isneginf(got), torch.isneginf(want))
    fin = torch.isfinite(want)
    if not bool(fin.any()):
        return
    scale = want[fin].abs().max()
    assert float((got[fin] - want[fin]).abs().max()) <= (1e-5 if dtype == "f32" else 1e-2) * float(scale)


def _definition(y, x, A, B, scale, b=None):
    x, A, B = (t.double().cpu() for t in (x, A, B))
    z = (x[:, None, :] * A[None]).sum(-1) + (0 if b is None else b.double().cpu())
    return y.double().cpu() + scale * (z[:, None, :] * B[None]).sum(-1)


def _run(dtype, rank, d_in, d_out, T, poison, direft=False, z_rank=0, lens=None):
    """lens: segment lengths where the T rows are not one prompt; every position counts."""
    lens = np.array([T] if lens is None else lens)
    tab = wl.from_lengths(lens, np.zeros(len(lens), int), lens)
    ss, sa, sp = (torch.from_numpy(a.copy()).cuda() for a in (tab.seg_start, tab.seg_adapter, tab.seg_prefill_len))
    x = wl.activations(T, d_in, dtype, device="cuda", seed=1)
    y = x if direft else wl.activations(T, d_out, dtype, device="cuda", seed=2)
    A = wl.activations(rank, d_in, dtype, device="cuda", seed=3)
    B = wl.activations(d_out, rank, dtype, device="cuda", seed=4)
    inf = float("inf")
    if poison == "factor":                         # single elements of the second factor, at the first, a middle and the last rank
        B[3, 0], B[d_out // 2, rank // 2], B[d_out - 1, rank - 1] = inf, -inf, inf
    elif poison == "nan factor":
        B[5, rank - 1] = float("nan")
    elif poison == "row":                          # an activation, so that this row's whole intermediate is infinite
        x[7, d_in - 1], x[T - 1, 0] = inf, -inf
    elif poison == "first factor":
        A[rank - 1, 2] = inf
    want = _definition(y, x, A, B, 0.5)
    ws = preft.new_workspace(T, tab.S, z_rank=z_rank)
    Ap, Bp = preft.pointer_table([A]), preft.pointer_table([B])
    out = y.clone()
    if direft:
        preft.preft_direft_apply(out, ss, sa, sp, Ap, Bp, None, rank, 0.5, preft.PREFT_PREFILL_ONLY, ws)
    else:
        preft.preft_lora_apply(out, x, ss, sa, sp, Ap, Bp, rank, 0.5, preft.PREFT_PREFILL_ONLY, ws)
    torch.cuda.synchronize()
    _same(out, want, dtype)


POISON = ["factor", "nan factor", "row", "first factor"]


@pytest.mark.parametrize("poison", POISON)
@pytest.mark.parametrize("rank", [1, 3, 5, 8, 12, 16, 20, 31, 36, 65, 100])
def test_fp32(rank, poison):
    _run("f32", rank, 132, 140, 100, poison)
    _run("f32", rank, 132, 132, 100, poison, direft=True)


@pytest.mark.parametrize("poison", POISON)
@pytest.mark.parametrize("rank", [1, 2, 3])
def test_bf16_rank_1_to_3_in_two_launches(rank, poison):
    prev = preft.set_test_flags(preft.test_flags(resident=1))
    try:
        _run("bf16", rank, 136, 520, 100, poison, z_rank=rank)
    finally:
        preft.set_test_flags(prev)


# Ranks above 16 that are no multiple of 4, on the kernels that the per-row kernels' calls have gone to: the small-batch kernel (prompts, tiles of a
# few decode rows), the column-split kernel (widths that are no multiples of 128; gathered tiles beside the row-split kernel's chunks)
ODD_CALLS = [(136, 264, [100], False), (128, 256, [1] * 3, False), (136, 136, [90, 1, 1, 7], True), (264, 136, [1100], False), (136, 136, [1100], True),
             (128, 256, [1] * 1100, False), (256, 256, [1] * 1050, True)]


@pytest.mark.parametrize("poison", POISON)
@pytest.mark.parametrize("rank", [17, 31, 45, 63, 66, 127])
def test_bf16_ranks_above_16_that_are_no_multiple_of_4(rank, poison):
    for d_in, d_out, lens, direft in ODD_CALLS:
        if poison == "row" and sum(lens) < 8:
            continue
        _run("bf16", rank, d_in, d_out, sum(lens), poison, direft=direft, lens=lens)


@pytest.mark.parametrize("rank", [17, 31, 45, 63, 66, 127])
def test_those_ranks_keep_an_intermediate_of_24_bits(rank):
    """Each row has z = 2^23 + 2^14 + 1 in one rank and 2^23 + 2^14 in another, with factors of 1 and -1: the result is 1 if z reaches it in 32 bits, and 0
    from 16 bits of it (2^23 and 2^14)."""
    from parity_util import dev_tables
    pairs = [(2 * i, 2 * i + 1 if 2 * i + 1 < rank else rank - 2) for i in range((rank + 1) // 2)]
    for d_in, d_out, lens, direft in ODD_CALLS:
        d, T = 512 if d_in % 128 == 0 else 520, sum(lens)
        tab = wl.from_lengths(np.array(lens), np.zeros(len(lens), int), np.array(lens))
        ss, sa, sp = dev_tables(tab)
        A = torch.zeros(rank, d)
        sign = torch.ones(rank)
        for i, (one, other) in enumerate(pairs):
            A[one, 3 * i:3 * i + 3] = torch.tensor([2048.0, 128.0, 1.0])
            A[other, 3 * i:3 * i + 3] = torch.tensor([2048.0, 128.0, 0.0])
            sign[other] = -1
        x = torch.zeros(T, d)
        for t in range(T):
            i = t % len(pairs)
            x[t, 3 * i:3 * i + 3] = torch.tensor([4096.0, 128.0, 1.0])
        A, x, sign = (v.to(torch.bfloat16).cuda() for v in (A, x, sign))
        B = torch.zeros(d if direft else d_out, rank, dtype=torch.bfloat16, device="cuda")
        B[d - 1 if direft else slice(None)] = sign
        Ap, Bp, ws = preft.pointer_table([A]), preft.pointer_table([B]), preft.new_workspace(T, tab.S)
        y = x if direft else torch.zeros(T, d_out, dtype=torch.bfloat16, device="cuda")
        if direft:
            preft.preft_direft_apply(x, ss, sa, sp, Ap, Bp, None, rank, 1.0, preft.PREFT_ALL_TOKENS, ws)
            y = y[:, d - 1]
        else:
            preft.preft_lora_apply(y, x, ss, sa, sp, Ap, Bp, rank, 1.0, preft.PREFT_ALL_TOKENS, ws)
        assert torch.equal(y, torch.ones_like(y)), (d, d_out, len(lens), direft)
