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


def _run(dtype, rank, d_in, d_out, T, poison, direft=False, z_rank=0):
    tab = wl.from_lengths(np.array([T]), np.array([0]), np.array([T]))
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
    ws = preft.new_workspace(T, 1, z_rank=z_rank)
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
