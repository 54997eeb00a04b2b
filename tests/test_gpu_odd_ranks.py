"""Ranks above 16 that are no multiple of 4, on widths that are multiples of 128 and on others: the small-batch kernel (up to 1024 rows), the
column-split kernel (chunks and gathered tiles of 32 and 16 rows), packed and in place, one layer and several.  Against the oracle
(parity_util's bars), and the last rank's factors to a value: an integer check that no neighbouring column's factor gets in."""
import shutil

import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [(17, 264, (136,)), (18, 128, (1000, 8)), (19, 1000, (256,)), (30, 136, (520, 264, 128)), (31, 520, (392,)), (33, 264, (136, 384)), (47, 128, (264,)),
         (50, 392, (1032,)), (63, 1000, (136, 8)), (65, 136, (264,)), (126, 264, (136,)), (127, 128, (520,))]


def _table(N, rows, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    lens = np.array([1, 15, 16, 17, 33, 5, 4, 3, 2, 129] + ([700, 600] if rows > 1024 else []) + [1] * 40)
    return wl.from_lengths(lens, rng.integers(-1, N + 1, size=len(lens)), np.where(lens > 1, lens, 0))


@pytest.mark.parametrize("rows", [200, 1500])
@pytest.mark.parametrize("rank,d_in,d_outs", CASES, ids=[f"r{c[0]}-{c[1]}-{'x'.join(map(str, c[2]))}" for c in CASES])
def test_against_the_oracle(rank, d_in, d_outs, rows):
    from oracle import preft_oracle as ora
    from parity_util import bits, check_guards, compare, dev_tables, direft_pools_to_device, lora_pools_to_device, padded
    N = 4
    tab = _table(N, rows, rank)
    assert (tab.T > 1024) == (rows > 1024)
    ss, sa, sp = dev_tables(tab)
    tables = (tab.seg_start, tab.seg_adapter, tab.seg_prefill_len)
    x = wl.activations(tab.T, d_in, "bf16", device="cuda", seed=1)
    y0s = [wl.activations(tab.T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
    pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=9 + i) for i, n in enumerate(d_outs)]
    dev = [lora_pools_to_device(pl) for pl in pools]
    dpool = wl.direft_pool(N, rank, d_in, "bf16", device="cuda", seed=20)
    W1, W2t, b, keep = direft_pools_to_device(dpool)
    for z_rank in (0, rank):
        ws = preft.new_workspace(tab.T, tab.S, z_rank=z_rank, z_proj=len(d_outs))
        for mode, pos in ((preft.PREFT_PREFILL_ONLY, ora.PROMPT_ONLY), (preft.PREFT_ALL_TOKENS, ora.ALL_POSITIONS)):
            ws.fill_(0x5a)
            owner = ora.positions(tab.T, *tables, N, pos)
            bufs = [padded(y, 8, 7.0) for y in y0s]
            hbuf, h = padded(x, 8, 7.0)
            preft.preft_lora_apply_packed([v[1] for v in bufs], x, ss, sa, sp, [t[0] for t in dev], [t[1] for t in dev], rank, 2.0, mode, ws)
            preft.preft_direft_apply(h, ss, sa, sp, W1, W2t, b, rank, 0.5, mode | preft.PREFT_SCHEDULE_READY, ws)
            for (buf, y), y0, pl in zip(bufs, y0s, pools):
                check_guards(buf, tab.T, y0.shape[1], 7.0)
                want = ora.lora(y0.cpu(), x.cpu(), *tables, [a.cpu() for a in pl.A], [m.cpu() for m in pl.B], rank, 2.0, pos)
                compare(y, y0, want, owner, "bf16")
            check_guards(hbuf, tab.T, d_in, 7.0)
            want = ora.direft(x.cpu(), *tables, [a.cpu() for a in dpool.A], [m.cpu() for m in dpool.B], [v.cpu() for v in dpool.b], rank, 0.5, pos)
            compare(h, x, want, owner, "bf16")
            if z_rank == 0:                                   # several layers: the bits of one
                hs = [x.clone(), x.clone()]
                layers = [torch.tensor([t.data_ptr()] * 2, dtype=torch.int64, device="cuda") for t in (W1, W2t, b)]
                preft.preft_direft_apply_layers(hs, preft.pointer_table(hs), ss, sa, sp, *layers, N, rank, 0.5, mode | preft.PREFT_SCHEDULE_READY, ws)
                assert all(torch.equal(bits(v), bits(h)) for v in hs)


@pytest.mark.parametrize("rows", [100, 1500])
@pytest.mark.parametrize("rank,d,d_out", [(17, 136, 264), (19, 128, 136), (31, 264, 264), (33, 136, 136), (45, 128, 264), (63, 264, 136), (66, 136, 136), (127, 128, 264)])
def test_every_rank_meets_its_own_factor(rank, d, d_out, rows):
    """x and A pick rank k in row k (mod rank); B holds a different integer in every place: y must be exactly that integer."""
    from parity_util import dev_tables
    tab = wl.from_lengths(np.array([rows]), np.array([0]), np.array([rows]))
    ss, sa, sp = dev_tables(tab)
    A = torch.zeros(rank, d, dtype=torch.bfloat16, device="cuda")
    A[torch.arange(rank), torch.arange(rank)] = 1
    x = torch.zeros(rows, d, dtype=torch.bfloat16, device="cuda")
    x[torch.arange(rows), torch.arange(rows) % rank] = 1
    B = ((torch.arange(d_out * rank, device="cuda").view(d_out, rank) * 7) % 251 - 125).to(torch.bfloat16)
    y = torch.zeros(rows, d_out, dtype=torch.bfloat16, device="cuda")
    preft.preft_lora_apply(y, x, ss, sa, sp, preft.pointer_table([A]), preft.pointer_table([B]), rank, 1.0, preft.PREFT_PREFILL_ONLY,
                           preft.new_workspace(rows, 1))
    assert torch.equal(y, B.t()[torch.arange(rows, device="cuda") % rank])


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="asks the dispatch through hipcc")
@pytest.mark.parametrize("rank,d", [(17, 128), (18, 4096), (30, 2048), (31, 1024)])
def test_in_place_on_widths_that_are_multiples_of_128(rank, d, tmp_path_factory):
    """Rank 17-31 in place: the column-split and the row-split kernel, which the test flags choose; both against the oracle on the same rows, and
    the default call the one that the dispatch names, to the bit: short prompts, long ones, a batch above 16 384 rows, and one of short prompts alone."""
    from oracle import preft_oracle as ora
    from paper_2605_14217_amd import binding as B
    from parity_util import bits, compare, dev_tables, direft_pools_to_device
    from test_host_rules import ask
    N = 4
    seen = set()
    for lens in ([1, 15, 16, 17, 33, 5, 4, 129, 700, 600] + [1] * 20, [17, 129, 700, 600], [1, 15, 16, 17, 33, 5, 4, 129, 700, 600] + [5100] * 3 + [1] * 20, [40] * 220):
        lens = np.array(lens)
        tab = wl.from_lengths(lens, np.random.Generator(np.random.PCG64(rank)).integers(-1, N + 1, size=len(lens)), np.where(lens > 1, lens, 0))
        ss, sa, sp = dev_tables(tab)
        tables = (tab.seg_start, tab.seg_adapter, tab.seg_prefill_len)
        x = wl.activations(tab.T, d, "bf16", device="cuda", seed=1)
        pool = wl.direft_pool(N, rank, d, "bf16", device="cuda", seed=20)
        W1, W2t, b, keep = direft_pools_to_device(pool)
        ws = preft.new_workspace(tab.T, tab.S, z_rank=rank)
        got = {}
        for variant in (0, 3, 4):
            h = x.clone()
            prev = B.set_test_flags(B.test_flags(variant=variant))
            try:
                preft.preft_direft_apply(h, ss, sa, sp, W1, W2t, b, rank, 0.5, preft.PREFT_ALL_TOKENS, ws)
            finally:
                B.set_test_flags(prev)
            got[variant] = h
        streams = int(ask(tmp_path_factory, [f"route {tab.T} {tab.S} {rank} {d} {d} 1"])[0].split()[1])
        seen.add(streams)
        assert torch.equal(bits(got[0]), bits(got[3 if streams else 4]))
        if tab.T <= 16384:
            owner = ora.positions(tab.T, *tables, N, ora.ALL_POSITIONS)
            want = ora.direft(x.cpu(), *tables, [a.cpu() for a in pool.A], [m.cpu() for m in pool.B], [v.cpu() for v in pool.b], rank, 0.5, ora.ALL_POSITIONS)
            for h in got.values():
                compare(h, x, want, owner, "bf16")
        else:
            assert (got[3].float() - got[4].float()).abs().max() <= 2 ** -6 * got[4].float().abs().max()      # two bf16 roundings of the largest value
    assert seen == ({1} if d >= 4096 else {0, 1})


@pytest.mark.parametrize("rank,d,outs,lens,in_place", [(127, 8523264, (128,), [5, 1], False), (64, 17301504, (128,), [5, 1], False), (31, 35791488, (), [5], True),
                                                       (63, 17432576, (128, 256), [600, 500, 1], False), (16, 71586816, (8, 16), [5, 1], False)])
def test_factors_beyond_the_column_split_kernels_offsets(rank, d, outs, lens, in_place):
    """First factors of more than 2^31 bytes, whose last rank lies beyond a signed 32-bit offset: only that rank's row holds anything, ones and minus ones, and
    x single ones, so that z is a small integer and y that integer times its factor, to the bit."""
    from parity_util import dev_tables
    lens = np.array(lens)
    T = int(lens.sum())
    tab = wl.from_lengths(lens, np.zeros(len(lens), int), np.where(lens > 1, lens, 0))
    ss, sa, sp = dev_tables(tab)
    g = torch.Generator(device="cuda").manual_seed(rank)
    A = torch.zeros(rank, d, dtype=torch.bfloat16, device="cuda")
    A[rank - 1] = 2 * torch.randint(0, 2, (d,), generator=g, device="cuda") - 1
    at = torch.randint(0, d, (T, 64), generator=g, device="cuda")          # places of x that hold a one
    x = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda").scatter_(1, at, 1.0)
    z = torch.stack([A[rank - 1][torch.unique(at[t])].float().sum() for t in range(T)]).view(T, 1)
    Ap = preft.pointer_table([A])
    ws = preft.new_workspace(T, len(lens), z_rank=min(rank, 64), z_proj=max(1, len(outs)))
    Bs = [torch.randint(-3, 4, (n, rank), generator=g, device="cuda").to(torch.bfloat16) for n in (outs or (d,))]
    if in_place:
        want = (x.float() + z * Bs[0][:, rank - 1].float()).to(torch.bfloat16)
        preft.preft_direft_apply(x, ss, sa, sp, Ap, preft.pointer_table(Bs), None, rank, 1.0, preft.PREFT_ALL_TOKENS, ws)
        assert torch.equal(x, want)
        return
    ys = [torch.zeros(T, n, dtype=torch.bfloat16, device="cuda") for n in outs]
    preft.preft_lora_apply_packed(ys, x, ss, sa, sp, [Ap] * len(outs), [preft.pointer_table([b]) for b in Bs], rank, 1.0, preft.PREFT_ALL_TOKENS, ws)
    for y, b in zip(ys, Bs):
        assert torch.equal(y, (z * b[:, rank - 1].float()).to(torch.bfloat16))
