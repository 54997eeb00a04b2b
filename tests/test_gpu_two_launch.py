"""LoRA as two launches (shrink into the workspace's z area, then the expand in 2-D tiles): every rank class, at the
edges of its tiles -- 32 rows x 512 columns, 128-column units, 32-column steps -- against the oracle, and bit for
bit against the single launch: how many bytes of workspace a call is handed decides which launches it takes, never what
it returns.  Bars of parity_util: row-wise 1e-2 for bf16 storage."""
import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu

# prompts of 1, 15..17, 31..33, 127..129 rows between decode rows, and one empty segment
LENS = [1, 15, 16, 17, 31, 32, 33, 5, 0, 127, 128, 129, 4, 560] + [1] * 40

CASES = [(1, 512, (512,)), (1, 136, (1032, 8, 520)), (2, 1096, (2056, 384)), (3, 1000, (520, 8)), (3, 4104, (136, 520, 1024)), (4, 128, (128, 1032, 512)), (5, 264, (640,)), (7, 1000, (2728, 2728)),
         (8, 136, (1544,)), (12, 520, (504, 512)), (16, 4104, (512,)), (16, 512, (1536, 256, 256)), (13, 384, (1288, 24, 512)),
         (17, 128, (128,)), (20, 256, (512, 256)), (24, 256, (384,)), (32, 512, (256, 128)), (28, 1024, (512, 640, 256)), (31, 384, (512, 128, 256)), (36, 128, (1152,)), (48, 256, (512,)),
         (63, 256, (640, 512)), (64, 128, (128, 1664)),
         # panels of 64 rows x 256 columns that share their factors (rank 33-64 in multiples of 4, every width a multiple of 256)
         (36, 384, (256,)), (40, 128, (512, 256)), (48, 256, (768, 256, 1024)), (52, 128, (256, 1280)), (60, 640, (512,)), (64, 128, (256, 512, 256)), (64, 1024, (1536,)),
         # the same at ranks that are no multiple of 4, and panels of 64 x 128 where a width is no multiple of 256
         (33, 128, (256,)), (37, 256, (768, 512)), (63, 128, (1024,)), (49, 128, (384, 256, 128)), (44, 256, (640,))]


@pytest.mark.parametrize("pad", [0, 8])
@pytest.mark.parametrize("rank,d_in,d_outs", CASES, ids=[f"r{c[0]}-{c[1]}-{'x'.join(map(str, c[2]))}" for c in CASES])
def test_two_launches_match_the_oracle_and_the_single_launch(rank, d_in, d_outs, pad):
    from oracle import preft_oracle as ora
    from parity_util import bits, check_guards, compare, dev_tables, lora_pools_to_device, padded
    N = 5
    rng = np.random.Generator(np.random.PCG64(rank * 31 + d_in))
    lens = np.array(LENS)
    ids = rng.integers(-1, N + 1, size=len(lens))              # -1 and N: no adapter
    tab = wl.from_lengths(lens, ids, np.where(np.arange(len(lens)) < 14, np.maximum(lens - (lens > 100), 0), 0))
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    x = wl.activations(T, d_in, "bf16", device="cuda", seed=1)
    y0s = [wl.activations(T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
    pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=9 + i) for i, n in enumerate(d_outs)]
    tables = [lora_pools_to_device(pl) for pl in pools]
    ws = preft.new_workspace(T, tab.S, z_rank=rank, z_proj=len(d_outs))

    def call(mode, flags):
        ws.fill_(0xa5)                                        # nothing in the workspace has to start at zero
        bufs = [padded(y, pad, 7.0) for y in y0s]
        prev = preft.set_test_flags(flags)
        try:
            preft.preft_lora_apply_packed([b[1] for b in bufs], x, ss, sa, sp, [t[0] for t in tables],
                                          [t[1] for t in tables], rank, 2.0, mode, ws)
        finally:
            preft.set_test_flags(prev)
        torch.cuda.synchronize()
        for (buf, _), n in zip(bufs, d_outs):
            check_guards(buf, T, n, 7.0)
        return [b[1] for b in bufs]

    for all_tokens in (False, True):
        mode = preft.PREFT_ALL_TOKENS if all_tokens else preft.PREFT_PREFILL_ONLY
        pos = ora.ALL_POSITIONS if all_tokens else ora.PROMPT_ONLY
        owner = ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, pos)
        two = call(mode, preft.test_flags(resident=1))
        for y, y0, pl in zip(two, y0s, pools):
            want = ora.lora(y0.cpu(), x.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len,
                            [a.cpu() for a in pl.A], [b.cpu() for b in pl.B], rank, 2.0, pos)
            compare(y, y0, want, owner, "bf16")
        one = call(mode, preft.test_flags(variant=5, colsplit=1) if rank >= 4 else preft.test_flags(variant=2))
        for y, y1 in zip(two, one):
            assert torch.equal(bits(y), bits(y1))


@pytest.mark.parametrize("rank,d", [(36, 256), (48, 384), (64, 128), (64, 1024), (33, 128), (63, 256), (50, 640)])
def test_in_place_as_two_launches(rank, d):
    """DiReFT at rank 33-64: against the oracle, and bit for bit what a workspace without room for z gets (one launch)."""
    from oracle import preft_oracle as ora
    from parity_util import bits, check_guards, compare, dev_tables, direft_pools_to_device, padded
    N = 5
    rng = np.random.Generator(np.random.PCG64(rank + d))
    lens = np.array(LENS)
    tab = wl.from_lengths(lens, rng.integers(-1, N + 1, size=len(lens)), np.where(np.arange(len(lens)) < 14, np.maximum(lens - (lens > 100), 0), 0))
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    h0 = wl.activations(T, d, "bf16", device="cuda", seed=3)
    pool = wl.direft_pool(N, rank, d, "bf16", device="cuda", seed=4)
    W1, W2t, b, keep = direft_pools_to_device(pool, bias=True)
    for mode, pos in ((preft.PREFT_PREFILL_ONLY, ora.PROMPT_ONLY), (preft.PREFT_ALL_TOKENS, ora.ALL_POSITIONS)):
        got = []
        for z_rank, flags in ((rank, preft.test_flags(resident=1)), (0, preft.test_flags(variant=4))):
            ws = preft.new_workspace(T, tab.S, z_rank=z_rank)
            ws.fill_(0xa5)
            buf, h = padded(h0, 8, 7.0)
            prev = preft.set_test_flags(flags)
            try:
                preft.preft_direft_apply(h, ss, sa, sp, W1, W2t, b, rank, 0.5, mode, ws)
            finally:
                preft.set_test_flags(prev)
            torch.cuda.synchronize()
            check_guards(buf, T, d, 7.0)
            got.append(h)
        want = ora.direft(h0.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, [a.cpu() for a in pool.A],
                          [m.cpu() for m in pool.B], [v.cpu() for v in pool.b], rank, 0.5, pos)
        compare(got[0], h0, want, ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, pos), "bf16")
        assert torch.equal(bits(got[0]), bits(got[1]))


def _table(rank, d, N, empty=0):
    rng = np.random.Generator(np.random.PCG64(rank + d))
    lens = np.array(LENS + [0] * empty)
    return wl.from_lengths(lens, rng.integers(-1, N + 1, size=len(lens)), np.where(np.arange(len(lens)) < 14, np.maximum(lens - (lens > 100), 0), 0))


def _lora(tab, N, rank, d_in, d_outs, sides):
    """Every side (flags, room for z) against the oracle, guards untouched, and all of them bit for bit alike; both position sets."""
    from oracle import preft_oracle as ora
    from parity_util import bits, check_guards, compare, dev_tables, lora_pools_to_device, padded
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    x = wl.activations(T, d_in, "bf16", device="cuda", seed=1)
    y0s = [wl.activations(T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
    pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=9 + i) for i, n in enumerate(d_outs)]
    tables = [lora_pools_to_device(pl) for pl in pools]
    for mode, pos in ((preft.PREFT_PREFILL_ONLY, ora.PROMPT_ONLY), (preft.PREFT_ALL_TOKENS, ora.ALL_POSITIONS)):
        owner = ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, pos)
        got = []
        for flags, room in sides:
            ws = preft.new_workspace(T, tab.S, z_rank=rank if room else 0, z_proj=len(d_outs))
            ws.fill_(0xa5)
            bufs = [padded(y, 8, 7.0) for y in y0s]
            prev = preft.set_test_flags(flags)
            try:
                preft.preft_lora_apply_packed([b[1] for b in bufs], x, ss, sa, sp, [t[0] for t in tables], [t[1] for t in tables], rank, 2.0, mode, ws)
            finally:
                preft.set_test_flags(prev)
            torch.cuda.synchronize()
            for (buf, _), n in zip(bufs, d_outs):
                check_guards(buf, T, n, 7.0)
            got.append([b[1] for b in bufs])
        for i, pl in enumerate(pools):
            want = ora.lora(y0s[i].cpu(), x.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, [a.cpu() for a in pl.A], [b.cpu() for b in pl.B], rank, 2.0, pos)
            compare(got[0][i], y0s[i], want, owner, "bf16")
            for other in got[1:]:
                assert torch.equal(bits(got[0][i]), bits(other[i]))


def _direft(tab, N, rank, d, sides, layers):
    """The same in place; `layers`: the flags of a call of two layers, each of which has the bits of its one-layer call."""
    from oracle import preft_oracle as ora
    from parity_util import bits, check_guards, compare, dev_tables, direft_pools_to_device, padded
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    h0 = wl.activations(T, d, "bf16", device="cuda", seed=3)
    pool = wl.direft_pool(N, rank, d, "bf16", device="cuda", seed=4)
    W1, W2t, b, keep = direft_pools_to_device(pool, bias=True)
    table = lambda t: torch.tensor([t.data_ptr()] * 2, dtype=torch.int64, device="cuda")
    for mode, pos in ((preft.PREFT_PREFILL_ONLY, ora.PROMPT_ONLY), (preft.PREFT_ALL_TOKENS, ora.ALL_POSITIONS)):
        got = []
        for flags, room in sides + [(layers, True)]:
            ws = preft.new_workspace(T, tab.S, z_rank=rank if room else 0)
            ws.fill_(0xa5)
            bufs = [padded(h0, 8, 7.0) for _ in range(2)]
            prev = preft.set_test_flags(flags)
            try:
                if len(got) < len(sides):
                    preft.preft_direft_apply(bufs[0][1], ss, sa, sp, W1, W2t, b, rank, 0.5, mode, ws)
                else:
                    hs = [v[1] for v in bufs]
                    preft.preft_direft_apply_layers(hs, torch.tensor([v.data_ptr() for v in hs], dtype=torch.int64, device="cuda"), ss, sa, sp, table(W1), table(W2t), table(b), N, rank, 0.5, mode, ws)
            finally:
                preft.set_test_flags(prev)
            torch.cuda.synchronize()
            for buf, _ in bufs:
                check_guards(buf, T, d, 7.0)
            got.append(bufs[0][1])
            if len(got) > len(sides):
                assert torch.equal(bits(bufs[0][1]), bits(bufs[1][1]))
        want = ora.direft(h0.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, [a.cpu() for a in pool.A], [m.cpu() for m in pool.B], [v.cpu() for v in pool.b],
                          rank, 0.5, pos)
        compare(got[0], h0, want, ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, pos), "bf16")
        for other in got[1:]:
            assert torch.equal(bits(got[0]), bits(other))


# the small-batch kernel's shrink as a launch of its own: one to four rank blocks a workgroup, ranks that end in a block, one to three outputs, widths that are no
# multiple of 128 or of a panel, d_in of one to three rounds of the wavefronts' units
SHRINK = [(20, 264, (1032, 8, 520)), (24, 4104, (512,)), (28, 128, (128, 1032)), (32, 1000, (520,)), (36, 136, (1096, 520)), (48, 4104, (264,)), (52, 512, (1536, 256, 264)),
          (64, 2056, (520,)), (68, 264, (136,)), (96, 1032, (1032, 520)), (100, 128, (264,)), (112, 512, (640,)), (128, 4104, (136, 1544))]


@pytest.mark.parametrize("rank,d_in,d_outs", SHRINK, ids=[f"r{c[0]}-{c[1]}-{'x'.join(map(str, c[2]))}" for c in SHRINK])
@pytest.mark.parametrize("many", [False, True])
def test_small_batch_shrink_then_expand(rank, d_in, d_outs, many):
    """Against the oracle, and bit for bit the small-batch kernel's single launch; many: so many segments that a workgroup takes three or four rank blocks."""
    tab = _table(rank, d_in, 5, 3000 if many else 0)
    _lora(tab, 5, rank, d_in, d_outs, [(preft.test_flags(resident=2), True), (preft.test_flags(resident=2), False), (preft.test_flags(colsplit=3), True)])


@pytest.mark.parametrize("rank", [36, 64, 128])
@pytest.mark.parametrize("decode", [True, False], ids=["decode", "prompts"])
def test_many_adapters_sum_in_the_same_groups(tmp_path_factory, rank, decode):
    """About as many adapters as segments: the single launch has 4 wavefronts instead of 8, and the shrink launch sums in as many groups.  With room for z, without, and
    with room as two launches in any case: the same bits."""
    from test_host_rules import ask
    rng = np.random.Generator(np.random.PCG64(rank))
    if decode:
        tab = wl.from_lengths(np.ones(512, int), rng.integers(0, 64, 512), np.zeros(512, int))
    else:
        lens = rng.integers(6, 20, 64)
        tab = wl.from_lengths(lens, rng.permutation(64), lens)
    d_in, d_out = 1544, 4104
    takes, _, _, waves, _ = ask(tmp_path_factory, [f"small {tab.T} {tab.S} 64 1 {rank} {d_in} {d_out} 0 0"])[0].split()
    assert (takes, waves) == ("1", "4")
    _lora(tab, 64, rank, d_in, (d_out,), [(0, True), (0, False), (preft.test_flags(resident=2), True)])


@pytest.mark.parametrize("rank,d", [(20, 8200), (32, 264), (36, 1032), (48, 4104), (64, 512), (68, 136), (96, 2056), (128, 264)])
def test_small_batch_shrink_then_expand_in_place(rank, d):
    flags = preft.test_flags(resident=2)
    _direft(_table(rank, d, 5), 5, rank, d, [(flags, True), (flags, False)], flags)


@pytest.mark.parametrize("rank,d_in,d_outs", [(68, 128, (128,)), (96, 256, (384, 128)), (100, 384, (256,)), (128, 1024, (640,)), (128, 256, (1152, 128, 128))])
@pytest.mark.parametrize("tall", [False, True])
def test_two_launches_above_rank_64(rank, d_in, d_outs, tall):
    """64-row tiles and (tall: by the number of segments) 128-row tiles of the row-split kernel's shrink, then the panels: out of place and in place."""
    tab = _table(rank, d_in, 5, 1100 if tall else 0)
    one = preft.test_flags(variant=5, colsplit=1)
    _lora(tab, 5, rank, d_in, d_outs, [(preft.test_flags(resident=1), True), (one, True)])
    _direft(tab, 5, rank, d_in, [(preft.test_flags(resident=1), True), (preft.test_flags(resident=1), False)], preft.test_flags(resident=1))


@pytest.mark.parametrize("rank,d,empty", [(64, 8192, 0), (63, 7680, 0), (96, 8192, 0), (96, 8192, 1100)])
def test_in_place_calls_that_the_cache_can_hold(rank, d, empty):
    """17 MB of h and more, without the non-temporal hint in either launch (above rank 64 in 64- and 128-row tiles): the bits of the single launch."""
    tab = _table(rank, d, 5, empty)
    assert tab.T * d * 2 >= 16 << 20
    _direft(tab, 5, rank, d, [(0, True), (preft.test_flags(variant=4), False)], 0)


@pytest.mark.parametrize("rank,d", [(20, 9224), (32, 10240), (28, 14336)])
def test_wide_rows_in_place_keep_units(rank, d):
    """Rank 20-32 on rows wider than 8192: 8 units a wavefront in registers, the bits of tiles that are streamed in both sweeps."""
    _direft(_table(rank, d, 5), 5, rank, d, [(0, True), (preft.test_flags(variant=3), True)], 0)


@pytest.mark.parametrize("rank,d", [(20, 9224), (32, 10240), (28, 14336)])
def test_wide_rows_of_long_prompts_keep_units(rank, d):
    """The same where the dispatch takes that form: segments of 72 rows and more on average."""
    tab = wl.from_lengths(np.array([700, 129, 500, 33, 161]), np.array([0, 3, -1, 2, 0]), np.array([700, 128, 500, 33, 0]))
    _direft(tab, 5, rank, d, [(0, True), (preft.test_flags(variant=3), True)], 0)
