"""The small-batch kernel's shapes, each reached by the sizes of a call and not by a test flag: deep workgroups of one unit up to
many, the shallow ones of rank 4-16, the 4-wavefront ones above rank 32; single and packed outputs, ragged widths, decode rows of many
adapters and prompts, both position sets.  The dispatch is asked on the host that a call takes the shape it is here for; the
result is compared with the oracle (parity_util's bars)."""
import shutil

import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(shutil.which("hipcc") is None, reason="asks the dispatch through hipcc")]

# (what the call is here for: deep, wavefronts, least units of a share), rank, d_in, outputs, decode rows, adapters, prompts
CASES = [
    ((0, 8, 8), 16, 264, (14336, 14336), 32, 32, ()), ((0, 8, 8), 7, 200, (13336, 14344), 40, 40, ()), ((0, 8, 8), 4, 512, (4104,), 512, 512, ()),
    ((0, 8, 8), 15, 128, (8192, 1032, 1024), 512, 400, ()), ((0, 8, 16), 12, 1000, (14336, 14336), 16, 5, (200,) * 4),
    ((1, 8, 8), 16, 512, (4096,), 500, 21, ()), ((1, 8, 4), 8, 512, (1024,), 3, 2, ()), ((1, 8, 2), 24, 512, (1024,), 16, 16, (200,)),
    ((1, 8, 2), 32, 264, (14336, 14344), 32, 32, ()), ((1, 8, 32), 20, 136, (14336, 14336, 4096), 512, 64, ()),
    ((1, 8, 1), 64, 376, (1024,), 2, 1, ()), ((1, 8, 1), 36, 136, (1096, 520), 10, 3, (17,)), ((1, 8, 1), 128, 256, (1024,), 20, 8, (60, 5)),
    ((1, 4, 8), 40, 256, (4096,), 512, 512, ()), ((1, 4, 8), 64, 264, (14336, 1032), 64, 64, ()), ((1, 4, 8), 96, 128, (6152,), 96, 96, ()),
    ((1, 4, 8), 128, 136, (4096, 4096, 136), 40, 40, ()),
]


@pytest.mark.parametrize("shape,rank,d_in,d_outs,decode,N,prompts", CASES, ids=[f"r{c[1]}-{c[2]}-{'x'.join(map(str, c[3]))}-{c[4]}of{c[5]}" for c in CASES])
def test_shape_against_the_oracle(tmp_path_factory, shape, rank, d_in, d_outs, decode, N, prompts):
    from oracle import preft_oracle as ora
    from parity_util import check_guards, compare, dev_tables, lora_pools_to_device, padded
    from test_host_rules import ask
    rng = np.random.Generator(np.random.PCG64(rank + d_in))
    lens = np.array(list(prompts) + [1] * decode)
    order = rng.permutation(len(lens))
    ids = np.concatenate([rng.integers(0, N, size=len(prompts)), rng.permutation(np.arange(decode) % N)]).astype(int)
    tab = wl.from_lengths(lens[order], ids[order], np.where(lens > 1, lens, 0)[order])
    T = tab.T
    widths = list(d_outs) + [0] * (3 - len(d_outs))
    answer = ask(tmp_path_factory, [f"small {T} {tab.S} {N} 1 {rank} {d_in} " + " ".join(map(str, widths))])[0].split()
    takes, units, deep, waves = (int(v) for v in answer[:4])
    assert takes == 1 and (deep, waves) == shape[:2] and units >= shape[2], answer
    ss, sa, sp = dev_tables(tab)
    x = wl.activations(T, d_in, "bf16", device="cuda", seed=1)
    y0s = [wl.activations(T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
    pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=9 + i) for i, n in enumerate(d_outs)]
    tables = [lora_pools_to_device(pl) for pl in pools]
    ws = preft.new_workspace(T, tab.S)
    for mode, pos in ((preft.PREFT_ALL_TOKENS, ora.ALL_POSITIONS), (preft.PREFT_PREFILL_ONLY, ora.PROMPT_ONLY)):
        bufs = [padded(y, 8, 7.0) for y in y0s]
        preft.preft_lora_apply_packed([b[1] for b in bufs], x, ss, sa, sp, [t[0] for t in tables], [t[1] for t in tables], rank, 2.0, mode, ws)
        owner = ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, pos)
        for (buf, y), y0, pl in zip(bufs, y0s, pools):
            check_guards(buf, T, y0.shape[1], 7.0)
            want = ora.lora(y0.cpu(), x.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len,
                            [a.cpu() for a in pl.A], [b.cpu() for b in pl.B], rank, 2.0, pos)
            compare(y, y0, want, owner, "bf16")


@pytest.mark.parametrize("rank,d,d_out", [(16, 512, 4096), (4, 136, 264), (7, 1000, 520), (32, 256, 1032), (64, 384, 512), (96, 128, 256)])
def test_tiles_of_one_to_sixteen_rows(rank, d, d_out):
    """Gathered tiles of 1, 4, 5 and 16 rows and prompts that end 1, 4 and 5 rows into a tile, out of place (where tiles of at most four rows load a
    quarter of what others do) and in place beside prompts (where they do not), against the oracle; and the row's bits are those it has
    beside others in a tile."""
    from oracle import preft_oracle as ora
    from parity_util import bits, compare, dev_tables, direft_pools_to_device, lora_pools_to_device
    counts, prompts = [1, 4, 5, 16], [17, 20, 21, 36]
    N = len(counts) + len(prompts)
    lens = np.array([1] * sum(counts) + prompts)
    ids = np.concatenate([np.repeat(np.arange(len(counts)), counts), len(counts) + np.arange(len(prompts))]).astype(int)
    order = np.random.Generator(np.random.PCG64(rank)).permutation(len(lens))
    x = None
    rows = {}                                                 # the same rows under one adapter each, and all under adapter 0 (fuller tiles)
    for kind, who in (("own", ids[order]), ("one", np.zeros(len(lens), dtype=int))):
        tab = wl.from_lengths(lens[order], who, np.where(lens > 1, lens, 0)[order])
        if x is None:
            x, y0, h0 = (wl.activations(tab.T, n, "bf16", device="cuda", seed=i) for i, n in enumerate((d, d_out, d)))
        ss, sa, sp = dev_tables(tab)
        pool, dpool = wl.lora_pool(N, rank, d, d_out, "bf16", device="cuda", seed=5), wl.direft_pool(N, rank, d, "bf16", device="cuda", seed=6)
        if kind == "own":                                     # every adapter has the same weights, so that rows can be compared
            for m in (pool.A, pool.B, dpool.A, dpool.B, dpool.b):
                for i in range(1, N):
                    m[i].copy_(m[0])
            same = pool, dpool
        pool, dpool = same
        A, B, keep = lora_pools_to_device(pool)
        W1, W2t, b, keep2 = direft_pools_to_device(dpool)
        ws = preft.new_workspace(tab.T, tab.S)
        y, h = y0.clone(), h0.clone()
        preft.preft_lora_apply(y, x, ss, sa, sp, A, B, rank, 2.0, preft.PREFT_ALL_TOKENS, ws)
        preft.preft_direft_apply(h, ss, sa, sp, W1, W2t, b, rank, 0.5, preft.PREFT_ALL_TOKENS, ws)
        owner = ora.positions(tab.T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, ora.ALL_POSITIONS)
        tables = (tab.seg_start, tab.seg_adapter, tab.seg_prefill_len)
        compare(y, y0, ora.lora(y0.cpu(), x.cpu(), *tables, [a.cpu() for a in pool.A], [m.cpu() for m in pool.B], rank, 2.0, ora.ALL_POSITIONS), owner, "bf16")
        compare(h, h0, ora.direft(h0.cpu(), *tables, [a.cpu() for a in dpool.A], [m.cpu() for m in dpool.B], [v.cpu() for v in dpool.b], rank, 0.5,
                                  ora.ALL_POSITIONS), owner, "bf16")
        rows[kind] = y, h
    assert bits(rows["own"][0]).equal(bits(rows["one"][0])) and bits(rows["own"][1]).equal(bits(rows["one"][1]))


@pytest.mark.parametrize("rank,d", [(4, 520), (12, 1024), (16, 1032), (4, 4096), (4, 8192), (5, 2120), (7, 4104), (7, 8192), (16, 2760), (16, 8192), (16, 14336), (17, 1000), (24, 4096),
                                    (24, 1000), (31, 1000), (31, 8192), (32, 4096), (33, 2056), (63, 1000), (63, 8192), (64, 4096), (64, 8192), (64, 264)])
def test_in_place_steps_of_decode_rows(tmp_path_factory, rank, d):
    """A step of single rows alone in place: the form that loads a quarter for tiles of at most four rows, at 1, 4, 5 and 16 rows of an adapter,
    one layer and several, against the oracle; and each row has the bits that it has in a batch beside a prompt, where the quarter form does not run."""
    from parity_util import bits, dev_tables, direft_pools_to_device, run_direft_layers_case
    from test_host_rules import ask
    counts, N, L = [1, 4, 5, 16], 40, 3
    ids = np.random.Generator(np.random.PCG64(rank + d)).permutation(np.repeat([3, 11, 17, 39], counts))
    tab = wl.from_lengths(np.ones(len(ids), int), ids, np.zeros(len(ids), int))
    beside = wl.from_lengths(np.append(np.ones(len(ids), int), 30), np.append(ids, 7), np.append(np.zeros(len(ids), int), 30))
    few, other = (tuple(map(int, a.split())) for a in ask(tmp_path_factory, [f"in_place {t.T} {t.S} {N} 1 {rank} {d}" for t in (tab, beside)]))
    assert few == (1, 1) and other[1] == 0
    pools = [wl.direft_pool(N, rank, d, "bf16", device="cuda", seed=l) for l in range(L)]
    hs = [wl.activations(tab.T, d, "bf16", device="cuda", seed=9 + l) for l in range(L)]
    run_direft_layers_case(tab, pools, hs, "bf16", 0.5, True, [True, False, True], pad_cols=8)
    if other[0]:                                              # beside the prompt the same kernel, in its other form
        W1, W2t, b, keep = direft_pools_to_device(pools[0])
        rows = []
        for t in (tab, beside):
            h = torch.zeros(t.T, d, dtype=torch.bfloat16, device="cuda")
            h[:tab.T] = hs[0]
            preft.preft_direft_apply(h, *dev_tables(t), W1, W2t, b, rank, 0.5, preft.PREFT_ALL_TOKENS, preft.new_workspace(t.T, t.S))
            rows.append(h[:tab.T])
        assert bits(rows[0]).equal(bits(rows[1]))


@pytest.mark.parametrize("rank", [4, 7, 16, 20, 32])
@pytest.mark.parametrize("d_in", [8, 1024, 1032, 2048, 2056, 4096, 4104, 6152, 9216])
def test_shrink_of_few_rows(rank, d_in):
    """Tiles of at most four rows: one, two and four units of d_in on their way in each wavefront, with and without a round that repeats, a last
    unit that is cut off and wavefronts without one; in place and out of place, against the oracle."""
    from parity_util import run_direft_case, run_lora_case
    N, counts = 5, [1, 3, 4, 6]
    ids = np.random.Generator(np.random.PCG64(rank + d_in)).permutation(np.repeat(np.arange(4), counts))
    tab = wl.from_lengths(np.ones(len(ids), int), ids, np.zeros(len(ids), int))
    x = wl.activations(tab.T, d_in, "bf16", device="cuda", seed=1)
    y0 = wl.activations(tab.T, 392, "bf16", device="cuda", seed=2)
    run_lora_case(tab, wl.lora_pool(N, rank, d_in, 392, "bf16", device="cuda", seed=3), x, y0, "bf16", 2.0, True, pad_cols=8)
    run_direft_case(tab, wl.direft_pool(N, rank, d_in, "bf16", device="cuda", seed=4), x, "bf16", 0.5, True, pad_cols=8)


@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("d_in,d_outs", [(264, (1032,)), (4104, (512,)), (1000, (520, 8, 2056)), (6152, (4096,))])
def test_small_ranks(rank, d_in, d_outs):
    """Ranks up to 8, of whose first factor a wavefront loads one or two groups of four ranks, and ranks 1-3, whose expand runs on the vector ALU: tiles of one
    to sixteen rows, prompts and decode rows, out of place and in place (one layer and several), infinite factors of one adapter, against the oracle."""
    from oracle import preft_oracle as ora
    from parity_util import check_guards, compare, dev_tables, lora_pools_to_device, padded, run_direft_case, run_direft_layers_case
    N, counts, prompts = 9, [1, 4, 5, 16], [17, 20, 36, 130]
    lens = np.array([1] * sum(counts) + prompts)
    ids = np.concatenate([np.repeat(np.arange(4), counts), 4 + np.arange(4)]).astype(int)
    order = np.random.Generator(np.random.PCG64(rank + d_in)).permutation(len(lens))
    tab = wl.from_lengths(lens[order], ids[order], np.where(lens > 1, lens, 0)[order])
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    x = wl.activations(T, d_in, "bf16", device="cuda", seed=1)
    y0s = [wl.activations(T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
    pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=9 + i) for i, n in enumerate(d_outs)]
    tables = [lora_pools_to_device(pl) for pl in pools]
    for mode, pos in ((preft.PREFT_ALL_TOKENS, ora.ALL_POSITIONS), (preft.PREFT_PREFILL_ONLY, ora.PROMPT_ONLY)):
        bufs = [padded(y, 8, 7.0) for y in y0s]
        preft.preft_lora_apply_packed([b[1] for b in bufs], x, ss, sa, sp, [t[0] for t in tables], [t[1] for t in tables], rank, 2.0, mode, preft.new_workspace(T, tab.S))
        owner = ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, pos)
        for (buf, y), y0, pl in zip(bufs, y0s, pools):
            check_guards(buf, T, y0.shape[1], 7.0)
            want = ora.lora(y0.cpu(), x.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, [a.cpu() for a in pl.A], [b.cpu() for b in pl.B], rank, 2.0, pos)
            compare(y, y0, want, owner, "bf16")
        run_direft_case(tab, wl.direft_pool(N, rank, d_in, "bf16", device="cuda", seed=4), x, "bf16", 0.5, pos == ora.ALL_POSITIONS, pad_cols=8)
    run_direft_layers_case(tab, [wl.direft_pool(N, rank, d_in, "bf16", device="cuda", seed=l) for l in range(2)],
                           [wl.activations(T, d_in, "bf16", device="cuda", seed=9 + l) for l in range(2)], "bf16", 0.5, True, [True, False], pad_cols=8)
    # an infinite factor makes infinities where its product with z does not vanish, never NaN, and only in its own adapter's rows
    pools[0].B[4][:] = float("inf")
    A, B, keep = lora_pools_to_device(pools[0])
    y = y0s[0].clone()
    preft.preft_lora_apply(y, x, ss, sa, sp, A, B, rank, 2.0, preft.PREFT_ALL_TOKENS, preft.new_workspace(T, tab.S))
    mine = torch.from_numpy(ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, ora.ALL_POSITIONS) == 4).cuda()
    assert bool(torch.isfinite(y[~mine]).all()) and not bool(torch.isfinite(y[mine]).any())
    if rank == 1:
        assert bool(torch.isinf(y[mine]).all())


@pytest.mark.parametrize("rank", [20, 24, 28, 32])
@pytest.mark.parametrize("d_in,d_out", [(264, 1032), (1000, 520), (4104, 2056)])
def test_forms_of_rank_20_to_32(rank, d_in, d_out):
    """Each rank has a form of its own (the groups of the first factor that are loaded, the way of the second): tiles of one to sixteen rows, prompts and decode rows, out of place
    and in place, one layer and several, against the oracle."""
    from parity_util import run_direft_case, run_direft_layers_case, run_lora_case
    lens = np.array([1] * 26 + [17, 20, 36, 130])
    ids = np.concatenate([np.repeat(np.arange(4), [1, 4, 5, 16]), 4 + np.arange(4)]).astype(int)
    order = np.random.Generator(np.random.PCG64(rank + d_in)).permutation(len(lens))
    tab = wl.from_lengths(lens[order], ids[order], np.where(lens > 1, lens, 0)[order])
    x = wl.activations(tab.T, d_in, "bf16", device="cuda", seed=1)
    y0 = wl.activations(tab.T, d_out, "bf16", device="cuda", seed=2)
    for all_tokens in (True, False):
        run_lora_case(tab, wl.lora_pool(8, rank, d_in, d_out, "bf16", device="cuda", seed=3), x, y0, "bf16", 2.0, all_tokens, pad_cols=8)
        run_direft_case(tab, wl.direft_pool(8, rank, d_in, "bf16", device="cuda", seed=4), x, "bf16", 0.5, all_tokens, pad_cols=8)
    run_direft_layers_case(tab, [wl.direft_pool(8, rank, d_in, "bf16", device="cuda", seed=l) for l in range(2)],
                           [wl.activations(tab.T, d_in, "bf16", device="cuda", seed=9 + l) for l in range(2)], "bf16", 0.5, True, [True, False], pad_cols=8)
