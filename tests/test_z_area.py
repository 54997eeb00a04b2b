"""The z area of a workspace (preft_workspace_bytes_z) holds every piece that a two-launch LoRA call writes: on the
host, for every rank, from the address function the kernels use; on the GPU, with guard bytes right behind it."""
import shutil

import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_the_area_covers_every_piece_the_kernels_write(tmp_path_factory):
    from test_host_rules import ask
    # batches whose chunk list fills its capacity best: few long segments, whole chunks; and segments just above a chunk
    # and batches of short segments, every one a gathered tile of its own (an adapter each)
    batches = [[2048], [128], [129], [1152], [4096], [1000] * 8, [700] * 50, [5] * 400, [129] * 30, [128] * 16 + [1] * 40, [1], [1] * 7, [1] * 500, [2] * 300, [4] * 200, [1] * 300 + [2048], [5] * 100 + [1] * 400]
    asked, lines = [], []
    for lens in batches:
        # whole chunks; the gathered tiles (at most one per short segment) lie behind them, and where there are none the last chunk counts up to the 64-row tile that holds its last row
        chunks = sum((n + 127) // 128 for n in lens if n > 4) * 8
        gathered = sum(1 for n in lens if n <= 4)
        if not gathered:
            last = [n for n in lens if n > 4][-1]
            chunks -= 4 if (last - 1) % 128 < 64 else 0
        for rank in range(1, 129):
            for n_proj in (1, 2, 3):
                asked.append((lens, rank, n_proj))
                lines.append(f"z {chunks + gathered} {rank} {n_proj}")
    ends = [int(v) for v in ask(tmp_path_factory, lines)]
    assert len(ends) == len(asked)
    for (lens, rank, n_proj), end in zip(asked, ends):
        T, S = sum(lens), len(lens)
        start = (preft.preft_workspace_bytes(T, S) + 255) // 256 * 256
        assert start + end <= preft.preft_workspace_bytes_z(T, S, rank, n_proj), (lens[:3], S, rank, n_proj)


@pytest.mark.gpu
@pytest.mark.parametrize("rank", [16, 17, 32, 33, 40, 47, 48, 49, 64])
@pytest.mark.parametrize("lens", [[2048], [1152, 1000]], ids=["one-segment", "two-segments"])
def test_nothing_is_written_behind_the_workspace(rank, lens):
    from oracle import preft_oracle as ora
    from parity_util import compare, dev_tables, lora_pools_to_device
    d_in, N, guard = 256, 2, 1 << 20
    tab = wl.from_lengths(np.array(lens), np.arange(len(lens)) % N, np.array(lens))
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    owner = ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, ora.PROMPT_ONLY)
    x = wl.activations(T, d_in, "bf16", device="cuda", seed=1)
    for n_proj in (1, 2, 3):
        d_outs = (512, 128, 384)[:n_proj]
        y0s = [wl.activations(T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
        pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=5 + i) for i, n in enumerate(d_outs)]
        tables = [lora_pools_to_device(pl) for pl in pools]
        need = preft.preft_workspace_bytes_z(T, tab.S, rank, n_proj)
        buf = torch.full((need + guard,), 0x5a, dtype=torch.uint8, device="cuda")
        ys = [y.clone() for y in y0s]
        prev = preft.set_test_flags(preft.test_flags(resident=1))
        try:
            preft.preft_lora_apply_packed(ys, x, ss, sa, sp, [t[0] for t in tables], [t[1] for t in tables], rank, 2.0,
                                          preft.PREFT_PREFILL_ONLY, buf[:need])
        finally:
            preft.set_test_flags(prev)
        torch.cuda.synchronize()
        assert bool((buf[need:] == 0x5a).all()), f"bytes behind the workspace were written (rank {rank}, {n_proj} outputs)"
        for i, pl in enumerate(pools):
            want = ora.lora(y0s[i].cpu(), x.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len,
                            [a.cpu() for a in pl.A], [b.cpu() for b in pl.B], rank, 2.0, ora.PROMPT_ONLY)
            compare(ys[i], y0s[i], want, owner, "bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("rank", [20, 48, 68, 128])
@pytest.mark.parametrize("lens", [[1152, 1000], [1] * 300, [129] * 3 + [1] * 40 + [4] * 30], ids=["prompts", "decode", "both"])
@pytest.mark.parametrize("resident", [1, 2])
def test_nothing_is_written_behind_the_workspace_above_rank_16(rank, lens, resident):
    """resident=2: the small-batch kernel's shrink, which writes the z of gathered tiles at every rank; 1: the row-split kernel's, of up to eight rank blocks.  An adapter for every segment."""
    from oracle import preft_oracle as ora
    from parity_util import compare, dev_tables, lora_pools_to_device
    d_in, N, guard = 256, len(lens), 1 << 20
    tab = wl.from_lengths(np.array(lens), np.arange(N), np.where(np.array(lens) > 4, lens, 0))
    T = tab.T
    ss, sa, sp = dev_tables(tab)
    owner = ora.positions(T, tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, N, ora.ALL_POSITIONS)
    x = wl.activations(T, d_in, "bf16", device="cuda", seed=1)
    d_outs = (512, 128, 384)[:1 if resident == 1 and rank > 64 else 3]
    y0s = [wl.activations(T, n, "bf16", device="cuda", seed=2 + i) for i, n in enumerate(d_outs)]
    pools = [wl.lora_pool(N, rank, d_in, n, "bf16", device="cuda", seed=5 + i) for i, n in enumerate(d_outs)]
    tables = [lora_pools_to_device(pl) for pl in pools]
    need = preft.preft_workspace_bytes_z(T, tab.S, rank, len(d_outs))
    buf = torch.full((need + guard,), 0x5a, dtype=torch.uint8, device="cuda")
    ys = [y.clone() for y in y0s]
    prev = preft.set_test_flags(preft.test_flags(resident=resident))
    try:
        preft.preft_lora_apply_packed(ys, x, ss, sa, sp, [t[0] for t in tables], [t[1] for t in tables], rank, 2.0, preft.PREFT_ALL_TOKENS, buf[:need])
    finally:
        preft.set_test_flags(prev)
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x5a).all()), f"bytes behind the workspace were written (rank {rank}, {len(d_outs)} outputs)"
    for i, pl in enumerate(pools):
        want = ora.lora(y0s[i].cpu(), x.cpu(), tab.seg_start, tab.seg_adapter, tab.seg_prefill_len, [a.cpu() for a in pl.A], [b.cpu() for b in pl.B], rank, 2.0, ora.ALL_POSITIONS)
        compare(ys[i], y0s[i], want, owner, "bf16")
