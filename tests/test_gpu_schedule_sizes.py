"""The scheduler at the sizes where its workgroup changes: one wavefront for 64 segments or 256 adapters, more above, one or several segments
per thread, chunks written by a lane (up to 16 of a segment) or by the wavefront.  Every list against a plain restatement."""
import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,N", [(1, 1), (63, 3), (64, 256), (65, 257), (128, 4096), (129, 4097), (700, 40), (1024, 64), (1025, 64), (2100, 5)])
@pytest.mark.parametrize("all_tokens", [False, True])
def test_lists(S, N, all_tokens):
    from parity_util import dev_tables
    rng = np.random.Generator(np.random.PCG64(S + N))
    lens = rng.choice([0, 1, 1, 2, 4, 5, 127, 128, 129, 2048, 2049], size=S, p=[.05, .3, .2, .1, .1, .1, .05, .04, .03, .02, .01])
    lens[0] = 2049
    ids = rng.integers(-1, N + 1, size=S)
    ids[0] = 0
    tab = wl.from_lengths(lens, ids, np.where(rng.random(S) < 0.5, lens, lens // 2))
    n = np.where((ids >= 0) & (ids < N), lens if all_tokens else np.minimum(tab.seg_prefill_len, lens), 0)
    ss, sa, sp = dev_tables(tab)
    ws = preft.new_workspace(tab.T, S)
    ws.fill_(0xab)
    preft.preft_schedule(ws, ss, sa, sp, tab.T, N, preft.PREFT_ALL_TOKENS if all_tokens else preft.PREFT_PREFILL_ONLY)
    head = ws[:64].view(torch.int32).cpu().numpy()
    chunks = [[ids[s], tab.seg_start[s] + c, min(128, n[s] - c), s] for s in range(S) if n[s] > 4 for c in range(0, n[s], 128)]
    rows = sorted((ids[s], tab.seg_start[s] + j) for s in range(S) if n[s] <= 4 for j in range(n[s]))
    assert list(head[:4]) == [len(chunks), len(rows), n.sum(), int(all_tokens)] and list(head[5:8]) == [tab.T, S, N]
    g0 = 64 + 16 * (tab.T // 128 + min(S, tab.T // 5) + 1)
    s0 = g0 + 16 * (min(4 * S, tab.T) + 1)
    assert ws[64:64 + 16 * len(chunks)].view(torch.int32).view(-1, 4).cpu().tolist() == [[int(v) for v in c] for c in chunks]
    shorts = ws[s0:s0 + 8 * len(rows)].view(torch.int32).view(-1, 2).cpu().numpy()
    assert sorted(map(tuple, shorts.tolist())) == [(int(a), int(r)) for a, r in rows]
    tiles = ws[g0:g0 + 16 * head[4]].view(torch.int32).view(-1, 4).cpu().numpy()
    seen = np.zeros(len(rows), dtype=int)
    for a, first, count, _ in tiles:
        assert 1 <= count <= 16 and np.all(shorts[first:first + count, 0] == a)
        seen[first:first + count] += 1
    assert np.all(seen == 1)
    if N <= 4096:
        owners, per = np.unique([a for a, _ in rows], return_counts=True) if rows else ([], np.zeros(0, dtype=int))
        assert len(tiles) == int(np.sum((per + 15) // 16))
