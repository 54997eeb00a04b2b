"""Where the lines of the dispatch lie that choose between kernels whose sums of z are grouped differently: such a choice is the same with and without room
for z, so it is made only where neither side of it is the slower one.  Asked from the sources' own rules on the host."""
import shutil

import pytest

from test_host_rules import ask

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def small(tmp_path_factory, cases):
    """Whether the small-batch kernel takes LoRA calls (T, S, N, all positions, rank, d_in, d_out)."""
    return [line.split()[0] == "1" for line in ask(tmp_path_factory, [" ".join(map(str, c)) + " 0 0" for c in (("small",) + c for c in cases)])]


@pytest.mark.parametrize("rank", [20, 32, 36, 64, 68, 128])
def test_calls_above_1024_rows_that_stay_with_the_kernels_of_larger_batches(tmp_path_factory, rank):
    decode = [(T, T, N, 1, rank, d, n) for T in (1025, 2000, 4096) for N in (1, 64, 500) for d, n in ((4096, 4096), (1000, 4096), (8192, 512), (512, 14336))]
    long = [(T, 20, 64, 0, rank, d, n) for T in (6145, 20000, 200000) for d, n in ((4096, 4096), (1000, 4096), (4096, 520), (1000, 12296))]
    assert not any(small(tmp_path_factory, decode + long))
    if rank > 32:
        short = [(2000, 101, 64, 0, rank, 1024, 4096), (2000, 300, 300, 0, rank, 1000, 2072)]
        ragged = [(1600, 4, 64, 0, rank, 1000, 4104), (1600, 4, 64, 0, rank, 1000, 12296), (2000, 4, 64, 0, rank, 4096, 264), (4097, 4, 64, 0, rank, 1000, 4096)]
        assert not any(small(tmp_path_factory, short + ragged))
    # and those that the small-batch kernel keeps
    assert all(small(tmp_path_factory, [(T, 4, 64, 0, rank, d, n) for T in (1025, 2000) for d, n in ((4096, 4096), (512, 14336), (1000, 2072))]))
