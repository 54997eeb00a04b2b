"""Where lines of the dispatch lie, asked from the sources' own rules on the host.  Those that choose between kernels whose sums of z are grouped differently choose
the same with and without room for z, so they do it only where neither side is the slower one."""
import os
import shutil
import subprocess

import pytest

from test_host_rules import ROOT, ask

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


ANSWERS = ("small", "two", "stay", "in_place_small", "in_place_two", "h_stays", "keeps_units", "ids")
_exe = {}


def lines(tmp_path_factory, cases):
    """The driver's answers for calls (T, S, N, all positions, rank, d_in, columns of the output, bytes of an element)."""
    if "exe" not in _exe:
        exe = tmp_path_factory.mktemp("dispatch_lines") / "driver"
        build = subprocess.run(["hipcc", "--cuda-host-only", "-std=c++17", os.path.join(ROOT, "tests", "dispatch_lines_driver.hip"), "-o", str(exe)], capture_output=True, text=True)
        assert build.returncode == 0, build.stderr
        _exe["exe"] = exe
    run = subprocess.run([str(_exe["exe"])], input="".join(" ".join(map(str, c)) + "\n" for c in cases), capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    out = [dict(zip(ANSWERS, (v == "1" for v in line.split()))) for line in run.stdout.splitlines()]
    assert len(out) == len(cases)
    return out


def test_the_second_launch_of_few_tiles_has_a_shrink_to_save(tmp_path_factory):
    one = [(3000, 8, 64, 0, rank, d, n, 2) for rank, d, n in ((20, 512, 112), (32, 4096, 4096), (40, 360, 1088), (48, 1848, 512), (60, 1024, 232), (56, 256, 2048), (68, 768, 128), (128, 4096, 512))]
    one += [(725, 725, 32, 1, 56, 8192, 9536, 2), (960, 960, 4, 1, 56, 384, 14336, 2), (234, 234, 200, 1, 64, 1416, 1952, 2), (900, 900, 500, 1, 96, 4096, 1024, 2)]
    assert not any(a["two"] for a in lines(tmp_path_factory, one))
    two = [(3000, 8, 64, 0, rank, d, n, 2) for rank, d, n in ((20, 4096, 8192), (48, 1024, 4096), (64, 4096, 1536), (68, 1024, 1024), (128, 512, 4096))] + [(900, 5, 5, 0, 64, 4096, 4096, 2), (512, 512, 64, 1, 96, 4096, 1024, 2)]
    assert all(a["two"] for a in lines(tmp_path_factory, two))
    in_place = lines(tmp_path_factory, [(180, 24, 64, 1, 68, 104, 104, 2), (362, 362, 32, 1, 68, 384, 384, 2), (286, 3, 4, 0, 128, 144, 144, 2), (300, 2, 5, 0, 128, 512, 512, 2), (300, 2, 5, 0, 96, 4096, 4096, 2), (426, 426, 200, 1, 96, 2880, 2880, 2)])
    assert [a["in_place_two"] for a in in_place] == [False, False, False, True, True, False]


def test_tiles_of_an_expand_launch_are_counted_as_they_are_numbered(tmp_path_factory):
    """64 rows a tile above rank 32, in panels of 256 columns where the width allows it and the rank is at most 64, else of 128; fewer than 2^31 ids."""
    T, S = 64 * 8192, 1
    got = lines(tmp_path_factory, [(T, S, 1, 0, rank, 4096, n, 2) for rank in (64, 68, 128) for n in (1 << 24, 1 << 25, 1 << 26)])
    assert [a["ids"] for a in got] == [True, True, False, True, False, False, True, False, False]


def test_units_stay_in_registers_where_the_tiles_are_full(tmp_path_factory):
    """In place, rank 20-32: not for segments that leave the 32-row tiles part-empty, prompts or decode rows."""
    short = [(2510, 239, 200, 0, 20, 8320, 8320, 2), (2588, 225, 32, 0, 28, 14336, 14336, 2), (6305, 130, 200, 0, 24, 8320, 8320, 2), (1613, 25, 64, 0, 20, 14336, 14336, 2), (900, 900, 4, 1, 32, 9216, 9216, 2)]
    assert not any(a["keeps_units"] for a in lines(tmp_path_factory, short + [(18000, 30, 64, 0, 32, 9208, 9208, 2), (7700, 14, 64, 0, 24, 9216, 9216, 2)]))
    assert all(a["keeps_units"] for a in lines(tmp_path_factory, [(18000, 30, 64, 0, 32, 10240, 10240, 2), (12000, 120, 64, 0, 20, 14336, 14336, 2)]))


def test_what_is_read_without_the_non_temporal_hint(tmp_path_factory):
    """Activations between the L2s together and a quarter (fp32: a third) of the memory-side cache, the factors of many adapters counted; in place 20 to 64 MB of h."""
    lora = [(2300, 4, 4, 0, 16, 4096, 4096, 4), (2600, 4, 4, 0, 16, 4096, 4096, 4), (3000, 4, 4, 0, 32, 4096, 4096, 2), (4400, 4, 4, 0, 32, 4096, 4096, 2), (1900, 4, 4, 0, 32, 4096, 4096, 2),
            (3000, 3000, 512, 1, 44, 4096, 4096, 2)]
    assert [a["stay"] for a in lines(tmp_path_factory, lora)] == [True, False, True, False, False, False]
    h = [(1200, 4, 4, 0, 64, 8192, 8192, 2), (1300, 4, 4, 0, 64, 8192, 8192, 2), (4000, 4, 4, 0, 64, 8192, 8192, 2), (4200, 4, 4, 0, 64, 8192, 8192, 2)]
    assert [a["h_stays"] for a in lines(tmp_path_factory, h)] == [False, True, True, False]


def test_ranks_1_to_3_that_stay_with_the_vector_alu(tmp_path_factory):
    """Next to nothing to expand, in place narrow rows, or tiles enough to fill the chip with the layers of one call."""
    lora = [(41, 34, 32, 0, 1, 8192, 512, 2), (850, 2, 1, 0, 1, 7040, 512, 2), (8, 1, 64, 0, 2, 9016, 1024, 2), (2000, 2000, 500, 1, 1, 4096, 512, 2), (1300, 38, 64, 1, 1, 1024, 1024, 2),
            (585, 130, 512, 0, 1, 512, 1024, 2), (41, 34, 32, 0, 1, 4096, 4096, 2), (41, 34, 32, 0, 3, 8192, 512, 2)]
    assert [a["small"] for a in lines(tmp_path_factory, lora)] == [False] * 6 + [True] * 2
    h = [(81, 74, 512, 1, 2, 896, 896, 2), (304, 57, 200, 1, 2, 3456, 3456, 2), (105, 14, 512, 0, 3, 128, 128, 2), (32, 32, 8, 1, 2, 896, 896, 2), (100, 2, 8, 0, 3, 1024, 1024, 2)]
    assert [a["in_place_small"] for a in lines(tmp_path_factory, h)] == [False, False, False, True, True]


def test_ranks_4_to_16_above_1024_rows_that_stay_with_the_kernels_of_larger_batches(tmp_path_factory):
    """Narrow inputs and outputs, and wide inputs with wide outputs."""
    no = [(3500, 2, 4, 0, 16, 768, 1296, 2), (2000, 106, 4, 0, 12, 2304, 1024, 2), (2800, 7, 32, 0, 8, 2048, 2048, 2), (2800, 7, 32, 0, 12, 8192, 6144, 2), (6000, 5, 64, 0, 16, 4096, 3256, 2)]
    yes = [(4000, 10, 32, 0, 8, 2048, 2048, 2), (2800, 7, 32, 0, 9, 2048, 2048, 2), (2800, 7, 32, 0, 12, 8192, 4096, 2), (2400, 7, 32, 0, 4, 4096, 8448, 2)]
    assert [a["small"] for a in lines(tmp_path_factory, no + yes)] == [False] * 5 + [True] * 4
