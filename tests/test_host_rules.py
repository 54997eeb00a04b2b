"""Layout and offset rules that the kernels share with their launches, asked from the sources' own functions on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
_exe = {}


def ask(tmp_path_factory, lines):
    """The driver's answers, one per line."""
    if "exe" not in _exe:
        exe = tmp_path_factory.mktemp("host_rules") / "driver"
        build = subprocess.run(["hipcc", "--cuda-host-only", "-std=c++17", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host",
                                "-fno-sanitize-recover=all", os.path.join(ROOT, "tests", "host_rules_driver.hip"), "-o", str(exe)],
                               capture_output=True, text=True)
        assert build.returncode == 0, build.stderr
        _exe["exe"] = exe
    run = subprocess.run([str(_exe["exe"])], input="\n".join(lines) + "\n", capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    return run.stdout.split("\n")[:-1]


def test_last_factor_piece_of_any_width_fits_32_bits(tmp_path_factory):
    """The last 16-byte piece a wavefront may read of a [d_out, rank] factor, from column c on: never past the matrix,
    never negative, whatever the width (2^25 columns at rank 64 are 2^31 values)."""
    cases = [(left, most, rank) for left in (8, 16, 24, 120, 128, 136, 4096, 1 << 22, 1 << 25, (1 << 28) + 8, (1 << 31) - 8)
             for most in (32, 128) for rank in (1, 3, 7, 15, 17, 36, 63, 64)]
    for (left, most, rank), got in zip(cases, ask(tmp_path_factory, [f"piece {l} {m} {r}" for l, m, r in cases])):
        assert int(got) == min(left, most) * rank // 8 - 1 >= 0


def test_the_column_split_kernel_takes_only_what_its_offsets_reach(tmp_path_factory):
    """Its lanes hold byte offsets from a factor's start in a signed 32-bit register, at most ((rank - 1) d_in + 120) * 2 (mfma_tile_body:
    the last rank's row, a lane's 16-byte piece of a 128-column unit).  Whatever sends a call to it must leave that below 2^31:
    chunks of ranks up to 16, of widths that are no multiple of 128 and, in place, of ranks up to 32."""
    widths = sorted({w for at in (1 << 20, 1 << 22, 8523264, 17301504, 35791488, 71583104, 1 << 28, (1 << 30) - 256) for w in range(at - 256, at + 257, 8)}
                    | {(1 << 31) - 8, (1 << 31) - 128})
    cases = [(T, rank, d, d_out, direft) for rank in (4, 5, 15, 16, 17, 20, 31, 32, 33, 63, 64, 65, 127, 128) for d in widths
             for T in (8, 2000, 400000) for d_out, direft in ((128, 0), (d, 1))]
    reached = set()
    for (T, rank, d, d_out, direft), got in zip(cases, ask(tmp_path_factory, [f"route {T} {1 + T // 600} {r} {d} {o} {i}" for T, r, d, o, i in cases])):
        takes, streams, fits = (int(v) for v in got.split())
        assert fits == (((rank - 1) * d + 120) * 2 < (1 << 31) - 15)         # 16 bytes from there on
        whole_units = d % 128 == 0 and d_out % 128 == 0
        columns = rank <= 16 or not whole_units or (rank % 4 != 0 and streams)
        assert not (takes and columns) or fits, (T, rank, d)
        assert takes == (fits and (rank <= 16 or rank % 4 == 0 or d <= 1 << 22) or (rank > 16 and whole_units)), (T, rank, d)
        reached.add((takes, columns, fits))
    assert reached == {(1, True, 1), (1, False, 1), (1, False, 0), (0, True, 0), (0, True, 1)}
