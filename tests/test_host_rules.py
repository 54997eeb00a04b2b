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
