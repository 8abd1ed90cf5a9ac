"""Which levels' Gauss-Seidel sweeps run in one launch: the library's own
headers, compiled for the host and asked at the edges of their rules."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_01287_amd", "csrc")
HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")


def ask(tmp_path, expressions):
    """The values of C++ expressions over a SweepData `q` (usable but for what
    the expression sets)."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    lines = "\n".join(f'    {{ SweepData q; q.ncolors = 14; q.apart = true; q.places = 1000; printf("%d\\n", int({e})); }}'
                      for e in expressions)
    src.write_text('#include <cstdio>\n#include "context.h"\nusing namespace amgp2;\nint main() {\n' + lines + "\n}\n")
    subprocess.check_call([HIPCC, "-std=c++17", "-w", "-x", "hip", "--offload-host-only", "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, str(src), "-o", str(exe)])
    return [int(v) for v in subprocess.check_output([str(exe)], text=True).split()]


def test_usable(tmp_path):
    """The colours' tables in LDS; one half of the swept values (32 bytes a
    place, 8 for a scalar vector) below 2 GiB, at 2^26 and 2^28 places."""
    cases = {"q.usable()": 1, "(q.apart = false, q.usable())": 0,
             "(q.ncolors = 0, q.usable())": 0, "(q.ncolors = 1023, q.usable())": 1, "(q.ncolors = 1024, q.usable())": 0,
             "(q.places = (1 << 26) - 1, q.usable())": 1, "(q.places = 1 << 26, q.usable())": 0,
             "(q.places = 1 << 27, q.usable())": 0, "(q.places = (1ll << 31) - 1, q.usable())": 0,
             "(q.stride = 1, q.places = (1 << 28) - 1, q.usable())": 1,
             "(q.stride = 1, q.places = 1 << 28, q.usable())": 0}
    assert ask(tmp_path, cases) == list(cases.values())


def test_large_colours_take_a_launch_each(tmp_path):
    """Both sides of every line, by entries a colour (finest levels: rows of 28
    entries, 14 colours; coarse ones: 70 and 30)."""
    def rule(mode, fp64, row, colours, entries, pre, post):
        nnz = int(entries * 1e3) * colours
        return f"sweep_by_colour({mode}, {fp64}, {nnz}ll, {nnz // row}, {colours}, {pre}, {post})"

    cases = {}
    for mode, fp64, row, colours, pre, post, below, above in (
            ("SWEEP_BLOCK", "true", 28, 14, 1, 1, 361, 538), ("SWEEP_BLOCK", "true", 28, 14, 2, 2, 309, 361),
            ("SWEEP_BLOCK", "true", 28, 14, 0, 1, 309, 361), ("SWEEP_BLOCK", "false", 28, 14, 1, 1, 1218, 1400),
            ("SWEEP_BLOCK", "false", 28, 14, 2, 2, 361, 538), ("SWEEP_BLOCK", "false", 70, 30, 1, 1, 1052, 1400),
            ("SWEEP_SCALAR3", "true", 28, 14, 1, 1, 901, 1051), ("SWEEP_SCALAR3", "true", 70, 30, 2, 2, 476, 711),
            ("SWEEP_SCALAR3", "false", 28, 14, 1, 1, 1817, 2310), ("SWEEP_SCALAR3", "false", 28, 14, 2, 2, 1399, 1817),
            ("SWEEP_SCALAR3", "false", 70, 30, 1, 1, 476, 711)):
        cases[rule(mode, fp64, row, colours, below, pre, post)] = 0
        cases[rule(mode, fp64, row, colours, above, pre, post)] = 1
    cases["sweep_by_colour(SWEEP_BLOCK, true, 0, 0, 0, 1, 1)"] = 0
    assert ask(tmp_path, cases) == list(cases.values())
