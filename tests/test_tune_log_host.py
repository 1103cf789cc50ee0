"""The log tells which rows of a tuning file select the transform (CPU).

A geometry other than the default makes its length compute with the
number-theoretic transform, also where an untuned call computes over GF(2).
Rows without an architecture name apply everywhere, so no GPU is needed.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
L = 1_572_864


def lines(tmp_path, rows, how):
    path = str(tmp_path / "rows.txt")
    with open(path, "w") as f:
        f.write("".join(r + "\n" for r in rows))
    env = dict(os.environ, PYTHONPATH=ROOT, PA_LOG="info")
    env.pop("PA_TUNE_CACHE", None)
    code = "import paper_1809_07592_amd as pa\n"
    if how == "cache":
        env["PA_TUNE_CACHE"] = path
        code += "pa.tune_get(%d, 0)\n" % L
    else:
        code += "pa.tune_load(%r)\n" % path
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    return [ln for ln in r.stderr.splitlines() if "tuning cache" in ln]


@pytest.mark.parametrize("how", ["cache", "load"])
def test_rows_that_select_the_transform_are_counted(tmp_path, how):
    # two rows that differ from the default (one in the row workgroup size
    # only), one default row, one length beyond the split form
    got = lines(tmp_path, ["%d 0 7 16" % L, "%d 1 0 0 0 512" % L, "%d 0 0 0" % (2 * L), "28311552 1 0 0 0 512"], how)
    assert any("4 of 4 rows" in ln for ln in got), got
    assert any("2 rows select the transform" in ln for ln in got), got


@pytest.mark.parametrize("how", ["cache", "load"])
def test_default_rows_say_nothing(tmp_path, how):
    got = lines(tmp_path, ["%d 0 0 0" % L], how)
    assert len(got) == 1 and "1 of 1 rows" in got[0], got
