"""Tuning results kept in a file (OD_TUNE_CACHE): what a grid does with entries
it can take and with entries it cannot.  The file is read once per process, so
each step is a process of its own; the entries under test are those a first
process wrote, changed here."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NO_BOXES = 16   # in the schedule column: tiles were quicker than passes over boxes
HEAD = """
import numpy as np
import oracle
import paper_2605_12734_amd as od
N = (96, 64, 40)
def grid(exec_, **kw):
    return od.Grid(N, odf=8, dtype="f64", exec=exec_, hints=1, seed=3, **kw)
def check(g, iters):
    want, _, r = oracle.solve(N, np.float64, seed=3, iters=iters)
    assert g.iterations() == iters and g.residual() == r
    assert np.array_equal(g.read(), want)
"""


def _child(cache, body):
    p = subprocess.run([sys.executable, "-c", HEAD + body], cwd=ROOT, timeout=100, capture_output=True, text=True,
                       env=dict(os.environ, OD_TUNE_CACHE=str(cache)))
    assert p.returncode == 0, p.stdout + p.stderr


def _entries(cache, execs):
    """One entry for each form, as a process that tunes writes them."""
    _child(cache, f"""
for e in {execs!r}:
    g = grid(e)
    g.autotune(1)
    g.close()
""")
    rows = [ln.split() for ln in cache.read_text().splitlines()]
    assert len(rows) == len(execs)
    return rows


def test_an_entry_that_cannot_be_applied_changes_nothing(tmp_path):
    cache = tmp_path / "tune"
    rows = _entries(cache, ["fused", "graph", "persistent"])
    for r in rows:
        r[1:4] = ["7", "7", "7"]   # not a compiled tile
        r[4] = str(int(r[4]) | NO_BOXES)
    cache.write_text("".join(" ".join(r) + "\n" for r in rows))
    _child(cache, """
for e in ("fused", "graph", "persistent"):
    g = grid(e)
    before = g.plan()
    g.iterate(4)
    g.iterate(4)   # (a graph for either parity)
    try:
        g.autotune(1)
    except Exception as ex:
        assert "compiled variant" in str(ex), ex
    else:
        raise AssertionError("a tile that is not compiled was taken")
    assert g.pass_info()["steps"] == 4 and g.plan() == before
    g.iterate(4)
    g.iterate(3)
    check(g, 15)
    g.close()
""")
