"""Tuning results kept in a file (OD_TUNE_CACHE): what a grid does with entries
it can take and with entries it cannot.  The library reads the file at the
process's first od_autotune, so the entries are written here when the tests are
collected; each is of a grid size that no other test tunes."""
import atexit
import os
import tempfile

import numpy as np
import pytest

import oracle
import paper_2605_12734_amd as od

pytestmark = pytest.mark.gpu

NO_BOXES = 16   # in the schedule column: tiles were quicker than passes over boxes
REFUSED = (104, 64, 40)


def _key(n, exec_):
    """The key of a grid of n, 8 chares, fp64, hints bit 0."""
    cfg, _keep = od.make_config(n=n, odf=8, dtype="f64", exec=exec_, hints=1)
    half = "x".join(str(v // 2) for v in n)
    return f"s8/e{cfg.exec}/n{n[0]}x{n[1]}x{n[2]}/{half}:8/h0/i0x0"


def _grid(n, exec_):
    return od.Grid(n, odf=8, dtype="f64", exec=exec_, hints=1, seed=3)


def _check(g, n, iters):
    want, _, r = oracle.solve(n, np.float64, seed=3, iters=iters)
    assert g.iterations() == iters and g.residual() == r
    assert np.array_equal(g.read(), want)


if "OD_TUNE_CACHE" not in os.environ:
    _fd, _path = tempfile.mkstemp(prefix="od_tune_")
    with os.fdopen(_fd, "w") as _f:
        for _e in ("fused", "graph", "persistent"):
            _f.write(f"{_key(REFUSED, _e)} 7 7 7 {NO_BOXES | (1 if _e == 'persistent' else 0)} 0\n")   # no such tile
    os.environ["OD_TUNE_CACHE"] = _path
    atexit.register(os.unlink, _path)


@pytest.mark.parametrize("exec_", ["fused", "graph", "persistent"])
def test_an_entry_that_cannot_be_applied_changes_nothing(exec_):
    g = _grid(REFUSED, exec_)
    try:
        before = g.plan()
        g.iterate(4)
        g.iterate(4)   # (a graph for either parity)
        with pytest.raises(Exception, match="compiled variant"):
            g.autotune(1)
        assert g.pass_info()["steps"] == 4 and g.plan() == before
        g.iterate(4)
        g.iterate(3)
        _check(g, REFUSED, 15)
    finally:
        g.close()
