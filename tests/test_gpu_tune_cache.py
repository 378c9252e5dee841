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
REFUSED, KEPT, OLD, FLAT = (104, 64, 40), (112, 64, 40), (120, 64, 40), (96, 1, 80)
FORMS = ("fused", "graph", "persistent")


def _key(n, exec_):
    """The key of a grid of n, 8 chares (FLAT: one), fp64, the 3D stencil, hints bit 0."""
    kw = dict(n=n, odf=1 if n == FLAT else 8, dtype="f64", exec=exec_, hints=1)
    cfg, _keep = od.make_config(**kw)
    boxes = len(od.host_plan(**kw)["pass"]["boxes"])
    chare = "x".join(str(v if n == FLAT else v // 2) for v in n)
    # (message-driven grids tune the scheduler at the planned tile, here of pairs)
    tile = "/t" + "x".join(map(str, od.host_plan(**kw)["tile"])) + "/p2" if exec_ == "msgdriven" else ""
    return (f"v2/s8/k7/e{cfg.exec}/n{n[0]}x{n[1]}x{n[2]}/b4x{boxes}/{chare}:{1 if n == FLAT else 8}{tile}/h0/i0x0",
            cfg.exec, chare)


def _grid(n, exec_):
    return od.Grid(n, odf=8, dtype="f64", exec=exec_, hints=1, seed=3)


def _check(g, n, iters):
    want, _, r = oracle.solve(n, np.float64, seed=3, iters=iters)
    assert g.iterations() == iters and g.residual() == r
    assert np.array_equal(g.read(), want)


def _in_file(key):
    with open(os.environ["OD_TUNE_CACHE"]) as f:
        return any(ln.startswith(key) for ln in f)


def _write_entries():
    rows = []
    for e in FORMS:
        sched = NO_BOXES | (1 if e == "persistent" else 0)
        rows.append(f"{_key(REFUSED, e)[0]} 7 7 7 {sched} 0")   # no such tile
        rows.append(f"{_key(KEPT, e)[0]} 32 16 8 {sched} 0")
        _, num, chare = _key(OLD, e)   # as files had it before boxes were part of the key
        rows.append(f"s8/e{num}/n{'x'.join(map(str, OLD))}/{chare}:8/h0/i0x0 32 16 8 {sched} 0")
    rows.append(f"{_key(KEPT, 'msgdriven')[0]} 0 0 0 {NO_BOXES | 1 | 2 << 2} 0")   # cursor, no publisher
    rows.append(f"{_key(FLAT, 'fused')[0]} 256 1 32 {NO_BOXES} 0")
    _, num, chare = _key(FLAT, "fused")
    rows.append(f"s8/e{num}/n{chare}/{chare}:1/h0/i0x0 256 1 32 {NO_BOXES} 0")
    fd, path = tempfile.mkstemp(prefix="od_tune_")
    with os.fdopen(fd, "w") as f:
        f.write("\n".join(rows) + "\n")
    os.environ["OD_TUNE_CACHE"] = path
    atexit.register(os.unlink, path)


if "OD_TUNE_CACHE" not in os.environ:
    try:
        _write_entries()
    except ImportError:   # nothing is built: no test here can run either
        pass


@pytest.mark.parametrize("exec_", FORMS)
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


@pytest.mark.parametrize("exec_", FORMS + ("msgdriven",))
def test_an_entry_without_boxes_runs_the_tile(exec_):
    g = _grid(KEPT, exec_)
    try:
        g.iterate(5)
        tile = (32, 16, 8) if exec_ != "msgdriven" else tuple(g.plan()["tile"])
        assert g.autotune(1) == tile and g.plan()["schedule"] == {"persistent": 1, "msgdriven": 9}.get(exec_, 0)
        assert g.pass_info()["steps"] == 2 and len(g.pass_info()["boxes"]) == 0
        g.iterate(4)
        g.iterate(3)
        _check(g, KEPT, 12)
    finally:
        g.close()


@pytest.mark.parametrize("exec_", FORMS)
def test_an_entry_from_before_the_boxes_is_not_taken(exec_):
    # it knows nothing of the boxes: the grid is tuned, and the file has it
    g = _grid(OLD, exec_)
    try:
        g.autotune(1)
        assert _in_file(_key(OLD, exec_)[0])
        g.iterate(9)
        _check(g, OLD, 9)
    finally:
        g.close()


def test_an_entry_of_the_other_stencil_is_not_taken():
    n = (FLAT[0], FLAT[2])
    g = od.Grid2D(n, odf=1, dtype="f64", exec="fused", hints=1, seed=3)
    try:
        g.autotune(1)
        assert _in_file(_key(FLAT, "fused")[0].split("/b")[0].replace("/k7", "/k5"))   # tuned, as the 2D stencil's
        g.iterate(9)
        want, _, r = oracle.solve2d(n, np.float64, 3, 9, (1.0, 0.0, 0.0, 0.0))
        assert np.array_equal(g.read(), want) and g.residual() == r
    finally:
        g.close()


def test_the_tuner_takes_the_planned_tile_or_boxes_on_a_thin_grid():
    n = (1, 2000, 600)
    g = od.Grid(n, odf=1, dtype="f32", exec="fused", hints=1, seed=3)
    try:
        assert g.pass_info()["steps"] == 2
        planned = tuple(g.plan()["tile"])
        g.iterate(3)
        tile = g.autotune(2)
        # the planned tile, pairs by which are the quickest, is among the candidates
        assert g.pass_info()["steps"] == 4 or tile == planned
        g.iterate(9)
        want, _, r = oracle.solve(n, np.float32, seed=3, iters=12)
        assert np.array_equal(g.read(), want) and g.residual() == r
    finally:
        g.close()
