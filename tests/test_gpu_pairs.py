"""Pairs of steps on grids that by default run passes over boxes: hints bit 14
keeps them to pairs, under every form, schedule, remainder and load imbalance,
also after tuning.  Compared with the CPU oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2605_12734_amd as od
import workloads

pytestmark = pytest.mark.gpu

DT = {"f64": np.float64, "f32": np.float32}
BC6 = (1.0, 0.5, 0.25, 0.125, 2.0, 3.0)
PAIRS = 1 | 1 << 14


def _run(n, odf, dtype, iters, exec_, tune=False, schedule=None, **kw):
    want, _, r_want = oracle.solve(n, DT[dtype], seed=5, iters=sum(iters), bc=BC6)
    g = od.Grid(n, odf=odf, dtype=dtype, exec=exec_, bc=BC6, seed=5, hints=PAIRS, **kw)
    try:
        assert g.pass_info()["steps"] == 2 and g.plan()["steps_per_pass"] == 2
        assert schedule is None or g.plan()["schedule"] == schedule
        for i, k in enumerate(iters):
            g.iterate(k)
            if tune and i == 0:
                g.autotune(1)
        U, r, it = g.read(), g.residual(), g.iterations()
    finally:
        g.close()
    assert np.array_equal(U, want), int((U != want).sum())
    assert r == r_want and it == sum(iters)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("iters", [[1], [2], [5], [12], [4, 3, 4]])
@pytest.mark.parametrize("exec_,schedule", [("fused", 0), ("graph", 0), ("persistent", 2), ("msgdriven", 0)])
def test_64cubed(dtype, iters, exec_, schedule):
    _run(64, 8, dtype, iters, exec_, schedule=schedule)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("exec_", ["fused", "graph", "persistent", "msgdriven"])
@pytest.mark.parametrize("n,odf", [((150, 90, 70), 27), ((37, 21, 19), 8), ((9, 8, 7), 27), ((40, 3, 33), 8)])
def test_ragged(dtype, exec_, n, odf):
    _run(n, odf, dtype, [7, 4], exec_)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("exec_", ["fused", "persistent", "msgdriven"])
def test_under_imbalance(dtype, exec_):
    _run((70, 45, 38), 27, dtype, [9, 4], exec_, imbalance_pct=50, imbalance_max_extra=3)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("exec_", ["fused", "graph", "persistent", "msgdriven"])
def test_uneven_blocks(dtype, exec_):
    blocks = workloads.octree_blocks(n=96, root=32, min_edge=8, p_refine=0.5, seed=7)
    _run(96, 1, dtype, [9, 4], exec_, blocks=blocks)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("iters", [[4, 9], [5, 8], [6, 7]])
def test_tuned_persistent(dtype, iters):
    # the tuned tile, schedule and waves cap are what the compared part runs
    # (a size of its own for each: tuned sizes are kept in the process)
    n = (150, 90, 60 + 4 * iters[0])
    want, _, r_want = oracle.solve(n, DT[dtype], seed=5, iters=13, bc=BC6)
    g = od.Grid(n, odf=27, dtype=dtype, exec="persistent", bc=BC6, seed=5, hints=PAIRS)
    try:
        g.iterate(iters[0])
        g.autotune(1)
        assert g.plan()["schedule"] in (1, 2, 3, 4) and g.pass_info()["steps"] <= 2
        g.iterate(iters[1])
        assert np.array_equal(g.read(), want) and g.residual() == r_want
    finally:
        g.close()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_tuned_message_driven(dtype):
    _run((96, 80, 56), 64, dtype, [5, 8], "msgdriven", tune=True)
