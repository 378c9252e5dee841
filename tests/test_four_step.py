"""Four Jacobi steps per pass: the boxes of a pass (host) and its bits (GPU).

The pass cuts the whole grid into boxes of 64 x 64 lanes that cross chares;
each computes a ring of four cells more than it writes, except at the grid's
faces.  Everything is compared with the CPU oracle bit for bit."""
import time

import numpy as np
import pytest

import oracle
import paper_2605_12734_amd as od
import workloads

DT = {"f64": np.float64, "f32": np.float32}
BC6 = (1.0, 0.5, 0.25, 0.125, 2.0, 3.0)
RING = 4


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,odf", [((1, 1, 1), 1), ((2, 3, 4), 8), ((9, 8, 7), 27), ((63, 15, 5), 1), ((64, 16, 1), 1),
                                   ((65, 17, 3), 1), ((64, 65, 2), 1), ((120, 120, 3), 1), ((124, 121, 4), 1),
                                   ((176, 177, 5), 1), ((180, 119, 16), 27), ((211, 163, 57), 27), ((300, 500, 7), 8),
                                   ((512, 512, 40), 64), ((1000, 66, 1), 1), ((130, 40, 6), 125)])
def test_boxes_write_each_cell_once_and_keep_their_ring(dtype, n, odf):
    p = od.host_plan(n=n, odf=odf, dtype=dtype, exec="graph")["pass"]
    assert p["steps"] == 4 and p["bytes"] == (8 if dtype == "f32" else 16) * n[0] * n[1] * n[2]
    seen = np.zeros((n[2], n[1], n[0]), dtype=np.int8)
    for cx0, cx1, cy0, cy1, x0, x1, y0, y1, z0, z1 in p["boxes"]:
        # the lanes stay in the grid, and no written cell is within the ring's
        # reach of the cells computed from nothing
        assert 0 <= cx0 <= x0 < x1 <= cx1 <= n[0] and 0 <= cy0 <= y0 < y1 <= cy1 <= n[1] and 0 <= z0 < z1 <= n[2]
        assert cx0 == 0 or x0 - cx0 >= RING
        assert cy0 == 0 or y0 - cy0 >= RING
        assert cx1 == n[0] or cx1 - x1 >= RING
        assert cy1 == n[1] or cy1 - y1 >= RING
        seen[z0:z1, y0:y1, x0:x1] += 1
    assert (seen == 1).all()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [(300, 300, 4), (250, 250, 12), (100, 100, 30), (64, 64, 64), (225, 391, 6)])
def test_boxes_of_message_driven_tasks(dtype, n):
    # a task costs more than its planes: fewer boxes of more planes where a pass
    # launched by itself takes as many as the chip holds; each cell once as ever
    one = od.host_plan(n=n, odf=1, dtype=dtype, exec="fused")["pass"]
    p = od.host_plan(n=n, odf=1, dtype=dtype, exec="msgdriven")["pass"]
    assert p["steps"] == 4 and len(p["boxes"]) <= len(one["boxes"])
    assert dtype == "f64" or len(p["boxes"]) <= 512 < len(one["boxes"]) or n == (64, 64, 64)
    seen = np.zeros((n[2], n[1], n[0]), dtype=np.int8)
    for cx0, cx1, cy0, cy1, x0, x1, y0, y1, z0, z1 in p["boxes"]:
        assert (cx0 == 0 or x0 - cx0 >= RING) and (cx1 == n[0] or cx1 - x1 >= RING)
        assert (cy0 == 0 or y0 - cy0 >= RING) and (cy1 == n[1] or cy1 - y1 >= RING)
        seen[z0:z1, y0:y1, x0:x1] += 1
    assert (seen == 1).all()


@pytest.mark.parametrize("kw,steps", [
    (dict(n=64), 4), (dict(n=(5, 3, 2), odf=1), 4), (dict(n=(65, 64, 8)), 4), (dict(n=(66, 64, 64), dtype="f32"), 4),
    (dict(n=64, exec="fused"), 4), (dict(n=64, exec="persistent"), 4), (dict(n=64, exec="msgdriven"), 4),
    (dict(n=64, exec="per_chare"), 1),
    (dict(n=64, exec="persistent", hints=1 << 4), 2),          # a schedule of tiles
    (dict(n=64, exec="persistent", hints=1 << 3), 1),          # the timeline is one of single steps
    (dict(n=64, exec="persistent", imbalance_pct=10, imbalance_max_extra=4), 2),
    (dict(n=64, exec="fused", imbalance_pct=10, imbalance_max_extra=4), 4),
    (dict(n=64, hints=1 << 14), 2), (dict(n=64, hints=1 << 12), 1),
    (dict(n=64, tile=(32, 16, 16)), 2),                        # the caller's tile shape is what runs
    (dict(n=(64, 1, 64), stencil=5), 8),                       # the 2D stencil
    (dict(n=(64, 1, 64), stencil=5, exec="persistent"), 1),
])
def test_which_grids_run_four_steps(kw, steps):
    kw = dict(dict(odf=8, dtype="f64", exec="graph"), **kw)
    if kw.get("stencil") == 5:
        kw["odf"] = 1
    assert od.host_plan(**kw)["pass"]["steps"] == steps


@pytest.mark.parametrize("dtype,exec_,n,odf,steps", [
    # most of a box's lanes outside the grid and enough tiles to fill the chip
    ("f64", "fused", (1, 2000, 2000), 1, 2), ("f64", "graph", (4, 8000, 2000), 1, 2), ("f64", "fused", (8, 2000, 2000), 1, 2),
    ("f64", "persistent", (1, 2000, 2000), 1, 2), ("f64", "msgdriven", (1, 2000, 2000), 1, 2),
    ("f64", "fused", (8000, 1, 8000), 1, 1), ("f32", "fused", (8000, 1, 8000), 1, 1), ("f64", "fused", (1, 1, 100000), 1, 1),
    ("f32", "fused", (4, 8000, 2000), 1, 2), ("f64", "fused", (1, 1000, 1000), 8, 2), ("f32", "msgdriven", (100000, 1, 1), 1, 1),
    # enough cells in the lanes, or too few tiles
    ("f64", "fused", (32, 2000, 2000), 1, 4), ("f64", "fused", (2000, 2000, 1), 1, 4), ("f64", "fused", (2000, 2, 2000), 1, 4),
    ("f64", "fused", (8, 300, 300), 1, 4), ("f64", "fused", (300, 1, 300), 1, 4), ("f64", "fused", (1, 300, 300), 1, 4),
    ("f32", "fused", (2000, 1, 2000), 1, 4), ("f64", "fused", (16, 16, 4096), 1, 4), ("f64", "fused", (4, 1000, 1000), 64, 4),
    ("f32", "msgdriven", (4, 2000, 2000), 1, 4)])
def test_thin_grids_run_the_quicker_passes(dtype, exec_, n, odf, steps):
    assert od.host_plan(n=n, odf=odf, dtype=dtype, exec=exec_)["pass"]["steps"] == steps


@pytest.mark.gpu
@pytest.mark.parametrize("exec_", ["fused", "graph", "persistent", "msgdriven"])
@pytest.mark.parametrize("dtype,n", [("f64", (1, 700, 900)), ("f64", (1500, 1, 3000)), ("f32", (3000, 1, 5000))])
def test_thin_grids(exec_, dtype, n):
    # whichever passes the rule takes
    want, _, r = oracle.solve(n, DT[dtype], seed=5, iters=11, bc=BC6)
    g = od.Grid(n, odf=1, dtype=dtype, exec=exec_, bc=BC6, seed=5, hints=1)
    try:
        g.iterate(4)
        g.iterate(7)
        U, got = g.read(), g.residual()
    finally:
        g.close()
    _same(U, want)
    assert got == r


def _same(U, want):
    if not np.array_equal(U, want):
        d = np.argwhere(~((U == want) | (np.isnan(U) & np.isnan(want))))
        if len(d):
            k, j, i = d[0]
            raise AssertionError(f"{len(d)} cells differ; first at padded (k,j,i)=({k},{j},{i}): "
                                 f"{U[k, j, i]!r} vs {want[k, j, i]!r}")


def _run(n, odf, dtype, iters, exec_="fused", seed=5, write=None, want_steps=4, **kw):
    g = od.Grid(n, odf=odf, dtype=dtype, exec=exec_, bc=BC6, seed=seed, hints=1, **kw)
    try:
        assert g.pass_info()["steps"] == want_steps
        if write is not None:
            g.write(write)
        for k in iters:
            g.iterate(k)
        return g.read(), g.residual()
    finally:
        g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,odf", [((64, 64, 1), 1), ((64, 64, 9), 1), ((68, 65, 3), 1), ((120, 121, 4), 1),
                                   ((124, 120, 5), 1), ((176, 70, 12), 1), ((180, 64, 20), 1), ((128, 72, 64), 64),
                                   ((64, 67, 30), 8), ((192, 130, 33), 27), ((256, 64, 48), 512),
                                   # vectors cut short by chares and by the grid; grids of one
                                   # strip, of fewer rows or vectors than lanes, of one cell
                                   ((211, 163, 37), 27), ((65, 70, 9), 1), ((67, 64, 9), 8), ((66, 130, 20), 8),
                                   ((1, 1, 1), 1), ((2, 1, 3), 1), ((9, 8, 7), 27), ((3, 40, 5), 1), ((40, 3, 33), 8),
                                   ((63, 15, 12), 1), ((64, 16, 12), 8), ((65, 17, 12), 8), ((130, 33, 5), 125),
                                   ((100, 100, 100), 512)])
def test_edges_of_boxes_and_chares(dtype, n, odf):
    want, _, r = oracle.solve(n, DT[dtype], seed=5, iters=8, bc=BC6)
    U, got = _run(n, odf, dtype, [8])
    _same(U, want)
    assert got == r


@pytest.mark.gpu
@pytest.mark.parametrize("exec_", ["fused", "graph", "persistent", "msgdriven"])
@pytest.mark.parametrize("iters", [[4], [5], [6], [7], [4, 4], [3, 8, 1, 4], [1, 11]])
def test_what_is_left_of_a_count(exec_, iters):
    want, _, r = oracle.solve((128, 64, 24), np.float64, seed=5, iters=sum(iters), bc=BC6)
    U, got = _run((128, 64, 24), 8, "f64", iters, exec_)
    _same(U, want)
    assert got == r


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("exec_,hints", [("persistent", 0), ("msgdriven", 0), ("msgdriven", 4), ("msgdriven", 64),
                                         ("msgdriven", 512)])
def test_boxes_in_one_launch(dtype, exec_, hints):
    # more boxes than workgroups and several passes; message-driven also with
    # the schedule check's delays, cursor claims and a publisher per XCD
    n, iters = (300, 300, 70), 20
    want, _, r = oracle.solve(n, DT[dtype], seed=5, iters=iters, bc=BC6)
    g = od.Grid(n, odf=27, dtype=dtype, exec=exec_, bc=BC6, seed=5, hints=1 | hints)
    try:
        assert g.pass_info()["steps"] == 4
        g.iterate(12)
        g.iterate(8)
        U, got = g.read(), g.residual()
    finally:
        g.close()
    _same(U, want)
    assert got == r


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("iters", [[40], [41], [42, 3], [2, 43, 40], [1, 40, 4, 44]])
def test_message_driven_boxes_and_tiles_in_turn(dtype, iters):
    # counts long enough for boxes, what is left of them, and short ones by tiles
    n = (128, 64, 24)
    want, _, r = oracle.solve(n, DT[dtype], seed=5, iters=sum(iters), bc=BC6)
    U, got = _run(n, 8, dtype, iters, "msgdriven")
    _same(U, want)
    assert got == r


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,n,count", [("f32", 128, 6), ("f64", 128, 10), ("f64", 64, 6), ("f32", 192, 4)])
def test_short_message_driven_counts_cost_no_more_than_pairs(dtype, n, count):
    # a launch of boxes, and another for the rest, took up to 1.7 times as long
    times = []
    for hints in (1, 1 | 1 << 14):
        g = od.Grid(n, odf=8, dtype=dtype, exec="msgdriven", hints=hints)
        took = []
        for _ in range(40):
            t0 = time.perf_counter()
            g.iterate(count)
            g.residual()
            took.append(time.perf_counter() - t0)
        g.close()
        times.append(sorted(took)[5])
    assert times[0] < 1.2 * times[1], times


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("odf,iters", [(64, [4]), (64, [3, 8]), (8, [11])])
def test_imbalance_re_runs_before_the_pass(dtype, odf, iters):
    # half the chares re-run up to four times a step: their re-runs write the
    # other parity before the pass overwrites it
    n = (128, 72, 40)
    want, _, r = oracle.solve(n, DT[dtype], seed=5, iters=sum(iters), bc=BC6)
    U, got = _run(n, odf, dtype, iters, imbalance_pct=50, imbalance_max_extra=4)
    _same(U, want)
    assert got == r


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_uneven_blocks(dtype):
    n = 128
    blocks = workloads.octree_blocks(n=n, root=64, min_edge=16, p_refine=0.5, seed=3)
    want, _, r = oracle.solve(n, DT[dtype], seed=5, iters=9, bc=BC6)
    U, got = _run(n, 1, dtype, [9], blocks=blocks)
    _same(U, want)
    assert got == r


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("field", ["shell", "signs", "tiny", "zeros", "huge"])
def test_values_the_division_and_the_boundary_can_go_wrong_on(dtype, field):
    # every shell cell its own value; sums of both signs; sums around and below
    # the smallest normal number, where the quotient rounds to fewer bits;
    # zeros of both signs; infinities (whose differences make NaNs)
    n = (132, 70, 14)
    rng = np.random.default_rng(7)
    U = rng.random((n[2] + 2, n[1] + 2, n[0] + 2))
    info = np.finfo(DT[dtype])
    if field == "signs":
        U = U - 0.5
    elif field == "tiny":
        U = (U - 0.3) * float(info.tiny) * 2.0 ** rng.integers(-info.nmant, 60, U.shape)
    elif field == "zeros":
        U = np.where(U < 0.7, 0.0, -0.0)
    elif field == "huge":
        U = np.where(U < 0.0005, np.inf, (U - 0.5) * float(info.max) / 8)
    U = U.astype(DT[dtype])
    for a in (0, 1, 2):   # shell edges and corners read back as 0
        for b in range(a):
            for i in (0, -1):
                for j in (0, -1):
                    at = [slice(None)] * 3
                    at[a], at[b] = i, j
                    U[tuple(at)] = 0
    want, _, r = oracle.jacobi(U.copy(), 8)
    got, gr = _run(n, 1, dtype, [8], write=U)
    assert np.array_equal(got.view(np.uint8), want.view(np.uint8)) or field == "huge"
    _same(got, want)
    assert gr == r


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1018, 1016, 1020])
def test_sums_below_the_quick_division_beside_huge_ones(scale):
    # odd in x about a plane of nearly subnormal values: in that plane the huge
    # x neighbours cancel, so each small sum stays beside one of 2^1017 and more,
    # whose high word reads as a signalling NaN
    n, c = (65, 64, 12), 33
    rng = np.random.default_rng(3)
    U = np.zeros((n[2] + 2, n[1] + 2, n[0] + 2))
    for d in range(1, 34):
        U[:, :, c + d] = 2.0 ** scale * (1 + rng.random(U.shape[:2]) / 8)
        U[:, :, c - d] = -U[:, :, c + d]
    U[:, :, c] = (rng.random(U.shape[:2]) - 0.3) * 2.0 ** -1018
    for a in (0, 1, 2):   # shell edges and corners read back as 0
        for b in range(a):
            for i in (0, -1):
                for j in (0, -1):
                    at = [slice(None)] * 3
                    at[a], at[b] = i, j
                    U[tuple(at)] = 0
    want, _, r = oracle.jacobi(U.copy(), 8)
    assert 0 < np.abs(want[1:-1, 1:-1, c]).max() < 2.0 ** -1016
    got, gr = _run(n, 1, "f64", [8], write=U)
    _same(got, want)
    assert gr == r


@pytest.mark.gpu
@pytest.mark.parametrize("exec_,dims,n", [("fused", 3, 3), ("fused", 3, 4), ("fused", 3, 7), ("fused", 3, 8), ("fused", 3, 12),
                                          ("fused", 3, 20), ("fused", 2, 8), ("fused", 2, 12), ("fused", 2, 16),
                                          ("persistent", 3, 4), ("persistent", 3, 8), ("persistent", 3, 12)])
def test_replays_of_a_captured_count_go_on(exec_, dims, n):
    # each replay continues where the last ended: the passes of the count keep
    # the parity they have by pairs, whatever part of it runs over boxes
    import torch

    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        if dims == 3:
            g = od.Grid((64, 64, 24), odf=8, dtype="f64", exec=exec_, seed=5, bc=BC6, hints=1, stream=s)
        else:
            g = od.Grid2D((300, 64), odf=4, dtype="f64", exec=exec_, seed=5, hints=1, stream=s)
    try:
        s.synchronize()
        g.iterate(8)   # (the first launches are not in the graph)
        g.residual()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s, capture_error_mode="relaxed"):
            g.iterate(n)
        assert g.pass_info()["steps"] == (4 if dims == 3 else 8)
        for i in range(1, 4):
            with torch.cuda.stream(s):
                graph.replay()
            s.synchronize()
            if dims == 3:
                want, _, r = oracle.solve((64, 64, 24), np.float64, seed=5, iters=8 + i * n, bc=BC6)
            else:
                want, _, r = oracle.solve2d((300, 64), np.float64, 5, 8 + i * n, (1.0, 0.0, 0.0, 0.0))
            _same(g.read(), want)
            assert g.residual() == r
    finally:
        g.close()


@pytest.mark.gpu
def test_a_long_axis_does_not_make_creation_long():
    # the table of planes behind a chare's: quadratic work on it took 0.36 s for a
    # chare of 60000 planes, so 16 s here, what is linear takes hundredths
    n = (8, 8, 400000)
    t0 = time.monotonic()
    g = od.Grid(n, odf=1, dtype="f64", exec="fused", bc=BC6, seed=5)
    took = time.monotonic() - t0
    try:
        assert took < 5, took
        g.iterate(8)
        _same(g.read(), oracle.solve(n, np.float64, seed=5, iters=8, bc=BC6)[0])
    finally:
        g.close()


@pytest.mark.gpu
def test_a_workspace_of_the_pairs_size_runs_pairs():
    import ctypes

    import torch

    from paper_2605_12734_amd import _binding as B

    kw = dict(n=(128, 64, 24), odf=8, dtype="f64", exec="fused", bc=BC6, seed=5)
    cfg, _keep = od.make_config(**kw)
    pairs, _k2 = od.make_config(hints=1 << 14, **kw)
    size = ctypes.c_size_t()
    od.check(od.lib().od_workspace_bytes(ctypes.byref(pairs), ctypes.byref(size)), "bytes")
    ws = torch.empty(size.value, dtype=torch.uint8, device="cuda:0")
    h = ctypes.c_void_p()
    od.check(od.lib().od_create(ctypes.byref(cfg), None, ctypes.c_void_p(ws.data_ptr()), size, ctypes.byref(h)),
             "od_create")
    try:
        assert od.pass_info(h)["steps"] == 2
        od.check(od.lib().od_iterate(h, 8), "od_iterate")
        r = ctypes.c_double()
        od.check(od.lib().od_residual(h, ctypes.byref(r)), "od_residual")
        assert r.value == oracle.solve((128, 64, 24), np.float64, seed=5, iters=8, bc=BC6)[2]
    finally:
        od.check(od.lib().od_destroy(h), "od_destroy")
    assert B.OD_F64 == 8


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,odf", [((1, 1), 1), ((5, 9), 1), ((252, 3), 1), ((253, 20), 1), ((256, 16), 4), ((257, 17), 9),
                                   ((512, 64), 16), ((1000, 700), 9), ((2048, 10), 64)])
def test_boxes_of_the_2d_stencil(dtype, n, odf):
    p = od.host_plan(n=(n[0], 1, n[1]), odf=odf, dtype=dtype, exec="graph", stencil=5)["pass"]
    assert p["steps"] == 8
    seen = np.zeros((n[1], n[0]), dtype=np.int8)
    for cx0, cx1, _, _, x0, x1, _, _, z0, z1 in p["boxes"]:
        assert 0 <= cx0 <= x0 < x1 <= cx1 <= n[0] and 0 <= z0 < z1 <= n[1]
        assert cx0 == 0 or x0 - cx0 >= 8
        assert cx1 == n[0] or cx1 - x1 >= 8
        seen[z0:z1, x0:x1] += 1
    assert (seen == 1).all()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("exec_", ["fused", "graph"])
@pytest.mark.parametrize("n,odf,iters", [((1, 1), 1, [8]), ((5, 9), 1, [16]), ((252, 30), 1, [8, 3]), ((253, 20), 1, [8]),
                                         ((256, 16), 4, [19]), ((257, 170), 9, [16]), ((512, 64), 16, [8, 8]),
                                         ((1000, 700), 9, [24]), ((500, 40), 1, [13])])
def test_2d_stencil(dtype, exec_, n, odf, iters):
    bc = (1.0, 0.5, 2.0, 3.0)
    want, _, r = oracle.solve2d(n, DT[dtype], 5, sum(iters), bc)
    g = od.Grid2D(n, odf=odf, dtype=dtype, exec=exec_, bc=bc, seed=5, hints=1)
    try:
        assert g.pass_info()["steps"] == 8
        for k in iters:
            g.iterate(k)
        U, got = g.read(), g.residual()
    finally:
        g.close()
    _same(U, want)
    assert got == r


# Served solves: passes of up to four steps.  Sizes at the edges of the boxes
# (one row a strip below 64, the lanes' 64 cells, full and partial vectors) and
# every remainder of the interval between checks; the reference is the oracle's
# solve with the same stopping rule, the tolerance 0.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("check_every", [0, 1, 2, 3, 4, 6, 9])
def test_served_passes_match_oracle(dtype, check_every):
    from paper_2605_12734_amd.serving import Server

    reqs = [dict(n=n, dtype=dtype, odf=odf, tol=tol, max_iters=iters, check_every=check_every, seed=n)
            for n, odf, tol, iters in [(1, 1, 0.0, 5), (4, 1, 0.0, 1), (31, 8, 0.0, 13), (63, 27, 2e-3, 40), (64, 8, 0.0, 7),
                                       (65, 1, 2e-3, 22), (96, 8, 0.0, 11), (130, 64, 0.0, 6)]]
    with Server(arena_bytes=1 << 30, max_slots=16) as srv:
        tickets = [srv.submit(**q) for q in reqs]
        for t, q in zip(tickets, reqs):
            res, field = srv.wait(t), srv.fetch(t)
            want, it, r = oracle.solve(q["n"], DT[dtype], seed=q["seed"], iters=q["max_iters"], tol=q["tol"],
                                       check_every=check_every)
            assert (res["iters"], res["residual"]) == (it, r), q
            assert np.array_equal(field, want), q


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("check_every", [1, 2, 3])
def test_served_short_passes_at_the_edges_of_their_boxes(dtype, check_every):
    # passes of up to one, two or three steps over boxes with a ring of as many
    # cells: of 62 to 58 and 14 to 10 rows, checked at every iteration also with
    # pieces of 4 to 10 planes
    from paper_2605_12734_amd.serving import Server

    reqs = [dict(n=n, dtype=dtype, odf=odf, tol=tol, max_iters=iters, check_every=check_every, seed=n)
            for n, odf, tol, iters in [(2, 1, 0.0, 3), (8, 8, 0.0, 9), (14, 1, 0.0, 5), (15, 1, 0.0, 6), (16, 8, 0.0, 17),
                                       (24, 27, 0.0, 8), (25, 1, 0.0, 8), (29, 8, 0.0, 7), (62, 1, 0.0, 6),
                                       (63, 1, 2e-3, 40), (125, 27, 0.0, 4), (126, 1, 0.0, 5), (190, 64, 0.0, 3)]]
    with Server(arena_bytes=2 << 30, max_slots=16) as srv:
        tickets = [srv.submit(**q) for q in reqs]
        for t, q in zip(tickets, reqs):
            res, field = srv.wait(t), srv.fetch(t)
            want, it, r = oracle.solve(q["n"], DT[dtype], seed=q["seed"], iters=q["max_iters"], tol=q["tol"],
                                       check_every=check_every)
            assert (res["iters"], res["residual"]) == (it, r), q
            assert np.array_equal(field, want), q
