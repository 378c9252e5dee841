"""What is timed: solves as programs that use this package run them.

A case is one program: a grid (or a server) that it keeps, and a pass that
advances the field and hands the result back, through the package's public
entry points only.  A pass goes on from where the previous one left the field.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2605_12734_amd as od

DEFAULT_BC = (1.0, 0.0, 0.0, 0.0, 0.0, 0.0)


def listed():
    return [
        # the smallest job: a short solve on a small grid, where launches and
        # the round trip to the host are most of the time
        dict(name="cube64", kind="cube", nx=64, ny=64, nz=64, odf=8, dtype="f64", exec="graph", iters=100,
             tune=False),
        # ragged box, odd extents and an odd iteration count, single precision,
        # one launch per pass: a grid nobody sized for the hardware
        dict(name="ragged_f32", kind="cube", nx=211, ny=163, nz=157, odf=27, dtype="f32", exec="fused", iters=401,
             tune=False),
        # solve to a tolerance: the residual is looked at every 10 iterations
        dict(name="converge128", kind="converge", n=128, odf=64, dtype="f64", exec="graph", iters=400, every=10),
        # the headline grid: 4096 chares of 32^3, graph replays, tuned
        dict(name="cube512_odf4096", kind="cube", nx=512, ny=512, nz=512, odf=4096, dtype="f64", exec="graph",
             iters=2000, tune=True),
        # the same grid in few large chares and single precision
        dict(name="cube512_f32", kind="cube", nx=512, ny=512, nz=512, odf=8, dtype="f32", exec="graph", iters=2000,
             tune=True),
        # one cooperative launch for all iterations, chares of 64^3
        dict(name="persistent512", kind="cube", nx=512, ny=512, nz=512, odf=512, dtype="f64", exec="persistent",
             iters=1000, tune=True),
        # the message-driven scheduler, chares of 128^3
        dict(name="msgdriven512", kind="cube", nx=512, ny=512, nz=512, odf=64, dtype="f64", exec="msgdriven",
             iters=1000, tune=False),
        # dynamic load imbalance: each step a tenth of the chares re-run 1-4 sweeps
        dict(name="imbalance512", kind="cube", nx=512, ny=512, nz=512, odf=512, dtype="f64", exec="fused", iters=500,
             tune=False, imbalance=10),
        # uneven blocks from octree refinement, one resolution, graph replays
        dict(name="octree512", kind="octree", n=512, dtype="f64", exec="graph", iters=500, multires=False, blocks=1),
        # the same refinement with 16 cells per leaf edge: ghost cells filled
        # by injection and averaging where the resolution changes
        dict(name="multires512", kind="octree", n=512, dtype="f64", exec="graph", iters=500, multires=True, blocks=1),
        # the paper's 2D workload, a quarter of its edge
        dict(name="jacobi2d", kind="plane", nx=8192, ny=8192, odf=64, dtype="f64", exec="graph", iters=1000),
        # serving: a burst of independent solves of mixed sizes and types
        dict(name="serve16", kind="serve", requests=16, lo=32, hi=256, iters=1000, mix=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cube", "cube", "cube", "cube", "imbalance", "converge", "octree", "plane", "serve"])
    dtype = rng.choice(["f64", "f64", "f32"])
    if kind == "octree":
        return dict(kind="octree", n=rng.choice([256, 384, 512]), dtype=dtype,
                    exec=rng.choice(["graph", "fused", "persistent"]), iters=rng.randint(60, 500),
                    multires=rng.random() < 0.4, blocks=rng.randint(1, 999))
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(1, 16), lo=32, hi=rng.randint(48, 256),
                    iters=10 * rng.randint(10, 100), mix=rng.randint(1, 999))
    if kind == "plane":
        nx, ny = _log(rng, 256, 8192), _log(rng, 256, 8192)
        return dict(kind="plane", nx=nx, ny=ny, odf=rng.choice([1, 4, 16, 64]), dtype=dtype,
                    exec=rng.choice(["graph", "fused"]), iters=_log(rng, 50, 1000))
    if kind == "converge":
        every = rng.choice([5, 10, 20])
        return dict(kind="converge", n=_log(rng, 32, 320), odf=rng.choice([1, 8, 64]), dtype=dtype,
                    exec=rng.choice(["graph", "persistent", "fused"]), iters=every * rng.randint(5, 40), every=every)
    n = _log(rng, 40, 512)
    side = [min(512, max(32, int(n * rng.uniform(0.6, 1.4)))) if rng.random() < 0.5 else n for _ in range(3)]
    case = dict(kind="cube", nx=side[0], ny=side[1], nz=side[2], odf=rng.choice([1, 8, 27, 64, 512, 4096]),
                dtype=dtype, exec=rng.choice(["graph", "graph", "fused", "persistent", "msgdriven"]),
                iters=_log(rng, 50, 2000), tune=rng.random() < 0.5)
    while round(case["odf"] ** (1 / 3)) * 8 > min(side):   # chares of at least 8 cells an edge
        case["odf"] = {4096: 512, 512: 64, 64: 27, 27: 8, 8: 1}[case["odf"]]
    if kind == "imbalance":
        case.update(exec=rng.choice(["fused", "persistent", "msgdriven"]), iters=min(case["iters"], 500),
                    imbalance=10, tune=False)
    if case["exec"] in ("msgdriven",):
        case["tune"] = False
    return case


# ---------------------------------------------------------------------------
# structure of the uneven and the served cases


def _leaves(case):
    """Octree leaves (origin, edge) of the case's domain: blocks of 128 split
    with probability 0.4 at each level, down to 16."""
    rng = np.random.default_rng(int(case["blocks"]))
    n, out = int(case["n"]), []
    level = [(x, y, z, 128) for z in range(0, n, 128) for y in range(0, n, 128) for x in range(0, n, 128)]
    while level:
        nxt = []
        for x, y, z, e in level:
            if e > 16 and rng.random() < 0.4:
                h = e // 2
                nxt += [(x + i, y + j, z + k, h) for k in (0, h) for j in (0, h) for i in (0, h)]
            else:
                out.append((x, y, z, e))
        level = nxt
    out.sort(key=lambda b: (b[2], b[1], b[0]))
    return out


def _requests(case):
    """Sizes log-uniform, half of them fp32, 1, 8 or 64 chares each."""
    rng = np.random.default_rng(int(case["mix"]))
    out = []
    for _ in range(int(case["requests"])):
        n = int(round(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"])))))
        out.append((n, "f32" if rng.random() < 0.5 else "f64", int(rng.choice([1, 8, 64]))))
    return out


def _cells(case):
    if case["kind"] == "cube":
        return case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "plane":
        return case["nx"] * case["ny"]
    if case["kind"] == "octree" and case["multires"]:
        return 4096 * len(_leaves(case))
    if case["kind"] == "serve":
        return sum(n ** 3 for n, _, _ in _requests(case))
    return case["n"] ** 3


def work(case):
    """The start field is drawn on the device and the result returned: the
    field is written and read at least once each; six operations an update."""
    cells = _cells(case)
    if case["kind"] == "serve":
        size = sum((4 if d == "f32" else 8) * n ** 3 for n, d, _ in _requests(case)) / cells
    else:
        size = 4 if case["dtype"] == "f32" else 8
    ops = 4 if case["kind"] == "plane" else 6
    return {"bytes": 2.0 * size * cells, "flops": float(ops) * cells * case["iters"]}


# ---------------------------------------------------------------------------


def prepare(case, seed):
    k = case["kind"]
    if k == "serve":
        reqs = _requests(case)
        srv = od.Server(od_arena(reqs), max_slots=len(reqs))
        return {"case": case, "server": srv, "requests": reqs, "seed": int(seed)}
    kw = dict(dtype=case["dtype"], exec=case["exec"], seed=int(seed), hints=1)
    if k == "octree":
        leaves = _leaves(case)
        kw["blocks"] = [((x, y, z), (e, e, e)) for x, y, z, e in leaves]
        if case["multires"]:
            kw["cell"] = [e // 16 for _, _, _, e in leaves]
        g = od.Grid(case["n"], **kw)
    elif k == "plane":
        g = od.Grid2D((case["nx"], case["ny"]), odf=case["odf"], **kw)
    elif k == "converge":
        g = od.Grid(case["n"], odf=case["odf"], **kw)
    else:
        if case.get("imbalance"):
            kw.update(imbalance_pct=case["imbalance"], imbalance_max_extra=4)
        g = od.Grid((case["nx"], case["ny"], case["nz"]), odf=case["odf"], **kw)
    if case.get("tune"):
        g.autotune(2)
    return {"case": case, "grid": g}


def od_arena(reqs):
    from paper_2605_12734_amd import serving
    need = sum(serving.request_bytes(n=n, dtype=d, odf=o) for n, d, o in reqs)
    return serving.control_bytes(len(reqs)) + need + (len(reqs) + 1) * 4096


def run(state):
    case = state["case"]
    if case["kind"] == "serve":
        srv, seed = state["server"], state["seed"]
        tickets = [srv.submit(n, d, odf=o, tol=1e-6, max_iters=case["iters"], check_every=10, seed=seed + i)
                   for i, (n, d, o) in enumerate(state["requests"])]
        info = [srv.wait(t) for t in tickets]
        return {"field": [srv.fetch(t) for t in tickets], "iters": [int(x["iters"]) for x in info],
                "residual": [float(x["residual"]) for x in info]}
    g = state["grid"]
    if case["kind"] == "converge":
        seen = []
        for _ in range(case["iters"] // case["every"]):
            g.iterate(case["every"])
            seen.append(g.residual())
        return {"residual": np.array(seen), "field": g.read()}
    g.iterate(case["iters"])
    r = g.residual()
    if case["kind"] == "octree" and case["multires"]:
        return {"residual": r, "field": np.stack([g.read_block(b) for b in range(g.plan()["nchares"])])}
    return {"residual": r, "field": g.read()}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch


def _unit(seed, index, dtype):
    """SplitMix64's (index + 1)-th output of `seed` as a number in [0, 1)."""
    def const(v):
        v &= (1 << 64) - 1
        return v - (1 << 64) if v >> 63 else v

    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)

    z = (index + 1) * const(0x9E3779B97F4A7C15) + const(int(seed))
    z = (z ^ shr(z, 30)) * const(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * const(0x94D049BB133111EB)
    z = z ^ shr(z, 31)
    if dtype == "f32":
        return shr(z, 40).double() * 2.0 ** -24
    return shr(z, 11).double() * 2.0 ** -53


def _where():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _box(nx, ny, nz, seed, dtype):
    """Padded start field: interior drawn, the shell's x- face 1."""
    u = torch.zeros((nz + 2, ny + 2, nx + 2), dtype=torch.float64, device=_where())
    for z in range(nz):   # plane by plane: the indices of a whole grid are large
        i = torch.arange(z * ny * nx, (z + 1) * ny * nx, dtype=torch.int64, device=u.device)
        u[z + 1, 1:-1, 1:-1] = _unit(seed, i, dtype).view(ny, nx)
    u[1:-1, 1:-1, 0] = DEFAULT_BC[0]
    return u


def _sweep(u, v, flat=False):
    """v's interior = the mean of u's neighbours (flat: no y neighbours)."""
    w = v[1:-1, 1:-1, 1:-1]
    torch.add(u[1:-1, 1:-1, :-2], u[1:-1, 1:-1, 2:], out=w)
    if not flat:
        w += u[1:-1, :-2, 1:-1]
        w += u[1:-1, 2:, 1:-1]
    w += u[:-2, 1:-1, 1:-1]
    w += u[2:, 1:-1, 1:-1]
    w /= 4.0 if flat else 6.0


def _solve(u, iters, flat=False, every=0):
    v, seen, r = u.clone(), [], 0.0
    for i in range(1, iters + 1):
        _sweep(u, v, flat)
        if i == iters or (every and i % every == 0):
            r = float((v[1:-1, 1:-1, 1:-1] - u[1:-1, 1:-1, 1:-1]).abs().max())
            seen.append(r)
        u, v = v, u
    return u, seen if every else r


def _multires(case, seed):
    """Every leaf holds 16^3 cells.  Before each sweep the ghost layer of a
    face is read from the neighbour: the cell of the same or a coarser
    neighbour that holds the ghost cell, or the mean of the finer cells of
    the touching layer that cover it; 1 or 0 on the domain's own faces."""
    leaves, n = np.array(_leaves(case)), case["n"]
    B, dev = len(leaves), _where()
    own = np.empty((n // 16,) * 3, dtype=np.int64)
    for b, (x, y, z, e) in enumerate(leaves // 16):
        own[z:z + e, y:y + e, x:x + e] = b
    h = leaves[:, 3] // 16
    u = torch.zeros((B, 18, 18, 18), dtype=torch.float64, device=dev)
    c = np.arange(16)
    for b in range(B):
        x, y, z, _ = leaves[b]
        q = ((z + c * h[b])[:, None, None] * n + (y + c * h[b])[None, :, None]) * n + (x + c * h[b])[None, None, :]
        u[b, 1:-1, 1:-1, 1:-1] = _unit(seed, torch.from_numpy(q).to(dev), case["dtype"])
    flat = lambda b, i, j, k: ((b * 18 + k + 1) * 18 + j + 1) * 18 + i + 1   # noqa: E731
    fills = {}   # cells averaged along an edge -> ([ghost index], [source indices])
    ones = []
    for b in range(B):
        o = leaves[b, :3]
        for d in range(3):
            for side in (0, 1):
                t = [a for a in range(3) if a != d]
                g1, g2 = [a.ravel() for a in np.meshgrid(c, c, indexing="ij")]
                ghost = [None] * 3
                ghost[d], ghost[t[0]], ghost[t[1]] = np.full(256, 16 if side else -1), g1, g2
                nrm = o[d] + leaves[b, 3] if side else o[d] - 1
                dst = flat(b, *ghost)
                if nrm < 0 or nrm >= n:
                    if d == 0 and side == 0:
                        ones.append(dst)
                    continue
                p = [None] * 3
                p[d], p[t[0]], p[t[1]] = np.full(256, nrm), o[t[0]] + g1 * h[b], o[t[1]] + g2 * h[b]
                nb = own[p[2] // 16, p[1] // 16, p[0] // 16]
                for r in np.unique(np.maximum(1, h[b] // h[nb])):
                    m = np.maximum(1, h[b] // h[nb]) == r
                    a2, a1 = np.meshgrid(np.arange(r), np.arange(r), indexing="ij")
                    src = [None] * 3
                    for a in range(3):
                        step = 0 if a == d else (a1 if a == t[0] else a2).ravel()[None, :]
                        hn = h[nb[m]][:, None]
                        src[a] = (p[a][m][:, None] - leaves[nb[m], a][:, None]) // hn + step + np.zeros((1, r * r), int)
                    lists = fills.setdefault(int(r), ([], []))
                    lists[0].append(dst[m])
                    lists[1].append(flat(nb[m][:, None], *src))
    put = [(torch.from_numpy(np.concatenate(d)).to(dev), torch.from_numpy(np.concatenate(s)).to(dev))
           for _, (d, s) in sorted(fills.items())]
    u.view(-1)[torch.from_numpy(np.concatenate(ones)).to(dev)] = DEFAULT_BC[0]
    v, r = u.clone(), 0.0
    for i in range(case["iters"]):
        for d, s in put:
            u.view(-1)[d] = u.view(-1)[s].mean(1)
        w = v[:, 1:-1, 1:-1, 1:-1]
        torch.add(u[:, 1:-1, 1:-1, :-2], u[:, 1:-1, 1:-1, 2:], out=w)
        for q in (u[:, 1:-1, :-2, 1:-1], u[:, 1:-1, 2:, 1:-1], u[:, :-2, 1:-1, 1:-1], u[:, 2:, 1:-1, 1:-1]):
            w += q
        w /= 6.0
        if i == case["iters"] - 1:
            r = float((w - u[:, 1:-1, 1:-1, 1:-1]).abs().max())
        u, v = v, u
    return {"residual": r, "field": u[:, 1:-1, 1:-1, 1:-1].contiguous()}


def exact(case, seed):
    k = case["kind"]
    if _cells(case) * case["iters"] > 4e11:   # about 20 seconds
        return None
    if k == "octree" and case["multires"]:
        return _multires(case, seed)
    if k == "serve":
        fields, res = [], []
        for i, (n, d, _) in enumerate(_requests(case)):
            u, r = _solve(_box(n, n, n, seed + i, d), case["iters"])
            fields.append(u)
            res.append(r)
        return {"field": fields, "iters": [case["iters"]] * len(fields), "residual": res}
    if k == "plane":
        u, r = _solve(_box(case["nx"], 1, case["ny"], seed, case["dtype"]), case["iters"], flat=True)
        return {"residual": r, "field": u[:, 1, :].contiguous()}
    if k == "converge":
        n = case["n"]
        u, seen = _solve(_box(n, n, n, seed, case["dtype"]), case["iters"], every=case["every"])
        return {"residual": np.array(seen), "field": u}
    nx, ny, nz = (case["nx"], case["ny"], case["nz"]) if k == "cube" else (case["n"],) * 3
    u, r = _solve(_box(nx, ny, nz, seed, case["dtype"]), case["iters"])
    return {"residual": r, "field": u}
