"""od_read hands back the padded field chunk by chunk, host threads copying
filled chunks while the device gathers the next: fields of one chunk, of a
few, of more chunks than staging slots, and with planes larger than a chunk."""
import numpy as np
import pytest

import paper_2605_12734_amd as od

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,odf,dtype", [((40, 30, 20), 1, "f64"), ((130, 120, 50), 8, "f64"), ((256, 200, 260), 27, "f32"),
                                         ((400, 390, 230), 64, "f32"), ((1100, 520, 3), 1, "f64")])
def test_read_returns_what_was_written(n, odf, dtype):
    U = np.random.default_rng(3).random((n[2] + 2, n[1] + 2, n[0] + 2)).astype({"f64": np.float64, "f32": np.float32}[dtype])
    out = [np.zeros(U.shape, dtype=bool) for _ in range(3)]
    for d in range(3):
        for i in (0, -1):
            out[d][tuple(i if a == d else slice(None) for a in range(3))] = True
    U[(out[0].astype(int) + out[1] + out[2]) > 1] = 0   # shell edges and corners read back as 0
    with od.Grid(n, odf=odf, dtype=dtype, exec="graph") as g:
        g.write(U)
        for _ in range(2):
            assert np.array_equal(g.read(), U)


# Blocks on both sides of the size (1 MiB) up to which a block is read in one
# launch, rows that fill no vector among them.
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 5, 50, 51, 64, 65])
def test_read_block_is_the_fields(n, dtype):
    g = od.Grid(n, odf=1, dtype=dtype, exec="fused", seed=3)
    try:
        g.iterate(3)
        assert np.array_equal(g.read_block(0), g.read()[1:-1, 1:-1, 1:-1])
    finally:
        g.close()
