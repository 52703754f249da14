"""Brick layout on both sides of 4 GiB (32-bit byte offsets below, node form above)
and on the smallest lattices: populations equal the row layout's bit for bit."""
import numpy as np
import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,q,prec", [
    ((16, 16, 16), 27, lbm.LBM_F16S), ((16, 32, 48), 19, lbm.LBM_F64), ((48, 16, 32), 27, lbm.LBM_F32),
    ((272, 272, 256), 27, lbm.LBM_F64), ((272, 272, 288), 27, lbm.LBM_F64)])
def test_bricks_equal_rows(shape, q, prec):
    """4.09 and 4.60 * 10^9 bytes in the two large cases."""
    nx, ny, nz = shape
    tags = inputs.random_tags(nx, ny, nz, seed=6, solid_frac=0.6, fluid_tags=(lbm.TAG_TRT,))
    n = tags.size
    cells = np.arange(n) if n < 100000 else np.unique(np.concatenate(
        [np.arange(0, n, 1999), np.arange(n - 3000, n), np.arange(3000), np.arange(n // 2, n // 2 + 3000)]))
    out = []
    for layout in ("rows", "bricks"):
        with lbm.Lattice(tags, q=q, prec=prec, tau=0.8, layout=layout, force=(1e-4, 2e-5, 0.0),
                         wall_velocity=[(0.05, 0.0, 0.02), (0.0, -0.04, 0.0)]) as L:
            L.init_equilibrium(*inputs.random_fields(nx, ny, nz, seed=3))
            L.step(5)
            out.append(L.read_cells(cells))
    fluid = tags.ravel()[cells] == lbm.TAG_TRT
    assert np.array_equal(out[0][fluid], out[1][fluid])
