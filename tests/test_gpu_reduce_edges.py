"""Moments and enstrophy where their kernels branch: one block of tile sums and one
more than that, axes of the fewest nodes the stencil takes, against numpy sums of the
fields read back.
"""
import numpy as np
import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu


def _lattice(shape, prec):
    nx, ny, nz = shape
    L = lbm.Lattice(inputs.all_fluid(nx, ny, nz), q=19, prec=prec, tau=0.6)
    L.init_equilibrium(*inputs.random_fields(nx, ny, nz, seed=8))
    L.step(3)
    return L, *L.read_fields()


@pytest.mark.parametrize("shape", [(5, 4, 3), (64, 64, 16), (64, 64, 17), (257, 3, 97), (64, 256, 65)])
def test_moments_equal_numpy(shape):
    """FP64 sums of at most a million terms, Neumaier and a tree: 1e-12 relative
    (the momentum, whose terms cancel, of the sum of their magnitudes)."""
    L, rho, u = _lattice(shape, lbm.LBM_F64)
    m = L.reduce()
    n = rho.size
    assert m["n_nonfinite"] == 0
    ke = 0.5 * (u ** 2).sum() / n
    assert abs(m["kinetic_energy"] - ke) <= 1e-12 * ke
    assert abs(m["mass"] - rho.sum()) <= 1e-12 * n
    for k, a in enumerate("xyz"):
        assert abs(m["momentum"][k] - (rho * u[k]).sum()) <= 1e-12 * np.abs(u[k]).sum()


@pytest.mark.parametrize("shape", [(9, 9, 9), (31, 10, 9), (64, 65, 17)])
def test_enstrophy_equals_numpy(shape):
    """The same stencil and fields; a few roundings per node, 1e-12 relative."""
    L, _, u = _lattice(shape, lbm.LBM_F32)

    def d(a, axis):
        return sum(c * (np.roll(a, -k, axis) - np.roll(a, k, axis))
                   for k, c in ((1, 4 / 5), (2, -1 / 5), (3, 4 / 105), (4, -1 / 280)))
    w = (d(u[2], 1) - d(u[1], 0), d(u[0], 0) - d(u[2], 2), d(u[1], 2) - d(u[0], 1))
    ref = 0.5 * sum((a ** 2).sum() for a in w) / u[0].size
    assert abs(L.enstrophy() - ref) <= 1e-12 * ref
