"""Reads to host memory at the edges of the staged copy (pieces of 2 MB, from 8 MB on):
planes that are and are not whole pieces, several chunks, one of two outputs, against
the same planes read node by node, and pinned memory.
"""
import numpy as np
import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu


def _lattice(shape, layout=None):
    nx, ny, nz = shape
    tags = inputs.random_tags(nx, ny, nz, seed=5)
    L = lbm.Lattice(tags, q=19, prec=lbm.LBM_F64, tau=0.6, layout=layout)
    L.init_equilibrium(*inputs.random_fields(nx, ny, nz, seed=2))
    L.step(3)
    return L, tags


@pytest.mark.parametrize("shape,layout", [((16, 16, 16), "bricks"), ((64, 64, 63), None), ((64, 64, 64), None),
                                          ((64, 64, 65), None), ((131, 67, 59), None), ((96, 112, 128), "bricks"),
                                          ((256, 256, 150), None)])
def test_reads_agree(shape, layout):
    """The populations of sampled nodes read as a list equal the planes (FP64, exact), and
    rho and rho u are their sums (19 terms of order one: 1e-14); rho alone and u alone equal
    the read of both; a destination that HIP pinned gets the same."""
    import torch
    L, tags = _lattice(shape, layout)
    rho, u = L.read_fields()
    n = rho.size
    cells = np.unique(np.concatenate([np.arange(0, n, 997), np.arange(262143, n, 262144), np.arange(0, n, 262144),
                                      [n - 1]]))
    fluid = (tags.ravel()[cells] >= 1) & (tags.ravel()[cells] <= 10)
    f = L.read_cells(cells).reshape(cells.size, 19)
    assert np.abs(rho.ravel()[cells] - f.sum(1))[fluid].max() <= 1e-14 * 19
    assert np.all(rho.ravel()[cells][~fluid] == 0.0)
    pops = L.read_populations().reshape(19, n)
    assert np.array_equal(pops[:, cells[fluid]].T, f[fluid])
    pin = torch.full((4, n), 7.0, dtype=torch.float64, pin_memory=True).numpy()
    r1, u1 = np.full_like(rho, 7.0), np.full_like(u, 7.0)
    lib = lbm.lib()
    assert lib.lbm_read_fields(L.h, lbm._ptr(r1), None) == lbm.LBM_OK
    assert lib.lbm_read_fields(L.h, None, lbm._ptr(u1)) == lbm.LBM_OK
    assert lib.lbm_read_fields(L.h, lbm._ptr(pin[0]), lbm._ptr(pin[1:])) == lbm.LBM_OK
    assert np.array_equal(rho, r1) and np.array_equal(u, u1)
    assert np.array_equal(pin[0], rho.ravel()) and np.array_equal(pin[1:].ravel(), u.ravel())


def test_reads_of_two_threads():
    """Two lattices, two threads, each its own stream and staging."""
    import threading

    import torch
    Ls = []
    for _ in range(2):
        nx, ny, nz = 96, 96, 97
        L = lbm.Lattice(inputs.all_fluid(nx, ny, nz), q=19, prec=lbm.LBM_F32, tau=0.6, stream=torch.cuda.Stream())
        L.init_equilibrium(*inputs.random_fields(nx, ny, nz, seed=len(Ls)))
        Ls.append(L)
    ref = [L.read_fields() for L in Ls]
    out = [None, None]

    def work(k):
        for _ in range(3):
            out[k] = Ls[k].read_fields()
    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for k in range(2):
        assert np.array_equal(ref[k][0], out[k][0]) and np.array_equal(ref[k][1], out[k][1])
    assert not np.array_equal(ref[0][0], ref[1][0])
