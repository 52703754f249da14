"""Lattices on the special stream handles (hipStreamLegacy 1, hipStreamPerThread 2): the
second names another stream in every thread, so the threads that copy a large read out
must not start before the gather has ended.
"""
import numpy as np
import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("handle", [1, 2])
def test_large_reads_follow_the_steps(handle):
    nx, ny, nz = 128, 120, 136  # 67 MB of fields, 317 MB of populations: staged copies, two chunks
    tags = inputs.all_fluid(nx, ny, nz)
    rho, u = inputs.random_fields(nx, ny, nz, seed=6)
    Ls = [lbm.Lattice(tags, q=19, prec=lbm.LBM_F64, tau=0.6, stream=s) for s in (None, handle)]
    for L in Ls:
        L.init_equilibrium(rho, u)
    for n in (9, 22):
        out = []
        for L in Ls:
            L.step(n)  # queued when the read is called
            out.append((*L.read_fields(), L.read_state()))
        for a, b in zip(*out):
            assert np.array_equal(a, b)
    assert np.abs(out[0][1]).max() > 0.0
    for L in Ls:
        L.close()
