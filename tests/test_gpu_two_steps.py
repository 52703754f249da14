"""The two-step kernel (csrc/lbm_two.h) against the one-step kernels.

A lattice large enough to take it steps by fours through a second array; an
explicit launch shape selects the one-step kernels.  Both do the same arithmetic
per node, so the populations are equal bit for bit (the regularized models, whose
products the compiler may fuse differently in the two kernels: a few roundings).
Sizes put tile and chunk edges everywhere: rows that are not whole tiles, one tile
and a bit, rows of several blocks, planes that are not whole blocks.
"""
import numpy as np
import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu
EPS = {lbm.LBM_F64: 2.0 ** -52, lbm.LBM_F32: 2.0 ** -23, lbm.LBM_F16S: 2.0 ** -10}
KW = dict(tau=0.6, smag_cs=0.1, wall_velocity=[(0.1, 0.02, 0.0), (0.0, -0.05, 0.03)])


def _run(tags, q, prec, force, one_step, torch_buffer=False):
    nz, ny, nx = tags.shape
    L = lbm.Lattice(tags, q=q, prec=prec, force=force, layout="rows", torch_buffer=torch_buffer, **KW)
    if one_step:
        L.set_launch(64, 4)
    L.init_equilibrium(*inputs.random_fields(nx, ny, nz, seed=4))
    L.step(9)  # two pairs of two, one step: the next run starts at odd layout parity
    a = L.read_state()
    series = L.step_reduce(11, 5)
    b = L.read_state()
    L.close()
    return a, b, series


def _check(tags, q, prec, model, force=(0.0, 0.0, 0.0), torch_buffer=False):
    one = _run(tags, q, prec, force, True)
    two = _run(tags, q, prec, force, False, torch_buffer)
    for k in range(2):
        if model in (lbm.TAG_REG, lbm.TAG_RR):
            # one rounding of a population per step and product fused differently
            assert np.abs(one[k] - two[k]).max() <= 40 * EPS[prec] * np.abs(one[k]).max()
        else:
            assert np.array_equal(one[k], two[k])
    for m, n in zip(one[2], two[2]):
        assert n["n_nonfinite"] == 0
        assert abs(m["kinetic_energy"] - n["kinetic_energy"]) <= 40 * EPS[prec] * m["kinetic_energy"]


@pytest.mark.parametrize("prec", [lbm.LBM_F64, lbm.LBM_F32, lbm.LBM_F16S])
@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("shape", [(129, 131, 127), (256, 96, 101), (90, 201, 160)])
def test_periodic_equals_one_step(shape, q, prec):
    nx, ny, nz = shape
    _check(inputs.all_fluid(nx, ny, nz, lbm.TAG_SMAG), q, prec, lbm.TAG_SMAG)


@pytest.mark.parametrize("prec", [lbm.LBM_F64, lbm.LBM_F32, lbm.LBM_F16S])
@pytest.mark.parametrize("tag,force", [(lbm.TAG_BGK, (1e-4, -2e-4, 5e-5)), (lbm.TAG_TRT, (0.0, 0.0, 0.0)),
                                       (lbm.TAG_TRT, (1e-4, -2e-4, 5e-5)), (lbm.TAG_RR, (0.0, 0.0, 1e-4)),
                                       (lbm.TAG_REG, (0.0, 0.0, 0.0))])
def test_walls_equal_one_step(tag, force, prec):
    """Random solid and moving-wall nodes (also across the periodic edges)."""
    tags = inputs.random_tags(192, 130, 141, 11, 0.15, 0.05, (tag,))
    _check(tags, 19, prec, tag, force)


@pytest.mark.parametrize("tag", [lbm.TAG_BGK, lbm.TAG_TRT])
def test_uniform_force_and_caller_buffer(tag):
    _check(inputs.all_fluid(140, 150, 130, tag), 27, lbm.LBM_F32, tag, (1e-4, 0.0, -1e-4), torch_buffer=True)


def test_d3q27_mixed_walls():
    tags = inputs.random_tags(150, 120, 131, 7, 0.1, 0.05, (lbm.TAG_BGK, lbm.TAG_SMAG))
    for prec in (lbm.LBM_F64, lbm.LBM_F32):
        _check(tags, 27, prec, lbm.TAG_SMAG)
