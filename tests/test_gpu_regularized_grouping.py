"""Regularized and recursive lattices: the populations do not depend on how calls group
the steps (calls of four and more take two steps a pass where there is memory for it),
nor on the storage layout or the launch shape.
"""
import numpy as np
import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu
KW = dict(tau=0.6, wall_velocity=[(0.1, 0.02, 0.0), (0.0, -0.05, 0.03)])


def _states(tags, q, prec, force, how):
    nz, ny, nx = tags.shape
    L = lbm.Lattice(tags, q=q, prec=prec, force=force, layout="rows", **KW)
    if how == "launch":
        L.set_launch(64, 4)
    L.init_equilibrium(*inputs.random_fields(nx, ny, nz, seed=4))
    out = []
    for n in (5, 6):  # the second run starts at odd layout parity
        for k in ([n] if how == "grouped" else [1] * n):
            L.step(k)
        out.append(L.read_state())
    L.close()
    return out


@pytest.mark.parametrize("force", [(0.0, 0.0, 0.0), (1e-4, -2e-4, 5e-5)])
@pytest.mark.parametrize("tag", [lbm.TAG_REG, lbm.TAG_RR])
@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("prec,geom", [("f64", "periodic"), ("f64", "walls"), ("f32", "periodic"), ("f32", "walls")])
def test_grouping_and_launch_are_bitwise_irrelevant(prec, geom, q, tag, force):
    nx, ny, nz = 210, 150, 141
    tags = inputs.all_fluid(nx, ny, nz, tag) if geom == "periodic" else \
        inputs.random_tags(nx, ny, nz, 11, 0.1, 0.05, (tag,))
    single = _states(tags, q, prec, force, "single")
    for how in ("grouped", "launch"):
        for a, b in zip(single, _states(tags, q, prec, force, how)):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("nx,ny,nz", [(256, 252, 124), (250, 254, 130)])
@pytest.mark.parametrize("q,tag", [(19, lbm.TAG_REG), (27, lbm.TAG_REG), (27, lbm.TAG_RR)])
def test_fp16_grouping_is_bitwise_irrelevant(nx, ny, nz, q, tag):
    tags = inputs.all_fluid(nx, ny, nz, tag)
    single = _states(tags, q, "f16s", (0.0, 0.0, 0.0), "single")
    for a, b in zip(single, _states(tags, q, "f16s", (0.0, 0.0, 0.0), "grouped")):
        assert np.array_equal(a, b)
