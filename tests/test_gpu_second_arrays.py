"""Second population arrays (two steps a pass) of one process hold at most a quarter of the
device together, so that a program that fills the memory with lattices gets nearly as
many as their own arrays allow, and are given back with their lattices.
"""

import pytest

from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu


def test_second_arrays_are_bounded_and_given_back():
    import torch
    total = torch.cuda.mem_get_info()[1]
    tags = inputs.all_fluid(512, 320, 256)  # D3Q27 FP64: 9.1 GB
    size = lbm.lbm_population_bytes(lbm.make_config(512, 320, 256, q=27, prec="f64"))
    Ls = []
    try:
        # twelve would take 109 GB of second arrays by the share of free memory alone
        for _ in range(12):
            Ls.append(lbm.Lattice(tags, q=27, prec="f64"))
        two = [L.steps_per_pass for L in Ls]
        held = size * two.count(2)
        assert two[0] == 2 and two[-1] == 1
        assert total / 4 - 2 * size < held <= total / 4
        # one that gives its array back makes room for another lattice's
        k = two.index(2)
        Ls.pop(k).close()
        Ls.append(lbm.Lattice(tags, q=27, prec="f64"))
        assert Ls[-1].steps_per_pass == 2
    finally:
        for L in Ls:
            L.close()
