"""Gradient and Adam kernels at the edges of their 128-sample blocks: fewer samples
than a wave or a block takes, one more than whole blocks, several passes of every
block, and sample indices out of range (which contribute nothing)."""
import numpy as np
import pytest

import oracle.mlp as om
from paper_2506_09242_amd import inputs, lbm

pytestmark = pytest.mark.gpu


def _data(n, seed):
    r = np.random.default_rng(seed)
    X = np.concatenate([2e-5 * r.normal(size=(n, 6)), 1.0 + 1e-3 * r.normal(size=(n, 1))], 1).astype(np.float32)
    P = inputs.mlp_he_init(seed)
    P[1345:1352], P[1352:1359] = X.mean(0), X.std(0) + (X.std(0) == 0)
    return X, np.abs(r.normal(1.0, 0.5, n)).astype(np.float32), P


def _dev(a):
    import torch
    return torch.tensor(np.asarray(a), device="cuda")


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 128, 129, 1000, 40000])
def test_gradient_block_edges(n):
    """FP32 sums over n samples against FP64: n eps at the most, 1e-4 as in test_gpu_mlp."""
    import torch
    X, Y, P = _data(n, 3)
    loss_o, g_o = om.loss_and_grad(P.astype(np.float64), X.astype(np.float64), Y.astype(np.float64))
    g, l = torch.empty(om.NP, device="cuda"), torch.empty(1, device="cuda")
    lbm.lbm_mlp_grad(_dev(P), _dev(X), _dev(Y), g, l)
    assert np.abs(g.cpu().numpy() - g_o).max() <= 1e-4 * np.abs(g_o).max()
    assert abs(l.item() / loss_o - 1.0) <= 1e-4


@pytest.mark.parametrize("n,batch", [(5, 5), (130, 64), (300, 299), (700, 1000)])
def test_out_of_range_indices_contribute_nothing(n, batch):
    """Replacing samples by out-of-range indices is the same as samples whose residual is
    left out: compared with the run over the remaining ones at the batch's own scale."""
    import torch
    X, Y, P = _data(n, 5)
    perm = np.arange(n, dtype=np.int64)
    bad = perm.copy()
    bad[::3] = np.array([n, -1, n + 7])[np.arange(len(bad[::3])) % 3]
    out = []
    for idx in (bad,):
        p, log = _dev(P), torch.empty(1, device="cuda")
        lbm.lbm_mlp_train(p, _dev(X), _dev(Y), _dev(idx), batch, 1, 1e-3, log)
        out.append((p.cpu().numpy(), log.item()))
    # oracle: one Adam step per batch on the kept samples, gradient scaled by kept / batch
    v = P.astype(np.float64)
    m1, m2, total, nb = np.zeros(1345), np.zeros(1345), 0.0, -(-n // batch)
    for b in range(nb):
        k = bad[b * batch:(b + 1) * batch]
        keep = k[(k >= 0) & (k < n)]
        loss, g = om.loss_and_grad(v, X[keep].astype(np.float64), Y[keep].astype(np.float64))
        loss, g = loss * len(keep) / len(k), g[:1345] * len(keep) / len(k)
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        t = b + 1
        v[:1345] -= 1e-3 * (m1 / (1 - 0.9 ** t)) / (np.sqrt(m2 / (1 - 0.999 ** t)) + 1e-8)
        total += loss / nb
    # a step moves a parameter by at most about lr; its direction is set by the gradient's
    # sign, so only parameters whose gradient is at FP32 rounding may differ by a whole step
    d = np.abs(out[0][0] - v)
    assert np.median(d) <= 1e-6 and np.mean(d > 1e-5) <= 0.01
    assert abs(out[0][1] / total - 1.0) <= 1e-4
