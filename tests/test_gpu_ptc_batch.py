"""Samples of a training batch that go through the kernels together.

The weight gradient is a matrix product over 64-site groups: lattices whose
parities end inside a group (8, 72 and 720 sites) against the FP64 oracle, at
the tolerance of the single-sample test (FP32 arithmetic: 1e-4).  A batch
larger than the workspace is cut into launches whose sums accumulate: for
copies of the same pairs loss and gradient do not depend on the number of
copies, except for the FP32 rounding of the factor 2/B (2^-24 each) and of the
result (2^-24): 1e-6.
"""
import numpy as np
import pytest
import torch

import paper_0710_2442_amd as wd
import synthetic as syn
from gpu_util import rel_err, round_c64, storage_round, to_field
from oracle import ptc

pytestmark = pytest.mark.gpu


def _net(g, act):
    rng = np.random.Generator(np.random.PCG64(71))
    W1 = 0.2 * (rng.standard_normal((9, 2, 1, 4, 4)) + 1j * rng.standard_normal((9, 2, 1, 4, 4)))
    W2 = 0.2 * (rng.standard_normal((9, 1, 2, 4, 4)) + 1j * rng.standard_normal((9, 1, 2, 4, 4)))
    return wd.Ptc(g, wd.ptc_weights_to_flat(W1, W2), act), W1, W2


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 3 * 2), (6, 4, 6, 10)])
@pytest.mark.parametrize("B", [1, 3])
def test_batch_gradient_matches_oracle(dims, B):
    U = syn.gauge_field(dims, 0.3, 72)
    rs = [syn.gaussian_spinor(dims, 73 + b) for b in range(B)]
    es = [syn.gaussian_spinor(dims, 83 + b) for b in range(B)]
    g = wd.Gauge(U, dims, -1, "f32")
    n, W1, W2 = _net(g, "f32")
    fr = torch.cat([to_field(g, x, "f32") for x in rs])
    fe = torch.cat([to_field(g, x, "f32") for x in es])
    loss, grad = wd.wd_ptc_loss_grad(n, fr, fe, B)
    L, g1, g2 = ptc.loss_and_grads(round_c64(U), W1, W2, [storage_round(x, "f32") for x in rs],
                                   [storage_round(x, "f32") for x in es])
    G1, G2 = wd.ptc_flat_to_weights(grad)
    assert abs(loss - L) <= 1e-5 * L
    assert rel_err(G1, g1) <= 1e-4 and rel_err(G2, g2) <= 1e-4
    n.close()
    g.close()


@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_batch_larger_than_the_workspace(act):
    dims = (4, 4, 4, 4)  # 1024 samples fill the workspace
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 75), dims, -1, "f32")
    n, _, _ = _net(g, act)
    fr = torch.cat([to_field(g, syn.gaussian_spinor(dims, 76 + b), "f32") for b in range(2)])
    fe = torch.cat([to_field(g, syn.gaussian_spinor(dims, 78 + b), "f32") for b in range(2)])
    l2, g2 = wd.wd_ptc_loss_grad(n, fr, fe, 2)
    for B in (2050, 4):
        lb, gb = wd.wd_ptc_loss_grad(n, fr.repeat(B // 2), fe.repeat(B // 2), B)
        assert abs(lb - l2) <= 1e-6 * l2
        assert np.linalg.norm(gb - g2) <= 1e-6 * np.linalg.norm(g2)
    n.close()
    g.close()
