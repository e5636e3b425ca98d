"""Training steps in a captured graph: the first step of a network can be
captured, and a replay stays valid when a larger batch has grown the workspace
since.  Weights against the same steps taken eagerly; the samples go one by one
in the graph and together without it, so the FP64 sums differ in order and the
FP32 gradient by at most a rounding: 1e-6 of weights of order 1."""
import numpy as np
import pytest
import torch

import paper_0710_2442_amd as wd
import synthetic as syn
from gpu_util import to_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_captured_first_step_survives_a_larger_batch(act):
    dims, B, big = (6, 4, 6, 10), 3, 8
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 121), dims, -1, "f32")
    r = torch.cat([to_field(g, syn.gaussian_spinor(dims, 122 + b), "f32") for b in range(big)])
    e = torch.cat([to_field(g, syn.gaussian_spinor(dims, 132 + b), "f32") for b in range(big)])
    m = r.numel() // big
    rng = np.random.Generator(np.random.PCG64(71))
    W = 0.2 * rng.standard_normal(1152).astype(np.float32)
    nets = [wd.Ptc(g, W, act) for _ in range(2)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        wd.wd_ptc_train_step(nets[0], r[:B * m], e[:B * m], B, 1e-3, want_loss=False)
    loss, _ = wd.wd_ptc_loss_grad(nets[0], r, e, big)  # the weights have not moved yet
    want, _ = wd.wd_ptc_loss_grad(nets[1], r, e, big)
    assert loss == want
    filler = [torch.full((m,), 0xCD, dtype=torch.uint8, device="cuda") for _ in range(64)]
    for step in range(3):
        graph.replay()
        torch.cuda.synchronize()
        if step == 0:
            wd.wd_ptc_train_step(nets[1], r[:B * m], e[:B * m], B, 1e-3)
            got, ref = wd.wd_ptc_get_weights(nets[0]), wd.wd_ptc_get_weights(nets[1])
            assert np.abs(ref - W).max() > 5e-4
            assert np.abs(got - ref).max() <= 1e-6
        wd.wd_ptc_loss_grad(nets[0], r, e, big)  # eager work between the replays
    assert all(bool((f == 0xCD).all()) for f in filler)
    for n in nets:
        n.close()
    g.close()
