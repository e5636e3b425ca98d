"""CG recurrences where a thread walks four packet runs side by side: fields
whose packets the grid covers more than four times, with a remainder.  Against
the two-apart form of the same systems (bit for bit: the scalars come from the
hops) and, for one FP64 system, the oracle's own residual."""
import pytest
import torch

import paper_0710_2442_amd as wd
import synthetic as syn
from gpu_util import from_field, to_field
from oracle import solvers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner", ["f32", "bf16"])
def test_many_systems_side_by_side(inner):
    """64 systems of 12096 sites a parity (192 padding slots): 31 blocks each,
    36 (BF16) or 72 (FP32) runs; 6 systems take 144 or 288 blocks, two apart."""
    dims, n, few = (12, 12, 12, 14), 64, 6
    U = syn.gauge_field((12, 12, 12, 2), 0.3, 97).repeat(7, axis=0)
    g = wd.Gauge(U, dims, -1, "f64")
    fields = [wd.wd_new_field(dims, "f64") for _ in range(n)]
    for r, f in enumerate(fields):
        wd.wd_gaussian_field(g, f, wd.WD_FULL, "f64", 11, r)
    m = fields[0].numel()
    p = wd.wd_solve_params_default(solver=wd.WD_SOLVER_DEFECT_CG, inner_prec=inner, inner_tol=1e-2)
    got = []
    for k in (n, few):
        x = torch.full((k * m,), 0xAB, dtype=torch.uint8, device="cuda")
        rc, infos = wd.wd_solve_mrhs(g, torch.cat(fields[:k]), x, k, 0.12, 1e-10, p)
        assert rc == 0 and max(i["true_rel_resid"] for i in infos) <= 1e-10
        got.append((x, [i["iters"] for i in infos]))
    assert got[0][1][:few] == got[1][1]
    assert torch.equal(got[0][0][:few * m], got[1][0])
    g.close()


@pytest.mark.parametrize("solver", ["CG", "CGLS_FULL"])
def test_one_system_side_by_side(solver):
    """179712 sites a parity: 1.03 times four runs per thread of 2047 blocks."""
    dims = (24, 24, 24, 26)
    U = syn.gauge_field((24, 24, 24, 2), 0.3, 98).repeat(13, axis=0)
    b = syn.gaussian_spinor(dims, 99)
    g = wd.Gauge(U, dims, -1, "f64")
    x = wd.wd_new_field(dims, "f64")
    x.fill_(0xAB)
    rc, info = wd.wd_solve(g, to_field(g, b), x, 0.12, 1e-9,
                           wd.wd_solve_params_default(solver=getattr(wd, "WD_SOLVER_" + solver)))
    assert rc == 0
    r = solvers.true_residual(U, b, from_field(g, x), 0.12)
    assert r <= 1e-9 and abs(r - info["true_rel_resid"]) <= 1e-3 * 1e-9
    g.close()
