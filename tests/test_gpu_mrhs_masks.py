"""Finished systems of a multi-RHS solve.  The hop walks the live systems of a
chunk only: whatever the others are (zero sources are finished from the start,
the rest stop at different iterations), a system's solution has the same bits,
and finished systems cost next to nothing."""
import time

import pytest
import torch

import paper_0710_2442_amd as wd
import synthetic as syn
from gpu_util import to_field

pytestmark = pytest.mark.gpu
KAPPA = 0.12


def _params(inner):
    return wd.wd_solve_params_default(solver=wd.WD_SOLVER_DEFECT_CG, inner_prec=inner,
                                      inner_tol=1e-3 if inner == "f32" else 1e-2)


@pytest.mark.parametrize("inner", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("rpl", [16, 4, 1])
def test_masked_systems_do_not_change_the_others(inner, rpl):
    """18 systems in chunks of 9, 4 and 1: first, last, alternate, all but one
    and a whole chunk masked; FP64 (one LDS buffer) runs in the residuals."""
    dims, n = (6, 4, 6, 10), 18
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 91), dims, -1, "f64")
    for prec in ("f64", inner):
        wd.wd_set_dslash_mrhs_variant(g, prec, 512, wd.WD_ORDER_RANGES, rpl)
    src = [syn.point_source(dims, 1, 2)] + [syn.gaussian_spinor(dims, 92 + r) for r in range(n - 1)]
    b = torch.cat([to_field(g, s) for s in src])
    m = b.numel() // n

    def solve(b):
        x = torch.full_like(b, 0xAB)
        rc, infos = wd.wd_solve_mrhs(g, b, x, n, KAPPA, 1e-10, _params(inner))
        assert rc == 0
        return x, [i["iters"] for i in infos]

    x0, it0 = solve(b)
    assert len(set(it0)) > 1  # the systems stop at different iterations by themselves
    for live in (range(1, n), range(n - 1), range(0, n, 2), [7], range(9), range(9, n), range(4, 8), []):
        bm = b.clone()
        for r in set(range(n)) - set(live):
            bm[r * m:(r + 1) * m] = 0
        x, it = solve(bm)
        for r in range(n):
            if r in live:
                assert it[r] == it0[r] and torch.equal(x[r * m:(r + 1) * m], x0[r * m:(r + 1) * m]), (list(live), r)
            else:
                assert it[r] == 0 and not x[r * m:(r + 1) * m].view(torch.float64).any(), (list(live), r)
    g.close()


def test_finished_systems_are_nearly_free():
    """One live system of twelve: less than half the time of twelve (a third on
    an idle device; 0.58 when the hop loaded and projected every system)."""
    dims, n = (16, 16, 16, 32), 12
    U = syn.gauge_field((16, 16, 16, 2), 0.3, 93).repeat(16, axis=0)
    g = wd.Gauge(U, dims, -1, "f64")
    fields = [wd.wd_new_field(dims, "f64") for _ in range(n)]
    for r, f in enumerate(fields):
        wd.wd_gaussian_field(g, f, wd.WD_FULL, "f64", 7, r)
    b = torch.cat(fields)
    one = b.clone()
    one[b.numel() // n:] = 0
    x = torch.empty_like(b)
    secs = {}
    for _ in range(5):
        for key, src in (("all", b), ("one", one)):
            torch.cuda.synchronize()
            t = time.perf_counter()
            rc, _ = wd.wd_solve_mrhs(g, src, x, n, KAPPA, 1e-10, _params("f32"))
            secs[key] = min(secs.get(key, 1e9), time.perf_counter() - t)
            assert rc == 0
    assert secs["one"] < 0.48 * secs["all"], secs
    g.close()


@pytest.mark.parametrize("inner", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("cap", [1000, 7])
def test_where_an_iteration_ends_does_not_change_a_system(inner, cap):
    """135168 sites a parity, one more tile than the consumers add up: 4 systems
    end an iteration in a launch of their own, 3 in the p update.  Same bits,
    same counts, also at the iteration cap and for a zero source."""
    dims = (16, 16, 16, 66)
    U = syn.gauge_field((16, 16, 16, 2), 0.3, 95).repeat(33, axis=0)
    g = wd.Gauge(U, dims, -1, "f64")
    fields = [wd.wd_new_field(dims, "f64") for _ in range(4)]
    for r, f in enumerate(fields):
        wd.wd_gaussian_field(g, f, wd.WD_FULL, "f64", 9, r)
    fields[1].zero_()
    m = fields[0].numel()
    p = _params(inner)
    p.max_iter = cap
    got = {}
    for n in (3, 4):
        x = torch.full((n * m,), 0xAB, dtype=torch.uint8, device="cuda")
        rc, infos = wd.wd_solve_mrhs(g, torch.cat(fields[:n]), x, n, KAPPA, 1e-10, p)
        assert (rc == 0) == (cap == 1000)
        got[n] = x, [(i["iters"], i["outer_iters"], i["status"]) for i in infos]
        assert cap == 7 or max(i["true_rel_resid"] for i in infos) <= 1e-10
    assert got[4][1][:3] == got[3][1] and got[3][1][1][0] == 0
    assert torch.equal(got[4][0][:3 * m], got[3][0])
    g.close()
