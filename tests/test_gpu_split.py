"""The hop and D_W with one wave per hop direction (WD_TUNE_SPLIT_DIRS and
one-launch tile 4, what a new handle runs): the same bytes as the
one-site-per-lane hop and as the march in every storage precision, order and
epilogue.  Sizes: one slot tile mostly padding (2^4: 8
sites), fewer tiles than XCDs, padding in the last tile, ranges whose last
blocks are empty, extents of 2 (forward and backward neighbours coincide)."""
import pytest
import torch

import paper_0710_2442_amd as wd
import synthetic as syn
from oracle import solvers
from gpu_util import BARS_L2, SITE_BARS, assert_close, from_field, to_field

pytestmark = pytest.mark.gpu

ORDERS = (0, 2, 8, -2, -8, -101, -108, wd.WD_ORDER_RANGES)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (2, 6, 2, 34), (8, 8, 8, 8), (16, 16, 8, 16)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_split_hop_is_bitwise_the_one_lane_hop(dims, prec):
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 61), dims, -1, prec)
    default = wd.wd_get_dslash_variant(g, prec)
    assert default[0] == 64 and default[2] & wd.WD_TUNE_SPLIT_DIRS
    psi = syn.gaussian_spinor(dims, 62)
    n = 0
    for parity in (wd.WD_EVEN, wd.WD_ODD):
        src = to_field(g, psi, prec, 1 - parity)
        for flags in (0, wd.WD_DAGGER):
            wd.wd_set_dslash_variant(g, prec, 256, 0, 0)
            ref = wd.wd_new_field(dims, prec, 1, parity)
            wd.wd_dslash_ex(g, src, ref, 0.7, parity, prec, flags)
            for variant in [default] + [(64, o, wd.WD_TUNE_SPLIT_DIRS | c) for o in ORDERS
                                        for c in (0, wd.WD_TUNE_CACHED_STORE)]:
                try:
                    wd.wd_set_dslash_variant(g, prec, *variant)
                except wd.WdError:
                    assert variant[1] not in (0, wd.WD_ORDER_RANGES)
                    continue
                assert wd.wd_get_dslash_variant(g, prec) == variant
                out = wd.wd_new_field(dims, prec, 1, parity)
                out.fill_(0xAB)
                wd.wd_dslash_ex(g, src, out, 0.7, parity, prec, flags)
                torch.cuda.synchronize()
                assert torch.equal(out, ref), (variant, parity, flags)
                n += 1
    assert n >= 4 * 5
    bit = wd.WD_TUNE_SPLIT_DIRS
    for bad in ((128, 0, bit), (64, 0, bit | 4), (64, 0, bit | wd.WD_TUNE_PRELOAD_LINKS),
                (64, 0, bit | wd.WD_TUNE_STAGE_LDS), (64, 0, bit | (1 << wd.WD_TUNE_SPL_SHIFT)),
                (64, wd.WD_ORDER_RANGES, 0), (64, 5, bit)):
        with pytest.raises(wd.WdError):
            wd.wd_set_dslash_variant(g, prec, *bad)
    g.close()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (8, 8, 8, 8)])
@pytest.mark.parametrize("inner", ["f64", "f32", "f16", "bf16"])
def test_split_hop_in_a_solve_is_bitwise_the_one_lane_hop(dims, inner):
    """Every epilogue and norm a solver fuses into the hop (64-site blocks on
    both sides, so the norm partials are the same sums)."""
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 63), dims, -1, "f64")
    b = to_field(g, syn.gaussian_spinor(dims, 64))
    p = wd.wd_solve_params_default(solver=wd.WD_SOLVER_CG) if inner == "f64" else wd.wd_solve_params_default(
        solver=wd.WD_SOLVER_DEFECT_CG, inner_prec=inner, inner_tol=1e-2)
    outs = []
    for groups, occ in ((0, 0), (0, wd.WD_TUNE_SPLIT_DIRS), (wd.WD_ORDER_RANGES, wd.WD_TUNE_SPLIT_DIRS)):
        for prec in ("f64", "f32", "f16", "bf16"):
            wd.wd_set_dslash_variant(g, prec, 64, groups, occ)
        x = wd.wd_new_field(dims, "f64")
        rc, info = wd.wd_solve(g, b, x, 0.12, 1e-10, p)
        assert rc == 0
        outs.append((x, info["iters"], info["outer_iters"]))
    for o in outs[1:]:
        assert o[1:] == outs[0][1:] and torch.equal(o[0], outs[0][0])
    g.close()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (2, 6, 2, 34), (16, 8, 8, 16), (16, 32, 32, 32)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_split_dirac_is_bitwise_the_march(dims, prec):
    """Tile 4, set and as a new handle chooses it (16x32^3: 2^18 sites per
    parity, the order of slice regions), against consecutive marching tiles."""
    gen = torch.Generator().manual_seed(65)
    L1, L2, L3, L4 = dims
    if L1 * L2 * L3 * L4 > 100000:  # links from one block repeated along x4
        U = syn.gauge_field((L1, L2, L3, 2), 0.3, 66)
        U = U.repeat(L4 // 2, axis=0)
    else:
        U = syn.gauge_field(dims, 0.3, 66)
    g = wd.Gauge(U, dims, -1, prec)
    canon = torch.randn(L1 * L2 * L3 * L4 * 24, generator=gen, dtype=torch.float64)
    src = to_field(g, torch.view_as_complex(canon.reshape(-1, 2)).numpy(), prec)
    for flags in (0, wd.WD_DAGGER):
        outs = []
        hops = wd.wd_new_field(dims, prec)
        hops.fill_(0xAB)
        wd.wd_dslash_ex(g, src, hops, 0.124, wd.WD_FULL, prec, flags)
        for variant in (None, (0, 4), (0, 0)):
            if variant:
                wd.wd_set_dirac_variant(g, prec, *variant)
                assert wd.wd_get_dirac_variant(g, prec) == variant
            out = wd.wd_new_field(dims, prec)
            out.fill_(0xAB)
            wd.wd_dslash_ex(g, src, out, 0.124, wd.WD_FULL, prec, flags | wd.WD_ONE_PASS)
            torch.cuda.synchronize()
            outs.append(out)
        assert all(torch.equal(o, outs[0]) for o in outs[1:]), flags
        # without WD_ONE_PASS the hops are added first: two roundings of the
        # same value, each within the precision's bars of it
        assert_close(from_field(g, hops, prec), from_field(g, outs[0], prec), prec, l2=2 * BARS_L2[prec],
                     site=2 * SITE_BARS[prec], what=f"D_W {dims} {prec}")
    g.close()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (8, 8, 8, 16)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nrhs", [1, 5, 17])
def test_split_mrhs_hop_is_bitwise_the_single_hop(dims, prec, nrhs):
    """Block 512 with 1, 2, 4 and 16 right-hand sides per block (even and
    ragged chunks, a buffer of one and of many), every order that fits, and
    the default's own choice."""
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 67), dims, -1, prec)
    psis = syn.gaussian_spinor(dims, 68, nrhs=nrhs)
    assert wd.wd_get_dslash_mrhs_variant(g, prec)[0] == 512
    for parity in (wd.WD_EVEN, wd.WD_ODD):
        src = torch.cat([to_field(g, p, prec, 1 - parity) for p in psis])
        hb = src.numel() // nrhs
        ref = torch.empty_like(src)
        for r in range(nrhs):
            wd.wd_dslash_ex(g, src[r * hb:(r + 1) * hb], ref[r * hb:(r + 1) * hb], 0.7, parity, prec)
        n = 0
        for variant in [None] + [(512, o, rpl) for o in ORDERS for rpl in (1, 2, 4, 16)]:
            if variant:
                try:
                    wd.wd_set_dslash_mrhs_variant(g, prec, *variant)
                except wd.WdError:
                    assert variant[1] not in (0, wd.WD_ORDER_RANGES)
                    continue
            out = torch.full_like(src, 0xAB)
            wd.wd_dslash_mrhs(g, src, out, 0.7, parity, prec, nrhs)
            torch.cuda.synchronize()
            assert torch.equal(out, ref), (variant, parity)
            n += 1
        assert n >= 9
    for bad in ((512, 0, 0), (512, 0, 17), (512, 5, 4)):
        with pytest.raises(wd.WdError):
            wd.wd_set_dslash_mrhs_variant(g, prec, *bad)
    g.close()


@pytest.mark.parametrize("inner", ["f32", "f16", "bf16"])
def test_split_mrhs_solve_matches_the_single_solves(inner):
    """Epilogues, per-RHS norms and skip flags of the multi-RHS hop in a solve
    whose systems stop at different iterations (a point source, a zero source
    and Gaussian ones) on a lattice with padding slots: each system's solution
    solves its own equation."""
    dims, kappa = (6, 4, 6, 10), 0.12
    U = syn.gauge_field(dims, 0.3, 69)
    g = wd.Gauge(U, dims, -1, "f64")
    b = [syn.point_source(dims, 1, 2), 0 * syn.point_source(dims, 0, 0)]
    b += [syn.gaussian_spinor(dims, 70 + r) for r in range(5)]
    fb = torch.cat([to_field(g, x) for x in b])
    fx = torch.empty_like(fb)
    p = wd.wd_solve_params_default(solver=wd.WD_SOLVER_DEFECT_CG, inner_prec=inner, inner_tol=1e-2)
    rc, infos = wd.wd_solve_mrhs(g, fb, fx, len(b), kappa, 1e-10, p)
    assert rc == 0 and all(i["status"] == 0 for i in infos)
    n = fb.numel() // len(b)
    for r, src in enumerate(b):
        x = from_field(g, fx[r * n:(r + 1) * n])
        if r == 1:
            assert not x.any()
        else:
            assert solvers.true_residual(U, src, x, kappa) <= 1.01e-10
    g.close()
