"""FP16 hop and D_W with one wave per hop direction: three waves sum a site's
components and agree on its scale.  The same bytes as one thread per site for
sites of zeros, of tiny and huge numbers, infinities and NaN, with and without
an epilogue, at block edges and in padding.  (Numbers below 2^-128 give NaN in
the stored input: the scale's reciprocal overflows.  A NaN's sign is not defined
by the arithmetic; the forms differ in it.)
"""
import numpy as np
import pytest
import torch

import paper_0710_2442_amd as wd
import synthetic as syn
from gpu_util import to_field

pytestmark = pytest.mark.gpu


def _spinor(dims, special):
    psi = syn.gaussian_spinor(dims, 102)
    flat = psi.reshape(-1, 12)
    rng = np.random.Generator(np.random.PCG64(103))
    flat[rng.random(len(flat)) < 0.5] = 0
    pick = rng.permutation(len(flat))
    for q, f in enumerate((1e-30, 1e-42, 1e30, 3e38)):
        flat[pick[q::16]] *= f
    if special:
        flat[pick[5], 7] = np.inf
        flat[pick[6], 0] = np.nan
        flat[pick[7]] = np.nan
    return psi


def _nan_positive(field):
    """The field's bytes with every FP16 NaN positive (scales, 16 bits a half, are
    never NaN: fmax skips them)."""
    h = field.view(torch.int16).clone()
    h[(h & 0x7FFF) == 0x7E00] = 0x7E00
    return h


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 6, 10), (8, 8, 8, 8)])
@pytest.mark.parametrize("special", [False, True])
def test_split_scale_is_the_sites(dims, special):
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 101), dims, -1, "f16")
    psi = _spinor(dims, special)
    default = wd.wd_get_dslash_variant(g, "f16")
    assert default[2] & wd.WD_TUNE_SPLIT_DIRS
    for flags in (0, wd.WD_DAGGER):
        for parity in (wd.WD_EVEN, wd.WD_ODD):
            src = to_field(g, psi, "f16", 1 - parity)
            outs = []
            for variant in ((256, 0, 0), default):
                wd.wd_set_dslash_variant(g, "f16", *variant)
                out = wd.wd_new_field(dims, "f16", 1, parity)
                out.fill_(0xAB)
                wd.wd_dslash_ex(g, src, out, 0.7, parity, "f16", flags)
                torch.cuda.synchronize()
                outs.append(_nan_positive(out))
            assert torch.equal(*outs), (parity, flags)
        src = to_field(g, psi, "f16")
        outs = []
        for slices, tile in ((dims[3], 0), (0, 4)):  # the march, and one wave per direction
            wd.wd_set_dirac_variant(g, "f16", slices, tile)
            out = wd.wd_new_field(dims, "f16")
            out.fill_(0xAB)
            wd.wd_dslash_ex(g, src, out, 0.12, wd.WD_FULL, "f16", flags | wd.WD_ONE_PASS)
            torch.cuda.synchronize()
            outs.append(_nan_positive(out))
        assert torch.equal(*outs), flags
    g.close()


def test_large_lattices_use_it_too():
    """2^18 sites a parity and more: the default is the same form."""
    dims = (16, 16, 32, 64)
    U = syn.gauge_field((16, 16, 32, 2), 0.3, 104).repeat(32, axis=0)
    g = wd.Gauge(U, dims, -1, "f16")
    block, groups, occ = wd.wd_get_dslash_variant(g, "f16")
    assert (block, groups) == (64, 8) and occ & wd.WD_TUNE_SPLIT_DIRS
    src, outs = wd.wd_new_field(dims, "f16", 1, wd.WD_ODD), []
    f32 = wd.wd_new_field(dims, "f32", 1, wd.WD_ODD)
    wd.wd_gaussian_field(g, f32, wd.WD_ODD, "f32", 7, 0)
    wd.wd_convert(g, f32, "f32", src, "f16", 1, 1.0)
    for variant in ((block, groups, occ), (256, 0, 0)):
        wd.wd_set_dslash_variant(g, "f16", *variant)
        out = wd.wd_new_field(dims, "f16", 1, wd.WD_EVEN)
        wd.wd_dslash_ex(g, src, out, 0.12, wd.WD_EVEN, "f16")
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(*outs)
    g.close()


@pytest.mark.parametrize("n", [12, 24])
def test_many_right_hand_sides_on_a_small_lattice(n):
    """8^4: the default takes 4.7 and 6.4 us where one lane per site takes 14;
    with all components of a site in one wave it took 24.  Same bytes."""
    dims = (8, 8, 8, 8)
    g = wd.Gauge(syn.gauge_field(dims, 0.3, 105), dims, -1, "f16")
    src = to_field(g, syn.gaussian_spinor(dims, 106), "f16", wd.WD_ODD).repeat(n)
    default, us, outs = wd.wd_get_dslash_mrhs_variant(g, "f16"), [], []
    for variant in (default, (128, 0, 4)):
        wd.wd_set_dslash_mrhs_variant(g, "f16", *variant)
        out = torch.full_like(src, 0xAB)
        wd.wd_dslash_mrhs(g, src, out, 0.12, wd.WD_EVEN, "f16", n)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                wd.wd_dslash_mrhs(g, src, out, 0.12, wd.WD_EVEN, "f16", n)
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            graph.replay()
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) * 1e3 / 20)
        us.append(min(times))
        outs.append(out)
    assert torch.equal(*outs)
    assert us[0] < us[1], us
    g.close()
