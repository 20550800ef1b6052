"""The Schwarz half-sweep kernel where its lane layout can go wrong, against the NumPy oracle.

A wave holds 32 pairs of sites: on 2^4 domains four (domain, right-hand side) pairs share
one wave, so with three right-hand sides of different kappa the lanes of a wave carry
different clover fields and kappas; on 4^4 and 8x4^3 domains a workgroup is four or eight
waves whose inner products meet in LDS. The number of MR steps reaches from one (the
accumulated odd-site correction is its first term only) to five. Tolerances are those of
the element-wise parity tests: about ten times the rounding of the storage precision.
"""
import numpy as np
import pytest

import synthetic
from oracle import sap as osap
from oracle import wilson

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-6, "f16": 1e-3, "f16l": 1e-3}


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1502_04025_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "f16l"])
@pytest.mark.parametrize("dims,block,nmr", [((8, 4, 4, 12), (2, 2, 2, 2), 1), ((8, 8, 8, 8), (4, 4, 4, 4), 5),
                                            ((16, 8, 8, 8), (8, 4, 4, 4), 1)])
def test_three_kappas_share_the_waves(ctx, dims, block, nmr, prec):
    kap = [0.125, 0.118, 0.121]
    u = synthetic.gauge_field(dims, 0.3, 81)
    eta = synthetic.gaussian_source(dims, len(kap), 82)
    t = wilson.clover_term(u, 1.0)
    f = ctx.load_gauge(u, block)
    f.compute_clover(1.0)
    out = f.sap(np.array(kap), eta, nmr=nmr, ncy=2, prec=prec)
    f.free()
    for r, k in enumerate(kap):
        ref = osap.sap(osap.BlockSystem(u, t, k, block), eta[r], 2, nmr)
        d = out[r] - ref
        assert np.linalg.norm(d) <= TOL[prec] * np.linalg.norm(ref), (r, prec)
        assert np.abs(d).max() <= 4 * TOL[prec] * np.abs(ref).max(), (r, prec)


@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_same_bits_from_either_form_of_the_launch(ctx, prec):
    """40 right-hand sides on 8 domains of a colour are 320 workgroups, which takes the FP32
    kernel's form for more than one workgroup per CU; one right-hand side takes the other."""
    dims, block = (16, 8, 8, 8), (8, 4, 4, 4)
    f = ctx.load_gauge(synthetic.gauge_field(dims, 0.3, 83), block)
    f.compute_clover(1.0)
    eta = synthetic.gaussian_source(dims, 40, 84)
    out = f.sap(0.123, eta, nmr=3, ncy=2, prec=prec)
    for r in (0, 17, 39):
        assert np.array_equal(out[r], f.sap(0.123, eta[r], nmr=3, ncy=2, prec=prec)), r
    f.free()


@pytest.mark.parametrize("dims,block", [((4, 4, 4, 4), (2, 2, 2, 2)), ((8, 8, 8, 8), (4, 4, 4, 4))])
def test_clover_inverse_with_row_exchanges(ctx, dims, block):
    """The 6x6 inverses where pivoting matters: a clover term that puts 1e-3 on the diagonal of
    1 + kappa T beside off-diagonal entries of order one. The bound is rounding times the
    condition number (below 1e5 here) times the few operations per entry: 1e-10."""
    kappa = 0.12
    lead = dims[::-1]
    rng = np.random.default_rng(85)
    t = np.zeros(lead + (12, 12), dtype=np.complex128)
    for k in range(2):
        g = rng.standard_normal(lead + (6, 6)) + 1j * rng.standard_normal(lead + (6, 6))
        h = g + np.conj(np.swapaxes(g, -1, -2))
        i = np.arange(6)
        h[..., i, i] = (1e-3 - 1.0) / kappa
        off = ~np.eye(6, dtype=bool)
        h[..., off] /= kappa
        t[..., 6 * k:6 * k + 6, 6 * k:6 * k + 6] = h
    assert np.linalg.cond(np.eye(12) + kappa * t).max() < 1e5
    u = synthetic.gauge_field(dims, 0.3, 86)
    eta = synthetic.gaussian_source(dims, 1, 87)
    f = ctx.load_gauge(u, block)
    f.load_clover(t)
    out = f.sap(kappa, eta, nmr=1, ncy=1, prec="f64")
    f.free()
    ref = osap.sap(osap.BlockSystem(u, t, kappa, block), eta[0], 1, 1)
    assert np.linalg.norm(out[0] - ref) <= 1e-10 * np.linalg.norm(ref)
