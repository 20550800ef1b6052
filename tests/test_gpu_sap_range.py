"""The Schwarz sweep on inputs whose domain norms reach the bottom of the arithmetic's range.

The MR step length is <p, r> / <p, p>. Where <p, p> is positive but below the reciprocal of
the largest number (2.9e-39 in FP32), 1 / <p, p> is infinite though the quotient is of order
one. With a point source and a small kappa the front of the sweep passes through that range
(oracle sweeps with FP32 step lengths: 256 to 2560 sites in it); in FP64 a source of size
2^-520 is there at once. The results have to be finite and as close to the oracle as any
other sweep; the far domains weigh nothing in the norm.
"""
import numpy as np
import pytest

import synthetic
from oracle import sap as osap
from oracle import wilson

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-6, "f16": 1e-3, "f16l": 1e-3}

CASES = [((8, 8, 8, 32), (4, 4, 4, 4), 0.02, 4), ((16, 8, 8, 24), (8, 4, 4, 4), 0.01, 3),
         ((4, 4, 4, 32), (2, 2, 2, 2), 0.03, 7)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1502_04025_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dims,block,kappa,ncy", CASES)
def test_point_source_front(ctx, dims, block, kappa, ncy):
    u = synthetic.gauge_field(dims, 0.3, 91)
    eta = synthetic.point_sources(dims)[0]
    t = wilson.clover_term(u, 1.0)
    ref = osap.sap(osap.BlockSystem(u, t, kappa, block), eta, ncy, 2)
    f = ctx.load_gauge(u, block)
    f.compute_clover(1.0)
    out = {p: f.sap(kappa, eta, nmr=2, ncy=ncy, prec=p) for p in TOL}
    f.free()
    for p in TOL:
        bad = int((~np.isfinite(out[p])).any(axis=(-1, -2)).sum())
        print(f"{dims} {block} {p}: {bad} sites not finite", flush=True)
    for p in TOL:
        assert np.isfinite(out[p]).all(), p
        assert np.linalg.norm(out[p] - ref) <= TOL[p] * np.linalg.norm(ref), p


@pytest.mark.parametrize("dims,block", [((4, 4, 4, 8), (2, 2, 2, 2)), ((8, 8, 8, 8), (4, 4, 4, 4)),
                                        ((16, 8, 8, 8), (8, 4, 4, 4))])
def test_small_source_fp64(ctx, dims, block):
    """The sweep scales with its source; a factor of a power of two changes no mantissa. The
    squares in the inner products are about 2^-1040, where FP64 numbers are 2^-1074 apart: each
    step length is off by at most 2^-33, and a psi of 2 cycles of 2 steps on 2 colours by 1e-9."""
    u = synthetic.gauge_field(dims, 0.3, 92)
    eta = synthetic.gaussian_source(dims, 1, 93)
    f = ctx.load_gauge(u, block)
    f.compute_clover(1.0)
    ref = f.sap(0.12, eta, nmr=2, ncy=2, prec="f64")
    out = f.sap(0.12, eta * 2.0 ** -520, nmr=2, ncy=2, prec="f64")
    f.free()
    assert np.isfinite(out).all()
    assert np.linalg.norm(out * 2.0 ** 520 - ref) <= 1e-9 * np.linalg.norm(ref)
