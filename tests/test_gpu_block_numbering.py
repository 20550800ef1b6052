"""The block operator's workgroup numbering for several right-hand sides.

A block's right-hand sides follow each other on one XCD, and their kernel is another instance
than that of a single right-hand side. Three of them, over every domain shape and precision,
on grids of 32 to 96 blocks with unequal extents: each against the oracle's M_B, so that a
block or a field taken for another one shows, and each with the bits it has alone.
Tolerances as for one right-hand side: the rounding of the storage precision.
"""
import numpy as np
import pytest

import synthetic
from oracle import wilson

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 5e-3}

CASES = [((4, 4, 8, 12), (2, 2, 2, 2)), ((8, 8, 24, 8), (4, 4, 4, 4)), ((16, 8, 8, 16), (8, 4, 4, 4))]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1502_04025_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dims,block", CASES)
@pytest.mark.parametrize("links12", [False, True])
def test_three_right_hand_sides(ctx, dims, block, links12):
    u = synthetic.gauge_field(dims, 0.3, 111)
    psi = synthetic.gaussian_source(dims, 3, 112)
    t = wilson.clover_term(u, 1.0)
    ref = [wilson.apply_M(u, t, 0.126, p, block=block) for p in psi]
    f = ctx.load_gauge(u, block)
    f.compute_clover(1.0)
    for prec in ("f32", "f16") if links12 else ("f64", "f32", "f16"):
        out = f.apply_block_D(0.126, psi, prec=prec, links12=links12)
        for r in range(3):
            assert np.linalg.norm(out[r] - ref[r]) <= TOL[prec] * np.linalg.norm(ref[r]), (prec, r)
            assert np.array_equal(out[r], f.apply_block_D(0.126, psi[r], prec=prec, links12=links12)), (prec, r)
    f.free()
