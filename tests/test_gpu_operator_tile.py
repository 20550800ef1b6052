"""The operator on blocks whose spinors pass through LDS: every right-hand side has the same bits
alone and among others (both ways of dealing the blocks to the XCDs), and follows the oracle
where the hops leave a tile: sources on the corners of tiles and next to the lattice's faces."""
import numpy as np
import pytest

import synthetic
from oracle import wilson
from test_gpu_operator import TOL, ctx, relerr  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture
def setup(ctx):  # noqa: F811
    fields = []

    def make(dims, block):
        u = synthetic.gauge_field(dims, 0.3, 5)
        f = ctx.load_gauge(u, block)
        f.compute_clover(1.0)
        fields.append(f)
        return u, wilson.clover_term(u, 1.0), f

    yield make
    for f in fields:
        f.free()


@pytest.mark.parametrize("dims,block", [((8, 8, 16, 24), (4, 4, 4, 4)), ((32, 8, 8, 16), (8, 4, 4, 4))])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_operator_alone_and_in_a_batch(setup, dims, block, prec):
    print(f"D tile {dims} {block} {prec}", flush=True)
    u, t, f = setup(dims, block)
    psi = synthetic.gaussian_source(dims, 6, 9)
    psi[1] = 0
    lx, ly, lz, lt = dims
    for x in (0, block[0] - 1, block[0], lx - 1):
        for tt in (0, 1, 2, 3, 4, lt - 1):
            psi[1, tt, (tt * block[2]) % lz, ly - 1 if tt % 2 else 0, x, tt % 4, x % 3] = 1 + 1j
    out = f.apply_D(0.124, psi, prec=prec)
    for r in range(6):
        np.testing.assert_array_equal(f.apply_D(0.124, psi[r:r + 1], prec=prec)[0], out[r])
    for r in (1, 5):
        assert relerr(out[r], wilson.apply_M(u, t, 0.124, psi[r])) <= TOL[prec]


@pytest.mark.parametrize("shift", [0, 1])
def test_operators_on_overlapping_arrays(setup, shift):
    """The output may be the input, or overlap it by some of its right-hand sides."""
    import torch
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    _, _, f = setup(dims, block)
    psi = torch.from_numpy(synthetic.gaussian_source(dims, 9, 12)).cuda()
    torch.cuda.synchronize()
    for call in (f.apply_D, f.apply_block_D, lambda *a, **k: f.apply_block_D(*a, links12=True, **k)):
        ref = call(0.124, psi[:8].clone(), prec="f32")
        x = psi.clone()
        torch.cuda.synchronize()
        call(0.124, x[:8], prec="f32", out=x[shift:8 + shift])
        assert torch.equal(x[shift:8 + shift], ref)
