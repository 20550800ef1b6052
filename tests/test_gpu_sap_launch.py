"""The FP32 Schwarz kernel's launches for one right-hand side on lattices that fill the chip.

Up to two right-hand sides on 8x4^3 domains take the form with the even sites' clover in LDS, and
one on 4^4 domains, from 512 workgroups on, a launch with LDS for one workgroup per CU; more
right-hand sides take the others. Neither changes an operation: the same bits alone and with
three, where the lattice has more than 256 workgroups of a colour (8x4^3) or 512 (4^4).
"""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block", [((16, 24, 24, 32), (8, 4, 4, 4)), ((16, 16, 32, 32), (4, 4, 4, 4)),
                                        ((16, 16, 24, 48), (4, 4, 4, 4))])
def test_same_bits_alone_and_with_three(dims, block):
    import torch
    from paper_1502_04025_amd import Context
    assert torch.cuda.is_available()
    c = Context(0)
    f = c.load_gauge(torch.from_numpy(synthetic.gauge_field(dims, 0.3, 121)).cuda(), block)
    f.compute_clover(1.0)
    eta = torch.from_numpy(synthetic.gaussian_source(dims, 3, 122)).cuda()
    out = f.sap(0.123, eta, nmr=2, ncy=2, prec="f32")
    ref = f.sap(0.123, eta, nmr=2, ncy=2, prec="f64")
    err = torch.linalg.vector_norm(out - ref) / torch.linalg.vector_norm(ref)
    one = [f.sap(0.123, eta[r:r + 1].contiguous(), nmr=2, ncy=2, prec="f32") for r in range(3)]
    two = f.sap(0.123, eta[:2].contiguous(), nmr=2, ncy=2, prec="f32")
    f.free()
    c.close()
    assert err.item() <= 1e-6
    for r in range(3):
        assert np.array_equal(one[r][0].cpu().numpy(), out[r].cpu().numpy()), r
    assert np.array_equal(two.cpu().numpy(), out[:2].cpu().numpy())
