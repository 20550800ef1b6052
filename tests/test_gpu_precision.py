"""Rounding errors of the device code held to those of a plain evaluation of the same formula.

Each test takes the exact result from extended precision and compares two errors: that of
the device and that of NumPy evaluating the formula once in the device's arithmetic. The
device may be 15% further off: it orders sums differently and fuses multiplications, while
one rounding too many per entry adds 30% or more.
"""
import numpy as np
import pytest

import synthetic
from oracle import lattice as lat

pytestmark = pytest.mark.gpu

SLACK = 1.15


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1502_04025_amd import Context
    c = Context(0)
    yield c
    c.close()


def gauss_jordan(a):
    """Inverses of a[n, 6, 6] with partial pivoting, Hermitian matrices: the mean of both
    triangles."""
    n = np.arange(len(a))
    a = a.copy()
    inv = np.broadcast_to(np.eye(6, dtype=a.dtype), a.shape).copy()
    for c in range(6):
        p = c + np.argmax(np.abs(a[:, c:, c]) ** 2, axis=1)
        for m in (a, inv):
            top = m[:, c].copy()
            m[:, c] = m[n, p]
            m[n, p] = top
        q = 1 / a[:, c, c]
        a[:, c] *= q[:, None]
        inv[:, c] *= q[:, None]
        for r in range(6):
            if r != c:
                f = a[:, r, c].copy()[:, None]
                a[:, r] -= f * a[:, c]
                inv[:, r] -= f * inv[:, c]
    return (inv + np.conj(np.swapaxes(inv, 1, 2))) / 2


@pytest.mark.parametrize("block", [(2, 2, 2, 2), (4, 4, 4, 4)])
def test_clover_inverse(ctx, block):
    """With all links zero a Schwarz sweep gives (1 + kappa T)^-1 eta on the odd sites, so unit
    sources show the inverse itself."""
    dims, kappa = (8, 8, 8, 8), 0.12
    lead = dims[::-1]
    rng = np.random.default_rng(101)
    g = rng.standard_normal(lead + (2, 6, 6)) + 1j * rng.standard_normal(lead + (2, 6, 6))
    h = 0.05 * (g + np.conj(np.swapaxes(g, -1, -2)))
    t = np.zeros(lead + (12, 12), dtype=np.complex128)
    for k in range(2):
        t[..., 6 * k:6 * k + 6, 6 * k:6 * k + 6] = h[..., k, :, :] / kappa
    eta = np.zeros((12,) + lead + (4, 3), dtype=np.complex128)
    for k in range(12):
        eta[k, ..., k // 3, k % 3] = 1
    f = ctx.load_gauge(np.zeros(lead + (4, 3, 3), dtype=np.complex128), block)
    f.load_clover(t)
    out = f.sap(kappa, eta, nmr=1, ncy=1, prec="f64")
    f.free()
    odd = lat.parity(dims) == 1
    got = np.moveaxis(out.reshape((12,) + lead + (12,)), 0, -1)[odd]
    for k in range(2):
        s = slice(6 * k, 6 * k + 6)
        a = np.eye(6) + kappa * t[odd][:, s, s]
        exact = gauss_jordan(a.astype(np.clongdouble))
        err = [float(np.linalg.norm((x - exact).astype(np.complex128))) for x in (got[:, s, s], gauss_jordan(a))]
        print(f"{block} chirality {k}: device {err[0]:.4e} numpy {err[1]:.4e}", flush=True)
        assert err[0] <= SLACK * err[1]
