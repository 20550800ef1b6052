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
from oracle.gamma import GAMMA

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


def odd_from_even(u, eta, kappa, psi, block, dtype):
    """eta + kappa (hops from other blocks) + kappa (hops inside the block) of psi, in dtype."""
    dims = lat.dims_of(eta)
    u, psi, out = u.astype(dtype), psi.astype(dtype), eta.astype(dtype)
    for inside in (False, True):
        h = np.zeros_like(out)
        for mu in range(4):
            g, um = GAMMA[mu].astype(dtype), u[..., mu, :, :]
            for back in (False, True):
                chi = lat.shift_bwd(psi, mu, True) if back else lat.shift_fwd(psi, mu, True)
                gchi = (g[:, :, None] * chi[..., None, :, :]).sum(axis=-2)  # one entry a row: exact
                half = chi + gchi if back else chi - gchi
                v = np.conj(np.swapaxes(lat.shift_bwd(um, mu), -1, -2)) if back else um
                hop = np.einsum("...ab,...sb->...sa", v, half)
                keep = (lat.internal_bwd if back else lat.internal_fwd)(dims, block, mu) == inside
                h = h + hop * keep[..., None, None].astype(dtype)
        out = out + dtype(kappa) * h
    return out


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dims,block", [((8, 8, 8, 8), (2, 2, 2, 2)), ((8, 8, 8, 8), (4, 4, 4, 4)),
                                        ((16, 8, 8, 8), (8, 4, 4, 4))])
def test_odd_correction_follows_the_even_one(ctx, dims, block, prec):
    """After one cycle the odd sites of the second colour solve their own equation exactly, given
    psi on the even sites; without a clover term it reads psi_o = eta_o + kappa H psi_e. Links,
    source and kappa are FP32 numbers, so the arithmetic alone makes the error."""
    kappa = 0.125
    low, high = (np.complex64, np.complex128) if prec == "f32" else (np.complex128, np.clongdouble)
    u = synthetic.gauge_field(dims, 0.3, 103).astype(np.complex64).astype(np.complex128)
    eta = synthetic.gaussian_source(dims, 1, 104)[0].astype(np.complex64).astype(np.complex128)
    f = ctx.load_gauge(u, block)
    f.compute_clover(0.0)
    psi = f.sap(kappa, eta, nmr=6, ncy=1, prec=prec)
    f.free()
    at = (lat.parity(dims) == 1) & (lat.block_colour(dims, block) == 1)
    exact = odd_from_even(u, eta, kappa, psi, block, high)[at]
    plain = odd_from_even(u, eta, kappa, psi, block, low)[at]
    err = [float(np.sqrt((np.abs(x - exact) ** 2).sum())) for x in (psi[at], plain)]
    print(f"{block} {prec}: device {err[0]:.4e} numpy {err[1]:.4e}", flush=True)
    assert err[0] <= SLACK * err[1]
