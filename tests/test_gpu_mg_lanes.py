"""The multigrid kernels at the sizes where their lane sums and their sharing of the stencil
change form: numbers of test vectors on both sides of each power of two, and one to six
systems solved together (a workgroup of the coarse operator takes one, two or four)."""
import numpy as np
import pytest

from oracle import mg as omg
from test_gpu_mg import _dense_from_stencil, _fields_from_cols, _setup, ctx  # noqa: F401

pytestmark = pytest.mark.gpu
DIMS, BLOCK, GRID = (8, 8, 8, 8), (4, 4, 4, 4), (2, 2, 2, 2)


@pytest.mark.parametrize("nvec", [6, 10, 16])
def test_coarse_operator_matches_oracle(ctx, nvec):  # noqa: F811
    print(f"mg P and D_c with {nvec} test vectors", flush=True)
    from paper_1502_04025_amd import Multigrid
    u, t, f, vecs = _setup(ctx, DIMS, BLOCK, nvec=nvec, seed=71)
    mg = Multigrid(f, 0.128, vecs, setup_iters=0, coarse_iters=4, prec="f64")
    cols = omg.prolongator(list(vecs), BLOCK)
    p_ref = _fields_from_cols(cols, nvec)
    # P and D_c are stored in FP32: one rounding of P, K <= 32 products of two of them in D_c
    assert np.abs(mg.prolongator() - p_ref).max() <= 1e-6 * np.abs(p_ref).max()
    ref = omg.coarse_dense(u, t, 0.128, cols, BLOCK)
    assert np.abs(_dense_from_stencil(mg.coarse_operator(), GRID) - ref).max() <= 1e-5 * np.abs(ref).max()
    mg.close()
    f.free()


@pytest.mark.parametrize("nvec,iters", [(2, 8), (6, 12), (16, 20)])
def test_coarse_solves_together_and_alone(ctx, nvec, iters):  # noqa: F811
    """Every system of a coarse solve has the same bits alone and with any others, in both
    forms of the Arnoldi step, and they follow GMRES with the stored operator: FP32 vectors of
    `iters` steps, each rounded once to 6e-8."""
    print(f"mg coarse solves with {nvec} test vectors, GMRES({iters})", flush=True)
    from paper_1502_04025_amd import Multigrid
    _, _, f, vecs = _setup(ctx, DIMS, BLOCK, nvec=nvec, seed=73)
    rng = np.random.default_rng(11)
    shape = (6, 2, 2, 2, 2, 2 * nvec)
    rhs = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    for form in (0, 1):
        mg = Multigrid(f, 0.128, vecs, setup_iters=0, coarse_iters=iters, prec="f64", coarse_form=form)
        dense = _dense_from_stencil(mg.coarse_operator(), GRID)
        alone = [mg.coarse_solve(rhs[i:i + 1])[0] for i in range(6)]
        for n in range(2, 7):
            got = mg.coarse_solve(rhs[6 - n:])
            for i in range(n):
                np.testing.assert_array_equal(got[i], alone[6 - n + i])
        for i in range(2):
            ref = omg.gmres_fixed(lambda v: (dense @ v.ravel()).reshape(v.shape), rhs[i], iters)
            assert np.linalg.norm(alone[i] - ref) <= 1e-4 * np.linalg.norm(ref)
        mg.close()
    f.free()
