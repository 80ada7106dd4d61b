"""The tridiagonal reduction of the leading-eigenpair solver at the edges of its
register layout: orders around the multiples of 64, where one workgroup gives
way to two, two to four and four to eight, graded spectra whose trailing rows
are tiny, and matrices of different orders in one launch.  Tolerances as for the
other orders: eigenvalues to a few n u lambda_max (the backward error of
Householder reduction), vectors orthonormal to float64, errors to 1e-10."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

ORDERS = [4, 8, 9, 16, 62, 66, 127, 129, 164, 165, 166, 191, 192, 193, 255, 257, 319, 320, 321, 383, 384, 385, 447, 511]


@pytest.mark.parametrize("n", ORDERS)
def test_leading_pairs_at_layout_edges(n):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    rng = np.random.default_rng(n)
    k = max(1, n // 5)
    B = rng.standard_normal((n, n + 3))
    for Z in (B @ B.T, np.outer(s := 0.8 ** np.arange(n), s) * (B @ B.T)):
        lam, Vt = rb.sym_eig_top(torch.from_numpy(Z).cuda(), k)
        lam, V = lam.cpu().numpy(), Vt.cpu().numpy().T
        w = np.linalg.eigvalsh(Z)[::-1]
        assert np.max(np.abs(lam - w[:k])) <= 4 * n * 2.0 ** -52 * w[0]
        assert np.linalg.norm(V.T @ V - np.eye(k), 2) <= 1e-12
        assert np.linalg.norm(Z @ V - V * lam, axis=0).max() <= 1e-12 * w[0]


@pytest.mark.parametrize("dims,ranks,p,q", [
    ((60, 50, 300), (10, 20, 80), 5, 1),     # bases of 30, 50 and 170 columns: one and two workgroups
    ((90, 300, 310), (20, 90, 130), 8, 1),   # 56, 196 and 276: one, two and four
])
def test_orders_together(dims, ranks, p, q):
    import torch
    import paper_2211_14828_amd as rb
    X = np.random.default_rng(sum(dims)).standard_normal(dims)
    _, _, err = rb.tucker(torch.from_numpy(X).cuda(), ranks, p=p, q=q, seed=4)
    _, _, ref = rbki_tucker(X, ranks, p, q, 4)
    assert abs(err - ref) <= 1e-10 * ref, (err, ref)
