"""Adaptive steps whose projected matrices outgrow the leading-eigenpair solver (512)
and then a cooperative Jacobi grid of all modes at once (982 of three modes), with
modes that stay below.  At the last step every basis spans its mode's space, so the
factors are the leading eigenvectors of X_(n) X_(n)^T; the error (second order in a
factor's) agrees to 1e-10, as in test_gpu_parity.py."""
import numpy as np
import pytest

from oracle.tensor import project_core

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,ranks,q", [((1000, 34, 33), (45, 25, 8), 19), ((600, 40, 30), (45, 8, 9), 11)])
def test_wide_steps(dims, ranks, q):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(5).standard_normal(dims)
    core, factors, err, used = rb.tucker_adaptive(torch.from_numpy(X).to("cuda"), ranks, p=5, max_q=q, fit_tol=-1.0,
                                                  seed=4)
    exact = []
    for n, R in enumerate(ranks):
        Xn = np.moveaxis(X, n, 0).reshape(dims[n], -1)
        exact.append(np.linalg.eigh(Xn @ Xn.T)[1][:, ::-1][:, :R])
    ref = np.sqrt(1 - np.sum(project_core(X, exact) ** 2) / np.sum(X ** 2))
    assert used == q
    assert abs(err - ref) <= 1e-10 * ref
    for U in factors:
        U = U.double().cpu().numpy()
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 1e-10
