"""Modes of low rank (fewer columns than the Krylov basis has directions), where a block's
last vectors are rounding noise after the projection: the basis is orthonormal to 1e-13
(a kept vector has at least a tenth of its length left in the second pass, so rounding
is amplified a hundredfold at most) and, where it spans the columns, the error is that of the
leading singular vectors to 1e-10 (float32 1e-5, as in test_gpu_parity.py).  Several
seeds each: which noise vectors pass the first tests is a matter of rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    ((128, 33), (10, 2), 2, 3), ((300, 61), (20, 2), 5, 3), ((64, 7, 7), (8, 2, 2), 5, 4), ((500, 90), (30, 2), 10, 3),
    ((1400, 129), (30, 3), 10, 4), ((90, 3, 3), (4, 2, 2), 1, 5), ((400, 150), (100, 2), 30, 1),
]


@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
@pytest.mark.parametrize("dims,ranks,p,q", CASES)
def test_basis_and_error(dims, ranks, p, q, dtype):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    J = int(np.prod(dims[1:]))
    for seed in range(12):
        X = np.random.default_rng(seed).standard_normal(dims)
        Xg = torch.from_numpy(X).to("cuda", getattr(torch, dtype))
        Qt, width = rb.basis(Xg, 0, ranks, p=p, q=q, seed=seed)
        Q = Qt[:width].cpu().numpy()
        assert np.abs(Q @ Q.T - np.eye(width)).max() <= 1e-13, seed
        if dtype == "bfloat16" or len(dims) > 2:
            continue
        core, factors, err = rb.tucker(Xg, ranks, p=p, q=q, seed=seed)
        assert width >= J
        X = Xg.double().cpu().numpy()
        U = np.linalg.svd(X, full_matrices=False)[0][:, :ranks[0]]
        V = factors[1].double().cpu().numpy()
        ref = np.linalg.norm(X - U @ (U.T @ X @ V) @ V.T) / np.linalg.norm(X)
        assert abs(err - ref) <= (1e-10 if dtype == "float64" else 1e-5) * ref, seed


def test_block_that_was_wrong():
    """The case in which it was seen: 33 columns, a signal 20 times the noise."""
    import torch
    import paper_2211_14828_amd as rb
    g = torch.Generator().manual_seed(737)
    X = torch.randn((128, 33), generator=g, dtype=torch.float64)
    for c in range(3):
        v = [torch.cos((c + 1.0) * 1.7 * torch.arange(d, dtype=torch.float64) + c) for d in (128, 33)]
        X = X + 3.0 / (c + 1) * torch.outer(*v)
    _, factors, err = rb.tucker(X.cuda(), [10, 2], p=2, q=3, seed=234706231126)
    U = factors[0].cpu().numpy()
    assert np.abs(U.T @ U - np.eye(10)).max() <= 1e-12
    assert abs(err - 0.54113922868850) <= 1e-9
