"""The blocked CholeskyQR step at the edges of its panels: sketches of one column,
around 16, 32, 48, 64 and 96 columns and of one more than it takes, rows that do not
fill a workgroup's 64, full rank and (the drop rule) a tensor of lower rank than the
sketch.  The basis is orthonormal to 1e-13 sqrt(S') (two float64 passes) and spans the
sketch's image of the float64 oracle, X X^T X Omega too, to 1e-10."""
import numpy as np
import pytest

from oracle.philox import omega

pytestmark = pytest.mark.gpu

SIZES = [(9, 1), (70, 2), (63, 15), (64, 16), (65, 17), (130, 31), (100, 33), (120, 48), (190, 49), (129, 64), (200, 65),
         (140, 80), (150, 95), (193, 96), (230, 97),
         # G formed by the step itself (few columns) and just past it
         (3, 2), (512, 14), (513, 14), (256, 20), (257, 20), (128, 40), (129, 40), (76, 64), (77, 64)]


@pytest.mark.parametrize("deficient", [False, True])
@pytest.mark.parametrize("I,S", SIZES)
def test_basis_at_panel_edges(I, S, deficient):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    rng = np.random.default_rng(1000 * I + S)
    J = 2 * I + 30
    X = rng.standard_normal((I, J))
    if deficient:
        r = max(1, S // 3)
        X = rng.standard_normal((I, r)) @ rng.standard_normal((r, J))
    Qt, width = rb.basis(torch.from_numpy(X).cuda(), 0, [S, 1], p=0, q=1, seed=5)
    Q = Qt.cpu().numpy()
    kept = Q[np.abs(Q).max(axis=1) > 0]
    assert np.linalg.norm(kept @ kept.T - np.eye(len(kept)), 2) <= 1e-13 * np.sqrt(len(kept)) * 10
    if deficient:
        assert len(kept) == r
    W = X @ omega(5, 0, J, S)
    for B in (W, X @ (X.T @ W)):
        B = B / np.linalg.norm(B, axis=0)
        assert np.linalg.norm(B - kept.T @ (kept @ B), axis=0).max() <= 1e-10
