"""Sketch values made inside the Gram kernel (float32 modes of at most 64 rows): rows
that start at even and odd indices of the stream, slabs shorter and longer than a K
tile, whole and partial tiles, all 64 sketch rows and one, and a sampled unfolding.
The sketch alone shows in a basis without Krylov steps (q = 0) of fewer columns than
the mode has: that basis has to contain X Omega of the float64 oracle's stream, to
1e-4 of each column's norm (float32 products, 1e-6, over the smallest singular value
of the Gaussian block, above 1e-2 of the largest at these shapes)."""
import numpy as np
import pytest

from oracle.philox import omega
from oracle.tensor import unfold

pytestmark = pytest.mark.gpu

CASES = [((64, 33, 16), 0, 20), ((64, 33, 16), 2, 10), ((21, 50, 9), 1, 30), ((21, 50, 9), 0, 3), ((7, 63, 33), 1, 58),
         ((9, 64, 3), 1, 17), ((11, 13, 64), 2, 40), ((5, 64, 47), 1, 59)]


@pytest.mark.parametrize("dims,mode,rank", CASES)
def test_basis_spans_the_sketch(dims, mode, rank):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims) + mode).standard_normal(dims).astype(np.float32)
    ranks = [1] * len(dims)
    ranks[mode] = rank
    Qt, width = rb.basis(torch.from_numpy(X).to("cuda"), mode, ranks, p=1, q=0, seed=31)
    Q = Qt[:width].cpu().numpy()
    Xn = unfold(X.astype(np.float64), mode)
    W = Xn @ omega(31, mode, Xn.shape[1], rank + 1)
    off = W - Q.T @ (Q @ W)
    assert np.linalg.norm(off, axis=0).max() <= 1e-4 * np.linalg.norm(W, axis=0).min()
