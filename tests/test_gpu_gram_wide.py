"""The wide float32 Gram form (256 x 256 tiles) at its edges, against the float64
oracle: one row past 128, whole and partly filled tiles, K tiles of 16 that a slab
exceeds by one value or just fills, K tiles of several slabs with a remainder (thin
trailing dimensions, the last mode), an unfolding shorter than a K tile, and
sketches of one, two and three groups beyond the 64 columns that the diagonal
tiles take.  White noise; tolerance on the reconstruction error as in
test_gpu_parity.py (float32 1e-5 relative)."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

CASES = [
    # last mode, rows across the lanes
    ((20, 6, 129), (5, 4, 9), 6), ((21, 7, 256), (5, 4, 9), 6), ((9, 17, 250), (5, 4, 60), 4), ((7, 2, 200), (3, 2, 8), 3),
    # several slabs to a K tile (16 / 3 and 16 / 15 of them)
    ((9, 200, 3), (4, 9, 2), 5), ((9, 200, 15), (4, 9, 5), 5),
    # slabs of one K tile, one value more, and one less than two
    ((4, 512, 16), (3, 20, 5), 5), ((3, 390, 17), (2, 12, 5), 5), ((5, 449, 31), (3, 12, 5), 5),
    # nine tiles of rows and columns; a matrix
    ((700, 90), (30, 20), 8),
    # sketches of 140 and 200 columns
    ((400, 450), (130, 20), 10), ((450, 400), (190, 20), 10),
]


@pytest.mark.parametrize("dims,ranks,p", CASES)
def test_wide_tiles_match_oracle(dims, ranks, p):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims).astype(np.float32)
    _, factors, err = rb.tucker(torch.from_numpy(X).to("cuda"), ranks, p=p, q=1, seed=13)
    X = X.astype(np.float64)
    _, exact, ref = rbki_tucker(X, ranks, p, 1, 13)
    assert abs(err - ref) <= 1e-5 * ref, (err, ref)
    for U, V in zip(factors, exact):
        U = U.double().cpu().numpy()
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 1e-5
