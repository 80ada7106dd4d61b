"""The float64 Gram form of 65 to 256 rows at its edges, against the float64 oracle:
one row past 64, whole and partly filled groups and blocks, one and two shares of the
blocks, sketches of one column, around 16 and 32 and of 64, slabs of exactly one K
tile, one value more and less, K tiles of several slabs with a remainder, the last
mode, an unfolding shorter than a K tile, and a sampled unfolding.  White noise;
reconstruction error to 1e-10 and basis orthonormality as in test_gpu_parity.py."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

CASES = [((65, 16, 3), (9, 4, 2), 1.0), ((128, 17), (12, 10), 1.0), ((129, 31), (27, 11), 1.0), ((3, 256, 16), (2, 26, 5), 1.0),
         ((5, 255, 33), (2, 59, 6), 1.0), ((9, 200, 3), (4, 11, 2), 1.0), ((9, 200, 15), (4, 10, 5), 1.0),
         ((20, 6, 97), (5, 4, 27), 1.0), ((21, 7, 256), (5, 4, 58), 1.0), ((7, 2, 160), (3, 2, 8), 1.0),
         ((70, 200, 40), (4, 9, 6), 0.25), ((250, 2, 3), (1, 1, 1), 1.0)]


@pytest.mark.parametrize("dims,ranks,rate", CASES)
def test_flat_form_matches_oracle(dims, ranks, rate):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims)
    _, factors, err = rb.tucker(torch.from_numpy(X).to("cuda"), ranks, p=5, q=1, seed=14, sample_rate=rate)
    _, _, ref = rbki_tucker(X, ranks, 5, 1, 14, sample_rate=rate)
    assert abs(err - ref) <= 1e-10 * ref, (err, ref)
    for U in factors:
        U = U.cpu().numpy()
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 1e-12
