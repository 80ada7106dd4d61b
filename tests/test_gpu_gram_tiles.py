"""Gram and sketch products at the edges of their tiles, against the float64
oracle: row counts around the 32-, 64-, 128- and 256-row boundaries, K tiles
that a slab does not fill, K tiles of several slabs (thin trailing dimensions,
the last mode) with and without a remainder, and unfoldings shorter than a K
tile.  White noise, so that every entry of X_(n) X_(n)^T moves the factors.

Tolerances (relative, on the reconstruction error, as in test_gpu_parity.py):
float64 1e-10, float32 1e-5; bfloat16 products 1e-3."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

TOL = {"float64": 1e-10, "float32": 1e-5, "bfloat16": 1e-3}

SHAPES = [
    (33, 65, 31),        # one past 32 and 64; slabs shorter than a K tile
    (64, 64, 64),        # thin tiles filled
    (63, 129, 32),       # a 128-row tile and one row; slab of exactly one float32 K tile
    (257, 40, 33),       # past 256 sketch columns; slab of one K tile and one value
    (50, 40, 7),         # four slabs to a float32 K tile, the last tile overlapping
    (2, 70, 7),          # fewer slabs than a K tile takes
    (3, 70, 5),          # an unfolding shorter than a K tile
    (40, 6, 90, 3),      # thin trailing dimension below a tall mode
    (1, 140, 130),       # a mode of one row
    (300, 90),           # a matrix
]


@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
@pytest.mark.parametrize("dims", SHAPES)
def test_tucker_at_tile_edges(dims, dtype):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims)
    Xg = torch.from_numpy(X).to({"float64": torch.float64, "float32": torch.float32, "bfloat16": torch.bfloat16}[dtype])
    T = int(np.prod(dims))
    ranks = [min(9, d, T // d) for d in dims]
    core, factors, err = rb.tucker(Xg.to("cuda"), ranks, p=6, q=1, seed=11)
    _, _, ref = rbki_tucker(Xg.double().numpy(), ranks, 6, 1, 11)
    assert abs(err - ref) <= TOL[dtype] * ref, (err, ref)
    for U in factors:
        U = U.double().cpu().numpy()
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 1e-5


def test_wide_sketches():
    """Sketches of more than 64 and more than 128 columns."""
    import torch
    import paper_2211_14828_amd as rb
    X = np.random.default_rng(3).standard_normal((150, 140, 20)).astype(np.float32)
    core, factors, err = rb.tucker(torch.from_numpy(X).to("cuda"), [90, 130, 12], p=5, q=1, seed=4)
    _, _, ref = rbki_tucker(X.astype(np.float64), [90, 130, 12], 5, 1, 4)
    assert abs(err - ref) <= 1e-5 * ref, (err, ref)
