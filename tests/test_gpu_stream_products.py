"""Streaming mode products and the streaming error pass at the edges of their
pieces, through whole decompositions against the float64 oracle: slabs of 1 to
9 values, inner dimensions below, at and past a stage, ranks around the 16-row
blocks and past 64 and 128, few and many rows in the last mode.  Tolerances on
the reconstruction error as in test_gpu_parity.py; the core is compared with
X x_n U_n^T of the returned factors in float64 (float32 products: 1e-5 of the
core's norm, the size of a few thousand float32 roundings)."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker
from oracle.tensor import project_core

pytestmark = pytest.mark.gpu

CASES = [
    ((70, 66, 9), (16, 17, 4)), ((65, 40, 5), (15, 33, 5)), ((40, 50, 3), (20, 30, 3)), ((40, 50, 2), (20, 30, 2)),
    ((90, 6, 4), (20, 3, 2)), ((150, 140, 21), (70, 48, 11)), ((150, 160, 12), (140, 130, 7)), ((15, 17, 300), (5, 6, 31)),
    ((130, 129, 131), (7, 65, 3)), ((3, 200, 129), (3, 12, 49)), ((300, 61), (30, 29)), ((20, 19, 18, 17), (8, 7, 6, 5)),
]


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("dims,ranks", CASES)
def test_products_and_error(dims, ranks, dtype):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims) + 1).standard_normal(dims).astype(dtype)
    core, factors, err = rb.tucker(torch.from_numpy(X).to("cuda"), ranks, p=4, q=1, seed=6)
    X = X.astype(np.float64)
    _, _, ref = rbki_tucker(X, ranks, 4, 1, 6)
    assert abs(err - ref) <= (1e-10 if dtype == np.float64 else 1e-5) * ref, (err, ref)
    G = project_core(X, [U.double().cpu().numpy() for U in factors])
    off = np.linalg.norm(core.double().cpu().numpy() - G) / np.linalg.norm(G)
    assert off <= (1e-12 if dtype == np.float64 else 1e-5), off
