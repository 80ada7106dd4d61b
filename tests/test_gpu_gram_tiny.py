"""Gram and sketch products of modes of at most eight rows, kept in registers:
against the float64 oracle, for slabs that a 16-byte piece divides, exceeds and does
not fit in, for the tiny mode first, in the middle and last, and with fewer K values
than a workgroup has threads.  White noise; tolerances on the reconstruction error
as in test_gpu_parity.py (float64 1e-10, float32 1e-5, bfloat16 products 1e-3)."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

TOL = {"float64": 1e-10, "float32": 1e-5, "bfloat16": 1e-3}
CASES = [((3, 90, 80), (2, 9, 8)), ((40, 4, 37), (6, 4, 5)), ((60, 50, 3), (9, 8, 2)), ((50, 8, 9), (7, 8, 4)),
         ((45, 7, 3), (6, 5, 2)), ((30, 5, 2, 31), (5, 4, 1, 6)), ((8, 8, 8), (5, 8, 6)), ((1, 300, 2), (1, 1, 1))]


@pytest.mark.parametrize("dtype", ["float64", "float32", "bfloat16"])
@pytest.mark.parametrize("dims,ranks", CASES)
def test_tiny_modes_match_oracle(dims, ranks, dtype):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims)
    Xg = torch.from_numpy(X).to({"float64": torch.float64, "float32": torch.float32, "bfloat16": torch.bfloat16}[dtype])
    _, factors, err = rb.tucker(Xg.to("cuda"), ranks, p=1, q=1, seed=17)
    _, _, ref = rbki_tucker(Xg.double().numpy(), ranks, 1, 1, 17)
    assert abs(err - ref) <= TOL[dtype] * max(ref, 1e-3), (err, ref)
    for U in factors:
        U = U.double().cpu().numpy()
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 1e-5
