"""The reduction of the pipelined Gram kernels' partial sums with few splits and with
many (four and sixteen groups of lanes), at row counts around its 64-value runs and
256-row tiles and at the smallest and largest sketch.  Float64 oracle on the same
bfloat16 values; 1e-5 relative on the reconstruction error, as in test_gpu_parity.py
for bfloat16 inputs."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

CASES = [((65, 70, 40), (6, 59, 5)), ((255, 130, 9), (5, 9, 4)), ((257, 64, 33), (9, 5, 6)), ((300, 320, 350), (3, 6, 9)),
         ((520, 66, 64), (12, 3, 4))]


@pytest.mark.parametrize("dims,ranks", CASES)
def test_partial_sums(dims, ranks):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = torch.from_numpy(np.random.default_rng(sum(dims)).standard_normal(dims)).to(torch.bfloat16)
    _, _, err = rb.tucker(X.to("cuda"), ranks, p=5, q=1, seed=2, precision="mixed_bf16")
    _, _, ref = rbki_tucker(X.double().numpy(), ranks, 5, 1, 2)
    assert abs(err - ref) <= 1e-5 * ref, (err, ref)
