"""Tall modes on both sides of the rule by steps (1030 rows: up to two steps from X
itself, from three on from X X^T; 1300: three and four), against the float64 oracle
with the tolerances of test_gpu_parity.py."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("dims,q,variant", [((1030, 40), 2, "krylov"), ((1030, 40), 3, "krylov"), ((20, 21, 1300), 3, "krylov"),
                                            ((20, 21, 1300), 4, "krylov"), ((1030, 40), 9, "power")])
def test_steps(dims, q, variant, dtype):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    ranks = [6] * len(dims)
    X = np.random.default_rng(q).standard_normal(dims).astype(dtype)
    core, factors, err = rb.tucker(torch.from_numpy(X).to("cuda"), ranks, p=4, q=q, seed=2, variant=variant)
    _, _, ref = rbki_tucker(X.astype(np.float64), ranks, 4, q, 2, variant=variant)
    assert abs(err - ref) <= (1e-10 if dtype == "float64" else 1e-5) * ref
