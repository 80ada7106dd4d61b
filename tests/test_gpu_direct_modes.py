"""Modes whose products with X X^T are formed from X itself (at least 1024 rows, at
most half as many columns): first and last modes, exactly half as many columns and
very few, each data type, Krylov and power iteration, the step-by-step solve, and a
neighbour just short of the rule (1023 rows; more than half as many columns).  Errors
against the float64 oracle as in test_gpu_parity.py (float64 1e-10, float32 1e-5,
bfloat16 inputs 1e-5: their values are exact and the sums float64 here)."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

CASES = [
    ((2100, 33, 31), (9, 8, 7), "float32", "krylov"), ((30, 33, 2100), (9, 8, 7), "float32", "krylov"),
    ((30, 33, 2100), (9, 8, 7), "float64", "power"), ((2048, 1024), (20, 15), "float64", "krylov"),
    ((2500, 3), (2, 2), "float32", "krylov"), ((17, 2300), (6, 12), "bfloat16", "krylov"),
    ((1023, 300), (20, 15), "float32", "krylov"), ((1024, 512), (20, 15), "float32", "krylov"), ((40, 27, 2100), (9, 8, 7), "float32", "power"),
]


@pytest.mark.parametrize("dims,ranks,dtype,variant", CASES)
def test_direct_modes_match_oracle(dims, ranks, dtype, variant):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims)
    Xg = torch.from_numpy(X).to({"float64": torch.float64, "float32": torch.float32, "bfloat16": torch.bfloat16}[dtype])
    Xd = Xg.to("cuda")
    core, factors, err = rb.tucker(Xd, ranks, p=5, q=2, seed=12, variant=variant)
    _, _, ref = rbki_tucker(Xg.double().numpy(), ranks, 5, 2, 12, variant=variant)
    assert abs(err - ref) <= (1e-10 if dtype == "float64" else 1e-5) * max(ref, 0.1), (err, ref)
    if variant == "krylov":
        c, fa, ea, _ = rb.tucker_adaptive(Xd, ranks, p=5, max_q=2, fit_tol=-1.0, seed=12)
        assert ea == err and torch.equal(c, core) and all(torch.equal(U, V) for U, V in zip(fa, factors))
