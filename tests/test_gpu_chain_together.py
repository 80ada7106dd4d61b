"""Krylov chains of modes beyond the persistent kernel, run in step: modes of
different widths in one launch (each orthonormalisation kernel at once), inner
dimensions split over workgroups, 64-row product tiles, and the same result for
a mode alone and among others.  Against the float64 oracle; tolerances on the
reconstruction error as in test_gpu_parity.py (float64 1e-10, float32 1e-5)."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

CASES = [
    # sketches of 75, 15 and 105 columns together
    ((300, 290, 280), (70, 10, 100), 5, 1, np.float64, "krylov", 1.0),
    # 4200 rows: 64-row tiles and a split inner dimension; two small modes
    ((4200, 45, 40), (50, 8, 8), 10, 1, np.float32, "krylov", 1.0),
    # power iteration, and sampled columns
    ((270, 300, 20), (9, 33, 6), 7, 2, np.float64, "power", 1.0),
    ((270, 300, 20), (9, 33, 6), 7, 2, np.float64, "krylov", 0.3),
]


@pytest.mark.parametrize("dims,ranks,p,q,dtype,variant,rate", CASES)
def test_chains_in_step_match_oracle(dims, ranks, p, q, dtype, variant, rate):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims).astype(dtype)
    _, _, err = rb.tucker(torch.from_numpy(X).to("cuda"), ranks, p=p, q=q, seed=21, variant=variant, sample_rate=rate)
    _, _, ref = rbki_tucker(X.astype(np.float64), ranks, p, q, 21, variant=variant, sample_rate=rate)
    assert abs(err - ref) <= (1e-10 if dtype == np.float64 else 1e-5) * ref, (err, ref)


def test_a_basis_alone_equals_the_one_among_others():
    """One mode's basis by its own call and inside a decomposition of several
    modes: the factor of the decomposition lies in it to float64 rounding."""
    import torch
    import paper_2211_14828_amd as rb
    X = np.random.default_rng(8).standard_normal((290, 40, 300))
    Xg = torch.from_numpy(X).to("cuda")
    _, factors, _ = rb.tucker(Xg, [12, 6, 20], p=5, q=2, seed=3)
    for n, U in enumerate(factors):
        Qt, width = rb.basis(Xg, n, [12, 6, 20], p=5, q=2, seed=3)
        Q = Qt[:width]
        assert float((U - Q.T @ (Q @ U)).abs().max()) <= 1e-12
