"""Mixed forms and stored bfloat16 with trailing dimensions of 1, where the mode before
them has no columns inside a slab, against the float64 oracle.  The tensors are nearly of
rank three, so what the operands' rounding adds to the error shows in full: at most
2^-9 of a value twice over (tensor and factor) in bfloat16, 2^-4 / sqrt(3) in e4m3, in
quadrature with the oracle's error.  Factors are orthonormal to 1e-5 and those of the
signal within 1e-2 (cosine) of the oracle's."""
import numpy as np
import pytest

from oracle.rbki import rbki_tucker

pytestmark = pytest.mark.gpu

CASES = [((13, 10, 1), (4, 4, 1)), ((28, 36, 1), (2, 3, 1)), ((300, 140, 1), (5, 4, 1)), ((9, 200, 1, 1), (3, 5, 1, 1)),
         ((6, 5, 150, 1), (3, 3, 6, 1)), ((150, 1), (1, 1)), ((1, 40, 1), (1, 1, 1)), ((70, 65, 1), (30, 64, 1))]


@pytest.mark.parametrize("dtype,precision", [("bfloat16", "plain"), ("float32", "mixed_bf16"), ("float32", "mixed_fp8")])
@pytest.mark.parametrize("dims,ranks", CASES)
def test_trailing_ones(dims, ranks, dtype, precision):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    rng = np.random.default_rng(sum(dims))
    U = [np.linalg.qr(rng.standard_normal((d, min(3, d))))[0] for d in dims]
    X = 0.02 * rng.standard_normal(dims) / np.sqrt(np.prod(dims))
    for c in range(3):
        t = np.array(2.0 ** -c)
        for V in U:
            t = np.multiply.outer(t, V[:, min(c, V.shape[1] - 1)])
        X = X + t
    Xg = torch.from_numpy(X).to("cuda", getattr(torch, dtype))
    core, factors, err = rb.tucker(Xg, ranks, p=5, q=1, seed=3, precision=precision)
    _, exact, ref = rbki_tucker(Xg.double().cpu().numpy(), ranks, 5, 1, 3)
    added = 2.0 ** -4 / np.sqrt(3) if precision == "mixed_fp8" else 2.0 ** -8
    assert err ** 2 <= ref ** 2 + added ** 2 and err >= ref - 1e-5
    for V in factors:
        V = V.double().cpu().numpy()
        assert np.abs(V.T @ V - np.eye(V.shape[1])).max() <= 1e-5
    for V, W, R in zip(factors, exact, ranks):
        k = min(R, 3)
        cos = np.abs(np.sum(V.double().cpu().numpy()[:, :k] * W[:, :k], 0))
        assert np.all(cos >= 1 - 1e-2)
