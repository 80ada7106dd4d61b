"""The launch that signs the factors and writes their copies: one row, rows that do
not fill a workgroup, one column, several modes of different sizes at once, in the
plans that keep the copies for the later products (small modes in one chain launch,
modes in step) and in the stages of the sequential form.  Factors asked for in
float32 and float64 are the same numbers, every column's largest entry is positive,
the core is the projection on them, and the step-by-step solve that stops at its
limit gives the fixed-step result to the bit."""
import numpy as np
import pytest

from oracle.tensor import project_core

pytestmark = pytest.mark.gpu

CASES = [((9, 1, 30), (5, 1, 4)), ((64, 70, 20), (1, 2, 2)), ((300, 40, 33), (5, 9, 4)), ((20, 300, 6, 5), (7, 13, 4, 2)),
         ((130, 90), (65, 64))]


@pytest.mark.parametrize("truncation", ["independent", "sequential"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("dims,ranks", CASES)
def test_factors_and_their_copies(dims, ranks, dtype, truncation):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    X = np.random.default_rng(sum(dims)).standard_normal(dims).astype(dtype)
    Xg = torch.from_numpy(X).to("cuda")
    kw = dict(p=3, q=1, seed=9)
    core, f64, err = rb.tucker(Xg, ranks, out_dtype=torch.float64, truncation=truncation, **kw)
    _, f32, err32 = rb.tucker(Xg, ranks, out_dtype=torch.float32, truncation=truncation, **kw)
    assert err == err32
    for U, V in zip(f64, f32):
        assert torch.equal(U.float(), V)
        U = U.cpu().numpy()
        assert (U[np.argmax(np.abs(U), axis=0), np.arange(U.shape[1])] > 0).all()
    G = project_core(X.astype(np.float64), [U.cpu().numpy() for U in f64])
    off = np.linalg.norm(core.cpu().numpy() - G) / np.linalg.norm(G)
    assert off <= (1e-12 if dtype == np.float64 else 1e-5), off
    if truncation == "independent":
        c, fa, ea, qa = rb.tucker_adaptive(Xg, ranks, p=3, max_q=1, fit_tol=-1.0, seed=9, out_dtype=torch.float64)
        assert qa == 1 and ea == err and torch.equal(c, core)
        assert all(torch.equal(U, V) for U, V in zip(fa, f64))
