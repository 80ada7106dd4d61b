"""The float32 sketch and Gram products to first order: the spans of W = X Omega (a basis
without Krylov steps) and of C Q_0 (one step of power iteration) against float64, in
every form of the Gram kernel (tiles, thin, wide, in registers), with slabs longer and
shorter than a K tile, the last mode, and values of 2^-58.

The values are +-2^e times a number that goes by the row's parity: 1, of one bfloat16
part, or one whose second and third parts are as large as they can be (2^-8 and 2^-17).
A part product that is lost or misplaced then turns the rows of one parity against the
others, by 2^-18 = 3.8e-6 (hl, lh) and more (mm), a component outside the span; parts
of the Gaussian sketch are worth 2e-6.  What is left in a right one is the sums'
rounding, some tens of additions of relative 2^-25 (1e-7 to 2e-7): the tolerance is
8e-7.  test_lost_part_products_show states what each is worth, on the CPU."""
import numpy as np
import pytest

from oracle.philox import omega
from oracle.tensor import unfold

TOL = 8e-7
S = 20

CASES = [
    ((100, 30, 20), 0), ((25, 24, 100), 2), ((9, 100, 7), 1),              # 128-row tiles
    ((60, 24, 25), 0), ((25, 24, 60), 2), ((30, 60, 7), 1),                # thin
    ((400, 20, 30), 0), ((20, 30, 400), 2), ((60, 400, 12), 1), ((7, 512, 100), 1),   # wide
    ((8, 30, 20), 0), ((30, 20, 8), 2),                                    # in registers
]


def parts(x):
    """The three bfloat16 parts of float32 values, exact."""
    out = []
    r = x.astype(np.float32)
    for _ in range(3):
        u = r.view(np.uint32).astype(np.uint64)
        h = ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)
        out.append(h.astype(np.float64))
        r = (r - h).astype(np.float32)
    assert not r.any()
    return out


def tensor(dims, mode):
    rng = np.random.default_rng(sum(dims) + mode)
    v = np.array([1 + 2.0 ** -8 - 2.0 ** -15 + 2.0 ** -17 - 2.0 ** -23, 1.0])
    X = rng.choice([-1.0, 1.0], dims) * 2.0 ** rng.integers(-1, 2, dims)
    shape = [1] * len(dims)
    shape[mode] = dims[mode]
    return (X * v[np.arange(dims[mode]) % 2].reshape(shape)).astype(np.float32)


def outside(Q, Y):
    return np.linalg.norm(Y - Q @ (Q.T @ Y)) / np.linalg.norm(Y)


def test_lost_part_products_show():
    """What each part product is worth, in float64."""
    dims, mode = (100, 30, 20), 0
    X = unfold(tensor(dims, mode), mode)
    Om = omega(31, mode, X.shape[1], S)
    x, o = parts(X), parts(Om.astype(np.float32))
    W = X.astype(np.float64) @ Om
    Q0 = np.linalg.qr(W)[0]
    C = X.astype(np.float64) @ X.T.astype(np.float64)
    for a, b in ((0, 2), (2, 0), (1, 1)):
        assert outside(np.linalg.qr(W - x[a] @ o[b])[0], W) > 1.5 * TOL
        assert outside(np.linalg.qr((C - x[a] @ x[b].T) @ Q0)[0], C @ Q0) > 1.5 * TOL


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [0, -58])
@pytest.mark.parametrize("dims,mode", CASES)
def test_spans(dims, mode, scale):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    s = min(S, dims[mode] // 2)
    X = tensor(dims, mode)
    ranks = [1] * len(dims)
    ranks[mode] = s - 1
    Xg = torch.from_numpy((X * np.float32(2.0 ** scale))).to("cuda")
    Xn = unfold(X.astype(np.float64), mode)
    W = Xn @ omega(31, mode, Xn.shape[1], s)
    Qt, width = rb.basis(Xg, mode, ranks, p=1, q=0, seed=31)
    assert width == s and outside(Qt[:width].cpu().numpy().T, W) <= TOL
    Qt, width = rb.basis(Xg, mode, ranks, p=1, q=1, seed=31, variant="power")
    assert width == s and outside(Qt[:width].cpu().numpy().T, Xn @ (Xn.T @ np.linalg.qr(W)[0])) <= TOL
