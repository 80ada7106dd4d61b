"""The float32 sketch stream against the float64 one, value by value: relative error
at most four units in the last place (a logarithm and a root of about one each, of
which the root halves the first, a sine or cosine of about one, and a product),
for small values too; an odd number of values."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,mode", [(0, 0), (5, 3), (2 ** 40 + 17, 1)])
def test_float32_values(seed, mode):
    import torch
    import paper_2211_14828_amd as rb
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    exact = rb.omega(seed, mode, 1234567, 7, torch.float64)
    z = rb.omega(seed, mode, 1234567, 7, torch.float32).double()
    assert float(((z - exact).abs() / exact.abs()).max()) <= 4 * 2.0 ** -23
