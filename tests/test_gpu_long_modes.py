"""Modes so long that a workgroup for every 64 values of C's partials would pass the
2^32 threads of a launch: from about 23073 rows on in the Gram kernels' reduction, and
about 46080 in the pipelined form's.  The rows' four columns are orthogonal with norms
apart, so that the factor is known: the columns divided by their norms, in order.  A
float64 sum has no error to speak of here; in float32 a value of C is rounded by 2^-24,
in bfloat16 the columns are whole numbers below 2^8, and the chain that follows is
float64: 1e-6 on a factor with gaps of a half between its squared values."""
import numpy as np
import pytest
import torch

import paper_2211_14828_amd as rb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,dtype,precision", [(23040, "float32", "plain"), (23200, "float32", "plain"),
                                                   (23200, "float64", "plain"), (46200, "float32", "mixed_bf16")])
def test_long_middle_mode(rows, dtype, precision):
    # signs of period 2, 4 and 8: orthogonal over whole periods, zero past them
    whole = rows - rows % 8
    i = np.arange(rows)
    cols = np.stack([s * np.where((i // p) % 2 == 0, 1.0, -1.0) * (i < whole)
                     for s, p in ((8.0, 1), (4.0, 2), (2.0, 4))] + [1.0 * (i < whole)], 1)
    X = torch.from_numpy(np.ascontiguousarray(cols.reshape(rows, 2, 2).transpose(1, 0, 2))).to("cuda",
                                                                                               getattr(torch, dtype))
    _, factors, _ = rb.tucker(X, [2, 4, 2], p=5, q=1, seed=1, precision=precision)
    want = cols / np.linalg.norm(cols, axis=0)
    got = factors[1].double().cpu().numpy()
    assert np.abs(np.abs((got * want).sum(0)) - 1).max() <= 1e-6
    assert np.linalg.norm(np.abs(got) - np.abs(want)) <= 1e-6
    assert np.linalg.norm(got[whole - 64:] - np.sign((got * want).sum(0)) * want[whole - 64:]) <= 1e-6
