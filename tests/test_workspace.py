"""Workspace sizes of plans whose chain sets come near what they may take: no larger than
they were without them (the sizes recorded then), so that a caller's buffer, or the fixed
scratch of rbki_tucker_noalloc, that was large enough still is."""
import pytest
import torch

import paper_2211_14828_amd as rb

CASES = [
    (([296, 238, 2, 2, 4, 2, 2], [11, 56, 2, 2, 4, 2, 2], 5, 17, torch.float32, "mixed_bf16"), 1631255104),
    (([296, 238, 2, 2, 4, 2, 2], [11, 56, 2, 2, 4, 2, 2], 5, 17, torch.float32, "plain"), 129864256),
]


@pytest.mark.parametrize("problem,before", CASES)
def test_no_larger(problem, before):
    assert 0 < rb.workspace_bytes(*problem) <= before
