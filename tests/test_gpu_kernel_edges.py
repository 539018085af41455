"""Sizes at which a kernel's tiling or a rule of its dispatch can go wrong (edges of tiles, remainders, the smallest and the
largest of a range), against the CPU oracle.  Every tolerance is derived beside its test."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_28115_amd import workloads as wl
from test_gpu_parity import log, to_dev, to_host, widen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bd():
    from paper_2605_28115_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return binding


@pytest.mark.parametrize("tokens", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("anchors", [1, 127, 129, 511, 513, 700])
def test_token_weight_columns_and_row_slots(bd, tokens, anchors):
    """Token weights over column groups of 64 and row slots of 128 x 4.  A weight is exp(logit) over its row's sum, logits
    are at most 1 (inv_tau = 1): operands rounded to bf16 move one by at most 2 * 2^-9, so a weight and its row's sum by
    2^-8 each, the weight's own rounding by 2^-9: 2^-6 relative covers them, and the fp32 sums' 2^-20."""
    log("token weights", tokens, anchors)
    rng = np.random.default_rng(1000 * tokens + anchors)
    x, x32 = wl.quantize(rng.standard_normal((2, tokens, 64)).astype(np.float32), "bf16")
    a, a32 = wl.quantize(rng.standard_normal((anchors, 64)).astype(np.float32), "bf16")
    _, tw = bd.civic_anchor_aggregate(to_dev(x), to_dev(a), 1.0, want_token_weight=True)
    _, ref = oracle.anchor_aggregate(x32, a32, 1.0, want_col_sum=True)
    got = to_host(tw).astype(np.float64)
    assert (np.abs(got - ref) <= 2.0 ** -6 * ref).all(), float((np.abs(got - ref) / ref).max())
