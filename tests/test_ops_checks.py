"""Argument checks of ops.py that need no GPU."""

import pytest
import torch

from paper_2607_27744_amd import ops


@pytest.mark.parametrize("fn", [ops.glm_linear, ops.ikbo_linear_combined])
def test_strided_request_bias_is_refused(fn):
    # The kernels read d_req consecutive floats.
    x, w = torch.zeros(2, 8), torch.zeros(4, 8)
    kw = dict(x_req=x, x_cand=x, w_rr=w, w_cr=w, w_cc=w,
              cand_offsets=torch.tensor([0, 1, 2], dtype=torch.int32))
    with pytest.raises(ValueError, match="contiguous float32"):
        fn(**kw, b_req=torch.zeros(8)[::2])
    with pytest.raises(ValueError, match="on the GPU"):
        fn(**kw, b_req=torch.zeros(4))
