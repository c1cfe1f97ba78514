"""The stand-alone depthwise kernel (gpu) where its blocks, strips and image borders can go wrong, against the
oracle.  Tolerance: 1e-4 * sum|w||x| per output, as for every fp32 kernel here."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("n,h,w,c", [
    (70, 9, 1, 4),           # rows of one quad, a block across many images
    (3, 13, 4, 20),          # a block ends within a row
    (2, 34, 8, 16),          # rows of 32 quads (stride 1), the longest of the narrow kernel; half of that (stride 2)
    (2, 34, 11, 12),         # and one more
    (1, 1, 1, 4),            # one pixel, one lane
    (2, 3, 1, 20),           # one column
    (1, 1, 40, 12),          # one row; rows of 120 quads (stride 1), 60 (stride 2)
    (3, 5, 16, 16),          # rows of exactly one block of 64 (stride 1), half of one (stride 2)
    (2, 6, 13, 1028),        # a channel quad past a block: columns cross blocks
    (5, 9, 14, 512),         # one-row strips, blocks of 256
    (9, 30, 29, 260),        # enough for four-row strips with a remainder; blocks of 64 and 256 with idle lanes
    (40, 13, 13, 512),
])
def test_depthwise_edges(n, h, w, c, stride):
    wt = W.normal_weights(9700 + c, (c, 3, 3), 0.4)
    b = W.small_bias(9701, c) * 10
    chain = S.sbn_chain_create([S.dw_item(wt, b, stride=stride, act=S.SBN_ACT_RELU)])
    x = W.uniform_activation(9702 + w, (n, h, w, c))
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, h, w)
    y = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), y, n, h, w, None)
    torch.cuda.synchronize()
    ref, bound = R.dwconv3x3_nhwc(x, wt, b, stride=stride, act=R.ACT_RELU)
    assert_within_bound(y.cpu().numpy(), ref, bound, f"depthwise {n, h, w, c} stride {stride}")
