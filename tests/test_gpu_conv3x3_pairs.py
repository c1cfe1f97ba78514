"""The 3x3 forms on pairs of 16-bit floats (gpu): edges of tiles, images and channels against the oracle, and
data outside the pairs' range.  Tolerance: 1e-4 * sum|w||x| per output, as for every fp32 kernel here
(observed 3e-7)."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu
FORMS = (2064, 2065, 2128)


def pack(K, N, pct, go=4, gi=4, relu=True):
    w = W.he_weights(9100 + K + N, N, 3, 3, K)
    b = W.small_bias(9101, N) * 20
    mask = S.sbn_prune_magnitude(w, S.SBN_CONV3X3, go, gi, pct)
    assert np.count_nonzero(mask) * go * gi * 9 >= 128 * N       # else the layer has no pairs and the test tests nothing
    p = S.sbn_pack(S.SBN_CONV3X3, w, go, gi, mask=mask, bias=b, act=S.SBN_ACT_RELU if relu else S.SBN_ACT_NONE)
    return p, w, mask, b


def run(p, x, N, form):
    n, h, w, _ = x.shape
    xd = torch.from_numpy(x).cuda()
    yd = torch.full((n, h, w, N), float("nan"), device="cuda")
    S.sbn_force_kernel_form(S.SBN_CONV3X3, form)
    try:
        S.sbn_conv3x3_sparse(p, xd, yd, n, h, w)
        torch.cuda.synchronize()
    finally:
        S.sbn_force_kernel_form(S.SBN_CONV3X3, 0)
    return yd.cpu().numpy()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n,h,w,K,N,pct,go,gi", [
    (1, 4, 4, 32, 64, 30, 4, 4),           # the smallest image, one sub-chunk
    (5, 5, 7, 36, 68, 20, 4, 2),           # a tile over four images; ragged channels on both sides
    (2, 8, 16, 64, 16, 50, 4, 4),          # tiles end where rows do; one bundle
    (1, 5, 127, 32, 48, 40, 4, 4),         # the widest image
    (1, 13, 63, 96, 72, 60, 8, 4),         # largest width of the middle image buffer of 128-pixel tiles, odd sub-chunks
    (1, 9, 47, 40, 64, 30, 4, 1),          # and of the small one of 64-pixel tiles
    (3, 9, 9, 256, 200, 80, 4, 4),
])
def test_edges(form, n, h, w, K, N, pct, go, gi):
    p, wt, mask, b = pack(K, N, pct, go, gi)
    x = W.uniform_activation(9102 + h + w, (n, h, w, K))
    ref, bound = R.sparse_conv_reference(x, wt, mask, go, gi, bias=b, stride=1, pad=1, act=R.ACT_RELU)
    assert_within_bound(run(p, x, N, form), ref, bound, f"form {form}")


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("kind", ["tiny image", "huge value", "first channels tiny", "later channels tiny", "all tiny", "all huge"])
def test_unusual_magnitudes(form, kind):
    p, wt, mask, b = pack(128, 64, 50, relu=False)
    x = W.uniform_activation(9103, (4, 6, 9, 128))
    if kind == "tiny image":
        x[1] *= np.float32(1e-15)
    elif kind == "huge value":
        x[1, 3, 4, 9] = 1e15
    elif kind == "first channels tiny":
        x[..., :64] *= np.float32(1e-12)
    elif kind == "later channels tiny":
        x[..., 64:] *= np.float32(1e-12)
    else:
        x *= np.float32(1e-25 if kind == "all tiny" else 1e25)
    ref, bound = R.sparse_conv_reference(x, wt, mask, 4, 4, bias=b, stride=1, pad=1)
    assert_within_bound(run(p, x, 64, form), ref, bound, kind)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_infinities_and_nan_reach_the_windows_that_hold_them_and_nothing_else(form, value):
    p, wt, mask, b = pack(64, 64, 50, relu=False)
    x = W.uniform_activation(9104, (3, 7, 6, 64))
    x[1, 0, 5, 18] = value
    y, y32 = run(p, x, 64, form), run(p, x, 64, 1)
    assert np.array_equal(np.isnan(y), np.isnan(y32)) and np.array_equal(np.isinf(y), np.isinf(y32))
    fin = np.isfinite(y32)
    assert not fin.all() and fin[0].all() and fin[2].all()
    assert np.allclose(y[fin], y32[fin], rtol=0, atol=1e-4)
