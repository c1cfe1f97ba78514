"""The few-pixel kernel (gpu): remainders of pixels, channels and bundles against the oracle, channel counts that are no
multiple of four, images smaller than a tile, strides, and activations that are not finite.

Tolerance: a 32-bit sum runs over at most 16 products, each rounded and added once (2 * 16 roundings of 2^-24 of the products'
magnitudes); everything after that is added in 64 bits and rounded once, as the oracle's result is."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W

pytestmark = pytest.mark.gpu


def run(kind, p, x, N, stride, form):
    n, h, w = x.shape[:3]
    y = torch.full((n, (h - 1) // stride + 1, (w - 1) // stride + 1, N), float("nan"), device="cuda")
    S.sbn_force_kernel_form(kind, form)
    try:
        (S.sbn_conv1x1_sparse if kind == S.SBN_CONV1X1 else S.sbn_conv3x3_sparse)(p, torch.from_numpy(x).cuda(), y, n, h, w)
        torch.cuda.synchronize()
    finally:
        S.sbn_force_kernel_form(kind, 0)
    return y.cpu().numpy()


def layer(kind, K, N, pct, go, gi, stride=1, relu=True):
    k = 3 if kind == S.SBN_CONV3X3 else 1
    w, b = W.he_weights(7100 + K + N, N, k, k, K), W.small_bias(7101, N) * 20
    mask = S.sbn_prune_magnitude(w, kind, go, gi, pct)
    return S.sbn_pack(kind, w, go, gi, mask=mask, bias=b, stride=stride, act=S.SBN_ACT_RELU if relu else S.SBN_ACT_NONE), w, mask, b


def check(y, ref, bound, what):
    assert np.isfinite(y).all(), what
    bad = np.abs(y.astype(np.float64) - ref) > 32 * 2.0 ** -24 * bound + np.abs(ref) * 2.0 ** -23
    assert not bad.any(), (what, int(bad.sum()), np.argwhere(bad)[:3])


@pytest.mark.parametrize("form", (3004, 3008))
@pytest.mark.parametrize("m,K,N,pct,go,gi", [
    (1, 4, 4, 0, 4, 4),                # one pixel, one block
    (15, 33, 12, 20, 4, 1),            # a piece of one channel, the last one of the tensor
    (16, 30, 16, 0, 4, 2),
    (17, 90, 200, 40, 8, 2),           # one pixel in the second tile, half a bundle at the end
    (33, 36, 20, 50, 4, 4),            # a second sub-chunk of one piece
    (49, 260, 68, 90, 4, 4),
    (200, 1024, 64, 70, 8, 8),
    (31, 640, 48, 100, 4, 4),          # every block removed
])
def test_1x1_edges(form, m, K, N, pct, go, gi):
    p, w, mask, b = layer(S.SBN_CONV1X1, K, N, pct, go, gi)
    x = W.uniform_activation(7102 + m, (1, 1, m, K))
    ref, bound = R.sparse_conv_reference(x, w, mask, go, gi, bias=b, act=R.ACT_RELU)
    check(run(S.SBN_CONV1X1, p, x, N, 1, form), ref, bound, f"form {form}")


@pytest.mark.parametrize("form", (3004, 3008, 3016))
@pytest.mark.parametrize("n,h,w,K,N,pct,go,gi,stride", [
    (1, 1, 1, 4, 4, 0, 4, 4, 1),       # eight of nine taps outside
    (40, 1, 1, 12, 20, 30, 4, 4, 1),   # a tile of sixteen images
    (7, 2, 3, 36, 16, 20, 4, 2, 1),
    (3, 5, 7, 32, 40, 50, 8, 4, 2),    # the last row and column are read by the stride
    (2, 8, 6, 64, 16, 0, 4, 1, 2),
    (1, 9, 11, 104, 72, 70, 8, 8, 1),
    (2, 17, 4, 256, 24, 90, 4, 4, 1),
])
def test_3x3_edges(form, n, h, w, K, N, pct, go, gi, stride):
    p, wt, mask, b = layer(S.SBN_CONV3X3, K, N, pct, go, gi, stride)
    x = W.uniform_activation(7103 + h, (n, h, w, K))
    ref, bound = R.sparse_conv_reference(x, wt, mask, go, gi, bias=b, stride=stride, pad=1, act=R.ACT_RELU)
    check(run(S.SBN_CONV3X3, p, x, N, stride, form), ref, bound, f"form {form}")


@pytest.mark.parametrize("kind", (S.SBN_CONV1X1, S.SBN_CONV3X3))
@pytest.mark.parametrize("value", (np.inf, -np.inf, np.nan))
@pytest.mark.parametrize("many", (False, True))
def test_what_is_not_finite_reaches_only_what_keeps_its_block(kind, value, many):
    """Removed blocks are multiplied as zeros, which an infinite activation must not turn into NaN."""
    K, N, n, h, w = 96, 48, 2, 6, 5
    p, wt, mask, b = layer(kind, K, N, 60, 4, 4, relu=False)
    x = W.uniform_activation(7104, (n, h, w, K))
    clean = run(kind, p, x, N, 1, 3008)
    at = [(1, 2, 3)] if not many else [(i, j, k) for i in range(n) for j in range(h) for k in range(w) if (i + j + k) % 3 == 0]
    ch = 37
    for i in at:
        x[i][ch] = value
    y = run(kind, p, x, N, 1, 3008)
    keeps = np.repeat(mask[:, ch // 4] != 0, 4)
    hit = np.zeros((n, h, w), bool)
    for i, j, k in at:
        if kind == S.SBN_CONV1X1:
            hit[i, j, k] = True
        else:
            hit[i, max(0, j - 1):j + 2, max(0, k - 1):k + 2] = True
    assert keeps.any() and not keeps.all()
    assert not np.isfinite(y[hit][:, keeps]).any()
    untouched = ~(hit[..., None] & keeps)
    # (done again in another order: 32-bit sums of up to 9 * 96 products)
    assert np.allclose(y[untouched], clean[untouched], rtol=0, atol=1e-4)
    assert np.array_equal(y[~hit], clean[~hit])


@pytest.mark.parametrize("m,K,N,pct", [(196, 512, 512, 30), (49, 1024, 1024, 90), (784, 128, 256, 50), (1, 1024, 1000, 0)])
def test_the_automatic_choice_takes_it_for_one_image(m, K, N, pct):
    """The same bits as the forced form: layers of a network on one image run on this kernel."""
    p, w, mask, b = layer(S.SBN_CONV1X1, K, N, pct, 4, 4)
    x = W.uniform_activation(7105, (1, 1, m, K))
    y = run(S.SBN_CONV1X1, p, x, N, 1, 0)
    assert any(np.array_equal(y, run(S.SBN_CONV1X1, p, x, N, 1, f)) for f in (3004, 3008))


@pytest.mark.parametrize("kind,h,w,K,N,pct,stride,form", [
    # 16 pixels x 16 channels = a tile, 32 channels of a tap = a unit
    (S.SBN_CONV3X3, 16, 16, 256, 64, 0, 1, 3016),      # 64 tiles of 72 units: sixteen waves
    (S.SBN_CONV3X3, 17, 16, 256, 64, 0, 1, 3008),      # 68 tiles
    (S.SBN_CONV3X3, 16, 16, 224, 64, 0, 1, 3008),      # 63 units
    (S.SBN_CONV3X3, 31, 32, 256, 64, 0, 2, 3016),      # (stride 2: 16 x 16 pixels)
    (S.SBN_CONV3X3, 32, 32, 32, 64, 0, 1, 3008),       # a tile per compute unit
    (S.SBN_CONV3X3, 33, 32, 32, 64, 0, 1, 3004),
    (S.SBN_CONV3X3, 60, 80, 32, 64, 0, 1, 3004),       # 4.7 tiles per compute unit
    (S.SBN_CONV3X3, 60, 81, 32, 64, 0, 1, None),
    (S.SBN_CONV3X3, 48, 60, 32, 64, 50, 1, 3004),      # half kept: 0.6 of it
    (S.SBN_CONV3X3, 49, 60, 32, 64, 50, 1, None),
    (S.SBN_CONV3X3, 52, 64, 512, 64, 0, 1, 3004),      # 470 units per compute unit
    (S.SBN_CONV3X3, 53, 64, 512, 64, 0, 1, None),
    (S.SBN_CONV3X3, 167, 189, 32, 64, 0, 2, 3004),     # stride 2: 7.8 tiles
    (S.SBN_CONV3X3, 168, 191, 32, 64, 0, 2, None),
    (S.SBN_CONV1X1, 32, 32, 256, 64, 0, 1, 3008),      # a tile per compute unit
    (S.SBN_CONV1X1, 25, 41, 256, 64, 0, 1, 3004),
    (S.SBN_CONV1X1, 64, 96, 64, 64, 0, 1, 3004),       # six tiles
    (S.SBN_CONV1X1, 5, 1229, 64, 64, 0, 1, None),
    (S.SBN_CONV1X1, 32, 60, 1024, 128, 0, 1, 3004),    # 120 units
    (S.SBN_CONV1X1, 17, 113, 1024, 128, 0, 1, None),
])
def test_the_automatic_choice_on_both_sides_of_its_lines(kind, h, w, K, N, pct, stride, form):
    """The same bits as the form that the rule names on a device of 256 compute units; as none of them where it takes another kernel."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 compute units")
    p = layer(kind, K, N, pct, 4, 4, stride)[0]
    x = W.uniform_activation(7106, (1, h, w, K))
    y = run(kind, p, x, N, stride, 0)
    for f in (3004, 3008) if kind == S.SBN_CONV1X1 else (3004, 3008, 3016):
        same = np.array_equal(y, run(kind, p, x, N, stride, f))
        assert same if f == form else form or not same, f
