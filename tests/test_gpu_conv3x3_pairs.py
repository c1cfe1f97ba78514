"""The 3x3 forms on triples of bfloat16 (gpu): edges of tiles, images and channels against the oracle, every bit
of single products, values of very different size side by side, and data outside the triples' range.

Tolerance: 1e-4 * sum|w||x| per output, as for every fp32 kernel here, where none is derived beside the test."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu
FORMS = (2064, 2065, 2128)


def pack_wide(w, go, gi, **kw):
    """A layer with the tables of the wide forms, whether or not the automatic choice would use them."""
    S.sbn_force_kernel_form(S.SBN_CONV3X3, 2064)
    try:
        return S.sbn_pack(S.SBN_CONV3X3, w, go, gi, **kw)
    finally:
        S.sbn_force_kernel_form(S.SBN_CONV3X3, 0)


def pack(K, N, pct, go=4, gi=4, relu=True, bias=True):
    w = W.he_weights(9100 + K + N, N, 3, 3, K)
    b = W.small_bias(9101, N) * 20 if bias else None
    mask = S.sbn_prune_magnitude(w, S.SBN_CONV3X3, go, gi, pct)
    p = pack_wide(w, go, gi, mask=mask, bias=b, act=S.SBN_ACT_RELU if relu else S.SBN_ACT_NONE)
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
    y = run(p, x, N, form)
    assert_within_bound(y, ref, bound, f"form {form}")
    # a rounding of 2^-23 of what has been summed per row of taps of 32 channels and six within it, 8 for the rest
    assert np.all(np.abs(y - ref) <= (3 * ((K + 31) // 32) + 14) * 2.0 ** -23 * (bound + np.abs(b)))


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


# ---- every bit of the operands, whatever stands beside them ------------------------------------

def kept_weights(w, mask, go, gi):
    """[c_out][3][3][c_in] in 64 bits, removed kernels zero."""
    N, K = w.shape[0], w.shape[-1]
    return w * np.repeat(np.repeat(mask.reshape(N // go, K // gi) != 0, go, 0), gi, 1).astype(np.float64)[:, None, None, :]


def convolve64(x, wm):
    n, h, w, K = x.shape
    xp = np.zeros((n, h + 2, w + 2, K))
    xp[:, 1:-1, 1:-1] = x
    return sum(xp[:, ky:ky + h, kx:kx + w] @ wm[:, ky, kx].T for ky in range(3) for kx in range(3))


@pytest.mark.parametrize("form", FORMS + (0,))
@pytest.mark.parametrize("n,h,w,K,N,pct,go,gi", [(30, 6, 9, 64, 64, 0, 4, 4), (7, 11, 23, 132, 68, 30, 4, 2), (40, 7, 7, 256, 96, 50, 8, 4)])
def test_single_products_keep_every_bit(form, n, h, w, K, N, pct, go, gi):
    """No two active activations within a window: an output is one product of a weight and an activation, off by the
    rounding of the result, that of the small sums and what the kernel leaves out (the 1x1 test has the figures)."""
    p, wt, mask, _ = pack(K, N, pct, go, gi, relu=False, bias=False)
    x = np.zeros((n, h, w, K), np.float32)
    at = np.stack(np.meshgrid(np.arange(n), np.arange(0, h, 3), np.arange(0, w, 3), indexing="ij"), -1).reshape(-1, 3)
    x[at[:, 0], at[:, 1], at[:, 2], np.arange(len(at)) % K] = W.uniform_activation(9105, (len(at),)) + np.float32(1.5)
    ref = convolve64(x, kept_weights(wt, mask, go, gi))
    assert np.all(np.abs(run(p, x, N, form) - ref) <= 2.25 * 2.0 ** -24 * np.abs(ref))


@pytest.mark.parametrize("form", FORMS + (0,))
@pytest.mark.parametrize("kind", [("weights", 40), ("weights", 48), ("taps", 40), ("removed", 1e12), ("removed", 1e20), ("one filter of four", 1e15),
                                  ("small beside one", 1e-33), ("small beside one", 1e-40), ("all", 1e-36), ("all", 1e30)], ids=str)
def test_large_values_cost_small_ones_nothing(form, kind):
    K, N = 64, 96
    w = W.he_weights(9106, N, 3, 3, K)
    x = np.abs(W.uniform_activation(9107, (40, 7, 9, K)))
    gi = 1 if kind[0] == "removed" else 4
    mask = np.ones((N // 4, K // gi), np.uint8)
    if kind[0] == "weights":                       # large activations, small weights
        x[..., ::4] *= np.float32(2.0) ** kind[1]
        w[..., ::4] *= np.float32(2.0) ** -kind[1]
    elif kind[0] == "taps":                        # large weights that only zeros meet
        w[:, 0] *= np.float32(2.0) ** kind[1]
        x[:, :-1] = 0
    elif kind[0] == "removed":
        mask[:, ::4] = 0
        x[..., ::4] = kind[1]
    elif kind[0] == "one filter of four":
        x[..., 9] = kind[1]
        w[np.arange(N) % 4 != 1, :, :, 8:12] = 0
    elif kind[0] == "small beside one":
        x[..., 1::2] *= np.float32(kind[1])
    else:
        x *= np.float32(kind[1])
    p = pack_wide(w, 4, gi, mask=mask)
    wm = kept_weights(w, mask, 4, gi)
    ref, bound = convolve64(x, wm), convolve64(x, np.abs(wm))
    # a rounding of 2^-23 of what has been summed, at most 9 * 64 of them (one per product in the 32-bit forms)
    err = np.abs(run(p, x, N, form) - ref)
    assert np.all(err <= 48 * 2.0 ** -23 * bound + 2.0 ** -149 * 9 * K), (err / np.maximum(bound, 1e-300)).max()


@pytest.mark.parametrize("form", FORMS)
def test_activations_below_the_range_against_huge_weights(form):
    K, N = 64, 64
    w, mask = W.he_weights(9108, N, 3, 3, K) * np.float32(1e30), np.ones((N // 4, K // 4), np.uint8)
    x = np.abs(W.uniform_activation(9109, (5, 9, 11, K)))
    x[1:4] *= np.float32(1e-36)
    x[2, 4] = 0
    p = pack_wide(w, 4, 4, mask=mask)
    wm = kept_weights(w, mask, 4, 4)
    assert np.all(np.abs(run(p, x, N, form) - convolve64(x, wm)) <= 9 * K * 2.0 ** -24 * convolve64(x, np.abs(wm)))


@pytest.mark.parametrize("K,N,pct", [(64, 64, 0), (256, 64, 50), (512, 96, 70)])
def test_long_sums_are_no_further_off_than_32_bit_ones(K, N, pct):
    """Against 64 bits, as a whole: at most what the 32-bit form shows."""
    p, w, mask, b = pack(K, N, pct, relu=False)
    x = np.maximum(W.normal_weights(9110, (4, 7, 9, K), 1.0), 0)
    ref = convolve64(x, kept_weights(w, mask, 4, 4)) + b
    limit = np.linalg.norm(run(p, x, N, 1) - ref)
    for form in FORMS:
        assert np.linalg.norm(run(p, x, N, form) - ref) <= limit


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("spoilt", [1, 3, 40])
def test_outputs_done_again_one_by_one_and_side_by_side(form, spoilt):
    """Up to 12 of a wave's outputs are done again by the wave together, more by their lanes."""
    p, wt, mask, b = pack(68, 96, 50, relu=False)
    x = W.uniform_activation(9111, (3, 7, 9, 68))
    at = np.zeros((3, 7, 9), bool)
    at.reshape(-1)[60:60 + spoilt] = True
    x[at, 33] = np.inf
    y = run(p, x, 96, form)
    x[at, 33] = 0
    wm = kept_weights(wt, mask, 4, 4)
    ref, bound = convolve64(x, wm) + b, convolve64(np.abs(x), np.abs(wm)) + np.abs(b)
    hot = np.zeros_like(x)
    hot[at, 33] = 1
    ok = convolve64(hot, np.abs(wm)) == 0
    assert np.array_equal(np.isfinite(y), ok)
    assert np.all(np.abs(y - ref)[ok] <= 9 * 68 * 2.0 ** -24 * bound[ok] + 2.0 ** -24 * np.abs(ref[ok]))
