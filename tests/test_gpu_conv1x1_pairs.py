"""The 1x1 forms on triples of bfloat16 (gpu): tile edges against the oracle, every bit of single products, values of
very different size side by side, and data outside the triples' range, where the kernel falls back on
32-bit multiply-adds.

Tolerance: that of every fp32 kernel here, 1e-4 * sum|w||x| per output, where none is derived beside the test."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu
FORMS = (2064, 2256)


def pack_wide(w, go, gi, **kw):
    """A layer with the tables of the wide forms, whether or not the automatic choice would use them."""
    S.sbn_force_kernel_form(S.SBN_CONV1X1, 2064)
    try:
        return S.sbn_pack(S.SBN_CONV1X1, w, go, gi, **kw)
    finally:
        S.sbn_force_kernel_form(S.SBN_CONV1X1, 0)


def pack(K, N, pct, go=4, gi=4, relu=True, bias=True):
    w = W.he_weights(9000 + K + N, N, 1, 1, K)
    b = W.small_bias(9001, N) * 20 if bias else None
    mask = S.sbn_prune_magnitude(w, S.SBN_CONV1X1, go, gi, pct)
    p = pack_wide(w, go, gi, mask=mask, bias=b, act=S.SBN_ACT_RELU if relu else S.SBN_ACT_NONE)
    return p, w, mask, b


def kept_weights(w, mask, go, gi):
    """[c_out][c_in] in 64 bits, removed blocks zero."""
    N, K = w.shape[0], w.shape[-1]
    return w.reshape(N, K) * np.repeat(np.repeat(mask.reshape(N // go, K // gi) != 0, go, 0), gi, 1).astype(np.float64)


def run(p, x, N, form):
    xd = torch.from_numpy(x).cuda()
    yd = torch.full((1, 1, x.shape[2], N), float("nan"), device="cuda")
    S.sbn_force_kernel_form(S.SBN_CONV1X1, form)
    try:
        S.sbn_conv1x1_sparse(p, xd, yd, 1, 1, x.shape[2])
        torch.cuda.synchronize()
    finally:
        S.sbn_force_kernel_form(S.SBN_CONV1X1, 0)
    return yd.cpu().numpy()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("m,K,N,pct,go,gi", [
    (1, 128, 128, 0, 4, 4),            # one pixel, two chunks
    (63, 132, 96, 0, 4, 4),            # a ragged last chunk of four channels
    (64, 192, 136, 10, 8, 4),          # channels past a tile
    (65, 256, 260, 30, 4, 1),          # one bundle of four channels in the second column tile
    (127, 324, 16, 50, 4, 2),          # one bundle
    (129, 512, 512, 70, 4, 4),
    (300, 1024, 256, 80, 8, 8),        # odd number of tiles, many chunks
])
def test_tile_edges(form, m, K, N, pct, go, gi):
    p, w, mask, b = pack(K, N, pct, go, gi)
    x = W.uniform_activation(9002 + m, (1, 1, m, K))
    ref, bound = R.sparse_conv_reference(x, w, mask, go, gi, bias=b, act=R.ACT_RELU)
    y = run(p, x, N, form)
    assert_within_bound(y, ref, bound, f"form {form}")
    # a rounding of 2^-23 of what has been summed per step of 16 channels, and 8 for the small sums, bias and oracle
    assert np.all(np.abs(y - ref) <= (K / 16 + 8) * 2.0 ** -23 * (bound + np.abs(b)))


@pytest.mark.parametrize("m", [128 * 256 * 2 + 3])
def test_more_tiles_than_workgroups(m):
    """The streaming form takes several tiles per workgroup; sums and marks start afresh with each."""
    p, w, mask, b = pack(128, 256, 0)
    x = W.uniform_activation(9003, (1, 1, m, 128))
    x[0, 0, ::2] *= np.float32(2.0 ** -9)
    x[0, 0, 5000:9000] *= np.float32(2.0 ** 20)
    ref, bound = R.sparse_conv_reference(x, w, mask, 4, 4, bias=b, act=R.ACT_RELU)
    for form in (2256, 0):
        assert_within_bound(run(p, x, 256, form), ref, bound, f"form {form}")


def unusual(kind, x):
    x = x.copy()
    if kind == "tiny pixel":
        x[0, 0, 5] *= np.float32(1e-15)
    elif kind == "huge value":                # filters that do not keep its block must not feel it, nor its neighbours
        x[0, 0, 5, 9] = 1e15
    elif kind == "first chunks tiny":         # the sums so far are rescaled
        x[..., :128] *= np.float32(1e-12)
    elif kind == "later chunks tiny":
        x[..., 128:] *= np.float32(1e-12)
    elif kind == "all tiny":
        x *= np.float32(1e-25)
    elif kind == "all huge":
        x *= np.float32(1e25)
    elif kind == "zero pixels":
        x[0, 0, 3:40] = 0
    return x


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("kind", ["tiny pixel", "huge value", "first chunks tiny", "later chunks tiny", "all tiny", "all huge",
                                  "zero pixels"])
def test_unusual_magnitudes(form, kind):
    p, w, mask, b = pack(256, 256, 30, relu=False)
    x = unusual(kind, W.uniform_activation(9004, (1, 1, 200, 256)))
    ref, bound = R.sparse_conv_reference(x, w, mask, 4, 4, bias=b)
    assert_within_bound(run(p, x, 256, form), ref, bound, kind)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38])
def test_infinities_and_nan_reach_what_keeps_their_block_and_nothing_else(form, value):
    p, w, mask, b = pack(256, 256, 30, relu=False)
    x = W.uniform_activation(9005, (1, 1, 200, 256))
    clean = run(p, x, 256, 504)
    x[0, 0, 7, 130] = value
    y, y32 = run(p, x, 256, form), run(p, x, 256, 504)
    assert np.array_equal(np.isnan(y), np.isnan(y32)) and np.array_equal(np.isinf(y), np.isinf(y32))
    keeps = np.repeat(mask.reshape(64, 64)[:, 130 // 4] != 0, 4)
    assert np.isfinite(y[0, 0, 7, ~keeps]).all()
    rows = np.arange(200) != 7
    assert np.allclose(y[0, 0, rows], clean[0, 0, rows], rtol=0, atol=1e-4)


# ---- every bit of the operands, whatever stands beside them ------------------------------------

# One product, exact but for what the kernel leaves out (at most 2^-24 of it), the rounding of the result (2^-24) and
# those of the small sums (five of 2^-23 of 2^-7 of it): 2.1 * 2^-24.
ONE_PRODUCT = 2.25 * 2.0 ** -24


@pytest.mark.parametrize("form", FORMS + (0,))
@pytest.mark.parametrize("K,N,pct,go,gi", [(128, 128, 0, 4, 4), (324, 260, 30, 4, 1), (512, 256, 50, 8, 4), (1024, 96, 70, 4, 2)])
def test_single_products_keep_every_bit(form, K, N, pct, go, gi):
    """One active channel per pixel: an output is one product of a weight and an activation."""
    p, w, mask, _ = pack(K, N, pct, go, gi, relu=False, bias=False)
    m = 4500 if N > 100 else 11300                    # (so many that the automatic choice is free to take a wide form)
    x = np.zeros((1, 1, m, K), np.float32)
    x[0, 0, np.arange(m), np.arange(m) % K] = W.uniform_activation(9006, (m,)) + np.float32(1.5)
    wm = kept_weights(w, mask, go, gi)
    ref = x[0, 0, np.arange(m), np.arange(m) % K].astype(np.float64)[:, None] * wm[:, np.arange(m) % K].T
    assert np.all(np.abs(run(p, x, N, form)[0, 0] - ref) <= ONE_PRODUCT * np.abs(ref))


def spread(kind, K, N):
    """Weights, block shape, mask and activations of a layer whose large values meet small or removed weights."""
    w = W.he_weights(9007, N, 1, 1, K)
    x = np.abs(W.uniform_activation(9008, (1, 1, 4500, K)))
    gi = 1 if kind[0] == "removed" else 4
    mask = np.ones((N // 4, K // gi), np.uint8)
    if kind[0] == "large activations, small weights":
        x[..., ::4] *= np.float32(2.0) ** kind[1]
        w[..., ::4] *= np.float32(2.0) ** -kind[1]
    elif kind[0] == "removed":
        mask[:, ::4] = 0
        x[..., ::4] = kind[1]
    elif kind[0] == "one piece":
        mask[:, :] = 1
        mask[:, 20:] = 0
        x[...] = 0
        x[..., 8:12] = 0.5
        x[..., 90] = kind[1]
    elif kind[0] == "one filter of four":
        x[..., 9] = kind[1]
        w[np.arange(N) % 4 != 1, :, :, 8:12] = 0
    elif kind[0] == "small beside one":
        x[..., 1::2] *= np.float32(kind[1])
    elif kind[0] == "all":
        x *= np.float32(kind[1])
    return w, gi, mask, x


@pytest.mark.parametrize("form", FORMS + (0,))
@pytest.mark.parametrize("kind", [("large activations, small weights", 32), ("large activations, small weights", 40),
                                  ("large activations, small weights", 48), ("removed", 1e12), ("removed", 1e15), ("removed", 1e20),
                                  ("one piece", 1e20), ("one filter of four", 1e15), ("small beside one", 1e-33),
                                  ("small beside one", 1e-40), ("all", 1e-30), ("all", 1e-36), ("all", 1e30)], ids=str)
def test_large_values_cost_small_ones_nothing(form, kind):
    K, N = 256, 256
    w, gi, mask, x = spread(kind, K, N)
    p = pack_wide(w, 4, gi, mask=mask)
    ref, bound = R.sparse_conv_reference(x, w, mask, 4, gi)
    err = np.abs(run(p, x, N, form) - ref)
    # every sum of 32-bit floats: a rounding of 2^-23 of what has been summed, c_in / 16 + 6 of them in the wide
    # form, and half of one in the oracle's result; 32-bit results below 2^-126 are multiples of 2^-149
    assert np.all(err <= 23 * 2.0 ** -23 * bound + 2.0 ** -149 * K), (err / bound).max()


def test_activations_below_the_range_against_huge_weights():
    """The last bits of an activation below 2^-110 do not fit a bfloat16; times a large weight they show."""
    K, N = 256, 256
    w, mask = W.he_weights(9009, N, 1, 1, K) * np.float32(1e30), np.ones((N // 4, K // 4), np.uint8)
    x = np.abs(W.uniform_activation(9010, (1, 1, 300, K)))
    x[0, 0, 17:250] *= np.float32(1e-36)
    x[0, 0, 100] = 0
    p = pack_wide(w, 4, 4, mask=mask)
    ref, bound = R.sparse_conv_reference(x, w, mask, 4, 4)
    for form in FORMS:
        assert np.all(np.abs(run(p, x, N, form) - ref) <= K * 2.0 ** -24 * bound)


@pytest.mark.parametrize("K,N,pct", [(128, 128, 0), (256, 256, 50), (512, 512, 30), (1024, 256, 70)])
def test_long_sums_are_no_further_off_than_32_bit_ones(K, N, pct):
    """Against 64 bits, as a whole: at most what one chain of 32-bit multiply-adds per output shows."""
    p, w, mask, b = pack(K, N, pct, relu=False)
    x = np.maximum(W.normal_weights(9011, (1, 1, 512, K), 1.0), 0)
    wm = kept_weights(w, mask, 4, 4)
    ref = x[0, 0].astype(np.float64) @ wm.T + b
    chain = np.broadcast_to(b, (512, N)).astype(np.float32)
    for k in range(K):                                 # (64-bit products are exact: one rounding per multiply-add)
        chain = (chain + x[0, 0, :, k:k + 1].astype(np.float64) * wm[:, k]).astype(np.float32)
    limit = np.linalg.norm(chain - ref)
    for form in FORMS:
        assert np.linalg.norm(run(p, x, N, form)[0, 0] - ref) <= limit


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("spoilt", [1, 12, 13, 200])
def test_outputs_done_again_one_by_one_and_side_by_side(form, spoilt):
    """Up to 12 of a wave's outputs are done again by the wave together, more by their lanes; an overflowing activation
    that only a part of the filters keeps."""
    p, w, mask, b = pack(324, 96, 30, relu=False)
    x = W.uniform_activation(9012, (1, 1, 200, 324))
    x[0, 0, :spoilt, 131] = np.inf
    y = run(p, x, 96, form)
    keeps = np.repeat(mask.reshape(24, 81)[:, 131 // 4] != 0, 4)
    assert not np.isfinite(y[0, 0, :spoilt, keeps]).any()
    x[0, 0, :spoilt, 131] = 0
    ref, bound = R.sparse_conv_reference(x, w, mask, 4, 4, bias=b)
    ok = np.isfinite(y)
    assert ok[0, 0, spoilt:].all() and ok[0, 0, :, ~keeps].all()
    assert np.all(np.abs(y - ref)[ok] <= 324 * 2.0 ** -24 * bound[ok] + 2.0 ** -23 * np.abs(ref[ok]))


@pytest.mark.parametrize("form", FORMS)
def test_marks_stay_with_their_tile(form):
    """Pixels below the range here and there in many tiles, which the streaming form walks one after the other."""
    K, N, m = 128, 256, 128 * 128 * 2 + 77
    w = W.he_weights(9013, N, 1, 1, K) * np.float32(1e30)
    mask = np.ones((N // 4, K // 4), np.uint8)
    x = np.abs(W.uniform_activation(9014, (1, 1, m, K)))
    x[0, 0, 5::97] *= np.float32(1e-36)
    p = pack_wide(w, 4, 4, mask=mask)
    wm = kept_weights(w, mask, 4, 4)
    ref, bound = x[0, 0].astype(np.float64) @ wm.T, x[0, 0].astype(np.float64) @ np.abs(wm).T
    assert np.all(np.abs(run(p, x, N, form)[0, 0] - ref) <= K * 2.0 ** -24 * bound)


@pytest.mark.parametrize("form", FORMS + (0,))
@pytest.mark.parametrize("value", [1e-38, 1e-44, 3.4e38])
def test_weights_outside_the_range_stay_with_the_32_bit_kernels(form, value):
    K, N, m = 128, 128, 300
    w = W.he_weights(9015, N, 1, 1, K)
    w[7, 0, 0, 60:64] = np.float32(value)
    mask = np.ones((N // 4, K // 4), np.uint8)
    x = np.zeros((1, 1, m, K), np.float32)
    x[0, 0, :, 60] = 0.25
    p = pack_wide(w, 4, 4, mask=mask)
    ref = 0.25 * w[:, 0, 0, 60].astype(np.float64)
    assert np.all(np.abs(run(p, x, N, form)[0, 0] - ref) <= 2.0 ** -23 * np.abs(ref) + 2.0 ** -149)
