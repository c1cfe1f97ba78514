"""The 1x1 forms on pairs of 16-bit floats (gpu): tile edges against the oracle, and data outside the
pairs' range, where the kernel has to fall back on 32-bit multiply-adds.

Tolerance: that of every fp32 kernel here, 1e-4 * sum|w||x| per output.  The pairs themselves are good to
about 2^-22 of the largest product of an output plus K / 32 roundings of the sum (observed 3e-7)."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu
FORMS = (2064, 2256)


def pack(K, N, pct, go=4, gi=4, relu=True):
    w = W.he_weights(9000 + K + N, N, 1, 1, K)
    b = W.small_bias(9001, N) * 20
    mask = S.sbn_prune_magnitude(w, S.SBN_CONV1X1, go, gi, pct)
    assert np.count_nonzero(mask) * go * gi >= 128 * N           # else the layer has no pairs and the test tests nothing
    p = S.sbn_pack(S.SBN_CONV1X1, w, go, gi, mask=mask, bias=b, act=S.SBN_ACT_RELU if relu else S.SBN_ACT_NONE)
    return p, w, mask, b


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
    assert_within_bound(run(p, x, N, form), ref, bound, f"form {form}")


@pytest.mark.parametrize("m", [128 * 256 * 2 + 3])
def test_more_tiles_than_workgroups(m):
    """The streaming form takes several tiles per workgroup; the exponents start afresh with each."""
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
