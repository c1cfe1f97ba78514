"""The 32 x 32 form on triples of bfloat16 (gpu), by the checks and tolerances of the other forms on triples: edges, every bit of
single products, values of very different size, data outside the triples' range; and launches in two parts."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
import test_gpu_conv1x1_pairs as T
import workloads as W

pytestmark = pytest.mark.gpu
FORM = 2032


@pytest.mark.parametrize("args", [
    (1, 128, 128, 0, 4, 4),            # one pixel, four units
    (31, 68, 96, 0, 4, 4),             # three units, the last one of one piece, a wave without any
    (32, 132, 4, 10, 4, 4),            # a pair of bundles with one group
    (33, 192, 136, 10, 8, 4),          # one pixel in the second tile
    (65, 256, 260, 30, 4, 1),          # a single bundle in the last pair
    (97, 324, 48, 50, 4, 2),
    (300, 1024, 256, 80, 8, 8),        # eight units per wave
], ids=str)
def test_tile_edges(args):
    T.test_tile_edges(FORM, *args)


@pytest.mark.parametrize("kind", ["tiny pixel", "huge value", "first chunks tiny", "later chunks tiny", "all tiny", "all huge", "zero pixels"])
def test_unusual_magnitudes(kind):
    T.test_unusual_magnitudes(FORM, kind)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38])
def test_infinities_and_nan(value):
    T.test_infinities_and_nan_reach_what_keeps_their_block_and_nothing_else(FORM, value)


@pytest.mark.parametrize("args", [(128, 128, 0, 4, 4), (324, 260, 30, 4, 1), (1024, 96, 70, 4, 2)], ids=str)
def test_single_products(args):
    T.test_single_products_keep_every_bit(FORM, *args)


@pytest.mark.parametrize("kind", [("large activations, small weights", 40), ("removed", 1e20), ("one piece", 1e20),
                                  ("small beside one", 1e-40), ("all", 1e-36), ("all", 1e30)], ids=str)
def test_large_and_small(kind):
    T.test_large_values_cost_small_ones_nothing(FORM, kind)


def test_outside_the_range_and_long_sums(monkeypatch):
    monkeypatch.setattr(T, "FORMS", (FORM,))
    T.test_activations_below_the_range_against_huge_weights()
    for args in [(128, 128, 0), (512, 512, 30), (1024, 256, 70)]:
        T.test_long_sums_are_no_further_off_than_32_bit_ones(*args)
    T.test_marks_stay_with_their_tile(FORM)
    for spoilt in (1, 13, 200):
        T.test_outputs_done_again_one_by_one_and_side_by_side(FORM, spoilt)


@pytest.mark.parametrize("m,K,N", [(50176, 512, 512), (49152 + 1, 388, 512)])
def test_whole_rounds_and_the_rest(m, K, N):
    """A launch whose last round would be short leaves as two: every pixel as in one launch of the form of the whole rounds."""
    p, w, mask, b = T.pack(K, N, 30)
    x = torch.from_numpy(W.uniform_activation(9020, (1, 1, m, K))).cuda()
    y, one = torch.full((1, 1, m, N), float("nan"), device="cuda"), torch.empty((1, 1, m, N), device="cuda")
    S.sbn_conv1x1_sparse(p, x, y, 1, 1, m)
    S.sbn_force_kernel_form(S.SBN_CONV1X1, 2256)
    try:
        S.sbn_conv1x1_sparse(p, x, one, 1, 1, m)
        torch.cuda.synchronize()
    finally:
        S.sbn_force_kernel_form(S.SBN_CONV1X1, 0)
    whole = m // 128 // 128 * 128 * 128            # (256 compute units, two column tiles)
    assert torch.equal(y[0, 0, :whole], one[0, 0, :whole])
    scale = x[0, 0].abs() @ torch.from_numpy(np.abs(T.kept_weights(w, mask, 4, 4))).float().cuda().T
    assert ((y - one).abs()[0, 0] <= (K / 16 + 16) * 2.0 ** -23 * scale + 2.0 ** -22).all()


@pytest.mark.parametrize("m,K,N,pct,taken", [
    (12544, 1024, 64, 70, True),       # up to 64 output channels
    (5121, 512, 64, 90, False),        # 1.26 tiles per compute unit, little kept
    (8225, 512, 64, 95, True),         # a little over two
    (5121, 192, 64, 80, True),         # the fewest input channels, a tile more than 1.25
    (16385, 192, 64, 80, False),       # a tile more than four
    (2500, 768, 64, 60, True),         # many input channels: from 0.6 tiles on
    (2400, 768, 64, 60, False),
    (2500, 764, 64, 60, False),
    (7186, 1024, 96, 70, True),        # more output channels, three tenths kept
    (7186, 1024, 96, 75, False),
    (3000, 260, 256, 60, True),
    (750, 512, 512, 60, False),        # few pixels for the channels
    (1372, 512, 512, 50, False),       # (a margin of 1.07)
    (1372, 512, 512, 40, True),        # (1.28)
])
def test_layers_that_keep_less(m, K, N, pct, taken):
    """The automatic choice and the forced form agree bit for bit where the rule takes the form, for 256 compute units; and are close elsewhere."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 compute units")
    w = W.he_weights(9030, N, 1, 1, K)
    mask = S.sbn_prune_magnitude(w, S.SBN_CONV1X1, 4, 4, pct)
    auto, forced = S.sbn_pack(S.SBN_CONV1X1, w, 4, 4, mask=mask), T.pack_wide(w, 4, 4, mask=mask)
    x = W.uniform_activation(9031, (1, 1, m, K))
    y, one = T.run(auto, x, N, 0), T.run(forced, x, N, FORM)
    assert np.array_equal(y, one) == taken
    scale = np.abs(x[0, 0]) @ np.abs(T.kept_weights(w, mask, 4, 4)).astype(np.float32).T
    assert (np.abs(y - one)[0, 0] <= K * 2.0 ** -23 * scale).all()
