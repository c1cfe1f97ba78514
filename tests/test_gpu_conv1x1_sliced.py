"""The 1x1 form whose workgroups share a tile's input channels between slices of four waves (gpu): edges of tiles, chunks and slices against
the oracle, which of them the launch rule takes, and non-finite values."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from helpers import assert_within_bound
from test_gpu_conv1x1 import run_layer
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture
def forced():
    yield lambda form: S.sbn_force_kernel_form(S.SBN_CONV1X1, form)
    S.sbn_force_kernel_form(S.SBN_CONV1X1, 0)


@pytest.mark.parametrize("form", [402, 404])
@pytest.mark.parametrize("m,K,N,go,gi,pct", [
    (1, 68, 4, 4, 4, 0),               # two chunks: slices without any; one pixel, one group
    (63, 128, 16, 4, 4, 50),
    (64, 132, 64, 4, 1, 70),           # the third chunk of one piece
    (65, 196, 68, 4, 4, 90),           # one pixel and one group in second tiles
    (130, 256, 72, 8, 4, 95),
    (200, 324, 120, 8, 2, 50),         # six chunks: slices of two and of one
    (129, 576, 192, 4, 8, 100),        # nothing kept
    (70, 1024, 64, 8, 8, 60),
])
def test_edges(forced, form, m, K, N, go, gi, pct):
    wt, b = W.he_weights(8100 + K, N, 1, 1, K), W.small_bias(8101, N) * 20
    x = W.uniform_activation(8102, (1, 1, m, K))
    forced(form)
    y, ref, bound = run_layer(x, wt, go, gi, bias=b, act=S.SBN_ACT_RELU, pct=pct)
    assert_within_bound(y, ref, bound, f"{form, m, K, N, go, gi, pct}")


@pytest.mark.parametrize("form", [402, 404])
def test_infinities_and_nan_reach_what_keeps_their_block_and_nothing_else(forced, form):
    m, K, N = 70, 324, 72
    wt = W.he_weights(8110, N, 1, 1, K)
    x = W.uniform_activation(8111, (1, 1, m, K))
    spoilt = x.copy()
    where = [(0, 0), (5, 63), (30, 64), (63, 200), (64, 323)]
    for i, (pix, ch) in enumerate(where):
        spoilt[0, 0, pix, ch] = (np.inf, np.nan, -np.inf)[i % 3]
    forced(form)
    y, y2 = run_layer(x, wt, 4, 4, pct=50)[0][0, 0], run_layer(spoilt, wt, 4, 4, pct=50)[0][0, 0]
    kept = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 50).reshape(N // 4, K // 4) != 0
    reached = np.zeros((m, N), bool)
    for pix, ch in where:
        reached[pix] = np.repeat(kept[:, ch // 4], 4)
    assert reached.any() and not np.isfinite(y2[reached]).any()
    assert np.array_equal(y[~reached], y2[~reached])


@pytest.mark.parametrize("m,K,N,pct,form", [
    (784, 1024, 1024, 90, 404),        # 0.81 tiles per compute unit
    (784, 256, 1024, 80, 402),
    (3136, 512, 512, 90, 402),         # 1.53 tiles
    (3136, 512, 512, 50, 0),
    (784, 192, 1024, 90, 0),
    (4096, 1024, 512, 90, 0),          # 2 tiles
    (569, 384, 1264, 70, 0),           # 0.70 tiles, more than 512 outputs: 1.1 times slower than the split form
    (690, 384, 1264, 70, 402),         # 0.86
    (4485, 680, 112, 95, 404),         # 0.55, of few outputs
    (821, 384, 912, 60, 0),            # 0.72: two slices would add up too long
    (768, 576, 880, 80, 0),            # 0.66
    (768, 576, 1200, 80, 404),         # 0.89
    (407, 960, 1056, 95, 0),           # the split form has eight waves,
    (5464, 720, 104, 95, 404),         # 16 outputs to each of which read the pixels again where they are many
    (2600, 520, 512, 97, 0),           # 1.28 tiles, of little work
    (2600, 640, 512, 80, 0),           # 1.28 tiles, 0.28 of them for split workgroups,
    (2304, 704, 640, 80, 402),         # 1.41, 0.47
    (12800, 1024, 128, 80, 0),         # 1.56, few outputs
    (1157, 1008, 1264, 99, 402),       # 1.48, 20 column tiles
    (2368, 768, 448, 95, 0),           # 1.01 tiles, 0.14 of them for split workgroups
    (2112, 768, 832, 95, 402),         # 1.68, 33 pixel tiles: 2.03 tiles per unit
])
def test_rule(forced, m, K, N, pct, form):
    """Counted for 256 compute units: the bits of the forced form, and on the other side of the lines other bits than either."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 compute units")
    wt = W.he_weights(8120 + K, N, 1, 1, K)
    mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, pct)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask)
    x = torch.from_numpy(W.uniform_activation(8121, (1, 1, m, K))).cuda()

    def run(f):
        y = torch.full((1, 1, m, N), float("nan"), device="cuda")
        forced(f)
        S.sbn_conv1x1_sparse(p, x, y, 1, 1, m)
        torch.cuda.synchronize()
        return y

    auto, two, four = run(0), run(402), run(404)
    assert not torch.equal(two, four)
    assert [torch.equal(auto, two), torch.equal(auto, four)] == [form == 402, form == 404]


@pytest.mark.parametrize("m,K,N,pct,replaced", [
    (3508, 200, 208, 99, 12),          # short sums: what counts is how few additions round
    (3508, 200, 208, 95, 12),          # two slices
    (784, 256, 1024, 80, 504),         # that add pairs in 32 bits
    (1143, 320, 776, 60, 504),         # long sums for two slices
    (784, 1024, 1024, 80, 504),        # four slices
    (3234, 3656, 152, 81, 508),        # where the split form has eight waves
    (6395, 592, 256, 99, 12),          # more than one tile per compute unit
    (1157, 1008, 1264, 99, 12),
    (3136, 1024, 512, 70, 12),
])
def test_no_further_from_the_exact_sum_than_the_form_it_replaces(forced, m, K, N, pct, replaced):
    """The rule's choice against the 32-bit form that would run without it: the same products, and in the sliced form every partial sum is
    shorter or joins in 64 bits, so the error's norm over all outputs must not be larger."""
    wt = W.he_weights(8140 + K, N, 1, 1, K)
    mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, pct)
    b = W.small_bias(8141, N)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, bias=b)
    x = np.maximum(W.uniform_activation(8142, (1, 1, m, K)), 0)
    xd = torch.from_numpy(x).cuda()
    kept = wt.reshape(N, K).astype(np.float64) * np.repeat(np.repeat(mask.reshape(N // 4, K // 4) != 0, 4, 0), 4, 1)
    ref = x[0, 0].astype(np.float64) @ kept.T + b

    def error(form):
        y = torch.full((1, 1, m, N), float("nan"), device="cuda")
        forced(form)
        S.sbn_conv1x1_sparse(p, xd, y, 1, 1, m)
        torch.cuda.synchronize()
        return np.linalg.norm(y.cpu().numpy()[0, 0] - ref) / np.linalg.norm(ref)

    chosen, before = error(0), error(replaced)
    assert chosen <= before, (chosen, before)


def test_tiles_are_spread_evenly(forced):
    """180 tiles of 64 x 64 are one round of workgroups of a device of 256 compute units, as 160 are, although 9 pixel tiles do not divide
    among its eight dies (with two rounds on one of them the launch takes 1.8 times as long)."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 compute units")
    K, N, took = 512, 1280, []
    wt = W.he_weights(8130, N, 1, 1, K)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 70))
    forced(404)
    for m in (8 * 64, 9 * 64):
        x = torch.from_numpy(W.uniform_activation(8131, (1, 1, m, K))).cuda()
        y = torch.empty((1, 1, m, N), device="cuda")
        S.sbn_conv1x1_sparse(p, x, y, 1, 1, m)
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(50):
                S.sbn_conv1x1_sparse(p, x, y, 1, 1, m)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        took.append(sorted(times)[4])
    assert took[1] < 1.4 * took[0], took
