"""Depthwise + 1x1 pairs in one launch (csrc/sbn_dwpw.hip) where a workgroup walks several tiles: more tiles than workgroups are
resident, in every form of the kernel (four and eight waves, stride 1 and 2, dense and pattern-pruned), against the oracle's two
layers.  Tolerance as for the fused pairs in test_gpu_chain.py: the 1x1 layer's, plus the depthwise layer's carried through the weights."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
import workloads as W
from helpers import assert_within_bound
from oracle import reference as R

pytestmark = pytest.mark.gpu


def resident(K, N, stride, tiles):
    """Workgroups that the kernel's form for these sizes keeps on the chip: as many as the waves that a compute unit holds of it allow."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if N > 64:
        return 2 * cus
    return (4 if stride == 1 else 3 if K == 32 or tiles <= 4 * cus else 2) * cus


@pytest.mark.parametrize("n,h,w,K,N,stride,patterned,one_launch", [
    (66, 33, 31, 32, 64, 1, False, True),        # 1320 tiles, ragged both ways
    (72, 40, 24, 64, 60, 1, True, True),         # 1080 whole tiles of two sub-chunks, fewer channels than the waves cover
    (72, 33, 23, 96, 36, 1, False, True),        # 1080 of three
    (108, 25, 17, 32, 12, 1, True, True),        # 1296 tiles, most of them at a border
    (35, 33, 31, 96, 128, 1, False, True),
    (35, 33, 31, 128, 100, 1, True, True),
    (35, 65, 61, 64, 128, 2, False, True),
    (60, 66, 62, 32, 64, 2, False, True),        # stride 2, four waves: 1200 tiles, three workgroups per compute unit
    (45, 65, 61, 64, 40, 2, True, True),         # 900 tiles
    (45, 66, 62, 96, 8, 2, False, True),
    (60, 65, 62, 64, 40, 2, True, True),         # 1200 tiles of several sub-chunks: two
    (60, 66, 61, 96, 64, 2, False, True),
    (600, 5, 3, 64, 96, 1, False, True),         # an image smaller than a tile: every step moves to another image
    (1, 1, 123400, 128, 8, 1, False, False),     # rows past the offsets' range: two launches, whatever the switch says
])
def test_tiles_in_a_stream(n, h, w, K, N, stride, patterned, one_launch):
    seed = 9900 + K + N + stride
    dw_w, dw_b = W.normal_weights(seed, (K, 3, 3), 0.4), W.small_bias(seed + 1, K) * 10
    pattern = S.sbn_dw_pattern_select(dw_w, 16) if patterned else None
    wt, b = W.he_weights(seed + 2, N, 1, 1, K), W.small_bias(seed + 3, N) * 10
    mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 50)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, bias=b, act=S.SBN_ACT_RELU)
    chain = S.sbn_chain_create([S.dw_item(dw_w, dw_b, stride=stride, act=S.SBN_ACT_RELU, pattern=pattern, go=16), S.sparse_item(p)])
    if patterned:
        dw_w = R.dw_pattern_apply(dw_w, pattern, 16)
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, h, w)
    tiles = n * ((oh + 7) // 8) * ((ow + 7) // 8)
    assert not one_launch or tiles > resident(K, N, stride, tiles), tiles
    x = W.uniform_activation(seed + 5, (n, h, w, K))
    ws = torch.full((S.sbn_chain_workspace(chain, n, h, w) // 4,), float("nan"), device="cuda")
    y = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    S.sbn_chain_set_fusion(chain, 2)
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), y, n, h, w, ws)
    torch.cuda.synchronize()
    assert bool(ws.isnan().all()) == one_launch
    mid, bound_dw = R.dwconv3x3_nhwc(x, dw_w, dw_b, stride=stride, act=R.ACT_RELU)
    ref, bound_pw = R.sparse_conv_reference(mid, wt, mask, 4, 4, bias=b, act=R.ACT_RELU)
    wm = np.abs(R.apply_mask(wt, mask, 4, 4).reshape(N, K).astype(np.float64))
    bound = bound_pw + (bound_dw.reshape(-1, K) @ wm.T).reshape(bound_pw.shape)
    assert_within_bound(y.cpu().numpy(), ref, bound, f"{n, h, w, K, N, stride, patterned}")


@pytest.mark.parametrize("n,h,w,N,patterned,acts,copies", [
    (1, 16, 16, 64, False, (1, 1, 1), None),     # one tile, a border on every side
    (2, 37, 45, 36, False, (1, 0, 0), None),     # odd extents: the last row and column of windows reach past the input
    (2, 36, 47, 12, True, (0, 1, 1), None),
    (40, 66, 81, 64, False, (1, 1, 1), None),    # 1200 tiles: several per workgroup
    (40, 66, 81, 60, True, (1, 1, 1), None),
    (3, 1, 1, 64, True, (1, 1, 1), None),        # one pixel
    (1, 2, 301, 64, False, (1, 1, 1), None),
    (2, 37, 45, 36, False, (1, 1, 1), 2),        # a copy of the result is the same launch
    (2, 37, 45, 36, False, (1, 1, 1), 1),        # of what is never in memory: the stem by itself
    (2, 37, 45, 36, False, (1, 1, 1), 0),        # ... and the pair as one
])
def test_stem_in_the_first_pairs_launch(n, h, w, N, patterned, acts, copies):
    """A 3 -> 32 channel stem of stride 2, a depthwise layer and a 1x1 layer as one launch against the oracle's three layers; every layer's
    bound is carried through the weights of those behind it (ReLU between them is 1-Lipschitz)."""
    K, seed = 32, 9950 + N
    act = [S.SBN_ACT_RELU if a else S.SBN_ACT_NONE for a in acts]
    st_w, st_b = W.he_weights(seed, 32, 3, 3, 3), W.small_bias(seed + 1, 32) * 10
    dw_w, dw_b = W.normal_weights(seed + 2, (K, 3, 3), 0.4), W.small_bias(seed + 3, K) * 10
    pattern = S.sbn_dw_pattern_select(dw_w, 16) if patterned else None
    wt, b = W.he_weights(seed + 4, N, 1, 1, K), W.small_bias(seed + 5, N) * 10
    mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 50)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, bias=b, act=act[2])
    chain = S.sbn_chain_create([S.stem_item(st_w, st_b, stride=2, act=act[0]),
                                S.dw_item(dw_w, dw_b, act=act[1], pattern=pattern, go=16), S.sparse_item(p)])
    if patterned:
        dw_w = R.dw_pattern_apply(dw_w, pattern, 16)
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, h, w)
    x = W.uniform_activation(seed + 6, (n, h, w, 3))
    ws = torch.full((S.sbn_chain_workspace(chain, n, h, w) // 4,), float("nan"), device="cuda")     # (fusion as it is by default: whatever the size)
    y = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    outs = None if copies is None else [torch.full((n, oh, ow, 32 if i < 2 else oc), float("nan"), device="cuda") if i == copies else None
                                        for i in range(3)]
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), y, n, h, w, ws, **({} if outs is None else {"layer_outputs": outs}))
    torch.cuda.synchronize()
    assert bool(ws.isnan().all()) == (copies in (None, 2))
    stem, b0 = R.conv_nhwc(x, st_w, st_b, stride=2, pad=1, act=acts[0] and R.ACT_RELU or R.ACT_NONE)
    mid, b1 = R.dwconv3x3_nhwc(stem, dw_w, dw_b, act=acts[1] and R.ACT_RELU or R.ACT_NONE)
    b1 = b1 + R.dwconv3x3_nhwc(b0.astype(np.float32), np.abs(dw_w), None)[0]
    ref, bound = R.sparse_conv_reference(mid, wt, mask, 4, 4, bias=b, act=acts[2] and R.ACT_RELU or R.ACT_NONE)
    wm = np.abs(R.apply_mask(wt, mask, 4, 4).reshape(N, K).astype(np.float64))
    bound = bound + (b1.reshape(-1, K).astype(np.float64) @ wm.T).reshape(bound.shape)
    assert_within_bound(y.cpu().numpy(), ref, bound, f"{n, h, w, N, patterned, acts}")
    if copies == 2:
        assert torch.equal(outs[2], y)


def test_small_stems_are_no_further_from_the_exact_result_than_three_launches():
    """Where the pair behind the stem would be two launches by the rule, the 1x1 layer's sums are exact to the last rounding but one in its
    few-pixel form.  The error's norm over all outputs, one launch against three, is the same but for which way single roundings fall: mean over
    the sizes at most 1.5 % more (1x1 sums kept in 32 bits and their bias added last: 6 % more)."""
    ratios = []
    for seed, (n, h, w, N) in enumerate([(4, 58, 45, 4), (7, 30, 46, 20), (3, 70, 19, 24), (2, 27, 50, 52), (6, 12, 58, 56), (5, 26, 82, 64)]):
        K, seed = 32, 9980 + 10 * seed
        st_w, st_b = W.he_weights(seed, 32, 3, 3, 3), W.small_bias(seed + 1, 32)
        dw_w, dw_b = W.normal_weights(seed + 2, (K, 3, 3), 0.4), W.small_bias(seed + 3, K)
        wt, b = W.he_weights(seed + 4, N, 1, 1, K), W.small_bias(seed + 5, N)
        mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 50)
        chain = S.sbn_chain_create([S.stem_item(st_w, st_b), S.dw_item(dw_w, dw_b),
                                    S.sparse_item(S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, bias=b, act=S.SBN_ACT_RELU))])
        x = torch.from_numpy(W.uniform_activation(seed + 6, (n, h, w, 3)))
        conv, f64 = torch.nn.functional.conv2d, lambda a: torch.from_numpy(np.asarray(a, np.float64))
        ref = conv(x.double().permute(0, 3, 1, 2), f64(st_w).permute(0, 3, 1, 2), f64(st_b), stride=2, padding=1).relu()
        ref = conv(ref, f64(dw_w)[:, None], f64(dw_b), padding=1, groups=K).relu()
        ref = conv(ref, f64(R.apply_mask(wt, mask, 4, 4).reshape(N, K, 1, 1)), f64(b)).relu().permute(0, 2, 3, 1)
        ws = torch.empty(S.sbn_chain_workspace(chain, n, h, w) // 4, device="cuda")
        errors = []
        for enable in (1, 0):
            S.sbn_chain_set_fusion(chain, enable)
            ws.fill_(float("nan"))
            y = torch.full(tuple(ref.shape), float("nan"), device="cuda")
            S.sbn_pointwise_chain(chain, x.cuda(), y, n, h, w, ws)
            torch.cuda.synchronize()
            assert bool(ws.isnan().all()) == (enable == 1)
            errors.append(float((y.cpu().double() - ref).norm()))
        ratios.append(errors[0] / errors[1])
    assert np.mean(ratios) <= 1.015, ratios


@pytest.mark.parametrize("stem", [False, True])
def test_images_of_more_than_two_to_the_31_elements(stem):
    """A depthwise input of 2.2 * 10^9 elements in one launch: the last rows against the oracle (they lie furthest from the tensors' starts), each
    of whose layers leaves out what the cut above them spoils."""
    K, N, h, w, seed = 32, 4, 60000, 1150, 9995
    st_w, dw_w, wt = W.he_weights(seed, 32, 3, 3, 3), W.normal_weights(seed + 1, (K, 3, 3), 0.4), W.he_weights(seed + 2, N, 1, 1, K)
    items = [S.dw_item(dw_w, None), S.sparse_item(S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4))]
    chain = S.sbn_chain_create([S.stem_item(st_w, None)] + items if stem else items)
    shape = (1, 2 * h, 2 * w, 3) if stem else (1, h, w, K)
    x = torch.rand(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed)).mul_(2).sub_(1)
    ws = torch.zeros(S.sbn_chain_workspace(chain, *shape[:3]) // 4, device="cuda")
    ws[:4096].fill_(float("nan"))
    y = torch.full((1, h, w, N), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, x, y, *shape[:3], ws)
    torch.cuda.synchronize()
    assert bool(ws[:4096].isnan().all())
    assert not bool(y.isnan().any())
    tail = x[:, -24 if stem else -12:].cpu().numpy()
    b0 = None
    if stem:
        tail, b0 = R.conv_nhwc(tail, st_w, None, stride=2, pad=1, act=R.ACT_RELU)
    mid, bound = R.dwconv3x3_nhwc(tail, dw_w, None, act=R.ACT_RELU)
    if stem:
        bound = bound + R.dwconv3x3_nhwc(b0.astype(np.float32), np.abs(dw_w), None)[0]
    ref, bound_pw = R.sparse_conv_reference(mid, wt, None, 4, 4)
    bound = bound_pw + (bound.reshape(-1, K).astype(np.float64) @ np.abs(wt.reshape(N, K).astype(np.float64)).T).reshape(bound_pw.shape)
    assert_within_bound(y[:, -8:].cpu().numpy(), ref[:, -8:], bound[:, -8:], f"stem {stem}")


@pytest.mark.parametrize("stem,n,h,w,K,N,stride,patterned", [
    (False, 2, 21, 19, 64, 60, 1, False),
    (False, 2, 21, 19, 32, 64, 1, True),
    (False, 2, 21, 19, 64, 128, 1, True),        # eight waves
    (False, 2, 37, 35, 64, 40, 2, False),        # three workgroups per unit
    (False, 65, 37, 35, 96, 40, 2, True),        # two: more than four tiles per unit
    (False, 2, 37, 35, 96, 100, 2, False),
    (True, 2, 37, 45, 32, 36, 1, False),         # sums in 64 bits
    (True, 6, 70, 66, 32, 64, 1, True),          # and in 32
])
def test_infinities_and_nan_reach_what_reads_them_and_nothing_else(stem, n, h, w, K, N, stride, patterned):
    """Without activations every output that a spoilt input reaches over kept taps and blocks is not finite and every other keeps its bits; with
    ReLU (of NaN: 0) infinities lie where they do in separate launches (whose depthwise kernel multiplies the zeros of removed taps: not compared where
    there are any)."""
    seed = 9960 + K + N
    st_w, dw_w, wt = W.he_weights(seed, 32, 3, 3, 3), W.normal_weights(seed + 1, (K, 3, 3), 0.4), W.he_weights(seed + 2, N, 1, 1, K)
    pattern = S.sbn_dw_pattern_select(dw_w, 16) if patterned else None
    mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 50)
    c_in = 3 if stem else K
    x = W.uniform_activation(seed + 3, (n, h, w, c_in))
    spoilt = x.copy()
    where = [(0, 0, 0, 0), (0, h - 1, w - 1, c_in - 1), (n - 1, 7, 8, 1), (n - 1, 16, w - 1, 2), (n - 1, h - 1, 15, 0)]
    for i, at in enumerate(where):
        spoilt[at] = (np.inf, np.nan, -np.inf)[i % 3]

    def run(x, act, fusion):
        p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, act=act)
        items = [S.dw_item(dw_w, None, stride=stride, act=act, pattern=pattern), S.sparse_item(p)]
        chain = S.sbn_chain_create([S.stem_item(st_w, None, act=act)] + items if stem else items)
        S.sbn_chain_set_fusion(chain, fusion)
        oh, ow, oc = S.sbn_chain_output_shape(chain, n, h, w)
        ws = torch.full((S.sbn_chain_workspace(chain, n, h, w) // 4,), 7.0, device="cuda")
        y = torch.full((n, oh, ow, oc), 7.0, device="cuda")
        S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), y, n, h, w, ws)
        torch.cuda.synchronize()
        assert bool((ws == 7.0).all()) == (fusion != 0)
        return y.cpu().numpy()

    fused = 1 if stem else 2
    taps = R.dw_pattern_apply(np.ones((K, 3, 3), np.float32), pattern, 16) if patterned else np.ones((K, 3, 3), np.float32)
    reach = (~np.isfinite(spoilt)).astype(np.float32)
    if stem:
        reach = (R.conv_nhwc(reach, np.ones((32, 3, 3, 3), np.float32), None, stride=2, pad=1)[0] > 0).astype(np.float32)
    reach = R.dwconv3x3_nhwc(reach, taps, None, stride=stride)[0] > 0
    kept = np.repeat(np.repeat(mask.reshape(N // 4, K // 4) != 0, 4, 0), 4, 1)
    reach = reach.reshape(-1, K).astype(np.float32) @ kept.T.astype(np.float32) > 0
    clean, y = run(x, S.SBN_ACT_NONE, fused).reshape(-1, N), run(spoilt, S.SBN_ACT_NONE, fused).reshape(-1, N)
    assert reach.any() and not np.isfinite(y[reach]).any()
    assert np.array_equal(y[~reach], clean[~reach])

    one, separate = run(spoilt, S.SBN_ACT_RELU, fused), run(spoilt, S.SBN_ACT_RELU, 0)
    assert not np.isnan(one).any() and np.isinf(one).any()
    assert patterned or np.array_equal(np.isinf(one), np.isinf(separate))
