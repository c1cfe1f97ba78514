"""Layer chaining on the GPU: sparse pointwise layers, dense depthwise 3x3 + ReLU between
them, global average pool and a dense classifier, checked layer by layer against the oracle
(each oracle layer is fed the GPU's previous output) and end to end on a small input."""
import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from oracle import reference as R
import workloads as W
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu


def build_stack(chans, hw, batch, pct, seed, strides):
    """Rearranged, pruned pointwise layers with depthwise layers in front of each."""
    L = len(chans) - 1
    pws = [dict(kind=S.SBN_CONV1X1, w=W.he_weights(seed + i, chans[i + 1], 1, 1, chans[i]), go=4, gi=4)
           for i in range(L)]
    perms = S.sbn_rearrange(pws, [-1] + list(range(L - 1)), pct, seed=seed, max_iters=300,
                            keep_output_order=[0] * (L - 1) + [1])
    perms = S.sbn_order_groups(pws, [-1] + list(range(L - 1)), pct, perms, keep_output_order=[0] * (L - 1) + [1])
    items, meta = [], []
    pin = None
    for i in range(L):
        dw_w = W.normal_weights(seed + 50 + i, (chans[i], 3, 3), 0.4)
        dw_b = W.small_bias(seed + 70 + i, chans[i])
        items.append(S.dw_item(dw_w, dw_b, stride=strides[i], act=S.SBN_ACT_RELU))
        meta.append(dict(kind="dw", w=dw_w, b=dw_b, stride=strides[i], order=pin))
        b = W.small_bias(seed + 90 + i, chans[i + 1])
        wp = R.permute_weights(pws[i]["w"], perms[i], pin)
        mask = S.sbn_prune_magnitude(wp, S.SBN_CONV1X1, 4, 4, pct)
        p = S.sbn_pack(S.SBN_CONV1X1, pws[i]["w"], 4, 4, mask=mask, bias=b, perm_out=perms[i], perm_in=pin,
                       act=S.SBN_ACT_RELU)
        items.append(S.sparse_item(p))
        meta.append(dict(kind="pw", w=pws[i]["w"], b=b, mask=mask, po=perms[i], pi=pin))
        pin = perms[i]
    return items, meta


def oracle_item(m, x):
    if m["kind"] == "dw":
        w, b = m["w"], m["b"]
        if m["order"] is not None:
            w, b = w[m["order"]], b[m["order"]]
        return R.dwconv3x3_nhwc(x, w, b, stride=m["stride"], act=R.ACT_RELU)
    if m["kind"] == "pw":
        return R.sparse_conv_reference(x, m["w"], m["mask"], 4, 4, bias=m["b"], perm_out=m["po"], perm_in=m["pi"],
                                       act=R.ACT_RELU)
    if m["kind"] == "pool":
        y = R.avgpool_nhwc(x)[:, None, None, :]
        return y, None
    raise AssertionError


def test_chain_layer_by_layer_and_end_to_end():
    chans, strides = [16, 32, 64, 64, 24], [1, 2, 1, 2]
    n, hw = 3, 18
    items, meta = build_stack(chans, hw, n, 50, 9000, strides)
    items.append(S.avgpool_item())
    meta.append(dict(kind="pool"))
    fc_w = W.he_weights(9100, 12, 1, 1, chans[-1])
    fc = S.sbn_pack(S.SBN_CONV1X1, fc_w, 4, 4, bias=W.small_bias(9101, 12))       # dense classifier: all blocks kept
    items.append(S.sparse_item(fc))
    meta.append(dict(kind="pw", w=fc_w, b=W.small_bias(9101, 12), mask=np.ones((3, chans[-1] // 4), np.uint8),
                     po=None, pi=None))
    meta[-1]["act_none"] = True
    chain = S.sbn_chain_create(items)
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, hw, hw)
    assert (oh, ow, oc) == (1, 1, 12)
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    x = W.uniform_activation(9200, (n, hw, hw, chans[0]))
    xd = torch.from_numpy(x).cuda()
    yd = torch.full((n, 1, 1, 12), float("nan"), device="cuda")
    # shapes of every item's output, to allocate the per-layer taps
    shapes, h, c = [], hw, chans[0]
    for m in meta:
        if m["kind"] == "dw":
            h = (h - 1) // m["stride"] + 1
        elif m["kind"] == "pw":
            c = m["w"].shape[0]
        else:
            h = 1
        shapes.append((n, h, h, c))
    taps = [torch.full(s, float("nan"), device="cuda") for s in shapes]
    S.sbn_pointwise_chain(chain, xd, yd, n, hw, hw, ws, layer_outputs=taps)
    torch.cuda.synchronize()
    outs = [t.cpu().numpy() for t in taps]
    assert np.array_equal(outs[-1], yd.cpu().numpy())

    # teacher-forced: oracle layer l is fed the GPU's output of layer l-1
    prev = x
    for i, m in enumerate(meta):
        if m.get("act_none"):
            ref, bound = R.sparse_conv_reference(prev, m["w"], m["mask"], 4, 4, bias=m["b"])
        else:
            ref, bound = oracle_item(m, prev)
        if bound is None:       # average pool: fp32 sum of 25 values vs fp64
            np.testing.assert_allclose(outs[i], ref, rtol=0, atol=1e-5)
        else:
            assert_within_bound(outs[i], ref, bound, f"chain item {i} ({m['kind']})")
        prev = outs[i]

    # end to end in original channel order, no rearrangement, same masks mapped back
    cur = x
    for m in meta:
        if m["kind"] == "dw":
            cur, _ = R.dwconv3x3_nhwc(cur, m["w"], m["b"], stride=m["stride"], act=R.ACT_RELU)
        elif m["kind"] == "pool":
            cur = R.avgpool_nhwc(cur)[:, None, None, :]
        else:
            wp = R.permute_weights(m["w"], m["po"], m["pi"])
            wt = R.unpermute_weights(R.apply_mask(wp, m["mask"], 4, 4), m["po"], m["pi"])
            cur, _ = R.conv_nhwc(cur, wt, m["b"], act=R.ACT_NONE if m.get("act_none") else R.ACT_RELU)
    np.testing.assert_allclose(outs[-1], cur, rtol=1e-3, atol=1e-4)


def test_chain_rejects_mismatched_orders_and_shapes():
    w1, w2 = W.he_weights(9300, 16, 1, 1, 8), W.he_weights(9301, 8, 1, 1, 16)
    po = W.random_permutation(9302, 16)
    a = S.sbn_pack(S.SBN_CONV1X1, w1, 4, 4, perm_out=po)
    b_bad = S.sbn_pack(S.SBN_CONV1X1, w2, 4, 4)                    # expects identity order
    b_ok = S.sbn_pack(S.SBN_CONV1X1, w2, 4, 4, perm_in=po)
    with pytest.raises(S.SbnError) as ei:
        S.sbn_chain_create([S.sparse_item(a), S.sparse_item(b_bad)])
    assert ei.value.code == -2
    chain = S.sbn_chain_create([S.sparse_item(a), S.sparse_item(b_ok)])
    with pytest.raises(S.SbnError):
        S.sbn_chain_create([S.sparse_item(a), S.sparse_item(a)])     # 16 channels out, 8 expected in
    with pytest.raises(S.SbnError):
        S.sbn_chain_create([S.sparse_item(a), S.dw_item(np.zeros((8, 3, 3), np.float32))])
    x = torch.zeros(1, 2, 2, 8, device="cuda")
    y = torch.zeros(1, 2, 2, 8, device="cuda")
    with pytest.raises(S.SbnError):
        S.sbn_pointwise_chain(chain, x, y, 1, 2, 2, None)            # workspace missing


def test_chain_with_3x3_layer():
    w3 = W.he_weights(9400, 16, 3, 3, 8)
    m3 = S.sbn_prune_magnitude(w3, S.SBN_CONV3X3, 4, 4, 50)
    a = S.sbn_pack(S.SBN_CONV3X3, w3, 4, 4, mask=m3, stride=2, act=S.SBN_ACT_RELU)
    w1 = W.he_weights(9401, 8, 1, 1, 16)
    b = S.sbn_pack(S.SBN_CONV1X1, w1, 4, 4)
    chain = S.sbn_chain_create([S.sparse_item(a), S.sparse_item(b)])
    n, hw = 2, 11
    assert S.sbn_chain_output_shape(chain, n, hw, hw) == (6, 6, 8)
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    x = W.uniform_activation(9402, (n, hw, hw, 8))
    yd = torch.empty(n, 6, 6, 8, device="cuda")
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), yd, n, hw, hw, ws)
    torch.cuda.synchronize()
    h1, _ = R.sparse_conv_reference(x, w3, m3, 4, 4, stride=2, pad=1, act=R.ACT_RELU)
    ref, bound = R.conv_nhwc(h1, w1)
    np.testing.assert_allclose(yd.cpu().numpy(), ref, rtol=1e-4, atol=1e-5)


def test_whole_mobilenet_chain_small_input():
    """Config 4 at a small input (2 x 64 x 64 x 3): stem -> 13 x (dw, sparse pw) -> pool -> classifier,
    every item checked against the oracle fed with the GPU's previous output."""
    import bench
    chain, meta = bench.build_mobilenet_chain(S, W, 50, max_iters=100)
    n, hw = 2, 64
    x = W.uniform_activation(9500, (n, hw, hw, 3))
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, hw, hw)
    assert (oh, ow, oc) == (1, 1, 1000)
    shapes, h, c = [], hw, 3
    for m in meta:
        if m["kind"] in ("dw", "stem"):
            h = (h - 1) // m["stride"] + 1
        if m["kind"] in ("pw", "stem"):
            c = m["w"].shape[0]
        if m["kind"] == "pool":
            h = 1
        shapes.append((n, h, h, c))
    taps = [torch.full(s, float("nan"), device="cuda") for s in shapes]
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    yd = torch.empty(n, 1, 1, 1000, device="cuda")
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), yd, n, hw, hw, ws, layer_outputs=taps)
    torch.cuda.synchronize()
    prev = x
    for i, m in enumerate(meta):
        out = taps[i].cpu().numpy()
        if m["kind"] == "stem":
            ref, bound = R.conv_nhwc(prev, m["w"], m["b"], stride=m["stride"], pad=1, act=R.ACT_RELU)
        elif m["kind"] == "dw":
            w, b = m["w"], m["b"]
            if m["order"] is not None:
                w, b = w[m["order"]], b[m["order"]]
            ref, bound = R.dwconv3x3_nhwc(prev, w, b, stride=m["stride"], act=R.ACT_RELU)
        elif m["kind"] == "pool":
            ref, bound = R.avgpool_nhwc(prev)[:, None, None, :], None
        else:
            ref, bound = R.sparse_conv_reference(prev, m["w"], m["mask"], m["go"], 4, bias=m["b"], perm_out=m["po"],
                                                 perm_in=m["pi"], act=m["act"])
        if bound is None:
            np.testing.assert_allclose(out, ref, rtol=0, atol=1e-5)
        else:
            assert_within_bound(out, ref, bound, f"mobilenet item {i} ({m['kind']})")
        prev = out
    assert np.array_equal(taps[-1].cpu().numpy(), yd.cpu().numpy())


@pytest.mark.parametrize("c_in,c_out,stride,hw", [(2, 8, 1, 9), (4, 16, 2, 10), (3, 32, 2, 13), (1, 4, 1, 5)])
def test_stem_item_alone(c_in, c_out, stride, hw):
    w = W.he_weights(9600 + c_in, c_out, 3, 3, c_in)
    b = W.small_bias(9601, c_out) * 10
    chain = S.sbn_chain_create([S.stem_item(w, b, stride=stride, act=S.SBN_ACT_RELU)])
    n = 3
    x = W.uniform_activation(9602, (n, hw, hw, c_in))
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, hw, hw)
    yd = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), yd, n, hw, hw, None)
    torch.cuda.synchronize()
    ref, bound = R.conv_nhwc(x, w, b, stride=stride, pad=1, act=R.ACT_RELU)
    assert_within_bound(yd.cpu().numpy(), ref, bound, "stem")


def test_stem_must_come_first():
    w1 = W.he_weights(9700, 4, 1, 1, 4)
    a = S.sbn_pack(S.SBN_CONV1X1, w1, 4, 4)
    with pytest.raises(S.SbnError) as ei:
        S.sbn_chain_create([S.sparse_item(a), S.stem_item(W.he_weights(9701, 8, 3, 3, 4))])
    assert ei.value.code == -2


def test_chain_replays_in_a_hip_graph():
    """Run calls neither allocate nor synchronise, so a caller may capture them in a HIP graph.
    The captured chain is replayed several times on new inputs, with eager work and
    synchronisations between the replays, and every replay must equal the eager result bit for bit."""
    chans, strides = [16, 32, 64, 32], [1, 2, 1]
    n, hw = 2, 12
    items, _ = build_stack(chans, hw, n, 50, 9300, strides)
    items.append(S.avgpool_item())
    chain = S.sbn_chain_create(items)
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, hw, hw)
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    ws_eager = torch.empty_like(ws)
    xd = torch.zeros((n, hw, hw, chans[0]), device="cuda")
    yd = torch.zeros((n, oh, ow, oc), device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        S.sbn_pointwise_chain(chain, xd, yd, n, hw, hw, ws, stream=side)          # warm-up outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        S.sbn_pointwise_chain(chain, xd, yd, n, hw, hw, ws, stream=side)
    for rep in range(4):
        x = torch.from_numpy(W.uniform_activation(9400 + rep, (n, hw, hw, chans[0]))).cuda()
        y_eager = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
        S.sbn_pointwise_chain(chain, x, y_eager, n, hw, hw, ws_eager)
        torch.cuda.synchronize()
        xd.copy_(x)
        yd.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(yd, y_eager), f"replay {rep} differs from the eager run"


@pytest.mark.parametrize("c,hw,stride,go", [(32, 14, 1, 16), (40, 9, 2, 16), (28, 7, 1, 16), (24, 11, 1, 8)])
def test_depthwise_layer_with_3_9_pattern_groups(c, hw, stride, go):
    """A 3:9 pattern-pruned depthwise layer (Section 3.2, DwConv3x3) behind a rearranged pointwise
    layer: the pattern groups are formed over the channels in the order the layer runs in, and the
    result must be the oracle's dense depthwise convolution of the select-masked weights."""
    n, c0 = 2, 16
    w1 = W.he_weights(9500, c, 1, 1, c0)
    perm = S.sbn_rearrange([dict(kind=S.SBN_CONV1X1, w=w1, go=4, gi=4)], [-1], 50, seed=9500, max_iters=200)[0]
    mask = S.sbn_prune_magnitude(R.permute_weights(w1, perm, None), S.SBN_CONV1X1, 4, 4, 50)
    p1 = S.sbn_pack(S.SBN_CONV1X1, w1, 4, 4, mask=mask, perm_out=perm, act=S.SBN_ACT_RELU)
    dw_w = W.normal_weights(9501, (c, 3, 3), 0.4)
    dw_b = W.small_bias(9502, c)
    n_groups = len(R.dw_pattern_groups(c, go))
    keep_dense = np.zeros(n_groups, np.uint8)
    keep_dense[-1] = 1 if n_groups > 1 else 0
    pattern = S.sbn_dw_pattern_select(dw_w[perm], go, keep_dense=keep_dense)       # on the order it runs in
    assert pattern.tolist() == R.dw_pattern_select(dw_w[perm], go, dense_groups=tuple(np.nonzero(keep_dense)[0])).tolist()
    chain = S.sbn_chain_create([S.sparse_item(p1),
                                S.dw_item(dw_w, dw_b, stride=stride, act=S.SBN_ACT_RELU, pattern=pattern, go=go)])
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, hw, hw)
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    x = W.uniform_activation(9503, (n, hw, hw, c0))
    mid = torch.empty((n, hw, hw, c), device="cuda")
    yd = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), yd, n, hw, hw, ws, layer_outputs=[mid, None])
    torch.cuda.synchronize()
    wm = R.dw_pattern_apply(dw_w[perm], pattern, go)
    assert (wm != 0).sum() < dw_w.size                                              # something was pruned
    y_ref, bound = R.dwconv3x3_nhwc(mid.cpu().numpy(), wm, dw_b[perm], stride=stride, act=R.ACT_RELU)
    assert_within_bound(yd.cpu().numpy(), y_ref, bound, "pattern-pruned depthwise layer")


FUSED_CASES = [
    # n, h, w, K, N, stride, pct, relu_dw, relu_pw, perm
    (2, 8, 8, 32, 64, 1, 30, True, True, False),        # one tile, one sub-chunk, one column tile
    (1, 13, 19, 64, 128, 1, 50, True, True, True),      # ragged tiles, two sub-chunks, two column tiles
    (2, 17, 9, 64, 128, 2, 50, True, False, True),      # stride 2, odd sizes
    (1, 21, 21, 128, 128, 1, 70, True, True, True),     # four sub-chunks
    (1, 12, 30, 128, 72, 2, 90, False, True, False),    # stride 2, no ReLU after the depthwise layer, ragged N
    (3, 1, 1, 32, 8, 1, 0, True, True, False),          # single pixels
    (1, 9, 9, 96, 24, 1, 100, True, True, False),       # everything pruned: act(bias) everywhere
]


@pytest.mark.parametrize("patterned", [False, True])
@pytest.mark.parametrize("n,h,w,K,N,stride,pct,relu_dw,relu_pw,perm", FUSED_CASES)
def test_depthwise_fused_into_small_pointwise_layer(n, h, w, K, N, stride, pct, relu_dw, relu_pw, perm, patterned):
    """A depthwise layer in front of a 1x1 layer with at most 128 channels on either side runs inside
    that layer's launch.  Checked against the oracle's two layers (the tolerance of the second carries
    the first's through the 1x1 weights: |err| <= 1e-4 (bound_pw + |W| bound_dw)), and against the
    same chain with the fusion switched off.  patterned: the depthwise layer is 3:9 pattern pruned in
    groups of 16 channels (one group left dense); the fused launch then skips the removed taps group
    by group, and the oracle convolves the select-masked weights densely."""
    seed = 9700 + K + N + stride + pct
    dw_w = W.normal_weights(seed, (K, 3, 3), 0.4)
    dw_b = W.small_bias(seed + 1, K) * 10
    pattern = None
    if patterned:
        keep_dense = np.zeros(K // 16, np.uint8)
        keep_dense[K // 32] = 1
        pattern = S.sbn_dw_pattern_select(dw_w, 16, keep_dense=keep_dense)
        assert len(set(pattern.tolist())) >= 2
    wt = W.he_weights(seed + 2, N, 1, 1, K)
    b = W.small_bias(seed + 3, N) * 10
    po = W.random_permutation(seed + 4, N) if perm else None
    mask = S.sbn_prune_magnitude(R.permute_weights(wt, po, None), S.SBN_CONV1X1, 4, 4, pct)
    act_pw = S.SBN_ACT_RELU if relu_pw else S.SBN_ACT_NONE
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, bias=b, perm_out=po, act=act_pw)
    chain = S.sbn_chain_create([S.dw_item(dw_w, dw_b, stride=stride, act=S.SBN_ACT_RELU if relu_dw else S.SBN_ACT_NONE,
                                          pattern=pattern, go=16),
                                S.sparse_item(p)])
    if patterned:
        dw_w = R.dw_pattern_apply(dw_w, pattern, 16)
    oh, ow, oc = S.sbn_chain_output_shape(chain, n, h, w)
    ws = torch.empty(S.sbn_chain_workspace(chain, n, h, w) // 4, device="cuda")
    x = W.uniform_activation(seed + 5, (n, h, w, K))
    xd = torch.from_numpy(x).cuda()
    y_fused = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    ws.fill_(float("nan"))
    S.sbn_chain_set_fusion(chain, 2)                       # whatever the size
    S.sbn_pointwise_chain(chain, xd, y_fused, n, h, w, ws)
    torch.cuda.synchronize()
    assert ws.isnan().all()                                # the depthwise output was never in memory
    S.sbn_chain_set_fusion(chain, False)
    y_plain = torch.full((n, oh, ow, oc), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, xd, y_plain, n, h, w, ws)
    torch.cuda.synchronize()
    assert not ws.isnan().all()

    mid, bound_dw = R.dwconv3x3_nhwc(x, dw_w, dw_b, stride=stride, act=R.ACT_RELU if relu_dw else R.ACT_NONE)
    ref, bound_pw = R.sparse_conv_reference(mid, wt, mask, 4, 4, bias=b, perm_out=po, act=act_pw)
    wm = np.abs(R.apply_mask(R.permute_weights(wt, po, None), mask, 4, 4).reshape(N, K).astype(np.float64))
    bound = bound_pw + (bound_dw.reshape(-1, K) @ wm.T).reshape(bound_pw.shape)
    assert_within_bound(y_fused.cpu().numpy(), ref, bound, f"fused {n,h,w,K,N,stride,pct}")
    assert_within_bound(y_plain.cpu().numpy(), ref, bound, f"separate {n,h,w,K,N,stride,pct}")


@pytest.mark.parametrize("tiles,K,N,stride,fused", [
    (64, 32, 64, 1, False), (65, 32, 64, 1, True),         # one tile of 8 x 8 pixels for every four compute units
    (65, 64, 128, 2, True),                                # more than 64 channels on one side only
    (96, 96, 72, 1, False), (97, 96, 72, 1, True),         # on both: six for every sixteen
])
def test_pairs_are_fused_from_enough_tiles_on(tiles, K, N, stride, fused):
    """Which pairs run as one launch on a device of 256 compute units, by the switch's three values: one that does never
    writes the depthwise output to the workspace.  The results against the oracle's two layers, as above."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 compute units")
    h, w = 8 * stride, 8 * stride * tiles
    dw_w, wt = W.normal_weights(9801, (K, 3, 3), 0.4), W.he_weights(9802, N, 1, 1, K)
    mask = S.sbn_prune_magnitude(wt, S.SBN_CONV1X1, 4, 4, 50)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, mask=mask, act=S.SBN_ACT_RELU)
    chain = S.sbn_chain_create([S.dw_item(dw_w, None, stride=stride, act=S.SBN_ACT_RELU), S.sparse_item(p)])
    oh, ow, oc = S.sbn_chain_output_shape(chain, 1, h, w)
    x = W.uniform_activation(9803, (1, h, w, K))
    xd = torch.from_numpy(x).cuda()
    mid, bound_dw = R.dwconv3x3_nhwc(x, dw_w, None, stride=stride, act=R.ACT_RELU)
    ref, bound_pw = R.sparse_conv_reference(mid, wt, mask, 4, 4, act=R.ACT_RELU)
    wm = np.abs(R.apply_mask(wt, mask, 4, 4).reshape(N, K).astype(np.float64))
    bound = bound_pw + (bound_dw.reshape(-1, K) @ wm.T).reshape(bound_pw.shape)
    ws = torch.empty(S.sbn_chain_workspace(chain, 1, h, w) // 4, device="cuda")
    for enable, expect in ((None, fused), (0, False), (2, True), (True, fused), (1, fused)):
        if enable is not None:
            S.sbn_chain_set_fusion(chain, enable)
        ws.fill_(float("nan"))
        y = torch.full((1, oh, ow, oc), float("nan"), device="cuda")
        S.sbn_pointwise_chain(chain, xd, y, 1, h, w, ws)
        torch.cuda.synchronize()
        assert bool(ws.isnan().all()) == expect, enable
        assert_within_bound(y.cpu().numpy(), ref, bound, f"enable={enable} {tiles,K,N,stride}")


def test_fusion_is_skipped_when_the_depthwise_output_is_requested():
    n, h, w, K, N = 1, 10, 10, 32, 32
    dw_w, dw_b = W.normal_weights(9801, (K, 3, 3), 0.4), W.small_bias(9802, K)
    wt = W.he_weights(9803, N, 1, 1, K)
    p = S.sbn_pack(S.SBN_CONV1X1, wt, 4, 4, act=S.SBN_ACT_RELU)
    chain = S.sbn_chain_create([S.dw_item(dw_w, dw_b, stride=1, act=S.SBN_ACT_RELU), S.sparse_item(p)])
    ws = torch.empty(S.sbn_chain_workspace(chain, n, h, w) // 4, device="cuda")
    x = W.uniform_activation(9804, (n, h, w, K))
    mid = torch.full((n, h, w, K), float("nan"), device="cuda")
    yd = torch.full((n, h, w, N), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, torch.from_numpy(x).cuda(), yd, n, h, w, ws, layer_outputs=[mid, None])
    torch.cuda.synchronize()
    ref_mid, bound_mid = R.dwconv3x3_nhwc(x, dw_w, dw_b, stride=1, act=R.ACT_RELU)
    assert_within_bound(mid.cpu().numpy(), ref_mid, bound_mid, "depthwise output copy")
    ref, bound = R.sparse_conv_reference(mid.cpu().numpy(), wt, None, 4, 4, act=R.ACT_RELU)
    assert_within_bound(yd.cpu().numpy(), ref, bound, "1x1 after the copied depthwise output")


def test_whole_mobilenet_batch64_full_size_sampled():
    """Config 4 at its full size and in the launch configuration the benchmark times (batch 64,
    224 x 224, the first three depthwise layers running inside their 1x1 layers): every launch's output
    is captured and, for sampled images, compared with the oracle fed with the GPU's previous output;
    a fused pair is compared with the oracle's two layers under the two-layer tolerance."""
    import bench
    chain, meta = bench.build_mobilenet_chain(S, W, 50, max_iters=100)
    n, hw, imgs = 64, 224, [0, 63]
    g = torch.Generator(device="cuda").manual_seed(4001)
    xd = torch.rand((n, hw, hw, 3), device="cuda", generator=g) * 2 - 1
    shapes, h, c = [], hw, 3
    for m in meta:
        if m["kind"] in ("dw", "stem"):
            h = (h - 1) // m["stride"] + 1
        if m["kind"] in ("pw", "stem"):
            c = m["w"].shape[0]
        if m["kind"] == "pool":
            h = 1
        shapes.append((n, h, h, c))
    fused = [i for i, m in enumerate(meta[:-1])
             if m["kind"] == "dw" and meta[i + 1]["kind"] == "pw" and meta[i + 1]["w"].shape[3] % 32 == 0
             and meta[i + 1]["w"].shape[3] <= 128 and meta[i + 1]["w"].shape[0] <= 128]
    assert len(fused) == 3
    taps = [None if i in fused else torch.full(s, float("nan"), device="cuda") for i, s in enumerate(shapes)]
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    yd = torch.empty(n, 1, 1, 1000, device="cuda")
    S.sbn_pointwise_chain(chain, xd, yd, n, hw, hw, ws, layer_outputs=taps)
    torch.cuda.synchronize()
    prev = xd[imgs].cpu().numpy()
    pending = None                      # a fused depthwise item waiting for its 1x1 layer
    for i, m in enumerate(meta):
        if i in fused:
            pending = m
            continue
        out = taps[i][imgs].cpu().numpy()
        if m["kind"] == "stem":
            ref, bound = R.conv_nhwc(prev, m["w"], m["b"], stride=m["stride"], pad=1, act=R.ACT_RELU)
        elif m["kind"] == "dw":
            w, b = m["w"], m["b"]
            if m["order"] is not None:
                w, b = w[m["order"]], b[m["order"]]
            ref, bound = R.dwconv3x3_nhwc(prev, w, b, stride=m["stride"], act=R.ACT_RELU)
        elif m["kind"] == "pool":
            ref, bound = R.avgpool_nhwc(prev)[:, None, None, :], None
        else:
            x_in, extra = prev, None
            if pending is not None:
                w, b = pending["w"], pending["b"]
                if pending["order"] is not None:
                    w, b = w[pending["order"]], b[pending["order"]]
                x_in, bound_dw = R.dwconv3x3_nhwc(prev, w, b, stride=pending["stride"], act=R.ACT_RELU)
                wp = R.apply_mask(R.permute_weights(m["w"], m["po"], m["pi"]), m["mask"], m["go"], 4)
                K = wp.shape[3]
                extra = bound_dw.reshape(-1, K) @ np.abs(wp.reshape(-1, K).astype(np.float64)).T
                pending = None
            ref, bound = R.sparse_conv_reference(x_in, m["w"], m["mask"], m["go"], 4, bias=m["b"], perm_out=m["po"],
                                                 perm_in=m["pi"], act=m["act"])
            if extra is not None:
                bound = bound + extra.reshape(bound.shape)
        if bound is None:
            np.testing.assert_allclose(out, ref, rtol=0, atol=1e-5)
        else:
            assert_within_bound(out, ref, bound, f"mobilenet batch 64 item {i} ({m['kind']})")
        prev = out
    assert torch.equal(taps[-1], yd)


def _teacher_forced(meta, outs, x):
    prev = x
    for i, m in enumerate(meta):
        ref, bound = oracle_item(m, prev)
        assert_within_bound(outs[i], ref, bound, f"multi-layer item {i} ({m['kind']})")
        prev = outs[i]


@pytest.mark.parametrize("n,hw", [(1, 14), (2, 9), (1, 7)])
def test_runs_of_small_items_go_out_as_one_launch(n, hw):
    """Few pixels (the paper's single-image setting): consecutive depthwise and 1x1 items run as
    phases of ONE launch with grid-wide barriers in between (opt-in).  Every item's output is captured
    (copies are phases of the same launch) and compared with the oracle fed with the GPU's previous
    output; the final output must also agree with the one-launch-per-item path, and the chain's
    barrier state must report no give-up."""
    chans, strides = [128, 256, 256, 512], [1, 2, 1]
    items, meta = build_stack(chans, hw, n, 50, 9900 + hw, strides)
    chain = S.sbn_chain_create(items)
    S.sbn_chain_set_multi_layer(chain, True)
    x = W.uniform_activation(9950 + hw, (n, hw, hw, chans[0]))
    xd = torch.from_numpy(x).cuda()
    shapes, h, c = [], hw, chans[0]
    for m in meta:
        if m["kind"] == "dw":
            h = (h - 1) // m["stride"] + 1
        else:
            c = m["w"].shape[0]
        shapes.append((n, h, h, c))
    ws = torch.empty(S.sbn_chain_workspace(chain, n, hw, hw) // 4, device="cuda")
    taps = [torch.full(s, float("nan"), device="cuda") for s in shapes]
    y_multi = torch.full(shapes[-1], float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, xd, y_multi, n, hw, hw, ws, layer_outputs=taps)
    torch.cuda.synchronize()
    S.sbn_chain_check(chain)
    outs = [t.cpu().numpy() for t in taps]
    assert np.array_equal(outs[-1], y_multi.cpu().numpy())
    _teacher_forced(meta, outs, x)
    # twice more without taps (the barrier words carry over from launch to launch), then item by item
    y_again = torch.full(shapes[-1], float("nan"), device="cuda")
    for _ in range(2):
        S.sbn_pointwise_chain(chain, xd, y_again, n, hw, hw, ws)
    torch.cuda.synchronize()
    S.sbn_chain_check(chain)
    assert torch.equal(y_again, y_multi)
    S.sbn_chain_set_multi_layer(chain, False)
    y_items = torch.full(shapes[-1], float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, xd, y_items, n, hw, hw, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(y_multi.cpu().numpy(), y_items.cpu().numpy(), rtol=2e-4, atol=2e-5)


def test_mobilenet_batch1_multi_layer_tail_matches_item_by_item():
    """Whole MobileNet-v1 on one image: the items from the fourth depthwise layer on (at most 784
    pixels each) leave as one launch; logits agree with the path of one launch per item."""
    import bench
    chain, meta = bench.build_mobilenet_chain(S, W, 50, max_iters=50)
    S.sbn_chain_set_multi_layer(chain, True)
    g = torch.Generator(device="cuda").manual_seed(4002)
    xd = torch.rand((1, 224, 224, 3), device="cuda", generator=g) * 2 - 1
    ws = torch.empty(S.sbn_chain_workspace(chain, 1, 224, 224) // 4, device="cuda")
    y_multi = torch.full((1, 1, 1, 1000), float("nan"), device="cuda")
    y_items = torch.full((1, 1, 1, 1000), float("nan"), device="cuda")
    S.sbn_pointwise_chain(chain, xd, y_multi, 1, 224, 224, ws)
    torch.cuda.synchronize()
    S.sbn_chain_check(chain)
    S.sbn_chain_set_multi_layer(chain, False)
    S.sbn_pointwise_chain(chain, xd, y_items, 1, 224, 224, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(y_multi).all()
    scale = float(y_items.abs().max())
    assert float((y_multi - y_items).abs().max()) <= 1e-4 * max(scale, 1.0)


def test_average_pool_of_more_images_than_one_launch_takes():
    """2^22 + 1 images of one pixel x 256 channels: four workgroups of 256 threads each, a little over the 2^32 work items
    that HIP takes per launch.  The pool of one pixel is that pixel, so every value is known."""
    n, c = (1 << 22) + 1, 256
    if torch.cuda.mem_get_info()[0] < 20 * (1 << 30):
        pytest.skip("needs 20 GiB of device memory")
    w = np.zeros((c, 3, 3), np.float32)
    w[:, 1, 1] = 1.0                                       # (a depthwise layer that copies: a chain cannot start with the pool)
    chain = S.sbn_chain_create([S.dw_item(w, None, act=S.SBN_ACT_NONE), S.avgpool_item()])
    x = torch.rand((n, 1, 1, c), device="cuda", generator=torch.Generator(device="cuda").manual_seed(9810))
    y = torch.full((n, 1, 1, c), float("nan"), device="cuda")
    ws = torch.empty(S.sbn_chain_workspace(chain, n, 1, 1) // 4, device="cuda")
    S.sbn_pointwise_chain(chain, x, y, n, 1, 1, ws)
    torch.cuda.synchronize()
    assert torch.equal(x, y)
