"""The calls whose speed matters, as a user's program makes them.

Four kinds of work, all through the public entry points:

  pw      one group-sparse 1x1 layer                      sbn_conv1x1_sparse
  pw13    the 13 pointwise layers of MobileNet-v1, one
          call each on its own resident input             sbn_conv1x1_sparse
  net     MobileNet-v1 forward, stem to logits, as one
          chain                                           sbn_pointwise_chain[_static]
  c3      a list of kernel-sparse 3x3 layers, one call
          each                                            sbn_conv3x3_sparse

Everything is fp32, the only data type of the library.  Weights are He-normal,
pruned by block magnitude, biases small, activations what the layers meet in a
network: U(-1, 1) images, non-negative half-zero activations (the output of a
ReLU) in front of single layers.  Layers are packed once and kept, outputs and
workspaces belong to the caller and are reused.
"""
import math

import numpy as np
import torch

import paper_2310_19509_amd as S

# (input extent as a divisor of the image's, channels in, channels out) of the 13 pointwise layers
PW13 = ((2, 32, 64), (4, 64, 128), (4, 128, 128), (8, 128, 256), (8, 256, 256), (16, 256, 512), (16, 512, 512),
        (16, 512, 512), (16, 512, 512), (16, 512, 512), (16, 512, 512), (32, 512, 1024), (32, 1024, 1024))
DW_STRIDE = (1, 2, 1, 2, 1, 2, 1, 1, 1, 1, 1, 2, 1)

# ResNet-50-shaped 3x3 layers: (extent, channels in, channels out, stride)
R50_3X3 = ((56, 64, 64, 1), (28, 128, 128, 1), (14, 256, 256, 1), (7, 512, 512, 1))


def _pw(name, n, h, w, c_in, c_out, pct, go=4, gi=4, relu=True, bias=True):
    return dict(name=name, kind="pw", n=n, h=h, w=w, c_in=c_in, c_out=c_out, pct=pct, go=go, gi=gi, relu=relu, bias=bias)


def _pw13(name, n, res, pct, go=4, gi=4):
    return dict(name=name, kind="pw13", n=n, res=res, pct=pct, go=go, gi=gi)


def _net(name, n, res, pct, go=4, pattern=False, static=False):
    return dict(name=name, kind="net", n=n, res=res, pct=pct, go=go, pattern=pattern, static=static)


def _c3(name, n, layers, pct, go=4, gi=4):
    # a case holds plain values: the layers travel as text, "extent:c_in:c_out:stride ..."
    return dict(name=name, kind="c3", n=n, layers=" ".join(":".join(str(v) for v in l) for l in layers), pct=pct, go=go, gi=gi)


def listed():
    return [
        # the smallest call: one layer on one 14 x 14 feature map
        _pw("layer_14x14_64_128", 1, 14, 14, 64, 128, 50, relu=False, bias=False),
        # a layer whose sizes fit no tile: blocks of 8 x 2, an odd feature map, odd channel counts
        _pw("layer_odd", 3, 37, 29, 90, 200, 40, go=8, gi=2),
        # one large layer, a server's batch
        _pw("layer_512_b512", 512, 14, 14, 512, 512, 50),
        # the pointwise stack on one image: single-image latency, layer by layer
        _pw13("pw13_b1", 1, 224, 30),
        # the pointwise stack at the batch of a throughput run: moderate, high and extreme sparsity
        _pw13("pw13_b64_30", 64, 224, 30),
        _pw13("pw13_b64_70", 64, 224, 70),
        # wider blocks, a medium batch
        _pw13("pw13_b16_90_go8", 16, 224, 90, go=8),
        # a whole network on one image (the latency setting), with the library's own workspace
        _net("net_b1", 1, 224, 50, static=True),
        # the same at throughput batch
        _net("net_b64", 64, 224, 50),
        # a smaller input, pattern-pruned depthwise layers, a batch that divides nothing
        _net("net_b11_160_pattern", 11, 160, 30, pattern=True),
        # kernel-sparse 3x3 layers of a ResNet-50 at batch 32
        _c3("c3_b32_70", 32, R50_3X3, 70),
        # few images, ragged extents, a strided layer among them, lower sparsity
        _c3("c3_b3_ragged", 3, ((57, 64, 64, 1), (45, 64, 128, 2), (23, 128, 128, 1), (9, 256, 200, 1)), 50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 1e14)


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("pw", "pw", "pw", "pw13", "pw13", "net", "net", "c3", "c3"))
        pct = rng.choice((30, 50, 70, 90, rng.randint(0, 95), rng.randint(0, 95)))
        go = rng.choice((4, 4, 8))
        gi = rng.choice((4, 4, 4, 1, 2, 8)) if go == 4 else rng.choice((4, 2, 8))
        if kind == "pw":
            unit = max(gi, 2) if rng.random() < 0.3 else 8 * max(gi, 4)
            c_in = max(1, _log_int(rng, 16, 1024) // unit) * unit
            c_out = max(1, _log_int(rng, 16, 1024) // go) * go
            h, w = _log_int(rng, 7, 112), _log_int(rng, 7, 112)
            case = _pw("", _log_int(rng, 1, 512), h, w, c_in, c_out, pct, go, gi, rng.random() < 0.8, rng.random() < 0.8)
        elif kind == "pw13":
            case = _pw13("", _log_int(rng, 1, 64), rng.choice((128, 160, 192, 224, 256, rng.randint(96, 256))), pct, go, 4)
        elif kind == "net":
            n = _log_int(rng, 1, 64)
            case = _net("", n, rng.choice((128, 160, 192, 224, 256, rng.randint(96, 256))), pct, go, rng.random() < 0.3,
                        n == 1 and rng.random() < 0.5)
        else:
            layers = []
            for _ in range(rng.randint(1, 4)):
                unit = max(gi, 4) * rng.choice((1, 4, 8))
                c_in = max(1, _log_int(rng, 16, 512) // unit) * unit
                layers.append((_log_int(rng, 7, 112), c_in, max(1, _log_int(rng, 16, 512) // go) * go, rng.choice((1, 1, 1, 2))))
            case = _c3("", _log_int(rng, 1, 32), layers, pct, go, gi)
        del case["name"]
        if _cost(case) <= limit:
            return case


# ---- shapes -----------------------------------------------------------------------------------

def _half(v, times):
    for _ in range(times):
        v = (v - 1) // 2 + 1
    return v


def _pw13_shapes(case):
    """(pixels, c_in, c_out) of the 13 layers."""
    return [(case["n"] * _half(case["res"], d.bit_length() - 1) ** 2, ci, co) for d, ci, co in PW13]


def _c3_layers(case):
    return [tuple(int(v) for v in l.split(":")) for l in case["layers"].split()]


def _kept(case, c_in, c_out):
    """Weights (per tap) that a layer keeps."""
    blocks = (c_out // case["go"]) * (c_in // case.get("gi", 4))
    return (blocks - blocks * case["pct"] // 100) * case["go"] * case.get("gi", 4)


def work(case):
    nbytes = flops = 0
    if case["kind"] in ("pw", "pw13"):
        shapes = _pw13_shapes(case) if case["kind"] == "pw13" else [(case["n"] * case["h"] * case["w"], case["c_in"], case["c_out"])]
        for m, ci, co in shapes:
            nbytes += 4 * (m * (ci + co) + _kept(case, ci, co))
            flops += 2 * m * _kept(case, ci, co)
    elif case["kind"] == "net":
        n, res = case["n"], case["res"]
        m = n * _half(res, 1) ** 2
        nbytes += 4 * (n * res * res * 3 + n * 1000 + 27 * 32 + 1024 * 1000)
        flops += 2 * m * 27 * 32 + 2 * n * 1024 * 1000
        for (m, ci, co) in _pw13_shapes(case):
            nbytes += 4 * (_kept(case, ci, co) + 9 * ci)
            flops += 2 * m * (_kept(case, ci, co) + (6 if case["pattern"] else 9) * ci)
    else:
        for hw, ci, co, stride in _c3_layers(case):
            o = case["n"] * ((hw - 1) // stride + 1) ** 2
            nbytes += 4 * (case["n"] * hw * hw * ci + o * co + 9 * _kept(case, ci, co))
            flops += 2 * o * 9 * _kept(case, ci, co)
    return dict(bytes=nbytes, flops=flops)


# ---- inputs -----------------------------------------------------------------------------------

def _he(rng, c_out, k, c_in):
    return (rng.standard_normal((c_out, k, k, c_in), dtype=np.float32) * np.float32(math.sqrt(2.0 / (k * k * c_in))))


def _bias(rng, n):
    return rng.standard_normal(n, dtype=np.float32) * np.float32(0.01)


def _pack(case, kind, rng, c_in, c_out, stride=1, relu=True, bias=True, perm_out=None, perm_in=None):
    w = _he(rng, c_out, 3 if kind == S.SBN_CONV3X3 else 1, c_in)
    wp = w if perm_out is None else w[perm_out]
    wp = wp if perm_in is None else wp[..., perm_in]
    go, gi = case["go"], case.get("gi", 4)
    mask = S.sbn_prune_magnitude(np.ascontiguousarray(wp), kind, go, gi, case["pct"])
    return S.sbn_pack(kind, w, go, gi, mask=mask, bias=_bias(rng, c_out) if bias else None, perm_out=perm_out,
                      perm_in=perm_in, stride=stride, act=S.SBN_ACT_RELU if relu else S.SBN_ACT_NONE)


def _activations(gen, *shape):
    """What a layer reads inside a network: the output of a ReLU."""
    return torch.randn(shape, device="cuda", generator=gen).clamp_(min=0.0)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    calls, chain = [], None
    if case["kind"] == "pw":
        n, h, w = case["n"], case["h"], case["w"]
        p = _pack(case, S.SBN_CONV1X1, rng, case["c_in"], case["c_out"], relu=case["relu"], bias=case["bias"])
        calls.append((S.sbn_conv1x1_sparse, p, _activations(gen, n, h, w, case["c_in"]),
                      torch.empty((n, h, w, case["c_out"]), device="cuda"), n, h, w))
    elif case["kind"] == "pw13":
        for m, ci, co in _pw13_shapes(case):
            p = _pack(case, S.SBN_CONV1X1, rng, ci, co)
            hw = math.isqrt(m // case["n"])
            calls.append((S.sbn_conv1x1_sparse, p, _activations(gen, case["n"], hw, hw, ci),
                          torch.empty((case["n"], hw, hw, co), device="cuda"), case["n"], hw, hw))
    elif case["kind"] == "c3":
        n = case["n"]
        for hw, ci, co, stride in _c3_layers(case):
            p = _pack(case, S.SBN_CONV3X3, rng, ci, co, stride=stride)
            o = (hw - 1) // stride + 1
            calls.append((S.sbn_conv3x3_sparse, p, _activations(gen, n, hw, hw, ci),
                          torch.empty((n, o, o, co), device="cuda"), n, hw, hw))
    else:
        # Channel orders as an earlier search for a rearrangement left them: a layer's filter order is
        # the next layer's channel order, the depthwise layers in between follow it.
        items = [S.stem_item(_he(rng, 32, 3, 3), _bias(rng, 32))]
        pin = None
        for (_, ci, co), stride in zip(PW13, DW_STRIDE):
            dw = rng.standard_normal((ci, 3, 3), dtype=np.float32) * np.float32(math.sqrt(2.0 / 9.0))
            pat = S.sbn_dw_pattern_select(dw if pin is None else np.ascontiguousarray(dw[pin])) if case["pattern"] else None
            items.append(S.dw_item(dw, _bias(rng, ci), stride=stride, pattern=pat))
            po = rng.permutation(co).astype(np.int32)
            items.append(S.sparse_item(_pack(case, S.SBN_CONV1X1, rng, ci, co, perm_out=po, perm_in=pin)))
            pin = po
        items.append(S.avgpool_item())
        items.append(S.sparse_item(S.sbn_pack(S.SBN_CONV1X1, _he(rng, 1000, 1, 1024), 4, 4, bias=_bias(rng, 1000), perm_in=pin)))
        chain = S.sbn_chain_create(items)
        n, res = case["n"], case["res"]
        ws = None if case["static"] else torch.empty(S.sbn_chain_workspace(chain, n, res, res) // 4, device="cuda")
        x = torch.rand((n, res, res, 3), device="cuda", generator=gen) * 2 - 1
        calls.append((x, torch.empty((n, 1, 1, 1000), device="cuda"), n, res, res, ws))
    return dict(calls=calls, chain=chain)


def run(state):
    """One pass; returns every output whole."""
    if state["chain"] is not None:
        x, y, n, h, w, ws = state["calls"][0]
        if ws is None:
            S.sbn_pointwise_chain_static(state["chain"], x, y, n, h, w)
        else:
            S.sbn_pointwise_chain(state["chain"], x, y, n, h, w, ws)
        return y
    for fn, p, x, y, n, h, w in state["calls"]:
        fn(p, x, y, n, h, w)
    return [c[3] for c in state["calls"]]


def tolerance(case):
    """fp32 products and sums, nothing shorter.  Against the same layers in 64 bits (listed cases and
    ten drawn ones on an MI355X) the largest relative 2-norm error of a layer was 2.5e-7, of a whole
    network 1.8e-7, and the largest single difference 2.8e-6 of the result's root mean square: four
    times that.  (For scale: rounding one operand to bf16 would show 1e-3, to 16 bits 4e-6.)"""
    return {"rel": 1e-6, "max": 1e-5}
