"""The compiled marshalling of the run calls: ordinary calls go through it, everything else keeps the behaviour of the Python
code (checks, messages, streams)."""

import warnings

import numpy as np
import pytest
import torch

import paper_2310_19509_amd as S
from paper_2310_19509_amd import _lib, api
import workloads as W


def layer(kind=S.SBN_CONV1X1, K=64, N=32, device=-1, **kw):
    k = 3 if kind == S.SBN_CONV3X3 else 1
    return S.sbn_pack(kind, W.he_weights(8100, N, k, k, K), 4, 4, device=device, **kw)


def test_other_calls_are_answered_with_none_on_the_host():
    m = _lib.marshal()
    p = layer()
    x, y = torch.zeros(1, 2, 2, 64), torch.zeros(1, 2, 2, 32)
    for args in [(0, p, x, y, 1, 2, 2, None), (0, None, x, y, 1, 2, 2, None), (0, p, 16, 32, 1, 2, 2, None), (0, p, x, y, 1, 2, 2, 0),
                 (0, p, x, y, 0, 2, 2, None), (0, p, x, y, np.int64(1), 2, 2, None), (0, p, x, y, 1 << 40, 2, 2, None), (2, p, x, y, 1, 2, 2, None)]:
        assert m.layer(*args) is None
    assert m.chain(None, x, y, 1, 2, 2, None, None) is None
    with pytest.raises(AssertionError):                      # a host tensor: refused as before
        S.sbn_conv1x1_sparse(p, x, y, 1, 2, 2)
    with pytest.raises(ValueError):
        S.sbn_conv1x1_sparse(p, x[:, :1], y, 1, 2, 2)
    with pytest.raises(S.SbnError):                          # packed without a device copy
        S.sbn_conv1x1_sparse(p, 256, 512, 1, 2, 2, 0)


@pytest.fixture
def elsewhere(tmp_path, monkeypatch):
    """The module not loaded yet, its folder an empty one."""
    _lib.lib()
    monkeypatch.setattr(_lib, "_PKG", str(tmp_path))
    monkeypatch.setattr(_lib, "_marshal", None)
    monkeypatch.setattr(api, "_native", None)
    return tmp_path


def compiler(path, body):
    path.write_text("#!/bin/sh\n" + body)
    path.chmod(0o755)
    return str(path)


def test_calls_without_the_module(elsewhere, monkeypatch):
    """No compiler: one warning, and the Python code answers every call; no half-written file is left to be loaded."""
    monkeypatch.setenv("CXX", compiler(elsewhere / "cxx", 'for out; do :; done; printf half > "$out"; exit 1'))
    p = layer()
    with pytest.warns(UserWarning, match="marshalled in Python"):
        with pytest.raises(S.SbnError):                      # packed without a device copy: the library's own answer
            S.sbn_conv1x1_sparse(p, 256, 512, 1, 2, 2, 0)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        with pytest.raises(S.SbnError):
            S.sbn_conv1x1_sparse(p, 256, 512, 1, 2, 2, 0)
        with pytest.raises(AssertionError):
            S.sbn_conv1x1_sparse(p, torch.zeros(1, 2, 2, 64), torch.zeros(1, 2, 2, 32), 1, 2, 2)
    assert [f.name for f in elsewhere.iterdir()] == ["cxx"]


def test_a_file_that_does_not_load(elsewhere, monkeypatch):
    open(_lib.marshal_path(), "w").write("not a shared object")
    with pytest.warns(UserWarning, match="marshalled in Python"):
        with pytest.raises(S.SbnError):
            S.sbn_conv1x1_sparse(layer(), 256, 512, 1, 2, 2, 0)


def test_another_torch_has_a_file_of_its_own(elsewhere, monkeypatch):
    path = _lib.marshal_path()
    monkeypatch.setattr(torch, "__version__", "0.0")
    assert _lib.marshal_path() != path


def test_the_file_appears_when_it_is_complete(elsewhere, monkeypatch):
    """While the compiler still writes, nothing lies under the name that a second process would load."""
    path = _lib.marshal_path()
    monkeypatch.setenv("CXX", compiler(elsewhere / "cxx", f'for out; do :; done; printf half > "$out"; [ -e "{path}" ] && exit 1; printf whole > "$out"'))
    assert _lib.build_marshal() == path
    assert open(path).read() == "whole"


@pytest.mark.gpu
def test_the_python_code_gives_the_same_results(elsewhere, monkeypatch):
    monkeypatch.setenv("CXX", "false")
    x, y, ref = torch.randn(2, 5, 7, 64, device="cuda"), torch.zeros(2, 5, 7, 32, device="cuda"), torch.zeros(2, 5, 7, 32, device="cuda")
    p = layer(device=0)
    with pytest.warns(UserWarning, match="marshalled in Python"):
        S.sbn_conv1x1_sparse(p, x, ref, 2, 5, 7)
    monkeypatch.undo()
    S.sbn_conv1x1_sparse(p, x, y, 2, 5, 7)
    assert torch.equal(y, ref) and not torch.equal(y, torch.zeros_like(y))


@pytest.mark.gpu
@pytest.mark.parametrize("kind,stride", [(S.SBN_CONV1X1, 1), (S.SBN_CONV3X3, 1), (S.SBN_CONV3X3, 2)])
def test_layers(kind, stride):
    m, fn = _lib.marshal(), S.sbn_conv1x1_sparse if kind == S.SBN_CONV1X1 else S.sbn_conv3x3_sparse
    p = layer(kind, device=0, stride=stride)
    x = torch.randn(2, 5, 7, 64, device="cuda")
    o = (2, (5 - 1) // stride + 1, (7 - 1) // stride + 1, 32)
    ref, y = torch.zeros(o, device="cuda"), torch.zeros(o, device="cuda")
    fn(p, x, ref, 2, 5, 7, stream=torch.cuda.current_stream())          # the Python code's way
    k = int(kind == S.SBN_CONV3X3)
    assert m.layer(k, p, x, y, 2, 5, 7, None) == 0
    assert torch.equal(ref, y)
    # the current stream is the one the launch goes to: a fill before and a copy after it, on a stream of its own
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        big = torch.randn(4096, 4096, device="cuda")
        for _ in range(8):
            big = big @ big * 1e-4
        y.fill_(7.0)
        fn(p, x, y, 2, 5, 7)
        got = y.clone()
    side.synchronize()
    assert torch.equal(ref, got)
    # refused and accepted as by the Python code
    class Sub(torch.Tensor):
        pass
    assert m.layer(k, p, x.as_subclass(Sub), y, 2, 5, 7, None) is None
    assert m.layer(k, p, x.transpose(1, 2), y, 2, 5, 7, None) is None
    assert m.layer(k, p, x.double(), y, 2, 5, 7, None) is None
    with pytest.raises(ValueError):
        fn(p, x[:1], y, 2, 5, 7)
    with pytest.raises(ValueError):
        fn(p, x, y[:1], 2, 5, 7)
    with pytest.raises(AssertionError):
        fn(p, x.transpose(1, 2), y, 2, 5, 7)
    flat = torch.zeros(2 * 5 * 7 * 64 + 1, device="cuda")
    with pytest.raises(S.SbnError):                          # not 16-byte aligned: the library's own check
        fn(p, flat[1:], y, 2, 5, 7)
    with pytest.raises(S.SbnError):
        (S.sbn_conv3x3_sparse if k == 0 else S.sbn_conv1x1_sparse)(p, x, torch.zeros(2, 5, 7, 32, device="cuda"), 2, 5, 7)
    S.sbn_free(p)
    with pytest.raises(S.SbnError):
        fn(p, x, y, 2, 5, 7)


@pytest.mark.gpu
def test_chains():
    m = _lib.marshal()
    items = [S.dw_item(W.he_weights(8101, 64, 3, 3, 1)[..., 0]), S.sparse_item(layer(device=0)), S.avgpool_item()]
    c = S.sbn_chain_create(items)
    x = torch.randn(2, 6, 6, 64, device="cuda")
    ws = torch.empty(S.sbn_chain_workspace(c, 2, 6, 6) // 4, device="cuda")
    ref, y = torch.zeros(2, 1, 1, 32, device="cuda"), torch.zeros(2, 1, 1, 32, device="cuda")
    S.sbn_pointwise_chain(c, x, ref, 2, 6, 6, ws, stream=torch.cuda.current_stream())
    assert m.chain(c, x, y, 2, 6, 6, ws, None) == 0 and torch.equal(ref, y)
    y.zero_()
    assert m.chain(c, x, y, 2, 6, 6, None, None) == 0 and torch.equal(ref, y)
    with pytest.raises(ValueError):
        S.sbn_pointwise_chain(c, x[:1], y, 2, 6, 6, ws)
    with pytest.raises(ValueError):
        S.sbn_pointwise_chain_static(c, x, y[:1], 2, 6, 6)
    with pytest.raises(S.SbnError):
        S.sbn_pointwise_chain(c, x, y, 2, 6, 6, ws[:8])
    assert m.layer(0, c, x, y, 2, 6, 6, None) is None        # a chain is no layer
