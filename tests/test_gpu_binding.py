"""The binding's native path against its interpreted one (which an explicit
stream selects): the same bytes for every form both take, the same errors for
what neither does."""
import numpy as np
import pytest
import torch

import paper_2608_12932_amd as w
from paper_2608_12932_amd import inputs as I
from helpers import bf16_dev, dev, pack, scales_dev

pytestmark = pytest.mark.gpu


class Record:
    """The native module with the results of its calls (None: declined)."""

    def __init__(self, monkeypatch):
        self.native, self.got = w._load_fast(), []
        monkeypatch.setattr(w, "_fast", self)

    def __getattr__(self, name):
        def call(*args):
            self.got.append(getattr(self.native, name)(*args))
            return self.got[-1]
        return call

    def last(self, f, *args, **kw):
        """f's result and what the last native call of it gave."""
        self.got.clear()
        r = f(*args, **kw)
        return r, self.got[-1]


def same(a, b):
    assert a.dtype == b.dtype and a.shape == b.shape
    assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("group", [False, True])
@pytest.mark.parametrize("M", [0, 3, 70])
def test_linear_paths_agree(M, group, swiglu):
    K, N = 256, 96
    x = bf16_dev(I.activations(M, K, 900 + M))
    W, s = I.weights(N, K, 901, group=group)
    wp, sd = pack(W), scales_dev(s)
    q, sx = w.w4a8_quantize_act(x)
    f = w.w4a8_linear_swiglu if swiglu else w.w4a8_linear
    mode = w.SCALE_GROUP_F16 if group else w.SCALE_CHANNEL_F32
    cur = torch.cuda.current_stream()
    for kind in (w.OUT_BF16, w.OUT_F32) + (() if swiglu else (w.OUT_I32_ACC,)):
        for xin, xs in ((x, None), (q, sx)):
            ref = f(xin, wp, sd, N, x_scale=xs, scale_mode=mode, out_kind=kind, stream=cur)
            ws = w.Workspace()
            tensor = torch.zeros(1 << 20, dtype=torch.uint8, device=dev())
            out = torch.empty_like(ref)
            for wk in (None, ws, ws, tensor):
                same(f(xin, wp, sd, N, x_scale=xs, scale_mode=mode, out_kind=kind, workspace=wk), ref)
                assert f(xin, wp, sd, N, x_scale=xs, scale_mode=mode, out_kind=kind, out=out, workspace=wk) is out
                same(out, ref)


def test_workspace_grows_and_changes_stream():
    K, N = 512, 64
    W, s = I.weights(N, K, 902)
    wp, sd, ws = pack(W), scales_dev(s), w.Workspace()
    side = torch.cuda.Stream()
    for M in (2, 200, 5):  # grows at the second
        x = bf16_dev(I.activations(M, K, 903))
        ref = w.w4a8_linear(x, wp, sd, N, stream=torch.cuda.current_stream())
        same(w.w4a8_linear(x, wp, sd, N, workspace=ws), ref)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):  # the buffer of the other stream, recorded for this one
            y = w.w4a8_linear(x, wp, sd, N, workspace=ws)
        side.synchronize()
        same(y, ref)
    assert ws.buf.numel() >= w.w4a8_linear_workspace_bytes(200, N, K)


def test_quantize_norm_and_flow_agree():
    cur = torch.cuda.current_stream()
    for M, K in ((1, 128), (5, 640), (70, 4096)):
        x = bf16_dev(I.activations(M, K, 904))
        g = torch.linspace(0.5, 1.5, K, device=dev()).to(torch.bfloat16)
        for a, b in ((w.w4a8_quantize_act(x), w.w4a8_quantize_act(x, stream=cur)),
                     (w.w4a8_rmsnorm_quantize_act(x, g, 1e-6), w.w4a8_rmsnorm_quantize_act(x, g, 1e-6, stream=cur))):
            same(a[0], b[0])
            same(a[1], b[1])
    for v_new, stats in ((True, True), (True, False), (False, False)):
        got = []
        for stream in (None, cur):
            x = torch.from_numpy(I.flow_state(3, 40, 905)).to(dev())
            v = bf16_dev(I.flow_velocity(3, 40, 906)) if v_new else None
            c = bf16_dev(I.flow_velocity(3, 40, 907))
            st = w.w4a8_flow_step(x, v, c, 0.125, stats=stats, repeat=2, stream=stream)
            got.append((x, c, st))
        same(got[0][0], got[1][0])
        same(got[0][1], got[1][1])
        assert (got[0][2] is None) == (not stats)
        if stats:
            same(got[0][2], got[1][2])


def test_refused_calls():
    K, N = 256, 64
    x = bf16_dev(I.activations(4, K, 908))
    W, s = I.weights(N, K, 909)
    wp, sd = pack(W), scales_dev(s)
    with pytest.raises(TypeError):
        w.w4a8_linear(x.float(), wp, sd, N)
    with pytest.raises(TypeError):
        w.w4a8_linear(x, wp, sd.half(), N)
    with pytest.raises(TypeError):
        w.w4a8_linear(x, wp.cpu(), sd, N)
    with pytest.raises(ValueError):
        w.w4a8_linear(x[:, ::2], wp, sd, N)
    with pytest.raises(ValueError):
        w.w4a8_linear(w.w4a8_quantize_act(x)[0], wp, sd, N)  # codes without scales
    with pytest.raises(ValueError):
        w.w4a8_linear(x, wp, sd, N, out=torch.empty(4, N + 1, dtype=torch.bfloat16, device=dev()))
    with pytest.raises(w.W4A8Error):
        w.w4a8_linear(x, wp, sd, 24)  # not a multiple of 16
    with pytest.raises(w.W4A8Error):
        w.w4a8_linear(x, wp, sd, N, workspace=torch.zeros(16, dtype=torch.uint8, device=dev()))
    with pytest.raises(w.W4A8Error):
        w.w4a8_rmsnorm_quantize_act(x, torch.ones(K, dtype=torch.bfloat16, device=dev()), -1.0)
    with pytest.raises(ValueError):
        w.w4a8_rmsnorm_quantize_act(x, torch.ones(K + 8, dtype=torch.bfloat16, device=dev()), 1e-6)
    with pytest.raises(ValueError):
        w.w4a8_flow_step(torch.zeros(2, 8, device=dev()), None, torch.zeros(2, 4, dtype=torch.bfloat16, device=dev()), 0.1)


def test_native_path_is_taken(monkeypatch):
    K, N, M = 512, 64, 20
    rec = Record(monkeypatch)
    x = bf16_dev(I.activations(M, K, 910))
    (q, sx), got = rec.last(w.w4a8_quantize_act, x)
    assert type(got) is tuple and got[0] is q
    r, got = rec.last(w.w4a8_rmsnorm_quantize_act, x, torch.ones(K, dtype=torch.bfloat16, device=dev()), 1e-6)
    assert r is got
    for f, group in ((w.w4a8_linear, False), (w.w4a8_linear, True), (w.w4a8_linear_swiglu, True)):
        W, s = I.weights(N, K, 911, group=group)
        wp, sd = pack(W), scales_dev(s)
        kw = dict(scale_mode=w.SCALE_GROUP_F16 if group else w.SCALE_CHANNEL_F32)
        ws = w.Workspace()
        need = w.w4a8_linear_workspace_bytes(M, N, K, int(group))
        assert need > 0 and w.w4a8_linear_workspace_bytes(M, N, K, int(group), w.IN_I8) == 0
        for wk in (ws, ws, None, torch.zeros(need, dtype=torch.uint8, device=dev())):
            y, got = rec.last(f, x, wp, sd, N, workspace=wk, **kw)
            assert y is got
        y, got = rec.last(f, q, wp, sd, N, x_scale=sx, **kw)
        assert y is got
        out = torch.empty_like(y)
        y, got = rec.last(f, x, wp, sd, N, workspace=ws, out=out, **kw)
        assert y is out and got is out
    f = lambda v, stats: rec.last(w.w4a8_flow_step, torch.zeros(2, 8, device=dev()), v,
                                  torch.zeros(2, 8, dtype=torch.bfloat16, device=dev()), 0.1, stats=stats)
    v = torch.ones(2, 8, dtype=torch.bfloat16, device=dev())
    st, got = f(v, True)
    assert st is got and st.shape == (2, 4)
    assert f(v, False) == (None, True) and f(None, False) == (None, True)


def test_native_path_declines(monkeypatch):
    import copy
    K, N, M = 512, 64, 20
    rec = Record(monkeypatch)
    x = bf16_dev(I.activations(M, K, 912))
    W, s = I.weights(N, K, 913)
    wp, sd, ws = pack(W), scales_dev(s), w.Workspace()
    ref = w.w4a8_linear(x, wp, sd, N, workspace=ws)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):  # a Workspace of another stream, a copy of one
        y, got = rec.last(w.w4a8_linear, x, wp, sd, N, workspace=ws)
        twin = copy.deepcopy(ws)
    assert got is None
    side.synchronize()
    same(y, ref)
    y, got = rec.last(w.w4a8_linear, x, wp, sd, N, workspace=twin)
    assert got is None
    same(y, ref)

    class Sub(torch.Tensor):
        pass

    y, got = rec.last(w.w4a8_linear, x.as_subclass(Sub), wp, sd, N)
    assert got is None
    same(y.as_subclass(torch.Tensor), ref)


def test_refused_calls_leave_the_workspace_alone():
    K, N, M = 512, 64, 20
    x = bf16_dev(I.activations(M, K, 912))
    W, s = I.weights(N, K, 913)
    wp, sd = pack(W), scales_dev(s)
    ws = w.Workspace()
    for bad in (dict(x=x.float()), dict(x=x[:, ::2]), dict(wp=wp.cpu()), dict(sd=sd.half()),
                dict(out=torch.empty(M, N + 1, dtype=torch.bfloat16, device=dev()))):
        a = dict(x=x, wp=wp, sd=sd, out=None) | bad
        with pytest.raises((TypeError, ValueError)):
            w.w4a8_linear(a["x"], a["wp"], a["sd"], N, out=a["out"], workspace=ws)
        assert ws.buf.numel() == 0, list(bad)
