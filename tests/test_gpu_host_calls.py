"""The compiled host part of the calls against the binding's own Python code: the same outputs for every
layout and every choice of buffers passed in, the same errors for what does not fit."""
import ctypes

import pytest
import torch

from paper_2509_24006_amd import binding as sla

pytestmark = pytest.mark.gpu


class _HandsEverythingBack:
    build_mask = forward = mask_forward = backward = staticmethod(lambda *a: None)


def _tensors(layout, dtype, B=2, H=3, N=333, d=64):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    new = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dtype)
    W = new(d, d) * 0.02
    if layout == sla.SLA_STRIDED:
        x = [new(B, N, 3, H, d)[:, :, i].transpose(1, 2) for i in range(3)] + [new(B, N, 3, H, d)[:, :, 0].transpose(1, 2)]
        return sla.make_params(B, H, N, d, 0.2, 0.2, dtype, layout=layout, strides=x[0].stride()[:3]), x, W
    shape = (B, N, H, d) if layout == sla.SLA_BNHD else (B, H, N, d)
    return sla.make_params(B, H, N, d, 0.2, 0.2, dtype, layout=layout), [new(*shape) for _ in range(4)], W


def _all(p, x, W, given):
    z, dev = sla.sla_sizes(p), "cuda"
    u8 = lambda n: torch.empty(n + 64, dtype=torch.uint8, device=dev)
    like = lambda t: torch.empty_strided(t.shape, t.stride(), dtype=t.dtype, device=dev)
    kw = [{}, {}, {}]
    if given:
        kw = [dict(workspace=u8(z.ws_mask_bytes), Mc=torch.empty((p.B, p.H, z.Tq, z.T), dtype=torch.int8, device=dev),
                   luts=u8(z.luts_bytes)),
              dict(O=like(x[0]), saved=u8(z.saved_bytes), workspace=u8(z.ws_forward_bytes), need_saved=False),
              dict(workspace=u8(z.ws_backward_bytes),
                   out=(like(x[0]), like(x[1]), like(x[2]), torch.empty(p.d, p.d, device=dev)))]
    Mc, luts, ws = sla.sla_build_mask(p, x[0], x[1], **kw[0])
    O, saved = sla.sla_forward(p, x[0], x[1], x[2], W, Mc, luts, **kw[1])
    grads = sla.sla_backward(p, x[0], x[1], x[2], W, Mc, luts, saved, x[3], **kw[2])
    if given:
        assert Mc is kw[0]["Mc"] and luts is kw[0]["luts"] and ws is kw[0]["workspace"]
        assert O is kw[1]["O"] and saved is kw[1]["saved"]
        assert all(a is b for a, b in zip(grads, kw[2]["out"]))
    assert sla.sla_forward(p, x[0], x[1], x[2], W, Mc, luts, need_saved=False)[1] is None
    return (Mc, O) + tuple(grads)


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("layout", [sla.SLA_BHND, sla.SLA_BNHD, sla.SLA_STRIDED])
def test_same_results_as_the_calls_step_by_step(monkeypatch, layout, dtype, given):
    p, x, W = _tensors(layout, dtype)
    got = _all(p, x, W, given)
    monkeypatch.setattr(sla, "_host_calls", lambda: _HandsEverythingBack)
    ref = _all(p, x, W, given)
    for a, b in zip(got, ref):
        assert a.stride() == b.stride() and a.dtype == b.dtype and a.device == b.device
        assert torch.equal(a, b)


def test_same_errors_as_the_calls_step_by_step(monkeypatch):
    p, x, W = _tensors(sla.SLA_BHND, torch.bfloat16)
    Q, K, V, dO = x
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)
    O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
    bad_p = sla.make_params(2, 3, 333, 64, 0.2, 0.2, torch.bfloat16, bkv=128)
    small = torch.empty(8, dtype=torch.uint8, device="cuda")
    calls = [
        lambda: sla.sla_build_mask(bad_p, Q, K),
        lambda: sla.sla_build_mask(p, Q.float(), K),
        lambda: sla.sla_build_mask(p, Q[:, :, :300], K),
        lambda: sla.sla_build_mask(p, Q.transpose(1, 2).contiguous().transpose(1, 2), K),
        lambda: sla.sla_build_mask(p, Q.cpu(), K),
        lambda: sla.sla_build_mask(p, Q, K, workspace=small),
        lambda: sla.sla_build_mask(p, Q, K, luts=small),
        lambda: sla.sla_forward(p, Q, K, V, W.float(), Mc, luts),
        lambda: sla.sla_forward(p, Q, K, V, W.t(), Mc, luts),
        lambda: sla.sla_forward(p, Q, K, V, W, Mc[:, :, :2], luts),
        lambda: sla.sla_forward(p, Q, K, V, W, Mc, luts, O=O.float()),
        lambda: sla.sla_forward(p, Q, K, V, W, Mc, luts, saved=small),
        lambda: sla.sla_forward(p, Q, K, None, W, Mc, luts),
        lambda: sla.sla_backward(p, Q, K, V, W, Mc, luts, small, dO),
        lambda: sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO, out=(Q, K, V, W)),
        lambda: sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO, out=(Q, K, V)),
        lambda: sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, None),
        # a workspace that is not 16-byte aligned: refused by the library itself
        lambda: sla.sla_forward(p, Q, K, V, W, Mc, luts,
                                workspace=torch.empty(sla.sla_sizes(p).ws_forward_bytes + 1, dtype=torch.uint8, device="cuda")[1:]),
    ]

    def errors():
        out = []
        for f in calls:
            with pytest.raises((sla.SLAError, ValueError, AttributeError, TypeError)) as e:
                f()
            out.append((type(e.value), str(e.value)))
        return out

    got = errors()
    monkeypatch.setattr(sla, "_host_calls", lambda: _HandsEverythingBack)
    assert got == errors()


def test_subclasses_take_the_python_path():
    class Plain(torch.Tensor):
        pass

    p, (Q, K, V, dO), W = _tensors(sla.SLA_BHND, torch.bfloat16)
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)
    O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
    assert torch.equal(Mc, sla.sla_build_mask(p, Q.as_subclass(Plain), K)[0])
    # the compiled calls hand every tensor of a subclass back, in any place, and take parameters
    host, addr = sla._host_calls(), ctypes.addressof(p)
    new = torch.empty_like
    ws = torch.empty(max(sla.sla_sizes(p).ws_backward_bytes, sla.sla_sizes(p).ws_mask_bytes), dtype=torch.uint8, device="cuda")
    calls = [(host.build_mask, [Q, K, ws, new(Mc), new(luts)], []),
             (host.forward, [Q, K, V, W, Mc, luts, new(O), new(saved), ws], [True]),
             (host.mask_forward, [Q, K, V, W], [True]),
             (host.backward, [Q, K, V, W, Mc, luts, saved, dO, ws, new(Q), new(K), new(V), torch.empty_like(W, dtype=torch.float32)],
              [False])]
    for call, tensors, rest in calls:
        assert type(call(addr, *tensors, *rest)) is tuple
        assert type(call(addr, *[torch.nn.Parameter(t, requires_grad=False) for t in tensors], *rest)) is tuple
        for i, t in enumerate(tensors):
            assert call(addr, *tensors[:i], t.as_subclass(Plain), *tensors[i + 1:], *rest) is None, (call, i)


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,H,d,bq,k_h,k_l", [(1, 3, 64, 64, 1.0, 0.0), (5, 2, 128, 64, 0.2, 0.2), (64, 1, 64, 128, 0.1, 0.1),
                                               (65, 2, 128, 64, 0.1, 0.1), (130, 1, 64, 256, 0.05, 0.2),
                                               (70, 3, 64, 64, 0.3, 0.7), (70, 1, 128, 64, 0.0, 0.1)])
def test_mask_and_forward_in_one_call(monkeypatch, T, H, d, bq, k_h, k_l, dtype, saved):
    # pooling or column tables beside the states; no marginal block (no states at all); no critical block
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    N = T * 64 - (7 if T > 1 else 0)
    Q, K, V, dO = (torch.randn(2, H, N, d, generator=g, device="cuda").to(dtype) for _ in range(4))
    W = (0.02 * torch.randn(d, d, generator=g, device="cuda")).to(dtype)
    p = sla.make_params(2, H, N, d, k_h, k_l, dtype, bq=bq)
    got = sla.sla_mask_forward(p, Q, K, V, W, need_saved=saved)
    with monkeypatch.context() as m:
        m.setattr(sla, "_host_calls", lambda: _HandsEverythingBack)
        ref = sla.sla_mask_forward(p, Q, K, V, W, need_saved=saved)
    names = lambda luts: sla.lut_views(p, luts)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[2], ref[2])
    for (k, a), b in zip(names(got[1]).items(), names(ref[1]).values()):
        assert torch.equal(a, b), k
    assert (got[3] is None) == (not saved)
    if saved:
        a, b = (sla.sla_backward(p, Q, K, V, W, x[0], x[1], x[3], dO) for x in (got, ref))
        assert all(torch.equal(x, y) for x, y in zip(a, b))
