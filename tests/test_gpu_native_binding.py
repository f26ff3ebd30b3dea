"""The native call path of the Python binding against its Python path: equal bits for every accepted form (bf16 and 16-bit
integer views, lists and tuples, absent outputs and adapters, a given stream), and the same exception for refused ones."""
import pytest

import paper_2309_00754_amd as H
import workloads as WL
from paper_2309_00754_amd import _binding as Bd
from gpu_helpers import dev as to_dev
from gpu_helpers import dev_bf16, say

pytestmark = pytest.mark.gpu


def _calls(dev):
    """(name, call, output tensors) over the entry points; a call runs on the current stream unless it says otherwise."""
    import torch
    z = lambda *s: torch.zeros(s, device=dev)  # noqa: E731
    c = WL.gen_linear(7100, 24, 264, 136, 8)
    x, W, A, B = (dev_bf16(v, dev) for v in (c.x, c.W, c.A, c.B))
    xb, Wb = x.view(torch.bfloat16), W.view(torch.bfloat16)
    o = [z(24, 136) for _ in range(6)]
    yield "linear", lambda: H.hydra_lora_linear(x, Wb, A, B, 2, o[0], o[1]), o[:2]
    yield "linear off only", lambda: H.hydra_lora_linear(xb, W, None, None, 1.0, o[0]), o[:1]
    st = torch.cuda.Stream()
    yield "linear on a stream", lambda: H.hydra_lora_linear(x, W, A, B, 2.0, None, o[1], stream=st), o[1:2]
    ws = torch.empty(H.hydra_lora_linear_workspace_bytes(24, 136, 8), dtype=torch.uint8, device=dev)
    yield "linear ws", lambda: H.hydra_lora_linear_ws(x, W, A, B, 2.0, o[0], o[1], ws), o[:2]
    yield "linear ws, own workspace", lambda: H.hydra_lora_linear_ws(x, W, A, B, 2.0, o[0], o[1]), o[:2]
    yield "group", lambda: H.hydra_lora_linear_group((x, x), [W, Wb], [A, None], [B, None], [2.0, 1], [o[0], o[2]],
                                                     (o[1], None)), o[:3]
    yield "group without outputs off", lambda: H.hydra_lora_linear_group([x], [W], [A], [B], (0.5,), None, [o[1]]), o[1:2]
    xd = x[:3].contiguous()
    gws = H.hydra_lora_linear_group_workspace(2, 3, 136, 8, dev)
    d = [z(3, 136) for _ in range(4)]
    yield "group ws", lambda: H.hydra_lora_linear_group_ws([xd, xd], [W, W], [A, A], [B, B], [2.0, 1.0], d[:2], d[2:],
                                                           gws), d
    yield "multi", lambda: H.hydra_lora_linear_multi(xd, W, [xd, xd], [A, A], [B, B], [2.0, 1.0], d[0], d[1:3]), d[:3]
    yield "multi without adapters", lambda: H.hydra_lora_linear_multi(None, W, [xd], None, None, [1.0], None, [d[1]]), d[1:2]
    mws = torch.empty(max(16, H.hydra_lora_linear_multi_workspace_bytes(3, 136, 8)), dtype=torch.uint8, device=dev)
    yield "multi ws", lambda: H.hydra_lora_linear_multi_ws(xd, W, [xd], [A], [B], [2.0], d[0], [d[1]], mws), d[:2]
    s = WL.gen_score_head(7200, 2, 20, 128, 300, 8)
    h, Wl, Al, Bl, wr = (dev_bf16(v, dev) for v in (s.h, s.W_lm, s.A, s.B, s.w_rm))
    tok, m = to_dev(s.ids, dev), [z(40) for _ in range(5)] + [z(2)]
    err = torch.zeros(1, dtype=torch.int32, device=dev)
    sws = torch.empty(H.hydra_score_workspace_bytes(40, 300), dtype=torch.uint8, device=dev)
    yield "score", lambda: H.hydra_score(h, Wl, Al, Bl, 2.0, tok, wr, 2, 20, *m[:3], reward=m[5], lse_on=m[3],
                                         lse_off=m[4], workspace=sws, err_flag=err), m
    yield "score, own workspace", lambda: H.hydra_score(h, Wl, None, None, 2.0, tok, None, 2, 20, *m[:3]), m[:3]
    yield "score two", lambda: H.hydra_score_two_input(h, h, Wl, Al, Bl, 2.0, tok, wr, 2, 20, *m[:3], reward=m[5],
                                                       workspace=sws), m[:3] + m[5:]
    yield "score noalloc", lambda: H.hydra_score_noalloc(h, Wl, Al, Bl, 2.0, tok, wr, 2, 20, *m[:3], reward=m[5]), m[:3] + m[5:]
    on = torch.randn(40, 301, device=dev)
    off = on + 0.1
    yield "logits", lambda: H.hydra_score_logits(on, off, tok, *m[:3], lse_on=m[3]), m[:4]
    a = WL.gen_advantages(7300, 2, 20, 128)
    kl, rew, hv, wv = to_dev(a.kl, dev), to_dev(a.reward, dev), dev_bf16(a.h, dev), dev_bf16(a.w_v, dev)
    yield "value head", lambda: H.hydra_value_head(hv, wv, m[0]), m[:1]
    yield "advantages", lambda: H.hydra_ppo_advantages(kl, rew, m[0], 2, 20, m[1], m[2], m[3], start=3), m[1:4]
    l3, g = z(3), [z(40), z(40)]
    yield "loss", lambda: H.hydra_ppo_loss(kl, m[3], m[1], m[0], m[2], 2, 20, l3, g[0], g[1], start=3, eps=0.1), [l3] + g
    Wt, dy = torch.empty(264, 136, dtype=W.dtype, device=dev), dev_bf16(WL.gen_linear(7400, 24, 136, 8, 0).x, dev)
    H.hydra_transpose_bf16(W, Wt)
    dx, dA, dB = z(24, 264), z(8, 264), z(136, 8)
    bws = torch.empty(H.hydra_lora_linear_backward_workspace_bytes(24, 136, 264, 8), dtype=torch.uint8, device=dev)
    yield "backward", lambda: H.hydra_lora_linear_backward(x, Wt, A, B, 2.0, dy, dx, dA, dB, bws), [dx, dA, dB]
    yield "backward, dB only", lambda: H.hydra_lora_linear_backward(x, None, A, B, 2.0, dy, dB=dB), [dB]
    yield "backward without adapter", lambda: H.hydra_lora_linear_backward(None, Wt, None, None, 1.0, dy, dx), [dx]


def test_accepted_forms_have_the_bits_of_the_python_path(dev, monkeypatch):
    import torch
    assert not isinstance(Bd._native(), Bd._NoNative), "_hydra_native is not built"
    native = Bd._native()
    took = []

    class Spy:
        def __getattr__(self, name):
            def call(*args):
                st = getattr(native, name)(*args)
                took.append(st != Bd._SLOW)
                return st
            return call

    for name, call, outs in _calls(dev):
        say("native binding", name)
        got = []
        for path in (Spy(), Bd._NoNative()):
            monkeypatch.setattr(Bd, "_nat", path)
            for o in outs:
                o.fill_(float("nan"))
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            got.append([o.clone() for o in outs])
        for p, q in zip(*got):
            assert torch.isfinite(q).all() and torch.equal(p, q), name
        # only what has to be allocated or lacks an adapter goes on to the Python path
        assert took.pop() != ("own workspace" in name or name in ("backward, dB only", "backward without adapter")), name


@pytest.mark.parametrize("what", ["host", "dtype", "strided", "shape", "numpy", "no tensor", "scale", "workspace", "sizes",
                                  "sizes past 64 bits"])
def test_refused_forms_raise_what_the_python_path_raises(what, dev, monkeypatch):
    import torch
    c = WL.gen_linear(7500, 24, 264, 136, 8)
    x, W, A, B = (dev_bf16(v, dev) for v in (c.x, c.W, c.A, c.B))
    y = torch.full((24, 136), 7.0, device=dev)
    tok, v = torch.zeros(24, dtype=torch.int32, device=dev), torch.zeros(24, device=dev)
    ws = torch.empty(H.hydra_score_workspace_bytes(24, 136), dtype=torch.uint8, device=dev)
    call = {
        "host": lambda: H.hydra_lora_linear(x.cpu(), W, A, B, 1.0, y),
        "dtype": lambda: H.hydra_lora_linear(x, W.float(), A, B, 1.0, y),
        "strided": lambda: H.hydra_lora_linear(x, W, A, B, 1.0, torch.empty(136, 24, device=dev).t()),
        "shape": lambda: H.hydra_lora_linear(x, W, A, B[:-1], 1.0, y),
        "numpy": lambda: H.hydra_lora_linear_group([c.x], [W], [A], [B], [1.0], [y]),
        "no tensor": lambda: H.hydra_value_head(None, x[0], v),
        "scale": None,
        "workspace": lambda: H.hydra_score(x, W, A, B, 1.0, tok, None, 1, 24, v, v, v, workspace=True),
        "sizes": lambda: H.hydra_score(x, W, A, B, 1.0, tok, None, 2, 24, v, v, v, workspace=ws),
        # 8 x (2^61 + 3) is 24, the rows of x, in 64 bits
        "sizes past 64 bits": lambda: H.hydra_score(x, W, A, B, 1.0, tok, None, 8, 2 ** 61 + 3, v, v, v, workspace=ws),
    }[what]
    if what == "scale":  # a text that float() reads is taken by both, as the number
        got = []
        for path in (Bd._native(), Bd._NoNative()):
            monkeypatch.setattr(Bd, "_nat", path)
            on = torch.full((24, 136), float("nan"), device=dev)
            H.hydra_lora_linear(x, W, A, B, "2", None, on)
            got.append(on)
        H.hydra_lora_linear(x, W, A, B, 2.0, None, y)
        torch.cuda.synchronize()
        assert torch.equal(got[0], y) and torch.equal(got[1], y)
        return
    kinds = []
    for path in (Bd._native(), Bd._NoNative()):
        monkeypatch.setattr(Bd, "_nat", path)
        with pytest.raises(Exception) as e:
            call()
        kinds.append((type(e.value), str(e.value)))
    torch.cuda.synchronize()
    assert kinds[0] == kinds[1] and (y == 7.0).all()
