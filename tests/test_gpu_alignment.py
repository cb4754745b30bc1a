"""Operands and results that lie at any multiple of their element's size: the
kernels' wide loads and stores (16 bytes, through buffers and pointers) give
the same bits at every such address."""
import pytest

import synth

from gpu_util import assert_bitwise, device_inputs, inputs, say

pytestmark = pytest.mark.gpu


def _shifted(t):
    """A contiguous copy of t that starts one element past an allocation's start."""
    if t is None:
        return None
    import torch
    v = torch.zeros(t.numel() + 64, dtype=t.dtype, device=t.device)[1:1 + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == t.element_size()
    return v


@pytest.mark.parametrize("base,kw", [
    ("lstm_h512_t1000", dict(batch=20, input=112, hidden=528)),                       # step_small by rows, fp32
    ("lstm_h512_t1000", dict(batch=3, input=16, hidden=80)),                          # ... by fragments
    ("lstm_h2048_bf16_t10000", dict(batch=20, input=1248, hidden=96, loss="mean_sq_all")),   # bf16, by rows
    ("lstm_h2048_bf16_t10000", dict(batch=100, input=64, hidden=672, loss="mean_sq_all")),   # wide bf16
    ("lstm_h4096_t20000", dict(batch=300, input=48, hidden=1040, w_scale=1.0 / 32, loss="mean_sq_all")),  # split fp32
    ("resmlp_w4096_l2000_bf16", dict(batch=70, hidden=160, w_scale=0.05)),            # wide residual MLP
    ("resmlp_w4096_l2000_bf16", dict(dtype="f32", batch=70, hidden=272, w_scale=0.05)),
    ("mlp_widths_l2000", dict(batch=40, hidden=128, widths=(128, 64, 128, 32))),
])
def test_any_element_address(base, kw):
    import torch

    import paper_1806_01117_amd as amb
    wl = synth.get(base).with_(n_steps=5, name=base + "_shifted", **kw)
    dev = device_inputs(wl, *inputs(wl))
    res = []
    for place in (lambda t: t, _shifted):
        r = amb.Runner(amb.ProblemSpec.from_workload(wl, fast_slots=3, slow_slots=0))
        try:
            if wl.cell in ("rnn", "lstm"):
                r.set("path", 1)
            x, W, b, h0, c0 = (place(t) for t in dev)
            out = {"dW": place(torch.zeros(W.shape, device="cuda")), "db": place(torch.zeros(b.shape, device="cuda")),
                   "dh0": place(torch.zeros(h0.shape, device="cuda")),
                   "dc0": place(torch.zeros(h0.shape, device="cuda")) if c0 is not None else None}
            say(wl.name, kw, "shifted" if place is _shifted else "aligned")
            got = r.run(x, W, b, h0, c0, out=out)
            res.append({k: v.cpu().numpy() if hasattr(v, "cpu") else v for k, v in got.items() if v is not None})
        finally:
            r.close()
    assert_bitwise(*res)
