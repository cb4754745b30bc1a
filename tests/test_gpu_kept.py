"""Pre-activations that a forward step keeps for its adjoint.  With an interval
of one nearly every adjoint forms them again, store-all keeps the last 16
steps' (the ring's size; 37 steps wrap it twice), Revolve on two slots and an
interval of 20 keep them in between: gradients and loss agree bit for bit, on
every path that keeps them."""
import pytest

import synth

from gpu_util import assert_bitwise, device_inputs, inputs, run_gpu

pytestmark = pytest.mark.gpu

N = 37


@pytest.mark.parametrize("base,kw,opts", [
    ("lstm_h512_t1000", dict(batch=20, input=16, hidden=48), {"path": 1}),                      # step_small, fp32
    ("rnn_h64_t128", dict(batch=5, input=16, hidden=48, loss="mean_sq_all"), {"path": 1}),
    ("lstm_h2048_bf16_t10000", dict(batch=9, input=32, hidden=64), {}),                         # ... bf16
    ("lstm_h2048_bf16_t10000", dict(batch=70, input=64, hidden=128, loss="mean_sq_all"), {}),   # wide bf16
    ("lstm_h2048_bf16_t10000", dict(cell="rnn", batch=50, input=64, hidden=192), {}),
    ("lstm_h4096_t20000", dict(batch=260, input=16, hidden=1040, w_scale=1.0 / 32, loss="mean_sq_all"), {}),  # split fp32
    ("lstm_h4096_t20000", dict(cell="rnn", batch=1100, input=16, hidden=272, w_scale=1.0 / 16), {}),
    ("resmlp_w4096_l2000_bf16", dict(batch=70, hidden=128, w_scale=0.05, loss="mean_sq_all"), {}),  # wide residual MLP
    ("resmlp_w4096_l2000_bf16", dict(batch=20, hidden=96, w_scale=0.05), {}),                   # resmlp_step
    ("resmlp_w4096_l2000_bf16", dict(dtype="f32", batch=20, hidden=80, w_scale=0.05, loss="mean_sq_all"), {}),
    ("mlp_widths_l2000", dict(batch=40, hidden=128, widths=(128, 64, 128, 32), loss="mean_sq_all"), {}),
])
def test_kept_equals_formed_again(base, kw, opts):
    wl = synth.get(base).with_(n_steps=N, name=base + "_kept", **kw)
    dev = device_inputs(wl, *inputs(wl))
    path = opts.get("path")
    again = run_gpu(wl, dev, path=path, fast_slots=3, slow_slots=N, interval_min=1)
    for slots, host, interval in ((N, 0, 0), (2, 0, 0), (4, N, 20), (6, N, 5)):
        if wl.cell == "mlp" and slots == N:
            slots = 12  # its sized schedule's table grows with the slots
        assert_bitwise(again, run_gpu(wl, dev, path=path, fast_slots=slots, slow_slots=host, interval_min=interval))


@pytest.mark.parametrize("base,kw", [
    ("lstm_h512_t1000", dict(batch=20, input=16, hidden=1040)),                                 # step_small
    ("lstm_h2048_bf16_t10000", dict(batch=70, input=64, hidden=128, loss="mean_sq_all")),       # wide bf16
    ("lstm_h4096_t20000", dict(batch=260, input=16, hidden=1040, w_scale=1.0 / 32, loss="mean_sq_all")),  # split fp32
    ("resmlp_w4096_l2000_bf16", dict(batch=70, hidden=128, w_scale=0.05, loss="mean_sq_all")),  # wide residual MLP
])
def test_fewer_places(base, kw):
    # the ring of kept steps may be smaller or absent: the workspace shrinks by
    # its places and the results stay
    import paper_1806_01117_amd as amb
    from paper_1806_01117_amd._lib import EINVAL, AmbpttError
    wl = synth.get(base).with_(n_steps=N, name=base + "_places", **kw)
    dev = device_inputs(wl, *inputs(wl))
    want = run_gpu(wl, dev, fast_slots=4, slow_slots=N, interval_min=20)
    place = -(-4 * wl.batch * wl.gates * wl.hidden // 256) * 256
    r = amb.Runner(amb.ProblemSpec.from_workload(wl, fast_slots=4, slow_slots=N, interval_min=20))
    full = r.ws.numel()
    assert r.L.ambptt_workspace_bytes(r.ctx) == full
    try:
        for kept in (5, 0, 1, 16):
            r.set("kept_steps", kept)
            assert r.ws.numel() == full - (16 - kept) * place
            got = r.run(*dev)
            assert_bitwise(want, {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in got.items() if v is not None})
        with pytest.raises(AmbpttError) as e:
            r.set("kept_steps", 17)
        assert e.value.status == EINVAL
        r.set("kept_steps", 3)
        with pytest.raises(AmbpttError) as e:  # the workspace that is bound has three places
            from paper_1806_01117_amd._lib import check
            check(r.L.ambptt_set_int(r.ctx, b"kept_steps", 4))
        assert e.value.status == EINVAL
        r.run(*dev)
    finally:
        r.close()
