"""The large-batch fp32 kernels on the bf16 matrix cores (operands split in
three bf16 parts), at sizes ragged against their tiles and 32-wide stages: row
tiles of 256 and 128, units past the last tile, an input that ends inside a
stage, no input at all.  Each run is compared with the oracle and, bit for
bit, across schedules, and must be no further from the oracle than the fp32
MFMA kernels on the same inputs (within the spread of two summation orders:
a factor of 1.5)."""
import numpy as np
import pytest

import synth

from gpu_util import TOL_F32, assert_bitwise, assert_close, device_inputs, inputs, rel_err, run_gpu, run_oracle, say

pytestmark = pytest.mark.gpu

KEYS = ("loss", "dW", "db", "dh0", "dc0")


def _rms(got, want):
    got, want = np.asarray(got, np.float64), np.asarray(want, np.float64)
    return float(np.sqrt(np.mean((got - want) ** 2)) / np.sqrt(np.mean(want ** 2)))


@pytest.mark.parametrize("cell,B,D,H,n", [
    ("lstm", 256, 16, 1024, 5),    # 128-row tiles, whole; the input fills half a stage
    ("lstm", 300, 48, 1040, 5),    # partial row tile, units past the last tile, input of one and a half stages
    ("lstm", 1030, 32, 1248, 3),   # 256-row tiles, the last of 6 rows
    ("rnn", 300, 0, 1040, 6),      # no input; one gate
    ("rnn", 1100, 80, 272, 6),     # K below two stages per part
    ("rnn", 4100, 16, 1104, 3),    # 256-row tiles with one gate, the last of 4 rows, units past the last tile
])
def test_against_oracle(cell, B, D, H, n):
    wl = synth.get("lstm_h4096_t20000").with_(cell=cell, loss="mean_sq_all", batch=B, input=D, hidden=H, n_steps=n,
                                              w_scale=H ** -0.5, h0_std=0.3, name=f"{cell}_f32x3")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    want = run_oracle(wl, *host)
    a = run_gpu(wl, dev, fast_slots=3, slow_slots=n, interval_min=2)
    assert_close(a, want, TOL_F32)
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=n, slow_slots=0))   # store-all
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=2, slow_slots=0))   # plain Revolve
    old = run_gpu(wl, dev, fast_slots=3, slow_slots=n, interval_min=2, opts={"lds_gemm": 2})
    assert not np.array_equal(a["dh0"], old["dh0"])  # other kernels
    for k in KEYS:
        if k in want and k != "loss":
            e, e0 = _rms(a[k], want[k]), _rms(old[k], want[k])
            say(k, f"{e:.2e} split, {e0:.2e} fp32 MFMA")
            assert e <= 1.5 * e0 + 1e-7, k


@pytest.mark.parametrize("B,D,H", [
    (8192, 0, 32),    # one stage for two wave groups: the first has none
    (16384, 0, 16),   # ... half of it padding
    (16390, 16, 16),  # a group for the input's, one for the state's; a last row tile of 6 rows
])
def test_shortest_reductions(B, D, H):
    wl = synth.get("lstm_h4096_t20000").with_(cell="rnn", loss="mean_sq_all", batch=B, input=D, hidden=H, n_steps=3,
                                              w_scale=H ** -0.5, h0_std=0.3, name="rnn_f32x3_short")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    a = run_gpu(wl, dev, fast_slots=3, slow_slots=0)
    assert a["stats"]["kernel_calls"][3] == 2  # the large-batch path
    assert_close(a, run_oracle(wl, *host), TOL_F32)
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=2, slow_slots=0))


@pytest.mark.parametrize("cell,B,D,H,n,window", [
    ("lstm", 1, 176, 80, 5, 1),     # windows of one row
    ("lstm", 20, 176, 80, 9, 1),    # ... of 20: less than a stage
    ("rnn", 3, 0, 48, 70, 24),      # no input; windows of 72 and 66 rows (three stages: a padded fourth)
    ("rnn", 3, 0, 48, 70, 40),      # ... of 120 and 90 rows (four stages, and three)
    ("lstm", 20, 48, 80, 32, 8),    # columns past the last tile of both operands
    ("lstm", 33, 144, 128, 9, 31),  # the input ends inside a column tile; one window of 297 rows
])
def test_weight_gradient_windows(cell, B, D, H, n, window):
    # one launch per step: only the windows run on the bf16 matrix cores
    wl = synth.get("lstm_h512_t1000").with_(cell=cell, loss="mean_sq_all", batch=B, input=D, hidden=H, n_steps=n,
                                            w_scale=H ** -0.5, h0_std=0.3, name=f"{cell}_dw_f32x3")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    want = run_oracle(wl, *host)
    a = run_gpu(wl, dev, path=1, window=window, fast_slots=3, slow_slots=n, interval_min=2)
    assert_close(a, want, TOL_F32)
    assert_bitwise(a, run_gpu(wl, dev, path=1, window=window, fast_slots=n, slow_slots=0))
    old = run_gpu(wl, dev, path=1, window=window, fast_slots=3, slow_slots=n, interval_min=2, opts={"lds_gemm": 2})
    assert not np.array_equal(a["dW"], old["dW"])  # two kernels, so two orders of summation
    for k in ("dW", "db"):
        e, e0 = _rms(a[k], want[k]), _rms(old[k], want[k])
        say(k, f"{e:.2e} split, {e0:.2e} fp32 MFMA")
        assert e <= 1.5 * e0 + 1e-7, k


def test_tiny_gradients():
    # dL/dh_0 about 1e-36: zbar's low parts would leave bf16's range unscaled
    wl = synth.get("lstm_h4096_t20000").with_(cell="rnn", loss="half_sq_last", batch=256, input=16, hidden=1024,
                                              n_steps=22, w_scale=0.0022, h0_std=0.3, name="rnn_f32x3_tiny")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    want = run_oracle(wl, *host)
    say("max |dh0|", float(np.max(np.abs(want["dh0"]))))
    assert 1e-37 < np.max(np.abs(want["dh0"])) < 1e-30
    a = run_gpu(wl, dev, fast_slots=22, slow_slots=0)
    assert rel_err(a["dh0"], want["dh0"]) <= 1e-5


def test_small_operands():
    # operands near the smallest normal value keep all their bits: inputs,
    # states and weights of about 1e-37 beside ordinary ones, each in gradients
    # that they alone make.  (Unscaled, their second and third bf16 parts leave
    # bf16's range: 1e-4 and more.)  Bound: 2^-24 per rounding, sums of up to
    # 2048 terms in some 70 roundings, against the largest of the region.
    B, D, H = 1024, 32, 256
    wl = synth.get("lstm_h4096_t20000").with_(cell="rnn", loss="half_sq_last", batch=B, input=D, hidden=H, n_steps=2,
                                              w_scale=H ** -0.5, h0_std=0.3, name="rnn_f32x3_small")
    x, W, b, x0 = inputs(wl)
    x, W, x0 = x.copy(), W.copy(), {k: v.copy() for k, v in x0.items()}
    b = np.zeros_like(b)
    x[:, :, 16:] *= 1e-37       # dW's columns 16 .. 31
    W[128:, :] *= 1e-37         # units 128 .. 255: states of that size
    x0["h"][:, 128:] *= 1e-37   # dW's columns D + 128 ..
    W[:, D + 64:D + 128] *= 1e-37  # dL/dh_0's columns 64 .. 127
    dev = device_inputs(wl, x, W, b, x0)
    want = run_oracle(wl, x, W, b, x0)
    a = run_gpu(wl, dev, fast_slots=2, slow_slots=0)
    assert a["stats"]["kernel_calls"][3] == 1  # the large-batch path
    for k, rows, cols in (("dW", slice(0, 128), slice(16, 32)), ("dW", slice(0, 128), slice(D + 128, D + 256)),
                          ("dh0", slice(0, B), slice(64, 128))):
        g, w = np.asarray(a[k], np.float64)[rows, cols], np.asarray(want[k], np.float64)[rows, cols]
        e = float(np.max(np.abs(g - w)) / np.max(np.abs(w)))
        say(k, cols, f"largest {np.max(np.abs(w)):.1e}, error {e:.1e}")
        assert 1e-39 < np.max(np.abs(w)) < 1e-33 and e <= 5e-6, (k, cols)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38, 1e25])  # 1e25: only the scaled sums overflow
def test_values_that_do_not_split(value):
    # an infinite, NaN or huge input behaves as with the fp32 MFMA kernels
    wl = synth.get("lstm_h4096_t20000").with_(loss="mean_sq_all", batch=270, input=16, hidden=1024, n_steps=3,
                                              w_scale=1.0 / 32, name="lstm_f32x3_nonfinite")
    x, W, b, x0 = inputs(wl)
    x = x.copy()
    x[1, 5, 3] = value
    dev = device_inputs(wl, x, W, b, x0)
    a = run_gpu(wl, dev, fast_slots=3, slow_slots=0)
    o = run_gpu(wl, dev, fast_slots=3, slow_slots=0, opts={"lds_gemm": 2})
    for k in KEYS:
        u, v = np.asarray(a[k], np.float64), np.asarray(o[k], np.float64)
        assert np.array_equal(np.isnan(u), np.isnan(v)), k
        assert np.array_equal(np.isinf(u), np.isinf(v)), k
        f = np.isfinite(u)
        if f.any():
            assert np.max(np.abs(u[f] - v[f])) <= 1e-4 * max(np.max(np.abs(v[f])), 1e-30), k
