"""The small-batch step kernels on both sides of the sizes at which their loads
go by rows through LDS: row lengths that end in the middle of a 128-byte block
and whole ones, batches ragged against 16 rows, short and long reductions of
the gate product (20 blocks) and of the h-adjoint product (16 blocks); against
the oracle and, bit for bit, across schedules."""
import numpy as np
import pytest

import synth

from gpu_util import TOL_BF16, TOL_F32, assert_bitwise, assert_close, device_inputs, inputs, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,cell,B,D,H,n", [
    ("f32", "lstm", 3, 16, 112, 7),     # neither: 4 and 14 blocks
    ("f32", "lstm", 17, 48, 144, 7),    # the h-adjoint alone: 18 blocks
    ("f32", "lstm", 20, 112, 528, 5),   # both: x and h end in the middle of a block
    ("f32", "rnn", 33, 0, 656, 6),      # no input; 21 blocks
    ("f32", "rnn", 1, 624, 16, 6),      # the gate product alone
    ("bf16", "lstm", 9, 32, 256, 7),    # the h-adjoint alone
    ("bf16", "lstm", 20, 1248, 96, 5),  # the gate product alone (21 blocks, whole and half)
    ("bf16", "rnn", 40, 352, 1056, 5),  # both, h and zbar end in the middle of a block
])
def test_against_oracle(dtype, cell, B, D, H, n):
    base = "lstm_h512_t1000" if dtype == "f32" else "lstm_h2048_bf16_t10000"
    wl = synth.get(base).with_(cell=cell, batch=B, input=D, hidden=H, n_steps=n, w_scale=H ** -0.5, h0_std=0.3,
                               loss="mean_sq_all", name=f"{cell}_{dtype}_small")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    a = run_gpu(wl, dev, path=1, wide=False, fast_slots=3, slow_slots=n, interval_min=2)
    assert_close(a, run_oracle(wl, *host), TOL_F32 if dtype == "f32" else TOL_BF16)
    assert_bitwise(a, run_gpu(wl, dev, path=1, wide=False, fast_slots=n, slow_slots=0))
    assert_bitwise(a, run_gpu(wl, dev, path=1, wide=False, fast_slots=2, slow_slots=0))


def test_rows_stay_apart():
    # what a block reads past the end of a row is the next row's: not even its NaNs count
    wl = synth.get("lstm_h512_t1000").with_(batch=20, input=112, hidden=528, n_steps=3, loss="mean_sq_all",
                                            w_scale=0.05, name="lstm_small_rows")
    x, W, b, x0 = inputs(wl)
    clean = run_gpu(wl, device_inputs(wl, x, W, b, x0), path=1, fast_slots=3, slow_slots=0)
    x = x.copy()
    x[1, 3, :] = np.nan
    x0 = {k: v.copy() for k, v in x0.items()}
    x0["h"][17, :] = np.inf
    r = run_gpu(wl, device_inputs(wl, x, W, b, x0), path=1, fast_slots=3, slow_slots=0)
    others = [m for m in range(20) if m not in (3, 17)]
    for k in ("dh0", "dc0"):
        assert np.array_equal(np.asarray(r[k])[others], np.asarray(clean[k])[others]), k
