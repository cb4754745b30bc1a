"""The wide bf16 kernels at widths that end in the middle of a 64-wide block
(odd multiples of 32), on tiles of 16, 32 and 64 rows, and at small batches
whose weights are many, and the small-batch kernels where such steps are too
small for them: against the oracle and, bit for bit, across schedules.  A row
of the batch that is not finite stays alone."""
import numpy as np
import pytest

import synth

from gpu_util import TOL_BF16, assert_bitwise, assert_close, assert_close_relu, device_inputs, inputs, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

HADJ = 3


@pytest.mark.parametrize("cell,B,D,H,n,wide", [
    ("lstm", 54, 160, 992, 4, True),   # both segments end in the middle of a block; 16-row tiles, the last of 6 rows
    ("lstm", 100, 64, 672, 4, True),   # 32-row tiles (42 column tiles)
    ("lstm", 70, 96, 992, 3, True),    # 32-row tiles, the last of 6 rows, both segments
    ("lstm", 200, 96, 992, 3, True),   # 64-row tiles, the last of 8 rows, both segments
    ("rnn", 260, 96, 1056, 4, True),   # 16-row tiles; the last column tile and the product's reduction end inside a block
    ("rnn", 150, 32, 2080, 3, True),   # 32-row tiles, the last of 22 rows
    ("rnn", 300, 0, 2080, 3, True),    # 64-row tiles, no input
    ("lstm", 18, 480, 1056, 3, True),  # a small batch with many weights
    ("lstm", 70, 32, 96, 9, False),    # steps of few products: the small-batch kernels
    ("lstm", 48, 96, 608, 5, False),
    ("lstm", 5, 32, 736, 4, False),
    ("rnn", 50, 160, 160, 9, False),
    ("rnn", 512, 480, 608, 3, False),
    ("rnn", 32, 992, 2048, 3, False),
])
def test_cells(cell, B, D, H, n, wide):
    wl = synth.get("lstm_h2048_bf16_t10000").with_(cell=cell, batch=B, input=D, hidden=H, n_steps=n, w_scale=H ** -0.5,
                                                   h0_std=0.3, loss="mean_sq_all", name=f"{cell}_wide_ragged")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    a = run_gpu(wl, dev, fast_slots=3, slow_slots=n, interval_min=2)
    assert a["stats"]["kernel_calls"][HADJ] == (n - 1 if wide else 0)  # which kernels ran
    assert_close(a, run_oracle(wl, *host), TOL_BF16)
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=n, slow_slots=0))
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=2, slow_slots=0))


@pytest.mark.parametrize("B,w,n", [
    (70, 160, 9), (200, 1056, 4), (7, 1056, 5),  # 16-row tiles
    (250, 1312, 4),                              # 32-row tiles, the last of 26 rows
    (250, 2592, 3),                              # 64-row tiles, the last of 58 rows
])
def test_residual_mlp(B, w, n):
    wl = synth.get("resmlp_w4096_l2000_bf16").with_(batch=B, hidden=w, n_steps=n, w_scale=0.9 / w ** 0.5,
                                                    name="resmlp_wide_ragged")
    host = inputs(wl)
    dev = device_inputs(wl, *host)
    a = run_gpu(wl, dev, fast_slots=n, slow_slots=0)
    assert a["stats"]["kernel_calls"][HADJ] == n - 1
    assert_close_relu(a, run_oracle(wl, *host), TOL_BF16)
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=2, slow_slots=n, interval_min=1))
    assert_bitwise(a, run_gpu(wl, dev, fast_slots=2, slow_slots=0))


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_rows_stay_apart(value):
    # what a block reads past the end of a row is the next row's: not even its NaNs count
    wl = synth.get("lstm_h2048_bf16_t10000").with_(batch=70, input=96, hidden=992, n_steps=4, loss="mean_sq_all",
                                                   w_scale=0.03, name="lstm_wide_rows")
    x, W, b, x0 = inputs(wl)
    clean = run_gpu(wl, device_inputs(wl, x, W, b, x0), fast_slots=4, slow_slots=0)
    assert clean["stats"]["kernel_calls"][HADJ] == 3  # the wide kernels ran
    x = x.copy()
    x[2, 3, :] = value
    x0 = {k: v.copy() for k, v in x0.items()}
    x0["h"][17, :] = value
    r = run_gpu(wl, device_inputs(wl, x, W, b, x0), fast_slots=4, slow_slots=0)
    others = [m for m in range(70) if m not in (3, 17)]
    for k in ("dh0", "dc0"):
        assert np.array_equal(np.asarray(r[k])[others], np.asarray(clean[k])[others]), k
