"""Forward products over few rows (16 x 16, 32 x 32 and 64 x 32 blocks whose waves split K)
against the fp64 oracle: row, column and K remainders, every activation mode (one and two
planes of A, f16 operands), and the head's layers.

Bars: those of the cross stack's forward (2e-2 for bf16 activations, 2e-3 / 5e-3 for hi +
lo pairs and f16) and of the head's logits (2e-3)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import FWD_TOL, need_gpu, relerr, to_np
from paper_2402_06859_amd.step import DeviceBatch
from paper_2402_06859_amd.synth import HeadSpec, Workload, make_inputs
from test_gpu_head import Y_TOL, run_head

pytestmark = pytest.mark.gpu


# (rows, categorical features, dense, rank): widths 16 cat + dense around a stage of K (64)
# and the eight waves' turns (512), ranks as K and as N
@pytest.mark.parametrize("mode,tol", [("storage", FWD_TOL["bf16"]), ("hilo", 2e-3), ("f16", 5e-3)])
@pytest.mark.parametrize("rows,cat,dense,rank", [
    (1, 2, 8, 8), (15, 4, 0, 24), (16, 4, 64, 64), (17, 30, 40, 72), (33, 32, 8, 256), (70, 96, 24, 136),
    (200, 100, 256, 264), (257, 120, 8, 128)])
def test_forward(rows, cat, dense, rank, mode, tol):
    need_gpu()
    wl = Workload("few", 41, rows, cat, 10_000, 100, 16, dense, 2, rank, False, "bf16", "sum", 1.1, act_mode=mode)
    inp = make_inputs(wl, bias_std=0.1)
    db = DeviceBatch(wl, inp)
    db.gather()
    db.forward()
    torch.cuda.synchronize()
    W, U, b = ([w.float().numpy() for w in inp[k]] for k in ("w_down", "u", "bias"))
    err = relerr(to_np(db.x_out), oracle.forward(to_np(db.x0), W, U, b, wl.alpha, wl.beta, wl.temperature))
    print(rows, wl.d, rank, mode, "rel err %.2g" % err, flush=True)
    # (x_out itself is bf16: at most 2^-9 of each value)
    assert err <= tol + (0 if mode == "storage" else 2.0 ** -9)
    assert db.lib.check_device_errors() == 0


@pytest.mark.parametrize("rows,hidden", [(1, (24,)), (13, (72, 40)), (50, (256, 128)), (90, (520, 264)), (130, (1000, 776))])
def test_head(rows, hidden):
    need_gpu()
    wl = Workload("fewhead", 42, rows, 40, 10_000, 100, 16, 72, 1, 16, False, "bf16", "sum", 1.1)
    dh, ref, _, _ = run_head(wl, HeadSpec("few", hidden), rows)
    assert relerr(to_np(dh.y), ref["y"]) <= Y_TOL
    assert relerr(to_np(dh.y_cal), ref["y_cal"]) <= Y_TOL
    assert relerr(to_np(dh.grads["W"][0]), ref["W"][0]) <= 1e-2
