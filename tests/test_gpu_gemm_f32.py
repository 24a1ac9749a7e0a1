"""Float models' products (all six of a layer) against the fp64 oracle at sizes around the
blocks, the waves' split of k and the split of a long batch over workgroups.

Bar: float products and sums over K <= 5000 terms; an error of sqrt(K) roundings of the
terms' magnitude is below 1e-5 of the result's norm."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import gemm_plan, need_gpu, relerr, to_np
from paper_2402_06859_amd.step import DeviceBatch
from paper_2402_06859_amd.synth import Workload, make_inputs

pytestmark = pytest.mark.gpu


def run_and_compare(wl, edit=None):
    inp = make_inputs(wl, bias_std=0.1)
    db = DeviceBatch(wl, inp)
    if edit is not None:
        edit(db)
    db.gather()
    db.forward()
    db.backward()
    torch.cuda.synchronize()
    x0 = to_np(db.x0)
    W, U, b = ([w.float().numpy() for w in inp[k]] for k in ("w_down", "u", "bias"))
    args = (wl.alpha, wl.beta, wl.temperature)
    xL = oracle.forward(x0, W, U, b, *args)
    gx0, gW, gU, gb = oracle.backward(x0, W, U, b, inp["grad_out"].float().numpy(), *args)
    errs = [relerr(to_np(db.x_out), xL), relerr(to_np(db.grad_x0), gx0)]
    for l in range(wl.num_layers):
        errs += [relerr(to_np(db.g_w_down[l]), gW[l]), relerr(to_np(db.g_u[l]), gU[l]), relerr(to_np(db.g_bias[l]), gb[l])]
    print(wl.batch, wl.d, wl.rank, "max rel err %.2g" % max(errs), flush=True)
    assert max(errs) <= 1e-5


# batch (K of the weight gradients): 1, below and above one step of 16 and one pass of the
# waves, several passes, long enough to be split over workgroups; rank and width: one
# remainder, one block and several, all on 32 x 32 blocks but the last's up and gx
@pytest.mark.parametrize("batch,cat,dense,rank,attn", [
    (1, 2, 4, 4, False), (17, 2, 8, 12, False), (130, 2, 8, 36, True), (515, 3, 20, 32, False), (2051, 4, 64, 64, False),
    (4099, 2, 32, 20, False), (300, 60, 64, 128, True), (1030, 31, 492, 132, False)])
def test_products(batch, cat, dense, rank, attn):
    need_gpu()
    run_and_compare(Workload("f32", 31, batch, cat, 10_000, 100, 16, dense, 2, rank, attn, "f32", "mul", 1.1))


# 64 x 64 blocks (four waves side by side, two groups along k): all six products, every
# combination of contiguous and strided operands, with remainders of rows, columns and k
# (1030, 988 and 532: none a multiple of 64 or of a pass of 128 k)
@pytest.mark.parametrize("batch,cat,dense,rank", [(1030, 31, 492, 532), (2053, 31, 492, 532)])
def test_products_of_64_blocks(batch, cat, dense, rank):
    need_gpu()
    d = 16 * cat + dense
    for M, N, K, grad in ((batch, rank, d, False), (batch, d, rank, False), (d, rank, batch, True), (rank, d, batch, True)):
        p = gemm_plan(M, N, K, "f32", grad)
        assert (p.bm, p.bn) == (64, 64)
    run_and_compare(Workload("f32", 32, batch, cat, 10_000, 100, 16, dense, 1, rank, False, "f32", "mul", 1.1))


def test_weights_aligned_to_a_float():
    """Float weights one float past a 16-byte boundary: the fragments' loads ask for no more."""
    need_gpu()

    def shift(ts):
        out = []
        for t in ts:
            v = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape)
            v.copy_(t)
            assert v.data_ptr() % 16 == 4
            out.append(v)
        return out

    def edit(db):
        db.w_down, db.u = shift(db.w_down), shift(db.u)

    run_and_compare(Workload("f32", 33, 130, 2, 10_000, 100, 16, 8, 2, 36, True, "f32", "mul", 1.1), edit)
