"""Products large enough for the 256 x 256, 256 x 128 and 128 x 128 blocks, with rows, columns and a
contracted dimension that are no multiples of a block or a stage (the remainder of K comes
first, per plane of A), against float64 products on the same device.

Bars: the cross stack's (2e-2 forward, 5e-2 gradients for bf16 activations), tighter for hi +
lo pairs and f16 (5e-3; x_out itself is bf16). bf16 gradients carry the roundings of gt and
[gv|gq|gk] (2^-9 each) through two layers."""
import pytest
import torch

from gpu_helpers import gemm_plan, need_gpu
from paper_2402_06859_amd.rdcn import Rdcn, make_config

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


# rows, dense inputs (16 more make the width), rank (no attention: any rank); the plans, as (tile rows,
# tile columns, splits, stages), of the down and up products and of the weight gradients
B256, B128, M3, M2, S64 = (256, 256, 1, 2), (256, 128, 1, 3), (128, 128, 1, 3), (128, 128, 1, 2), (64, 64, 1, 3)


@pytest.mark.parametrize("mode,tol", [("storage", 1e-2), ("hilo", 5e-3), ("f16", 5e-3)])
@pytest.mark.parametrize("rows,dense,rank,down,up,grads", [
    (2003, 2088, 2056, B128, B128, B128), (4100, 1032, 2184, B256, B128, (128, 128, 3, 2)),
    (1537, 3080, 1736, M3, B128, B128),
    (8300, 1976, 2024, B256, B256, (256, 256, 4, 2)),    # the batch in 4
    (20500, 1512, 1000, B256, B256, (256, 256, 10, 2)),  # ... in 10 (24 tiles)
    (33000, 984, 1016, B256, B256, (256, 256, 16, 2)),   # ... in 16 (16 tiles, the last split short)
    (16500, 984, 1016, B256, B256, (128, 128, 6, 2)),
    (8100, 2024, 504, M3, B256, (128, 128, 6, 2)),       # down: 256 blocks
    (2500, 1080, 1064, M3, S64, (128, 128, 2, 3)),
    (1700, 1984, 1048, S64, M3, (128, 128, 1, 3)),        # fused epilogues on 128 x 128, three stages
    (1301, 1048, 408, S64, S64, (64, 64, 2, 3)),
    # fewer rows than a load's clamp, over many column tiles
    (5, 20488, 64, S64, S64, S64), (5, 30984, 64, S64, M2, M3)])
def test_products(rows, dense, rank, down, up, grads, mode, tol):
    plans = [gemm_plan(rows, rank, 16 + dense), gemm_plan(rows, 16 + dense, rank, fused_out=True),
             gemm_plan(16 + dense, rank, rows, weight_grad=True), gemm_plan(rank, 16 + dense, rows, weight_grad=True)]
    assert [(p.bm, p.bn, p.splits, p.stages) for p in plans] == [down, up, grads, grads]
    need_gpu()
    dev = "cuda"
    d, L = 16 + dense, 2
    g = torch.Generator(device=dev)
    g.manual_seed(rows)
    rand = lambda *s, std=1.0: (torch.randn(*s, device=dev, generator=g) * std).bfloat16()
    x0, go = rand(rows, d), rand(rows, d)
    std = (2.0 / (d + rank)) ** 0.5
    W, U, b = [[rand(*s, std=t) for _ in range(L)] for s, t in (((rank, d), std), ((d, rank), std), ((d,), 0.1))]
    lib = Rdcn(make_config(rows, 1, 16, dense, rank, L, 40, 40, 1600, activation_mode=mode))
    sb, tb = lib.workspace_bytes(rows)
    saved, scratch = (torch.empty(max(n, 1), dtype=torch.uint8, device=dev) for n in (sb, tb))
    x_out, gx0 = torch.empty_like(x0), torch.empty(rows, d, device=dev)
    gW, gU, gb = ([torch.full(t.shape, float("nan"), device=dev) for t in ts] for ts in (W, U, b))
    print("large blocks", mode, rows, d, rank, flush=True)
    lib.rdcn_forward(rows, x0, W, U, b, x_out, saved, scratch)
    lib.rdcn_backward(rows, x0, W, U, b, saved, go, gx0, gW, gU, gb, scratch)
    torch.cuda.synchronize()
    assert lib.check_device_errors() == 0
    X, xs, hs, ts = x0.double(), [x0.double()], [], []
    for l in range(L):
        hs.append(xs[l] @ W[l].double().t())
        ts.append(hs[l] @ U[l].double().t() + b[l].double())
        xs.append(X * ts[l] + xs[l])
    errs = {"x": rel(x_out, xs[L])}
    gr, acc = go.double(), torch.zeros_like(X)
    for l in reversed(range(L)):
        gt = gr * X
        acc += gr * ts[l]
        gh = gt @ U[l].double()
        errs.update({"gU%d" % l: rel(gU[l], gt.t() @ hs[l]), "gb%d" % l: rel(gb[l], gt.sum(0)),
                     "gW%d" % l: rel(gW[l], gh.t() @ xs[l])})
        gr = gr + gh @ W[l].double()
    errs["gx0"] = rel(gx0, acc + gr)
    print({k: "%.2g" % v for k, v in errs.items()}, flush=True)
    assert all(v <= (tol if k == "x" else 1e-2) for k, v in errs.items()), errs
