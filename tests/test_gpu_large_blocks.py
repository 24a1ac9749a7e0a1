"""Products large enough for the 256 x 256, 256 x 128 and 128 x 128 blocks, with rows, columns and a
contracted dimension that are no multiples of a block or a stage (the remainder of K comes
first, per plane of A), against float64 products on the same device.

Bars: the cross stack's (2e-2 forward, 5e-2 gradients for bf16 activations), tighter for hi +
lo pairs and f16 (5e-3; x_out itself is bf16). bf16 gradients carry the roundings of gt and
[gv|gq|gk] (2^-9 each) through two layers."""
import pytest
import torch

from gpu_helpers import need_gpu
from paper_2402_06859_amd.rdcn import Rdcn, make_config

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float((a.double() - b).norm() / b.norm())


# rows, categorical features x 16 + dense = width, rank (no attention: any rank)
@pytest.mark.parametrize("mode,tol", [("storage", 1e-2), ("hilo", 5e-3), ("f16", 5e-3)])
@pytest.mark.parametrize("rows,dense,rank", [(2003, 2088, 2056), (4100, 1032, 2184), (1537, 3080, 1736),
                                             (8300, 1976, 2024),   # weight gradients: 256 x 256, the batch in 4
                                             (16500, 984, 1016),   # ... in 16: 16 tiles, ragged, uneven splits
                                             (8100, 2024, 504),    # 256 blocks of 128 x 128, three stages
                                             (2500, 1080, 1064),   # fewer of them; weight gradients split too
                                             (1301, 1048, 408),    # weight gradients on 64 x 64 blocks
                                             # fewer rows than a load's clamp, over many column tiles
                                             (5, 20488, 64), (5, 30984, 64)])
def test_products(rows, dense, rank, mode, tol):
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
