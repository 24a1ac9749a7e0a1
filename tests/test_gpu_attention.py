"""The bf16 attention kernels' two forms (panel sums and direct sums, chosen per sample by
its range of scores) against the fp64 oracle, where the choice and its tiles have edges.

One layer without depth: q, k and v come from x0 and W through exact bf16 products with
float sums, so the float weight gradients see the attention through two bf16 roundings
only (gt or x0's products, and [gv|gq|gk] or h: 2^-9 each) and must be within 2^-8 of the
oracle in norm; softmax errors of one f16 rounding (2^-11) stay below that. The key
gradient sum_i A_ij a_i (v_j - o_i) nearly cancels where the softmax is close to one-hot
(o_i = v_j): the rounding of its terms is bounded by 2^-11 of their magnitudes' sum, which
is added to its bar.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import need_gpu, relerr, to_np
from paper_2402_06859_amd.rdcn import Rdcn, make_config
from paper_2402_06859_amd.step import DeviceBatch
from paper_2402_06859_amd.synth import Workload, make_inputs

pytestmark = pytest.mark.gpu
TOL = 2.0 ** -8


def compare(wl, edit=None):
    inp = make_inputs(wl, bias_std=0.1)
    if edit is not None:
        edit(inp)
    db = DeviceBatch(wl, inp)
    db.gather()
    db.forward()
    db.backward()
    torch.cuda.synchronize()
    x0 = to_np(db.x0)
    W, U, b = ([w.float().numpy() for w in inp[k]] for k in ("w_down", "u", "bias"))
    args = (wl.alpha, wl.beta, wl.temperature)
    xL = oracle.forward(x0, W, U, b, *args)
    gx0, gW, gU, gb = oracle.backward(x0, W, U, b, inp["grad_out"].float().numpy(), *args)
    r = wl.rank
    # magnitudes of the key gradient's terms against the gradient, from q, k, v and gh in float64
    P = x0.astype(np.float64) @ W[0].T.astype(np.float64)
    v, q, k = (P[:, i * r:(i + 1) * r] for i in range(3))
    gh = (inp["grad_out"].float().numpy().astype(np.float64) * x0) @ U[0]
    S = q[:, :, None] * k[:, None, :] / wl.temperature
    A = np.exp(S - S.max(2, keepdims=True))
    A /= A.sum(2, keepdims=True)
    o = np.einsum("bij,bj->bi", A, v)
    w = A * (gh * q / wl.temperature)[:, :, None]
    gk = (w * (v[:, None, :] - o[:, :, None])).sum(1)
    mag = (np.abs(w) * (np.abs(v[:, None, :]) + np.abs(o[:, :, None]))).sum(1)
    tol = {"gk": TOL + 2.0 ** -11 * np.linalg.norm(mag) / max(np.linalg.norm(gk), 1e-3 * np.linalg.norm(gh))}
    errs = {"x": relerr(to_np(db.x_out), xL), "gx0": relerr(to_np(db.grad_x0), gx0),
            "gU": relerr(to_np(db.g_u[0]), gU[0])}
    scale = 1e-3 * np.linalg.norm(gW[0])  # (a part that vanishes exactly is measured on the whole)
    for i, n in enumerate(("gv", "gq", "gk")):
        ref = gW[0][i * r:(i + 1) * r]
        errs[n] = np.linalg.norm(to_np(db.g_w_down[0])[i * r:(i + 1) * r] - ref) / max(np.linalg.norm(ref), scale)
    print(wl.rank, wl.batch, wl.temperature, {n: "%.2g" % e for n, e in errs.items()}, "gk bar %.2g" % tol["gk"],
          flush=True)
    assert all(e <= tol.get(n, TOL) for n, e in errs.items()), errs


# rank: 24, 40 and 120 (always direct), 128 and 136 (one tile and the next), 256 | 264 (one
# wave | four), 512 | 520 (one tile per wave | two), 1024; batches leave waves of the last
# workgroup without a sample. Temperatures: one group of panels, several, several sweeps
# over the entries, and so sharp that samples take the direct sums (rank 256 at 0.08 mixes both).
@pytest.mark.parametrize("rank,batch,tau", [
    (24, 9, 1.0), (40, 7, 0.5), (120, 7, 1.0), (128, 6, 1.0), (136, 5, 0.3), (256, 6, 4.0), (256, 33, 0.08),
    (256, 5, 0.02), (264, 3, 1.0), (264, 3, 0.1), (512, 3, 0.2), (520, 3, 1.0), (1024, 3, 1.0), (1024, 24, 0.05),
    (1024, 2, 0.02)])
def test_forms(rank, batch, tau):
    need_gpu()
    compare(Workload("att", 21, batch, 4, 20_000, 150, 16, 64, 1, rank, True, "bf16", "sum", 1.1, temperature=tau))


@pytest.mark.parametrize("rank", [40, 256, 600])
@pytest.mark.parametrize("what", ["keys", "queries", "values", "one_sided"])
def test_degenerate_ranges(rank, what):
    """All keys equal (a range of width 0), all queries zero, all values zero, and queries and
    keys of one sign far from zero (a shifted range)."""
    need_gpu()

    def edit(inp):
        w = inp["w_down"][0]
        if what == "keys":
            w[2 * rank:] = w[2 * rank]
        elif what == "queries":
            w[rank:2 * rank] = 0
        elif what == "values":
            w[:rank] = 0
        else:  # a strong common direction on the dense inputs
            inp["dense"][:] = 1
            w[rank:, 64:] += 0.08

    compare(Workload("att_deg", 22, 5, 4, 20_000, 150, 16, 64, 1, rank, True, "bf16", "sum", 1.1), edit)


def one_hot_layer(rank, spread, B, seed, edit=None, **cfg):
    """One layer over B unit vectors: sample b of x0 is e_b, so its v, q, k are column b of W and its gh row
    b of U, exactly, and column b of W's gradient holds its stored [gv|gq|gk]. Returns the float64
    [B, 1, r] v and k, [B, r, 1] q and gh, the stored gradient [3 r, B] and the saved buffer."""
    dev, d = "cuda", 64
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    rand = lambda *s: torch.randn(*s, device=dev, generator=g)
    W = rand(3 * rank, d)
    W[rank:2 * rank] *= spread
    W, U, b = W.bfloat16(), rand(d, rank).bfloat16(), torch.zeros(d, dtype=torch.bfloat16, device=dev)
    if edit is not None:
        edit(W)
    x0 = torch.zeros(B, d, dtype=torch.bfloat16, device=dev)
    x0[range(B), range(B)] = 1
    lib = Rdcn(make_config(B, 1, 16, d - 16, rank, 1, 40, 40, 1600, attn_alpha=1.0, **cfg))
    saved, scratch = (torch.zeros(n, dtype=torch.uint8, device=dev) for n in lib.workspace_bytes(B))
    x_out, gx0 = torch.empty_like(x0), torch.empty(B, d, device=dev)
    gW, gU, gb = (torch.empty(t.shape, device=dev) for t in (W, U, b))
    lib.rdcn_forward(B, x0, [W], [U], [b], x_out, saved, scratch)
    lib.rdcn_backward(B, x0, [W], [U], [b], saved, torch.ones_like(x0), gx0, [gW], [gU], [gb], scratch)
    torch.cuda.synchronize()
    assert lib.check_device_errors() == 0
    v, q, k = (W[i * rank:(i + 1) * rank, :B].double().t()[:, None, :] for i in range(3))
    return v, q.transpose(1, 2), k, U[:B].double()[:, :, None], gW[:, :B].double(), saved


# 192 and 256: one wave per sample; 264, 520 and 1024: four; spread: of the logits (16 to 96 panels)
@pytest.mark.parametrize("rank,spread", [(192, 1.0), (256, 0.3), (256, 3.0), (264, 1.0), (512, 3.0), (520, 1.0),
                                         (1024, 1.0)])
def test_panel_sums_precision(rank, spread):
    """The backward's column sums before [gv|gq|gk] are stored as bf16 (exact inputs; skip_beta is
    0, so that gv is the softmax's sum alone). How many stored values are not the float64
    value's bf16 measures the error: one of eps relative to a value flips a share of about
    eps / 2^-7.5 (the spacing of bf16). The direct form's, and that of panels whose exponentials
    are rounded to f16, is 2e-4 or so and flips 2 to 5%; with hi + lo exponentials the forward's
    rounded Z and o remain, below 1e-4 in the typical sample. Bar: 1.5% over gv and gk. (gq is
    the forward's sum and keeps its one rounding: at most the 2^-11 that the bars above allow.)"""
    need_gpu()
    v, q, k, go, got, _ = one_hot_layer(rank, spread, 8, rank, skip_beta=0.0)
    A = torch.softmax(q * k, 2)
    D = A * (v - (A * v).sum(2, keepdim=True))
    ref = torch.cat([(A * go).sum(1), (go * D * k).sum(2), (D * go * q).sum(1)], 1).t()    # [3 r, B]
    assert torch.equal(got, got.bfloat16().double())
    shares = []
    for i in range(3):
        y, x = ref[i * rank:(i + 1) * rank], got[i * rank:(i + 1) * rank]
        big = y.abs() >= 0.25 * y.square().mean(0, keepdim=True).sqrt()
        shares.append(float((y.float().bfloat16().double() != x)[big].double().mean()))
    print(rank, spread, "flipped roundings gv %.4f gq %.4f gk %.4f" % tuple(shares), flush=True)
    assert (shares[0] + shares[2]) / 2 <= 0.015


# 120: direct sums; 128, 136 and 256: panels of one wave; 264, 520, 1024: of four; spread 60:
# samples beyond the panels, in the same kernels
@pytest.mark.parametrize("mode", ["hilo", "f16"])
@pytest.mark.parametrize("rank,spread", [(120, 1.0), (128, 1.0), (136, 1.0), (256, 1.0), (256, 60.0), (264, 1.0), (520, 1.0),
                                         (520, 60.0), (1024, 1.0)])
def test_second_planes_of_h(rank, spread, mode):
    """h as the forward keeps it: bf16, and a second plane with the bf16 rounding's remainder or the
    f16 value. The saved buffer of one layer starts with [v|q|k] (float), then the two planes, each
    256-byte aligned. Bars: what the planes hold (2^-17 of h, or 2^-11 for f16) in the largest element
    and the sums' 2^-11 (one f16 rounding of the exponentials) in norm."""
    need_gpu()
    B = 5
    v, q, k, _, _, saved = one_hot_layer(rank, spread, B, 100 + rank, activation_mode=mode)
    h = (v + (torch.softmax(q * k, 2) * v).sum(2)[:, None, :])[:, 0]
    al = lambda n: -(-n // 256) * 256
    o1 = al(B * 3 * rank * 4)
    o2 = o1 + al(B * rank * 2)
    plane = lambda o, dt: saved[o:o + B * rank * 2].view(dt).view(B, rank).double()
    hi = plane(o1, torch.bfloat16)
    full = hi + plane(o2, torch.bfloat16) if mode == "hilo" else plane(o2, torch.float16)
    held = 2.0 ** -17 if mode == "hilo" else 2.0 ** -11
    err = float((full - h).norm() / h.norm())
    print(rank, spread, mode, "rel err %.2g" % err, flush=True)
    assert err <= 2.0 ** -11 + held  # (h as bf16 alone: 1e-3)
    assert float(((hi - full).abs() / full.abs().clamp_min(1e-3)).max()) <= 2.0 ** -8


@pytest.mark.parametrize("rank", [120, 136, 256, 520, 1024])
@pytest.mark.parametrize("what,part,value", [("query", 1, "nan"), ("query", 1, "inf"), ("key", 2, "nan"), ("key", 2, "inf"),
                                             ("value", 0, "nan")])
def test_nonfinite_inputs(rank, what, part, value):
    """One non-finite coordinate: W has it in sample 1's column, and the products with the other samples' zeros
    make theirs NaN. h is NaN wherever float64 has NaN; a bad query leaves the other rows within the
    usual bar (in the direct form all but row 7 + 16, whose exponentials share a matrix operand's
    column with row 7's: zero times NaN)."""
    need_gpu()
    B = 6

    def edit(W):
        W[part * rank + 7, 1] = float(value)

    # q, k, v as the projection left them, and h (bf16), from the saved buffer
    saved = one_hot_layer(rank, 1.0, B, 7, edit)[5]
    n = B * 3 * rank * 4
    P = saved[:n].view(torch.float32).view(B, 3, rank).double()
    v, q, k = P[:, 0, None, :], P[:, 1, :, None], P[:, 2, None, :]
    h = v[:, 0] + (torch.softmax(q * k, 2) * v).sum(2)
    o1 = -(-n // 256) * 256
    hd = saved[o1:o1 + B * rank * 2].view(torch.bfloat16).view(B, rank).double()
    print(rank, what, value, "NaN of %d: %d, device %d" % (h.numel(), h.isnan().sum(), hd.isnan().sum()), flush=True)
    assert hd[h.isnan()].isnan().all()
    if what == "query":
        rest = h.isfinite()
        assert rest.sum() == B * (rank - 1)
        if rank < 128:
            rest[:, 7 + 16] = False
        assert float((hd - h)[rest].norm() / h[rest].norm()) <= TOL
