"""Which blocks a product gets (csrc/gemm.hip, plan_gemm), on both sides of the lines between the
plans; the figures each line rests on stand beside it there."""
import pytest

from gpu_helpers import gemm_plan


def tiles(M, N, bm, bn):
    return -(-M // bm) * -(-N // bn)


# 160 to 239 tiles of 128 x 128: a fused epilogue or a short K leaves them to 64 x 64 blocks
@pytest.mark.parametrize("M,N,K,fused,bm", [
    (4096, 640, 64, True, 64), (4096, 640, 2048, True, 64), (4096, 768, 256, True, 64), (2048, 1792, 512, True, 64),
    (2048, 1792, 1016, True, 64), (2048, 1792, 1024, True, 128), (600, 5376, 1024, True, 128),
    (4096, 768, 512, False, 64), (4096, 768, 1024, False, 128), (4096, 768, 1856, False, 128),
    (5120, 640, 504, False, 64), (5120, 640, 512, False, 128),
    (4096, 512, 4096, False, 64), (4096, 1024, 64, True, 128)])  # 128 tiles and 256
def test_mid_size_products(M, N, K, fused, bm):
    p = gemm_plan(M, N, K, fused_out=fused)
    assert (p.bm, p.bn, p.splits) == (bm, bm, 1), (p.bm, p.bn, p.splits)
    # 128 x 128 blocks of at most one per CU run three stages
    assert p.stages == 3


# rows of the batch, then width and rank of the gradient: 256 x 256 blocks that split the batch
@pytest.mark.parametrize("K,M,N,splits", [
    (8300, 1992, 2024, 4), (16384, 4352, 512, 7), (20500, 1528, 1000, 10), (32767, 1000, 1016, 0), (33000, 1000, 1016, 16),
    (65536, 1856, 256, 16), (65535, 1856, 256, 0),
    # fewer than 8 tiles: 16 splits of them would leave more than half of the chip idle
    (300_000, 1792, 256, 0), (600_000, 256, 256, 0), (131_072, 1024, 256, 0)])
def test_split_weight_gradients(K, M, N, splits):
    p = gemm_plan(M, N, K, weight_grad=True)
    blocks = tiles(M, N, p.bm, p.bn) * p.splits
    if splits:
        assert (p.bm, p.bn, p.splits) == (256, 256, splits)
        assert blocks >= 128
    else:
        assert p.bm < 256 and p.splits > 1 and blocks >= 128
    assert -(-K // p.splits) >= 512
