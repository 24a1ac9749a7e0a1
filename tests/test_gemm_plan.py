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
