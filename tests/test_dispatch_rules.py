"""Which kernel a product or convolution takes, at sizes on either side of the rules' lines where the other choice was measured to be the slower one
(or, for long reductions of convolutions, the less precise one).  Host code only."""
import pytest

from paper_2312_14227_amd import binding as et

DIRECT, RING = {11, 13, 15}, {23, 25, 29}
RASTER = {33, 35}


@pytest.mark.parametrize("M,N,K,kw,allowed", [
    (1377, 640, 4032, {}, RING),                             # 7.1 GFLOP, 63 slices: 18.1 us against 22.5 on tiles of 64 x 128
    (1576, 3072, 768, dict(c_f32=1, residual=1), RING),      # 7.4 GFLOP: 18.4 / 19.7
    (1159, 3904, 768, dict(b_t=1, epilogue=2), RING | {1, 3}),   # 6.9 GFLOP: 16.4 / 18.4
    (4970, 1088, 960, dict(b_t=1, epilogue=2), RING),        # 10.4 GFLOP, GELU backward: 19.3 / 21.6
    (3072, 1856, 1024, dict(b_t=1, epilogue=2), RING),       # 11.7 GFLOP: 19.8 / 22.0
    (12608, 3072, 768, {}, DIRECT),
    (12608, 3072, 768, dict(epilogue=1), DIRECT),
    (12608, 768, 3072, dict(c_f32=1, residual=1), DIRECT),
    (6304, 4096, 1024, dict(b_t=1, epilogue=2), DIRECT),
])
def test_products(M, N, K, kw, allowed):
    assert et.et_debug_gemm_tile(M, N, K, **kw) in allowed


@pytest.mark.parametrize("batch,side,C,raster", [
    (16, 7, 1024, False), (36, 4, 1024, False), (48, 7, 1024, False), (28, 7, 1024, False), (8, 14, 576, False),
    (32, 7, 512, True), (32, 14, 256, True), (32, 28, 128, True), (64, 7, 512, True), (16, 7, 512, False), (40, 14, 256, False),
])
def test_convolutions(batch, side, C, raster):
    tile, split = et.et_debug_conv3x3_plan(batch, side, side, C, C)
    assert (tile in RASTER) == raster and (split == 1 or not raster)
