"""The ring tile of the bf16 GEMM (64 x 64, direct-to-LDS slices of 64): one, a few and many slices around the ring's depth, ragged
lengths of every dimension, split reductions, and its implicit convolutions over any number of pixels.  References and
bounds are those of the other tiles' tests."""
import pytest

from test_gpu_conv3x3 import _case, _case_dw, _case_gathered, _case_split
from test_gpu_gemm import _run

pytestmark = pytest.mark.gpu

RING = 23


@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (3, 8, 8), (65, 72, 128), (63, 136, 191), (130, 64, 192), (64, 200, 193), (200, 72, 256),
                                   (72, 104, 321), (197, 64, 509), (100, 330, 1000)])
def test_ring_tile(M, N, K, a_t, b_t):
    _run(M, N, K, a_t, b_t, 1, True, a_t == 0 and b_t == 0, 1, RING, seed=M + N + K)
    _run(M, N, K, a_t, b_t, 0, True, False, 1, RING, seed=M + K)


@pytest.mark.parametrize("M,N,K,split", [(64, 64, 640, 2), (136, 200, 1999, 5), (40, 72, 5000, 19), (128, 64, 64 * 200 + 8, 50)])
def test_ring_tile_split_reduction(M, N, K, split):
    _run(M, N, K, 1, 1, 1, False, False, split, RING, seed=split)


@pytest.mark.parametrize("batch,H,W,C,N", [(1, 1, 1, 64, 64), (1, 5, 7, 64, 72), (2, 9, 8, 128, 64), (3, 13, 13, 192, 200)])
def test_ring_convolution(batch, H, W, C, N):
    for mode in (0, 1, 2):
        _case(batch, H, W, C, N, mode, RING, seed=H + C + mode)
    for split in (2, 4):
        _case_split(batch, H, W, C, N, 3, split, RING, seed=H + split)


@pytest.mark.parametrize("batch,H,W,C,N,split", [(1, 5, 5, 8, 8, 1), (1, 1, 3, 64, 64, 1), (3, 13, 13, 64, 72, 1), (2, 25, 25, 24, 40, 4), (5, 7, 9, 128, 136, 1)])
def test_ring_convolution_weight_gradient(batch, H, W, C, N, split):
    _case_dw(batch, H, W, C, N, split, RING, seed=H + N)


@pytest.mark.parametrize("taps,stride", [(3, 2), (1, 2), (1, 1)])
def test_ring_convolution_with_stride(taps, stride):
    _case_gathered(3, 15, 17, 64, 72, taps, stride, RING, seed=taps + stride)
    _case_gathered(2, 16, 8, 64, 72, taps, stride, RING, seed=taps + stride, split=0)   # (weight gradient with the planned tile)


@pytest.mark.parametrize("batch,H,W,C,N", [(1, 25, 25, 128, 128), (3, 13, 13, 256, 256), (2, 7, 7, 512, 512)])
def test_planned_convolution_over_odd_maps(batch, H, W, C, N):
    """Tile and split from the planner, pixel counts that are not multiples of 64."""
    _case_split(batch, H, W, C, N, 3, 0, 0, seed=C)
    _case_dw(batch, H, W, C, N, 0, 0, seed=C + 1)


@pytest.mark.parametrize("tile", [25, 29])
@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(64, 128, 64), (3, 8, 8), (129, 136, 191), (130, 260, 193), (72, 104, 509), (260, 130, 1000)])
def test_eight_wave_ring_tiles(M, N, K, a_t, b_t, tile):
    _run(M, N, K, a_t, b_t, 1, True, a_t == 0 and b_t == 0, 1, tile, seed=M + N + K)
    _run(M, N, K, a_t, b_t, 0, True, False, 1, tile, seed=M + K)
    if a_t and N % 4 == 0 and K > 500:
        _run(M, N, K, 1, 1, 1, False, False, 3, tile, seed=K)


@pytest.mark.parametrize("tile", [25, 27, 29])
@pytest.mark.parametrize("batch,H,W,C,N", [(1, 1, 1, 64, 64), (1, 5, 7, 64, 72), (2, 9, 8, 128, 64), (3, 13, 13, 192, 200)])
def test_eight_wave_ring_convolution(batch, H, W, C, N, tile):
    for mode in (0, 1, 2):
        _case(batch, H, W, C, N, mode, tile, seed=H + C + mode)
    _case_split(batch, H, W, C, N, 3, 2, tile, seed=H)
    if tile != 29:
        _case_dw(batch, H, W, C, N, 2 if H > 10 else 1, tile, seed=H + N)


@pytest.mark.parametrize("tile", [25, 27])
def test_eight_wave_ring_convolution_with_stride(tile):
    for taps, stride in ((3, 2), (1, 2)):
        _case_gathered(3, 15, 17, 64, 72, taps, stride, tile, seed=taps + stride)
