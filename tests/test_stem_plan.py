"""Weight gradient of the 7x7 stem, [N channels x 256 window elements] reduced over the output pixels: the chunks of the reduction that
its plan asks for, read off the scratch size, against the tiles that exist for it (64 x 512, 128 x 256, 256 x 192, 256 x 256: one or
two tiles for at most 256 channels).  With one workgroup per (tile, chunk), the plan has to give seven of eight compute units one wherever the
pixels suffice for chunks of four slices of 64 (an eighth is what whole slices can cost: 1 568 slices make 224 chunks of 7)."""
import pytest

from paper_2312_14227_amd import binding as et

CUS = 256


def _chunks(batch, side, N):
    Ho = (side - 1) // 2 + 1
    padded = 2 * (Ho - 1) + 8
    up = lambda v: (v + 255) // 256 * 256
    fixed = up(batch * padded * padded * 4 * 2) + up(N * 256 * 2) + up(N * 256 * 4)
    left = et.et_debug_stem_ws_bytes(batch, side, side, 3, N) - fixed - 256
    assert left >= 0
    return max(1, round(left / (N * 256 * 4))), batch * Ho * Ho


@pytest.mark.parametrize("batch,side,N", [(32, 224, 64), (8, 224, 64), (64, 224, 64), (16, 256, 64), (32, 224, 32), (32, 96, 64), (32, 224, 128)])
def test_the_stem_gradient_fills_the_chip(batch, side, N):
    chunks, pixels = _chunks(batch, side, N)
    assert pixels >= 64 * 4 * CUS
    assert CUS * 7 // 8 <= chunks <= CUS
