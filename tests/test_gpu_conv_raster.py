"""The 3x3 convolution of small images from windows of a raster of all their pixels: images of a single pixel and of a row, windows that cover
many images, the widest one, ragged ends; one chunk of input channels and many, odd and even; one workgroup, and enough to share CUs; every
epilogue.  References and bounds are those of the gathered convolution's tests."""
import pytest

from test_gpu_conv3x3 import _case, _case_split

pytestmark = pytest.mark.gpu

@pytest.mark.parametrize("batch,H,W,C,N", [(1, 1, 1, 64, 64), (40, 1, 1, 64, 64), (5, 1, 9, 128, 64), (2, 7, 7, 512, 128), (33, 3, 5, 64, 64),
                                           (3, 14, 14, 192, 192), (1, 62, 62, 64, 64), (2, 30, 31, 64, 128), (1, 9, 30, 128, 64),
                                           (37, 14, 14, 64, 256), (2, 28, 28, 320, 64)])
def test_raster_convolution(batch, H, W, C, N):
    for tile in (33, 35) if W <= 30 else (33,):   # 128, 256 positions per workgroup
        for mode in (0, 1, 2):
            _case(batch, H, W, C, N, mode, tile, seed=H + W + mode)
        _case_split(batch, H, W, C, N, 3, 1, tile, seed=H + N)


def test_raster_convolution_refuses_other_layers():
    import torch
    from paper_2312_14227_amd import binding as et
    t = torch.zeros(1 << 22, device="cuda:0", dtype=torch.bfloat16)
    p, stream = t.data_ptr(), torch.cuda.current_stream().cuda_stream
    for (H, W, C, N, tile) in ((8, 63, 64, 64, 33), (8, 31, 64, 64, 35), (8, 8, 96, 64, 33), (8, 8, 64, 96, 33), (8, 8, 64, 32, 35)):
        assert et.et_debug_conv3x3(p, p, p, 1, H, W, C, N, p, p, 0, tile, stream) == et.ET_EINVAL
