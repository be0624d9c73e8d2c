"""The 3x3 convolution of 64 channels from tiles of the input with their border: images of one tile and many, ragged ends in both directions,
one and several blocks of output channels, more tiles than workgroups; every epilogue.  References and bounds are those of the gathered
convolution's tests; against its ring tile, whose sums run in the same order, the results are the same bit for bit."""
import pytest

from test_gpu_conv3x3 import _case, _case_split

pytestmark = pytest.mark.gpu

HALO = 31


@pytest.mark.parametrize("batch,H,W,N", [(1, 8, 32, 64), (1, 6, 30, 64), (2, 16, 25, 128), (3, 13, 60, 64), (1, 7, 113, 192), (2, 56, 56, 64)])
def test_halo_convolution(batch, H, W, N):
    for mode in (0, 1, 2):
        _case(batch, H, W, 64, N, mode, HALO, seed=H + W + mode)
    _case_split(batch, H, W, 64, N, 3, 1, HALO, seed=H + N)


@pytest.mark.parametrize("batch,H,W,N", [(2, 16, 25, 128), (9, 50, 50, 64), (8, 112, 112, 64), (5, 64, 64, 128)])
def test_halo_convolution_gives_the_bits_of_the_ring_tile(batch, H, W, N):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(batch)
    dev = lambda *s: torch.randn(*s, generator=gen).bfloat16().to("cuda:0")  # noqa: E731
    x, w, bias, u, gain = dev(batch, H, W, 64), dev(N, 3, 3, 64), dev(N), dev(batch * H * W, N), dev(N)
    p = lambda t: t.data_ptr()  # noqa: E731
    part = torch.empty(16, device="cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    for mode in (0, 1, 2, 3):
        res = []
        for tile in (23, HALO):
            out = torch.full((batch * H * W + 1, N), float("nan"), device="cuda:0", dtype=torch.bfloat16)
            z = torch.full_like(out, float("nan"))
            if mode == 3:
                st = et.et_debug_conv3x3_split(p(x), p(w), p(out), p(z), batch, H, W, 64, N, p(bias), p(gain), 0, 3, 1, p(part), tile, stream)
            else:
                st = et.et_debug_conv3x3(p(x), p(w), p(out), batch, H, W, 64, N, p(bias), p(u), mode, tile, stream)
            assert st == 0
            torch.cuda.synchronize()
            res.append((out.view(torch.int16), z.view(torch.int16)))
        assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1]), mode


def test_halo_convolution_refuses_other_layers():
    import torch
    from paper_2312_14227_amd import binding as et
    t = torch.zeros(1 << 20, device="cuda:0", dtype=torch.bfloat16)
    p, stream = t.data_ptr(), torch.cuda.current_stream().cuda_stream
    for (H, W, C, N) in ((8, 32, 128, 64), (8, 32, 64, 72), (8, 32, 64, 32), (7, 7, 64, 64)):
        assert et.et_debug_conv3x3(p, p, p, 1, H, W, C, N, p, p, 0, HALO, stream) == et.ET_EINVAL
