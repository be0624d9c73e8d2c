"""First 3x3 convolution without a column matrix, where its tiles of 32 pixels and 32 or 64 channels end: one pixel, one row, ragged pixel and
channel counts, one to three input channels, both strides, with bias + ReLU and with affine + clamp.  Reference: torch in float64 on
the CPU; a result is an fp32 sum of at most 27 products rounded to bf16 once (2^-8 of the value), the affine is applied to the
rounded value."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("batch,H,W,C,N", [(1, 1, 1, 3, 8), (2, 7, 5, 3, 64), (1, 33, 1, 1, 40), (3, 16, 19, 2, 72), (1, 2, 50, 3, 136), (5, 13, 14, 3, 32)])
def test_first_convolution(batch, H, W, C, N, stride):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(H * W + C + N)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    x = torch.randn(batch, H, W, C, generator=gen).bfloat16()
    w = (torch.randn(N, 3, 3, C, generator=gen) / 3).bfloat16()
    gain, shift = (1 + torch.randn(N, generator=gen) / 4).bfloat16(), torch.randn(N, generator=gen).bfloat16()
    ref = torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), w.double().permute(0, 3, 1, 2), stride=stride, padding=1).permute(0, 2, 3, 1)
    mag = torch.nn.functional.conv2d(x.double().abs().permute(0, 3, 1, 2), w.double().abs().permute(0, 3, 1, 2), stride=stride, padding=1).permute(0, 2, 3, 1)
    xt, wt, gt, st = (a.to("cuda:0") for a in (x, w, gain, shift))
    z = torch.full((batch, Ho, Wo, N), float("nan"), device="cuda:0", dtype=torch.bfloat16)
    y, y2, y3 = (torch.full_like(z, float("nan")) for _ in range(3))
    call = lambda g, zz, yy: et.et_debug_conv_first(xt.data_ptr(), wt.data_ptr(), g, st.data_ptr(), zz, yy, batch, H, W, C, N, stride, 0.0, 6.0,
                                                    torch.cuda.current_stream().cuda_stream)
    assert call(gt.data_ptr(), z.data_ptr(), y.data_ptr()) == 0
    assert call(gt.data_ptr(), 0, y2.data_ptr()) == 0
    assert call(0, 0, y3.data_ptr()) == 0
    torch.cuda.synchronize()
    zc, sums = z.cpu().double(), 27 * 2.0 ** -24 * mag
    assert torch.all((zc - ref).abs() <= 2.0 ** -8 * ref.abs() + sums)
    want = (zc * gain.double() + shift.double()).clamp(0, 6)      # one fp32 fused operation, rounded
    assert torch.all((y.cpu().double() - want).abs() <= (2.0 ** -8 + 2.0 ** -22) * want)
    assert torch.equal(y.cpu(), y2.cpu())
    want = (ref + shift.double()).clamp(min=0)
    assert torch.all((y3.cpu().double() - want).abs() <= 2.0 ** -8 * want + 2 * sums + 2.0 ** -22)


@pytest.mark.parametrize("batch,H,W,C,N,stride", [(1, 5, 70, 3, 64, 1), (2, 4, 140, 3, 40, 2), (1, 6, 100, 1, 8, 1), (1, 4, 140, 2, 32, 2)])
def test_first_convolution_with_tiles_inside_the_image(batch, H, W, C, N, stride):
    """Rows of 70 output pixels and more: 32 consecutive ones without a border pixel among them, which are gathered without a test."""
    Wo = (W - 1) // stride + 1
    inside = lambda p: 0 < p // Wo % ((H - 1) // stride + 1) * stride < H - 1 and 0 < p % Wo * stride < W - 1
    pixels = batch * ((H - 1) // stride + 1) * Wo
    assert any(all(inside(p) for p in range(t, t + 32)) for t in range(0, pixels - 31, 32))
    test_first_convolution(batch, H, W, C, N, stride)


def test_first_convolution_rejects():
    import torch
    from paper_2312_14227_amd import binding as et
    p = torch.zeros(65536, device="cuda:0").data_ptr()
    call = lambda **k: et.et_debug_conv_first(k.get("x", p), p, k.get("g", p), p, k.get("z", 0), p, 1, 4, 4, k.get("C", 3), k.get("N", 8), k.get("s", 1), 0.0, 6.0)
    assert call() == 0
    torch.cuda.synchronize()
    for bad in (dict(C=4), dict(C=0), dict(N=12), dict(N=0), dict(s=3), dict(x=0), dict(x=p + 2), dict(g=0, z=p)):
        assert call(**bad) == -1
