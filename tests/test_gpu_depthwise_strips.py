"""Depthwise 3x3 kernels where their strips and channel groups end: strips with a remainder, one row, one column, channel counts
with no divisor for a workgroup (a tail of idle threads), odd maps at stride 2.  Reference: torch in float64 on the CPU.  Tolerances:
outputs are rounded to bf16 once (2^-8 of the value) after an fp32 sum of nine products; the weight gradient is an fp32 sum, its
error below n * 2^-24 of the sum of magnitudes for n terms added in a chain."""
import pytest

pytestmark = pytest.mark.gpu

# batch, H, W, C, stride
SHAPES = [(4, 35, 96, 848, 1), (4, 35, 95, 848, 2), (1, 1, 1, 8, 1), (1, 1, 1, 8, 2), (2, 1, 5, 200, 1), (2, 2, 1, 424, 2),
          (8, 19, 64, 416, 1), (3, 5, 3, 16, 2)]


@pytest.mark.parametrize("batch,H,W,C,stride", SHAPES)
def test_depthwise_strips(batch, H, W, C, stride):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(C + H)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    x = torch.randn(batch, H, W, C, generator=gen).bfloat16()
    w = (torch.randn(C, 9, generator=gen) / 3).bfloat16()
    d = torch.randn(batch, Ho, Wo, C, generator=gen).bfloat16()
    act = (4 * torch.randn(batch, H, W, C, generator=gen) + 3).clamp(0, 6).bfloat16()
    one = torch.ones(C).bfloat16()

    def shifted(a, ky, kx):       # a[h * stride + ky - 1, w * stride + kx - 1], zeros outside
        p = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1))
        return p[:, ky:ky + (Ho - 1) * stride + 1:stride, kx:kx + (Wo - 1) * stride + 1:stride]

    xd, wd, dd = x.double(), w.double(), d.double()
    z = torch.zeros(batch, Ho, Wo, C, dtype=torch.float64)
    dw, mag = torch.zeros(C, 9, dtype=torch.float64), torch.zeros(C, 9, dtype=torch.float64)
    g = torch.zeros(batch, H + 2, W + 2, C, dtype=torch.float64)
    for t in range(9):
        ky, kx = divmod(t, 3)
        s = shifted(xd, ky, kx)
        z += s * wd[:, t]
        dw[:, t] = (dd * s).sum((0, 1, 2))
        mag[:, t] = (dd * s).abs().sum((0, 1, 2))
        g[:, ky:ky + (Ho - 1) * stride + 1:stride, kx:kx + (Wo - 1) * stride + 1:stride] += dd * wd[:, t]
    dx = g[:, 1:H + 1, 1:W + 1] * ((act > 0) & (act < 6))

    dev = lambda a: a.to("cuda:0")
    xt, wt, dt, at, ot = dev(x), dev(w), dev(d), dev(act), dev(one)
    zt = torch.full((batch, Ho, Wo, C), float("nan"), device="cuda:0", dtype=torch.bfloat16)
    yt, out = torch.full_like(zt, float("nan")), torch.full_like(xt, float("nan"))
    dwt = torch.full((C, 9), float("nan"), device="cuda:0")
    ws = torch.full((et.et_debug_depthwise3x3_ws_floats(batch, H, W, C, stride),), float("nan"), device="cuda:0")
    st = torch.cuda.current_stream().cuda_stream
    run = lambda *a: et.et_debug_depthwise3x3(*a, batch, H, W, C, stride, st)
    assert run(0, xt.data_ptr(), wt.data_ptr(), ot.data_ptr(), ot.data_ptr(), zt.data_ptr(), yt.data_ptr(), 0) == 0
    assert run(1, dt.data_ptr(), wt.data_ptr(), 0, at.data_ptr(), out.data_ptr(), 0, 0) == 0
    assert run(2, dt.data_ptr(), xt.data_ptr(), 0, 0, dwt.data_ptr(), 0, ws.data_ptr()) == 0
    torch.cuda.synchronize()
    zg = zt.cpu().double()
    assert torch.all((zg - z).abs() <= 2.0 ** -8 * z.abs() + 1e-5)
    assert torch.equal(yt.cpu(), (zg + 1).clamp(0, 6).bfloat16())
    assert torch.all((out.cpu().double() - dx).abs() <= 2.0 ** -8 * dx.abs() + 1e-5)
    assert torch.all((dwt.cpu().double() - dw).abs() <= batch * Ho * Wo * 2.0 ** -24 * mag + 1e-6)
