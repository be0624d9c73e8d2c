"""Backward pass of a per-channel affine in one launch: one row, remainders of its row groups and chunks, channel counts with no
divisor for a workgroup, every source of the mask, in place.  Element-wise results are bf16 roundings of single operations
and have to be equal to torch's; the sums are fp32 sums of n terms, their error below n * 2^-24 of the sum of magnitudes.  z and y of
the masked cases come from the forward kernels (a depthwise convolution with a single tap), so that a mask taken from z has
to be the mask of the stored y, also where y is rounded to a bound."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(1, 8), (3, 24), (517, 144), (300, 296), (4100, 16), (70, 960), (33, 2048), (20000, 64)])
def test_affine_back(rows, cols):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(rows + cols)
    dev = lambda a: a.to("cuda:0")
    rnd = lambda *s: torch.randn(*s, generator=gen).bfloat16()
    d, add, x = rnd(rows, cols), rnd(rows, cols), 2 * rnd(rows, cols)
    gain, shift = 1 + rnd(cols) / 4, 2 + rnd(cols)
    one_tap = torch.zeros(cols, 9).bfloat16()
    one_tap[:, 4] = 1
    st = torch.cuda.current_stream().cuda_stream
    dt, at, xt, gt, ht, wt = map(dev, (d, add, x, gain, shift, one_tap))
    z, y = torch.empty_like(dt), torch.empty_like(dt)
    p = lambda a: 0 if a is None else a.data_ptr()
    assert et.et_debug_depthwise3x3(0, p(xt), p(wt), p(gt), p(ht), p(z), p(y), 0, 1, rows, 1, cols, 1, st) == 0
    z32 = torch.randn(rows, cols, generator=gen).to("cuda:0")
    ws = torch.full((et.et_debug_affine_back_ws_floats(rows, cols),), float("nan"), device="cuda:0")
    for use_add in (False, True):
        for mask in ("none", "y", "z", "z32"):
            for want in ((1, 1, 1, 1), (1, 0, 0, 1), (0, 1, 1, 0), (0, 0, 1, 0)):
                if mask == "z32" and use_add:
                    continue
                src, addend = dt.clone(), at.clone()
                dmid = (addend if use_add else src) if want[0] else None       # in place
                dout = torch.full_like(dt, float("nan")) if want[1] else None
                total, mul = (torch.full((cols,), float("nan"), device="cuda:0") if k else None for k in want[2:])
                zz = z32 if mask == "z32" else z
                assert et.et_debug_affine_back(p(src), p(addend) if use_add else 0, p(y) if mask == "y" else 0, 0 if mask == "z32" else p(z),
                                               p(z32) if mask == "z32" else 0, p(gt), p(ht), p(dmid), p(dout), p(total), p(mul), p(ws), 6.0,
                                               int(mask == "z"), rows, cols, st) == 0
                torch.cuda.synchronize()
                m = (d.float() + add.float()).bfloat16() if use_add else d
                if mask in ("y", "z"):
                    yc = y.cpu().float()
                    m = torch.where((yc > 0) & (yc < 6), m, torch.zeros_like(m))
                if want[0]:
                    assert torch.equal(dmid.cpu(), m)
                if want[1]:
                    assert torch.equal(dout.cpu(), (m.float() * gain.float()).bfloat16())
                for got, terms in ((total, m.double()), (mul, m.double() * zz.cpu().double())):
                    if got is not None:
                        err = (got.cpu().double() - terms.sum(0)).abs()
                        assert torch.all(err <= rows * 2.0 ** -24 * terms.abs().sum(0) + 1e-30)


@pytest.mark.parametrize("producer", ["two-group", "ring", "split two-group", "split ring", "first convolution"])
def test_mask_from_z_is_that_of_the_stored_activation(producer):
    """z and y as the product's epilogue, its split reduction and the first convolution store them, values spread around either bound of ReLU6
    (the first convolution: of ReLU): the mask computed from z has to close exactly where the stored y lies on a bound."""
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(3)
    st = torch.cuda.current_stream().cuda_stream
    first = producer == "first convolution"
    batch, H, W, C, N = (2, 40, 40, 3, 64) if first else (2, 16, 24, 64, 64)
    rows, hi = batch * H * W, float("inf") if first else 6.0
    dev = lambda a: a.bfloat16().to("cuda:0")
    x, w = dev(torch.randn(batch, H, W, C, generator=gen)), dev(torch.randn(N, 3, 3, C, generator=gen) / (9 * C) ** 0.5)
    # every second channel around 0, the others around 6, steps of y near a rounding unit of the bound
    shift = dev(torch.where(torch.arange(N) % 2 == 0, 0.0, 0.0 if first else 6.0) + torch.randn(N, generator=gen) / 64)
    gain = dev((1 + torch.rand(N, generator=gen)) / 32)
    z, y, d, m = (torch.full((rows, N), float("nan"), device="cuda:0", dtype=torch.bfloat16) for _ in range(4))
    d.copy_(torch.randn(rows, N, generator=gen))
    p = lambda a: a.data_ptr()
    if first:
        assert et.et_debug_conv_first(p(x), p(w), p(gain), p(shift), p(z), p(y), batch, H, W, C, N, 1, 0.0, hi, st) == 0
    else:
        split = 3 if producer.startswith("split") else 1
        part = torch.empty(rows * N * split, device="cuda:0")
        assert et.et_debug_conv3x3_split(p(x), p(w), p(y), p(z), batch, H, W, C, N, p(shift), p(gain), 0, 3, split, p(part), 23 if "ring" in producer else 17, st) == 0
    ws = torch.empty(et.et_debug_affine_back_ws_floats(rows, N), device="cuda:0")
    assert et.et_debug_affine_back(p(d), 0, 0, p(z), 0, p(gain), p(shift), p(m), 0, 0, 0, p(ws), hi, 1, rows, N, st) == 0
    torch.cuda.synchronize()
    yf = y.float()
    is_open = (yf > 0) & (yf < hi)
    assert 0.2 < is_open.float().mean().item() < 0.8
    assert torch.equal(m, torch.where(is_open, d, torch.zeros_like(d)))


def test_affine_back_rejects():
    import torch
    from paper_2312_14227_amd import binding as et
    t = torch.zeros(4096, device="cuda:0")
    p = t.data_ptr()
    call = lambda **k: et.et_debug_affine_back(*(k.get(n, 0) for n in "d add y z z32 gain shift dmid dout total mul".split()), p, 6.0, k.get("f", 0),
                                               k.get("rows", 2), k.get("cols", 8))
    assert call(d=p, dmid=p) == 0
    torch.cuda.synchronize()
    for bad in (dict(d=p), dict(dmid=p), dict(d=p, dmid=p, cols=12), dict(d=p, dmid=p, rows=0), dict(d=p, mul=p), dict(d=p, dout=p),
                dict(d=p, dmid=p, f=1, z=p), dict(d=p, dmid=p, z=p, z32=p), dict(d=p + 2, dmid=p)):
        assert call(**bad) == -1


def test_mirrored_weights():
    """Blocks of 64 x 64 channels with remainders in either direction, several weights in a launch and more than a launch holds."""
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(1)
    shapes = [(64, 64), (8, 8), (72, 200), (128, 56), (64, 136)] + [(8, 16)] * 120
    ws = [torch.randn(o, 9, c, generator=gen).bfloat16() for o, c in shapes]
    wt = [w.to("cuda:0") for w in ws]
    out = [torch.full((c, 9, o), float("nan"), device="cuda:0", dtype=torch.bfloat16) for o, c in shapes]
    call = lambda O, Cs: et.et_debug_flip3x3([w.data_ptr() for w in wt], [t.data_ptr() for t in out], O, Cs, torch.cuda.current_stream().cuda_stream)
    assert call([o for o, _ in shapes], [c for _, c in shapes]) == 0
    torch.cuda.synchronize()
    for w, t in zip(ws, out):
        assert torch.equal(t.cpu(), w.flip(1).permute(2, 1, 0))
    assert call([4] * len(shapes), [c for _, c in shapes]) == -1
