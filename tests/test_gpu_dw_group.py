"""Weight gradients in a group (one launch for many) against float64 products of the same bf16 inputs, and bit for bit against the same gradients
run one at a time with the same split: what a gradient is does not depend on what runs beside it.  Groups of few and many jobs, of one
kind and mixed, with one to many chunks of one to many slices and ragged sizes of everything; enough large ones for the resident tiles to
take several units each, and more jobs than one launch takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PLAIN = [(8, 8, 1, 1), (16, 24, 63, 1), (72, 40, 64, 1), (64, 200, 65, 1), (136, 72, 500, 2), (264, 520, 130, 1), (96, 16, 5000, 19), (64, 64, 9000, 40)]
CONV = [(64, 1, 1, 3, 8, 3, 1, 1), (72, 2, 5, 7, 64, 3, 1, 1), (40, 3, 13, 12, 24, 3, 2, 2), (64, 2, 9, 9, 64, 1, 2, 1), (128, 4, 25, 25, 64, 3, 1, 7)]   # out, batch, H, W, C, taps, stride, split
LARGE = [(768, 768, 1000, 1), (1000, 520, 777, 3), (256, 1536, 640, 2), (2304, 768, 833, 1), (300, 264, 64, 1), (1536, 2000, 200, 1)]
GROUPS = {"one_small": PLAIN[:1], "small": PLAIN, "gathered": CONV, "large": LARGE, "large_many": LARGE * 5, "mixed": PLAIN + CONV + LARGE,
          "more_than_a_launch": [PLAIN[1 + i % 5] for i in range(100)], "gathered_many": [CONV[i % 4] for i in range(50)]}


def _job(shape, gen):
    import torch
    if len(shape) == 4:
        M, N, K, split = shape
        A, B = torch.randn(K, M, generator=gen), torch.randn(K, N, generator=gen)
        return (M, N, K, split, 0, 0, 0, 0, 0), A, B, B
    M, batch, H, W, Cin, taps, stride, split = shape
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    K, N = batch * Ho * Wo, taps * taps * Cin
    A, x = torch.randn(K, M, generator=gen), torch.randn(batch, H, W, Cin, generator=gen)
    pad = taps // 2
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    cols = torch.stack([xp[:, ky:ky + stride * Ho:stride, kx:kx + stride * Wo:stride][:, :Ho, :Wo] for ky in range(taps) for kx in range(taps)], dim=3)
    return (M, N, K, split, H, W, Cin, taps, stride), A, x, cols.reshape(K, N)


@pytest.mark.parametrize("name", GROUPS)
def test_group_of_weight_gradients(name):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(len(GROUPS[name]))
    stream = torch.cuda.current_stream().cuda_stream
    shapes, dev, refs, scales = [], [], [], []
    for s in GROUPS[name]:
        shape, A, B, cols = _job(s, gen)
        M8, N8 = (shape[0] + 7) // 8 * 8, (shape[1] + 7) // 8 * 8
        A, B, cols = A.bfloat16(), B.bfloat16(), cols.bfloat16()
        a, c = A.double(), cols.double()
        refs.append(a.T @ c)
        scales.append(a.abs().T @ c.abs())
        pad = lambda t, n: torch.nn.functional.pad(t, (0, n - t.shape[-1]))  # noqa: E731
        dev.append((pad(A, M8).to("cuda:0"), (pad(B, N8) if shape[6] == 0 else B).contiguous().to("cuda:0")))
        shapes.append(shape)
    out = [torch.full((s[0] + 1, s[1]), float("nan"), device="cuda:0") for s in shapes]
    elems = sum(s[0] * s[1] * s[3] for s in shapes)
    part = torch.full((elems,), float("nan"), device="cuda:0")
    p = lambda t: t.data_ptr()  # noqa: E731
    run = lambda idx, o: et.et_debug_dw_group([p(dev[i][0]) for i in idx], [p(dev[i][1]) for i in idx], [p(t) for t in o], [shapes[i] for i in idx],  # noqa: E731
                                              p(part), elems, stream)
    assert run(range(len(shapes)), out) == 0
    torch.cuda.synchronize()
    for i, (s, o) in enumerate(zip(shapes, out)):
        assert torch.isnan(o[s[0]]).all()                              # nothing beyond the result
        err = (o[:s[0]].double().cpu() - refs[i]).abs()
        assert torch.all(err <= 2e-6 * np.sqrt(s[2]) * scales[i] + 1e-6), (s, float(err.max()))
    for i in list(range(len(shapes)))[:24]:
        alone = torch.full_like(out[i], float("nan"))
        s = shapes[i]
        assert run([i], [alone]) == 0
        torch.cuda.synchronize()
        assert torch.equal(alone[:s[0]], out[i][:s[0]]), s
        if s[6] == 0:                                                  # the product on its own
            M8, N8 = (s[0] + 7) // 8 * 8, (s[1] + 7) // 8 * 8
            single = torch.full_like(out[i], float("nan"))
            assert et.et_debug_gemm_bf16(p(dev[i][0]), p(dev[i][1]), p(single), s[0], s[1], s[2], M8, N8, s[1], 1, 1, 1, 1.0, 0, 0, s[3], p(part), 0,
                                         stream) == 0
            torch.cuda.synchronize()
            assert torch.equal(single[:s[0]], out[i][:s[0]]), s


def test_group_refuses_what_its_kernels_do_not_take():
    import torch
    from paper_2312_14227_amd import binding as et
    t = torch.zeros(4096, device="cuda:0", dtype=torch.bfloat16)
    o = torch.zeros(4096, device="cuda:0")
    p = t.data_ptr()
    ok = (16, 16, 16, 1, 0, 0, 0, 0, 0)
    for bad in ((16, 18, 16, 1, 0, 0, 0, 0, 0), (0, 16, 16, 1, 0, 0, 0, 0, 0), (16, 16, 16, 0, 0, 0, 0, 0, 0), (16, 72, 16, 1, 4, 4, 9, 3, 1), (16, 72, 17, 1, 4, 4, 8, 3, 1)):
        assert et.et_debug_dw_group([p], [p], [o.data_ptr()], [bad], o.data_ptr(), 4096) == et.ET_EINVAL
    assert et.et_debug_dw_group([p + 2], [p], [o.data_ptr()], [ok], o.data_ptr(), 4096) == et.ET_EINVAL
    assert et.et_debug_dw_group([p], [p], [o.data_ptr()], [(16, 16, 512, 8, 0, 0, 0, 0, 0)], o.data_ptr(), 100) == et.ET_EINVAL
