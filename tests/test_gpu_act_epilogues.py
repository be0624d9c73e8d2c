"""Bias + ReLU, affine + clamp and affine + second branch + clamp as epilogues of plain products, on the tiles that load their operands straight to LDS (256 x 256, 192 x
256, 128 x 256), on the 64 x 64 ring tile with three and with five slices in flight, and on the tile that the sizes take: against float64 of the same bf16
inputs, and bit for bit against the register-staged tile, whose sums run in the same order.  Whole tiles, ragged rows and columns, leading dimensions and
alignments that allow no 16-byte access, several units per workgroup, z stored and not, the second branch with and without a gain of its own."""
import pytest

pytestmark = pytest.mark.gpu

DIRECT, RING, STAGED = [11, 13, 15], 23, 1
SIZES = [(3, 8, 64, 8), (256, 256, 128, 256), (257, 264, 192, 264), (193, 508, 256, 508), (520, 772, 320, 776), (700, 516, 64, 516)]


def _run(M, N, K, ldc, kind, tile, shift=0):
    """kind: "bias", "affine", "affine_z", "add", "add_z", "add_gain_z"; shift: elements by which y and U miss a 16-byte boundary"""
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(M + N + K)
    r = lambda *s: torch.randn(*s, generator=gen).bfloat16()  # noqa: E731
    A, B, bias, gain, gain2, bias2, U = r(M, K), (r(N, K) * K ** -0.5).bfloat16(), r(N), r(N), r(N), r(N), r(M, ldc)
    dev = lambda t: t.to("cuda:0").contiguous()  # noqa: E731
    a, b = dev(A), dev(B)
    acc, scale = A.double() @ B.double().T, A.double().abs() @ B.double().abs().T
    vec = [dev(t) for t in (bias, gain, gain2, bias2)]

    def place(fill, shift):   # [M][ldc] `shift` elements behind a 16-byte boundary, with a guard row behind it
        flat = torch.full((shift + (M + 1) * ldc,), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        if fill is not None:
            flat[shift:shift + M * ldc] = fill.to("cuda:0").reshape(-1)
        return flat, flat[shift:shift + M * ldc].view(M, ldc)

    def call(t):
        zf, z = place(None, 0)
        yf, y = place(None, shift)
        _, u = place(U, shift)
        affine, add = kind != "bias", kind.startswith("add")
        p = lambda t_, on=True: t_.data_ptr() if on else 0  # noqa: E731
        own = "gain" in kind
        rc = et.et_debug_gemm_bf16_act(a.data_ptr(), b.data_ptr(), p(z, kind.endswith("z")), p(y), M, N, K, K, K, ldc, p(vec[0]), p(vec[1], affine), p(u, add),
                                       p(vec[2], own), p(vec[3], own), -0.5 if affine else 0.0, 2.0 if affine else 0.0, t, torch.cuda.current_stream().cuda_stream)
        assert rc == 0, (rc, t)
        torch.cuda.synchronize()
        for flat, body, at, used in ((zf, z, 0, kind.endswith("z")), (yf, y, shift, True)):   # nothing in front, behind, or beyond the N columns
            assert torch.isnan(flat[:at]).all() and torch.isnan(flat[at + M * ldc:]).all() and torch.isnan(body[:, N:]).all()
            assert used or torch.isnan(body).all()
        return z[:, :N].clone(), y[:, :N].clone()

    z, y = call(tile)
    err = 2e-6 * scale * K ** 0.5 + 1e-6          # fp32 sums of exact products
    if kind == "bias":
        want, slack = (acc + bias.double()).clamp_min(0), err
    else:
        if kind.endswith("z"):
            assert ((z.cpu().double() - acc).abs() <= err + 2.0 ** -8 * acc.abs()).all()
        # y from z as rounded: up to a rounding of z away from the product, and of fp32 arithmetic
        want, slack = acc * gain.double() + bias.double(), (err + 2.0 ** -8 * acc.abs()) * gain.double().abs()
        if kind.startswith("add"):
            want = want + (U[:, :N].double() * gain2.double() + bias2.double() if "gain" in kind else U[:, :N].double())
        slack = slack + 1e-6 * (want.abs() + acc.abs() + 4)
        want = want.clamp(-0.5, 2.0)
    assert ((y.cpu().double() - want).abs() <= slack + 2.0 ** -8 * want.abs()).all()
    z1, y1 = call(STAGED)
    assert torch.equal(y, y1) and (not kind.endswith("z") or torch.equal(z, z1))


KINDS = ["bias", "affine", "affine_z", "add", "add_z", "add_gain_z"]


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("kind", KINDS)
def test_direct_tiles(kind, tile):
    for M, N, K, ldc in SIZES:
        _run(M, N, K, ldc, kind, tile)
    if kind != "bias":   # (the first output is 16-byte aligned)
        _run(257, 264, 192, 272, kind, tile, shift=4)
        _run(512, 512, 64, 512, kind, tile, shift=4)


@pytest.mark.parametrize("kind", ["affine_z", "add_gain_z"])
def test_direct_tiles_several_units_per_workgroup(kind):
    _run(5000, 5204, 128, 5204, kind, 15)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("M,N,K", [(64, 64, 2048), (130, 72, 2112), (200, 136, 2056), (500, 332, 2304)])
def test_ring_tile_with_five_slices_in_flight(M, N, K, kind):
    _run(M, N, K, N, kind, RING)
    _run(M, N, 256, N, kind, RING)     # (three)


@pytest.mark.parametrize("kind", ["affine_z", "add_z"])
def test_sizes_that_take_the_direct_tiles_by_themselves(kind):
    """1 x 1 convolutions of 32 images of 256 x 256 in a 50-layer residual network: 8.6 GFLOP each."""
    _run(32768, 256, 512, 256, kind, 0)
    _run(8192, 512, 1024, 512, kind, 0)
