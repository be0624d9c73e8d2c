"""Column sums that the GELU-backward epilogue leaves over every 32 rows of its result, on every tile that has this epilogue: row counts that
end inside a block of 32, in its first row and on its end, columns that end inside a tile, a wave's columns and a lane's four.
A sum is at most 32 fp32 additions of the stored bf16 values, error below 32 * 2^-24 of the sum of their magnitudes; rows and
columns beyond are not written."""
import pytest

pytestmark = pytest.mark.gpu

TILES = {"staged 128x128": 1, "staged 128x64": 3, "direct 256x256": 5, "direct 256x128": 7, "two-group 256x256": 11, "two-group 256x192": 13,
         "ring 64x64": 23, "ring 64x128": 25, "ring 128x128": 29, "planned": 0}


@pytest.mark.parametrize("tile", TILES, ids=[t.replace(" ", "_") for t in TILES])
@pytest.mark.parametrize("M,N", [(1, 8), (33, 72), (64, 200), (97, 264), (300, 392), (530, 520)])
def test_column_sums_of_the_gelu_backward_epilogue(M, N, tile):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(M + N)
    K = 128
    dev = lambda a: a.bfloat16().to("cuda:0")
    A, B, aux = dev(torch.randn(M, K, generator=gen)), dev(torch.randn(K, N, generator=gen)), dev(torch.rand(M, N, generator=gen))
    out = torch.full((M, N), float("nan"), device="cuda:0", dtype=torch.bfloat16)
    parts = (M + 31) // 32
    sums = torch.full((parts + 1, N), float("nan"), device="cuda:0")
    p = lambda t: t.data_ptr()
    assert et.et_debug_gemm_bf16_colsum(p(A), p(B), p(out), p(aux), p(sums), M, N, K, K, N, N, TILES[tile], torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    got = out.double().cpu()
    ref = (A.double() @ B.double() * aux.double()).cpu()
    scale = (A.double().abs() @ B.double().abs() * aux.double()).cpu()
    assert torch.all((got - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -23 * scale)
    padded = torch.zeros(parts * 32, N, dtype=torch.float64)
    padded[:M] = got
    blocks = padded.view(parts, 32, N)
    err = (sums[:parts].double().cpu() - blocks.sum(1)).abs()
    assert torch.all(err <= 32 * 2.0 ** -24 * blocks.abs().sum(1) + 1e-30)
    assert torch.all(torch.isnan(sums[parts]))
