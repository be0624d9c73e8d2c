"""The two-group tiles that load their operands straight to LDS (256 x 256, 192 x 256, 128 x 256): one to many slices of 64, so that the requests run ahead
into the same tile, the workgroup's next one and the one after that; ragged rows and columns; more tiles than CUs; split reductions with a shorter
last chunk; every epilogue (those with an activation that is no GELU in test_gpu_act_epilogues.py).  References and bounds are those of the other tiles' tests."""
import pytest

from test_gpu_gemm import _run
from test_gpu_gemm import test_gemm_gelu_epilogues as gelu_epilogues
from test_gpu_gemm_colsum import TILES
from test_gpu_gemm_colsum import test_column_sums_of_the_gelu_backward_epilogue as column_sums

pytestmark = pytest.mark.gpu

DIRECT = [11, 13, 15]


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(3, 8, 64), (192, 256, 128), (256, 256, 192), (257, 264, 256), (193, 510, 320), (700, 520, 704)])
def test_direct_tile(M, N, K, a_t, b_t, tile):
    _run(M, N, K, a_t, b_t, 1, True, a_t == 0 and b_t == 0, 1, tile, seed=tile + M)
    _run(M, N, K, a_t, b_t, 0, True, False, 1, tile, seed=tile + N)


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("K", [64, 128, 192])
def test_direct_tile_several_units_per_workgroup(K, tile):
    """More tiles than CUs: short reductions, where a request is up to two tiles ahead of the multiplication."""
    _run(5000, 5200, K, 0, 0, 1, True, True, 1, tile, seed=K)
    _run(5000, 5200, K, 1, 1, 0, True, False, 1, tile, seed=K + 1)


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("M,N,K,split", [(768, 520, 4992, 6), (1536, 2000, 64 * 23, 7), (260, 256, 64 * 9, 2), (264, 512, 64 * 9 + 8, 2), (520, 264, 1000, 3),
                                           (256, 256, 4097, 5)])
def test_direct_tile_split_reduction(M, N, K, split, tile):
    _run(M, N, K, 1, 1, 1, False, False, split, tile, seed=split)


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("M,N,K", [(700, 520, 192), (513, 300, 128), (77, 136, 64)])
def test_direct_tile_gelu(M, N, K, tile):
    gelu_epilogues(M, N, K, tile)


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("M,N", [(1, 8), (33, 72), (97, 264), (530, 520)])
def test_direct_tile_column_sums(M, N, tile, monkeypatch):
    monkeypatch.setitem(TILES, "direct", tile)
    column_sums(M, N, "direct")


@pytest.mark.parametrize("tile", DIRECT)
@pytest.mark.parametrize("K", [1, 63, 65, 130, 191, 1000])
def test_direct_tile_weight_gradient_over_any_number_of_rows(K, tile):
    """The last slice of a reduction over rows holds zeros beyond them; with more tiles than CUs every tile has one."""
    _run(264, 520, K, 1, 1, 1, True, False, 1, tile, seed=K)
    if K == 65:
        _run(4500, 5200, K, 1, 1, 1, False, False, 1, tile, seed=K)
