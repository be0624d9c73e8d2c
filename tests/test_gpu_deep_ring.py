"""The 64 x 64 ring tile with five slices in flight, taken by products of at most one tile per CU and 32 slices or more (36 where the second operand is
transposed): reductions of these lengths and around them, with whole and ragged ends, in every layout and epilogue that has it (the affine ones in
test_gpu_act_epilogues.py).  References and bounds are those of the other tiles' tests."""
import pytest

from test_gpu_gemm import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(64, 64, 2048), (3, 8, 2056), (130, 72, 2111), (200, 136, 2049), (197, 64, 4100), (500, 330, 2304), (72, 136, 3072), (130, 64, 3073)])
def test_deep_ring(M, N, K):
    for a_t, b_t in ((0, 0), (0, 1)):
        _run(M, N, K, a_t, b_t, 0, True, False, 1, 23, seed=M + N + K)
        _run(M, N, K, a_t, b_t, 1, True, a_t == 0 and b_t == 0, 1, 23, seed=M + K)
