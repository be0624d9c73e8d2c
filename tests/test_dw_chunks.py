"""Chunks of a weight gradient's reduction.  They decide how many rows one fp32 accumulator adds up, and with that the error of the sum: each
matrix instruction adds 16 rows to the accumulator, whose rounding errors (2^-24 of a running sum that grows with the square root of the rows)
leave about 2^-24 sqrt(rows / 96) of the result for operands of random sign.  A longer chunk is a less precise gradient, whatever runs it."""
import pytest

from paper_2312_14227_amd import binding as et

# M, N, rows: chunks.  Transformers of width 768 (batch 64, 32, 128; 577 tokens), 1024 and 384
CHUNKS = {(2304, 768, 12608): 7, (768, 768, 12608): 3, (3072, 768, 12608): 5, (768, 3072, 12608): 5, (2304, 768, 6304): 8, (768, 768, 6304): 3,
          (3072, 768, 6304): 7, (768, 768, 25216): 21, (3072, 768, 25216): 7, (768, 768, 4616): 3, (3072, 1024, 6304): 5, (4096, 1024, 6304): 4,
          (1024, 4096, 6304): 4, (1152, 384, 6304): 4, (1536, 384, 6304): 3, (768, 768, 788): 1}


@pytest.mark.parametrize("shape", CHUNKS)
def test_chunks_are_no_longer_than_these(shape):
    assert et.et_debug_dw_chunks(*shape) >= CHUNKS[shape]


def test_no_empty_chunk_and_no_split_that_cannot_be_stored():
    for M in (8, 200, 256, 1000, 3072):
        for N in (8, 254, 256, 768, 3000):
            for K in (1, 64, 500, 4096, 6304, 12608, 40000, 401408):
                s, slices = et.et_debug_dw_chunks(M, N, K), (K + 63) // 64
                assert s == 1 or (N % 4 == 0 and -(-slices // -(-slices // s)) == s), (M, N, K, s)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(2304, 768, 12608), (3072, 1024, 6304), (2304, 768, 6304), (768, 768, 4616)])
def test_error_against_64_bits(shape):
    import torch
    M, N, K = shape
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    A, B = (torch.randn(K, n, generator=gen, device="cuda").bfloat16() for n in (M, N))
    ref = A.double().t().contiguous() @ B.double()
    s = et.et_debug_dw_chunks(M, N, K)
    out, part = torch.full((M, N), float("nan"), device="cuda"), torch.empty(s * M * N, device="cuda")
    assert et.et_debug_gemm_bf16(A.data_ptr(), B.data_ptr(), out.data_ptr(), M, N, K, M, N, N, 1, 1, 1, 1.0, 0, 0, s, part.data_ptr(), 0,
                                 torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    # the estimate above for chunks of K / CHUNKS rows, with a quarter for the sum of the chunks
    assert float((out.double() - ref).norm() / ref.norm()) <= 1.25 * 2.0 ** -24 * (K / CHUNKS[shape] / 96) ** 0.5
