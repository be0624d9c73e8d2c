"""Attention with few (batch, head) items, where two workgroups share one, bit for bit against the same heads among many, where each has its own: the
forward pass splits the query tiles (more than four of them), the backward pass its two passes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 33, 100, 128, 129, 160, 197, 224])
def test_shared_items_give_the_same_bits(T):
    import torch
    from paper_2312_14227_amd import binding as et
    gen = torch.Generator().manual_seed(T)
    H, many = 3, 44                                     # 132 items: one workgroup each; 3 and 126: two
    D = 64 * H
    qkv = torch.randn(many, T, 3 * D, generator=gen).bfloat16().to("cuda:0")
    dout = torch.randn(many, T, D, generator=gen).bfloat16().to("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream

    def run(B):
        out = torch.full((B, T, D), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        lse = torch.full((B, H, T), float("nan"), device="cuda:0")
        dqkv = torch.full((B, T, 3 * D), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        p = lambda t: t.data_ptr()  # noqa: E731
        assert et.et_debug_attention(0, p(qkv), p(out), p(lse), 0, 0, B, T, H, stream) == 0
        assert et.et_debug_attention(1, p(qkv), p(out), p(lse), p(dout), p(dqkv), B, T, H, stream) == 0
        torch.cuda.synchronize()
        return out, lse, dqkv

    full = run(many)
    for B in (1, 42):
        for a, b in zip(run(B), full):
            assert torch.equal(a, b[:B])
