"""The streaming attention kernels against the oracle's definition: one and several chunks of 64 rows and blocks of 128 own rows, ragged
ends of both, fewer (batch, head) items than the 8 shares of the grid and more."""
import numpy as np
import pytest

from gpu_util import rel_l2
from oracle import attention as oatt
from test_gpu_attention import _bf16

pytestmark = pytest.mark.gpu


def _run(B, T, H, seed, q_gain=1.0):
    import torch
    from paper_2312_14227_amd import binding as et
    D = 64 * H
    rng = np.random.default_rng(seed)
    qkv = rng.standard_normal((B, T, 3 * D))
    qkv[..., :D] *= q_gain
    qkv_t, dout_t = _bf16(qkv).cuda(), _bf16(rng.standard_normal((B, T, D))).cuda()
    out_t = torch.full((B, T, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse_t = torch.full((B, H, T), float("nan"), dtype=torch.float32, device="cuda")
    dqkv_t = torch.full((B, T, 3 * D), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert et.et_debug_attention_long(0, qkv_t.data_ptr(), out_t.data_ptr(), lse_t.data_ptr(), 0, 0, B, T, H) == 0
    assert et.et_debug_attention_long(1, qkv_t.data_ptr(), out_t.data_ptr(), lse_t.data_ptr(), dout_t.data_ptr(), dqkv_t.data_ptr(), B, T, H) == 0
    torch.cuda.synchronize()
    qkv64 = qkv_t.float().cpu().numpy().astype(np.float64)
    dout64 = dout_t.float().cpu().numpy().astype(np.float64)
    out_ref, lse_ref, _ = oatt.attention_forward(qkv64, H)
    g_ref = oatt.attention_backward(qkv64, dout64, H)
    # one bf16 rounding of the probabilities and one of the results, as in the on-chip kernels' tests
    out, lse, g = out_t.float().cpu().numpy(), lse_t.cpu().numpy(), dqkv_t.float().cpu().numpy()
    assert np.isfinite(out).all() and np.isfinite(lse).all() and np.isfinite(g).all()
    assert rel_l2(out, out_ref) <= 6e-3, rel_l2(out, out_ref)
    np.testing.assert_allclose(lse, lse_ref, rtol=0, atol=2e-5 * max(1.0, np.abs(lse_ref).max()))
    for i, name in enumerate(("dq", "dk", "dv")):
        a, b = g[..., i * D:(i + 1) * D], g_ref[..., i * D:(i + 1) * D]
        if T == 1 and i < 2:
            assert np.abs(a).max() <= 1e-6 * np.abs(g_ref).max(), name
            continue
        assert rel_l2(a, b) <= 1e-2, (name, rel_l2(a, b))


@pytest.mark.parametrize("B,T,H", [(1, 1, 1), (2, 63, 3), (1, 64, 9), (3, 65, 1), (1, 127, 2), (2, 128, 4), (1, 129, 1), (2, 225, 3), (1, 256, 2), (1, 257, 2),
                                   (2, 577, 2), (1, 1000, 1)])
def test_streaming_attention_matches_the_definition(B, T, H):
    _run(B, T, H, seed=T + B)


def test_streaming_attention_with_rising_scores():
    # score standard deviation 4: the running maximum moves several times per row
    _run(2, 400, 2, seed=5, q_gain=4.0)
