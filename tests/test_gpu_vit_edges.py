"""Transformer steps where the last block's gradient covers only the CLS rows, against the oracle over many masks: one block (the CLS rows and
the embedding meet in the same block), two tokens, sequences around the attention kernels' tiles and beyond what fits on chip,
widths between the LayerNorm kernels' register sizes, two blocks whose biases of 3 x width and mlp come from the attention
and matrix kernels over a ragged number of rows, and a head size without a fused attention kernel (dense zero rows)."""
import numpy as np
import pytest

from gpu_util import sample_masks, tol_for
from oracle import nets
from synth import make_workload
from synth.configs import ViTConfig
from test_gpu_step import _check_step, _session

pytestmark = pytest.mark.gpu

#                 batch, tokens, patch_dim, width, heads, mlp, blocks, classes
CASES = {"one_block": (9, 33, 64, 64, 1, 72, 1, 8), "two_tokens": (17, 2, 16, 128, 2, 256, 2, 16), "on_chip_limit": (2, 224, 24, 64, 1, 64, 2, 8),
         "streamed": (2, 257, 24, 128, 2, 136, 1, 8), "streamed_bias_sums": (3, 385, 16, 64, 1, 72, 2, 8), "bias_sums": (9, 193, 16, 128, 2, 200, 2, 8), "width_320": (5, 20, 40, 320, 5, 200, 3, 24), "width_1984": (2, 5, 16, 1984, 31, 64, 1, 8),
         "width_2112": (2, 5, 16, 2112, 33, 64, 1, 8), "heads_of_32": (3, 19, 24, 96, 3, 64, 2, 8)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_last_block_on_cls_rows_matches_oracle(name):
    B, T, P, D, H, F, L, C = CASES[name]
    cfg = ViTConfig(name, B, T, P, D, H, F, L, C)
    wl = make_workload(cfg, seed=B + T, init="random")
    N = len(wl.weights)
    ref = nets.step(cfg, wl.weights, wl.x, wl.y, [1] * N)
    s = _session(cfg, wl)
    xt, yt = s.put_input(wl.x, wl.y)
    rng = np.random.default_rng(T)
    last = 4 + 12 * (L - 1)
    for mask in sample_masks(N, rng, extra=tuple(range(last, last + 12)) + (N - 4, N - 5)):
        _check_step(s, cfg, wl, xt, yt, mask, ref, tol_for(cfg))
    s.close()
