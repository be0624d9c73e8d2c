"""The fp32 MLP step at sizes around the edges of its 16- and 32-wide tiles and of the four waves' turns over the reduction, against
the oracle: losses and every gradient to 1e-5 (fp32 products and sums)."""
import numpy as np
import pytest

from oracle import nets
from synth import make_workload
from synth.configs import MLPConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch", [((16, 16, 16), 16), ((5, 3, 2), 1), ((67, 131, 33, 10), 37), ((64, 65, 63, 17), 15), ((257, 260, 255, 12), 33),
                                        ((300, 1024, 40, 1000, 7), 19), ((512, 544, 513, 200), 530), ((1024, 1024, 24), 512)])
def test_mlp_step_matches_oracle(dims, batch):
    import torch  # noqa: F401
    from paper_2312_14227_amd.session import Session
    cfg = MLPConfig("mlp_sizes", dims, batch)
    wl = make_workload(cfg, seed=len(dims) + batch)
    ref = nets.step(cfg, wl.weights, wl.x, wl.y, [1] * len(wl.weights))
    s = Session(cfg, wl.weights)
    xt, yt = s.put_input(wl.x, wl.y)
    loss = s.train_step(xt, yt, np.ones(len(wl.weights), dtype=np.uint8))
    assert abs(loss - ref["loss"]) <= 1e-5 * abs(ref["loss"])
    for k, g in enumerate(ref["grads"]):
        err = np.linalg.norm(s.grads_host(k) - g.ravel()) / max(np.linalg.norm(g), 1e-30)
        assert err <= 1e-5, (k, err)
    s.close()
