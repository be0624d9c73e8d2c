"""A context is bound to as much workspace as the caller has: the least is what a pass needs whose weight gradients run one at a time, and with
less than it can use a pass runs some of them by themselves and the others in more and smaller groups.  Loss and gradients are compared bit for bit
with those of the whole workspace, and of a pass whose kernels are timed, which runs every weight gradient by itself, plain or gathered;
nothing is written beyond the workspace that was given.  One model has more gradients than a group takes."""
import numpy as np
import pytest

from paper_2312_14227_amd import binding as et
from synth import CONFIGS
from synth.configs import MobileNetConfig, ResNetConfig, ViTConfig

# bytes that sufficed when every weight gradient ran by itself
SUFFICED = {"vit_b": 4639113472, "vit_l": 5944913920, "vgg16": None, "mlp": None}


def _ctx(cfg):
    from paper_2312_14227_amd.session import desc_from_config
    return et.et_create(desc_from_config(cfg))


@pytest.mark.parametrize("name", SUFFICED)
def test_what_sufficed_suffices(name):
    ctx = _ctx(CONFIGS[name])
    least, most = et.et_workspace_min_bytes(ctx), et.et_workspace_bytes(ctx)
    if SUFFICED[name] is None:
        assert least == most          # (these keep no gradients)
    else:
        assert least <= SUFFICED[name] < most
    with pytest.raises(et.EtError) as e:
        n = et.et_num_tensors(ctx)
        et.et_bind(ctx, [4096] * n, None, [4096] * n, 4096, least - 1)
    assert e.value.status == et.ET_ENOMEM
    et.et_destroy(ctx)


MODELS = {
    "transformer": ViTConfig("room_vit", 24, 65, 96, 256, 4, 512, 4, 24),
    "transformer_131_weights": ViTConfig("room_many", 3, 20, 64, 64, 1, 128, 33, 16),
    "unfused_attention": ViTConfig("room_dh32", 2, 40, 64, 128, 4, 256, 3, 16),
    "resnet": ResNetConfig("room_resnet", 4, 64, 3, 64, (2, 2, 1), (64, 64, 128), 24),
    "mobilenet": MobileNetConfig("room_mobile", 4, 64, 3, 16, ((1, 16, 1, 1), (6, 24, 2, 2), (6, 32, 2, 2)), 64, 24),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", MODELS)
def test_the_same_bits_with_any_room(name):
    import torch
    from paper_2312_14227_amd.session import Session
    from synth import make_workload
    cfg = MODELS[name]
    wl = make_workload(cfg, seed=2, init="random")
    N = len(wl.weights)
    s = Session(cfg, wl.weights, with_state=False)
    xt, yt = s.put_input(wl.x, wl.y)
    least, most = et.et_workspace_min_bytes(s.ctx), et.et_workspace_bytes(s.ctx)
    assert least < most == s.ws_bytes
    rng = np.random.default_rng(7)
    masks = [np.ones(N, np.uint8)] + [(rng.random(N) < p).astype(np.uint8) for p in (0.3, 0.7)]

    def run(room, timed=False):
        at = s.ws_ptr - s.ws.data_ptr()
        s.ws.fill_(0xFF)                                    # (NaNs: nothing beyond the least is cleared)
        et.et_bind(s.ctx, [w.data_ptr() for w in s.w], None, [g.data_ptr() for g in s.grad], s.ws_ptr, room)
        if timed:
            et.et_kernel_timing(s.ctx, 1)
        out, launches = [], []
        for m in masks:
            for g in s.grad:
                g.fill_(float("nan"))
            loss = s.train_step(xt, yt, m)
            out.append([torch.tensor(loss)] + [s.grad[i].clone() for i in range(N) if m[i]])
            launches.append(s.launch_counts()[1])
        if timed:
            et.et_kernel_timing(s.ctx, 0)
        assert bool((s.ws[at + room:] == 0xFF).all())       # nothing beyond what was given
        return out, launches

    want, fewest = run(most)
    alone, each = run(most, timed=True)
    rooms = [least, least + 256] + [least + int((most - least) * f) for f in (0.03, 0.1, 0.25, 0.5, 0.8, 0.97)] + [most - 256]
    counts = []
    for got, launches in [(alone, each)] + [run(r) for r in rooms]:
        for a, b in zip(want, got):
            assert len(a) == len(b) and all(torch.equal(x.cpu(), y.cpu()) and bool(torch.isfinite(x).all()) for x, y in zip(a, b))
        counts.append(launches[0])
    assert fewest[0] < counts[1] <= counts[0]               # (the least room: hardly any gradient finds a place)
    assert any(fewest[0] < n < counts[1] for n in counts)   # (some run by themselves, some in groups)
    s.close()
