"""Frames at any alignment that the encoder's own launch reads (raw: words, a ring's:
bytes), and at one that it leaves to the separate launches, give the bits of aligned
frames."""
import pytest
import torch

from paper_2602_21203_amd import synthetic
from tests import helpers as H
from tests.test_gpu_encoder_frames import _shifted

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api


@pytest.mark.parametrize("stored,offsets", [(False, (4, 12, 2)), (True, (1, 2, 4, 13))])
def test_update(stored, offsets):
    print(f"update frames stored={stored}", flush=True)
    cfg, B, cap = H.cfg("full"), 100, 256
    rep = synthetic.replay(cap, cfg["H"], cfg["W"], cfg["C"], cfg["proprio"], cfg["action"], seed=3, device="cuda")
    if stored:   # the block means, as a ring holds them
        side = cfg["H"] // cfg["k"]
        for f in ("obs", "next_obs"):
            m = rep[f].view(cap, side, cfg["k"], side, cfg["k"], cfg["C"]).float().mean((2, 4))
            rep[f] = m.round().to(torch.uint8).contiguous()
    want = None
    for by in (0, *offsets):
        ag = api.Agent(cfg, torch.tensor(H.params("full"), dtype=torch.float32, device="cuda"), B, prec=1, seed=7)
        r = {k: _shifted(v, by) if k in ("obs", "next_obs") else v for k, v in rep.items()}
        view = api.Ring.__new__(api.Ring)   # a view of these buffers, as a ring gives one
        view.view = api.replay_struct(r)
        view.view.squinted = int(stored)
        stats = ag.sac_update(view, 3).clone()
        torch.cuda.synchronize()
        got = (stats, ag.params.clone(), ag.target.clone(), ag.grads.clone())
        ag.close()
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), by


@pytest.mark.parametrize("n", [1, 700])
def test_act(n):
    print(f"act frames n={n}", flush=True)
    cfg = H.cfg("full")
    ag = api.Agent(cfg, torch.tensor(H.params("full"), dtype=torch.float32, device="cuda"), 64, prec=1, seed=7)
    frames = synthetic.frames(n, cfg["H"], cfg["W"], cfg["C"], seed=n, device="cuda")
    prop = torch.randn((n, cfg["proprio"]), device="cuda")
    want = ag.act(frames, prop, sample=True, request_id=5)
    for by in (4, 12, 2):
        assert torch.equal(want, ag.act(_shifted(frames, by), prop, sample=True, request_id=5)), by
