"""Batches of the act() server that are admitted together run at once on the device,
however short they are: each one's first work is enqueued before any one's last."""
import pytest
import torch

from paper_2602_21203_amd import synthetic
from tests import helpers as H

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api


@pytest.mark.parametrize("name", ["full", "state_tiny"])
def test_batches_admitted_together_overlap(name):
    print(f"server overlap {name}", flush=True)
    cfg, slots, rows = H.cfg(name), 3, 4
    agent = api.Agent(cfg, H.params(name), 32, prec=1)
    frames = synthetic.frames(slots * rows, cfg["H"], cfg["W"], cfg["C"], seed=4, device="cuda")
    prop = torch.randn(slots * rows, cfg["proprio"], device="cuda")
    part = lambda t, i: t[rows * i:rows * (i + 1)]
    want = [agent.act(part(frames, i), part(prop, i), sample=True, request_id=i) for i in range(slots)]
    torch.cuda.synchronize()
    srv = api.Server(agent, mem_budget=1 << 30, max_batch_obs=rows, n_slots=slots)   # a request fills a batch
    for k in range(1, 6):
        srv.hold(True)
        outs = [srv.submit(part(frames, i), part(prop, i), i, sample=True) for i in range(slots)]
        srv.hold(False)
        srv.drain()
        torch.cuda.synchronize()
        st = srv.stats()
        print("  server stats:", st, flush=True)
        assert st["batches"] == slots * k and st["max_slots_busy"] == slots
        assert st["overlapped_batches"] == (slots - 1) * k
        for a, b in zip(want, outs):
            assert torch.equal(a, b)
    srv.close()
    agent.close()
