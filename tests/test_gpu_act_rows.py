"""A policy query's rows do not depend on how many share it: few rows, whose products
normalise their own input, equal the same rows of a larger query bit for bit."""
import pytest
import torch

from paper_2602_21203_amd import synthetic
from tests import helpers as H

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api


@pytest.mark.parametrize("n", [1, 2, 5, 15, 16, 17])
@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("name,prec", [("full", 0), ("full", 1), ("full32", 1), ("tiny", 0)])
def test_few_rows_equal_many(name, prec, sample, n):
    print(f"act rows {name} prec={prec} sample={sample} n={n}", flush=True)
    cfg = H.cfg(name)
    ag = api.Agent(cfg, torch.tensor(H.params(name), dtype=torch.float32, device="cuda"), 64, prec=prec, seed=7)
    frames = synthetic.frames(50, cfg["H"], cfg["W"], cfg["C"], seed=n, device="cuda")
    prop = torch.randn((50, cfg["proprio"]), device="cuda")
    many = ag.act(frames, prop, sample=sample, request_id=5)
    few = ag.act(frames[:n].contiguous(), prop[:n].contiguous(), sample=sample, request_id=5)
    assert torch.equal(few, many[:n])
