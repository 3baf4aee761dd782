"""Calls large enough for the pairs of products on the 64 x 64 tile: the twin critics on
2,001 rows (input and weight gradient of a layer in one launch) and on 5,800 (the
k-concatenated first-layer gradient), updates whose forward pairs fill the chip.  A row's
results equal those of the same row in a small call bit for bit; gradients of parameters
are the sum of the small calls'; bfloat16 updates with and without operand copies agree
bit for bit; FP32 updates match the oracle."""
import pytest
import torch

from oracle import layout as olayout
from tests import helpers as H
from tests.test_gpu_bf16_copies import _run
from tests.test_gpu_update import test_one_update_matches_oracle as one_update_matches_oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api

STEP = 300   # rows of a small call: at most 2 x 5 x 8 tiles of 64 x 64


@pytest.mark.parametrize("n,prec", [(1100, 0), (2001, 0), (2001, 1), (5800, 0), (5800, 1)])
def test_critic_rows_equal_small_calls(n, prec):
    print(f"large critic n={n} prec={prec}", flush=True)
    cfg = H.cfg("full")
    d = olayout.dims(**cfg)
    c0, c1 = olayout.blocks(d)["critic"]
    p = torch.tensor(H.params("full")[c0:c1], dtype=torch.float32, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    feat, s, a = torch.relu(r(n, 288)), r(n, cfg["proprio"]), torch.tanh(r(n, cfg["action"]))
    dl = 0.1 * r(2, n, cfg["atoms"])
    logits, ws = api.critic_fwd(cfg, prec, p, feat, s, a)
    dp, df, da = api.critic_bwd(cfg, prec, p, ws, dl)
    total = torch.zeros_like(dp, dtype=torch.float64)
    mass = torch.zeros_like(total)
    for i in range(0, n, STEP):
        cut = lambda t: t[i:i + STEP].contiguous()
        lo, w = api.critic_fwd(cfg, prec, p, cut(feat), cut(s), cut(a))
        gp, gf, ga = api.critic_bwd(cfg, prec, p, w, dl[:, i:i + STEP].contiguous())
        assert torch.equal(logits[:, i:i + STEP], lo), i
        assert torch.equal(df[i:i + STEP], gf) and torch.equal(da[i:i + STEP], ga), i
        total += gp.double()
        mass += gp.double() ** 2
    # every parameter's gradient is a sum over the rows of FP32 products (equal terms in both):
    # n additions on either side, each within 2^-24 of a running sum whose size is at most a few
    # times the terms' root of squares (they are of random sign), so norm-wise 2 n 2^-24 sqrt(n)
    # of a row's; a block's squares stand for STEP rows'
    err = (dp.double() - total).norm() / mass.sum().sqrt()
    assert err <= 2 * n * 2.0 ** -24, err


def test_fp32_update_with_large_pairs_matches_oracle():
    one_update_matches_oracle("full", 1500, 2048, 0)


def test_bf16_update_with_large_pairs_equals_one_without_copies():
    print("large update, copies on and off", flush=True)
    out = []
    for copies in (True, False):
        ag, stats, n = _run("full", 1900, 1, copies, n_blocks=1)
        out.append((torch.tensor(stats), ag.params.clone(), ag.target.clone(), ag.grads.clone()))
        ag.close()
        assert (n > 0) == copies
    for x, y in zip(*out):
        assert torch.equal(x, y)
