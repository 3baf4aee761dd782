"""The FP32 encoder on 32 x 32 inputs: its forward equals the general convolutions bit
for bit (a caller's image that is only 4-byte aligned still takes those), and on small
integers, where every FP32 sum is exact, forward and backward equal float64
convolutions."""
import pytest
import torch
import torch.nn.functional as F

from oracle import layout as olayout
from tests import helpers as H

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api

SIDE, CH = 32, 9


def _layers(flat):
    tab, _ = olayout.offsets(olayout.dims(**H.cfg("full32")))
    cut = lambda t: flat[t[0]:t[0] + torch.Size(t[1]).numel()].double().cpu().reshape(t[1])
    return [(cut(tab[f"enc.conv{i}.W"]), cut(tab[f"enc.conv{i}.b"])) for i in (1, 2, 3)], tab


@pytest.mark.parametrize("n", [1, 2, 37, 257])
def test_forward_equals_general_path(n):
    print(f"encoder32 forward n={n}", flush=True)
    cfg = H.cfg("full32")
    gen = torch.Generator().manual_seed(n)
    end = olayout.blocks(olayout.dims(**cfg))["enc"][1]
    p = (torch.randn(end, generator=gen) * 0.1).cuda()
    size = n * CH * SIDE * SIDE
    store = torch.zeros(size + 1, device="cuda")
    x = torch.rand((n, CH, SIDE, SIDE), generator=gen).cuda()
    off = store[1:].view(x.shape)
    off.copy_(x)
    want = api.encoder_fwd_noalloc(cfg, 0, p, off)   # 4-byte aligned: the general convolutions
    assert torch.equal(api.encoder_fwd_noalloc(cfg, 0, p, x), want)
    assert torch.equal(api.encoder_fwd(cfg, 0, p, x)[0], want)


@pytest.mark.parametrize("n", [1, 3, 65])
def test_integers_are_exact(n):
    print(f"encoder32 integers n={n}", flush=True)
    cfg = H.cfg("full32")
    gen = torch.Generator().manual_seed(100 + n)
    end = olayout.blocks(olayout.dims(**cfg))["enc"][1]
    ints = lambda lo, hi, *s: torch.randint(lo, hi + 1, s, generator=gen).float()
    flat = ints(-1, 1, end)
    x = ints(0, 3, n, CH, SIDE, SIDE)
    layers, tab = _layers(flat)
    ws = [(W.requires_grad_(), b.requires_grad_()) for W, b in layers]
    h = x.double()
    for i, (W, b) in enumerate(ws):
        h = F.relu(F.conv2d(h, W, b, stride=2 if i == 0 else 1))
    feat, wsp = api.encoder_fwd(cfg, 0, flat.cuda(), x.cuda())
    assert torch.equal(feat.cpu().double(), h.detach().reshape(n, -1))
    d = ints(-1, 1, *h.shape) * (ints(0, 7, *h.shape) == 0)
    h.backward(d.double())
    g = api.encoder_bwd(cfg, 0, flat.cuda(), wsp, d.reshape(n, -1).contiguous().cuda(), end).cpu().double()
    for i, (W, b) in enumerate(ws):
        for nm, t in (("W", W), ("b", b)):
            o = tab[f"enc.conv{i + 1}.{nm}"][0]
            assert W.grad.abs().max() < 2 ** 24
            assert torch.equal(g[o:o + t.numel()], t.grad.reshape(-1)), (i, nm)
