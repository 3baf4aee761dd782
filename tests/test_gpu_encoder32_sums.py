"""The FP32 encoder backward on 32 x 32 inputs adds four partial sums per output, as the
general convolutions do: next to one term of 2^24 (whose neighbours are 2 apart) terms of
1/4 are lost where they share its sum, and kept in the other three.  The four sums take 16
of every 64 terms each, so at most 16 ceil(K / 64) terms share the large one's, and the
three additions of the sums round by at most 1 each: the bound below.  A single sum loses
all of the small terms."""
import math

import pytest
import torch

from oracle import layout as olayout
from tests import helpers as H

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api

SIDE, CH, F = 32, 9, 32
OUT = (15, 13, 11)
BIG = 2.0 ** 24


def _grad(params, x, dfeat):
    """The gradients of the weights and biases by layer."""
    cfg = H.cfg("full32")
    tab, blocks = olayout.offsets(olayout.dims(**cfg))[0], olayout.blocks(olayout.dims(**cfg))
    flat = torch.zeros(blocks["enc"][1])
    for i, (W, b) in enumerate(params):
        for name, t in ((f"enc.conv{i + 1}.W", W), (f"enc.conv{i + 1}.b", b)):
            flat[tab[name][0]:tab[name][0] + t.numel()] = t.reshape(-1)
    flat = flat.cuda()
    _, ws = api.encoder_fwd(cfg, 0, flat, x.cuda())
    g = api.encoder_bwd(cfg, 0, flat, ws, dfeat.reshape(1, -1).contiguous().cuda(), flat.numel()).cpu()
    cut = lambda n, t: g[tab[n][0]:tab[n][0] + t.numel()].reshape(t.shape).double()
    return [(cut(f"enc.conv{i + 1}.W", W), cut(f"enc.conv{i + 1}.b", b)) for i, (W, b) in enumerate(params)]


def _zeros():
    return [[torch.zeros(F, CH if i == 0 else F, 3, 3), torch.zeros(F)] for i in range(3)]


def _bound(terms):
    return 16 * math.ceil(terms / 64) * 0.25 + 3


# the large term first, and inside a later slice
@pytest.mark.parametrize("f_big,tap_big", [(0, 0), (20, 5)])
@pytest.mark.parametrize("layer", [1, 2])
def test_input_gradient(layer, f_big, tap_big):
    """K = (f, tap) of one input pixel; every other pixel below is masked, so the bias
    gradient of the layer below is that pixel's input gradient."""
    print(f"encoder32 sums dx layer={layer}", flush=True)
    p = _zeros()
    x = torch.zeros(1, CH, SIDE, SIDE)
    x[0, 0, 15, 15] = 1.0            # seen by pixel (7, 7) of the first layer through its centre tap
    p[0][0][:, 0, 1, 1] = 1.0
    if layer == 2:                   # and by pixel (6, 6) of the second
        p[1][0][:, 0, 1, 1] = 1.0
    else:                            # the upper layer passes its gradient straight down
        p[1][1][:] = 1.0
        for f in range(F):
            p[2][0][f, f, 1, 1] = 1.0
    W = p[layer][0]
    W[:] = 0.25
    W.view(F, F, 9)[f_big, :, tap_big] = BIG
    if layer == 2:
        p[1][0][1:, 0, 1, 1] = 1.0
    p[2][1][:] = 1.0                 # every feature positive
    got = _grad(p, x, torch.ones(F, OUT[2], OUT[2]))[layer - 1][1]
    exact = BIG + 0.25 * (9 * F - 1)
    assert (got - exact).abs().max() <= _bound(9 * F), (got - exact).abs().max()


@pytest.mark.parametrize("q_big", [0, 70])
@pytest.mark.parametrize("layer", [0, 1, 2])
def test_weight_gradient(layer, q_big):
    """K = the output pixels; the layer's input is 1/4 everywhere, its output gradient 1
    but for one pixel."""
    print(f"encoder32 sums dw layer={layer}", flush=True)
    o, top = OUT[layer], OUT[2]
    p = _zeros()
    for i in range(3):
        p[i][1][:] = 0.25            # every output positive, and the layers' inputs 1/4
        if i > layer:                # pass the gradient straight down, at the centre tap
            for f in range(F):
                p[i][0][f, f, 1, 1] = 1.0
    x = torch.full((1, CH, SIDE, SIDE), 0.25)
    m = (o - top) // 2               # pixels of the layer that no feature's gradient reaches
    d = torch.ones(F, top, top)
    y, xx = divmod(q_big, o)
    y, xx = max(y, m), max(xx, m)
    d[:, y - m, xx - m] = BIG / 0.25
    got = _grad(p, x, d)[layer][0]
    exact = BIG + 0.25 * (top * top - 1)
    assert (got - exact).abs().max() <= _bound(o * o), (got - exact).abs().max()
