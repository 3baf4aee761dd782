"""encoder_fwd keeps its input for encoder_bwd and writes the features wherever the
caller's buffers lie: over the images, or 4-byte aligned, as apart and aligned."""
import ctypes

import pytest
import torch

from oracle import layout as olayout
from tests import helpers as H

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import _lib, api


@pytest.mark.parametrize("name,prec", [("full", 0), ("full", 1), ("full32", 0), ("full32", 1), ("tiny", 0), ("tiny", 1)])
@pytest.mark.parametrize("x_off,feat_off", [(0, None), (1, None), (0, 1), (2, 0), (3, 2)])
def test_buffers(name, prec, x_off, feat_off):
    print(f"encoder buffers {name} prec={prec} x+{x_off} feat+{feat_off}", flush=True)
    cfg, n = H.cfg(name), 5
    end = olayout.blocks(olayout.dims(**cfg))["enc"][1]
    p = torch.tensor(H.params(name)[:end], dtype=torch.float32, device="cuda")
    gen = torch.Generator().manual_seed(1)
    side, width = cfg["H"] // cfg["k"], _lib.feat_width(cfg)
    x = (torch.rand((n, cfg["C"], side, side), generator=gen) - 0.5).cuda()
    dfeat = torch.randn((n, width), generator=gen).cuda()
    want, ws = api.encoder_fwd(cfg, prec, p, x)
    gwant = api.encoder_bwd(cfg, prec, p, ws, dfeat, end)
    store = torch.zeros(max(x.numel(), n * width) + 8, device="cuda")
    store[x_off:x_off + x.numel()] = x.flatten()
    # feat_off None: the features over the images, from their start
    fbuf = store if feat_off is None else torch.zeros(n * width + 8, device="cuda")
    off = x_off if feat_off is None else feat_off
    ws2 = torch.empty_like(ws)
    _lib.check(_lib.LIB.encoder_fwd(ctypes.byref(_lib.make_dims(cfg)), prec, p.data_ptr(),
                                    store.data_ptr() + 4 * x_off, n, fbuf.data_ptr() + 4 * off, ws2.data_ptr(),
                                    _lib.stream_handle()))
    assert torch.equal(fbuf[off:off + n * width].view(n, width), want)
    assert torch.equal(api.encoder_bwd(cfg, prec, p, ws2, dfeat, end), gwant)
