"""The categorical projection on dyadic values, where positions, weights and sums are
exact in FP32: equal to the oracle for every support width, run length and direction of
the shifted atoms, clamped ends, and rewards or probabilities that are not finite."""
import numpy as np
import pytest
import torch

from oracle import nets
from tests import helpers as H

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2602_21203_amd import api


@pytest.mark.parametrize("N", [2, 3, 63, 64, 65, 101, 128, 129, 255, 256])
@pytest.mark.parametrize("gamma", [0.0, 0.25, 1.0, 2.0, -1.0])
def test_projection_is_exact_on_dyadic_values(N, gamma):
    print(f"projection N={N} gamma={gamma}", flush=True)
    n = 203   # a ragged last workgroup
    rng = np.random.default_rng(N)
    lo, hi = -float(N // 2), float(N - 1 - N // 2)   # atoms one apart
    p = rng.integers(0, 64, size=(n, N)).astype(np.float32) / 4096
    r = rng.integers(-3 * N, 3 * N + 1, size=n).astype(np.float32) / 4
    done = (rng.uniform(size=n) < 0.3).astype(np.uint8)
    bonus = rng.integers(-8, 9, size=n).astype(np.float32) / 2
    r[:3] = np.nan, np.inf, -np.inf
    p[5, N // 2] = np.inf
    p[6, 0] = np.nan
    p[7] = -p[7]
    dev = lambda v: torch.as_tensor(v).cuda()
    cfg = dict(H.cfg("full"), atoms=N, v_min=lo, v_max=hi)
    for b in (bonus, None):
        got = api.c51_project(cfg, dev(p), dev(r), dev(done), None if b is None else dev(b), gamma).cpu().numpy()
        with np.errstate(invalid="ignore"):
            want = nets.c51_project(p.astype(np.float64), r.astype(np.float64), done.astype(np.float64), gamma,
                                    0.0 * bonus if b is None else b.astype(np.float64), lo, hi)
        np.testing.assert_array_equal(got, want)
