"""Router gradient at the edges of its token groups (32 tokens with eight lanes each, 64 with
four from 32769 tokens and up to 32 heads, 256 with one up to 8 heads) and of the head and
selection counts, against the formula in float64.

Bounds: each float32 operation adds at most 2^-24 relative; an affinity carries the
rounding of its exponent argument (the logit range R), two units of expf, the sum of at
most 13 additions in a row, a reciprocal and a product, below R + 24 units; a sum over K
entries adds K + 1."""
import numpy as np
import pytest

import oracle as O
from gpu_util import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if torch.cuda.is_available():
    import paper_2609_38832_amd._lib as L


@pytest.mark.parametrize("BT,H,K", [((1, 1), 1, 1), ((1, 31), 7, 3), ((1, 33), 33, 5),
                                    ((3, 43), 64, 64), ((2, 1000), 32, 8),
                                    ((1, 255), 8, 8), ((1, 257), 5, 2), ((2, 128), 8, 1),
                                    ((1, 513), 9, 9), ((1, 32768), 32, 4), ((1, 32769), 9, 2),
                                    ((3, 10950), 32, 4), ((1, 33000), 33, 3), ((1, 33000), 8, 3)])
@pytest.mark.parametrize("gate_mode", [O.GATE_SOFTMAX_SELECTED, O.GATE_SOFTMAX_ALL])
def test_route_bwd_edges(BT, H, K, gate_mode):
    say(f"route backward {BT} H {H} K {K} gate_mode {gate_mode}")
    B, T = BT
    rng = np.random.default_rng(B * T + H)
    lg = torch.from_numpy(3 * rng.standard_normal((B, T, H)).astype(np.float32)).cuda()
    dg = torch.from_numpy(rng.standard_normal((B, T, K)).astype(np.float32)).cuda()
    r = L.route(lg, K, gate_mode)
    got = L.route_bwd(lg, r, dg, gate_mode).cpu().double()
    top = r["topk_idx"].cpu().long()
    lo, d = lg.cpu().double(), dg.cpu().double()
    if gate_mode == O.GATE_SOFTMAX_SELECTED:
        g = r["gates"].cpu().double()
        s, sa = (g * d).sum(-1, keepdim=True), (g * d.abs()).sum(-1, keepdim=True)
        want = torch.zeros_like(lo).scatter_(-1, top, g * (d - s))
        mass = torch.zeros_like(lo).scatter_(-1, top, g * (d.abs() + sa))
        units = K + 4
    else:
        a = torch.softmax(lo, -1)
        da = torch.zeros_like(lo).scatter_(-1, top, d)
        want = a * (da - (a * da).sum(-1, keepdim=True))
        mass = a * (da.abs() + (a * da.abs()).sum(-1, keepdim=True))
        units = 2 * (float(lo.max() - lo.min()) + 24) + K + 4
    assert bool(((got - want).abs() <= units * 2.0 ** -24 * mass + 1e-37).all())
