"""Query-range parts on the key side of the bf16 backward: key blocks of long
segments, against float64 autograd on the host.

Tolerance: the other backward tests' bound, 2e-2 of the largest gradient and
1e-2 relative L2 (operands rounded to bf16, float32 sums).
"""
import math

import pytest

torch = pytest.importorskip("torch")

from paper_2609_38832_amd import _lib as L  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L.lib()


from gpu_util import DEV, say  # noqa: E402


def _rope(x, base=1e4):
    n, d = x.shape
    a = torch.arange(n, dtype=torch.float64)[:, None] * base ** (
        -2.0 * torch.arange(d // 2, dtype=torch.float64) / d)
    x1, x2 = x[:, :d // 2], x[:, d // 2:]
    return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)


def _grads(q, k, v, do):
    x = [y.cpu().double().requires_grad_(True) for y in (q, k, v)]
    n, d = q.shape
    s = _rope(x[0]) @ _rope(x[1]).T / math.sqrt(d)
    s.masked_fill_(torch.ones(n, n, dtype=torch.bool).triu_(1), float("-inf"))
    return torch.autograd.grad(((torch.softmax(s, -1) @ x[2]) * do).sum(), x)


# T: the longest T without parts; 65 and 66 key tiles; an odd count of tiles
# with a ragged end.  A second head takes the other tokens (whole blocks).
@pytest.mark.parametrize("T,first", [(4096, 4096), (4160, 4160), (4224, 4224), (4400, 4259)])
@pytest.mark.parametrize("d", [64, 128])
def test_key_parts(T, first, d):
    say(f"key-side parts T {T}, {first} tokens in head 0, d {d}")
    g = torch.Generator(device=DEV).manual_seed(T + d)
    logits = torch.zeros(1, T, 2, device=DEV)
    pick = torch.randperm(T, generator=g, device=DEV)
    logits[0, pick[:first], 0] = 1.0
    logits[0, pick[first:], 1] = 1.0
    q, k, v = (torch.randn(1, 2, T, d, generator=g, device=DEV, dtype=torch.bfloat16)
               for _ in range(3))
    dout = torch.randn(1, T, d, generator=g, device=DEV)
    r = L.route(logits, 1)
    off, perm = r["seg_offsets"].cpu().tolist(), r["perm_token"].cpu()
    assert off[1] == first
    packed = L.attn_bwd(q, k, v, r, 1, 1e4, dout, packed=True)
    dense = L.attn_bwd(q, k, v, r, 1, 1e4, dout)
    again = L.attn_bwd(q, k, v, r, 1, 1e4, dout, packed=True)
    for name in ("dq", "dk", "dv", "dgates"):
        assert torch.equal(packed[name], again[name]), name
    for h in range(2):
        t = perm[off[h]:off[h + 1]].long()
        if len(t) == 0:
            continue
        ref = _grads(q[0, h, t.to(DEV)], k[0, h, t.to(DEV)], v[0, h, t.to(DEV)],
                     dout.cpu().double()[0, t])
        for name, x in zip(("dq", "dk", "dv"), ref):
            got = packed[name][off[h]:off[h + 1]]
            assert torch.equal(dense[name][0, h, t.to(DEV)], got), name
            err = (got.cpu().double() - x).abs()
            assert float(err.max()) <= 2e-2 * float(x.abs().max()), name
            assert float(err.norm() / x.norm()) <= 1e-2, name


@pytest.mark.parametrize("d", [64, 128])
def test_saved_backward_repeats(d, T=4400):
    # the parts' records and sums lie in workspace that the saved state does not
    # need: a second backward from the same state gives the same gradients, and so
    # does a workspace sized for as many tokens in shorter sequences
    say(f"saved backward twice, T {T}, d {d}")
    g = torch.Generator(device=DEV).manual_seed(d)
    logits = torch.randn(1, T, 8, generator=g, device=DEV)
    logits[..., 0] += 9.0
    q, k, v = (torch.randn(1, 8, T, d, generator=g, device=DEV, dtype=torch.bfloat16)
               for _ in range(3))
    dout = torch.randn(1, T, d, generator=g, device=DEV)
    r = L.route(logits, 1)
    want = L.attn_bwd(q, k, v, r, 1, 1e4, dout, packed=True)
    ws = L.workspace(L.lib().namoh_attn_bwd_workspace_size(4, 4096, 8, 1, d), DEV)
    L.attn_fwd_train(q, k, v, r, 1, 1e4, ws)
    for rep in range(2):
        got = L.attn_bwd(q, k, v, r, 1, 1e4, dout, ws=ws, packed=True, saved=True)
        for name in ("dq", "dk", "dv", "dgates"):
            assert torch.equal(got[name], want[name]), (rep, name)


def test_parts_longer_than_a_fair_share(T=16384, d=128):
    # one head of 16384 tokens: the query side's parts leave too few partial rows
    # for the key side's at a fair share of 65 tiles (573 + 2 x 286 of 1024)
    say(f"key-side parts that share the partial rows, T {T}, d {d}")
    g = torch.Generator(device=DEV).manual_seed(3)
    q, k, v = (torch.randn(1, 1, T, d, generator=g, device=DEV, dtype=torch.bfloat16)
               for _ in range(3))
    dout = torch.randn(1, T, d, generator=g, device=DEV)
    r = L.route(torch.zeros(1, T, 1, device=DEV), 1)
    got = L.attn_bwd(q, k, v, r, 1, 1e4, dout, packed=True)
    qd, kd = (_rope(x[0, 0].cpu().double()).to(DEV) for x in (q, k))
    vd, do = v[0, 0].double(), dout[0].double()
    dq, dk, dv = (torch.zeros(T, d, dtype=torch.float64, device=DEV) for _ in range(3))
    for lo in range(0, T, 2048):
        hi = lo + 2048
        s = (qd[lo:hi] @ kd[:hi].T) / math.sqrt(d)
        i, j = torch.arange(lo, hi, device=DEV)[:, None], torch.arange(hi, device=DEV)[None]
        p = torch.softmax(s.masked_fill_(j > i, float("-inf")), -1)
        o = p @ vd[:hi]
        dv[:hi] += p.T @ do[lo:hi]
        ds = p * (do[lo:hi] @ vd[:hi].T - (do[lo:hi] * o).sum(-1, keepdim=True)) / math.sqrt(d)
        dq[lo:hi] = ds @ kd[:hi]
        dk[:hi] += ds.T @ qd[lo:hi]
    for name, x in (("dq", dq), ("dk", dk), ("dv", dv)):
        y = got[name].double()
        if name != "dv":   # into the rotated frame
            y = _rope(y.cpu()).to(DEV)
        err = (y - x).abs()
        assert float(err.max()) <= 2e-2 * float(x.abs().max()), name
        assert float(err.norm() / x.norm()) <= 1e-2, name
