"""Decode steps at the edges of the history chunks, against float64 on the
host.  Cache rows past the histories hold NaN: none of them may be used, the
new token's own row before it is written included.

Tolerance: outputs are float32 here; float32 arithmetic for one or two query
heads per cached row (bf16 caches are exact inputs; the appended key is
rounded to bf16, 2^-9), bf16 queries and probabilities for four and eight:
check_out's bf16 bound covers both.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2609_38832_amd import _lib as L  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L.lib()


from gpu_util import DEV, check_out, say  # noqa: E402

BASE = 1e4


def _rope(x, pos):
    d = x.shape[-1]
    a = pos * BASE ** (-2.0 * torch.arange(d // 2, dtype=torch.float64) / d)
    x1, x2 = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)


def _attend(q, k, v):
    p = torch.softmax(k @ q / math.sqrt(q.shape[-1]), 0)
    return p @ v


# histories around the multiples of 128, 256 and 512 rows
LENS = [0, 1, 31, 127, 128, 129, 255, 256, 257, 383, 384, 511, 512, 513, 640, 1023, 1024, 1030]


# cap 1100: three chunks of up to 512 rows; few sequences spread a history
# over them, 64 x 8 heads (more than 1024 workgroups) do not; cap 300: one
@pytest.mark.parametrize("B,K,cap", [(9, 2, 1100), (64, 8, 1100), (9, 2, 300)])
@pytest.mark.parametrize("d,g", [(64, 1), (128, 1), (64, 2), (128, 4), (64, 8), (128, 8)])
def test_routed_chunks(B, K, cap, d, g):
    say(f"decode chunks B{B} K{K} cap{cap} d{d} g{g}")
    H = 2 * K
    gen = torch.Generator(device=DEV).manual_seed(B + cap + d + g)
    lens = [n for n in LENS if n < cap]
    n0 = torch.tensor([[lens[(b * H + h) % len(lens)] for h in range(H)] for b in range(B)],
                      dtype=torch.int32)
    bf = dict(generator=gen, device=DEV, dtype=torch.bfloat16)
    kc, vc = (torch.randn(B, H, cap, d, **bf) for _ in range(2))
    past = torch.arange(cap, device=DEV)[None, None] >= n0.to(DEV)[..., None]
    kc[past], vc[past] = float("nan"), float("nan")
    k0, v0 = kc.cpu().double(), vc.cpu().double()
    logits = torch.randn(B, H, generator=gen, device=DEV)
    q, k, v = torch.randn(B, H * g, d, **bf), torch.randn(B, H, d, **bf), torch.randn(B, H, d, **bf)
    clen = n0.to(DEV)
    step = L.decode_step_grouped if g > 1 else L.decode_step
    res = step(logits, q, k, v, kc, vc, clen, K, BASE, out_dtype=torch.float32)
    torch.cuda.synchronize()
    top = torch.sort(logits.cpu(), dim=-1, descending=True, stable=True)[1][:, :K]
    assert torch.equal(res["topk_idx"].cpu().long(), top)
    want = n0.clone()
    got, ref = [], []
    qd, kd, vd = (x.cpu().double() for x in (q, k, v))
    for b in range(B):
        gates = torch.softmax(logits[b].cpu().double()[top[b]], 0)
        o = torch.zeros(d, dtype=torch.float64)
        for j, h in enumerate(top[b].tolist()):
            n = int(n0[b, h])
            want[b, h] += 1
            kn = _rope(kd[b, h], n)
            row = kc[b, h, n].cpu().double()
            assert float((row - kn).abs().max()) <= 2 ** -8 * float(kn.abs().max())
            assert torch.equal(vc[b, h, n].cpu().double(), vd[b, h])
            kk = torch.cat([k0[b, h, :n], row[None]])
            vv = torch.cat([v0[b, h, :n], vd[b, h][None]])
            for u in range(g):
                o += gates[j] * _attend(_rope(qd[b, h * g + u], n), kk, vv)
        got.append(res["out"][b].cpu().numpy())
        ref.append(o.numpy())
    assert torch.equal(clen.cpu(), want)
    check_out(np.array(got), np.array(ref), "bf16", what="decode out")


@pytest.mark.parametrize("window,p", [(0, 0), (0, 511), (0, 512), (0, 1024), (128, 127), (128, 128),
                                      (700, 511), (700, 699), (700, 700), (700, 1500)])
@pytest.mark.parametrize("B", [3, 300])
def test_shared_chunks(B, window, p, d=64, Hs=2):
    say(f"shared decode chunks B{B} window {window} p {p}")
    cap = window if window else 1100
    gen = torch.Generator(device=DEV).manual_seed(p + B)
    bf = dict(generator=gen, device=DEV, dtype=torch.bfloat16)
    kc, vc = (torch.full((B, Hs, cap, d), float("nan"), device=DEV, dtype=torch.bfloat16)
              for _ in range(2))
    m = min(p, window - 1) if window else p          # tokens the new one sees besides itself
    slots = torch.arange(p - m, p, device=DEV) % cap
    hk, hv = torch.randn(B, Hs, m, d, **bf), torch.randn(B, Hs, m, d, **bf)
    kc[:, :, slots], vc[:, :, slots] = hk, hv
    q, k, v = (torch.randn(B, Hs, d, **bf) for _ in range(3))
    clen = torch.full((B,), p, dtype=torch.int32, device=DEV)
    out = torch.full((B, d), 2.0, device=DEV)
    L.shared_decode_step(q, k, v, kc, vc, clen, window, BASE, out=out, accumulate=True)
    torch.cuda.synchronize()
    assert (clen == p + 1).all()
    got, ref = [], []
    for b in range(min(B, 4)):
        o = torch.full((d,), 2.0, dtype=torch.float64)
        for s in range(Hs):
            row = kc[b, s, p % cap].cpu().double()
            kk = torch.cat([hk[b, s].cpu().double(), row[None]])
            vv = torch.cat([hv[b, s].cpu().double(), v[b, s].cpu().double()[None]])
            o += _attend(_rope(q[b, s].cpu().double(), p), kk, vv)
        got.append(out[b].cpu().numpy())
        ref.append(o.numpy())
    check_out(np.array(got), np.array(ref), "bf16", what="shared decode out")


@pytest.mark.parametrize("n", [0, 40, 700])
@pytest.mark.parametrize("g,dtype", [(1, torch.bfloat16), (2, torch.bfloat16), (1, torch.float32)])
def test_infinite_value_of_the_new_token(n, g, dtype, d=64, cap=900):
    # infinite in one column of the new value: that column is infinite (its
    # weight is positive), the others what they are without it
    say(f"infinite new value, {n} rows before, group {g}, {dtype}")
    gen = torch.Generator(device=DEV).manual_seed(n)
    kw = dict(generator=gen, device=DEV, dtype=dtype)
    kc, vc = (torch.randn(1, 2, cap, d, **kw) for _ in range(2))
    q, k, v = torch.randn(1, 2 * g, d, **kw), torch.randn(1, 2, d, **kw), torch.randn(1, 2, d, **kw)
    logits = torch.randn(1, 2, generator=gen, device=DEV)
    step = L.decode_step_grouped if g > 1 else L.decode_step
    outs = []
    for x in (1.0, float("inf")):
        v[0, :, 5] = x
        outs.append(step(logits, q, k, v, kc.clone(), vc.clone(),
                         torch.full((1, 2), n, dtype=torch.int32, device=DEV), 2, BASE,
                         out_dtype=torch.float32)["out"][0].cpu())
    assert torch.isfinite(outs[0]).all() and outs[1][5] == float("inf")
    keep = torch.arange(d) != 5
    assert torch.equal(outs[1][keep], outs[0][keep])
    s = torch.full((1, d), 1.0, device=DEV)   # shared heads, added to out
    v[0, :, 5] = float("inf")
    L.shared_decode_step(q[:, :2].contiguous(), k, v, kc, vc,
                         torch.full((1,), n, dtype=torch.int32, device=DEV), 0, BASE, out=s,
                         accumulate=True)
    s = s[0].cpu()
    assert s[5] == float("inf") and torch.isfinite(s[keep]).all()


# Many sequences with short caches are routed in a launch before the attention;
# the same sequences in small batches are routed in its workgroups.  The appends
# and the routing are the same arithmetic; the outputs differ by the order of
# float32 sums (one or two heads a row) or by the maximum that bf16 probabilities
# are rounded against (four and eight).
@pytest.mark.parametrize("d,g,dtype,cap,rope,biased", [
    (64, 1, torch.bfloat16, 300, 0, False), (128, 1, torch.bfloat16, 200, 1, False),
    (64, 2, torch.bfloat16, 400, 0, False), (128, 2, torch.bfloat16, 150, 2, False),
    (64, 4, torch.bfloat16, 1100, 0, False), (128, 8, torch.bfloat16, 300, 1, False),
    (64, 8, torch.bfloat16, 40, 2, False), (128, 4, torch.bfloat16, 1792, 0, False),
    (32, 1, torch.bfloat16, 600, 0, True), (32, 1, torch.float32, 300, 1, False),
    (64, 1, torch.float32, 257, 2, True), (128, 1, torch.float32, 200, 0, False)])
def test_routed_ahead(d, g, dtype, cap, rope, biased, B=336, K=6, H=9):
    say(f"decode routed ahead: d{d} g{g} {dtype} cap{cap} rope{rope} biased{biased}")
    gen = torch.Generator(device=DEV).manual_seed(d + g + cap)
    kw = dict(generator=gen, device=DEV, dtype=dtype)
    lens = [n for n in LENS + [cap - 1, cap - 2, cap] if n <= cap]
    n0 = torch.tensor([[lens[(b * H + h) % len(lens)] for h in range(H)] for b in range(B)],
                      dtype=torch.int32, device=DEV)
    kc, vc = (torch.randn(B, H, cap, d, **kw) for _ in range(2))
    past = torch.arange(cap, device=DEV)[None, None] >= n0[..., None]
    kc[past], vc[past] = float("nan"), float("nan")
    logits = torch.randn(B, H, generator=gen, device=DEV)
    logits[::7] = torch.round(logits[::7])   # ties
    logits[::7][logits[::7] == 0] *= -1      # zeros of both signs
    q, k, v = torch.randn(B, H * g, d, **kw), torch.randn(B, H, d, **kw), torch.randn(B, H, d, **kw)
    pos = torch.randint(0, 5000, (B,), generator=gen, device=DEV, dtype=torch.int32)
    extra = {"bias": torch.randn(H, generator=gen, device=DEV) * 0.1} if biased else {}

    def run(lo, hi):
        c = [x[lo:hi].clone() for x in (kc, vc, n0)]
        st = torch.zeros(1, dtype=torch.int32, device=DEV)
        step = L.decode_step_grouped if g > 1 else L.decode_step
        r = step(logits[lo:hi], q[lo:hi], k[lo:hi], v[lo:hi], *c, K, BASE, rope,
                 seq_pos=pos[lo:hi] if rope == 1 else None, out_dtype=torch.float32, dev_status=st,
                 **extra)
        return [r["topk_idx"], r["gates"], *c, r["out"]], int(st.item())

    whole, status = run(0, B)
    parts = [run(lo, lo + 42) for lo in range(0, B, 42)]
    assert status == max(p[1] for p in parts) == 1    # (some selected head's cache is full)
    same = [torch.cat([p[0][i] for p in parts]) for i in range(6)]
    for a, b in zip(whole[:2] + whole[4:5], same[:2] + same[4:5]):
        assert torch.equal(a, b)
    for a, b in zip(whole[2:4], same[2:4]):            # caches, their unused rows NaN
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert torch.isfinite(whole[5]).all()
    if g >= 4:
        check_out(whole[5].cpu().numpy(), same[5].cpu().double().numpy(), "bf16", what="outputs")
    else:
        err = (whole[5] - same[5]).abs().max()
        assert float(err) <= 1e-5 * float(same[5].abs().max())
