"""GPU parity of the routed projections' tiled kernel at the edges of its
tiles and of its dispatch, against float64 products on the host.

Tolerance: check_out's bf16 bound (operands bf16, float32 accumulation; the
roundings are the bf16 results, and the bf16 gated rows before the dense
output product: 2^-9 relative each).
"""
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


def _routing(B, T, H, K, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return g, L.route(torch.randn(B, T, H, generator=g, device=DEV), K)


def _sample(B, T, n=40):
    g = np.random.default_rng(5)
    bt = {(0, 0), (B - 1, T - 1)}
    while len(bt) < min(n, B * T):
        bt.add((int(g.integers(B)), int(g.integers(T))))
    return sorted(bt)


# (B, T, H, K, d): one head's rows 1, 127 .. 129, 255 .. 257 (K = H: a head
# holds every token); sequences joined into one tile; more than 128 tiles of a
# share (unsplit) and a split tail after full rounds; more than 256 sequences
QKV = [(1, 1, 1, 1, 64), (1, 127, 2, 2, 64), (1, 129, 1, 1, 128), (1, 255, 3, 3, 64),
       (1, 257, 2, 2, 128), (5, 51, 2, 2, 64), (256, 3, 4, 2, 64), (257, 3, 4, 2, 64),
       (2, 4400, 8, 4, 64), (3, 2900, 64, 8, 128),
       # 256-row tiles (more than 512 of the small ones) at the same edges; 510 and 513 of them
       (1, 129, 64, 64, 128), (1, 255, 64, 64, 128), (1, 257, 48, 48, 128), (1, 500, 64, 16, 128),
       (1, 20480, 10, 1, 64), (1, 20480, 11, 1, 64)]


@pytest.mark.parametrize("B,T,H,K,d", QKV)
def test_qkv_tiles(B, T, H, K, d, dm=256):
    say(f"qkv tiles B{B} T{T} H{H} K{K} d{d}")
    g, r = _routing(B, T, H, K, 3)
    x = torch.randn(B, T, dm, generator=g, device=DEV, dtype=torch.bfloat16)
    w = torch.randn(H, 3, d, dm, generator=g, device=DEV, dtype=torch.bfloat16) * dm ** -0.5
    mark = 12288.0   # exact in bf16; rows of unrouted pairs keep it
    out = {n: torch.full((B, H, T, d), mark, dtype=torch.bfloat16, device=DEV) for n in "qkv"}
    L.qkv_proj(x, w, r, H, K, out=out)
    torch.cuda.synchronize()
    routed = torch.zeros(B, T, H, dtype=torch.bool, device=DEV)
    routed.scatter_(2, r["topk_idx"].long(), True)
    routed = routed.transpose(1, 2)
    for n in "qkv":   # every routed row written, no other
        assert (out[n][~routed] == mark).all() and not (out[n][routed] == mark).all(1).any()
    topk, xs, ws = r["topk_idx"].cpu(), x.cpu().double(), w.cpu().double()
    got, ref = [], []
    for b, t in _sample(B, T):
        for i in topk[b, t].tolist():
            for j, n in enumerate("qkv"):
                got.append(out[n][b, i, t].float().cpu().numpy())
                ref.append((ws[i, j] @ xs[b, t]).numpy())
    check_out(np.array(got), np.array(ref), "bf16", what="q/k/v rows")


# (B, T, H, K, d, dm): tokens around a tile and its half; 136 tiles (unsplit),
# 288 (a round and a split tail); H = 64 (128-column tiles); the dense form
# past 384 K: 512 K with 96 tiles, one tile less (per-pair), d = 128 at
# 1024 K with 256 tiles, one less (per-pair); d_model 128, where the dense
# form's rows do not fit the per-pair workspace
OUT = [(1, 1, 4, 2, 64, 256), (1, 128, 4, 2, 64, 256), (1, 129, 4, 2, 64, 128),
       (1, 257, 1, 1, 64, 256), (2, 2176, 4, 2, 64, 2048), (1, 9100, 4, 2, 128, 2048),
       (1, 300, 64, 11, 64, 512), (1, 3072, 16, 2, 64, 2048), (1, 2816, 16, 2, 64, 2048),
       (1, 8192, 16, 2, 128, 2048), (1, 7936, 16, 2, 128, 2048), (1, 25000, 16, 2, 64, 128),
       # 256 small tiles, and 256-row tiles just past them (1, 128 and 129 rows in the last)
       (1, 1024, 4, 2, 64, 2048), (1, 1025, 4, 2, 64, 2048), (1, 1152, 4, 2, 64, 2048),
       (1, 1153, 4, 2, 64, 2048), (1, 4225, 64, 11, 64, 512)]


@pytest.mark.parametrize("hdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,T,H,K,d,dm", OUT)
def test_out_tiles(B, T, H, K, d, dm, hdt):
    say(f"out tiles B{B} T{T} H{H} K{K} d{d} dm{dm} {hdt}")
    g, r = _routing(B, T, H, K, 4)
    ho = torch.randn(B * T * K, d, generator=g, device=DEV).to(hdt)
    w = torch.randn(H, dm, d, generator=g, device=DEV, dtype=torch.bfloat16) * d ** -0.5
    odt = torch.bfloat16 if hdt == torch.float32 else torch.float32
    o = L.out_proj(ho, w, r, B, T, H, K, out_dtype=odt,
                   out=torch.full((B, T, dm), float("nan"), dtype=odt, device=DEV))
    torch.cuda.synchronize()
    assert torch.isfinite(o).all()
    _check_out_rows(o, ho, w, r, _sample(B, T))


def _check_out_rows(o, ho, w, r, sample):
    ws = w.cpu().double()
    got, ref = [], []
    for b, t in sample:
        top, gates, slot = (r[n][b, t].cpu() for n in ("topk_idx", "gates", "slot_pos"))
        h = ho[slot.to(DEV).long()].cpu().double()
        got.append(o[b, t].float().cpu().numpy())
        ref.append(sum(gates[k].double() * (ws[top[k]] @ h[k])
                       for k in range(len(top))).numpy())
    check_out(np.array(got), np.array(ref), "bf16", what="output rows")


def test_out_rows_past_4_gib():
    # the gated rows end past 2^32 bytes: rows are addressed in 64 bits
    B, T, H, K, d, dm = 1, 262145, 64, 64, 128, 128
    say("output projection, 4 GiB of gated rows")
    g, r = _routing(B, T, H, K, 6)
    ho = torch.randn(B * T * K, d, generator=g, device=DEV, dtype=torch.bfloat16)
    w = torch.randn(H, dm, d, generator=g, device=DEV, dtype=torch.bfloat16) * d ** -0.5
    o = L.out_proj(ho, w, r, B, T, H, K, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _check_out_rows(o, ho, w, r, _sample(B, T, 12))


# every row of short inputs (128 x 64 tiles), whose reduction runs in rounds of
# three chunks: 32 and 64 chunks, and 2, 6 and 10 (a round cut short, whole ones,
# one chunk over); output: H d / 64 chunks of 1, 2, 3, 4, 32 and 64
@pytest.mark.parametrize("T,H,K,d,dm", [(300, 32, 8, 64, 2048), (300, 32, 8, 128, 4096),
                                        (97, 8, 4, 64, 128), (97, 8, 4, 64, 384),
                                        (97, 8, 4, 64, 640)])
def test_small_qkv_all_rows(T, H, K, d, dm):
    say(f"short qkv, all rows: T{T} H{H} K{K} d{d} dm{dm}")
    g, r = _routing(1, T, H, K, 7)
    x = torch.randn(1, T, dm, generator=g, device=DEV, dtype=torch.bfloat16)
    w = torch.randn(H, 3, d, dm, generator=g, device=DEV, dtype=torch.bfloat16) * dm ** -0.5
    out = {n: torch.full((1, H, T, d), float("nan"), dtype=torch.bfloat16, device=DEV) for n in "qkv"}
    for rep in range(3):
        L.qkv_proj(x, w, r, H, K, out=out)
    top, xd = r["topk_idx"][0].long(), x[0].double()
    for j, n in enumerate("qkv"):
        got, ref = [], []
        for h in range(H):
            t = (top == h).any(1).nonzero()[:, 0]
            got.append(out[n][0, h, t].float())
            ref.append(xd[t] @ w[h, j].double().T)
        check_out(torch.cat(got).cpu().numpy(), torch.cat(ref).cpu().numpy(), "bf16", what=n)


@pytest.mark.parametrize("T,H,K,d,dm", [(300, 32, 8, 64, 2048), (300, 32, 16, 128, 2048),
                                        (130, 1, 1, 64, 256), (130, 2, 1, 64, 256),
                                        (130, 3, 1, 64, 256), (130, 2, 1, 128, 256)])
def test_small_out_all_rows(T, H, K, d, dm):
    say(f"short output projection, all rows: T{T} H{H} K{K} d{d} dm{dm}")
    g, r = _routing(1, T, H, K, 8)
    ho = torch.randn(T * K, d, generator=g, device=DEV)
    w = torch.randn(H, dm, d, generator=g, device=DEV, dtype=torch.bfloat16) * d ** -0.5
    for rep in range(3):
        o = L.out_proj(ho, w, r, 1, T, H, K, out_dtype=torch.float32,
                       out=torch.full((1, T, dm), float("nan"), device=DEV))
    ref = torch.zeros(T, dm, dtype=torch.float64, device=DEV)
    rows = (r["gates"][0].double()[..., None] * ho[r["slot_pos"][0].long()].double())   # [T, K, d]
    for h in range(H):
        t, k = (r["topk_idx"][0] == h).nonzero(as_tuple=True)
        ref[t] += rows[t, k] @ w[h].double().T
    check_out(o[0].cpu().numpy(), ref.cpu().numpy(), "bf16", what="output rows")


# each dense tile form (short inputs; 256 x 256 up to 384 K, at 512 K and at
# 1024 K; 128 columns for 64 heads; a split tail's half tiles), and the per-pair form
@pytest.mark.parametrize("T,H,K,d,dm", [(300, 4, 2, 64, 256), (3072, 4, 2, 128, 2048),
                                        (3072, 16, 2, 64, 2048), (8192, 16, 2, 128, 2048),
                                        (4225, 64, 11, 64, 512), (2816, 16, 2, 64, 2048)])
@pytest.mark.parametrize("odt", [torch.float32, torch.bfloat16])
def test_non_finite_weights_stay_with_their_heads(T, H, K, d, dm, odt):
    say(f"non-finite weights: T{T} H{H} K{K} d{d} dm{dm} {odt}")
    g, r = _routing(1, T, H, K, 9)
    ho = torch.randn(T * K, d, generator=g, device=DEV)
    w = torch.randn(H, dm, d, generator=g, device=DEV, dtype=torch.bfloat16) * d ** -0.5
    inf, nan = float("inf"), float("nan")
    clean = L.out_proj(ho, w, r, 1, T, H, K, out_dtype=odt)
    w2 = w.clone()
    w2[1, 5, 3], w2[1, dm - 1, d - 1], w2[H - 1, 37] = inf, nan, -inf
    o = L.out_proj(ho, w2, r, 1, T, H, K, out_dtype=odt)
    bad = torch.zeros(1, T, dm, dtype=torch.bool, device=DEV)
    for h, cols in ((1, [5, dm - 1]), (H - 1, [37])):
        t = (r["topk_idx"][0] == h).any(1)
        for col in cols:
            bad[0, t, col] = True
    assert torch.equal(~torch.isfinite(o), bad)
    same = o == clean
    touched = torch.zeros(dm, dtype=torch.bool, device=DEV)
    touched[[5, 37, dm - 1]] = True
    assert same[..., ~touched].all()
    # the touched columns of the other tokens: float32 sums in another order
    a, b = o[..., touched].double(), clean[..., touched].double()
    keep = ~bad[..., touched]
    lim = 1e-5 if odt == torch.float32 else 2 ** -7
    assert ((a - b).abs()[keep] <= lim * (1 + b.abs()[keep])).all()
