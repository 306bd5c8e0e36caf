"""Dense gradients of the bf16 backward: the rows of tokens that a head did not select are
exactly zero and the others equal the packed gradients, in outputs that hold NaN.

Token counts around the fill's units (16 tokens at d = 64, 8 at d = 128), more units than
fill workgroups, every head selected, 64 heads, fills on both sides of 512 MB (written beside
the query side's products, or by a launch of their own), and past it on both sides of 400
products a filled row (beside again from there on)."""
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


@pytest.mark.parametrize("B,T,H,K,d", [(1, 1, 1, 1, 64), (2, 7, 5, 2, 128), (3, 17, 64, 9, 64),
                                       (2, 33, 4, 4, 64), (3, 700, 8, 2, 128), (1, 2307, 6, 1, 64),
                                       (1, 5548, 64, 1, 128),
                                       (1, 5549, 64, 1, 128), (2, 5548, 64, 1, 64),
                                       (3, 3699, 64, 1, 64),
                                       (110, 799, 8, 4, 128), (110, 800, 8, 4, 128)])
def test_dense_rows(B, T, H, K, d):
    say(f"dense gradients B {B} T {T} H {H} K {K} d {d}")
    g = torch.Generator(device=DEV).manual_seed(T)
    r = L.route(torch.randn(B, T, H, generator=g, device=DEV), K)
    q, k, v = (torch.randn(B, H, T, d, generator=g, device=DEV, dtype=torch.bfloat16)
               for _ in range(3))
    dout = torch.randn(B, T, d, generator=g, device=DEV)
    packed = L.attn_bwd(q, k, v, r, K, 1e4, dout, packed=True)
    out = {n: torch.full((B, H, T, d), float("nan"), device=DEV) for n in ("dq", "dk", "dv")}
    out["dgates"] = torch.full((B, T, K), float("nan"), device=DEV)
    dense = L.attn_bwd(q, k, v, r, K, 1e4, dout, out=out)
    b, t, s = torch.meshgrid(*(torch.arange(n, device=DEV) for n in (B, T, K)), indexing="ij")
    h, pos = r["topk_idx"].long(), r["slot_pos"].long()
    for name in ("dq", "dk", "dv"):
        want = torch.zeros(B, H, T, d, device=DEV)
        want[b, h, t] = packed[name][pos]
        assert torch.equal(dense[name], want), name
    assert torch.equal(dense["dgates"], packed["dgates"])
