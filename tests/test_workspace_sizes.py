"""Workspace sizes: a workspace sized for a program's largest call serves its smaller ones.
The size queries run on the host; the steps that reuse one workspace need the GPU."""
import os

import pytest

torch = pytest.importorskip("torch")

from paper_2609_38832_amd import _lib as L  # noqa: E402

HEADS = [1, 2, 3, 7, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 128, 255, 256, 257, 300, 1024]
CAPS = [1, 64, 127, 128, 129, 256, 300, 511, 512, 513, 640, 1024, 1025, 4000, 32768]


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(L.LIB_PATH):
        pytest.skip("libnamoh.so not built")
    return L.lib()


def _never_smaller(sizes):
    assert all(s > 0 for s in sizes)
    assert sizes == sorted(sizes), sizes


@pytest.mark.parametrize("d", [32, 64, 128])
def test_decode_sizes_never_decrease(lib, d):
    for cap in CAPS:
        for K in (1, 4, 8):
            _never_smaller([lib.namoh_decode_workspace_size(B, 64, K, d, cap) for B in HEADS])
        for B in (1, 3, 16, 17, 64):
            _never_smaller([lib.namoh_decode_workspace_size(B, 64, K, d, cap) for K in range(1, 65)])
            _never_smaller([lib.namoh_shared_decode_workspace_size(B, s, d, cap) for s in HEADS])
        _never_smaller([lib.namoh_shared_decode_workspace_size(B, 2, d, cap) for B in HEADS])
        if d != 32:
            for g in (1, 2, 4, 8):
                _never_smaller([lib.namoh_decode_grouped_workspace_size(B, 16, 4, g, d, cap)
                                for B in HEADS])
            for B in (1, 16, 33):
                _never_smaller([lib.namoh_decode_grouped_workspace_size(B, 16, 4, g, d, cap)
                                for g in (1, 2, 4, 8)])
    for B in (1, 16, 17, 64):
        _never_smaller([lib.namoh_decode_workspace_size(B, 64, 8, d, cap) for cap in CAPS])
        _never_smaller([lib.namoh_shared_decode_workspace_size(B, 2, d, cap) for cap in CAPS])


@pytest.mark.gpu
@pytest.mark.parametrize("g,K,B0,batches", [(1, 8, 17, (17, 16, 5, 1)), (4, 4, 33, (33, 32, 9, 1))])
def test_decode_workspace_of_a_larger_batch(lib, g, K, B0, batches):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_util import DEV, say
    d, cap, H = 128, 512, 2 * K
    n = (lib.namoh_decode_workspace_size(B0, H, K, d, cap) if g == 1 else
         lib.namoh_decode_grouped_workspace_size(B0, H, K, g, d, cap))
    ws = L.workspace(n, DEV)
    sws = L.workspace(lib.namoh_shared_decode_workspace_size(B0 * 4, 2, d, cap), DEV)
    step = L.decode_step if g == 1 else L.decode_step_grouped
    for B in batches:
        say(f"workspace of {B0} sequences, {B} used, group {g}")
        gen = torch.Generator(device=DEV).manual_seed(B)
        bf = dict(generator=gen, device=DEV, dtype=torch.bfloat16)
        kc, vc = (torch.randn(B, H, cap, d, **bf) for _ in range(2))
        lens = torch.randint(0, cap - 1, (B, H), generator=gen, device=DEV).int()
        logits = torch.randn(B, H, generator=gen, device=DEV)
        q, k, v = (torch.randn(B, H * m, d, **bf) for m in (g, 1, 1))
        outs = [step(logits, q, k, v, kc.clone(), vc.clone(), lens.clone(), K, 1e4,
                     out_dtype=torch.float32, **kw)["out"] for kw in ({}, {"ws": ws})]
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
        skc, svc = (torch.randn(B, 2, cap, d, **bf) for _ in range(2))
        sq, sk, sv = (torch.randn(B, 2, d, **bf) for _ in range(3))
        plen = torch.full((B,), 400, dtype=torch.int32, device=DEV)
        outs = [L.shared_decode_step(sq, sk, sv, skc.clone(), svc.clone(), plen.clone(), 0, 1e4,
                                     out_dtype=torch.float32, **kw) for kw in ({}, {"ws": sws})]
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("d", [64, 128])
def test_backward_size_follows_the_rows(lib, d):
    # one more token costs its rows, also where key blocks start to run as
    # parts (past 4096 tokens); long sequences need no more than as many
    # tokens in short ones, but for their rotation table and block counts
    for H, K in ((8, 1), (32, 4), (64, 8)):
        size = [lib.namoh_attn_bwd_workspace_size(1, T, H, K, d) for T in range(4064, 4130)]
        _never_smaller(size)
        assert max(b - a for a, b in zip(size, size[1:])) < (1 << 18) * K
        long = lib.namoh_attn_bwd_workspace_size(1, 16384, H, K, d)
        short = lib.namoh_attn_bwd_workspace_size(4, 4096, H, K, d)
        assert long <= short + 16384 * d // 2 * 8
