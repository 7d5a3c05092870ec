"""Rings whose workgroups have two key groups: the references of later segments, found before the loop and taken at a segment's first sub-tile."""
import pytest
import torch

from gpu_util import RING, attn_shape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2412_20501_amd.build import ensure_built
    ensure_built()
    import paper_2412_20501_amd as tr
    return tr


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("std", [1.0, 4.0])   # of Q and K: 4 moves a row's largest score by tens from segment to segment
@pytest.mark.parametrize("H,seg,n,D", [
    (2, 64, 4, 64),       # as short as segments of key groups can be: every step but the first renews
    (2, 64, 4, 128),
    (2, 95, 3, 64),       # renewed every 64 keys, rows and keys end inside a sub-tile
    (1, 97, 5, 128),      # an odd number of sub-tiles a segment: either key group holds its first one
    (2, 161, 2, 128),     # one reference, for one key group
    (3, 260, 4, 64),      # references beyond the tiles that are loaded before the loop
    (1, 600, 6, 128),     # renewed between inner tiles
])
def test_references_of_later_segments(lib, H, seg, n, D, std, causal):
    S, scale = seg * n, D ** -0.5
    gen = torch.Generator(device="cuda").manual_seed(100 * seg + D)
    q, k, v = ((torch.randn((1, H, S, D), device="cuda", generator=gen) * s).bfloat16() for s in (std, std, 1.0))
    assert attn_shape(lib, RING, 1, H, H, S, S, D, 0 if causal else None, n) == (64, 2)
    out, lse = torch.full((1, H, S, D), float("nan"), device="cuda"), torch.full((1, H, S), float("nan"), device="cuda")
    lib.tr_ring_attn(q, k, v, n, causal, out, lse)
    torch.cuda.synchronize()
    s = (q.double() * scale) @ k.double().transpose(-1, -2).contiguous()
    if causal:
        s.masked_fill_(torch.ones((S, S), dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    want = torch.softmax(s, -1) @ v.double()
    # weights rounded to bf16: at most 2^-8 of the largest value, where one key has all the weight; lse from fp32 scores and sums
    assert float((out - want).abs().max()) <= 2 ** -8 * float(v.abs().max()) * 1.02 + 1e-4
    assert float((lse - torch.logsumexp(s, -1)).abs().max()) <= 1e-5 * max(1.0, float(s[torch.isfinite(s)].abs().max()) / 8)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_packed_heads(lib, D, causal):
    """Rings whose query heads share a row space (fewer rounds of workgroups): Query rows of two heads in one workgroup, references renewed."""
    B, Hq, Hkv, seg, n = 300, 4, 2, 40, 3
    S, scale = seg * n, D ** -0.5
    assert attn_shape(lib, RING, B, Hq, Hkv, S, S, D, 0 if causal else None, n)[1] == 1
    gen = torch.Generator(device="cuda").manual_seed(D)
    q, k, v = (torch.randn((B, h, S, D), device="cuda", generator=gen).bfloat16() for h in (Hq, Hkv, Hkv))
    out, lse = torch.full((B, Hq, S, D), float("nan"), device="cuda"), torch.full((B, Hq, S), float("nan"), device="cuda")
    lib.tr_ring_attn(q, k, v, n, causal, out, lse)
    torch.cuda.synchronize()
    kk, vv = (x.double().repeat_interleave(Hq // Hkv, 1) for x in (k, v))
    s = (q.double() * scale) @ kk.transpose(-1, -2).contiguous()
    if causal:
        s.masked_fill_(torch.ones((S, S), dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    want = torch.softmax(s, -1) @ vv
    assert float((out - want).abs().max()) <= 2 ** -8 * float(v.abs().max()) * 1.02 + 1e-4
    assert float((lse - torch.logsumexp(s, -1)).abs().max()) <= 1e-5
