"""Rings whose workgroups have two key groups: the references of later segments, found before the loop and taken at a segment's first sub-tile."""
import pytest
import torch

from gpu_util import RING, STEP_F32, attn_shape

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


@pytest.mark.parametrize("B,H,Sq,Sk,n,causal", [
    (4, 32, 300, 300, 1, True),       # row tiles that see one tile of keys to five
    (4, 32, 300, 337, 1, True), (4, 24, 449, 449, 1, True),   # the sixth tile, the eighth: a group of six and more; one row in the last workgroup
    (3, 32, 385, 290, 1, True),       # rows that see no key
    (4, 8, 1089, 1089, 1, True),      # groups of inner tiles
    (16, 8, 257, 1345, 1, False), (16, 8, 257, 1409, 1, True), (16, 8, 257, 1601, 1, False),   # tails of one to six tiles behind them
    (4, 8, 1152, 1152, 3, True), (4, 8, 1300, 1300, 4, True),   # rings
    (2, 8, 2304, 2304, 9, True),      # as many references as it keeps
])
def test_three_workgroups_a_compute_unit(lib, B, H, Sq, Sk, n, causal):
    """512 to 768 workgroups of 64 rows at D 64."""
    D, off = 64, Sk - Sq if causal else None
    assert 512 <= B * H * -(-Sq // 64) <= 768 and attn_shape(lib, RING if n > 1 else STEP_F32, B, H, H, Sq, Sk, D, off, n) == (64, 2)
    gen = torch.Generator(device="cuda").manual_seed(Sq + 7 * Sk)
    q, k, v = (torch.randn((B, H, S, D), device="cuda", generator=gen).bfloat16() for S in (Sq, Sk, Sk))
    out, lse = torch.full((B, H, Sq, D), float("nan"), device="cuda"), torch.full((B, H, Sq), float("nan"), device="cuda")
    if n > 1:
        lib.tr_ring_attn(q, k, v, n, causal, out, lse)
    elif causal:
        lib.tr_block_attn_causal_at(q, k, v, max(off, 0), max(-off, 0), D ** -0.5, out, lse)
    else:
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, D ** -0.5, out, lse)
    torch.cuda.synchronize()
    s = (q.double() * D ** -0.5) @ k.double().transpose(-1, -2).contiguous()
    if causal:
        s.masked_fill_(torch.arange(Sk, device="cuda")[None, :] > torch.arange(Sq, device="cuda")[:, None] + off, float("-inf"))
    want_l = torch.logsumexp(s, -1)
    want_o = torch.exp(s - want_l.masked_fill(torch.isinf(want_l), 0.0)[..., None]) @ v.double()
    seen = ~torch.isneginf(want_l)
    assert torch.equal(torch.isneginf(lse), ~seen)
    assert float((out - want_o).abs().max()) <= 2 ** -8 * float(v.abs().max()) * 1.02 + 1e-4 and float((lse - want_l)[seen].abs().max()) <= 1e-5
