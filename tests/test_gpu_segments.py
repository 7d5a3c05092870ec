"""Rings whose workgroups have two key groups: the references of later segments, found before the loop and taken at a segment's first sub-tile."""
import pytest
import torch

from gpu_util import RING, STEP_BF16, STEP_F32, STEP_MERGE, attn_per_unit, attn_plan, attn_shape

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
    (2, 75, 4, 64),       # renewed every 64 keys, rows and keys end inside a sub-tile
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
    assert float((out - want).abs().max()) <= (1e-2 if std == 1.0 else 2 ** -8 * float(v.abs().max()) * 1.02 + 1e-4)   # (1e-2: as for every block step)
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
    assert float((out - want).abs().max()) <= 1e-2
    assert float((lse - torch.logsumexp(s, -1)).abs().max()) <= 1e-5


@pytest.mark.parametrize("B,H,Sq,Sk,n,causal", [
    (4, 32, 256, 256, 1, True),       # row tiles that see one tile of keys to four
    (4, 32, 200, 300, 1, True),       # five
    (4, 32, 193, 337, 1, True), (4, 24, 449, 449, 1, True),   # the sixth tile, the eighth: a group of six and more; one row in the last workgroup
    (3, 32, 385, 290, 1, True),       # rows that see no key
    (4, 8, 1089, 1089, 1, True),      # groups of inner tiles
    (16, 8, 257, 1345, 1, False), (16, 8, 257, 1409, 1, True), (16, 8, 257, 1601, 1, False),   # tails of one to six tiles behind them
    (4, 8, 1152, 1152, 3, True), (4, 8, 1300, 1300, 4, True),   # rings
    (2, 8, 2304, 2304, 9, True),      # as many references as it keeps
])
def test_three_workgroups_a_compute_unit(lib, B, H, Sq, Sk, n, causal):
    """512 to 768 workgroups of 64 rows at D 64."""
    D, off = 64, Sk - Sq if causal else None
    form = RING if n > 1 else STEP_F32
    assert attn_shape(lib, form, B, H, H, Sq, Sk, D, off, n) == (64, 2) and attn_per_unit(lib, form, B, H, H, Sq, Sk, D, off, n) == 3
    gen = torch.Generator(device="cuda").manual_seed(Sq + 7 * Sk)
    q, k, v = (torch.randn((B, H, S, D), device="cuda", generator=gen).bfloat16() for S in (Sq, Sk, Sk))
    out, lse = torch.full((B, H, Sq, D), float("nan"), device="cuda"), torch.full((B, H, Sq), float("nan"), device="cuda")
    if n > 1:
        lib.tr_ring_attn(q, k, v, n, causal, out, lse)
    else:
        _step(lib, q, k, v, off, out, lse)
    torch.cuda.synchronize()
    want_o, want_l = _exact(q, k, v, off)
    seen = ~torch.isneginf(want_l)
    assert torch.equal(torch.isneginf(lse), ~seen)
    assert float((out - want_o).abs().max()) <= 1e-2 and float((lse - want_l)[seen].abs().max()) <= 1e-5


def _step(lib, q, k, v, off, out, lse):
    if off is None:
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, q.shape[-1] ** -0.5, out, lse)
    else:
        lib.tr_block_attn_causal_at(q, k, v, max(off, 0), max(-off, 0), q.shape[-1] ** -0.5, out, lse)


def _exact(q, k, v, off):
    g = q.shape[1] // k.shape[1]
    s = (q.double() * q.shape[-1] ** -0.5) @ k.double().repeat_interleave(g, 1).transpose(-1, -2).contiguous()
    if off is not None:
        s.masked_fill_(torch.arange(k.shape[2], device="cuda")[None, :] > torch.arange(q.shape[2], device="cuda")[:, None] + off, float("-inf"))
    lse = torch.logsumexp(s, -1)
    return torch.exp(s - lse.masked_fill(torch.isinf(lse), 0.0)[..., None]) @ v.double().repeat_interleave(g, 1), lse


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,off,form,renewed", [
    (4, 16, 4, 537, 2850, 2313, STEP_BF16, False),      # bf16 results, grouped heads
    (2, 12, 12, 1777, 1777, 0, STEP_MERGE, False),      # merged into accumulators
    (1, 16, 2, 2201, 2201, 0, STEP_F32, True),          # rounds as the parts it is not cut into would
    (1, 16, 2, 2201, 2201, 0, STEP_MERGE, True),
    (1, 4, 1, 9001, 9001, 0, STEP_F32, True),
])
def test_steps_of_three_workgroups_a_compute_unit(lib, B, Hq, Hkv, Sq, Sk, off, form, renewed):
    """Every way out of the kernel, with grouped heads in the token-major layout; renewed: the reference is taken anew at the parts that
    256-row workgroups would cut the keys into."""
    D = 64
    assert attn_per_unit(lib, form, B, Hq, Hkv, Sq, Sk, D, off) == 3 and attn_plan(lib, B, Hq, Hkv, Sq, Sk, D, off) == (1, 0)
    gen = torch.Generator(device="cuda").manual_seed(Sq + form)
    def tensor(H, S):
        return torch.randn((B, S, H, D), device="cuda", generator=gen).bfloat16().permute(0, 2, 1, 3)
    q, k, v = tensor(Hq, Sq), tensor(Hkv, Sk), tensor(Hkv, Sk)
    out = torch.full((B, Sq, Hq, D), float("nan"), device="cuda", dtype=torch.bfloat16 if form == STEP_BF16 else torch.float32).permute(0, 2, 1, 3)
    lse = torch.full((B, Hq, Sq), float("nan"), device="cuda")
    want_o, want_l = zip(*(_exact(*(x[b:b + 1, lo:hi] for x, lo, hi in ((q, h * (Hq // Hkv), (h + 1) * (Hq // Hkv)), (k, h, h + 1), (v, h, h + 1))), off)
                           for b in range(B) for h in range(Hkv)))
    want_o, want_l = torch.cat(want_o).view(B, Hq, Sq, D), torch.cat(want_l).view(B, Hq, Sq)
    if form == STEP_MERGE:
        out.copy_(torch.randn((B, Hq, Sq, D), device="cuda", generator=gen))
        lse.copy_(torch.randn((B, Hq, Sq), device="cuda", generator=gen) * 2 + 6)
        lse[:, 0, 0], out[:, 0, 0] = float("-inf"), float("nan")   # an empty row
        a, b, new = lse.double(), want_l, torch.logaddexp(lse.double(), want_l)
        want_o = torch.where(torch.isneginf(a)[..., None], want_o, torch.exp(a - new)[..., None] * out.double() + torch.exp(b - new)[..., None] * want_o)
        want_l = new
        lib.tr_block_attn_merge(q, k, v, lib.TR_MASK_CAUSAL_DIAG, D ** -0.5, out, lse)
    else:
        _step(lib, q, k, v, off, out, lse)
    torch.cuda.synchronize()
    rounding = 2 ** -8 * float(v.abs().max()) if form == STEP_BF16 else 0.0     # of a result to bf16
    assert float((out - want_o).abs().max()) <= 1e-2 + rounding and float((lse - want_l).abs().max()) <= 1e-5


@pytest.mark.parametrize("B,Hq,Hkv,S,form,n", [
    (2, 12, 12, 1777, STEP_F32, 1), (2, 12, 12, 1777, STEP_MERGE, 1), (2, 12, 12, 1777, STEP_BF16, 1),
    (4, 32, 8, 225, RING, 1),                                                                   # four tiles of 64 keys, the last one with 33
    (4, 8, 8, 1089, STEP_F32, 1),                                                               # groups of inner tiles
    (2, 16, 8, 1024, RING, 4), (1, 16, 16, 2001, RING, 3), (2, 8, 8, 2304, RING, 9),            # references of later segments
])
def test_same_bits_as_one_workgroup_a_compute_unit(lib, B, Hq, Hkv, S, form, n):
    """Heads alone, as a ring (which is not cut), whose workgroups of 64 rows have a unit each, against the same heads where three share one."""
    D, g = 64, Hq // Hkv
    assert attn_shape(lib, form, B, Hq, Hkv, S, S, D, 0, n) == (64, 2) and attn_per_unit(lib, form, B, Hq, Hkv, S, S, D, 0, n) == 3
    assert attn_shape(lib, RING, 1, g, 1, S, S, D, 0, n) == (64, 2) and attn_per_unit(lib, RING, 1, g, 1, S, S, D, 0, n) == 1
    gen = torch.Generator(device="cuda").manual_seed(S + n)
    q, k, v = (torch.randn((B, H, S, D), device="cuda", generator=gen).bfloat16() for H in (Hq, Hkv, Hkv))
    out = torch.full((B, Hq, S, D), float("nan"), device="cuda", dtype=torch.bfloat16 if form == STEP_BF16 else torch.float32)
    lse = torch.full((B, Hq, S), float("-inf") if form == STEP_MERGE else float("nan"), device="cuda")
    if form == RING:
        lib.tr_ring_attn(q, k, v, n, True, out, lse)
    elif form == STEP_MERGE:   # onto empty accumulators, which take the block as it is
        lib.tr_block_attn_merge(q, k, v, lib.TR_MASK_CAUSAL_DIAG, D ** -0.5, out, lse)
    else:
        _step(lib, q, k, v, 0, out, lse)
    for b, h in ((0, 0), (B // 2, Hkv // 2), (B - 1, Hkv - 1)):
        heads = slice(h * g, (h + 1) * g)
        alone, alone_lse = torch.full((1, g, S, D), float("nan"), device="cuda"), torch.full((1, g, S), float("nan"), device="cuda")
        lib.tr_ring_attn(q[b:b + 1, heads], k[b:b + 1, h:h + 1], v[b:b + 1, h:h + 1], n, True, alone, alone_lse)
        torch.cuda.synchronize()
        assert torch.equal(alone.to(out.dtype), out[b:b + 1, heads]) and torch.equal(alone_lse, lse[b:b + 1, heads])
