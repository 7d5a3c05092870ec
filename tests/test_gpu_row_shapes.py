"""Shapes of an attention workgroup: 128 Query rows (two or three workgroups to a compute unit), and 128 or 64 rows whose waves
share the keys out among themselves, against what a full chip takes, workgroups of 128 or 256 rows with one key group: the same inputs as one
entry of a batch so large that the launch takes those.  The shape a case stands for is beside it.  All round the same weights (one
exponent reference for a row and segment, renewed at the same keys whatever the shape), so only fp32 sums differ: a few 2^-23 of values of size 1
(out) and 10 (lse).  Sizes sit at the edges of row groups, workgroups, sub-tiles and tiles of keys, and where a segment's
reference is renewed."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import RING, RING_BF16, STEP_BF16, STEP_F32, STEP_MERGE, attn_per_unit, attn_plan, attn_shape, bits_to_dev, f64, max_abs, rand_bits, to_np

pytestmark = pytest.mark.gpu
MANY = 2048      # (batch, head, row tile) triples of 256 rows from which on the launches here take 128 rows and one key group
ROWS_256, ROWS_128, ROWS_128_GROUPS, ROWS_64_GROUPS = (256, 1), (128, 1), (128, 2), (64, 2)    # Query rows of a workgroup, key groups


def _qkv(Hq, Hkv, Sq, Sk, D, seed, token=False):
    def tensor(H, S, s):
        x = rand_bits((1, H, S, D), s)
        return bits_to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3))).permute(0, 2, 1, 3) if token else bits_to_dev(x)
    return tensor(Hq, Sq, seed), tensor(Hkv, Sk, seed + 1), tensor(Hkv, Sk, seed + 2)


def _new(B, H, S, D, dtype=torch.float32, lse=float("nan")):
    return torch.full((B, H, S, D), float("nan"), device="cuda", dtype=dtype), torch.full((B, H, S), lse, device="cuda")


def _agree(few, many, tol=1e-5):
    (o, l), (bo, bl) = few, many
    assert torch.equal(torch.isneginf(l[0]), torch.isneginf(bl[-1]))
    seen = ~torch.isneginf(l[0])
    worst = float((o[0].float() - bo[-1].float()).abs().max()), float((l[0] - bl[-1])[seen].abs().max()) if bool(seen.any()) else 0.0
    print("out, lse:", worst)
    assert max(worst) <= tol


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Hq,Hkv,seg,n,D,token,shape", [
    (1, 1, 1, 1, 64, False, ROWS_256),
    (2, 1, 33, 2, 128, True, ROWS_256),            # a reference every sub-tile, which key groups don't take
    (1, 1, 96, 4, 128, False, ROWS_64_GROUPS),     # segments of three sub-tiles: their first one belongs to either key group
    (3, 1, 65, 1, 64, True, ROWS_256),
    (2, 2, 129, 1, 128, False, ROWS_64_GROUPS),    # one row in the third workgroup
    (2, 1, 191, 3, 64, False, ROWS_64_GROUPS),
    (1, 1, 128, 33, 128, False, ROWS_128),         # 32 later references, by 128-row workgroups on either side
    (1, 1, 288, 33, 128, False, ROWS_64_GROUPS),   # as many later references as key groups keep
    (8, 2, 1024, 2, 128, False, ROWS_64_GROUPS),   # renewed between groups of inner tiles
    (4, 4, 1536, 2, 64, False, ROWS_64_GROUPS),
    (24, 8, 1000, 1, 64, True, ROWS_128_GROUPS),
    (20, 20, 768, 1, 128, False, ROWS_64_GROUPS),
])
def test_rings(lib, Hq, Hkv, seg, n, D, token, shape, causal):
    S = seg * n
    q, k, v = _qkv(Hq, Hkv, S, S, D, 700, token)
    few = _new(1, Hq, S, D)
    lib.tr_ring_attn(q, k, v, n, causal, *few)
    B = -(-MANY // (Hq * -(-S // 256)))
    assert attn_shape(lib, RING, 1, Hq, Hkv, S, S, D, 0 if causal else None, n) == shape
    assert attn_shape(lib, RING, B, Hq, Hkv, S, S, D, 0 if causal else None, n) == ROWS_128
    many = _new(B, Hq, S, D)
    lib.tr_ring_attn(q.expand(B, -1, -1, -1), k.expand(B, -1, -1, -1), v.expand(B, -1, -1, -1), n, causal, *many)
    torch.cuda.synchronize()
    _agree(few, many)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("seg,n,D", [(1024, 2, 64), (1000, 3, 64), (545, 4, 64), (2000, 2, 64), (4096, 2, 64), (478, 4, 128), (700, 3, 128), (2000, 2, 128)])
def test_rings_renew_at_the_same_keys(lib, seg, n, D, causal):
    """One head alone and as one of several, which take workgroups of other shapes: segments that start between the
    tiles and groups of tiles of any of them round the same weights, so that fp32 sums are all that differs."""
    q, k, v = _qkv(1, 1, seg * n, seg * n, D, 780)
    few = _new(1, 1, seg * n, D)
    lib.tr_ring_attn(q, k, v, n, causal, *few)
    shapes = [attn_shape(lib, RING, 1, 1, 1, seg * n, seg * n, D, 0 if causal else None, n)]
    compared = {(*shapes[0], 1)}
    for heads in (2, 4, 8, 12, 16, 24, 32, 96):
        shapes.append(attn_shape(lib, RING, 1, heads, heads, seg * n, seg * n, D, 0 if causal else None, n))
        launch = (*shapes[-1], attn_per_unit(lib, RING, 1, heads, heads, seg * n, seg * n, D, 0 if causal else None, n))
        if launch in compared:
            continue
        compared.add(launch)
        many = _new(1, heads, seg * n, D)
        lib.tr_ring_attn(*(x.expand(-1, heads, -1, -1) for x in (q, k, v)), n, causal, *many)
        torch.cuda.synchronize()
        _agree(few, [x.transpose(0, 1) for x in many])
    assert shapes[0] == ROWS_64_GROUPS and ROWS_128 in shapes
    assert (64, 2, 3) in compared or D == 128 or not causal
    assert ROWS_256 in shapes or (causal and (seg, n) in ((1024, 2), (545, 4), (478, 4)))
    assert ROWS_128_GROUPS in shapes or (seg, n) not in ((4096, 2), (2000, 2)) or (seg, causal) in ((2000, False), (4096, True))


@pytest.mark.parametrize("Hq,Hkv,seg,n", [(1, 1, 501, 3), (2, 1, 700, 4), (2, 2, 32, 34)])
def test_rings_against_the_oracle(lib, Hq, Hkv, seg, n):
    """Segments that start between groups of inner tiles, or that are as short or as many as key groups don't take."""
    S, D = seg * n, 128
    q, k, v = _qkv(Hq, Hkv, S, S, D, 710)
    ref = oracle.attention_full(f64(q.cpu().view(torch.int16).numpy().view(np.uint16)), f64(k.cpu().view(torch.int16).numpy().view(np.uint16)),
                                f64(v.cpu().view(torch.int16).numpy().view(np.uint16)), D ** -0.5, True)
    out, lse = _new(1, Hq, S, D)
    lib.tr_ring_attn(q, k, v, n, True, out, lse)
    torch.cuda.synchronize()
    assert max_abs(to_np(out), ref[0]) <= 1e-2 and max_abs(to_np(lse), ref[1]) <= 1e-5


def _exact(q, k, v, off):
    g = q.shape[1] // k.shape[1]
    s = (q.double() * q.shape[-1] ** -0.5) @ k.double().repeat_interleave(g, 1).transpose(-1, -2).contiguous()
    if off is not None:
        rows, keys = torch.arange(q.shape[2], device="cuda"), torch.arange(k.shape[2], device="cuda")
        s = s.masked_fill(keys[None, :] > rows[:, None] + off, float("-inf"))
    lse = torch.logsumexp(s, -1)
    return torch.exp(s - lse.masked_fill(torch.isinf(lse), 0.0)[..., None]) @ v.double().repeat_interleave(g, 1), lse


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,off,shape", [
    (2, 24, 8, 300, 300, 128, None, ROWS_64_GROUPS),    # a ragged last workgroup
    (2, 24, 8, 300, 300, 64, None, ROWS_64_GROUPS),
    (9, 24, 8, 300, 300, 128, None, ROWS_128),          # two workgroups to a compute unit
    (4, 24, 8, 300, 300, 64, None, ROWS_128),           # three
    (3, 32, 32, 129, 31, 64, None, ROWS_128),           # one row in the second workgroup, less than a sub-tile
    (3, 32, 32, 129, 65, 64, None, ROWS_128),           # one key in the second tile
    (3, 32, 32, 129, 193, 64, 64, ROWS_128),            # a ring of three tiles once round, and one key more
    (3, 32, 32, 140, 257, 64, 117, ROWS_128),
    (3, 32, 32, 140, 161, 128, 21, ROWS_64_GROUPS),
    (4, 32, 32, 140, 161, 128, 21, ROWS_128),           # a ring of four tiles of 32 keys once round, and one more
    (4, 32, 32, 140, 129, 128, None, ROWS_128),         # one key in the fifth tile
    (3, 32, 32, 250, 700, 128, 500, ROWS_128_GROUPS),   # inner tiles, keys that no row sees
    (4, 32, 32, 250, 700, 128, 500, ROWS_128),
    (3, 32, 32, 250, 700, 64, -100, ROWS_128),          # rows without any key
    (1, 64, 16, 1024, 1024, 64, 0, ROWS_128),
    (1, 64, 16, 1024, 1024, 128, 0, ROWS_128),
])
def test_small_workgroups(lib, B, Hq, Hkv, Sq, Sk, D, off, shape):
    assert attn_shape(lib, STEP_F32, B, Hq, Hkv, Sq, Sk, D, off) == shape
    q, k, v = (bits_to_dev(rand_bits((B, h, S, D), 740 + i)) for i, (h, S) in enumerate(((Hq, Sq), (Hkv, Sk), (Hkv, Sk))))
    out, lse = _new(B, Hq, Sq, D)
    if off is None:
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, D ** -0.5, out, lse)
    else:
        lib.tr_block_attn_causal_at(q, k, v, max(off, 0), max(-off, 0), D ** -0.5, out, lse)
    torch.cuda.synchronize()
    want_o, want_l = _exact(q, k, v, off)
    assert torch.equal(torch.isneginf(lse), torch.isneginf(want_l))
    seen = ~torch.isneginf(want_l)
    assert float((out - want_o).abs().max()) <= 1e-2 and float((lse - want_l)[seen].abs().max()) <= 1e-5   # as for every block step


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_bf16_blocks_of_small_workgroups(lib, D, causal):
    """96 heads of 3 chunks of 300 rows in the chunk form."""
    B, H, chunk, n = 4, 24, 300, 3
    assert attn_shape(lib, RING_BF16, B, H, H, chunk * n, chunk * n, D, 0 if causal else None, n) == ROWS_128
    q, k, v = (bits_to_dev(rand_bits((B, H, chunk * n, D), 760 + i)) for i in range(3))
    out, lse = _new(B, H, chunk * n, D)
    ws = torch.empty(lib.tr_ring_attn_blocks_workspace_bytes(q, n, lib.TR_BF16), dtype=torch.uint8, device="cuda")
    lib.tr_ring_attn_blocks(q, k, v, n, causal, out, lse, lib.TR_BF16, ws, D ** -0.5)
    torch.cuda.synchronize()
    want_o, want_l = _exact(q, k, v, 0 if causal else None)
    # a bf16 rounding of each later block on top of a block step's distance
    assert float((out - want_o).abs().max()) <= 1e-2 + 2 ** -8 * float(v.abs().max()) and float((lse - want_l).abs().max()) <= 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, None])   # None: merged into accumulators
@pytest.mark.parametrize("Hq,Hkv,Sq,Sk,D,off,shape", [
    (1, 1, 1, 1, 64, None, ROWS_256),
    (2, 1, 31, 33, 128, None, ROWS_256),           # one sub-tile and one key
    (2, 2, 64, 64, 64, 0, ROWS_256),
    (2, 2, 129, 97, 128, None, ROWS_64_GROUPS),    # an odd sub-tile of one key, the second key group's
    (1, 1, 130, 500, 128, 370, ROWS_64_GROUPS),    # causal, the last row sees the last key
    (3, 3, 70, 129, 64, 20, ROWS_256),             # keys that no row sees
    (2, 1, 200, 450, 128, -90, ROWS_64_GROUPS),    # rows that see none
    (12, 4, 500, 512, 64, 12, ROWS_64_GROUPS),
    (16, 8, 700, 300, 128, None, ROWS_64_GROUPS),
    (32, 32, 624, 738, 64, None, ROWS_128_GROUPS),
    (32, 32, 612, 964, 128, 352, ROWS_128_GROUPS),
])
def test_steps(lib, Hq, Hkv, Sq, Sk, D, off, shape, dtype):
    if dtype is None and off is not None:
        pytest.skip("the merging step has no causal rule at arbitrary positions")
    q, k, v = _qkv(Hq, Hkv, Sq, Sk, D, 720, True)
    B = -(-MANY // (Hq * -(-Sq // 256)))
    form = {None: STEP_MERGE, torch.float32: STEP_F32, torch.bfloat16: STEP_BF16}[dtype]
    assert attn_shape(lib, form, 1, Hq, Hkv, Sq, Sk, D, off) == shape and attn_shape(lib, form, B, Hq, Hkv, Sq, Sk, D, off) == ROWS_128

    def run(B, q, k, v):
        out, lse = _new(B, Hq, Sq, D, dtype or torch.float32)
        if dtype is None:
            gen = torch.Generator(device="cuda").manual_seed(5)
            out.copy_(torch.randn((1, Hq, Sq, D), device="cuda", generator=gen))
            lse.copy_(torch.randn((1, Hq, Sq), device="cuda", generator=gen) * 4)
            lse[:, 0, 0] = float("-inf")
            out[:, 0, 0] = float("nan")
            lib.tr_block_attn_merge(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
        elif off is None:
            lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
        else:
            lib.tr_block_attn_causal_at(q, k, v, max(off, 0), max(-off, 0), 0.1, out, lse)
        return out, lse

    few, many = run(1, q, k, v), run(B, *(x.expand(B, -1, -1, -1) for x in (q, k, v)))
    torch.cuda.synchronize()
    _agree(few, many, 2 ** -8 * 4 if dtype is torch.bfloat16 else 1e-5)   # a bf16 ulp of values below 4, where a sum lies at a tie


@pytest.mark.parametrize("merge", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,off,parts", [
    (4, 3, 1, 935, 1385, 128, None, 3),
    (1, 12, 4, 1611, 1611, 128, 0, 3),
    (1, 16, 16, 1594, 2428, 64, 834, 2),
    (2, 4, 2, 2272, 2339, 128, 67, 3),
    (1, 8, 8, 2900, 2900, 128, 0, 2),
])
def test_uncut_calls_round_as_their_parts(lib, B, Hq, Hkv, Sq, Sk, D, off, parts, merge):
    """Block steps that workgroups of fewer rows run in one piece: the weights are those of the parts that 256-row ones would cut
    the keys into, attended one by one here (none of them as large as to be cut again), so that fp32 sums are all that differs."""
    assert attn_plan(lib, B, Hq, Hkv, Sq, Sk, D, off) == (1, 0)
    if merge and off is not None:
        pytest.skip("the merging step has no causal rule at arbitrary positions")
    q, k, v = (bits_to_dev(rand_bits((B, h, S, D), 790 + i)) for i, (h, S) in enumerate(((Hq, Sq), (Hkv, Sk), (Hkv, Sk))))

    def step(k, v, k0, out, lse):
        if merge:
            out.fill_(float("nan"))
            lse.fill_(float("-inf"))
            lib.tr_block_attn_merge(q, k, v, lib.TR_MASK_NONE, D ** -0.5, out, lse)
        elif off is None:
            lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, D ** -0.5, out, lse)
        else:
            lib.tr_block_attn_causal_at(q, k, v, off, k0, D ** -0.5, out, lse)

    whole = _new(B, Hq, Sq, D)
    step(k, v, 0, *whole)
    keys = max(512, -(-Sk // parts) + 127 & -128)
    outs, lses = zip(*(_new(B, Hq, Sq, D) for _ in range(parts)))
    for i in range(parts):
        part = slice(i * keys, (i + 1) * keys)
        assert attn_plan(lib, B, Hq, Hkv, Sq, k[:, :, part].shape[2], D, off if off is None else off - i * keys) == (1, 0)
        step(k[:, :, part], v[:, :, part], i * keys, outs[i], lses[i])
    folded = _new(B, Hq, Sq, D)
    lib.tr_merge_n(*folded, list(outs), list(lses))
    torch.cuda.synchronize()
    for b in range(B):
        _agree([x[b:b + 1] for x in whole], [x[b:b + 1] for x in folded])


def test_more_rows_than_a_grid_of_small_workgroups_holds(lib):
    """65536 workgroups of 128 rows are one too many for a grid's second dimension; 32769 of 256 rows are not."""
    S, D = 65536 * 128 + 5, 64
    q = torch.randn((1, 1, S, D), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).bfloat16()
    k, v = (bits_to_dev(rand_bits((1, 1, 3, D), 770 + i)) for i in range(2))
    out, lse = torch.full((1, 1, S, D), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.full((1, 1, S), float("nan"), device="cuda")
    lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, D ** -0.5, out, lse)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(lse).all())
    for r in (slice(0, 300), slice(S // 2 - 200, S // 2 + 200), slice(S - 300, S)):
        want_o, want_l = _exact(q[:, :, r], k, v, None)
        assert float((out[:, :, r] - want_o).abs().max()) <= 1e-2 * 2 and float((lse[:, :, r] - want_l).abs().max()) <= 1e-5   # (and bf16's rounding of values to 4)


def test_scores_beyond_the_fast_path(lib):
    """Scores 40 wide: references are raised per key group and the groups' sums meet at different ones."""
    S, D = 320, 64
    q, k, v = _qkv(2, 2, S, S, D, 730)
    q, k = (q.float() * 6).bfloat16(), (k.float() * 6).bfloat16()
    out, lse = _new(1, 2, S, D)
    lib.tr_ring_attn(q, k, v, 1, False, out, lse)
    torch.cuda.synchronize()
    s = (q.double() * D ** -0.5) @ k.double().transpose(-1, -2).contiguous()
    want = torch.softmax(s, -1) @ v.double()
    # all weight on a few keys: 2^-8 of the largest value
    assert float((out - want).abs().max()) <= 2 ** -8 * float(v.abs().max()) * 1.02 + 1e-4
    assert float((lse - torch.logsumexp(s, -1)).abs().max()) <= 1e-3
