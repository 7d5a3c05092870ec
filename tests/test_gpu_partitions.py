"""Attention on grids that leave the chip idle: keys cut into parts, grouped query heads packed into one row space.

Sizes sit where the form can go wrong: row counts around a wave and a tile, a last part of one key, parts
that no row of a tile sees, heads that share a wave; the expected form, and the shape of the workgroups, stand beside each.  Reference: the fp64 oracle, tolerances as for every
block step.  Without scratch (under graph capture, on a stream beyond those that have a region) the keys are one piece.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import STEP_BF16, STEP_F32, STEP_MERGE, attn_plan, attn_shape, bits_to_dev, f64, max_abs, rand_bits, to_np

pytestmark = pytest.mark.gpu
OUT_TOL, LSE_TOL = 1e-2, 1e-3

FORMS = {
    # B, Hq, Hkv, Sq, Sk, D, offset of the causal rule (None: no mask): parts of the keys, packed heads
    (1, 8, 1, 1, 4097, 128, None): (9, 1),        # decode: eight heads in one wave, last part of one key
    (2, 6, 2, 11, 1500, 64, None): (3, 1),        # three heads, 33 rows: one row in the second wave
    (1, 4, 1, 64, 3000, 128, None): (6, 1),       # 256 packed rows: exactly a tile
    (1, 3, 1, 86, 2049, 64, None): (5, 1),        # 258 packed rows: two in the second tile
    (1, 2, 2, 300, 8192, 128, None): (16, 0),     # no packing, two tiles, sixteen parts
    (1, 4, 2, 40, 2600, 128, 2560): (6, 1),       # causal, packed heads that share waves
    (1, 4, 1, 300, 1100, 128, 744): (3, 1),       # causal, packed: a tile whose rows see two of three parts
    (1, 8, 1, 600, 1600, 64, 1000): (4, 1),       # the same over several tiles of a head
    (1, 2, 2, 2048, 2048, 64, 0): (4, 0),         # diagonal: early tiles see one part only
    (1, 2, 1, 20, 4000, 128, 2100): (5, 1),       # later keys that no row sees
    (1, 2, 2, 1600, 2500, 128, -300): (3, 0),     # rows without any key, and a tile with one part
    (1, 2, 2, 2600, 2300, 64, -300): (5, 0),
    (40, 8, 1, 1, 300, 64, None): (1, 1),         # one piece, packed for one round of workgroups instead of two
    (30, 12, 4, 30, 500, 128, 480): (1, 1),       # the same, causal, three heads in 90 rows
    (9, 32, 8, 300, 330, 64, 20): (1, 1),         # the same, a tile that ends one head and starts the next
    (66, 32, 8, 2, 70, 64, None): (1, 1),         # more than two rounds of packed tiles
    (1, 32, 8, 73, 5186, 64, None): (11, 1),      # 256-row workgroups, packed: 292 rows
    (8, 8, 1, 53, 4110, 128, 4057): (9, 1),       # the same, causal: 424 rows of eight heads
    (2, 12, 4, 135, 4095, 128, 3960): (8, 1),     # 128-row workgroups, packed, causal: 405 rows of three heads
    (2, 4, 4, 299, 5172, 64, None): (11, 0),      # not packed: 43 rows in the second tile
    (1, 8, 8, 388, 4460, 128, 4072): (9, 0),      # the same, causal
    (3, 6, 3, 129, 2825, 128, None): (6, 0),      # 128-row workgroups: one row in the second
    (4, 6, 2, 45, 6006, 128, None): (12, 1),      # the same, packed: 135 rows
    (1, 16, 16, 133, 2797, 128, 2664): (6, 0),    # 128 rows and two key groups, causal
    (4, 12, 4, 43, 2730, 128, None): (6, 1),      # the same, packed: 129 rows
    (1, 32, 16, 68, 2637, 128, 2569): (6, 1),     # the same, causal: 136 rows of two heads
}
CASES = list(FORMS)
ROWS_256, ROWS_128, ROWS_128_GROUPS, ROWS_64_GROUPS = (256, 1), (128, 1), (128, 2), (64, 2)    # Query rows of a workgroup, key groups
SHAPES = dict.fromkeys(CASES, ROWS_64_GROUPS)
SHAPES.update({
    (1, 8, 1, 600, 1600, 64, 1000): ROWS_128,
    (1, 2, 2, 2600, 2300, 64, -300): ROWS_128_GROUPS,
    (30, 12, 4, 30, 500, 128, 480): ROWS_256,
    (9, 32, 8, 300, 330, 64, 20): ROWS_128,
    (66, 32, 8, 2, 70, 64, None): ROWS_128,
    (1, 32, 8, 73, 5186, 64, None): ROWS_256,
    (8, 8, 1, 53, 4110, 128, 4057): ROWS_256,
    (2, 12, 4, 135, 4095, 128, 3960): ROWS_128,
    (2, 4, 4, 299, 5172, 64, None): ROWS_256,
    (1, 8, 8, 388, 4460, 128, 4072): ROWS_256,
    (3, 6, 3, 129, 2825, 128, None): ROWS_128,
    (4, 6, 2, 45, 6006, 128, None): ROWS_128,
    (1, 16, 16, 133, 2797, 128, 2664): ROWS_128_GROUPS,
    (4, 12, 4, 43, 2730, 128, None): ROWS_128_GROUPS,
    (1, 32, 16, 68, 2637, 128, 2569): ROWS_128_GROUPS,
})


def _inputs(case, seed):
    B, Hq, Hkv, Sq, Sk, D, _ = case
    return rand_bits((B, Hq, Sq, D), seed), rand_bits((B, Hkv, Sk, D), seed + 1), rand_bits((B, Hkv, Sk, D), seed + 2)


def _attend(lib, case, q, k, v, scale, out, lse, stream=None):
    off = case[6]
    if off is None:
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, scale, out, lse, stream)
    else:
        lib.tr_block_attn_causal_at(q, k, v, max(off, 0), max(-off, 0), scale, out, lse, stream)


def _reference(case, qb, kb, vb, scale):
    off = case[6]
    if off is None:
        return oracle.attention_block(f64(qb), f64(kb), f64(vb), scale)
    return oracle.attention_block(f64(qb), f64(kb), f64(vb), scale, causal_diag=True, q_offset=max(off, 0), k_offset=max(-off, 0))


@pytest.mark.parametrize("case", CASES, ids=str)
def test_the_cases_take_the_forms_they_stand_for(lib, case):
    assert attn_plan(lib, *case) == FORMS[case]
    assert {attn_shape(lib, form, *case) for form in (STEP_BF16, STEP_F32, STEP_MERGE)} == {SHAPES[case]}


def test_parts_of_small_workgroups_that_scratch_does_not_hold(lib):
    """136 rows are 160 of a 256-row workgroup's slot and 256 of two 128-row ones: 144 heads in 5 parts fit the 33 MiB of a region
    only in the first form, which the call goes back to (96 heads take 128 rows)."""
    B, H, Sq, Sk, D = 6, 24, 136, 29362, 64
    assert attn_plan(lib, 4, H, H, Sq, Sk, D) == (5, 0) and attn_shape(lib, STEP_F32, 4, H, H, Sq, Sk, D) == ROWS_128
    assert attn_plan(lib, B, H, H, Sq, Sk, D) == (5, 0) and attn_shape(lib, STEP_F32, B, H, H, Sq, Sk, D) == ROWS_256
    assert B * H * 5 * 160 * (D + 1) * 4 <= 33 << 20 < B * H * 5 * 256 * (D + 1) * 4
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.randn((B, H, S, D), device="cuda", generator=gen).bfloat16() for S in (Sq, Sk, Sk))
    out, lse = torch.full((B, H, Sq, D), float("nan"), device="cuda"), torch.full((B, H, Sq), float("nan"), device="cuda")
    lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, D ** -0.5, out, lse)
    torch.cuda.synchronize()
    for b in range(B):
        s = (q[b].double() * D ** -0.5) @ k[b].double().transpose(-1, -2).contiguous()
        want_l = torch.logsumexp(s, -1)
        want_o = torch.exp(s - want_l[..., None]) @ v[b].double()
        assert float((out[b] - want_o).abs().max()) <= OUT_TOL and float((lse[b] - want_l).abs().max()) <= LSE_TOL


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_parts_reach_the_oracle(lib, case, out_dtype):
    B, Hq, Hkv, Sq, Sk, D, _ = case
    qb, kb, vb = _inputs(case, 300)
    scale = 1.0 / np.sqrt(D)
    # token-major tensors: head and row strides change places
    q, k, v = (bits_to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3))).permute(0, 2, 1, 3) for x in (qb, kb, vb))
    out = torch.full((B, Sq, Hq, D), float("nan"), dtype=out_dtype, device="cuda").permute(0, 2, 1, 3)
    lse = torch.full((B, Hq, Sq), float("nan"), dtype=torch.float32, device="cuda")
    _attend(lib, case, q, k, v, scale, out, lse)
    torch.cuda.synchronize()
    ref_o, ref_l = _reference(case, qb, kb, vb, scale)
    assert np.array_equal(np.isneginf(to_np(lse)), np.isneginf(ref_l))
    assert max_abs(to_np(out), ref_o) <= OUT_TOL and max_abs(to_np(lse), ref_l) <= LSE_TOL


@pytest.mark.parametrize("case", [c for c in CASES if c[6] is None or c[3] == c[4]], ids=str)
def test_parts_merge_into_accumulators(lib, case):
    B, Hq, Hkv, Sq, Sk, D, off = case
    mask = lib.TR_MASK_NONE if off is None else lib.TR_MASK_CAUSAL_DIAG
    qb, kb, vb = _inputs(case, 330)
    rng = np.random.default_rng(333)
    acc_o = rng.standard_normal((B, Hq, Sq, D)).astype(np.float32)
    acc_l = rng.uniform(-5, 15, (B, Hq, Sq)).astype(np.float32)
    acc_l[:, 0, 0] = -np.inf
    clean = acc_o.copy()
    clean[:, 0, 0] = 0.0
    acc_o[:, 0, 0] = np.nan                                # an empty row may hold garbage
    d_o, d_l = torch.from_numpy(acc_o).cuda(), torch.from_numpy(acc_l).cuda()
    lib.tr_block_attn_merge(bits_to_dev(qb), bits_to_dev(kb), bits_to_dev(vb), mask, 0.1, d_o, d_l)
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.merge_pair(clean, acc_l, *_reference(case, qb, kb, vb, 0.1))
    assert max_abs(to_np(d_o), ref_o) <= OUT_TOL and max_abs(to_np(d_l), ref_l) <= LSE_TOL


@pytest.mark.parametrize("form", ["bf16", "fp32", "merge"])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_without_scratch_the_result_is_the_same_up_to_rounding(lib, case, form):
    """More streams at a time than have a scratch region, and a captured call: one pass over all keys, to the oracle's
    tolerance; the replays of a graph agree bitwise."""
    if form == "merge" and case[6] is not None and case[3] != case[4]:
        pytest.skip("the merging step has no causal rule at arbitrary positions")
    B, Hq, Hkv, Sq, Sk, D, _ = case
    bits = _inputs(case, 360)
    q, k, v = (bits_to_dev(x) for x in bits)
    ref_o, ref_l = _reference(case, *bits, 0.1)
    dtype = torch.bfloat16 if form == "bf16" else torch.float32
    empty = float("-inf") if form == "merge" else float("nan")     # merge: onto an empty accumulator that holds garbage

    def new():
        return torch.full((B, Hq, Sq, D), float("nan"), dtype=dtype, device="cuda"), torch.full((B, Hq, Sq), empty, device="cuda")

    def run(out, lse, stream=None):
        if form == "merge":
            mask = lib.TR_MASK_NONE if case[6] is None else lib.TR_MASK_CAUSAL_DIAG
            lib.tr_block_attn_merge(q, k, v, mask, 0.1, out, lse, stream)
        else:
            _attend(lib, case, q, k, v, 0.1, out, lse, stream)

    def check(out, lse):
        assert np.array_equal(np.isneginf(to_np(lse)), np.isneginf(ref_l))
        assert max_abs(to_np(out), ref_o) <= OUT_TOL and max_abs(to_np(lse), ref_l) <= LSE_TOL

    streams = [torch.cuda.Stream() for _ in range(6)]
    results = [new() for _ in streams]
    torch.cuda.synchronize()
    for s, (o, l) in zip(streams, results):
        run(o, l, s)
    torch.cuda.synchronize()
    for o, l in results:
        check(o, l)
    graph_o, graph_l = new()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(graph_o, graph_l)
    first = None
    for _ in range(3):
        graph_o.fill_(float("nan")); graph_l.fill_(empty)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(graph_o, graph_l)
        first = first or (graph_o.clone(), graph_l.clone())
        assert torch.equal(graph_o, first[0]) and torch.equal(graph_l, first[1])
