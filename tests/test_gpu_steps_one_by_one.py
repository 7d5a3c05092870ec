"""Algorithm 1 spelled out by the caller with fp32 blocks: tr_block_attn and tr_merge, or tr_block_attn_merge, chunk by chunk in
the schedule's order, against the fp64 oracle and against the ring entry points, which run the same schedule as one
launch and round the same weights (whole segments of sub-tiles: only fp32 sums differ).  Chunks of sixteen and twelve tiles reach the
kernel's inner-tile loop at either head dim.  A workspace handed to a ring is left alone."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import attn_plan, bits_to_dev, f64, max_abs, rand_bits, to_np

pytestmark = pytest.mark.gpu
OUT_TOL, LSE_TOL = 1e-2, 1e-3


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,chunk,n,D", [
    (2, 4, 2, 96, 4, 128),
    (1, 3, 1, 160, 3, 64),
    (1, 12, 4, 1024, 2, 128),
    (1, 20, 10, 1536, 2, 64),
])
def test_steps_one_by_one_and_the_ring_agree(lib, B, Hq, Hkv, chunk, n, D, causal):
    S, scale = chunk * n, 1.0 / np.sqrt(D)
    assert attn_plan(lib, B, Hq, Hkv, chunk, chunk, D)[0] == attn_plan(lib, B, Hq, Hkv, chunk, chunk, D, 0)[0] == 1   # steps in one piece, like the ring
    qb, kb, vb = (rand_bits((B, h, S, D), 640 + i) for i, h in enumerate((Hq, Hkv, Hkv)))
    q, k, v = bits_to_dev(qb), bits_to_dev(kb), bits_to_dev(vb)
    ref_o, ref_l = oracle.attention_full(f64(qb), f64(kb), f64(vb), scale, causal)
    new = lambda S: (torch.full((B, Hq, S, D), float("nan"), device="cuda"), torch.full((B, Hq, S), float("nan"), device="cuda"))
    part = lambda t, c: t[:, :, c * chunk:(c + 1) * chunk]
    two, fused, (blk_o, blk_l) = new(S), new(S), new(chunk)
    two[1].fill_(float("-inf"))                          # empty accumulators, out uninitialised
    fused[1].fill_(float("-inf"))
    for _, j, c in oracle.ring_schedule(n, causal):
        mask = lib.TR_MASK_CAUSAL_DIAG if causal and j == c else lib.TR_MASK_NONE
        lib.tr_block_attn(part(q, c), part(k, j), part(v, j), mask, scale, blk_o, blk_l)
        lib.tr_merge(part(two[0], c), part(two[1], c), blk_o, blk_l)
        lib.tr_block_attn_merge(part(q, c), part(k, j), part(v, j), mask, scale, part(fused[0], c), part(fused[1], c))
    ring, given, noalloc = new(S), new(S), new(S)
    lib.tr_ring_attn(q, k, v, n, causal, *ring, scale)
    ws = torch.full((lib.tr_ring_attn_workspace_bytes(q, n),), 171, dtype=torch.uint8, device="cuda")
    lib.tr_ring_attn(q, k, v, n, causal, *given, scale, ws)
    lib.tr_ring_attn_noalloc(q, k, v, n, causal, *noalloc, scale)
    torch.cuda.synchronize()
    assert bool((ws == 171).all())
    for o, l in (two, fused, ring, given, noalloc):
        assert max_abs(to_np(o), ref_o) <= OUT_TOL and max_abs(to_np(l), ref_l) <= LSE_TOL
    for o, l in (given, noalloc):
        assert torch.equal(o, ring[0]) and torch.equal(l, ring[1])
    # the same weights, fp32 sums in another order: a few 2^-23 of values of size 1 (out) and 10 (lse), measured 7e-7 and 2e-6
    worst = [max_abs(to_np(x), to_np(y)) for o, l in (two, fused) for x, y in ((o, ring[0]), (l, ring[1]))]
    print("steps against ring (out, lse; two kernels, fused):", worst)
    assert max(worst) <= 1e-5
