"""tr_ring_attn_blocks with bf16 blocks against Algorithm 1 spelled out by the caller: tr_block_attn into a bf16
block_out (the first block of a chunk straight into the accumulators), tr_merge after it, in the schedule's
order.  The same bits where both share the keys out alike (the number of key groups, asserted; with another one fp32 sums differ,
and so does what is rounded to bf16).  Chunk lengths sit around tiles; up to 512 keys a block step is one pass over its keys."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import RING_BF16, STEP_BF16, STEP_F32, attn_shape, bits_to_dev, rand_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,chunk,n,D,token", [
    (1, 2, 2, 1, 5, 64, False),        # chunks of one row
    (2, 6, 2, 24, 7, 64, True),        # less than a wave, token-major
    (1, 4, 2, 256, 4, 128, False),     # exactly one query tile
    (1, 3, 3, 257, 3, 64, False),      # one row in the second tile
    (1, 8, 8, 400, 3, 128, True),      # XCD-aware placement, ragged tiles
    (1, 2, 1, 320, 1, 128, False),     # a single chunk: nothing is merged
])
def test_bf16_blocks_are_the_steps_one_by_one(lib, B, Hq, Hkv, chunk, n, D, token, causal):
    S, off = chunk * n, 0 if causal else None
    groups = {attn_shape(lib, RING_BF16, B, Hq, Hkv, S, S, D, off, n)[1], attn_shape(lib, STEP_F32, B, Hq, Hkv, chunk, chunk, D, off)[1]}
    groups |= {attn_shape(lib, STEP_BF16, B, Hq, Hkv, chunk, chunk, D)[1]} if n > 1 else set()
    assert len(groups) == 1 or chunk <= 32               # (a sub-tile belongs to one group)
    _same_bits(lib, B, Hq, Hkv, chunk, n, D, token, causal)


@pytest.mark.parametrize("B,Hq,Hkv,chunk,n,D,token,causal,shape", [
    (16, 16, 16, 20, 3, 64, False, True, (128, 1)),     # no wave has 32 rows
    (4, 24, 24, 45, 3, 64, False, False, (128, 1)),     # one that has, one of 13
    (8, 24, 8, 45, 3, 64, True, True, (128, 1)),
    (4, 24, 24, 45, 3, 128, True, False, (128, 1)),
    (8, 24, 24, 45, 3, 128, False, True, (128, 1)),
    (8, 40, 10, 131, 4, 64, True, False, (128, 1)),     # three rows in the second workgroup
    (8, 40, 10, 131, 4, 128, False, True, (128, 1)),
    (2, 48, 48, 257, 3, 64, False, True, (128, 1)),
    (4, 40, 40, 127, 2, 64, True, True, (256, 1)),      # half of the waves have no rows
    (4, 40, 40, 128, 2, 64, False, True, (256, 1)),
    (4, 32, 8, 128, 2, 128, False, False, (256, 1)),
    (1, 40, 8, 768, 2, 128, True, False, (256, 1)),
    (4, 30, 30, 127, 4, 128, False, True, (256, 1)),
    (4, 40, 40, 90, 3, 128, True, True, (256, 1)),
])
def test_updates_in_the_lanes_are_the_steps_one_by_one(lib, B, Hq, Hkv, chunk, n, D, token, causal, shape):
    """One key group on either side: between two blocks the accumulators lie in the result as they lie in the lanes."""
    S, off = chunk * n, 0 if causal else None
    assert attn_shape(lib, RING_BF16, B, Hq, Hkv, S, S, D, off, n) == shape
    assert attn_shape(lib, STEP_F32, B, Hq, Hkv, chunk, chunk, D, off)[1] == attn_shape(lib, STEP_BF16, B, Hq, Hkv, chunk, chunk, D)[1] == 1
    _same_bits(lib, B, Hq, Hkv, chunk, n, D, token, causal)


def _same_bits(lib, B, Hq, Hkv, chunk, n, D, token, causal):
    S, scale = chunk * n, 1.0 / np.sqrt(D)

    def tensor(H, seed):
        x = rand_bits((B, H, S, D), seed)
        return bits_to_dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3))).permute(0, 2, 1, 3) if token else bits_to_dev(x)

    q, k, v = tensor(Hq, 400), tensor(Hkv, 401), tensor(Hkv, 402)
    new = lambda S: (torch.full((B, Hq, S, D), float("nan"), device="cuda"), torch.full((B, Hq, S), float("nan"), device="cuda"))
    out, lse = new(S)
    ws = torch.empty(lib.tr_ring_attn_blocks_workspace_bytes(q, n, lib.TR_BF16), dtype=torch.uint8, device="cuda")
    lib.tr_ring_attn_blocks(q, k, v, n, causal, out, lse, lib.TR_BF16, ws, scale)

    ref_o, ref_l = new(S)
    blk_o, blk_l = torch.empty((B, Hq, chunk, D), dtype=torch.bfloat16, device="cuda"), torch.empty((B, Hq, chunk), device="cuda")
    part = lambda t, c: t[:, :, c * chunk:(c + 1) * chunk]
    seen = set()
    for _, j, c in oracle.ring_schedule(n, causal):
        mask = lib.TR_MASK_CAUSAL_DIAG if causal and j == c else lib.TR_MASK_NONE
        o, l = (blk_o, blk_l) if c in seen else (part(ref_o, c), part(ref_l, c))
        lib.tr_block_attn(part(q, c), part(k, j), part(v, j), mask, scale, o, l)
        if c in seen:
            lib.tr_merge(part(ref_o, c), part(ref_l, c), blk_o, blk_l)
        seen.add(c)
    torch.cuda.synchronize()
    assert torch.equal(out, ref_o) and torch.equal(lse, ref_l)


@pytest.mark.parametrize("causal,n,B,D", [(False, 1, 1, 64), (True, 3, 1, 64), (True, 3, 150, 64), (True, 2, 150, 128)])   # from 150 on one key group
def test_a_first_block_is_stored_as_it_is(lib, causal, n, B, D):
    chunk = 96
    assert n == 1 or attn_shape(lib, RING_BF16, B, 2, 1, chunk * n, chunk * n, D, 0, n)[1] == (2 if B == 1 else 1)
    q, k, v = (bits_to_dev(rand_bits((B, h, chunk * n, D), 530 + i)) for i, h in enumerate((2, 1, 1)))
    q[0, 1, 7, 0] = float("nan")                         # a row that meets one block only (chunk 0)
    out, lse = torch.zeros((B, 2, chunk * n, D), device="cuda"), torch.zeros((B, 2, chunk * n), device="cuda")
    ws = torch.empty(lib.tr_ring_attn_blocks_workspace_bytes(q, n, lib.TR_BF16), dtype=torch.uint8, device="cuda")
    lib.tr_ring_attn_blocks(q, k, v, n, causal, out, lse, lib.TR_BF16, ws, 0.1)
    torch.cuda.synchronize()
    assert torch.isnan(out[0, 1, 7]).all() and bool(torch.isneginf(lse[0, 1, 7]))
    keep = torch.ones((2, chunk * n), dtype=torch.bool, device="cuda")
    keep[1, 7] = False
    assert torch.isfinite(out[0][keep]).all() and torch.isfinite(lse[0][keep]).all()
    assert torch.isfinite(out[1:]).all() and torch.isfinite(lse[1:]).all()
