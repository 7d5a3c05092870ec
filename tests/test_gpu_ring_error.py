"""The ring entry points are no further from 64-bit attention than the block steps they stand for: tr_block_attn into
fp32 blocks and tr_merge, chunk by chunk in the schedule's order.  Every block has an exponent reference of its own,
so that its largest weights reach the PV product unrounded; one reference for a whole sequence costs 14 % at four
chunks of 64 keys and 50 % at sixteen of 16.  Both sides round the same weights, so 2 % is left for the fp32 sums."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import bits_to_dev, rand_bits

pytestmark = pytest.mark.gpu


def _exact(q, k, v, scale, causal):
    B, Hq, S, D = q.shape
    out = torch.empty(q.shape, dtype=torch.float64)
    for h in range(Hq):
        g = h // (Hq // k.shape[1])
        s = (q[:, h].double().cpu() * scale) @ k[:, g].double().cpu().transpose(1, 2)
        if causal:
            s = s.masked_fill(torch.ones((S, S), dtype=torch.bool).triu(1), float("-inf"))
        out[:, h] = torch.softmax(s, -1) @ v[:, g].double().cpu()
    return out


def _distance(x, exact):
    return float(((x.double().cpu() - exact).square().sum() / exact.square().sum()).sqrt())


@pytest.mark.parametrize("entry", ["ring", "blocks", "zigzag"])
@pytest.mark.parametrize("Hq,Hkv,chunk,n,D,causal,std", [
    (2, 2, 64, 4, 64, False, 1.0),
    (2, 1, 64, 8, 128, True, 1.0),
    (4, 4, 16, 16, 128, False, 1.0),  # chunks shorter than a sub-tile
    (4, 2, 23, 12, 64, True, 1.0),
    (4, 4, 40, 8, 128, False, 1.0),   # sub-tiles that hold the end of one chunk and the start of the next
    (2, 2, 100, 6, 64, True, 1.0),
    (2, 2, 256, 4, 128, False, 1.0),
    (1, 1, 512, 8, 128, True, 1.0),   # renewed between groups of inner tiles
    (1, 1, 768, 4, 64, False, 4.0),   # scores 16 wide: references that are not lowered, and sums beyond the fast path's
])
def test_ring_is_as_exact_as_its_block_steps(lib, entry, Hq, Hkv, chunk, n, D, causal, std):
    if entry == "zigzag" and (not causal or n % 2):
        pytest.skip("the zigzag partition is causal and has an even number of segments")
    S, scale = chunk * n, 1.0 / np.sqrt(D)
    q, k, v = (bits_to_dev(rand_bits((2, h, S, D), 540 + i, std if i < 2 else 1.0)) for i, h in enumerate((Hq, Hkv, Hkv)))
    out, lse = torch.empty((2, Hq, S, D), device="cuda"), torch.empty((2, Hq, S), device="cuda")
    if entry == "ring":
        lib.tr_ring_attn(q, k, v, n, causal, out, lse, scale)
    elif entry == "blocks":
        ws = torch.empty(lib.tr_ring_attn_blocks_workspace_bytes(q, n, lib.TR_F32), dtype=torch.uint8, device="cuda")
        lib.tr_ring_attn_blocks(q, k, v, n, causal, out, lse, lib.TR_F32, ws, scale)
    else:
        lib.tr_ring_attn_sched(q, k, v, n // 2, True, lib.TR_SCHED_ZIGZAG, out, lse, scale)

    acc_o, acc_l = torch.empty_like(out), torch.full_like(lse, float("-inf"))
    blk_o, blk_l = torch.empty((2, Hq, chunk, D), device="cuda"), torch.empty((2, Hq, chunk), device="cuda")
    part = lambda t, c: t[:, :, c * chunk:(c + 1) * chunk]
    for _, j, c in oracle.ring_schedule(n, causal):
        mask = lib.TR_MASK_CAUSAL_DIAG if causal and j == c else lib.TR_MASK_NONE
        lib.tr_block_attn(part(q, c), part(k, j), part(v, j), mask, scale, blk_o, blk_l)
        lib.tr_merge(part(acc_o, c), part(acc_l, c), blk_o, blk_l)
    exact = _exact(q, k, v, scale, causal)
    ring, steps = _distance(out, exact), _distance(acc_o, exact)
    print(f"ring {ring:.4e}, block steps {steps:.4e}")
    assert ring <= 1.02 * steps
    # fp32 sums of the same unrounded weights; a score of size s is itself rounded to s * 2^-23 or so
    assert float((lse - acc_l).abs().max()) <= 1e-5 * max(1.0, float(acc_l.abs().max()) / 8)
