"""Query rows on their way into registers, and Updates that stay in the lanes between two blocks: row counts around the row groups and
tiles of a workgroup, few and many keys, dense and token-major rows, against the same operation in 64 bits.  Out to 1e-2 and lse
to 1e-3 (bf16 weights); blocks rounded to bf16 add 2^-8 of the largest value for each that is merged (test_gpu_block_transport.py compares their
bits).  The shape that a case stands for is asserted."""
import math

import pytest
import torch

from gpu_util import RING_BF16, STEP_F32, attn_plan, attn_shape

pytestmark = pytest.mark.gpu


def rows(gen, B, H, S, D, token):
    if token:
        wide = torch.randn((B, S, H + 1, D), device="cuda", dtype=torch.bfloat16, generator=gen)   # a row of other heads between two rows
        return wide[:, :, :H].permute(0, 2, 1, 3)
    return torch.randn((B, H, S, D), device="cuda", dtype=torch.bfloat16, generator=gen)


def attend(q, k, v, scale, causal):
    g = q.shape[1] // k.shape[1]
    k, v = (x.double().repeat_interleave(g, 1).contiguous() for x in (k, v))
    s = torch.matmul(q.double().contiguous() * scale, k.transpose(2, 3).contiguous())
    if causal:
        past = k.shape[2] - q.shape[2]
        keep = torch.arange(k.shape[2], device="cuda")[None, :] <= torch.arange(q.shape[2], device="cuda")[:, None] + past
        s.masked_fill_(~keep, float("-inf"))
    return torch.matmul(torch.softmax(s, -1), v), torch.logsumexp(s, -1)


def block_step(lib, D, Sq, B, Hq, Hkv, Sk, token, shape, causal):
    assert attn_shape(lib, STEP_F32, B, Hq, Hkv, Sq, Sk, D, Sk - Sq if causal else None) == shape
    gen = torch.Generator(device="cuda").manual_seed(31 * Sq + Sk + D)
    q, k, v = rows(gen, B, Hq, Sq, D, token), rows(gen, B, Hkv, Sk, D, token), rows(gen, B, Hkv, Sk, D, token)
    scale = 1.0 / math.sqrt(D)
    out = torch.full((B, Hq, Sq, D), float("nan"), device="cuda")
    lse = torch.full((B, Hq, Sq), float("nan"), device="cuda")
    if causal:
        lib.tr_block_attn_causal_at(q, k, v, Sk - Sq, 0, scale, out, lse)
    else:
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, scale, out, lse)
    ref_o, ref_l = attend(q, k, v, scale, causal)
    assert (out.double() - ref_o).abs().max().item() <= max(1e-2, v.abs().max().item() / 256)   # weights rounded to bf16: 2^-8 of a value
    assert (lse.double() - ref_l).abs().max().item() <= 1e-3


# Query rows of a workgroup, key groups: those that each row count below takes, without a mask and under the causal rule.
SHAPES = {"a": (256, 1), "b": (128, 1), "c": (128, 2), "d": (64, 2)}
SQ = [1, 2, 31, 33, 63, 65, 100, 129, 257]


@pytest.mark.parametrize("Sq", SQ)
@pytest.mark.parametrize("D,B,Hq,Hkv,Sk,shapes,causal_shapes", [
    (64, 1, 2, 2, 70, "aaaaaaadd", "aaaaaaadd"), (64, 1, 6, 2, 1100, "ddddddddd", "ddddddddd"),
    (64, 4, 16, 16, 200, "dddaaaadb", "dddaaaadb"), (64, 2, 48, 12, 333, "dddddddbb", "dddddddbb"),
    (128, 1, 2, 2, 70, "aaaaaaadd", "aaaaaaadd"), (128, 1, 6, 2, 1100, "ddddddddd", "ddddddddd"),
    (128, 4, 16, 16, 200, "dddaaaadb", "dddaaaadd"), (128, 2, 48, 12, 333, "dddddaaba", "dddddaabb"),
])
@pytest.mark.parametrize("token", [False, True])
def test_rows_of_a_block_step(lib, D, Sq, B, Hq, Hkv, Sk, shapes, causal_shapes, token):
    at = SQ.index(Sq)
    block_step(lib, D, Sq, B, Hq, Hkv, max(Sk, Sq), token, SHAPES[shapes[at]], False)
    block_step(lib, D, Sq, B, Hq, Hkv, max(Sk, Sq), token, SHAPES[causal_shapes[at]], True)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,causal", [
    (2, 48, 12, 129, 1000, False), (2, 48, 12, 129, 1000, True),      # one row in the second workgroup: three of four row groups have none
    (1, 64, 64, 257, 1000, False), (1, 24, 8, 641, 641, False),
    (1, 24, 8, 1000, 1000, True),                                     # the first row tiles see one tile of keys to three, which wait for all loads
    (1, 24, 24, 1300, 1300, True),
])
def test_rows_of_128_row_workgroups_with_key_groups(lib, D, B, Hq, Hkv, Sq, Sk, causal):
    """At D 128 the only workgroups whose K_3 and V_1 both lie where the rows pass through."""
    block_step(lib, D, Sq, B, Hq, Hkv, Sk, False, SHAPES["c"], causal)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,Sq,Sk", [(8, 8, 1, 1500), (8, 8, 15, 1500), (8, 8, 16, 1500), (8, 8, 17, 1500), (8, 2, 1, 2048), (8, 2, 4, 2048), (8, 2, 5, 2048)])
@pytest.mark.parametrize("token", [False, True])
def test_few_rows_of_a_cut_step(lib, D, Hq, Hkv, Sq, Sk, token):
    """Up to 16 rows of a K/V head, one query head's or its whole group's, and 17 and more."""
    parts, packed = attn_plan(lib, 1, Hq, Hkv, Sq, Sk, D)
    assert parts > 1 and packed == int(Hq > Hkv)
    for causal in (False, True):
        block_step(lib, D, Sq, 1, Hq, Hkv, Sk, token, SHAPES["d"], causal)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [1, 16, 17, 32, 45, 127, 128, 131, 300])
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,H,token", [(1, 3, True), (8, 40, False)])
def test_rows_of_bf16_blocks(lib, D, chunk, n, causal, B, H, token):
    gen = torch.Generator(device="cuda").manual_seed(17 * chunk + n + D)
    S = n * chunk
    rows_wg, groups = attn_shape(lib, RING_BF16, B, H, H, S, S, D, 0 if causal else None, n)
    assert groups == 1 if B == 8 or (n == 1 and chunk <= 128) else (rows_wg, groups) == (64, 2)
    q, k, v = (rows(gen, B, H, S, D, token) for _ in range(3))
    scale = 1.0 / math.sqrt(D)
    guard = torch.full((B, S + 2, H, D), 7.0, device="cuda")   # rows on both sides of the result, which stay as they are
    out = guard[:, 1:S + 1].permute(0, 2, 1, 3)
    lse = torch.full((B, H, S), float("nan"), device="cuda")
    ws = torch.empty(lib.tr_ring_attn_blocks_workspace_bytes(q, n, lib.TR_BF16), dtype=torch.uint8, device="cuda")
    lib.tr_ring_attn_blocks(q, k, v, n, causal, out, lse, lib.TR_BF16, ws, scale)
    ref_o, ref_l = attend(q, k, v, scale, causal)
    top = v.abs().max().item()
    assert (out.double() - ref_o).abs().max().item() <= max(1e-2, top / 256) + (n - 1) * top / 256
    assert (lse.double() - ref_l).abs().max().item() <= 1e-3
    assert (guard[:, 0] == 7.0).all() and (guard[:, S + 1] == 7.0).all()
