"""NaN and infinity through the forms an attention call can take.  A row whose scores hold a NaN gets out = NaN and
lse = -inf, whether its keys are one pass or cut into parts (which Sk = 4097 with few rows are); merged into an
accumulator such a block counts as empty.  An infinite value of V reaches out as that infinity."""
import numpy as np
import pytest
import torch

from gpu_util import bits_to_dev, rand_bits

pytestmark = pytest.mark.gpu


def _qkv(B, Hq, Hkv, Sq, Sk, D, seed):
    return tuple(bits_to_dev(rand_bits((B, h, s, D), seed + i)) for i, (h, s) in enumerate(((Hq, Sq), (Hkv, Sk), (Hkv, Sk))))


@pytest.mark.parametrize("Sk", [200, 4097])            # one pass, and cut into parts
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_bad_key_reaches_the_result(lib, Sk, dtype, bad):
    q, k, v = _qkv(1, 8, 2, 3, Sk, 128, 500)
    k[0, 1, Sk // 2, 5] = bad                            # K/V head 1: query heads 4 .. 7
    q[:, :, :, 5] = 1.0                                  # inf: a score of +inf, whose weight is exp(inf - inf)
    out = torch.zeros((1, 8, 3, 128), dtype=dtype, device="cuda")
    lse = torch.zeros((1, 8, 3), device="cuda")
    lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
    torch.cuda.synchronize()
    assert torch.isnan(out[:, 4:]).all() and torch.isneginf(lse[:, 4:]).all()
    assert torch.isfinite(out[:, :4]).all() and torch.isfinite(lse[:, :4]).all()


@pytest.mark.parametrize("Sk", [200, 4097])
def test_a_bad_block_leaves_the_accumulator(lib, Sk):
    q, k, v = _qkv(1, 8, 2, 3, Sk, 128, 510)
    k[0, 1, Sk - 1, 0] = float("nan")
    out, lse = torch.randn((1, 8, 3, 128), device="cuda"), torch.randn((1, 8, 3), device="cuda")
    lse[0, 5] = float("-inf")                            # an empty accumulator stays empty, with out = 0
    was_o, was_l = out.clone(), lse.clone()
    was_o[0, 5] = 0.0
    lib.tr_block_attn_merge(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
    torch.cuda.synchronize()
    assert torch.equal(out[:, 4:], was_o[:, 4:]) and torch.equal(lse[:, 4:], was_l[:, 4:])
    assert torch.isfinite(out[:, :4]).all() and not torch.equal(lse[:, :4], was_l[:, :4])


@pytest.mark.parametrize("Sk", [200, 4097])
def test_an_infinite_value_stays_infinite(lib, Sk):
    q, k, v = _qkv(1, 8, 2, 3, Sk, 128, 520)
    v[0, 1, 7, 3], v[0, 1, Sk // 2, 9] = float("inf"), float("-inf")
    out, lse = torch.zeros((1, 8, 3, 128), device="cuda"), torch.zeros((1, 8, 3), device="cuda")
    lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
    torch.cuda.synchronize()
    assert torch.isposinf(out[:, 4:, :, 3]).all() and torch.isneginf(out[:, 4:, :, 9]).all()
    out[:, 4:, :, 3] = out[:, 4:, :, 9] = 0.0
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
