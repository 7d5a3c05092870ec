"""tr_merge where whole waves hold only empty accumulators (their out is not read) beside waves that hold one row
that is not, and the reverse: fp32 blocks against the fp64 oracle, max-abs 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import max_abs, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [4, 36, 64, 128, 640])
@pytest.mark.parametrize("pattern", ["all", "one_held", "one_empty", "first_half", "blocks_empty_too"])
def test_merge_onto_empty_accumulators(lib, D, pattern):
    B, H, S = 1, 2, 131
    rng = np.random.default_rng(D)
    a, b = (rng.standard_normal((B, H, S, D)).astype(np.float32) for _ in range(2))
    la, lb = (rng.uniform(-5, 15, (B, H, S)).astype(np.float32) for _ in range(2))
    empty = np.ones((B, H, S), bool)
    if pattern == "one_held":
        empty[0, 1, 77] = False
    elif pattern == "one_empty":
        empty[:] = False
        empty[0, 1, 77] = True
    elif pattern == "first_half":
        empty[:, :, S // 2:] = False
    elif pattern == "blocks_empty_too":
        lb[:, :, ::3] = -np.inf
    la[empty] = -np.inf
    clean = np.where(empty[..., None], np.float32(0), a)
    a[empty] = np.nan
    acc_o, acc_l = torch.from_numpy(a).cuda(), torch.from_numpy(la).cuda()
    lib.tr_merge(acc_o, acc_l, torch.from_numpy(b).cuda(), torch.from_numpy(lb).cuda())
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.merge_pair(clean, la, b, lb)
    got_o, got_l = to_np(acc_o), to_np(acc_l)
    live = np.isfinite(ref_l)
    assert np.array_equal(np.isneginf(got_l), ~live) and not np.isnan(got_o).any()
    assert max_abs(got_o, ref_o) <= 1e-5 and max_abs(got_l[live], ref_l[live]) <= 1e-5
