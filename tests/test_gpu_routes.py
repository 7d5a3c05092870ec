"""Where the partial results of a call whose keys are cut can go decides its route: a scratch region of the library, or
(graph capture, no region idle) one launch over all keys."""
import numpy as np
import pytest
import torch

from gpu_util import bits_to_dev, rand_bits

pytestmark = pytest.mark.gpu


def _captured(run):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    return graph


@pytest.mark.parametrize("D", [64, 128])
def test_a_captured_step_is_one_pass_over_its_keys(lib, D):
    """2048 rows x 2 heads are cut when a region is there.  The reference of one pass is the chunk form with a single chunk."""
    S, scale = 2048, 1.0 / np.sqrt(D)
    q, k, v = (bits_to_dev(rand_bits((1, 2, S, D), 560 + i)) for i in range(3))
    new = lambda: (torch.full((1, 2, S, D), float("nan"), device="cuda"), torch.full((1, 2, S), float("nan"), device="cuda"))
    one_o, one_l = new()
    ws = torch.empty(lib.tr_ring_attn_blocks_workspace_bytes(q, 1, lib.TR_BF16), dtype=torch.uint8, device="cuda")
    lib.tr_ring_attn_blocks(q, k, v, 1, True, one_o, one_l, lib.TR_BF16, ws, scale)
    out, lse = new()
    lib.tr_block_attn(q, k, v, lib.TR_MASK_CAUSAL_DIAG, scale, out, lse)      # sets the kernels up before the capture
    torch.cuda.synchronize()
    assert not torch.equal(out, one_o)                                        # cut: sums in another order
    graph = _captured(lambda: lib.tr_block_attn(q, k, v, lib.TR_MASK_CAUSAL_DIAG, scale, out, lse))
    for _ in range(3):
        out.fill_(float("nan")); lse.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, one_o) and torch.equal(lse, one_l)


def test_a_ring_gives_the_same_bits_on_every_route(lib):
    S = 2048
    q, k, v = (bits_to_dev(rand_bits((1, 2, S, 128), 570 + i)) for i in range(3))
    new = lambda: (torch.full((1, 2, S, 128), float("nan"), device="cuda"), torch.full((1, 2, S), float("nan"), device="cuda"))
    out, lse = new()
    lib.tr_ring_attn(q, k, v, 4, True, out, lse)
    graph_o, graph_l = new()
    torch.cuda.synchronize()
    graph = _captured(lambda: lib.tr_ring_attn(q, k, v, 4, True, graph_o, graph_l))
    for _ in range(3):
        graph_o.fill_(float("nan")); graph_l.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(graph_o, out) and torch.equal(graph_l, lse)
