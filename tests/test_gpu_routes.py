"""Where the partial results of a call whose keys are cut can go decides its route: a scratch region of the library, or
(graph capture, no region idle) one launch over all keys."""
import threading

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


def test_a_region_serves_one_stream_after_another(lib):
    """Streams come and go; whoever calls while the regions are idle gets the cut form, so the bits do not depend on how
    many streams were there before (a bf16 result of one pass is rounded from other sums)."""
    q = bits_to_dev(rand_bits((1, 8, 5, 128), 580))
    k, v = (bits_to_dev(rand_bits((1, 2, 6000, 128), 581 + i)) for i in range(2))
    new = lambda: (torch.empty((1, 8, 5, 128), dtype=torch.bfloat16, device="cuda"), torch.empty((1, 8, 5), device="cuda"))
    out, lse = new()
    lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(9)]
    for s in streams * 2:
        o, l = new()
        torch.cuda.synchronize()
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, o, l, s)
        s.synchronize()
        assert torch.equal(o, out) and torch.equal(l, lse)


def test_an_eager_call_beside_a_capture_leaves_the_capture_alone(lib):
    q = bits_to_dev(rand_bits((1, 8, 5, 128), 590))
    k, v = (bits_to_dev(rand_bits((1, 2, 6000, 128), 591 + i)) for i in range(2))
    new = lambda: (torch.full((1, 8, 5, 128), float("nan"), device="cuda"), torch.full((1, 8, 5), float("nan"), device="cuda"))
    out, lse = new()
    lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, out, lse)
    graph_o, graph_l = new()
    beside = [new() for _ in range(6)]
    # torch deals its streams out in turn, and the one that captures is one of them
    streams = [s for s in (torch.cuda.Stream() for _ in range(len(beside) + 1)) if s != torch.cuda.graph.default_capture_stream]
    torch.cuda.synchronize()

    def run():
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, graph_o, graph_l)
        for s, (o, l) in zip(streams, beside):
            lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, o, l, s)

    graph = _captured(run)
    torch.cuda.synchronize()
    for o, l in beside:                                  # region or not: the same up to the order of fp32 sums
        assert float((o - out).abs().max()) <= 1e-2 and float((l - lse).abs().max()) <= 1e-5
    for o, l in beside:
        o.fill_(7.0)
    graph.replay()
    torch.cuda.synchronize()
    assert float((graph_o - out).abs().max()) <= 1e-2 and float((graph_l - lse).abs().max()) <= 1e-5
    assert all(bool((o == 7.0).all()) for o, _ in beside)  # the eager calls are no part of the graph


def test_a_busy_region_is_not_taken(lib):
    """Four streams hold the regions behind long work of their own; a call on a fifth does not wait for them: it takes its
    keys in one piece, like a captured call.  Once they are done it gets a region again."""
    q = bits_to_dev(rand_bits((1, 8, 5, 128), 600))
    k, v = (bits_to_dev(rand_bits((1, 2, 6000, 128), 601 + i)) for i in range(2))
    new = lambda: (torch.full((1, 8, 5, 128), float("nan"), device="cuda"), torch.full((1, 8, 5), float("nan"), device="cuda"))
    step = lambda o, l, s=None: lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, o, l, s)
    cut, one = new(), new()
    step(*cut)
    torch.cuda.synchronize()
    graph = _captured(lambda: step(*one))
    graph.replay()
    long = torch.randn((8192, 8192), device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert not torch.equal(cut[0], one[0])
    busy, fifth = [torch.cuda.Stream() for _ in range(4)], torch.cuda.Stream()
    held = [new() for _ in busy]
    (o, l), (o2, l2) = new(), new()
    torch.cuda.synchronize()
    for s, (ho, hl) in zip(busy, held):
        step(ho, hl, s)                                  # each owns a region
        s.synchronize()
    with torch.cuda.stream(busy[0]):
        for _ in range(100):
            long @ long                                  # about 80 ms
    for s in busy[1:]:
        s.wait_stream(busy[0])
    for s, (ho, hl) in zip(busy, held):
        step(ho, hl, s)
    step(o, l, fifth)
    fifth.synchronize()
    still_busy = not busy[0].query()
    assert torch.equal(o, one[0]) and torch.equal(l, one[1])
    assert still_busy                                    # else the case above has not been met
    torch.cuda.synchronize()
    step(o2, l2, fifth)
    torch.cuda.synchronize()
    for x in held + [(o2, l2)]:
        assert torch.equal(x[0], cut[0]) and torch.equal(x[1], cut[1])


def test_two_threads_on_one_stream(lib):
    """Attention and fold of one call go out together, whoever else enqueues on the stream."""
    stream = torch.cuda.Stream()
    sides = []
    for seed, Sk in ((620, 6000), (630, 3500)):
        q = bits_to_dev(rand_bits((1, 8, 5, 128), seed))
        k, v = (bits_to_dev(rand_bits((1, 2, Sk, 128), seed + 1 + i)) for i in range(2))
        outs = [(torch.empty((1, 8, 5, 128), device="cuda"), torch.empty((1, 8, 5), device="cuda")) for _ in range(200)]
        want = (torch.empty((1, 8, 5, 128), device="cuda"), torch.empty((1, 8, 5), device="cuda"))
        lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, *want, stream)
        sides.append((q, k, v, outs, want))
    torch.cuda.synchronize()

    def work(side):
        q, k, v, outs, _ = side
        for o, l in outs:
            lib.tr_block_attn(q, k, v, lib.TR_MASK_NONE, 0.1, o, l, stream)

    threads = [threading.Thread(target=work, args=(s,)) for s in sides]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for _, _, _, outs, want in sides:
        for o, l in outs:
            assert torch.equal(o, want[0]) and torch.equal(l, want[1])
