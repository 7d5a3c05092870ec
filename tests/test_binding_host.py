"""Marshalling of the Python calls (csrc/binding.cpp): what is refused, and with which exception, before anything is launched."""
import pytest
import torch


@pytest.fixture(scope="module")
def tr():
    from paper_2412_20501_amd.build import ensure_built
    ensure_built()
    import paper_2412_20501_amd as m
    return m


class Stream:
    cuda_stream = 0


def _args(D=64, dtype=torch.bfloat16):
    q, k, v = (torch.zeros((1, 2, 8, D), dtype=dtype) for _ in range(3))
    return q, k, v, torch.zeros((1, 2, 8, D)), torch.zeros((1, 2, 8))


def test_tensors_that_are_no_operands(tr):
    q, k, v, o, l = _args()
    step = lambda q=q, o=o, l=l: tr.tr_block_attn(q, k, v, 0, 0.1, o, l, Stream)
    with pytest.raises(TypeError, match="unsupported dtype"):
        step(q=q.half())
    with pytest.raises(ValueError, match=r"\[B,H,S,D\]"):
        step(q=q[0, 0])
    with pytest.raises(ValueError, match="innermost"):
        step(o=o.transpose(2, 3))
    with pytest.raises(AttributeError):
        step(l=None)
    with pytest.raises((RuntimeError, ValueError)):
        step(q=q.float().to_sparse())
    with pytest.raises(ValueError, match="differ in length"):
        tr.tr_merge_n(o, l, [o, o], [l], False, Stream)
    with pytest.raises(TypeError, match="unsupported dtype"):
        tr.tr_merge_n(o, l, [o, o.half()], [l, l], False, Stream)


def test_the_library_answers(tr):
    """Sizes, strides and values reach the library as they are: it names them when it refuses."""
    q, k, v, o, l = _args()
    with pytest.raises(tr.TokenRingError, match="head dim 96") as e:
        tr.tr_block_attn(*_args(96)[:3], 0, 0.1, torch.zeros((1, 2, 8, 96)), l, stream=Stream)
    assert e.value.status == 3
    with pytest.raises(tr.TokenRingError, match="mask kind 7"):
        tr.tr_block_attn(q, k, v, 7, 0.1, o, l, Stream)
    with pytest.raises(tr.TokenRingError, match="scale"):
        tr.tr_block_attn(q, k, v, 0, -1, o, l, Stream)
    with pytest.raises(tr.TokenRingError, match="positions"):
        tr.tr_block_attn_causal_at(q, k, v, -(1 << 40), 0, 0.1, o, l, Stream)
    with pytest.raises(tr.TokenRingError, match="overlap"):
        tr.tr_merge(o, l, o, l, Stream)
    with pytest.raises(tr.TokenRingError, match="out of range"):
        tr.tr_merge_n(o, l, [], [], False, Stream)
    with pytest.raises(tr.TokenRingError, match="not a multiple of n_chunks 3"):
        tr.tr_ring_attn(q, k, v, 3, False, o, l, stream=Stream)
    with pytest.raises(tr.TokenRingError, match="unknown schedule 9"):
        tr.tr_ring_attn_sched(q, k, v, 2, True, 9, o, l, stream=Stream)
    with pytest.raises(tr.TokenRingError, match="aligned|too small"):
        tr.tr_ring_attn_blocks(q, k, v, 2, True, o, l, tr.TR_BF16, torch.zeros(64, dtype=torch.uint8), stream=Stream)
    with pytest.raises(tr.TokenRingError, match="stride"):
        tr.tr_ring_attn_noalloc(q, k, v, 2, True, torch.zeros((1, 1, 8, 64)).expand(1, 2, 8, 64), l, stream=Stream)


def test_other_number_types_and_tensor_subclasses(tr):
    class Sub(torch.Tensor):
        pass
    q, k, v, o, l = _args()
    with pytest.raises(tr.TokenRingError, match="mask kind 7"):
        tr.tr_block_attn(q.as_subclass(Sub), torch.nn.Parameter(k, requires_grad=False), v, torch.tensor(7), torch.tensor(0.1), o, l, Stream)
    with pytest.raises(tr.TokenRingError, match="n_chunks must be >= 1"):
        tr.tr_ring_attn(q, k, v, 1 << 32, False, o, l, stream=Stream)      # the C ABI's int: the low bits
    with pytest.raises(ValueError):
        tr.tr_block_attn(q, k, v, 0, "a", o, l, Stream)
