"""Accumulators around the size whose rows the Update keeps in the caches (224 MiB): the first rows of a large one and those behind
them take different branches of the kernel, and a wave may hold rows of both."""
import pytest
import torch

pytestmark = pytest.mark.gpu

KEPT = 224 << 20


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("extra", [-1, 0, 1, 2, 4099])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_on_both_sides_of_the_kept_ones(lib, D, extra, dtype):
    rows = KEPT // (4 * D) + extra
    gen = torch.Generator(device="cuda").manual_seed(20600 + D + extra)
    out = torch.full((1, 1, rows, D), float("nan"), device="cuda")
    lse = torch.full((1, 1, rows), float("-inf"), device="cuda")
    blocks = [(torch.randn((1, 1, rows, D), device="cuda", dtype=dtype, generator=gen),
               torch.rand((1, 1, rows), device="cuda", generator=gen) * 20 - 5) for _ in range(2)]
    for o, l in blocks:
        lib.tr_merge(out, lse, o, l)
    ref = torch.logsumexp(torch.stack([l.double() for _, l in blocks]), 0)
    assert (lse.double() - ref).abs().max().item() <= 1e-5
    worst = 0.0
    for r0 in range(0, rows, 1 << 17):
        part = slice(r0, min(rows, r0 + (1 << 17)))
        want = sum(torch.exp(l[:, :, part].double() - ref[:, :, part])[..., None] * o[:, :, part].double() for o, l in blocks)
        worst = max(worst, (out[:, :, part].double() - want).abs().max().item())
    assert worst <= 1e-5          # the bound of the merges on N(0, 1) partials (a handful of fp32 operations an element)
