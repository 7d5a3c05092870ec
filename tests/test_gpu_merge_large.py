"""Accumulators around the size (128 MiB) from which on the Update goes past the caches, dense and token-major, against the same sums in 64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LINE = 128 << 20


def _check(lib, H, S, D, dtype, token, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def rows(fill):
        if token:
            return fill((1, S, H, D)).permute(0, 2, 1, 3)
        return fill((1, H, S, D))

    out = rows(lambda shape: torch.full(shape, float("nan"), device="cuda"))
    lse = torch.full((1, H, S), float("-inf"), device="cuda")
    blocks = [(rows(lambda shape: torch.randn(shape, device="cuda", dtype=dtype, generator=gen)),
               torch.rand((1, H, S), device="cuda", generator=gen) * 20 - 5) for _ in range(2)]
    for o, l in blocks:
        lib.tr_merge(out, lse, o, l)
    ref = torch.logsumexp(torch.stack([l.double() for _, l in blocks]), 0)
    assert (lse.double() - ref).abs().max().item() <= 1e-5
    worst = 0.0
    for r0 in range(0, S, 1 << 16):
        part = slice(r0, min(S, r0 + (1 << 16)))
        want = sum(torch.exp(l[:, :, part].double() - ref[:, :, part])[..., None] * o[:, :, part].double() for o, l in blocks)
        worst = max(worst, (out[:, :, part].double() - want).abs().max().item())
    assert worst <= 1e-5          # the bound of the merges on N(0, 1) partials (a handful of fp32 operations an element)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("extra", [-1, 0, 1, 2, 4099])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_around_the_line(lib, D, extra, dtype):
    _check(lib, 1, LINE // (4 * D) + extra, D, dtype, False, 20600 + D + extra)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("H,S,D", [(3, 87382, 128), (5, 70001, 96), (2, 458753, 64)])   # just beyond the line; odd heads and rows; 224 MiB and a row
def test_token_major(lib, H, S, D, dtype):
    _check(lib, H, S, D, dtype, True, 20700 + H)
