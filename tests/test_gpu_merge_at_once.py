"""tr_merge around the size up to which a launch requests the accumulator together with the block: 699050 threads, each with two chunks of four columns."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2412_20501_amd.build import ensure_built
    ensure_built()
    import paper_2412_20501_amd as tr
    return tr


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,D,strided", [
    (1, 4, False), (77, 8, True), (300, 12, False), (300, 20, True), (300, 24, False), (300, 40, False),   # one chunk, threads without a second one, more than two
    (3001, 64, True), (1000, 128, True), (200, 256, False), (200, 512, True), (200, 516, False),
    (87381, 64, False), (87382, 64, False), (43690, 128, False), (43691, 128, False),                      # the line
])
def test_updates_around_the_line(lib, rows, D, strided, dtype):
    gen = torch.Generator(device="cuda").manual_seed(rows + D)
    def tensor(dtype):
        wide = torch.randn((1, rows, 2, D), device="cuda", generator=gen).to(dtype)
        return wide[:, :, :1].permute(0, 2, 1, 3) if strided else wide[:, :, 0][:, None].contiguous()
    out, blk = tensor(torch.float32), tensor(dtype)
    lse, blk_lse = (torch.rand((1, 1, rows), device="cuda", generator=gen) * 20 - 5 for _ in range(2))
    lse[..., 0::5], blk_lse[..., 1::5] = float("-inf"), float("-inf")
    lse[..., 2::25], blk_lse[..., 2::25] = float("-inf"), float("-inf")
    a, b = lse.double(), blk_lse.double()
    want_l = torch.logaddexp(a, b)
    weight = lambda x: torch.where(torch.isneginf(x), torch.zeros_like(x), torch.exp(x - want_l.masked_fill(torch.isinf(want_l), 0.0)))[..., None]
    want_o = weight(a) * out.double() + weight(b) * blk.double()
    out[0, 0, 0::5], blk[0, 0, 1::5] = float("nan"), float("nan")   # what an empty side holds is not looked at
    lib.tr_merge(out, lse, blk, blk_lse)
    torch.cuda.synchronize()
    assert torch.equal(torch.isneginf(lse), torch.isneginf(want_l))
    seen = ~torch.isneginf(want_l)
    assert float((out - want_o).abs().max()) <= 1e-5 and float((lse - want_l)[seen].abs().max()) <= 1e-5
