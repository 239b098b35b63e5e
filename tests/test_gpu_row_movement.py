"""Forms of the kernels around a pruning point at their edges: scores for every split of a row over lanes, pack and zero-filling
unpack with none to many rows per wavefront, rows that are held in registers and longer ones, and masks of several passes."""
import pytest
import torch

from paper_2604_15408_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
_TD = {"f16": torch.float16, "bf16": torch.bfloat16}


_WIDTHS = [8, 64, 72, 128, 192, 200, 384, 392, 512, 640, 768, 776, 1024, 1032, 1536, 1544]


@pytest.mark.parametrize("C", _WIDTHS)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_scores_every_split(dtype, C):
    """fp64 sums of exact squares: any order is within C roundings of the true sum."""
    for rows in (1, 3, 33, 130):
        x = torch.randn(rows, 1, C, generator=torch.Generator().manual_seed(C + rows)).to(_TD[dtype])
        scores = torch.full((rows + 1, 1), -1.0, dtype=torch.float64, device=DEV)
        binding.ragged_token_scores_l2(x.to(DEV), scores[:rows])
        want = (x.double() ** 2).sum(2)
        assert torch.all((scores[:rows].cpu() - want).abs() <= C * 2.0 ** -53 * want)
        assert scores[rows].item() == -1.0


@pytest.mark.parametrize("C", _WIDTHS)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_scores_order_of_sums(dtype, C):
    """The bits are those of 64 lanes with chunks l, l + 64, ... of eight values on lane l and exchanges 32, 16, ... 1 apart, whatever
    the split, for values over so many binades that every sum is rounded (a square is exact in fp64)."""
    gen = torch.Generator().manual_seed(C)
    wide = {"f16": 10, "bf16": 30}[dtype]
    x = (torch.randn(65, C, generator=gen) * torch.exp2(torch.randint(-wide, wide, (65, C), generator=gen))).to(_TD[dtype])
    x[x.isinf()] = 1.0
    square = x.double() ** 2
    lane = torch.zeros(65, 64, dtype=torch.float64)
    for k in range(C):
        lane[:, k // 8 % 64] += square[:, k]
    for half in (32, 16, 8, 4, 2, 1):
        lane = lane[:, :half] + lane[:, half:]
    scores = torch.zeros(65, 1, dtype=torch.float64, device=DEV)
    binding.ragged_token_scores_l2(x[:, None, :].to(DEV), scores)
    assert torch.equal(scores.cpu(), lane)


# Pack takes rows of up to 1024 values ahead of its prefix count if the mask has at most 16 KB (and its chunks, then, 8 tokens).  Beyond
# that its chunks have 16 tokens, over 32 768 tokens 32, over 65 536 64; those of the unpack have half as many.
@pytest.mark.parametrize("B,N,C,keep,spare", [
    (2, 197, 768, 1.0, 0),          # every row kept
    (1, 64, 1024, 0.5, 0),          # the longest rows ahead of the count
    (3, 65, 1032, 0.7, 0),          # longer ones, one by one
    (90, 197, 768, 0.5, 0),         # two words a lane in the smallest chunks
    (30, 577, 1024, 1.0, 0),        # the longest of those, every row kept
    (90, 197, 520, 0.05, 0),        # the shortest, hardly any kept
    (256, 197, 768, 0.6, 0),        # chunks of 32 and 16: several passes over two words a lane
    (120, 577, 776, 0.9, 0),        # chunks of 64 and 32
    (90, 197, 512, 0.5, 0),         # one word a lane in the smallest chunks
    (90, 197, 192, 1.0, 0),
    (220, 197, 8, 0.6, 0),          # 43 KB of mask, chunks of 32 and 16: one word a lane
    (220, 197, 512, 1.0, 0),
    (300, 577, 64, 0.9, 0),         # 173 KB of mask, chunks of 64: more than four rows for a wavefront
    (300, 577, 64, 0.02, 0),        # wavefronts without rows
    (220, 197, 512, 1.0, -1000),    # fewer packed rows than kept ones
    (90, 197, 1024, 0.8, -3001),
    (256, 197, 768, 0.7, -30002),
    (30, 577, 1032, 1.0, -4003),
])
def test_pack_unpack_forms(B, N, C, keep, spare):
    gen = torch.Generator().manual_seed(B + N + C)
    x = torch.randint(-30000, 30000, (B, N, C), generator=gen, dtype=torch.int16)
    mask = torch.rand(B, N, generator=gen) < keep
    lens = mask.sum(1)
    T = int(lens.sum())
    cap = T + spare
    xd, kd = x.view(torch.float16).to(DEV), mask.to(torch.uint8).to(DEV)
    packed = torch.zeros(cap + 1, C, dtype=torch.int16, device=DEV).view(torch.float16)
    cu, gidx = torch.zeros(B + 1, dtype=torch.int32, device=DEV), torch.full((cap + 1,), -1, dtype=torch.int32, device=DEV)
    binding.ragged_pack(xd, kd, packed[:cap], cu, gidx[:cap])
    flat = torch.nonzero(mask.flatten()).flatten()
    want = x.reshape(B * N, C)[flat]
    assert torch.equal(cu.cpu()[1:].long(), torch.cumsum(lens, 0)) and cu[0].item() == 0
    assert torch.equal(packed.view(torch.int16).cpu()[:cap], want[:cap]) and not torch.any(packed.view(torch.int16)[cap])
    assert torch.equal(gidx.cpu()[:cap].long(), flat[:cap]) and gidx[cap].item() == -1
    if spare < 0:
        return
    out = torch.full((B, N, C), 77, dtype=torch.int16, device=DEV)
    binding.ragged_unpack(packed[:cap], kd, cu, gidx[:cap], out.view(torch.float16), 1)
    assert torch.equal(out.cpu(), torch.where(mask[:, :, None], x, torch.zeros_like(x)))
