"""Forms of the kernels around a pruning point at their edges: scores for every split of a row over lanes."""
import pytest
import torch

from paper_2604_15408_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
_TD = {"f16": torch.float16, "bf16": torch.bfloat16}


@pytest.mark.parametrize("C", [8, 192, 384, 512, 640, 768, 1024, 1032])
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
