"""ragged_layernorm in every form of its kernel: widths that fill 16, 32 or 64 lanes with 8, 10, 12, 14 or 16 values and widths
that do not, with so many rows that a group of lanes takes several (one of them the last), fewer rows than the capacity, in place.
Bound: fp32 statistics (relative 1e-6) and one rounding to the output type, as in test_gpu_block.py."""
import pytest
import torch

from paper_2604_15408_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("C", [8, 128, 192, 256, 384, 504, 512, 640, 768, 896, 1000, 1024, 1032, 2048])
def test_layernorm_forms(C, dtype):
    tdt, ulp = {"f16": (torch.float16, 2.0 ** -10), "bf16": (torch.bfloat16, 2.0 ** -7)}[dtype]
    lanes = {128: 16, 192: 16, 256: 32, 384: 32}.get(C, 64)
    at_once = 16384 * 64 // lanes
    gen = torch.Generator(device=DEV).manual_seed(C)
    g, b = torch.randn(2, C, generator=gen, device=DEV).to(tdt)
    for cap, rows in ((at_once + 5, at_once + 3), (2 * at_once + 1, at_once + at_once // 2), (33, 33), (65, 1)):
        x = (torch.randn(cap, C, generator=gen, device=DEV) * 2 + 0.75).to(tdt)
        y = x.clone()
        binding.ragged_layernorm(y, g, b, y, torch.tensor([rows], dtype=torch.int32, device=DEV), 1e-6)
        assert torch.equal(y[rows:], x[rows:])
        for first in range(0, rows, 1 << 15):                  # (a stretch at a time: the reference is in fp64)
            s = slice(first, min(first + (1 << 15), rows))
            want = torch.nn.functional.layer_norm(x[s].double(), (C,), g.double(), b.double(), 1e-6)
            err = (y[s].double() - want).abs()
            assert torch.all(err <= ulp * want.abs() + 1e-5 * (1 + want.abs())), (cap, rows, first, float(err.max()))
