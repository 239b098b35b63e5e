"""ragged_layernorm in every form of its kernel: 16, 32 and 64 lanes a row, widths that fill them and widths that do not, with so many
rows that a lane takes several (one of them the last), fewer rows than the capacity, in place.  Bound: fp32 statistics (relative
1e-6) and one rounding to the output type, as in test_gpu_block.py; and, bit for bit, the one order of summation that all forms have."""
import re

import numpy as np
import pytest
import torch

from paper_2604_15408_amd import binding
from paper_2604_15408_amd.build import CSRC

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _constant(name):
    return int(re.search(rf"constexpr int {name} = (\d+);", (CSRC / "linear.hip").read_text()).group(1))


_TYPES = {"f16": (torch.float16, 2.0 ** -10), "bf16": (torch.bfloat16, 2.0 ** -7)}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("C", [8, 128, 192, 256, 384, 504, 512, 640, 768, 896, 1000, 1024, 1032, 2048])
def test_layernorm_forms(C, dtype):
    tdt, ulp = _TYPES[dtype]
    lanes = 16 if C <= 384 else 32 if C <= 768 else 64         # (of the form for many rows)
    at_once = _constant("kLnWaves") * 64 // lanes
    few = _constant("kLnFewRows")
    gen = torch.Generator(device=DEV).manual_seed(C)
    g, b = torch.randn(2, C, generator=gen, device=DEV).to(tdt)
    for cap, rows in ((at_once + 5, at_once + 3), (2 * at_once + 1, at_once + at_once // 2), (few + 1, few - 1), (few, few), (33, 33), (65, 1)):
        x = (torch.randn(cap, C, generator=gen, device=DEV) * 2 + 0.75).to(tdt)
        y = x.clone()
        binding.ragged_layernorm(y, g, b, y, torch.tensor([rows], dtype=torch.int32, device=DEV), 1e-6)
        assert torch.equal(y[rows:], x[rows:])
        for first in range(0, rows, 1 << 15):                  # (a stretch at a time: the reference is in fp64)
            s = slice(first, min(first + (1 << 15), rows))
            want = torch.nn.functional.layer_norm(x[s].double(), (C,), g.double(), b.double(), 1e-6)
            err = (y[s].double() - want).abs()
            assert torch.all(err <= ulp * want.abs() + 1e-5 * (1 + want.abs())), (cap, rows, first, float(err.max()))


def _in_order(x, g, b, eps):
    """LayerNorm of fp32 rows on the CPU as 64 lanes do it: chunks of eight values, number l, l + 64, ... to lane l, one fp32 partial
    sum a lane, pairs of lanes 8, 4, 2, 1, 16 and 32 apart.  (An fma is formed in fp64, where its product is exact; rounding
    the sum twice could differ from rounding it once in some 2^-28 of all cases.)"""
    rows, C = x.shape
    fma = lambda p, q, r: (p.double() * q.double() + r.double()).float()

    def total(add):
        lane = torch.zeros(rows, 64)
        for k in range(C):
            lane[:, k // 8 % 64] = add(k, lane[:, k // 8 % 64])
        lane = lane.view(rows, 4, 16)
        for apart in (8, 4, 2, 1):
            lane = lane + lane.roll(apart, 2)
        return (lane[:, 0, 0] + lane[:, 1, 0]) + (lane[:, 2, 0] + lane[:, 3, 0])

    n = torch.tensor(float(C))
    mean = total(lambda k, s: s + x[:, k]) / n
    v = x - mean[:, None]
    var = total(lambda k, s: fma(v[:, k], v[:, k], s)) / n
    rstd = 1.0 / torch.from_numpy(np.sqrt((var + torch.tensor(eps)).numpy()))      # (torch.sqrt does not round every fp32 root correctly)
    return fma(v * rstd[:, None], g, b)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("C", [64, 128, 192, 256, 320, 384, 512, 576, 640, 768, 896, 1024, 1536, 2048])
def test_layernorm_order_of_sums(C, dtype):
    """A row's bits are the same whatever the number of rows, and those of the order above: few rows and many are summed up
    by different numbers of lanes."""
    tdt, _ = _TYPES[dtype]
    n = 256
    gen = torch.Generator().manual_seed(C)
    x = (torch.randn(n, C, generator=gen) * 2 + 0.75).to(tdt)
    g, b = torch.randn(2, C, generator=gen).to(tdt)
    want = _in_order(x.float(), g.float(), b.float(), 1e-6).to(tdt)
    for cap in (n, _constant("kLnFewRows") + 1):
        xd = torch.zeros(cap, C, dtype=tdt, device=DEV)
        xd[cap - n:] = x.to(DEV)
        y = torch.zeros_like(xd)
        binding.ragged_layernorm(xd, g.to(DEV), b.to(DEV), y, torch.tensor([cap], dtype=torch.int32, device=DEV), 1e-6)
        differ = int((y[cap - n:].cpu().view(torch.int16) != want.view(torch.int16)).sum())
        assert differ == 0, (cap, differ)
