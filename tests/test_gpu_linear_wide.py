"""ragged_linear with rows of millions of features, where the 32-bit offsets of outputs and residual come to their end (a tile's rows
together have up to 2^32 bytes: 256 rows below 2^23 features, 32 below 2^26) and the form with 64-bit addresses begins.  Reference:
the same in fp32 on the GPU, a stretch of features at a time, with the bound that test_gpu_block.py derives."""
import pytest
import torch

from paper_2604_15408_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows,N,dtype,act,residual", [(257, 1 << 22, "f16", "none", True), (3, 1 << 22, "bf16", "gelu", False),
                                                       (3, (1 << 22) + 64, "f16", "gelu", True),
                                                       (65, (1 << 22) + 64, "bf16", "none", False),
                                                       (257, (1 << 23) - 256, "f16", "none", True),
                                                       (257, (1 << 23) + 256, "bf16", "none", True),
                                                       (33, (1 << 26) - 64, "bf16", "none", False),
                                                       (2, 1 << 26, "f16", "gelu", True), (33, 1 << 26, "bf16", "none", False)])
def test_linear_wide_rows(rows, N, dtype, act, residual):
    K = 64
    tdt, ulp = {"f16": (torch.float16, 2.0 ** -10), "bf16": (torch.bfloat16, 2.0 ** -7)}[dtype]
    g = torch.Generator(device=DEV).manual_seed(rows)
    rand = lambda *shape, scale=1.0: torch.randn(*shape, generator=g, device=DEV, dtype=tdt) * scale
    x, w, b = rand(rows + 1, K), rand(N, K, scale=K ** -0.5), rand(N)
    r = rand(rows + 1, N) if residual else None
    y = torch.full((rows + 1, N), 77.0, dtype=tdt, device=DEV)
    binding.ragged_linear(x, w, b, r, y, torch.tensor([rows], dtype=torch.int32, device=DEV), act)
    assert torch.all(y[rows] == 77.0)
    xf = x[:rows].float()
    for n in range(0, N, 1 << 18):
        s = slice(n, min(n + (1 << 18), N))
        wt = w[s].float().T.contiguous()
        want = xf @ wt + b[s].float()
        if act == "gelu":
            want = torch.nn.functional.gelu(want)
        if residual:
            want = want + r[:rows, s].float()
        bound = ulp * want.abs() + 2.0 ** -15 * (xf.abs() @ wt.abs()) + 1e-6
        assert torch.all((y[:rows, s].float() - want).abs() <= bound), (n, float(((y[:rows, s].float() - want).abs() / bound).max()))
