"""The linear layers' tile of 192 features x 128 rows, two work-groups to a CU (the widest with two), against the oracle: contractions of
one step, of two and of twelve, where the residual is requested two steps early."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_15408_amd import binding
from paper_2604_15408_amd import workloads as wl
from tests import linear_rule as rule

SHAPE = (6, 4, 2)
TN, TM = 192, 128


@pytest.mark.gpu
@pytest.mark.parametrize("act", ["none", "gelu"])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_linear_wide_pairs(dtype, residual, act):
    """Row counts around a tile edge and one where work-groups take several tiles, one k-step and several; bound as in
    test_gpu_block.py."""
    tdt, ulp = {"f16": (torch.float16, 2.0 ** -10), "bf16": (torch.bfloat16, 2.0 ** -7)}[dtype]
    gen = torch.Generator().manual_seed(1)
    for K in (64, 128, 768):
        hint, N = rule.call_for(SHAPE, act, K)
        for rows in (TM - 1, TM, TM + 1, TM * (700 // (N // TN) + 1) + TM // 2 + 1):
            assert rule.pick(hint, rows, N, K, act)[0] == SHAPE
            cap = max(rows, hint)
            x, w = torch.randn(cap, K, generator=gen).to(tdt), (torch.randn(N, K, generator=gen) * K ** -0.5).to(tdt)
            b, r = (torch.randn(N, generator=gen) * 0.5).to(tdt), torch.randn(cap, N, generator=gen).to(tdt)
            y = torch.full((cap, N), 77.0, dtype=tdt, device="cuda:0")
            binding.ragged_linear(x.cuda(), w.cuda(), b.cuda(), r.cuda() if residual else None, y,
                                  torch.tensor([rows], dtype=torch.int32, device="cuda:0"), act, rows_hint=hint)
            torch.cuda.synchronize()
            assert torch.all(y[rows:] == 77.0) and not torch.any(y[:rows] == 77.0)
            last = (rows - 1) // TM * TM
            near = {e + d for e in (0, 16, 64, TM, last, last + 64) for d in (-1, 0, 1, 15)} | {rows - 1}
            pick = sorted(v for v in near if 0 <= v < rows)
            want = oracle.linear(wl.to_words(x[pick]), wl.to_words(w), wl.to_words(b), wl.to_words(r[pick]) if residual else None, act, dtype,
                                 threads=oracle.max_threads())
            S = oracle.linear(wl.to_words(x[pick].abs()), wl.to_words(w.abs()), dtype=dtype, threads=oracle.max_threads())
            err = np.abs(y[pick].cpu().to(torch.float64).numpy() - want)
            bound = ulp * np.abs(want) + 2.0 ** -15 * S + 1e-6
            assert np.all(err <= bound), (N, K, rows, float((err / bound).max()))
