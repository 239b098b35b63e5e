"""The linear layers' tile of 192 features x 128 rows, two work-groups to a CU: its walk over tiles and loads on the CPU, as
test_linear_walk.py has it for the other shapes, and its results against the oracle."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_2604_15408_amd import binding
from paper_2604_15408_amd import workloads as wl
from paper_2604_15408_amd.build import CSRC
from tests import linear_rule as rule

SHAPE = (6, 4, 2)
TN, TM = 192, 128


def test_every_load_stays_inside_its_operand(tmp_path):
    src, so = tmp_path / "check.cpp", tmp_path / "check.so"
    src.write_text('#include "linear_walk.h"\n#undef LINEAR_SHAPES\n#define LINEAR_SHAPES(X) LINEAR_WIDE_PAIRS(X)\n#include "linear_walk_check.cpp"\n')
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}",
                    f"-I{os.path.dirname(os.path.abspath(__file__))}", "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))
    out = (ctypes.c_int * 4)()
    lib.linear_shape(0, out)
    assert lib.linear_shape_count() == 1 and tuple(out) == (*SHAPE, 2)

    def follow(rows, N, K, cap=None):
        assert lib.linear_walk_check(*SHAPE, max(rows, 1) if cap is None else cap, rows, N, K) == 0, (rows, N, K, cap)

    for K in (64, 128, 192, 768):
        for rows in (1, TM - 1, TM, TM + 1, 3 * TM + 17, 9 * TM + 1):
            for feature_tiles in (1, 3, 7, 13):
                follow(rows, TN * feature_tiles, K)
        follow(40 * TM + 5, TN * 20, K)                        # several tiles per work-group
        follow(TM + 3, TN * 2, K, cap=50 * TM)                 # far fewer rows than the capacity
    follow(2 * TM + 1, TN, 1 << 22)
    for rows in (0, -1, -TM - 1, -(1 << 31)):
        follow(rows, TN * 33, 64, cap=300)


@pytest.mark.gpu
@pytest.mark.parametrize("act", ["none", "gelu"])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_linear_wide_pairs(dtype, residual, act):
    """Row counts around a tile edge and one where work-groups take several tiles, one k-step and several; bound as in
    test_gpu_block.py."""
    tdt, ulp = {"f16": (torch.float16, 2.0 ** -10), "bf16": (torch.bfloat16, 2.0 ** -7)}[dtype]
    gen = torch.Generator().manual_seed(1)
    ran = 0
    for K in (64, 128, 768):
        call = rule.call_for(SHAPE, act, K)
        if call is None:
            continue
        hint, N = call
        for rows in (TM - 1, TM, TM + 1, TM * (700 // (N // TN) + 1) + TM // 2 + 1):
            if rule.pick(hint, rows, N, K, act)[0] != SHAPE:
                continue
            ran += 1
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
    assert ran >= 4
