"""Rank counts that fill no tiling exactly, at the edges of every tiling of the scoring
kernel: one node more than the next smaller one holds, one node less than it holds itself,
and exactly as many; both routes, with missing samples and signs among the plain steps.  One
step per workgroup; runs of several are in the parity tests of carried hints."""
import numpy as np
import pytest
import torch

import gpu_harness
from gpu_harness import oracle_params, run_and_compare

pytestmark = pytest.mark.gpu

# ranks that the tilings hold (threads x rows x 4), of the batch route and of the per-column one
HOLD = (256, 512, 1024, 2048, 3072, 4096, 6144, 8192, 10240, 12288, 14336, 16384, 20480, 24576, 28672, 32768, 40960,
        49152, 57344, 65536)
EDGES = sorted({r for h in HOLD for r in (h - 8, h, h + 8) if r <= 65536})


@pytest.mark.parametrize("steps_per_column_route", [0, 64])
@pytest.mark.parametrize("R,M", [(R, 2) for R in EDGES] + [(R, M) for R in EDGES if 2000 < R < 4200 for M in (1, 5)])
def test_edges_of_the_tilings(R, M, steps_per_column_route):
    T = 4
    print(f"case edges R={R} M={M} route={steps_per_column_route}", flush=True)
    g = torch.Generator().manual_seed(R)
    x = torch.exp(0.02 * torch.randn((T, M, R), generator=g, dtype=torch.float64))
    x[:, 1::2] = 400.0 / x[:, 1::2]                          # lower is worse
    x[:, 0::2, -8:] *= 1.3                                   # the last node is slow ...
    x[:, 1::2, -8:] /= 1.3
    x = x.to(torch.float32)
    x[2, 0, -3:] = float("nan")                              # ... and some of its samples are missing
    x[3, M - 1] -= 400.0 if M == 2 else 1.0                  # signs
    p = oracle_params(R=R, M=M, W=3, k=2, directions=(1, -1, 1, -1, 1)[:M], min_signals=min(2, M))
    gpu_harness.STREAMING_STEPS = steps_per_column_route
    try:
        rep = run_and_compare(p, x, topk_k=min(8, R // 8), chunks=[2, 2], label=f"edge{R}")
    finally:
        gpu_harness.STREAMING_STEPS = None
    assert rep["z_bit_exact"] and rep["node_flags"] >= 1
