"""Thresholds of either zero: a score exceeds when it is strictly greater, and neither zero is
greater than the other, so the two thresholds give the same decisions -- for ranks that sit
exactly on the median (scores of +0: a constant column, a third of the ranks alike) and for
missing samples, which never exceed."""
import pytest
import torch

import gpu_harness
from gpu_harness import oracle_params, run_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps_per_column_route", [0, 64])
@pytest.mark.parametrize("thr", [0.0, -0.0])
@pytest.mark.parametrize("R,M", [(64, 3), (1000, 3), (3000, 1), (3000, 3), (4104, 3), (8000, 3), (16384, 3), (40000, 3)])
def test_scores_of_zero_do_not_exceed_a_threshold_of_zero(R, M, thr, steps_per_column_route):
    T = 4
    print(f"case threshold {thr} R={R} M={M} route={steps_per_column_route}", flush=True)
    g = torch.Generator().manual_seed(R)
    x = torch.exp(0.02 * torch.randn((T, M, R), generator=g))
    x[1] = 1.0                                                           # every rank on the median
    x[2][torch.rand((M, R), generator=g) < 0.34] = x[2].median()         # many of them
    x[3][torch.rand((M, R), generator=g) < 0.02] = float("nan")          # some samples missing ...
    x[3, :, 8:16] = float("nan")                                         # ... those of a whole node among them
    p = oracle_params(R=R, M=M, W=3, k=2, thr=thr, directions=(1, 0, -1)[:M], min_signals=1)
    gpu_harness.STREAMING_STEPS = steps_per_column_route
    try:
        rep = run_and_compare(p, x, topk_k=min(8, R // 8), label=f"threshold {thr}, {R} ranks")
    finally:
        gpu_harness.STREAMING_STEPS = None
    assert rep["z_bit_exact"]
