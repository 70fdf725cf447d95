"""Runs of steps that each miss some samples: the selection led by the step before with ranks
that follow the samples present, missing samples scored in the median's place (thresholds from
zero up, scaled-sum rule, primary metric that does not fall) or by the general route."""
import pytest
import torch

import oracle
from gpu_harness import oracle_params, run_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", [1, -1, 0])
@pytest.mark.parametrize("thr,agg", [(2.5, oracle.NODE_SUM_SCALED), (0.0, oracle.NODE_SUM_SCALED),
                                     (-0.5, oracle.NODE_SUM_SCALED), (2.5, oracle.NODE_MAX)])
@pytest.mark.parametrize("R,T", [(4096, 3100), (5000, 2100), (16384, 2060), (20000, 1030)])
def test_runs_of_steps_with_missing_samples(R, T, thr, agg, direction):
    print(f"case missing runs R={R} T={T} thr={thr} agg={agg} direction={direction}", flush=True)
    g = torch.Generator().manual_seed(R + 7 * direction)
    x = torch.exp(0.02 * torch.randn((T, 1, R), generator=g, dtype=torch.float32))
    gone = torch.rand((T, R // 8, 1), generator=g) < 0.01                # whole nodes: a node score of zero
    x[:, 0] = torch.where(gone.expand(T, R // 8, 8).reshape(T, R), float("nan"), x[:, 0])
    x[torch.rand(x.shape, generator=g) < 0.002] = float("nan")           # single samples: odd and even numbers present
    x[T // 2, 0, :] = float("nan")                                       # a step of which nothing arrived
    x[T // 2 + 1, 0, 5:] = float("nan")
    p = oracle_params(R=R, M=1, W=8, k=4, thr=thr, node_agg=agg, directions=(direction,), min_signals=1)
    run_and_compare(p, x, topk_k=8, label=f"missing runs R{R}", want_z=False)
