"""Columns that one wave scores (up to 4 096 ranks): few distinct values, missing samples, signs,
and a sample that misleads -- its 64 ranks made far off, too tight, missing, negative or the
lowest -- against the oracle, one step and several, at the register rows' edges."""
import numpy as np
import pytest
import torch

from gpu_harness import bits32, detector_for, oracle_params, run_and_compare

pytestmark = pytest.mark.gpu

ROWS = (1, 2, 4, 8, 12, 16)


def sampled_ranks(R):
    """The ranks of a column's sample: lane l looks at element 4 * l of one register row of 256
    ranks, the row by the lane's group."""
    rows = next(r for r in ROWS if R <= 256 * r)
    lane = np.arange(64)
    if rows == 1:
        row = np.zeros(64, int)
    elif rows == 2:
        row = lane // 32
    else:
        row = lane // 16 * (rows // 4)
    rank = 256 * row + 4 * lane
    return rank[rank < R]


def column(kind, T, M, R, g):
    x = torch.exp(0.02 * torch.randn((T, M, R), generator=g, dtype=torch.float64))
    at = torch.from_numpy(sampled_ranks(R))
    if kind == "whole degrees":
        x = torch.round(65 * x)
    elif kind == "tenths":
        x = torch.round(10 * x) / 10
    elif kind == "two values":
        x = torch.where(torch.rand(x.shape, generator=g) < 0.5, 1.0, 2.0).to(x.dtype)
    elif kind == "equal":
        x = torch.ones_like(x)
    elif kind == "missing":
        x[torch.rand(x.shape, generator=g) < 0.2] = float("nan")
    elif kind == "missing degrees":
        x = torch.round(65 * x)
        x[torch.rand(x.shape, generator=g) < 0.3] = float("nan")
    elif kind == "signs":
        x = x - 1
        x[:, :, ::7] = -0.0
    elif kind == "signs and missing":
        x = torch.round(100 * (x - 1))
        x[torch.rand(x.shape, generator=g) < 0.1] = float("nan")
    elif kind == "sample far above":
        x[:, :, at] *= 1e6
    elif kind == "sample far below":
        x[:, :, at] *= 1e-6
    elif kind == "sample too tight":
        x[:, :, at] = 1.3
    elif kind == "sample missing":
        x[:, :, at] = float("nan")
    elif kind == "sample negative":
        x[:, :, at] *= -1
    elif kind == "sample on two values":
        x[:, :, at] = torch.where(torch.arange(len(at)) % 2 == 0, 0.5, 1.7).to(x.dtype)
    x[:, 0, -8:] *= 1.3
    return x.to(torch.float32)


KINDS = ("whole degrees", "tenths", "two values", "equal", "missing", "missing degrees", "signs", "signs and missing",
         "sample far above", "sample far below", "sample too tight", "sample missing", "sample negative",
         "sample on two values")


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("R", [64, 72, 248, 256, 264, 512, 520, 800, 1024, 1032, 2048, 2056, 3072, 3080, 4088, 4096])
def test_awkward_columns(R, kind):
    print(f"case small columns R={R} {kind}", flush=True)
    g = torch.Generator().manual_seed(R + len(kind))
    x = column(kind, 6, 2, R, g)
    p = oracle_params(R=R, M=2, W=3, k=2, thr=2.5, directions=(1, 0), min_signals=1)
    run_and_compare(p, x, topk_k=min(8, R // 8), chunks=[5, 1], label=f"small-{R}-{kind}")


@pytest.mark.parametrize("R", [8, 56, 64, 512, 1024, 2048])
def test_infinite_medians_repeat(R):
    """Infinities are unsupported input, but one call gives what another gives: nothing that an
    earlier launch left in the work area is read."""
    print(f"case infinite medians R={R}", flush=True)
    det = detector_for(oracle_params(R=R, M=2, W=3, k=2))
    g = torch.Generator().manual_seed(R)
    x = torch.exp(0.02 * torch.randn((1, 2, R), generator=g))
    x[0, 0, : 5 * R // 8] = float("inf")
    x[0, 1, : 3 * R // 4] = float("-inf")
    seen = set()
    for i in range(6):
        other = det.alloc_outputs(64)
        det.score_batch(torch.exp((1 + i) * torch.randn((64, 2, R), generator=g)).cuda(), other)
        out = det.alloc_outputs(1)
        det.score_batch(x.cuda(), out)
        seen.add(bits32(out["med"].cpu()).tobytes() + bits32(out["mad"].cpu()).tobytes())
    det.close()
    assert len(seen) == 1


def _so_many_between_the_pivots(R, n, rng):
    """A column of which exactly n values lie between the pivots that its sample gives (a quarter of the sample's
    64 about its middle, both ends included): 64 fill the wave's list of last candidates."""
    at = sampled_ranks(R)
    ns = len(at)
    reach = 4 + ns // 16
    lo, hi = ns // 2 - reach, ns // 2 + reach
    sample = (1.0 + (np.arange(ns) - ns // 2) * 1e-3).astype(np.float32)
    x = np.empty(R, np.float32)
    x[at] = rng.permutation(sample)
    rest = rng.permutation(np.setdiff1d(np.arange(R), at))
    inside = n - (hi - lo + 1)
    x[rest[:inside]] = rng.uniform(sample[lo] + 1e-5, sample[hi] - 1e-5, inside)
    out = rest[inside:]
    below = (R - n) // 2 - lo                                   # the median's ranks lie in the middle of the n
    x[out[:below]] = 0.9 * (1.0 + 0.01 * rng.random(below))
    x[out[below:]] = 1.1 * (1.0 + 0.01 * rng.random(len(out) - below))
    assert ((x >= sample[lo]) & (x <= sample[hi])).sum() == n
    return x


@pytest.mark.parametrize("R,M", [(64, 8), (256, 8), (512, 8), (1000, 8), (1024, 4), (2048, 8), (3000, 4), (3072, 2), (4000, 8), (4096, 2)])
def test_last_candidates_that_fill_their_list(R, M):
    """62 to 66 candidates in every wave of a workgroup, whose lists lie one behind another; a column of
    64 ranks is such a list by itself, also with values missing or of either sign."""
    rng = np.random.default_rng(R)
    counts = [62, 63, 64, 65, 66, 64]
    x = np.empty((len(counts) * 4, M, R), np.float32)
    for t in range(len(x)):
        for m in range(M):
            if R == 64:
                col = (1.0 + 0.02 * rng.standard_normal(R)).astype(np.float32)
                kind = (t + m) % 4
                if kind == 1:
                    col[rng.integers(R)] = np.nan
                elif kind == 2:
                    col[rng.permutation(R)[:20]] = 1.0
                elif kind == 3:
                    col = col - np.float32(1.0)
            else:
                col = _so_many_between_the_pivots(R, counts[(t + m) % len(counts)], rng)
                if t % 4 == 3:
                    col = -col
            x[t, m] = col
    p = oracle_params(R=R, M=M, W=4, k=2, directions=(1, -1, 0, 1, -1, 1, 0, 1)[:M], min_signals=min(2, M))
    run_and_compare(p, torch.from_numpy(x), topk_k=min(8, R // 8), chunks=[len(x) - 1, 1], label=f"full lists R{R} M{M}")
