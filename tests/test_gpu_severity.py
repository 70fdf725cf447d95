"""The severity tiers where the selection of the middle quotient changes its way: few quotients
(sorted at once), many, an odd number of them, ties throughout, a sample that misleads, and
several flagged nodes within one workgroup's group of neighbours."""
import pytest
import torch

import oracle
from gpu_harness import compare_severity, detector_for, gpu_score, oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "ties", "two values", "missing", "ramp", "signs"])
@pytest.mark.parametrize("T,W", [(1, 4), (8, 8), (9, 9), (70, 64), (300, 257), (1030, 1024)])
@pytest.mark.parametrize("direction", [1, -1, 0])
def test_the_middle_quotient(kind, T, W, direction):
    R = 8 * 19
    print(f"case severity {kind} T={T} W={W} direction={direction}", flush=True)
    g = torch.Generator().manual_seed(T + len(kind))
    x = torch.exp(0.02 * torch.randn((T, 1, R), generator=g, dtype=torch.float64))
    slow = 1.25 if direction >= 0 else 0.8
    for n in (0, 5, 6, 7, 8, 18):                           # neighbours, the first and the last
        x[:, :, 8 * n: 8 * n + 8] *= slow
    if kind == "ties":
        x = torch.round(x * 4) / 4
    elif kind == "two values":                              # the two middle quotients far apart
        x[:, :, 0: 4] = 1.1
        x[:, :, 4: 8] = 1.9
    elif kind == "missing":
        x[torch.rand(x.shape, generator=g) < 0.3] = float("nan")
        x[:, :, 40: 47] = float("nan")
    elif kind == "ramp":                                    # sorted in time: a sample in order
        x = x * torch.linspace(0.5, 2.0, T, dtype=torch.float64)[:, None, None] ** 3
    elif kind == "signs":
        x[:, :, 3::8] *= -1
    x = x.to(torch.float32)
    p = oracle_params(R=R, M=1, W=W, k=1, thr=2.0, directions=(direction,), min_signals=1)
    d = oracle.detect(p, x.numpy(), topk_k=4, want_z=False)
    det = detector_for(p)
    out = gpu_score(det, x, want_z=False)
    det.update_window(out, T)
    rep = compare_severity(p, d, det, x, out, label=f"{kind}-{T}")
    assert sum(rep["tiers"][1:]) > 0 or T == 1
    det.close()
