"""The hinted selection's lists and its search for the MAD's edges, where they change course:
lists of up to 64, 512 and more values about the median and about median -+ MAD (a wave's list of
rows that overflows among them), and hints of the MAD that put the search 64 edges off or more on
either side, or off the histogram.  One step per call, hinted; bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import compare_scores, detector_for, oracle_params

pytestmark = pytest.mark.gpu


def _column(R, kind, seed):
    rng = np.random.default_rng(seed)
    x = np.exp(0.02 * rng.standard_normal(R))
    dev = np.median(np.abs(x - 1.0))
    at = rng.permutation(R)
    if kind == "plain":
        return x
    where, share = kind
    n = max(2, int(share * R))
    jitter = 1e-6 * rng.standard_normal(n)                  # a few keys, within one bucket
    if where == "median":
        x[at[:n]] = 1.0 + jitter
    elif where == "mad":                                    # (half of them on either side)
        x[at[:n]] = 1.0 + dev * (1.0 + jitter) * np.where(np.arange(n) % 2, 1.0, -1.0)
    else:                                                   # one wave's ranks, all at the MAD's distance
        x[:n] = 1.0 + dev * (1.0 + jitter) * np.where(np.arange(n) % 2, 1.0, -1.0)
    return x


KINDS = ["plain", ("median", 1e-3), ("median", 6e-3), ("median", 0.02), ("mad", 2e-3), ("mad", 0.01), ("mad", 0.05),
         ("wave", 0.03)]


@pytest.mark.parametrize("R", [4104, 16384, 20000, 32768, 65536])
@pytest.mark.parametrize("mad_factor", [0.25, 0.85, 1.0, 1.15, 1.6, 8.0])
def test_lists_and_edges_of_the_hinted_selection(R, mad_factor):
    print(f"case hint edges R={R} mad x {mad_factor}", flush=True)
    M = len(KINDS)
    x = torch.from_numpy(np.stack([_column(R, k, 31 * R + i) for i, k in enumerate(KINDS)])[None].astype(np.float32))
    p = oracle_params(R=R, M=M, W=4, k=2, directions=(1, -1, 1, 0, -1, 1, 0, 1), min_signals=2)
    o = oracle.score(p, x.numpy(), want_z=True)
    det = detector_for(p)
    med = torch.from_numpy(o.med.reshape(-1)).cuda()
    mad = torch.from_numpy(o.mad.reshape(-1) * np.float32(mad_factor)).cuda()
    det.set_streaming_hints(med, mad)
    out = det.alloc_outputs(1, want_z=True)
    det.score_batch(x.cuda(), out)
    torch.cuda.synchronize()
    assert compare_scores(o, out, f"R={R} x{mad_factor}")["z_bit_exact"]
    det.set_streaming_hints(None, None)
    det.close()
