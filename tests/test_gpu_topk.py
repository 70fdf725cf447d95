"""The ranking kernel at the edges of its dispatch: one wave, one / two / four / eight keys
per thread, requests up to and beyond 64, and rankings in which the likely candidates sit
where the threshold of the short route does not expect them (all keys equal but for the
node index, the best ones all with one wave of threads, sorted input)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import gpu_topk
from paper_2605_17879_amd import Config, Detector

pytestmark = pytest.mark.gpu

PATTERNS = ("random", "equal", "one wave", "ascending", "few values", "one thread column")


def _scores(pattern, N, rng):
    z = rng.standard_normal(N).astype(np.float32)
    n = np.arange(N)
    if pattern == "equal":
        z[:] = np.float32(-0.0)
    elif pattern == "one wave":
        z[n % 1024 < 64] += 100.0
    elif pattern == "ascending":
        z = (n * 1e-6).astype(np.float32)
    elif pattern == "few values":
        z = rng.integers(-2, 3, N).astype(np.float32)
    elif pattern == "one thread column":
        z[n % 1024 < 8] += 100.0
    return z


@pytest.mark.parametrize("pattern", PATTERNS)
@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 128, 129, 1000, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192])
def test_slowest_nodes_at_the_edges_of_the_dispatch(N, pattern):
    rng = np.random.default_rng(N * 7 + len(pattern))
    det = Detector(Config(n_ranks=8 * N, n_metrics=1, window=4, persist_k=2))
    out = det.alloc_outputs(1)
    z = _scores(pattern, N, rng)
    bits = rng.random(det.NW * 64) < 0.03
    bits[N:] = False
    words = np.packbits(bits.reshape(-1, 8), axis=1, bitorder="little").reshape(-1).view(np.int64)
    out["rank_anom"].zero_()
    out["node_anom"].copy_(torch.from_numpy(words.copy())[None])
    out["node_z"].copy_(torch.from_numpy(z)[None])
    det.update_window(out, 1)
    for k in sorted({1, min(N, 7), min(N, 63), min(N, 64), min(N, 65), N}):
        want_idx, want_key = oracle.topk(bits[:N].astype(np.uint16), z, k)
        idx, key = gpu_topk(det, k)
        assert np.array_equal(idx, want_idx), (N, pattern, k)
        assert np.array_equal(key, want_key), (N, pattern, k)
    det.close()


@pytest.mark.parametrize("spread", ["within 32 of each other", "wide", "at both ends of the range", "equal"])
@pytest.mark.parametrize("N", [65, 1024, 3230, 8192])
def test_ranking_by_sums_that_agree_in_their_leading_bits(N, spread):
    rng = np.random.default_rng(N + len(spread))
    W = 1024 if spread == "at both ends of the range" else 4
    det = Detector(Config(n_ranks=8 * N, n_metrics=1, window=W, persist_k=2))
    q = {"within 32 of each other": rng.integers(-8, 8, (W, N)), "wide": rng.integers(-30000, 30000, (W, N)),
         "at both ends of the range": np.repeat(rng.choice([-32768, 32767], (1, N)), W, axis=0),
         "equal": np.full((W, N), 5)}[spread]
    out = det.alloc_outputs(W)
    out["exceed_mask"].zero_()
    node_mask = rng.random((W, N)) < 0.01
    out["node_mask"].copy_(torch.from_numpy(node_mask.astype(np.uint8)))
    out["node_z"].copy_(torch.from_numpy((q / 64.0).astype(np.float32)))      # (exact: the default grid is 1/64)
    det.alloc_ledger(W)
    det.update_ledger(out, W)
    for k in (1, 33, 64):
        want_idx, want_key = oracle.topk_mean(node_mask.sum(0).astype(np.uint16), q.sum(0).astype(np.int32), k)
        tk = det.alloc_topk(k)
        det.topk_nodes_mean(k, tk)
        assert np.array_equal(tk["idx"].cpu().numpy(), want_idx), (N, spread, k)
        assert np.array_equal(tk["key"].cpu().numpy().view(np.uint64), want_key), (N, spread, k)
    det.close()
