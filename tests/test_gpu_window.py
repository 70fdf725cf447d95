"""The batch kernel of the persistence window at its edges: rank counts around a tile of
2 048 items, windows around whole 64-step blocks and up to the longest, batches around
whole blocks and stretches (several stretches of a tile find first flagged steps and
leave the ring to the first), one-step calls between them -- counts, flags, first
flagged steps and the ring's further use against the oracle's re-summed windows."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import compare_decision, detector_for, oracle_params

pytestmark = pytest.mark.gpu

CASES = [  # ranks, window, persist, batches
    (64, 1, 1, [1, 2, 63, 64, 65]),
    (2048, 63, 20, [64, 1, 300, 255]),
    (2056, 64, 30, [257, 63, 1, 513]),
    (2040, 65, 2, [4 * 64 + 1, 4 * 64, 1, 1, 700]),
    (16384, 256, 60, [2700, 70, 1, 300]),
    (16392, 100, 85, [1, 1000, 1300]),
    (4104, 1024, 300, [1000, 24, 1, 2100, 64]),
    (520, 1023, 1023, [1100, 1, 1500]),
    (65536, 20, 15, [350, 1]),
    # around the longest batch that is walked step by step, and whole blocks behind it
    (64, 1, 1, [255, 256, 257, 320, 321]),
    (2056, 63, 20, [257, 383, 256, 384, 2]),
    (2040, 511, 100, [511, 512, 3, 576]),
    (4104, 1024, 300, [1023, 1024, 1025, 64, 1]),
    (32776, 300, 100, [256, 257, 300]),
]


def _words(bits):
    T, n = bits.shape
    padded = np.zeros((T, (n + 63) // 64 * 64), np.uint8)
    padded[:, :n] = bits
    return np.packbits(padded.reshape(T, -1, 64), axis=2, bitorder="little").view(np.uint64).reshape(T, -1)


@pytest.mark.parametrize("R,W,k,batches", CASES)
def test_batches_around_blocks_tiles_and_stretches(R, W, k, batches):
    rng = np.random.default_rng(R + 7 * W + k)
    T, N = sum(batches), R // 8
    quiet = rng.random((T, R), dtype=np.float32) < 0.02
    bits = quiet | (rng.random((T, R), dtype=np.float32) < rng.choice([0.0, 0.0, 0.0, 0.3, 0.7, 1.0], size=(1, R)))
    bits[:, -1] = 1                                                     # the last item of the last word
    bits[T // 2:, 3] = 0                                                # a flag that falls again
    node_bits = rng.random((T, N), dtype=np.float32) < rng.choice([0.02, 0.5, 0.98], size=(1, N))
    ra, na = _words(bits), _words(node_bits)
    node_z = rng.standard_normal((T, N)).astype(np.float32)
    p = oracle_params(R=R, M=1, W=W, k=k, min_signals=1)
    pr, pn = oracle.window(R, ra, W, k), oracle.window(N, na, W, k)
    d = dict(ranks=pr, nodes=pn, node_flag_byte=oracle.node_flag_byte(8, pn.flag, pr.flag))
    top = min(N, 64)
    d["topk_idx"], d["topk_key"] = oracle.topk(pn.count, node_z[-1], top)
    det = detector_for(p, topk=top)
    dra, dna = (torch.from_numpy(a.view(np.int64)).cuda() for a in (ra, na))
    dnz = torch.from_numpy(node_z).cuda()
    t0 = 0
    for c in batches:
        det.update_window(dict(rank_anom=dra[t0:t0 + c], node_anom=dna[t0:t0 + c], node_z=dnz[t0:t0 + c]), c)
        t0 += c
    compare_decision(p, d, det, top, label=f"R={R} W={W} k={k} {batches}")
    det.close()


@pytest.mark.parametrize("R,W,k,T", [(2056, 64, 30, 700), (4096, 65, 60, 641), (65536, 256, 200, 900), (1024, 100, 80, 703)])
@pytest.mark.parametrize("share", [0.002, 0.05, 0.6])
def test_items_flagged_together(R, W, k, T, share):
    """Few and many candidates of a block: walked item by item, or all items at once.  Some fall
    behind at one step, some in the last, partial block, some come and go; a second batch
    finds most of them flagged already."""
    print(f"case flagged together R={R} W={W} k={k} T={T} share={share}", flush=True)
    rng = np.random.default_rng(R + W + int(1000 * share))
    N, t = R // 8, np.arange(2 * T)[:, None]

    def history(n):
        kind = rng.permutation(np.where(rng.random(n) < share, rng.integers(1, 5, n), 0))[None]
        noise = rng.random((2 * T, n), dtype=np.float32) < 0.02
        return noise | ((kind == 1) & (t > T // 3)) | ((kind == 2) & (t > T - k - 3)) | \
            ((kind == 3) & (t // W % 2 == 0)) | ((kind == 4) & (rng.random((2 * T, n), dtype=np.float32) < k / W))

    ra, na = _words(history(R)), _words(history(N))
    p = oracle_params(R=R, M=1, W=W, k=k, min_signals=1)
    pr, pn = oracle.window(R, ra, W, k), oracle.window(N, na, W, k)
    node_z = rng.standard_normal((2 * T, N)).astype(np.float32)
    d = dict(ranks=pr, nodes=pn, node_flag_byte=oracle.node_flag_byte(8, pn.flag, pr.flag))
    d["topk_idx"], d["topk_key"] = oracle.topk(pn.count, node_z[-1], min(N, 64))
    det = detector_for(p, topk=min(N, 64))
    for a in (0, T):
        det.update_window({name: torch.from_numpy(v[a:a + T]).cuda() for name, v in
                           (("rank_anom", ra.view(np.int64)), ("node_anom", na.view(np.int64)), ("node_z", node_z))}, T)
    compare_decision(p, d, det, min(N, 64), label=f"together-{R}-{share}")
    det.close()
