"""The selection's lists and its search for the MAD's edges, where they change course: up to 64,
512 and more values about the median and about median -+ MAD, spread over all waves, and hints of the
MAD that put the search 64 edges off or more on either side, or off the histogram (one step per
call, hinted); buckets of values that are too many for the lists of rows of one wave or of all of
them (runs of steps in every width of workgroup).  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import compare_scores, detector_for, oracle_params, run_and_compare

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


def _ranks_of_one_wave(R, threads, n):
    """n ranks that one wave of a column's `threads` holds, each in a register row of its own."""
    i = np.arange(n)
    blocks = R // (4 * threads)                             # whole register rows
    assert n <= 64 * blocks
    return (i % blocks) * 4 * threads + 256 + 4 * (i // blocks)


# (40 and more rows of a wave, none of the others; shares of all waves; from 300 values on in one
# bucket for the general way, which counts them once more)
CROWDS = [("wave", 60), ("wave", 70), ("wave", 128), ("wave", 200), ("wave", 250), ("all", 130), ("all", 240),
          ("all", 330), ("all", 450), ("all", 700), None]


@pytest.mark.parametrize("signs", [False, True])
@pytest.mark.parametrize("R,T,threads", [(5000, 2600, 256), (8184, 2600, 256), (16384, 2060, 256), (20000, 1030, 512),
                                         (32768, 1030, 512), (40000, 520, 1024), (65536, 520, 1024), (16384, 12, 1024),
                                         (65536, 12, 1024)])
def test_buckets_too_crowded_for_the_lists(R, T, threads, signs):
    """Two steps a run and more, so that each kind of column is followed by another (T = 12: one
    workgroup per column).  Some lists hold the bucket, some are a row too short, some overflow in
    one wave alone, and some buckets hold more than is ranked at all."""
    print(f"case crowded buckets R={R} T={T} signs={signs}", flush=True)
    rng = np.random.default_rng(R + T)
    x = np.exp(0.02 * rng.standard_normal((T, 1, R), dtype=np.float32))
    for t in range(T):
        kind = CROWDS[int(rng.integers(len(CROWDS)))]
        if kind is None:
            continue
        where, n = kind
        n = min(n, 64 * (R // (4 * threads)))
        at = _ranks_of_one_wave(R, threads, n) if where == "wave" else rng.permutation(R)[:n]
        x[t, 0, at] = 1.0 + 2e-6 * rng.standard_normal(n)              # about the median, within a bucket or two
    if signs:
        x -= np.float32(1.0)
    p = oracle_params(R=R, M=1, W=8, k=4, directions=(1,), min_signals=1)
    run_and_compare(p, torch.from_numpy(x), topk_k=8, label=f"crowded buckets R{R}", want_z=False)


# (values on a grid of 1/q of the MAD: about 0.27 R / q of them alike in the middle, so that the gathered
# candidates and those ranked at last go from a few to beyond what one wave takes)
GRIDS = [None, 4000, 1000, 400, 250, 120, 60, 30]


@pytest.mark.parametrize("missing", [0, 1, 64])
@pytest.mark.parametrize("R", [4104, 8192, 16384, 24000, 40960, 57344, 65536])
def test_gathered_candidates_up_to_their_limits(R, missing):
    """Few and many alike values in the buckets of the median and of the MAD, odd and even numbers of
    samples: 16, 32 and 64 candidates and more, one step hinted and runs of steps."""
    print(f"case candidates R={R} missing={missing}", flush=True)
    rng = np.random.default_rng(R + missing)
    M, T = len(GRIDS), 3
    z = rng.standard_normal((T, M, R))
    for m, q in enumerate(GRIDS):
        if q:
            z[:, m] = np.round(z[:, m] * q) / q
    x = (1.0 + 0.02 * z).astype(np.float32)
    for t in range(T):
        for m in range(M):
            x[t, m, rng.permutation(R)[:missing * t]] = np.nan
    x = torch.from_numpy(x)
    p = oracle_params(R=R, M=M, W=4, k=2, directions=(1, -1, 1, 0, -1, 1, 0, 1), min_signals=2)
    o = oracle.score(p, x.numpy(), want_z=False)
    det = detector_for(p)
    out = det.alloc_outputs(1)
    for t in range(1, T):                                    # one step per call, hinted by the one before
        det.set_streaming_hints(torch.from_numpy(o.med[t - 1].copy()).cuda(), torch.from_numpy(o.mad[t - 1].copy()).cuda())
        det.score_batch(x[t:t + 1].cuda(), out)
        torch.cuda.synchronize()
        compare_scores(oracle.score(p, x[t:t + 1].numpy(), want_z=False), out, f"R={R} step {t}")
    det.set_streaming_hints(None, None)
    det.close()
    run_and_compare(p, x.repeat(400, 1, 1)[:max(6, 2200 * 4096 // R)], topk_k=8, label=f"candidates R{R}", want_z=False)


# (the gap between the two middle values, in thousandths of the MAD, of which a bucket is one to two:
# neighbours in one bucket, in two, a few and up to 63 apart, and beyond)
GAPS = [0, 1, 2, 3, 8, 30, 60, 75, 100, 140, 160, 400]


@pytest.mark.parametrize("R,T", [(4104, 2600), (5000, 2600), (8192, 2600), (16384, 2060), (24000, 1030), (65536, 520),
                                 (16384, 24), (65536, 24)])
def test_middle_ranks_in_buckets_apart(R, T):
    """The two middle ranks far apart, in runs of steps and (T = 24) one or a few steps a workgroup; in
    every second step the distances about the MAD are unevenly spread besides, so that the place
    that an even spread gives to the wanted one is off by up to all of them."""
    print(f"case middle ranks apart R={R} T={T}", flush=True)
    rng = np.random.default_rng(R + T)
    d = np.abs(rng.standard_normal((T, 1, R)))                  # distances from the middle, in standard deviations
    for t in range(1, T, 2):
        n = 2 * int(rng.integers(10, 120))
        at = rng.permutation(R)[:n]
        d[t, 0, at] = 0.6745 * (1.0 + 2e-3 * rng.random(n) ** float(rng.integers(2, 12)) * rng.choice([-1.0, 1.0]))
    gap = 0.6745e-3 * np.array([GAPS[t % len(GAPS)] for t in range(T)])[:, None, None]
    side = np.where(rng.permuted(np.tile(np.arange(R) % 2, (T, 1, 1)), axis=2), 1.0, -1.0)
    x = torch.from_numpy((1.0 + 0.02 * side * (d + 0.5 * gap)).astype(np.float32))
    p = oracle_params(R=R, M=1, W=8, k=4, directions=(1,), min_signals=1)
    run_and_compare(p, x, topk_k=8, label=f"middle ranks apart R{R}", want_z=False, chunks=[T] if T > 24 else [4] * 6)


def _negative_and_tiny(R, kind, seed):
    """Values that no shifted bits of a real column hold: -2.0 to -2.0095, whose bits are 0xC0000000 and
    a little more, negative subnormals, -0 and plain negative numbers."""
    rng = np.random.default_rng(seed)
    if kind == "below_minus_two":
        b = np.uint32(0xC0000000) + rng.integers(0, 40000, R).astype(np.uint32)
    elif kind == "negative_subnormals":
        b = np.uint32(0x80000000) + rng.integers(0, 40000, R).astype(np.uint32)
    elif kind == "mixed":
        b = (np.float32(1.0) + np.float32(0.02) * rng.standard_normal(R, dtype=np.float32)).view(np.uint32).copy()
        at = rng.permutation(R)
        b[at[: R // 8]] = np.uint32(0xC0000000) + rng.integers(0, 40000, R // 8).astype(np.uint32)
        b[at[R // 8:R // 4]] = np.uint32(0x80000000)
    elif kind == "subnormals":                              # (no signs: units about 44)
        b = rng.integers(20, 69, R).astype(np.uint32)
    elif kind == "wider_subnormals":                        # (a bracket wide enough to count in, from near 0 on)
        b = rng.integers(1, 60000, R).astype(np.uint32)
    else:
        b = (-400.0 * np.exp(0.02 * rng.standard_normal(R))).astype(np.float32).view(np.uint32)
    return b.astype(np.uint32).view(np.float32)


TINY_KINDS = ["below_minus_two", "negative_subnormals", "mixed", "subnormals", "wider_subnormals", "negative"]
# (median and MAD hinted, in units of the last place of zero)
TINY_HINTS = [(50, 20), (44, 30), (64, 50), (65, 51), (200, 3), (3000, 1500), (30000, 15000), (1, 1)]


@pytest.mark.parametrize("R", [4096, 4104, 8192, 16384, 20000, 40000, 65536])
def test_hints_of_a_few_subnormal_units(R):
    """Brackets that begin next to zero, narrower and wider than the counters, over columns with signs and
    without: hints cost time, never results."""
    print(f"case tiny hints R={R}", flush=True)
    M = len(TINY_KINDS)
    x = torch.from_numpy(np.stack([_negative_and_tiny(R, k, 7 * R + i) for i, k in enumerate(TINY_KINDS)])[None].copy())
    p = oracle_params(R=R, M=M, W=4, k=2, directions=(1, -1, 1, 0, -1, 1), min_signals=2)
    o = oracle.score(p, x.numpy(), want_z=True)
    det = detector_for(p)
    xd = x.cuda()
    for med, mad in TINY_HINTS:
        hints = [torch.from_numpy(np.full(M, v, dtype=np.uint32).view(np.float32)).cuda() for v in (med, mad)]
        det.set_streaming_hints(*hints)
        out = det.alloc_outputs(1, want_z=True)
        for v in out.values():
            v.view(torch.uint8).fill_(0xA5)
        det.score_batch(xd, out)
        torch.cuda.synchronize()
        assert compare_scores(o, out, f"R={R} hints {med} {mad}")["z_bit_exact"]
    det.set_streaming_hints(None, None)
    det.close()


@pytest.mark.parametrize("R,T", [(4104, 2600), (16384, 2060), (24000, 1030), (40000, 520), (65536, 520)])
def test_steps_of_a_few_subnormal_units_before_negative_ones(R, T):
    """The same from step to step: a column of subnormal values leaves its hints to one with signs."""
    print(f"case tiny steps R={R} T={T}", flush=True)
    order = ["subnormals", "subnormals", "below_minus_two", "wider_subnormals", "mixed", "subnormals", "negative_subnormals"]
    x = torch.from_numpy(np.stack([_negative_and_tiny(R, order[t % len(order)], 11 * R + t % 21) for t in range(T)])[:, None].copy())
    p = oracle_params(R=R, M=1, W=8, k=4, directions=(1,), min_signals=1)
    run_and_compare(p, x, topk_k=8, label=f"tiny steps R{R}", want_z=False)


@pytest.mark.parametrize("R,T", [(4104, 2600), (8192, 2600), (16384, 2060), (24000, 1030), (40960, 520), (57344, 520), (65536, 520)])
def test_gathered_candidates_from_step_to_step(R, T):
    """The columns of the test above -- few and many alike values, odd and even numbers of samples -- in batches of
    more than twice the steps that the chip takes at once, so that each workgroup's later steps are hinted by
    its own earlier ones, over columns of another kind."""
    print(f"case candidates from step to step R={R} T={T}", flush=True)
    rng = np.random.default_rng(3 * R)
    n = 3 * len(GRIDS)                                          # steps that differ, given again and again
    x = np.empty((n, 2, R), np.float32)
    for t in range(n):
        for m in range(2):
            z = rng.standard_normal(R)
            q = GRIDS[(t + 3 * m * (t // len(GRIDS) + 1)) % len(GRIDS)]
            z = np.round(z * q) / q if q else z
            x[t, m] = 1.0 + 0.02 * z
            x[t, m, rng.permutation(R)[:(0, 1, 64, 0)[(t + m) % 4]]] = np.nan
    x = torch.from_numpy(x).repeat((T + n - 1) // n, 1, 1)[:T].contiguous()
    p = oracle_params(R=R, M=2, W=4, k=2, directions=(1, -1), min_signals=2)
    run_and_compare(p, x, topk_k=8, label=f"candidates from step to step R{R}", want_z=False)
