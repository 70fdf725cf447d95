"""Inputs whose answers take more looking for must not cost many times what plain ones do:
both are timed in turn in this process, so that only their ratio counts.  The bounds lie
far from what either form of a kernel takes, with the ratios measured beside them."""
import numpy as np
import pytest
import torch

from gpu_harness import detector_for, oracle_params

pytestmark = pytest.mark.gpu


def device_us(prepare, call, n=7):
    """The median device time of `call` behind an untimed `prepare`."""
    got = []
    for _ in range(n + 2):
        prepare()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        call()
        ev[1].record()
        torch.cuda.synchronize()
        got.append(1e3 * ev[0].elapsed_time(ev[1]))
    return sorted(got[2:])[n // 2]


def packed(bits):
    T, n = bits.shape
    padded = np.zeros((T, (n + 63) // 64 * 64), np.uint8)
    padded[:, :n] = bits
    words = np.packbits(padded.reshape(T, -1, 64), axis=2, bitorder="little").view(np.int64).reshape(T, -1)
    return torch.from_numpy(words.copy()).cuda()


@pytest.mark.parametrize("kind", ["fall behind together", "come and go", "hover"])
@pytest.mark.parametrize("R,T,W,k", [(65536, 1024, 256, 200), (16384, 2048, 20, 15), (1024, 2000, 100, 80)])
def test_window_of_many_items_flagged(R, T, W, k, kind):
    """Measured, 65 536 ranks: 13 us with nothing flagged; many items at once by the walk of
    one item after another 396, 733 and 1 179 us, in bit slices 16, 18 and 26 us."""
    rng = np.random.default_rng(R)
    quiet = rng.random((T, R), dtype=np.float32) < 0.01
    sick = rng.random(R) < 0.3
    t = np.arange(T)[:, None]
    many = {"fall behind together": quiet | (sick & (t > T // 3)), "come and go": quiet | (sick & (t // W % 2 == 0)),
            "hover": rng.random((T, R), dtype=np.float32) < k / W}[kind]
    us = []
    for bits in (quiet, many):
        det = detector_for(oracle_params(R=R, M=1, W=W, k=k, min_signals=1))
        out = dict(rank_anom=packed(bits), node_anom=packed(bits[:, ::8]), node_z=torch.zeros((T, R // 8), device="cuda"))
        us.append(device_us(det.state.zero_, lambda: det.update_window(out, T, 0)))
        det.close()
    print(f"{kind}, {R} ranks: {us[0]:.1f} us quiet, {us[1]:.1f} us many", flush=True)
    assert us[1] < 8 * us[0]


@pytest.mark.parametrize("T", [2, 64])
def test_window_of_short_batches(T):
    """A short batch's cost follows its steps, not the window.  Measured, 65 536 ranks, ten
    calls in a row, windows 64 and 1 024: where the whole window was counted afresh 9 and 13 us
    a call, from the stored counts 4 to 5 with either."""
    R = 65536
    us = []
    for W in (64, 1024):
        det = detector_for(oracle_params(R=R, M=1, W=W, k=W // 2, min_signals=1))
        rng = np.random.default_rng(T)
        out = dict(rank_anom=packed(rng.random((T, R), dtype=np.float32) < 0.01),
                   node_anom=packed(rng.random((T, R // 8), dtype=np.float32) < 0.01),
                   node_z=torch.zeros((T, R // 8), device="cuda"))
        us.append(device_us(lambda: det.update_window(out, T), lambda: [det.update_window(out, T) for _ in range(10)]) / 10)
        det.close()
    print(f"{T} steps: {us[0]:.2f} us window 64, {us[1]:.2f} us window 1024", flush=True)
    assert us[1] < 1.4 * us[0] and us[1] < 12


@pytest.mark.parametrize("kind,bound", [("fall behind together", 2.5), ("come and go", 3), ("hover", 8)])
def test_ledger_of_many_items_flagged(kind, bound):
    """Measured, 65 536 ranks x 512 steps: 35 us with nothing flagged; many items at once by the
    walk of one word after another 116, 173 and 497 us, in bit slices 60, 59 and 163 (of which
    the episodes' own bookkeeping is the most where every node hovers)."""
    R, T, W, k = 65536, 512, 100, 80
    rng = np.random.default_rng(R)
    quiet = rng.random((T, R), dtype=np.float32) < 0.01
    sick = rng.random(R) < 0.3
    t = np.arange(T)[:, None]
    many = {"fall behind together": quiet | (sick & (t > T // 3)), "come and go": quiet | (sick & (t // W % 2 == 0)),
            "hover": rng.random((T, R), dtype=np.float32) < k / W}[kind]
    us = []
    for bits in (quiet, many):
        det = detector_for(oracle_params(R=R, M=4, W=W, k=k, min_signals=2))
        mask = 15 * bits.astype(np.uint8)
        out = dict(exceed_mask=torch.from_numpy(mask).cuda(), node_mask=torch.from_numpy(mask[:, ::8].copy()).cuda(),
                   node_z=torch.zeros((T, R // 8), device="cuda"))
        led = det.alloc_ledger(T)
        us.append(device_us(led.zero_, lambda: det.update_ledger(out, T, 0)))
        det.close()
    print(f"{kind}, {R} ranks: {us[0]:.1f} us quiet, {us[1]:.1f} us many", flush=True)
    assert us[1] < bound * us[0]


def test_ledger_of_short_batches_in_a_wide_window():
    """65 536 ranks, window 1 024, ten calls in a row: a 32-step batch next to one of 24 steps.
    Measured: 19 and 38 us a call where the longer one loaded the whole window, 19 and 23."""
    R, W, us = 65536, 1024, []
    for T in (24, 32):
        det = detector_for(oracle_params(R=R, M=4, W=W, k=W // 2, min_signals=2))
        mask = (np.random.default_rng(T).random((T, R), dtype=np.float32) < 0.01).astype(np.uint8)
        out = dict(exceed_mask=torch.from_numpy(mask).cuda(), node_mask=torch.from_numpy(mask[:, ::8].copy()).cuda(),
                   node_z=torch.zeros((T, R // 8), device="cuda"))
        det.alloc_ledger(T)
        us.append(device_us(lambda: det.update_ledger(out, T), lambda: [det.update_ledger(out, T) for _ in range(10)]) / 10)
        det.close()
    print(f"ledger, window {W}: {us[0]:.1f} us for 24 steps, {us[1]:.1f} us for 32", flush=True)
    assert us[1] < 1.6 * us[0]


@pytest.mark.parametrize("pattern", ["equal", "ascending", "few values"])
@pytest.mark.parametrize("N", [1000, 5000, 8192])
def test_slowest_nodes_of_alike_scores(N, pattern):
    """Twenty calls in a row.  Measured, 8 192 nodes, k = 64: 6 us a call for scores in random
    order; equal ones 70, rising ones 40 where many alike were sorted, 11 and 14 by the
    threads' best keys."""
    rng = np.random.default_rng(N)
    plain = rng.standard_normal(N).astype(np.float32)
    alike = {"equal": np.zeros(N, np.float32), "ascending": (1 + 1e-6 * np.arange(N)).astype(np.float32),
             "few values": rng.integers(-2, 3, N).astype(np.float32)}[pattern]
    det = detector_for(oracle_params(R=8 * N, M=1, W=4, k=2, min_signals=1))
    out, tk, us = det.alloc_outputs(1), det.alloc_topk(64), []
    out["rank_anom"].zero_()
    out["node_anom"].zero_()
    for z in (plain, alike):
        out["node_z"].copy_(torch.from_numpy(z)[None])
        det.update_window(out, 1)
        us.append(device_us(lambda: None, lambda: [det.topk_nodes(64, tk) for _ in range(20)]) / 20)
    det.close()
    print(f"{pattern}, {N} nodes: {us[0]:.1f} us in random order, {us[1]:.1f} us", flush=True)
    assert us[1] < 3 * us[0]


@pytest.mark.parametrize("nodes,W", [(128, 16), (2048, 16), (8192, 16), (8192, 256)])
def test_severity_of_neighbouring_nodes(nodes, W):
    """Eight flagged nodes side by side next to eight far apart, ten calls in a row.  Measured,
    window 16: 17 us a call against 7 where one workgroup took the neighbours one after
    another, 6 either way since; window 256: 48 against 12, 10.5 either way."""
    R, us = 8 * nodes, []
    det = detector_for(oracle_params(R=R, M=1, W=W, k=max(1, W // 2), min_signals=1))
    x = torch.exp(0.02 * torch.randn((W, 1, R), device="cuda"))
    out, sev = det.alloc_outputs(W), det.alloc_severity()
    det.score_batch(x, out)
    for where in (np.arange(8) * (nodes // 8) + np.arange(8), 16 + np.arange(8)):
        bits = np.zeros((W, nodes), bool)
        bits[:, where] = True
        out["rank_anom"].zero_()
        out["node_anom"].copy_(packed(bits))
        det.state.zero_()
        det.update_window(out, W, 0)
        us.append(device_us(lambda: None, lambda: [det.severity(x, out, sev) for _ in range(10)]) / 10)
        assert int((sev["tier"] > 0).sum()) == 8
    det.close()
    print(f"severity, {nodes} nodes, window {W}: {us[0]:.1f} us apart, {us[1]:.1f} us side by side", flush=True)
    assert us[1] < 1.8 * us[0]


@pytest.mark.parametrize("kind,bound", [("missing", 1.25), ("whole degrees", 2.0)])
def test_scoring_of_small_awkward_columns(kind, bound):
    """4 000 ranks x 2 metrics x 256 steps.  Measured: 40 us for plain values; one sample in a
    hundred missing 57 where their keys were mapped like those of signs, 43; whole degrees 90
    before their sample's middle value was tried alone, 66."""
    R, M, T, us = 4000, 2, 256, []
    det = detector_for(oracle_params(R=R, M=M, W=4, k=2))
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.exp(0.02 * torch.randn((T, M, R), device="cuda", generator=g))
    other = torch.round(65 * x) if kind == "whole degrees" else \
        torch.where(torch.rand(x.shape, device="cuda", generator=g) < 0.01, float("nan"), x)
    out = det.alloc_outputs(T)
    for v in (x, other):
        us.append(device_us(lambda: None, lambda: [det.score_batch(v, out) for _ in range(10)]) / 10)
    det.close()
    print(f"{kind}, {R} ranks: {us[0]:.1f} us plain, {us[1]:.1f} us", flush=True)
    assert us[1] < bound * us[0]


@pytest.mark.parametrize("R,T", [(48000, 1024), (20000, 1000)])
def test_scoring_of_a_bucket_crowded_by_one_wave(R, T):
    """200 values about the median, all of them in the ranks of one wave.  Measured, 48 000 ranks x
    1 024 steps: 87 us for plain columns; 156 where a wave's list that is too short had the column
    selected anew, 103 where its bucket is gathered again; 20 000 x 1 000: 46, 80 and 56."""
    us = []
    det = detector_for(oracle_params(R=R, M=1, W=4, k=2, min_signals=1))
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.exp(0.02 * torch.randn((T, 1, R), device="cuda", generator=g))
    block, i = 4 * (512 if R <= 32768 else 1024), torch.arange(200, device="cuda")
    at = (i % (R // block)) * block + 256 + 4 * (i // (R // block))
    crowded = x.clone()
    crowded[:, :, at] = 1.0 + 2e-6 * torch.randn((T, 1, 200), device="cuda", generator=g)
    out = det.alloc_outputs(T)
    for v in (x, crowded):
        us.append(device_us(lambda: None, lambda: [det.score_batch(v, out) for _ in range(10)]) / 10)
    det.close()
    print(f"crowded by one wave, {R} ranks: {us[0]:.1f} us plain, {us[1]:.1f} us", flush=True)
    assert us[1] < 1.5 * us[0]


@pytest.mark.parametrize("R", [56000, 65528])
def test_scoring_of_skewed_columns(R):
    """Exponential values next to log-normal ones: a bucket on the left of the median is several times
    as narrow as its mirror image.  Measured, 56 000 ranks x 1 024 steps: 104 and 112 to 122 us; 143
    where the distances ranked reached a wide bucket further in.  65 528 ranks: 121 and 146 us, a ratio of
    1.21; the bound lies halfway to 1.37."""
    T, us = 1024, []
    det = detector_for(oracle_params(R=R, M=1, W=4, k=2, min_signals=1))
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.exp(0.02 * torch.randn((T, 1, R), device="cuda", generator=g))
    skewed = torch.empty_like(x).exponential_(generator=g) + 1e-6
    out = det.alloc_outputs(T)
    for v in (x, skewed):
        us.append(device_us(lambda: None, lambda: [det.score_batch(v, out) for _ in range(10)]) / 10)
    det.close()
    print(f"skewed, {R} ranks: {us[0]:.1f} us plain, {us[1]:.1f} us", flush=True)
    assert us[1] < 1.29 * us[0]


@pytest.mark.parametrize("R,T", [(32768, 1024), (56000, 512)])
def test_scoring_of_a_crowd_at_the_edge_of_the_mad(R, T):
    """400 alike values where the median plus MAD lies, spread over all ranks: too many distances to
    compare each with all.  Measured, 32 768 ranks x 1 024 steps x 2: 88 us for plain columns; 163 where
    they were ranked, 116 where the column's distances are selected; 56 000 x 512 x 4: 142, 274 and 188."""
    M, us = 2 if R <= 32768 else 4, []
    det = detector_for(oracle_params(R=R, M=M, W=4, k=2, min_signals=1, directions=(1,) * M))
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.exp(0.02 * torch.randn((T, M, R), device="cuda", generator=g))
    crowded = x.clone()
    at = torch.randperm(R, device="cuda", generator=g)[:400]
    crowded[:, :, at] = 1.0 + 0.6745 * 0.02 + 2e-6 * torch.randn((T, M, 400), device="cuda", generator=g)
    out = det.alloc_outputs(T)
    for v in (x, crowded):
        us.append(device_us(lambda: None, lambda: [det.score_batch(v, out) for _ in range(10)]) / 10)
    det.close()
    print(f"crowd at the MAD's edge, {R} ranks: {us[0]:.1f} us plain, {us[1]:.1f} us", flush=True)
    assert us[1] < 1.6 * us[0]


@pytest.mark.parametrize("R,T,M", [(5000, 1000, 2), (7000, 1000, 8), (8000, 1000, 4), (12000, 1000, 4), (24000, 512, 8), (32768, 512, 8),
                                   (4096, 256, 1), (16384, 200, 1), (15000, 1024, 4), (16384, 1024, 4)])
@pytest.mark.parametrize("kind", ["exponential", "log-normal of sigma 1"])
def test_scoring_of_skewed_columns_in_runs_of_one_step_or_two(kind, R, T, M):
    """Columns whose quartiles lie unevenly about the median, and whose first hints are a sample's.  Measured,
    plain / exponential / log-normal, us: 8 000 ranks x 1 000 steps x 4 45 / 90 / 88 with half the interquartile
    distance in place of the MAD, 45 / 50 / 49 with the sides' unevenness taken into account; 24 000 x 512 x 8 102 /
    182 / 172 and 103 / 110 / 110; 5 000 x 1 000 x 2 26 / 46 / 44 and 26 / 27 / 27; columns sampled one by one, 16 384 x
    1 024 x 4 69 / 115 / 95 and 69 / 73 / 75, 4 096 x 256 x 1 12 / 20 / 20 and 12 / 12 / 12.  The bound lies half way
    between 1.1 and 1.6."""
    us = []
    det = detector_for(oracle_params(R=R, M=M, W=4, k=2, min_signals=1, directions=(1,) * M))
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((T, M, R), device="cuda", generator=g)
    skewed = torch.exp(x) if kind != "exponential" else torch.empty_like(x).exponential_(generator=g) + 1e-6
    x = torch.exp(0.02 * x)
    out = det.alloc_outputs(T)
    for v in (x, skewed):
        us.append(device_us(lambda: None, lambda: [det.score_batch(v, out) for _ in range(10)]) / 10)
    det.close()
    print(f"{kind}, {R} ranks x {T} x {M}: {us[0]:.1f} us plain, {us[1]:.1f} us", flush=True)
    assert us[1] < 1.35 * us[0]
