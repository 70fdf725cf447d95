"""What this framework's speed is measured on: the work that a user has it do, through
the public entry points of ``paper_2605_17879_amd.Detector``.

The listed cases cover the five configurations of the repository's benchmark and tests
(64 to 65 536 ranks, one to eight metrics, one step per call to 10 000 steps per batch)
and, beside them, rank counts that are no power of two, telemetry with samples missing,
the optional full z output, the ledger and the follow-up on flagged nodes.  ``draw``
makes more cases of the same kinds, with sizes spread over the whole range.

A case is a dict of plain values:
  kind     "stream"   one evaluation appended per call, hinted by the call before
           "batch"    a whole batch: scores, window, flags, slowest nodes
           "missing"  the same for a job whose membership changes: ranks that took no
                      part in a step are marked missing first
           "scores"   a batch with the full z output written as well
           "ledger"   the bookkeeping that follows a scored batch
           "followup" severity tiers of the flagged nodes and scoring of sweep results
  ranks, metrics, steps, window, persist, noise ("lognormal" or "heavy")
"""
from __future__ import annotations

import math
import random

import torch

from paper_2605_17879_amd import Config, Detector

DEVICE = "cuda:0"
TOPK = 64

# Metrics of the heavy-tailed recipe: step time (s), compute time (s), collective wait
# (s), achieved TFLOPS, GPU temperature (C), GPU clock (GHz), power (W), NIC rate (Gb/s),
# and whether each rises (+1) or falls (-1) when a rank slows down.
BASES = (1.0, 0.7, 0.3, 400.0, 65.0, 1.93, 700.0, 400.0)
DIRECTIONS = (1, 1, 1, -1, 1, -1, -1, -1)

STREAM_HISTORY = 32          # steps that a streaming state goes through in turn


def _case(name, kind, ranks, metrics, steps, window, persist, noise):
    return {"name": name, "kind": kind, "ranks": ranks, "metrics": metrics, "steps": steps,
            "window": window, "persist": persist, "noise": noise}


def listed():
    return [
        # a small job watched live: the smallest call there is, all latency and launches
        _case("stream-1000x4", "stream", 1000, 4, 1, 50, 40, "lognormal"),
        # the streaming configuration: 32 768 ranks, every metric, one step per call
        _case("stream-32768x8", "stream", 32768, 8, 1, 256, 200, "heavy"),
        # the smallest job's history scored in one go: one metric, 200 steps
        _case("batch-64x1x200", "batch", 64, 1, 200, 20, 15, "lognormal"),
        # a 1 024-GPU job's history
        _case("batch-1024x4x2000", "batch", 1024, 4, 2000, 50, 40, "lognormal"),
        # a job of an odd size (625 nodes), two metrics
        _case("batch-5000x2x1000", "batch", 5000, 2, 1000, 100, 80, "lognormal"),
        # the 16 384-rank configuration in a single scoring pass
        _case("batch-16384x4x10000", "batch", 16384, 4, 10000, 100, 80, "lognormal"),
        # a large job of an odd size (5 000 nodes), every metric
        _case("batch-40000x8x1024", "batch", 40000, 8, 1024, 256, 200, "heavy"),
        # the largest configuration: 65 536 ranks x 4 096 steps x 8 metrics
        _case("batch-65536x8x4096", "batch", 65536, 8, 4096, 256, 200, "heavy"),
        # ranks that joined late, left or were not polled in time
        _case("missing-16384x4x1024", "missing", 16384, 4, 1024, 100, 80, "lognormal"),
        # an analyst's pass: every sample's score is wanted, not the decisions alone
        _case("scores-32768x8x512", "scores", 32768, 8, 512, 256, 200, "heavy"),
        # per-indicator persistence, averaged scores and recurrence behind a scored batch
        _case("ledger-65536x8x4096", "ledger", 65536, 8, 4096, 256, 200, "heavy"),
        # the tiers of the nodes that the window flagged, and a sweep over all nodes
        _case("followup-65536x8x512", "followup", 65536, 8, 512, 256, 200, "heavy"),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the most samples (ranks x metrics x steps) of a drawn case of each kind
_MOST_SAMPLES = {"batch": 1_000_000_000, "missing": 134_000_000, "scores": 268_000_000,
                 "ledger": 1_000_000_000, "followup": 268_000_000}


def draw(rng: random.Random):
    kind = rng.choice(("stream", "stream", "batch", "batch", "batch", "missing", "scores", "ledger", "followup"))
    ranks = max(64, min(65536, 8 * (_log_between(rng, 64, 65536) // 8)))
    noise = rng.choice(("lognormal", "heavy"))
    metrics = rng.randint(1, 4 if noise == "lognormal" else 8)
    window = _log_between(rng, 16, 512)
    persist = max(1, (window * rng.randint(70, 85)) // 100)
    if kind == "stream":
        steps = 1
    else:
        most = max(64, min(10000, _MOST_SAMPLES[kind] // (ranks * metrics)))
        steps = _log_between(rng, 64, most) if most > 64 else 64
        if kind == "followup":
            window = min(window, 256)
            persist = max(1, (window * 75) // 100)
    return {"kind": kind, "ranks": ranks, "metrics": metrics, "steps": steps, "window": window,
            "persist": persist, "noise": noise}


# ---- inputs ----------------------------------------------------------------------------

def _slowdown(R, T, g):
    """Who is slow, how much and since when: (factor[R], onset[R], ramp).  A few whole
    nodes drift to +20 %, a few single GPUs sit at +10 %, everybody else at 1."""
    N = R // 8
    factor = torch.ones(R, device=DEVICE)
    onset = torch.zeros(R, device=DEVICE)
    order = torch.randperm(N, device=DEVICE, generator=g)
    n_nodes, n_gpus = max(1, N // 256), max(1, N // 512)
    nodes = order[:n_nodes]
    factor.view(N, 8)[nodes] = 1.2
    onset.view(N, 8)[nodes] = (torch.rand(n_nodes, device=DEVICE, generator=g) * 0.5 * T)[:, None]
    gpus = order[n_nodes:n_nodes + n_gpus] * 8 + 3
    factor[gpus] = 1.1
    return factor, onset, max(1.0, 0.1 * T)


def _telemetry(case, seed, steps):
    """x[steps][metrics][ranks] fp32 on the GPU."""
    R, M = case["ranks"], case["metrics"]
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    factor, onset, ramp = _slowdown(R, steps, g)
    x = torch.empty((steps, M, R), dtype=torch.float32, device=DEVICE)
    chunk = max(1, min(steps, 33_554_432 // (M * R)))
    for t0 in range(0, steps, chunk):
        n = min(chunk, steps - t0)
        t = torch.arange(t0, t0 + n, dtype=torch.float32, device=DEVICE)[:, None]
        slow = 1.0 + (factor - 1.0) * ((t - onset) / ramp).clamp_(0.0, 1.0)          # [n][R]
        if case["noise"] == "lognormal":
            # one step time, the other metrics follow from it; one-step spikes of a factor of two
            step = torch.exp(0.02 * torch.randn((n, R), device=DEVICE, generator=g)) * slow
            step = torch.where(torch.rand((n, R), device=DEVICE, generator=g) < 0.005, 2.0 * step, step)
            compute = 0.7 * step
            for m, v in enumerate((step, compute, step - compute, 400.0 / step)[:M]):
                x[t0:t0 + n, m] = v
        else:
            # independent metrics with Student-t(3) noise of 2 % in log space
            z = torch.randn((n, M, R), device=DEVICE, generator=g)
            c = torch.zeros_like(z)
            for _ in range(3):
                c += torch.randn((n, M, R), device=DEVICE, generator=g).square_()
            z.mul_(0.02).div_(c.div_(3.0).sqrt_())
            for m in range(M):
                s = slow if DIRECTIONS[m] > 0 else 1.0 / slow
                x[t0:t0 + n, m] = BASES[m] * s * torch.exp(z[:, m])
    return x


def _membership(R, T, seed):
    """Bit words [T][ceil(R/64)]: one rank in a hundred is out for the whole batch, and
    in every step one node in five hundred was not polled in time."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed + 1)
    RW = (R + 63) // 64
    out = torch.rand(R, device=DEVICE, generator=g) < 0.01
    place = torch.arange(64, dtype=torch.int64, device=DEVICE)
    active = torch.empty((T, RW), dtype=torch.int64, device=DEVICE)
    chunk = max(1, 16_777_216 // R)
    for t0 in range(0, T, chunk):
        n = min(chunk, T - t0)
        missed = torch.rand((n, R // 8, 1), device=DEVICE, generator=g) < 0.002
        here = torch.zeros((n, RW * 64), dtype=torch.bool, device=DEVICE)
        here[:, :R] = ~(missed.expand(n, R // 8, 8).reshape(n, R) | out)
        active[t0:t0 + n] = (here.view(n, RW, 64).to(torch.int64) << place).sum(-1)
    return active


def _detector(case):
    M = case["metrics"]
    directions = (1, 1, 1, -1)[:M] if case["noise"] == "lognormal" else DIRECTIONS[:M]
    return Detector(Config(n_ranks=case["ranks"], n_metrics=M, window=case["window"],
                           persist_k=case["persist"], direction=directions), device=DEVICE)


def prepare(case, seed):
    kind, T = case["kind"], case["steps"]
    det = _detector(case)
    k = min(TOPK, det.N)
    s = {"kind": kind, "det": det, "steps": T, "k": k}
    if kind == "stream":
        s["x"] = _telemetry(case, seed, STREAM_HISTORY)
        s["at"] = 0
        s["out"], s["flags"], s["top"] = det.alloc_outputs(1), det.alloc_flags(), det.alloc_topk(k)
        s["out"]["med"].zero_()
        s["out"]["mad"].zero_()
        # each call starts looking at the medians and MADs of the one before
        det.set_streaming_hints(s["out"]["med"].view(-1), s["out"]["mad"].view(-1))
        return s
    s["x"] = _telemetry(case, seed, T)
    s["out"] = det.alloc_outputs(T, want_z=kind == "scores")
    if kind in ("batch", "missing", "scores"):
        s["flags"], s["top"] = det.alloc_flags(), det.alloc_topk(k)
    if kind == "missing":
        s["active"] = _membership(case["ranks"], T, seed)
    if kind == "ledger":
        det.score_batch(s["x"], s["out"])
        del s["x"]
        det.alloc_ledger(T)
        s["flags"], s["top"] = det.alloc_ledger_flags(), det.alloc_topk(k)
    if kind == "followup":
        det.score_batch(s["x"], s["out"])
        det.update_window(s["out"], T)
        s["tiers"] = det.alloc_severity()
        g = torch.Generator(device=DEVICE)
        g.manual_seed(seed + 2)
        # sweep results: throughputs and pairwise bandwidths within a few percent, the
        # odd GPU or link well below
        flops = 1.0 + 0.01 * torch.randn((det.N, 8), device=DEVICE, generator=g)
        bw = 1.0 + 0.02 * torch.randn((det.N, 8, 8), device=DEVICE, generator=g)
        flops[torch.rand(flops.shape, device=DEVICE, generator=g) < 0.005] *= 0.85
        bw[torch.rand(bw.shape, device=DEVICE, generator=g) < 0.001] *= 0.7
        s["flops"], s["bw"] = 1200.0 * flops, 140.0 * bw
    return s


def run(s):
    kind, det, T = s["kind"], s["det"], s["steps"]
    if kind == "ledger":
        det.update_ledger(s["out"], T)
        det.ledger_flags(s["flags"])
        det.topk_nodes_mean(s["k"], s["top"])
        return {"flags": s["flags"], "top": s["top"]}
    if kind == "followup":
        det.severity(s["x"], s["out"], s["tiers"])
        return {"tiers": s["tiers"], "sweep": det.sweep_score(s["flops"], s["bw"])}
    x = s["x"]
    if kind == "stream":
        x = x[s["at"]:s["at"] + 1]
        s["at"] = (s["at"] + 1) % STREAM_HISTORY
    elif kind == "missing":
        det.apply_membership(x, s["active"])
    det.score_batch(x, s["out"])
    det.update_window(s["out"], T)
    det.flags(s["flags"])
    det.topk_nodes(s["k"], s["top"])
    return {"scores": s["out"], "flags": s["flags"], "top": s["top"], "window": det.state}


# ---- what a pass cannot do without --------------------------------------------------------

def work(case):
    kind, R, M, T, W = case["kind"], case["ranks"], case["metrics"], case["steps"], case["window"]
    N, RW, NW, keep = R // 8, (R + 63) // 64, (R // 8 + 63) // 64, min(case["steps"], case["window"])
    top = min(TOPK, N) * 12
    if kind == "ledger":
        read = T * (R + N) + keep * N * 4                           # exceed bytes, the window's node scores
        rings = 2 * keep * (R + N) + keep * N * 2 + min(W, T) * N * 2
        counts = 2 * (R + N) * 20 + N * 50                          # per-metric counts, first steps, episode starts
        outs = (R + N) * 6 + N * 9 + top
        return {"bytes": read + rings + counts + outs, "flops": T * (R + N) * 8}
    if kind == "followup":
        slow = max(1, N // 256) + max(1, N // 512)                  # nodes whose samples must be read
        tiers = R * 2 + N * 2 + slow * 8 * keep * 4 + keep * 4 + N * 5
        sweep = N * (8 + 64) * 4 + N * (8 * 4 + 1 + 4 + 1)
        return {"bytes": tiers + sweep, "flops": slow * 8 * keep + N * 100}
    x = 4 * M * R * T
    scores = T * (8 * M + R + 8 * RW + 4 * N + N + 8 * NW) + (x if kind == "scores" else 0)
    window = 2 * keep * (RW + NW) * 8 + 2 * (R + N) * 6 + N * 8     # rings, counts and first steps, latest node scores
    outs = (R + N) * 7 + top
    active = T * RW * 8 if kind == "missing" else 0
    return {"bytes": x + scores + window + outs + active, "flops": 2 * M * R * T}


def tolerance(case):
    # Medians, MADs, masks, counters, flags, first steps, rankings and node scores follow from
    # comparisons and from operations rounded once each: one correct implementation gives the
    # same bits as another.  The full z output is held to 1e-6 (its quotient may be formed from
    # a reciprocal), which is also the bound that the repository's tests put on it.
    return {"rel": 1e-6} if case["kind"] == "scores" else "exact"
