"""The hints of a run's first step come from samples of its columns, taken all at once: here exactly the
sampled ranks mislead, as the kernel's own header (gd_sample.h, compiled for the host) gives them, in
every share of waves and columns -- four, two and one wave to a column, two columns to a wave.  The
selection must notice and still return the exact statistics.  Bit for bit against the oracle."""
import os
import subprocess

import numpy as np
import pytest
import torch

from gpu_harness import oracle_params, run_and_compare

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2605_17879_amd", "csrc")

HIP = """
#define __device__
#define __forceinline__ inline
"""

MAIN = r"""
#include "gd_sample.h"
#include <stdio.h>
#include <stdlib.h>
int main(int, char** argv) {
    const uint32_t R = atoi(argv[1]), columns = atoi(argv[2]), waves = atoi(argv[3]);
    for (uint32_t place = 0; place < 64u << sample_parts_log(columns, waves); ++place) printf("%u\n", sample_rank(place, R));
    return 0;
}
"""

# threads of the run-of-steps tiling of a rank count, where all columns of the first step are sampled at once
THREADS = [(4097, 14336, 256), (16385, 32768, 512), (32769, 65536, 1024)]


def threads_of(R):
    return next(nt for lo, hi, nt in THREADS if lo <= R <= hi)


@pytest.fixture(scope="module")
def sampled_ranks(tmp_path_factory):
    d = tmp_path_factory.mktemp("sample")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(HIP)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "ranks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{d}", f"-I{CSRC}", str(d / "main.cpp"), "-o", exe], check=True)

    def ranks(R, M):
        out = subprocess.run([exe, str(R), str(M), str(threads_of(R) // 64)], check=True, capture_output=True, text=True).stdout
        return np.array(out.split(), dtype=np.int64)            # the first of four neighbours each
    return ranks


# (four waves a column, two, one, and more columns than waves, in each width of workgroup that has them)
SIZES = [(4104, 1), (5000, 2), (8184, 3), (10000, 8), (14336, 5), (16392, 2), (24000, 4), (32768, 8), (32776, 4), (40000, 8),
         (65528, 3), (65536, 8)]


@pytest.mark.parametrize("R,M", SIZES)
def test_the_sampled_ranks_lie_in_the_column_and_all_over_it(sampled_ranks, R, M):
    first = sampled_ranks(R, M)
    waves = threads_of(R) // 64
    assert len(first) == 64 * (4 if 4 * M <= waves else 2 if 2 * M <= waves else 1)
    assert first.min() >= 0 and first.max() + 4 <= R and np.all(first % 4 == 0)
    assert len(set(first.tolist())) == len(first)
    # sixteen multiples of the golden ratio leave no gap wider than its fifth power, 0.09: a piece in each eighth
    assert np.all(np.bincount(first * 8 // R, minlength=8) >= 4)


# what the sampled values are instead of themselves (c: the column's median, s: its sampled values, [n][4] with
# a lot of the wave's sort in each of the four places)
def _mislead(kind, c, s, rng):
    if kind == "far above":
        return s * 50.0
    if kind == "other scale":
        return np.abs(c + (s - c) * 300.0) + 1e-3 * c
    if kind == "too tight":
        return c + (s - c) * 1e-3
    if kind == "missing":
        return np.full_like(s, np.nan)
    if kind == "one lot arrived":
        s = s.copy(); s[:, 1:] = np.nan; return s
    if kind == "three lots arrived":
        s = s.copy(); s[:, 2] = np.nan; return s
    if kind == "few arrived":                                  # (fewer than a lot needs, in each of them)
        s = s.copy(); s[rng.permutation(len(s))[10:]] = np.nan; return s
    if kind == "negative":
        return -s
    if kind == "one negative":
        s = s.copy(); s[0, 0] = -s[0, 0]; return s
    if kind == "constant":
        return np.full_like(s, c)
    if kind == "alike in one lot":
        s = s.copy(); s[:, 0] = c; return s
    if kind == "alike in two lots":
        s = s.copy(); s[:, :2] = c * 1.001; return s
    if kind == "next to infinity":
        s = s.copy(); s[rng.random(s.shape) < 0.3] = 3.0e38; return s
    if kind == "skewed":                                       # (one side hundreds of times the other)
        return np.where(s < c, c - (c - s) * 1e-2, c + (s - c) * 20.0)
    if kind == "next to zero":
        return (np.abs(s - c) / c * 1e-38 + 1e-44)
    assert kind == "as they are"
    return s


KINDS = ["far above", "other scale", "too tight", "missing", "one lot arrived", "three lots arrived", "few arrived", "negative",
         "one negative", "constant", "alike in one lot", "alike in two lots", "next to infinity", "skewed", "next to zero", "as they are"]


@pytest.mark.gpu
@pytest.mark.parametrize("R,M", SIZES)
def test_misleading_samples_of_a_run_s_first_step(sampled_ranks, R, M):
    """Every step of these short batches is a run's first; each kind meets each metric, the whole column's
    values are even, skewed and of few distinct values in turn."""
    print(f"case first samples R={R} M={M}", flush=True)
    rng = np.random.default_rng(R + M)
    T = len(KINDS)
    at = sampled_ranks(R, M)[:, None] + np.arange(4)
    x = np.empty((T, M, R))
    for t in range(T):
        for m in range(M):
            n = rng.standard_normal(R)
            shape = (t + 2 * m) % 3
            col = np.exp(0.02 * n) if shape == 0 else np.exp(n) if shape == 1 else np.round(65.0 + 4.0 * n)
            kind = KINDS[(t + 5 * m) % T]
            col[at] = _mislead(kind, np.median(col), col[at], rng)
            x[t, m] = col
    x = torch.from_numpy(x.astype(np.float32))
    p = oracle_params(R=R, M=M, W=4, k=2, directions=(1, -1, 0, 1, -1, 1, 0, 1)[:M], min_signals=min(2, M))
    import gpu_harness
    gpu_harness.STREAMING_STEPS = 0                             # whole-run route
    try:
        run_and_compare(p, x, topk_k=8, chunks=[T], label=f"first samples R{R} M{M}", want_z=False)
    finally:
        gpu_harness.STREAMING_STEPS = None
