"""The scoring kernel's design rests on a whole column living in registers with 16 waves
per compute unit: at most 128 vector registers per lane and nothing spilled.  The
compiler's own resource report (-Rpass-analysis=kernel-resource-usage, written beside the
objects by the build) is parsed here; no GPU is needed."""
import os
import re

import pytest

from paper_2605_17879_amd import build as hip_build

SOURCES = ("score.hip", "score_z.hip")


def _report(src):
    path = hip_build.resource_file(src)
    source = os.path.join(hip_build.CSRC, "score.hip")
    if not os.path.exists(path) or os.path.getmtime(path) < os.path.getmtime(source):
        hip_build.build()                       # (the build writes the reports)
    with open(path) as f:
        return hip_build.parse_resources(f.read())


@pytest.mark.parametrize("src", SOURCES)
def test_every_scoring_instantiation_is_within_the_register_budget(src):
    res = _report(src)
    tilings = {k: hip_build.tiling_of(k) for k in res if hip_build.tiling_of(k)}
    want_z = 1 if src == "score_z.hip" else 0
    # the exact-fit tilings of whole batches and those of the per-column route
    batch = {(64, 1, 10), (64, 4, 10), (256, 4, 11), (256, 16, 11), (512, 16, 12), (1024, 16, 12)}
    column = {(64, 1, 10), (64, 4, 10), (256, 4, 11), (1024, 4, 12), (1024, 8, 12), (1024, 16, 12)}
    seen_batch = {t[:3] for t in tilings.values() if t[4] == 0 and t[5] == want_z}
    seen_column = {t[:3] for t in tilings.values() if t[4] == 1 and t[5] == want_z}
    assert seen_batch == batch and seen_column == column, (seen_batch, seen_column)
    assert hip_build.check_register_budget(res) == []
    for name, t in tilings.items():
        r = res[name]
        assert r["VGPRs"] + r["AGPRs"] <= hip_build.VGPR_BUDGET, name
        assert r["Occupancy [waves/SIMD]"] >= 4, name
        assert r["LDS Size [bytes/block]"] == 0, name          # all of its LDS is dynamic (sized by the launcher)
        if t[3] and t[0] >= 256 and not t[4]:                  # exact-fit batch tilings: nothing in scratch memory
            assert r["VGPRs Spill"] == 0 and r["ScratchSize [bytes/lane]"] == 0, (name, r)


RAGGED = {"few": {(64, 1, 10), (64, 2, 10), (64, 4, 10), (64, 8, 10), (64, 12, 10), (64, 16, 10), (256, 4, 11),
                  (256, 6, 11), (256, 8, 11)},
          "many": {(nt, rows, log) for nt, log in ((256, 11), (512, 12), (1024, 12)) for rows in (10, 12, 14, 16)},
          "columns": {(256, 4, 11)} | {(1024, rows, 12) for rows in (2, 4, 6, 8, 10, 12, 14, 16)}}


@pytest.mark.parametrize("src", hip_build.RAGGED_SOURCES)
def test_every_ragged_instantiation_is_within_the_register_budget(src):
    res = {k: r for k, r in _report(src).items() if hip_build.is_ragged(k)}
    seen = {tuple(int(g) for g in re.search(r"score_ragged_kernelILi(\d+)ELi(\d+)ELi(\d+)E", k).groups()) for k in res}
    kind = re.match(r"score_ragged_([a-z]+?)(_z)?\.hip", src).group(1)
    assert seen == RAGGED[kind], seen
    assert hip_build.check_register_budget(res) == []
    for name, r in res.items():
        assert r["VGPRs"] + r["AGPRs"] <= hip_build.VGPR_BUDGET and r["Occupancy [waves/SIMD]"] >= 4, name


def test_the_parser_reads_the_compiler_remarks():
    text = """x.hip:1:1: remark: Function Name: _ZN1_12score_kernelILi1024ELi16ELi12ELb1ELb0ELb0EEEv13gd_score_args [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     VGPRs: 129 [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     AGPRs: 0 [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     ScratchSize [bytes/lane]: 16 [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     Dynamic Stack: False [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     Occupancy [waves/SIMD]: 3 [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     VGPRs Spill: 4 [-Rpass-analysis=kernel-resource-usage]
"""
    res = hip_build.parse_resources(text)
    (name, r), = res.items()
    assert hip_build.tiling_of(name) == (1024, 16, 12, 1, 0, 0)
    assert r == {"VGPRs": 129, "AGPRs": 0, "ScratchSize [bytes/lane]": 16, "Dynamic Stack": False,
                 "Occupancy [waves/SIMD]": 3, "VGPRs Spill": 4}
    bad = hip_build.check_register_budget(res)
    assert len(bad) == 3, bad


@pytest.mark.parametrize("kernel,needed", [
    ("score_ragged_kernelILi256ELi8ELi11ELb0ELb0EEE", 5), ("score_ragged_kernelILi256ELi8ELi11ELb0ELb1EEE", 4),
    ("score_ragged_kernelILi256ELi10ELi11ELb0ELb0EEE", 4), ("score_kernelILi256ELi4ELi11ELb1ELb0ELb0EEE", 5),
    ("score_kernelILi256ELi4ELi11ELb1ELb0ELb1EEE", 4), ("score_kernelILi512ELi16ELi12ELb1ELb0ELb0EEE", 4)])
def test_the_check_asks_for_the_waves_that_the_launcher_counts_on(kernel, needed):
    name = f"_ZN1_1{kernel}v13gd_score_args"
    for waves in (needed - 1, needed):
        res = {name: {"VGPRs": 96, "AGPRs": 0, "ScratchSize [bytes/lane]": 0, "Occupancy [waves/SIMD]": waves,
                      "VGPRs Spill": 0, "Dynamic Stack": False}}
        assert len(hip_build.check_register_budget(res)) == (1 if waves < needed else 0)
