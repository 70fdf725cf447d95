"""The counter records under profiles/ describe one state of the scoring kernel: the
benchmark's guard on them has to see a change to any file that the kernel is made of."""
import json
import os
import shutil

import bench

CSRC = os.path.join("paper_2605_17879_amd", "csrc")


def test_every_file_of_the_kernel_counts(tmp_path, monkeypatch):
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    whole = bench._score_source_hash()
    (tmp_path / "profiles" / "r.json").write_text(json.dumps({"score_sources_sha256": whole}))
    assert bench._profile_record("r.json") is not None
    for name in ("score.hip", "score_small.h", "gd_lanes.h", "gd_internal.h", "gd_grant.h"):
        path = tmp_path / CSRC / name
        text = path.read_text()
        path.write_text(text + "\n// changed\n")
        assert bench._score_source_hash() != whole and bench._profile_record("r.json") is None, name
        path.write_text(text)
    (tmp_path / CSRC / "window.hip").write_text("// another kernel\n")
    assert bench._score_source_hash() == whole and bench._profile_record("r.json") is not None
