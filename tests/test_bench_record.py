"""The committed counter record is dropped when what the pair kernel's launch depends on changes."""
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

CSRC = "paper_astro_ph_0703100_amd/csrc/"


@pytest.mark.parametrize("rel,old,new", [
    (CSRC + "api.cpp", "blocks >= 1000000 ? 4", "blocks >= 2000000 ? 4"),  # records per lane
    (CSRC + "tuning.cpp", "return {1, 256, 0};", "return {1, 128, 0};"),   # built-in shape
    (CSRC + "gravity.h", "s_nop 2", "s_nop 1"),
    (bench.TUNING_FILE, '"nseg": 40', '"nseg": 41')])
def test_hash_follows_the_launch(tmp_path, monkeypatch, rel, old, new):
    for f in bench.KERNEL_SOURCES + [bench.TUNING_FILE]:
        os.makedirs(tmp_path / os.path.dirname(f), exist_ok=True)
        shutil.copy(os.path.join(ROOT, f), tmp_path / f)
    before = bench.sources_hash()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.sources_hash() == before
    path = tmp_path / rel
    assert old in path.read_text()
    path.write_text(path.read_text().replace(old, new))
    assert bench.sources_hash() != before
