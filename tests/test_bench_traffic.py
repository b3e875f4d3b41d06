"""CPU checks of bench.py's HBM-traffic figures: each committed counter summary is quoted only while the sources it was
counted on are unchanged, the shared tile order among them, and only for launches of the size that was counted."""
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CSRC = os.path.join("paper_2007_03638_amd", "csrc")
SUMMARIES = {"gett_f32_chi24_counters.md": ("gett<f32,192x192,Am,Bn,v,k2>", "gett.hip"),
             "gett_split_chi24_counters.md": ("gett<f32,128x192,Am,Bn,v,k2,s3>", "gett_split_device.h")}


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """A copy of what the figures are read from."""
    shutil.copytree(os.path.join(ROOT, "profiles"), tmp_path / "profiles")
    os.makedirs(tmp_path / CSRC)
    for f in ("gett.hip", "gett_split_device.h", "gett_device.h"):
        shutil.copy(os.path.join(ROOT, CSRC, f), tmp_path / CSRC / f)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return tmp_path


@pytest.mark.parametrize("summary", SUMMARIES)
def test_quoted_for_its_sources_and_size_only(tree, summary):
    variant, source = SUMMARIES[summary]
    text = (tree / "profiles" / summary).read_text()
    fields = dict(l.split(": ", 1) for l in text.splitlines() if ": " in l and not l.startswith("|"))
    size, traffic = float(fields["algorithmic_bytes_per_launch"]), float(fields["traffic_bytes_per_launch"])
    assert traffic > 0.9 * size
    assert bench.counter_traffic(variant) == bench.counter_traffic(variant, size) == traffic
    assert bench.counter_traffic(variant, 1.05 * size) == traffic
    assert bench.counter_traffic(variant, 2.0 * size) is None and bench.counter_traffic(variant, 0.01 * size) is None
    for changed in (source, "gett_device.h"):
        path = tree / CSRC / changed
        kept = path.read_bytes()
        path.write_bytes(kept + b"\n")
        assert bench.counter_traffic(variant) is None
        path.write_bytes(kept)
    assert bench.counter_traffic(variant) == traffic
