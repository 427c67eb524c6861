"""bench.py quotes a measured profile only where it was taken on the current device sources: a
change to any of them, the grouped GEMMs' headers and files among them, makes it unmeasured."""
import json
import os
import shutil
from types import SimpleNamespace

import pytest

import bench

CSRC = os.path.join("paper_2607_09686_amd", "csrc")
DEVICE = sorted(f for f in os.listdir(os.path.join(bench.ROOT, CSRC)) if f.endswith((".hip", ".h")))


@pytest.mark.parametrize("name", DEVICE)
def test_a_changed_device_source_ends_a_profile(tmp_path, monkeypatch, name):
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    record = {"kernel_sources_sha256_16": bench.kernel_sources_sha256_16(), "workload": "w",
              "traffic_bytes_per_launch": 5}
    (tmp_path / "k_traffic.json").write_text(json.dumps(record))
    args = SimpleNamespace(profiles=str(tmp_path), policy="lru")
    wl = SimpleNamespace(name="w", budget_slots=3)
    assert bench.measured_traffic(args, "k", wl, 3) == 5
    with open(tmp_path / CSRC / name, "a") as f:
        f.write("\n// changed\n")
    assert bench.measured_traffic(args, "k", wl, 3) is None

