"""The committed HBM traffic of the dominant sweep counts only for the sources
it was taken on: a change to its kernel, its plan or its dispatch drops it."""
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join("paper_1702_08521_amd", "csrc")
KEY = "landau_3d3v/f32"


@pytest.fixture
def copy(tmp_path, monkeypatch):
    sys.path.insert(0, ROOT)
    import bench

    shutil.copytree(os.path.join(ROOT, CSRC), tmp_path / CSRC)
    shutil.copytree(os.path.join(ROOT, "profiles"), tmp_path / "profiles")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return bench, tmp_path


def test_record_is_of_these_sources(copy):
    bench, _ = copy
    assert bench.read_traffic(KEY) > 0


@pytest.mark.parametrize("name", ["sweep_device.hpp", "sweep_kernels.hpp", "sweep_launch.hpp", "slmpp_internal.hpp",
                                  "sweep.hip", "sweep_f32.hip", "api.hip"])
def test_record_is_dropped_when_a_source_changes(copy, name):
    bench, root = copy
    with open(root / CSRC / name, "a") as f:
        f.write("\n")
    assert bench.read_traffic(KEY) is None
