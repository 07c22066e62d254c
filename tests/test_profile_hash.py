"""The hash that ties a kernel profile to its sources changes with every local header that the
rollout kernels' sources include, so that the bench takes no counters of another kernel."""
import os
import re
import shutil

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CS = os.path.join("paper_2409_10469_amd", "csrc")


def _included(names):
    seen, todo = set(), list(names)
    while todo:
        n = todo.pop()
        if n in seen or not os.path.exists(os.path.join(ROOT, CS, n)):
            continue
        seen.add(n)
        with open(os.path.join(ROOT, CS, n)) as f:
            todo += re.findall(r'#include "([^"]+)"', f.read())
    return sorted(seen)


def test_profile_hash_covers_the_kernels_sources(tmp_path, monkeypatch):
    names = _included(["mppi_kernels.hip", "rollout16.hip"])
    assert "mppi_device.h" in names
    os.makedirs(tmp_path / CS)
    for n in names:
        shutil.copy(os.path.join(ROOT, CS, n), tmp_path / CS / n)
    shutil.copy(os.path.join(ROOT, "paper_2409_10469_amd", "build.py"), tmp_path / "paper_2409_10469_amd" / "build.py")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    base = bench.kernel_source_hash()
    for n in names:
        with open(tmp_path / CS / n, "a") as f:
            f.write("\n// changed\n")
        new = bench.kernel_source_hash()
        assert new != base, n
        base = new
