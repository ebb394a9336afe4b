"""What the benchmark reports of the kernels.

Committed HBM counters only for the kernels they were taken on: a change in any source that holds
a timed kernel, or a header that such a source includes, has to change the digest that the
counter files carry.  The classes that share the strokes' launches as one row."""
import os
import re
import shutil

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_0907_4863_amd", "csrc")


def timed_sources():
    """The sources whose launchers take a kernel timer, and the headers they include."""
    todo = [f for f in os.listdir(CSRC) if f.endswith(".hip") and f != "timer.hip"
            and re.search(r"\bKTimer\b", open(os.path.join(CSRC, f)).read())]
    seen = set()
    while todo:
        f = todo.pop()
        if f in seen or not os.path.exists(os.path.join(CSRC, f)):
            continue
        seen.add(f)
        todo += re.findall(r'#include "([a-z_]+\.h)"', open(os.path.join(CSRC, f)).read())
    return sorted(seen - {"host_prep.h"})


@pytest.mark.parametrize("name", timed_sources())
def test_a_change_of_a_kernel_source_changes_the_digest(name, tmp_path, monkeypatch):
    copy = tmp_path / "paper_0907_4863_amd" / "csrc"
    shutil.copytree(CSRC, copy)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench._kernel_sources_digest()
    with open(copy / name, "a") as fh:
        fh.write("\n")
    assert bench._kernel_sources_digest() != before


def test_counters_of_other_sources_are_not_reported(tmp_path, monkeypatch):
    shutil.copytree(CSRC, tmp_path / "paper_0907_4863_amd" / "csrc")
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    text = "fetch_bytes_per_launch 3e8\nwrite_bytes_per_launch 1e8\nsources_sha256 "
    path = tmp_path / "profiles" / "traffic_cg_xr_box.txt"
    path.write_text(text + bench._kernel_sources_digest() + "\n")
    assert bench.measured_traffic("cg_xr", "box") == 4e8
    path.write_text(text + "0" * 64 + "\n")
    assert bench.measured_traffic("cg_xr", "box") is None


def _rows(launches):
    return {k: {"total_ms": ms, "launches": n, "avg_us": 1e3 * ms / n, "alg_bytes_per_launch": b / n,
                "achieved_GBs": b / (ms * 1e-3) / 1e9}
            for (k, n), ms, b in zip(launches.items(), (3.0, 1.0, 1.0, 1.0, 4.0), (6e9, 2e9, 2e9, 2e9, 9e9))}


def test_strokes_are_one_class_of_the_bench():
    """The shares of a stroke's launch in four classes add up to one row with the strokes' time,
    launches, bytes and rate; step kernels (three smoother launches a prolongation) keep theirs."""
    kinds = {"l0_cheb": 46, "l0_resid": 23, "l0_restrict": 23, "l0_prolong": 23, "cg_xr": 22}
    got = bench.join_strokes(_rows(kinds))
    assert set(got) == {"l0_strokes", "cg_xr"}
    s = got["l0_strokes"]
    assert s["launches"] == 46 and s["total_ms"] == 6.0 and abs(s["achieved_GBs"] - 2000.0) < 1e-9
    assert abs(s["alg_bytes_per_launch"] * 46 - 12e9) < 1.0 and abs(s["avg_us"] * 46 - 6000.0) < 1e-9
    by_steps = _rows(dict(kinds, l0_cheb=69))
    assert bench.join_strokes(by_steps) is by_steps
