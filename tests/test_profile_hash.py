"""A committed counter summary counts as current only while the kernel's file and
every header that it includes are unchanged (host only)."""
import json
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("prec,kernel", [("fp64", "lbe_moment.hip"), ("fp32", "lbe_fluid.hip")])
def test_summary_is_dropped_when_a_header_changes(prec, kernel, tmp_path, monkeypatch):
    import bench
    from paper_1109_3277_amd import profile_summary as P

    shutil.copytree(os.path.join(ROOT, "paper_1109_3277_amd", "csrc"), tmp_path / "pkg" / "csrc")
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    monkeypatch.setattr(P, "HERE", str(tmp_path / "pkg"))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    path = P.fluid_source(prec == "fp64")
    assert os.path.basename(path) == kernel
    os.makedirs(tmp_path / "profiles")
    rec = {"source_sha256_16": P.source_hash(path), "bytes_per_launch": 17}
    json.dump(rec, open(tmp_path / "profiles" / f"fused_{prec}_some_pmc.json", "w"))
    assert bench.measured_traffic("some", prec) == 17
    headers = ["lbe_device.h", "lbe_internal.h"] + (["lbe_moment.h"] if prec == "fp64" else [])
    for name in [kernel] + headers:
        f = tmp_path / "pkg" / "csrc" / name
        old = f.read_bytes()
        f.write_bytes(old + b"\n// changed\n")
        assert bench.measured_traffic("some", prec) is None, name
        f.write_bytes(old)
        assert bench.measured_traffic("some", prec) == 17, name
