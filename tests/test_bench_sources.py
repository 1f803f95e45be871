"""The hash by which bench.py knows stale counter figures covers every source
that defines or launches a matrix-core kernel or chooses a launch's shape."""
import os
import shutil

import bench


def test_hash_covers_every_kernel_and_launch_source(tmp_path, monkeypatch):
    pkg = tmp_path / "paper_2604_22718_amd"
    shutil.copytree(os.path.join(bench.ROOT, "paper_2604_22718_amd"), pkg, ignore=shutil.ignore_patterns("*.so*", "__pycache__"))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    start = bench.src_hash()
    others = {"rtt_tt.hpp", "rtt_narrow.hpp", "rtt_net.hpp"}
    for f in sorted(os.listdir(pkg / "csrc")) + ["../build.py"]:
        p = pkg / "csrc" / f
        text = p.read_bytes()
        p.write_bytes(text + b"\n")
        assert (bench.src_hash() == start) == (f in others), f
        p.write_bytes(text)
    assert bench.src_hash() == start
