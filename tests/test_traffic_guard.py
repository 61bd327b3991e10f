"""bench.py reports committed HBM traffic only for the kernels it was counted
on: their source, the header with their layouts and waves per SIMD, and the
compiler flags (CPU)."""
import hashlib
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


@pytest.mark.parametrize("change", ["none", "pair_kernels.hip", "cp_internal.h", "flags"])
def test_traffic_only_for_the_build_it_was_counted_on(change, tmp_path, monkeypatch):
    import bench
    from paper_1911_08275_amd import build
    csrc = os.path.join(ROOT, "paper_1911_08275_amd", "csrc")
    files = []
    for name in ("pair_kernels.hip", "cp_internal.h"):
        with open(os.path.join(csrc, name), "rb") as f:
            files.append(tmp_path / name)
            files[-1].write_bytes(f.read())
    monkeypatch.setattr(bench, "KERNEL_FILES", [str(f) for f in files])
    summary = tmp_path / "traffic.md"
    summary.write_text("- pair_kernels.hip sha256: `%s`\n- pair kernel build sha256: `%s`\n"
                       "- refine: `2,2,2`\n- fetch bytes per launch: `5`\n"
                       "- write bytes per launch: `7`\n"
                       % (hashlib.sha256(files[0].read_bytes()).hexdigest(),
                          bench.kernel_build_hash()))
    monkeypatch.setattr(bench, "TRAFFIC_FILES", [str(summary)])
    if change == "flags":
        monkeypatch.setattr(build, "FLAGS", build.FLAGS + ["-O2"])
    elif change != "none":
        path = tmp_path / change
        path.write_bytes(path.read_bytes() + b"\n")
    assert bench.measured_traffic([2, 2, 2]) == (12 if change == "none" else None)
    assert bench.measured_traffic([2, 2, 3]) is None
