"""The few-edge tables (one edge per table cell, decided by the sign of a
difference) against the decision tables and the definition: every certain
decision holds for all binary64 values within the error bound of the binary32
estimate, at and around every edge, band end and cell boundary (CPU)."""
import os
import subprocess

from paper_1911_08275_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_few_edge_tables(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path / "few_edge_checks")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    src, obj = os.path.join(ROOT, "tests", "host", "few_edge_checks.hip"), exe + ".o"
    lib = os.path.dirname(build.LIB)
    for cmd in ([build.HIPCC, "-O1"] + flags + ["-c", src, "-o", obj],
                [build.HIPCC, "--offload-arch=gfx950", obj, "-L" + lib, "-lcountpairs",
                 "-Wl,-rpath," + lib, "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "few-edge checks passed" in r.stdout, (r.stdout, r.stderr)
