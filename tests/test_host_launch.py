"""The host's choices and checks around the pair launch, compiled from the
library's host source and run without a GPU."""
import os
import subprocess

from paper_1911_08275_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_checks(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path / "launch_checks")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    src, obj = os.path.join(ROOT, "tests", "host", "launch_checks.hip"), exe + ".o"
    lib = os.path.dirname(build.LIB)
    for cmd in ([build.HIPCC, "-O1"] + flags + ["-c", src, "-o", obj],
                [build.HIPCC, "--offload-arch=gfx950", obj, "-L" + lib, "-lcountpairs",
                 "-Wl,-rpath," + lib, "-o", exe]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, CP_AUTOTUNE_CACHE=str(tmp_path / "tune.json")))
    assert r.returncode == 0 and "launch checks passed" in r.stdout, (r.stdout, r.stderr)
