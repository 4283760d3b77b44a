"""The two-stream exchange calls of the host layer under the sanitizers, with
the stand-ins of test_host_threads.  CPU only."""
import os
import shutil
import subprocess

import pytest

from test_host_threads import CSRC, HARNESS, ROOT, SANITIZERS


@pytest.mark.parametrize("kind", list(SANITIZERS))
def test_two_lanes_under_sanitizer(tmp_path, kind):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    host_src = tmp_path / "lace_api_host.cpp"
    shutil.copyfile(os.path.join(CSRC, "lace_api.hip"), host_src)
    exe = tmp_path / f"drive_{kind}"
    cmd = [gxx, "-std=c++17", "-O1", "-g", *SANITIZERS[kind],
           "-I", HARNESS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           str(host_src), *(os.path.join(HARNESS, f) for f in
                            ("stub_runtime.cpp", "stub_launch.cpp", "drive_lanes.cpp")),
           "-o", str(exe), "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    env = dict(os.environ, TSAN_OPTIONS="halt_on_error=1 exitcode=66",
               ASAN_OPTIONS="detect_leaks=1 exitcode=67")
    r = subprocess.run([str(exe), "4", "2"], capture_output=True, text=True,
                       timeout=300, env=env)
    out = r.stdout + r.stderr
    assert r.returncode == 0, out[-4000:]
    assert "two lanes: 4 threads x 2 reps ok" in out
    for bad in ("ThreadSanitizer", "AddressSanitizer", "runtime error",
                "LeakSanitizer"):
        assert bad not in out, out[-4000:]
