"""Host-only checks of C-ABI calls (csrc/api.cpp) on models: tests/host/calls_driver.cpp with
stand-ins for the HIP runtime and the kernel launchers (tests/host/fake_runtime.cpp), under
AddressSanitizer and UndefinedBehaviorSanitizer.  No GPU is used."""
import os
import subprocess

import pytest

from tests.test_host_sanitizers import CSRC, HIPCC, HOST, ROOT, SAN


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("calls"))
    common = ["-O1", "-g", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"), "-I", CSRC] + SAN
    objs = []
    for src, lang in [(os.path.join(CSRC, "api.cpp"), ["-x", "hip"]), (os.path.join(HOST, "fake_runtime.cpp"), ["-x", "hip"]),
                      (os.path.join(HOST, "calls_driver.cpp"), [])]:
        obj = os.path.join(out, os.path.basename(src) + ".o")
        r = subprocess.run([HIPCC] + common + lang + ["-c", src, "-o", obj], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        objs.append(obj)
    exe = os.path.join(out, "calls_driver")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950"] + SAN + objs + ["-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("check", ["large_orders", "points_errors", "tuned_tiles", "tune_keys"])
def test_host_calls(driver, check, tmp_path):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1",
               DSX_TUNE_CACHE=str(tmp_path / "tune.txt"))
    r = subprocess.run([driver, check], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-6000:])
    assert "passed" in r.stdout
