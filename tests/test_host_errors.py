"""Error paths of plora_batch_begin, the way of its image and the items of its lists, on the CPU: tests/native/host_errors.cpp links the library's host
code against the stand-in HIP runtime of tests/native/fake_hip.cpp, whose calls can be made to fail."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_errors") / "host_errors")
    nat = os.path.join(ROOT, "tests", "native")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
           "-I" + os.path.join(ROOT, "paper_2512_20210_amd", "csrc"), "-I" + nat,
           os.path.join(nat, "host_errors.cpp"), os.path.join(nat, "fake_hip.cpp"),
           os.path.join(ROOT, "paper_2512_20210_amd", "csrc", "plora_pool.cpp"), "-o", out]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:]
    return out


@pytest.mark.parametrize("check", ["image_in_flight", "callers_error", "counters_cleared", "fp32_thresholds", "panel_route", "fp32_route", "rest_tables"])
def test_batch_begin(exe, check):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe, check], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120, env=env)
    assert r.returncode == 0 and check + " OK" in r.stdout, r.stdout[-3000:]
