"""The library's host code over a stand-in for the HIP runtime and the kernels (CPU only): what
calls launch and allocate, and their error paths. See host_calls_driver.cpp for the scenarios."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_18022_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_calls") / "driver")
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
         "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", out,
         os.path.join(ROOT, "tests", "host_calls_driver.cpp"),
         *(os.path.join(CSRC, f) for f in ("split_host.cpp", "nn_host.cpp", "search_host.cpp"))])
    return out


@pytest.mark.parametrize("scenario", [
    "flag-of-a-failed-pass", "scenarios-after-a-failed-allocation",
    "autotune-times-the-own-choice", "graph-replays-choose-by-their-tours",
    "two-wavefronts-by-length-and-items", "sums-of-batches", "prep-workgroups",
    "timing-names-the-dominant-kernel",
])
def test_host_calls(driver, scenario):
    # nothing preloaded comes before the sanitizer's runtime, which the driver links first
    env = {**os.environ, "ASAN_OPTIONS": "detect_leaks=0:verify_asan_link_order=0"}
    res = subprocess.run([driver, scenario], capture_output=True, text=True, env=env, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr[-2000:]
