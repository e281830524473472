"""The runtime behind the C boundary on a device made of host memory (no GPU): tests/host_device_driver.cpp defines the
HIP calls and the launches, is built with the host sources under AddressSanitizer and UndefinedBehaviorSanitizer, and checks
what happens when memory runs out and what the kernels are handed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1903_00757_amd", "csrc")
DRIVER = os.path.join(ROOT, "tests", "host_device_driver.cpp")
HIPCC = "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = tmp_path_factory.mktemp("host_device")
    sanitizers = "-Xarch_host -fsanitize=address -Xarch_host -fsanitize=undefined -Xarch_host -fno-omit-frame-pointer".split()
    link = "-fsanitize=address -fsanitize=undefined -fno-gpu-sanitize".split()
    common = [HIPCC, "-std=c++17", "-O1", "-g", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
              "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objects = []
    for src in [os.path.join(CSRC, f) for f in ("gv_api.cpp", "gv_plan.cpp", "gv_augment.cpp")] + [DRIVER]:
        obj = str(out / (os.path.basename(src) + ".o"))
        subprocess.run([*common, "-x", "hip", *sanitizers, "-c", src, "-o", obj], check=True, capture_output=True, text=True)
        objects.append(obj)
    exe = str(out / "driver")
    subprocess.run([HIPCC, "--offload-arch=gfx950", *link, *objects, "-o", exe, "-lpthread"], check=True, capture_output=True,
                   text=True)
    return exe


@pytest.mark.parametrize("check", [
    "contexts after failed allocations",
    "levels after failed allocations",
    "flowing pools",
    "narrow pools",
    "patience of waiting",
    "pools that give up",
    "refused scratch",
    "early ends",
    "pools in parts",
    "walks after failed allocations",
    "packed walks leave room",
    "reports of evaluation",
    "plans of pools",
    "counted launches",
    "ranking where it can be done",
])
def test_host_runtime(driver, check):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1:alloc_dealloc_mismatch=0",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    done = subprocess.run([driver, check], capture_output=True, text=True, env=env, timeout=300)
    assert done.returncode == 0, done.stdout + done.stderr
    assert "all checks passed" in done.stdout
    assert "runtime error" not in done.stderr and "Sanitizer" not in done.stderr, done.stderr
