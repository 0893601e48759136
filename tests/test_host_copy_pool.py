"""The proxy threads' copies through the shared batches, with a CPU thread in the place of the device, under
ThreadSanitizer and AddressSanitizer: every row arrives, no event is reused while its batch is under way."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_19849_amd", "csrc")


@pytest.mark.parametrize("sanitizer", ["thread", "address,undefined"])
def test_copies_through_shared_batches(tmp_path, sanitizer):
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("g++ or the HIP headers are not available")
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", f"-fsanitize={sanitizer}", "-fno-omit-frame-pointer",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(CSRC, "proxy.cpp"),
                    os.path.join(CSRC, "api.cpp"), os.path.join(ROOT, "tests", "native", "copy_pool_driver.cpp"), "-o", exe,
                    "-L/opt/rocm/lib", "-lamdhip64", "-lpthread", "-lrt", "-Wl,-rpath,/opt/rocm/lib"],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0 protect_shadow_gap=0"))
    assert r.returncode == 0 and r.stdout == "bad 0\n", r.stdout + r.stderr[-3000:]
    assert "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, r.stderr[-3000:]
