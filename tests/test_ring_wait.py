"""How long a Push waits for room, and what it counts: the kernel's loop compiled for the CPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_each_command_of_a_pair_waits_for_itself(tmp_path):
    """The time limit bounds every wait: the second command's wait starts when the first has left, and each counts."""
    if not shutil.which("g++"):
        pytest.skip("g++ is not available")
    with open(os.path.join(ROOT, "paper_2512_19849_amd", "csrc", "ep_device.h")) as f:
        loop = re.search(r"^template <int N>\nEP_DEV unsigned long long ring_publish_run\(.*?^}\n", f.read(), re.M | re.S)
    (tmp_path / "run.inc").write_text(loop.group(0))
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-w", f'-DRING_PUBLISH_RUN="{tmp_path}/run.inc"', "-o", exe,
                    os.path.join(ROOT, "tests", "native", "ring_wait_driver.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout.split("\n")
    assert out[:4] == ["2 error 0 stored 2 stalls 1",      # (room for both at once: one wait)
                       "2 error 0 stored 2 stalls 2",      # 60 and then 60 more, the limit is 100
                       "-1 error -5 stored 1 stalls 2",
                       "-1 error -5 stored 0 stalls 1"]
