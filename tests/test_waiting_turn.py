"""At most one context at a time has launches on a device whose workgroups wait for their first one (csrc/waiting_turn.h):
the rule by itself, in one thread and in four, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_one_context_at_a_time(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "turn"
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", "-I", os.path.join(ROOT, "paper_2412_00099_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "waiting_turn_driver.cpp"), "-o", str(exe)], check=True,
                   capture_output=True, text=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stderr[-2000:]
    bad, waited, without, most = map(int, run.stdout.split())
    assert bad == 0 and waited + without == 80000 and waited > 0 and most == 1
