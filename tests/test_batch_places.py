"""The records of a routed batch are checked before an index in them is used (csrc/batch_places.h), on the CPU with the
sanitizers: a damaged record is reported and touches nothing."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path_factory.mktemp("places") / "places"
    subprocess.run([gxx, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-static-libubsan", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2412_00099_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "batch_places_driver.cpp"), "-o", str(exe)], check=True,
                   capture_output=True, text=True)
    return exe


@pytest.mark.parametrize("expert,slot,expect", [(4, 4, (-1, 1, 14)), (4, 6, (3, 1, 9)), (4, -1, (3, 1, 9)), (9, 0, (3, 1, 9)),
                                                (-1, 0, (3, 1, 9)), (0, 1 << 28, (3, 1, 9)), (0, -(1 << 31), (3, 1, 9))])
def test_a_damaged_record_is_reported(driver, expert, slot, expect):
    run = subprocess.run([str(driver), str(expert), str(slot)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stderr[-2000:]
    assert tuple(map(int, run.stdout.split())) == expect
