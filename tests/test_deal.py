"""How a workgroup's list of records (shared ones, then routed ones) is dealt out to its eight wavefronts, on the CPU: the order
in which a wavefront adds its records up is part of what y's bits depend on."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NW = 8


def test_lists_are_dealt_in_list_order(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "deal"
    subprocess.run([gxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-static-libubsan", "-I",
                    os.path.join(ROOT, "paper_2412_00099_amd", "csrc"), os.path.join(ROOT, "tests", "host", "deal_driver.cpp"),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    lists = [(ns, nr) for ns in (0, 1, 2, 7, 8, 9, 11, 22, 64) for nr in (0, 1, 5, 8, 13, 33, 34, 100)] + [(1 << 22, 0), (5, 1 << 22)]
    run = subprocess.run([str(exe)], input="\n".join(f"{a} {b}" for a, b in lists), capture_output=True, text=True, check=True)
    for (ns, nr), line in zip(lists, run.stdout.splitlines()):
        v = list(map(int, line.split()))
        for i, step in enumerate((NW, 1)):
            for w in range(NW):
                first_sh, n_sh, first_rt, n_rt = v[4 * (i * NW + w):4 * (i * NW + w) + 4]
                if ns + nr > 1000:  # (long lists: the ends only)
                    assert n_sh + n_rt in ((ns + nr) // NW, (ns + nr + NW - 1) // NW)
                    continue
                got = [first_sh + k * step for k in range(n_sh)] + [ns + first_rt + k * step for k in range(n_rt)]
                if step == 1:  # one contiguous block of the whole list
                    want = list(range(w * (ns + nr) // NW, (w + 1) * (ns + nr) // NW))
                else:  # every NW-th entry
                    want = list(range(w, ns + nr, NW))
                assert got == want and all(e < ns for e in got[:n_sh]) and all(e >= ns for e in got[n_sh:]), (ns, nr, step, w)
