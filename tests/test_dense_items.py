"""The cut of an expert's routed rows into items of the dense launches, compiled
for the host: the items cover the rows in order, hold at most R of them, and differ
by at most one 32-row group, so that their tiles take nearly equal time and cost
what the split of the tiles over the XCDs counts them as."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the HIP headers")
def test_dense_items(tmp_path):
    exe = str(tmp_path / "dense_items")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2609_33385_amd", "csrc"),
                    os.path.join(HERE, "native", "dense_items.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("ALL OK"), r.stdout[-500:]
