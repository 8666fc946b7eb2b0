"""How a persistent plane kernel's items are shared among workgroups and XCDs
(paper_1905_01348_amd/csrc/item_map.hpp), on the CPU, built with g++ and the address and
undefined-behaviour sanitizers: each item is visited once, in range, and the XCDs' shares are even
to 5% wherever each has one of its own."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")
def test_item_map(tmp_path):
    exe = str(tmp_path / "item_map_check")
    build = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
             "-fno-sanitize-recover=undefined",
             "-I" + os.path.join(ROOT, "paper_1905_01348_amd", "csrc"),
             os.path.join(ROOT, "tests", "item_map_check.cpp"), "-o", exe]
    r = subprocess.run(build, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    out = r.stdout + r.stderr
    assert r.returncode == 0, out[-4000:]
    assert out.strip().splitlines()[-1] == "ok", out[-2000:]
