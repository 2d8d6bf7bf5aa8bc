"""The copy kernel's source on the CPU under AddressSanitizer and ThreadSanitizer: arrays ending
in every remainder of an 8-byte word, tails alone, six arrays at once, and more words than the
largest grid takes in one step of its threads."""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SMALL = [[2], [8], [4, 6], [2 * n for n in (1, 2, 3, 4, 5, 1021)], [8 * 1024, 8 * 1024 + 2], [2, 30000, 6, 4, 8, 2048]]
# 256 workgroups of 256 threads with 4 words each move 2 MB in a step: three arrays over that
LARGE = [[1 << 20, (1 << 20) + 6, 3000]]


@pytest.fixture(scope="module", params=["address", "thread"])
def run(request, tmp_path_factory):
    exe = tmp_path_factory.mktemp("copy") / "run_copy"
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-g", "-x", "c++", f"-fsanitize={request.param}",
                           "-fno-omit-frame-pointer", "-pthread", "-I" + os.path.join(HERE, "emu"),
                           "-I" + os.path.join(ROOT, "paper_2004_04334_amd", "csrc"),
                           os.path.join(HERE, "emu", "run_copy.cpp"), "-o", str(exe)])

    def go(to_host, sizes):
        r = subprocess.run([str(exe), str(int(to_host)), *map(str, sizes)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
    go.sanitizer = request.param
    return go


@pytest.mark.parametrize("to_host", [False, True])
def test_copy_kernel(run, to_host):
    for sizes in SMALL + (LARGE if run.sanitizer == "address" and to_host else []):
        run(to_host, sizes)
