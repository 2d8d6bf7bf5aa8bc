"""Which host arrays the copy kernel may move, asked of the library's own rule with made-up
answers of the runtime: it reads every byte between an array's ends, so all of them must lie
in one allocation that the device can address, and its accesses are coherent with the host's
only in coherent memory."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = """
#include <cstddef>
#include <cstdio>
#include "pxcl_internal.h"
int main() {
    unsigned long long host, bytes, pinned, dev, base, size;   // pinned: 1, and non-coherent: 2
    while (scanf("%llu %llu %llu %llu %llu %llu", &host, &bytes, &pinned, &dev, &base, &size) == 6)
        printf("%d\\n", pxcl::copy_kernel_takes(host, bytes, pxcl::HostMemory{pinned != 0, pinned != 2, dev, base, size}) ? 1 : 0);
}
"""
P = 1 << 20                       # a block of 4,096 bytes at P, the device's view of it at P + D
D = 1 << 32
CASES = [
    ("the whole block", (P, 4096, 1, P + D, P + D, 4096), 1),
    ("its inside", (P + 8, 4080, 1, P + D + 8, P + D, 4096), 1),
    ("its last word and a tail", (P + 4080, 14, 1, P + D + 4080, P + D, 4096), 1),
    ("one byte past its end", (P, 4097, 1, P + D, P + D, 4096), 0),
    # ends in another pinned block: first and last byte have a device address, the gap has none
    ("a hole before its last byte", (P, 3 * 4096, 1, P + D, P + D, 4096), 0),
    ("before the block", (P - 8, 16, 1, P + D - 8, P + D, 4096), 0),
    ("at the block's end", (P + 4096, 8, 1, P + D + 4096, P + D, 4096), 0),
    ("off 8-byte alignment", (P + 2, 64, 1, P + D + 2, P + D, 4096), 0),
    ("the device's view off alignment", (P, 64, 1, P + D + 4, P + D, 4096), 0),
    ("non-coherent", (P, 4096, 2, P + D, P + D, 4096), 0),
    ("pageable", (P, 64, 0, 0, 0, 0), 0),
    ("pageable inside what an earlier answer held", (P, 64, 0, P + D, P + D, 4096), 0),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "t.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-Wno-unused-function",
                           "-I" + os.path.join(ROOT, "paper_2004_04334_amd", "csrc"), str(d / "t.cpp"), "-o", str(d / "t")])

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        return [int(x) for x in subprocess.run([str(d / "t")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return ask


def test_copy_kernel_takes_whole_allocations_only(rule):
    got = rule([c[1] for c in CASES])
    assert len(got) == len(CASES)
    assert [(c[0], g) for c, g in zip(CASES, got)] == [(c[0], c[2]) for c in CASES]
