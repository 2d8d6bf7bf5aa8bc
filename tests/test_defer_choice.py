"""When a server's batches defer the big-module kernel, asked of the library's own rule: batches
that need their second launch nearly always must nearly always launch every kernel at once, and
batches that never need it must all be deferred."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = """
#include <cstdio>
#include <deque>
#include "pxcl_internal.h"
// batches with `inflight` on the device at once; every `period`-th of the stretch up to `turn`
// needs no second launch (0: none), after it every one needs none
int main() {
    int n, inflight, period, turn;
    while (scanf("%d %d %d %d", &n, &inflight, &period, &turn) == 4) {
        pxcl::DeferChoice c;
        std::deque<int> flying;            // of each batch: -1 not deferred, else whether it needs the second launch
        int deferred = 0, second = 0, after = 0;
        for (int i = 0; i < n; ++i) {
            if (int(flying.size()) == inflight) {
                if (flying.front() >= 0) c.done(flying.front() != 0);
                flying.pop_front();
            }
            const bool needs = i < turn && !(period && i % period == 0), d = c.next();
            deferred += d;
            second += d && needs;
            after += d && i >= turn;
            flying.push_back(d ? int(needs) : -1);
        }
        printf("%d %d %d\\n", deferred, second, after);
    }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("defer")
    (d / "t.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-Wno-unused-function",
                           "-I" + os.path.join(ROOT, "paper_2004_04334_amd", "csrc"), str(d / "t.cpp"), "-o", str(d / "t")])

    def ask(*row):
        r = subprocess.run([str(d / "t")], input=" ".join(map(str, row)), capture_output=True, text=True, check=True)
        return tuple(int(x) for x in r.stdout.split())
    return ask


@pytest.mark.parametrize("inflight", [1, 6])
def test_batches_defer_only_while_that_saves_the_second_kernel(rule, inflight):
    n = 4000
    deferred, second, _ = rule(n, inflight, 0, n)          # every batch needs it: the first ones, then 1 in 256
    assert second == deferred <= 3 + inflight + n // 256
    deferred, second, _ = rule(n, inflight, 0, 0)          # none does
    assert (deferred, second) == (n, 0)
    deferred, second, _ = rule(n, inflight, 2, n)          # every other one: never three in a row
    assert (deferred, second) == (n, n // 2)
    # the load changes at half time: at most one retry period and what is in flight later, all defer
    deferred, second, after = rule(n, inflight, 0, n // 2)
    assert after >= n // 2 - 256 - inflight
