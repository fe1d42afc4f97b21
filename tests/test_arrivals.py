"""CPU checks of how the workgroups of a sequence find out which of them ends last (csrc/space_arrivals.h)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "space_arrivals.h"
using namespace space;

static std::mt19937 rng(3);
static uint32_t count = 0;
struct Call {
    int n;
    std::vector<int> order;  // its workgroups as they end
    int at = 0, lasts = 0, last_at = -1;
};
static Call make(int n) {
    Call c{n, std::vector<int>(n)};
    for (int i = 0; i < n; ++i) c.order[i] = i;
    std::shuffle(c.order.begin(), c.order.end(), rng);
    return c;
}
static void arrive(Call& c) {
    const uint32_t share = arrival_share(c.n, c.order[c.at]), before = count;
    count += share;
    if (arrival_is_last(before, share)) { ++c.lasts; c.last_at = c.at; }
    ++c.at;
}

int main() {
    long wrong = 0;
    for (int n = 1; n <= 1024; ++n)
        for (int rep = 0; rep < 3; ++rep) {  // a call by itself: the one that ends last, and no other, is told so
            Call c = make(n);
            while (c.at < n) arrive(c);
            if ((c.lasts != 1 || c.last_at != n - 1) && wrong++ < 5) printf("%d workgroups, %d lasts at %d\n", n, c.lasts, c.last_at);
        }
    for (int rep = 0; rep < 4000; ++rep) {  // calls that meet on the count (not allowed), then calls by themselves again
        std::vector<Call> met;
        for (int k = 2 + rng() % 3; k > 0; --k) met.push_back(make(1 + rng() % 96));
        for (;;) {
            std::vector<Call*> open;
            for (Call& c : met)
                if (c.at < c.n) open.push_back(&c);
            if (open.empty()) break;
            arrive(*open[rng() % open.size()]);
        }
        for (int k = 0; k < 3; ++k) {
            Call c = make(1 + rng() % 96);
            while (c.at < c.n) arrive(c);
            if ((c.lasts != 1 || c.last_at != c.n - 1) && wrong++ < 5) printf("after an overlap: %d workgroups, %d lasts at %d\n", c.n, c.lasts, c.last_at);
        }
    }
    printf("%ld wrong\n", wrong);
    return wrong != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_the_last_of_a_call_is_found_whatever_came_before(tmp_path):
    """Calls of 1 to 1024 workgroups that end in any order, and calls behind others that met on the same count: exactly the workgroup that
    ends last is told so.  Nothing tells one call from another, so a replay of a captured call is a call like any other."""
    src = tmp_path / "arrivals.cpp"
    src.write_text(_PROGRAM)
    exe = tmp_path / "arrivals"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2402_11809_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
