"""CPU check of how the workgroups of a batch's attention are paired on the CUs (csrc/space_attn_plan.h)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "space_attn_plan.h"
using namespace space;

int main() {
    int wrong = 0, kinds[3] = {0, 0, 0};
    for (int heads = 1; heads <= 512; ++heads)
        for (int places = 1; places <= 2100; ++places) {
            const int shared = attention_shared(places, heads);
            ++kinds[shared < 0 ? 0 : shared == 0 ? 1 : 2];
            std::vector<char> seen(places, 0);
            bool ok = true;
            for (int p = 0; p < places; ++p) {
                const int item = attention_item(p, places, shared);
                ok = ok && item >= 0 && item < places && !seen[item];
                if (ok) seen[item] = 1;
            }
            if (!ok && wrong++ < 5) printf("%d heads, %d places: shared %d\n", heads, places, shared);
        }
    printf("%d wrong\n", wrong);
    return wrong || !kinds[0] || !kinds[1] || !kinds[2];
}
"""


def test_every_place_takes_one_item(tmp_path):
    """Head counts and batches of every size: no item of the table is left out, taken twice or outside it."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "attn_plan.cpp"
    src.write_text(_PROGRAM)
    exe = tmp_path / "attn_plan"
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2402_11809_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
