"""CPU checks of how the workgroups of a batch's attention are paired on the CUs and how its keys are cut by length
(csrc/space_attn_plan.h)."""
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

_TABLE_PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "space_attn_plan.h"
using namespace space;

static long tables = 0, cuts = 0, full = 0, wrong = 0;

static void check(const std::vector<int>& lens, int block_chunks, int slots, int streams) {
    const int batch = (int)lens.size();
    std::vector<KeySeq> seq;
    int longest = 0, total = 0;
    for (int len : lens) {
        seq.push_back(key_seq((len + 31) / 32, block_chunks));
        longest = std::max(longest, seq.back().chunks);
        total += seq.back().chunks;
    }
    const KeyCut cut = key_cut(batch, slots, streams, longest, total, [&](int size) {
        int parts = 0;
        for (const KeySeq& s : seq) parts += key_parts(s, size, longest);
        return parts;
    });
    std::vector<int> n, part;
    for (const KeySeq& s : seq) {
        n.push_back(key_parts(s, cut.size, longest));
        part.push_back(key_part_chunks(s, n.back()));
    }
    std::vector<KeyPart> table(slots, KeyPart{-2, 0, 0, 0});
    bool ok = cut.parts <= slots && slots <= kMaxKeySlots;
    int parts = 0, largest = 0;
    for (int b = 0; b < batch; ++b) {
        const int first = key_first_place(b, part[b], batch, [&](int i) { return part[i]; }, [&](int i) { return n[i]; });
        ok = ok && n[b] >= 1 && n[b] <= kMaxKeyParts && first >= 0 && first + n[b] <= cut.parts;
        ok = ok && (n[b] == 1 || ((lens[b] + 31) / 32 >= 4 * n[b] && part[b] >= 4));  // every wave has a cached chunk
        for (int j = 0; ok && j < n[b]; ++j) {
            ok = table[first + j].b == -2;  // nobody else's place
            table[first + j] = KeyPart{b, j, n[b], lens[b]};
        }
        parts += n[b];
        largest = std::max(largest, part[b]);
    }
    ok = ok && parts == cut.parts;
    for (int r = 0; ok && r < slots; ++r) ok = (table[r].b >= 0) == (r < parts);  // the rest is marked as left over
    for (int r = 1; ok && r < parts; ++r) ok = part[table[r].b] <= part[table[r - 1].b];  // largest first
    const bool cutting = parts > batch;
    ok = ok && (!cutting || (slots > batch && largest < longest));
    ++tables;
    cuts += cutting;
    full += parts == slots;
    if (!ok && wrong++ < 5) printf("batch %d, block %d, slots %d, streams %d: wrong table\n", batch, block_chunks, slots, streams);
}

int main() {
    std::mt19937 rng(1);
    auto upto = [&](int n) { return (int)(rng() % (unsigned)n); };
    for (int streams = 1; streams <= 512; streams += streams < 72 ? 1 : 8)
        for (int batch = 2; batch <= 64; ++batch)
            for (int kind = 0; kind < 6; ++kind) {
                std::vector<int> lens(batch);
                const int most = 1 << (6 + upto(11));
                for (int b = 0; b < batch; ++b)
                    lens[b] = kind == 0 ? most : kind == 1 ? upto(most) : kind == 2 ? (b == batch / 2 ? most : upto(40))
                              : kind == 3 ? 0 : kind == 4 ? most * b / batch : (b & 1 ? most : most / 3);
                const int slots[] = {batch, batch + 1, 256 / streams, 512 / streams, batch + upto(512)};
                for (int s : slots)
                    if (s >= batch && s <= kMaxKeySlots) check(lens, 1 + upto(32), s, streams);
            }
    printf("%ld tables, %ld with cuts, %ld without a slot to spare, %ld wrong\n", tables, cuts, full, wrong);
    return wrong || tables < 10000 || cuts < 1000 || full < 1000;
}
"""


_ROUNDS_PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "space_attn_plan.h"
using namespace space;

int main() {
    int wrong = 0;
    for (int chunks = 0; chunks <= 4100; ++chunks)
        for (int n = 1; n <= key_seq(chunks, 2).most; ++n) {
            const int rounds = (chunks + 3) / 4, even = (rounds + kBlockRounds + n - 1) / n;
            int at = 0, busiest = 0;
            bool ok = key_part_first(rounds, n, 0) == 0 && key_part_first(rounds, n, n) == rounds;
            for (int p = 0; p < n; ++p) {
                const int own = key_part_first(rounds, n, p + 1) - at;
                ok = ok && own >= (p < n - 1) && (p == 0 || p == n - 1 || own <= at - key_part_first(rounds, n, p - 1));
                busiest = std::max(busiest, p < n - 1 ? own : own + kBlockRounds);
                at += own;
            }
            // (a part of no cached rounds still has the block)
            ok = ok && at == rounds && busiest <= std::max(even, kBlockRounds) && busiest <= (rounds + n - 1) / n + kBlockRounds;
            if (!ok && wrong++ < 5) printf("%d chunks in %d parts: busiest %d\n", chunks, n, busiest);
        }
    return wrong;
}
"""


_PRICE_PROGRAM = r"""
#include <cstdio>
#include "space_attn_plan.h"
using namespace space;

static int parts(int staging, int streams, int slots, int a, int b) {
    const KeySeq s[2] = {key_seq(a, 8), key_seq(b, 8)};
    const int longest = b + 8;
    return key_cut(2, slots, streams, longest, a + b + 16, [&](int size) { return key_parts(s[0], size, longest) + key_parts(s[1], size, longest); }, staging).parts;
}
int main() {
    // 256 rows of 32 heads: four query groups, two workgroups per CU in all; behind 2000 and 4000 positions
    const int rows = parts(kRowsStaging, 128, 4, 63, 125), few = parts(kPartStaging, 128, 4, 63, 125), none = parts(kRowsStaging, 128, 2, 63, 125), equal = parts(kRowsStaging, 128, 3, 125, 125);
    printf("%d %d %d %d\n", rows, few, none, equal);
    return !(rows == 3 && few == 2 && none == 2 && equal == 2);
}
"""


def _run(tmp_path, program):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "attn_plan.cpp"
    src.write_text(program)
    exe = tmp_path / "attn_plan"
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2402_11809_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout


def test_every_place_takes_one_item(tmp_path):
    """Head counts and batches of every size: no item of the table is left out, taken twice or outside it."""
    _run(tmp_path, _PROGRAM)


def test_every_part_has_one_place_in_the_table(tmp_path):
    """Batches of 2 to 64 sequences (equal, ragged, one long, empty, ascending, two lengths), blocks of 1 to 32 chunks and every
    number of slots: the parts fit the slots, every part of every sequence has one place, those of a sequence lie side by side, larger
    ones in front; a sequence is cut into at most 16 parts of at least four cached chunks; left-over slots are at the end."""
    _run(tmp_path, _TABLE_PROGRAM)


def test_rounds_of_a_part(tmp_path):
    """Every number of cached chunks and of parts that a sequence may have: the parts lie end to end and hold every round once, no part
    before the last is empty, and the busiest, the last one's block included, has no more than rounds and block dealt out evenly, nor more
    than it had with equal parts."""
    _run(tmp_path, _ROUNDS_PROGRAM)


def test_a_batch_of_prompt_chunks_is_cut_at_its_own_price(tmp_path):
    """Two sequences whose query groups give every CU one workgroup: the longer one is cut where a part costs next to nothing
    beside its chunks, not where it stages the block; never without a slot to spare, nor equal ones that cannot both be cut."""
    _run(tmp_path, _PRICE_PROGRAM)
