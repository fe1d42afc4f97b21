// How the many-row projection kernel cuts its work, decided on the host (no HIP in here: compiles with any
// C++17 compiler).
#pragma once
#include <stdint.h>

namespace space {

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int round_up(int a, int b) { return ceil_div(a, b) * b; }

constexpr int kWideDepth = 2;          // weight tiles in flight per wave and tile row: partial sums are whole rounds of them
constexpr int kWideSearchGroups = 32;  // longest blocks (in groups of 32 rows) whose cuts are compared

// How the rows of every weight group are cut: count[c] pieces of 4 - c groups of two row tiles (8, 6, 4,
// 2 row tiles), laid end to end in this order; the groups add up to ceil(ceil(m / 16) / 2).
struct WideParts {
    int count[4];
    int by_size;  // launch order: 0 = weight group by weight group, 1 = all pieces of a size before any smaller one
};

// What a launch costs: the work of its busiest CU, in units of 17.4 us / 1280.  A CU gets through one piece after
// the other, or two at half speed each; workgroup i runs on XCD i % 8, the first two rounds on its 32 CUs
// in turn, later ones where a place is free.  A piece of g groups over kt contraction tiles takes 17.4 us *
// (kt / 128 * (0.6 + g) + 0.4), one of a single group 0.2 * kt / 128 more: fitted on 790 x 4 launches (224 .. 1024
// rows at 7B and 13B width, all projections, up to 26 cuts, both orders, 1, 2 and 4 partial sums; off by
// 7.9 % rms).  gk8: weight groups x partial sums per XCD.
constexpr double kWideUnitUs = 17.4 / 1280;
inline int64_t wide_piece_cost(int g, int kt) { return (int64_t)kt * (10 * g + (g == 1 ? 8 : 6)) + 512; }

// The cost, or any value >= bar once it is known not to lie below bar.  This runs in front of the first launch at
// a row count, with the GPU idle, so the workgroups are not placed one by one: the CUs are kept as levels of equal
// load, lowest first, and a run of equal pieces fills a level at a time.
inline int64_t wide_cost(const WideParts& parts, int gk8, int kt, int64_t bar = INT64_MAX) {
    constexpr int kCus = 32;
    int64_t piece[4], total = 0;
    for (int c = 0, pieces = 0; c < 4; ++c) {
        piece[c] = wide_piece_cost(4 - c, kt);
        total += piece[c] * parts.count[c] * gk8;
        pieces += parts.count[c] * gk8;
        if (ceil_div(pieces, kCus) * piece[c] >= bar) return bar;  // some CU has that many of at least this size
    }
    if (total / kCus >= bar) return bar;
    const int n_runs = parts.by_size ? 4 : 4 * gk8, per_run = parts.by_size ? gk8 : 1;
    int run = 0, left = parts.count[0] * per_run;
    auto skip_empty = [&]() {  // to the next run with pieces left; false: none
        while (left == 0) {
            if (++run >= n_runs) return false;
            left = parts.count[run & 3] * per_run;
        }
        return true;
    };
    // the first two rounds
    int64_t first[kCus] = {0};
    for (int i = 0; i < 2 * kCus && skip_empty(); ++i, --left) first[i % kCus] += piece[run & 3];
    struct Level {
        int64_t load;
        int cus;
    } level[kCus + 1];
    int n = 0;  // levels, level[n - 1] the lowest
    auto insert = [&](int64_t load, int cus) {
        int at = n;
        while (at > 0 && level[at - 1].load < load) --at;
        if (at > 0 && level[at - 1].load == load) {
            level[at - 1].cus += cus;
            return;
        }
        for (int j = n; j > at; --j) level[j] = level[j - 1];
        level[at] = Level{load, cus};
        ++n;
    };
    for (int i = kCus - 1; i >= 0; --i) insert(first[i], 1);  // loads mostly fall with i
    // the rest, where a place is free
    while (level[0].load < bar && skip_empty()) {
        Level& low = level[n - 1];
        const int take = left < low.cus ? left : low.cus;
        const int64_t load = low.load + piece[run & 3];
        left -= take;
        low.cus -= take;
        if (low.cus == 0) --n;
        insert(load, take);
    }
    return level[0].load;
}

struct WideCut {
    WideParts parts;
    int ksplit;  // partial sums over the contraction
};

// By how much another cut has to be ahead of pieces of 128 rows and one for the rest, in percent of their cost.
// Measured at 7B, 13B and 70B width (97 .. 1024 rows, all projections): 115 picks more than 9 % ahead are 10 %
// faster on average and at most 1.3 % slower; 19 picks 5 .. 9 % ahead where the matrix has up to 512 MB are 1.7 %
// faster on average (7B LM head at 648 rows 273 -> 258 us) and at most 5 % slower; 6 of them at 940 MB (70B gate /
// up) are 2.4 % slower on average (480 rows 1381 -> 1538 us, whole 70B layers 3.5 .. 5.8 % slower): every size in a
// launch streams the matrix again, there from memory and not from a cache, which the model knows nothing of.
inline int wide_cut_bar(int n, int k_tiles) { return (int64_t)n * k_tiles * 64 > ((int64_t)512 << 20) ? 91 : 95; }

// Cut of the rows and number of partial sums with the lowest cost, a partial sum beyond the first charged
// with the time to read it.  Pieces of 128 rows and one for the rest, large ones first, unless another cut is
// ahead (wide_cut_bar).  Why it matters: gate / up at 333 rows and 7B width makes 258 workgroups of 128 and 96 rows,
// i.e. two CUs with two of them, 140 us; the cut picked here 120.  O and down at 224 rows 28 -> 21 and 63 -> 45 us.
// Beyond 1024 rows there are many rounds and the cut matters little.
//   n_groups, n, k_tiles  the matrix: weight groups (workgroups along its rows), rows, contraction tiles
//   m                     rows of the launch
//   smax                  most partial sums (1 .. 4); force_ksplit > 0: that many
//   cut                   that cut; the partial sums are still those of the plan without it, so that a cut
//                         alone changes no sum's order
inline WideCut plan_wide_cut(int n_groups, int n, int k_tiles, int m, int smax, int force_ksplit, const WideParts* cut) {
    const int groups = ceil_div(ceil_div(m, 16), 2);
    WideParts plain{};
    plain.count[0] = groups / 4;
    if (groups % 4) plain.count[4 - groups % 4] = 1;
    plain.by_size = 1;
    WideCut p{plain, 1};
    int64_t best = INT64_MAX;
    for (int ks = 1; ks <= smax && !(cut && force_ksplit > 0); ks *= 2) {
        if (force_ksplit > 0 && ks != (force_ksplit < smax ? force_ksplit : smax)) continue;
        if (force_ksplit <= 0 && ks > 1 && k_tiles / ks < 16) break;
        const int gk8 = ceil_div(n_groups * ks, 8), kt = round_up(ceil_div(k_tiles, ks), kWideDepth);
        WideParts parts = plain;
        int64_t cost = wide_cost(parts, gk8, kt);
        int64_t bar = cost * wide_cut_bar(n, k_tiles) / 100;
        for (int a = groups <= kWideSearchGroups ? groups / 4 : -1; a >= 0; --a)
            for (int b = (groups - 4 * a) / 3; b >= 0; --b) {
                const int rest = groups - 4 * a - 3 * b;
                for (int order = 0; order < 2; ++order) {
                    const WideParts c{{a, b, rest / 2, rest % 2}, order};
                    const int64_t t = wide_cost(c, gk8, kt, bar);
                    if (t < bar) {
                        bar = cost = t;
                        parts = c;
                    }
                }
            }
        cost += (int64_t)((ks - 1) * (double)m * n * 4.0 / (4.5e6 * kWideUnitUs));
        if (cost < best) {
            best = cost;
            p = WideCut{parts, ks};
        }
    }
    if (force_ksplit > 0) p.ksplit = force_ksplit < smax ? force_ksplit : smax;
    if (cut) p.parts = *cut;
    return p;
}

}  // namespace space
