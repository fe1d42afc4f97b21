// How the many-row projection kernel cuts its work, decided on the host (no HIP in here: compiles with any
// C++17 compiler).
#pragma once
#include <stdint.h>

namespace space {

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int round_up(int a, int b) { return ceil_div(a, b) * b; }

constexpr int kWideDepth = 2;          // weight tiles in flight per wave and tile row: partial sums are whole rounds of them
constexpr int kWideSearchGroups = 32;  // longest blocks (in groups of 32 rows) whose cuts are compared

// Whether the many-row kernel takes a projection over m rows, or the weight-streaming kernel in passes of 96 rows.  The
// passes cost next to nothing while all their workgroups run at once, one per CU, and a round each beyond; the many-row
// kernel has a fixed cost of 3 - 5 us more and fewer, larger workgroups, but uses the matrix unit better and shares the operand
// planes.  So: from the second round of workgroups on, or from the third where a round is short and the sums have to be
// complete (the many-row kernel then cannot be cut over the contraction and has few workgroups: gate / up of a 1024-wide model
// at 128 rows, 352 workgroups of 8 rounds, 12.1 us in passes against 15.1).  Short: a wave requests at most 128 tiles of 1 KB in its lq
// contraction tiles, r_pack of weights and 12 of operands (6 row tiles, two planes) each; the line
// lies between that gate / up, 112 tiles, and the LM head of 32000 of the same model, 160.  Measured on 9 shapes from 256 to 8192 wide, all
// projections, 12 row counts from 100 to 1000, passes / many-row kernel in us: 128 rows, 256 wide down 6.8 / 12.0; 1024 wide QKV 8.0 /
// 10.4; 2048 wide QKV 23.0 / 13.7; 7B gate / up 79.8 / 60.4, LM head 110 / 72; 70B down 176 / 125; 288 rows, 256 wide QKV 5.1 / 7.7;
// 1024 wide LM head of 32000 69.5 / 44.9; 800 rows, 512 wide gate / up 14.6 / 10.4.  Over all of them, on which the rule was made, it is 0.3 % behind
// the better of the two, fixed lines at 97 and 193 rows 13 and 12 %.
//   groups, splits, lq, r_pack  how the matrix is packed (PackedW);  plain: the sums may be partial ones
constexpr int kPassRows = 96;
inline bool wide_is_faster(int groups, int splits, int lq, int r_pack, int m, bool plain) {
    if (m <= kPassRows) return false;
    const long long wgs = (long long)groups * splits * ceil_div(m, kPassRows);
    return wgs > 512 || (wgs > 256 && (plain || lq * (r_pack + 12) > 128));
}

// How the rows of every weight group are cut: count[c] pieces of 4 - c groups of two row tiles (8, 6, 4,
// 2 row tiles), laid end to end in this order; the groups add up to ceil(ceil(m / 16) / 2).
struct WideParts {
    int count[4];
    int by_size;  // launch order: 0 = weight group by weight group, 1 = all pieces of a size before any smaller one, 2 = before any larger one (with a tail)
};

// What a launch costs: the work of its busiest CU, in units of 17.4 us / 1280.  A CU gets through one piece after
// the other, or two at half speed each; workgroup i runs on XCD i % 8, the first two rounds on its 32 CUs
// in turn, later ones where a place is free.  A piece of g groups over kt contraction tiles takes 17.4 us *
// (kt / 128 * (0.6 + g) + 0.4), one of a single group 0.2 * kt / 128 more: fitted on 790 x 4 launches (224 .. 1024
// rows at 7B and 13B width, all projections, up to 26 cuts, both orders, 1, 2 and 4 partial sums; off by
// 7.9 % rms).  gk8: weight groups x partial sums per XCD.
constexpr double kWideUnitUs = 17.4 / 1280;
inline int64_t wide_piece_cost(int g, int kt) { return (int64_t)kt * (10 * g + (g == 1 ? 8 : 6)) + 512; }

// The load of the busiest CU once `runs` runs of equal pieces (cost_of(run) each, count_of(run) of them) are placed, or
// any value >= bar once it is known not to lie below bar.  This runs in front of the first launch at
// a row count, with the GPU idle, so the workgroups are not placed one by one: the CUs are kept as levels of equal
// load, lowest first, and a run of equal pieces fills a level at a time.
constexpr int kWideCus = 32;  // per XCD
template <class Cost, class Count>
inline int64_t wide_place(int runs, Cost cost_of, Count count_of, int64_t bar) {
    int run = 0, left = count_of(0);
    auto skip_empty = [&]() {  // to the next run with pieces left; false: none
        while (left == 0) {
            if (++run >= runs) return false;
            left = count_of(run);
        }
        return true;
    };
    // the first two rounds
    int64_t first[kWideCus] = {0};
    for (int i = 0; i < 2 * kWideCus && skip_empty(); ++i, --left) first[i % kWideCus] += cost_of(run);
    struct Level {
        int64_t load;
        int cus;
    } level[kWideCus + 1];
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
    for (int i = kWideCus - 1; i >= 0; --i) insert(first[i], 1);  // loads mostly fall with i
    // the rest, where a place is free
    while (level[0].load < bar && skip_empty()) {
        Level& low = level[n - 1];
        const int take = left < low.cus ? left : low.cus;
        const int64_t load = low.load + cost_of(run);
        left -= take;
        low.cus -= take;
        if (low.cus == 0) --n;
        insert(load, take);
    }
    return level[0].load;
}

// The cost, or any value >= bar once it is known not to lie below bar.
inline int64_t wide_cost(const WideParts& parts, int gk8, int kt, int64_t bar = INT64_MAX) {
    int64_t piece[4], total = 0;
    for (int c = 0, pieces = 0; c < 4; ++c) {
        piece[c] = wide_piece_cost(4 - c, kt);
        total += piece[c] * parts.count[c] * gk8;
        pieces += parts.count[c] * gk8;
        if (ceil_div(pieces, kWideCus) * piece[c] >= bar) return bar;  // some CU has that many of at least this size
    }
    if (total / kWideCus >= bar) return bar;
    const int per_run = parts.by_size ? gk8 : 1;
    return wide_place(parts.by_size ? 4 : 4 * gk8, [&](int run) { return piece[run & 3]; },
                      [&](int run) { return parts.count[run & 3] * per_run; }, bar);
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

// The last `pieces` pieces of every XCD, in launch order, are cut over the contraction: `parts` workgroups each, whose sums
// the one that ends last adds up in part order (same bits whichever that is) before the epilogue.  0: none.
constexpr int kWideTailMinK = 64;    // contraction tiles (shorter: a workgroup's fixed cost outweighs it)
constexpr int kWideTailSlots = 32;  // most workgroups per XCD with a part of a piece (partial sums of 128 KB each)
struct WideTail {
    int pieces, parts;
};

// A part costs its share of the piece and 3 us to write the sums and count itself; the one that ends last another
// 2 us, and 2 us to read each part's sums: a wave has room for one part's in flight.  (Measured at 7B: 256 rows, O and down, all
// pieces in 8 parts 19 -> 35 and 42 -> 54 us; QKV at 208 rows, 12 of 18 pieces in 2 parts 49 -> 50; but gate / up, one piece
// of 33 in 4 to 16 parts, 288 rows 89 -> 82 and 333 rows 107 -> 94: there all of it lies beside whole pieces.  These are launches
// whose weights come from memory; in two layers run again and again, most of them out of the cache behind L2, 288 rows are level.)
inline int64_t wide_part_cost(int g, int kt, int parts, bool last) {
    return wide_piece_cost(g, round_up(ceil_div(kt, parts), kWideDepth)) + 220 + (last ? 147 + 147 * parts : 0);
}

// Whether a tail is 10 % ahead of the cut `c` in this model (complete sums only), and which.  Rounds of workgroups that
// are nearly empty are what it removes: gate / up at 333 rows and 7B width is 11 weight groups per XCD in pieces of 128, 128
// and 96 rows, one piece more than an XCD has CUs, and either two pieces share a CU or smaller ones stream the
// weights more often.  Two tails are tried with every cut: what exceeds whole rounds of workgroups, and all pieces of
// the last size.  Measured, without / with: 7B gate / up at 208 and 224 rows 84 / 74 us, 333 and 352 rows 113 / 99, QKV at
// 704 rows 118 / 113; 13B gate / up at 288 and 333 rows 133 / 122 and 159 / 148; 70B gate / up at 512 and 896 rows 688 /
// 635 and 1203 / 1117.  5 to 10 % ahead in the model is within what cards differ by: 7B QKV at 648 and 1024 rows 102.4 / 101.7 and
// 161 / 157 on one, 108.9 / 113.0 and level on another that holds a lower clock.  Whole prompts of six layers, us a
// layer: 7B 208 rows -4.4, 288 -3.2, 320 -5.4, 333 and 352 -11.6; 13B 288 rows -5.5, 333 and 352 -4.2; level (-2.6 .. +1.7,
// which is also what runs differ by) at the other 23 of 32 row counts from 208 to 896.
inline bool plan_wide_tail(int n_groups, int n, int k_tiles, int m, const WideCut& c, WideCut* cut, WideTail* tail) {
    const int groups = ceil_div(ceil_div(m, 16), 2), gk8 = ceil_div(n_groups, 8);
    if (groups > kWideSearchGroups || k_tiles < kWideTailMinK) return false;
    const int kt_c = round_up(ceil_div(k_tiles, c.ksplit), kWideDepth), kt = round_up(k_tiles, kWideDepth);
    const int64_t now = wide_cost(c.parts, ceil_div(n_groups * c.ksplit, 8), kt_c) +
                        (int64_t)((c.ksplit - 1) * (double)m * n * 4.0 / (4.5e6 * kWideUnitUs));
    int64_t bar = now * 90 / 100;
    bool found = false;
    int64_t piece[4];
    for (int q = 0; q < 4; ++q) piece[q] = wide_piece_cost(4 - q, kt);
    for (int a = groups / 4; a >= 0; --a)
        for (int b = (groups - 4 * a) / 3; b >= 0; --b) {
            const int rest = groups - 4 * a - 3 * b;
            const WideParts w{{a, b, rest / 2, rest % 2}, 1};
            int64_t total = 0;
            int all = 0, big = -1, small = 0;  // largest and smallest size there is
            for (int q = 0; q < 4; ++q) {
                total += piece[q] * w.count[q] * gk8;
                all += w.count[q] * gk8;
                if (w.count[q]) {
                    if (big < 0) big = q;
                    small = q;
                }
            }
            if (total / kWideCus >= bar) continue;
            for (int order = 1; order <= 2; ++order) {
                if (order == 2 && big == small) break;
                const int last = order == 1 ? small : big;
                const int sizes[2] = {all % kWideCus, w.count[last] * gk8};
                for (int which = 0; which < 2; ++which) {
                    const int t = sizes[which];
                    if (t < 1 || t > w.count[last] * gk8 || 2 * t > kWideTailSlots || (which && t == sizes[0])) continue;
                    for (int parts = 2; parts <= 8 && parts * t <= kWideTailSlots && kt / parts >= 16; parts += parts < 4 ? 1 : 2) {
                        if ((parts - 1) * round_up(ceil_div(kt, parts), kWideDepth) >= kt) continue;  // an empty part
                        const int64_t part = wide_part_cost(4 - last, kt, parts, false), end = wide_part_cost(4 - last, kt, parts, true);
                        if ((total + t * ((parts - 1) * part + end - piece[last])) / kWideCus >= bar) continue;
                        auto size_of = [&](int run) { return order == 1 ? run : 3 - run; };
                        const int64_t cost = wide_place(6, [&](int run) { return run == 5 ? end : run == 4 ? part : piece[size_of(run)]; },
                                                        [&](int run) { return run == 5 ? t : run == 4 ? t * (parts - 1) : w.count[size_of(run)] * gk8 - (size_of(run) == last ? t : 0); }, bar);
                        if (cost < bar) {
                            bar = cost;
                            found = true;
                            *cut = WideCut{{{w.count[0], w.count[1], w.count[2], w.count[3]}, order}, 1};
                            *tail = WideTail{t, parts};
                        }
                    }
                }
            }
        }
    return found;
}

}  // namespace space
