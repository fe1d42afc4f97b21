// How the key-split attention of a batch deals its workgroups out by length: into how many parts each sequence is cut,
// where the parts lie in the table, and which workgroup takes which place of it.  The same functions on the host and in the
// kernels (constexpr functions are both), plain C++ so that they can be checked without a GPU.
#pragma once

namespace space {

// How many places at the end of `places` (each one workgroup per head) share a CU with the first ones; negative: not all
// workgroups fit the chip at once.  At most half of them: the workgroups beyond 256 rarely fill whole places, and 21
// places of 24 heads (504 workgroups, 248 beyond 256) would round to 11, one more than has a partner.
constexpr int attention_shared(int places, int n_heads) {
    const int over = places * n_heads - 256;
    if (over <= 0) return 0;
    if (over > 256) return -1;
    const int shared = (over + n_heads - 1) / n_heads;
    return shared < places / 2 ? shared : places / 2;
}

// Batches with more workgroups than CUs and one workgroup for all keys of a (sequence, head, query group): who shares a
// CU with whom, and who starts first, goes by length.  Workgroup 256 + i runs on the CU of workgroup i while all fit
// (two per CU), each at half speed.  shared > 0: that many places at the end of the `places` share a CU with the
// first ones; the longest sequences get the places between, alone, and of the others the longest go with the shortest.
// shared < 0: more than fit at once, longest first.  Returns the place's rank by length (of its part).
// (648 rows of 8 sequences, 458 to 3685 cached positions: in batch order 1377 and 3685 shared a CU, 87 us per layer, by length 79;
// 70B, 8 ragged sequences of 81 rows, 1024 workgroups, 134 / 82.)
constexpr int attention_item(int place, int places, int shared) {
    if (shared < 0) return place;
    if (place < shared) return places - 2 * shared + place;
    if (place >= places - shared) return places - 1 - (place - (places - shared));
    return place - shared;
}

// A workgroup's share of a batch: part `part` of n_parts over the keys of sequence b, `len` cached ones; b < 0: none.  The table
// holds the parts that every (head, query group) has, largest first, the parts of a sequence one behind the other.
constexpr int kMaxKeyParts = 16, kMaxKeySlots = 512;
struct KeyPart {
    int b, part, n_parts, len;
};

// Chunks of a sequence, the block's included (0: no sequence), and the most parts it may have: at least four cached chunks
// (a round of the four waves of a workgroup) for each.
struct KeySeq {
    int chunks, most;
};
constexpr KeySeq key_seq(int cached_chunks, int block_chunks) {
    const int most = cached_chunks / 4 < kMaxKeyParts ? cached_chunks / 4 : kMaxKeyParts;
    return KeySeq{cached_chunks + block_chunks, most > 1 ? most : 1};
}
// Parts of a sequence if none is to have more than `size` chunks (as far as it may be cut); at size >= longest: one.
constexpr int key_parts(const KeySeq& s, int size, int longest) {
    if (s.chunks == 0) return 0;
    if (size >= longest) return 1;
    const int n = (s.chunks + size - 1) / size;
    return n < s.most ? n : s.most;
}
// An even share of a sequence's chunks, by which the parts are ordered and the cut is priced: how many of them the last part has
// (below) does not belong there.  (Sizes in whole rounds, the block counted as kBlockRounds: 20 sequences of 8 heads of 64 277.5 ->
// 292 us a step of six layers, 30 of them 289 -> 301, 8 of 40 heads of 128 813 -> 827; none of 70 batches ahead.)
constexpr int key_part_chunks(const KeySeq& s, int n) { return n ? (s.chunks + n - 1) / n : 0; }

// First round of cached chunks (a chunk per wave each) of part p, of part n_parts the end, where the last part alone stages the
// block's keys and values and takes its chunks.  That costs as much as kBlockRounds rounds (measured in a batch of 8 x 36 rows, us: staging 14
// instead of 6, the block's chunks 2, a round 4.4 while HBM is busy; with equal parts the last ones ended 10 us behind all others;
// 1, 3 and 4 rounds are level with 2 over 70 ragged batches of one to three query tiles, heads of 64 and of 128).  So no part has more than
// rounds and block dealt out evenly: the last one what the others leave at that size, down to none, and they share the rest evenly, one
// more for the first ones.  No part before the last is empty.
constexpr int kBlockRounds = 2;
constexpr int key_part_first(int rounds, int n_parts, int p) {
    if (p <= 0) return 0;
    if (p >= n_parts) return rounds;
    const int others = n_parts - 1, full = others * ((rounds + kBlockRounds + n_parts - 1) / n_parts), rest = rounds < full ? rounds : full;
    const int one_more = rest % others;
    return p * (rest / others) + (p < one_more ? p : one_more);
}

// What the busiest CU spends on `parts` parts of at most `largest` chunks: these and, worth `staging` chunks, what a part does in
// front of them; beyond a workgroup per CU the mean over the CUs, of which 232 are taken to be busy, counts as well.  kPartStaging: the
// kernel for few rows stages the block.  kRowsStaging: attn_rows_kernel only asks for its queries, and while a CU has one of its
// workgroups leaves a third of its time unused, so long sequences are better cut than alone (priced at 16 it was up to 9 %
// behind the kernel for few rows there; five-layer prompts, that kernel / priced at 16 / at 2, us: 2 sequences of 256 rows behind 2000 and 4000
// positions, 32 heads of 128 1199 / 1230 / 1140, of 64 788 / 853 / 783; 4 of 512 rows behind 512 to 2048, 8 heads of 64, 449 / 491 / 445; 6 and
// 10 lie in between, equal lengths are level).
constexpr int kPartStaging = 16, kRowsStaging = 2;
constexpr int key_cut_cost(int parts, int largest, int total, int streams, int staging) {
    const int alone = largest + staging;
    const int mean = parts * streams > 256 ? (total + parts * staging) * streams / 232 : 0;
    return alone > mean ? alone : mean;
}

struct KeyCut {
    int size;   // for key_parts
    int parts;  // of all sequences
};
// The smallest largest part that the slots allow; no cut (size = longest) where it is not 8 % ahead of none.
//   longest, total  chunks of the longest sequence and of all of them;  parts_at(size): parts of all sequences
template <class PartsAt>
constexpr KeyCut key_cut(int batch, int slots, int streams, int longest, int total, PartsAt parts_at, int staging = kPartStaging) {
    const KeyCut none{longest, batch};
    if (slots <= batch) return none;
    int size = total / slots > 1 ? total / slots : 1, parts = batch;
    for (;;) {  // ends: at size >= longest every sequence has one part
        parts = parts_at(size);
        if (size >= longest || parts <= slots) break;
        size += size >> 3 > 1 ? size >> 3 : 1;
    }
    if (key_cut_cost(parts, size, total, streams, staging) * 100 > key_cut_cost(batch, longest, total, streams, staging) * 92) return none;
    return KeyCut{size, parts};
}

// First place of sequence b in the table: the parts of sequences with larger ones lie in front (equal ones by index).
template <class Chunks, class Parts>
constexpr int key_first_place(int b, int own_chunks, int batch, Chunks part_chunks_of, Parts parts_of) {
    int first = 0;
    for (int i = 0; i < batch; ++i) {
        const int other = part_chunks_of(i), n = parts_of(i);
        first += other > own_chunks || (other == own_chunks && i < b) ? n : 0;
    }
    return first;
}

}  // namespace space
