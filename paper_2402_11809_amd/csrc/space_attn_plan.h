// Which workgroup of a batch's attention takes which place in the order by length: the same functions on the host and
// in the kernel (constexpr functions are both), plain C++ so that they can be checked without a GPU.
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

}  // namespace space
