// When a long ingest runs its last layer only for the rows that are used (run_body).
#pragma once
#include "osprey.h"

namespace osp {

constexpr int kNarrowFp32Rows = 16;          // the vector body computes eight rows at a time
constexpr int kNarrowBf16Rows = 64;          // up to here a layer costs its launches, not its rows
constexpr long kNarrowWeights = 32L << 20;
constexpr long kNarrowFp32Bytes = 150000000;

// `rows` new rows of which `keep` (one per sequence) are used.  Narrowing costs a key/value
// product for every row beside the kept rows' whole QKV product, an append and a gather; it
// saves the other rows' query part, O projection and FFN (`w` weights).
//
// bf16: whole ingests with one draft, never / always narrowed, us:
//   d 1024 (w 16M): 48 sequences of 2 rows 422 / 435, of 3 467 / 460; 64 of 2 479 / 493, of 3
//     522 / 516; 96 of 1 560 / 610, of 3 688 / 695, of 4 723 / 719; 128 of 4 891 / 892, of 6
//     982 / 946; one of 65 261 / 250
//   d 2560 (w 106M): 33 of 2 685 / 662; 64 of 2 922 / 865; 96 of 2 945 / 998, of 3 1103 / 1099
//   d 2048, 64-wide heads (w 63M): 64 of 1 or 2 884 / 895, of 2 1003 / 989; 96 of 2 1080 / 1122,
//     of 3 1322 / 1303
// so two rows per sequence pay, three where the weights are few or the kept rows are more
// than one streaming pass, four where both hold.
//
// fp32: d 256: 2 of 8 rows 82 / 77, 4 of 4 83 / 88, 4 of 8 90 / 90, 8 of 4 97 / 109, 16 of 8
// 132 / 131, 32 of 8 203 / 188; d 1024 (63 MB per group of eight rows): 4 of 4 449 / 450, 4 of 6
// 491 / 456, 8 of 3 670 / 680, 8 of 4 704 / 685, 16 of 1 or 2 1153 / 1166: eight rows per
// sequence, or as many groups less as read 150 MB of weights.
inline bool narrow_pays(const osprey_config& c, long rows, long keep) {
  const long d = c.d_model, o = (long)c.n_q_heads * c.head_dim;
  const long w = 3 * d * o + 3 * d * c.d_ffn;
  if (c.dtype == OSPREY_BF16) {
    const long per = 2 + (w < kNarrowWeights ? 1 : 0) + (keep > kNarrowBf16Rows ? 1 : 0);
    return rows > kNarrowBf16Rows && rows >= per * keep;
  }
  if (rows < kNarrowFp32Rows || rows <= keep) return false;
  // (up to eight kept rows cost the vector body 1, 2, 4 or 8 of a group)
  const long kept = keep <= 1 ? 1 : (keep <= 2 ? 2 : (keep <= 4 ? 4 : (keep + 7) / 8 * 8));
  return rows >= 8 * keep || ((rows + 7) / 8 * 8 - kept) * 4 * w / 8 >= kNarrowFp32Bytes;
}

}  // namespace osp
