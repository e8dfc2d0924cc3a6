// How a decode call splits the live lists over workgroups. Plain C++: no HIP in here.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "ikv.h"

namespace ikv {

constexpr int DEC_ROUND = 512;                     // workgroups of one resident round (two per CU on 256 CUs)
constexpr int DEC_MAX_SPLITS = 64;                 // of a live list

// Adjacent KV heads that a workgroup of the decode kernel takes: up to four in the head-group
// kernel (bf16, D = 128), one otherwise.
inline int decode_heads_per_wg(const ikv_pool &p) {
  if (p.kv_dtype != IKV_BF16 || p.D != 128) return 1;
  return p.Hkv % 4 == 0 ? 4 : (p.Hkv % 2 == 0 ? 2 : 1);
}

// Workgroups per split of a session.
inline int64_t decode_units(const ikv_pool &p) { return int64_t(p.L) * (p.Hkv / decode_heads_per_wg(p)); }

// An upper bound on the live positions a session holds after a retention event: the forced
// set (at most pi + qe - qs positions) plus the budget, and never more than N. A slot map
// that was never pruned may hold more; the decode is then still exact, only with longer
// splits.
inline int64_t decode_live_bound(const ikv_session &s) {
  const int64_t forced = int64_t(std::max(0, s.pi)) + std::max(0, s.qe - s.qs);
  return std::max<int64_t>(1, std::min<int64_t>(s.N, std::max<int64_t>(s.C, forced)));
}

// Percent of its rounds' workgroups that a grid of n > 0 workgroups fills.
inline int64_t decode_fill(int64_t n) { return 100 * n / ((n + DEC_ROUND - 1) / DEC_ROUND * DEC_ROUND); }

// Splits of every session's live list, from bounds known on the host. Every session has the
// same number, so that every workgroup has work wherever the dispatcher puts it (with splits
// per session and empty workgroups after them, whole XCDs went without).
//
// One resident round of workgroups, at least 64 live positions per split, at most 64 splits.
// A workgroup ends with its split's stores, and its slot takes no new work until they are
// done; long splits in one round pay that once per slot. At the Qwen3-8B 32k step (8192 live,
// 72 units) that is 7 splits of 1171 positions: the head-group kernel 196 us against 212 with
// 32 splits of 256 (without the stores, 32 splits ran in 191).
//
// Several sessions that one round holds fewer than three splits of (calls of the head-group
// kernel, us):
//  - more splits where they fill their rounds better, up to four of at least 256 positions:
//    8 x 72 units of 3000 positions 636 with one split, 574 with four; 16 x 48 units 817 and
//    765 with two; where one split fills them, one is best (5 x 96 units of 2400 to 3000
//    positions: 433, 438 with two; of 1200 to 1500: 239 and 247).
//  - lists of uneven bounds (the longest 1.15 times the mean or more): up to eight splits of
//    at least 768 positions in up to ten rounds, so that the last workgroups are short ones.
//    5 x 96 units of 1200 to 12,000 positions 1402 with one split, 1155 with eight; 16 x 48
//    units of 517 to 8192 positions 1813 with one, 1642 with two, 1536 with six. Below 768
//    positions the splits cost more than they even out (16 x 96 units of 375 to 1500: 586 with
//    one, 608 with four).
inline int decode_splits(const ikv_pool &p, const ikv_session *sess, int B) {
  int64_t longest = 1, sum = 0;
  for (int b = 0; b < B; ++b) {
    const int64_t n = decode_live_bound(sess[b]);
    longest = std::max(longest, n);
    sum += n;
  }
  const int64_t wgs = std::max<int64_t>(1, decode_units(p) * std::max(1, B));
  int64_t s = std::max<int64_t>(1, DEC_ROUND / wgs);
  if (B > 1 && s < 3) {
    for (int64_t k = s + 1; k <= 4 && longest >= 256 * k && decode_fill(s * wgs) < 90; ++k)
      if (decode_fill(k * wgs) > decode_fill(s * wgs)) s = k;
    if (20 * longest * B >= 23 * sum) {
      const int64_t most = std::min<int64_t>(8, std::min<int64_t>(longest / 768, 10 * DEC_ROUND / wgs));
      for (int64_t k = most; k > s; --k)
        if (decode_fill(k * wgs) >= 90) s = k;
    }
  }
  s = std::min<int64_t>(s, (longest + 63) / 64);
  return int(std::min<int64_t>(s, DEC_MAX_SPLITS));
}

}  // namespace ikv
