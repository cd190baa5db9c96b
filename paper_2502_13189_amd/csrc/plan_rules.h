// Which rows of a batch are not routed: host rules of the plans (plain C++, no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace moba {

// Rows of a sequence's first topk blocks keep every past block, i.e. attend
// their whole prefix: a causal tile then does what routed tiles, their partials
// and the merge would, and the gate has nothing to choose.  But such a tile is
// up to topk blocks long, so only where the sequence's causal tiles alone keep
// half of the chip's 512 128-row work-groups busy for that long.  (Of the
// sequence alone, so that its rows do not depend on the batch.)  Returns the blocks
// taken out of the routing: topk, or 1 (block 0, which has no past).  The whole
// forward, all rows routed, then with the head: 8192 tokens, 32 heads, B = 512,
// top-3: 366 -> 352 us; 32K tokens, B = 256, top-32: 8.64 -> 7.97 ms; 112K ragged
// tokens, B = 1024, top-4: 8.93 -> 8.76 ms.
inline int head_blocks(int64_t L, int Hq, int B, int topk) {
  if (B < 1 || topk < 2) return 1;
  const double h = (double)std::min<int64_t>(L, (int64_t)topk * B);
  const double pairs = 0.5 * h * h + 0.5 * B * (L - h);
  return pairs * Hq / 128 >= 256.0 * h ? topk : 1;
}

// Whether the backward takes the forward's head blocks.  A head row saves it
// (topk - 1) / 2 fp32 dQ partials (about 0.38 ns each) but costs dK/dV a masked row for
// every key of the head (8e-5 ns each, topk B / 2 per row: all of the saving at B = 4600),
// and the head's last causal tile, one work-group per CU, holds up the dQ launch for
// up to 16 ns per key of its length; per row of one query head the saving must exceed
// that with a margin: Hq (topk - 1) (1 - B / 4600) >= 130.  dK/dV and dQ without and with
// head blocks: 16K tokens, 32/8 heads, B = 256, top-16 (453): 5475 -> 5105 us; 32K, 32/8, B =
// 512, top-8 (199): 8903 -> 8703; 48K, 32/8, B = 1024, top-8 (174): 23.10 -> 22.85 ms; 32K,
// 32/8, B = 700, top-5 (109): 7223 -> 7203 us; 48K, 32/8, B = 2048, top-8 (124): 38.84 -> 38.95
// ms; 8192, 32/8, B = 512, top-4 (85): 1084 -> 1102 us; 16K, 16/16, B = 512, top-4 (43): 1236 ->
// 1300; 24000, 16/16, B = 3000, top-5 (22): 7.13 -> 7.43 ms.  (Few blocks of 4096 keys would gain
// up to 5%, as their own tiles fill the chip badly, but others of that length lose.)
// Below top-4 it was never faster.
inline bool bwd_head_blocks(int Hq, int B, int topk) {
  return topk >= 4 && (double)Hq * (topk - 1) * (1.0 - B / 4600.0) >= 130.0;
}

}  // namespace moba
