// Worklist of the pipelined decoder cross-attention, built on the host.
#pragma once

#include <cstdint>
#include <vector>

#include "tx_internal.h"

namespace tx {

// One tile set per kind: whole-request tiles (rows written normalised) and
// kv-split tiles (partial slots, merged afterwards); each is a per-XCD list
// set of its own, the XCDs' loads balanced over both.
struct XTileSet {
  std::vector<XTile> tiles;   // per-XCD lists, concatenated
  std::vector<int32_t> xoff;  // 9 entries: XCD x owns tiles[xoff[x] .. xoff[x + 1])
  int longest() const {
    int n = 0;
    for (int x = 0; x + 1 < (int)xoff.size(); ++x) n = n > xoff[x + 1] - xoff[x] ? n : xoff[x + 1] - xoff[x];
    return n;
  }
};
struct XPlan {
  XTileSet whole, split;
  std::vector<XMerge> merges;
  int n_parts = 0;  // partial slots used (kv-split tiles)
};

// Histories of fewer pages are never split: whether one is, and into how many
// parts, depends on the work of the whole batch, and parts change the order of
// the sums. A score of a request with at most kXWholePages - 1 pages (1984
// tokens) is therefore bitwise the same whatever users and candidates share the
// call and however the call is cut into passes; past that it may differ by the
// rounding of another order of summing. (Splitting from 8 pages on ran a call
// of 8 users of 500-4000 tokens in 358 us against 404.)
constexpr int kXWholePages = 32;

// Fewest pages a kv-split part covers. A part costs a partial slot written and
// read back (66 KB each way), a page of its block about 1 us; with 4 pages
// instead of 16 (and the whole-request tiles in the same launch) a layer of one
// user of 16384 (64-page parts before, 37 now) went from 97 + 19 us (split, merge)
// to 79 + 8.
constexpr int kXMinSplitPages = 4;

// Tiles for the requests of one cross-attention launch (queries of request r:
// reqs[r].qa_n + reqs[r].qb_n, keys: its first kv_len cached tokens) on a GPU
// with `resident_blocks` resident blocks, using at most max_parts partial
// slots.
void xattn_plan(const std::vector<AttnReq>& reqs, int H, int resident_blocks, int max_parts, XPlan& out);

}  // namespace tx
