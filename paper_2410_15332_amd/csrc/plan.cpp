// Host planner of the link step: integer work only, no device calls.
//
// Builds, for a batch of requests, the selected set S (LegoLink-k, Sec. 4.2:
// the first k tokens of every chunk but the first, plus the suffix; k < 0 =
// every token, Sec. 2.3), the linked block tables (chunks concatenated in
// order, then the suffix), the request-private blocks that receive recomputed
// K/V (copy-on-write when a block also keeps cached rows), and the attention
// work decomposition (query tiles x split-KV key ranges).
#include <algorithm>
#include <cstring>
#include <functional>
#include <vector>

#include "plan_internal.h"
#include "status.h"

namespace epic {

epic_status validate_attn_cfg(const epic_attn_cfg* cfg) {
  EPIC_CHECK_ARG(cfg != nullptr, "attention config is NULL");
  if (cfg->num_kv_heads <= 0 || cfg->num_q_heads <= 0 || cfg->num_q_heads % cfg->num_kv_heads != 0)
    return fail(EPIC_ERR_INVALID_ARG, "num_q_heads (%d) must be a positive multiple of num_kv_heads (%d)",
                cfg->num_q_heads, cfg->num_kv_heads);
  const int G = cfg->num_q_heads / cfg->num_kv_heads;
  if ((G & (G - 1)) != 0 || G > kTileRowsSmall)
    return fail(EPIC_ERR_UNSUPPORTED, "query heads per KV head (%d) must be a power of two <= %d", G,
                kTileRowsSmall);
  if (cfg->head_dim != 64 && cfg->head_dim != 128)
    return fail(EPIC_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", cfg->head_dim);
  if (cfg->block_size != kBlock)
    return fail(EPIC_ERR_UNSUPPORTED, "block_size %d not supported (16)", cfg->block_size);
  if (cfg->kv_split_blocks < 0)
    return fail(EPIC_ERR_INVALID_ARG, "kv_split_blocks %d < 0", cfg->kv_split_blocks);
  if (cfg->tile_rows != 0 && !valid_tile_rows(cfg->tile_rows))
    return fail(EPIC_ERR_UNSUPPORTED, "tile_rows %d (expected 0, %d, %d or %d)", cfg->tile_rows, kTileRowsTiny,
                kTileRowsSmall, kTileRowsLarge);
  if (cfg->tile_rows == kTileRowsTiny && G > kTileRowsTiny)
    return fail(EPIC_ERR_UNSUPPORTED, "tile_rows %d needs at most %d query heads per KV head (%d)", kTileRowsTiny,
                kTileRowsTiny, G);
  if (!(cfg->softmax_scale >= 0.0f)) return fail(EPIC_ERR_INVALID_ARG, "softmax_scale must be >= 0");
  return EPIC_OK;
}

namespace {

int cdiv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

struct ReqShape {
  int64_t n_chunk_tokens = 0;
  int n_s = 0, n_lb = 0, n_priv = 0, n_rerot = 0;
};

// Re-rotation applies to the cached rows of chunks after the first (chunk 0 sits
// at offset 0, where the compile rotation is already the linked one).
bool rerotates(const epic_link_request& r, int j) { return r.rerotate != 0 && r.k >= 0 && j > 0; }

// Number of tokens of chunk j that belong to S.
int selected_in_chunk(const epic_link_request& r, int j) {
  if (r.k < 0) return r.chunk_len[j];
  if (j == 0) return 0;  // the first chunk is never recomputed
  return std::min(r.k, r.chunk_len[j]);
}

epic_status validate_request(const epic_link_request& r, int idx, ReqShape* sh) {
  EPIC_CHECK_ARG(r.num_chunks >= 0, "request %d: num_chunks %d < 0", idx, r.num_chunks);
  EPIC_CHECK_ARG(r.suffix_len >= 0, "request %d: suffix_len %d < 0", idx, r.suffix_len);
  EPIC_CHECK_ARG(r.rerotate == 0 || r.rerotate == 1, "request %d: rerotate %d (0 or 1)", idx, r.rerotate);
  if (r.num_chunks > 0) {
    EPIC_CHECK_ARG(r.chunk_len && r.chunk_block_off && r.chunk_blocks,
                   "request %d: chunk arrays are NULL", idx);
    EPIC_CHECK_ARG(r.chunk_block_off[0] == 0, "request %d: chunk_block_off[0] != 0", idx);
  }
  *sh = ReqShape{};
  for (int j = 0; j < r.num_chunks; ++j) {
    const int L = r.chunk_len[j];
    EPIC_CHECK_ARG(L >= 1, "request %d chunk %d: length %d < 1", idx, j, L);
    const int nb = r.chunk_block_off[j + 1] - r.chunk_block_off[j];
    EPIC_CHECK_ARG(nb == cdiv(L, kBlock), "request %d chunk %d: %d blocks given, %d needed", idx, j, nb,
                   cdiv(L, kBlock));
    sh->n_chunk_tokens += L;
    const int sel = selected_in_chunk(r, j);
    sh->n_s += sel;
    sh->n_lb += nb;
    if (rerotates(r, j)) {
      sh->n_priv += nb;                                   // every block: a rotated copy
      sh->n_rerot += sel >= L ? 0 : nb - sel / kBlock;    // those that keep a cached row
    } else {
      sh->n_priv += cdiv(sel, kBlock);
    }
  }
  sh->n_s += r.suffix_len;
  sh->n_lb += cdiv(r.suffix_len, kBlock);
  sh->n_priv += cdiv(r.suffix_len, kBlock);
  EPIC_CHECK_ARG(sh->n_chunk_tokens + r.suffix_len < (int64_t(1) << 30), "request %d: too many tokens", idx);
  return EPIC_OK;
}

// Linked positions of S for one request, ascending.
void select_positions(const epic_link_request& r, std::vector<int32_t>* pos) {
  int64_t off = 0;
  for (int j = 0; j < r.num_chunks; ++j) {
    const int sel = selected_in_chunk(r, j);
    for (int t = 0; t < sel; ++t) pos->push_back(static_cast<int32_t>(off + t));
    off += r.chunk_len[j];
  }
  for (int t = 0; t < r.suffix_len; ++t) pos->push_back(static_cast<int32_t>(off + t));
}

// Linked block table of one request: (pos0, len) of each block in position order.
void linked_blocks(const epic_link_request& r, std::vector<int32_t>* pos0, std::vector<int32_t>* len) {
  int64_t off = 0;
  for (int j = 0; j < r.num_chunks; ++j) {
    for (int t = 0; t < r.chunk_len[j]; t += kBlock) {
      pos0->push_back(static_cast<int32_t>(off + t));
      len->push_back(std::min(kBlock, r.chunk_len[j] - t));
    }
    off += r.chunk_len[j];
  }
  for (int t = 0; t < r.suffix_len; t += kBlock) {
    pos0->push_back(static_cast<int32_t>(off + t));
    len->push_back(std::min(kBlock, r.suffix_len - t));
  }
}

struct Tile {
  int req, row0, nrows, nblk;
};

// S positions and linked-block first positions of one request.
struct ReqRows {
  std::vector<int32_t> pos, p0;
};

// Query tiles: consecutive S rows of one request, rows_per_tile at a time.  A
// tile needs the linked blocks whose first position is <= its last row's position.
void make_tiles(const std::vector<ReqRows>& rr, int rows_per_tile, std::vector<Tile>* tiles) {
  int row_base = 0;
  for (size_t b = 0; b < rr.size(); ++b) {
    const std::vector<int32_t>& pos = rr[b].pos;
    const std::vector<int32_t>& p0 = rr[b].p0;
    for (size_t r0 = 0; r0 < pos.size(); r0 += rows_per_tile) {
      const int n = static_cast<int>(std::min<size_t>(rows_per_tile, pos.size() - r0));
      const int32_t last = pos[r0 + n - 1];
      const int nblk = static_cast<int>(std::upper_bound(p0.begin(), p0.end(), last) - p0.begin());
      tiles->push_back(Tile{static_cast<int>(b), row_base + static_cast<int>(r0), n, nblk});
    }
    row_base += static_cast<int>(pos.size());
  }
}

// Work items of a split, in launch order: longest key range first, so the
// dispatcher's greedy fill of freed workgroup slots ends with the short items;
// among equal lengths segment-major (all first segments, then all second
// segments, ...) and tiles with the longest key range first, so workgroups that
// start together read the same KV blocks through their XCD's L2.  Each entry:
// (tile, segment).
std::vector<std::pair<int, int>> item_order(const std::vector<Tile>& tiles, int split) {
  std::vector<int> order(tiles.size());
  for (size_t t = 0; t < tiles.size(); ++t) order[t] = static_cast<int>(t);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return tiles[x].nblk > tiles[y].nblk; });
  int max_splits = 1;
  for (const Tile& t : tiles) max_splits = std::max(max_splits, cdiv(t.nblk, split));
  std::vector<std::pair<int, int>> items;
  for (int seg = 0; seg < max_splits; ++seg)
    for (int t : order)
      if (seg < std::max(1, cdiv(tiles[t].nblk, split))) items.emplace_back(t, seg);
  auto blocks = [&](const std::pair<int, int>& it) {
    return std::min(tiles[it.first].nblk, (it.second + 1) * split) - it.second * split;
  };
  std::stable_sort(items.begin(), items.end(),
                   [&](const std::pair<int, int>& x, const std::pair<int, int>& y) { return blocks(x) > blocks(y); });
  return items;
}

// Kernel shape of a tile size: workgroup slots per launch round, and the time of
// one 64-key step of one workgroup and its fixed prologue / epilogue charge, in
// steps (the split search compares splits of one shape only).
// A split item also writes its fp32 partial tile, which the combine reads back.
struct TileShape {
  int rows, slots;
  double step_cost, item_overhead, partial_cost;
};
constexpr TileShape kShapeLarge{kTileRowsLarge, 256, 1.0, 3.0, 4.0};   // one 8-wavefront workgroup per CU, 256 CUs
constexpr TileShape kShapeSmall{kTileRowsSmall, 512, 1.0, 2.0, 4.0};   // two 4-wavefront workgroups per CU
constexpr TileShape kShapeTiny{kTileRowsTiny, 768, 1.0, 2.0, 1.0};      // three 4-wavefront workgroups per CU

// Estimated duration of the attention launch for a split: the items (times the
// KV heads, head-minor as in the grid) are dealt in launch order to the
// workgroup slots, each to the slot that frees up first -- as the hardware
// dispatcher does -- and an item costs its steps plus a fixed prologue /
// epilogue charge.  An item's heads cost the same, so where the heads divide the slots
// evenly the slots stay in groups of equal finish times, one per head, and one slot of
// each group stands for it: the same times from a heap of slots / heads entries.
double estimate_makespan(const std::vector<Tile>& tiles, int split, int hkv, const TileShape& sh) {
  const int same = sh.slots % hkv == 0 ? hkv : 1;       // slots per group
  std::vector<double> slots(sh.slots / same, 0.0);   // min-heap of slot finish times
  double makespan = 0.0;
  for (const auto& [t, seg] : item_order(tiles, split)) {
    const int blocks = std::min(tiles[t].nblk, (seg + 1) * split) - seg * split;
    const bool partial = tiles[t].nblk > split;
    const double cost = cdiv(std::max(blocks, 1), kKvTileBlocks) * sh.step_cost + sh.item_overhead +
                        (partial ? sh.partial_cost : 0.0);
    for (int g = 0; g < hkv; g += same) {
      std::pop_heap(slots.begin(), slots.end(), std::greater<double>());
      slots.back() += cost;
      makespan = std::max(makespan, slots.back());
      std::push_heap(slots.begin(), slots.end(), std::greater<double>());
    }
  }
  return makespan;
}

// Key blocks per split-KV work item: among splits max_nblk / n (n from 1 to 128
// in about geometric steps, rounded up to whole 4-block tiles), the one with the
// shortest estimated launch, where a finer split must be 3% shorter to win (fewer
// partials).  Below 64 blocks only while every item has a CU to itself: there the
// launch lasts as long as its longest item, whatever the others do (4 x 128 + 16
// tokens, 8 heads of 64: 9 steps in one item 14.9 us, a step each 4.8 and 3.7 for
// the combine); with more items the partials that every split writes and re-reads
// cost more than they gain (10 x 512 tokens, 32 heads: 64 blocks 34 + 5 us, 32
// blocks 33 + 7, 16 blocks 48 + 10).  *time receives that estimate.
int split_blocks(const epic_attn_cfg* cfg, const std::vector<Tile>& tiles, const TileShape& sh, double* time) {
  const int hkv = cfg->num_kv_heads;
  if (cfg->kv_split_blocks > 0) {
    const int split = std::max(kKvTileBlocks, cfg->kv_split_blocks / kKvTileBlocks * kKvTileBlocks);
    *time = estimate_makespan(tiles, split, hkv, sh);
    return split;
  }
  constexpr int kMinSplit = 64;        // ... in general
  constexpr int64_t kCus = 256;
  constexpr int64_t kMaxRounds = 16;   // past this many dispatch rounds, splitting cannot balance better
  int max_nblk = kKvTileBlocks;
  for (const Tile& t : tiles) max_nblk = std::max(max_nblk, t.nblk);
  auto n_items = [&](int split) {
    int64_t n = 0;
    for (const Tile& t : tiles) n += std::max(1, cdiv(t.nblk, split));
    return n;
  };
  // A first split adds the combine's launch, which a short decode item does not repay
  // (in steps; called one by one, 14 blocks unsplit 13.5 us, split 15.2; 125 blocks of 128
  // dims 23 -> 15; on the GPU, 120 items of 110 blocks of 64 dims in two parts 22.6 -> 19.2).
  const double first_split = sh.rows == kTileRowsTiny ? 8.0 : 0.0;
  const int whole = cdiv(max_nblk, kKvTileBlocks) * kKvTileBlocks;
  // Likewise link items of up to 8 steps of 64 dims.  Calls made one by one go at the host's
  // pace, two launches whole (7 / 8 / 9 steps 13.6 / 15.9 / 16.5 us), three split (17.3 / 17.5 /
  // 17.0); replayed from a HIP graph whole takes 21.0 / 23.2 / 23.7, split 19-21 / 19-21 / 20, so
  // there the line would lie at 6.  Not 128 dims, whose steps take longer (5 steps: whole 15.3,
  // split 17.2, in a graph 22.8 and 19.3; 6 steps: 19.5 and 16.9, 27.2 and 20.7).  And decode items
  // of up to 16 steps of 64 dims: two launches, 15 us on the GPU, are through when three are enqueued.
  if (cfg->head_dim == 64 && whole <= (sh.rows == kTileRowsTiny ? 16 : 8) * kKvTileBlocks) {
    *time = estimate_makespan(tiles, whole, hkv, sh);
    return whole;
  }
  int best = whole;
  double best_time = estimate_makespan(tiles, whole, hkv, sh);
  if (n_items(whole) * hkv < kMaxRounds * sh.slots) {
    int prev = whole;
    static constexpr int kParts[] = {2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 96, 128};
    for (const int n : kParts) {
      int split = cdiv(cdiv(max_nblk, n), kKvTileBlocks) * kKvTileBlocks;
      if (split < kMinSplit && n_items(split) * hkv > kCus) split = kMinSplit;
      if (split >= prev) continue;
      prev = split;
      if (n_items(split) * hkv > kMaxRounds * sh.slots) break;
      const double t = estimate_makespan(tiles, split, hkv, sh) + first_split;
      if (t < best_time * 0.97) {               // finer splits must pay for their partials clearly
        best_time = t;
        best = split;
      }
    }
  }
  *time = best_time;
  return best;
}

int64_t align16(int64_t n) { return (n + 15) & ~int64_t(15); }

}  // namespace

}  // namespace epic

using namespace epic;

namespace {

// Tile size and split-KV split for these S rows; fills s->tile_rows, n_tiles,
// n_work, n_partials.  256-row tiles share each staged K/V block between twice
// the rows, which pays when their rows need nearly the same keys and the tiles
// still balance over the CUs.  Take them when they cost at most 5% more
// (row x 64-key) steps than 128-row tiles, their estimated launch is at most
// kLargeEdge times that of 128-row tiles (each estimate in its own kernel's
// steps: the 8-wavefront kernel runs a 256-row step in about 1/1.07-1/1.13 of
// the time two 4-wavefront workgroups take for two 128-row steps, measured), and
// they give every CU a workgroup.
void choose_tiles(const std::vector<ReqRows>& rr, const epic_attn_cfg* cfg, epic_plan_sizes* s,
                  std::vector<Tile>* tiles_out, int* split_out) {
  const int G = cfg->num_q_heads / cfg->num_kv_heads;
  std::vector<Tile>& tiles = *tiles_out;
  // 16-row tiles (the decode kernel) when every request has at most 16 / G S rows:
  // a 128-row tile would hold almost only empty rows
  bool few_rows = G <= kTileRowsTiny;
  size_t any_rows = 0;
  for (const ReqRows& r : rr) {
    few_rows = few_rows && r.pos.size() <= static_cast<size_t>(kTileRowsTiny / G);
    any_rows += r.pos.size();
  }
  if (cfg->tile_rows == kTileRowsTiny || (cfg->tile_rows == 0 && few_rows && any_rows > 0)) {
    make_tiles(rr, kTileRowsTiny / G, &tiles);
    s->tile_rows = kTileRowsTiny;
    double est = 0.0;
    const int split = split_blocks(cfg, tiles, kShapeTiny, &est);
    *split_out = split;
    int64_t n_work = 0, n_part = 0;
    for (const Tile& t : tiles) {
      const int ns = std::max(1, cdiv(t.nblk, split));
      n_work += ns;
      if (ns > 1) n_part += ns;
    }
    s->n_tiles = static_cast<int32_t>(tiles.size());
    s->n_work = static_cast<int32_t>(n_work);
    s->n_partials = static_cast<int32_t>(n_part);
    return;
  }
  std::vector<Tile> small, large;
  make_tiles(rr, kTileRowsSmall / G, &small);
  make_tiles(rr, kTileRowsLarge / G, &large);
  auto row_steps = [](const std::vector<Tile>& ts, int rows) {
    int64_t n = 0;
    for (const Tile& t : ts) n += int64_t(cdiv(t.nblk, kKvTileBlocks)) * rows;
    return n;
  };
  constexpr double kLargeEdge = 1.07;
  double est = 0.0, est_small = 0.0;
  int split = split_blocks(cfg, large, kShapeLarge, &est);
  int64_t large_items = 0;
  for (const Tile& t : large) large_items += std::max(1, cdiv(t.nblk, split));
  bool use_large = cfg->tile_rows == kTileRowsLarge;
  int split_small = 0;
  if (cfg->tile_rows == 0 && row_steps(large, kTileRowsLarge) * 100 <= row_steps(small, kTileRowsSmall) * 105 &&
      large_items * cfg->num_kv_heads >= kShapeLarge.slots) {
    split_small = split_blocks(cfg, small, kShapeSmall, &est_small);
    use_large = est <= kLargeEdge * est_small;
  }
  if (use_large) {
    tiles.swap(large);
    s->tile_rows = kTileRowsLarge;
  } else {
    tiles.swap(small);
    s->tile_rows = kTileRowsSmall;
    split = split_small > 0 ? split_small : split_blocks(cfg, tiles, kShapeSmall, &est);
  }
  *split_out = split;
  int64_t n_work = 0, n_part = 0;
  for (const Tile& t : tiles) {
    const int ns = std::max(1, cdiv(t.nblk, split));
    n_work += ns;
    if (ns > 1) n_part += ns;
  }
  s->n_tiles = static_cast<int32_t>(tiles.size());
  s->n_work = static_cast<int32_t>(n_work);
  s->n_partials = static_cast<int32_t>(n_part);
}

void finish_sizes(epic_plan_sizes* s) {
  s->total_ints = 3 * align16(s->n_s) + 2 * align16(s->batch + 1) + 3 * align16(s->n_linked_blocks) +
                  3 * align16(s->n_private) + align16(int64_t(s->n_private) * kBlock) +
                  align16(4 * int64_t(s->n_tiles)) + align16(kWorkInts * int64_t(s->n_work));
}

// Attention tiles and split-KV work items of a plan whose S rows and linked
// tables are written.  Work items go in item_order's launch order (longest key
// range first; among equal lengths key segment first, so that workgroups that
// start together read the same KV blocks through their XCD's L2).
epic_status write_work(const std::vector<Tile>& tiles, int split, const epic_plan_sizes& chk, epic_plan* plan) {
  int part = 0;
  for (size_t t = 0; t < tiles.size(); ++t) {
    const int ns = std::max(1, cdiv(tiles[t].nblk, split));
    plan->tiles[4 * t + 0] = tiles[t].row0;
    plan->tiles[4 * t + 1] = tiles[t].nrows;
    plan->tiles[4 * t + 2] = ns > 1 ? part : -1;
    plan->tiles[4 * t + 3] = ns;
    if (ns > 1) part += ns;
  }
  // work items in launch order
  int w = 0;
  for (const auto& [t, seg] : item_order(tiles, split)) {
    const int ns = plan->tiles[4 * t + 3];
    const int base = plan->blk_off[tiles[t].req];
    const int b0 = base + seg * split;
    const int b1 = base + std::min(tiles[t].nblk, (seg + 1) * split);
    // Leading KV tiles (kKvTileBlocks blocks each) that need no mask: all
    // blocks full and every key at or before the tile's first row.
    const int32_t first_pos = plan->s_pos[tiles[t].row0];
    int n_fast = 0;
    for (int b = b0; b + kKvTileBlocks <= b1; b += kKvTileBlocks) {
      bool ok = true;
      for (int i = 0; i < kKvTileBlocks; ++i) ok = ok && plan->block_len[b + i] == kBlock;
      const int last = b + kKvTileBlocks - 1;
      ok = ok && plan->block_pos0[last] + kBlock - 1 <= first_pos;
      if (!ok) break;
      ++n_fast;
    }
    int32_t* wk = plan->work + int64_t(kWorkInts) * w;
    wk[0] = static_cast<int32_t>(t);
    wk[1] = b0;
    wk[2] = b1;
    wk[3] = ns > 1 ? plan->tiles[4 * t + 2] + seg : -1;
    wk[4] = n_fast;
    wk[5] = wk[6] = wk[7] = 0;
    ++w;
  }
  if (w != chk.n_work || part != chk.n_partials)
    return fail(EPIC_ERR_INVALID_ARG, "internal planner inconsistency (work)");
  return EPIC_OK;
}

// Sizes of the link plan, plus its attention tiles and split (shared by the sizes
// query and the plan builder, so the split search runs once per call).
epic_status plan_shape(const epic_link_request* reqs, int32_t batch, const epic_attn_cfg* cfg, int32_t n_free,
                       epic_plan_sizes* out, std::vector<Tile>* tiles_out, int* split_out) {
  EPIC_CHECK_ARG(out != nullptr, "output sizes pointer is NULL");
  EPIC_CHECK_ARG(batch >= 0, "batch %d < 0", batch);
  EPIC_CHECK_ARG(batch == 0 || reqs != nullptr, "requests pointer is NULL");
  EPIC_CHECK_ARG(n_free >= 0, "n_free %d < 0", n_free);
  epic_status st = validate_attn_cfg(cfg);
  if (st != EPIC_OK) return st;
  epic_plan_sizes s{};
  s.batch = batch;
  int64_t n_s = 0, n_lb = 0, n_priv = 0, n_rerot = 0, max_pos = 0;
  for (int b = 0; b < batch; ++b) {
    ReqShape sh;
    st = validate_request(reqs[b], b, &sh);
    if (st != EPIC_OK) return st;
    n_s += sh.n_s;
    n_lb += sh.n_lb;
    n_priv += sh.n_priv;
    n_rerot += sh.n_rerot;
    max_pos = std::max<int64_t>(max_pos, sh.n_chunk_tokens + reqs[b].suffix_len);
  }
  EPIC_CHECK_ARG(n_s < (int64_t(1) << 30) && n_lb < (int64_t(1) << 30), "batch too large");
  if (n_priv > n_free)
    return fail(EPIC_ERR_NO_PRIVATE_BLOCKS, "plan needs %lld private blocks, %d free", (long long)n_priv, n_free);
  std::vector<ReqRows> rr(static_cast<size_t>(batch));
  for (int b = 0; b < batch; ++b) {
    std::vector<int32_t> ln;
    select_positions(reqs[b], &rr[b].pos);
    linked_blocks(reqs[b], &rr[b].p0, &ln);
  }
  choose_tiles(rr, cfg, &s, tiles_out, split_out);
  s.n_s = static_cast<int32_t>(n_s);
  s.n_linked_blocks = static_cast<int32_t>(n_lb);
  s.n_private = static_cast<int32_t>(n_priv);
  s.n_rerotated = static_cast<int32_t>(n_rerot);
  s.max_pos = static_cast<int32_t>(max_pos);
  finish_sizes(&s);
  *out = s;
  return EPIC_OK;
}

}  // namespace

extern "C" epic_status epic_plan_sizes_get(const epic_link_request* reqs, int32_t batch,
                                           const epic_attn_cfg* cfg, int32_t n_free,
                                           epic_plan_sizes* out) {
  clear_error();
  std::vector<Tile> tiles;
  int split = 0;
  return plan_shape(reqs, batch, cfg, n_free, out, &tiles, &split);
}

extern "C" epic_status epic_plan_layout(const epic_plan_sizes* s, int32_t* base, epic_plan* p) {
  clear_error();
  EPIC_CHECK_ARG(s && p, "NULL argument");
  int32_t* cur = base;
  auto take = [&](int64_t n) {
    int32_t* r = cur;
    cur += align16(n);
    return r;
  };
  p->s_pos = take(s->n_s);
  p->s_req = take(s->n_s);
  p->s_slot = take(s->n_s);
  p->s_off = take(s->batch + 1);
  p->linked_blocks = take(s->n_linked_blocks);
  p->block_pos0 = take(s->n_linked_blocks);
  p->block_len = take(s->n_linked_blocks);
  p->blk_off = take(s->batch + 1);
  p->priv_block = take(s->n_private);
  p->priv_src = take(s->n_private);
  p->priv_rows = take(int64_t(s->n_private) * kBlock);
  p->tiles = take(4 * int64_t(s->n_tiles));
  p->work = take(kWorkInts * int64_t(s->n_work));
  p->priv_rot = take(s->n_private);
  if (cur - base != s->total_ints) return fail(EPIC_ERR_INVALID_ARG, "plan sizes are inconsistent");
  return EPIC_OK;
}

extern "C" epic_status epic_plan_link(const epic_link_request* reqs, int32_t batch,
                                      const epic_attn_cfg* cfg, const int32_t* free_blocks,
                                      int32_t n_free, int32_t num_blocks,
                                      const epic_plan_sizes* sizes, epic_plan* plan) {
  clear_error();
  epic_plan_sizes chk;
  std::vector<Tile> tiles;
  int split = 0;
  epic_status st = plan_shape(reqs, batch, cfg, n_free, &chk, &tiles, &split);
  if (st != EPIC_OK) return st;
  EPIC_CHECK_ARG(sizes && plan, "NULL sizes or plan");
  EPIC_CHECK_ARG(std::memcmp(&chk, sizes, sizeof(chk)) == 0, "sizes do not match these requests");
  EPIC_CHECK_ARG(num_blocks > 0, "num_blocks %d <= 0", num_blocks);
  EPIC_CHECK_ARG(chk.n_private == 0 || free_blocks != nullptr, "free_blocks is NULL");

  // Block ids: chunk blocks and free blocks in range, free blocks distinct and unused by chunks.
  std::vector<uint8_t> used(static_cast<size_t>(num_blocks), 0);
  for (int b = 0; b < batch; ++b) {
    const epic_link_request& r = reqs[b];
    const int nb = r.num_chunks > 0 ? r.chunk_block_off[r.num_chunks] : 0;
    for (int i = 0; i < nb; ++i) {
      const int id = r.chunk_blocks[i];
      EPIC_CHECK_ARG(id >= 0 && id < num_blocks, "request %d: chunk block id %d out of range [0, %d)", b, id,
                     num_blocks);
      used[id] = 1;
    }
  }
  for (int i = 0; i < chk.n_private; ++i) {
    const int id = free_blocks[i];
    EPIC_CHECK_ARG(id >= 0 && id < num_blocks, "free block id %d out of range [0, %d)", id, num_blocks);
    EPIC_CHECK_ARG(used[id] == 0, "free block %d is a chunk block or listed twice", id);
    used[id] = 2;
  }

  const int bs = kBlock;
  int row = 0, lb = 0, pv = 0;
  for (int b = 0; b < batch; ++b) {
    const epic_link_request& r = reqs[b];
    plan->s_off[b] = row;
    plan->blk_off[b] = lb;
    int64_t off = 0;
    // chunk tokens
    for (int j = 0; j < r.num_chunks; ++j) {
      const int L = r.chunk_len[j];
      const int sel = selected_in_chunk(r, j);  // tokens [0, sel) of the chunk are in S
      const int32_t* cb = r.chunk_blocks + r.chunk_block_off[j];
      for (int i = 0; i * bs < L; ++i) {
        const int t0 = i * bs, len = std::min(bs, L - t0);
        plan->block_pos0[lb] = static_cast<int32_t>(off + t0);
        plan->block_len[lb] = len;
        if (t0 < sel || rerotates(r, j)) {
          const int id = free_blocks[pv];
          const bool keeps_cached = sel < t0 + len;  // some valid slot is not recomputed
          plan->priv_block[pv] = id;
          plan->priv_src[pv] = keeps_cached ? cb[i] : -1;
          plan->priv_rot[pv] = keeps_cached && rerotates(r, j) ? static_cast<int32_t>(off) : 0;
          for (int o = 0; o < bs; ++o) {
            const int t = t0 + o;
            int32_t rr = -1;
            if (t < sel) {
              rr = row++;
              plan->s_pos[rr] = static_cast<int32_t>(off + t);
              plan->s_req[rr] = b;
              plan->s_slot[rr] = id * bs + o;
            }
            plan->priv_rows[int64_t(pv) * bs + o] = rr;
          }
          plan->linked_blocks[lb] = id;
          ++pv;
        } else {
          plan->linked_blocks[lb] = cb[i];
        }
        ++lb;
      }
      off += L;
    }
    // suffix tokens: all new, all in S
    for (int t0 = 0; t0 < r.suffix_len; t0 += bs) {
      const int len = std::min(bs, r.suffix_len - t0);
      const int id = free_blocks[pv];
      plan->block_pos0[lb] = static_cast<int32_t>(off + t0);
      plan->block_len[lb] = len;
      plan->linked_blocks[lb] = id;
      plan->priv_block[pv] = id;
      plan->priv_src[pv] = -1;
      plan->priv_rot[pv] = 0;
      for (int o = 0; o < bs; ++o) {
        int32_t rr = -1;
        if (o < len) {
          rr = row++;
          plan->s_pos[rr] = static_cast<int32_t>(off + t0 + o);
          plan->s_req[rr] = b;
          plan->s_slot[rr] = id * bs + o;
        }
        plan->priv_rows[int64_t(pv) * bs + o] = rr;
      }
      ++pv;
      ++lb;
    }
  }
  plan->s_off[batch] = row;
  plan->blk_off[batch] = lb;
  if (row != chk.n_s || lb != chk.n_linked_blocks || pv != chk.n_private)
    return fail(EPIC_ERR_INVALID_ARG, "internal planner inconsistency");

  return write_work(tiles, split, chk, plan);
}

// ---------------------------------------------------------------- decode

namespace {

// One request of a decode plan: its blocks in the previous plan, its length there,
// the free slots of its last block when that block may take the new tokens, and
// the new blocks it needs.
struct DecodeReq {
  int a = 0, e = 0;        // linked blocks [a, e) of the previous plan
  int64_t n = 0;           // tokens linked so far
  int t = 0;               // new tokens
  int room = 0;            // new tokens that go into the last block
  int extra = 0;           // new blocks
};

// ---- Decode over shared chunk caches.  Requests that link the same cached blocks each
// read them for the sake of a few rows.  Where that repeats enough, the plan lets one
// work item carry the rows of several requests over the blocks they have in common: the
// blocks are read once per 16-row tile instead of once per request.  Each row still
// gets one partial per item, in the slots of its own request's tile, so the combine is
// the ordinary one.
//
// Item kinds (work[7]): kItemRange as ever; kItemShared: blocks [work[1], work[2]) of one
// request's table with no causal mask, work[5] S rows listed as pairs (S row, partial * 16 +
// row within its tile); kItemList: work[2] blocks (work[1] = 0) of the tile's own request
// listed by index, with the mask.  Lists sit in extension entries from entry work[6] on:
// work[0] = -1, work[2..7] six int32 of the list.

struct SharedWork {
  std::vector<int32_t> tiles, work;        // plan arrays
  int n_partials = 0;
};

struct SharedRun {                          // blocks [i, i + n) of request b's table, and who else links them
  int b, i, n;
  std::vector<std::pair<int, int>> members; // (request, first block in its table)
};

// Longest-first makespan of items (cost each) on the slots one head gets.
double makespan(std::vector<double> cost, int slots) {
  std::sort(cost.begin(), cost.end(), std::greater<double>());
  std::vector<double> heap(static_cast<size_t>(slots), 0.0);
  double end = 0.0;
  for (const double c : cost) {
    std::pop_heap(heap.begin(), heap.end(), std::greater<double>());
    heap.back() += c;
    end = std::max(end, heap.back());
    std::push_heap(heap.begin(), heap.end(), std::greater<double>());
  }
  return end;
}

// Estimated us of a decode step, over shared items and with every request reading its own
// blocks, fitted to 220 random batches of which a quarter of the block reads or more could be
// shared (2-32 requests of 1-64 chunks of 33-2048 tokens; deviation 10% rms).  The reads are what
// sharing saves.  It costs launch slots for more and shorter items and their list entries, and
// partials: a row of 30 chunks of 100 tokens has one per chunk where its own blocks need two or three.
// Sharing whenever a quarter of the reads were saved made 58 of the 220 slower: 25 requests of 34 x
// 59 tokens from 102 chunks, 32/4 heads of 128, 22.8 -> 43.6 us (us on the GPU); 10 of 30 x 137 from 120,
// 16/8 heads, 31.3 -> 34.2; 4 of 14 x 396 from 14, 14.8 -> 18.2.  Shared where that is 10% shorter by these
// estimates: 119 of the 220, none slower, all together 1.303 times as fast as plain (sharing every
// one 1.276, the faster of the two 1.327); at 5% shorter 131, one slower by 4%, 1.309.
struct ShareCost {
  double blk_mb, row_mb;                                    // a block's K and V, a partial row, of all heads
  int hkv, dim;
  double plain(int64_t blocks) const { return 11.05 + 0.118 * double(blocks) * blk_mb; }
  double shared(int64_t blocks, double makespan, int64_t entries, int64_t part_rows) const {
    return 9.84 + 0.297 * makespan * dim / 128 + 0.107 * double(blocks) * blk_mb +
           0.818 * double(entries) * hkv / kShapeTiny.slots + 1.01 * double(part_rows) * row_mb;
  }
  bool pays(double shared_us, int64_t total) const { return shared_us <= 0.9 * plain(total); }
  // partial rows past which sharing cannot pay, at least `blocks` read
  int64_t most_parts(int64_t blocks, int64_t total) const {
    return static_cast<int64_t>(std::max(0.0, (0.9 * plain(total) - shared(blocks, 0.0, 0, 0)) / (1.01 * row_mb)));
  }
};

// Work items over shared blocks for 16-row tiles; false where sharing does not pay.
// A block is shared if several requests link it with the same valid length, none twice,
// and all of it precedes their new rows (so it needs no causal mask).
// A plan is built for every token, so each refusal comes as soon as its reason is known
// (requests x chunks x tokens, both planner calls: 400 x 8 x 256 of 3000 chunks, nothing to
// save, 1.7 ms against 5.5 with the work list built first; 300 x 64 x 20 of 200 chunks, over
// the partials' limit, 1.0 against 12).
bool shared_decode(const epic_plan_sizes* ps, const epic_plan* prev, const std::vector<DecodeReq>& dr,
                   const epic_attn_cfg* cfg, SharedWork* out) {
  const int G = cfg->num_q_heads / cfg->num_kv_heads, R = kTileRowsTiny / G;
  const int batch = static_cast<int>(dr.size());
  if (R < 2) return false;
  // not for requests of under 1024 tokens, whose items are too short to repay the combine
  int64_t total = 0, n_rows = 0;
  for (const DecodeReq& d : dr) {
    if (d.t == 0) continue;
    total += d.e - d.a + d.extra;
    ++n_rows;
  }
  if (total < 64 * n_rows) return false;
  // a caller with the fixed scratch array must not lose a plan that fitted it: most partials
  const int64_t max_parts = (int64_t(EPIC_NOALLOC_SCRATCH_BYTES) / ((cfg->head_dim + 1) * 4) - 64) /
                            (int64_t(cfg->num_kv_heads) * kTileRowsTiny);
  // entry of every linked block by its physical id: the id itself where the ids are about
  // as many as the blocks, else open addressing
  struct Ref {
    uint64_t sig = 0;
    int count = 0, last = -1, len = 0, run = -1;            // run: the one that starts with this block
    bool bad = false;
  };
  int max_id = 0, min_id = 0;
  for (int i = 0; i < ps->n_linked_blocks; ++i) {
    max_id = std::max(max_id, prev->linked_blocks[i]);
    min_id = std::min(min_id, prev->linked_blocks[i]);
  }
  if (min_id < 0) return false;                             // (rejected later)
  const bool dense = max_id < 2 * int64_t(ps->n_linked_blocks);
  std::vector<int> hashed;                                  // !dense: entries of the blocks
  size_t slots_n = static_cast<size_t>(max_id) + 1;
  if (!dense) {
    slots_n = 64;
    while (slots_n < 2 * static_cast<size_t>(ps->n_linked_blocks)) slots_n *= 2;
    std::vector<int> ids(slots_n, -1);
    hashed.resize(static_cast<size_t>(ps->n_linked_blocks));
    for (int i = 0; i < ps->n_linked_blocks; ++i) {
      const int id = prev->linked_blocks[i];
      size_t at = (static_cast<uint32_t>(id) * 2654435761u) & (slots_n - 1);
      while (ids[at] >= 0 && ids[at] != id) at = (at + 1) & (slots_n - 1);
      ids[at] = id;
      hashed[i] = static_cast<int>(at);
    }
  }
  const int32_t* entry = dense ? prev->linked_blocks : hashed.data();
  auto frozen = [&](int b) { return dr[b].e - dr[b].a - (dr[b].room > 0 ? 1 : 0); };   // blocks that take no new row
  // Not where fewer than a quarter of the block reads are saved: counted exactly below, here
  // at most (R rows share a read; R divides 256, so the counts may wrap).
  std::vector<uint8_t> count(slots_n, 0);
  int64_t saved = 0;
  for (int b = 0; b < batch; ++b) {
    if (dr[b].t == 0) continue;
    const int32_t* at = entry + dr[b].a;
    for (int i = 0, n = frozen(b); i < n; ++i) saved += (count[at[i]]++ & (R - 1)) != 0;
  }
  const ShareCost us{cfg->num_kv_heads * 16.0 * cfg->head_dim * 4e-6, double(cfg->num_q_heads) * cfg->head_dim * 4e-6,
                     cfg->num_kv_heads, cfg->head_dim};
  if ((total - saved) * 4 > total * 3 || !us.pays(us.shared(total - saved, 0.0, 0, 0), total)) return false;
  std::vector<Ref> ref(slots_n);
  for (int b = 0; b < batch; ++b) {
    if (dr[b].t == 0) continue;
    uint64_t h = (uint64_t(b) + 1) * 0x9E3779B97F4A7C15ull;
    h = (h ^ (h >> 29)) * 0xBF58476D1CE4E5B9ull;
    const int32_t *at = entry + dr[b].a, *lens = prev->block_len + dr[b].a;
    for (int i = 0, n = frozen(b); i < n; ++i) {
      Ref& x = ref[at[i]];
      x.bad = x.bad || x.last == b || (x.count > 0 && x.len != lens[i]);
      x.sig += h;
      x.last = b;
      x.len = lens[i];
      ++x.count;
    }
  }
  auto sig_of = [&](int b, int i) {
    const Ref& x = ref[entry[dr[b].a + i]];
    return x.count > 1 && !x.bad ? x.sig : uint64_t(0);
  };
  // runs of blocks with the same set of requests; a run of one request is its own
  std::vector<SharedRun> runs;
  std::vector<std::vector<std::pair<int, int>>> own(batch);       // [i0, i1) of each request, unshared
  auto add_own = [&](int b, int i, int n) {
    if (!own[b].empty() && own[b].back().second == i) own[b].back().second = i + n;
    else own[b].emplace_back(i, i + n);
  };
  int64_t parts_least = n_rows;             // a partial per member of a run, and one of a request's own blocks
  const int64_t parts_limit = std::min(max_parts, us.most_parts(total - saved, total));
  for (int b = 0; b < batch; ++b) {
    if (dr[b].t == 0) continue;
    const int fz = frozen(b), nb = dr[b].e - dr[b].a + dr[b].extra;
    uint64_t sig = 0 < fz ? sig_of(b, 0) : 0;
    for (int i = 0; i < nb;) {
      uint64_t next = 0;
      int j = i + 1;
      while (j < nb && (next = j < fz ? sig_of(b, j) : 0) == sig) ++j;
      if (sig == 0) {
        add_own(b, i, j - i);
      } else {
        const int32_t* ids = prev->linked_blocks + dr[b].a + i;
        int& r = ref[entry[dr[b].a + i]].run;
        if (r < 0) {
          r = static_cast<int>(runs.size());
          runs.push_back(SharedRun{b, i, j - i, {{b, i}}});
          ++parts_least;
        } else if (runs[r].n == j - i &&
                   std::equal(ids, ids + (j - i), prev->linked_blocks + dr[runs[r].b].a + runs[r].i)) {
          runs[r].members.emplace_back(b, i);
          ++parts_least;
        } else {
          add_own(b, i, j - i);                           // the same blocks in another order
        }
      }
      i = j;
      sig = next;
    }
    if (parts_least > parts_limit) return false;
  }
  // groups of at most R rows over a run, about equal
  struct Group {
    int run, m0, m1;                                       // members [m0, m1) of the run
  };
  std::vector<Group> groups;
  int64_t read = 0;
  for (size_t r = 0; r < runs.size(); ++r) {
    const auto& members = runs[r].members;
    int rows = 0;
    for (const auto& m : members) rows += dr[m.first].t;
    const int parts = cdiv(rows, R), each = cdiv(rows, parts);
    int fill = 0, m0 = 0;
    for (int k = 0; k < static_cast<int>(members.size()); ++k) {
      const int t = dr[members[k].first].t;
      if (fill > 0 && (fill + t > R || fill >= each)) {
        groups.push_back(Group{static_cast<int>(r), m0, k});
        m0 = k;
        fill = 0;
      }
      fill += t;
    }
    groups.push_back(Group{static_cast<int>(r), m0, static_cast<int>(members.size())});
  }
  for (const Group& g : groups) read += runs[g.run].n;
  for (const auto& o : own)
    for (const auto& x : o) read += x.second - x.first;
  if (read * 4 > total * 3) return false;
  // Unshared blocks: ranges of at least kListBelow blocks as items of their own, the
  // rest of a request's listed together.
  constexpr int kListBelow = 48, kListMost = 96;
  struct Item {
    int kind, group, b, i0, i1;                           // blocks [i0, i1) of b's table, or of its list
    int parts;
  };
  std::vector<std::vector<int>> lists(batch);
  std::vector<Item> whole;
  for (size_t k = 0; k < groups.size(); ++k) {
    const SharedRun& r = runs[groups[k].run];
    whole.push_back(Item{kItemShared, static_cast<int>(k), r.b, r.i, r.i + r.n, groups[k].m1 - groups[k].m0});
  }
  for (int b = 0; b < batch; ++b) {
    for (const auto& x : own[b]) {
      if (x.second - x.first >= kListBelow) whole.push_back(Item{kItemRange, -1, b, x.first, x.second, 1});
      else
        for (int i = x.first; i < x.second; ++i) lists[b].push_back(i);
    }
    for (int i = 0; i < static_cast<int>(lists[b].size()); i += kListMost)
      whole.push_back(Item{kItemList, -1, b, i, std::min<int>(i + kListMost, static_cast<int>(lists[b].size())), 1});
  }
  // split: pieces of at most `split` blocks, by the estimated launch as in split_blocks, among
  // those whose partials fit; whole where even whole items make more rounds than balancing needs
  const int slots = std::max(1, kShapeTiny.slots / cfg->num_kv_heads);
  auto pieces = [](const Item& it, int split) { return cdiv(it.i1 - it.i0, split); };
  int longest = 16;
  int64_t whole_parts = 0;
  for (const Item& it : whole) {
    longest = std::max(longest, it.i1 - it.i0);
    whole_parts += it.parts;
  }
  if (whole_parts > max_parts) return false;
  int best = longest;
  double best_time = 0.0;
  std::vector<double> cost;
  for (const int parts : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64}) {
    const int split = std::max(16, cdiv(longest, parts));
    int64_t n_parts = 0;
    cost.clear();
    for (const Item& it : whole) {
      const int p = pieces(it, split);
      n_parts += int64_t(p) * it.parts;
      cost.insert(cost.end(), p, cdiv(cdiv(it.i1 - it.i0, p), kKvTileBlocks) + kShapeTiny.item_overhead +
                                     kShapeTiny.partial_cost * (it.kind == kItemShared ? 1 + 0.25 * it.parts : 1));
    }
    if (n_parts > max_parts || cost.size() > 16u * static_cast<size_t>(slots)) break;
    const double t = makespan(cost, slots);
    if (parts == 1 || t < best_time * 0.97) best_time = t, best = split;
    if (split == 16) break;
  }
  int64_t entries = 0, part_rows = 0;
  for (const Item& it : whole) {
    const int p = pieces(it, best);
    int rows = dr[it.b].t, listed = it.kind == kItemList ? cdiv(it.i1 - it.i0, p) : 0;
    if (it.kind == kItemShared) {
      rows = 0;
      for (int k = groups[it.group].m0; k < groups[it.group].m1; ++k) rows += dr[runs[groups[it.group].run].members[k].first].t;
      listed = 2 * rows;
    }
    entries += int64_t(p) * (1 + cdiv(listed, kExtInts));
    part_rows += int64_t(p) * rows;
  }
  if (!us.pays(us.shared(read, best_time, entries, part_rows), total)) return false;
  // tiles: one per request with rows; partials of a tile are consecutive
  std::vector<int> tile_of(batch, -1), n_part(batch, 0), row0(batch, 0), base(batch, 0);
  int n_tiles = 0, rows = 0, lb = 0;
  for (int b = 0; b < batch; ++b) {
    row0[b] = rows;
    base[b] = lb;
    rows += dr[b].t;
    lb += dr[b].e - dr[b].a + dr[b].extra;
    if (dr[b].t > 0) tile_of[b] = n_tiles++;
  }
  std::vector<Item> items;
  for (const Item& it : whole) {
    const int p = pieces(it, best), n = it.i1 - it.i0;
    for (int k = 0; k < p; ++k)
      items.push_back(Item{it.kind, it.group, it.b, it.i0 + int(int64_t(n) * k / p), it.i0 + int(int64_t(n) * (k + 1) / p),
                           it.parts});
  }
  // longest first; equal lengths keep their order, so the groups of one run stay together
  std::stable_sort(items.begin(), items.end(), [](const Item& x, const Item& y) { return x.i1 - x.i0 > y.i1 - y.i0; });
  for (const Item& it : items) {
    if (it.kind == kItemShared)
      for (int k = groups[it.group].m0; k < groups[it.group].m1; ++k) ++n_part[runs[groups[it.group].run].members[k].first];
    else
      ++n_part[it.b];
  }
  int part = 0;
  std::vector<int> next(batch, 0);
  out->tiles.clear();
  for (int b = 0; b < batch; ++b) {
    if (tile_of[b] < 0) continue;
    const bool split_tile = n_part[b] > 1;
    out->tiles.insert(out->tiles.end(), {row0[b], dr[b].t, split_tile ? part : -1, n_part[b]});
    next[b] = split_tile ? part : -1;
    if (split_tile) part += n_part[b];
  }
  out->n_partials = part;
  auto take = [&](int b) { return next[b] < 0 ? -1 : next[b]++; };
  const int n_items = static_cast<int>(items.size());
  std::vector<int32_t> ext;
  auto extend = [&](const std::vector<int32_t>& list) {   // returns the first extension entry's index
    const int at = n_items + static_cast<int>(ext.size()) / kWorkInts;
    for (size_t i = 0; i < list.size(); i += kExtInts) {
      ext.insert(ext.end(), {-1, 0});
      for (size_t j = i; j < i + kExtInts; ++j) ext.push_back(j < list.size() ? list[j] : 0);
    }
    return at;
  };
  out->work.clear();
  for (const Item& it : items) {
    int32_t wk[kWorkInts] = {tile_of[it.b], base[it.b] + it.i0, base[it.b] + it.i1, -1, 0, 0, 0, it.kind};
    std::vector<int32_t> list;
    if (it.kind == kItemShared) {
      for (int k = groups[it.group].m0; k < groups[it.group].m1; ++k) {
        const auto& m = runs[groups[it.group].run].members[k];
        const int p = take(m.first);
        for (int t = 0; t < dr[m.first].t; ++t) {
          list.push_back(row0[m.first] + t);
          list.push_back(p < 0 ? -1 : p * kTileRowsTiny + t);
        }
      }
      wk[5] = static_cast<int32_t>(list.size()) / 2;
      wk[6] = extend(list);
    } else {
      wk[3] = take(it.b);
      if (it.kind == kItemList) {
        for (int i = it.i0; i < it.i1; ++i) list.push_back(base[it.b] + lists[it.b][i]);
        wk[1] = 0;
        wk[2] = wk[5] = static_cast<int32_t>(list.size());
        wk[6] = extend(list);
      }
    }
    out->work.insert(out->work.end(), wk, wk + kWorkInts);
  }
  out->work.insert(out->work.end(), ext.begin(), ext.end());
  return true;
}

epic_status decode_shape(const epic_plan_sizes* ps, const epic_plan* prev, const int32_t* new_tokens,
                         const epic_attn_cfg* cfg, int32_t n_free, epic_plan_sizes* out,
                         std::vector<Tile>* tiles_out, int* split_out, std::vector<DecodeReq>* dr_out,
                         SharedWork* shared) {
  EPIC_CHECK_ARG(ps && prev && out, "NULL previous plan, sizes or output");
  EPIC_CHECK_ARG(n_free >= 0, "n_free %d < 0", n_free);
  epic_status st = validate_attn_cfg(cfg);
  if (st != EPIC_OK) return st;
  const int batch = ps->batch;
  EPIC_CHECK_ARG(batch == 0 || (new_tokens && prev->blk_off && prev->linked_blocks && prev->block_pos0 &&
                                prev->block_len),
                 "NULL new_tokens or previous plan array");
  EPIC_CHECK_ARG(ps->n_private == 0 || prev->priv_block, "previous plan has no private block list");
  // blocks the previous step wrote: only those may take further tokens
  std::vector<int32_t> written(prev->priv_block, prev->priv_block + ps->n_private);
  std::sort(written.begin(), written.end());
  std::vector<DecodeReq>& dr = *dr_out;
  dr.assign(static_cast<size_t>(batch), DecodeReq{});
  int64_t n_s = 0, n_lb = 0, n_priv = 0, n_take = 0, max_pos = 0;
  for (int b = 0; b < batch; ++b) {
    DecodeReq& d = dr[b];
    d.a = prev->blk_off[b];
    d.e = prev->blk_off[b + 1];
    EPIC_CHECK_ARG(0 <= d.a && d.a <= d.e && d.e <= ps->n_linked_blocks, "previous plan: bad blk_off at %d", b);
    d.t = new_tokens[b];
    EPIC_CHECK_ARG(d.t >= 0, "request %d: %d new tokens", b, d.t);
    if (d.e > d.a) {
      const int last = d.e - 1, len = prev->block_len[last];
      d.n = int64_t(prev->block_pos0[last]) + len;
      if (len < kBlock && std::binary_search(written.begin(), written.end(), prev->linked_blocks[last]))
        d.room = std::min(d.t, kBlock - len);
    }
    d.extra = cdiv(d.t - d.room, kBlock);
    EPIC_CHECK_ARG(d.n + d.t < (int64_t(1) << 30), "request %d: too many tokens", b);
    n_s += d.t;
    n_lb += (d.e - d.a) + d.extra;
    n_priv += (d.room > 0 ? 1 : 0) + d.extra;
    n_take += d.extra;
    max_pos = std::max<int64_t>(max_pos, d.n + d.t);
  }
  EPIC_CHECK_ARG(n_s < (int64_t(1) << 30) && n_lb < (int64_t(1) << 30), "batch too large");
  if (n_take > n_free)
    return fail(EPIC_ERR_NO_PRIVATE_BLOCKS, "plan needs %lld new blocks, %d free", (long long)n_take, n_free);
  epic_plan_sizes s{};
  s.batch = batch;
  // plans for the decode kernel, one tile per request: perhaps over shared blocks
  const int G = cfg->num_q_heads / cfg->num_kv_heads;
  bool tiny = (cfg->tile_rows == 0 || cfg->tile_rows == kTileRowsTiny) && cfg->kv_split_blocks == 0 && G <= kTileRowsTiny;
  int n_tiles = 0;
  for (const DecodeReq& d : dr) {
    tiny = tiny && d.t <= kTileRowsTiny / G;
    n_tiles += d.t > 0;
  }
  if (tiny && n_tiles > 1 && shared_decode(ps, prev, dr, cfg, shared)) {
    s.tile_rows = kTileRowsTiny;
    s.n_tiles = n_tiles;
    s.n_work = static_cast<int32_t>(shared->work.size()) / kWorkInts;
    s.n_partials = shared->n_partials;
  } else {
    std::vector<ReqRows> rr(static_cast<size_t>(batch));
    for (int b = 0; b < batch; ++b) {
      const DecodeReq& d = dr[b];
      rr[b].p0.reserve(static_cast<size_t>(d.e - d.a) + d.extra);
      rr[b].p0.assign(prev->block_pos0 + d.a, prev->block_pos0 + d.e);
      for (int i = 0; i < d.extra; ++i) rr[b].p0.push_back(static_cast<int32_t>(d.n + d.room + int64_t(i) * kBlock));
      for (int i = 0; i < d.t; ++i) rr[b].pos.push_back(static_cast<int32_t>(d.n + i));
    }
    choose_tiles(rr, cfg, &s, tiles_out, split_out);
  }
  s.n_s = static_cast<int32_t>(n_s);
  s.n_linked_blocks = static_cast<int32_t>(n_lb);
  s.n_private = static_cast<int32_t>(n_priv);
  s.max_pos = static_cast<int32_t>(max_pos);
  finish_sizes(&s);
  *out = s;
  return EPIC_OK;
}

}  // namespace

extern "C" epic_status epic_plan_decode_sizes(const epic_plan_sizes* prev_sizes, const epic_plan* prev,
                                              const int32_t* new_tokens, const epic_attn_cfg* cfg, int32_t n_free,
                                              epic_plan_sizes* out) {
  clear_error();
  std::vector<Tile> tiles;
  std::vector<DecodeReq> dr;
  SharedWork shared;
  int split = 0;
  return decode_shape(prev_sizes, prev, new_tokens, cfg, n_free, out, &tiles, &split, &dr, &shared);
}

extern "C" epic_status epic_plan_decode(const epic_plan_sizes* prev_sizes, const epic_plan* prev,
                                        const int32_t* new_tokens, const epic_attn_cfg* cfg,
                                        const int32_t* free_blocks, int32_t n_free, int32_t num_blocks,
                                        const epic_plan_sizes* sizes, epic_plan* plan) {
  clear_error();
  epic_plan_sizes chk;
  std::vector<Tile> tiles;
  std::vector<DecodeReq> dr;
  SharedWork shared;
  int split = 0;
  epic_status st = decode_shape(prev_sizes, prev, new_tokens, cfg, n_free, &chk, &tiles, &split, &dr, &shared);
  if (st != EPIC_OK) return st;
  EPIC_CHECK_ARG(sizes && plan, "NULL sizes or plan");
  EPIC_CHECK_ARG(std::memcmp(&chk, sizes, sizeof(chk)) == 0, "sizes do not match this previous plan");
  EPIC_CHECK_ARG(num_blocks > 0, "num_blocks %d <= 0", num_blocks);
  int64_t n_take = 0;
  for (const DecodeReq& d : dr) n_take += d.extra;
  EPIC_CHECK_ARG(n_take == 0 || free_blocks != nullptr, "free_blocks is NULL");
  // free blocks: in range, distinct, not linked by the previous plan
  std::vector<uint8_t> used(static_cast<size_t>(num_blocks), 0);
  for (int i = 0; i < prev_sizes->n_linked_blocks; ++i) {
    const int id = prev->linked_blocks[i];
    EPIC_CHECK_ARG(id >= 0 && id < num_blocks, "previous plan: block id %d out of range [0, %d)", id, num_blocks);
    used[id] = 1;
  }
  for (int64_t i = 0; i < n_take; ++i) {
    const int id = free_blocks[i];
    EPIC_CHECK_ARG(id >= 0 && id < num_blocks, "free block id %d out of range [0, %d)", id, num_blocks);
    EPIC_CHECK_ARG(used[id] == 0, "free block %d is already linked or listed twice", id);
    used[id] = 2;
  }
  const int bs = kBlock;
  int row = 0, lb = 0, pv = 0, fl = 0;
  auto add_row = [&](int b, int64_t pos, int id, int o) {
    plan->s_pos[row] = static_cast<int32_t>(pos);
    plan->s_req[row] = b;
    plan->s_slot[row] = id * bs + o;
    return row++;
  };
  for (int b = 0; b < chk.batch; ++b) {
    const DecodeReq& d = dr[b];
    plan->s_off[b] = row;
    plan->blk_off[b] = lb;
    for (int i = d.a; i < d.e; ++i, ++lb) {
      plan->linked_blocks[lb] = prev->linked_blocks[i];
      plan->block_pos0[lb] = prev->block_pos0[i];
      plan->block_len[lb] = prev->block_len[i] + (i == d.e - 1 ? d.room : 0);
    }
    int64_t pos = d.n;
    if (d.room > 0) {                          // the last block takes the first new tokens
      const int id = prev->linked_blocks[d.e - 1], len = prev->block_len[d.e - 1];
      plan->priv_block[pv] = id;
      plan->priv_src[pv] = id;                 // its earlier tokens stay: copied onto themselves
      plan->priv_rot[pv] = 0;
      for (int o = 0; o < bs; ++o)
        plan->priv_rows[int64_t(pv) * bs + o] = (o >= len && o < len + d.room) ? add_row(b, pos++, id, o) : -1;
      ++pv;
    }
    for (int i = 0; i < d.extra; ++i, ++lb, ++pv) {
      const int id = free_blocks[fl++];
      const int len = static_cast<int>(std::min<int64_t>(bs, d.n + d.t - pos));
      plan->linked_blocks[lb] = id;
      plan->block_pos0[lb] = static_cast<int32_t>(pos);
      plan->block_len[lb] = len;
      plan->priv_block[pv] = id;
      plan->priv_src[pv] = -1;
      plan->priv_rot[pv] = 0;
      for (int o = 0; o < bs; ++o) plan->priv_rows[int64_t(pv) * bs + o] = o < len ? add_row(b, pos++, id, o) : -1;
    }
  }
  plan->s_off[chk.batch] = row;
  plan->blk_off[chk.batch] = lb;
  if (row != chk.n_s || lb != chk.n_linked_blocks || pv != chk.n_private || fl != n_take)
    return fail(EPIC_ERR_INVALID_ARG, "internal planner inconsistency (decode)");
  if (!shared.work.empty()) {
    std::copy(shared.tiles.begin(), shared.tiles.end(), plan->tiles);
    std::copy(shared.work.begin(), shared.work.end(), plan->work);
    return EPIC_OK;
  }
  return write_work(tiles, split, chk, plan);
}

// ---------------------------------------------------------------- compile

namespace {

// The compile step (Sec. 2.2) prefills every chunk alone; LegoLink-0 (Sec. 5.4)
// first prepends n_dummy dummy tokens to each chunk and afterwards drops their
// K/V.  Each chunk is one request of the plan: S = its n_dummy + L tokens at
// positions 0 .. n_dummy + L - 1, the dummies first.  Without dummies the
// chunk's own blocks are its linked (attention) blocks.  With dummies the
// attention reads n_dummy + L tokens from staging blocks taken from the free
// list, and the chunk's blocks are further private blocks outside the linked
// table that receive chunk token t at slot t (rows n_dummy + t).
epic_status compile_shape(const epic_compile_batch* cb, const epic_attn_cfg* cfg, int32_t n_free,
                          epic_plan_sizes* out, std::vector<Tile>* tiles_out, int* split_out,
                          int64_t* n_staging) {
  EPIC_CHECK_ARG(cb && out, "NULL compile batch or output sizes");
  EPIC_CHECK_ARG(n_free >= 0, "n_free %d < 0", n_free);
  epic_status st = validate_attn_cfg(cfg);
  if (st != EPIC_OK) return st;
  const int n = cb->num_chunks;
  EPIC_CHECK_ARG(n >= 0, "num_chunks %d < 0", n);
  EPIC_CHECK_ARG(cb->n_dummy >= 0 && cb->n_dummy <= (1 << 20), "n_dummy %d outside [0, 2^20]", cb->n_dummy);
  if (n > 0) {
    EPIC_CHECK_ARG(cb->chunk_len && cb->chunk_block_off && cb->chunk_blocks, "chunk arrays are NULL");
    EPIC_CHECK_ARG(cb->chunk_block_off[0] == 0, "chunk_block_off[0] != 0");
  }
  const int nd = cb->n_dummy;
  std::vector<ReqRows> rr(static_cast<size_t>(n));
  int64_t n_s = 0, n_lb = 0, n_priv = 0, stage = 0, max_pos = 0;
  for (int j = 0; j < n; ++j) {
    const int L = cb->chunk_len[j];
    EPIC_CHECK_ARG(L >= 1, "chunk %d: length %d < 1", j, L);
    EPIC_CHECK_ARG(int64_t(L) + nd < (int64_t(1) << 30), "chunk %d: too many tokens", j);
    const int nb = cb->chunk_block_off[j + 1] - cb->chunk_block_off[j];
    EPIC_CHECK_ARG(nb == cdiv(L, kBlock), "chunk %d: %d blocks given, %d needed", j, nb, cdiv(L, kBlock));
    const int total = nd + L, lb = cdiv(total, kBlock);
    for (int p = 0; p < total; ++p) rr[j].pos.push_back(p);
    for (int i = 0; i < lb; ++i) rr[j].p0.push_back(i * kBlock);
    n_s += total;
    n_lb += lb;
    n_priv += nb + (nd > 0 ? lb : 0);
    stage += nd > 0 ? lb : 0;
    max_pos = std::max<int64_t>(max_pos, total);
  }
  EPIC_CHECK_ARG(n_s < (int64_t(1) << 30) && n_priv < (int64_t(1) << 30), "batch too large");
  if (stage > n_free)
    return fail(EPIC_ERR_NO_PRIVATE_BLOCKS, "plan needs %lld staging blocks, %d free", (long long)stage, n_free);
  epic_plan_sizes s{};
  s.batch = n;
  choose_tiles(rr, cfg, &s, tiles_out, split_out);
  s.n_s = static_cast<int32_t>(n_s);
  s.n_linked_blocks = static_cast<int32_t>(n_lb);
  s.n_private = static_cast<int32_t>(n_priv);
  s.max_pos = static_cast<int32_t>(max_pos);
  finish_sizes(&s);
  *out = s;
  *n_staging = stage;
  return EPIC_OK;
}

}  // namespace

extern "C" epic_status epic_plan_compile_sizes(const epic_compile_batch* batch, const epic_attn_cfg* cfg,
                                               int32_t n_free, epic_plan_sizes* out) {
  clear_error();
  std::vector<Tile> tiles;
  int split = 0;
  int64_t stage = 0;
  return compile_shape(batch, cfg, n_free, out, &tiles, &split, &stage);
}

extern "C" epic_status epic_plan_compile(const epic_compile_batch* batch, const epic_attn_cfg* cfg,
                                         const int32_t* free_blocks, int32_t n_free, int32_t num_blocks,
                                         const epic_plan_sizes* sizes, epic_plan* plan) {
  clear_error();
  epic_plan_sizes chk;
  std::vector<Tile> tiles;
  int split = 0;
  int64_t stage = 0;
  epic_status st = compile_shape(batch, cfg, n_free, &chk, &tiles, &split, &stage);
  if (st != EPIC_OK) return st;
  EPIC_CHECK_ARG(sizes && plan, "NULL sizes or plan");
  EPIC_CHECK_ARG(std::memcmp(&chk, sizes, sizeof(chk)) == 0, "sizes do not match this compile batch");
  EPIC_CHECK_ARG(num_blocks > 0, "num_blocks %d <= 0", num_blocks);
  EPIC_CHECK_ARG(stage == 0 || free_blocks != nullptr, "free_blocks is NULL");
  const int n = batch->num_chunks, nd = batch->n_dummy, bs = kBlock;
  // every block is written: chunk blocks and staging blocks in range and all distinct
  std::vector<uint8_t> used(static_cast<size_t>(num_blocks), 0);
  const int n_chunk_blocks = n > 0 ? batch->chunk_block_off[n] : 0;
  for (int i = 0; i < n_chunk_blocks; ++i) {
    const int id = batch->chunk_blocks[i];
    EPIC_CHECK_ARG(id >= 0 && id < num_blocks, "chunk block id %d out of range [0, %d)", id, num_blocks);
    EPIC_CHECK_ARG(used[id] == 0, "chunk block %d is listed twice", id);
    used[id] = 1;
  }
  for (int64_t i = 0; i < stage; ++i) {
    const int id = free_blocks[i];
    EPIC_CHECK_ARG(id >= 0 && id < num_blocks, "free block id %d out of range [0, %d)", id, num_blocks);
    EPIC_CHECK_ARG(used[id] == 0, "free block %d is a chunk block or listed twice", id);
    used[id] = 2;
  }
  int row = 0, lb = 0, pv = 0, fl = 0;
  for (int j = 0; j < n; ++j) {
    const int L = batch->chunk_len[j], total = nd + L;
    const int32_t* cbk = batch->chunk_blocks + batch->chunk_block_off[j];
    const int row0 = row;
    plan->s_off[j] = row;
    plan->blk_off[j] = lb;
    // linked (attention) blocks: the chunk's own blocks, or staging blocks with dummies
    for (int i = 0; i * bs < total; ++i, ++lb, ++pv) {
      const int id = nd > 0 ? free_blocks[fl++] : cbk[i];
      const int len = std::min(bs, total - i * bs);
      plan->linked_blocks[lb] = id;
      plan->block_pos0[lb] = i * bs;
      plan->block_len[lb] = len;
      plan->priv_block[pv] = id;
      plan->priv_src[pv] = -1;
      plan->priv_rot[pv] = 0;
      for (int o = 0; o < bs; ++o) {
        int32_t r = -1;
        if (o < len) {
          r = row++;
          plan->s_pos[r] = i * bs + o;
          plan->s_req[r] = j;
          plan->s_slot[r] = id * bs + o;
        }
        plan->priv_rows[int64_t(pv) * bs + o] = r;
      }
    }
    // the chunk's cache without the dummies: chunk token t (row row0 + nd + t) at slot t
    if (nd > 0) {
      for (int i = 0; i * bs < L; ++i, ++pv) {
        plan->priv_block[pv] = cbk[i];
        plan->priv_src[pv] = -1;
        plan->priv_rot[pv] = 0;
        for (int o = 0; o < bs; ++o) {
          const int t = i * bs + o;
          plan->priv_rows[int64_t(pv) * bs + o] = t < L ? row0 + nd + t : -1;
        }
      }
    }
  }
  plan->s_off[n] = row;
  plan->blk_off[n] = lb;
  if (row != chk.n_s || lb != chk.n_linked_blocks || pv != chk.n_private || fl != stage)
    return fail(EPIC_ERR_INVALID_ARG, "internal planner inconsistency (compile)");
  return write_work(tiles, split, chk, plan);
}
