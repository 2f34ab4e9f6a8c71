// Host-side integer planner of libmpic (no GPU calls in this file).
//
// Selection rule, Sec. 4.2: the recompute set is every text token plus the first k
// tokens of every image chunk.  Linking, Fig. 7 step 2 / Sec. 4.1: rows of the
// recompute set are replaced by freshly generated K/V (text slots are only
// placeholders before that), every other row comes from the stored chunk cache.
// The planner turns a batch of segment lists into range-wise filled index maps,
// the rotary tables of the chunk shifts and the launch order of attention tiles.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <new>
#include <numeric>

#include "common.h"

namespace mpic {

int fail(mpic_ctx* ctx, int code, const std::string& msg) {
  if (ctx) ctx->last_error = msg;
  return code;
}

int fail_hip(mpic_ctx* ctx, hipError_t e, const char* what) {
  if (ctx) ctx->last_error = std::string(what) + ": " + hipGetErrorString(e);
  return MPIC_ERR_HIP;
}

namespace {

constexpr int kXcds = 8;  // L2 domains of the chip; workgroup i is dispatched to domain i % 8
constexpr int kComputeUnits = 256;

// Cut the recompute set of every request into attention tiles and order them for launch.
//
// A tile is a range of "flattened rows" of one (request, kv head): all G query heads
// of a fresh row are adjacent, fresh rows follow each other in position order.  Tiles
// are cut every kAttnTileRows rows regardless of run boundaries: the kernel masks per
// row and every wavefront stops at the last key its own rows can see, so a tile that
// straddles two runs costs no more than its parts while full tiles keep the K/V
// stream per flop low.
//
// A launch ends when its last tile does, and a tile's work grows with the position of its rows.
// Where the longest tile is more than half of a compute unit's share, tiles are also cut along the
// keys: every piece visits a range of 64-key blocks and leaves a partial result (normalised output
// + log-sum-exp) that a merge kernel combines.  How long the pieces are is decided by list
// scheduling of a few candidates (choose_cut below).
//
// Launch order: tiles that read the same K/V (same request and kv head) are dealt to the
// same L2 domain, and inside a domain the longest tiles come first so the tail of the
// launch is made of short work.
void build_tiles(mpic_plan& p, int group, int n_kv_heads) {
  struct Item {
    AttnTile t;
    int64_t cost;
  };
  constexpr int64_t kBlock = 64;          // keys per block of the attention kernel
  constexpr int64_t kMinPieceBlocks = 4;
  // Fixed costs in blocks (1.3 us each with one workgroup per compute unit): of a tile, of a piece, of
  // the merge launch, and the rows of partial results that are written and read again in the time of
  // one block (11 MB, 8.5 TB/s).  Measured over three sets of 104 batches of 0.1 to 300 GFLOP against
  // pieces of one size for a whole launch that had to fit one or two rounds over the chip (attention
  // and merge, both sides in turn): 0.84, 0.85 and 0.88 of that time, 33 of the 312 batches more than
  // 3 % above it, most of them launches of less than 20 us.  With 10 blocks for a piece whatever its
  // rows and 4 for the merge launch: 0.85, 0.87 and 0.89, 45 batches; with 16 for a piece up to 22 %
  // more.  One request of 2177 rows with 87-block tiles 91 -> 70 us, 8 requests of 13K tokens 197 -> 179 us.
  constexpr int64_t kTileCost = 6, kPieceCost = 5, kMergeCost = 2, kPartRowsPerBlock = 10667;
  constexpr int64_t kUnit = 10;
  const int B = p.n_requests;
  const int n_combo = B * n_kv_heads;
  auto last_pos = [&](int b, int64_t row_end) {  // position of the last fresh row below flattened row `row_end`
    return static_cast<int64_t>(p.q_pos[p.q_off[b] + (row_end - 1) / group]);
  };
  // Tile height: full tiles unless even pieces of the smallest size would leave compute
  // units without work; then the height is halved (down to two wavefronts' worth of rows).
  int64_t tile_rows = kAttnTileRows;
  auto count_pieces = [&](int64_t h, int64_t* total_blocks) {
    int64_t n = 0, tot = 0;
    for (int b = 0; b < B; ++b) {
      const int64_t rows = static_cast<int64_t>(p.q_off[b + 1] - p.q_off[b]) * group;
      for (int64_t row = 0; row < rows; row += h) {
        const int64_t blocks = (last_pos(b, std::min(rows, row + h)) + 1 + kBlock - 1) / kBlock;
        n += (blocks + kMinPieceBlocks - 1) / kMinPieceBlocks * n_kv_heads;
        tot += blocks * n_kv_heads;
      }
    }
    if (total_blocks) *total_blocks = tot;
    return n;
  };
  while (tile_rows > 64 && count_pieces(tile_rows, nullptr) < kComputeUnits) tile_rows /= 2;
  // the tiles of one kv head
  struct RowTile {
    int b;
    int64_t row, n, n_keys, blocks;
  };
  std::vector<RowTile> row_tiles;
  int64_t total_blocks = 0, longest = 0;
  for (int b = 0; b < B; ++b) {
    const int64_t rows = static_cast<int64_t>(p.q_off[b + 1] - p.q_off[b]) * group;
    for (int64_t row = 0; row < rows; row += tile_rows) {
      const int64_t n = std::min<int64_t>(tile_rows, rows - row), n_keys = last_pos(b, row + n) + 1;
      row_tiles.push_back(RowTile{b, row, n, n_keys, (n_keys + kBlock - 1) / kBlock});
      total_blocks += row_tiles.back().blocks * n_kv_heads;
      longest = std::max(longest, row_tiles.back().blocks);
    }
  }
  const int64_t per_cu = (total_blocks + kComputeUnits - 1) / kComputeUnits;
  // How a tile of `blocks` blocks is cut: tiles longer than `cap` into even pieces, or into pieces
  // of exactly `cap` and a remainder.  Even pieces suit launches of one round, where the longest
  // piece decides; equal pieces with remainders fill the end of a launch of several.
  struct Cut {
    int64_t cap;
    bool even;
  };
  auto n_pieces = [&](int64_t blocks, const Cut& c) {
    if (blocks <= c.cap) return int64_t{1};
    if (c.even) return std::max<int64_t>(1, std::min((blocks + c.cap - 1) / c.cap, blocks / kMinPieceBlocks));
    return blocks % c.cap >= kMinPieceBlocks ? blocks / c.cap + 1 : blocks / c.cap;
  };
  auto piece_begin = [&](int64_t blocks, const Cut& c, int64_t parts, int64_t i) {
    // (a remainder shorter than the smallest piece is shared by the others)
    return c.even || blocks % c.cap < kMinPieceBlocks || i == parts ? blocks * i / parts : i * c.cap;
  };
  // How long a piece of `keys` keys of tile t (cut into `parts`) occupies a compute unit.
  auto duration = [&](const RowTile& t, int64_t keys, int64_t parts) {
    const int64_t blocks = (keys + kBlock - 1) / kBlock + (parts > 1 ? kPieceCost : kTileCost);
    return blocks * (t.n > kAttnTileRows / 2 ? kUnit : kUnit * 4 / 5);
  };
  // Predicted end of the launch, in blocks / kUnit: list scheduling, longest piece first, over the compute
  // units that one kv head has to itself.
  int64_t heads = n_kv_heads, per_head_cus = kComputeUnits;
  while (heads % 2 == 0 && per_head_cus > kComputeUnits / kXcds) heads /= 2, per_head_cus /= 2;
  std::vector<int64_t> costs, load;
  auto simulate = [&](const Cut& c, int64_t best) {
    costs.clear();
    int64_t sum = 0, part_rows = 0;
    for (const RowTile& t : row_tiles) {
      const int64_t parts = n_pieces(t.blocks, c);
      if (parts > 1) part_rows += parts * t.n * n_kv_heads;
      for (int64_t i = 0; i < parts; ++i) {
        const int64_t cost = duration(t, (piece_begin(t.blocks, c, parts, i + 1) - piece_begin(t.blocks, c, parts, i)) * kBlock, parts);
        costs.push_back(cost);  // (once for all heads)
        sum += cost * heads;
      }
    }
    const int64_t merge = part_rows > 0 ? kMergeCost * kUnit + part_rows * kUnit / kPartRowsPerBlock : 0;
    if (sum / per_head_cus + merge >= best) return best;  // cannot be better
    std::sort(costs.begin(), costs.end(), std::greater<int64_t>());
    if (costs.empty() || costs.front() + merge >= best) return best;
    load.assign(per_head_cus, 0);
    int64_t end = 0;
    for (const int64_t cost : costs)
      for (int64_t h = 0; h < heads; ++h) {
        // the lightest unit takes the piece and sinks to its place in the heap
        const int64_t now = load.front() + cost;
        size_t at = 0;
        for (size_t kid = 1; kid < load.size(); kid = 2 * at + 1) {
          if (kid + 1 < load.size() && load[kid + 1] < load[kid]) ++kid;
          if (load[kid] >= now) break;
          load[at] = load[kid];
          at = kid;
        }
        load[at] = now;
        end = std::max(end, now);
        if (end + merge >= best) return best;
      }
    return end + merge;
  };
  auto choose_cut = [&]() {
    Cut chosen{longest, true};  // uncut
    if (2 * longest <= per_cu) return chosen;
    int64_t best = simulate(chosen, INT64_MAX);
    best -= best * 3 / 100;  // a cut launch has to be worth its partial results
    // Long launches are only cut where a few tiles stand out, coarsely: finer pieces end the launch
    // up to 2 % earlier, but the linking of the next layer then no longer fits beside its end.
    const bool is_long = per_cu > 256;
    const std::vector<int64_t> percents =
        is_long ? std::vector<int64_t>{70, 60, 50, 40} : std::vector<int64_t>{100, 80, 115, 90, 65, 130, 150, 55, 180, 220, 270, 330};
    int64_t last = 0;
    for (const int64_t percent : percents) {
      const int64_t cap = std::max<int64_t>(kMinPieceBlocks, (per_cu * percent + 99) / 100);
      if (cap >= longest || cap == last) continue;
      last = cap;
      for (const bool even : {true, false}) {
        if (is_long && !even) continue;
        const int64_t m = simulate(Cut{cap, even}, best);
        if (m < best) {
          best = m;
          chosen = Cut{cap, even};
        }
      }
    }
    return chosen;
  };
  const Cut cut = choose_cut();
  // The launch: the tiles cut, dealt to the L2 domains and ordered inside each.
  struct Layout {
    std::vector<std::vector<Item>> queue;  // per L2 domain, in launch order
    std::vector<AttnMerge> merges;
    int32_t n_parts = 0;
  };
  auto by_cost = [](const Item& a, const Item& b) { return a.cost > b.cost; };
  Layout chosen;
  std::vector<std::vector<Item>> per_combo(n_combo);
  for (const RowTile& rt : row_tiles) {
    const int b = rt.b;
    const int64_t row = rt.row, n = rt.n;
    const int64_t parts = n_pieces(rt.blocks, cut);
    for (int64_t i = 0; i < parts; ++i) {
      const int64_t key0 = piece_begin(rt.blocks, cut, parts, i) * kBlock;
      const int64_t key1 = std::min<int64_t>(rt.n_keys, piece_begin(rt.blocks, cut, parts, i + 1) * kBlock);
      const int64_t cost = duration(rt, key1 - key0, parts);
      for (int g = 0; g < n_kv_heads; ++g) {
        Item it{};
        it.t.req = b;
        it.t.kv_head = g;
        it.t.row0 = static_cast<int32_t>(row);
        it.t.n_rows = static_cast<int32_t>(n);
        it.t.n_keys = static_cast<int32_t>(key1);
        it.t.key0 = static_cast<int32_t>(key0);
        it.t.part = -1;  // set below for the pieces of a cut tile
        it.cost = cost;
        per_combo[b * n_kv_heads + g].push_back(it);
      }
    }
    if (parts > 1) {
      for (int g = 0; g < n_kv_heads; ++g) {
        AttnMerge m{};
        m.req = b;
        m.kv_head = g;
        m.row0 = static_cast<int32_t>(row);
        m.n_rows = static_cast<int32_t>(n);
        m.first_part = chosen.n_parts;
        m.n_parts = static_cast<int32_t>(parts);
        m.q_off = p.q_off[b];
        chosen.n_parts += static_cast<int32_t>(parts);
        chosen.merges.push_back(m);
        // the pieces of this (tile, g) were pushed last into their group, in key order
        auto& v = per_combo[b * n_kv_heads + g];
        for (int64_t i = 0; i < parts; ++i) v[v.size() - parts + i].t.part = m.first_part + static_cast<int32_t>(i);
      }
    }
  }
  chosen.queue.assign(kXcds, {});
  std::vector<int64_t> total(n_combo, 0);
  int64_t sum = 0;
  for (int c = 0; c < n_combo; ++c) {
    for (const Item& it : per_combo[c]) total[c] += it.cost;
    sum += total[c];
  }
  // whole (request, kv head) groups go to the currently lightest domain, heaviest first ...
  std::vector<int> order(n_combo), home(n_combo);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return total[a] > total[b]; });
  std::vector<int64_t> domain(kXcds, 0);
  for (int c : order) {
    home[c] = static_cast<int>(std::min_element(domain.begin(), domain.end()) - domain.begin());
    domain[home[c]] += total[c];
  }
  if (n_combo > 0 && kXcds % n_combo == 0) {
    // (few groups: each has its own share of the domains, which get its tiles in turn)
    const int share = kXcds / n_combo;
    for (int c = 0; c < n_combo; ++c) {
      std::stable_sort(per_combo[c].begin(), per_combo[c].end(), by_cost);
      for (size_t i = 0; i < per_combo[c].size(); ++i)
        chosen.queue[c * share + static_cast<int>(i % share)].push_back(per_combo[c][i]);
    }
  } else if (*std::max_element(domain.begin(), domain.end()) * kXcds <= sum + sum * 3 / 100) {
    for (int c : order) chosen.queue[home[c]].insert(chosen.queue[home[c]].end(), per_combo[c].begin(), per_combo[c].end());
  } else {
    // ... unless that leaves some domain idle at the end (12 groups on 8 domains: a quarter of
    // the chip): then the groups lie on a line that is cut into eight equal parts, and the tiles
    // of a group that spans several domains are dealt to them, longest first, by what each lacks
    int64_t begin = 0;
    for (int c = 0; c < n_combo; ++c) {
      int64_t lack[kXcds] = {};
      for (int x = 0; x < kXcds; ++x)
        lack[x] = std::min(begin + total[c], sum * (x + 1) / kXcds) - std::max(begin, sum * x / kXcds);
      begin += total[c];
      std::stable_sort(per_combo[c].begin(), per_combo[c].end(), by_cost);
      for (const Item& it : per_combo[c]) {
        const int x = static_cast<int>(std::max_element(lack, lack + kXcds) - lack);
        lack[x] -= it.cost;
        chosen.queue[x].push_back(it);
      }
    }
  }
  for (auto& q : chosen.queue) std::stable_sort(q.begin(), q.end(), by_cost);
  // Predicted duration of the launch, in blocks: every L2 domain hands its tiles in order to whichever
  // of its compute units is free first; a tile costs two blocks more than its keys, a piece of a cut
  // one five.  (Smaller fixed costs than `duration` has, which are relative to the time of a block in
  // small launches: what hangs on the estimate is whether it leaves anything idle and whether it
  // comes to half a millisecond.)
  int64_t busy_blocks = 0;  // compute-unit time the tiles take, in blocks
  auto predicted_makespan = [&]() {
    int64_t worst = 0;
    auto heavier = std::greater<int64_t>();
    for (const auto& q : chosen.queue) {
      std::vector<int64_t> load(kComputeUnits / kXcds, 0);  // min-heap of compute unit loads
      for (const Item& it : q) {
        std::pop_heap(load.begin(), load.end(), heavier);
        const int64_t cost = (it.t.n_keys - it.t.key0 + kBlock - 1) / kBlock + 2 + (it.t.part >= 0 ? 3 : 0);
        load.back() += cost;
        busy_blocks += cost;
        std::push_heap(load.begin(), load.end(), heavier);
      }
      worst = std::max(worst, *std::max_element(load.begin(), load.end()));
    }
    return worst;
  };
  // what the launch is predicted to leave idle: room for work that rides along in its tail
  p.est_makespan_blocks = predicted_makespan();
  p.est_idle_blocks = p.est_makespan_blocks * kComputeUnits - busy_blocks;
  p.merges = std::move(chosen.merges);
  p.n_parts = chosen.n_parts;
  size_t depth = 0;
  for (const auto& q : chosen.queue) depth = std::max(depth, q.size());
  p.tiles.clear();
  p.tiles.reserve(depth * kXcds);
  for (size_t i = 0; i < depth; ++i)
    for (int x = 0; x < kXcds; ++x) {
      if (i < chosen.queue[x].size()) {
        p.tiles.push_back(chosen.queue[x][i].t);
      } else {
        p.tiles.push_back(AttnTile{});  // padding keeps the i % 8 dealing intact
      }
    }
  while (!p.tiles.empty() && p.tiles.back().n_rows == 0) p.tiles.pop_back();
}

// Work items of the fp32 attention: tiles of 32 flattened rows, longest first, and where that leaves compute
// units idle the same launch with the long tiles cut along the keys into even pieces, whose partial results a
// second launch merges.
//
// How long the pieces are is decided by list scheduling over the compute units that one kv head has to itself, a
// workgroup at a time on each.  Costs in units of 0.85 us: a wavefront multiplies a block of 32 keys in 3.4 us (heads
// of 64: 1.7) and shares its SIMD with one other, every block it takes costs latencies besides, and so do a
// workgroup and the merge launch.  Fitted to a sweep of the piece length over nine requests of 300 to 2.5K tokens (both
// head sizes), where the choice is within 5 % of the best length.  Attention and merge, uncut and cut: 149 rows over 693
// keys with 32 heads 38.3 -> 26.5 us, 76 over 360 22.5 -> 16.3, 4 heads of 64 over 2.6K keys 64.5 -> 18.4; batches that fill
// the chip stay whole (396 rows over 1.9K keys with 32 heads 95 us, cut at best 105).
void build_pieces_f32(mpic_plan& p, int group, int n_kv_heads, int head_dim) {
  p.tiles_f32.clear();
  p.pieces_f32.clear();
  p.merges_f32.clear();
  p.n_parts_f32 = 0;
  constexpr int64_t kKeys = 32, kWaves = 8, kSimds = 4;
  std::vector<AttnPieceF32>& tiles = p.tiles_f32;
  for (int b = 0; b < p.n_requests; ++b) {
    const int64_t rows = static_cast<int64_t>(p.q_off[b + 1] - p.q_off[b]) * group;
    for (int64_t row = 0; row < rows; row += kAttnTileRowsF32) {
      const int64_t n = std::min<int64_t>(kAttnTileRowsF32, rows - row);
      const int32_t last = p.q_pos[p.q_off[b] + (row + n - 1) / group];
      tiles.push_back(AttnPieceF32{b, static_cast<int32_t>(row), static_cast<int32_t>(n), 0, last + 1, -1, p.q_off[b], p.ctx_off[b]});
    }
  }
  auto longer = [](const AttnPieceF32& x, const AttnPieceF32& y) { return x.key1 - x.key0 > y.key1 - y.key0; };
  std::stable_sort(tiles.begin(), tiles.end(), longer);
  auto blocks_of = [](const AttnPieceF32& t) { return (t.key1 - t.key0 + kKeys - 1) / kKeys; };
  const int64_t longest = tiles.empty() ? 0 : blocks_of(tiles.front());
  if (longest <= kWaves) return;
  int64_t heads = n_kv_heads, cus = kComputeUnits;
  while (heads % 2 == 0 && cus > kSimds) heads /= 2, cus /= 2;
  auto cost = [&](int64_t blocks) {
    const int64_t on_simd = (blocks + kSimds - 1) / kSimds, rounds = (blocks + kWaves - 1) / kWaves;
    return head_dim == 64 ? 3 + 2 * on_simd + 3 * rounds : 4 + 4 * on_simd + 5 * rounds;
  };
  constexpr int64_t kMergeCost = 3;
  const int64_t part_rows_per_unit = int64_t{425000} / head_dim;  // (8 bytes a coordinate, 4 TB/s)
  std::vector<int64_t> load;
  auto simulate = [&](int64_t cap, int64_t best) {
    int64_t sum = 0, n_parts = 0;
    for (const AttnPieceF32& t : tiles) {
      const int64_t blocks = blocks_of(t), parts = (blocks + cap - 1) / cap;
      sum += (parts - blocks % parts) * cost(blocks / parts) + blocks % parts * cost(blocks / parts + 1);
      if (parts > 1) n_parts += parts;
    }
    const int64_t merge = n_parts > 0 ? kMergeCost + n_parts * kAttnTileRowsF32 * n_kv_heads / part_rows_per_unit : 0;
    if (sum * heads / cus + merge >= best) return best;  // cannot be better
    load.assign(cus, 0);                                 // min-heap
    const auto heavier = std::greater<int64_t>();
    int64_t end = 0;
    for (const AttnPieceF32& t : tiles) {
      const int64_t blocks = blocks_of(t), parts = (blocks + cap - 1) / cap;
      for (int64_t i = 0; i < parts * heads; ++i) {
        std::pop_heap(load.begin(), load.end(), heavier);
        load.back() += cost(blocks / parts + (i % parts < blocks % parts));
        end = std::max(end, load.back());
        std::push_heap(load.begin(), load.end(), heavier);
        if (end + merge >= best) return best;
      }
    }
    return end + merge;
  };
  int64_t total = 0;
  for (const AttnPieceF32& t : tiles) total += blocks_of(t);
  if (total * heads >= 4 * longest * cus) return;  // several rounds of the longest tile: even enough
  int64_t cut = longest, best = simulate(longest, INT64_MAX);
  best -= best * 5 / 100;  // a cut launch has to be worth its partial results
  std::vector<int64_t> caps;
  for (int64_t cap = kSimds; cap < longest; cap += std::max<int64_t>(1, cap / 5)) caps.push_back(cap);
  // Tried from a compute unit's share outwards, where the best one mostly lies: the others are then seen to be no better
  // without a look at most of their pieces.  Of equally good ones the shortest is taken.
  const int64_t share = total * heads / cus;
  size_t lo = std::lower_bound(caps.begin(), caps.end(), share) - caps.begin(), hi = lo;
  while (lo > 0 || hi < caps.size()) {
    const bool up = lo == 0 || (hi < caps.size() && caps[hi] * caps[lo - 1] <= share * share);
    const int64_t cap = up ? caps[hi++] : caps[--lo];
    const int64_t bound = best + (cap < cut && cut < longest);
    const int64_t end = simulate(cap, bound);
    if (end < bound) {
      best = end;
      cut = cap;
    }
  }
  if (cut == longest) return;
  for (const AttnPieceF32& t : tiles) {
    const int64_t blocks = blocks_of(t), parts = (blocks + cut - 1) / cut;
    if (parts > 1) {
      p.merges_f32.push_back(AttnMerge{t.req, 0, t.row0, t.n_rows, p.n_parts_f32, static_cast<int32_t>(parts), t.q_off, 0});
    }
    for (int64_t i = 0; i < parts; ++i) {
      AttnPieceF32 x = t;
      x.key0 = static_cast<int32_t>(blocks * i / parts * kKeys);
      x.key1 = std::min(t.key1, static_cast<int32_t>(blocks * (i + 1) / parts * kKeys));
      if (parts > 1) x.part = p.n_parts_f32++;
      p.pieces_f32.push_back(x);
    }
  }
  std::stable_sort(p.pieces_f32.begin(), p.pieces_f32.end(), longer);
}

// Key blocks of a lazy_rope plan (see KeyBlock), as the kernels walk them.  The list of a request
// holds its fresh blocks first and its stored blocks after them, each part in position order: a
// kernel that walks a tile in list order changes the shift its queries are turned back by once per
// chunk instance (softmax does not care about the order of the keys).  A tile visits the blocks
// that start at or before its last row, a prefix of both parts; the pieces of a tile that was cut
// along the keys share those blocks in proportion to their key ranges, in list order.
void build_key_blocks(mpic_plan& p) {
  const int B = p.n_requests;
  p.key_order.clear();
  p.key_order.reserve(p.n_ctx);
  for (int b = 0; b < B; ++b) {
    for (int32_t r = p.q_off[b]; r < p.q_off[b + 1]; ++r) p.key_order.push_back(p.ctx_off[b] + p.q_pos[r]);
    for (int32_t pos = p.ctx_off[b]; pos < p.ctx_off[b + 1]; ++pos)
      if (p.src_inst[pos] >= 0) p.key_order.push_back(pos);
  }
  // where the tile that a piece belongs to ends
  std::vector<int32_t> tile_end(p.n_parts);
  for (const AttnTile& t : p.tiles)
    if (t.n_rows > 0 && t.part >= 0) tile_end[t.part] = t.n_keys;
  for (const AttnMerge& m : p.merges)  // (the last piece ends where the tile does)
    for (int32_t i = 0; i + 1 < m.n_parts; ++i) tile_end[m.first_part + i] = tile_end[m.first_part + m.n_parts - 1];

  for (int s = 0; s < kNumBlockSizes; ++s) {
    const int32_t bn = kBlockSizes[s];
    auto& blocks = p.kblk[s];
    auto& first = p.kblk_first[s];
    auto& mid = p.kblk_mid[s];
    auto& parts = p.kblk_parts[s];
    blocks.clear();
    first.assign(1, 0);
    mid.clear();
    parts.clear();
    for (int b = 0; b < B; ++b) {
      const int32_t ctx0 = p.ctx_off[b], n = p.ctx_off[b + 1] - ctx0, n_fresh = p.q_off[b + 1] - p.q_off[b];
      const int32_t* order = p.key_order.data() + ctx0;
      for (int32_t i = 0; i < n_fresh; i += bn) blocks.push_back(KeyBlock{order[i] - ctx0, std::min(bn, n_fresh - i), -1, i});
      mid.push_back(static_cast<int32_t>(blocks.size()));
      for (int32_t i = n_fresh; i < n;) {
        const int32_t inst = p.src_inst[order[i]];
        int32_t end = i + 1;
        while (end < n && end - i < bn && p.src_inst[order[end]] == inst) ++end;
        blocks.push_back(KeyBlock{order[i] - ctx0, end - i, inst, i - n_fresh});
        i = end;
      }
      first.push_back(static_cast<int32_t>(blocks.size()));
      parts.insert(parts.end(), {first[b], mid[b], first[b + 1]});
    }
    auto& ranges = p.lazy_range[s];
    ranges.clear();
    if (bn == 32) continue;  // the decode kernel splits its blocks at launch
    ranges.reserve(p.tiles.size() * 4);
    for (const AttnTile& t : p.tiles) {
      if (t.n_rows <= 0) {
        ranges.insert(ranges.end(), {0, 0, 0, 0});
        continue;
      }
      const int32_t end = t.part >= 0 ? tile_end[t.part] : t.n_keys;
      auto before_end = [&](int32_t lo, int32_t hi) {  // blocks of [lo, hi) that start below the tile's end
        const KeyBlock* it = std::lower_bound(blocks.data() + lo, blocks.data() + hi, end,
                                              [](const KeyBlock& k, int32_t v) { return k.pos0 < v; });
        return static_cast<int32_t>(it - (blocks.data() + lo));
      };
      // no piece is empty: a piece owns more than 192 keys' worth of positions, and a gathered block
      // holds 96 keys at most.  Every row sees a key of the first piece, which starts with the
      // request's first fresh row
      const int32_t nf = before_end(first[t.req], mid[t.req]), ns = before_end(mid[t.req], first[t.req + 1]);
      const int32_t lo = static_cast<int32_t>(static_cast<int64_t>(nf + ns) * t.key0 / end);
      const int32_t hi = static_cast<int32_t>(static_cast<int64_t>(nf + ns) * t.n_keys / end);
      const int32_t r[4] = {std::min(lo, nf), std::min(hi, nf), std::max(lo, nf) - nf, std::max(hi, nf) - nf};
      ranges.insert(ranges.end(), r, r + 4);
    }
  }
}

// Whether the attention over caches in place runs in half tiles, two workgroups of four wavefronts for each, or in whole
// ones of eight.  Halves start sooner, fill each other's gaps on a compute unit, skip blocks that only the other half's rows
// reach, and pad a chunk's last key block to 64 keys instead of 96; whole tiles read every block once for all rows and have
// fewer barriers per key.  Time of 350 launches of 11 to 510 us in halves, relative to whole tiles:
//   tall tiles (more than half the rows) hold most of the blocks: 0.76 to 1.08 (0.90 on average) up to 60 blocks per compute
//     unit, except cut into long pieces, which gain neither start nor balance (0.98 to 1.07); above that it is the padding of
//     short chunks that decides: 0.78 to 1.03 (0.92) where halves walk up to 0.975 of the keys that whole tiles walk, padding
//     counted, 0.95 to 1.12 (1.01) where they save less; more than 180 blocks per compute unit 1.0 to 1.14;
//   low tiles, which leave one wavefront on a SIMD in either shape: up to four blocks per compute unit 0.68 to 1.05 (0.95), but
//     1.0 to 1.09 where they have more than two wavefronts of rows; with more blocks 0.86 to 1.33 (1.04).
// Of 191 drawn launches that this rule runs in halves, 12 took more than 1.015 of the time, 0.906 on average.
bool runs_in_halves(const mpic_plan& p) {
  int64_t pieces = 0, cut = 0, blocks = 0, tall = 0, low = 0, low_rows = 0;
  for (const AttnTile& t : p.tiles) {
    if (t.n_rows <= 0) continue;
    const int64_t b = (t.n_keys - t.key0 + 63) / 64;
    ++pieces;
    cut += t.part >= 0;
    blocks += b;
    if (t.n_rows > kAttnTileRows / 2) {
      tall += b;
    } else {
      ++low;
      low_rows += t.n_rows;
    }
  }
  if (2 * tall < blocks) return blocks <= 4 * kComputeUnits && low_rows <= 64 * low;
  if (blocks > 180 * kComputeUnits || (3 * cut >= 2 * pieces && blocks > 28 * pieces)) return false;
  if (blocks <= 60 * kComputeUnits) return true;
  auto keys_walked = [&](int32_t bn) {
    int64_t n = 0;
    const auto& r = p.lazy_range[block_size_index(bn)];
    for (size_t i = 0; i < r.size(); i += 2) n += r[i + 1] - r[i];
    return n * bn;
  };
  return 1000 * keys_walked(kHalfTileBlock) <= 975 * keys_walked(96);
}

// The block ranges of the tiles' halves of rows (lazy_half): the first one reaches less far.  At least one block each, so that
// a half whose rows see nothing of a piece has something to walk.
void build_half_ranges(mpic_plan& p, int group) {
  const int s = block_size_index(kHalfTileBlock);
  p.lazy_half.clear();
  if (!p.half_tiles) return;
  p.lazy_half.reserve(p.tiles.size() * 8);
  for (size_t i = 0; i < p.tiles.size(); ++i) {
    const AttnTile& t = p.tiles[i];
    const int32_t* r = p.lazy_range[s].data() + 4 * i;
    for (int32_t row = 0; row < kAttnTileRows; row += kAttnTileRows / 2) {
      if (row >= t.n_rows) {
        p.lazy_half.insert(p.lazy_half.end(), {0, 0, 0, 0});
        continue;
      }
      const int32_t last_row = t.row0 + std::min(t.n_rows, row + kAttnTileRows / 2) - 1;
      const int32_t reach = p.q_pos[p.q_off[t.req] + last_row / group];
      // of blocks lo .. hi - 1 behind block `from`, the first that starts behind the reach
      auto up_to = [&](int32_t from, int32_t lo, int32_t hi) {
        const KeyBlock* part = p.kblk[s].data() + from;
        return static_cast<int32_t>(std::upper_bound(part + lo, part + hi, reach,
                                                     [](int32_t v, const KeyBlock& k) { return v < k.pos0; }) - part);
      };
      int32_t f1 = up_to(p.kblk_first[s][t.req], r[0], r[1]);
      int32_t s1 = up_to(p.kblk_mid[s][t.req], r[2], r[3]);
      if (f1 == r[0] && s1 == r[2]) (r[0] < r[1] ? f1 : s1) += 1;
      p.lazy_half.insert(p.lazy_half.end(), {r[0], f1, r[2], s1});
    }
  }
}

// Rotary tables of the fresh rows, for contexts whose fresh Q/K arrive without positions:
// one table row per distinct position id of the batch (requests with the same layout share
// all of them) and an index per fresh row.  cos/sin of p * w_i are evaluated in double
// from p = 256 * hi + lo by the angle-addition formulas, which needs (max_p / 256 + 256)
// evaluations per frequency instead of one per position, and are rounded once to float.
void build_fresh_rope(mpic_plan& p, const mpic_config& c) {
  const int half = c.head_dim / 2;
  const size_t nq = p.q_pos.size();
  p.fresh_rot.resize(nq);
  if (nq == 0) return;
  const int32_t max_pos = *std::max_element(p.q_pos.begin(), p.q_pos.end());
  std::vector<int32_t> row_of(static_cast<size_t>(max_pos) + 1, -1);
  std::vector<int32_t> uniq;
  for (size_t r = 0; r < nq; ++r) {
    int32_t& u = row_of[p.q_pos[r]];
    if (u < 0) {
      u = static_cast<int32_t>(uniq.size());
      uniq.push_back(p.q_pos[r]);
    }
    p.fresh_rot[r] = u;
  }
  constexpr int kLo = 256;
  const int n_hi = max_pos / kLo + 1;
  std::vector<double> hi_c(static_cast<size_t>(n_hi) * half), hi_s(hi_c.size());
  std::vector<double> lo_c(static_cast<size_t>(kLo) * half), lo_s(lo_c.size());
  for (int j = 0; j < half; ++j) {
    const double w = std::pow(c.rope_theta, -2.0 * j / c.head_dim);
    for (int h = 0; h < n_hi; ++h) {
      const double phi = static_cast<double>(h) * kLo * w;
      hi_c[static_cast<size_t>(h) * half + j] = std::cos(phi);
      hi_s[static_cast<size_t>(h) * half + j] = std::sin(phi);
    }
    for (int l = 0; l < kLo; ++l) {
      const double phi = static_cast<double>(l) * w;
      lo_c[static_cast<size_t>(l) * half + j] = std::cos(phi);
      lo_s[static_cast<size_t>(l) * half + j] = std::sin(phi);
    }
  }
  p.fresh_cos.resize(uniq.size() * half);
  p.fresh_sin.resize(uniq.size() * half);
  for (size_t u = 0; u < uniq.size(); ++u) {
    const double* hc = &hi_c[static_cast<size_t>(uniq[u] / kLo) * half];
    const double* hs = &hi_s[static_cast<size_t>(uniq[u] / kLo) * half];
    const double* lc = &lo_c[static_cast<size_t>(uniq[u] % kLo) * half];
    const double* ls = &lo_s[static_cast<size_t>(uniq[u] % kLo) * half];
    for (int j = 0; j < half; ++j) {
      p.fresh_cos[u * half + j] = static_cast<float>(hc[j] * lc[j] - hs[j] * ls[j]);
      p.fresh_sin[u * half + j] = static_cast<float>(hs[j] * lc[j] + hc[j] * ls[j]);
    }
  }
}

}  // namespace
}  // namespace mpic

using mpic::fail;

extern "C" int mpic_create(mpic_ctx** out, const mpic_config* config) {
  if (!out || !config) return MPIC_ERR_INVALID;
  *out = nullptr;
  const mpic_config& c = *config;
  if (c.n_q_heads <= 0 || c.n_kv_heads <= 0 || c.head_dim <= 0 || c.n_q_heads % c.n_kv_heads != 0 ||
      (c.head_dim & 1) || !(c.rope_theta > 0.0) || !std::isfinite(c.rope_theta) || c.page_size < 0 ||
      (c.rope_interleaved != 0 && c.rope_interleaved != 1) || (c.fresh_pre_rope != 0 && c.fresh_pre_rope != 1) ||
      (c.lazy_rope != 0 && c.lazy_rope != 1))
    return MPIC_ERR_INVALID;
  if (c.dtype == MPIC_F32) {
    if (c.head_dim != 64 && c.head_dim != 128) return MPIC_ERR_UNSUPPORTED;
  } else if (c.dtype == MPIC_BF16) {
    if (c.head_dim != 128) return MPIC_ERR_UNSUPPORTED;
  } else {
    return MPIC_ERR_INVALID;
  }
  mpic_ctx* ctx = nullptr;
  try {
    ctx = new mpic_ctx();
  } catch (const std::bad_alloc&) {
    return MPIC_ERR_OOM;
  }
  ctx->cfg = c;
  ctx->group = c.n_q_heads / c.n_kv_heads;
  *out = ctx;
  return MPIC_OK;
}

extern "C" int mpic_plan_create(mpic_ctx* ctx, int32_t n_requests, const int32_t* seg_off,
                                const mpic_segment* segs, int32_t default_k,
                                const int32_t* page_table, const int32_t* page_table_off,
                                int64_t n_pool_pages, mpic_plan** out) {
  return mpic_plan_create_selected(ctx, n_requests, seg_off, segs, default_k, nullptr, nullptr, page_table,
                                   page_table_off, n_pool_pages, out);
}

extern "C" int mpic_plan_create_selected(mpic_ctx* ctx, int32_t n_requests, const int32_t* seg_off,
                                         const mpic_segment* segs, int32_t default_k,
                                         const int32_t* sel_off, const int32_t* sel_idx,
                                         const int32_t* page_table, const int32_t* page_table_off,
                                         int64_t n_pool_pages, mpic_plan** out) {
  if (!ctx) return MPIC_ERR_INVALID;
  if (!out) return fail(ctx, MPIC_ERR_INVALID, "plan_create: out is NULL");
  *out = nullptr;
  if (n_requests < 1 || !seg_off || default_k < 0)
    return fail(ctx, MPIC_ERR_INVALID, "plan_create: need n_requests >= 1, seg_off, default_k >= 0");
  const int ps = ctx->cfg.page_size;
  if (ps > 0 && (!page_table_off || n_pool_pages <= 0))
    return fail(ctx, MPIC_ERR_INVALID, "plan_create: paged layout needs page table offsets and a pool size");
  if (seg_off[0] != 0) return fail(ctx, MPIC_ERR_INVALID, "plan_create: seg_off[0] must be 0");
  for (int b = 0; b < n_requests; ++b)
    if (seg_off[b + 1] < seg_off[b]) return fail(ctx, MPIC_ERR_INVALID, "plan_create: seg_off must not decrease");
  if (seg_off[n_requests] > 0 && !segs) return fail(ctx, MPIC_ERR_INVALID, "plan_create: segs is NULL");

  // pass 1: validate and size
  int64_t n_ctx = 0, n_q = 0;
  for (int32_t s = 0; s < seg_off[n_requests]; ++s) {
    const mpic_segment& g = segs[s];
    if (g.len < 0 || (g.kind != 0 && g.kind != 1)) return fail(ctx, MPIC_ERR_INVALID, "plan_create: bad segment kind or negative len");
    if (g.kind == 1 && g.chunk < 0) return fail(ctx, MPIC_ERR_INVALID, "plan_create: negative chunk index");
    n_ctx += g.len;
    if (g.kind == 0) {
      n_q += g.len;
    } else if (g.k == MPIC_K_LISTED) {
      if (!sel_off || sel_off[s + 1] < sel_off[s] || (sel_off[s + 1] > sel_off[s] && !sel_idx))
        return fail(ctx, MPIC_ERR_INVALID, "plan_create: a listed recompute set needs sel_off / sel_idx");
      for (int32_t i = sel_off[s]; i < sel_off[s + 1]; ++i)
        if (sel_idx[i] < 0 || sel_idx[i] >= g.len) return fail(ctx, MPIC_ERR_INVALID, "plan_create: listed token outside its chunk");
      n_q += std::min<int64_t>(sel_off[s + 1] - sel_off[s], g.len);  // upper bound (duplicates allowed)
    } else {
      const int64_t k = g.k < 0 ? default_k : g.k;
      n_q += std::min<int64_t>(k, g.len);
    }
  }
  const int64_t slot_limit = ps > 0 ? n_pool_pages * ps : n_ctx;
  if (n_ctx >= INT32_MAX || slot_limit >= INT32_MAX || n_q * ctx->group >= INT32_MAX)
    return fail(ctx, MPIC_ERR_INVALID, "plan_create: batch too large for 32-bit indices");

  mpic_plan* p = new (std::nothrow) mpic_plan();
  if (!p) return fail(ctx, MPIC_ERR_OOM, "plan_create: out of host memory");
  try {
    p->ctx = ctx;
    p->n_requests = n_requests;
    p->n_ctx = n_ctx;
    p->ctx_off.assign(1, 0);
    p->q_off.assign(1, 0);
    p->q_pos.reserve(n_q);
    p->q_req.reserve(n_q);
    p->slot_map.reserve(n_q);
    p->src_inst.resize(n_ctx);
    p->src_row.resize(n_ctx);
    p->dst_slot.resize(n_ctx);
    std::vector<char> page_used, mark;
    if (ps > 0) page_used.assign(n_pool_pages, 0);

    for (int b = 0; b < n_requests; ++b) {
      const int32_t ctx0 = p->ctx_off.back();
      const int32_t q0 = p->q_off.back();
      int32_t pos = 0;  // position inside the request
      int32_t row = q0; // next fresh row
      auto take_fresh = [&](int32_t first, int32_t count) {
        if (count <= 0) return;
        const bool extends = !p->runs.empty() && p->runs[p->runs.size() - 4] == b &&
                             p->runs[p->runs.size() - 1] + p->runs[p->runs.size() - 2] == first;
        if (extends) {
          p->runs[p->runs.size() - 2] += count;
        } else {
          p->runs.insert(p->runs.end(), {b, row, count, first});
        }
        for (int32_t t = 0; t < count; ++t) {
          p->src_inst[ctx0 + first + t] = -1;
          p->src_row[ctx0 + first + t] = row;
          p->q_pos.push_back(first + t);
          p->q_req.push_back(b);
          ++row;
        }
      };
      for (int32_t s = seg_off[b]; s < seg_off[b + 1]; ++s) {
        const mpic_segment& g = segs[s];
        if (g.kind == 0) {
          take_fresh(pos, g.len);
        } else {
          // which tokens of the chunk are recomputed: the first k, or the listed ones
          mark.assign(g.len, 0);
          if (g.k == MPIC_K_LISTED) {
            for (int32_t i = sel_off[s]; i < sel_off[s + 1]; ++i) mark[sel_idx[i]] = 1;
          } else {
            const int64_t k = g.k < 0 ? default_k : g.k;
            std::fill(mark.begin(), mark.begin() + std::min<int64_t>(k, g.len), 1);
          }
          int32_t k_eff = 0;  // length of the leading recomputed run
          while (k_eff < g.len && mark[k_eff]) ++k_eff;
          const int32_t inst = static_cast<int32_t>(p->inst_src.size());
          p->inst_src.push_back(g.chunk);
          p->inst_delta.push_back(pos);
          p->inst_len.push_back(g.len);
          p->inst_k.push_back(k_eff);
          p->inst_req.push_back(b);
          p->max_src = std::max(p->max_src, g.chunk);
          int32_t cached = 0;
          for (int32_t t = 0; t < g.len;) {
            int32_t e = t;
            if (mark[t]) {
              while (e < g.len && mark[e]) ++e;
              take_fresh(pos + t, e - t);
            } else {
              while (e < g.len && !mark[e]) {
                p->src_inst[ctx0 + pos + e] = inst;
                p->src_row[ctx0 + pos + e] = e;
                ++e;
              }
              cached += e - t;
            }
            t = e;
          }
          p->inst_cached.push_back(cached);
        }
        pos += g.len;
      }
      // physical slots
      if (ps > 0) {
        const int64_t have = static_cast<int64_t>(page_table_off[b + 1]) - page_table_off[b];
        const int64_t need = (static_cast<int64_t>(pos) + ps - 1) / ps;
        if (have < need || (need > 0 && !page_table)) {
          delete p;
          return fail(ctx, MPIC_ERR_INVALID, "plan_create: page table missing or shorter than the request");
        }
        const int32_t* tab = page_table + page_table_off[b];
        for (int64_t pg = 0; pg < need; ++pg) {
          const int32_t id = tab[pg];
          if (id < 0 || id >= n_pool_pages || page_used[id]) {
            delete p;
            return fail(ctx, MPIC_ERR_INVALID, "plan_create: page id out of range or used twice");
          }
          page_used[id] = 1;
        }
        for (int32_t t = 0; t < pos; ++t) p->dst_slot[ctx0 + t] = tab[t / ps] * ps + t % ps;
      } else {
        for (int32_t t = 0; t < pos; ++t) p->dst_slot[ctx0 + t] = ctx0 + t;
      }
      for (int32_t r = q0; r < row; ++r) p->slot_map.push_back(p->dst_slot[ctx0 + p->q_pos[r]]);
      p->ctx_off.push_back(ctx0 + pos);
      p->q_off.push_back(row);
    }
    for (int32_t s : p->dst_slot) p->max_slot = std::max<int64_t>(p->max_slot, s);
    p->n_q = static_cast<int64_t>(p->q_pos.size());

    // rotary tables: one angle vector per chunk instance, evaluated in double
    const int half = ctx->cfg.head_dim / 2;
    p->rope_cos.resize(p->inst_src.size() * half);
    p->rope_sin.resize(p->inst_src.size() * half);
    for (size_t i = 0; i < p->inst_src.size(); ++i)
      for (int j = 0; j < half; ++j) {
        const double inv_freq = std::pow(ctx->cfg.rope_theta, -2.0 * j / ctx->cfg.head_dim);
        const double phi = static_cast<double>(p->inst_delta[i]) * inv_freq;
        p->rope_cos[i * half + j] = static_cast<float>(std::cos(phi));
        p->rope_sin[i * half + j] = static_cast<float>(std::sin(phi));
      }
    if (ctx->cfg.fresh_pre_rope) mpic::build_fresh_rope(*p, ctx->cfg);
    mpic::build_tiles(*p, ctx->group, ctx->cfg.n_kv_heads);
    if (ctx->cfg.dtype == MPIC_F32) mpic::build_pieces_f32(*p, ctx->group, ctx->cfg.n_kv_heads, ctx->cfg.head_dim);
    if (ctx->cfg.lazy_rope) {
      mpic::build_key_blocks(*p);
      p->half_tiles = mpic::runs_in_halves(*p);
      mpic::build_half_ranges(*p, ctx->group);
    }
    {
      auto clamp = [](int64_t x) { return static_cast<int32_t>(std::min<int64_t>(x, INT32_MAX)); };
      p->launch_est = {clamp(p->est_makespan_blocks), clamp(p->est_idle_blocks),
                       mpic::can_link_in_attention(ctx, p) ? 1 : 0,
                       mpic::can_link_in_attention(ctx, p) && mpic::link_fits_attention_tail(ctx, p) ? 1 : 0};
    }
  } catch (const std::bad_alloc&) {
    delete p;
    return fail(ctx, MPIC_ERR_OOM, "plan_create: out of host memory");
  }
  *out = p;
  return MPIC_OK;
}

extern "C" int mpic_plan_get(const mpic_plan* plan, int32_t what, const int32_t** host_ptr, size_t* n) {
  if (!plan || !host_ptr || !n) return MPIC_ERR_INVALID;
  const std::vector<int32_t>* v = nullptr;
  switch (what) {
    case MPIC_PLAN_CTX_OFF: v = &plan->ctx_off; break;
    case MPIC_PLAN_Q_OFF: v = &plan->q_off; break;
    case MPIC_PLAN_Q_POS: v = &plan->q_pos; break;
    case MPIC_PLAN_Q_REQ: v = &plan->q_req; break;
    case MPIC_PLAN_SLOT_MAP: v = &plan->slot_map; break;
    case MPIC_PLAN_SRC_INST: v = &plan->src_inst; break;
    case MPIC_PLAN_SRC_ROW: v = &plan->src_row; break;
    case MPIC_PLAN_DST_SLOT: v = &plan->dst_slot; break;
    case MPIC_PLAN_INST_SRC: v = &plan->inst_src; break;
    case MPIC_PLAN_INST_DELTA: v = &plan->inst_delta; break;
    case MPIC_PLAN_INST_LEN: v = &plan->inst_len; break;
    case MPIC_PLAN_INST_K: v = &plan->inst_k; break;
    case MPIC_PLAN_INST_REQ: v = &plan->inst_req; break;
    case MPIC_PLAN_RUNS: v = &plan->runs; break;
    case MPIC_PLAN_LAUNCH_ESTIMATE: v = &plan->launch_est; break;
    case MPIC_PLAN_LAZY_TILES_64: v = &plan->lazy_range[1]; break;
    case MPIC_PLAN_LAZY_TILES_96: v = &plan->lazy_range[2]; break;
    case MPIC_PLAN_KEY_BLOCK_PARTS_32: v = &plan->kblk_parts[0]; break;
    case MPIC_PLAN_KEY_BLOCK_PARTS_64: v = &plan->kblk_parts[1]; break;
    case MPIC_PLAN_KEY_BLOCK_PARTS_96: v = &plan->kblk_parts[2]; break;
    case MPIC_PLAN_KEY_BLOCK_ORDER: v = &plan->key_order; break;
    case MPIC_PLAN_KEY_BLOCKS_32:
    case MPIC_PLAN_KEY_BLOCKS_64:
    case MPIC_PLAN_KEY_BLOCKS_96: {
      const auto& blocks = plan->kblk[what - MPIC_PLAN_KEY_BLOCKS_32];
      *host_ptr = reinterpret_cast<const int32_t*>(blocks.data());
      *n = blocks.size() * 4;
      return MPIC_OK;
    }
    case MPIC_PLAN_ATTN_TILES:
      *host_ptr = reinterpret_cast<const int32_t*>(plan->tiles.data());
      *n = plan->tiles.size() * 8;
      return MPIC_OK;
    default:
      return fail(plan->ctx, MPIC_ERR_INVALID, "plan_get: unknown selector");
  }
  *host_ptr = v->data();
  *n = v->size();
  return MPIC_OK;
}

extern "C" int mpic_plan_get_rope(const mpic_plan* plan, const float** cos_tab, const float** sin_tab,
                                  size_t* n) {
  if (!plan || !cos_tab || !sin_tab || !n) return MPIC_ERR_INVALID;
  *cos_tab = plan->rope_cos.data();
  *sin_tab = plan->rope_sin.data();
  *n = plan->rope_cos.size();
  return MPIC_OK;
}

extern "C" int mpic_plan_get_fresh_rope(const mpic_plan* plan, const int32_t** table_row,
                                        const float** cos_tab, const float** sin_tab, size_t* n_rows) {
  if (!plan || !table_row || !cos_tab || !sin_tab || !n_rows) return MPIC_ERR_INVALID;
  *table_row = plan->fresh_rot.data();
  *cos_tab = plan->fresh_cos.data();
  *sin_tab = plan->fresh_sin.data();
  *n_rows = plan->fresh_cos.size() / (plan->ctx->cfg.head_dim / 2);
  return MPIC_OK;
}

extern "C" const char* mpic_strerror(int status) {
  switch (status) {
    case MPIC_OK: return "ok";
    case MPIC_ERR_INVALID: return "invalid argument";
    case MPIC_ERR_UNSUPPORTED: return "unsupported configuration";
    case MPIC_ERR_OOM: return "out of memory";
    case MPIC_ERR_HIP: return "HIP runtime error";
    case MPIC_ERR_IO: return "file of the disk tier could not be written";
    case MPIC_ERR_CACHE_MISS: return "stored cache missing or failed to load";
    default: return "unknown status";
  }
}

extern "C" const char* mpic_last_error(const mpic_ctx* ctx) { return ctx ? ctx->last_error.c_str() : ""; }
