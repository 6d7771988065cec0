#include "plan.hpp"

#include <algorithm>
#include <cmath>
#include <functional>
#include <queue>

namespace dk {

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

PlanConfig default_config(int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, bool bf16) {
  PlanConfig c;
  c.n_q_heads = n_q_heads;
  c.n_kv_heads = n_kv_heads;
  c.head_dim = head_dim;
  c.use_mfma = true;  // (route_config() decides for each call)
  c.tile_rows = 256;
  c.stream_rows = 96;
  c.kv_tile = 64;
  // stream items: never cut a slot's keys finer than one CU's fair share of the batch (256 CUs); every extra
  // item costs a ramp-up, a partial write and merge work, and the planner's chains balance the rest
  c.stream_target = std::max(1, 256 / n_kv_heads);
  c.tile_wave_slots = std::max(1, 256 / n_kv_heads);
  c.tile_min_chunk = 128;
  c.tile_item_cost = 5;
  c.stream_min_chunk = 512;
  c.stream_chains = 256;
  c.stream_item_cost = 512;
  // Workgroup w of a launch runs on XCD w % 8, and on every MI355X measured the odd XCDs stream K/V 5-10 % slower
  // than the even ones while the whole chip pulls on HBM: chains planned on the host give them that much less.
  for (int x = 0; x < 8; ++x) c.xcd_speed[x] = (x & 1) ? 0.95f : 1.f;
  c.stream_queue = 1;
  c.small_units = 256;
  c.arrivals = ARRIVALS_PER_SLICE;
  c.row_fixed_us = 10.f;
  c.row_step_us = 1.8f;
  c.unit_us = {7.0f, 9.2f, 11.4f};
  c.key_us = {0.69f, 0.96f, 1.28f};
  c.cost = {{9.3f, 11.4f, 14.6f}, {0.59f, 1.02f, 1.69f}, 3.5f, 1.4f, 6.8f, 1.72f, 3.0f, 1.4f, 1.0f, 0.08f, 0.42f, 0.04f, 5.3f};
  c.once_cells = std::max<int64_t>(1, (int64_t(256) << 20) / ((int64_t)2 * n_kv_heads * head_dim * (bf16 ? 2 : 4)));
  c.inline_blob_bytes = INLINE_BLOB_BYTES;
  return c;
}

PlanConfig route_config(const PlanConfig& cfg, Route r, int32_t n_seqs, const int32_t* cu_delta) {
  PlanConfig c = cfg;
  c.use_mfma = r != Route::kRef;
  if (cfg.small_units > 0 && (r == Route::kGeneral || r == Route::kF32)) {
    const bool wide = cfg.head_dim > 64;
    if (r == Route::kGeneral)
      c.scalar = wide ? ScalarCost{7.5f, 2.3f, 2.5f, 3.7f, 9.9f, 6.26f, 0.67f, 1.14f, 7.f, 2.5f}
                      : ScalarCost{7.1f, 0.69f, 2.9f, 2.3f, 9.4f, 5.45f, 0.38f, 0.47f, 7.f, 6.f};
    else
      c.scalar = wide ? ScalarCost{7.3f, 5.3f, 6.9f, 3.5f, 8.6f, 9.95f, 2.4f, 2.8f, 5.f, 2.f}
                      : ScalarCost{7.1f, 1.45f, 6.5f, 0.2f, 7.6f, 7.1f, 1.0f, 1.34f, 5.f, 2.f};
  }
  if (r == Route::kGeneral) {
    // block kernel: items of 128 rows, two workgroups on a compute unit; an item's fixed cost (first tiles, merge of
    // the half-waves, store) is about three of its shorter key steps
    c.tile_rows = 128;
    if (cfg.head_dim == 64) {
      c.row_fixed_us = 8.f;
      c.row_step_us = 1.4f;
      c.unit_us = {7.5f, 9.2f, 11.5f};
      c.key_us = {0.5f, 0.8f, 1.1f};
    } else {
      c.unit_us = {8.5f, 9.7f, 13.f};
      c.key_us = {0.76f, 1.25f, 1.65f};
    }
    c.cost = PlanCost();
    // (Measured with the streaming kernel's key loop as it was before it became a pipeline, like the scalar kernel's rival prices
    // above.)  With 64-wide heads the stream kernel's third row block is slower than the block kernel (16 sessions of 12-24 new
    // tokens on 500-4000: 57 us / 42 us); a batch with any longer entry runs in the block kernel as a whole, as long as
    // the short ones read no more than some 800 MB there, 20 % slower than the stream kernel does, but beside the others
    // and without a launch of their own (two chunks of 256 tokens and 14 decoding sessions 77 us / 64 us, two of 512 and
    // 46 longer ones 219 / 189; 64 verifying sessions alone, 1.3 GB: stream kernel 243, block kernel 298).
    if (cfg.head_dim == 64) c.stream_rows = std::min(c.stream_rows, 64);
    c.join_keys = (int64_t(800) << 20) / ((int64_t)4 * cfg.n_kv_heads * cfg.head_dim);
    c.tile_wave_slots = 2 * cfg.tile_wave_slots;
    c.tile_item_cost = std::min(cfg.tile_item_cost, 3);
  }
  if (r == Route::kF32) {
    // fp32 kernel: every row goes through it, in items of 32 rows once those fill the chip, else of 16.  A workgroup
    // works through 128 keys of 64 in about a microsecond; a cut costs a merge launch (6 us), so no piece is made
    // shorter than that is worth.
    int64_t items = 0;
    const int64_t group = cfg.n_q_heads / cfg.n_kv_heads;
    for (int32_t b = 0; b < n_seqs; ++b) items += (group * ((int64_t)cu_delta[b + 1] - cu_delta[b]) + 31) / 32;
    c.tile_rows = items * cfg.n_kv_heads >= 256 ? 32 : 16;
    c.stream_rows = 0;
    c.small_units = 0;
    c.tile_min_chunk = std::max(cfg.tile_min_chunk, 65536 / cfg.head_dim);
  }
  return c;
}

namespace {
typedef PlanRowTile RowTile;

// Work items of the streaming kernel: each entry's visible key range [0, kv_hi) is cut into nearly equal chunks
// (multiples of kv_tile) so that there are about `target` items per KV head and none is shorter than min_chunk;
// longest first.  Entries whose range is cut get partial rows and a merge record.
void cut_stream_items(const std::vector<RowTile>& tiles, int32_t kv_tile, int32_t target, int32_t min_chunk,
                      std::vector<DkItem>* items, std::vector<DkMerge>* merges, int64_t* part_rows) {
  if (tiles.empty()) return;
  int64_t total = 0;
  for (const RowTile& t : tiles) total += t.kv_hi;
  int64_t chunk = std::max<int64_t>(min_chunk, (total + target - 1) / target);
  chunk = (chunk + kv_tile - 1) / kv_tile * kv_tile;
  const size_t first = items->size();
  for (const RowTile& t : tiles) {
    int32_t ns = (int32_t)((t.kv_hi + chunk - 1) / chunk);
    if (ns > 1 && t.kv_hi - (int64_t)(ns - 1) * chunk < chunk / 4) --ns;  // no sliver at the end
    const int64_t each = ((t.kv_hi + ns - 1) / ns + kv_tile - 1) / kv_tile * kv_tile;
    ns = (int32_t)((t.kv_hi + each - 1) / each);
    int32_t part0 = -1;
    if (ns > 1) {
      part0 = (int32_t)*part_rows;
      *part_rows += (int64_t)ns * t.nrows;
      merges->push_back({t.entry, t.row0, t.nrows, part0, ns, 0, {0, 0}});
    }
    for (int32_t sp = 0; sp < ns; ++sp) {
      DkItem it{};
      it.entry = t.entry;
      it.row0 = t.row0;
      it.nrows = t.nrows;
      it.kv_lo = (int32_t)(sp * each);
      it.kv_hi = sp + 1 == ns ? t.kv_hi : (int32_t)((sp + 1) * each);
      it.part_row0 = ns > 1 ? part0 + sp * t.nrows : -1;
      if (ns > 1 && ns < 256 && merges->size() <= 256) {
        it.merge = (int32_t)(merges->size() - 1) * 256 + ns;
        it.part_base = part0;
      }
      items->push_back(it);
    }
  }
  std::stable_sort(items->begin() + (std::ptrdiff_t)first, items->end(), [](const DkItem& a, const DkItem& b) {
    return (int64_t)(a.kv_hi - a.kv_lo) * a.nrows > (int64_t)(b.kv_hi - b.kv_lo) * b.nrows;
  });
}

int row_blocks(const DkItem& it) { return (it.nrows + 31) / 32; }

// The streaming kernel runs one workgroup per compute unit, and a workgroup walks a chain of units
// (item, KV head).  Its workgroups share no K/V rows, so a unit may run on any XCD.  The units arrive
// longest first and each joins the chain that is free first (longest-processing-time rule on machines of
// unequal speed: workgroup w runs on XCD w % 8, and the XCDs do not stream from HBM equally fast; among
// idle chains the faster ones are served first, so they get the longest units), so that all compute
// units finish together whatever the mix of context lengths.  With very many small units, runs of
// consecutive units are handed out as one block to keep the planning time down.
// A workgroup takes the body for as many 32-row blocks as its first unit has, so that one has the most of its chain.
void chain_units(const std::vector<DkItem>& items, const PlanConfig& cfg, std::vector<std::pair<double, int32_t>>& heap,
                 std::vector<int32_t>& tail, std::vector<int32_t>* links, int32_t* n_chains) {
  const int64_t n_units = (int64_t)items.size() * cfg.n_kv_heads;
  const int32_t chains = (int32_t)std::min<int64_t>(n_units, std::max(cfg.stream_chains, 1));
  *n_chains = chains;
  links->assign((size_t)(chains + n_units), -1);
  int32_t* head = links->data();
  int32_t* next = links->data() + chains;
  if (n_units == chains) {  // one unit each: nothing to balance
    for (int32_t c = 0; c < chains; ++c) head[c] = c;
    return;
  }
  double inv_speed[8];
  for (int x = 0; x < 8; ++x) inv_speed[x] = 1.0 / (cfg.xcd_speed[x] > 0.f ? cfg.xcd_speed[x] : 1.f);
  typedef std::pair<double, int32_t> Free;  // (time at which the chain is free, chain)
  heap.resize((size_t)chains);
  for (int32_t c = 0; c < chains; ++c) heap[c] = {1e-6 * inv_speed[c & 7], c};
  const auto later = [](const Free& a, const Free& b) { return a > b; };
  std::make_heap(heap.begin(), heap.end(), later);
  tail.assign((size_t)chains, -1);
  const int64_t per_block = (n_units + 8 * (int64_t)chains - 1) / (8 * (int64_t)chains);
  for (int64_t u0 = 0; u0 < n_units; u0 += per_block) {
    const int64_t u1 = std::min(n_units, u0 + per_block);
    std::pop_heap(heap.begin(), heap.end(), later);
    Free& f = heap.back();
    const int32_t c = f.second;
    int64_t cost = 0;
    for (int64_t u = u0; u < u1; ++u) {
      const DkItem& it = items[(size_t)(u / cfg.n_kv_heads)];
      cost += (int64_t)(it.kv_hi - it.kv_lo) + cfg.stream_item_cost;
      if (tail[c] < 0) {
        head[c] = tail[c] = (int32_t)u;
      } else if (row_blocks(it) > row_blocks(items[(size_t)(head[c] / cfg.n_kv_heads)])) {
        next[u] = head[c];
        head[c] = (int32_t)u;
      } else {
        next[tail[c]] = (int32_t)u;
        tail[c] = (int32_t)u;
      }
    }
    f.first += (double)cost * inv_speed[c & 7];
    std::push_heap(heap.begin(), heap.end(), later);
  }
}
// Work items of the tile kernel.  `slots` workgroups per KV head each walk a chain of items; an item is a row
// tile against a piece of its visible key range.  Costs are counted in key tiles: an item of n tiles takes
// n + item_cost (pipeline ramp, output store).
//   1. Pieces: with at least as many row tiles as workgroups nothing is cut; with fewer, every entry's key range
//      is cut into floor(slots / row tiles) equal chunks, the same boundaries for all row tiles of the entry --
//      the workgroups walking one chunk read the same K/V tiles at the same time and share them through L2.
//   2. Longest piece first, each to the chain that is free first (pieces of one (entry, chunk) group are equally
//      long, so they stay neighbours and start together).
//   3. Levelling: while the busiest chain is more than a few tiles above the idlest, the tail of one of its
//      pieces is cut off and handed to the idlest chain, sized so that the two end together.  This is what makes
//      the chains finish together whatever the mix of lengths; it costs one more item and the partial rows of
//      the row tile that was cut.
// Row tiles that end up in several pieces get partial rows and a merge record.  Items are emitted chain by chain.
void cut_tile_items(AttendPlan* p, const PlanConfig& cfg) {
  const std::vector<RowTile>& tiles = p->tile_tiles;
  p->tile_chains = 0;
  if (tiles.empty()) return;
  const int32_t kt = cfg.kv_tile;
  const int32_t slots = std::max(cfg.tile_wave_slots, 1);
  const int32_t fixed = std::max(cfg.tile_item_cost, 0);
  const int32_t min_piece = std::max<int32_t>(std::max<int32_t>(1, cfg.tile_min_chunk / kt), fixed);  // tiles
  const int32_t n_tiles = (int32_t)tiles.size();
  const auto len_of = [&](const PlanPiece& q) { return (q.hi - q.lo + kt - 1) / kt; };

  std::vector<PlanPiece>& pieces = p->pieces;
  pieces.clear();
  const int32_t k0 = n_tiles < slots ? slots / n_tiles : 1;
  for (int32_t b = 0; b < n_tiles;) {  // tiles of one entry are consecutive
    int32_t e = b, hi_max = 0;
    while (e < n_tiles && tiles[e].entry == tiles[b].entry) hi_max = std::max(hi_max, tiles[e++].kv_hi);
    const int32_t longest = (hi_max + kt - 1) / kt;
    const int32_t k = std::max(1, std::min(k0, longest / min_piece));
    const int32_t each = (longest + k - 1) / k * kt;  // keys per chunk
    for (int32_t t = b; t < e; ++t)
      for (int32_t lo = 0; lo < tiles[t].kv_hi;) {
        int32_t hi = std::min(tiles[t].kv_hi, lo + each);
        if (tiles[t].kv_hi - hi < each / 4) hi = tiles[t].kv_hi;  // no sliver at the end
        pieces.push_back({t, lo, hi, -1});
        lo = hi;
      }
    b = e;
  }

  std::vector<int32_t>& order = p->order;
  order.resize(pieces.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int32_t)i;
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
    const PlanPiece &a = pieces[x], &b = pieces[y];
    const int32_t la = len_of(a), lb = len_of(b);
    if (la != lb) return la > lb;
    if (tiles[a.tile].entry != tiles[b.tile].entry) return tiles[a.tile].entry < tiles[b.tile].entry;
    if (a.lo != b.lo) return a.lo < b.lo;
    return tiles[a.tile].row0 > tiles[b.tile].row0;
  });

  std::vector<int32_t>&head = p->chain_head, &tail = p->chain_tail;
  std::vector<int64_t>& load = p->chain_load;
  head.assign((size_t)slots, -1);
  tail.assign((size_t)slots, -1);
  load.assign((size_t)slots, 0);
  const auto append = [&](int32_t c, int32_t i) {
    if (tail[c] < 0) head[c] = i; else pieces[tail[c]].next = i;
    tail[c] = i;
    pieces[i].next = -1;
    load[c] += len_of(pieces[i]) + fixed;
  };
  {
    typedef std::pair<double, int32_t> Free;  // (time at which the chain is free, chain)
    std::vector<Free>& heap = p->heap;
    heap.resize((size_t)slots);
    for (int32_t c = 0; c < slots; ++c) heap[c] = {0.0, c};
    const auto later = [](const Free& a, const Free& b) { return a > b; };
    std::make_heap(heap.begin(), heap.end(), later);
    for (int32_t i : order) {
      std::pop_heap(heap.begin(), heap.end(), later);
      Free& f = heap.back();
      append(f.second, i);
      f.first = (double)load[f.second];
      std::push_heap(heap.begin(), heap.end(), later);
    }
  }

  for (int32_t round = 0; round < 4 * slots; ++round) {
    int32_t busy = 0, idle = 0;
    for (int32_t c = 1; c < slots; ++c) {
      if (load[c] > load[busy]) busy = c;
      if (load[c] < load[idle]) idle = c;
    }
    // tiles to hand over so that both chains end together (the new item pays its fixed cost on the idle chain)
    const int64_t give = (load[busy] - load[idle] - fixed) / 2;
    if (give < min_piece) break;
    int32_t donor = -1;  // the last piece of the busy chain that stays a piece after giving
    for (int32_t i = head[busy]; i >= 0; i = pieces[i].next)
      if (len_of(pieces[i]) >= give + min_piece) donor = i;
    if (donor < 0) break;
    const int32_t cut = pieces[donor].lo + (len_of(pieces[donor]) - (int32_t)give) * kt;
    pieces.push_back({pieces[donor].tile, cut, pieces[donor].hi, -1});
    pieces[donor].hi = cut;
    load[busy] -= give;
    append(idle, (int32_t)pieces.size() - 1);
  }

  // partial rows and merge records of the row tiles that were cut
  std::vector<int32_t>&count = p->tile_pieces, &part0 = p->tile_part0;
  count.assign((size_t)n_tiles, 0);
  part0.assign((size_t)n_tiles, -1);
  for (const PlanPiece& q : pieces) ++count[q.tile];
  for (int32_t t = 0; t < n_tiles; ++t)
    if (count[t] > 1) {
      part0[t] = (int32_t)p->part_rows;
      p->part_rows += (int64_t)count[t] * tiles[t].nrows;
      p->merges.push_back({tiles[t].entry, tiles[t].row0, tiles[t].nrows, part0[t], count[t], 0, {0, 0}});
      count[t] = 0;  // from here on: pieces of the tile emitted so far
    } else {
      count[t] = -1;
    }

  std::vector<int32_t>& links = p->tile_links;
  int32_t chains = 0;
  for (int32_t c = 0; c < slots; ++c) chains += head[c] >= 0;
  p->tile_chains = chains;
  links.assign((size_t)chains + pieces.size(), -1);
  int32_t cc = 0;
  for (int32_t c = 0; c < slots; ++c) {
    if (head[c] < 0) continue;
    links[cc++] = (int32_t)p->tile_items.size();
    for (int32_t i = head[c]; i >= 0; i = pieces[i].next) {
      const PlanPiece& q = pieces[i];
      const RowTile& t = tiles[q.tile];
      DkItem it{};
      it.entry = t.entry;
      it.row0 = t.row0;
      it.nrows = t.nrows;
      it.kv_lo = q.lo;
      it.kv_hi = q.hi;
      it.part_row0 = count[q.tile] < 0 ? -1 : part0[q.tile] + count[q.tile]++ * t.nrows;
      const int32_t idx = (int32_t)p->tile_items.size();
      p->tile_items.push_back(it);
      if (pieces[i].next >= 0) links[(size_t)chains + idx] = idx + 1;
    }
  }
}

// Small batches: what they take is latency, not bandwidth or arithmetic.  A unit of the streaming kernel costs a fixed
// part (descriptors, first requests, merge of the four wavefronts, store) and then 0.7 us per 128 keys with 32 rows, 1.3 with
// 96; so while every unit can have a compute unit of its own, short row tiles on many compute units beat long ones on few, and
// a turn of a few hundred rows often runs better here than in the tile kernel, which pays 9 us an item, 1.8 us per 64 keys and
// mostly a merge launch.  Rows and pieces are chosen entry by entry (small_shapes): a single height for the whole batch, as
// this was planned before, gives the short entries units that the long ones lack.  Measured, 32 query heads on 8 KV heads of
// 128 (us per step, one height and cut for all entries / entry by entry): 150 tokens on 4000 cached 39 / 26.5, on 8000
// 43.5 / 35, three sessions of 40-80 tokens on 1000-3000 30.6 / 20.1; one token on 3000 11.4 / 11.2.
// PlanConfig::unit_us and key_us have the kernel's measurements, in microseconds, and the plan of least estimated time is the
// candidate.  They are of 8 KV heads and keys that the caches hold; so in place of work of the tile kernel the candidate is
// only taken if step_us(), fitted over many shapes, has it cheaper too.  (64-wide heads and odd groups, block kernel / here:
// two turns of up to 450 tokens on 5000, 64-wide, 51.5 / 42; four of up to 370 on 3000, 16 heads on 4 of 64, 40 / 31.5;
// twelve of up to 60 on 8000, three heads to a KV head, 77 / 63; 16 of up to 110 on 4000, six heads to one, 48 / 41.  The
// general forms have unit and key prices of their own, but no fit of step_us().)
constexpr double kMergeUs = 4.0, kMergeRoundUs = 1.2;           // merge launch, and each round of eight splits that it reads
constexpr double kMergeInsideUs = 2.0, kMergeInsideSplitUs = 0.05;  // merge by the streaming kernel itself
constexpr int32_t kMergeInsideRows = 8, kMergeInsideParts = 64;  // most rows, and partial rows, of such a merge
// All compute units together: 8.7 TB/s with 128-wide heads, which is what the Infinity Cache and HBM give between them on
// batches of this size.  With the rate of HBM alone the planner left compute units idle that a batch could have used (us per
// step, at 10500 / 17000: one token on 8000 13.5 / 11.6, on 16000 19.2 / 16.5, three sessions of 7000-20000 38 / 36, four of
// 2000 13.8 / 11.2, six of 9000-20000 103 / 67, three of 2500-18000 with 64-wide heads 26.2 / 18.7).
constexpr double kKeysPerUs = 17000.0;
constexpr int32_t kMostSplits = 32;

// Batches of more K/V than the Infinity Cache holds (AttendPlan::once) come from HBM, and the units share what it gives: one
// alone takes 1.3 us for 64 KiB, so that half of the compute units do not reach HBM's rate, and a unit that is longer than the
// others goes on at its own pace when they have ended.  With the estimate above such batches were cut too little or too much
// (13 sessions of up to 27000 tokens, not cut because HBM seemed the limit, 264 us, 193 in 36 items; six sessions of up to
// 40000, 22 / 33 items, 139 / 183).  A further row tile of an entry costs little by itself -- its reads follow the first one's
// -- but the non-temporal loads are lost with it, and chains of two units end later than their lengths say.  Fitted to 189
// plans of 63 batches (4 to 30 sessions, 256-1500 MB, 1 to 32 new tokens, 64- and 128-wide heads, groups of three and four;
// 7 % off, root mean square, where the estimate above is 21 % off), of which it picks one 0.5 % slower than the best of three,
// on average.
constexpr double kHbmBytesPerUs = 6.5e6, kHbmUnitBytesPerUs = 65536 / 1.3, kReadAgain = 0.1, kReadCached = 1.1, kChained = 1.1;

// A streaming unit: a launch with it, and a piece of `keys` keys.
double key_us(const PlanConfig& cfg, bool hbm, int32_t blocks) {
  const double us = cfg.key_us[blocks - 1];
  return hbm ? std::max(us, 128.0 * 4.0 * cfg.head_dim / kHbmUnitBytesPerUs) : us;
}
double unit_us(const PlanConfig& cfg, bool hbm, int32_t blocks, double keys) {
  return cfg.unit_us[blocks - 1] + key_us(cfg, hbm, blocks) * keys / 128.0;
}

// How long units take that read from HBM side by side: while they ask for more than it gives, all are slowed down alike.
double shared_us(const PlanConfig& cfg, bool cached, std::vector<PlanLoad>* loads) {
  std::sort(loads->begin(), loads->end(), [](const PlanLoad& a, const PlanLoad& b) { return a.us < b.us; });
  const double rate = kHbmBytesPerUs / (4.0 * cfg.head_dim * cfg.n_kv_heads) / (cached ? kReadCached : 1.0);
  double demand = 0.0, us = 0.0, own = 0.0;
  for (const PlanLoad& l : *loads) demand += l.keys / l.us;
  for (const PlanLoad& l : *loads) {
    us += (l.us - own) * std::max(1.0, demand / rate);
    own = l.us;
    demand -= l.keys / l.us;
  }
  return us;
}

double merge_us(const PlanConfig& cfg, int32_t tile_rows, int64_t split) {
  if (split <= 1) return 0.0;
  const bool inside = cfg.arrivals > 0 && tile_rows <= kMergeInsideRows && split * tile_rows <= kMergeInsideParts;
  return inside ? kMergeInsideUs + kMergeInsideSplitUs * (double)split : kMergeUs + kMergeRoundUs * (double)((split + 7) / 8);
}

// Descriptor bytes of a plan, as build_plan lays them out (a queue's counter, never in the kernel arguments, left out).
size_t blob_size(const AttendPlan& p, bool with_cells, size_t tile_items, size_t tile_links, size_t stream_items, size_t stream_links,
                 size_t merges) {
  const auto part = [](size_t n, size_t each) { return align_up(n * each, 16); };
  return part(p.entries.size(), sizeof(DkEntry)) + part(p.segs.size(), sizeof(DkSeg)) + part(tile_items, sizeof(DkItem)) +
         part(tile_links, sizeof(int32_t)) + part(stream_items, sizeof(DkItem)) + part(stream_links, sizeof(int32_t)) +
         part(merges, sizeof(DkMerge)) + part(with_cells ? (size_t)p.total_tokens : 0, sizeof(int32_t));
}

// Workspace of a plan: its descriptors, then its partial rows.
size_t workspace_of(const PlanConfig& cfg, size_t blob_bytes, int64_t part_rows) {
  return align_up(align_up(blob_bytes, 256) + (size_t)part_rows * cfg.n_kv_heads * (cfg.head_dim + 2) * sizeof(float), 256) + 256;
}

// The best way to run the whole batch through the streaming kernel with at most one unit per workgroup and at most
// max_blob bytes of descriptors: every entry's row tiles get as many 32-row blocks, and its keys as many pieces, as it takes
// for no unit to last longer than the estimate, which is made as short as the number of workgroups allows -- short tiles for
// the entries with the most keys, wide ones for the others.  shapes[i]: of entry i.  Returns the estimate, 0 if there is none.
double small_shapes(AttendPlan& p, const PlanConfig& cfg, int32_t group, bool with_cells, size_t max_blob) {
  std::vector<PlanShape>&shapes = p.shapes, &trial = p.trial_shapes;
  int32_t most_rows = 0;
  int64_t all_keys = 0;
  for (const DkEntry& e : p.entries)
    if (e.delta > 0) {
      most_rows = std::max(most_rows, group * e.delta);
      all_keys += (int64_t)e.n + e.delta;
    }
  if (most_rows == 0 || (cfg.small_rows > 0 && most_rows > cfg.small_rows)) return 0.0;
  const int64_t most_items = std::min(cfg.small_units, cfg.stream_chains) / cfg.n_kv_heads;
  const double floor_us = cfg.unit_us[0] + (double)all_keys * cfg.n_kv_heads / kKeysPerUs;
  const double least_us = p.once ? 0.0 : floor_us;  // no estimate is below it: the search ends where it is reached
  const int32_t narrowest = std::min(3, (most_rows + 31) / 32);
  shapes.resize(p.entries.size());
  trial.resize(p.entries.size());
  // Shapes whose units last `us` at most: the fewest units for every entry.  Returns what they come to, 0 if they are too many.
  const auto fit = [&](double us, int32_t most_splits, std::vector<PlanShape>* out) {
    int64_t items = 0, merges = 0;
    double longest = 0.0, merge = 0.0;
    bool several = false;
    p.loads.clear();
    for (size_t i = 0; i < p.entries.size(); ++i) {
      const DkEntry& e = p.entries[i];
      if (e.delta <= 0) continue;
      const int64_t rows = (int64_t)group * e.delta;
      const double keys = (double)e.n + e.delta;
      PlanShape best;
      int64_t best_units = INT64_MAX;
      for (int32_t b = 1; b <= narrowest && (b == 1 || (b - 1) * 32 < rows); ++b) {
        const double room = (us - cfg.unit_us[b - 1]) * 128.0 / key_us(cfg, p.once, b);  // keys of a unit
        if (room < 1.0) continue;
        const int64_t split = std::max<int64_t>(1, (int64_t)std::ceil(keys / room));
        if (split > most_splits || (split > 1 && keys < 128.0 * (double)split)) continue;
        const int64_t units = (rows + 32 * b - 1) / (32 * b) * split;
        if (units < best_units || (p.once && units == best_units)) {  // (rather one row tile in two pieces than two tiles)
          best_units = units;
          best.rows = 32 * b;
          best.chunk = (int32_t)((((int64_t)e.n + e.delta + split - 1) / split + cfg.kv_tile - 1) / cfg.kv_tile * cfg.kv_tile);
        }
      }
      if (best.rows == 0) return 0.0;
      const int64_t split = ((int64_t)keys + best.chunk - 1) / best.chunk, tiles = (rows + best.rows - 1) / best.rows;
      items += tiles * split;
      merges += split > 1 ? tiles : 0;
      if (items > most_items) return 0.0;
      const double alone = unit_us(cfg, p.once, best.rows / 32, std::min(keys, (double)best.chunk));
      longest = std::max(longest, alone);
      several = several || tiles > 1;
      if (p.once) p.loads.push_back({alone, keys * (1.0 + kReadAgain * (double)(tiles - 1))});
      merge = std::max(merge, merge_us(cfg, (int32_t)std::min<int64_t>(rows, best.rows), split));
      (*out)[i] = best;
    }
    if (blob_size(p, with_cells, 0, 0, (size_t)items, 0, (size_t)merges) > max_blob) return 0.0;
    return (p.once ? shared_us(cfg, several, &p.loads) : std::max(longest, floor_us)) + merge;
  };
  double best_us = 0.0;
  for (const int32_t most_splits : {1, kMostSplits}) {
    // shortest duration that fits, to a few percent
    double lo = cfg.unit_us[0], hi = 0.0;
    for (const DkEntry& e : p.entries)
      if (e.delta > 0)
        hi = std::max(hi, unit_us(cfg, p.once, std::min<int32_t>(narrowest, (group * e.delta + 31) / 32), (double)e.n + e.delta));
    if (most_splits > 1) hi = std::min(hi, best_us > 0.0 ? best_us : hi);
    hi *= 1.001;
    for (int step = 0; step < 7; ++step) {
      const double us = step == 0 ? hi : 0.5 * (lo + hi);
      const double got = fit(us, most_splits, &trial);
      if (got > 0.0 && (best_us == 0.0 || got < best_us)) {
        best_us = got;
        shapes.swap(trial);
      }
      if (best_us > 0.0 && best_us <= least_us) return best_us;
      if (got > 0.0) hi = us;
      else if (step == 0) break;
      else lo = us;
    }
  }
  return best_us;
}

void unmark_once(AttendPlan* p) {
  for (DkSeg& s : p->segs) s.once = 0;
  p->once = false;
}

// Marks the segments that the streaming kernel may read past the caches (non-temporal loads): all that no two entries
// share, once the batch's cells are more than the Infinity Cache holds -- nothing of them can be there from an earlier
// call, and keeping them costs a tenth of the HBM rate.  Measured, us, cached / non-temporal: 64 verifying sessions of
// 4096-16384 tokens 416 / 372, 256 decoding ones of 512-8192 789 / 709; 64 sessions sharing 8192 of 8500 tokens 157 / 169.
// By the size of the K/V (decoding sessions of 4000 tokens; the same pass again and again, K/V that appends have just
// written, after 600 MB of other writes): 125 MB 27.7 / 31.4, 32.4 / 42.6, 60 / 35; 250 MB 43.6 / 49.8, 64.4 / 59.2, 104 / 54;
// 281 MB 48.7 / 50.9, 69.7 / 64.2, 112 / 55; 312 MB 54.4 / 53.1, 75.3 / 69.8, 119 / 57; 500 MB 96 / 87, 132 / 113, 160 / 90.
// A segment is taken for shared if another entry has one that starts at the same cell (an aliased prefix does).
void mark_once(AttendPlan* p, const PlanConfig& cfg) {
  int64_t cells = 0;
  size_t n = 0;
  for (const DkSeg& s : p->segs) cells += s.src == 0 ? s.len : 0;
  if (cfg.once_cells <= 0 || cells < cfg.once_cells) return;
  size_t size = 16;
  while (size < 2 * p->segs.size()) size *= 2;
  std::vector<int32_t>& table = p->seg_table;  // open addressing by start cell
  table.assign(size, -1);
  for (DkSeg& s : p->segs) {
    const int32_t i = (int32_t)n++;
    if (s.src != 0) continue;
    s.once = 1;
    size_t at = (size_t)((uint64_t)s.start * 0x9E3779B97F4A7C15ull >> 32) & (size - 1);
    while (table[at] >= 0 && p->segs[(size_t)table[at]].start != s.start) at = (at + 1) & (size - 1);
    if (table[at] < 0) {
      table[at] = i;
      continue;
    }
    DkSeg& other = p->segs[(size_t)table[at]];
    cells -= std::min(s.len, other.len);
    s.once = other.once = 0;
    if (s.len > other.len) table[at] = i;
  }
  p->once = true;
  if (cells < cfg.once_cells) unmark_once(p);
}

// Merging inside the streaming kernel: nothing else has split rows, every workgroup has one unit, every (row tile, KV
// head) a counter of its own, and the last workgroup of a row tile reads all of its partial rows in a round or two --
// one workgroup is slow with more (us per step, merge launch / inside: one token on 3000 cached 13.8 / 12.0, with 64-wide
// heads 13.9 / 10.8; 9 tokens, 36 rows, on 2000 13.7 / 20.0; 20 tokens on 4000 15 / 25).
bool merges_inside(const AttendPlan& p, const PlanConfig& cfg) {
  if (p.tile_chains > 0 || p.merges.empty() || p.merges.size() * (size_t)cfg.n_kv_heads > (size_t)cfg.arrivals ||
      (int64_t)p.stream_items.size() * cfg.n_kv_heads > std::max(cfg.stream_chains, 1))
    return false;
  for (const DkMerge& m : p.merges)
    if (m.nrows > kMergeInsideRows || m.nsplit * m.nrows > kMergeInsideParts) return false;
  return true;
}

bool one_tile_each(const AttendPlan& p) {  // no entry has more than one row tile
  for (const DkItem& it : p.stream_items)
    if (it.row0 > 0) return false;
  return true;
}

// The same estimate for the plan that the rules for large batches made.
double planned_us(AttendPlan& p, const PlanConfig& cfg) {
  double us = 0;
  if (p.tile_chains > 0) {
    const int64_t load = *std::max_element(p.chain_load.begin(), p.chain_load.end());
    us += cfg.row_fixed_us + cfg.row_step_us * (double)load;
  }
  if (!p.stream_items.empty()) {
    const int64_t units = (int64_t)p.stream_items.size() * cfg.n_kv_heads, chains = std::max(cfg.stream_chains, 1);
    if (p.once) {
      // the items of one KV head on its share of the workgroups, longest first, each where most room is (one row tile to an entry)
      const size_t room = (size_t)std::max<int64_t>(1, chains / cfg.n_kv_heads);
      const auto later = [](const PlanLoad& a, const PlanLoad& b) { return a.us > b.us; };
      p.loads.clear();
      for (const DkItem& it : p.stream_items) {
        const PlanLoad l{unit_us(cfg, true, row_blocks(it), it.kv_hi - it.kv_lo), (double)(it.kv_hi - it.kv_lo)};
        if (p.loads.size() < room) {
          p.loads.push_back(l);
        } else {
          std::pop_heap(p.loads.begin(), p.loads.end(), later);
          p.loads.back().us += l.us;
          p.loads.back().keys += l.keys;
        }
        std::push_heap(p.loads.begin(), p.loads.end(), later);
      }
      us += shared_us(cfg, false, &p.loads) * (units > chains ? kChained : 1.0);
    } else {
      double longest = 0;
      int64_t keys = 0;
      for (const DkItem& it : p.stream_items) {
        longest = std::max(longest, unit_us(cfg, false, row_blocks(it), it.kv_hi - it.kv_lo));
        keys += it.kv_hi - it.kv_lo;
      }
      longest *= (double)((units + chains - 1) / chains);  // (one after the other where the workgroups are fewer)
      us += std::max(longest, cfg.unit_us[0] + (double)keys * cfg.n_kv_heads / kKeysPerUs) * (units > chains ? kChained : 1.0);
    }
  }
  double merge = p.merges.empty() || p.tile_chains == 0 ? 0.0 : 7.0;
  if (p.tile_chains == 0)
    for (const DkMerge& m : p.merges) merge = std::max(merge, merge_us(cfg, m.nrows, m.nsplit));
  return us + merge;
}

// What a step of the plan's work items takes, with `blob` bytes of descriptors, by prices fitted to 2081 measured steps: 1 to
// 16 sessions of up to 16000 tokens with 1 to 300 new ones, groups of 1 to 16 query heads on 1 to 16 KV heads, planned with
// different numbers of units; 7 % off, root mean square.  The streaming kernel's prices are of its key loop before that became
// a pipeline, a fifth too high for three row blocks, and were fitted with one height to a batch.  Each unit is taken at its own
// height: with the price of the tallest on the keys of the longest, which mostly are two units, batches of mixed turns went to
// the tile kernel that are faster here (us per step, 14 sessions of up to 31 new tokens on 5700, 90.9 / 54.1, 11 of up to 47 on
// 4200, 68 / 38, four of up to 95 on 4000, 48 / 31; of 80 such batches 14 changed, none of them slower).
double step_us(const AttendPlan& p, const PlanConfig& cfg, size_t blob) {
  const PlanCost& c = cfg.cost;
  double us = blob > (size_t)cfg.inline_blob_bytes ? c.upload : 0.0;
  if (p.tile_chains > 0) {
    const int64_t load = *std::max_element(p.chain_load.begin(), p.chain_load.end());
    us += c.row_fixed + c.row_step * (double)load + c.row_items * (double)p.tile_items.size() * cfg.n_kv_heads / 256.0;
  }
  if (!p.stream_items.empty()) {
    double longest = 0;
    int64_t keys = 0, all = 0;  // keys: those of each entry once
    for (const DkItem& it : p.stream_items) {
      const int mb = row_blocks(it) - 1;
      longest = std::max(longest, c.unit[mb] + c.per128[mb] * (it.kv_hi - it.kv_lo) / 128.0);
      all += it.kv_hi - it.kv_lo;
      const DkEntry& e = p.entries[(size_t)it.entry];
      if (it.kv_hi == e.n + e.delta) keys += it.kv_hi;  // (the last piece of the entry's last row tile)
    }
    us += longest + (c.keys * (double)keys + c.again * (double)(all - keys)) * cfg.n_kv_heads * 1e-5;
  }
  if (!p.merges.empty()) {
    int32_t split = 0;
    for (const DkMerge& m : p.merges) split = std::max(split, m.nsplit);
    us += merges_inside(p, cfg) ? c.merge_inside + c.inside_split * split
                                : c.merge + c.split * split + c.parts * 1e-4 * (double)(p.part_rows * cfg.n_kv_heads) * cfg.head_dim / 128.0;
  }
  return us;
}

// Many short sessions on the general and fp32 routes: from some 35 of them on the descriptors no longer fit the kernel
// arguments, and the upload, with the host work that goes with it, costs a step more than the scalar kernel, whose descriptors
// have no items and no chains, loses on a few hundred keys (us a step with its append, matrix / scalar kernel: 40 sessions of
// 20 cached tokens, 24 query heads of 128 on 8, 23.9 / 15.8; 48 of 20, 32 heads of 64 on 8, 24.4 / 15.9; fp32, 4 heads of 64
// on 1, 40 of 20, 21.7 / 15.5; 200 of 200, 9 heads of 64, 61.5 / 26.1).  The prices are fitted to 1232 steps of 1 to 100
// sessions, up to 4 new tokens each, on either kernel; beyond that they hold while the scalar kernel's waves take few rounds
// (fp32, 400 sessions of 120 tokens, 2.8 rounds: 57.7 / 75.7; 128 of 60, 24 heads of 128 on 8, 3 rounds: 35.2 / 40.5).  Of 280
// batches of 34 to 400 sessions the scalar kernel gets 37 in staged mode, all of them 1.12 times faster or more by it, 1.56
// times on average, and 46 in appended mode, 1.3 times on average.  18 of the 280 stay more than 5 % slower than there (50 are
// without the rule), where prices that take them would also take some that the matrix kernels serve faster.
bool scalar_is_cheaper(const AttendPlan& p, const PlanConfig& cfg, size_t row_tiles, size_t stream_tiles) {
  const ScalarCost& c = cfg.scalar;
  if (c.launch == 0.f) return false;
  const size_t tiles = row_tiles + stream_tiles, units = stream_tiles * (size_t)cfg.n_kv_heads;
  const size_t chains = (size_t)std::max(cfg.stream_chains, 1), limit = (size_t)cfg.inline_blob_bytes;
  const size_t row_links = row_tiles ? row_tiles + std::min(row_tiles, (size_t)std::max(cfg.tile_wave_slots, 1)) : 0;
  const size_t stream_links = units > chains ? units + chains : 0;
  const size_t own = p.entries.size() * sizeof(DkEntry) + p.segs.size() * sizeof(DkSeg);
  if (own + tiles * sizeof(DkItem) + (row_links + stream_links) * sizeof(int32_t) <= limit) return false;
  const double rounds = (double)p.total_tokens * cfg.n_q_heads / (256.0 * (cfg.head_dim > 64 ? 4 : 9));
  if (rounds > c.rounds) return false;
  int64_t n = 0;
  for (const DkEntry& e : p.entries)
    if (e.delta > 0) n = std::max<int64_t>(n, (int64_t)e.n + e.delta);
  const double steps = (double)((n + 63) / 64), waves = (double)tiles * cfg.n_kv_heads / 256.0;
  return c.launch + c.step * steps + (c.round_step * steps + c.round) * rounds + (own > limit ? c.upload : 0.0) <
         c.matrix + c.wave * std::max(0.0, waves - 1.0) + (c.keys + c.wave_keys * waves) * (double)n / 128.0 + c.upload;
}
}  // namespace

int32_t build_plan(Pool& pool, const PlanConfig& cfg, int32_t n_seqs, const int32_t* slots, const int32_t* cu_delta,
                   bool staged, AttendPlan* p, bool with_cells) {
  int32_t rc = pool.check_batch(n_seqs, slots, cu_delta);
  if (rc != OK) return rc;
  p->entries.clear();
  p->segs.clear();
  p->tile_items.clear();
  p->stream_items.clear();
  p->merges.clear();
  p->stream_links.clear();
  p->stream_chains = 0;
  p->tile_links.clear();
  p->tile_chains = 0;
  p->part_rows = 0;
  p->total_tokens = n_seqs ? cu_delta[n_seqs] : 0;
  const int32_t group = cfg.n_q_heads / cfg.n_kv_heads;
  std::vector<Extent>& ext = p->ext;
  std::vector<RowTile>& tile_tiles = p->tile_tiles;
  std::vector<RowTile>& stream_tiles = p->stream_tiles;
  tile_tiles.clear();
  stream_tiles.clear();
  for (int32_t b = 0; b < n_seqs; ++b) {
    const int32_t delta = cu_delta[b + 1] - cu_delta[b];
    int64_t len = 0;
    rc = pool.extents_locked(slots[b], &ext, &len);
    if (rc != OK) return rc;
    if (!staged && delta > len) return ERR_INVALID;
    if (len + delta > INT32_MAX / 2) return ERR_UNSUPPORTED;
    DkEntry e{};
    e.seg_begin = (int32_t)p->segs.size();
    e.n = (int32_t)(staged ? len : len - delta);
    e.delta = delta;
    e.tok0 = cu_delta[b];
    if (delta > 0) {
      for (const Extent& x : ext) p->segs.push_back({x.cell, (int32_t)x.pos, (int32_t)x.len, 0, 0});
      if (staged) p->segs.push_back({(int64_t)cu_delta[b], e.n, delta, 1, 0});
    }
    e.seg_end = (int32_t)p->segs.size();
    p->entries.push_back(e);
    if (delta == 0 || !cfg.use_mfma) continue;
    const int32_t rows = group * delta;
    const int32_t ei = (int32_t)p->entries.size() - 1;
    if (rows <= cfg.stream_rows) {
      stream_tiles.push_back({ei, 0, rows, e.n + delta});
    } else {
      for (int32_t r0 = 0; r0 < rows; r0 += cfg.tile_rows) {
        const int32_t nr = std::min(cfg.tile_rows, rows - r0);
        const int32_t last_tok = (r0 + nr - 1) / group;
        tile_tiles.push_back({ei, r0, nr, e.n + last_tok + 1});
      }
    }
  }
  p->scalar = scalar_is_cheaper(*p, cfg, tile_tiles.size(), stream_tiles.size());
  if (p->scalar) {
    tile_tiles.clear();
    stream_tiles.clear();
  }
  if (!tile_tiles.empty() && !stream_tiles.empty()) {
    int64_t keys = 0;
    for (const RowTile& t : stream_tiles) keys += t.kv_hi;
    if (keys <= cfg.join_keys) {
      tile_tiles.insert(tile_tiles.end(), stream_tiles.begin(), stream_tiles.end());
      stream_tiles.clear();
    }
  }
  cut_tile_items(p, cfg);
  cut_stream_items(stream_tiles, cfg.kv_tile, cfg.stream_target, cfg.stream_min_chunk, &p->stream_items, &p->merges,
                   &p->part_rows);
  p->largest_bytes = 0;
  bool small = false;
  const bool may_be_small = !p->scalar && cfg.small_units > 0 && (int64_t)(tile_tiles.size() + stream_tiles.size()) * cfg.n_kv_heads <= cfg.small_units;
  p->once = false;
  if (may_be_small || !p->stream_items.empty()) mark_once(p, cfg);
  if (may_be_small) {
    // (a call whose descriptors travel in the kernel arguments goes on doing so)
    const size_t units = p->stream_items.size() * (size_t)cfg.n_kv_heads;
    const size_t chains = std::min(units, (size_t)std::max(cfg.stream_chains, 1));
    const size_t blob = blob_size(*p, with_cells, p->tile_items.size(), p->tile_links.size(), p->stream_items.size(),
                                  units == chains ? 0 : units + chains, p->merges.size());
    p->largest_bytes = workspace_of(cfg, blob, p->part_rows);
    // (no small plan has more partial rows than this, whatever its descriptors may come to)
    const int64_t most_items = std::min(cfg.small_units, cfg.stream_chains) / cfg.n_kv_heads;
    p->largest_bytes = std::max(p->largest_bytes, workspace_of(cfg, blob_size(*p, with_cells, 0, 0, (size_t)most_items, 0, (size_t)most_items),
                                                               std::min(most_items * 96, p->total_tokens * group * kMostSplits)));
    const double small_us = small_shapes(*p, cfg, group, with_cells,
                                         blob <= (size_t)cfg.inline_blob_bytes ? (size_t)cfg.inline_blob_bytes : SIZE_MAX);
    const double planned = small_us > 0.0 ? planned_us(*p, cfg) : 0.0;
    if (small_us > 0.0 && small_us < planned) {
      // (step_us() knows no HBM: there a plan that is clearly cheaper goes without it.  Of 56 such batches with work of the tile
      // kernel the 17 that this lets through are 1.06 to 1.4 times faster, of the seven closer ones three 5 to 11 % slower.)
      const bool clearly = p->once && small_us * 1.2 < planned;
      const bool weigh = !clearly && p->tile_chains > 0 && cfg.cost.row_step > 0.f;
      const double large_us = weigh ? step_us(*p, cfg, blob) : 0.0;
      const int32_t large_chains = p->tile_chains;
      const int64_t large_parts = p->part_rows;
      std::vector<RowTile>& small_tiles = p->small_tiles;
      small_tiles.clear();
      p->swap_spare();  // the plan made so far waits there
      p->stream_items.clear();
      p->merges.clear();
      p->tile_items.clear();
      p->tile_links.clear();
      p->tile_chains = 0;
      p->part_rows = 0;
      for (int32_t ei = 0; ei < (int32_t)p->entries.size(); ++ei) {
        const DkEntry& e = p->entries[ei];
        const int32_t rows = group * e.delta;
        small_tiles.clear();
        for (int32_t r0 = 0; r0 < rows; r0 += p->shapes[(size_t)ei].rows) {
          const int32_t nr = std::min(p->shapes[(size_t)ei].rows, rows - r0);
          small_tiles.push_back({ei, r0, nr, e.n + (r0 + nr - 1) / group + 1});
        }
        cut_stream_items(small_tiles, cfg.kv_tile, INT32_MAX, p->shapes[(size_t)ei].chunk, &p->stream_items, &p->merges, &p->part_rows);
      }
      if (!weigh || step_us(*p, cfg, blob_size(*p, with_cells, 0, 0, p->stream_items.size(), 0, p->merges.size())) < large_us) {
        small = true;
      } else {
        p->swap_spare();
        p->tile_chains = large_chains;
        p->part_rows = large_parts;
      }
    }
  }
  // (marked for one row tile per entry: nothing else reads the keys)
  if (p->once && (p->stream_items.empty() || (small && !one_tile_each(*p)))) unmark_once(p);
  for (DkMerge& m : p->merges) m.tok0 = p->entries[(size_t)m.entry].tok0;
  // Streaming units: with at least four units per workgroup they form a queue that the workgroups draw from at
  // run time (measured: +3-5 % on 700 decode slots, +1.5 % on 2048, because the compute units do not stream equally
  // fast; with two units per workgroup, as in a 64-slot verification batch, the queue has nothing to balance with
  // and the chains planned here are 1-2 % faster).  Not for a launch whose descriptors travel in the kernel
  // arguments (the queue's counter needs device memory) -- decided on a lower bound of the blob's size, and abi.hip
  // uploads every blob of a queued plan.
  p->stream_units = (int64_t)p->stream_items.size() * cfg.n_kv_heads;
  const size_t floor_bytes = p->entries.size() * sizeof(DkEntry) + p->segs.size() * sizeof(DkSeg) +
                             (p->tile_items.size() + p->stream_items.size()) * sizeof(DkItem);
  const int64_t per_wg = cfg.stream_queue == 2 ? 1 : 4;  // (2: queue whenever some workgroup gets a second unit)
  p->stream_queued = cfg.stream_queue != 0 && p->stream_units >= per_wg * (int64_t)std::max(cfg.stream_chains, 1) &&
                     p->stream_units > std::max(cfg.stream_chains, 1) && floor_bytes > (size_t)cfg.inline_blob_bytes;
  if (p->stream_queued) {
    p->stream_links.clear();
    p->stream_chains = (int32_t)std::min<int64_t>(p->stream_units, std::max(cfg.stream_chains, 1));
  } else {
    chain_units(p->stream_items, cfg, p->heap, p->tail, &p->stream_links, &p->stream_chains);
  }
  p->stream_single = !p->stream_queued && p->stream_units == p->stream_chains;
  p->stream_merges = p->stream_single && merges_inside(*p, cfg);

  size_t off = 0;
  p->off_entries = off;
  off = align_up(off + p->entries.size() * sizeof(DkEntry), 16);
  p->off_segs = off;
  off = align_up(off + p->segs.size() * sizeof(DkSeg), 16);
  p->off_tile = off;
  off = align_up(off + p->tile_items.size() * sizeof(DkItem), 16);
  p->off_tile_links = off;
  off = align_up(off + p->tile_links.size() * sizeof(int32_t), 16);
  p->off_stream = off;
  off = align_up(off + p->stream_items.size() * sizeof(DkItem), 16);
  p->off_links = off;
  if (!p->stream_single) off = align_up(off + p->stream_links.size() * sizeof(int32_t), 16);
  p->off_merges = off;
  off = align_up(off + p->merges.size() * sizeof(DkMerge), 16);
  p->off_queue = off;
  if (p->stream_queued) off += 16;
  p->off_cells = off;
  if (with_cells) off = align_up(off + (size_t)p->total_tokens * sizeof(int32_t), 16);
  p->blob_bytes = off;  // descriptors: small blobs travel in the kernel arguments, larger ones are uploaded
  p->off_parts = align_up(off, 256);
  p->total_bytes = workspace_of(cfg, p->blob_bytes, p->part_rows);
  p->largest_bytes = std::max(p->largest_bytes, p->total_bytes);
  return OK;
}

}  // namespace dk
