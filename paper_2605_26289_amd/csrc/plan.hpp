// Host-side planning of one dk_delta_attend call: resolves every slot's logical view into
// segments, cuts the work into workgroup-sized items (with the key range split when there are
// too few query rows to fill the chip) and lays the descriptors out for upload.
#pragma once
#include <array>
#include <cstddef>
#include <cstdint>
#include <utility>
#include <vector>

#include "device_types.h"
#include "pool.hpp"

namespace dk {

// Which kernels carry an attention call.
enum class Route {
  kRef = 0,      // scalar reference kernel: variant 1, a scale that is not positive and finite, calls with room for no other,
             // many short sessions (ScalarCost), bf16 pools of 2^24 bytes of K a token and more
  kTile = 1,     // bf16, 128-wide heads, groups of 2^k <= 16 query heads: tile and stream kernels
  kGeneral = 2,  // bf16, any other shape: block kernel and the stream kernel's general form
  kF32 = 3,      // fp32 pools
};

// What a step costs, in microseconds.
struct PlanCost {
  float unit[3] = {}, per128[3] = {};  // streaming kernel, by row blocks of its widest tile: a launch, 128 keys of its longest unit
  float keys = 0, again = 0;           // 1e5 keys of one KV head that it reads: the first time, by further row tiles
  float row_fixed = 0, row_step = 0, row_items = 0;  // row-tile kernel: a launch, 64 keys of its longest chain, 256 (item, KV head)
  float merge = 0, parts = 0, split = 0;     // merge launch, 1e4 partial rows of 128, each split of the row tile cut most often
  float merge_inside = 0, inside_split = 0;  // merge inside the streaming kernel, each split
  float upload = 0;                                  // descriptors that do not fit the kernel arguments
};

// What a step of many short sessions takes on the scalar kernel and on the matrix kernels, in microseconds.
struct ScalarCost {
  float launch = 0, step = 0, round_step = 0, round = 0;  // scalar kernel: a launch, 64 keys of the longest row; per round: 64 keys, its start
  float matrix = 0, wave = 0, keys = 0, wave_keys = 0;    // matrix kernels: a launch, 256 units more, 128 keys; 128 keys per 256 units
  float upload = 0;                                       // descriptors that do not fit the kernel arguments
  float rounds = 0;                                       // most rounds of the scalar kernel's waves that the prices hold for
};

// Every field starts as zero ("never", "none"), however the object that holds it is made.
struct PlanConfig {
  int32_t n_q_heads = 0, n_kv_heads = 0, head_dim = 0;
  bool use_mfma = false;  // matrix kernels serve the call: work items are cut (the scalar kernel needs entries and segments only)
  int32_t tile_rows = 0;  // packed query rows per workgroup of the tile kernel
  int32_t stream_rows = 0;  // max packed rows handled by the streaming (small-Delta) kernel
  int32_t kv_tile = 0;  // keys per inner step; split boundaries are multiples of it
  int32_t tile_wave_slots = 0;  // tile-kernel workgroups of one KV head that run at a time (its share of the CUs)
  int32_t stream_target = 0;  // same, streaming kernel
  int32_t tile_min_chunk = 0, stream_min_chunk = 0;  // smallest key range worth its own item
  int32_t tile_item_cost = 0;  // fixed cost of a tile item inside a chain, in key tiles (store phase, pipeline ramp)
  int32_t stream_chains = 0;  // workgroups of the streaming kernel: one per compute unit
  int32_t stream_item_cost = 0;  // fixed cost of an item in the chain balance, in keys
  float xcd_speed[8] = {};  // relative K/V streaming rate of the XCD that workgroup w lands on (w % 8)
  int32_t stream_queue = 0;  // 1: streaming units are drawn from a queue at run time when the blob is uploaded
  int64_t join_keys = 0;  // short entries join the row-tile kernel's launch if they see at most this many keys (0: never)
  int64_t once_cells = 0;  // batches of at least this many cells are read past the caches (0: none are)
  float row_fixed_us = 0, row_step_us = 0;  // estimated cost of the row-tile kernel: a launch, and an item's 64-key step
  // estimated cost of a streaming unit, by its 32-row blocks: a launch, and 128 of its keys
  std::array<float, 3> unit_us = {}, key_us = {};
  PlanCost cost;  // prices by which plans of a small batch are weighed against the tile kernel's (row_step 0: they are not)
  ScalarCost scalar;  // prices by which short sessions go to the scalar kernel (launch 0: they do not)
  int32_t arrivals = 0;  // counters for merges inside the streaming kernel (0: none)
  int32_t small_units = 0;  // a batch of at most this many streaming units may be planned as a small one (0: never)
  int32_t small_rows = 0;   // ... unless an entry has more packed rows than this (0: however many)
  int32_t inline_blob_bytes = 0;  // a descriptor blob up to this size travels in the kernel arguments
};

// What a pool of this shape starts with, and what a call of a pool with the configuration cfg is planned by on route r
// (of a batch whose offsets have been checked).
PlanConfig default_config(int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, bool bf16);
PlanConfig route_config(const PlanConfig& cfg, Route r, int32_t n_seqs, const int32_t* cu_delta);

// One packed row tile of an entry before its key range is cut: rows [row0, row0 + nrows) see keys [0, kv_hi).
struct PlanRowTile {
  int32_t entry, row0, nrows, kv_hi;
};
// A piece of a row tile's key range on its way to becoming a work item of the tile kernel.
struct PlanPiece {
  int32_t tile;    // index of its row tile
  int32_t lo, hi;  // key positions
  int32_t next;    // next piece of the same chain, -1 at the end
};

// How an entry is cut for the streaming kernel in a small batch.
struct PlanShape {
  int32_t rows = 0;   // rows per tile: 32, 64 or 96
  int32_t chunk = 0;  // keys per unit
};

// Streaming units side by side: how long one takes alone, and the keys that all of the kind read.
struct PlanLoad {
  double us, keys;
};

// A plan object may be reused from call to call: build_plan() clears it but keeps the capacity of its
// vectors, so that planning a batch like the previous one only allocates what sorting and the check for
// slots that occur twice need.
struct AttendPlan {
  // working storage of build_plan
  std::vector<Extent> ext;
  std::vector<PlanRowTile> tile_tiles, stream_tiles, small_tiles;
  std::vector<std::pair<double, int32_t>> heap;
  std::vector<int32_t> tail;
  std::vector<PlanPiece> pieces;
  std::vector<int32_t> order, chain_head, chain_tail, tile_pieces, tile_part0;
  std::vector<int64_t> chain_load;
  std::vector<int32_t> seg_table;
  std::vector<PlanShape> shapes, trial_shapes;
  std::vector<PlanLoad> loads;

  std::vector<DkEntry> entries;
  std::vector<DkSeg> segs;
  std::vector<DkItem> tile_items, stream_items;
  std::vector<DkMerge> merges;
  // the work items of the plan for large batches while one for a small batch is weighed against it
  std::vector<DkItem> spare_tile_items, spare_stream_items;
  std::vector<DkMerge> spare_merges;
  std::vector<int32_t> spare_tile_links;
  void swap_spare() {
    std::swap(tile_items, spare_tile_items);
    std::swap(stream_items, spare_stream_items);
    std::swap(merges, spare_merges);
    std::swap(tile_links, spare_tile_links);
  }
  int64_t total_tokens = 0;
  int64_t part_rows = 0;
  // Streaming kernel: unit u = item u / n_kv_heads for KV head u % n_kv_heads.  Workgroup w walks the
  // chain stream_links[w], stream_links[n_chains + that unit], ... until a link is negative.
  std::vector<int32_t> stream_links;
  int32_t stream_chains = 0;
  // ... or, when stream_queued, starts with unit w and draws every further unit from a counter (off_queue, one
  // int32 that is uploaded holding stream_chains): the units are in longest-first order, no links are built.
  bool stream_queued = false;
  // ... or has one unit per workgroup, unit w for workgroup w: the links say nothing and are not part of the blob.
  bool stream_single = false;
  // The streaming kernel can merge the split rows itself (the workgroup that finishes the last split of a row tile does).
  bool stream_merges = false;
  bool once = false;  // some segments are marked DkSeg::once
  bool scalar = false;  // planned for the scalar kernel by PlanConfig::scalar: there are entries and segments only
  int64_t stream_units = 0;
  size_t off_queue = 0;
  // Tile kernel: tile_wave_slots workgroups per KV head, workgroup c of a head walks the items
  // tile_links[c], tile_links[tile_chains + that item], ...; the chains are the same for every KV head.
  std::vector<int32_t> tile_links;
  int32_t tile_chains = 0;
  size_t off_entries = 0, off_segs = 0, off_tile = 0, off_tile_links = 0, off_stream = 0, off_links = 0, off_merges = 0;
  size_t off_cells = 0;    // destination cell of every new token (int32), only when the plan was built with_cells
  size_t blob_bytes = 0;   // descriptors
  size_t off_parts = 0;    // fp32 partial rows, each (head_dim + 2) floats per KV head
  size_t total_bytes = 0;  // whole workspace
  // Whether a small batch is planned as one, and how it is then cut, depends on the size of its descriptors: on how many
  // segments its slots have, and on with_cells.  This is the largest workspace that a plan of the same batch comes to
  // whatever the outcome (up to the segments themselves).
  size_t largest_bytes = 0;
};

// Caller holds pool.mutex().  with_cells reserves, inside the descriptor blob, one int32 per new token for the
// cell it is to be written to (the call that appends and attends in one launch fills them in).
int32_t build_plan(Pool& pool, const PlanConfig& cfg, int32_t n_seqs, const int32_t* slots, const int32_t* cu_delta,
                   bool staged, AttendPlan* plan, bool with_cells = false);

}  // namespace dk
