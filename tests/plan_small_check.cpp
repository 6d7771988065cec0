// Host check of what is planned for the batches of a pool, with the configuration that its shape gets (no GPU): on every route,
// as a small batch or by the rules for large ones, every (row, key) pair is covered once, split rows have a merge record
// with partial rows of their own, a call whose descriptors fit the kernel arguments still does, the streaming kernel merges
// only what its counters can count, short entries join the row-tile kernel whole, and no cells that two entries share are
// read past the caches.  Built and run by tests/test_host_plan_small.py.  Exits 0 when every check held.
#include <algorithm>
#include <cstdio>
#include <map>
#include <mutex>
#include <new>
#include <random>
#include <vector>

#include "../paper_2605_26289_amd/csrc/plan.hpp"

static int failures = 0;
#define CHECK(cond)                                               \
  do {                                                            \
    if (!(cond)) {                                                \
      ++failures;                                                 \
      std::printf("FAILED %s (line %d)\n", #cond, __LINE__);      \
    }                                                             \
  } while (0)

// A configuration made in storage that held something else, as a member of an object with a constructor of its own is:
// what its maker does not set is zero, not what the storage held.
struct Holder {
  int other;
  dk::PlanConfig cfg;
  explicit Holder(int o) : other(o) {}
};
static void check_fields_start_at_zero() {
  alignas(Holder) static unsigned char storage[sizeof(Holder)];
  for (unsigned char& b : storage) b = 0x5a;
  const Holder* h = new (storage) Holder(1);
  CHECK(h->cfg.join_keys == 0);
  CHECK(h->cfg.once_cells == 0);
  CHECK(h->cfg.arrivals == 0);
  CHECK(h->cfg.small_units == 0);
}

struct Shape {
  int hq, hkv, d;
  bool bf16;
  dk::Route route;
};
static const Shape kShapes[] = {
    {32, 8, 128, true, dk::Route::kTile},    {8, 2, 128, true, dk::Route::kTile},    {16, 16, 128, true, dk::Route::kTile},
    {16, 1, 128, true, dk::Route::kTile},    {4, 4, 128, true, dk::Route::kTile},    {32, 8, 64, true, dk::Route::kGeneral},
    {14, 2, 64, true, dk::Route::kGeneral},  {24, 8, 128, true, dk::Route::kGeneral}, {48, 3, 64, true, dk::Route::kGeneral},
    {32, 1, 128, true, dk::Route::kGeneral}, {4, 1, 64, false, dk::Route::kF32},     {32, 8, 128, false, dk::Route::kF32},
};

// Many short sessions: where they are planned for the scalar kernel there is nothing but entries and segments, the matrix
// kernels' plan of the same batch would not fit the kernel arguments, and its workspace is the larger one.
static void check_short_sessions() {
  std::mt19937 rng(11);
  auto uni = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int scalar[2] = {}, matrix[2] = {};
  for (int rep = 0; rep < 800; ++rep) {
    const Shape& sh = kShapes[rng() % (sizeof(kShapes) / sizeof(kShapes[0]))];
    const int nseq = uni(1, 100), top = uni(0, 1) ? uni(1, 60) : uni(1, 400), most = uni(0, 3);
    const bool staged = uni(0, 1);
    std::vector<int32_t> slots(nseq), cu(nseq + 1, 0);
    for (int b = 0; b < nseq; ++b) cu[b + 1] = cu[b] + (b == 0 ? 1 : uni(0, most));
    dk::Pool pool(nseq, 0, (int64_t)nseq * 512, 16);
    for (int b = 0; b < nseq; ++b) {
      CHECK(pool.acquire(0, 0, &slots[b]) == dk::OK);
      const int32_t c2[2] = {0, uni(std::max(1, most), std::max({1, most, top}))};
      std::vector<int64_t> dst;
      CHECK(pool.append(1, &slots[b], c2, nullptr, &dst) == dk::OK);
    }
    const dk::PlanConfig base = dk::default_config(sh.hq, sh.hkv, sh.d, sh.bf16);
    const dk::PlanConfig cfg = dk::route_config(base, sh.route, nseq, cu.data());
    const dk::PlanConfig ref = dk::route_config(base, dk::Route::kRef, nseq, cu.data());
    dk::PlanConfig never = cfg, off = base;
    never.scalar = dk::ScalarCost();
    off.small_units = 0;
    CHECK(dk::route_config(off, sh.route, nseq, cu.data()).scalar.launch == 0.f);
    dk::AttendPlan p, m, r;
    {
      std::lock_guard<std::mutex> g(pool.mutex());
      CHECK(dk::build_plan(pool, cfg, nseq, slots.data(), cu.data(), staged, &p) == dk::OK);
      CHECK(dk::build_plan(pool, never, nseq, slots.data(), cu.data(), staged, &m) == dk::OK);
      CHECK(dk::build_plan(pool, ref, nseq, slots.data(), cu.data(), staged, &r) == dk::OK);
    }
    CHECK(!m.scalar && !r.scalar && (!p.scalar || sh.route != dk::Route::kTile));
    if (m.blob_bytes <= 3072) CHECK(!p.scalar);
    ++(p.scalar ? scalar : matrix)[nseq > 35];
    if (!p.scalar) continue;
    CHECK(p.tile_items.empty() && p.stream_items.empty() && p.merges.empty() && p.tile_chains == 0 && p.stream_units == 0);
    CHECK(p.part_rows == 0 && !p.stream_queued && !p.once);
    CHECK(p.blob_bytes == r.blob_bytes && p.total_bytes == r.total_bytes && p.off_segs == r.off_segs);
    CHECK(p.entries.size() == r.entries.size() && p.segs.size() == r.segs.size() && p.total_tokens == r.total_tokens);
    CHECK(p.total_bytes <= m.total_bytes);
  }
  std::printf("short sessions: %d planned for the scalar kernel, %d for the others\n", scalar[1], matrix[1]);
  CHECK(scalar[1] > 40 && matrix[1] > 40 && matrix[0] > 40);
}

// Batches of more K/V than the caches hold are bound by the memory: a second row tile of an entry would read its keys again, and
// past no cache.  So nearly every entry that fits one row tile gets one, cut into pieces where the chip has room for them.
static void check_large_histories() {
  std::mt19937 rng(13);
  auto uni = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  const Shape shapes[] = {{32, 8, 128, true, dk::Route::kTile}, {8, 2, 128, true, dk::Route::kTile}, {24, 8, 128, true, dk::Route::kGeneral}};
  int seen = 0, several = 0, cached = 0;
  for (int rep = 0; rep < 1500; ++rep) {
    const Shape& sh = shapes[rep % 3];
    const int group = sh.hq / sh.hkv, nseq = uni(6, 30), most = 96 / group, delta = uni(1, most);
    const int64_t cells = ((int64_t)300 << 20) / (sh.hkv * 512);
    const int lo = (int)(cells / nseq), hi = uni(lo, 4 * lo);
    std::vector<int32_t> slots(nseq), cu(nseq + 1, 0);
    std::vector<int> n(nseq);
    for (int& x : n) x = uni(lo, hi);
    dk::Pool pool(nseq, 0, (int64_t)nseq * (hi + 1024), 256);
    for (int b = 0; b < nseq; ++b) {
      CHECK(pool.acquire(0, 0, &slots[b]) == dk::OK);
      const int32_t c2[2] = {0, n[b]};
      std::vector<int64_t> dst;
      CHECK(pool.append(1, &slots[b], c2, nullptr, &dst) == dk::OK);
      cu[b + 1] = cu[b] + delta;
    }
    const dk::PlanConfig cfg = dk::route_config(dk::default_config(sh.hq, sh.hkv, sh.d, sh.bf16), sh.route, nseq, cu.data());
    dk::AttendPlan p;
    {
      std::lock_guard<std::mutex> g(pool.mutex());
      CHECK(dk::build_plan(pool, cfg, nseq, slots.data(), cu.data(), true, &p) == dk::OK);
    }
    CHECK(p.tile_items.empty());
    ++seen;
    cached += !p.once;
    bool one = true;
    for (const DkItem& it : p.stream_items) one = one && it.row0 == 0;
    several += !one;
  }
  std::printf("more than the caches hold: %d batches, %d with several row tiles to an entry, %d read through the caches\n", seen, several, cached);
  CHECK(seen == 1500 && several <= 50 && cached <= 50);
}

// Turns of different length, the longest of more rows than a streaming unit takes: each unit is priced at its own height, so
// that nearly all of such batches are streamed as a whole.
static void check_mixed_heights() {
  std::mt19937 rng(17);
  auto uni = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int streamed = 0;
  for (int rep = 0; rep < 200; ++rep) {
    const int nseq = uni(8, 14), most = uni(26, 44);
    std::vector<int32_t> slots(nseq), cu(nseq + 1, 0);
    dk::Pool pool(nseq, 0, (int64_t)nseq * 6144, 256);
    for (int b = 0; b < nseq; ++b) {
      CHECK(pool.acquire(0, 0, &slots[b]) == dk::OK);
      const int32_t c2[2] = {0, uni(2000, 5000)};
      std::vector<int64_t> dst;
      CHECK(pool.append(1, &slots[b], c2, nullptr, &dst) == dk::OK);
      cu[b + 1] = cu[b] + (uni(0, 1) ? most : uni(most / 8, most));
    }
    const dk::PlanConfig cfg = dk::route_config(dk::default_config(32, 8, 128, true), dk::Route::kTile, nseq, cu.data());
    dk::AttendPlan p;
    std::lock_guard<std::mutex> g(pool.mutex());
    CHECK(dk::build_plan(pool, cfg, nseq, slots.data(), cu.data(), true, &p) == dk::OK);
    streamed += p.tile_items.empty();
  }
  std::printf("mixed turns: %d of 200 streamed as a whole\n", streamed);
  CHECK(streamed >= 190);
}

int main() {
  check_fields_start_at_zero();
  check_mixed_heights();
  check_short_sessions();
  check_large_histories();
  std::mt19937 rng(7);
  auto uni = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int small = 0, cut = 0, near = 0, inside = 0, joined = 0, once = 0, shared = 0;
  for (int rep = 0; rep < 6000; ++rep) {
    const Shape& sh = kShapes[rng() % (sizeof(kShapes) / sizeof(kShapes[0]))];
    const int hq = sh.hq, hkv = sh.hkv, group = hq / hkv;
    const bool big = uni(0, 3) == 0;  // enough cells to be read past the caches
    const int nseq = big ? uni(4, 24) : uni(1, 12);
    std::vector<int> n(nseq), delta(nseq);
    std::vector<int32_t> slots(nseq), cu(nseq + 1, 0);
    int64_t cells = 4096;
    const int prefix = nseq > 1 && uni(0, 2) == 0 ? uni(1, 2000) : 0;  // aliased by some of the others
    for (int b = 0; b < nseq; ++b) {
      n[b] = big ? uni(4000, 40000) : uni(0, 1) ? uni(0, 6000) : uni(0, 300);
      delta[b] = uni(0, 3) == 0 ? uni(0, 300) : uni(0, 20);
      cells += n[b] + prefix + 768;
      cu[b + 1] = cu[b] + delta[b];
    }
    dk::Pool pool(nseq, 0, cells, 256);
    const auto append = [&](int32_t slot, int count) {
      const int32_t c2[2] = {0, count};
      std::vector<int64_t> dst;
      if (count > 0) CHECK(pool.append(1, &slot, c2, nullptr, &dst) == dk::OK);
    };
    for (int b = 0; b < nseq; ++b) {
      CHECK(pool.acquire(0, 0, &slots[b]) == dk::OK);
      if (b == 0) append(slots[0], prefix);
      const bool alias = b > 0 && prefix > 0 && uni(0, 1);
      if (alias) CHECK(pool.alias(slots[0], slots[b], 0, prefix) == dk::OK);
      append(slots[b], n[b]);
      n[b] += b == 0 || alias ? prefix : 0;
    }
    const bool cells_too = uni(0, 1);
    dk::AttendPlan p, large;
    const dk::PlanConfig cfg = dk::route_config(dk::default_config(hq, hkv, sh.d, sh.bf16), sh.route, nseq, cu.data());
    dk::PlanConfig off = cfg;
    off.small_units = 0;
    {
      std::lock_guard<std::mutex> g(pool.mutex());
      CHECK(dk::build_plan(pool, cfg, nseq, slots.data(), cu.data(), true, &p, cells_too) == dk::OK);
      CHECK(dk::build_plan(pool, off, nseq, slots.data(), cu.data(), true, &large, cells_too) == dk::OK);
    }
    CHECK(p.largest_bytes >= p.total_bytes && p.largest_bytes >= large.total_bytes);
    const bool other = p.tile_items.size() != large.tile_items.size() || p.stream_items.size() != large.stream_items.size();
    small += other;
    if (other) CHECK(p.tile_items.empty() && p.stream_units <= 256 && p.stream_single && p.tile_chains == 0);
    if (large.blob_bytes <= 3072) CHECK(p.blob_bytes <= 3072);
    near += large.blob_bytes <= 3072 && large.blob_bytes > 3072 - 128;
    std::map<std::pair<int, int>, std::vector<DkItem>> cover;
    const int stream_rows = sh.d == 64 && !other ? 64 : 96;
    for (const DkItem& it : p.tile_items) {
      CHECK(it.nrows <= cfg.tile_rows && it.merge == 0);
      cover[{it.entry, it.row0}].push_back(it);
    }
    for (const DkItem& it : p.stream_items) {
      CHECK(it.nrows <= stream_rows && sh.route != dk::Route::kF32);
      cover[{it.entry, it.row0}].push_back(it);
    }
    std::vector<int> rows(nseq, 0);
    std::vector<char> part((size_t)p.part_rows, 0);
    size_t split = 0;
    for (auto& kv : cover) {
      auto& v = kv.second;
      std::sort(v.begin(), v.end(), [](const DkItem& a, const DkItem& b) { return a.kv_lo < b.kv_lo; });
      const int e = kv.first.first, row0 = kv.first.second, nr = v[0].nrows;
      rows[e] += nr;
      CHECK(v.front().kv_lo == 0 && v.back().kv_hi == n[e] + (row0 + nr - 1) / group + 1);
      for (size_t i = 1; i < v.size(); ++i) CHECK(v[i].kv_lo == v[i - 1].kv_hi && v[i].nrows == nr);
      split += v.size() > 1;
      for (const DkItem& it : v) {
        CHECK(it.kv_lo < it.kv_hi && (it.part_row0 >= 0) == (v.size() > 1));
        for (int r = 0; it.part_row0 >= 0 && r < nr; ++r) {
          CHECK(it.part_row0 + r < p.part_rows && !part[(size_t)(it.part_row0 + r)]);
          if (it.part_row0 + r < p.part_rows) part[(size_t)(it.part_row0 + r)] = 1;
        }
      }
    }
    CHECK(split == p.merges.size());
    cut += split > 0 && other;
    for (const DkMerge& m : p.merges) {
      const auto& v = cover[{m.entry, m.row0}];
      CHECK((int)v.size() == m.nsplit && v[0].nrows == m.nrows && m.tok0 == cu[m.entry]);
      std::vector<int> at;
      for (const DkItem& it : v) at.push_back(it.part_row0);
      std::sort(at.begin(), at.end());
      for (int s = 0; s < m.nsplit; ++s) CHECK(at[(size_t)s] == m.part_row0 + s * m.nrows);
    }
    for (int b = 0; b < nseq; ++b) CHECK(rows[b] == group * delta[b]);

    // merges inside the streaming kernel
    inside += p.stream_merges;
    if (p.stream_merges) {
      CHECK(p.stream_single && p.tile_chains == 0 && p.merges.size() * (size_t)hkv <= (size_t)dk::ARRIVALS_PER_SLICE);
      for (const DkItem& it : p.stream_items) {
        CHECK((it.merge != 0) == (it.part_row0 >= 0));
        if (it.merge == 0) continue;
        CHECK((size_t)(it.merge >> 8) < p.merges.size());
        const DkMerge& m = p.merges[(size_t)(it.merge >> 8) % p.merges.size()];
        CHECK(m.entry == it.entry && m.row0 == it.row0 && m.nrows == it.nrows && m.nsplit == (it.merge & 255) && m.part_row0 == it.part_base);
      }
    }
    // short entries beside long ones on the general route: all in the row-tile kernel, or all in the streaming kernel
    if (sh.route == dk::Route::kGeneral && !other && !p.tile_items.empty()) {
      std::vector<char> seen(nseq, 0);
      int64_t short_keys = 0;
      for (int b = 0; b < nseq; ++b)
        if (delta[b] > 0 && group * delta[b] <= cfg.stream_rows) short_keys += n[b] + delta[b];
      for (const DkItem& it : p.tile_items) seen[it.entry] = 1;
      for (int b = 0; b < nseq; ++b)
        if (delta[b] > 0 && group * delta[b] <= cfg.stream_rows) {
          CHECK((seen[b] != 0) == (short_keys <= cfg.join_keys));
          joined += seen[b];
        }
    }
    // non-temporal loads: arena cells of one entry only, in batches that exceed the caches
    std::map<int64_t, int> starts, lengths;
    int64_t marked = 0, distinct = 0;
    for (const DkSeg& s : p.segs)
      if (s.src == 0) {
        ++starts[s.start];
        lengths[s.start] = std::max(lengths[s.start], s.len);
      }
    for (const auto& kv : lengths) distinct += kv.second;
    for (const DkSeg& s : p.segs) {
      if (!s.once) continue;
      CHECK(s.src == 0 && starts[s.start] == 1);
      marked += s.len;
    }
    for (const auto& kv : starts) shared += kv.second > 1 && marked > 0;
    CHECK((marked > 0) <= p.once);
    if (p.once) CHECK(!p.stream_items.empty() && distinct >= cfg.once_cells);
    once += p.once;
  }
  std::printf("planned as small %d, cut %d, close below the limit of the kernel arguments %d, merged inside %d, joined %d, "
              "read past the caches %d, beside shared ones %d, failures %d\n", small, cut, near, inside, joined, once, shared, failures);
  CHECK(small > 400 && cut > 100 && near > 10 && inside > 20 && joined > 20 && once > 20 && shared > 20);
  return failures ? 1 : 0;
}
