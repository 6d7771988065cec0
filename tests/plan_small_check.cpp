// Host check of small batches (no GPU): planned as a small batch or by the rules for large ones, every (row, key) pair is
// covered once, split rows have a merge record with partial rows of their own, and a call whose descriptors fit the kernel
// arguments still does.  Built and run by tests/test_host_plan_small.py.  Exits 0 when every check held.
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

static dk::PlanConfig config(int hq, int hkv, int small) {
  dk::PlanConfig c{};
  c.n_q_heads = hq;
  c.n_kv_heads = hkv;
  c.head_dim = 128;
  c.use_mfma = true;
  c.tile_rows = 256;
  c.stream_rows = 96;
  c.kv_tile = 64;
  c.tile_wave_slots = c.stream_target = std::max(1, 256 / hkv);
  c.tile_min_chunk = 128;
  c.tile_item_cost = 5;
  c.stream_min_chunk = 512;
  c.stream_chains = 256;
  c.stream_item_cost = 512;
  for (float& x : c.xcd_speed) x = 1.f;
  c.stream_queue = 1;
  c.small_units = small;
  c.row_fixed_us = 10.f;
  c.row_step_us = 1.8f;
  c.unit_scale = 1.f;
  c.inline_blob_bytes = 3072;
  return c;
}

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

int main() {
  check_fields_start_at_zero();
  std::mt19937 rng(7);
  auto uni = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int small = 0, cut = 0, near = 0;
  for (int rep = 0; rep < 4000; ++rep) {
    static const int heads[][2] = {{32, 8}, {8, 2}, {16, 16}, {16, 1}, {4, 4}, {48, 3}};
    const int* hh = heads[rng() % 6];
    const int hq = hh[0], hkv = hh[1], group = hq / hkv, nseq = uni(1, 12);
    std::vector<int> n(nseq), delta(nseq);
    std::vector<int32_t> slots(nseq), cu(nseq + 1, 0);
    int64_t cells = 4096;
    for (int b = 0; b < nseq; ++b) {
      n[b] = uni(0, 1) ? uni(0, 6000) : uni(0, 300);
      delta[b] = uni(0, 3) == 0 ? uni(0, 300) : uni(0, 20);
      cells += n[b] + 512;
      cu[b + 1] = cu[b] + delta[b];
    }
    dk::Pool pool(nseq, 0, cells, 256);
    for (int b = 0; b < nseq; ++b) {
      CHECK(pool.acquire(0, 0, &slots[b]) == dk::OK);
      const int32_t c2[2] = {0, n[b]};
      std::vector<int64_t> dst;
      if (n[b] > 0) CHECK(pool.append(1, &slots[b], c2, nullptr, &dst) == dk::OK);
    }
    const bool cells_too = uni(0, 1);
    dk::AttendPlan p, large;
    {
      std::lock_guard<std::mutex> g(pool.mutex());
      CHECK(dk::build_plan(pool, config(hq, hkv, 256), nseq, slots.data(), cu.data(), true, &p, cells_too) == dk::OK);
      CHECK(dk::build_plan(pool, config(hq, hkv, 0), nseq, slots.data(), cu.data(), true, &large, cells_too) == dk::OK);
    }
    const bool other = p.tile_items.size() != large.tile_items.size() || p.stream_items.size() != large.stream_items.size();
    small += other;
    if (other) CHECK(p.tile_items.empty() && p.stream_units <= 256 && p.stream_single && p.tile_chains == 0);
    if (large.blob_bytes <= 3072) CHECK(p.blob_bytes <= 3072);
    near += large.blob_bytes <= 3072 && large.blob_bytes > 3072 - 128;
    std::map<std::pair<int, int>, std::vector<DkItem>> cover;
    for (const DkItem& it : p.tile_items) cover[{it.entry, it.row0}].push_back(it);
    for (const DkItem& it : p.stream_items) {
      CHECK(it.nrows <= 96);
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
      CHECK((int)v.size() == m.nsplit && v[0].nrows == m.nrows);
      std::vector<int> at;
      for (const DkItem& it : v) at.push_back(it.part_row0);
      std::sort(at.begin(), at.end());
      for (int s = 0; s < m.nsplit; ++s) CHECK(at[(size_t)s] == m.part_row0 + s * m.nrows);
    }
    for (int b = 0; b < nseq; ++b) CHECK(rows[b] == group * delta[b]);
  }
  CHECK(small > 400 && cut > 100 && near > 10);
  std::printf("planned as small %d, cut %d, close below the limit of the kernel arguments %d, failures %d\n", small, cut, near, failures);
  return failures ? 1 : 0;
}
