// bf16 MFMA delta-prefill attention for the shapes the tile kernel does not serve: 64-wide heads, and groups of query
// heads per KV head that are no power of two up to 16 (gfx950, more packed rows than the stream kernel takes).
//
// A workgroup owns 128 packed query rows of one KV head (4 wavefronts x 32 rows) and walks the visible keys in 64-key
// tiles that the wavefronts share through an LDS ring (HBM -> LDS by global_load_lds_dwordx4, one barrier per tile).
// Two workgroups fit a compute unit (256 registers a lane, at most 64 KiB of LDS), so every SIMD holds two wavefronts:
// while one turns its scores into probabilities the other one's MFMAs run.  The products are transposed as in the tile
// kernel (S^T = K Q^T, O^T = V^T P^T, a lane owns one query row) and P never touches LDS.
//
// The probabilities enter the second product as hi + lo, two bf16 whose sum carries 16 bits of the fp32 weight: 16 S^T and
// 2 x 16 PV MFMAs per tile and wavefront with 128-wide heads, 8 and 2 x 8 with 64-wide ones.  That keeps the results as
// exact as those of the scalar fp32 kernel that served these shapes (1.7e-3 of the result's norm either way: the bf16
// store).  Bound by the softmax arithmetic and the split with 64-wide heads, by the MFMAs with 128-wide ones; in small
// batches by the chain of key steps of one item.  Measured, two 256-token chunks among 14 decoding or
// verifying sessions of 512-4096 tokens, 32 query heads on 8 KV heads of 64, all in this kernel: 50 us, 1630 in the scalar
// kernel; 80 MB read from beyond L2, which is each K/V row once, 15 MB written.
#include <hip/hip_runtime.h>

#include <mutex>

#include "attend_common.hpp"
#include "kernels.hpp"

namespace dk {
namespace mfma {

namespace {

constexpr int BLOCK_KT = 64;  // keys per tile
constexpr float BLOCK_RESCALE_SLACK = 8.f;  // log2 units, as in the tile kernel

template <int HD>
struct BlockGeo {
  static constexpr int TILE_BYTES = BLOCK_KT * Geo<HD>::ROW;       // K or V of one tile
  static constexpr int STAGE_BYTES = 2 * TILE_BYTES;
  static constexpr int STAGES = HD == 128 ? 2 : 4;                 // 64 KiB of LDS either way
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static constexpr int LOADS = STAGE_BYTES / 1024 / 4;             // 1 KiB requests per wavefront and tile
};

__device__ __forceinline__ float block_max3(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// LDS reads of this wavefront have returned; K/V requests stay in flight (no vmcnt wait here).
__device__ __forceinline__ void block_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace

// grid = n_chains * n_kv_heads: workgroup w serves KV head w % n_kv_heads (with 8 KV heads also its XCD, so the row
// tiles of a head share one L2) and walks chain w / n_kv_heads of the planner's items.
template <int HD, bool INLINE>
__global__ __launch_bounds__(256, 2) void attend_block_kernel(BlobArg<INLINE> blob, Ctx c, const int32_t* links,
                                                              int n_chains) {
  typedef Geo<HD> G;
  typedef BlockGeo<HD> B;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  (void)blob;
  touch_descs<INLINE>();
  c.entries = resolve_desc<INLINE>(c.entries);
  c.segs = resolve_desc<INLINE>(c.segs);
  c.items = resolve_desc<INLINE>(c.items);
  links = resolve_desc<INLINE>(links);
  const int g = blockIdx.x % c.n_kv_heads;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5;
  const uint32_t koff = k_lane_off<HD>(lane), voff = v_lane_off<HD>(lane);

  bool first = true;
  for (int item_idx = load_desc(links, blockIdx.x / c.n_kv_heads); item_idx >= 0;
       item_idx = load_desc(links, n_chains + item_idx)) {
    const DkItem it = load_desc(c.items, item_idx);
    const DkEntry e = load_desc(c.entries, it.entry);
    const int last_row = it.row0 + it.nrows - 1;
    const int row0 = it.row0 + wave * 32;
    const bool active = row0 <= last_row;
    const int row = min(row0 + (lane & 31), last_row);
    const int tok = row_token<true>(c, row);
    const int limit = e.n + tok;  // last visible position (bottom-right causal alignment)
    const int min_limit = e.n + row_token<true>(c, min(row0, last_row));
    const int max_limit = active ? e.n + row_token<true>(c, min(row0 + 31, last_row)) : -1;

    bf16x8 qf[G::KS];
    {
      const __bf16* qp = c.q + ((int64_t)(e.tok0 + tok) * c.n_q_heads + g * c.group + row_head<true>(c, row, tok)) * HD + 8 * h;
#pragma unroll
      for (int ks = 0; ks < G::KS; ++ks) qf[ks] = *(const bf16x8*)(qp + ks * 16);
    }

    KvCursor<G::ROW> cur{c.segs, e.seg_begin, e.seg_end, it.kv_lo, it.kv_hi};
    // tiles requested and not yet computed, oldest first: (valid rows, position of row 0)
    int cnt[B::STAGES] = {}, pos[B::STAGES] = {};
    int stage_wr = 0;
    KvTile t;
    auto request = [&](int slot) {  // the next tile of the range, if any, into the ring
      cnt[slot] = 0;
      if (!cur.next(c, g, BLOCK_KT, t)) return;
      cnt[slot] = t.cnt;
      pos[slot] = t.pos;
      char* kl = smem + stage_wr * B::STAGE_BYTES;
      char* vl = kl + B::TILE_BYTES;
#pragma unroll
      for (int b = 0; b < B::LOADS / 2; ++b) load_kib<false, HD>(t.k, t.stride, t.cnt, kl, b * 4 + wave, lane);
#pragma unroll
      for (int b = 0; b < B::LOADS / 2; ++b) load_kib<true, HD>(t.v, t.stride, t.cnt, vl, b * 4 + wave, lane);
      stage_wr = stage_wr + 1 == B::STAGES ? 0 : stage_wr + 1;
    };
    block_barrier();  // nobody reads the previous item's last tiles any more
#pragma unroll
    for (int s = 0; s < B::STAGES - 1; ++s) request(s);
    if (first) scatter_new_rows<INLINE, G::ROW>(c);
    first = false;
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) asm volatile("" ::"v"(qf[ks]));  // Q is waited for here, once

    f32x16 o[G::DB];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int db = 0; db < G::DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = 0.f;

    int stage_rd = 0;
    while (cnt[0] > 0) {
      // tile 0 of the queue has landed when only the younger tiles' requests are still out
      int younger = 0;
#pragma unroll
      for (int s = 1; s < B::STAGES - 1; ++s) younger += cnt[s] > 0;
      if (B::STAGES > 3 && younger == 2) wait_vmcnt<2 * B::LOADS>();
      else if (B::STAGES > 2 && younger == 1) wait_vmcnt<B::LOADS>();
      else wait_vmcnt<0>();
      block_barrier();  // landed for every wavefront, and the tile before it is finished everywhere
      request(B::STAGES - 1);
      const char* k_lds = smem + stage_rd * B::STAGE_BYTES;
      const char* v_lds = k_lds + B::TILE_BYTES;
      stage_rd = stage_rd + 1 == B::STAGES ? 0 : stage_rd + 1;
      const int tcnt = cnt[0], tpos = pos[0];
#pragma unroll
      for (int s = 0; s < B::STAGES - 1; ++s) {
        cnt[s] = cnt[s + 1];
        pos[s] = pos[s + 1];
      }
      if (tpos > max_limit) continue;  // no row of this wavefront sees the tile

      f32x16 s[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k_frag<HD>(k_lds, koff, kb, ks), qf[ks], s[kb], 0, 0, 0);
      // block_max3 is inline assembly, in front of which the compiler does not wait for the products as it does elsewhere
      // (a step of the two chunks and 14 sessions above: 57.5 us without the wait, 57.6 with it)
      asm volatile("s_nop 11" : "+v"(s[0]), "+v"(s[1]));

      if (tcnt < BLOCK_KT || tpos + BLOCK_KT - 1 > min_limit) {
        // accumulator r of key block kb is key 32 kb + 8 (r / 4) + 4 h + r % 4 of the tile
        const int lim = min(tcnt - 1, limit - tpos) - 4 * h;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (32 * kb + 8 * (r >> 2) + (r & 3) > lim) s[kb][r] = -INFINITY;
      }
      float mx = block_max3(s[0][0], s[1][0], s[0][1]);
      mx = fmaxf(mx, s[1][1]);
#pragma unroll
      for (int r = 2; r < 16; ++r) mx = block_max3(mx, s[0][r], s[1][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * c.c;
      // the reference maximum is only raised when the tile outgrows it by more than the slack
      if (__builtin_amdgcn_ballot_w64(mx > m + BLOCK_RESCALE_SLACK) != 0) {
        const float mn = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f(m - ((mn == -INFINITY) ? 0.f : mn));
        m = mn;
        l *= alpha;
#pragma unroll
        for (int db = 0; db < G::DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      }
      const float ms = (m == -INFINITY) ? 0.f : m;
      float rs[2] = {0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x8 hi, lo;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[j >> 1][8 * (j & 1) + 2 * w], c.c, -ms));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[j >> 1][8 * (j & 1) + 2 * w + 1], c.c, -ms));
          rs[w & 1] += p0 + p1;
          split_pair(p0, p1, hi, lo, w);
        }
#pragma unroll
        for (int db = 0; db < G::DB; ++db) {
          const bf16x8 v = read_v_frag<HD>(v_lds, voff, j, db);
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, hi, o[db], 0, 0, 0);
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, lo, o[db], 0, 0, 0);
        }
      }
      l += rs[0] + rs[1];
    }

    if (active) {
      const float lt[1] = {l + __shfl_xor(l, 32)}, mm[1] = {m};
#pragma unroll
      for (int db = 0; db < G::DB; ++db) {
        f32x4 quads[4];
#pragma unroll
        for (int r = 0; r < 16; ++r) quads[r >> 2][r & 3] = o[db][r];
        store_quads<HD, true>(c, e, it, g, wave * 32 + (lane & 31), db * 32 + 4 * h, quads, lt[0]);
      }
      store_ml<1, true>(c, e, it, g, wave * 32, lane, mm, lt);
      float z = 0.f;  // NaN if any of the row's sums is not finite
#pragma unroll
      for (int db = 0; db < G::DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) z = __builtin_fmaf(o[db][r], 0.f, z);
      const uint64_t bad = __builtin_amdgcn_ballot_w64(z != 0.f);
      if (bad != 0) {
#pragma unroll 1
        for (int db = 0; db < G::DB; ++db)  // (one at a time: all of them do not fit the registers)
          redo_rows<HD, true>(c, e, it, g, wave * 32, (uint32_t)(bad | bad >> 32), m, lt[0], lane, db, [](int) { return true; });
      }
    }
  }
}

namespace {

template <int HD, bool INLINE>
hipError_t launch_block(const BlobArg<INLINE>& blob, const Ctx& c, const int32_t* links, int32_t n_chains,
                        hipStream_t stream) {
  // once per process and instantiation, whatever thread or pool gets here first
  static std::once_flag once;
  static hipError_t status = hipSuccess;
  std::call_once(once, [] {
    status = hipFuncSetAttribute((const void*)attend_block_kernel<HD, INLINE>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, BlockGeo<HD>::LDS_BYTES);
  });
  if (status != hipSuccess) return status;
  const dim3 grid((unsigned)n_chains * (unsigned)c.n_kv_heads);
  attend_block_kernel<HD, INLINE><<<grid, 256, BlockGeo<HD>::LDS_BYTES, stream>>>(blob, c, links, n_chains);
  return hipGetLastError();
}

}  // namespace

}  // namespace mfma

hipError_t launch_attend_block(const AttendArgs& a, const DkItem* items, const int32_t* links, int32_t n_chains,
                               hipStream_t stream) {
  using namespace mfma;
  if (n_chains <= 0) return hipSuccess;
  if (a.arena.dtype != 1 || (a.arena.head_dim != 64 && a.arena.head_dim != 128)) return hipErrorInvalidValue;
  const Ctx c = make_ctx(a, items);
  if (a.inline_blob) {
    const BlobArg<true> blob{*a.inline_blob};
    return a.arena.head_dim == 64 ? launch_block<64>(blob, c, links, n_chains, stream)
                                  : launch_block<128>(blob, c, links, n_chains, stream);
  }
  const BlobArg<false> none{0};
  return a.arena.head_dim == 64 ? launch_block<64>(none, c, links, n_chains, stream)
                                : launch_block<128>(none, c, links, n_chains, stream);
}

}  // namespace dk
