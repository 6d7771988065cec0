// fp32 delta-prefill attention on the fp32 matrix instructions (gfx950, head_dim 64 and 128, any group of query heads).
//
// Transposed products as in the bf16 kernels, with v_mfma_f32_16x16x4_f32: S^T = K Q^T over blocks of 16 keys and 16 packed
// query rows, O^T += V^T P^T, a lane owning one query row (column l % 16 of every result), so that the probabilities leave
// the first product in the layout the second one takes as its B operand.  Everything is fp32; which depth or key a lane's
// operand element stands for is free as long as both operands agree, and is chosen so that K, V and Q come straight from
// memory in 16-byte pieces, 64 bytes of a K row or a whole 256 bytes of a V row together:
//   K, Q   element 4 i + j of quarter-wave h (h = l / 16) is depth 16 i + 4 h + j
//   S^T    accumulator r of quarter-wave h is key 4 h + r of the block, and so is the operand of PV product r
//   V      element 4 u + j of lane column m (m = l % 16) is depth 64 u + 4 m + j: result block 4 u + j of O^T
// There is no LDS in the key loop: a 16x16x4 product takes 32 cycles for 8 bytes of operands a lane, so the caches keep up,
// and V of a block travels under its S^T, the next block's K under its softmax and PV.
//
// A workgroup is 8 wavefronts that split the keys of one item (16 RB packed rows of one KV head) and merge their states
// through LDS.  RB = 2 halves the K/V traffic and is taken when 32-row items still fill the chip; with fewer rows RB = 1
// keeps more compute units busy.  Bound by the fp32 matrix rate (153 TFLOP/s for a large product) in long turns, by HBM in
// decoding, by the chain of blocks of one wavefront in small calls.  Measured against the scalar kernel: one 150-token turn
// of 4 heads of 64 on 200 tokens 10.9 us (19.7, kernel time); four turns of up to 300 tokens of 32 heads of 128 on ~1750
// tokens 197 us (4390); 16 decoding sessions of 4000-8000 tokens, same heads, 163 us (1214); error against float64
// 2.3-4.3e-7 of the result's norm (3.3-4.7e-7).
#include <hip/hip_runtime.h>

#include <mutex>

#include "attend_common.hpp"
#include "kernels.hpp"

namespace dk {
namespace mfma {

namespace {

constexpr int F32_WAVES = 8;
constexpr int F32_KT = 16;                 // keys per block
constexpr float F32_RESCALE_SLACK = 8.f;   // log2 units, as in the bf16 kernels

template <int HD, int RB>
struct F32Geo {
  static constexpr int ROW = 4 * HD;       // bytes
  static constexpr int NI = HD / 16;       // 16-byte pieces of a K or Q row per lane; 16-row blocks of O^T
  static constexpr int NU = HD / 64;       // 16-byte pieces of a V row per lane
  static constexpr int QUADS = RB * NI;    // fp32 quads of O^T per lane
  static constexpr int ML_OFFSET = F32_WAVES * QUADS * 64 * 16;
  static constexpr int LDS_BYTES = ML_OFFSET + F32_WAVES * RB * 16 * 8;
};

// redo_rows for fp32: rows rl0 .. rl0 + 15 of the item (m and l of row rl0 + i in the lanes of column i), the depths
// 64 u + 4 (4 h + r) .. + 3 that this wavefront has stored.
template <int HD>
__device__ __forceinline__ void redo_quad(const Ctx& c, const DkEntry& e, const DkItem& it, int g, int rl0, uint32_t bad, float m, float l,
                                          int lane, int u, int r) {
  constexpr int ROW = 4 * HD, NI = HD / 16;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // after the ordinary store of the same rows
  const int col = lane & 15, h = lane >> 4;
  const int last_row = it.row0 + it.nrows - 1;
  const int row = min(it.row0 + rl0 + col, last_row);
  const int tok = row_token<true>(c, row);
  const int limit = e.n + tok;
  const int64_t orow = (int64_t)(e.tok0 + tok) * c.n_q_heads + g * c.group + row_head<true>(c, row, tok);
  f32x4 qf[NI], o[4];
  NonFinite nf[4];
#pragma unroll
  for (int i = 0; i < NI; ++i) qf[i] = *(const f32x4*)((const float*)c.q + orow * HD + 16 * i + 4 * h);
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int max_limit = e.n + row_token<true>(c, min(it.row0 + rl0 + 15, last_row));
  KvCursor<ROW> cur{c.segs, e.seg_begin, e.seg_end, it.kv_lo, min(it.kv_hi, max_limit + 1)};
  KvTile t;
  while (cur.next(c, g, F32_KT, t)) {
    const char* kp = t.k + (uint32_t)min(col, t.cnt - 1) * t.stride + 16 * h;
    f32x4 kf[NI], vf[4];
#pragma unroll
    for (int i = 0; i < NI; ++i) kf[i] = *(const f32x4*)(kp + 64 * i);
#pragma unroll
    for (int k = 0; k < 4; ++k) vf[k] = *(const f32x4*)(t.v + (uint32_t)min(4 * h + k, t.cnt - 1) * t.stride + 16 * col + 256 * u);
    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][j], qf[i][j], s[j & 1], 0, 0, 0);
    const int lim = min(t.cnt - 1, limit - t.pos) - 4 * h;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][k] + s[1][k], c.c, -m));
      if (k > lim) p = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool odd = nf[j].see(__float_as_uint(vf[k][j]), t.pos + min(4 * h + k, t.cnt - 1));
        o[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? 0.f : vf[k][j], p, o[j], 0, 0, 0);
      }
    }
  }
  f32x4 x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    nf[j].merge_lanes(16);
    nf[j].merge_lanes(32);
    const float sum = r == 0 ? o[j][0] : r == 1 ? o[j][1] : r == 2 ? o[j][2] : o[j][3];
    x[j] = nf[j].of_lane(4 * h + r).apply(sum, limit);
  }
  if ((bad >> col & 1) == 0 || rl0 + col >= it.nrows || l != l) return;
  const int depth = 64 * u + 4 * (4 * h + r);
  if (it.part_row0 >= 0) *(f32x4*)(c.parts + ((int64_t)(it.part_row0 + rl0 + col) * c.n_kv_heads + g) * HD + depth) = x;
  else *(f32x4*)((float*)c.out + orow * HD + depth) = x * (1.f / l);
}

}  // namespace

// grid = n_chains * n_kv_heads, as the tile kernel: workgroup w walks chain w / n_kv_heads of the planner's items.
template <int HD, int RB, bool INLINE>
__global__ __launch_bounds__(64 * F32_WAVES, 2) void attend_f32_kernel(BlobArg<INLINE> blob, Ctx c, const int32_t* links,
                                                                       int n_chains) {
  typedef F32Geo<HD, RB> G;
  constexpr int NI = G::NI, NU = G::NU;
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
  const int col = lane & 15, h = lane >> 4;
  f32x4* xo = (f32x4*)smem;                      // [wave][quad][lane]
  float2* xml = (float2*)(smem + G::ML_OFFSET);  // [wave][row]: running maximum, weight sum

  bool first = true;
  for (int item_idx = load_desc(links, blockIdx.x / c.n_kv_heads); item_idx >= 0;
       item_idx = load_desc(links, n_chains + item_idx)) {
    const DkItem it = load_desc(c.items, item_idx);
    const DkEntry e = load_desc(c.entries, it.entry);
    const int last_row = it.row0 + it.nrows - 1;
    const int min_limit = e.n + row_token<true>(c, it.row0);  // last position the item's first row sees

    f32x4 qf[RB][NI];
    int limit[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int row = min(it.row0 + rb * 16 + col, last_row);
      const int tok = row_token<true>(c, row);
      limit[rb] = e.n + tok;
      const float* qp = (const float*)c.q + ((int64_t)(e.tok0 + tok) * c.n_q_heads + g * c.group + row_head<true>(c, row, tok)) * HD + 4 * h;
#pragma unroll
      for (int i = 0; i < NI; ++i) qf[rb][i] = *(const f32x4*)(qp + 16 * i);
    }

    // this wavefront's share of the item's keys
    const int blocks = (it.kv_hi - it.kv_lo + F32_KT - 1) / F32_KT;
    const int per = (blocks + F32_WAVES - 1) / F32_WAVES * F32_KT;
    const int lo = min(it.kv_hi, it.kv_lo + wave * per);
    KvCursor<G::ROW> cur{c.segs, e.seg_begin, e.seg_end, lo, min(it.kv_hi, lo + per)};
    KvTile t;
    f32x4 kf[NI], vf[4][NU];
    // rows past the end of a ragged block re-read the last valid one; their scores are masked
    const auto load_k = [&]() __attribute__((always_inline)) {
      const char* p = t.k + (uint32_t)min(col, t.cnt - 1) * t.stride + 16 * h;
#pragma unroll
      for (int i = 0; i < NI; ++i) kf[i] = *(const f32x4*)(p + 64 * i);
    };
    const auto load_v = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const char* p = t.v + (uint32_t)min(4 * h + r, t.cnt - 1) * t.stride + 16 * col;
#pragma unroll
        for (int u = 0; u < NU; ++u) vf[r][u] = *(const f32x4*)(p + 256 * u);
      }
    };
    bool have = cur.next(c, g, F32_KT, t);
    if (have) load_k();
    if (first) scatter_new_rows<INLINE, G::ROW, 64 * F32_WAVES>(c);
    first = false;

    f32x4 o[RB][NI];
    float m[RB], l[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      m[rb] = -INFINITY;
      l[rb] = 0.f;
#pragma unroll
      for (int b = 0; b < NI; ++b) o[rb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    while (have) {
      const int cnt = t.cnt, pos = t.pos;
      load_v();
      __builtin_amdgcn_sched_barrier(0);
      constexpr int CH = 2;  // two chains per score: shorter ones round less, and products of one row need not wait in line
      f32x4 s[RB][CH];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) s[rb][0] = s[rb][CH - 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            s[rb][j % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][j], qf[rb][i][j], s[rb][j % CH], 0, 0, 0);
      have = cur.next(c, g, F32_KT, t);
      if (have) load_k();
      __builtin_amdgcn_sched_barrier(0);

      bool grow = false;
      float mx[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        s[rb][0] = s[rb][0] + s[rb][1];
        if (cnt < F32_KT || pos + F32_KT - 1 > min_limit) {
          const int lim = min(cnt - 1, limit[rb] - pos) - 4 * h;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (r > lim) s[rb][0][r] = -INFINITY;
        }
        mx[rb] = fmaxf(fmaxf(s[rb][0][0], s[rb][0][1]), fmaxf(s[rb][0][2], s[rb][0][3])) * c.c;
        grow |= mx[rb] > m[rb] + F32_RESCALE_SLACK;
      }
      // The reference maximum of a row is only raised when a score outgrows it by more than the slack, so the four
      // lanes of a row need not exchange their maxima for every block.
      if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          float v = fmaxf(mx[rb], __shfl_xor(mx[rb], 16));
          v = fmaxf(v, __shfl_xor(v, 32));
          const float mn = fmaxf(m[rb], v);
          const float alpha = __builtin_amdgcn_exp2f(m[rb] - ((mn == -INFINITY) ? 0.f : mn));
          m[rb] = mn;
          l[rb] *= alpha;
#pragma unroll
          for (int b = 0; b < NI; ++b) o[rb][b] *= alpha;
        }
      }
      f32x4 p[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float ms = (m[rb] == -INFINITY) ? 0.f : m[rb];  // no key seen yet: keep the arithmetic finite
#pragma unroll
        for (int r = 0; r < 4; ++r) p[rb][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][0][r], c.c, -ms));
        l[rb] += (p[rb][0] + p[rb][1]) + (p[rb][2] + p[rb][3]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              o[rb][4 * u + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][u][j], p[rb][r], o[rb][4 * u + j], 0, 0, 0);
    }

    // ---- merge the wavefronts' states: quad (rb, u, r) of a lane is depths 64 u + 4 (4 h + r) .. + 3 of row rb * 16 + col
    // (the lane number is laundered so that the per-lane offsets of this part are computed here instead of being hoisted
    // out of the item loop, where they would sit in registers the key loop needs)
    int el = lane;
    asm volatile("" : "+v"(el));
    const int ecol = el & 15, eh = el >> 4;
    __syncthreads();  // the previous item's exchange has been read
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float lt = l[rb] + __shfl_xor(l[rb], 16);
      lt += __shfl_xor(lt, 32);
      if (el < 16) xml[(wave * RB + rb) * 16 + el] = make_float2(m[rb], lt);
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          xo[((wave * RB + rb) * NI + u * 4 + r) * 64 + el] =
              f32x4{o[rb][4 * u][r], o[rb][4 * u + 1][r], o[rb][4 * u + 2][r], o[rb][4 * u + 3][r]};
    }
    __syncthreads();
    for (int quad = wave; quad < G::QUADS; quad += F32_WAVES) {
      const int rb = quad / NI, u = (quad % NI) >> 2, r = quad & 3;
      const int rl = rb * 16 + ecol;
      float2 ml[F32_WAVES];
      float mm = -INFINITY;
#pragma unroll
      for (int w = 0; w < F32_WAVES; ++w) {
        ml[w] = xml[(w * RB + rb) * 16 + ecol];
        mm = fmaxf(mm, ml[w].x);
      }
      const float ms = (mm == -INFINITY) ? 0.f : mm;
      float lsum = 0.f;
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < F32_WAVES; ++w) {
        const float f = __builtin_amdgcn_exp2f(ml[w].x - ms);
        lsum += f * ml[w].y;
        acc += f * xo[(w * G::QUADS + quad) * 64 + el];
      }
      const bool finite = acc[0] * 0.f + acc[1] * 0.f + acc[2] * 0.f + acc[3] * 0.f == 0.f;
      uint64_t bad = __builtin_amdgcn_ballot_w64(!finite && rl < it.nrows);
      const int depth = 64 * u + 4 * (4 * eh + r);
      if (rl >= it.nrows) {
      } else if (it.part_row0 >= 0) {
        const int64_t prow = (int64_t)(it.part_row0 + rl) * c.n_kv_heads + g;
        *(f32x4*)(c.parts + prow * HD + depth) = acc;
        if (u == 0 && r == 0 && eh == 0) *(float2*)(c.parts_ml + prow * 2) = make_float2(mm, lsum);
      } else {
        const int row = it.row0 + rl;
        const int tok = row_token<true>(c, row);
        const int64_t orow = (int64_t)(e.tok0 + tok) * c.n_q_heads + g * c.group + row_head<true>(c, row, tok);
        *(f32x4*)((float*)c.out + orow * HD + depth) = acc * (1.f / lsum);
        if (c.lse && u == 0 && r == 0 && eh == 0) c.lse[orow] = (mm + log2f(lsum)) * 0.6931471805599453f;
      }
      if (bad != 0) {
        bad |= bad >> 32;
        redo_quad<HD>(c, e, it, g, rb * 16, (uint32_t)(bad | bad >> 16) & 0xffffu, mm, lsum, el, u, r);
      }
    }
  }
}

namespace {

template <int HD, int RB, bool INLINE>
hipError_t launch_f32(const BlobArg<INLINE>& blob, const Ctx& c, const int32_t* links, int32_t n_chains,
                      hipStream_t stream) {
  // once per process and instantiation, whatever thread or pool gets here first
  static std::once_flag once;
  static hipError_t status = hipSuccess;
  std::call_once(once, [] {
    status = hipFuncSetAttribute((const void*)attend_f32_kernel<HD, RB, INLINE>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, F32Geo<HD, RB>::LDS_BYTES);
  });
  if (status != hipSuccess) return status;
  const dim3 grid((unsigned)n_chains * (unsigned)c.n_kv_heads);
  attend_f32_kernel<HD, RB, INLINE><<<grid, 64 * F32_WAVES, F32Geo<HD, RB>::LDS_BYTES, stream>>>(blob, c, links, n_chains);
  return hipGetLastError();
}

template <bool INLINE>
hipError_t launch_f32_shape(int head_dim, bool wide, const BlobArg<INLINE>& blob, const Ctx& c, const int32_t* links,
                            int32_t n_chains, hipStream_t stream) {
  if (head_dim == 64)
    return wide ? launch_f32<64, 2, INLINE>(blob, c, links, n_chains, stream)
                : launch_f32<64, 1, INLINE>(blob, c, links, n_chains, stream);
  return wide ? launch_f32<128, 2, INLINE>(blob, c, links, n_chains, stream)
              : launch_f32<128, 1, INLINE>(blob, c, links, n_chains, stream);
}

}  // namespace

}  // namespace mfma

hipError_t launch_attend_f32(const AttendArgs& a, const DkItem* items, const int32_t* links, int32_t n_chains,
                             int32_t tile_rows, hipStream_t stream) {
  using namespace mfma;
  if (n_chains <= 0) return hipSuccess;
  if (a.arena.dtype != 0 || (a.arena.head_dim != 64 && a.arena.head_dim != 128)) return hipErrorInvalidValue;
  if (tile_rows != 16 && tile_rows != 32) return hipErrorInvalidValue;
  const Ctx c = make_ctx(a, items);
  if (a.inline_blob)
    return launch_f32_shape<true>(a.arena.head_dim, tile_rows == 32, BlobArg<true>{*a.inline_blob}, c, links, n_chains, stream);
  return launch_f32_shape<false>(a.arena.head_dim, tile_rows == 32, BlobArg<false>{0}, c, links, n_chains, stream);
}

}  // namespace dk
