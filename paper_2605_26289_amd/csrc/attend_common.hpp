// Shared device code of the bf16 MFMA attention kernels (gfx950): descriptor access, the walk over a
// slot's key segments, HBM -> LDS tile loads, MFMA operand reads and result stores.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace dk {
namespace mfma {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(3))) bf16x4* lds_bf16x4_ptr;
typedef __attribute__((address_space(1))) const void* glb_void_ptr;

constexpr int D = 128;
constexpr int ROW_BYTES = 256;

// What the head dimension decides.  The swizzles spread the 16-byte chunks of consecutive K/V rows over the LDS banks
// (64 banks of 4 bytes: one 256-byte row, or two 128-byte rows, per pass): K rows are read one per lane, 16 lanes to a
// pass, V rows in blocks of four rows x 64 bytes.
template <int HD>
struct Geo {
  static_assert(HD == 64 || HD == 128, "head dimensions of the MFMA kernels");
  static constexpr int ROW = 2 * HD;             // bytes of a K/V/Q/O row
  static constexpr int CHUNKS = ROW / 16;        // 16-byte chunks per row
  static constexpr int ROWS_PER_KIB = 1024 / ROW;
  static constexpr int KS = HD / 16;             // depth steps of S^T = K Q^T
  static constexpr int DB = HD / 32;             // depth blocks of O^T = V^T P^T
  static __device__ __forceinline__ int k_swizzle(int row) { return HD == 128 ? (row & 15) : ((row >> 1) & 7); }
  static __device__ __forceinline__ int v_swizzle(int row) { return HD == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2); }
};
// Split partials: per (partial row, KV head) D unnormalised fp32 sums in `parts` (512-byte rows) and the pair
// (running maximum in log2 units, weight sum) in `parts_ml`.

// Descriptors are read through the constant address space so that uniform reads become scalar loads
// (they must not take part in the vector-memory counter that tracks the K/V tiles in flight).
template <typename T>
__device__ __forceinline__ T load_desc(const T* base, int idx) {
  static_assert(sizeof(T) % 4 == 0, "descriptor structs are made of 32-bit words");
  typedef const __attribute__((address_space(4))) uint32_t* const_u32_ptr;
  const_u32_ptr p = (const_u32_ptr)((uintptr_t)base + (size_t)idx * sizeof(T));
  T out;
  uint32_t* o = (uint32_t*)&out;
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) o[i] = p[i];
  return out;
}

// A segment is asked for as a whole: left to itself the compiler first fetches what the search for the right one needs and
// the rest when that is over, another round trip of 500 cycles in front of the first K/V request.
__device__ __forceinline__ DkSeg load_seg(const DkSeg* segs, int idx) {
  DkSeg s = load_desc(segs, idx);
  asm volatile("" : "+s"(s.start), "+s"(s.pos), "+s"(s.len), "+s"(s.src), "+s"(s.once));
  return s;
}

// Kernel-argument form of the descriptor blob: the kernels take it as their FIRST argument, so in the inline
// instantiation it starts the kernel-argument segment and descriptor "pointers" are byte offsets from there.
template <bool INLINE> struct BlobArg;
template <> struct BlobArg<true> { InlineBlob blob; };
template <> struct BlobArg<false> { char unused; };

// Touches the first KiB of an inline blob, every line of it, in the round trip that brings the kernel's other arguments: item,
// entry and segment, which lead to one another, are then found in the scalar cache (or on their way there) one after the
// other, 100 cycles each instead of 500.
template <bool INLINE>
__device__ __forceinline__ void touch_descs() {
  if constexpr (INLINE) {
    typedef const __attribute__((address_space(4))) uint32_t* const_u32_ptr;
    const_u32_ptr base = (const_u32_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(INLINE_BLOB_BYTES >= 1024, "lines of the blob only");
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = base[16 * i];
    asm volatile("" : : "s"(w[0]), "s"(w[1]), "s"(w[2]), "s"(w[3]), "s"(w[4]), "s"(w[5]), "s"(w[6]), "s"(w[7]), "s"(w[8]), "s"(w[9]),
                 "s"(w[10]), "s"(w[11]), "s"(w[12]), "s"(w[13]), "s"(w[14]), "s"(w[15]));
  }
}

template <bool INLINE, typename T>
__device__ __forceinline__ const T* resolve_desc(const T* p) {
  if constexpr (INLINE) {
    typedef const __attribute__((address_space(4))) char* const_char_ptr;
    const_char_ptr base = (const_char_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    return (const T*)((uintptr_t)base + (uintptr_t)p);
  } else {
    return p;
  }
}

struct Ctx {
  const DkEntry* entries;
  const DkSeg* segs;
  const DkItem* items;
  const __bf16* __restrict__ q;
  const char* __restrict__ k_arena;
  const char* __restrict__ v_arena;
  const char* __restrict__ k_new;
  const char* __restrict__ v_new;
  __bf16* __restrict__ out;
  float* __restrict__ lse;
  float* __restrict__ parts;
  float* __restrict__ parts_ml;
  float c;  // softmax scale * log2(e): scores are handled in log2 units
  int32_t n_q_heads, n_kv_heads, gshift;
  int32_t group;    // query heads per KV head
  uint32_t gmagic;  // ceil(2^32 / group), 0 for group 1: see row_token
  uint32_t kvmagic;  // the same of n_kv_heads: see unit_item
  int64_t arena_cells;
  const int32_t* cells;  // small append-and-attend calls: arena cell of every new token
  int32_t n_scatter;     // how many tokens this launch writes into the arena (0: none)
};

// Token and head (inside the KV group) of a packed query row.  ANYG: any group size, by a multiply-high with the
// rounded-up reciprocal -- exact while row * (group - 1) < 2^32, which the host checks for the whole batch before it
// takes a kernel of this kind; otherwise the group is a power of two and this is a shift.
template <bool ANYG>
__device__ __forceinline__ int row_token(const Ctx& c, int row) {
  if constexpr (ANYG) return c.gmagic ? (int)__umulhi((uint32_t)row, c.gmagic) : row;
  else return row >> c.gshift;
}
// Item of a unit, and its KV head: unit = item * n_kv_heads + head.  The rounded-up reciprocal is at most one too high
// whatever the unit, and the remainder tells.
__device__ __forceinline__ int unit_item(const Ctx& c, int unit, int& g) {
  uint32_t item = c.kvmagic ? __umulhi((uint32_t)unit, c.kvmagic) : (uint32_t)unit;
  uint32_t head = (uint32_t)unit - item * (uint32_t)c.n_kv_heads;
  if (head >= (uint32_t)c.n_kv_heads) {
    --item;
    head += (uint32_t)c.n_kv_heads;
  }
  g = (int)head;
  return (int)item;
}
template <bool ANYG>
__device__ __forceinline__ int row_head(const Ctx& c, int row, int tok) {
  if constexpr (ANYG) return row - tok * c.group;
  else return row & ((1 << c.gshift) - 1);
}

// A run of at most KT consecutive K/V rows, all inside one segment.
struct KvTile {
  const char* k;
  const char* v;
  uint32_t stride;  // bytes between consecutive rows
  int32_t cnt;      // valid rows (>= 1)
  int32_t pos;      // logical position of row 0
  int32_t once;     // DkSeg::once
};

// Walks the logical key positions [p, hi) of an entry, segment by segment.  The state of the segment
// being walked (row pointers at position p, row stride, end position) is kept in a handful of scalars,
// so the common step touches neither the segment table nor the kernel arguments.
template <int ROW = ROW_BYTES>
struct KvCursor {
  const DkSeg* segs;
  int32_t si, se, p, hi;
  int32_t seg_end = 0;  // first position past the current segment (0: no segment loaded yet)
  const char* k = nullptr;
  const char* v = nullptr;
  uint32_t stride = 0;
  int32_t once = 0;

  __device__ __forceinline__ void enter_segment(const Ctx& c, int g) {
    DkSeg s = load_seg(segs, si);
    while (s.pos + s.len <= p && si + 1 < se) s = load_seg(segs, ++si);
    const int32_t off = p - s.pos;
    seg_end = s.pos + s.len;
    once = s.once;
    if (s.src == 0) {
      const int64_t byte = ((int64_t)g * c.arena_cells + s.start + off) * ROW;
      k = c.k_arena + byte;
      v = c.v_arena + byte;
      stride = ROW;
    } else {
      const int64_t byte = ((s.start + off) * c.n_kv_heads + g) * (int64_t)ROW;
      k = c.k_new + byte;
      v = c.v_new + byte;
      stride = (uint32_t)c.n_kv_heads * ROW;
    }
  }

  __device__ __forceinline__ bool next(const Ctx& c, int g, int kt, KvTile& t) {
    if (p >= hi) return false;
    if (p >= seg_end) enter_segment(c, g);
    t.cnt = min(kt, min(seg_end, hi) - p);
    t.k = k;
    t.v = v;
    t.stride = stride;
    t.pos = p;
    t.once = once;
    p += t.cnt;
    const uint32_t adv = (uint32_t)t.cnt * stride;
    k += adv;
    v += adv;
    return true;
  }
};

// One wavefront moves 1 KiB (4 rows of 256 bytes or 8 of 128) HBM -> LDS: lane l lands at lds + 16 l, i.e. (256-byte
// rows) row l / 16, chunk slot l % 16, and fetches the chunk that the swizzle assigns to that slot.  Rows past the end of a
// ragged tile re-read the last valid row; their scores are masked.
// The load is issued from inline assembly on purpose: the compiler then keeps no account of it and
// inserts no vmcnt(0) of its own in front of later LDS reads, so a tile can stay in flight while
// the previous one is being consumed.  Completion is awaited explicitly with wait_vmcnt<N>().
template <bool IS_V, int HD = D>
__device__ __forceinline__ uint32_t kib_lane_off(uint32_t stride, int cnt, int blk, int lane) {
  typedef Geo<HD> G;
  const int row = blk * G::ROWS_PER_KIB + lane / G::CHUNKS;
  const int slot = lane % G::CHUNKS;
  const int chunk = slot ^ (IS_V ? G::v_swizzle(row) : G::k_swizzle(row));
  return __umul24((uint32_t)min(row, cnt - 1), stride) + chunk * 16;  // (stride: KV heads x row bytes; dk_pool::choose_route keeps 2^24 out)
}
template <bool IS_V, int HD = D>
__device__ __forceinline__ void load_kib(const char* gbase, uint32_t stride, int cnt, char* lds_region, int blk, int lane) {
  const uint32_t voff = kib_lane_off<IS_V, HD>(stride, cnt, blk, lane);
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_ptr)(lds_region + blk * 1024);
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2"
      :
      : "s"(lds_addr), "v"(voff), "s"(gbase)
      : "memory", "m0");
}
// Eight such blocks, a whole tile of 8 KiB, with the lane's offsets at hand.  The instruction's offset counts for both
// addresses, so M0 is written once for four blocks; the lane's offsets make up for that on the side of memory, and for the
// bias that keeps them from getting negative (a ragged tile's last rows).  ONCE: non-temporal loads, for rows that nothing
// else reads (see DkSeg::once).
constexpr int KIB_BIAS = 3072;
template <bool IS_V, int HD = D>
__device__ __forceinline__ uint32_t kib_biased_off(uint32_t stride, int cnt, int blk, int lane) {
  return kib_lane_off<IS_V, HD>(stride, cnt, blk, lane) + KIB_BIAS - 1024 * (blk & 3);
}
template <bool ONCE>
__device__ __forceinline__ void load_eight_kib(const char* gbase, const uint32_t (&voff)[8], uint32_t lds_addr) {
#define DK_EIGHT_KIB(HOW)                                                                                          \
  asm volatile(                                                                                                    \
      "s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %9" HOW "\n\t"                                   \
      "global_load_lds_dwordx4 %2, %9 offset:1024" HOW "\n\tglobal_load_lds_dwordx4 %3, %9 offset:2048" HOW "\n\t"  \
      "global_load_lds_dwordx4 %4, %9 offset:3072" HOW "\n\ts_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\t"               \
      "global_load_lds_dwordx4 %5, %9" HOW "\n\tglobal_load_lds_dwordx4 %6, %9 offset:1024" HOW "\n\t"              \
      "global_load_lds_dwordx4 %7, %9 offset:2048" HOW "\n\tglobal_load_lds_dwordx4 %8, %9 offset:3072" HOW          \
      :                                                                                                            \
      : "s"(lds_addr), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "v"(voff[4]), "v"(voff[5]),           \
        "v"(voff[6]), "v"(voff[7]), "s"(gbase - KIB_BIAS)                                                            \
      : "memory", "m0", "scc")
  if constexpr (ONCE) DK_EIGHT_KIB(" nt");
  else DK_EIGHT_KIB("");
#undef DK_EIGHT_KIB
}

// A operand of S^T = K Q^T for key block kb and depth step ks: lane (row l%32, half h = l/32) holds
// K[kb*32 + l%32][ks*16 + 8h .. +7], which the swizzle keeps in chunk (2ks + h) ^ (row & 15) of its row.
// Because 2ks has bit 0 clear, that chunk is (2ks) ^ (h ^ (row & 15)): the per-lane part of the address
// is computed once (k_lane_off) and each depth step only XORs in ks << 5.
template <int HD = D>
__device__ __forceinline__ uint32_t k_lane_off(int lane) {
  const int r = lane & 31;
  return (uint32_t)(r * Geo<HD>::ROW + (((lane >> 5) ^ Geo<HD>::k_swizzle(r)) << 4));
}
template <int HD = D>
__device__ __forceinline__ bf16x8 read_k_frag(const char* k_lds, uint32_t lane_off, int kb, int ks) {
  return *(const bf16x8*)(k_lds + (lane_off ^ (uint32_t)(ks << 5)) + kb * (32 * Geo<HD>::ROW));
}

// A operand of O^T = V^T P^T for key step j (16 keys) and depth block db: lane (column l%32, half
// h = l/32) holds V[16j + 8u + 4h + e][db*32 + l%32] for u = 0,1 and e = 0..3 -- the same key order
// in which the S^T accumulators hand over P.  Two transposing 64-bit LDS reads: within 16 lanes, lane i
// supplies the address of row i/4, 4-column piece i%4 and receives column i of the four rows.
// (256-byte rows) The row's chunk is ((db ^ (row & 3)) << 2) | x, so again only db << 6 is XORed per read.
template <int HD = D>
__device__ __forceinline__ uint32_t v_lane_off(int lane) {
  const int i = lane & 15, qd = lane >> 4;
  const int rsub = i >> 2;                         // row inside the 4-row block == row & 3
  const int x = ((qd & 1) << 1) | ((i & 3) >> 1);  // 16-byte chunk inside the 64-byte column block
  return (uint32_t)((4 * (qd >> 1) + rsub) * Geo<HD>::ROW + (Geo<HD>::v_swizzle(rsub) << 4) + (x << 4) + ((i & 1) << 3));
}
template <int HD = D>
__device__ __forceinline__ bf16x8 read_v_frag(const char* v_lds, uint32_t lane_off, int j, int db) {
  const char* p0 = v_lds + (lane_off ^ (uint32_t)(db << 6)) + j * (16 * Geo<HD>::ROW);
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)p0);
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p0 + 8 * Geo<HD>::ROW));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Issues the loads of a wavefront's Q fragments; wait_q() below is where they must have arrived.  What is
// put between the two (finding the first K/V tiles and requesting them) overlaps with the Q round trip.
template <int MB>
__device__ __forceinline__ void load_q(const Ctx& c, const DkEntry& e, int g, int row_base, int last_row, int lane,
                                       bf16x8 (&qf)[MB][8], int (&limit)[MB]) {
  const int gmask = (1 << c.gshift) - 1;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int row = min(row_base + mb * 32 + (lane & 31), last_row);
    const int tok = row >> c.gshift;
    const int head = (g << c.gshift) + (row & gmask);
    limit[mb] = e.n + tok;  // last visible absolute position (bottom-right causal alignment)
    const __bf16* qp = c.q + ((int64_t)(e.tok0 + tok) * c.n_q_heads + head) * D + 8 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[mb][ks] = *(const bf16x8*)(qp + ks * 16);
  }
}

// Makes the compiler wait for Q here, once, instead of at first use inside the key loop, where its
// vmcnt(0) would also drain the K/V tiles that are meant to stay in flight.  (The wait it emits here is a
// vmcnt(0) as well: K/V tiles requested before this point land before the key loop starts.)
template <int MB>
__device__ __forceinline__ void wait_q(const bf16x8 (&qf)[MB][8]) {
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) asm volatile("" ::"v"(qf[mb][ks]));
}

// A pair of fp32 weights as hi + lo, both bf16: hi is the upper half of the bits (truncated), lo the rest rounded to
// bf16.  What is lost is below 2^-16 of the weight.  Written to pair w of the two B-operand fragments.
__device__ __forceinline__ uint32_t pack_pair(float p0, float p1) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  bf16x2 w;
  w[0] = (__bf16)p0;
  w[1] = (__bf16)p1;
  return __builtin_bit_cast(uint32_t, w);
}
__device__ __forceinline__ void split_pair(float p0, float p1, uint32_t& hi, uint32_t& lo) {
  const uint32_t u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
  hi = __builtin_amdgcn_perm(u1, u0, 0x07060302);  // upper halves of (p0, p1)
  lo = pack_pair(p0 - __uint_as_float(u0 & 0xffff0000u), p1 - __uint_as_float(u1 & 0xffff0000u));
}
__device__ __forceinline__ void split_pair(float p0, float p1, bf16x8& hi, bf16x8& lo, int w) {
  typedef __attribute__((ext_vector_type(4))) uint32_t words;
  words h = __builtin_bit_cast(words, hi), l = __builtin_bit_cast(words, lo);
  uint32_t hw, lw;
  split_pair(p0, p1, hw, lw);
  h[w] = hw;
  l[w] = lw;
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}

// Partial rows that another workgroup of the same launch reads: every store goes through to the memory that all XCDs see and
// every load comes from there (agent scope), so neither side has an L2 to write back or to invalidate.
template <typename T>
__device__ __forceinline__ void store_for_others(T* p, const T& x) {
  static_assert(sizeof(T) % 8 == 0, "in pieces of 8 bytes");
  struct Words { uint64_t w[sizeof(T) / 8]; };
  const Words words = __builtin_bit_cast(Words, x);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 8); ++i)
    __hip_atomic_store((uint64_t*)p + i, words.w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_of_others(const T* p) {
  static_assert(sizeof(T) % 8 == 0, "in pieces of 8 bytes");
  struct Words { uint64_t w[sizeof(T) / 8]; } words;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 8); ++i)
    words.w[i] = __hip_atomic_load((uint64_t*)p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_bit_cast(T, words);
}

// Stores one row's results of a lane: quad i holds depths depth0 + 8 i .. + 3 (the order of the 32x32 accumulators,
// depth0 including the half-wave's 4 h), as fp32 partials or, divided by the weight sum, as bf16 output.
// rl: the row inside the item (rows past its end are skipped).
template <int HD, bool ANYG, int NQ>
__device__ __forceinline__ void store_quads(const Ctx& c, const DkEntry& e, const DkItem& it, int g, int rl, int depth0,
                                            const f32x4 (&o)[NQ], float ltot, bool for_others = false) {
  if (rl >= it.nrows) return;
  if (it.part_row0 >= 0) {
    float* p = c.parts + ((int64_t)(it.part_row0 + rl) * c.n_kv_heads + g) * HD + depth0;
    if (for_others) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) store_for_others((f32x4*)(p + 8 * i), o[i]);
      return;
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) *(f32x4*)(p + 8 * i) = o[i];
  } else {
    const int row = it.row0 + rl;
    const int t = row_token<ANYG>(c, row);
    const int head = g * c.group + row_head<ANYG>(c, row, t);
    const float inv = 1.f / ltot;
    __bf16* dst = c.out + ((int64_t)(e.tok0 + t) * c.n_q_heads + head) * HD + depth0;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      bf16x4 v;
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = (__bf16)(o[i][u] * inv);
      *(bf16x4*)(dst + 8 * i) = v;
    }
  }
}

// The same store through a private LDS staging area of 8 KiB, so that every store instruction of the wavefront
// writes eight whole 128-byte pieces of eight rows instead of 64 scattered 8-byte pieces: the accumulator
// layout (lane = row) is turned into (8 lanes = 128 bytes of one row) on the way.  16-byte chunks of a staged
// row are XOR-swizzled with the row number, which keeps both the writes (one row per lane) and the reads
// (eight lanes per row) free of bank conflicts.  Covers 64 rows x all 128 depths: four passes of one depth
// block for fp32 partials, two passes of two depth blocks for the bf16 output.  LDS operations of one
// wavefront execute in order, so no wait is needed between a pass's writes and reads or between passes.
template <int MB>
__device__ __forceinline__ void store_rows_staged(const Ctx& c, const DkEntry& e, const DkItem& it, int g,
                                                  int row_local0, int lane, char* stage, const f32x16 (&o)[4][MB],
                                                  const float (&ltot)[MB]) {
  static_assert(MB == 2, "64 rows per wavefront");
  const int h = lane >> 5, r = lane & 31;
  const int rd_row = lane >> 3, rd_chunk = lane & 7;  // reader: row inside a group of eight, 16-byte chunk
  const int gmask = (1 << c.gshift) - 1;
  if (it.part_row0 >= 0) {
#pragma unroll
    for (int db = 0; db < 4; ++db) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int R = mb * 32 + r;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *(f32x4*)(stage + R * 128 + (((2 * r4 + h) ^ (R & 7)) << 4)) =
              f32x4{o[db][mb][4 * r4], o[db][mb][4 * r4 + 1], o[db][mb][4 * r4 + 2], o[db][mb][4 * r4 + 3]};
      }
#pragma unroll
      for (int ps = 0; ps < 8; ++ps) {
        const int R = ps * 8 + rd_row;
        const f32x4 v = *(const f32x4*)(stage + R * 128 + ((rd_chunk ^ (R & 7)) << 4));
        const int rl = row_local0 + R;
        if (rl < it.nrows)
          *(f32x4*)(c.parts + ((int64_t)(it.part_row0 + rl) * c.n_kv_heads + g) * D + db * 32 + rd_chunk * 4) = v;
      }
      __builtin_amdgcn_sched_barrier(0);  // one pass at a time: keeps the passes' registers from piling up
    }
  } else {
    float inv[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) inv[mb] = 1.f / ltot[mb];
#pragma unroll
    for (int dp = 0; dp < 2; ++dp) {  // depth blocks 2 dp and 2 dp + 1: 64 bf16 = 128 bytes per row
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int R = mb * 32 + r;
#pragma unroll
        for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            bf16x4 v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = (__bf16)(o[2 * dp + d2][mb][4 * r4 + t] * inv[mb]);
            // bf16 columns d2*32 + 8*r4 + 4h .. +3: 8-byte piece (8*d2 + 2*r4 + h) of the 128-byte row
            const int piece = 8 * d2 + 2 * r4 + h;
            *(bf16x4*)(stage + R * 128 + ((((piece >> 1) ^ (R & 7)) << 4) | ((piece & 1) << 3))) = v;
          }
      }
#pragma unroll
      for (int ps = 0; ps < 8; ++ps) {
        const int R = ps * 8 + rd_row;
        const bf16x8 v = *(const bf16x8*)(stage + R * 128 + ((rd_chunk ^ (R & 7)) << 4));
        const int rl = row_local0 + R;
        if (rl < it.nrows) {
          const int row = it.row0 + rl;
          const int tok = e.tok0 + (row >> c.gshift);
          const int head = (g << c.gshift) + (row & gmask);
          *(bf16x8*)(c.out + ((int64_t)tok * c.n_q_heads + head) * D + dp * 64 + rd_chunk * 8) = v;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// A product of matrix instructions multiplies every V row of a tile into every query row, hidden keys with weight zero --
// and 0 * inf or 0 * NaN is NaN.  So where V holds such values at positions some of a tile's rows may not see, those rows
// come out non-finite although what they attend to is not (and an infinity the row does see may come out as NaN, where the
// lower half of its weight is zero).  Kernels of shapes that were always free of that look at their sums once, before the
// store, and have the row blocks with non-finite sums done again (nobody pays for this otherwise): by the same products, but
// with the non-finite elements of V taken out, so that the sums are those of the finite ones; then a depth that has such
// elements at positions a row sees is set to what they make of it -- infinite if they are infinities of one sign, else NaN.
// The first position of each kind decides that, since a row sees all positions up to its limit.
//
// One wavefront does a row block over all keys of its item, straight from memory, relative to each row's final maximum m and
// weight sum l, which V has no part in; a row whose weight sum is NaN has a NaN weight, is NaN throughout, and stays as it
// is.  Every element is written by the wavefront that stored it before, so the bits are the same on every call.
// The value may well be one that every row sees, in every item of a long turn, so this has to keep up with the scalar kernel,
// which has a wavefront for every row.  Measured, a session of 2000 tokens with an infinity at its start, us a call, this /
// scalar kernel / one wavefront going row by row and key by key, as it was first: 32 heads of 64, 9 new tokens 24 / 41 / 763,
// 256 new tokens 136 / 496 / 8800; 24 heads of 128 on 8, 200 new tokens 120 / 615 / 7194; fp32, 8 heads of 128 on 2, 150 new
// tokens 169 / 443 / 3025.  (Slower than the scalar kernel: fp32 decoding with 64-wide heads, 96 / 61, bound by the latency
// of a block's loads.)
struct NonFinite {  // first positions of a depth's non-finite elements
  int32_t nan = INT32_MAX, pos = INT32_MAX, neg = INT32_MAX;
  __device__ __forceinline__ bool see(uint32_t bits, int32_t at) {  // an element's fp32 bits; true if it is not finite
    nan = min(nan, (bits & 0x7fffffffu) > 0x7f800000u ? at : INT32_MAX);
    pos = min(pos, bits == 0x7f800000u ? at : INT32_MAX);
    neg = min(neg, bits == 0xff800000u ? at : INT32_MAX);
    return (bits & 0x7f800000u) == 0x7f800000u;
  }
  __device__ __forceinline__ void merge_lanes(int mask) {
    nan = min(nan, __shfl_xor(nan, mask));
    pos = min(pos, __shfl_xor(pos, mask));
    neg = min(neg, __shfl_xor(neg, mask));
  }
  __device__ __forceinline__ NonFinite of_lane(int lane) const { return {__shfl(nan, lane), __shfl(pos, lane), __shfl(neg, lane)}; }
  // the sum of a row that sees the positions up to `limit`
  __device__ __forceinline__ float apply(float sum, int32_t limit) const {
    if (nan <= limit || (pos <= limit && neg <= limit)) return __uint_as_float(0x7fc00000u);
    if (pos <= limit) return INFINITY;
    return neg <= limit ? -INFINITY : sum;
  }
};

// bf16: rows rl0 .. rl0 + 31 of the item (bit i of `bad`: row rl0 + i is to be replaced; m and l in lanes i and 32 + i), depth
// block db; of it, the quads of depths that owns() says this wavefront has stored.
template <int HD, bool ANYG, typename Owns>
__device__ __forceinline__ void redo_rows(const Ctx& c, const DkEntry& e, const DkItem& it, int g, int rl0, uint32_t bad, float m,
                                          float l, int lane, int db, Owns owns) {
  typedef Geo<HD> G;
  asm volatile("" : "+v"(lane));  // (per-lane offsets are made here, not hoisted into registers that the key loop needs)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // after the ordinary store of the same rows
  const int col = lane & 31, h = lane >> 5;
  const int last_row = it.row0 + it.nrows - 1;
  const int row = min(it.row0 + rl0 + col, last_row);
  const int tok = row_token<ANYG>(c, row);
  const int limit = e.n + tok;
  const int64_t orow = (int64_t)(e.tok0 + tok) * c.n_q_heads + g * c.group + row_head<ANYG>(c, row, tok);
  bf16x8 qf[G::KS];
#pragma unroll
  for (int ks = 0; ks < G::KS; ++ks) qf[ks] = *(const bf16x8*)(c.q + orow * HD + ks * 16 + 8 * h);
  f32x16 o;
  NonFinite nf;
#pragma unroll
  for (int r = 0; r < 16; ++r) o[r] = 0.f;
  const int max_limit = e.n + row_token<ANYG>(c, min(it.row0 + rl0 + 31, last_row));
  KvCursor<G::ROW> cur{c.segs, e.seg_begin, e.seg_end, it.kv_lo, min(it.kv_hi, max_limit + 1)};
  KvTile t;
  while (cur.next(c, g, 32, t)) {
    const char* kp = t.k + (uint32_t)min(col, t.cnt - 1) * t.stride + 16 * h;
    bf16x8 kf[G::KS];
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) kf[ks] = *(const bf16x8*)(kp + 32 * ks);
    uint16_t vb[2][8];  // element 4 u + i of key step j is key 16 j + 8 u + 4 h + i, depth 32 db + col
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int x = 0; x < 8; ++x)
        vb[j][x] = *(const uint16_t*)(t.v + (uint32_t)min(16 * j + 8 * (x >> 2) + 4 * h + (x & 3), t.cnt - 1) * t.stride + 64 * db + 2 * col);
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
    const int lim = min(t.cnt - 1, limit - t.pos) - 4 * h;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c.c, -m));
      s[r] = 8 * (r >> 2) + (r & 3) > lim ? 0.f : p;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8 hi, lo;
#pragma unroll
      for (int w = 0; w < 4; ++w) split_pair(s[8 * j + 2 * w], s[8 * j + 2 * w + 1], hi, lo, w);
      bf16x8 v;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const bool odd = nf.see((uint32_t)vb[j][x] << 16, t.pos + min(16 * j + 8 * (x >> 2) + 4 * h + (x & 3), t.cnt - 1));
        v[x] = __builtin_bit_cast(__bf16, (uint16_t)(odd ? 0 : vb[j][x]));
      }
      o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, hi, o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, lo, o, 0, 0, 0);
    }
  }
  const bool mine = (bad >> col & 1) != 0 && rl0 + col < it.nrows && l == l;
  const float inv = 1.f / l;
  nf.merge_lanes(32);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f32x4 x;
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = nf.of_lane(8 * i + 4 * h + r).apply(o[4 * i + r], limit);
    const int depth = 32 * db + 8 * i + 4 * h;
    if (!mine || !owns(depth)) continue;
    if (it.part_row0 >= 0) {
      store_for_others((f32x4*)(c.parts + ((int64_t)(it.part_row0 + rl0 + col) * c.n_kv_heads + g) * HD + depth), x);
    } else {
      bf16x4 y;
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = (__bf16)(x[r] * inv);
      *(bf16x4*)(c.out + orow * HD + depth) = y;
    }
  }
}

// Running maximum and weight sum of each row (partials) or the row's log-sum-exp (final output).
template <int MB, bool ANYG = false>
__device__ __forceinline__ void store_ml(const Ctx& c, const DkEntry& e, const DkItem& it, int g, int row_local0,
                                         int lane, const float (&m)[MB], const float (&ltot)[MB], bool for_others = false) {
  if (lane >= 32) return;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int rl = row_local0 + mb * 32 + lane;
    if (rl >= it.nrows) continue;
    if (it.part_row0 >= 0) {
      float* p = c.parts_ml + ((int64_t)(it.part_row0 + rl) * c.n_kv_heads + g) * 2;
      const float2 ml = make_float2(m[mb], ltot[mb]);
      if (for_others) store_for_others((float2*)p, ml);
      else *(float2*)p = ml;
    } else if (c.lse) {
      const int row = it.row0 + rl;
      const int t = row_token<ANYG>(c, row);
      const int head = g * c.group + row_head<ANYG>(c, row, t);
      c.lse[(int64_t)(e.tok0 + t) * c.n_q_heads + head] = (m[mb] + __builtin_amdgcn_logf(ltot[mb])) * 0.6931471805599453f;
    }
  }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Append-and-attend calls small enough for their descriptors to travel in the kernel arguments: the attention
// kernel also writes the call's new K/V rows (token-major, as staged in k_new / v_new) into their arena cells, so
// that no separate copy kernel has to be launched.  The cells are fresh ones that no attention work of this launch
// reads (the new tokens are attended from the staged rows), so the order against the rest of the kernel is free:
// every workgroup copies an equal run where its own reads have something to hide under.
// The copy is cut into 16-byte pieces, piece p = (token, K or V, KV head, position in the row); a thread has up to four
// loads in flight before its first store.  load() asks for the first of them, store() writes them and does the others.
template <bool INLINE, int ROW = ROW_BYTES, int THREADS = 256>
struct RowCopy {
  typedef __attribute__((ext_vector_type(4))) uint32_t Piece;
  Piece v[4];
  char* dst[4];
  int at = 0, end = 0;  // pieces [at, end) of this workgroup are still to be done

  __device__ __forceinline__ void load_four(const Ctx& c) {
    const int32_t* cells = resolve_desc<INLINE>(c.cells);
    const int vecs = c.n_kv_heads * (ROW / 16);  // pieces of one token's K (as many for V)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (at + k * THREADS >= end) continue;
      const int p = min(at + k * THREADS + (int)threadIdx.x, end - 1);  // (threads past the end repeat the last piece)
      const int t = (int)((uint32_t)p / (uint32_t)(2 * vecs)), r = p - t * (2 * vecs);
      const bool is_v = r >= vecs;
      const int j = is_v ? r - vecs : r;
      const int g = j / (ROW / 16), piece = j % (ROW / 16);
      const int64_t cell = cells[t];
      v[k] = *(const Piece*)((is_v ? c.v_new : c.k_new) + ((int64_t)t * c.n_kv_heads + g) * ROW + piece * 16);
      dst[k] = const_cast<char*>(is_v ? c.v_arena : c.k_arena) + ((int64_t)g * c.arena_cells + cell) * ROW + piece * 16;
    }
  }
  __device__ __forceinline__ void store_four() {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (at + k * THREADS < end) *(Piece*)dst[k] = v[k];
    }
    at += 4 * THREADS;
  }
  __device__ __forceinline__ void load(const Ctx& c) {
    if (c.n_scatter <= 0) return;
    const int total = c.n_scatter * 2 * c.n_kv_heads * (ROW / 16);
    const int per = ((total + (int)gridDim.x - 1) / (int)gridDim.x + THREADS - 1) / THREADS * THREADS;
    at = min(total, (int)blockIdx.x * per);
    end = min(total, at + per);
    load_four(c);
  }
  __device__ __forceinline__ void store(const Ctx& c) {
    if (at >= end) return;
    store_four();
    while (at < end) {
      load_four(c);
      store_four();
    }
  }
};
template <bool INLINE, int ROW = ROW_BYTES, int THREADS = 256>
__device__ __forceinline__ void scatter_new_rows(const Ctx& c) {
  RowCopy<INLINE, ROW, THREADS> copy;
  copy.load(c);
  copy.store(c);
}

inline Ctx make_ctx(const AttendArgs& a, const DkItem* items) {
  Ctx c;
  c.entries = a.entries;
  c.segs = a.segs;
  c.items = items;
  c.q = (const __bf16*)a.q;
  c.k_arena = (const char*)a.arena.k_arena;
  c.v_arena = (const char*)a.arena.v_arena;
  c.k_new = (const char*)a.k_new;
  c.v_new = (const char*)a.v_new;
  c.out = (__bf16*)a.out;
  c.lse = a.lse;
  c.parts = a.parts;
  c.parts_ml = a.parts_ml;
  c.c = a.scale * 1.4426950408889634f;
  c.n_q_heads = a.arena.n_q_heads;
  c.n_kv_heads = a.arena.n_kv_heads;
  int group = a.arena.n_q_heads / a.arena.n_kv_heads, sh = 0;
  while ((1 << sh) < group) ++sh;
  c.gshift = sh;
  c.group = group;
  c.gmagic = group > 1 ? (uint32_t)(((1ull << 32) + group - 1) / group) : 0u;
  c.kvmagic = c.n_kv_heads > 1 ? (uint32_t)(((1ull << 32) + c.n_kv_heads - 1) / c.n_kv_heads) : 0u;
  c.arena_cells = a.arena.arena_cells;
  c.cells = a.cells;
  c.n_scatter = a.scatter ? a.total_tokens : 0;
  return c;
}

}  // namespace mfma
}  // namespace dk
