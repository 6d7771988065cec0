// bf16 MFMA delta-prefill attention kernels for gfx950.
//
// Both kernels compute, for the packed query rows of one KV head (row r = token r / G, head r % G of
// the group), the transposed products S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16.
// In that orientation a lane owns one query row (column l % 32 of the 32x32 result), so the online
// softmax needs one cross-lane exchange per row block and the probabilities leave the first MFMA in
// exactly the register layout the second one wants as its B operand: P never touches LDS.
//
//   tile kernel    large Delta: a workgroup owns 256 packed rows (4 wavefronts x 64 rows) and all
//                  wavefronts share each 64-key K/V tile through LDS (compute bound, MFMA roofline)
//   stream kernel  small Delta (row tiles of at most 96 packed rows: entries of G*Delta <= 96, and
//                  longer ones of small batches in several row tiles): every wavefront streams its
//                  own slice of the keys through private LDS stages with no barriers, the four
//                  states are merged at the end (HBM bound, in small batches latency)
//
// K/V tiles go HBM -> LDS with global_load_lds_dwordx4 (no VGPR staging).  Rows are 256 B; the 16-byte
// chunks of a row are XOR-swizzled so that the K reads (ds_read_b128, one row per lane) and the V
// reads (ds_read_b64_tr_b16, 4 rows x 16 columns per 16 lanes) are bank-conflict free.
#include <hip/hip_runtime.h>

#include <mutex>
#include <utility>

#include "attend_common.hpp"
#include "kernels.hpp"

namespace dk {
namespace mfma {

#ifdef DK_TRACE  // timeline build: wall-clock stamps (100 MHz) per workgroup and unit
__device__ unsigned long long g_strace[256][8][12];
#define DK_STR(seq, ph)                                                                                      \
  do {                                                                                                       \
    if (lane == 0 && (seq) < 8 && blockIdx.x < 256) g_strace[blockIdx.x][(seq)][(ph)] = wall_clock64();       \
  } while (0)
#else
#define DK_STR(seq, ph)
#endif

// HD: head dimension.  GEN: the general form, for everything but 128-wide heads in groups of 2^k <= 16 query heads per
// KV head -- any group size, and the probabilities enter the second product as a sum of two bf16 (p = hi + lo, about
// 2^-17 relative), i.e. with what matters of their 32 bits, for twice the PV products: the shapes it serves used to be
// computed with fp32 probabilities, and next to HBM the extra MFMAs cost little.  Measured, four turns of up to
// 200 tokens on 256-2048 of 24 query heads on 8 KV heads of 128: 44 us, 1345 in the scalar kernel.
// A tile is 8 KiB of K and 8 KiB of V: 32 keys of 256 bytes or 64 of 128.
template <int HD>
struct Tile {
  static constexpr int KB = 128 / HD;  // 32-key blocks per tile
  static constexpr int KT = 32 * KB;   // keys per tile
};

template <int MB, int HD>
struct RowState {
  f32x16 o[Geo<HD>::DB][MB];  // O^T accumulators: [depth block][row block], unnormalised
  float m[MB];      // running maximum of the scaled scores (log2 units), -inf before the first key
  float l[MB];      // this lane's share of the weight sum (the other half-wave holds the rest)
};

// MFMA operand fragments of one tile, read out of its LDS stage into registers: once a half of the stage (K or V) has been
// read it can take the next HBM load while the tile is still being computed.
template <int HD>
struct TileFrags {
  bf16x8 k[Tile<HD>::KB][Geo<HD>::KS];      // [key block][depth step]
  bf16x8 v[2 * Tile<HD>::KB][Geo<HD>::DB];  // [key step][depth block]
};
template <int HD>
__device__ __forceinline__ void read_k_frags(const char* k_lds, uint32_t koff, TileFrags<HD>& f) {
#pragma unroll
  for (int ks = 0; ks < Geo<HD>::KS; ++ks)
#pragma unroll
    for (int kb = 0; kb < Tile<HD>::KB; ++kb) f.k[kb][ks] = read_k_frag<HD>(k_lds, koff, kb, ks);
}
constexpr float STREAM_RESCALE_SLACK = 8.f;  // log2 units, as in the tile kernel

__device__ __forceinline__ float stream_max3(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// The products are issued from inline assembly so that the accumulators (O and the scores), and Q where QFrags says so, live in
// the accumulation registers and nowhere else: with plain C++ the compiler keeps a second copy of all of O in ordinary registers, for the sake
// of the rarely taken rescale.  It does not see then that these registers come out of the matrix pipeline; where a read can
// follow a product closely they pass through settle() first.
template <bool Q_ACC>
__device__ __forceinline__ void mfma_first(f32x16& s, const bf16x8& k, const bf16x8& q) {
  if constexpr (Q_ACC) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&a"(s) : "v"(k), "a"(q));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&a"(s) : "v"(k), "v"(q));
}
template <bool Q_ACC>
__device__ __forceinline__ void mfma_more(f32x16& s, const bf16x8& k, const bf16x8& q) {
  if constexpr (Q_ACC) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(s) : "v"(k), "a"(q));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(s) : "v"(k), "v"(q));
}
__device__ __forceinline__ void settle(f32x16& a) { asm volatile("s_nop 15\n\ts_nop 7" : "+a"(a)); }

// Q as B operand: lane (row l%32 of block mb, half l/32) holds Q[row][ks*16 + 8*(l/32) .. +7].  With one or two
// row blocks the unit's Q fragments stay in registers for the whole unit; with three (96 registers next to 192
// of accumulators) they would not fit, so each tile reads them from the Q area in LDS again (24 ds_read_b128 per
// tile next to the tile's own 16: LDS bandwidth is idle here).
// IN_ACC: two blocks around a loop over units, where they are asked for in accumulation registers.  In ordinary ones the
// compiler needs all 256 of them there and spills one in the form with non-temporal loads and inline descriptors; a single
// unit's body fits as it is (245 ordinary registers at most), and one block's fragments need no such help.
template <int MB, int HD, bool SINGLE>
struct QFrags {
  static constexpr bool IN_LDS = MB > 2;
  static constexpr bool IN_ACC = MB == 2 && !SINGLE;
  bf16x8 r[IN_LDS ? 1 : MB][Geo<HD>::KS];
  const char* q_lds;
  uint32_t koff;
  __device__ __forceinline__ void load() {
    if constexpr (!IN_LDS) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int ks = 0; ks < Geo<HD>::KS; ++ks) r[mb][ks] = read_k_frag<HD>(q_lds, koff, mb, ks);
      if constexpr (IN_ACC) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int ks = 0; ks < Geo<HD>::KS; ++ks) asm volatile("" : "+a"(r[mb][ks]));
      }
    }
  }
  __device__ __forceinline__ bf16x8 get(int mb, int ks) const {
    if constexpr (IN_LDS) return read_k_frag<HD>(q_lds, koff, mb, ks);
    else return r[mb][ks];
  }
};

template <int N>
struct Num {
  static constexpr int value = N;
};
template <typename F, int... Is>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, Is...>) {
  (f(Num<Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled(f, std::make_integer_sequence<int, N>{});
}

// Keeps a value's computation where the source has it.
template <typename T>
__device__ __forceinline__ void stay(const T& x) {
  asm volatile("" : : "v"(x));
}
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// The key loop is a software pipeline, because a compute unit runs one of these wavefronts per SIMD and nothing but the
// wavefront's own instructions can fill the time that a product, an exponential or a load takes.  Step t issues
//     S^T(t)                K fragments of tile t, read from LDS at the end of step t-1
//     O^T += V^T P^T(t-1)   V fragments of tile t-1, read at the beginning of step t
// and between those MFMAs, slot by slot in the order that is fixed here, the VALU turns S^T(t-1) into P(t-1), pair by pair,
// each just in time for its product, and takes the row maxima of S^T(t), whose accumulators are copied on the way (the next
// step's products overwrite them while the copy is being turned into weights).
// What bounds a step is the number of instructions, 4 cycles each, 8 an exponential and an MFMA.  Measured with cycle stamps,
// keys in L2: one row block of 128-wide heads 2300 cycles a step with the parts one after the other, 1560 like this (its 16
// MFMAs alone: 512); two row blocks with split weights 4100 / 2950 (48 MFMAs: 1540).  One 150-token turn on 800 cached tokens
// 13.9 -> 11.4 us, four turns of up to 200 tokens with three query heads to a KV head 41.4 -> 33.5.
template <int MB, int HD, bool GEN, bool SINGLE>
struct StreamStep {
  typedef QFrags<MB, HD, SINGLE> Q;
  static constexpr int KB = Tile<HD>::KB, KS = Geo<HD>::KS, DB = Geo<HD>::DB;
  static constexpr int S_PER = KS * KB, S_SLOTS = MB * S_PER;             // S^T products: of a row block (8), all
  static constexpr int NJ = 2 * KB, PIECES = MB * NJ;                     // a piece: eight weights a lane, one B operand
  static constexpr int O_PER = DB * (GEN ? 2 : 1), O_SLOTS = PIECES * O_PER;  // O^T products: of a piece, all
  static constexpr int PAIRS = 4 * PIECES;
  // Slot of a pair of weights: spread evenly up to the first product of the last piece.
  static constexpr int slot_of(int pair) { return pair * (S_SLOTS + O_SLOTS - O_PER) / PAIRS; }
  static constexpr bool in_time() {  // (two slots between a piece's last weights and its first product: no hazard)
    for (int p = 0; p < PIECES; ++p)
      if (slot_of(4 * p + 3) + 2 > S_SLOTS + p * O_PER) return false;
    return true;
  }
  static_assert(in_time(), "weights of a piece before its products");

  const Q& qf;
  RowState<MB, HD>& st;
  float c;
  TileFrags<HD> f;
  f32x16 acc[MB][KB];  // S^T of the tile
  f32x16 s[MB][KB];    // the copy, hidden keys at -inf
  float mx[MB], ms[MB], rs[MB][2];
  bf16x8 q[3];
  u32x4 hi[PIECES], lo[GEN ? PIECES : 1];  // weights, bf16: GEN their upper halves and what these leave

  template <int I>  // product I of S^T
  __device__ __forceinline__ void score() {
    constexpr int mb = I / S_PER, r = I % S_PER, ks = r / KB, kb = r % KB, n = mb * KS + ks;
    constexpr bool AHEAD = Q::IN_LDS;  // fragments of Q come from LDS, two depth steps ahead
    if constexpr (AHEAD && I == 0) {
      q[0] = qf.get(0, 0);
      q[1] = qf.get(0, 1);
    }
    if constexpr (AHEAD && kb == 0 && n + 2 < MB * KS) q[(n + 2) % 3] = qf.get((n + 2) / KS, (n + 2) % KS);
    bf16x8 b;
    if constexpr (AHEAD) b = q[n % 3];
    else b = qf.get(mb, ks);
    if constexpr (ks == 0) mfma_first<Q::IN_ACC>(acc[mb][kb], f.k[kb][ks], b);
    else mfma_more<Q::IN_ACC>(acc[mb][kb], f.k[kb][ks], b);
  }
  template <int I>  // product I of O^T
  __device__ __forceinline__ void output() {
    constexpr int P = I / O_PER, r = I % O_PER, mb = P / NJ, j = P % NJ, db = GEN ? r / 2 : r;
    mfma_more<false>(st.o[db][mb], f.v[j][db], __builtin_bit_cast(bf16x8, GEN && r % 2 == 1 ? lo[GEN ? P : 0] : hi[P]));
  }
  template <int N>  // pair N of weights
  __device__ __forceinline__ void weights() {
    constexpr int P = N / 4, W = N % 4, mb = P / NJ, j = P % NJ, r = 8 * (j & 1) + 2 * W;
    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][j >> 1][r], c, -ms[mb]));
    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mb][j >> 1][r + 1], c, -ms[mb]));
    if constexpr (j == 0 && W < 2) rs[mb][W] = p0 + p1;
    else rs[mb][W & 1] += p0 + p1;  // (no v_dot2 here: the dot instructions queue behind the MFMAs)
    uint32_t w;
    if constexpr (GEN) {
      uint32_t rest;
      split_pair(p0, p1, w, rest);
      stay(rest);
      lo[P][W] = rest;
    } else {
      w = pack_pair(p0, p1);
    }
    stay(w);
    hi[P][W] = w;
    if constexpr (j == NJ - 1 && W == 3) {
      st.l[mb] += rs[mb][0] + rs[mb][1];
      stay(st.l[mb]);
    } else {
      stay(rs[mb][W & 1]);
    }
  }
  // Copy and maximum, eight steps a row block: steps N .. N + COUNT - 1 of them, an asm statement each (a statement that
  // reads what the one before it wrote gets a wait state in between).
  template <int N, int COUNT>
  __device__ __forceinline__ void take() {
    constexpr int mb = N / 8, op = N % 8;
    if constexpr (KB == 1) {
      f32x16 &d = s[mb][0], &a = acc[mb][0];
      if constexpr (COUNT == 2) {
        if constexpr (op == 0)
          asm volatile(
              "v_accvgpr_read_b32 %0, %5\n\tv_accvgpr_read_b32 %1, %6\n\tv_accvgpr_read_b32 %2, %7\n\tv_accvgpr_read_b32 %3, %8\n\t"
              "v_max_f32 %4, %0, %1\n\tv_max3_f32 %4, %4, %2, %3"
              : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]), "=&v"(mx[mb])
              : "a"(a[0]), "a"(a[1]), "a"(a[2]), "a"(a[3]));
        else
          asm volatile(
              "v_accvgpr_read_b32 %0, %5\n\tv_accvgpr_read_b32 %1, %6\n\tv_accvgpr_read_b32 %2, %7\n\tv_accvgpr_read_b32 %3, %8\n\t"
              "v_max3_f32 %4, %4, %0, %1\n\tv_max3_f32 %4, %4, %2, %3"
              : "=&v"(d[2 * op]), "=&v"(d[2 * op + 1]), "=&v"(d[(2 * op + 2) & 15]), "=&v"(d[(2 * op + 3) & 15]), "+v"(mx[mb])
              : "a"(a[2 * op]), "a"(a[2 * op + 1]), "a"(a[(2 * op + 2) & 15]), "a"(a[(2 * op + 3) & 15]));
      } else if constexpr (op == 0) {
        asm volatile("v_accvgpr_read_b32 %0, %3\n\tv_accvgpr_read_b32 %1, %4\n\tv_max_f32 %2, %0, %1"
                     : "=&v"(d[0]), "=&v"(d[1]), "=&v"(mx[mb])
                     : "a"(a[0]), "a"(a[1]));
      } else {
        asm volatile("v_accvgpr_read_b32 %0, %3\n\tv_accvgpr_read_b32 %1, %4\n\tv_max3_f32 %2, %2, %0, %1"
                     : "=&v"(d[2 * op]), "=&v"(d[2 * op + 1]), "+v"(mx[mb])
                     : "a"(a[2 * op]), "a"(a[2 * op + 1]));
      }
    } else {
      f32x16 &d = s[mb][0], &e = s[mb][KB - 1], &a = acc[mb][0], &b = acc[mb][KB - 1];
      if constexpr (op == 0)
        asm volatile(
            "v_accvgpr_read_b32 %0, %5\n\tv_accvgpr_read_b32 %1, %6\n\tv_accvgpr_read_b32 %2, %7\n\tv_accvgpr_read_b32 %3, %8\n\t"
            "v_max_f32 %4, %0, %1\n\tv_max3_f32 %4, %4, %2, %3"
            : "=&v"(d[0]), "=&v"(d[1]), "=&v"(e[0]), "=&v"(e[1]), "=&v"(mx[mb])
            : "a"(a[0]), "a"(a[1]), "a"(b[0]), "a"(b[1]));
      else
        asm volatile(
            "v_accvgpr_read_b32 %0, %5\n\tv_accvgpr_read_b32 %1, %6\n\tv_accvgpr_read_b32 %2, %7\n\tv_accvgpr_read_b32 %3, %8\n\t"
            "v_max3_f32 %4, %4, %0, %1\n\tv_max3_f32 %4, %4, %2, %3"
            : "=&v"(d[2 * op]), "=&v"(d[2 * op + 1]), "=&v"(e[2 * op]), "=&v"(e[2 * op + 1]), "+v"(mx[mb])
            : "a"(a[2 * op]), "a"(a[2 * op + 1]), "a"(b[2 * op]), "a"(b[2 * op + 1]));
      if constexpr (COUNT == 2) take<8 * mb + (op + 1) % 8, 1>();
    }
  }
  template <int N>
  __device__ __forceinline__ void max_step() {
    constexpr int mb = N / 8, op = N % 8;
    if constexpr (op == 0) mx[mb] = fmaxf(s[mb][0][0], s[mb][0][1]);
    else mx[mb] = stream_max3(mx[mb], s[mb][0][2 * op], s[mb][0][2 * op + 1]);
    if constexpr (KB == 2) mx[mb] = stream_max3(mx[mb], s[mb][KB - 1][2 * op], s[mb][KB - 1][2 * op + 1]);
  }
  template <int SLOT, int... Ns>
  __device__ __forceinline__ void weights_of_slot(std::integer_sequence<int, Ns...>) {
    ((slot_of(Ns) == SLOT ? weights<Ns>() : (void)0), ...);
  }

  // The first tile: S^T alone.  In either function request(0) asks for the K rows of the tile after next, once the fragments
  // of K have all been read, and request(1) for the V rows of the next one, once those of V have.
  template <typename Request>
  __device__ __forceinline__ void first(Request&& request) {
    unrolled<S_SLOTS>([&](auto slot) __attribute__((always_inline)) {
      constexpr int I = decltype(slot)::value;
      score<I>();
      if constexpr (I == 1) request(Num<0>{});
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) settle(acc[MB - 1][kb]);
    unrolled<8 * MB>([&](auto n) __attribute__((always_inline)) { take<decltype(n)::value, 1>(); });
  }
  template <typename Request>
  __device__ __forceinline__ void next(const char* v_lds, uint32_t voff, Request&& request) {
    unrolled<S_SLOTS + O_SLOTS>([&](auto slot) __attribute__((always_inline)) {
      constexpr int I = decltype(slot)::value, o = I - S_SLOTS;
      if constexpr (I < S_SLOTS) score<I>();
      else output<(o > 0 ? o : 0)>();
      weights_of_slot<I>(std::make_integer_sequence<int, PAIRS>{});
      if constexpr (I == 1) request(Num<0>{});
      if constexpr (I >= 2 && I < 6)  // the fragments of V, in the order of their use
        unrolled<NJ * DB / 4>([&](auto n) __attribute__((always_inline)) {
          constexpr int F = (I >= 2 && I < 6 ? I - 2 : 0) * (NJ * DB / 4) + decltype(n)::value, j = F / DB, db = F % DB;
          f.v[j][db] = read_v_frag<HD>(v_lds, voff, j, db);
        });
      if constexpr (I == 7) request(Num<1>{});
      if constexpr (o >= 0) {
        // row block mb's weights are all made before the products of its last piece: its copy may be overwritten
        constexpr int mb = o / O_PER / NJ;
        if constexpr (o / O_PER % NJ == NJ - 1) take<8 * mb + 8 / O_PER * (o % O_PER), 8 / O_PER>();
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  // accumulator r of key block kb is key 32 kb + 8*(r/4) + 4h + r%4 of the tile
  // limit(mb): the last position that this lane's row of row block mb sees.
  template <typename Limit>
  __device__ __forceinline__ void mask(Limit&& limit, int lane, int cnt, int pos) {
    const int h = lane >> 5;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int lim = min(cnt - 1, limit(mb) - pos) - 4 * h;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * kb + 8 * (r >> 2) + (r & 3) > lim) s[mb][kb][r] = -INFINITY;
    }
    unrolled<8 * MB>([&](auto n) __attribute__((always_inline)) { max_step<decltype(n)::value>(); });
  }
  // The reference maximum of a row is only raised (and O, l rescaled) when the tile outgrows it by more than the slack, so
  // after the first tiles the multiplies on O are rare.  At the first tile O and l are zero and stay as they are.
  template <bool FIRST>
  __device__ __forceinline__ void raise() {
    bool grow = FIRST;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx[mb]), __float_as_uint(mx[mb]), false, false);
      mx[mb] = stream_max3(__uint_as_float(r[0]), __uint_as_float(r[1]), __uint_as_float(r[1])) * c;
      if constexpr (!FIRST) grow |= mx[mb] > st.m[mb] + STREAM_RESCALE_SLACK;
    }
    if (FIRST || __builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const float mn = fmaxf(st.m[mb], mx[mb]);
        const float mz = (mn == -INFINITY) ? 0.f : mn;  // every key so far masked: keep the arithmetic finite
        const float alpha = __builtin_amdgcn_exp2f(st.m[mb] - mz);
        st.m[mb] = mn;
        ms[mb] = mz;
        if constexpr (!FIRST) {
          st.l[mb] *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db) {  // (whole registers only; padded on both sides)
            settle(st.o[db][mb]);
            f32x16 t = st.o[db][mb];
            t = t * alpha;
            st.o[db][mb] = t;
            settle(st.o[db][mb]);
          }
        }
      }
    }
  }
};

// Accumulator r of depth block db is depth db*32 + 8*(r/4) + 4h + r%4: four consecutive depths per r/4.
// ------------------------------------------------------------------------------------------------
// Stream kernel.  grid = chains, block = 256.  A workgroup walks a chain of units (item, KV head).  Each
// wavefront owns a quarter of the unit's key range and two private 32-key stages (K 8 KiB + V 8 KiB
// each); no barrier in the key loop.  At the end of a unit the four (O, m, l) states are merged through
// LDS, wavefront w finishing depth block w.
//
// Unit changes.  The merge buffer is the wavefronts' second stages only, one row block at a time, so that a
// wavefront that has finished its quarter can at once request the next unit's first K/V tile into its first
// stage; the next unit's Q rows are requested into an LDS area of their own right after the first merge
// barrier (no wavefront reads the current Q any more then), and the second tile as soon as the merge buffer
// has been read.  The merge thus runs under the latency of those requests instead of in front of it.
//
// Which unit comes next.  With at most one unit per workgroup there is none; otherwise small launches (descriptors in
// the kernel arguments) walk the chains the planner linked.
// Otherwise the units form one queue, longest first: workgroup w starts with unit w and every further unit is
// drawn from a counter in device memory (uploaded with the descriptors, starting at the number of workgroups) by
// one atomic add.  The compute units do not stream equally fast -- by 10 % and more between XCDs, differently from
// box to box and batch to batch -- so chains of equal length planned on the host end up to 25 % apart; with the
// queue a faster workgroup simply takes the next unit earlier.  Wavefront 0 draws half-way through its share of
// the current unit (the order of drawing is the order of finishing, and the round trip is hidden), fetches the
// drawn unit's descriptors and hands them to the other wavefronts through LDS at the unit's end.  Which workgroup
// computes a unit has no influence on the unit's result.
//
// LDS map: [0, 128 KiB) stages, wavefront w at w * 32 KiB (stage 0, stage 1); then the (m, l) exchange
// (2 KiB); then the Q rows of the unit, laid out and swizzled like a K tile of MB * 32 rows; then the next
// unit's descriptors as published by wavefront 0.
// ------------------------------------------------------------------------------------------------
constexpr int STREAM_TILE_BYTES = 8192;                         // K or V of one tile
constexpr int STREAM_STAGE_BYTES = 2 * STREAM_TILE_BYTES;      // 16 KiB
constexpr int STREAM_WAVE_BYTES = 2 * STREAM_STAGE_BYTES;      // 32 KiB
constexpr int STREAM_ML_OFFSET = 4 * STREAM_WAVE_BYTES;        // after the stages
constexpr int STREAM_MAX_MB = 3;                               // row blocks of the widest instantiation
constexpr int STREAM_ML_ROWS = STREAM_MAX_MB * 32;             // rows per wavefront in the (m, l) exchange
constexpr int STREAM_Q_OFFSET = STREAM_ML_OFFSET + 4 * STREAM_ML_ROWS * 2 * 4;
constexpr int STREAM_NEXT_OFFSET = STREAM_Q_OFFSET + STREAM_MAX_MB * 32 * ROW_BYTES;
constexpr int STREAM_LDS_BYTES = STREAM_NEXT_OFFSET + 128;
static_assert(STREAM_LDS_BYTES <= 160 * 1024, "one workgroup per compute unit: all of its LDS, no more");

// One wavefront moves 1 KiB of query rows HBM -> LDS into the Q area: packed row `blk * ROWS_PER_KIB + l / CHUNKS` of
// the unit (clamped to its last row), chunk slots swizzled as for a K tile so that read_k_frag serves as the
// reader of Q's B-operand fragments.
template <int HD, bool GEN>
__device__ __forceinline__ void load_q_kib(const Ctx& c, const char* q_tok0, int g, int row0, int last_row,
                                           char* q_lds, int blk, int lane) {
  typedef Geo<HD> G;
  const int row = blk * G::ROWS_PER_KIB + lane / G::CHUNKS;
  const int chunk = (lane % G::CHUNKS) ^ G::k_swizzle(row);
  const int arow = min(row0 + row, last_row);
  const int tok = row_token<GEN>(c, arow);
  const uint32_t voff = (uint32_t)((tok * c.n_q_heads + g * c.group + row_head<GEN>(c, arow, tok)) * G::ROW + chunk * 16);
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_ptr)(q_lds + blk * 1024);
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2"
      :
      : "s"(lds_addr), "v"(voff), "s"(q_tok0)
      : "memory", "m0");
}

__device__ __forceinline__ void lds_barrier() {
  // LDS traffic of this wavefront has completed; K/V requests stay in flight (no vmcnt wait here)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Arrival counters: zero whenever no kernel that uses them runs (the last arrival takes its counter back to zero).
__device__ uint32_t g_arrivals[ARRIVAL_SLICES * ARRIVALS_PER_SLICE];

// Split rows of a small batch, merged by the workgroup that finishes the last of the splits (every workgroup has one unit):
// a merge launch costs the stream 5 us and the host 4 more, of 14 and 16 for one decoding session on 3000 tokens.  The
// partial rows were written by workgroups on other XCDs, whose L2 is not this one's: they are stored through to memory and
// loaded from there (agent scope, see store_for_others), every wavefront waits until its own stores have arrived, the workgroup
// meets, and one lane counts.  The last one to count merges.  Nobody waits for anybody: a workgroup that is not the last one
// ends.  (With ordinary stores, the count a release that writes the L2 back and an acquire that invalidates the caches, the one
// session's step took 11.2 us instead of 10.2.)
// D / 4 lanes take a row; with few rows the splits of one row are spread over several lane groups, whose sums meet in LDS.
// The order of the additions depends on the plan alone, not on who comes last.
template <int HD, bool GEN>
__device__ __forceinline__ void merge_if_last(const Ctx& c, const DkEntry& e, const DkItem& it, int g, uint32_t* arrivals,
                                              char* smem) {
  constexpr int LANES = HD / 4, GROUPS = 256 / LANES, AHEAD = 8;
  const int nsplit = it.merge & 255;
  uint32_t* counter = arrivals + (it.merge >> 8) * c.n_kv_heads + g;
  uint32_t* seen = (uint32_t*)(smem + STREAM_NEXT_OFFSET);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *seen = before;
    if (before == (uint32_t)nsplit - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (*seen != (uint32_t)nsplit - 1) return;

  int spread = 1;  // lane groups per row
  while (2 * spread * it.nrows <= GROUPS) spread *= 2;
  const int lane = threadIdx.x % LANES, grp = threadIdx.x / LANES;
  const int first = grp % spread;
  f32x4* xo = (f32x4*)smem;                       // [lane group][lane]
  float2* xml = (float2*)(smem + 256 * 16);       // [lane group]
  const int64_t srow = (int64_t)it.nrows * c.n_kv_heads;  // partial rows from one split of a row to the next
  for (int r0 = 0; r0 < it.nrows; r0 += GROUPS / spread) {
    const int rl = r0 + grp / spread;
    const int64_t prow = (int64_t)(it.part_base + min(rl, it.nrows - 1)) * c.n_kv_heads + g;
    const f32x4* p = (const f32x4*)(c.parts + prow * HD) + lane;
    const float2* ml = (const float2*)c.parts_ml + prow;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f, m = -INFINITY;
    const auto add = [&](float wm, float wl, const f32x4& v) {
      const float mn = fmaxf(m, wm);
      const float ms = (mn == -INFINITY) ? 0.f : mn;
      const float a = __builtin_amdgcn_exp2f(m - ms), f = __builtin_amdgcn_exp2f(wm - ms);
      m = mn;
      l = l * a + f * wl;
      acc = acc * a + f * v;
    };
    for (int s0 = first; s0 < nsplit; s0 += spread * AHEAD) {
      f32x4 v[AHEAD];
      float2 w[AHEAD];
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {  // (a split past the end repeats the last one and is left out below)
        const int64_t at = min(s0 + k * spread, nsplit - 1) * srow;
        w[k] = load_of_others(ml + at);
        v[k] = load_of_others(p + at * LANES);
      }
#pragma unroll
      for (int k = 0; k < AHEAD; ++k)
        if (s0 + k * spread < nsplit) add(w[k].x, w[k].y, v[k]);
    }
    if (spread > 1) {  // (one round: the rows fit the lane groups)
      xo[threadIdx.x] = acc;
      if (lane == 0) xml[grp] = make_float2(m, l);
      __syncthreads();
      if (first == 0)
        for (int k = 1; k < spread; ++k) add(xml[grp + k].x, xml[grp + k].y, xo[threadIdx.x + k * LANES]);
    }
    if (first != 0 || rl >= it.nrows) continue;
    const int row = it.row0 + rl;
    const int tok = row_token<GEN>(c, row);
    const int64_t orow = (int64_t)(e.tok0 + tok) * c.n_q_heads + g * c.group + row_head<GEN>(c, row, tok);
    const float inv = 1.f / l;
    bf16x4 o;
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = (__bf16)(acc[u] * inv);
    *(bf16x4*)(c.out + orow * HD + lane * 4) = o;
    if (c.lse && lane == 0) c.lse[orow] = (m + log2f(l)) * 0.6931471805599453f;
  }
}

// What a workgroup does whose units have at most MB 32-row blocks.
// SINGLE: it has one unit and ends.  (A form of its own, because around a loop over units the compiler makes all of the
// loop's constants first: 1230 instructions in front of the first product instead of 850.  One 150-token turn on 800 cached
// tokens 11.5 / 10.9 us, one decoding session 12.1 / 11.4.)
template <int MB, int HD, bool GEN, bool ONCE, bool INLINE, bool SINGLE>
__device__ __forceinline__ void stream_units(const Ctx& c, const int32_t* links, int n_chains, int32_t* queue, int n_units,
                                             int arrival_slice, char* smem, int unit, int g, DkItem it) {
  int thread = threadIdx.x;
  asm volatile("" : "+v"(thread));  // (nothing of this body is computed ahead of the branch to it)
  const int lane = thread & 63;
  const int wave = __builtin_amdgcn_readfirstlane(thread >> 6);
  char* my = smem + wave * STREAM_WAVE_BYTES;
  const uint32_t my_lds = (uint32_t)(uintptr_t)(lds_void_ptr)my;
  float* ml = (float*)(smem + STREAM_ML_OFFSET);  // [wave][row 0..95][m, l]
  char* q_lds = smem + STREAM_Q_OFFSET;
  int32_t* next_lds = (int32_t*)(smem + STREAM_NEXT_OFFSET);  // [0] unit, [4..11] its DkItem, [12..19] its DkEntry
  constexpr int KT = Tile<HD>::KT, DB = Geo<HD>::DB;
  const uint32_t koff = k_lane_off<HD>(lane), voff = v_lane_off<HD>(lane);
  const bool queued = !INLINE && !SINGLE && queue != nullptr;  // units are drawn from the queue (else: the planner's chains)
  int trace_seq = 0;
  (void)trace_seq;

  // ---- the unit being streamed, and the requests that open a unit ----------------------------------
  DkEntry e = load_desc(c.entries, it.entry);
  KvCursor<Geo<HD>::ROW> cur{c.segs, 0, 0, 0, 0};
  KvTile t0, t1, t2;  // tiles t, t+1 and t+2 of a step
  bool have0 = false, have1 = false, have2 = false;

  // Where this lane finds its 16 bytes of each KiB of K or V rows: made again when a tile's row count or stride changes.
  constexpr int BLOCKS = STREAM_TILE_BYTES / 1024;
  uint32_t k_at[BLOCKS], v_at[BLOCKS];
  int k_cnt = KT, v_cnt = KT;
  uint32_t k_stride = Geo<HD>::ROW, v_stride = Geo<HD>::ROW;
  auto aim = [&](uint32_t (&at)[BLOCKS], auto is_v) __attribute__((always_inline)) {
    constexpr bool IS_V = decltype(is_v)::value != 0;
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b) at[b] = kib_biased_off<IS_V, HD>(IS_V ? v_stride : k_stride, IS_V ? v_cnt : k_cnt, b, lane);
  };
  auto aim_k = [&](const KvTile& t) {
    if (t.cnt == k_cnt && t.stride == k_stride) return;
    k_cnt = t.cnt;
    k_stride = t.stride;
    aim(k_at, Num<0>{});
  };
  auto aim_v = [&](const KvTile& t) {
    if (t.cnt == v_cnt && t.stride == v_stride) return;
    v_cnt = t.cnt;
    v_stride = t.stride;
    aim(v_at, Num<1>{});
  };
  aim(k_at, Num<0>{});
  aim(v_at, Num<1>{});
  auto issue_k = [&](const KvTile& t, int stage) __attribute__((always_inline)) {
    const uint32_t lds = my_lds + (uint32_t)(stage * STREAM_STAGE_BYTES);
    if (ONCE && t.once) load_eight_kib<true>(t.k, k_at, lds);
    else load_eight_kib<false>(t.k, k_at, lds);
  };
  auto issue_v = [&](const KvTile& t, int stage) __attribute__((always_inline)) {
    const uint32_t lds = my_lds + (uint32_t)(stage * STREAM_STAGE_BYTES + STREAM_TILE_BYTES);
    if (ONCE && t.once) load_eight_kib<true>(t.v, v_at, lds);
    else load_eight_kib<false>(t.v, v_at, lds);
  };
  auto issue = [&](const KvTile& t, int stage) {
    aim_k(t);
    issue_k(t, stage);
    aim_v(t);
    issue_v(t, stage);
  };
  // The unit's Q rows (this wavefront's share of them), then this wavefront's quarter of its keys: cursor, first tile
  // requested into stage 0.
  auto open = [&](const DkItem& u, const DkEntry& ue, int ug) {
    const char* q_tok0 = (const char*)c.q + (int64_t)ue.tok0 * c.n_q_heads * Geo<HD>::ROW;
    int q_lane = lane;
    asm volatile("" : "+v"(q_lane));  // (per-lane offsets are made here, not kept in registers that the key loop needs)
#pragma unroll
    for (int b = 0; b < MB * 8 / Tile<HD>::KB; b += 4)
      load_q_kib<HD, GEN>(c, q_tok0, ug, u.row0, u.row0 + u.nrows - 1, q_lds, b + wave, q_lane);
    const int ntile = (u.kv_hi - u.kv_lo + KT - 1) / KT;
    const int per = (ntile + 3) / 4 * KT;
    const int lo = min(u.kv_hi, u.kv_lo + wave * per);
    const int hi = min(u.kv_hi, lo + per);
    cur = KvCursor<Geo<HD>::ROW>{c.segs, ue.seg_begin, ue.seg_end, lo, hi};
    have0 = cur.next(c, ug, KT, t0);
    if (have0) issue(t0, 0);
  };
  auto open_second = [&](int ug) {
    have1 = have0 && cur.next(c, ug, KT, t1);
    if (have1) issue(t1, 1);
  };

  open(it, e, g);
  open_second(g);
  if (wave == 0) DK_STR(0, 10);  // (kernel entry, a few scalar loads late)
  while (true) {
    // The descriptors of the next unit are fetched while this one is being streamed, so that a unit change
    // does not start with a chain of dependent memory round trips.
    int next_unit = -1;
    DkItem next_it = it;
    DkEntry next_e = e;
    if (!queued && !SINGLE) {
      next_unit = load_desc(links, n_chains + unit);
      if (!SINGLE && next_unit >= 0) {
        int head;
        next_it = load_desc(c.items, unit_item(c, next_unit, head));
        next_e = load_desc(c.entries, next_it.entry);
      }
    }
    // queue: wavefront 0 draws in iteration draw_at of its key loop (an ordinary atomic: the compiler keeps account
    // of it and waits for the answer where it is first used, after the loop, when no K/V request is in flight)
    const bool drawer = queued && wave == 0;
    int drawn = 0;
    bool drew = false;
    const auto draw = [&]() {
      if (lane == 0) drawn = __hip_atomic_fetch_add(queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      drew = true;
    };
    const int last_row = it.row0 + it.nrows - 1;
    const int min_limit = e.n + row_token<GEN>(c, it.row0);

    RowState<MB, HD> st;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      st.m[mb] = -INFINITY;
      st.l[mb] = 0.f;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        f32x16 z = {0};
        asm volatile("" : "+a"(z));  // born in an accumulation register tuple as a whole
        st.o[db][mb] = z;
      }
    }

    // This wavefront's share of Q and its first K rows have arrived (younger: the first V rows and the second tile), and
    // everybody's share of Q.
    if (wave == 0) DK_STR(trace_seq, 0);
    if (have1) wait_vmcnt<24>(); else if (have0) wait_vmcnt<8>(); else wait_vmcnt<0>();
    lds_barrier();
    QFrags<MB, HD, SINGLE> qf;
    qf.q_lds = q_lds;
    qf.koff = koff;
    if (have0) qf.load();
    if (wave == 0) DK_STR(trace_seq, 1);

    // Two private stages per wavefront, each a half for K and one for V.  Step t reads V(t-1) and at its end K(t+1); as soon
    // as K(t) and V(t-1) have been read their places take K(t+2) and V(t+1), so 16 to 32 KiB per wavefront are in flight.
    // (wavefront 0's share of the unit is at least this many tiles: ragged segment ends only add some)
    const auto limit = [&](int mb) { return e.n + row_token<GEN>(c, min(it.row0 + mb * 32 + (lane & 31), last_row)); };
    const int my_tiles = ((it.kv_hi - it.kv_lo + KT - 1) / KT + 3) / 4;
    const int draw_at = my_tiles / 2;
    if (have0) {
      StreamStep<MB, HD, GEN, SINGLE> step{qf, st, c.c};
      int stage = 0, iter = 0;  // where tile t lives, and t
      // end of step t: K(t+1) and V(t) have landed when only what step t requested is still out
      auto finish = [&](const KvTile& t, auto is_first) __attribute__((always_inline)) {
        if (have2) wait_vmcnt<16>(); else if (have1) wait_vmcnt<8>(); else wait_vmcnt<0>();
        if (have1) read_k_frags<HD>(my + (stage ^ 1) * STREAM_STAGE_BYTES, koff, step.f);
        if (t.cnt < KT || t.pos + KT - 1 > min_limit) step.mask(limit, lane, t.cnt, t.pos);
        step.template raise<decltype(is_first)::value != 0>();
      };
      read_k_frags<HD>(my, koff, step.f);
      have2 = have1 && cur.next(c, g, KT, t2);
      if (have2) aim_k(t2);
      step.first([&](auto) __attribute__((always_inline)) {
        if (!have2) return;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue_k(t2, 0);
      });
      finish(t0, Num<1>{});
      while (true) {
        const bool last = !have1;  // there is no tile t: S^T(t) comes out as something nobody reads
        t0 = t1;
        t1 = t2;
        have1 = have2;
        stage ^= 1;
        ++iter;
        have2 = have1 && cur.next(c, g, KT, t2);
        if (drawer && !drew && iter >= draw_at) draw();
        if (have2) aim_k(t2);
        if (have1) aim_v(t1);
        step.next(my + (stage ^ 1) * STREAM_STAGE_BYTES + STREAM_TILE_BYTES, voff, [&](auto of_v) __attribute__((always_inline)) {
          if constexpr (decltype(of_v)::value == 0) {
            if (!have2) return;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_k(t2, stage);
          } else {
            if (!have1) return;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_v(t1, stage ^ 1);
          }
        });
        if (last) break;
        finish(t0, Num<0>{});
      }
    }
    DK_STR(trace_seq, 2 + wave);  // each wavefront's own end of streaming

    // ---- unit change: both stages of this wavefront are free ----------------------------------------
    if (drawer) {
      if (!drew) draw();  // (a share with no tiles at all)
      const int q = __builtin_amdgcn_readfirstlane(drawn);
      next_unit = q < n_units ? q : -1;
      if (!SINGLE && next_unit >= 0) {
        int head;
        next_it = load_desc(c.items, unit_item(c, next_unit, head));
        next_e = load_desc(c.entries, next_it.entry);
      }
      if (lane == 0) {
        next_lds[0] = next_unit;
        next_lds[4] = next_it.entry;
        next_lds[5] = next_it.row0;
        next_lds[6] = next_it.nrows;
        next_lds[7] = next_it.kv_lo;
        next_lds[8] = next_it.kv_hi;
        next_lds[9] = next_it.part_row0;
        next_lds[12] = next_e.seg_begin;
        next_lds[13] = next_e.seg_end;
        next_lds[14] = next_e.n;
        next_lds[15] = next_e.delta;
        next_lds[16] = next_e.tok0;
      }
    }

    // small append-and-attend calls: this workgroup's share of the new rows is read now and goes into the arena after the
    // merge, which takes as long as the reads do
    RowCopy<INLINE, Geo<HD>::ROW> copy;
    if constexpr (INLINE) {
      if (SINGLE || next_unit < 0) copy.load(c);
    }

    // ---- merge the four wavefront states ------------------------------------------------------------
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int db = 0; db < DB; ++db) settle(st.o[db][mb]);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const float lt = st.l[mb] + __shfl_xor(st.l[mb], 32);
      if (lane < 32) {
        ml[(wave * STREAM_ML_ROWS + mb * 32 + lane) * 2] = st.m[mb];
        ml[(wave * STREAM_ML_ROWS + mb * 32 + lane) * 2 + 1] = lt;
      }
    }
    int next_g = 0;
    uint32_t bad_rows[MB];  // GEN: rows whose sums are not finite, see redo_rows
    float bad_m[MB], bad_l[MB];
    // the four wavefronts share out the depth blocks: a whole one each (HD 128) or half of one (HD 64)
    constexpr int NACC = DB * 4;  // accumulators of a row block per wavefront after the merge
    const int db = wave * DB / 4, r0 = wave * NACC % 16;
    const bool for_others = SINGLE && arrival_slice >= 0 && it.merge != 0;  // see merge_if_last
    int store_lane = lane;
    asm volatile("" : "+v"(store_lane));  // (addresses of the output are made here, each time)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      // row block mb of every wavefront's O goes through the wavefronts' second stages: [db][r / 4][lane][r % 4]
      f32x4* mine = (f32x4*)(my + STREAM_STAGE_BYTES);
#pragma unroll
      for (int d4 = 0; d4 < DB; ++d4)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          mine[(d4 * 4 + i) * 64 + lane] = f32x4{st.o[d4][mb][4 * i], st.o[d4][mb][4 * i + 1], st.o[d4][mb][4 * i + 2], st.o[d4][mb][4 * i + 3]};
      lds_barrier();
      if (mb == 0) {
        if (wave == 0) DK_STR(trace_seq, 6);
        if (queued) {  // what wavefront 0 drew (field by field: the values must stay in scalar registers)
          const auto word = [&](int i) { return __builtin_amdgcn_readfirstlane(next_lds[i]); };
          next_unit = word(0);
          next_it.entry = word(4);
          next_it.row0 = word(5);
          next_it.nrows = word(6);
          next_it.kv_lo = word(7);
          next_it.kv_hi = word(8);
          next_it.part_row0 = word(9);
          next_e.seg_begin = word(12);
          next_e.seg_end = word(13);
          next_e.n = word(14);
          next_e.delta = word(15);
          next_e.tok0 = word(16);
        }
        if (!SINGLE && next_unit >= 0) (void)unit_item(c, next_unit, next_g);
        // every wavefront is past its key loop: its first stage may take the next unit's first tile, and no
        // wavefront reads the current unit's Q any more
        if (!SINGLE && next_unit >= 0) open(next_it, next_e, next_g);  // (have0, t0, cur now belong to the next unit)
      }
      const int row = mb * 32 + (lane & 31);
      float mw[4], lw[4];
      float mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        mw[w] = ml[(w * STREAM_ML_ROWS + row) * 2];
        lw[w] = ml[(w * STREAM_ML_ROWS + row) * 2 + 1];
        mx = fmaxf(mx, mw[w]);
      }
      const float ms = (mx == -INFINITY) ? 0.f : mx;
      float lsum = 0.f;
      f32x4 acc[NACC / 4];
#pragma unroll
      for (int i = 0; i < NACC / 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float f = __builtin_amdgcn_exp2f(mw[w] - ms);
        lsum += f * lw[w];
        const f32x4* theirs = (const f32x4*)(smem + w * STREAM_WAVE_BYTES + STREAM_STAGE_BYTES);
#pragma unroll
        for (int i = 0; i < NACC / 4; ++i) acc[i] += f * theirs[(db * 4 + r0 / 4 + i) * 64 + lane];
      }
      // the buffer has been read everywhere: the next row block, or the next unit's second tile, may overwrite it
      if (mb + 1 < MB || !SINGLE && next_unit >= 0) lds_barrier();
      // (one row block's result at a time: the merged rows of all blocks together would not fit the registers)
      const float mm[1] = {mx}, ll[1] = {lsum};
      store_quads<HD, GEN>(c, e, it, g, row, db * 32 + 2 * r0 + 4 * (store_lane >> 5), acc, lsum, for_others);
      if (wave == 0) store_ml<1, GEN>(c, e, it, g, mb * 32, lane, mm, ll, for_others);
      if constexpr (GEN) {
        float z = 0.f;  // NaN if any of the row's sums is not finite
#pragma unroll
        for (int i = 0; i < NACC / 4; ++i)
#pragma unroll
          for (int u = 0; u < 4; ++u) z = __builtin_fmaf(acc[i][u], 0.f, z);
        const uint64_t bad = __builtin_amdgcn_ballot_w64(z != 0.f);
        bad_rows[mb] = (uint32_t)(bad | bad >> 32);
        bad_m[mb] = mx;
        bad_l[mb] = lsum;
      }
    }
    if constexpr (GEN) {
      uint32_t any = bad_rows[0];
#pragma unroll
      for (int mb = 1; mb < MB; ++mb) any |= bad_rows[mb];
      if (any != 0) {
#pragma unroll 1
        for (int mb = 0; mb < MB; ++mb) {
          const int i1 = MB > 1 ? 1 : 0, i2 = MB > 2 ? 2 : 0;
          const uint32_t rows = mb == 0 ? bad_rows[0] : mb == 1 ? bad_rows[i1] : bad_rows[i2];
          const float m = mb == 0 ? bad_m[0] : mb == 1 ? bad_m[i1] : bad_m[i2];
          const float l = mb == 0 ? bad_l[0] : mb == 1 ? bad_l[i1] : bad_l[i2];
          if (rows != 0) redo_rows<HD, true>(c, e, it, g, mb * 32, rows, m, l, lane, db, [&](int depth) { return depth / (HD / 4) == wave; });
        }
      }
    }
    // (after the stores: the wait that opens the next unit lets exactly this request stay in flight)
    if (!SINGLE && next_unit >= 0) open_second(next_g);
    if (wave == 0) DK_STR(trace_seq, 7);
#ifdef DK_TRACE
    if (threadIdx.x == 0 && trace_seq < 8 && blockIdx.x < 256) g_strace[blockIdx.x][trace_seq][8] = (unsigned long long)(it.kv_hi - it.kv_lo);
    ++trace_seq;
#endif
    if (SINGLE || next_unit < 0) {
      if constexpr (INLINE) copy.store(c);
      break;
    }
    unit = next_unit;
    it = next_it;
    e = next_e;
    g = next_g;
  }
  if (SINGLE && arrival_slice >= 0 && it.merge != 0) merge_if_last<HD, GEN>(c, e, it, g, g_arrivals + arrival_slice * ARRIVALS_PER_SLICE, smem);
}

// INLINE: the descriptors arrive inside the kernel arguments (first argument) and the descriptor pointers are byte
// offsets into them; otherwise they point into the uploaded workspace.
// ONCE: the launch has segments marked DkSeg::once (an instantiation of its own: the choice per tile costs the others 3-7 %).
// A workgroup's first unit has the most rows of those it walks (of a queue, the caller says how many blocks any unit has):
// it takes the body for one, two or three 32-row blocks, so that decoding sessions, verification batches and the row tiles
// of longer turns run side by side in one launch.  A workgroup with a single unit pays that unit's price; a chain pays its
// tallest unit's for all of them, a queued launch the tallest of the launch.
template <int HD, bool GEN, bool ONCE, bool INLINE, bool SINGLE>
__global__ __launch_bounds__(256, 1) void attend_stream_kernel(BlobArg<INLINE> blob, Ctx c, const int32_t* links, int n_chains,
                                                               int32_t* queue, int n_units, int queue_rows, int arrival_slice) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  (void)blob;
  touch_descs<INLINE>();
  c.entries = resolve_desc<INLINE>(c.entries);
  c.segs = resolve_desc<INLINE>(c.segs);
  c.items = resolve_desc<INLINE>(c.items);
  links = resolve_desc<INLINE>(links);
  const bool queued = !INLINE && !SINGLE && queue != nullptr;
  const int unit = queued || SINGLE ? (int)blockIdx.x : load_desc(links, blockIdx.x);
  int g;
  const DkItem it = load_desc(c.items, unit_item(c, unit, g));
  const int rows = queued ? queue_rows : it.nrows;
  if (rows <= 32) stream_units<1, HD, GEN, ONCE, INLINE, SINGLE>(c, links, n_chains, queue, n_units, arrival_slice, smem, unit, g, it);
  else if (rows <= 64) stream_units<2, HD, GEN, ONCE, INLINE, SINGLE>(c, links, n_chains, queue, n_units, arrival_slice, smem, unit, g, it);
  else stream_units<3, HD, GEN, ONCE, INLINE, SINGLE>(c, links, n_chains, queue, n_units, arrival_slice, smem, unit, g, it);
}


namespace {

template <int HD, bool GEN, bool ONCE, bool INLINE, bool SINGLE>
hipError_t launch_form(int32_t max_rows, const BlobArg<INLINE>& blob, const Ctx& c, const int32_t* links, int32_t n_chains,
                       int32_t* queue, int32_t n_units, int32_t slice, hipStream_t stream) {
  // once per process and instantiation, whatever thread or pool gets here first
  static std::once_flag once;
  static hipError_t status = hipSuccess;
  std::call_once(once, [] {
    status = hipFuncSetAttribute((const void*)attend_stream_kernel<HD, GEN, ONCE, INLINE, SINGLE>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, STREAM_LDS_BYTES);
  });
  if (status != hipSuccess) return status;
  attend_stream_kernel<HD, GEN, ONCE, INLINE, SINGLE><<<dim3((unsigned)n_chains), 256, STREAM_LDS_BYTES, stream>>>(
      blob, c, links, n_chains, queue, n_units, max_rows, slice);
  return hipGetLastError();
}

template <int HD, bool GEN, bool ONCE, bool INLINE>
hipError_t launch_one(int32_t max_rows, const BlobArg<INLINE>& blob, const Ctx& c, const int32_t* links, bool single,
                      int32_t n_chains, int32_t* queue, int32_t n_units, int32_t slice, hipStream_t stream) {
  return single ? launch_form<HD, GEN, ONCE, INLINE, true>(max_rows, blob, c, links, n_chains, queue, n_units, slice, stream)
                : launch_form<HD, GEN, ONCE, INLINE, false>(max_rows, blob, c, links, n_chains, queue, n_units, slice, stream);
}

template <bool ONCE, bool INLINE>
hipError_t launch_shape(const AttendArgs& a, int32_t max_rows, const BlobArg<INLINE>& blob, const Ctx& c,
                        const int32_t* links, bool single, int32_t n_chains, int32_t* queue, int32_t n_units,
                        hipStream_t stream) {
  const int32_t slice = a.arrival_slice;
  if (a.arena.head_dim == 64) return launch_one<64, true, ONCE, INLINE>(max_rows, blob, c, links, single, n_chains, queue, n_units, slice, stream);
  if (a.general) return launch_one<128, true, ONCE, INLINE>(max_rows, blob, c, links, single, n_chains, queue, n_units, slice, stream);
  return launch_one<128, false, ONCE, INLINE>(max_rows, blob, c, links, single, n_chains, queue, n_units, slice, stream);
}

}  // namespace

}  // namespace mfma

hipError_t launch_attend_stream(const AttendArgs& a, const DkItem* items, const int32_t* links, bool single,
                                int32_t n_chains, int32_t max_rows, int32_t* queue, int32_t n_units,
                                hipStream_t stream) {
  using namespace mfma;
  if (n_chains <= 0) return hipSuccess;
  if (a.arena.dtype != 1 || max_rows > STREAM_MAX_MB * 32) return hipErrorInvalidValue;
  if (a.arena.head_dim != 128 && !(a.arena.head_dim == 64 && a.general)) return hipErrorInvalidValue;
  if (queue && a.inline_blob) return hipErrorInvalidValue;  // the queue's counter needs device memory
  const Ctx c = make_ctx(a, items);
  if (a.inline_blob) {
    const BlobArg<true> blob{*a.inline_blob};
    return a.once ? launch_shape<true, true>(a, max_rows, blob, c, links, single, n_chains, queue, n_units, stream)
                  : launch_shape<false, true>(a, max_rows, blob, c, links, single, n_chains, queue, n_units, stream);
  }
  const BlobArg<false> none{0};
  return a.once ? launch_shape<true, false>(a, max_rows, none, c, links, single, n_chains, queue, n_units, stream)
                : launch_shape<false, false>(a, max_rows, none, c, links, single, n_chains, queue, n_units, stream);
}

}  // namespace dk
