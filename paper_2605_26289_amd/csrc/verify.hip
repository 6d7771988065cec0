// Greedy verification of speculative batches on the device (paper Sec. 3.8: batched on-device argmax
// over the vocabulary; Alg. 2: accept the drafts that match, front to back).
//
//   argmax_partial_kernel   one workgroup per (row, 32 KiB chunk of the row): 16-byte loads, eight in
//                           flight per lane, running (max, first index) per lane, wavefront shuffle
//                           reduction, one (value, index) pair per chunk.  HBM bound: every logit is
//                           read exactly once, past the caches where there are many of them.
//   verify_finish_kernel    one wavefront per slot: folds the chunk pairs of each of its rows, a lane per row, then
//                           finds the first draft that differs from the row's argmax, in registers.
//
// Measured, 64 slots of nine rows over 128 256 bf16 logits (148 MB), us a call, and the same in fp32: cached loads and
// the argmax of every row through memory 32.4 and 55.1; non-temporal loads alone 29.4 and 49.6; both 28.7 and 48.3.
// Which loads, by the size of the logits (us a call, cached / non-temporal; the same logits again and again, logits that
// a kernel has just written, logits after 600 MB of other writes): 17 MB 8.4 / 8.6, 12.5 / 12.8, 16.8 / 13.3; 52 MB
// 14.7 / 13.5, 17.5 / 20.2, 28.7 / 18.7; 70 MB 17.4 / 16.0, 20.0 / 21.0, 35.0 / 21.4; 105 MB 22.7 / 21.4, 25.4 / 25.6, 49 / 26.6;
// 140 MB 28.3 / 27.0, 31.4 / 31.1, 61 / 32.  From 64 MiB on the non-temporal loads lose at most a microsecond where the
// logits are fresh and win as much or much more elsewhere; below, fresh logits lose up to 3 us.
//
// Ties go to the lowest token id; a NaN logit counts as +infinity.
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace dk {

namespace {

constexpr int VERIFY_THREADS = 256;
constexpr int VERIFY_UNROLL = 8;
constexpr int VERIFY_CHUNK_BYTES = VERIFY_THREADS * 16 * VERIFY_UNROLL;  // 32 KiB of one row per workgroup

struct Best {
  float v;
  int32_t i;
};

__device__ __forceinline__ float as_key(float x) { return x != x ? INFINITY : x; }

// `a` wins over `b` if it is larger, or equal with the lower index
__device__ __forceinline__ Best better(Best a, Best b) {
  const bool take_b = b.v > a.v || (b.v == a.v && b.i < a.i);
  return take_b ? b : a;
}

__device__ __forceinline__ float elem_to_float(float x) { return x; }
__device__ __forceinline__ float elem_to_float(uint16_t bits) { return __uint_as_float((uint32_t)bits << 16); }

template <typename T, bool ONCE>
__global__ __launch_bounds__(VERIFY_THREADS) void argmax_partial_kernel(const T* __restrict__ logits, int64_t row_stride,
                                                                        int64_t vocab, int32_t n_chunks,
                                                                        Best* __restrict__ parts) {
  constexpr int VEC = 16 / (int)sizeof(T);
  constexpr int64_t CHUNK = (int64_t)VERIFY_THREADS * VEC * VERIFY_UNROLL;
  const int32_t row = blockIdx.y, chunk = blockIdx.x;
  const T* p = logits + (int64_t)row * row_stride;
  const int64_t base = (int64_t)chunk * CHUNK;
  typedef uint32_t words __attribute__((ext_vector_type(4)));
  words raw[VERIFY_UNROLL];
  bool full[VERIFY_UNROLL];
#pragma unroll
  for (int u = 0; u < VERIFY_UNROLL; ++u) {
    const int64_t e0 = base + ((int64_t)u * VERIFY_THREADS + threadIdx.x) * VEC;
    full[u] = e0 + VEC <= vocab;
    raw[u] = words{0, 0, 0, 0};
    if (full[u]) raw[u] = ONCE ? __builtin_nontemporal_load((const words*)(p + e0)) : *(const words*)(p + e0);
  }
  Best best{-INFINITY, INT32_MAX};
#pragma unroll
  for (int u = 0; u < VERIFY_UNROLL; ++u) {
    const int64_t e0 = base + ((int64_t)u * VERIFY_THREADS + threadIdx.x) * VEC;
    if (full[u]) {
      const T* lane_vals = (const T*)&raw[u];
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const float v = as_key(elem_to_float(lane_vals[j]));
        // indices only grow along a lane's walk, so "strictly larger" keeps the first maximum
        if (v > best.v || best.i == INT32_MAX) best = Best{v, (int32_t)(e0 + j)};
      }
    } else {
      for (int64_t e = e0; e < vocab && e < e0 + VEC; ++e) {  // ragged end of the row
        const float v = as_key(elem_to_float(p[e]));
        if (v > best.v || best.i == INT32_MAX) best = Best{v, (int32_t)e};
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Best o{__shfl_xor(best.v, off), __shfl_xor(best.i, off)};
    best = better(best, o);
  }
  __shared__ float sv[VERIFY_THREADS / 64];
  __shared__ int32_t si[VERIFY_THREADS / 64];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sv[wave] = best.v;
    si[wave] = best.i;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    Best b{sv[0], si[0]};
#pragma unroll
    for (int w = 1; w < VERIFY_THREADS / 64; ++w) b = better(b, Best{sv[w], si[w]});
    parts[(int64_t)row * n_chunks + chunk] = b;
  }
}

// One wavefront per slot.  Batch rows [r0, r1) of the slot hold [G_last, draft 0, ..., draft k-1]: lane s of a round of 64
// has row r0 + s, its argmax, and the draft that has to equal it.
constexpr int FINISH_AHEAD = 8;  // chunk pairs of a row requested at once
__global__ __launch_bounds__(64) void verify_finish_kernel(const int32_t* __restrict__ cu_delta,
                                                           const Best* __restrict__ parts, int32_t n_chunks,
                                                           const int32_t* __restrict__ batch_tokens,
                                                           int32_t* __restrict__ argmax_rows,
                                                           int32_t* __restrict__ n_keep_out,
                                                           int32_t* __restrict__ next_token_out) {
  const int32_t b = blockIdx.x, lane = threadIdx.x;
  const int32_t r0 = cu_delta[b], r1 = cu_delta[b + 1];
  if (r1 <= r0) {
    if (lane == 0) {
      n_keep_out[b] = 0;
      next_token_out[b] = -1;
    }
    return;
  }
  int32_t first_bad = -1, next = -1;  // of the slot: the first row whose argmax is not the draft after it (or the last row)
  for (int32_t base = r0; base < r1; base += 64) {
    const int32_t r = min(base + lane, r1 - 1);
    const int32_t draft = batch_tokens[min(r + 1, r1 - 1)];
    Best best{-INFINITY, INT32_MAX};
    for (int32_t c = 0; c < n_chunks; c += FINISH_AHEAD) {
      Best p[FINISH_AHEAD];
#pragma unroll
      for (int u = 0; u < FINISH_AHEAD; ++u) p[u] = parts[(int64_t)r * n_chunks + min(c + u, n_chunks - 1)];
#pragma unroll
      for (int u = 0; u < FINISH_AHEAD; ++u) best = better(best, p[u]);
    }
    if (argmax_rows && base + lane < r1) argmax_rows[r] = best.i;
    const uint64_t bad = __builtin_amdgcn_ballot_w64(r == r1 - 1 || best.i != draft);
    if (first_bad < 0 && bad != 0) {
      const int s = __builtin_ctzll(bad);
      first_bad = base - r0 + s;
      next = __shfl(best.i, s);
    }
  }
  if (lane == 0) {
    n_keep_out[b] = 1 + first_bad;
    next_token_out[b] = next;
  }
}

}  // namespace

int64_t verify_workspace_bytes(int32_t total_rows, int64_t vocab, int32_t dtype) {
  const int64_t elem = dtype == 1 ? 2 : 4;
  const int64_t n_chunks = (vocab * elem + VERIFY_CHUNK_BYTES - 1) / VERIFY_CHUNK_BYTES;
  const int64_t pairs = (int64_t)total_rows * n_chunks;
  return ((pairs * 8 + (int64_t)total_rows * 4 + 255) / 256) * 256 + 256;
}

hipError_t launch_verify_greedy(int32_t n_seqs, int32_t total_rows, const int32_t* cu_delta_dev, const void* logits,
                                int32_t dtype, int64_t vocab, int64_t row_stride, const int32_t* batch_tokens,
                                int32_t* argmax_out, int32_t* n_keep_out, int32_t* next_token_out, void* workspace,
                                hipStream_t stream) {
  if (n_seqs <= 0) return hipSuccess;
  const int64_t elem = dtype == 1 ? 2 : 4;
  const int32_t n_chunks = (int32_t)((vocab * elem + VERIFY_CHUNK_BYTES - 1) / VERIFY_CHUNK_BYTES);
  Best* parts = (Best*)workspace;
  if (total_rows > 0) {
    const dim3 grid((unsigned)n_chunks, (unsigned)total_rows);
    const bool once = (int64_t)total_rows * vocab * elem >= (int64_t)64 << 20;
    if (dtype == 1) {
      const auto kernel = once ? argmax_partial_kernel<uint16_t, true> : argmax_partial_kernel<uint16_t, false>;
      kernel<<<grid, VERIFY_THREADS, 0, stream>>>((const uint16_t*)logits, row_stride, vocab, n_chunks, parts);
    } else {
      const auto kernel = once ? argmax_partial_kernel<float, true> : argmax_partial_kernel<float, false>;
      kernel<<<grid, VERIFY_THREADS, 0, stream>>>((const float*)logits, row_stride, vocab, n_chunks, parts);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  verify_finish_kernel<<<dim3((unsigned)n_seqs), 64, 0, stream>>>(cu_delta_dev, parts, n_chunks, batch_tokens, argmax_out,
                                                                   n_keep_out, next_token_out);
  return hipGetLastError();
}

}  // namespace dk
