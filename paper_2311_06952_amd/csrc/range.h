// range.h -- block-range helpers of the kernels that list or count the samples
// with some property: a block takes a contiguous range of samples (about two
// blocks per CU) and reserves its share of the output with one global add.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace mh {
namespace {

// The chunk of samples [c0, min(c0 + 256, j1)) of a block's range: its
// members (pred true) are numbered in thread order, their count returned and,
// for member number l, put(l, i) called before the block's next barrier.
// Must be called by all threads of a 256-thread block with the same c0, j1.
template <typename Pred, typename Fn>
__device__ __forceinline__ uint32_t chunk_members(uint32_t c0, uint32_t j1, Pred pred, Fn put,
                                                  uint32_t *s_w) {
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  const uint32_t i = c0 + threadIdx.x;
  const bool m = i < j1 && pred(i);
  const uint64_t bal = __ballot(m);
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  __syncthreads();  // the previous chunk's readers of s_w and the staged members are done
  if (lane == 0) s_w[w] = (uint32_t)__popcll(bal);
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    off += q < w ? s_w[q] : 0u;
    tot += s_w[q];
  }
  if (m) put(off + (uint32_t)__popcll(bal & lt), i);
  return tot;
}

// Members of [j0, j1) (pred true), counted by a 256-thread block, and the
// start of their range from one add to *cursor.
template <typename Pred>
__device__ __forceinline__ uint32_t range_reserve(uint32_t j0, uint32_t j1, Pred pred,
                                                  uint32_t *__restrict__ cursor, uint32_t *s_w,
                                                  uint32_t *s_base) {
  uint32_t c = 0;
  for (uint32_t i = j0 + threadIdx.x; i < j1; i += 256u) c += pred(i) ? 1u : 0u;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((threadIdx.x & 63u) == 0) s_w[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t t = s_w[0] + s_w[1] + s_w[2] + s_w[3];
    *s_base = t ? atomicAdd(cursor, t) : 0u;
  }
  __syncthreads();
  return *s_base;
}

inline uint32_t nblk(uint32_t n, uint32_t b = 256) { return (n + b - 1) / b; }
// Samples per block of the range kernels: a multiple of 256, about two blocks
// per CU; and the blocks that cover n.  Their loops step by 256 without
// wrapping for n <= RANGE_MAX_N.
constexpr uint32_t RANGE_MAX_N = 0xFFFFFF00u;
inline uint32_t range_span(const Ctx *ctx, uint32_t n) {
  const uint64_t nb = 2u * (uint64_t)(ctx->num_cu > 0 ? ctx->num_cu : 1);
  const uint64_t s = ((((uint64_t)n + nb - 1) / nb) + 255) / 256 * 256;
  return (uint32_t)(s < 256 ? 256 : s);
}
inline uint32_t range_blocks(uint32_t n, uint32_t span) {
  return (uint32_t)(((uint64_t)n + span - 1) / span);
}

}  // namespace
}  // namespace mh
