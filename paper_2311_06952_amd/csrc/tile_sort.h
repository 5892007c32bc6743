// tile_sort.h -- one wave sorts one (tile, feature): the sorted ranks, the
// prefix masks and the sorted positions of the tile layout.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "internal.h"
#include "xcd.h"

namespace mh {
namespace {

// v of lane ^ J.  J = 1, 2 by a quad permutation, J = 4, 8 by shifts within
// rows of 16 (lane + J where lane & J is zero, else lane - J; the lanes whose
// shift leaves the row are the ones that take the other shift), all DPP moves
// without the LDS pipe; J = 16, 32 by a permute through it.
template <uint32_t J>
__device__ __forceinline__ uint32_t xor_lane32(uint32_t v, uint32_t lane) {
  if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);
  else if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);
  else if constexpr (J == 4 || J == 8) {
    const uint32_t up = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x100 + (int)J, 0xF, 0xF, false);
    const uint32_t dn = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x110 + (int)J, 0xF, 0xF, false);
    return (lane & J) ? dn : up;
  } else {
    return (uint32_t)__shfl_xor((int)v, (int)J, 64);
  }
}
template <uint32_t J, typename KT>
__device__ __forceinline__ KT xor_lane(KT v, uint32_t lane) {
  if constexpr (sizeof(KT) == 4) {
    return (KT)xor_lane32<J>((uint32_t)v, lane);
  } else {
    const uint32_t lo = xor_lane32<J>((uint32_t)v, lane);
    const uint32_t hi = xor_lane32<J>((uint32_t)(v >> 32), lane);
    return ((KT)hi << 32) | lo;
  }
}
// One compare-exchange stage of the bitonic network: merge size K, distance J.
template <uint32_t K, uint32_t J, typename KT>
__device__ __forceinline__ KT bitonic_stage(KT v, uint32_t lane) {
  const KT o = xor_lane<J>(v, lane);
  const bool up = (lane & K) == 0, lo = (lane & J) == 0;
  const KT mn = v < o ? v : o, mx = v < o ? o : v;
  return (lo == up) ? mn : mx;
}
// Inclusive OR-scan of a 64-bit value over the wave: within rows of 16 by
// row shifts of 1, 2, 4 and 8 (a lane without a source in the row ORs zero),
// then the row totals across rows (row broadcasts of lanes 15 and 31).
__device__ __forceinline__ uint64_t or_scan64(uint64_t x) {
  uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
  auto step = [&](auto ctrl_tag, auto mask_tag) {
    constexpr int ctrl = decltype(ctrl_tag)::value, rmask = decltype(mask_tag)::value;
    lo |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, ctrl, rmask, 0xF, false);
    hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, ctrl, rmask, 0xF, false);
  };
  step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});  // row_shr:1
  step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});  // row_shr:2
  step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});  // row_shr:4
  step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});  // row_shr:8
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});  // row_bcast:15
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});  // row_bcast:31
  return ((uint64_t)hi << 32) | lo;
}

// One wave per (tile, feature): sort the tile's ranks with their positions
// (bitonic network across the 64 lanes), write the sorted ranks and the
// prefix masks of the positions in sorted order.  The composite key (rank,
// position) is 32 bits wide when every rank is below 2^26 (fewer than 2^26
// samples), else 64.
//
// Block b works on feature f and tiles 4 q .. 4 q + 3 (one per wave), with
// (f, q) = block xcd_order(b) of the feature-major list (xcd.h), so that an
// XCD's random reads of a feature's ranks stay in its own L2.
template <typename KT>
__device__ __forceinline__ void tile_sort_body(const uint32_t *__restrict__ ranks, uint32_t ld,
                                               TileHdr *__restrict__ hdr, uint32_t bx) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t F = hdr->F;
  const uint32_t tq = (hdr->max_tiles + 3u) / 4u;  // tile quads per feature
  const uint32_t grid = (tq * F + 7u) & ~7u;  // (tile_sort_blocks)
  if (bx >= grid) return;
  const uint32_t bi = xcd_order(bx, grid);
  const uint32_t f = bi / tq, tile = (bi % tq) * 4u + (threadIdx.x >> 6);
  if (f >= F || tile >= hdr->n_tiles) return;
  uint8_t *base = reinterpret_cast<uint8_t *>(hdr);
  const uint32_t info = reinterpret_cast<const uint32_t *>(base + hdr->off_info)[tile];
  const uint32_t *order = reinterpret_cast<const uint32_t *>(base + hdr->off_order);
  const uint32_t cnt = info & 0xFFu;
  // unused lanes sort last: all ones
  constexpr uint32_t KB = sizeof(KT) * 8;
  uint32_t key = (uint32_t)(~KT(0) >> 6);
  if (lane < cnt) key = ranks[(size_t)f * ld + order[tile * TILE_W + lane]];
  // composite (key, position): distinct, so the network sorts a total order
  KT v = ((KT)key << 6) | lane;
  (void)KB;
  // the network: merges of size 2, 4, ..., 64, each halving its distance
  v = bitonic_stage<2, 1>(v, lane);
  v = bitonic_stage<4, 2>(v, lane);
  v = bitonic_stage<4, 1>(v, lane);
  v = bitonic_stage<8, 4>(v, lane);
  v = bitonic_stage<8, 2>(v, lane);
  v = bitonic_stage<8, 1>(v, lane);
  v = bitonic_stage<16, 8>(v, lane);
  v = bitonic_stage<16, 4>(v, lane);
  v = bitonic_stage<16, 2>(v, lane);
  v = bitonic_stage<16, 1>(v, lane);
  v = bitonic_stage<32, 16>(v, lane);
  v = bitonic_stage<32, 8>(v, lane);
  v = bitonic_stage<32, 4>(v, lane);
  v = bitonic_stage<32, 2>(v, lane);
  v = bitonic_stage<32, 1>(v, lane);
  v = bitonic_stage<64, 32>(v, lane);
  v = bitonic_stage<64, 16>(v, lane);
  v = bitonic_stage<64, 8>(v, lane);
  v = bitonic_stage<64, 4>(v, lane);
  v = bitonic_stage<64, 2>(v, lane);
  v = bitonic_stage<64, 1>(v, lane);
  // unused entries: 0x7FFFFFFF, above every rank and threshold (n < 2^31)
  const uint32_t skey = lane < cnt ? (uint32_t)(v >> 6) : 0x7FFFFFFFu;
  const uint32_t pos = (uint32_t)(v & 63u);
  // inclusive OR-scan over lanes: pm[lane + 1]
  const uint64_t bit = or_scan64((lane < cnt) ? (1ull << pos) : 0ull);
  uint8_t *rec = base + hdr->off_data + (size_t)tile * tile_bytes(F);
  uint32_t *sorted = reinterpret_cast<uint32_t *>(rec) + f * TILE_W;
  uint64_t *pm = reinterpret_cast<uint64_t *>(rec + (size_t)F * TILE_W * 4) + f * TILE_W;
  sorted[lane] = skey;
  if (lane < 63u) pm[lane + 1] = bit;
  else pm[0] = 0ull;
  // the compact form: past the count the last sample's position again, so
  // that a running union of (1 << position) stays correct without a test
  const uint32_t last = (uint32_t)__shfl((int)pos, (int)(cnt ? cnt - 1u : 0u), 64);
  base[hdr->off_perm + ((size_t)tile * F + f) * TILE_W + lane] = (uint8_t)(lane < cnt ? pos : last);
}

// Blocks of 256 threads that cover a layout: F per quad of tiles, a multiple
// of 8 (xcd.h).
inline uint32_t tile_sort_blocks(uint32_t max_tiles, uint32_t F) {
  return xcd_grid((uint32_t)(((uint64_t)max_tiles + 3) / 4 * F));
}

}  // namespace
}  // namespace mh
