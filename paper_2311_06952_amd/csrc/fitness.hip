// fitness.hip -- population fitness of classification trees (Algorithm 1;
// eq. opt_c; eq. opt_all; the soft-constraint fitness of Section 3.2).
//
// Main kernel (depth 1..5): lane = tree, 64 trees per wave, all trees of the
// block sharing one LDS-staged tile of up to 63 same-class samples.  For each
// branch node the lane finds c = #{tile ranks < tau} of its feature by a
// 6-step binary search over the tile's sorted column and takes the prefix
// mask pm[c] = the tile samples going left.  The samples reaching node t are
// a 64-bit mask R_t: R_1 = the tile, R_2t = R_t & pm, R_2t+1 = R_t & ~pm.  The
// lane accumulates popcount(R_t & pm) per node in registers; since the tile
// is single-class these are the per-(tree, node, class) left counts, and the
// leaf counts follow from them and the class totals in the epilogue:
// reach(1) = N_k, reach(2t) = left(t), reach(2t+1) = reach(t) - left(t).
//
// Walk kernel (any depth 1..10): lane = sample, the Algorithm 1 walk of one
// tree at a time with an LDS histogram per (leaf, class).
#include <hip/hip_ext.h>

#include <cstdio>

#include "de_body.h"
#include "device_common.h"
#include "epilogue.h"
#include "fitness_core.h"
#include "internal.h"

namespace mh {

size_t walk_scratch_bytes(uint32_t P, uint32_t D, uint32_t K) {
  return (size_t)P * ((size_t)1 << D) * K * 4;
}

size_t cnt_bytes(uint32_t n_problems, uint32_t D, uint32_t K, uint32_t P) {
  return CNT_REP * cnt_copy_elems(n_problems, (1u << D) - 1u, K, P) * 4;
}

namespace {

// After its last flush, a block of the fused kernel takes a ticket on every
// problem its tiles touched; the block that completes a problem's count (all
// blocks covering its tiles have flushed) runs that problem's epilogue and
// DE step at once, with its threads as the individuals and the tile buffer as
// scratch.  The counts are the only data that cross blocks inside a launch
// and are device-coherent atomics: every wave waits for its atomics to
// complete before the ticket is taken, and the finishing block reads the
// counts with agent-scope loads (no L2 write-back or invalidate needed).
template <int D, int WAVES>
__device__ __forceinline__ void fused_tail(const FuseArgs &fa, const uint32_t *__restrict__ info,
                                           uint32_t n_tiles, uint32_t t_begin, uint32_t t_end,
                                           uint32_t K, uint8_t *lds) {
  constexpr int SB = (1 << D) - 1;
  constexpr uint32_t NT = WAVES * 64;
  __shared__ uint32_t s_last;
  const uint32_t P = fa.a.P, Ppad = pad64(P), nb = gridDim.x;
  __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0) expcnt(0) lgkmcnt(0): this wave's atomics are done
  __syncthreads();
  const uint32_t s_lo = info[t_begin] >> 16, s_hi = info[t_end - 1] >> 16;
  // scratch carved from the (now free) dynamic LDS
  double *s_cost = reinterpret_cast<double *>(lds);
  uint32_t *s_idx = reinterpret_cast<uint32_t *>(lds + NT * 8);
  uint32_t *s_nu = reinterpret_cast<uint32_t *>(lds + NT * 12);
  double *rows = fa.rows_in_lds ? reinterpret_cast<double *>(lds + NT * 12 + 1024) : nullptr;
  for (uint32_t s = s_lo; s <= s_hi; ++s) {
    if (threadIdx.x == 0) {
      const uint32_t t0 = fa.segoff[s * K], t1 = fa.segoff[s * K + K];
      // blocks covering tiles [t0, t1): block b covers [T b / nb, T (b + 1) / nb),
      // at least one tile each when nb <= T, at most one when nb > T
      uint32_t covering;
      if (nb > n_tiles) {
        covering = t1 - t0;
      } else {
        const uint32_t bf = (uint32_t)(((uint64_t)(t0 + 1) * nb - 1) / n_tiles);
        const uint32_t bl = (uint32_t)(((uint64_t)t1 * nb - 1) / n_tiles);
        covering = bl - bf + 1;
      }
      const uint32_t expected = covering * gridDim.y;
      const uint32_t old = atomicAdd(&fa.done[s], 1u);
      s_last = (old + 1 == expected) ? 1u : 0u;
      if (s_last) fa.done[s] = 0;  // nobody else touches it in this launch
    }
    __syncthreads();
    if (s_last) de_gen_body<D, CNT_REP, true, false>(fa.a, fa.e, s, s_cost, s_idx, rows, s_nu);
    __syncthreads();
  }
}

// One block's share of a population evaluation on one tile set: block bx of
// nbx takes tiles [n_tiles bx / nbx, n_tiles (bx + 1) / nbx) for the trees
// by * NT .. by * NT + NT - 1.
template <int D, int WAVES, bool FUSE>
__device__ __forceinline__ void fitness_block(const TileHdr *__restrict__ hdr,
                                              const uint8_t *__restrict__ feat,
                                              const uint32_t *__restrict__ tau, uint32_t P,
                                              uint32_t *__restrict__ cnt, const FuseArgs &fa,
                                              uint32_t bx, uint32_t nbx, uint32_t by,
                                              uint8_t *lds) {
  constexpr int SB = (1 << D) - 1;
  constexpr uint32_t NT = WAVES * 64;
  const uint8_t *base = reinterpret_cast<const uint8_t *>(hdr);
  const uint32_t F = hdr->F, K = hdr->K;
  const uint32_t n_tiles = hdr->n_tiles;
  const uint32_t t_begin = (uint32_t)((uint64_t)n_tiles * bx / nbx);
  const uint32_t t_end = (uint32_t)((uint64_t)n_tiles * (bx + 1) / nbx);
  if (t_begin >= t_end) return;
  const uint32_t *__restrict__ info = reinterpret_cast<const uint32_t *>(base + hdr->off_info);
  const uint8_t *__restrict__ data = base + hdr->off_data;
  const size_t rec_bytes = tile_bytes(F);
  const uint32_t nchunk = 48u * F;
  const uint32_t r = by * NT + threadIdx.x;
  const bool live = r < P;
  const uint32_t Ppad = pad64(P);
  const uint32_t mregion = mask_region(F);
  // absolute LDS addresses: sorted column f at s0 + f * SCOL; after the
  // search a = s0 + f * SCOL + 4c, and pm[c] of column f is at kmask + 2a
  const uint32_t s0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint8_t *)lds);
  const uint32_t kmask = s0 + mregion - 2u * s0;

  NodeState<D> ns;
  uint32_t cur_sub = 0xFFFFFFFFu, cur_cls = 0xFFFFFFFFu;
#pragma unroll
  for (int t = 0; t < SB; ++t) ns.acc[t] = 0;

  uint32_t *const cnt_rep =
      cnt + (bx % CNT_REP) * cnt_copy_elems(hdr->n_problems, SB, K, P);
  auto flush = [&](uint32_t sub, uint32_t cls) {
    if (!live) return;
    uint32_t *c = cnt_rep + ((size_t)sub * SB * K + cls) * Ppad + r;
#pragma unroll
    for (int t = 0; t < SB; ++t) {
      if (ns.acc[t]) atomicAdd(c + (size_t)t * K * Ppad, ns.acc[t]);
      ns.acc[t] = 0;
    }
  };

  uint4 pf[PF];
  auto prefetch = [&](uint32_t tile) {
    const uint4 *__restrict__ src = reinterpret_cast<const uint4 *>(data + (size_t)tile * rec_bytes);
#pragma unroll
    for (int k = 0; k < PF; ++k) {
      const uint32_t c = threadIdx.x + k * NT;
      if (c < nchunk) pf[k] = src[c];
    }
  };
  // the next tile's info word travels with its prefetch
  prefetch(t_begin);
  uint32_t inf_next = info[t_begin];

  for (uint32_t tile = t_begin; tile < t_end; ++tile) {
    const uint32_t inf = inf_next;
    const uint32_t sub = inf >> 16, cls = (inf >> 8) & 0xFFu, count = inf & 0xFFu;
    if (sub != cur_sub || cls != cur_cls) {
      if (cur_sub != 0xFFFFFFFFu) flush(cur_sub, cur_cls);
      if (sub != cur_sub) {
        const uint8_t *fr = feat + ((size_t)sub * P + (live ? r : 0)) * SB;
        const uint32_t *tr = tau + ((size_t)sub * P + (live ? r : 0)) * SB;
#pragma unroll
        for (int t = 0; t < SB; ++t) {
          uint32_t f = live ? fr[t] : 0u;
          f = f <= F ? f : 0u;  // an out-of-range feature is treated as no split
          ns.col[t] = s0 + (f ? f - 1u : 0u) * SCOL;
          ns.thr[t] = f ? tr[t] : 0u;
        }
        // the parameters must have landed before the prefetch below is
        // issued, or every later wait would have to drain the prefetch too
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      }
      cur_sub = sub;
      cur_cls = cls;
    }
    __syncthreads();  // the previous tile is no longer read
#pragma unroll
    for (int k = 0; k < PF; ++k) {
      const uint32_t c = threadIdx.x + k * NT;
      if (c < nchunk) stage_chunk(lds, mregion, F, c, pf[k]);
    }
    if (nchunk > PF * NT) {  // wide rows: the rest without prefetch
      const uint4 *__restrict__ src =
          reinterpret_cast<const uint4 *>(data + (size_t)tile * rec_bytes);
      for (uint32_t c = threadIdx.x + PF * NT; c < nchunk; c += NT)
        stage_chunk(lds, mregion, F, c, src[c]);
    }
    __syncthreads();
    if (tile + 1 < t_end) {
      prefetch(tile + 1);
      inf_next = info[tile + 1];
    }
    uint64_t R[1 << D];
    R[1] = (1ull << count) - 1ull;  // count <= 63
    eval_nodes<D, 1>(kmask, ns, R);
  }
  flush(cur_sub, cur_cls);
  if constexpr (FUSE) {
    __syncthreads();  // the tile buffer becomes DE scratch
    fused_tail<D, WAVES>(fa, info, n_tiles, t_begin, t_end, K, lds);
  }
}

template <int D, int WAVES, bool FUSE>
__global__ __launch_bounds__(WAVES * 64) void k_fitness_bits(
    const TileHdr *__restrict__ hdr, const uint8_t *__restrict__ feat,
    const uint32_t *__restrict__ tau, uint32_t P, uint32_t *__restrict__ cnt, FuseArgs fa) {
  extern __shared__ __align__(16) uint8_t lds[];
  fitness_block<D, WAVES, FUSE>(hdr, feat, tau, P, cnt, fa, blockIdx.x, gridDim.x, blockIdx.y,
                                lds);
}

// Several independent population evaluations (one per job, each on its own
// tile set with its own trees and counters) in one launch: block b works for
// job job_of[b] as its block b - blk0 of nblk.  Every job's population fits
// one block (P <= WAVES * 64).
template <int D, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_fitness_jobs(const FitJob *__restrict__ jobs,
                                                             const uint16_t *__restrict__ job_of) {
  extern __shared__ __align__(16) uint8_t lds[];
  const FitJob jb = jobs[job_of[blockIdx.x]];
  fitness_block<D, WAVES, false>(jb.hdr, jb.feat, jb.tau, jb.P, jb.cnt, FuseArgs{},
                                 blockIdx.x - jb.blk0, jb.nblk, 0, lds);
}

// Epilogue from node left counts (tile path).  One thread per (sub, tree).
template <int D>
__global__ void k_epilogue_nodes(uint32_t *__restrict__ cnt, const uint32_t *__restrict__ ctot,
                                 const uint8_t *__restrict__ feat, uint32_t P, uint32_t K,
                                 uint32_t n_problems, uint32_t n_min, double alpha,
                                 FitnessOut out) {
  constexpr int SB = (1 << D) - 1, SL = 1 << D;
  const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= n_problems * P) return;
  const uint32_t sub = gid / P, r = gid % P;
  const uint32_t Ppad = pad64(P);
  const size_t tr = (size_t)sub * P + r;
  TreeScore sc = epilogue_node_counts<D, CNT_REP>(
      cnt + (size_t)sub * SB * K * Ppad, ctot + (size_t)sub * K, K, Ppad, r, feat + tr * SB,
      n_min, alpha, out.counts ? out.counts + tr * SL * K : nullptr,
      out.label ? out.label + tr * SL : nullptr, cnt_copy_elems(n_problems, SB, K, P));
  if (out.correct) out.correct[tr] = sc.correct;
  if (out.cost) out.cost[tr] = sc.cost;
}

constexpr uint32_t EPI_THREADS = 256;

// One tree's epilogue from its leaf counts [SL][K] (eq. opt_c, eq. opt_all
// and the soft-constraint fitness of Section 3.2), by a block of EPI_THREADS
// threads: labels (lowest class of the largest count, an empty leaf class
// 0), correct count and cost, and the counts cleared after they are read.
// Called by every thread of the block.  (Scoring a group's trees in the walk
// launch's last block instead of this separate launch was measured slower: that
// block's coherent loads ran one after another at the end of the launch.)
__device__ __forceinline__ void leaf_epilogue_tree(uint32_t *__restrict__ leafcnt,
                                                   const uint8_t *__restrict__ feat, uint32_t r,
                                                   uint32_t D, uint32_t K, uint32_t n_min,
                                                   double alpha, const FitnessOut &out,
                                                   uint32_t (*s_red)[EPI_THREADS / 64]) {
  const uint32_t SB = (1u << D) - 1u, SL = 1u << D;
  uint32_t correct = 0, nviol = 0, nsplit = 0, n_sub = 0;
  for (uint32_t l = threadIdx.x; l < SL; l += EPI_THREADS) {
    uint32_t *c = leafcnt + ((size_t)r * SL + l) * K;
    uint32_t best = 0, bk = 0, nl = 0;
    for (uint32_t k = 0; k < K; ++k) {
      const uint32_t v = c[k];
      c[k] = 0;
      if (out.counts) out.counts[((size_t)r * SL + l) * K + k] = v;
      nl += v;
      if (v > best) {
        best = v;
        bk = k;
      }
    }
    n_sub += nl;
    correct += best;
    nviol += (nl > 0 && nl < n_min) ? 1u : 0u;
    if (out.label) out.label[(size_t)r * SL + l] = (uint8_t)bk;
  }
  for (uint32_t t = threadIdx.x; t < SB; t += EPI_THREADS) nsplit += feat[(size_t)r * SB + t] != 0;
  uint32_t v4[4] = {correct, nviol, nsplit, n_sub};
  __syncthreads();  // s_red may still be read from an earlier call
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    for (uint32_t o = 32; o > 0; o >>= 1) v4[q] += __shfl_xor(v4[q], o, 64);
    if ((threadIdx.x & 63u) == 0) s_red[q][threadIdx.x >> 6] = v4[q];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int q = 0; q < 4; ++q) {
    v4[q] = 0;
    for (uint32_t w = 0; w < EPI_THREADS / 64; ++w) v4[q] += s_red[q][w];
  }
  correct = v4[0];
  nviol = v4[1];
  nsplit = v4[2];
  n_sub = v4[3];
  if (out.correct) out.correct[r] = correct;
  if (out.cost) {
    double v = (double)(n_sub - correct);
    v = __dadd_rn(v, __dmul_rn(alpha, (double)nsplit));
    v = __dadd_rn(v, (double)nviol);
    out.cost[r] = v;
  }
}

// ---------------------------------------------------------------------------
// Walk kernel (any depth): lane = sample.  A block owns a range of samples and
// a group of TG trees.  It stages its samples T at a time in LDS, every rank
// column and the labels, and walks them through its trees (Algorithm 1: t <-
// 2t if rank < tau else 2t + 1, D steps), adding to the (tree, leaf, class)
// histogram in LDS, which goes to memory once per block (global adds directly
// where it does not fit).  The block's 1,024 threads are NG = 1024 / T sets of
// T lanes; set s walks every sample through the trees s GI .. s GI + GI - 1,
// then + NG GI, ..., GI independent chains of dependent LDS reads per lane.
//
// The LDS pipe bounds it (a read that no bank conflict slows takes a CU 2.7
// cycles per wave, one of 64 random words 4.4, of 128 5.9), and next the
// vector unit.  A node is one LDS word, tau << 8 | 2 column, and a staged rank
// is rank << 8 | 2 column, so that the comparison needs no unpacking: per step
// a read of the node, a byte product for the rank's address (columns of 64
// samples are 256 bytes; from 129 features on, whose doubled column passes a
// byte, a mask and a shift), its read, a compare, a select and a shift-add
// for the child's address (node t at base + 4 (t - 1): child 2t + b at 2 addr
// - base + 4 + 4 b).  The nodes of a level are consecutive words, and lane i
// reads word i of a column whatever column its node names, so the rank reads
// never conflict.  That takes ranks and thresholds below 2^24 - 1; larger ones
// (WIDE, from that many samples on) use 64-bit nodes and plain ranks.  The
// next tile's chunks are loaded into registers while the current one is
// walked.
//
// Measured per launch, against 256-thread blocks of up to 32 64-bit-node trees
// without prefetch: depth 8, n = 10^5, F = 16, P = 100: 40.9 -> 37.2 us;
// depth 6, n = 2 10^5, F = 100, P = 64 (ranks read from memory at every step
// before): 810 -> 55 us.  A call for four depth-2 trees on three quarters of
// n = 2 10^5, F = 120: 52 us with every column staged, 43 with SEL.
// ---------------------------------------------------------------------------
constexpr uint32_t WT_THREADS = 1024;
constexpr uint32_t WT_NPF = 8;  // 16-byte chunks of the next tile per thread
constexpr uint32_t WT_RANK_MAX = 0xFFFFFFu;

struct WalkArgs {
  const uint32_t *ranks;
  uint32_t ld;
  const uint8_t *labels;
  const uint32_t *idx;     // the samples (null: 0 .. n_sub - 1)
  const uint32_t *weight;  // times each sample counts (null: once)
  const uint32_t *n_unique;
  uint32_t n_sub, n;
  const uint8_t *feat;
  const uint32_t *tau;
  uint32_t P, D, F, K;
  uint32_t TG;      // trees per block
  uint32_t per;     // samples per block (gridDim.x ranges), in units of 64
  uint32_t hist_in_lds;
  uint32_t vec4;  // rank columns readable as 16-byte chunks (aligned, ld % 4 == 0)
  uint32_t *leafcnt;  // [P][2^D][K]
};

// The sample at position j of the evaluation: its index, class (0xFF: left
// out) and weight.
__device__ __forceinline__ uint32_t walk_label(const WalkArgs &a, uint32_t j, uint32_t &i,
                                               uint32_t &w) {
  i = a.idx ? a.idx[j] : j;
  w = 1;
  if (i >= a.n) return 0xFFu;
  if (a.weight) w = a.weight[i];
  const uint32_t y = a.labels[i];
  return y < a.K && w ? y : 0xFFu;
}

// The block's share straight from memory: for a data set whose ranks do not
// fit the packed words although its sample count promised it (columns cut out
// of a larger encoding).
__device__ __forceinline__ void walk_plain(const WalkArgs &a, uint32_t r0, uint32_t tg, uint32_t s0,
                                        uint32_t s1) {
  const uint32_t SB = (1u << a.D) - 1u, SL = 1u << a.D;
  for (uint64_t j = (uint64_t)s0 + threadIdx.x; j < s1; j += WT_THREADS) {
    uint32_t i, w;
    const uint32_t y = walk_label(a, (uint32_t)j, i, w);
    if (y == 0xFFu) continue;
    for (uint32_t g = 0; g < tg; ++g) {
      const size_t tr = (size_t)(r0 + g) * SB;
      uint32_t t = 1;
      for (uint32_t d = 0; d < a.D; ++d) {
        const uint32_t f = a.feat[tr + t - 1];
        const bool left = f != 0 && f <= a.F && a.ranks[(size_t)(f - 1) * a.ld + i] < a.tau[tr + t - 1];
        t = left ? 2 * t : 2 * t + 1;
      }
      atomicAdd(&a.leafcnt[((size_t)(r0 + g) * SL + (t - SL)) * a.K + y], w);
    }
  }
}

// SEL: only the columns that the block's trees split on are staged (few trees
// of a wide data set), numbered by their order.
template <uint32_t T, int GI, bool WIDE, bool SEL>
__global__ __launch_bounds__(WT_THREADS) void k_walk_tiles(WalkArgs a) {
  extern __shared__ __align__(16) uint32_t wl[];
  constexpr uint32_t NG = WT_THREADS / T, NW = WIDE ? 8u : 4u;  // bytes of a node
  // the column is held shifted left by FS
  constexpr uint32_t FS = T > 128 ? 1 : 0;
  __shared__ uint8_t s_num[256], s_col[256];  // SEL: column to number and back
  __shared__ uint32_t s_cols;
  const uint32_t SB = (1u << a.D) - 1u, SL = 1u << a.D, K = a.K;
  const uint32_t r0 = blockIdx.y * a.TG;
  const uint32_t tg = min(a.TG, a.P - r0);
  uint32_t F = a.F;  // columns staged
  if constexpr (SEL) {
    if (threadIdx.x < 256) s_num[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < tg * SB; e += WT_THREADS) {
      const uint32_t f = a.feat[(size_t)r0 * SB + e];
      if (f != 0 && f <= a.F) s_num[f - 1u] = 1;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
      uint32_t run = 0;
      for (uint32_t f = threadIdx.x; f < 256; f += 64) {
        const bool on = s_num[f] != 0;
        const uint64_t all = __ballot(on);
        const uint32_t at = run + (uint32_t)__popcll(all & ((1ull << threadIdx.x) - 1ull));
        if (on) {
          s_col[at] = (uint8_t)f;
          s_num[f] = (uint8_t)at;
        }
        run += (uint32_t)__popcll(all);
      }
      if (threadIdx.x == 0) {
        if (run == 0) s_col[0] = 0;  // no split at all: nodes name column 0
        s_cols = run ? run : 1u;
      }
    }
    __syncthreads();
    F = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cols);
  }
  auto source = [&](uint32_t f) { return SEL ? (uint32_t)s_col[f] : f; };
  uint32_t *tile = wl;                                           // [T / 64][F][64]
  uint32_t *wgt = wl + F * T;                                    // [T] weights
  uint8_t *ylab = reinterpret_cast<uint8_t *>(wgt + T);          // [T]
  uint32_t *nodes = wgt + T + T / 4;                             // [TG][SB] words of NW bytes
  uint32_t *hist = nodes + ((a.TG * SB * (NW / 4) + 1u) & ~1u);  // [TG][SL][K]
  // absolute LDS byte addresses
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint32_t *)wl);
  const uint32_t node0 = lds0 + 4u * (F * T + T + T / 4);
  const uint32_t hist0 = lds0 + 4u * (uint32_t)(hist - wl);
  // the block's sample range (a multiple of 64, so that every tile starts at
  // a multiple of 4 samples for the 16-byte loads)
  const uint64_t per = 64ull * a.per;  // (64-bit: no wrap for counts near 2^32)
  const uint32_t s0 = (uint32_t)min((uint64_t)a.n_sub, blockIdx.x * per);
  const uint32_t s1 = (uint32_t)min((uint64_t)a.n_sub, s0 + per);
  if (!WIDE) {
    // (every wave finds the same, so the block leaves together)
    bool big = false;
    for (uint32_t f = threadIdx.x & 63u; f < a.F; f += 64) big |= a.n_unique[f] >= WT_RANK_MAX;
    if (__ballot(big) != 0ull) {
      walk_plain(a, r0, tg, s0, s1);
      return;
    }
  }
  const uint32_t i = threadIdx.x & (T - 1u);
  const uint32_t set = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / T));
  // the sample's rank in column 0; column f is 256 f bytes on
  const uint32_t lane_off = lds0 + 4u * (i % 64u) + 256u * F * (i / 64u);
  constexpr uint32_t T4 = T / 4;
  const uint32_t nch = F * T4;
  uint4 pf[WT_NPF];
  const bool chunked = !a.idx && a.vec4;  // (from four samples on)
  // the thread's number, opaque: what follows from it is worked out in place
  // rather than kept in registers across the walk
  auto thread = [] {
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  };
  // Loads without a branch (a skipped one would make each of the next wait
  // for those before it): columns and samples past the end come as the last
  // whole chunk, and the last samples of a ragged column when it is stored.
  const uint32_t j_last = (a.n - 4u) & ~3u;
  auto prefetch = [&](uint32_t base) {
    const uint32_t tid = thread();
#pragma unroll
    for (uint32_t k = 0; k < WT_NPF; ++k) {
      if (k * WT_THREADS >= nch) break;
      const uint32_t c = min(k * WT_THREADS + tid, nch - 1u), j = min(base + 4u * (c % T4), j_last);
      pf[k] = *reinterpret_cast<const uint4 *>(a.ranks + (size_t)source(c / T4) * a.ld + j);
    }
  };
  auto word = [&](uint32_t rank, uint32_t f) {
    return WIDE ? rank : (min(rank, WT_RANK_MAX) << 8) | (f << FS);
  };
  if (chunked) prefetch(s0);
  // this block's trees: nodes into LDS, histogram cleared
  for (uint32_t e = threadIdx.x; e < tg * SB; e += WT_THREADS) {
    const uint32_t f = a.feat[(size_t)r0 * SB + e], t = a.tau[(size_t)r0 * SB + e];
    const bool split = f != 0 && f <= a.F;
    const uint32_t th = split ? t : 0u, col = split ? (SEL ? s_num[f - 1u] : f - 1u) : 0u;
    if constexpr (WIDE)
      reinterpret_cast<uint64_t *>(nodes)[e] = ((uint64_t)th << 32) | (col << 8);
    else
      nodes[e] = (min(th, WT_RANK_MAX) << 8) | (col << FS);
  }
  if (a.hist_in_lds)
    for (uint32_t e = threadIdx.x; e < tg * SL * K; e += WT_THREADS) hist[e] = 0;
  for (uint32_t base = s0, next; base < s1; base = next) {
    const uint32_t cnt = min(T, s1 - base);
    next = base + cnt;
    __syncthreads();  // the previous tile (and the node set-up) is done
    if (threadIdx.x < T) {
      // a sample that is left out counts 0 times, in class 0
      uint32_t y = 0xFFu, w = 0, smp;
      if (threadIdx.x < cnt) y = walk_label(a, base + threadIdx.x, smp, w);
      ylab[threadIdx.x] = y == 0xFFu ? (uint8_t)0 : (uint8_t)y;
      wgt[threadIdx.x] = y == 0xFFu ? 0u : w;
    }
    const uint32_t tid = thread();
    if (chunked) {
      uint4 *tile4 = reinterpret_cast<uint4 *>(tile);
#pragma unroll
      for (uint32_t k = 0; k < WT_NPF; ++k) {
        const uint32_t c = k * WT_THREADS + tid, f = c / T4, q = c % T4;
        if (c >= nch) continue;
        if (const uint32_t j = base + 4u * q; j < s1 && j > j_last) {
          const uint32_t *p = a.ranks + (size_t)source(f) * a.ld + j;
          pf[k] = make_uint4(p[0], j + 1u < s1 ? p[1] : 0u, j + 2u < s1 ? p[2] : 0u, 0u);
        }
        tile4[((q / 16u) * F + f) * 16u + q % 16u] =
            make_uint4(word(pf[k].x, f), word(pf[k].y, f), word(pf[k].z, f), word(pf[k].w, f));
      }
    } else {
      // SG loads in flight per thread before their stores
      constexpr uint32_t SG = 8;
      for (uint32_t e0 = tid; e0 < F * T; e0 += SG * WT_THREADS) {
        uint32_t v[SG];
#pragma unroll
        for (uint32_t u = 0; u < SG; ++u) {
          const uint32_t e = e0 + u * WT_THREADS, f = e / T, q = e % T;
          v[u] = 0;
          if (e < F * T && q < cnt) {
            const uint32_t smp = a.idx ? a.idx[base + q] : base + q;
            if (smp < a.n) v[u] = a.ranks[(size_t)source(f) * a.ld + smp];
          }
        }
#pragma unroll
        for (uint32_t u = 0; u < SG; ++u) {
          const uint32_t e = e0 + u * WT_THREADS, f = e / T, q = e % T;
          if (e < F * T) tile[((q / 64u) * F + f) * 64u + q % 64u] = word(v[u], f);
        }
      }
    }
    __syncthreads();
    if (chunked && next < s1) prefetch(next);
    const uint32_t y = ylab[i], w = wgt[i];
    if (__ballot(w != 0u) == 0ull) continue;  // (uniform over the wave; no barrier inside)
    const uint32_t y4 = hist0 + 4u * y;
    // GI trees at a time; a batch past the last tree repeats the last one and
    // leaves its count out
    for (uint32_t g0 = set * GI; g0 < tg; g0 += NG * GI) {
      uint32_t na[GI], cl[GI], cr[GI];
#pragma unroll
      for (int gg = 0; gg < GI; ++gg) {
        na[gg] = node0 + NW * SB * min(g0 + gg, tg - 1);
        // child of address x: 2 x + cl or cr
        cl[gg] = NW - na[gg];
        cr[gg] = 2u * NW - na[gg];
        // (in vector registers: a select takes one scalar operand at most)
        asm volatile("" : "+v"(cl[gg]), "+v"(cr[gg]));
      }
      for (uint32_t lv = 0; lv < a.D; ++lv) {
        if constexpr (WIDE) {
#pragma unroll
          for (int gg = 0; gg < GI; ++gg) {
            const uint64_t x = lds_rd64(na[gg]);
            const uint32_t rk = lds_rd32((uint32_t)x + lane_off);
            na[gg] = 2u * na[gg] + (rk < (uint32_t)(x >> 32) ? cl[gg] : cr[gg]);
          }
        } else {
          uint32_t x[GI], rk[GI];
#pragma unroll
          for (int gg = 0; gg < GI; ++gg) x[gg] = lds_rd32(na[gg]);
#pragma unroll
          for (int gg = 0; gg < GI; ++gg) {
            // the word's low byte times 128 or 256, plus the lane's offset
            const uint32_t at = FS ? __builtin_amdgcn_udot4(x[gg], 128u, lane_off, false)
                                   : ((x[gg] & 0xFFu) << 8) + lane_off;
            rk[gg] = lds_rd32(at);
          }
#pragma unroll
          for (int gg = 0; gg < GI; ++gg)
            na[gg] = 2u * na[gg] + (rk[gg] < x[gg] ? cl[gg] : cr[gg]);
        }
      }
#pragma unroll
      for (int gg = 0; gg < GI; ++gg) {
        const uint32_t g = g0 + gg;
        if (g >= tg) continue;
        // the leaf's word of class 0, in bytes from the tree's histogram
        const uint32_t leaf0 = node0 + NW * SB * g + NW * (SL - 1u);
        if (a.hist_in_lds) {
          // (both factors below 2^24)
          const uint32_t at = __umul24(na[gg] - leaf0, K) / (NW / 4u) + 4u * g * SL * K + y4;
          __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t *)at, w,
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else if (w) {
          atomicAdd(&a.leafcnt[((size_t)(r0 + g) * SL + (na[gg] - leaf0) / NW) * K + y], w);
        }
      }
    }
  }
  if (a.hist_in_lds) {
    __syncthreads();
    // two counters at a time (each stays below 2^32, so no carry passes from
    // one to the other).  The ranges start at different words, so that the
    // blocks of a group, which end together, do not add to the same ones at
    // the same time.
    const uint32_t pairs = tg * (SL / 2) * K, rot = (uint64_t)pairs * blockIdx.x / gridDim.x;
    const uint64_t *hist2 = reinterpret_cast<const uint64_t *>(hist);
    unsigned long long *out =
        reinterpret_cast<unsigned long long *>(a.leafcnt + (size_t)r0 * SL * K);
#pragma unroll 4
    for (uint32_t e = threadIdx.x; e < pairs; e += WT_THREADS) {
      const uint32_t at = e + rot < pairs ? e + rot : e + rot - pairs;
      const uint64_t v = hist2[at];
      if (v) atomicAdd(&out[at], (unsigned long long)v);
    }
  }
}

// The walk with every rank read from memory where its node asks for it: a lane
// per sample, the block's trees in LDS as 64-bit nodes (tau, column), GI
// independent chains per lane.  The memory system bounds it (a wave's read of 64
// ranks is up to 64 lines), but it reads D ranks per tree where k_walk_tiles
// stages F columns for every group of trees, and the columns leave it room for
// few trees.  Measured per launch, there and here: n = 1.55 10^5, a sorted quarter
// of it, F = 120, K = 20, depth 7, P = 178 500 and 105 us; 2,700 samples of 1.35
// 10^5, F = 145, K = 5, depth 6, P = 5 33 and 12 us.
constexpr uint32_t WD_THREADS = 256;

template <int GI>
__global__ __launch_bounds__(WD_THREADS) void k_walk_direct(WalkArgs a) {
  extern __shared__ __align__(16) uint32_t wl[];
  const uint32_t SB = (1u << a.D) - 1u, SL = 1u << a.D, K = a.K;
  const uint32_t r0 = blockIdx.y * a.TG, tg = min(a.TG, a.P - r0);
  uint64_t *nodes = reinterpret_cast<uint64_t *>(wl);                     // [TG][SB]
  uint32_t *hist = reinterpret_cast<uint32_t *>(nodes + (size_t)a.TG * SB);  // [TG][SL][K]
  const uint32_t node0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint32_t *)wl);
  for (uint32_t e = threadIdx.x; e < tg * SB; e += WD_THREADS) {
    const uint32_t f = a.feat[(size_t)r0 * SB + e], t = a.tau[(size_t)r0 * SB + e];
    const bool split = f != 0 && f <= a.F;
    nodes[e] = split ? ((uint64_t)t << 32) | (f - 1u) : 0ull;
  }
  if (a.hist_in_lds)
    for (uint32_t e = threadIdx.x; e < tg * SL * K; e += WD_THREADS) hist[e] = 0;
  __syncthreads();
  const uint64_t per = 64ull * a.per;  // (64-bit: no wrap for counts near 2^32)
  const uint32_t s0 = (uint32_t)min((uint64_t)a.n_sub, blockIdx.x * per);
  const uint32_t s1 = (uint32_t)min((uint64_t)a.n_sub, s0 + per);
  for (uint32_t base = s0, next; base < s1; base = next) {
    const uint32_t cnt = min(WD_THREADS, s1 - base);
    next = base + cnt;
    uint32_t smp, w, y = 0xFFu;
    if (threadIdx.x < cnt) y = walk_label(a, base + threadIdx.x, smp, w);
    if (y == 0xFFu) continue;
    const uint32_t *rank = a.ranks + smp;
    for (uint32_t g0 = 0; g0 < tg; g0 += GI) {
      uint32_t nb[GI], na[GI];
#pragma unroll
      for (int gg = 0; gg < GI; ++gg) na[gg] = nb[gg] = node0 + 8u * SB * min(g0 + gg, tg - 1);
      for (uint32_t lv = 0; lv < a.D; ++lv) {
        uint64_t x[GI];
        uint32_t rk[GI];
#pragma unroll
        for (int gg = 0; gg < GI; ++gg) x[gg] = lds_rd64(na[gg]);
#pragma unroll
        for (int gg = 0; gg < GI; ++gg) rk[gg] = rank[(size_t)(uint32_t)x[gg] * a.ld];
#pragma unroll
        for (int gg = 0; gg < GI; ++gg)
          na[gg] = 2u * na[gg] - nb[gg] + (rk[gg] < (uint32_t)(x[gg] >> 32) ? 8u : 16u);
      }
#pragma unroll
      for (int gg = 0; gg < GI; ++gg) {
        if (g0 + gg >= tg) continue;
        const uint32_t leaf = (na[gg] - nb[gg]) / 8u + 1u - SL;
        if (a.hist_in_lds)
          atomicAdd(&hist[((g0 + gg) * SL + leaf) * K + y], w);
        else
          atomicAdd(&a.leafcnt[((size_t)(r0 + g0 + gg) * SL + leaf) * K + y], w);
      }
    }
  }
  if (!a.hist_in_lds) return;
  __syncthreads();
  for (uint32_t e = threadIdx.x; e < tg * SL * K; e += WD_THREADS)
    if (hist[e]) atomicAdd(&a.leafcnt[(size_t)r0 * SL * K + e], hist[e]);
}

// How often each sample is named by idx (entries past n are invalid input).
// (A launch takes fewer than 2^32 threads, a subset as many entries.)
__global__ __launch_bounds__(256) void k_walk_weight(const uint32_t *__restrict__ idx,
                                                     uint32_t n_sub, uint32_t n,
                                                     uint32_t *__restrict__ weight) {
  for (uint64_t j = blockIdx.x * 256ull + threadIdx.x; j < n_sub; j += gridDim.x * 256ull)
    if (idx[j] < n) atomicAdd(&weight[idx[j]], 1u);
}

// Epilogue from leaf counts (walk path), any depth.  Block per tree: the
// threads share out the leaves (and the nodes for the split count) and the
// integer sums meet in a block reduction, so the result does not depend on
// the order.
__global__ __launch_bounds__(EPI_THREADS) void k_epilogue_leaves(
    uint32_t *__restrict__ leafcnt, const uint8_t *__restrict__ feat, uint32_t P, uint32_t D,
    uint32_t K, uint32_t n_min, double alpha, FitnessOut out) {
  __shared__ uint32_t s_red[4][EPI_THREADS / 64];
  if (blockIdx.x >= P) return;
  leaf_epilogue_tree(leafcnt, feat, blockIdx.x, D, K, n_min, alpha, out, s_red);
}

// Launches on st; when e0/e1 are given the launch records them at the
// kernel's start and end.
template <int D, int WAVES>
hipError_t launch_bits(const TileHdr *hdr, uint32_t F, uint32_t gx, uint32_t gy,
                       const uint8_t *feat, const uint32_t *tau, uint32_t P, uint32_t *cnt,
                       const FuseArgs *fa, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  size_t lds = (size_t)mask_region(F) + (size_t)F * MCOL;
  if (fa) {
    const size_t need = WAVES * 64 * 12 + 1024 +
                        (fa->rows_in_lds ? (size_t)P * 2 * ((1u << D) - 1u) * 8 : 0);
    lds = lds > need ? lds : need;
    hipExtLaunchKernelGGL((k_fitness_bits<D, WAVES, true>), dim3(gx, gy), dim3(WAVES * 64), lds,
                          st, e0, e1, 0, hdr, feat, tau, P, cnt, *fa);
  } else {
    hipExtLaunchKernelGGL((k_fitness_bits<D, WAVES, false>), dim3(gx, gy), dim3(WAVES * 64), lds,
                          st, e0, e1, 0, hdr, feat, tau, P, cnt, FuseArgs{});
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_bits_w(uint32_t waves, const TileHdr *hdr, uint32_t F, uint32_t gx, uint32_t gy,
                         const uint8_t *feat, const uint32_t *tau, uint32_t P, uint32_t *cnt,
                         const FuseArgs *fa, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (waves == 1) return launch_bits<D, 1>(hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1);
  if (waves == 2) return launch_bits<D, 2>(hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1);
  if (waves == 4) return launch_bits<D, 4>(hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1);
  return launch_bits<D, 8>(hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1);
}

template <int D>
void launch_epi(uint32_t *cnt, const uint32_t *ctot, const uint8_t *feat, uint32_t P, uint32_t K,
                uint32_t n_problems, uint32_t n_min, double alpha, const FitnessOut &out,
                hipStream_t st) {
  uint32_t n = n_problems * P;
  k_epilogue_nodes<D><<<(n + 127) / 128, 128, 0, st>>>(cnt, ctot, feat, P, K, n_problems, n_min,
                                                       alpha, out);
}

}  // namespace

// Block threads of the fitness kernel for population P, and the power of two
// (>= P, >= 64) the fused DE step needs.
uint32_t fitness_block_threads(uint32_t P) {
  uint32_t waves = pad64(P) / 64;
  waves = waves > 4 ? 8 : (waves > 2 ? 4 : waves);
  return waves * 64;
}
uint32_t fused_threads(uint32_t P) {
  uint32_t t = 64;
  while (t < P) t <<= 1;
  return t;
}

mh_status launch_fitness_count(Ctx *ctx, const void *tiles, uint32_t F, uint32_t K,
                               uint32_t n_sub, uint32_t n_problems, uint32_t max_tiles,
                               const uint8_t *feat, const uint32_t *tau, uint32_t P, uint32_t D,
                               uint32_t *cnt, const FuseArgs *fa) {
  if (D < 1 || D > 5) return fail(ctx, MH_EINVAL, "tile fitness kernel supports depth 1..5");
  const TileHdr *hdr = reinterpret_cast<const TileHdr *>(tiles);
  hipStream_t st = ctx->stream;
  const uint32_t Ppad = pad64(P);
  // one block covers up to 8 waves of 64 trees, so a tile is staged once for
  // populations up to 512
  uint32_t waves = Ppad / 64;
  waves = waves > 4 ? 8 : (waves > 2 ? 4 : waves);
  const uint32_t gy = (Ppad + waves * 64 - 1) / (waves * 64);
  // blocks: about blocks_per_cu per CU over all tree groups, each with at
  // least min_tiles tiles
  uint32_t want = (uint32_t)ctx->num_cu * ctx->fit_blocks_per_cu;
  want = (want + gy - 1) / gy;
  const uint32_t cap = (max_tiles + ctx->fit_min_tiles - 1) / ctx->fit_min_tiles;
  uint32_t gx = want < cap ? want : cap;
  if (gx == 0) gx = 1;
  if (fa && (gy != 1 || fused_threads(P) > waves * 64))
    return fail(ctx, MH_EINVAL, "fused fitness + DE needs one block per tile to hold every tree");
  hipEvent_t e0, e1;
  const bool timed = prof_pair(ctx, &e0, &e1);
  hipError_t e = hipSuccess;
  switch (D) {
    case 1: e = launch_bits_w<1>(waves, hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1); break;
    case 2: e = launch_bits_w<2>(waves, hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1); break;
    case 3: e = launch_bits_w<3>(waves, hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1); break;
    case 4: e = launch_bits_w<4>(waves, hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1); break;
    case 5: e = launch_bits_w<5>(waves, hdr, F, gx, gy, feat, tau, P, cnt, fa, st, e0, e1); break;
  }
  if (e != hipSuccess) return hip_fail(ctx, e, "k_fitness_bits");
  if (timed) ctx->prof_launches += 1;
  ctx->prof_evals += (uint64_t)n_sub * P;
  ctx->prof_tiles += max_tiles;
  (void)K;
  (void)n_problems;
  return MH_OK;
}

mh_status launch_fitness_jobs(Ctx *ctx, uint32_t D, uint32_t waves, uint32_t F_max,
                              const FitJob *jobs, const uint16_t *job_of, uint32_t n_blocks) {
  if (n_blocks == 0) return MH_OK;
  const size_t lds = (size_t)mask_region(F_max) + (size_t)F_max * MCOL;
  hipStream_t st = ctx->stream;
  const dim3 grid(n_blocks), block(waves * 64);
#define MH_JOBS_W(DD)                                                                       \
  switch (waves) {                                                                          \
    case 1: k_fitness_jobs<DD, 1><<<grid, block, lds, st>>>(jobs, job_of); break;           \
    case 2: k_fitness_jobs<DD, 2><<<grid, block, lds, st>>>(jobs, job_of); break;           \
    case 4: k_fitness_jobs<DD, 4><<<grid, block, lds, st>>>(jobs, job_of); break;           \
    case 8: k_fitness_jobs<DD, 8><<<grid, block, lds, st>>>(jobs, job_of); break;           \
    default: return fail(ctx, MH_EINVAL, "fitness jobs: waves must be 1, 2, 4 or 8");      \
  }
  switch (D) {
    case 1: MH_JOBS_W(1) break;
    case 2: MH_JOBS_W(2) break;
    case 3: MH_JOBS_W(3) break;
    case 4: MH_JOBS_W(4) break;
    case 5: MH_JOBS_W(5) break;
    default: return fail(ctx, MH_EINVAL, "fitness jobs support depth 1..5");
  }
#undef MH_JOBS_W
  MH_LAUNCHED(ctx, "k_fitness_jobs");
  return MH_OK;
}

mh_status launch_fitness_epilogue(Ctx *ctx, const void *tiles, uint32_t F, uint32_t K,
                                  uint32_t n_sub, uint32_t n_problems, const uint8_t *feat,
                                  uint32_t P, uint32_t D, uint32_t n_min, double alpha,
                                  uint32_t *cnt, const FitnessOut &out) {
  const uint8_t *b = reinterpret_cast<const uint8_t *>(tiles);
  const TileHdr h = tile_layout(n_sub, F, K, n_problems);
  const uint32_t *ctot = reinterpret_cast<const uint32_t *>(b + h.off_ctot);
  hipStream_t st = ctx->stream;
  switch (D) {
    case 1: launch_epi<1>(cnt, ctot, feat, P, K, n_problems, n_min, alpha, out, st); break;
    case 2: launch_epi<2>(cnt, ctot, feat, P, K, n_problems, n_min, alpha, out, st); break;
    case 3: launch_epi<3>(cnt, ctot, feat, P, K, n_problems, n_min, alpha, out, st); break;
    case 4: launch_epi<4>(cnt, ctot, feat, P, K, n_problems, n_min, alpha, out, st); break;
    case 5: launch_epi<5>(cnt, ctot, feat, P, K, n_problems, n_min, alpha, out, st); break;
    default: return fail(ctx, MH_EINVAL, "tile epilogue supports depth 1..5");
  }
  MH_LAUNCHED(ctx, "k_epilogue_nodes");
  return MH_OK;
}

mh_status launch_fitness_tiles(Ctx *ctx, const void *tiles, uint32_t F, uint32_t K, uint32_t n_sub,
                               uint32_t n_problems, uint32_t max_tiles, const uint8_t *feat,
                               const uint32_t *tau, uint32_t P, uint32_t D, uint32_t n_min,
                               double alpha, uint32_t *cnt, const FitnessOut &out) {
  mh_status s = launch_fitness_count(ctx, tiles, F, K, n_sub, n_problems, max_tiles, feat, tau, P,
                                     D, cnt, nullptr);
  if (s) return s;
  return launch_fitness_epilogue(ctx, tiles, F, K, n_sub, n_problems, feat, P, D, n_min, alpha,
                                 cnt, out);
}

// How a walk over n_sub samples shares out its trees and samples over the
// blocks, and the cycles its fullest CU is expected to take.
struct WalkPlan {
  double cycles = 1e300;
  bool direct = false, sel = false, wide = false, hist_in_lds = false;
  uint32_t T = 0;  // samples per tile, or the trees a lane walks at once (direct)
  uint32_t TG = 0, per = 0, ranges = 0, groups = 0;
  size_t lds = 0;
};

// The 128-byte lines that 64 samples of one column lie on: two when they follow
// each other; of a subset, whose order is not known here, between the sorted
// case (2 n / n_sub) and the random one (64).
static double walk_lines(const mh_dataset *ds, uint32_t n_sub, bool gather) {
  return gather ? std::min(64.0, 8.0 * ds->n / n_sub) : 2.0;
}

// k_walk_tiles.  LDS, one block per CU: a tile of T samples with its labels and
// weights, TG trees' nodes and, when it fits, their histograms.  The largest
// tile that leaves the trees at least 60 KiB: its waves then share nothing but
// the trees, and a tile's barriers are paid for by more walks.
// Groups of trees times ranges of samples, at most one block per CU: the choice
// with the least work for a block, counted in CU cycles (measured): 8.4 per 64
// samples, tree (in batches of four) and level, 12 per 64 samples and column
// staged, 2,000 per tile for its barriers and the chains' latency, and 1.5 per
// histogram word cleared and added to memory.  With a multiple of 8 ranges every
// block of one range is on the same XCD (blocks go round-robin over the 8 XCDs in
// launch order), whose L2 then serves the range's ranks to all groups but one;
// that saves 4 per column.  Through an index 64 ranks of a column cost a block
// about 50 cycles and 1.2 per line, and the chip 30 and 4.2 per line (a CU's
// share of the memory bandwidth).
static WalkPlan plan_tiles(const Ctx *ctx, const mh_dataset *ds, uint32_t n_sub, bool gather,
                           uint32_t P, uint32_t D) {
  const uint32_t SB = (1u << D) - 1u, SL = 1u << D, K = ds->K, F = ds->F;
  WalkPlan w;
  w.wide = ds->n >= WT_RANK_MAX;
  // few trees on a wide data set stage only the columns they split on, at most
  // one per node (Fs: the columns a block stages, at most)
  w.sel = (uint64_t)P * SB <= F && !w.wide;
  const uint32_t Fs = w.sel ? P * SB : F;
  const uint32_t T = Fs <= 24 ? 1024u : Fs <= 48 ? 512u : Fs <= 128 ? 256u : 128u;
  const uint32_t NG = WT_THREADS / T;
  const size_t budget = ctx->max_lds - 4096;
  const size_t tile_bytes = (size_t)Fs * T * 4 + T * 4 + T;
  const size_t tree_nodes = (size_t)SB * (w.wide ? 8 : 4), tree_hist = (size_t)SL * K * 4;
  if (tile_bytes + tree_nodes + 16 > budget) return w;
  w.T = T;
  w.hist_in_lds = true;
  size_t TG = (budget - tile_bytes - 16) / (tree_nodes + tree_hist);
  if (TG == 0) {
    // histograms in memory: the nodes alone decide the trees per block
    w.hist_in_lds = false;
    TG = (budget - tile_bytes - 16) / tree_nodes;
  }
  const uint32_t cus = (uint32_t)ctx->num_cu, units = (uint32_t)(((uint64_t)n_sub + 63) / 64);
  const uint32_t g_min = (uint32_t)((P + TG - 1) / TG);
  uint32_t best_units = 0;
  for (uint32_t g = g_min; g <= std::max(g_min, std::min(P, cus)); ++g) {
    const uint32_t tg = (P + g - 1) / g;
    if (g > g_min && tg == (P + g - 2) / (g - 1)) continue;
    const uint32_t rg = std::max(1u, std::min(units, cus / g));
    const uint32_t chains = tg > 2 * NG ? (tg + 3) / 4 * 4 : tg;
    for (uint32_t r = rg;; r &= ~7u) {
      const uint32_t per = (units + r - 1) / r;
      const uint32_t rounds = (g * r + cus - 1) / cus;  // (more groups than CUs)
      const double unit = 8.4 * chains * D + (r % 8 ? 12.0 : 8.0) * Fs + 2000.0 * 64 / T;
      const double c = rounds * (per * unit + 1.5 * tg * SL * K);
      if (c < w.cycles) {
        w.cycles = c;
        w.groups = g;
        w.ranges = r;
        best_units = rounds * per;
      }
      if (r < 8 || r % 8 == 0) break;
    }
  }
  w.cycles += 6000.0;  // (launch and set-up, against k_walk_direct's)
  if (gather) {
    const double lines = walk_lines(ds, n_sub, true);
    w.cycles +=
        Fs * (best_units * (40.0 + 1.2 * lines) + (double)units / cus * (30.0 + 4.2 * lines));
  }
  w.TG = (P + w.groups - 1) / w.groups;
  w.groups = (P + w.TG - 1) / w.TG;
  w.per = (units + w.ranges - 1) / w.ranges;
  w.ranges = (units + w.per - 1) / w.per;
  w.lds = tile_bytes + ((w.TG * tree_nodes + 7) & ~(size_t)7) +
          (w.hist_in_lds ? w.TG * tree_hist : 0);
  return w;
}

// k_walk_direct: about three blocks per CU, at most 32 trees each.  Its cycles,
// fitted to measured launches (n = 3,000 to 2.5 10^6, F = 2 to 240, P = 1 to 512,
// depth 1 to 10, all samples and subsets): 12 per wave, tree and level, 0.8 per
// line that these touch and 5 per line that a block's trees touch first, 700 for
// a block's dependent reads, 1.3 per histogram word, 2,400 per wave and tree for
// counts in memory.
static WalkPlan plan_direct(const Ctx *ctx, const mh_dataset *ds, uint32_t n_sub, bool gather,
                            uint32_t P, uint32_t D) {
  const uint32_t SB = (1u << D) - 1u, SL = 1u << D, K = ds->K, F = ds->F;
  WalkPlan w;
  w.direct = true;
  const size_t budget = std::max<size_t>(48 * 1024, (ctx->max_lds - 4096) / 3);
  const size_t tree_nodes = (size_t)SB * 8, tree_hist = (size_t)SL * K * 4;
  size_t TG = budget / (tree_nodes + tree_hist);
  w.hist_in_lds = TG > 0;
  if (!TG) TG = budget / tree_nodes;
  TG = std::min<size_t>({TG, 32, P});
  const uint32_t GI = TG >= 8 ? 8u : 4u;
  if (TG > GI) TG -= TG % GI;
  w.T = GI;
  w.TG = (uint32_t)TG;
  w.groups = (P + w.TG - 1) / w.TG;
  if (w.groups > 65535) return w;  // (a grid's second dimension)
  w.lds = TG * (tree_nodes + (w.hist_in_lds ? tree_hist : 0));
  const uint32_t cus = (uint32_t)ctx->num_cu;
  const uint32_t per_cu = std::max<uint32_t>(
      1u, std::min<uint32_t>(8u, (uint32_t)(ctx->max_lds / std::max<size_t>(w.lds, 1))));
  const uint32_t tiles = (uint32_t)(((uint64_t)n_sub + WD_THREADS - 1) / WD_THREADS);
  w.ranges = std::max(1u, std::min(tiles, per_cu * cus / w.groups));
  if (w.ranges >= 8) w.ranges &= ~7u;
  const uint32_t rows = (tiles + w.ranges - 1) / w.ranges;  // of 256 samples, per block
  w.per = rows * (WD_THREADS / 64);
  w.ranges = (tiles + rows - 1) / rows;
  const double lines = walk_lines(ds, n_sub, gather), units = ((double)n_sub + 63) / 64;
  double touched = 0, cols = 0;  // of one tree, per 64 samples
  for (uint32_t lv = 0; lv < D; ++lv) {
    touched += std::min(64.0, (double)(1u << lv) * lines);
    cols += std::min(64u, 1u << lv);
  }
  const double first = std::min(std::min<double>(F, w.TG * cols) * lines, w.TG * touched);
  const double blocks = (double)w.groups * w.ranges;
  w.cycles = units / cus * (P * (12.0 * D + 0.8 * touched) + 5.0 * w.groups * first) +
             700.0 * rows * ((w.TG + GI - 1) / GI) * D * std::max(1.0, blocks / (per_cu * cus)) +
             (w.hist_in_lds ? 1.3 * w.TG * SL * K * std::max(1.0, blocks / cus)
                            : 2400.0 * units * P / cus);
  return w;
}

// The faster form as expected; k_walk_direct for rows wider than 48 columns
// (narrower ones leave a tile's columns room for many trees).
static WalkPlan walk_plan(const Ctx *ctx, const mh_dataset *ds, uint32_t n_sub, bool gather,
                          uint32_t P, uint32_t D) {
  const WalkPlan t = plan_tiles(ctx, ds, n_sub, gather, P, D);
  if (ds->F <= 48 && t.groups) return t;
  const WalkPlan d = plan_direct(ctx, ds, n_sub, gather, P, D);
  return d.cycles < t.cycles ? d : t;
}

// A subset can also be walked as all samples in order, each counted as often as
// the subset names it: the columns then stream in, where a gather reads a line of
// 128 bytes per rank, but the samples outside it are walked as well.  Counting
// takes two launches, 10,000 cycles, and 4.4 and 5 per 256 samples and entries.
// Measured: a random half of n = 2.7 10^5, F = 46, K = 3, depth 6, P = 196: 126 us
// so, 185 through the index; a sorted quarter of n = 1.8 10^6, F = 4, P = 169: 640
// and 160.
bool walk_weighs(const Ctx *ctx, const mh_dataset *ds, uint32_t n_sub, uint32_t P, uint32_t D,
                 uint32_t evaluations) {
  if (n_sub == 0 || ds->n == 0 || P == 0) return false;
  const double count = 10000.0 + (4.4 * ds->n + 5.0 * n_sub) / ctx->num_cu;
  return plan_tiles(ctx, ds, ds->n, false, P, D).cycles + count / evaluations <
         walk_plan(ctx, ds, n_sub, true, P, D).cycles;
}

const uint32_t *walk_weights(Ctx *ctx, const mh_dataset *ds, const uint32_t *idx, uint32_t n_sub) {
  uint32_t *w = (uint32_t *)arena_get(ctx, "walk_weight", (size_t)ds->n * 4);
  if (!w) {
    (void)hipGetLastError();  // no room for it: the subset is gathered
    return nullptr;
  }
  if (launch_zero(ctx, {{w, (size_t)ds->n * 4}})) return nullptr;
  const uint32_t blocks = (uint32_t)std::min<uint64_t>(((uint64_t)n_sub + 255) / 256, 1u << 16);
  k_walk_weight<<<blocks, 256, 0, ctx->stream>>>(idx, n_sub, ds->n, w);
  return w;
}

mh_status launch_fitness_walk(Ctx *ctx, const mh_dataset *ds, const uint32_t *idx, uint32_t n_sub,
                              const uint8_t *feat, const uint32_t *tau, uint32_t P, uint32_t D,
                              uint32_t n_min, double alpha, const FitnessOut &out,
                              uint32_t *leafcnt, const uint32_t *weight) {
  const uint32_t K = ds->K;
  // only the context's own buffer is known to stay clear between calls (a
  // caller's scratch may have held anything since)
  const size_t bytes = walk_scratch_bytes(P, D, K);
  const bool own = leafcnt == nullptr;
  if (own) leafcnt = (uint32_t *)arena_get(ctx, "walk_leafcnt", bytes);
  if (!leafcnt) return MH_ENOMEM;
  hipStream_t st = ctx->stream;
  if (!(own && ctx->walk_zero == leafcnt && ctx->walk_zero_bytes >= bytes))
    if (mh_status zs = launch_zero(ctx, {{leafcnt, bytes}})) return zs;
  if (own) ctx->walk_zero = nullptr;
  if (n_sub > 0 && P > 0 && ds->n > 0) {
    const WalkPlan w = weight ? plan_tiles(ctx, ds, ds->n, false, P, D)
                              : walk_plan(ctx, ds, n_sub, idx != nullptr, P, D);
    if (w.groups == 0)
      return fail(ctx, MH_EDEVICE, "the device's LDS is too small for the walk kernel");
    WalkArgs a;
    a.ranks = ds->ranks;
    a.ld = ds->ld;
    a.labels = ds->labels;
    a.idx = weight ? nullptr : idx;
    a.weight = weight;
    a.n_unique = ds->n_unique;
    a.n_sub = weight ? ds->n : n_sub;
    a.n = ds->n;
    a.feat = feat;
    a.tau = tau;
    a.P = P;
    a.D = D;
    a.F = ds->F;
    a.K = K;
    a.TG = w.TG;
    a.per = w.per;
    a.hist_in_lds = w.hist_in_lds ? 1u : 0u;
    a.vec4 = (ds->n >= 4 && ds->ld % 4 == 0 && ((uintptr_t)ds->ranks & 15u) == 0) ? 1u : 0u;
    a.leafcnt = leafcnt;
    const size_t lds = (w.lds + 15) & ~(size_t)15;
    if (ctx->debug)
      std::fprintf(stderr, "%s: grid %u x %u, %u trees and %u samples per block, LDS %zu bytes%s\n",
                   w.direct ? "k_walk_direct" : "k_walk_tiles", w.ranges, w.groups, w.TG,
                   64u * w.per, lds, weight ? ", weights" : "");
    hipEvent_t e0, e1;
    const bool timed = prof_pair(ctx, &e0, &e1);
    const dim3 grid(w.ranges, w.groups);
#define MH_WALK(TV, GIV, WV, SV)                                                              \
  hipExtLaunchKernelGGL((k_walk_tiles<TV, GIV, WV, SV>), grid, dim3(WT_THREADS), lds, st, e0, \
                        e1, 0, a)
#define MH_WALK_T(GIV, WV, SV)                    \
  switch (w.T) {                                  \
    case 1024: MH_WALK(1024, GIV, WV, SV); break; \
    case 512: MH_WALK(512, GIV, WV, SV); break;   \
    case 256: MH_WALK(256, GIV, WV, SV); break;   \
    default: MH_WALK(128, GIV, WV, SV); break;    \
  }
    // trees a lane walks at once
    const uint32_t NG = WT_THREADS / w.T, gi = (w.TG + NG - 1) / NG;
    if (w.direct) {
      if (w.T == 8)
        hipExtLaunchKernelGGL(k_walk_direct<8>, grid, dim3(WD_THREADS), lds, st, e0, e1, 0, a);
      else
        hipExtLaunchKernelGGL(k_walk_direct<4>, grid, dim3(WD_THREADS), lds, st, e0, e1, 0, a);
    } else if (w.wide) {
      MH_WALK_T(4, true, false);
    } else if (w.sel && gi <= 2) {
      MH_WALK_T(1, false, true);
    } else if (w.sel) {
      MH_WALK_T(4, false, true);
    } else if (gi <= 1) {
      MH_WALK_T(1, false, false);
    } else if (gi <= 2) {
      MH_WALK_T(2, false, false);
    } else {
      MH_WALK_T(4, false, false);
    }
#undef MH_WALK_T
#undef MH_WALK
    MH_LAUNCHED(ctx, w.direct ? "k_walk_direct" : "k_walk_tiles");
    if (timed) ctx->prof_launches += 1;
    ctx->prof_evals += (uint64_t)n_sub * P;
  }
  if (P > 0) {
    k_epilogue_leaves<<<P, EPI_THREADS, 0, st>>>(leafcnt, feat, P, D, K, n_min, alpha, out);
    MH_LAUNCHED(ctx, "k_epilogue_leaves");
  }
  // (the epilogue read and cleared every count of the P trees)
  if (own && P > 0) {
    ctx->walk_zero = leafcnt;
    ctx->walk_zero_bytes = bytes;
  }
  return MH_OK;
}

}  // namespace mh
