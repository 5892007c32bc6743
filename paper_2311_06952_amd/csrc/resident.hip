// resident.hip -- a whole DEOCT run (Algorithm 4) as one launch with the tiles
// resident in LDS, for problems small enough that every block keeps its share
// of the tile layout beside the DE state.
//
// As in persist.hip every block holds the whole population and repeats the DE
// arithmetic, so that the counts are the only data that cross blocks (through
// device-scope adds and a grid barrier; three rotating copies, cleared two
// generations ahead).  What differs is the split of the work.  Such a run is
// bound by the latency of its generations' serial phases, not by throughput,
// so a block has 1,024 threads (H groups of the population's lanes; thread r
// of a group belongs to individual r) and every phase is cut into H parts:
//  - counting: group h takes the (tile, part of the tree) tasks h, h + H, ..;
//    a part is a subtree below depth L with the path to it, so that a deep
//    tree's searches spread over 2^L groups.  A wave adds its left counts to
//    LDS counters by class when the class changes and at the end;
//  - the block's counters go to memory, after the barrier all counts come back
//    into LDS, one load per (node, class) and individual over all groups;
//  - costs: a group scores its share of the last-level nodes' leaf pairs;
//  - mutation, crossover and decode: group h makes the nodes h NA ...
// With one block there is no exchange at all: the LDS counters are the counts.
// The number of blocks follows the tiles (resident_shape).
//
// Against the form of two groups per block with all of a tree's nodes unrolled
// in each thread (a generation's cycles at n = 3 10^4, F = 13, K = 5, depth 5,
// P = 100: 63,000, of them 13,000 in the costs, 12,000 in the decode, 10,000
// in the mutation: one wave per SIMD runs tens of kilobytes of straight-line
// code once): 26.6 -> 16.1 us per generation there; n = 2 10^4, F = 18, K = 6,
// depth 4, P = 128: 13.5 -> 10.8; n = 1000, F = 4, depth 2, P = 32 (one block
// instead of 512): 5.0 -> 3.1.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <type_traits>
#include <vector>

#include "device_common.h"
#include "fitness_core.h"
#include "grid_sync.h"
#include "internal.h"
#include "persist.h"

namespace mh {
namespace {

constexpr uint32_t RES_THREADS = 1024;
constexpr uint32_t RES_MAX_TILES = 160;  // info words of a block's tiles

// LDS: rows f64 [2 SB][P] | thresholds u32 [SB][P] | column offsets u16 [SB][P]
// | counters u32 [SB][slots][P] (or, with split costs, the block's individuals'
// counts [own][SB][K], own = own_max) | per-individual scratch u32 [3][P] | n_unique
// [F] | class totals [K] | argmin scratch | info words | tiles.
struct ResLds {
  uint32_t thr, col, cnt, ind, nu, tot, best, info, tiles, total;
};
__host__ __device__ __forceinline__ ResLds res_lds(uint32_t SB, uint32_t P, uint32_t F, uint32_t K,
                                                   uint32_t slots, uint32_t tiles,
                                                   uint32_t own_max) {
  ResLds l;
  uint32_t o = align16u(2 * SB * P * 8);
  l.thr = o;
  o += align16u(SB * P * 4);
  l.col = o;
  o += align16u(SB * P * 2);
  l.cnt = o;
  const uint32_t c1 = SB * slots * P, c2 = own_max * SB * K;
  o += align16u((c1 > c2 ? c1 : c2) * 4);
  l.ind = o;
  o += align16u(3 * P * 4);
  l.nu = o;
  o += align16u(F * 4);
  l.tot = o;
  o += align16u(K * 4);
  l.best = o;
  o += 16 * 12;
  l.info = o;
  o += RES_MAX_TILES * 4;
  l.tiles = o;
  l.total = o + tiles * align16u(mask_region(F) + F * MCOL);
  return l;
}

// Searches and counts one tile for one part of a tree: the path nodes (depths
// 0 .. L - 1 above the part's subtree) and the subtree's nodes, all searches
// interleaved.  col/thr/acc: path nodes first, then the subtree in heap order.
template <int D, int L>
__device__ __forceinline__ void eval_part(uint32_t kmask, uint32_t off, uint32_t part,
                                          uint64_t R, const uint32_t *col, const uint32_t *thr,
                                          uint32_t *acc) {
  constexpr int DS = D - L, NS = (1 << DS) - 1, NN = L + NS;
  uint32_t a[NN];
#pragma unroll
  for (int i = 0; i < NN; ++i) a[i] = col[i] + off;
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    uint32_t v[NN];
#pragma unroll
    for (int i = 0; i < NN; ++i) v[i] = lds_rd32(a[i] + (s - 1) * 4);
#pragma unroll
    for (int i = 0; i < NN; ++i) a[i] = step_if_less(a[i], v[i], thr[i], s);
  }
  uint64_t m[NN];
#pragma unroll
  for (int i = 0; i < NN; ++i) m[i] = lds_rd64(kmask - off + 2 * a[i]);
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const uint64_t A = R & m[j];
    acc[j] += (uint32_t)__popcll(A);
    R = (part >> (L - 1 - j)) & 1u ? R & ~m[j] : A;
  }
  uint64_t S[1 << DS];
  S[1] = R;
#pragma unroll
  for (int t = 1; t <= NS; ++t) {
    const uint64_t A = S[t] & m[L + t - 1];
    acc[L + t - 1] += (uint32_t)__popcll(A);
    if (2 * t < (1 << DS)) {
      S[2 * t + 1] = S[t] & ~m[L + t - 1];
      S[2 * t] = A;
    }
  }
}

// The part's node i (0-based heap node - 1): path nodes, then the subtree.
template <int D, int L>
__device__ __forceinline__ uint32_t part_node(uint32_t part, int i) {
  if (i < L) return (1u << i) + (part >> (L - i)) - 1u;
  int s = i - L + 1, d = 0;
  while ((2 << d) <= s) ++d;
  return (((1u << L) + part) << d) + (uint32_t)(s - (1 << d)) - 1u;
}

// The arguments are read as scalars where they are used.
typedef const __attribute__((address_space(4))) RunArgs *ArgPtr;

// SPLIT: whether a run may share out its costs (xcost).
template <int D, int WAVES, bool SPLIT>
__device__ __forceinline__ void resident_body(const ArgPtr pa, uint32_t bx, uint64_t wait_ticks,
                                              uint8_t *lds) {
  constexpr int SB = (1 << D) - 1, m = 2 * SB;
  constexpr uint32_t NTH = WAVES * 64, H = RES_THREADS / NTH;
  constexpr int NA = (SB + H - 1) / H;            // nodes a group mutates
  constexpr int L = D < 4 ? 0 : (D == 5 && H >= 4 ? 2 : 1);  // 2^L divides H
  constexpr uint32_t PARTS = 1u << L;
  constexpr int NN = L + (1 << (D - L)) - 1;      // nodes of a counting task
  constexpr uint32_t LN = 1u << (D - 1);          // last-level nodes
  constexpr int XN = (int)((LN + H - 1) / H);     // of them per group
  const uint32_t P = pa->P, Ppad = pad64(P), K = pa->K, F = pa->F, slots = pa->slots;
  const uint32_t b = bx - pa->blk0, nb = pa->nblk;
  // groups are whole waves, so the group index is wave-uniform
  const uint32_t h = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / NTH));
  uint32_t r = threadIdx.x % NTH;
  const bool live = r < P;
  const int n_lo = (int)h * NA < SB ? (int)h * NA : SB;  // this group's nodes
  const int n_hi = n_lo + NA < SB ? n_lo + NA : SB;
  const bool solo = nb == 1;
  // split costs: the block scores the individuals [i0, i1) alone
  const bool split = SPLIT && pa->xcost != nullptr;
  const uint32_t own_max = split ? (P + nb - 1) / nb : 0u;
  const uint32_t i0 = (uint32_t)((uint64_t)P * b / nb);
  const uint32_t i1 = (uint32_t)((uint64_t)P * (b + 1) / nb);
  const uint32_t n_cnt = max(SB * slots * P, own_max * SB * K);  // words of the counters
  uint32_t bk = 0;  // grid barriers passed

  const uint8_t *base = reinterpret_cast<const uint8_t *>(pa->hdr);
  // the range comes from host-side counts; never past the built tiles
  const uint32_t n_tiles = pa->hdr->n_tiles;
  const uint32_t T0 = min(pa->tile0, n_tiles), T1 = min(pa->tile1, n_tiles);
  const uint32_t *__restrict__ info = reinterpret_cast<const uint32_t *>(base + pa->hdr->off_info);
  const uint8_t *__restrict__ data = base + pa->hdr->off_data;
  const uint32_t *__restrict__ ctot =
      reinterpret_cast<const uint32_t *>(base + pa->hdr->off_ctot) + (size_t)pa->sub * K;
  const uint32_t t_begin = T0 + (uint32_t)((uint64_t)(T1 - T0) * b / nb);
  const uint32_t t_end = T0 + (uint32_t)((uint64_t)(T1 - T0) * (b + 1) / nb);
  uint32_t nt = t_end - t_begin;
  if (nt > pa->tiles_max) {
    // more tiles than slots: cannot happen with the host's bound; stay inside
    // the LDS and report
    nt = pa->tiles_max;
    if (threadIdx.x == 0) __hip_atomic_store(pa->err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const ResLds lo = res_lds(SB, P, F, K, slots, pa->tiles_max, own_max);
  double *rows = reinterpret_cast<double *>(lds);
  uint32_t *x_thr = reinterpret_cast<uint32_t *>(lds + lo.thr);
  uint16_t *x_col = reinterpret_cast<uint16_t *>(lds + lo.col);  // (feature - 1) SCOL
  uint32_t *s_cnt = reinterpret_cast<uint32_t *>(lds + lo.cnt);
  uint32_t *s_cor = reinterpret_cast<uint32_t *>(lds + lo.ind);  // correct, then violations, splits
  uint32_t *s_vio = s_cor + P, *s_spl = s_vio + P;
  uint32_t *s_nu = reinterpret_cast<uint32_t *>(lds + lo.nu);
  uint32_t *s_tot = reinterpret_cast<uint32_t *>(lds + lo.tot);
  double *s_bc = reinterpret_cast<double *>(lds + lo.best);
  uint32_t *s_bi = reinterpret_cast<uint32_t *>(s_bc + 16);
  uint32_t *s_info = reinterpret_cast<uint32_t *>(lds + lo.info);
  const uint32_t mregion = mask_region(F), tile_lds = align16u(mregion + F * MCOL);
  const uint32_t s0 =
      (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint8_t *)lds) + lo.tiles;
  const uint32_t kmask = s0 + mregion - 2u * s0;

  // ---- the tiles, n_unique and the initial population
  {
    const uint32_t nchunk = 48u * F;
    const size_t rec = tile_bytes(F);
    for (uint32_t i = 0; i < nt; ++i) {
      const uint4 *__restrict__ src =
          reinterpret_cast<const uint4 *>(data + (size_t)(t_begin + i) * rec);
      for (uint32_t c = threadIdx.x; c < nchunk; c += RES_THREADS)
        stage_chunk(lds + lo.tiles + i * tile_lds, mregion, F, c, src[c]);
    }
    for (uint32_t i = threadIdx.x; i < nt; i += RES_THREADS) s_info[i] = info[t_begin + i];
    for (uint32_t k = threadIdx.x; k < K; k += RES_THREADS) s_tot[k] = ctot[k];
    for (uint32_t f = threadIdx.x; f < F; f += RES_THREADS) s_nu[f] = pa->n_unique[f];
    for (uint32_t e = threadIdx.x; e < n_cnt; e += RES_THREADS) s_cnt[e] = 0;
    for (uint32_t e = threadIdx.x; e < 3 * P; e += RES_THREADS) s_cor[e] = 0;
  }
  uint32_t n_sub = 0;
  for (uint32_t k = 0; k < K; ++k) n_sub += ctot[k];
  double gt[2 * NA];  // trial genes of the group's nodes
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int t = n_lo + j;
    gt[j] = gt[NA + j] = 0.0;
    if (t < n_hi && live) {
      gt[j] = pa->pop[(size_t)t * P + r];
      gt[NA + j] = pa->pop[(size_t)(SB + t) * P + r];
      rows[(size_t)t * P + r] = gt[j];
      rows[(size_t)(SB + t) * P + r] = gt[NA + j];
    }
  }
  __syncthreads();
  // decode the group's nodes of the trial
  auto put_nodes = [&]() {
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int t = n_lo + j;
      if (t < n_hi && live) {
        uint32_t f = 0, th = 0;
        decode_node(gt[j], gt[NA + j], F, s_nu, f, th);
        // (a node without a split reads column 0 with threshold 0: all right)
        x_col[t * P + r] = (uint16_t)(f ? (f - 1u) * SCOL : 0u);
        x_thr[t * P + r] = th;
        if (f) atomicAdd(&s_spl[r], 1u);
      }
    }
    __syncthreads();
  };
  put_nodes();

  const size_t cstride = (size_t)SB * K * Ppad;
  const uint64_t key = de_key(pa->seed, pa->prob);
  double cost_r = 0.0, cost_fin = 0.0;
  uint32_t bst_fin = 0;
  const uint32_t part = h % PARTS;
  const uint32_t cls0 = nt ? (s_info[0] >> 8) & 0xFFu : 0u;  // slot of class c: c - cls0
  const bool whole = slots == K;  // a counter for every class: slot = class
  double *const xcost = pa->xcost;
  const uint32_t cbase = whole ? 0u : cls0;
  // generation G + 1, when the best tree is wanted, counts that tree alone
  const uint32_t g_end = pa->out_label ? pa->G + 1 : pa->G;
  for (uint32_t g = 0; g <= g_end; ++g) {
    // the lane index is re-read each generation, so that the compiler
    // recomputes the addresses derived from it instead of holding them in
    // registers across the whole loop (1,024 threads leave 128 per lane)
    asm volatile("" : "+v"(r));
    uint32_t *cnt = pa->cnt + (size_t)(g % 3) * cstride;
    if (!solo) {
      uint32_t *z = pa->cnt + (size_t)((g + 1) % 3) * cstride;
      for (size_t i = (size_t)b * RES_THREADS + threadIdx.x; i < cstride; i += (size_t)nb * RES_THREADS)
        __hip_atomic_store(z + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // ---- left counts of this block's tiles.  (In the pass for the best tree
    // every lane holds that tree; lane 0 adds.)
    {
      const bool adds = live && (g <= pa->G || r == 0);
      const uint32_t rr = live ? r : 0u;
      uint32_t col[NN], thr[NN], acc[NN];
#pragma unroll
      for (int i = 0; i < NN; ++i) {
        const uint32_t t = part_node<D, L>(part, i);
        col[i] = s0 + x_col[t * P + rr];
        thr[i] = x_thr[t * P + rr];
        acc[i] = 0;
      }
      uint32_t cur = 0xFFFFFFFFu;
      auto flush = [&]() {
        if (cur == 0xFFFFFFFFu || !adds) return;
        const uint32_t slot = cur - cbase;
#pragma unroll
        for (int i = 0; i < NN; ++i) {
          // a path node is counted by the leftmost part below it
          if (i < L && (part & ((1u << (L - i)) - 1u)) != 0u) continue;
          const uint32_t t = part_node<D, L>(part, i);
          if (slot < slots) atomicAdd(&s_cnt[(t * slots + slot) * P + r], acc[i]);
          else if (acc[i]) atomicAdd(cnt + ((size_t)t * K + cur) * Ppad + r, acc[i]);
        }
      };
      for (uint32_t i = h / PARTS; i < nt; i += H / PARTS) {
        const uint32_t inf = s_info[i], cls = (inf >> 8) & 0xFFu;
        if (cls != cur) {
          flush();
          cur = cls;
#pragma unroll
          for (int q = 0; q < NN; ++q) acc[q] = 0;
        }
        eval_part<D, L>(kmask, i * tile_lds, part, (1ull << (inf & 0xFFu)) - 1ull, col, thr, acc);
      }
      flush();
    }
    __syncthreads();
    if (!solo) {
      // the block's counts to memory: slot c of node t is class cbase + c
      if (whole) {
        if (live)
          for (uint32_t y = h; y < SB * K; y += H) {
            const uint32_t v = s_cnt[y * P + r];
            if (v) atomicAdd(cnt + (size_t)y * Ppad + r, v);
          }
      } else if (live) {
        const uint32_t ce = min(slots, K - cls0), inv = 0xFFFFFFFFu / slots + 1u;
        for (uint32_t y = h; y < SB * slots; y += H) {
          const uint32_t t = slots == 1 ? y : __umulhi(y, inv), c = y - t * slots;
          const uint32_t v = c < ce ? s_cnt[y * P + r] : 0u;
          if (v) atomicAdd(cnt + ((size_t)t * K + cls0 + c) * Ppad + r, v);
        }
      }
      barrier_arrive(pa->bar, bk, b, nb);
    }

    // ---- the random draws of generation g + 1 (they depend only on the seed,
    // the generation, the individual and the slot), made while the other
    // blocks finish
    const uint32_t gg = g + 1;
    double Mr = pa->M;
    uint32_t r1 = 0, r2 = 0, qr = 0, cross = 0;
    if (live && g < pa->G && n_lo < n_hi) {
      // draw (gg, r, slot) is SplitMix64 output (base counter + slot)
      const uint64_t dbase =
          key + ((((uint64_t)gg << 40) | ((uint64_t)r << 20)) + 1ull) * 0x9E3779B97F4A7C15ull;
      auto draw = [&](uint32_t slot) {
        return sm64_fmix(dbase + (uint64_t)slot * 0x9E3779B97F4A7C15ull);
      };
      if (pa->M < 0.0) Mr = to_unit(draw(0));
      r1 = to_below(draw(1), P - 1u);
      r1 += (r1 >= r) ? 1u : 0u;
      r2 = to_below(draw(2), P - 2u);
      const uint32_t a = r < r1 ? r : r1, c = r < r1 ? r1 : r;
      r2 += (r2 >= a) ? 1u : 0u;
      r2 += (r2 >= c) ? 1u : 0u;
      qr = to_below(draw(3), m);
#pragma unroll
      for (int jj = 0; jj < 2 * NA; ++jj) {
        const int t = n_lo + (jj < NA ? jj : jj - NA);
        if (t >= n_hi) continue;
        const uint32_t q = (uint32_t)(t + (jj < NA ? 0 : SB));
        if (to_unit(draw(4u + q)) <= pa->CR || q == qr) cross |= 1u << jj;
      }
    }
    if (!solo) barrier_wait(pa->bar, bk++, pa->err, wait_ticks);

    if (g > pa->G) {
      // ---- the best tree's nodes, leaf classes (the largest count, ties to
      // the lower class, an empty leaf class 0), correct count and cost
      if (b == 0) {
        auto count = [&](uint32_t t, uint32_t k) {
          return solo ? s_cnt[(t * slots + k) * P]
                      : __hip_atomic_load(cnt + ((size_t)t * K + k) * Ppad, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
        };
        if (threadIdx.x < LN) {  // a thread per last-level node: its two leaves
          const uint32_t x = threadIdx.x;
          uint32_t bv[2] = {0, 0}, bk[2] = {0, 0};
          for (uint32_t k = 0; k < K; ++k) {
            uint32_t v = s_tot[k], node = 1;
            for (int d = D - 2; d >= 0; --d) {
              const uint32_t left = count(node - 1, k), bit = (x >> d) & 1u;
              v = bit ? v - left : left;
              node = 2 * node + bit;
            }
            const uint32_t left = count(node - 1, k), two[2] = {left, v - left};
            for (int q = 0; q < 2; ++q)
              if (two[q] > bv[q]) {
                bv[q] = two[q];
                bk[q] = k;
              }
          }
          pa->out_label[2 * x] = (uint8_t)bk[0];
          pa->out_label[2 * x + 1] = (uint8_t)bk[1];
          atomicAdd(&s_cor[0], bv[0] + bv[1]);  // (cleared after the last costs)
        }
        if (threadIdx.x < SB) {
          uint32_t f = 0, th = 0;
          decode_node(rows[(size_t)threadIdx.x * P + bst_fin],
                      rows[(size_t)(SB + threadIdx.x) * P + bst_fin], F, s_nu, f, th);
          pa->out_feat[threadIdx.x] = (uint8_t)f;
          pa->out_tau[threadIdx.x] = th;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
          *pa->out_correct = s_cor[0];
          *pa->out_cost = run_cost(cost_fin, pa->alpha, s_spl[0]);
        }
      }
      break;
    }

    // ---- costs (eq. opt_all and the soft-constraint fitness)
    double tc = 0.0;
    if (split) {
      // The block's own individuals: their counts into LDS (consecutive
      // threads load consecutive individuals of one counter), a thread per
      // individual and last-level node, and every cost back through memory
      // and a second barrier.
      const uint32_t own = i1 - i0, ny = SB * K;
      for (uint32_t e = threadIdx.x; e < own * ny; e += RES_THREADS) {
        const uint32_t y = e / own, i = e - y * own;
        s_cnt[i * ny + y] = __hip_atomic_load(cnt + (size_t)y * Ppad + i0 + i, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      for (uint32_t e = threadIdx.x; e < own * LN; e += RES_THREADS) {
        const uint32_t i = e / LN, x = e % LN;
        const uint32_t *c = s_cnt + i * ny;
        uint32_t nl0 = 0, nl1 = 0, b0 = 0, b1 = 0;
#pragma unroll 2
        for (uint32_t k = 0; k < K; ++k) {
          uint32_t v = s_tot[k], node = 1;
#pragma unroll
          for (int d = D - 2; d >= 0; --d) {
            const uint32_t left = c[(node - 1) * K + k], bit = (x >> d) & 1u;
            v = bit ? v - left : left;
            node = 2 * node + bit;
          }
          const uint32_t a = c[(node - 1) * K + k], z = v - a;
          nl0 += a;
          nl1 += z;
          b0 = a > b0 ? a : b0;
          b1 = z > b1 ? z : b1;
        }
        const uint32_t vio = (nl0 > 0 && nl0 < pa->n_min ? 1u : 0u) + (nl1 > 0 && nl1 < pa->n_min ? 1u : 0u);
        atomicAdd(&s_cor[i0 + i], b0 + b1);
        if (vio) atomicAdd(&s_vio[i0 + i], vio);
      }
      __syncthreads();
      if (threadIdx.x < own) {
        const uint32_t i = i0 + threadIdx.x;
        double v = (double)(n_sub - s_cor[i]);
        v = __dadd_rn(v, __dmul_rn(pa->alpha, (double)s_spl[i]));
        v = __dadd_rn(v, (double)s_vio[i]);
        __hip_atomic_store(xcost + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      barrier_arrive(pa->bar, bk, b, nb);
      barrier_wait(pa->bar, bk++, pa->err, wait_ticks);
      if (live) tc = __hip_atomic_load(xcost + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      // a group scores its last-level nodes' leaves over all classes, the
      // groups' sums meet in LDS
    {
        uint32_t nl[2 * XN], bl[2 * XN];
#pragma unroll
        for (int q = 0; q < 2 * XN; ++q) nl[q] = bl[q] = 0;
        for (uint32_t k0 = 0; k0 < K; k0 += slots) {
          const uint32_t kc = min(slots, K - k0);
          if (!solo) {
            // counts of classes k0 .. k0 + kc - 1: group h takes the (node,
            // class) pairs h, h + H, ..., up to 12 loads in flight; a batch's
            // loads past the last pair repeat it, so that none carries a branch
            if (k0) __syncthreads();  // the last chunk is scored
            const uint32_t *src = cnt + (live ? r : 0u), ny = SB * kc;
            // y / kc by a reciprocal (exact: y kc < 2^32)
            const uint32_t inv = 0xFFFFFFFFu / kc + 1u;
            auto batch = [&](uint32_t y0, auto size) {
              constexpr uint32_t CB = decltype(size)::value;
              uint32_t v[CB], at[CB];
#pragma unroll
              for (uint32_t u = 0; u < CB; ++u) {
                const uint32_t y = min(y0 + u * H, ny - 1u);
                at[u] = y;
                uint32_t m_y = y;  // in memory: [node][K]
                if (!whole) {
                  const uint32_t t = kc == 1 ? y : __umulhi(y, inv), c = y - t * kc;
                  at[u] = t * slots + c;
                  m_y = t * K + k0 + c;
                }
                v[u] = __hip_atomic_load(src + (size_t)m_y * Ppad, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
              }
#pragma unroll
              for (uint32_t u = 0; u < CB; ++u)
                if (live) s_cnt[at[u] * P + r] = v[u];
            };
            uint32_t y0 = h;
            for (; y0 + 8 * H < ny; y0 += 12 * H) batch(y0, std::integral_constant<uint32_t, 12>{});
            if (y0 + 4 * H < ny) batch(y0, std::integral_constant<uint32_t, 8>{});
            else if (y0 + H < ny) batch(y0, std::integral_constant<uint32_t, 4>{});
            else if (y0 < ny) batch(y0, std::integral_constant<uint32_t, 1>{});
            __syncthreads();
          }
          if (live)
#pragma unroll 2
            for (uint32_t kk = 0; kk < kc; ++kk) {
              const uint32_t tot = s_tot[k0 + kk];
#pragma unroll
              for (int q = 0; q < XN; ++q) {
                const uint32_t x = h + (uint32_t)q * H;
                if (x >= LN) continue;
                uint32_t v = tot, node = 1;
#pragma unroll
                for (int d = D - 2; d >= 0; --d) {
                  const uint32_t left = s_cnt[((node - 1) * slots + kk) * P + r];
                  const uint32_t bit = (x >> d) & 1u;
                  v = bit ? v - left : left;
                  node = 2 * node + bit;
                }
                const uint32_t a = s_cnt[((node - 1) * slots + kk) * P + r], c = v - a;
                nl[2 * q] += a;
                nl[2 * q + 1] += c;
                bl[2 * q] = a > bl[2 * q] ? a : bl[2 * q];
                bl[2 * q + 1] = c > bl[2 * q + 1] ? c : bl[2 * q + 1];
              }
            }
        }
        uint32_t cor = 0, vio = 0;
#pragma unroll
        for (int q = 0; q < 2 * XN; ++q) {
          cor += bl[q];
          vio += (nl[q] > 0 && nl[q] < pa->n_min) ? 1u : 0u;
        }
        if (live && h < LN) {
          atomicAdd(&s_cor[r], cor);
          if (vio) atomicAdd(&s_vio[r], vio);
        }
      }
      __syncthreads();
      if (live) {
        tc = (double)(n_sub - s_cor[r]);
        tc = __dadd_rn(tc, __dmul_rn(pa->alpha, (double)s_spl[r]));
        tc = __dadd_rn(tc, (double)s_vio[r]);
      }
    }
    // ---- selection (eq. selection; the trial wins ties), or the initial cost
    if (g == 0) {
      cost_r = tc;
    } else if (live && tc <= cost_r) {
      cost_r = tc;
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const int t = n_lo + j;
        if (t < n_hi) {
          rows[(size_t)t * P + r] = gt[j];
          rows[(size_t)(SB + t) * P + r] = gt[NA + j];
        }
      }
    }
    // ---- best: lowest index of the minimum cost (every group holds the same
    // costs: the first group's waves reduce them); the counters are cleared
    // for the next generation meanwhile
    if (h == 0) {
      double bc = live ? run_key(cost_r) : ARGMIN_NONE;
      uint32_t bi = r;
      wave_argmin(bc, bi);
      if ((threadIdx.x & 63u) == 0) {
        s_bc[threadIdx.x >> 6] = bc;
        s_bi[threadIdx.x >> 6] = bi;
      }
    }
    for (uint32_t e = threadIdx.x; e < n_cnt; e += RES_THREADS) s_cnt[e] = 0;
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < 3 * P; e += RES_THREADS) s_cor[e] = 0;
    double bc = s_bc[0];
    uint32_t bst = s_bi[0];
#pragma unroll
    for (uint32_t x = 1; x < WAVES; ++x) {
      const double c2 = s_bc[x];
      const uint32_t i2 = s_bi[x];
      const bool better = (c2 < bc) | ((c2 == bc) & (i2 < bst));
      bc = better ? c2 : bc;
      bst = better ? i2 : bst;
    }
    if (g == pa->G) {
      if (b == 0 && live) {
#pragma unroll
        for (int j = 0; j < NA; ++j) {
          const int t = n_lo + j;
          if (t < n_hi) {
            pa->pop[(size_t)t * P + r] = rows[(size_t)t * P + r];
            pa->pop[(size_t)(SB + t) * P + r] = rows[(size_t)(SB + t) * P + r];
          }
        }
        if (h == 0) pa->cost[r] = cost_r;
      }
      if (b == 0 && threadIdx.x == 0) *pa->best = bst;
      if (!pa->out_label) break;
      // one more pass counts the best tree alone (every lane holds it)
      bst_fin = bst;
      cost_fin = bc;
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const int t = n_lo + j;
        if (t < n_hi) {
          gt[j] = rows[(size_t)t * P + bst];
          gt[NA + j] = rows[(size_t)(SB + t) * P + bst];
        }
      }
    } else if (live) {
      // ---- DE/best/1 mutation and binomial crossover of generation g + 1,
      // this group's nodes (the feature gene t and the threshold gene SB + t)
      const double Fp1 = (double)F + 1.0;
#pragma unroll
      for (int jj = 0; jj < 2 * NA; ++jj) {
        const int t = n_lo + (jj < NA ? jj : jj - NA);
        if (t >= n_hi) continue;
        const size_t q = (size_t)(t + (jj < NA ? 0 : SB)) * P;
        const double d = __dsub_rn(rows[q + r1], rows[q + r2]);
        double v = __dadd_rn(rows[q + bst], __dmul_rn(Mr, d));
        const double hiq = jj < NA ? Fp1 : 1.0;
        if (!(v >= 0.0)) v = 0.0;
        if (v > hiq) v = hiq;
        gt[jj] = (cross >> jj) & 1u ? v : rows[q + r];
      }
    }
    __syncthreads();  // the split counts are cleared
    put_nodes();
  }
}

// Block bx's run: from the array, or the kernel's own first argument.
__device__ __forceinline__ ArgPtr run_args(const RunArgs *runs, const uint32_t *run_of_block,
                                           uint32_t bx) {
  return runs ? (ArgPtr)(uintptr_t)(runs + __builtin_amdgcn_readfirstlane((int)run_of_block[bx]))
              : (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
}

template <int D, int WAVES, bool SPLIT>
__global__ __launch_bounds__(RES_THREADS) void k_deoct_resident(
    RunArgs one, const RunArgs *__restrict__ runs, const uint32_t *__restrict__ run_of_block,
    uint64_t wait_ticks) {
  extern __shared__ __align__(16) uint8_t lds[];
  resident_body<D, WAVES, SPLIT>(run_args(runs, run_of_block, blockIdx.x), blockIdx.x, wait_ticks, lds);
}

// Runs of different depths, more of them than the CUs hold at once: the runs'
// blocks are numbered in order, and a block of the launch takes the next
// number whenever it is free.  A run's blocks so start in order, and every
// block with a lower number has started: only the last run started can still
// wait at its barrier for members, and these come as earlier runs, all of whose
// blocks are running, end.
template <int WAVES>
__global__ __launch_bounds__(RES_THREADS) void k_deoct_resident_queue(
    const RunArgs *__restrict__ runs, const uint32_t *__restrict__ run_of_block,
    uint32_t n_blocks, uint32_t *__restrict__ ticket, uint64_t wait_ticks) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ uint32_t s_next;
  for (;;) {
    if (threadIdx.x == 0) s_next = atomicAdd(ticket, 1u);
    __syncthreads();
    const uint32_t bx = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_next);
    if (bx >= n_blocks) return;
    const ArgPtr pa = run_args(runs, run_of_block, bx);
    switch (pa->D) {
      case 1: resident_body<1, WAVES, true>(pa, bx, wait_ticks, lds); break;
      case 2: resident_body<2, WAVES, true>(pa, bx, wait_ticks, lds); break;
      case 3: resident_body<3, WAVES, true>(pa, bx, wait_ticks, lds); break;
      case 4: resident_body<4, WAVES, true>(pa, bx, wait_ticks, lds); break;
      default: resident_body<5, WAVES, true>(pa, bx, wait_ticks, lds); break;
    }
    __syncthreads();  // the LDS and s_next are free again
  }
}

template <bool SPLIT>
const void *resident_kernel(uint32_t D, uint32_t waves) {
#define MH_RES(DD)                                                                     \
  case DD:                                                                             \
    switch (waves) {                                                                   \
      case 1: return reinterpret_cast<const void *>(k_deoct_resident<DD, 1, SPLIT>);   \
      case 2: return reinterpret_cast<const void *>(k_deoct_resident<DD, 2, SPLIT>);   \
      case 4: return reinterpret_cast<const void *>(k_deoct_resident<DD, 4, SPLIT>);   \
      default: return reinterpret_cast<const void *>(k_deoct_resident<DD, 8, SPLIT>);  \
    }
  switch (D) {
    MH_RES(1)
    MH_RES(2)
    MH_RES(3)
    MH_RES(4)
    case 5:  // (at depth 5 more than 256 individuals do not fit the LDS)
      switch (waves) {
        case 1: return reinterpret_cast<const void *>(k_deoct_resident<5, 1, SPLIT>);
        case 2: return reinterpret_cast<const void *>(k_deoct_resident<5, 2, SPLIT>);
        case 4: return reinterpret_cast<const void *>(k_deoct_resident<5, 4, SPLIT>);
      }
  }
#undef MH_RES
  return nullptr;
}

uint32_t waves_of(uint32_t P) {
  const uint32_t w = pad64(P) / 64;
  return w > 4 ? 8 : (w > 2 ? 4 : w);
}

}  // namespace

// Whether the blocks of a run share out the costs.  Every block reading all P
// SB K counts takes one batch of 12 loads per thread and group; past that, each
// block scores its own individuals and a second barrier (about 3,500 cycles)
// brings the costs back, with counters only for the classes of the block's own
// tiles.  Measured, cycles of a generation: n = 10^4, F = 20, K = 10, depth 4, P
// = 128 on 34 blocks 36,900 -> 29,300, on 85 blocks 29,300 -> 25,200; n = 3
// 10^4, F = 13, K = 5, depth 5, P = 100 on 256 blocks 39,500 -> 35,800.
bool split_costs(uint32_t P, uint32_t SB, uint32_t K, uint32_t nb) {
  return nb > 1 && SB * K > 12u * (RES_THREADS / (waves_of(P) * 64));
}

RunShape resident_fit(const Ctx *ctx, uint32_t D, uint32_t P, uint32_t F, uint32_t K,
                      uint32_t tiles, uint32_t nb) {
  RunShape r;
  if (!ctx->coop || D < 1 || D > 5 || P > 512 || F > 80 || nb == 0) return r;
  if (!resident_kernel<false>(D, waves_of(P))) return r;
  const uint32_t SB = (1u << D) - 1u, max_lds = ctx->max_lds - 2048;  // (coop_per_cu's margin)
  const uint32_t tm = (std::max(tiles, 1u) + nb - 1) / nb;
  if (tm > RES_MAX_TILES) return r;
  // class counters: as many as fit (a block's counts of the classes past them
  // add to memory, and the costs take the classes in chunks of them); all for
  // one block
  const bool split = split_costs(P, SB, K, nb);
  const uint32_t own = split ? (P + nb - 1) / nb : 0u;
  uint32_t slots = split ? std::min(K, tm) : K;
  while (nb > 1 && slots > 1 && res_lds(SB, P, F, K, slots, tm, own).total > max_lds) --slots;
  const uint32_t lds = res_lds(SB, P, F, K, slots, tm, own).total;
  if (lds <= max_lds) r = RunShape{nb, tm, slots, lds, split};
  return r;
}

// Cycles of a generation of a run of the given shape (2.4 GHz) over `tiles`
// tiles, by the parts that a block works through one after another: its
// group's nodes (mutation, crossover, decode), its searches (33 cycles of a CU's
// LDS each), its leaf scores, and with several blocks the exchange.  Against
// 7,900 measured runs (n = 300 to 16,000, F = 2 to 20, K = 2 to 40, depth 1 to 5,
// P = 8 to 512, 1 to 256 blocks): 4 % too long on average, standard deviation 12 %.
double resident_cycles(uint32_t D, uint32_t P, uint32_t K, const RunShape &r, uint32_t tiles) {
  const uint32_t SB = (1u << D) - 1u, LN = 1u << (D - 1), w = waves_of(P), H = 16 / w;
  const uint32_t per = std::max(1u, (tiles + r.nblk - 1) / r.nblk);
  const double searches = D < 4 ? SB : (D == 4 ? 16 : (H >= 4 ? 36 : 32));  // of a tile and wave
  double t = 900.0 + 770.0 * D + 500.0 * w + 3700.0 * ((SB + H - 1) / H) + 33.0 * per * w * searches;
  if (!r.split) t += 100.0 * K * ((LN + H - 1) / H) * D;
  if (r.split) t += 16600.0 - 47.0 * std::min(r.nblk, 128u);  // (a block scores P / nblk)
  else if (r.nblk > 1) t += (r.slots < K ? 14000.0 : w == 1 && D > 3 ? 7500.0 : 6000.0) + 12.0 * r.nblk;
  return t;
}

// The same of the form with all of a tree's nodes in a thread's registers and
// few tiles per block (persist.hip): standard deviation 10 % over 590 runs.
static double unrolled_cycles(uint32_t D, uint32_t P, uint32_t K) {
  const uint32_t SB = (1u << D) - 1u, w = waves_of(P), H = w <= 4 ? 2 : 1;
  return 8100.0 - 1220.0 * D + 130.0 * w + 280.0 * SB + 2430.0 * ((SB + H - 1) / H) + 80.0 * SB * K;
}

RunShape resident_shape(const Ctx *ctx, uint32_t D, uint32_t P, uint32_t F, uint32_t K,
                        uint32_t tiles, uint32_t tiles_likely, uint32_t max_blocks) {
  // Several blocks only where the groups are many: up to 128 individuals (eight
  // groups), from depth 3 on.  Elsewhere two groups per block with all of a
  // tree's nodes in registers (persist.hip) are as fast or faster.  Per
  // generation, there against here: n = 5 10^4, F = 21, P = 100, depth 3: 9.5
  // and 8.6 us; n = 5000, F = 10, P = 128, depth 3: 7.5 and 7.2; n = 2000, F =
  // 20, P = 100, depth 1: 4.0 and 4.9; n = 4000, F = 4, P = 128, depth 2: 5.0 and
  // 5.4; n = 10^5, F = 16, P = 256, depth 3: 10.4 and 10.8; n = 2 10^4, F = 8, P =
  // 512, depth 3: 11.5 and 13.3.  At depth 1 its several blocks per CU get in
  // each other's way when they add to few classes' counters: n = 6.4 10^4, F =
  // 4, K = 2, P = 128 6.1 and 5.3, n = 3.2 10^4, F = 12, K = 3, P = 64 6.6 and 4.7,
  // but n = 10^4, K = 3 4.4 and 4.5, n = 6.4 10^4, F = 5, K = 10, P = 8 4.7 and 5.5.
  const bool contended = D == 1 && K <= (P <= 64 ? 4u : 2u) &&
                         (P > 32 ? 3u : 2u) * tiles_likely >= (uint32_t)ctx->num_cu * K;
  const bool several = (P <= 128 && D >= 3) || (P <= 128 && contended) || ctx->resident_blocks;
  RunShape best;
  double best_t = 1e300;
  for (uint32_t nb = 1; nb <= (several ? max_blocks : 1u); ++nb) {
    const RunShape r = resident_fit(ctx, D, P, F, K, tiles, nb);
    if (!r.nblk) continue;
    const double t = resident_cycles(D, P, K, r, tiles_likely);
    // One block alone against that form: it needs no exchange but has all the
    // searches.  n = 300, F = 4, K = 2, P = 512, depth 2 (7 tiles) 5.8 us there
    // and 7.2 here; n = 2000, P = 200, depth 3 (33 tiles) 7.4 and 16.2, n = 1000,
    // F = 4, P = 32, depth 2 (17 tiles) 4.9 and 3.5.
    if (!several && t > unrolled_cycles(D, P, K)) continue;
    if (ctx->resident_blocks ? nb == ctx->resident_blocks : t < best_t) {
      best_t = t;
      best = r;
    }
  }
  return best;
}

mh_status launch_resident(Ctx *ctx, const std::vector<RunArgs> &runs, uint32_t lds,
                          RunArgs *runs_dev, uint32_t *map_dev, bool *used) {
  *used = false;
  uint32_t grid = 0, Pmax = 0;
  for (const RunArgs &r : runs) {
    grid += r.nblk;
    Pmax = std::max(Pmax, r.P);
  }
  const uint32_t D = runs[0].D, waves = waves_of(Pmax);
  bool split = false;
  for (const RunArgs &r : runs) split = split || r.xcost;
  const void *kern = split ? resident_kernel<true>(D, waves) : resident_kernel<false>(D, waves);
  if (!kern || grid == 0 || grid > (uint32_t)ctx->num_cu) return MH_OK;
  if (coop_per_cu(ctx, kern, RES_THREADS, lds) < 1 || coop_is_bad(ctx, kern, grid)) return MH_OK;
  RunArgs one = runs[0];
  const RunArgs *rd = nullptr;
  const uint32_t *md = nullptr;
  if (runs.size() > 1) {
    std::vector<uint32_t> map;
    for (size_t i = 0; i < runs.size(); ++i) map.insert(map.end(), runs[i].nblk, (uint32_t)i);
    MH_HIP(ctx, hipMemcpyAsync(runs_dev, runs.data(), runs.size() * sizeof(RunArgs),
                               hipMemcpyHostToDevice, ctx->stream));
    MH_HIP(ctx, hipMemcpyAsync(map_dev, map.data(), map.size() * 4, hipMemcpyHostToDevice,
                               ctx->stream));
    MH_HIP(ctx, hipStreamSynchronize(ctx->stream));  // the host vectors go out of scope
    rd = runs_dev;
    md = map_dev;
  }
  uint64_t ticks = ctx->wait_ticks;
  if (ctx->debug)
    std::fprintf(stderr, "k_deoct_resident<%u,%u>: %zu runs, grid %u, tiles %u per block, %u class slots, LDS %u bytes\n",
                 D, waves, runs.size(), grid, one.tiles_max, one.slots, lds);
  void *args[] = {&one, &rd, &md, &ticks};
  const hipError_t e = launch_grid_sync(ctx, kern, dim3(grid), dim3(RES_THREADS), args, lds);
  if (e == hipErrorInvalidValue || e == hipErrorCooperativeLaunchTooLarge ||
      e == hipErrorInvalidConfiguration) {
    (void)hipGetLastError();
    return MH_OK;
  }
  if (e != hipSuccess) return hip_fail(ctx, e, "k_deoct_resident");
  ctx->last_coop_kern = kern;
  ctx->last_coop_grid = grid;
  *used = true;
  return MH_OK;
}

mh_status launch_resident_queue(Ctx *ctx, uint32_t P_max, uint32_t n_blocks, uint32_t lds,
                                const RunArgs *runs_dev, const uint32_t *map_dev,
                                uint32_t *ticket, bool *used) {
  *used = false;
  const uint32_t waves = waves_of(P_max);
  const void *kern = waves == 1   ? reinterpret_cast<const void *>(k_deoct_resident_queue<1>)
                     : waves == 2 ? reinterpret_cast<const void *>(k_deoct_resident_queue<2>)
                                  : nullptr;
  const uint32_t grid = std::min(n_blocks, (uint32_t)ctx->num_cu);
  if (!kern || grid == 0) return MH_OK;
  if (coop_per_cu(ctx, kern, RES_THREADS, lds) < 1 || coop_is_bad(ctx, kern, grid)) return MH_OK;
  uint64_t ticks = ctx->wait_ticks;
  if (ctx->debug)
    std::fprintf(stderr, "k_deoct_resident_queue<%u>: %u blocks of work, grid %u, LDS %u bytes\n",
                 waves, n_blocks, grid, lds);
  void *args[] = {&runs_dev, &map_dev, &n_blocks, &ticket, &ticks};
  const hipError_t e = launch_grid_sync(ctx, kern, dim3(grid), dim3(RES_THREADS), args, lds);
  if (e == hipErrorInvalidValue || e == hipErrorCooperativeLaunchTooLarge ||
      e == hipErrorInvalidConfiguration) {
    (void)hipGetLastError();
    return MH_OK;
  }
  if (e != hipSuccess) return hip_fail(ctx, e, "k_deoct_resident_queue");
  ctx->last_coop_kern = kern;
  ctx->last_coop_grid = grid;
  *used = true;
  return MH_OK;
}

}  // namespace mh
