// split.hip -- the exact depth-1 split (Algorithm 2's horizon-1 branch), batched
// over subsets, and CART built from it.
//
// The elements are the (member sample, feature) pairs, per feature in the order
// (subset, rank).  In that order a threshold right after position p of a
// subset's run (tau = rank_p + 1, taken where the rank changes) leaves L_k =
// #{class k in the run up to p} samples of class k on the left; its correct
// count is max_k L_k + max_k (N_k - L_k).  The winner per subset is the first
// strict maximum in the order (no split, then feature, then tau): the largest
// correct count, ties to the smallest (feature, tau), and no split unless a
// split is strictly better.
//
// The same machinery gives CART's split (Gini impurity): the candidate's
// score is sum_k L_k^2 / |L| + sum_k R_k^2 / |R| in f64 (the integer sums of
// squares divided by the side sizes, then added, each correctly rounded), the
// winner the first strict maximum over (feature, tau); a subset splits iff it
// holds two or more classes and has a candidate.  Scores are positive, so
// their bit patterns order as u64.
//
// The order is sorted once (stable LSD radix passes over the rank's bytes, one
// segment per feature, then over the subset's where there are several).  CART
// keeps it from level to level: the two children of a node are a stable
// two-way partition of the node's run, one streaming pass, where sorting every
// level anew took a pass over 12 bytes an element for each byte of the key.
// Measured: CART of depth 8 at n = 4 10^5, F = 20, K = 3: 6.67 -> 1.82 ms; a
// level's evaluation 118 us twice -> 77 us, its order 400 us of radix passes
// -> 66 us of partition.
#include <algorithm>
#include <vector>

#include "device_common.h"
#include "internal.h"
#include "range.h"
#include "xcd.h"

namespace mh {
namespace {

// An element: rank and class in the high word, the sample in the low one.
// The class travels in the rank's top byte while ranks fit 24 bits, else it
// is read from the labels.
constexpr uint32_t SPLIT_PACK_MAX_N = 1u << 24;

struct ClassOf {
  const uint8_t *labels;  // null: packed
  __device__ __forceinline__ uint32_t cls(uint64_t e) const {
    return labels ? labels[(uint32_t)e] : (uint32_t)(e >> 56);
  }
  __device__ __forceinline__ uint32_t rank(uint64_t e) const {
    const uint32_t hi = (uint32_t)(e >> 32);
    return labels ? hi : hi & 0xFFFFFFu;
  }
};

// The members of the subsets (sub_of < nsub, or every sample when sub_of is
// null; valid labels), in whatever order the block adds give.
__global__ __launch_bounds__(256) void k_split_members(const uint32_t *__restrict__ sub_of,
                                                       uint32_t n, uint32_t nsub,
                                                       const uint8_t *__restrict__ labels,
                                                       uint32_t K, uint32_t span,
                                                       uint32_t *__restrict__ cursor,
                                                       uint32_t *__restrict__ mem) {
  __shared__ uint32_t s_w[4], s_base;
  const uint32_t j0 = blockIdx.x * span;
  const uint32_t j1 = (uint32_t)min((uint64_t)n, (uint64_t)j0 + span);  // no wrap near 2^32
  auto member = [&](uint32_t i) { return (sub_of ? sub_of[i] : 0u) < nsub && labels[i] < K; };
  uint32_t base = range_reserve(j0, j1, member, cursor, s_w, &s_base);
  for (uint32_t c0 = j0; c0 < j1; c0 += 256u)
    base += chunk_members(c0, j1, member, [&](uint32_t l, uint32_t i) { mem[base + l] = i; }, s_w);
}

// Elements of feature blockIdx.y, in member order.
__global__ __launch_bounds__(256) void k_split_elems(const uint32_t *__restrict__ mem, uint32_t M,
                                                     const uint32_t *__restrict__ ranks,
                                                     uint32_t ld,
                                                     const uint8_t *__restrict__ labels,
                                                     uint32_t packed, uint64_t *__restrict__ out) {
  const uint32_t f = blockIdx.y;
  const uint32_t *col = ranks + (size_t)f * ld;
  uint64_t *o = out + (size_t)f * M;
#pragma unroll
  for (uint32_t u = 0; u < 4; ++u) {
    const uint32_t q = (blockIdx.x * 4u + u) * 256u + threadIdx.x;
    if (q < M) {
      const uint32_t i = mem[q];
      const uint32_t hi = packed ? ((uint32_t)labels[i] << 24) | col[i] : col[i];
      o[q] = ((uint64_t)hi << 32) | i;
    }
  }
}

// Where the subsets lie: seg[s] the first position of subset s inside every
// feature (seg[nsub] the end), cum[s][k] the class-k members of the subsets
// before s, and even[s] the members of the even-numbered subsets before s (the
// left children, when subsets 2 q and 2 q + 1 are the children of q).  Block k
// < K scans class k, block K the sizes, block K + 1 the even sizes.
__global__ __launch_bounds__(256) void k_split_plan(const uint32_t *__restrict__ tot, uint32_t nsub,
                                                    uint32_t K, uint32_t *__restrict__ seg,
                                                    uint32_t *__restrict__ cum,
                                                    uint32_t *__restrict__ even) {
  __shared__ uint32_t s_w[4];
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6, k = blockIdx.x;
  uint32_t run = 0;
  for (uint32_t s0 = 0; s0 < nsub; s0 += 256u) {
    const uint32_t s = s0 + threadIdx.x;
    uint32_t v = 0;
    if (s < nsub) {
      if (k < K) v = tot[(size_t)s * K + k];
      else if (k == K || !(s & 1u))
        for (uint32_t c = 0; c < K; ++c) v += tot[(size_t)s * K + c];
    }
    uint32_t x = v;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    uint32_t before = run;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      before += q < w ? s_w[q] : 0u;
      run += s_w[q];
    }
    __syncthreads();
    if (s < nsub) {
      if (k < K) cum[(size_t)s * K + k] = before + x - v;
      else (k == K ? seg : even)[s] = before + x - v;
    }
  }
  if (threadIdx.x == 0 && k >= K) (k == K ? seg : even)[nsub] = run;
}

// A wave's share of a feature's run: SP_ROUNDS x 64 consecutive positions.
// Eight rounds keep eight loads of a lane in flight and leave a wave
// independent of the others (no barrier); its class counts start from the
// scanned counts of the spans before it.
constexpr uint32_t SP_ROUNDS = 8, SP_SPAN = 64 * SP_ROUNDS;

// Class counts of every span: sums[(f K + k) nspan + i].
__global__ __launch_bounds__(256) void k_split_class_sums(const uint64_t *__restrict__ el, uint32_t M,
                                                          uint32_t F, uint32_t K, uint32_t nspan,
                                                          ClassOf co,
                                                          uint32_t *__restrict__ sums) {
  const uint32_t bi = xcd_order(blockIdx.x, gridDim.x);
  const uint32_t g = bi * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
  if (g >= F * nspan) return;
  const uint32_t f = g / nspan, i = g % nspan;
  const uint64_t *e = el + (size_t)f * M;
  uint32_t c[SP_ROUNDS];
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint32_t p = i * SP_SPAN + r * 64u + lane;
    c[r] = p < M ? co.cls(e[p]) : 0xFFFFFFFFu;
  }
  // lane l ends up with the count of class k0 + l
  for (uint32_t k0 = 0; k0 < K; k0 += 64u) {
    uint32_t mine = 0;
    const uint32_t kn = min(64u, K - k0);
    for (uint32_t k = 0; k < kn; ++k) {
      uint32_t t = 0;
#pragma unroll
      for (uint32_t r = 0; r < SP_ROUNDS; ++r) t += (uint32_t)__popcll(__ballot(c[r] == k0 + k));
      mine = lane == k ? t : mine;
    }
    if (lane < kn) sums[((size_t)f * K + k0 + lane) * nspan + i] = mine;
  }
}

// Exclusive scan of each of `rows` rows of `len` counts, a wave per row.
__global__ __launch_bounds__(256) void k_split_row_scan(uint32_t *__restrict__ v, uint32_t rows,
                                                        uint32_t len) {
  const uint32_t row = blockIdx.x * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
  if (row >= rows) return;
  uint32_t *p = v + (size_t)row * len;
  uint32_t run = 0, next = lane < len ? p[lane] : 0u;
  for (uint32_t q0 = 0; q0 < len; q0 += 64u) {
    const uint32_t mine = next, q = q0 + lane;
    next = q + 64u < len ? p[q + 64u] : 0u;  // in flight during the scan
    uint32_t x = mine;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (q < len) p[q] = run + x - mine;
    run += __shfl(x, 63, 64);
  }
}

// The same by a block per row, SCAN_LONG counts in turn: the steps of a row wait
// for each other, and a wave's 64 counts at a time are 1,830 steps at 6 10^7
// elements.  The exact split of so many samples, one column, 2 and 5 classes:
// 9.38 -> 8.39 and 9.43 -> 8.43 ms.
constexpr uint32_t SCAN_LONG = 4096;
__global__ __launch_bounds__(1024) void k_split_row_scan_long(uint32_t *__restrict__ v,
                                                              uint32_t len) {
  __shared__ uint32_t s_wave[2][16];
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  uint32_t *p = v + (size_t)blockIdx.x * len;
  uint32_t run = 0, next[4];
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    const uint32_t q = 4u * threadIdx.x + i;
    next[i] = q < len ? p[q] : 0u;
  }
  for (uint32_t q0 = 0, b = 0; q0 < len; q0 += SCAN_LONG, b ^= 1u) {
    const uint32_t q = q0 + 4u * threadIdx.x;
    uint32_t mine[4], x = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      mine[i] = next[i];
      x += next[i];
      next[i] = q + SCAN_LONG + i < len ? p[q + SCAN_LONG + i] : 0u;  // in flight meanwhile
    }
    const uint32_t sum = x;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63u) s_wave[b][w] = x;
    __syncthreads();  // (one per step: the steps take the two rows in turn)
    uint32_t before = run + x - sum;
#pragma unroll
    for (uint32_t j = 0; j < 16; ++j) {
      const uint32_t t = s_wave[b][j];
      before += j < w ? t : 0u;
      run += t;
    }
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      if (q + i < len) p[q + i] = before;
      before += mine[i];
    }
  }
}

// A wave per row up to 4 steps of it: a block's one step takes as long.
mh_status row_scan(Ctx *ctx, uint32_t *v, uint32_t rows, uint32_t len) {
  if (len > 256u)
    k_split_row_scan_long<<<rows, 1024, 0, ctx->stream>>>(v, len);
  else
    k_split_row_scan<<<(rows + 3) / 4, 256, 0, ctx->stream>>>(v, rows, len);
  MH_LAUNCHED(ctx, "k_split_row_scan");
  return MH_OK;
}

// The last subset whose run starts at or before position p (the runs of the
// subsets cover the M positions of a feature; an empty one shares its start
// with the next).
__device__ __forceinline__ uint32_t seg_at(const uint32_t *__restrict__ seg, uint32_t nsub,
                                           uint32_t p) {
  uint32_t lo = 0, hi = nsub;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (seg[mid] <= p) lo = mid;
    else hi = mid;
  }
  return lo;
}

// A candidate or none (ft all ones): score, then the smaller (feature, tau).
struct SplitBest {
  uint64_t score, ft;
};
__device__ __forceinline__ void take_better(SplitBest &a, uint64_t score, uint64_t ft) {
  const bool b = score > a.score || (score == a.score && ft < a.ft);
  a.score = b ? score : a.score;
  a.ft = b ? ft : a.ft;
}
__device__ __forceinline__ SplitBest wave_best(SplitBest v) {
  for (int d = 32; d > 0; d >>= 1) {
    const uint64_t s = __shfl_xor(v.score, d, 64), t = __shfl_xor(v.ft, d, 64);
    take_better(v, s, t);
  }
  return v;
}

// The best candidate of every (span, subset) piece.  The pieces of a feature
// form a staircase in (span i, subset s), so i + s numbers them: piece
// f (nspan + nsub) + i + s.  A span inside one subset (nearly all of them)
// takes its subset's totals from scalar loads, the others per lane.
// What bounds it: 8 B read per element, and the K ballots and squares of a
// position; the earlier form wrote K counts per element to memory, read them
// back twice and found the winner in a second evaluation pass.
template <bool GINI>
__global__ __launch_bounds__(256) void k_split_eval(
    const uint64_t *__restrict__ el, uint32_t M, uint32_t F, uint32_t K, uint32_t nspan,
    uint32_t nsub, ClassOf co, const uint32_t *__restrict__ seg, const uint32_t *__restrict__ cum,
    const uint32_t *__restrict__ tot, const uint32_t *__restrict__ sums,
    SplitBest *__restrict__ pieces) {
  const uint32_t bi = xcd_order(blockIdx.x, gridDim.x);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)(bi * 4u + (threadIdx.x >> 6)));
  if (g >= F * nspan) return;
  const uint32_t f = g / nspan, i = g % nspan;
  const uint64_t *e = el + (size_t)f * M;
  const uint32_t p0 = i * SP_SPAN, p1 = min(M, p0 + SP_SPAN) - 1u;  // p0 < M
  const uint32_t s_first = seg_at(seg, nsub, p0), s_last = seg_at(seg, nsub, p1);
  const bool uniform = s_first == s_last;
  uint32_t c[SP_ROUNDS], rk[SP_ROUNDS], sv[SP_ROUNDS];
  bool cand[SP_ROUNDS];
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint32_t p = p0 + r * 64u + lane;
    const uint64_t x = p < M ? e[p] : 0ull;
    // the next position's element: the next lane's, the last lane loads it
    const uint32_t nr_own = lane == 63 && p + 1 < M ? co.rank(e[p + 1]) : 0u;
    rk[r] = co.rank(x);
    c[r] = p < M ? co.cls(x) : 0xFFFFFFFFu;
    const uint32_t nr_sh = __shfl_down(rk[r], 1, 64);
    const uint32_t nr = lane == 63 ? nr_own : nr_sh;
    sv[r] = uniform || p >= M ? s_first : seg_at(seg, nsub, p);
    // a boundary: the rank changes between p and p + 1 inside the run
    cand[r] = p < M && p + 1 < seg[sv[r] + 1] && nr != rk[r];
  }
  // GINI: sums of squares of the two sides; else the two largest counts
  uint64_t A[SP_ROUNDS], B[SP_ROUNDS];
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) A[r] = B[r] = 0;
  const uint64_t le = ~0ull >> (63u - lane);
  for (uint32_t k = 0; k < K; ++k) {
    uint32_t run = sums[((size_t)f * K + k) * nspan + i];
    const uint32_t cum_u = uniform ? cum[(size_t)s_first * K + k] : 0u;
    const uint32_t tot_u = uniform ? tot[(size_t)s_first * K + k] : 0u;
#pragma unroll
    for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
      const uint64_t bal = __ballot(c[r] == k);
      const uint32_t cb = uniform ? cum_u : cum[(size_t)sv[r] * K + k];
      const uint32_t T = uniform ? tot_u : tot[(size_t)sv[r] * K + k];
      const uint32_t L = run + (uint32_t)__popcll(bal & le) - cb, R = T - L;
      run += (uint32_t)__popcll(bal);
      if (GINI) {
        A[r] += (uint64_t)L * L;
        B[r] += (uint64_t)R * R;
      } else {
        A[r] = L > A[r] ? L : A[r];
        B[r] = R > B[r] ? R : B[r];
      }
    }
  }
  uint64_t score[SP_ROUNDS], ft[SP_ROUNDS];
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint32_t p = p0 + r * 64u + lane;
    score[r] = 0;
    ft[r] = ~0ull;
    if (cand[r]) {
      if (GINI)
        score[r] = (uint64_t)__double_as_longlong(
            __dadd_rn(__ddiv_rn((double)A[r], (double)(p + 1 - seg[sv[r]])),
                      __ddiv_rn((double)B[r], (double)(seg[sv[r] + 1] - 1 - p))));
      else
        score[r] = A[r] + B[r];
      ft[r] = ((uint64_t)(f + 1) << 32) | (rk[r] + 1u);
    }
  }
  SplitBest *out = pieces + (size_t)f * (nspan + nsub) + i;
  for (uint32_t s = s_first; s <= s_last; ++s) {
    if (seg[s] == seg[s + 1]) continue;  // an empty subset has no piece
    SplitBest b{0ull, ~0ull};
#pragma unroll
    for (uint32_t r = 0; r < SP_ROUNDS; ++r)
      if (sv[r] == s) take_better(b, score[r], ft[r]);
    b = wave_best(b);
    if (lane == 0) out[s] = b;
  }
}

// Best of a (subset, feature): its pieces, a wave each.
__global__ __launch_bounds__(256) void k_split_best(const SplitBest *__restrict__ pieces, uint32_t F,
                                                    uint32_t nspan, uint32_t nsub,
                                                    const uint32_t *__restrict__ seg,
                                                    SplitBest *__restrict__ best) {
  const uint32_t g = blockIdx.x * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
  if (g >= nsub * F) return;
  const uint32_t s = g / F, f = g % F;
  SplitBest b{0ull, ~0ull};
  if (seg[s] < seg[s + 1]) {
    const uint32_t i1 = (seg[s + 1] - 1) / SP_SPAN;
    const SplitBest *p = pieces + (size_t)f * (nspan + nsub) + s;
    for (uint32_t i = seg[s] / SP_SPAN + lane; i <= i1; i += 64u)
      take_better(b, p[i].score, p[i].ft);
  }
  b = wave_best(b);
  if (lane == 0) best[g] = b;
}

// The winner of every subset over its features (best null: no elements at
// all), a wave each.
__global__ __launch_bounds__(256) void k_split_final(const uint32_t *__restrict__ tot, uint32_t nsub,
                                                     uint32_t K, uint32_t F, uint32_t gini,
                                                     const SplitBest *__restrict__ best,
                                                     uint8_t *__restrict__ feat,
                                                     uint32_t *__restrict__ tau,
                                                     uint32_t *__restrict__ correct) {
  const uint32_t s = blockIdx.x * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
  if (s >= nsub) return;
  SplitBest b{0ull, ~0ull};
  if (best)
    for (uint32_t f = lane; f < F; f += 64u) take_better(b, best[(size_t)s * F + f].score, best[(size_t)s * F + f].ft);
  b = wave_best(b);
  uint32_t m = 0, classes = 0;
  for (uint32_t k = 0; k < K; ++k) {
    const uint32_t v = tot[(size_t)s * K + k];
    m = v > m ? v : m;
    classes += v ? 1u : 0u;
  }
  if (lane != 0) return;
  // no split (misclassification): every sample gets the largest class
  const bool split = b.ft != ~0ull && (gini ? classes > 1 : b.score > m);
  feat[s] = split ? (uint8_t)(b.ft >> 32) : (uint8_t)0;
  tau[s] = split ? (uint32_t)b.ft : 0u;
  if (correct) correct[s] = gini ? 0u : split ? (uint32_t)b.score : m;
}

// The two-way partition of every node's run for the next level: an element
// goes left when its sample's new location is even.  Pass 1: the left flags
// (bits[span][round]) and their count per span; after a scan of the counts
// along each feature, pass 2 moves the elements.  8 B read and written per
// element and a random byte-sized gather in pass 1.
__global__ __launch_bounds__(256) void k_part_count(const uint64_t *__restrict__ el, uint32_t M,
                                                    uint32_t F, uint32_t nspan,
                                                    const uint32_t *__restrict__ loc,
                                                    uint64_t *__restrict__ bits,
                                                    uint32_t *__restrict__ lsum) {
  const uint32_t bi = xcd_order(blockIdx.x, gridDim.x);
  const uint32_t g = bi * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
  if (g >= F * nspan) return;
  const uint32_t f = g / nspan, i = g % nspan;
  const uint32_t *id = reinterpret_cast<const uint32_t *>(el + (size_t)f * M);  // low words
  uint32_t left[SP_ROUNDS];
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint32_t p = i * SP_SPAN + r * 64u + lane;
    left[r] = p < M ? ~loc[id[2 * (size_t)p]] & 1u : 0u;
  }
  uint32_t t = 0;
  uint64_t mine = 0;
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint64_t bal = __ballot(left[r]);
    t += (uint32_t)__popcll(bal);
    mine = lane == r ? bal : mine;
  }
  if (lane < SP_ROUNDS) bits[(size_t)g * SP_ROUNDS + lane] = mine;
  if (lane == 0) lsum[g] = t;
}

// seg: the runs of the nsub nodes; seg2, even2: the plan of their 2 nsub
// children.
__global__ __launch_bounds__(256) void k_part_move(
    const uint64_t *__restrict__ el, uint64_t *__restrict__ out, uint32_t M, uint32_t F,
    uint32_t nspan, uint32_t nsub, const uint32_t *__restrict__ seg,
    const uint32_t *__restrict__ seg2, const uint32_t *__restrict__ even2,
    const uint64_t *__restrict__ bits, const uint32_t *__restrict__ lsum) {
  const uint32_t bi = xcd_order(blockIdx.x, gridDim.x);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)(bi * 4u + (threadIdx.x >> 6)));
  if (g >= F * nspan) return;
  const uint32_t f = g / nspan, i = g % nspan;
  const uint64_t *e = el + (size_t)f * M;
  uint64_t *o = out + (size_t)f * M;
  const uint32_t p0 = i * SP_SPAN, p1 = min(M, p0 + SP_SPAN) - 1u;
  const uint32_t s_first = seg_at(seg, nsub, p0);
  const bool uniform = seg_at(seg, nsub, p1) == s_first;
  const uint64_t lt = lane ? ~0ull >> (64u - lane) : 0ull;
  uint64_t x[SP_ROUNDS];
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint32_t p = p0 + r * 64u + lane;
    x[r] = p < M ? e[p] : 0ull;
  }
  uint32_t run = lsum[g];  // left elements of the feature before this span
#pragma unroll
  for (uint32_t r = 0; r < SP_ROUNDS; ++r) {
    const uint32_t p = p0 + r * 64u + lane;
    const uint64_t bal = bits[(size_t)g * SP_ROUNDS + r];
    if (p < M) {
      const uint32_t s = uniform ? s_first : seg_at(seg, nsub, p);
      // left elements of the node's run before p
      const uint32_t l = run + (uint32_t)__popcll(bal & lt) - even2[2 * s];
      const uint32_t to = (bal >> lane) & 1ull ? seg2[2 * s] + l : seg2[2 * s + 1] + (p - seg[s]) - l;
      if (to < M) o[to] = x[r];  // (always, for consistent plans)
    }
    run += (uint32_t)__popcll(bal);
  }
}

// sub_of for an explicit subset: 0 for idx members, 1 for the rest; and the
// subset's class totals, counted per block in LDS (one global add per block
// and class: a million samples over a few classes would otherwise serialise
// on a few addresses).
__global__ __launch_bounds__(256) void k_mark_subset(const uint32_t *__restrict__ idx,
                                                     uint32_t n_sub, uint32_t n,
                                                     const uint8_t *__restrict__ labels,
                                                     uint32_t K, uint32_t *__restrict__ sub_of,
                                                     uint32_t *__restrict__ tot) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n_sub) {
    const uint32_t i = idx ? idx[j] : j;
    // a repeated index counts once
    if (i < n && labels[i] < K && atomicExch(&sub_of[i], 0u) != 0u) atomicAdd(&h[labels[i]], 1u);
  }
  __syncthreads();
  if (threadIdx.x < K && h[threadIdx.x]) atomicAdd(&tot[threadIdx.x], h[threadIdx.x]);
}

// ---------------------------------------------------------------------------
// CART of depth D on each of nsub subsets at once, level by level: loc[i] is
// the node (heap numbering inside its subset's tree) sample i sits at; the
// nodes of a level are split subproblems s = sub 2^l + (u - 2^l) of the
// Gini split above.
// ---------------------------------------------------------------------------
__global__ void k_cart_sub(const uint32_t *__restrict__ sub_of, uint32_t n, uint32_t nsub,
                           const uint32_t *__restrict__ loc, uint32_t l,
                           uint32_t *__restrict__ sub_l) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t s = sub_of[i];
  sub_l[i] = s < nsub ? (s << l) + loc[i] - (1u << l) : nsub << l;
}

__global__ void k_cart_put(const uint8_t *__restrict__ fl, const uint32_t *__restrict__ tl,
                           uint32_t cnt, uint32_t l, uint32_t SB, uint8_t *__restrict__ feat,
                           uint32_t *__restrict__ tau) {
  const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= cnt) return;
  const uint32_t sub = q >> l, u = (1u << l) + (q & ((1u << l) - 1u));
  feat[(size_t)sub * SB + u - 1] = fl[q];
  tau[(size_t)sub * SB + u - 1] = tl[q];
}

__global__ void k_cart_route(const uint32_t *__restrict__ sub_of, uint32_t n, uint32_t nsub,
                             uint32_t *__restrict__ loc, uint32_t l,
                             const uint8_t *__restrict__ fl, const uint32_t *__restrict__ tl,
                             const uint32_t *__restrict__ ranks, uint32_t ld, uint32_t F) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t s = sub_of[i];
  if (s >= nsub) return;
  const uint32_t u = loc[i], q = (s << l) + u - (1u << l);
  const uint32_t f = fl[q];
  const bool left = f != 0 && f <= F && ranks[(size_t)(f - 1) * ld + i] < tl[q];
  loc[i] = left ? 2 * u : 2 * u + 1;
}

// Elements of the members of nsub subsets in (subset, rank) order, and where
// the subsets lie.  plan/plan2 alternate between a level and the next.
struct SplitOrder {
  uint32_t M = 0, F = 0, K = 0, nspan = 0;
  uint64_t *el = nullptr, *alt = nullptr;
  ClassOf co{nullptr};
  struct Plan {
    uint32_t *seg, *even, *cum;
  } plan{}, plan2{};
};

mh_status order_build(Ctx *ctx, const mh_dataset *ds, const uint32_t *sub_of, uint32_t nsub,
                      uint32_t max_sub, SplitOrder &o) {
  hipStream_t st = ctx->stream;
  const uint32_t n = ds->n, F = ds->F, K = ds->K;
  uint32_t sbits = 0;
  while ((1u << sbits) < nsub) ++sbits;
  // ranks lie below n
  uint32_t rb = 1;
  while ((1ull << rb) < n) ++rb;
  uint32_t *cursor = (uint32_t *)arena_get(ctx, "sp_cursor", 256);
  uint32_t *mem = (uint32_t *)arena_get(ctx, "sp_mem", (size_t)(n ? n : 1) * 4);
  uint32_t *h = host_words(ctx);
  if (!cursor || !mem || !h) return MH_ENOMEM;
  o.F = F;
  o.K = K;
  uint32_t *pl = (uint32_t *)arena_get(ctx, "sp_plan", ((size_t)max_sub * (K + 2) + 2) * 2 * 4);
  if (!pl) return MH_ENOMEM;
  for (SplitOrder::Plan *p : {&o.plan, &o.plan2}) {
    p->seg = pl;
    p->even = p->seg + max_sub + 1;
    p->cum = p->even + max_sub + 1;
    pl = p->cum + (size_t)max_sub * K;
  }
  if (n) {
    mh_status s = launch_zero(ctx, {{cursor, 4}});
    if (s) return s;
    const uint32_t span = range_span(ctx, n);
    k_split_members<<<range_blocks(n, span), 256, 0, st>>>(sub_of, n, nsub, ds->labels, K, span,
                                                           cursor, mem);
    MH_LAUNCHED(ctx, "k_split_members");
    MH_HIP(ctx, hipMemcpyAsync(h, cursor, 4, hipMemcpyDeviceToHost, st));
    MH_HIP(ctx, hipStreamSynchronize(st));
    o.M = h[0];
  }
  const uint64_t N64 = (uint64_t)o.M * F;
  if (N64 >= 0xFFFFFFFFull) return fail(ctx, MH_EINVAL, "split1: too many elements");
  if (!o.M) return MH_OK;
  const uint32_t M = o.M;
  o.nspan = (M + SP_SPAN - 1) / SP_SPAN;
  const bool packed = n <= SPLIT_PACK_MAX_N;
  o.co.labels = packed ? nullptr : ds->labels;
  o.el = (uint64_t *)arena_get(ctx, "sp_el_a", (size_t)N64 * 8);
  o.alt = (uint64_t *)arena_get(ctx, "sp_el_b", (size_t)N64 * 8);
  if (!o.el || !o.alt) return MH_ENOMEM;
  k_split_elems<<<dim3((M + 1023) / 1024, F), 256, 0, st>>>(mem, M, ds->ranks, ds->ld, ds->labels,
                                                            packed ? 1u : 0u, o.el);
  MH_LAUNCHED(ctx, "k_split_elems");
  for (uint32_t shift = 0; shift < rb; shift += 8) {
    mh_status s = seg_radix_pass(ctx, o.el, o.alt, M, F, 32 + shift, nullptr);
    if (s) return s;
    std::swap(o.el, o.alt);
  }
  for (uint32_t shift = 0; shift < sbits; shift += 8) {
    mh_status s = seg_radix_pass(ctx, o.el, o.alt, M, F, shift, sub_of);
    if (s) return s;
    std::swap(o.el, o.alt);
  }
  return MH_OK;
}

mh_status order_plan(Ctx *ctx, const SplitOrder &o, const SplitOrder::Plan &p, const uint32_t *tot,
                     uint32_t nsub) {
  k_split_plan<<<o.K + 2, 256, 0, ctx->stream>>>(tot, nsub, o.K, p.seg, p.cum, p.even);
  MH_LAUNCHED(ctx, "k_split_plan");
  return MH_OK;
}

// The winners of the nsub subsets of the order's plan.
mh_status order_eval(Ctx *ctx, const SplitOrder &o, const uint32_t *tot, uint32_t nsub, bool gini,
                     uint8_t *feat, uint32_t *tau, uint32_t *correct) {
  hipStream_t st = ctx->stream;
  const uint32_t M = o.M, F = o.F, K = o.K, nspan = o.nspan;
  SplitBest *best = nullptr;
  if (M) {
    uint32_t *sums = (uint32_t *)arena_get(ctx, "sp_csum", (size_t)F * K * nspan * 4);
    SplitBest *pieces =
        (SplitBest *)arena_get(ctx, "sp_pieces", (size_t)F * (nspan + nsub) * sizeof(SplitBest));
    best = (SplitBest *)arena_get(ctx, "sp_best", (size_t)nsub * F * sizeof(SplitBest));
    if (!sums || !pieces || !best) return MH_ENOMEM;
    const uint32_t blocks = xcd_grid((F * nspan + 3) / 4);
    k_split_class_sums<<<blocks, 256, 0, st>>>(o.el, M, F, K, nspan, o.co, sums);
    MH_LAUNCHED(ctx, "k_split_class_sums");
    if (mh_status s = row_scan(ctx, sums, F * K, nspan)) return s;
    if (gini)
      k_split_eval<true><<<blocks, 256, 0, st>>>(o.el, M, F, K, nspan, nsub, o.co, o.plan.seg,
                                                 o.plan.cum, tot, sums, pieces);
    else
      k_split_eval<false><<<blocks, 256, 0, st>>>(o.el, M, F, K, nspan, nsub, o.co, o.plan.seg,
                                                  o.plan.cum, tot, sums, pieces);
    MH_LAUNCHED(ctx, "k_split_eval");
    k_split_best<<<(nsub * F + 3) / 4, 256, 0, st>>>(pieces, F, nspan, nsub, o.plan.seg, best);
    MH_LAUNCHED(ctx, "k_split_best");
  }
  k_split_final<<<(nsub + 3) / 4, 256, 0, st>>>(tot, nsub, K, F, gini ? 1u : 0u, best, feat, tau,
                                                correct);
  MH_LAUNCHED(ctx, "k_split_final");
  return MH_OK;
}

// The order for the next level, whose 2 nsub subsets have the totals tot2:
// each run partitioned by the new locations.
mh_status order_partition(Ctx *ctx, SplitOrder &o, uint32_t nsub, const uint32_t *loc,
                          const uint32_t *tot2) {
  if (!o.M) return MH_OK;
  hipStream_t st = ctx->stream;
  const uint32_t M = o.M, F = o.F, nspan = o.nspan;
  uint64_t *bits = (uint64_t *)arena_get(ctx, "sp_bits", (size_t)F * nspan * SP_ROUNDS * 8);
  uint32_t *lsum = (uint32_t *)arena_get(ctx, "sp_lsum", (size_t)F * nspan * 4);
  if (!bits || !lsum) return MH_ENOMEM;
  mh_status s = order_plan(ctx, o, o.plan2, tot2, 2 * nsub);
  if (s) return s;
  const uint32_t blocks = xcd_grid((F * nspan + 3) / 4);
  k_part_count<<<blocks, 256, 0, st>>>(o.el, M, F, nspan, loc, bits, lsum);
  MH_LAUNCHED(ctx, "k_part_count");
  s = row_scan(ctx, lsum, F, nspan);
  if (s) return s;
  k_part_move<<<blocks, 256, 0, st>>>(o.el, o.alt, M, F, nspan, nsub, o.plan.seg, o.plan2.seg,
                                      o.plan2.even, bits, lsum);
  MH_LAUNCHED(ctx, "k_part_move");
  std::swap(o.el, o.alt);
  std::swap(o.plan, o.plan2);
  return MH_OK;
}

// Limits of a split over nsub subsets.
mh_status check_split(Ctx *ctx, const mh_dataset *ds, uint32_t nsub) {
  uint32_t fbits = 1, sbits = 0;
  while ((1u << fbits) < ds->F) ++fbits;
  while (sbits < 32 && (1ull << sbits) < nsub) ++sbits;
  if (fbits + sbits > 31) return fail(ctx, MH_EINVAL, "too many subsets for split1");
  if (ds->n > RANGE_MAX_N) return fail(ctx, MH_EINVAL, "too many samples for split1");
  return MH_OK;
}

}  // namespace

mh_status launch_split1(Ctx *ctx, const mh_dataset *ds, const uint32_t *sub_of, uint32_t nsub,
                        const uint32_t *tot, uint8_t *feat, uint32_t *tau, uint32_t *correct) {
  mh_status s = check_split(ctx, ds, nsub);
  if (s || nsub == 0) return s;
  SplitOrder o;
  s = order_build(ctx, ds, sub_of, nsub, nsub, o);
  if (!s) s = order_plan(ctx, o, o.plan, tot, nsub);
  if (!s) s = order_eval(ctx, o, tot, nsub, false, feat, tau, correct);
  return s;
}

mh_status cart_batched(Ctx *ctx, const mh_dataset *ds, const uint32_t *sub_of, uint32_t nsub,
                       uint32_t D, uint8_t *feat, uint32_t *tau) {
  hipStream_t st = ctx->stream;
  const uint32_t n = ds->n, K = ds->K, SB = (1u << D) - 1u;
  if (nsub == 0) return MH_OK;
  const size_t maxq = (size_t)nsub << (D - 1);
  if (maxq > 0xFFFFFFFFull / 2) return fail(ctx, MH_EINVAL, "CART: too many subsets");
  mh_status s = check_split(ctx, ds, (uint32_t)maxq);
  if (s) return s;
  uint32_t *loc = (uint32_t *)arena_get(ctx, "ct_loc", (size_t)(n ? n : 1) * 4);
  uint32_t *sub_l = (uint32_t *)arena_get(ctx, "ct_sub", (size_t)(n ? n : 1) * 4);
  uint32_t *hist = (uint32_t *)arena_get(ctx, "ct_hist", maxq * K * 4);
  uint8_t *fl = (uint8_t *)arena_get(ctx, "ct_f", maxq);
  uint32_t *tl = (uint32_t *)arena_get(ctx, "ct_t", maxq * 4);
  if (!loc || !sub_l || !hist || !fl || !tl) return MH_ENOMEM;
  if (n) {
    s = launch_fill(ctx, loc, n, 1u);
    if (s) return s;
  }
  SplitOrder o;
  s = order_build(ctx, ds, sub_of, nsub, (uint32_t)maxq, o);
  if (s) return s;
  for (uint32_t l = 0; l < D; ++l) {
    const uint32_t cnt = nsub << l;
    s = launch_zero(ctx, {{hist, (size_t)cnt * K * 4}});
    if (s) return s;
    if (n) {
      k_cart_sub<<<nblk(n), 256, 0, st>>>(sub_of, n, nsub, loc, l, sub_l);
      MH_LAUNCHED(ctx, "k_cart_sub");
      s = launch_level_hist(ctx, sub_l, ds->labels, n, K, 0, cnt, hist);
      if (s) return s;
    }
    s = l == 0 ? order_plan(ctx, o, o.plan, hist, cnt) : order_partition(ctx, o, cnt / 2, loc, hist);
    if (!s) s = order_eval(ctx, o, hist, cnt, true, fl, tl, nullptr);
    if (s) return s;
    k_cart_put<<<nblk(cnt), 256, 0, st>>>(fl, tl, cnt, l, SB, feat, tau);
    MH_LAUNCHED(ctx, "k_cart_put");
    if (l + 1 < D && n) {
      k_cart_route<<<nblk(n), 256, 0, st>>>(sub_of, n, nsub, loc, l, fl, tl, ds->ranks, ds->ld,
                                            ds->F);
      MH_LAUNCHED(ctx, "k_cart_route");
    }
  }
  return MH_OK;
}

mh_status cart_subset(Ctx *ctx, const mh_dataset *ds, const uint32_t *idx, uint32_t n_sub,
                      uint32_t D, uint8_t *feat, uint32_t *tau) {
  hipStream_t st = ctx->stream;
  const uint32_t n = ds->n, SB = (1u << D) - 1u;
  uint32_t *sub_of = (uint32_t *)arena_get(ctx, "s1_sub_of", (size_t)(n ? n : 1) * 4);
  uint32_t *tot = (uint32_t *)arena_get(ctx, "s1_tot", (size_t)ds->K * 4);
  uint8_t *f = (uint8_t *)arena_get(ctx, "ct_tree_f", SB);
  uint32_t *t = (uint32_t *)arena_get(ctx, "ct_tree_t", (size_t)SB * 4);
  if (!sub_of || !tot || !f || !t) return MH_ENOMEM;
  MH_HIP(ctx, hipMemsetAsync(tot, 0, (size_t)ds->K * 4, st));
  if (n)
    if (mh_status s = launch_fill(ctx, sub_of, n, 1u)) return s;
  if (n_sub) {
    k_mark_subset<<<nblk(n_sub), 256, 0, st>>>(idx, n_sub, n, ds->labels, ds->K, sub_of, tot);
    MH_LAUNCHED(ctx, "k_mark_subset");
  }
  mh_status s = cart_batched(ctx, ds, sub_of, 1, D, f, t);
  if (s) return s;
  MH_HIP(ctx, hipMemcpyAsync(feat, f, SB, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(tau, t, (size_t)SB * 4, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipStreamSynchronize(st));
  return MH_OK;
}

mh_status split1_subset(Ctx *ctx, const mh_dataset *ds, const uint32_t *idx, uint32_t n_sub,
                        uint8_t *feat, uint32_t *tau, uint32_t *correct) {
  hipStream_t st = ctx->stream;
  const uint32_t n = ds->n;
  uint32_t *sub_of = (uint32_t *)arena_get(ctx, "s1_sub_of", (size_t)(n ? n : 1) * 4);
  uint32_t *tot = (uint32_t *)arena_get(ctx, "s1_tot", (size_t)ds->K * 4);
  uint8_t *f = (uint8_t *)arena_get(ctx, "s1_f", 256);
  uint32_t *t = (uint32_t *)arena_get(ctx, "s1_t", 256);
  uint32_t *c = (uint32_t *)arena_get(ctx, "s1_c", 256);
  if (!sub_of || !tot || !f || !t || !c) return MH_ENOMEM;
  MH_HIP(ctx, hipMemsetAsync(tot, 0, (size_t)ds->K * 4, st));
  if (n)
    if (mh_status s = launch_fill(ctx, sub_of, n, 1u)) return s;
  if (n_sub) {
    k_mark_subset<<<nblk(n_sub), 256, 0, st>>>(idx, n_sub, n, ds->labels, ds->K, sub_of, tot);
    MH_LAUNCHED(ctx, "k_mark_subset");
  }
  mh_status s = launch_split1(ctx, ds, sub_of, 1, tot, f, t, c);
  if (s) return s;
  MH_HIP(ctx, hipMemcpyAsync(feat, f, 1, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(tau, t, 4, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(correct, c, 4, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipStreamSynchronize(st));
  return MH_OK;
}

}  // namespace mh
