// mh.hip -- the moving-horizon driver (Algorithm 2; Section 4).
//
// The tree is grown level by level.  node_of[i] is the node sample i sits at
// (heap numbering); the subset of node t is {i : node_of[i] == t}.  Nodes of a
// level have disjoint subsets and depend only on their ancestors, so solving
// them one after another (Algorithm 2's order) or all at once gives the same
// tree: the batched form runs one multi-problem DEOCT (or one batched split)
// per level, the sequential form one per node.
#include <algorithm>
#include <cstring>
#include <vector>

#include "de_body.h"
#include "device_common.h"
#include "internal.h"
#include "range.h"

namespace mh {
namespace {

__global__ void k_fill_u32(uint32_t *__restrict__ p, uint32_t n, uint32_t v) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Class histogram of the nodes of one level: hist[(t - t0) * K + y] for
// samples with node_of in [t0, t0 + width).  Block-aggregated in LDS.
__global__ __launch_bounds__(256) void k_level_hist(const uint32_t *__restrict__ node_of,
                                                    const uint8_t *__restrict__ labels, uint32_t n,
                                                    uint32_t K, uint32_t t0, uint32_t width,
                                                    uint32_t span, uint32_t *__restrict__ hist,
                                                    int in_lds) {
  extern __shared__ uint32_t h[];
  const uint32_t cells = width * K;
  if (in_lds)
    for (uint32_t c = threadIdx.x; c < cells; c += blockDim.x) h[c] = 0;
  __syncthreads();
  const uint32_t j0 = blockIdx.x * span;
  const uint32_t j1 = (uint32_t)min((uint64_t)n, (uint64_t)j0 + span);  // no wrap near 2^32
  for (uint32_t i = j0 + threadIdx.x; i < j1; i += blockDim.x) {
    const uint32_t t = node_of[i], y = labels[i];
    if (t >= t0 && t - t0 < width && y < K) atomicAdd(in_lds ? &h[(t - t0) * K + y] : &hist[(t - t0) * K + y], 1u);
  }
  __syncthreads();
  if (in_lds)
    for (uint32_t c = threadIdx.x; c < cells; c += blockDim.x)
      if (h[c]) atomicAdd(&hist[c], h[c]);
}

// Subproblem of every sample: sub_map[t - t0] for samples at a node of the
// level, else n_problems (not in any).
__global__ void k_assign_sub(const uint32_t *__restrict__ node_of, uint32_t n, uint32_t t0,
                             uint32_t width, const uint32_t *__restrict__ sub_map,
                             uint32_t n_problems, uint32_t *__restrict__ sub_of) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t t = node_of[i];
  sub_of[i] = (t >= t0 && t - t0 < width) ? sub_map[t - t0] : n_problems;
}

// Move every sample at a node of the level to its child (Section 2: left iff
// the node splits and rank < tau; a node without a split sends all right).
__global__ void k_route_level(uint32_t *__restrict__ node_of, uint32_t n, uint32_t t0,
                              uint32_t width, const uint8_t *__restrict__ feat,
                              const uint32_t *__restrict__ tau, const uint32_t *__restrict__ ranks,
                              uint32_t ld, uint32_t F) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t t = node_of[i];
  if (t < t0 || t - t0 >= width) return;
  const uint32_t f = feat[t - 1];
  const bool left = f != 0 && f <= F && ranks[(size_t)(f - 1) * ld + i] < tau[t - 1];
  node_of[i] = left ? 2 * t : 2 * t + 1;
}

// Scatter the root node of each problem's best tree into the full tree.
__global__ void k_put_roots(const uint8_t *__restrict__ f1, const uint32_t *__restrict__ t1,
                            uint32_t SB1, const uint32_t *__restrict__ nodes, uint32_t cnt,
                            uint8_t *__restrict__ feat, uint32_t *__restrict__ tau) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= cnt) return;
  feat[nodes[s] - 1] = f1[(size_t)s * SB1];
  tau[nodes[s] - 1] = t1[(size_t)s * SB1];
}

// Samples at node t, in whatever order the block adds give (the counts of a
// subset do not depend on the order of its samples).  Block b takes the
// samples [b span, (b + 1) span) and reserves their slots with one add.
__global__ __launch_bounds__(256) void k_compact(const uint32_t *__restrict__ node_of, uint32_t n,
                                                 uint32_t t, uint32_t span,
                                                 uint32_t *__restrict__ cursor,
                                                 uint32_t *__restrict__ idx) {
  __shared__ uint32_t s_w[4], s_base;
  const uint32_t j0 = blockIdx.x * span;
  const uint32_t j1 = (uint32_t)min((uint64_t)n, (uint64_t)j0 + span);  // no wrap near 2^32
  auto in = [&](uint32_t i) { return node_of[i] == t; };
  uint32_t base = range_reserve(j0, j1, in, cursor, s_w, &s_base);
  for (uint32_t c0 = j0; c0 < j1; c0 += 256u)
    base += chunk_members(c0, j1, in, [&](uint32_t l, uint32_t i) { idx[base + l] = i; }, s_w);
}

}  // namespace

mh_status launch_fill(Ctx *ctx, uint32_t *p, uint32_t n, uint32_t v) {
  k_fill_u32<<<nblk(n), 256, 0, ctx->stream>>>(p, n, v);
  MH_LAUNCHED(ctx, "k_fill_u32");
  return MH_OK;
}

mh_status launch_level_hist(Ctx *ctx, const uint32_t *node_of, const uint8_t *labels, uint32_t n,
                            uint32_t K, uint32_t t0, uint32_t width, uint32_t *hist) {
  if (n > RANGE_MAX_N) return fail(ctx, MH_EINVAL, "too many samples for the level counts");
  const bool in_lds = (size_t)width * K * 4 <= 32768;
  // a range of samples per block (about two blocks per CU): the few cells of
  // a shallow level take a few hundred global adds each
  const uint32_t span = range_span(ctx, n);
  k_level_hist<<<range_blocks(n, span), 256, in_lds ? (size_t)width * K * 4 : 0, ctx->stream>>>(
      node_of, labels, n, K, t0, width, span, hist, in_lds ? 1 : 0);
  MH_LAUNCHED(ctx, "k_level_hist");
  return MH_OK;
}

mh_status launch_compact(Ctx *ctx, const uint32_t *node_of, uint32_t n, uint32_t t, uint32_t *idx) {
  uint32_t *cursor = (uint32_t *)arena_get(ctx, "mh_cursor", 256);
  if (!cursor) return MH_ENOMEM;
  MH_HIP(ctx, hipMemsetAsync(cursor, 0, 4, ctx->stream));
  if (n > RANGE_MAX_N) return fail(ctx, MH_EINVAL, "too many samples for the compaction");
  if (n) {
    const uint32_t span = range_span(ctx, n);
    k_compact<<<range_blocks(n, span), 256, 0, ctx->stream>>>(node_of, n, t, span, cursor, idx);
    MH_LAUNCHED(ctx, "k_compact");
  }
  return MH_OK;
}

// Multi-problem DEOCT: one tile set over all problems, one fitness launch and
// one fused epilogue + DE step (a block per problem) per generation.
mh_status deoct_batched(Ctx *ctx, const mh_dataset *ds, const uint32_t *sub_of,
                        uint32_t n_problems, const uint64_t *prob_ids, const uint64_t *host_ids,
                        uint32_t D, const mh_de_params *prm, const uint32_t *class_counts,
                        const double *warm, uint32_t W, uint8_t *feat_out, uint32_t *tau_out) {
  const uint32_t P = prm->P, SB = (1u << D) - 1u, m = 2 * SB, K = ds->K, F = ds->F;
  if (D > 5 || F > 80) return fail(ctx, MH_EINVAL, "batched DEOCT needs depth <= 5 and F <= 80");
  hipStream_t st = ctx->stream;
  TileHdr h = tile_layout(ds->n, F, K, n_problems);
  void *tiles = arena_get(ctx, "mb_tiles", h.total_bytes);
  const size_t cb = cnt_bytes(n_problems, D, K, P);
  uint32_t *cnt = (uint32_t *)arena_get(ctx, "mb_cnt", cb);
  double *pop = (double *)arena_get(ctx, "mb_pop", (size_t)n_problems * P * m * 8);
  double *trial = (double *)arena_get(ctx, "mb_trial", (size_t)n_problems * P * m * 8);
  double *cost = (double *)arena_get(ctx, "mb_cost", (size_t)n_problems * P * 8);
  uint8_t *feat = (uint8_t *)arena_get(ctx, "mb_feat", (size_t)n_problems * P * SB);
  uint32_t *tau = (uint32_t *)arena_get(ctx, "mb_tau", (size_t)n_problems * P * SB * 4);
  uint32_t *best = (uint32_t *)arena_get(ctx, "mb_best", (size_t)n_problems * 4);
  if (!tiles || !cnt || !pop || !trial || !cost || !feat || !tau || !best) return MH_ENOMEM;
  mh_status s = launch_tile_build(ctx, ds, nullptr, sub_of, ds->n, n_problems, tiles, h.total_bytes);
  if (s) return s;
  MH_HIP(ctx, hipMemsetAsync(cnt, 0, cb, st));
  const uint32_t *ctot =
      reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(tiles) + h.off_ctot);
  DeDev de{P, D, F, prm->G, prm->M, prm->CR, prm->seed, ds->n_unique, true};
  s = launch_de_init(ctx, P, D, F, prm->seed, prob_ids, 0, n_problems, warm, W, pop, true);
  if (s) return s;
  if (class_counts && ctx->persist) {
    // every problem's whole run in one cooperative launch (a block group
    // per problem)
    uint32_t *err = (uint32_t *)arena_get(ctx, "mb_err", 256);
    if (!err) return MH_ENOMEM;
    bool used = false;
    s = launch_deoct_persist_multi(ctx, tiles, F, K, ds->n, n_problems, class_counts, D, prm,
                                   prob_ids, host_ids, ds->n_unique, pop, cost, best, err, &used);
    if (s) return s;
    if (used) {
      s = launch_decode(ctx, pop, P, D, F, ds->n_unique, feat_out, tau_out, n_problems, best, true);
      if (s) return s;
      uint32_t h_err = 0;
      MH_HIP(ctx, hipMemcpyAsync(&h_err, err, 4, hipMemcpyDeviceToHost, st));
      MH_HIP(ctx, hipStreamSynchronize(st));
      if (!h_err) return MH_OK;
      // the cooperative grid did not run all at once: not again; the level
      // runs on the per-generation kernels from a fresh start
      coop_note_failure(ctx);
      MH_HIP(ctx, hipMemsetAsync(cnt, 0, cb, st));
      s = launch_de_init(ctx, P, D, F, prm->seed, prob_ids, 0, n_problems, warm, W, pop, true);
      if (s) return s;
    }
  }
  s = launch_decode(ctx, pop, P, D, F, ds->n_unique, feat, tau, n_problems, nullptr, true);
  if (s) return s;
  const bool fuse = ctx->fuse_de && fusable(P, D, F);
  uint32_t *done = (uint32_t *)arena_get(ctx, "mb_done", (size_t)n_problems * 4);
  if (!done) return MH_ENOMEM;
  MH_HIP(ctx, hipMemsetAsync(done, 0, (size_t)n_problems * 4, st));
  const uint32_t *segoff =
      reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(tiles) + h.off_segoff);
  for (uint32_t g = 0; g <= prm->G; ++g) {
    if (fuse) {
      // one launch per generation for every problem of the level: the block
      // that completes a problem's counts runs its DE step
      FuseArgs fa = make_fuse(de, prob_ids, 0, n_problems, g + 1, g == 0, pop, cost, trial, best,
                              g < prm->G ? trial : nullptr, feat, tau, cnt, ctot, K, prm->n_min,
                              prm->alpha, done, segoff);
      s = launch_fitness_count(ctx, tiles, F, K, ds->n, n_problems, h.max_tiles, feat, tau, P, D,
                               cnt, &fa);
      if (s) return s;
      continue;
    }
    s = launch_fitness_count(ctx, tiles, F, K, ds->n, n_problems, h.max_tiles, feat, tau, P, D, cnt,
                             nullptr);
    if (s) return s;
    s = launch_de_gen(ctx, de, prob_ids, 0, n_problems, g + 1, g == 0, pop, cost, trial, best,
                      g < prm->G ? trial : nullptr, feat, tau, cnt, ctot, K, prm->n_min,
                      prm->alpha);
    if (s) return s;
  }
  return launch_decode(ctx, pop, P, D, F, ds->n_unique, feat_out, tau_out, n_problems, best, true);
}

// Warm-start genes of na nodes of a level (Algorithm 2's warm-start branch):
// per node, the whole-tree run's subtree of depth De at the node (when whole
// is given; subtree node u at depth k is tree node t 2^k + u - 2^k) and then
// the node's CART subtree (cf / ct, device [na][2^De - 1], when given),
// encoded into genes (device [na][W][2 (2^De - 1)]).
static mh_status level_warm(Ctx *ctx, const mh_dataset *ds, const uint32_t *nodes, uint32_t na,
                            uint32_t D, uint32_t De, const mh_tree *whole, const uint8_t *cf,
                            const uint32_t *ct, uint32_t W, double *genes) {
  hipStream_t st = ctx->stream;
  const uint32_t SBe = (1u << De) - 1u, SB = (1u << D) - 1u;
  uint8_t *wf = (uint8_t *)arena_get(ctx, "mh_wf", (size_t)na * W * SBe);
  uint32_t *wt = (uint32_t *)arena_get(ctx, "mh_wt", (size_t)na * W * SBe * 4);
  if (!wf || !wt) return MH_ENOMEM;
  if (whole) {
    std::vector<uint8_t> hf((size_t)na * W * SBe, 0);
    std::vector<uint32_t> ht((size_t)na * W * SBe, 0);
    for (uint32_t a = 0; a < na; ++a)
      for (uint32_t u = 1; u <= SBe; ++u) {
        uint32_t k = 0;
        while ((2u << k) <= u) ++k;
        const uint64_t v = ((uint64_t)nodes[a] << k) + (u - (1u << k));
        if (v > SB) continue;
        hf[(size_t)a * W * SBe + u - 1] = whole->feat[v - 1];
        ht[(size_t)a * W * SBe + u - 1] = whole->tau[v - 1];
      }
    MH_HIP(ctx, hipMemcpyAsync(wf, hf.data(), hf.size(), hipMemcpyHostToDevice, st));
    MH_HIP(ctx, hipMemcpyAsync(wt, ht.data(), ht.size() * 4, hipMemcpyHostToDevice, st));
    MH_HIP(ctx, hipStreamSynchronize(st));  // the host vectors go out of scope
  }
  if (cf) {
    const size_t w = W - 1;
    MH_HIP(ctx, hipMemcpy2DAsync(wf + w * SBe, (size_t)W * SBe, cf, SBe, SBe, na,
                                 hipMemcpyDeviceToDevice, st));
    MH_HIP(ctx, hipMemcpy2DAsync(wt + w * SBe, (size_t)W * SBe * 4, ct, (size_t)SBe * 4,
                                 (size_t)SBe * 4, na, hipMemcpyDeviceToDevice, st));
  }
  return launch_tree_encode(ctx, wf, wt, na * W, De, ds->F, ds->n_unique, genes);
}

// Algorithm 2.  flags: MH_SEQUENTIAL or MH_BATCHED, and the warm starts
// MH_WS_CART, MH_WS_DEOCT, MH_WS_DEOCT_CART.
// solve_one(ctx, ds, node_of, t, depth, prm, warm, W, &feat, &tau): the root
// of the DEOCT subtree of node t (sequential form), warm-started with the
// device genes warm [W][2 SB].
// solve_all(ctx, ds, D, prm, warm, W, &tree): DEOCT of the whole tree on
// every sample (problem id 0).
mh_status mh_train_impl(Ctx *ctx, const mh_dataset *ds, uint32_t D, uint32_t D_MH,
                        const mh_de_params *prm, uint32_t flags, mh_tree *out,
                        SolveNodeFn solve_one, SolveAllFn solve_all) {
  hipStream_t st = ctx->stream;
  const uint32_t n = ds->n, K = ds->K, SB = (1u << D) - 1u, SL = 1u << D;
  const bool batched = (flags & MH_BATCHED) != 0;
  const bool ws_cart = (flags & MH_WS_CART) != 0, ws_deoct = (flags & MH_WS_DEOCT) != 0;
  const uint32_t W = (ws_cart ? 1u : 0u) + (ws_deoct ? 1u : 0u);
  uint32_t *node_of = (uint32_t *)arena_get(ctx, "mh_node_of", (size_t)(n ? n : 1) * 4);
  uint32_t *sub_of = (uint32_t *)arena_get(ctx, "mh_sub_of", (size_t)(n ? n : 1) * 4);
  uint8_t *tfeat = (uint8_t *)arena_get(ctx, "mh_feat", SB);
  uint32_t *ttau = (uint32_t *)arena_get(ctx, "mh_tau", (size_t)SB * 4);
  const uint32_t maxw = 1u << (D - 1);
  uint32_t *hist = (uint32_t *)arena_get(ctx, "mh_hist", (size_t)maxw * K * 4);
  uint32_t *smap = (uint32_t *)arena_get(ctx, "mh_smap", (size_t)maxw * 4);
  uint64_t *pids = (uint64_t *)arena_get(ctx, "mh_pids", (size_t)maxw * 8);
  uint32_t *nodes_d = (uint32_t *)arena_get(ctx, "mh_nodes", (size_t)maxw * 4);
  uint8_t *rf = (uint8_t *)arena_get(ctx, "mh_rf", (size_t)maxw * 31);
  uint32_t *rt = (uint32_t *)arena_get(ctx, "mh_rt", (size_t)maxw * 31 * 4);
  uint32_t *scorr = (uint32_t *)arena_get(ctx, "mh_scorr", (size_t)maxw * 4);
  uint32_t *idx = (uint32_t *)arena_get(ctx, "mh_idx", (size_t)(n ? n : 1) * 4);
  if (!node_of || !sub_of || !tfeat || !ttau || !hist || !smap || !pids || !nodes_d || !rf || !rt ||
      !scorr || !idx)
    return MH_ENOMEM;
  MH_HIP(ctx, hipMemsetAsync(tfeat, 0, SB, st));
  MH_HIP(ctx, hipMemsetAsync(ttau, 0, (size_t)SB * 4, st));
  if (n) {
    k_fill_u32<<<nblk(n), 256, 0, st>>>(node_of, n, 1u);
    MH_LAUNCHED(ctx, "k_fill_u32");
  }
  // the whole-tree DEOCT run whose subtrees warm-start the nodes
  mh_tree whole;
  if (ws_deoct) {
    const double *wg = nullptr;
    uint32_t Wd = 0;
    if (flags & MH_WS_DEOCT_CART) {
      uint8_t *cf = (uint8_t *)arena_get(ctx, "mh_cf", SB);
      uint32_t *ct = (uint32_t *)arena_get(ctx, "mh_ct", (size_t)SB * 4);
      double *g = (double *)arena_get(ctx, "mh_wgenes", (size_t)2 * SB * 8);
      if (!cf || !ct || !g) return MH_ENOMEM;
      if (n) {
        k_fill_u32<<<nblk(n), 256, 0, st>>>(sub_of, n, 0u);
        MH_LAUNCHED(ctx, "k_fill_u32");
      }
      mh_status s = cart_batched(ctx, ds, sub_of, 1, D, cf, ct);
      if (!s) s = launch_tree_encode(ctx, cf, ct, 1, D, ds->F, ds->n_unique, g);
      if (s) return s;
      wg = g;
      Wd = 1;
    }
    mh_status s = solve_all(ctx, ds, D, prm, wg, Wd, &whole);
    if (s) return s;
  }
  std::vector<uint32_t> hh((size_t)maxw * K);
  for (uint32_t L = 0; L < D; ++L) {
    const uint32_t t0 = 1u << L, width = 1u << L;
    // class histogram of the level's nodes
    MH_HIP(ctx, hipMemsetAsync(hist, 0, (size_t)width * K * 4, st));
    if (n)
      if (mh_status s = launch_level_hist(ctx, node_of, ds->labels, n, K, t0, width, hist)) return s;
    MH_HIP(ctx, hipMemcpyAsync(hh.data(), hist, (size_t)width * K * 4, hipMemcpyDeviceToHost, st));
    MH_HIP(ctx, hipStreamSynchronize(st));
    // which nodes are solved (more than n_min samples of more than one class)
    std::vector<uint32_t> active, map(width, 0xFFFFFFFFu);
    for (uint32_t w = 0; w < width; ++w) {
      uint32_t size = 0, classes = 0;
      for (uint32_t k = 0; k < K; ++k) {
        size += hh[(size_t)w * K + k];
        classes += hh[(size_t)w * K + k] ? 1u : 0u;
      }
      if (size > prm->n_min && classes > 1) {
        map[w] = (uint32_t)active.size();
        active.push_back(t0 + w);
      }
    }
    const uint32_t De = std::min(D_MH, D - L);
    const uint32_t na = (uint32_t)active.size();
    if (na > 0) {
      for (uint32_t w = 0; w < width; ++w)
        if (map[w] == 0xFFFFFFFFu) map[w] = na;
      MH_HIP(ctx, hipMemcpyAsync(smap, map.data(), (size_t)width * 4, hipMemcpyHostToDevice, st));
      MH_HIP(ctx, hipMemcpyAsync(nodes_d, active.data(), (size_t)na * 4, hipMemcpyHostToDevice, st));
      std::vector<uint64_t> pid(active.begin(), active.end());
      MH_HIP(ctx, hipMemcpyAsync(pids, pid.data(), (size_t)na * 8, hipMemcpyHostToDevice, st));
      MH_HIP(ctx, hipStreamSynchronize(st));  // map / pid host buffers are reused below
      // roots land in rf/rt with stride SB1 (batched trees) or 1 (one root)
      uint32_t SB1 = (De == 1 || !batched) ? 1u : (1u << De) - 1u;
      if (batched || De == 1) {
        k_assign_sub<<<nblk(n), 256, 0, st>>>(node_of, n, t0, width, smap, na, sub_of);
        MH_LAUNCHED(ctx, "k_assign_sub");
      }
      if (De == 1) {
        // exact split of every active node (one batched launch; the result of
        // a node does not depend on the others)
        std::vector<uint32_t> tot((size_t)na * K);
        for (uint32_t a = 0; a < na; ++a)
          for (uint32_t k = 0; k < K; ++k) tot[(size_t)a * K + k] = hh[(size_t)(active[a] - t0) * K + k];
        MH_HIP(ctx, hipMemcpyAsync(hist, tot.data(), tot.size() * 4, hipMemcpyHostToDevice, st));
        MH_HIP(ctx, hipStreamSynchronize(st));
        mh_status s = launch_split1(ctx, ds, sub_of, na, hist, rf, rt, scorr);
        if (s) return s;
      } else if (batched) {
        std::vector<uint32_t> cc((size_t)na * K);
        for (uint32_t a = 0; a < na; ++a)
          for (uint32_t k = 0; k < K; ++k) cc[(size_t)a * K + k] = hh[(size_t)(active[a] - t0) * K + k];
        const uint32_t SBe = (1u << De) - 1u;
        double *wg = nullptr;
        if (W) {
          uint8_t *cf = (uint8_t *)arena_get(ctx, "mh_cf", (size_t)na * SBe);
          uint32_t *ct = (uint32_t *)arena_get(ctx, "mh_ct", (size_t)na * SBe * 4);
          wg = (double *)arena_get(ctx, "mh_wgenes", (size_t)na * W * 2 * SBe * 8);
          if (!cf || !ct || !wg) return MH_ENOMEM;
          mh_status s = ws_cart ? cart_batched(ctx, ds, sub_of, na, De, cf, ct) : MH_OK;
          if (!s)
            s = level_warm(ctx, ds, active.data(), na, D, De, ws_deoct ? &whole : nullptr,
                           ws_cart ? cf : nullptr, ct, W, wg);
          if (s) return s;
        }
        mh_status s = deoct_batched(ctx, ds, sub_of, na, pids, pid.data(), De, prm, cc.data(), wg, W, rf, rt);
        if (s) return s;
      } else {
        std::vector<uint8_t> hf(na);
        std::vector<uint32_t> ht(na);
        const uint32_t SBe = (1u << De) - 1u;
        for (uint32_t a = 0; a < na; ++a) {
          double *wg = nullptr;
          if (W) {
            // node t's own subset (subset 0) for its CART subtree
            uint32_t *one = (uint32_t *)arena_get(ctx, "mh_smap1", 4);
            uint8_t *cf = (uint8_t *)arena_get(ctx, "mh_cf", SBe);
            uint32_t *ct = (uint32_t *)arena_get(ctx, "mh_ct", (size_t)SBe * 4);
            wg = (double *)arena_get(ctx, "mh_wgenes", (size_t)W * 2 * SBe * 8);
            if (!one || !cf || !ct || !wg) return MH_ENOMEM;
            mh_status s = MH_OK;
            if (ws_cart) {
              MH_HIP(ctx, hipMemsetAsync(one, 0, 4, st));
              if (n) {
                k_assign_sub<<<nblk(n), 256, 0, st>>>(node_of, n, active[a], 1, one, 1, sub_of);
                MH_LAUNCHED(ctx, "k_assign_sub");
              }
              s = cart_batched(ctx, ds, sub_of, 1, De, cf, ct);
            }
            if (!s)
              s = level_warm(ctx, ds, &active[a], 1, D, De, ws_deoct ? &whole : nullptr,
                             ws_cart ? cf : nullptr, ct, W, wg);
            if (s) return s;
          }
          mh_status s = solve_one(ctx, ds, node_of, active[a], De, prm, wg, W, &hf[a], &ht[a]);
          if (s) return s;
        }
        MH_HIP(ctx, hipMemcpyAsync(rf, hf.data(), na, hipMemcpyHostToDevice, st));
        MH_HIP(ctx, hipMemcpyAsync(rt, ht.data(), (size_t)na * 4, hipMemcpyHostToDevice, st));
        MH_HIP(ctx, hipStreamSynchronize(st));  // host vectors go out of scope
      }
      k_put_roots<<<nblk(na), 256, 0, st>>>(rf, rt, SB1, nodes_d, na, tfeat, ttau);
      MH_LAUNCHED(ctx, "k_put_roots");
    }
    if (L + 1 < D && n) {
      k_route_level<<<nblk(n), 256, 0, st>>>(node_of, n, t0, width, tfeat, ttau, ds->ranks, ds->ld,
                                             ds->F);
      MH_LAUNCHED(ctx, "k_route_level");
    }
  }
  // leaf classes and objective of the final tree over all training samples
  uint8_t *lab = (uint8_t *)arena_get(ctx, "mh_lab", SL);
  uint32_t *corr = (uint32_t *)arena_get(ctx, "mh_corr", 256);
  double *cst = (double *)arena_get(ctx, "mh_cost", 256);
  if (!lab || !corr || !cst) return MH_ENOMEM;
  FitnessOut fo;
  fo.label = lab;
  fo.correct = corr;
  fo.cost = cst;
  mh_status s = launch_fitness_walk(ctx, ds, nullptr, n, tfeat, ttau, 1, D, prm->n_min, prm->alpha, fo);
  if (s) return s;
  std::memset(out, 0, sizeof(*out));
  out->D = D;
  MH_HIP(ctx, hipMemcpyAsync(out->feat, tfeat, SB, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(out->tau, ttau, (size_t)SB * 4, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(out->label, lab, SL, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(&out->correct, corr, 4, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipMemcpyAsync(&out->cost, cst, 8, hipMemcpyDeviceToHost, st));
  MH_HIP(ctx, hipStreamSynchronize(st));
  return MH_OK;
}

}  // namespace mh
