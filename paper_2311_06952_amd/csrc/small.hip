// small.hip -- preparation of small data sets, one launch for any number of
// them.
//
// A data set of up to SMALL_MAX_N samples is bound by launches and barriers,
// not by its bytes: the cooperative rank encoding passes nine grid barriers
// and the tile build six launches of a few microseconds each.  Here a block
// sorts a whole feature in LDS (no exchange between blocks) and another plans
// the tiles and lists their samples, so that the blocks of all features of all
// data sets run side by side.  Measured at n = 1000, F = 4: ranks 29.6 -> 11.7
// us, tile build 20 us in six launches -> 9.5 in two (the initial population
// included); 10 to 20 served requests of up to 2 10^4 samples: 65 us each, one
// after another -> 100 us together.
#include <algorithm>

#include "device_common.h"
#include "internal.h"
#include "small.h"
#include "tile_sort.h"

namespace mh {
namespace {

constexpr uint32_t SM_THREADS = 1024, SM_WAVES = SM_THREADS / 64;

// Exclusive scan of one value per thread over the block; *total receives the
// sum.  s_w: SM_WAVES words of LDS.
__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t *s_w, uint32_t *total) {
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) s_w[w] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (uint32_t q = 0; q < SM_WAVES; ++q) {
    const uint32_t t = s_w[q];
    before += q < w ? t : 0u;
    all += t;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

__host__ __device__ __forceinline__ uint32_t rank_small_lds(uint32_t n) {
  return SM_WAVES * 256 * 4 + SM_WAVES * 4 + n * 6 + 64;
}

// Dense ranks of feature f: four stable LSD radix passes of 8 bits over the
// order-preserving value bits.  Wave w holds positions [w S, (w + 1) S) in
// registers, 64 at a time; a pass counts its digits per wave, turns the counts
// into slots (digit-major, then wave), and writes every pair to its slot (the
// pairs of a wave with the same digit numbered by ballot match); the pairs
// sit in registers between read and write, so one LDS copy suffices.
template <int E>
__device__ __forceinline__ void rank_body(const __attribute__((address_space(4))) SmallJob *jb,
                                          uint32_t f, uint8_t *lds) {
  const uint32_t n = jb->n, F = jb->F;
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  uint32_t *wc = reinterpret_cast<uint32_t *>(lds);  // [SM_WAVES][256]
  uint32_t *s_w = wc + SM_WAVES * 256;
  uint32_t *key = s_w + SM_WAVES;
  uint16_t *id = reinterpret_cast<uint16_t *>(key + n);
  const uint32_t p0 = w * (E * 64u) + lane;  // position of round k: p0 + 64 k
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t kv[E], iv[E];
  bool nan = false;
  const float *X = jb->X;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    // (past the end the last row again, unused: the loads carry no branch)
    iv[k] = min(p0 + 64u * k, n - 1u);
    kv[k] = __float_as_uint(X[(size_t)iv[k] * F + f]);
  }
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const uint32_t u = kv[k];
    nan |= (u & 0x7FFFFFFFu) > 0x7F800000u;
    const uint32_t z = (u << 1) == 0u ? 0u : u;  // -0 == +0
    kv[k] = (z & 0x80000000u) ? ~z : (z | 0x80000000u);
  }
  if (__ballot(nan) && lane == 0) atomicOr(jb->nan, 1u);
#pragma unroll 1
  for (uint32_t pass = 0; pass < 4; ++pass) {
    const uint32_t shift = 8 * pass;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) wc[w * 256 + q * 64 + lane] = 0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < E; ++k)
      if (p0 + 64u * k < n) atomicAdd(&wc[w * 256 + ((kv[k] >> shift) & 0xFFu)], 1u);
    __syncthreads();
    {
      // thread d < 256: digit d's slots, wave by wave
      uint32_t tot = 0, all;
      if (threadIdx.x < 256)
        for (uint32_t q = 0; q < SM_WAVES; ++q) tot += wc[q * 256 + threadIdx.x];
      uint32_t run = block_exscan(tot, s_w, &all);
      if (threadIdx.x < 256)
        for (uint32_t q = 0; q < SM_WAVES; ++q) {
          const uint32_t c = wc[q * 256 + threadIdx.x];
          wc[q * 256 + threadIdx.x] = run;
          run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < E; ++k) {
      // (one round's ballots at a time: hoisted together they would spill)
      asm volatile("" : "+v"(kv[k])::"memory");
      const bool valid = p0 + 64u * k < n;
      const uint32_t d = (kv[k] >> shift) & 0xFFu;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (uint32_t bit = 0; bit < 8; ++bit) {
        const bool on = (d >> bit) & 1u;
        const uint64_t bal = __ballot(on);
        peers &= on ? bal : ~bal;
      }
      const uint32_t below = (uint32_t)__popcll(peers & lt);
      const uint32_t slot = valid ? wc[w * 256 + d] : 0u;
      __builtin_amdgcn_wave_barrier();
      if (valid) {
        key[slot + below] = kv[k];
        id[slot + below] = (uint16_t)iv[k];
        if (below == 0) wc[w * 256 + d] = slot + (uint32_t)__popcll(peers);
      }
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const uint32_t p = p0 + 64u * k;
      if (p < n) {
        kv[k] = key[p];
        iv[k] = id[p];
      }
    }
    __syncthreads();
  }
  // ranks: the starts of new values up to a position, minus one
  uint32_t loc[E], starts = 0;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    loc[k] = 0;
    const uint32_t p = p0 + 64u * k;
    const bool start = p < n && (p == 0 || key[p - 1] != kv[k]);
    const uint64_t b = __ballot(start);
    loc[k] = starts + (uint32_t)__popcll(b & lt) + (start ? 1u : 0u);
    starts += (uint32_t)__popcll(b);
  }
  uint32_t total;
  const uint32_t mine = block_exscan(lane == 0 ? starts : 0u, s_w, &total);
  const uint32_t base = __shfl(mine, 0, 64);
  uint32_t *rk = jb->ranks + (size_t)f * jb->ld;
#pragma unroll
  for (int k = 0; k < E; ++k)
    if (p0 + 64u * k < n) rk[iv[k]] = base + loc[k] - 1u;
  if (threadIdx.x == 0) jb->n_unique[f] = total;
}

// The tile plan of one data set (the header, class totals, segment offsets and
// info words) and the samples of every tile.  Lanes of a wave with the same
// label add once (few classes: adds of a whole wave to one word serialise).
__device__ __forceinline__ void plan_body(const __attribute__((address_space(4))) SmallJob *jb,
                                          uint8_t *lds) {
  uint32_t *h = reinterpret_cast<uint32_t *>(lds);  // [256] counts, then cursors
  uint32_t *off = h + 256;                          // [257] first tile of a class
  uint32_t *s_w = off + 257;
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  const uint32_t n_sub = jb->n_sub, n = jb->n, K = jb->K;
  uint8_t *base = reinterpret_cast<uint8_t *>(jb->tiles);
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  // sample j's index and class (K: invalid input, left out)
  auto label_of = [&](uint32_t j, uint32_t &i) {
    i = 0;
    if (j >= n_sub) return K;
    i = jb->idx ? jb->idx[j] : j;
    if (i >= n) return K;
    const uint32_t y = jb->labels[i];
    return y < K ? y : K;
  };
  // h[y] += 1 for every valid lane; returns the lane's number in its class
  auto add = [&](uint32_t y) {
    uint64_t pending = __ballot(y < K);
    uint32_t pos = 0;
    while (pending) {
      const int leader = __builtin_ctzll(pending);
      const uint32_t yl = (uint32_t)__builtin_amdgcn_readlane((int)y, leader);
      const uint64_t same = __ballot(y == yl);
      uint32_t b = 0;
      if (lane == (uint32_t)leader) b = atomicAdd(&h[yl], (uint32_t)__popcll(same));
      b = (uint32_t)__builtin_amdgcn_readlane((int)b, leader);
      if (y == yl) pos = b + (uint32_t)__popcll(same & lt);
      pending &= ~same;
    }
    return pos;
  };
  // (whole waves take part in every round)
  const uint32_t rounds = (n_sub + SM_THREADS - 1) / SM_THREADS;
  for (uint32_t q = 0; q < rounds; ++q) {
    uint32_t i;
    (void)add(label_of(q * SM_THREADS + threadIdx.x, i));
  }
  __syncthreads();
  uint32_t *ctot = reinterpret_cast<uint32_t *>(base + jb->hdr.off_ctot);
  uint32_t *segoff = reinterpret_cast<uint32_t *>(base + jb->hdr.off_segoff);
  uint32_t *cursor = reinterpret_cast<uint32_t *>(base + jb->hdr.off_cursor);
  uint32_t *info = reinterpret_cast<uint32_t *>(base + jb->hdr.off_info);
  uint32_t *order = reinterpret_cast<uint32_t *>(base + jb->hdr.off_order);
  const uint32_t c = threadIdx.x < K ? h[threadIdx.x] : 0u;
  uint32_t n_tiles;
  const uint32_t t0 = block_exscan((c + TILE_CAP - 1) / TILE_CAP, s_w, &n_tiles);
  if (threadIdx.x < K) {
    ctot[threadIdx.x] = c;
    segoff[threadIdx.x] = t0;
    cursor[threadIdx.x] = 0;
    off[threadIdx.x] = t0;
  }
  if (threadIdx.x == 0) {
    segoff[K] = n_tiles;
    off[K] = n_tiles;
  }
  if (threadIdx.x < 64) {
    // the header, with the tile count
    const __attribute__((address_space(4))) uint32_t *src =
        (const __attribute__((address_space(4))) uint32_t *)&jb->hdr;
    uint32_t v = src[threadIdx.x];
    if (threadIdx.x == offsetof(TileHdr, n_tiles) / 4) v = n_tiles;
    reinterpret_cast<uint32_t *>(base)[threadIdx.x] = v;
  }
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < n_tiles; t += SM_THREADS) {
    uint32_t lo = 0, hi = K;  // the last class whose tiles start at or before t
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (off[mid] <= t) lo = mid;
      else hi = mid;
    }
    info[t] = (lo << 8) | min(TILE_CAP, h[lo] - (t - off[lo]) * TILE_CAP);
  }
  __syncthreads();
  if (threadIdx.x < 256) h[threadIdx.x] = 0;  // cursors
  __syncthreads();
  for (uint32_t q = 0; q < rounds; ++q) {
    uint32_t i;
    const uint32_t y = label_of(q * SM_THREADS + threadIdx.x, i);
    const uint32_t pos = add(y);
    if (y < K) order[(off[y] + pos / TILE_CAP) * TILE_W + pos % TILE_CAP] = i;
  }
}

// The initial population (k_de_init's draws), gene-major.
__device__ __forceinline__ void init_body(const __attribute__((address_space(4))) SmallJob *jb) {
  const uint32_t P = jb->P, SB = jb->SB, m = 2 * SB;
  const uint64_t key = de_key(jb->seed, jb->prob);
  const double Fp1 = (double)jb->F + 1.0;
  for (uint32_t e = threadIdx.x; e < P * m; e += SM_THREADS) {
    const uint32_t q = e / P, r = e % P;
    const double u = to_unit(de_draw(key, 0, r, q));
    jb->pop[e] = q < SB ? __dmul_rn(u, Fp1) : u;
  }
}

// Block (x, job): feature x while ranks are wanted (x < x_rank), then the
// plan, then the population.
template <bool RANK>
__global__ __launch_bounds__(SM_THREADS) void k_prep_small(SmallJob one,
                                                           const SmallJob *__restrict__ jobs,
                                                           uint32_t what, uint32_t x_rank) {
  extern __shared__ __align__(16) uint8_t lds[];
  typedef const __attribute__((address_space(4))) SmallJob *JobPtr;
  const JobPtr jb = jobs ? (JobPtr)(uintptr_t)(jobs + blockIdx.y)
                         : (JobPtr)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t x = blockIdx.x;
  if (x < x_rank) {
    if constexpr (RANK) {
      if (x >= jb->F) return;
      // rounds of 1,024 samples by the block's own data set
      const uint32_t e = (jb->n + SM_THREADS - 1) / SM_THREADS;
      if (e <= 1) rank_body<1>(jb, x, lds);
      else if (e <= 2) rank_body<2>(jb, x, lds);
      else if (e <= 4) rank_body<4>(jb, x, lds);
      else if (e <= 8) rank_body<8>(jb, x, lds);
      else if (e <= 14) rank_body<14>(jb, x, lds);
      else rank_body<22>(jb, x, lds);
    }
    return;
  }
  x -= x_rank;
  if (what & PREP_PLAN) {
    if (x == 0) {
      plan_body(jb, lds);
      return;
    }
    x -= 1;
  }
  if (x == 0) init_body(jb);
}

__global__ __launch_bounds__(256) void k_tile_sort_jobs(SmallJob one,
                                                        const SmallJob *__restrict__ jobs) {
  typedef const __attribute__((address_space(4))) SmallJob *JobPtr;
  const JobPtr jb = jobs ? (JobPtr)(uintptr_t)(jobs + blockIdx.y)
                         : (JobPtr)__builtin_amdgcn_kernarg_segment_ptr();
  tile_sort_body<uint32_t>(jb->ranks, jb->ld, reinterpret_cast<TileHdr *>(jb->tiles), blockIdx.x);
}

__global__ __launch_bounds__(64) void k_pack_jobs(const PackJob *__restrict__ jobs) {
  const PackJob j = jobs[blockIdx.x];
  const uint32_t SB = (1u << j.D) - 1u, SL = 1u << j.D;
  for (uint32_t i = threadIdx.x; i < SL; i += 64u) {
    if (i < SB) {
      j.out->tree.feat[i] = j.f1[i];
      j.out->tree.tau[i] = j.t1[i];
    }
    j.out->tree.label[i] = j.lab1[i];
  }
  if (threadIdx.x == 0) {
    j.out->tree.D = j.D;
    j.out->tree.correct = *j.corr1;
    j.out->tree.cost = *j.cost1;
    j.out->flag = (*j.flag_a ? 1u : 0u) | (*j.flag_b << 1);
  }
}

}  // namespace

mh_status launch_prep_small(Ctx *ctx, const std::vector<SmallJob> &jobs, const SmallJob *jobs_dev,
                            uint32_t what) {
  uint32_t n = 0, F = 0;
  for (const SmallJob &j : jobs) {
    if (j.n > SMALL_MAX_N && (what & PREP_RANK)) return fail(ctx, MH_EINVAL, "not a small data set");
    n = std::max(n, j.n);
    F = std::max(F, j.F);
  }
  const uint32_t x_rank = (what & PREP_RANK) ? F : 0u;
  const dim3 grid(x_rank + ((what & PREP_PLAN) ? 1u : 0u) + ((what & PREP_INIT) ? 1u : 0u),
                  (uint32_t)jobs.size());
  const size_t lds = std::max<size_t>(x_rank ? rank_small_lds(n) : 0, (256 + 257 + 16) * 4);
  hipStream_t st = ctx->stream;
  if (x_rank)
    k_prep_small<true><<<grid, SM_THREADS, lds, st>>>(jobs[0], jobs_dev, what, x_rank);
  else
    k_prep_small<false><<<grid, SM_THREADS, lds, st>>>(jobs[0], jobs_dev, what, x_rank);
  MH_LAUNCHED(ctx, "k_prep_small");
  return MH_OK;
}

mh_status launch_tile_sort_small(Ctx *ctx, const std::vector<SmallJob> &jobs,
                                 const SmallJob *jobs_dev) {
  uint32_t blocks = 0;
  for (const SmallJob &j : jobs)
    blocks = std::max(blocks, tile_sort_blocks(j.hdr.max_tiles, j.F));
  k_tile_sort_jobs<<<dim3(blocks, (uint32_t)jobs.size()), 256, 0, ctx->stream>>>(jobs[0], jobs_dev);
  MH_LAUNCHED(ctx, "k_tile_sort_jobs");
  return MH_OK;
}

mh_status launch_pack_jobs(Ctx *ctx, const PackJob *jobs_dev, uint32_t n) {
  k_pack_jobs<<<n, 64, 0, ctx->stream>>>(jobs_dev);
  MH_LAUNCHED(ctx, "k_pack_jobs");
  return MH_OK;
}

}  // namespace mh
