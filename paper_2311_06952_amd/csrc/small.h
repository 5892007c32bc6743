// small.h -- data sets small enough that one block holds a whole feature (or a
// whole problem's sample list): their preparation in one launch.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "internal.h"

namespace mh {

// The most samples of a small data set (a feature's keys and 16-bit sample
// numbers in one block's LDS, 22 per thread).
constexpr uint32_t SMALL_MAX_N = 22u * 1024u;

// One data set; only the fields of the parts asked for are read.
struct SmallJob {
  TileHdr hdr;            // PREP_PLAN: the layout
  const float *X;         // PREP_RANK: [n][F]
  const uint8_t *labels;  // PREP_PLAN
  const uint32_t *idx;    // PREP_PLAN: the subset's samples (null: all)
  uint32_t *ranks, *n_unique, *nan;  // PREP_RANK out ([F][ld], [F], flag to or into)
  void *tiles;            // PREP_PLAN out
  double *pop;            // PREP_INIT out, gene-major
  uint64_t seed, prob;
  uint32_t n, F, K, ld;
  uint32_t n_sub, P, SB, pad;
};
enum { PREP_RANK = 1u, PREP_PLAN = 2u, PREP_INIT = 4u };

// The parts `what` of every job in one launch: the ranks of each feature (a
// block sorts it in LDS), the tile plan and sample lists (the layout without
// its sorted records), the initial population.  jobs_dev: the jobs on the
// device (null for one job, which travels as the kernel's argument).
mh_status launch_prep_small(Ctx *ctx, const std::vector<SmallJob> &jobs, const SmallJob *jobs_dev,
                            uint32_t what);
// The sorted records of every job's planned layout.
mh_status launch_tile_sort_small(Ctx *ctx, const std::vector<SmallJob> &jobs,
                                 const SmallJob *jobs_dev);

// A served run's result: the buffers it is packed from and where it goes.
struct PackJob {
  const uint8_t *f1, *lab1;
  const uint32_t *t1, *corr1, *flag_a, *flag_b;
  const double *cost1;
  ResultOut *out;
  uint32_t D, pad;
};
mh_status launch_pack_jobs(Ctx *ctx, const PackJob *jobs_dev, uint32_t n);

}  // namespace mh
