// persist.h -- what the two whole-run DEOCT kernels (persist.hip: tiles staged
// every generation; resident.hip: tiles resident in LDS) share.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <vector>

#include "internal.h"

namespace mh {
namespace {

__host__ __device__ __forceinline__ uint32_t align16u(uint32_t x) { return (x + 15u) & ~15u; }

// (cost, index) of the wave's smallest cost, ties to the lower index: DPP
// row shifts (1, 2, 4, 8) reduce each row of 16 lanes into its last lane,
// two row broadcasts fold the four rows into lane 63, which is read back.
// A lane with no source in a step sees (infinity, the largest index), which
// never wins: an infinite cost has a lower index.
__device__ __forceinline__ void wave_argmin(double &c, uint32_t &i) {
  auto step = [&](auto ctrl_tag, auto mask_tag) {
    constexpr int ctrl = decltype(ctrl_tag)::value, rmask = decltype(mask_tag)::value;
    const uint32_t lo = (uint32_t)__double2loint(c), hi = (uint32_t)__double2hiint(c);
    const uint32_t nlo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, ctrl,
                                                               rmask, 0xF, false);
    const uint32_t nhi = (uint32_t)__builtin_amdgcn_update_dpp((int)0x7FF00000u, (int)hi, ctrl,
                                                               rmask, 0xF, false);
    const uint32_t ni = (uint32_t)__builtin_amdgcn_update_dpp((int)0xFFFFFFFFu, (int)i, ctrl,
                                                              rmask, 0xF, false);
    const double cn = __hiloint2double((int)nhi, (int)nlo);
    const bool better = (cn < c) | ((cn == c) & (ni < i));
    c = better ? cn : c;
    i = better ? ni : i;
  };
  step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});  // row_shr:1
  step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});  // row_shr:2
  step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});  // row_shr:4
  step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});  // row_shr:8
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});  // row_bcast:15
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});  // row_bcast:31
  const int lo = __builtin_amdgcn_readlane(__double2loint(c), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(c), 63);
  c = __hiloint2double(hi, lo);
  i = (uint32_t)__builtin_amdgcn_readlane((int)i, 63);
}

}  // namespace

// One run of the resident kernel.
struct RunArgs {
  const TileHdr *hdr;        // tile set; the run's tiles are [tile0, tile1)
  const uint32_t *n_unique;  // [F]
  double *pop;               // gene-major [2 SB][P]: initial population in, final out
  double *cost;              // [P] out
  uint32_t *best;            // [1] out
  uint32_t *cnt;             // 3 copies of [SB][K][Ppad], zero on entry (unused by one block)
  uint32_t *bar;             // barrier words, zero on entry
  uint32_t *err;             // non-zero after a barrier wait gave up
  // the best tree after the last generation (null out_label: not wanted):
  // nodes [SB], leaf classes [SL], correct count and cost
  uint8_t *out_feat;
  uint32_t *out_tau;
  uint8_t *out_label;
  uint32_t *out_correct;
  double *out_cost;
  double *xcost;             // [P] the costs shared out over the blocks (null: every
                             // block scores all individuals)
  double M, CR, alpha;
  uint64_t seed, prob;
  uint32_t P, G, n_min, F, K, D;
  uint32_t tile0, tile1;     // clipped to the tiles built
  uint32_t sub;              // the run's subproblem in the tile set
  uint32_t blk0, nblk;       // its blocks
  uint32_t tiles_max;        // tile slots of a block
  uint32_t slots;            // classes with an LDS counter (all K for one block)
};

// The blocks of a run with at most `tiles` tiles: nblk blocks of at most
// tiles_max tiles each, `lds` bytes and `slots` class counters; nblk 0 when
// the run does not fit the kernel.
struct RunShape {
  uint32_t nblk = 0, tiles_max = 0, slots = 0, lds = 0;
  bool split = false;  // costs shared out over the blocks (needs RunArgs::xcost)
};
// resident_shape: the number of blocks (up to max_blocks) expected to be the
// fastest, none where another form is, for at most `tiles` tiles, likely
// tiles_likely; resident_fit: nb blocks, if the run fits them; resident_cycles:
// the expected cycles of a generation.
RunShape resident_shape(const Ctx *ctx, uint32_t D, uint32_t P, uint32_t F, uint32_t K,
                        uint32_t tiles, uint32_t tiles_likely, uint32_t max_blocks);
double resident_cycles(uint32_t D, uint32_t P, uint32_t K, const RunShape &r, uint32_t tiles);
RunShape resident_fit(const Ctx *ctx, uint32_t D, uint32_t P, uint32_t F, uint32_t K,
                      uint32_t tiles, uint32_t nb);
// Launches runs of one depth and one population width (P padded to a power of
// two of waves) together: `runs` on the host, their blocks numbered from 0
// (blk0, nblk) and at most one per CU in all.  lds: the largest of their
// shapes.  runs_dev / map_dev: device room for the runs and the run of each
// block (unused for a single run).  Sets *used to false when the launch is
// refused.
mh_status launch_resident(Ctx *ctx, const std::vector<RunArgs> &runs, uint32_t lds,
                          RunArgs *runs_dev, uint32_t *map_dev, bool *used);
// Launches any number of runs of up to P_max <= 128 individuals, of any
// depths: their n_blocks blocks are numbered from 0 in the order of the runs,
// none with more than one block per CU; runs_dev and map_dev (the run of each
// block) on the device; ticket: a device word, zero on entry.
mh_status launch_resident_queue(Ctx *ctx, uint32_t P_max, uint32_t n_blocks, uint32_t lds,
                                const RunArgs *runs_dev, const uint32_t *map_dev,
                                uint32_t *ticket, bool *used);

}  // namespace mh
