// Stress kernels (sampled path stress, exact path stress, differentiable loss)
// and the utility kernels of stress_kernels.hip: launch arguments and launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace pgsgd {

constexpr uint32_t kStreamSpsSlot = 6;  // Philox stream of the window-major sampled path stress slots
constexpr uint32_t kStreamLossSlot = 7; // Philox stream of the window-major loss slots

struct StressLaunch {
  const StepRec* rec;
  const float* coords;
  const float2* work;      // interleaved copy of coords (sampled path stress only)
  const uint32_t* inv;     // renumbered graph: caller id of every device node id (else NULL)
  const float2* work2;     // not NULL: the SPS of two layouts on the same pairs, whose copy work and work2 hold
                           // (k_to_work_pair)
  const uint64_t* path_off;
  const uint32_t* zipf;
  const uint16_t* guide;
  uint64_t n_nodes;
  uint64_t S;
  uint64_t count;          // steps (SPS) or pairs (loss)
  uint32_t m;              // SPS pairs per step
  uint32_t n_paths;
  uint32_t path_slots;
  uint32_t path_top;
  uint32_t W;
  uint32_t word2;          // counter word 2
  uint32_t c3;
  uint32_t k0, k1;
  // the sampled path stress, when out_count is set: pairs with stress
  // above out_threshold are appended (i, j, e_i | e_j << 1, stress; the first
  // out_max kept) and counted in *out_count
  uint64_t* out_count;
  uint64_t out_max;
  double out_threshold;
  uint64_t* out_i;
  uint64_t* out_j;
  uint8_t* out_e;
  double* out_s;
};

constexpr uint32_t kStressBlocks = 2048;
constexpr uint32_t kStressThreads = 256;
// Grids of the sampled path stress, full occupancy each: 2 sums of two doubles
// per block (one layout) or 5 (two layouts), within the 3 * kStressBlocks
// doubles of partials that a graph holds.
constexpr uint32_t kSpsBlocks = 1024, kSpsThreads = 512;
constexpr uint32_t kSpsPairBlocks = 512, kSpsPairThreads = 1024;
// Chunks of a step's m pairs so that a small graph still has a pair for every
// thread of the grid: as many as it takes (S >= 1, m >= 1), no more threads
// than the grid has; chunk c holds the pairs [c * per, min(m, (c + 1) * per)).
// In 64 bits: m may be any 32-bit number.
struct SpsSplit {
  uint32_t per, chunks;
};
inline SpsSplit sps_split(uint64_t S, uint32_t m, uint64_t threads) {
  const uint64_t want = S >= threads ? 1 : std::max<uint64_t>(1, std::min<uint64_t>(m, threads / S));
  const uint64_t per = (m + want - 1) / want;
  return {(uint32_t)per, (uint32_t)((m + per - 1) / per)};
}
static_assert(4 * kSpsBlocks <= 3 * kStressBlocks && 10 * kSpsPairBlocks <= 3 * kStressBlocks, "partials");
// The sums of one evaluation on the host: hi + lo of the sums of a, a^2 and, for
// two layouts, b, b^2, a b; the valid and skipped pairs; the outliers found.
struct SpsHostSums {
  double hi[5], lo[5];
  uint64_t n[2];
  uint64_t outliers;
};
hipError_t launch_sps(const StressLaunch& P, int mode, double* part_f, uint64_t* part_n, uint64_t* part_skip,
                      uint32_t* n_parts, hipStream_t s);
hipError_t launch_reduce_sps(const StressLaunch& P, const double* part_f, const uint64_t* part_n,
                             const uint64_t* part_skip, uint32_t n_parts, SpsHostSums* out, hipStream_t s);
// out_f[0] = sum of part_f; out_n[0] = sum of part_n; loss_out[0] their ratio.
hipError_t launch_reduce_parts(const double* part_f, const uint64_t* part_n, uint32_t n_parts, double* out_f,
                               uint64_t* out_n, float* loss_out, uint64_t* n_valid_out, hipStream_t s);
// Sampled path stress in window-major order: segments (the windows of
// 2^win_shift steps cut at path boundaries, in step order) get the counts of
// the plain pair draws that fall in them; each segment's slots draw their pair
// inside it.  Runs: XCD x takes the segments [sbeg[x], sbeg[x + 1]).
struct SpsWinLaunch {
  StressLaunch P;             // rec, work, path_off, S, m, path table, c3 of the plain pair draws, key
  uint32_t slot_c3;           // Philox word 3 of the slot draws
  uint32_t win_shift;
  uint32_t n_seg;
  uint32_t xstride;           // row length of xitem
  uint32_t count_blocks;
  const uint64_t* seg_start;  // [n_seg + 1], seg_start[n_seg] = S
  const uint32_t* seg_path;   // [n_seg]
  const uint32_t* path_extra; // [n_paths] a path's first segment less the window it starts in
  uint32_t* count;            // [n_seg] histogram (zeroed again by the scan)
  uint64_t* seg_off;          // [n_seg + 1] first slot of every segment
  const uint32_t* sbeg;       // [kXcds + 1] first segment of every run
  uint64_t* xitem;            // [kXcds][xstride] prefix of 64-slot items over the segments of each run
  uint64_t* queue;            // [2][kXcds][16] item counters of the loss's passes or the SPS (zeroed by the scan)
  uint64_t loss_pairs;        // the loss's window-major pairs (reading R22): the number of plain pairs; 0 = SPS
};
// runs: also the runs' item prefixes and counters, which the passes by tiles do not read
hipError_t launch_sps_win_count_scan(const SpsWinLaunch& W, bool runs, hipStream_t s);
hipError_t launch_sps_win(const SpsWinLaunch& W, double* part_f, uint64_t* part_n, uint64_t* part_skip,
                          uint32_t* n_parts, hipStream_t s);
// The loss (reading R22) over the segments' slots counted with loss_pairs:
// forward per-block sums (grid: blocks a multiple of kXcds), and the adjoint
// added into the planar gradient.
hipError_t launch_loss_win_fwd(const SpsWinLaunch& W, double* part_f, uint64_t* part_n, uint32_t blocks,
                               hipStream_t s);
hipError_t launch_loss_win_bwd(const SpsWinLaunch& W, const float* grad_out, const uint64_t* n_valid, float* grad,
                               uint32_t blocks, hipStream_t s);
// The loss by tiles: tile t covers the segments seg[off[t] .. off[t + 1]) (at
// most kTileMaxSeg), whose lowest device node ids lie in kTileNodes ids from
// base[t] on, and keeps the endpoints of up to kTileRange ids from base[t] on in
// LDS: their coordinates, and in the adjoint an image of their gradient, flushed
// with one atomic add per touched entry; other endpoints are read and added
// directly.  Block b starts with unit b and takes the others from *queue.  The
// pairs are the window-major loss pairs of W, the same slots as
// launch_loss_win_bwd.
//
// A segment's steps climb through up to ~2,000 ids, so what lies above the range
// grows fast once the range is less than that beyond a tile's last start: over
// 1e7 pairs the adjoint with 3,072 ids in LDS takes 207 us with tiles of 1,024
// ids, 227 with 1,536 and 321 with 2,048; tiles of 512 zero and flush twice as
// many images (253).
constexpr uint32_t kTileNodes = 1024;
constexpr uint32_t kTileRange = 4096;
constexpr uint32_t kTileMaxSeg = 256;    // a segment's number in its tile is a byte of k_loss_tile's guide
constexpr uint32_t kTileGuide = 1024;
constexpr uint32_t kTileThreads = 1024;
constexpr uint32_t kTileDone = 32;
// The forms of k_loss_tile (see there).
enum TileForm { kTileFwd, kTileFwdStaged, kTileBwd32, kTileBwd64, kTileBwd64Staged };
constexpr bool tile_grad(TileForm f) { return f != kTileFwd && f != kTileFwdStaged; }
constexpr bool tile_double(TileForm f) { return f == kTileBwd64 || f == kTileBwd64Staged; }
constexpr bool tile_staged(TileForm f) { return f == kTileFwdStaged || f == kTileBwd64Staged; }
// Blocks of 16 waves that a CU holds: the images of the gradient leave room for one.
constexpr uint32_t tile_blocks(TileForm f) { return tile_grad(f) ? 1 : 2; }
struct TileLaunch {
  const uint32_t* seg;
  const uint32_t* off;
  const uint32_t* base;
  uint32_t n_tiles;
  uint32_t split;  // parts of a tile's pairs, a unit of work each
  TileForm form;
  uint32_t entries;  // loss_tile_entries
  uint32_t* queue;   // [0] the next unit, [kTileDone] the blocks that have taken their last; both 0 between launches
  const float* planes;  // the caller's coordinates, read in place; NULL: the working copy
};
// Parts of a tile.  A gradient unit zeroes and flushes the tile's whole image,
// so its tiles stay whole while they fill the blocks; below that (and in the
// forward pass, which has no image) a tile is cut until the blocks have `rounds`
// units each, with at least one pair for every thread.  Forward over 1e7 pairs
// with 1, 2 and 4 units a block: 172, 161 and 165 us.
inline uint32_t loss_tile_split(uint32_t n_tiles, uint32_t blocks, uint64_t n_pairs, bool grad) {
  const uint64_t rounds = grad ? 1 : 2;
  const uint64_t want = (rounds * blocks + n_tiles - 1) / std::max(1u, n_tiles);
  const uint64_t room = n_pairs / ((uint64_t)kTileThreads * std::max(1u, n_tiles));
  if (grad && n_tiles >= blocks) return 1;
  return (uint32_t)std::max<uint64_t>(1, std::min(want, room));
}
// kTileFwd*: per-block sums into part_f / part_n[0 .. blocks); kTileBwd*: the
// adjoint of grad_out added to grad.
hipError_t launch_loss_tile(const SpsWinLaunch& W, const TileLaunch& T, const float* grad_out,
                            const uint64_t* n_valid, float* grad, double* part_f, uint64_t* part_n, uint32_t blocks,
                            hipStream_t s);
// Endpoints (two a node) of a tile's range that fit beside the power-law tables
// of window W, at most 2 * kTileRange; 0 if they are too few for the form to be
// the faster one.
uint32_t loss_tile_entries(uint32_t W, TileForm form, size_t lds_limit);
constexpr size_t kTileStaticLds = 10 * 1024;  // static LDS of k_loss_tile (a tile's segment table), rounded up
// out[g] = the lowest device node id over the steps [start[g], start[g + 1])
hipError_t launch_segment_min_node(const StepRec* rec, const uint64_t* start, uint32_t nseg, uint32_t* out,
                                   hipStream_t s);
// max_path_steps, d_max: the graph's longest path in steps and in nucleotides
hipError_t launch_path_stress_exact(const StressLaunch& P, uint64_t max_path_steps, int64_t d_max, double* part_f,
                                    uint64_t* part_n, uint32_t* n_parts, hipStream_t s);
// Static LDS of k_path_stress_exact, rounded up.
constexpr size_t kExactStaticLds = 25 * 1024;
hipError_t launch_stress_fwd(const StressLaunch& P, double* part_f, uint64_t* part_n, hipStream_t s);
hipError_t launch_stress_bwd(const StressLaunch& P, const float* grad_out, const uint64_t* n_valid, float* grad,
                             hipStream_t s);
hipError_t launch_init_coords(const StepRec* rec, const uint64_t* first_step, uint64_t n_nodes, const uint32_t* inv,
                              uint32_t k0, uint32_t k1, uint32_t c3, float jitter, float* coords, hipStream_t s);
hipError_t launch_first_visit(const StepRec* rec, uint64_t S, uint64_t n_nodes, uint64_t* first_step,
                              hipStream_t s);
hipError_t launch_adam(float* x, const float* g, float* m, float* v, uint64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s);

}  // namespace pgsgd
