// Window-major schedule: the structures shared by the host runtime and the
// kernels of local_kernels.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "internal.h"

namespace pgsgd {

constexpr uint32_t kStreamWindow = 5;       // Philox stream of the window-slot draws
constexpr uint32_t kLocalShift = 14;        // preferred window: 2^14 steps (about 1 MB of records and coordinates)
constexpr uint32_t kLocalMinWindows = 16;   // smaller windows for small graphs, down to 2^6 steps
constexpr uint32_t kLocalMaxWindows = 32768;
constexpr uint32_t kLocalStreams = 1;       // runs per XCD worked on at the same time
constexpr uint32_t kLocalMaxStreams = 16;
constexpr uint32_t kLocalGrab = 4;          // items a wave takes from its run's counter at once
// Automatic wave cap: waves <= nodes_w / 8, nodes_w ~ 2^shift * n_nodes *
// n_paths / S the node ids a window spans (an XCD's in-flight terms then
// number about as many as its window's node ids), never above the whole-graph cap.
// With the far-first update order of uniform-partner terms, layout quality on
// locality-ordered graphs is flat up to this cap.
constexpr uint64_t kLocalNodesPerWave = 8;
// In the iterations whose terms all have power-law partners (t >= n_iters /
// 2) both endpoints of every in-flight term lie in the XCD's active window, so
// lost Hogwild updates concentrate there: the automatic cap is nodes_w / 32
// (measured on a 9.9M-node, 90-path graph against the oracle's layout, on the
// same pairs of Eq. 2 at m = 3000: nodes_w / 8 left 5.3% more stress, nodes_w /
// 32 2.6%, for 0.6 s more per layout of 3.5 s).
constexpr uint64_t kLocalNodesPerWaveCooling = 32;
// Both caps stay below n_nodes / 512 waves up to this many (1.8M nodes, 32
// paths, 15 mixed iterations: 183 ms at 862 waves, 150 at 2,048, 139 at 3,000,
// 142 at 4,096; 7.2M nodes: 538 at 3,466, 544 at 4,096; the paired stress flat
// within 1%), and below n_nodes / 2048 beyond.
constexpr uint64_t kLocalMostWaves = 3584;
// Up to this many waves the iterations with uniform partners draw the next item
// while the current one's records load, as the all-cooling ones do: 15 such
// iterations on 51K / 342K / 985K nodes took 5.9 / 42.8 / 70.8 ms without and
// 4.8 / 35.0 / 60.7 with (500 to 1,900 waves); from about 3,500 waves on their
// far lines fill the fabric and it is slower (2.7M nodes: 167.9 and 173.0 ms,
// 7.2M: 437 and 448).  Graphs below kManyWaveNodes keep their pace.
constexpr uint64_t kLocalAheadWaves = 3072;
constexpr uint64_t kLocalEarlyWaves = 512;    // cap of the first eighth of the iterations below 1M nodes

// log2 of the window length for S steps: 2^14, halved while there would be
// fewer than 16 windows (not below 2^6), doubled while there would be more
// than 32768.  Part of the sampling definition (the slot draws depend on it).
inline uint32_t window_shift(uint64_t S) {
  auto n = [&](uint32_t sh) { return (S + (1ull << sh) - 1) >> sh; };
  uint32_t sh = kLocalShift;
  while (sh > 6 && n(sh) < kLocalMinWindows) --sh;
  while (n(sh) > kLocalMaxWindows) ++sh;
  return sh;
}

// Automatic cap of a whole graph.  One wave keeps the sampled path stress of the
// sequential loop on a 2.6K-node graph and two waves raise it by 12%, but what
// counts there are the XCDs: each works on its own L2's copy of the coordinates
// until the launch ends.  On 51K nodes the stress is 1.0 / 1.23 / 1.33 / 1.45 of
// one wave's on 1 / 2 / 4 / 8 XCDs, and with 24 paths within 0.5% from 24 to
// 1,024 waves while the time falls as 1 / waves (240 ms at 24, 10.5 at 780).  So
// below kManyWaveNodes the cap is n_nodes / 2048 waves, one or two per XCD, whose
// runs repeat to about 3e-4 of the coordinates (one wave: exactly) where more
// waves would move the layout by 1e-3, and at 16 and 17 blocks, whose XCDs share
// evenly, raise the stress: to 1.055 times on average over nine graphs of 33K to
// 36.6K nodes and 8 to 40 paths (1.00 to 1.17; 240 ms at 16 waves, 8.7 at 520),
// against 1.015 over seven of 37K to 41K.  From there on n_nodes / 64 waves up to
// 1,024, and where that is more n_nodes / 512 up to kLocalMostWaves, and
// n_nodes / 2048.
//
// With few paths a node has few updates an iteration, in few windows, to make
// up for the lost ones, and the waves that leave the stress alone fall with the
// steps: S / 512, S / 1024 and S / 2048 waves had 1.13 / 1.05 / 1.00 times the
// stress of n_nodes / 2048 on one path over 84K nodes (n_nodes / 64: 1.25), 1.13
// / 1.05 / 1.00 on four over 48K (1.15), 1.17 / 1.11 / 1.02 on six over 86K
// (1.17), and n_nodes / 64 had 1.00 to 1.04 on twelve over 83K in four runs.  So
// the cap is S / 2048 waves up to seven steps a node (eleven paths), rising with
// the fourth power of the steps a node beyond (sixteen paths: S / 560), and
// never below n_nodes / 2048.  It costs the six paths 24.6 ms for 6.0 (131 at
// n_nodes / 2048).
//
// In the plain order every term reads the whole graph and 512 waves are as many
// as the fabric serves: 157K / 326K nodes 21.0 / 45.5 ms at 512 and 21.1 / 46.3
// at 1,024 with 1.013 / 1.003 and 1.031 / 1.008 times the stress of n_nodes /
// 2048; 85K nodes 13.9 and 13.3 ms, 1.026 and 1.052.  Few paths take (S / 1500)
// waves a step of a node: one path over 84K nodes 1.02 times the stress, four
// over 70K at 450 waves 1.01 (at 1,024: 1.05).
constexpr uint32_t kManyWaveNodes = 36864;
constexpr uint32_t kManyWaveNodesPlain = 16384;  // plain order: runs of 8 waves already differ by 6e-4 to 9e-4
inline uint64_t few_path_waves(uint64_t n, uint64_t S) {
  const double per_node = (double)S / (double)std::max<uint64_t>(n, 1);
  const double w = (double)S / 2048.0 * std::max(1.0, std::pow(per_node / 7.0, 4.0));
  return std::max<uint64_t>({1, n / 2048, (uint64_t)std::min(w, 1e15)});
}
inline uint64_t auto_inflight_waves(uint64_t n, uint64_t S) {
  if (n < kManyWaveNodes) return std::max<uint64_t>(1, n / 2048);
  const uint64_t some = std::min<uint64_t>(n / 64, 1024), most = std::min<uint64_t>(n / 512, kLocalMostWaves);
  return std::min(std::max({n / 2048, some, most}), few_path_waves(n, S));
}
inline uint64_t auto_inflight_waves_plain(uint64_t n, uint64_t S) {
  const uint64_t least = std::max<uint64_t>(1, n / 2048);
  if (n < kManyWaveNodesPlain) return least;
  const double few = (double)S / 1500.0 * ((double)S / (double)n);
  return std::max(least, std::min({n / 64, (uint64_t)512, (uint64_t)std::min(few, 1e15)}));
}

// Iterations of a layout by their launch shape: the first eighth, whose steps
// are full corrections (mu = 1 for every pair), the rest of the iterations
// with uniform partners, and the all-cooling ones (t >= n_iters / 2).
enum LocalPhase : uint32_t { kPhaseEarly = 0, kPhaseMixed, kPhaseCooling, kPhases };

inline LocalPhase local_phase(uint32_t iter, uint32_t n_iters) {
  return iter >= n_iters / 2 ? kPhaseCooling : iter < n_iters / 8 ? kPhaseEarly : kPhaseMixed;
}

// Automatic wave cap of the windowed schedule (see kLocalNodesPerWave; the
// all-cooling iterations use kLocalNodesPerWaveCooling).  A lost update of the
// first iterations moves a node by a whole correction, and the next ones do
// not bring the layout's place on the axes back: with 1,024 waves in them a
// layout of 148K nodes lands 450 nt further along x than with 72 (6.5e-4 of
// the coordinates, runs differ by 3.6e-4), with 512 or fewer it does not.
// Graphs of a batch run `scale` times n_nodes / 2048 waves in every iteration
// (scale = 0: no batch), twice that below 65,536 nodes where scale > 1.
// Several of them share each L2, and what one evicts of another's coordinates
// the other XCDs then see, so a graph's place depends on the pace of its
// neighbours: all must gain alike, and not by much.  Six graphs of 60K to 351K
// nodes took 1,080 ms at scale 1 and 475 / 270 / 195 at 2 / 4 / 8; graph by
// graph, layouts of scale 1 / 2 / 4 / 8 lie 1.1 / 1.1 / 1.3 / 1.5 times as far
// from a set of scale 1 as its own lie from each other (means over 24).  With
// the caps of single layouts (174 ms) the smallest graph lay five times as far.
// Four graphs of 33K to 59K nodes: 401 ms at n_nodes / 2048 waves, 182 at twice
// and 101 at four times that; the stress of 19 graphs in six batches is 1.003
// and 0.987 of that at n_nodes / 2048 on average (0.96 to 1.14 and 0.89 to 1.07).
constexpr uint32_t kBatchScale = 2;
constexpr uint32_t kBatchNodes = 32768;  // a batch with a smaller graph runs at scale 1

inline uint64_t auto_local_waves(uint32_t n_nodes, uint32_t n_paths, uint64_t S, LocalPhase phase, uint32_t scale) {
  const uint32_t sh = window_shift(S);
  const double nodes_w =
      std::min<double>((double)n_nodes, std::ldexp(1.0, (int)sh) * (double)n_nodes * n_paths / (double)S);
  const uint64_t per = phase == kPhaseCooling ? kLocalNodesPerWaveCooling : kLocalNodesPerWave;
  uint64_t w = (uint64_t)(nodes_w / (double)per);
  if (scale) {
    const uint64_t times = scale > 1 && n_nodes < 65536 ? 2 * scale : scale;
    w = std::min<uint64_t>(w, times * std::max(1u, n_nodes / 2048));
    w = std::min(w, few_path_waves(n_nodes, S));
  } else {
    w = std::min<uint64_t>(w, auto_inflight_waves(n_nodes, S));
    if (phase == kPhaseEarly) w = std::min(w, std::max<uint64_t>(n_nodes / 2048, kLocalEarlyWaves));
  }
  return std::max<uint64_t>(1, w);
}

// Grids of k_layout_local: the in-flight wave cap (params.max_inflight_waves,
// automatic: auto_local_waves) and the waves that the device holds give the
// waves, which no phase exceeds; 256-thread blocks in a multiple of 8 (one
// share per XCD), or 64-thread blocks below 32 waves.  Automatic caps of graphs
// of fewer than 65,536 nodes keep the proportion between the XCDs that n_nodes /
// 2048 one-wave blocks have (21 blocks: three on XCDs 0..4, two on 5..7), so
// that the same XCDs end their shares last: an XCD writes its copy of the
// coordinates back when it is done, and the last one's stand.  With equal XCDs a
// layout of 44.5K nodes lay 2e-3 to 3e-3 away (runs differ by 3e-4), with the
// proportion kept 6e-4.  Caps below four waves for each of those blocks (few
// paths, or paths that revisit nodes; batches) keep it with 64-thread blocks.
struct LocalGrids {
  uint32_t blocks[kPhases], threads[kPhases];
  uint32_t quota_hi[kPhases], quota_lo[kPhases], hi_xcds[kPhases];  // blocks of an XCD's share that take work
  bool ahead[kPhases];  // draw the next item ahead also beside uniform partners (see kLocalAheadWaves)
};

inline LocalGrids local_grids(uint32_t n_nodes, uint32_t n_paths, uint64_t S, uint64_t max_inflight_waves,
                              uint64_t resident_waves, uint32_t scale) {
  LocalGrids out{};
  const uint32_t base = n_nodes / 2048;
  for (uint32_t ph = 0; ph < kPhases; ++ph) {
    const uint64_t cap =
        max_inflight_waves ? max_inflight_waves : auto_local_waves(n_nodes, n_paths, S, (LocalPhase)ph, scale);
    const uint64_t waves = std::max<uint64_t>(1, std::min(resident_waves, cap));
    out.ahead[ph] = !max_inflight_waves && scale != 1 && waves <= kLocalAheadWaves &&
                    n_nodes >= (scale ? kBatchNodes : kManyWaveNodes);
    out.quota_hi[ph] = out.quota_lo[ph] = 0xFFFFFFFFu;
    out.hi_xcds[ph] = kXcds;
    const bool wide = waves >= 4ull * kXcds;
    if (!max_inflight_waves && wide && base < 4 * kXcds) {
      const uint32_t block = waves >= 4ull * base ? 4 : 1;  // waves
      const uint32_t k = (uint32_t)waves / (block * base);  // blocks for one of base
      out.hi_xcds[ph] = base % kXcds;
      out.quota_lo[ph] = base / kXcds * k;
      out.quota_hi[ph] = out.quota_lo[ph] + k;
      out.threads[ph] = 64 * block;
      out.blocks[ph] = kXcds * (base % kXcds ? out.quota_hi[ph] : out.quota_lo[ph]);
      continue;
    }
    out.threads[ph] = wide ? 256 : 64;
    out.blocks[ph] = (uint32_t)(wide ? (waves / 4) / kXcds * kXcds : waves);
  }
  return out;
}

// log2 of the segment length of the loss's window-major pairs (reading R22):
// 2^10 steps, halved while there would be fewer than 16 windows (not below
// 2^6), doubled while there would be more than 32768.  Part of the loss's pair
// definition.
inline uint32_t loss_shift(uint64_t S) {
  auto n = [&](uint32_t sh) { return (S + (1ull << sh) - 1) >> sh; };
  uint32_t sh = 10;
  while (sh > 6 && n(sh) < kLocalMinWindows) --sh;
  while (n(sh) > kLocalMaxWindows) ++sh;
  return sh;
}

// One term of the ordered form: the two endpoints, their reference distance and
// the step length of the iteration; a = kNoTerm where the slot has no update.
struct alignas(16) OrderedTerm {
  uint32_t a, b;
  float d, mu;
};
constexpr uint32_t kNoTerm = 0xFFFFFFFFu;
// The ordered form of a windowed iteration that one wave runs: the terms of all
// slots first (any order, the whole chip), then one wave applies them in the
// order in which it would have drawn them.  list: 64 * ordered_items(T, n_win)
// terms.
constexpr uint32_t kOrderedChunk = 32;        // items a block stages at a time (two buffers)
constexpr uint32_t kOrderedLdsNodes = 4096;   // coordinates are held in LDS up to this many nodes
constexpr uint64_t kOrderedMaxBytes = 64u << 20;
inline uint64_t ordered_items(uint64_t n_terms, uint32_t n_win) { return n_terms / 64 + n_win; }

// Processing order: kXcds * streams runs of windows; run sigma = x * streams +
// r is stream r of XCD x and holds the windows starting in piece sigma of
// every path (paths cut into kXcds * streams equal pieces), in id order.
struct LocalLaunch {
  LayoutLaunch L;          // sampling parameters, coordinates, trace pointers (trace range in slot order)
  uint32_t n_win;          // ceil(S / 2^win_shift)
  uint32_t win_shift;
  uint32_t count_blocks;   // grid of the count kernel
  uint32_t streams;        // concurrent window streams per XCD
  uint32_t xstride;        // row length of xitem
  uint32_t ahead;          // iterations with uniform partners draw the next item ahead too
  uint32_t grab;           // items a wave takes from its stream's counter at once
  uint32_t quota_hi, quota_lo, hi_xcds;  // blocks of XCDs [0, hi_xcds) and of the others (see LocalGrids)
  uint32_t* wcount;        // [n_win] histogram (zeroed by the scan for the next iteration)
  uint64_t* woff;          // [n_win + 1] first slot of every window (window-id order)
  const uint32_t* worder;  // [n_win] windows in region order
  const uint32_t* sbeg;    // [kXcds * streams + 1] first position in worder of every run
  const uint32_t* wpath;   // [n_win] path holding the whole window, or bit 31 set if it spans paths
  uint64_t* xitem;         // [kXcds * streams][xstride] prefix of 64-slot groups over the windows of each run
  OrderedTerm* list;       // the ordered form's terms (see launch_layout_ordered), or NULL
  uint64_t* queue;         // [kXcds * streams * 16] item counters (zeroed by the scan), one per run on its own 128-byte line
};

hipError_t launch_local_count_scan(const LocalLaunch& P, hipStream_t s);
// Terms of every item into P.list, then their application by one wave.
hipError_t launch_layout_ordered(const LocalLaunch& P, hipStream_t s);
hipError_t launch_layout_local(const LocalLaunch& P, uint32_t blocks, uint32_t threads, hipStream_t s);
const void* layout_local_kernel();

}  // namespace pgsgd
