// How the work of a launch is split, from sizes alone (host code without HIP).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace f4 {

// The leaf blocks of one mesh in a launch.
struct BlockSet {
  int N;           // cells per block and axis
  int64_t blocks;
};

// Work items of the plane-marching stage kernel: blocks per workgroup (8 x 8
// tiles share one) and tiles per block plane, in 2D and 3D.
constexpr int stage_blocks_per_item(int N) { return N == 8 ? 4 : 1; }
constexpr int stage_tiles_per_block(int N) { return N == 32 ? 4 : 1; }
inline int64_t stage_items(int ndim, int N, int64_t nb, int ks) {
  const int64_t tiles = nb * stage_tiles_per_block(N), per = stage_blocks_per_item(N);
  return ((tiles + per - 1) / per) * (ndim == 3 ? ks : 1);
}

// Planes per work item of a MUSCL stage launch over the given meshes (3D): a
// tile is split along z into slabs of a power of two of planes where whole
// tiles leave CUs idle or end in a nearly empty round.  A launch of I items
// puts n = ceil(I / CUs) on a CU; S of them run at once (by registers and
// LDS), and a round of r <= S items takes about (r + 1.25 S) / (2.25 S) of a
// full one, because few waves wait more on their own chains.  An item costs
// its planes plus two (the planes around a slab are loaded and converted
// again).  The least of rounds x planes is taken; where block sizes are mixed, of
// the mean item's, plus what the longest exceeds it by (38,540 blocks of 8^3, 16^3
// and 32^3: 14.1 ms a step whole*, 14.6 with 16 planes per item).  Measured, two
// Heun steps in us by planes per item (the choice marked): FP32 180 blocks of
// 16^3: 163 (16), 126 (8), 102 (4)*, 105 (2); 512: 190 (16), 152 (8)*, 173 (4);
// 720: 211 (16)*, 219 (8); 80 blocks of 32^3: 327 (32), 219 (16)*, 218 (8),
// 235 (4); one: 275 (32), 52 (1)*; 512 of 8^3: 96 (8), 82 (4), 85 (2)*; FP64 180
// of 16^3: 210 (16), 176 (8)*, 188 (4); 27 of 32^3: 212 (16), 176 (8)*, 208 (4);
// 512 of 8^3: 136 (8), 95 (4)*, 127 (2).
inline int slab_planes(const BlockSet *sets, size_t n_sets, bool f64, int n_cu) {
  int largest = 0, smallest = 64;
  for (size_t i = 0; i < n_sets; i++) {
    largest = std::max(largest, sets[i].N);
    smallest = std::min(smallest, sets[i].N);
  }
  const bool mixed = smallest != largest;
  const int at_once = f64 ? (smallest == 8 || mixed ? 1 : 2) : (smallest == 8 || mixed ? 3 : 4);
  int best = largest;
  double best_cost = 0.0;
  for (int kd = largest; kd >= 1; kd /= 2) {
    int64_t items = 0, planes = 0;
    for (size_t i = 0; i < n_sets; i++) {
      const int N = sets[i].N;
      const int64_t it = stage_items(3, N, sets[i].blocks, std::max(1, N / kd));
      items += it;
      planes += it * (std::min(N, kd) + 2);
    }
    const int64_t n = (items + n_cu - 1) / n_cu, full = n / at_once, rest = n % at_once;
    const double rounds = (double)full + (rest ? (rest + 1.25 * at_once) / (2.25 * at_once) : 0.0);
    const double mean = items ? (double)planes / items : 0.0;
    const double cost = rounds * mean + (kd + 2 - mean);
    if (kd == largest || cost < best_cost) {
      best = kd;
      best_cost = cost;
    }
  }
  return best;
}

// k-slabs per tile of a mesh in a batch (3D): as configured, at least 8 planes
// each, or where nothing is configured (0) the model's depth.
inline int batch_slabs(int configured, int N, int planes) {
  return configured > 0 ? std::min(configured, N / 8) : std::max(1, N / planes);
}

// Planes per workgroup of a WENO5 stage launch (3D): a tile's whole depth, or
// slabs of it (halved as long as needed) where whole tiles leave CUs without
// work.  A slab converts six more planes of its columns and reconstructs two
// more cells of each.  The line lies at three workgroups of 256 threads a CU,
// where a second one no longer pays, and at four of one wave: 80 blocks of 32^3
// (320 tiles), FP32, 256 CUs, two Heun steps: 701 us whole, 404 us in 4 slabs,
// 464 us in 16; 512 blocks of 16^3: 381, 322 (2 slabs), 374 us (8); 512 of 8^3:
// 156, 107 (2), 135 us (8); one 32^3 block: 527 and 54 us (32 slabs).
inline int weno_planes(int64_t nblocks, int N, int n_cu) {
  const int ts = N == 8 ? 8 : 16;
  const int64_t tiles = nblocks * (N / ts) * (N / ts), fill = (ts == 8 ? 4 : 3) * (int64_t)n_cu;
  int kd = N;
  while (kd > 1 && tiles * (N / kd) < fill) kd /= 2;
  return kd;
}

// log2 of the slabs per block of a scalar advection launch (3D): a block per
// workgroup, or slabs of its planes (halved as long as needed) where whole
// blocks leave CUs without waves to hide their loads behind: up to two
// workgroups of 256 threads a CU, one of 64.  256 CUs, two Heun steps, van Leer,
// us: FP32 180 blocks of 16^3 61 whole, 48; 27 of 32^3 132 and 46; 80 of 32^3
// 135 and 86 (100 with twice as many); one of 32^3 124 and 29; 512 of 8^3 49 and
// 59; FP64 WENO5 80 of 32^3 462 and 248.
inline int advect_log2_slabs(int64_t nblocks, int N, int n_cu) {
  const int64_t threads = N * N, want = (N == 8 ? 64 : 512) * (int64_t)n_cu;
  int ls = 0;
  while ((N >> ls) > 1 && ((nblocks * threads) << ls) < want) ls++;
  return ls;
}

// Workgroups per record of a ghost round: a record's elements take several
// rounds of one workgroup (an FP64 16^3 prolongation: ten), each as long as a
// load from memory.  Launches of few records take more workgroups per record, up
// to eight per CU in all.  The walls of 225 16^2 columns (450 records): 14.6 us
// with one workgroup each, 11.7 us; what is left is the launch and four
// dependent loads.
inline int ghost_split(int64_t records, int64_t face_values, int n_cu) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((face_values + 511) / 512, 8 * (int64_t)n_cu / records));
}

}  // namespace f4
