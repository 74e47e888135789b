// How domains are split into the work items of the two-step kernel
// (lbm_two_step.hpp) and of the tile kernel (lbm_tile_steps.hpp), and whether
// those kernels are the faster ones for them.  Host code without GPU calls.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "lbm_params.hpp"

namespace rmrt {

struct SweepPlan {
  uint32_t cx = 0, cy = 0, cz = 0;   // inner columns of a patch, planes of a chunk
  uint32_t w = 0;                    // patch width, ring included
  double us = 1e300;                 // estimated time of a pass
};

// Time of one plane of one patch, in GPU clocks of a workgroup that has a CU
// to itself: about 7 per cache line and population stream that a row of the
// patch touches (a load or store of a wave that spans several rows or starts
// inside a line touches more of them), plus the collision of every thread's
// column, about 1/3 clock per column and population (half as much again in
// FP64).  On 256 x 256 x 128 (us per plane visit, estimated / measured):
// rD3Q19 FP32 whole rows 8.4 / 8.0, rD3Q27 FP32 7.6 / 6.4, rD3Q19 FP64 in
// patches of 64 columns 13.0 / 12.9.
inline double plane_clocks(double row_lines, double ring_lines, uint32_t cy, uint32_t columns, int q, int es) {
  const double lines = (row_lines + ring_lines) * (cy + 2) + (row_lines + 0.75 * ring_lines) * cy;
  return q * (7.0 * lines + (es == 8 ? 0.5 : 0.33) * columns);
}

// The split with the shortest pass for workgroups of `columns` columns, one
// per CU.  A patch of cx x cy inner columns takes (cx + 2)(cy + 2), or
// nx (cy + 2) when it spans x; a chunk of cz planes collides cz + 2 and starts
// its stores a plane late, hence the cz + 3 visits.
inline SweepPlan plan_sweep(uint32_t nx, uint32_t ny, uint32_t nz, int q, int es, uint32_t columns, uint32_t cus) {
  SweepPlan best;
  for (uint32_t ntx = 1; ntx <= nx; ++ntx) {
    const uint32_t cx = (nx + ntx - 1) / ntx;
    if ((uint64_t)(ntx - 1) * cx >= nx) continue;   // the same width as a smaller count
    if (ntx > 1 && cx * es < 64) break;             // rows of less than half a cache line
    const uint32_t w = ntx == 1 ? nx : cx + 2;
    const uint32_t rows = columns / w;
    if (rows < 3) continue;
    uint32_t nty = (ny + std::min(ny, rows - 2) - 1) / std::min(ny, rows - 2), cy = (ny + nty - 1) / nty;
    // the kernel's spare threads need three entries past the patch
    if (columns > w * (cy + 2) && columns - w * (cy + 2) < 3) {
      if (cy < 2) continue;
      cy -= 1;
      nty = (ny + cy - 1) / cy;
    }
    // whole rows lie end to end in memory; others start anywhere in a line
    const double row = cx * es / 128.0 + ((ntx > 1 && (cx * es) % 128 != 0) ? 1.0 : 0.0);
    const double clocks = plane_clocks(row, ntx == 1 ? 0.0 : 2.0, cy, columns, q, es);
    for (uint32_t ntz = 1; ntz <= nz; ++ntz) {
      const uint32_t cz = (nz + ntz - 1) / ntz;
      if ((uint64_t)(ntz - 1) * cz >= nz) continue;
      const uint64_t items = (uint64_t)ntx * nty * ntz, rounds = (items + cus - 1) / cus;
      const double us = (double)rounds * (cz + 3.0) * clocks / 2400.0;   // 2.4 GHz
      if (us < best.us) best = SweepPlan{cx, cy, cz, w, us};
      if (items > 4ull * cus) break;
    }
  }
  return best;
}

// Is the pass faster than two single steps (which move 2 q es bytes a node
// each at about 6.3 TB/s, after about 2.5 us of launch and ramp)?  The
// estimate above is an upper one (most measured passes take 0.8 - 0.95 of
// it), and where the two come close the single steps stay: they need no second
// buffer.  Measured single / two-step, us a step: rD3Q19 FP32 64^3 12.9 /
// 11.4 and 40 x 150 x 90 16.2 / 16.9 (not taken), 128 x 128 x 96 40 / 28,
// 160^3 111 / 74, 256 x 256 x 128 196.5 / 135; rD3Q27 FP32 223 x 116 x 100
// 89.7 / 92.2 (not taken), 512 x 128 x 64 147 / 127, 192^3 258 / 163; rD3Q19
// FP64 128 x 128 x 96 85 / 62, 256 x 256 x 128 449 / 303.  Of 240 random sizes
// of 2.5e5 to 8e6 nodes 130 are taken, at 0.62 to 0.98 of their single steps.
inline bool sweep_pays(const SweepPlan& p, uint64_t nodes, int q, int es) {
  const double single = (double)nodes * 2.0 * q * es / 6.3e6 + 2.5;
  return 0.85 * p.us < 0.9 * 2.0 * single;
}

// The items of a plan, in the order the workgroups take them.  Workgroups are
// dealt round-robin to the eight XCDs: each XCD gets a contiguous run of
// patches, so that their rings share its L2.
inline std::vector<SweepItem> sweep_items(const SweepPlan& p, uint32_t nx, uint32_t ny, uint32_t nz) {
  std::vector<SweepItem> list;
  for (uint32_t z = 0; z < nz; z += p.cz)
    for (uint32_t y = 0; y < ny; y += p.cy)
      for (uint32_t x = 0; x < nx; x += p.cx)
        list.push_back(SweepItem{x, std::min(p.cx, nx - x), y, std::min(p.cy, ny - y), z, std::min(p.cz, nz - z)});
  const size_t n = list.size(), q8 = n / 8, rem = n % 8;
  std::vector<SweepItem> out(n);
  for (size_t b = 0; b < n; ++b) {
    const size_t xcd = b % 8, first = xcd * q8 + std::min(xcd, rem);
    out[b] = list[first + b / 8];
  }
  return out;
}

// ---------------------------------------------------------------------------
// Tiles of several steps (rD2Q9)
// ---------------------------------------------------------------------------
struct TileSplit {
  uint32_t cx = 0, cy = 0, w = 0;   // inner nodes of a tile, width with the ring
  uint64_t tiles = ~0ull;
};

// The split of an nx x ny domain into the fewest tiles of at most `nodes`
// nodes, ring included (a tile over the whole of x has none there).
inline TileSplit split_tiles(uint32_t nx, uint32_t ny, uint32_t nodes, uint32_t ring) {
  TileSplit best;
  for (uint32_t ntx = 1; ntx <= nx; ++ntx) {
    const uint32_t cx = (nx + ntx - 1) / ntx;
    if ((uint64_t)(ntx - 1) * cx >= nx) continue;
    const uint32_t w = ntx == 1 ? nx : cx + 2 * ring;
    if (ntx > 1 && cx < 8) break;
    const uint32_t rows = nodes / w;
    if (rows < 2 * ring + 1) continue;
    const uint32_t cymax = std::min(ny, rows - 2 * ring), nty = (ny + cymax - 1) / cymax;
    const uint64_t tiles = (uint64_t)ntx * nty;
    if (tiles < best.tiles) best = TileSplit{cx, (ny + nty - 1) / nty, w, tiles};
  }
  return best;
}

// What the time of a step on rD2Q9 depends on besides the sizes: the storage,
// walls or solid nodes, solid masks (link words), constant sources, a batch.
struct TileKind {
  int es = 4;
  bool bounded = false, links = false, sourced = false, batch = false;
};

// Time of a pass of `tiles` tiles of up to `blocks` nodes per thread and `steps`
// steps on `cus` CUs (us): a launch, and per round of the workgroups that run at
// once (two on a CU, one of 512 threads in FP64) their first loads, then each
// thread's nodes; the last round is half paid for however few tiles it has, and
// where each workgroup has a CU to itself it is the shorter.  Two buffers that
// the 256 MB memory-side cache does not hold bound short passes (3.2 TB/s).
// Fitted to 650 measured passes of 3 and 4 steps (32 x 32 .. 2048 x 2048 nodes,
// single domains and batches), 90% of them within 13%; estimated / measured, 4 steps: FP32
// 2048 x 1024 54 / 49, with walls and force 78 / 67, 256 x 256 8.4 / 7.4, 64 x 32
// 5.9 / 5.7; FP64 2048 x 1024 116 / 120, 64 x 32 6.2 / 5.8.
inline double tile_pass_us(const TileKind& k, uint64_t nodes, uint64_t tiles, uint32_t blocks, uint32_t cus,
                           uint32_t threads, uint32_t steps) {
  const bool alone = k.es == 8 && threads > 256;
  const double x = (double)tiles / (alone ? cus : 2.0 * cus);
  double rounds = std::max(1.0, 0.5 * (x + std::ceil(x)));
  if (!alone && tiles <= cus) rounds = 0.65;
  double us;
  if (k.es == 4)
    us = 3.0 + rounds * (0.8 + blocks * (1.1 + steps * (0.63 + (k.bounded ? 0.28 : 0.0) + (k.sourced ? 0.19 : 0.0))));
  else if (!alone)
    us = 2.8 + rounds * (0.85 + blocks * (0.83 + steps * (0.64 + (k.bounded ? 0.16 : 0.0))));
  else
    us = rounds * (3.2 + blocks * (1.5 + steps * (0.66 + (k.bounded ? 0.13 : 0.0))));
  const double mb = nodes * 18.0 * k.es / 1e6;
  return mb > 256.0 ? std::max(us, mb / 3.2) : us;
}

// Time of a single step (us): a replayed launch and the bytes at the rate of the
// memory-side cache, which falls from 9.6 TB/s as the state outgrows it (most
// estimates within 10%; estimated / measured: FP32 64 x 32 2.4 / 2.4, 512 x 512
// 4.4 / 4.2, 2048 x 1024 19.7 / 20.8; FP64 2048 x 1024 43 / 42, 2048 x 2048 97 / 99).
inline double single_step_us(const TileKind& k, uint64_t nodes) {
  const double mb = nodes * 18.0 * k.es / 1e6;
  double us = 2.4 + mb / 9.6 + std::max(0.0, mb - 100.0) * (k.es == 4 ? 0.03 : 0.045);
  us += std::max(0.0, mb - 400.0) * 0.045;
  if (k.links)
    us *= k.es == 4 ? 1.2 : 1.14;
  else if (k.es == 4)
    us *= 1.0 + (k.bounded ? 0.04 : 0.0) + (k.sourced ? 0.05 : 0.0);
  return k.batch ? us + std::min(3.2, nodes / 8e4) : us;
}

// The passes that the tiles of a context can take, and single steps, by their
// estimated time (us).  A pass loads and exchanges its ring however few steps it
// takes: us a step, single / passes of four, three and two: FP32 700 x 700 6.3 /
// 4.7, 5.3, 6.5, 1500 x 700 10.2 / 8.1, 9.2, 11.6, with walls and force 11.4 / 11.0,
// 12.5, 15.9; a batch of 30 of 64 x 48 6.5 / 2.8, 3.3, 3.9.  The shorter the pass,
// the larger its share that the estimate may be wrong by: passes of four are
// taken up to 1.05 of their single steps, of three below 0.96, of two below 0.87
// (or where launches are all there is, with a tile of one node per thread on each
// CU: calls of four steps 17.7 against 19.6 us).
struct TileRule {
  double pass[5] = {}, single = 0.0;   // a pass of 2 .. 4 steps, weighted as above; a single step
};
inline TileRule tile_rule(const TileKind& k, uint64_t tiles, uint32_t blocks, uint32_t cus, uint32_t threads,
                          uint64_t nodes) {
  TileRule r;
  r.single = single_step_us(k, nodes);
  const double weight[5] = {0.0, 0.0, 1.15, 1.04, 0.95};
  for (uint32_t n = 2; n <= 4; ++n) r.pass[n] = weight[n] * tile_pass_us(k, nodes, tiles, blocks, cus, threads, n);
  if (blocks == 1 && tiles <= cus) r.pass[2] = std::min(r.pass[2], 1.9 * r.single);
  return r;
}

// The passes of a call that takes m (even) steps on the tile path: an even number
// of each length, so that the state ends in the buffer where single steps would
// leave it; single steps for what is left.  Of the splits with up to four passes
// of three and two of two the one with the shortest estimated time.
struct TileCall {
  int fours = 0, threes = 0, twos = 0;
  int passes() const { return fours + threes + twos; }
  int steps() const { return 4 * fours + 3 * threes + 2 * twos; }
  int pass_steps(int k) const { return k < fours ? 4 : k < fours + threes ? 3 : 2; }
};
inline TileCall tile_call(const TileRule& r, int m) {
  TileCall best;
  double best_us = m * r.single;
  for (int threes = 0; threes <= 4; threes += 2)
    for (int twos = 0; twos <= 2; twos += 2) {
      TileCall c;
      c.threes = threes;
      c.twos = twos;
      if (c.steps() > m) continue;
      if (r.pass[4] < 4.0 * r.single) c.fours = (m - c.steps()) / 8 * 2;
      const double us = c.fours * r.pass[4] + threes * r.pass[3] + twos * r.pass[2] + (m - c.steps()) * r.single;
      if (us < best_us) {
        best_us = us;
        best = c;
      }
    }
  return best;
}

// How much longer a split may be estimated and still be preferred for each node
// per thread that its tiles have more than another's: larger tiles have less ring
// (700 x 700 FP32, 4 nodes per thread 18.7 us a pass, estimated 18.3; 2 nodes
// 19.8, estimated 17.9).
constexpr double kTileSizeBias = 0.02;

}  // namespace rmrt
