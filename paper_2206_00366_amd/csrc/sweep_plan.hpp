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
// 11.4 and 40 x 150 x 90 16.2 / 16.9 (not taken), 128 x 128 x 96 37.9 / 27.7,
// 160^3 111 / 72, 256 x 256 x 128 196.5 / 133; rD3Q27 FP32 512 x 128 x 64
// 146 / 152 and 223 x 116 x 100 89.7 / 92.2 (not taken), 192^3 258 / 183;
// rD3Q19 FP64 128 x 128 x 96 78.8 / 60.9, 256 x 256 x 128 449 / 303.
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

// Time of a pass of `tiles` tiles of up to `blocks` nodes per thread and `steps`
// steps with `slots` workgroups at once (us): a launch, and per round the first
// loads, then each thread's nodes.  rD2Q9 FP32 with 512 threads, FP64 with 256
// or 512; estimated / measured: FP32 2048 x 1024 58.5 / 57, 256 x 256 6.9 / 8.2,
// FP64 2048 x 1024 (512 threads) 128 / 121, 64 x 32 (256 threads) 7.0 / 6.5.
inline double tile_pass_us(uint64_t tiles, uint32_t blocks, uint32_t slots, int es, uint32_t threads, uint32_t steps) {
  const double rounds = (double)((tiles + slots - 1) / slots);
  const double load = es == 8 && threads <= 256 ? 0.8 : 0.9, step = es == 4 ? 0.75 : threads <= 256 ? 0.8 : 1.0;
  return 1.5 + rounds * (1.5 + blocks * (load + steps * step));
}
// Is a pass faster than the single steps it stands for?  Those take a replayed
// launch and their bytes at the rate of the memory-side cache (FP32 64 x 32 2.7
// us, 512 x 512 4.5, 2048 x 1024 21; FP64 2048 x 1024 42).
inline bool tiles_pay(double pass_us, uint64_t nodes, int es, uint32_t steps) {
  const double single = 2.5 + (double)nodes * 18.0 * es / 8.4e6;
  return pass_us < 0.9 * steps * single;
}

}  // namespace rmrt
