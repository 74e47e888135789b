// The split of domains into two-step work items: every node belongs to exactly
// one item, every patch fits its workgroup, every XCD gets its share.  Prints
// "ok <plans>" and exits 0.
#include <stdio.h>

#include "../../paper_2206_00366_amd/csrc/sweep_plan.hpp"

using namespace rmrt;

static int check(uint32_t nx, uint32_t ny, uint32_t nz, int q, int es, uint32_t columns, uint32_t cus) {
  const SweepPlan p = plan_sweep(nx, ny, nz, q, es, columns, cus);
  if (p.cx == 0) {   // no patch of three rows fits
    if (nx < columns / 3) return fprintf(stderr, "no plan for %u x %u x %u\n", nx, ny, nz), 1;
    return 0;
  }
  const std::vector<SweepItem> items = sweep_items(p, nx, ny, nz);
  std::vector<unsigned char> seen((size_t)nx * ny * nz, 0);
  for (const SweepItem& t : items) {
    const uint32_t w = t.cx == nx ? nx : t.cx + 2;
    if (w > p.w || (uint64_t)w * (t.cy + 2) > columns || t.cx < 1 || t.cy < 1 || t.cz < 1 || t.x0 + t.cx > nx ||
        t.y0 + t.cy > ny || t.z0 + t.cz > nz)
      return fprintf(stderr, "bad item in %u x %u x %u\n", nx, ny, nz), 1;
    const uint32_t spare = columns - w * (t.cy + 2);
    if (spare == 1 || spare == 2) return fprintf(stderr, "%u spare threads in %u x %u x %u\n", spare, nx, ny, nz), 1;
    for (uint32_t z = t.z0; z < t.z0 + t.cz; ++z)
      for (uint32_t y = t.y0; y < t.y0 + t.cy; ++y)
        for (uint32_t x = t.x0; x < t.x0 + t.cx; ++x) seen[x + (size_t)nx * (y + (size_t)ny * z)] += 1;
  }
  for (unsigned char s : seen)
    if (s != 1) return fprintf(stderr, "a node of %u x %u x %u in %d items\n", nx, ny, nz, s), 1;
  return 0;
}

static int check_tiles(uint32_t nx, uint32_t ny, uint32_t nodes, uint32_t ring) {
  const TileSplit t = split_tiles(nx, ny, nodes, ring);
  if (t.cx == 0) return 0;   // no tile fits: single steps
  uint64_t n = 0;
  std::vector<unsigned char> seen((size_t)nx * ny, 0);
  for (uint32_t y = 0; y < ny; y += t.cy)
    for (uint32_t x = 0; x < nx; x += t.cx) {
      const uint32_t cx = std::min(t.cx, nx - x), cy = std::min(t.cy, ny - y), w = cx == nx ? nx : cx + 2 * ring;
      if (w > t.w || (uint64_t)w * (cy + 2 * ring) > nodes) return fprintf(stderr, "bad tile in %u x %u\n", nx, ny), 1;
      for (uint32_t j = y; j < y + cy; ++j)
        for (uint32_t i = x; i < x + cx; ++i) seen[i + (size_t)nx * j] += 1;
      ++n;
    }
  for (unsigned char s : seen)
    if (s != 1) return fprintf(stderr, "a node of %u x %u in %d tiles\n", nx, ny, s), 1;
  return n > t.tiles;
}

int main() {
  const uint32_t sizes[] = {4, 5, 7, 16, 31, 32, 33, 64, 65, 100, 127, 223, 256, 257, 512, 513, 700, 1300};
  const struct { int q, es; uint32_t columns; } kinds[] = {{19, 4, 1536}, {19, 8, 1024}, {27, 4, 1024}};
  int bad = 0, n = 0;
  for (const auto& k : kinds)
    for (uint32_t nx : sizes)
      for (uint32_t ny : sizes)
        for (uint32_t nz : sizes) {
          if ((uint64_t)nx * ny * nz > 2000000u) continue;
          bad += check(nx, ny, nz, k.q, k.es, k.columns, 256);
          bad += check(nx, ny, nz, k.q, k.es, k.columns, 7);
          n += 2;
        }
  const uint32_t flat[] = {8, 9, 13, 64, 77, 128, 255, 256, 257, 512, 777, 1024, 2048, 5000};
  for (uint32_t nodes = 256; nodes <= 2048; nodes += 256)
    for (uint32_t nx : flat)
      for (uint32_t ny : flat) {
        bad += check_tiles(nx, ny, nodes, 4);
        ++n;
      }
  if (bad) return 1;
  printf("ok %d\n", n);
  return 0;
}
