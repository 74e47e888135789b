// The rules that choose between single steps and passes of several steps.
// Prints "ok" and exits 0.
#include <stdio.h>

#include "../../paper_2206_00366_amd/csrc/sweep_plan.hpp"

using namespace rmrt;

static int bad = 0;
#define CHECK(cond, ...) \
  if (!(cond)) { fprintf(stderr, __VA_ARGS__); fprintf(stderr, "\n"); bad = 1; }

// a call's passes: an even number of each length, lengths that pay, never more
// steps than asked for, and no split of the same kind that is estimated shorter
static void calls() {
  for (int mask = 0; mask < 27; ++mask) {
    TileRule r;
    r.single = 1.0;
    for (int s = 2, v = mask; s <= 4; ++s, v /= 3) r.pass[s] = s * (v % 3 == 0 ? 0.5 : v % 3 == 1 ? 0.9 : 1.2);
    for (int m = 0; m <= 256; m += 2) {
      const TileCall c = tile_call(r, m);
      CHECK(c.fours % 2 == 0 && c.threes % 2 == 0 && c.twos % 2 == 0, "an odd number of passes for %d steps", m);
      int steps = 0;
      double us = 0.0;
      for (int k = 0; k < c.passes(); ++k) {
        const int s = c.pass_steps(k);
        CHECK(s >= 2 && s <= 4 && r.pass[s] < s, "a pass of %d steps for %d (mask %d)", s, m, mask);
        steps += s;
        us += r.pass[s];
      }
      CHECK(steps == c.steps() && steps <= m && steps % 2 == 0, "%d of %d steps", steps, m);
      us += m - steps;
      if (r.pass[4] < 4) CHECK(m - steps < 8, "%d of %d steps left over", m - steps, m);
      for (int f = 0; 8 * f <= m; ++f)
        for (int t = 0; 8 * f + 6 * t <= m && t <= 2; ++t)
          for (int w = 0; 8 * f + 6 * t + 4 * w <= m && w <= 1; ++w)
            CHECK(us <= 2 * (f * r.pass[4] + t * r.pass[3] + w * r.pass[2]) + (m - 8 * f - 6 * t - 4 * w) + 1e-9,
                  "a shorter split of %d steps (mask %d)", m, mask);
    }
  }
}

// the rule of the tiles that the library chooses
static TileRule rule_of(const TileKind& k, uint32_t nx, uint32_t ny, uint32_t count) {
  double best = 1e300;
  TileRule out;
  for (uint32_t twice = 0; twice < (k.es == 8 ? 2u : 1u); ++twice)
    for (uint32_t blocks = 1; blocks <= 4; ++blocks) {
      const uint32_t nt = (k.es == 8 ? 256u : 512u) << twice;
      const TileSplit t = split_tiles(nx, ny, blocks * nt, 4);
      if (t.cx == 0) continue;
      const uint64_t nodes = (uint64_t)count * nx * ny, tiles = count * t.tiles;
      const double us = tile_pass_us(k, nodes, tiles, blocks, 256, nt, 4) * (1.0 + kTileSizeBias * (4 - blocks));
      if (us < best) {
        best = us;
        out = tile_rule(k, tiles, blocks, 256, nt, nodes);
      }
    }
  return out;
}
static bool pays(const TileKind& k, uint32_t nx, uint32_t ny, uint32_t count, uint32_t steps) {
  const TileRule r = rule_of(k, nx, ny, count);
  return r.pass[steps] < steps * r.single;
}

// measured time of passes of 4, 3 and 2 steps over that of as many single ones
// (0: not told apart from the launches); a loss of more than 4% is not taken, a
// gain of more than 40% is
static void tiles() {
  const struct { int es, bounded, links, sourced; uint32_t nx, ny; double of[5]; } rows[] = {
      {4, 0, 0, 0, 64, 32, {0, 0, 0, 0.69, 0.59}},       {4, 0, 0, 0, 700, 700, {0, 0, 1.03, 0.85, 0.74}},
      {4, 0, 0, 0, 1024, 1024, {0, 0, 1.13, 0.85, 0.74}}, {4, 0, 0, 0, 1500, 700, {0, 0, 1.14, 0.90, 0.80}},
      {4, 0, 0, 0, 2048, 1024, {0, 0, 0.86, 0.68, 0.59}}, {4, 0, 0, 0, 2048, 2048, {0, 0, 1.11, 0.67, 0.60}},
      {4, 1, 0, 1, 256, 256, {0, 0, 1.37, 1.01, 0.90}},   {4, 1, 0, 1, 700, 700, {0, 0, 1.34, 1.07, 0.96}},
      {4, 1, 0, 1, 1500, 700, {0, 0, 1.40, 1.10, 0.96}},  {4, 1, 0, 1, 100, 3000, {0, 0, 1.22, 1.00, 0.89}},
      {4, 1, 0, 1, 1024, 512, {0, 0, 1.32, 1.06, 0.95}},  {4, 1, 1, 1, 1500, 700, {0, 0, 1.19, 0.95, 0.82}},
      {4, 1, 1, 1, 64, 32, {0, 0, 0, 0.63, 0.56}},        {4, 1, 1, 1, 2048, 1024, {0, 0, 0.96, 0.76, 0.63}},
      {8, 0, 0, 0, 64, 32, {0, 0, 0, 0.57, 0.53}},           {8, 0, 0, 0, 700, 700, {0, 0, 1.16, 0.92, 0.83}},
      {8, 1, 0, 0, 700, 700, {0, 0, 1.31, 1.03, 0.89}},   {8, 1, 0, 0, 1024, 512, {0, 0, 1.19, 0.94, 0.80}},
      {8, 1, 0, 0, 2048, 1024, {0, 0, 1.11, 0.87, 0.75}}, {8, 0, 0, 0, 2048, 2048, {0, 0, 0.98, 0.73, 0.65}},
  };
  for (const auto& r : rows)
    for (uint32_t s = 2; s <= 4; ++s) {
      if (r.of[s] == 0) continue;
      TileKind k;
      k.es = r.es;
      k.bounded = r.bounded;
      k.links = r.links;
      k.sourced = r.sourced;
      const bool p = pays(k, r.nx, r.ny, 1, s);
      if (r.of[s] > 1.04) CHECK(!p, "passes of %u steps taken on %u x %u, es %d, at %.2f", s, r.nx, r.ny, r.es, r.of[s]);
      if (r.of[s] < 0.6) CHECK(p, "passes of %u steps refused on %u x %u, es %d, at %.2f", s, r.nx, r.ny, r.es, r.of[s]);
    }
  // batches of equal domains: 30 of about 64 x 48 at 0.60, 0.50 and 0.43
  TileKind k;
  k.batch = true;
  for (uint32_t s = 2; s <= 4; ++s) CHECK(pays(k, 64, 48, 30, s), "passes of %u steps refused on a batch", s);
}

// two steps per pass in 3D: single step and step of a pass, us; a gain of more than
// 20% is taken, a loss is not
static void sweeps() {
  const struct { int q, es; uint32_t nx, ny, nz; double single, two; } rows[] = {
      {19, 4, 40, 150, 90, 16.2, 16.9},    {19, 4, 128, 128, 96, 40.1, 28.3},   {19, 4, 160, 160, 160, 111.7, 74.4},
      {19, 4, 256, 256, 128, 196.5, 135.5}, {19, 4, 250, 203, 121, 155.3, 132.6}, {19, 4, 512, 140, 90, 158.6, 129.9},
      {19, 4, 340, 128, 96, 105.9, 83.6},  {27, 4, 223, 116, 100, 89.7, 92.2},  {27, 4, 512, 128, 64, 147.1, 127.4},
      {27, 4, 192, 192, 192, 258.6, 163.5}, {27, 4, 160, 160, 160, 152.3, 103.8}, {27, 4, 64, 256, 128, 70.7, 51.3},
      {27, 4, 512, 140, 90, 240.0, 186.9}, {19, 8, 128, 128, 96, 85.1, 61.6},   {19, 8, 256, 256, 128, 449.0, 303.0},
      {19, 8, 512, 128, 64, 212.7, 160.7}, {19, 8, 160, 160, 160, 211.8, 148.4}, {19, 8, 96, 96, 96, 46.6, 34.9},
  };
  for (const auto& r : rows) {
    const uint32_t columns = r.q == 27 || r.es == 8 ? 1024 : 1536;
    const SweepPlan p = plan_sweep(r.nx, r.ny, r.nz, r.q, r.es, columns, 256);
    const bool pays = sweep_pays(p, (uint64_t)r.nx * r.ny * r.nz, r.q, r.es);
    if (r.two > r.single) CHECK(!pays, "two steps per pass taken on %u x %u x %u, q %d, es %d", r.nx, r.ny, r.nz, r.q, r.es);
    if (r.two < 0.83 * r.single) CHECK(pays, "two steps per pass refused on %u x %u x %u, q %d, es %d", r.nx, r.ny, r.nz, r.q, r.es);
  }
}

int main() {
  calls();
  tiles();
  sweeps();
  if (bad) return 1;
  printf("ok\n");
  return 0;
}
