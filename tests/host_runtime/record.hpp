#pragma once
#include <vector>

struct Launch {
  int kind, steps;   // kind 0: a single step, 1: two steps of a 3D domain, 2: a pass of rD2Q9 tiles
};
extern std::vector<Launch> launches;
