// How many clustering rounds the host launches before it looks at what they left, and with how many workgroups each.
// Plain C++: a host check runs it too.  The tree does not depend on it.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace srt {

constexpr int kPlocTail = 1024;    // clusters that one workgroup takes over
constexpr int kPlocBlocks = 1024;  // most blocks of a round: each sums the others' counts
// Fewest blocks of a round, where a scene has work for them.  A round leaves 0.57 of the clusters at first and 0.81 to
// 0.83 later, but clusters of very different sizes in one place merge slower: a million triangles around one point, of
// random sizes, leave 0.97.  Rounds launched for the usual share then find a hundred times the clusters they are made
// for.  Build of that scene: 169 ms with grids that shrink as usual to the end and are never corrected, 30 with the
// corrections of look(), 20.6 with these blocks besides (64 instead: 25.2, 512: 20.1); 1M needles of random lengths
// 141, 32 and 24.  Scattered triangles, 200k: 0.81, 0.79 and 0.74 ms.
constexpr int kPlocLeast = 256;

struct ClusterPlan {
  int64_t triangles;
  double expected;       // clusters that the next round should find
  double usual = 0.83;   // the share of them it should leave
  double seen;           // clusters at the last look ...
  int rounds = 0, looked = 0;  // rounds so far and down to that look

  explicit ClusterPlan(int64_t T) : triangles(T), expected(double(T)), seen(double(T)) {}

  // Blocks of the next round, whose tiles are `own` clusters.
  int64_t blocks(int64_t own) const {
    const double all = std::ceil(double(triangles) / double(own)), tiles = std::ceil(expected / double(own));
    return int64_t(std::min<double>(kPlocBlocks, std::max(1.0, std::min(all, std::max<double>(kPlocLeast, tiles)))));
  }
  void next() {
    expected = std::max<double>(kPlocTail, expected * (rounds == 0 ? 0.6 : usual));
    ++rounds;
  }
  // Rounds to launch before anything is known: none where the one-workgroup kernel can start at once.
  int first() const {
    return triangles <= kPlocTail ? 0 : 2 + int(std::ceil(std::log(double(triangles) / kPlocTail) / 0.2));
  }
  // The rounds so far left n clusters: how many more to launch.
  int look(int64_t n) {
    expected = double(n);
    usual = std::max(0.83, std::pow(expected / seen, 1.0 / std::max(1, rounds - looked)));
    seen = expected;
    looked = rounds;
    const double more = 2 + std::ceil(std::log(expected / kPlocTail) / -std::log(std::min(usual, 0.999)));
    return int(std::min(64.0, std::max(16.0, more)));
  }
};

}  // namespace srt
