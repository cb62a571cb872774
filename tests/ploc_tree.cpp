// The clustering builder's whole tree on the host, from the leaf boxes in Morton order: rounds by the partner rule of
// paper_1702_01530_amd/csrc/ploc_rule.h, one node a mutual pair with indices handed out from T-2 downwards, the
// surface-area cost table of the 4-wide cut, and the collapse level by level.  Arithmetic is FP32, each operation
// rounded by itself but for the fused ones of half_area_of.
//
//   ploc_tree BOXES REFS    BOXES: T records of six floats (lower, upper corner); REFS: four int32 a node, children in
//                           slot order: a node, or ~(leaf << 2); unused slots repeat the first child
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1702_01530_amd/csrc/ploc_rule.h"

struct V3 {
  float x, y, z;
};
struct Node {
  int left, right;    // a node, or ~leaf
  float cost[5];      // C(1..4)
  int split[5];       // of the slots j = 2..4, how many go to the left child
  bool open[5];       // whether opening the node is cheaper than keeping it whole
};

static float area(V3 lo, V3 hi) { return srt::half_area_of(hi.x - lo.x, hi.y - lo.y, hi.z - lo.z); }

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  std::vector<float> in;
  FILE* f = std::fopen(argv[1], "rb");
  if (!f) return 2;
  float buf[6];
  while (std::fread(buf, 4, 6, f) == 6) in.insert(in.end(), buf, buf + 6);
  std::fclose(f);
  const int64_t T = int64_t(in.size()) / 6;
  if (T < 2) return 2;

  std::vector<V3> lo(T), hi(T);
  std::vector<int> ref(T);
  std::vector<Node> nodes(T - 1);
  std::vector<float> leaf_cost(T);
  for (int64_t i = 0; i < T; ++i) {
    lo[i] = {in[6 * i], in[6 * i + 1], in[6 * i + 2]};
    hi[i] = {in[6 * i + 3], in[6 * i + 4], in[6 * i + 5]};
    ref[i] = ~int(i);
    leaf_cost[i] = 0.5f * area(lo[i], hi[i]);
  }
  auto cost = [&](int r, int j) { return r < 0 ? leaf_cost[~r] : nodes[r].cost[j]; };

  // rounds
  int64_t left = T - 1;  // nodes not yet made
  while (ref.size() > 1) {
    const int64_t n = int64_t(ref.size());
    std::vector<int64_t> partner(n);
    for (int64_t i = 0; i < n; ++i) partner[i] = srt::ploc_partner(lo.data(), hi.data(), 0, i, n, 32);
    int64_t merges = 0;
    for (int64_t i = 0; i < n; ++i) merges += partner[i] > i && partner[partner[i]] == i;
    if (merges < 1 || merges > left) return 3;
    int64_t next = left - merges;
    left = next;
    std::vector<V3> nlo, nhi;
    std::vector<int> nref;
    for (int64_t i = 0; i < n; ++i) {
      const int64_t j = partner[i];
      const bool mutual = partner[j] == i;
      if (mutual && j < i) continue;
      V3 a = lo[i], b = hi[i];
      int r = ref[i];
      if (mutual) {
        a = {std::fmin(a.x, lo[j].x), std::fmin(a.y, lo[j].y), std::fmin(a.z, lo[j].z)};
        b = {std::fmax(b.x, hi[j].x), std::fmax(b.y, hi[j].y), std::fmax(b.z, hi[j].z)};
        r = int(next++);
        Node& m = nodes[r];
        m.left = ref[i];
        m.right = ref[j];
        float D[5];
        for (int s = 2; s <= 4; ++s) {
          D[s] = INFINITY;
          m.split[s] = 1;
          for (int k = 1; k < s; ++k) {
            const float c = cost(m.left, k) + cost(m.right, s - k);
            if (c < D[s]) D[s] = c, m.split[s] = k;
          }
        }
        m.cost[1] = area(a, b) + D[4];
        for (int s = 2; s <= 4; ++s) {
          m.open[s] = D[s] < m.cost[1];
          m.cost[s] = std::fmin(m.cost[1], D[s]);
        }
      }
      nlo.push_back(a);
      nhi.push_back(b);
      nref.push_back(r);
    }
    lo.swap(nlo);
    hi.swap(nhi);
    ref.swap(nref);
  }
  if (left != 0 || ref[0] != 0) return 3;

  // collapse: a node's four slots go to its children by its split; a child with several is opened where that is cheaper
  std::vector<int> level = {0}, out;
  int made = 1;
  while (!level.empty()) {
    std::vector<int> next;
    for (int b : level) {
      std::vector<int> r = {nodes[b].left, nodes[b].right}, slots = {nodes[b].split[4], 4 - nodes[b].split[4]};
      for (size_t k = 0; k < r.size();) {
        if (r[k] >= 0 && slots[k] > 1 && nodes[r[k]].open[slots[k]]) {
          const Node& m = nodes[r[k]];
          const int s = slots[k], sl = m.split[s];
          r[k] = m.left;
          slots[k] = sl;
          r.insert(r.begin() + k + 1, m.right);
          slots.insert(slots.begin() + k + 1, s - sl);
        } else {
          ++k;
        }
      }
      if (r.size() > 4) return 3;
      int refs[4];
      for (size_t k = 0; k < 4; ++k) {
        if (k >= r.size()) {
          refs[k] = refs[0];
        } else if (r[k] < 0) {
          refs[k] = ~((~r[k]) << 2);
        } else {
          refs[k] = made++;
          next.push_back(r[k]);
        }
      }
      out.insert(out.end(), refs, refs + 4);
    }
    level.swap(next);
  }
  f = std::fopen(argv[2], "wb");
  if (!f || std::fwrite(out.data(), 4, out.size(), f) != out.size()) return 2;
  return std::fclose(f) ? 2 : 0;
}
