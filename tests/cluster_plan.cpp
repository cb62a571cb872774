// Host-side check of paper_1702_01530_amd/csrc/cluster_plan.h: scenes whose rounds leave a given share of the clusters
// are run through the plan.  From the first look at the clusters on, a round has a workgroup for every tile it finds (up
// to the most a round takes); before it, at least kPlocLeast or one a tile.  Prints one line per case and exits non-zero
// on a failure.
#include <cstdio>

#include "../paper_1702_01530_amd/csrc/cluster_plan.h"

int main() {
  int failures = 0;
  for (int64_t T : {1025, 5000, 65536, 1000000, 1 << 29}) {
    for (double share : {0.5, 0.83, 0.9, 0.97, 0.99, 0.999}) {
      for (int64_t own : {64, 416}) {
        srt::ClusterPlan plan(T);
        double n = double(T);
        int looks = 0, todo = plan.first();
        bool ok = todo > 0;
        while (ok && n > srt::kPlocTail && looks < 4096) {
          for (; todo > 0; --todo) {
            const double tiles = std::ceil(n / double(own)), most = std::min<double>(srt::kPlocBlocks, tiles);
            const double least = looks ? std::floor(0.9 * most) : std::min<double>(srt::kPlocLeast, most);
            if (n > srt::kPlocTail && double(plan.blocks(own)) < least) ok = false;
            if (plan.blocks(own) < 1 || plan.blocks(own) > srt::kPlocBlocks) ok = false;
            plan.next();
            if (n > srt::kPlocTail) n = std::floor(n * share);
          }
          if (n <= srt::kPlocTail) break;
          ++looks;
          todo = plan.look(int64_t(n));
          if (todo < 16 || todo > 64) ok = false;
        }
        ok = ok && n <= srt::kPlocTail;
        // each look is followed by 16 to 64 rounds
        if (looks > 3 + plan.rounds / 16) ok = false;
        std::printf("%s T=%lld share=%g own=%lld rounds=%d looks=%d\n", ok ? "OK" : "FAIL", (long long)T, share,
                    (long long)own, plan.rounds, looks);
        if (!ok) ++failures;
      }
    }
  }
  return failures ? 1 : 0;
}
