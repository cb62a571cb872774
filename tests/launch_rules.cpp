// Host-side check of paper_1702_01530_amd/csrc/launch_rules.h.  Prints one line per claim and exits non-zero on a failure.
#include <cstdio>

#include "../paper_1702_01530_amd/csrc/launch_rules.h"

using namespace srt;

static int failures = 0;
static void claim(bool ok, const char* what) {
  std::printf("%s %s\n", ok ? "OK" : "FAIL", what);
  if (!ok) ++failures;
}

static void spheres_are_work() {
  const int64_t small = 2 * 256 * 256, large = 2 * 1920 * 1080;
  claim(path_wins({0, 8, 1, 1, true}, small), "a few spheres go through k_path");
  claim(path_wins({0, 8, 1, 8, true}, small), "with any lights");
  claim(!path_wins({0, 4096, 1, 1, true}, small), "a small frame of many spheres does not");
  claim(!path_wins({0, 1, 4096, 1, true}, small), "nor one of many planes");
  claim(!path_wins({100, 500, 0, 2, true}, small), "nor one of triangles and many spheres");
  claim(path_wins({0, 256, 1, 1, true}, small) && !path_wins({0, 256, 1, 4, true}, small), "lights count");
  claim(path_wins({0, 1024, 1, 4, true}, large), "a large frame has waves to run meanwhile");
  claim(path_wins({256, 0, 0, 8, true}, small) && !path_wins({257, 0, 0, 1, true}, large), "triangles as before");
  claim(!flat_splits({511, 0, 0, 1, true}) && flat_splits({512, 0, 0, 1, true}), "triangles split as before");
  claim(!flat_splits({0, 510, 1, 1, true}) && flat_splits({0, 511, 1, 1, true}), "spheres and planes split too");
  claim(flat_splits({100, 412, 0, 1, true}) && flat_splits({0, 1 << 20, 1 << 16, 1, true}), "all together");
}

static void spheres_beside_a_tree() {
  const int64_t paths = 2 * 640 * 480;
  claim(path_wins({13000, 0, 0, 2, false}, paths), "a small frame of a tree goes through k_path");
  claim(path_wins({13000, 8, 1, 2, false}, paths), "with a few spheres too");
  claim(!path_wins({5000, 2000, 1, 2, false}, paths), "not with many");
  claim(!path_wins({100, 0, 1024, 1, false}, paths), "nor with many planes");
  claim(!path_wins({13000, 0, 0, 8, false}, paths), "rays count as before");
}

static void batches() {
  claim(min_rays_log2(false) == 3, "a wave of one image starts with eight rays or more");
  claim(min_rays_log2(true) == 0, "of a batch with one or more: each may be of another scene");
}

static void small_frames() {
  const int waves = 4;
  bool covers = true, bounded = true;
  for (bool flat : {false, true})
    for (int64_t full : {1, 255, 256, 768, 2048})
      for (int64_t resident : {0, 1, 256, 1280, 1536, 4096})
        for (int64_t paths = 1; paths < 20000000; paths = paths * 5 / 4 + 127) {
          const PathLaunch l = path_launch(flat, paths, waves, full, resident);
          covers = covers && (l.dynamic || (l.grid * waves << l.log2n) >= paths);
          bounded = bounded && l.grid >= 1 && l.grid <= full && l.log2n >= 3 && l.log2n <= 6;
        }
  claim(covers, "a launch that is not dynamic has a wave for every batch");
  claim(bounded, "grids hold at least one workgroup and no more than the spill area has room for");
  const int64_t frame = int64_t(81) * 60 * 128;  // 641x479
  claim(path_launch(false, frame, waves, 256, 256).grid == 256, "one workgroup per CU is one on every CU");
  claim(path_launch(false, frame, waves, 2048, 1280).grid == 1280 && path_launch(false, frame, waves, 2048, 1280).dynamic,
        "a full grid has what is resident");
}

int main() {
  small_frames();
  batches();
  spheres_are_work();
  spheres_beside_a_tree();
  return failures ? 1 : 0;
}
