// Which launches a render takes, from the sizes of its scene and image.  Plain C++: a host check runs it too.
// Results never depend on these rules.
#pragma once

#include <algorithm>
#include <cstdint>

namespace srt {

struct SceneSize {
  int32_t T, S, P, L;
  bool flat;  // without a tree, or rendered as if it had none
};

// Primitives that every ray of the scene is tested against.
inline int64_t walked(const SceneSize& s) { return int64_t(s.S) + s.P + (s.flat ? s.T : 0); }

// The fewest rays a traversal wave starts with, as a power of two: one image, or a batch of them.
constexpr int min_rays_log2(bool batch) { return batch ? 0 : 3; }

// Whether the waves of a workgroup share a batch's walk (k_trace_flat).  A launch of few rays lasts as long as one walk;
// a full one gains nothing from the shares and pays for joining them.  64x48, depth 0, 1 light: 120 triangles 75 us
// alone and 51 shared, 511: 160 and 63; 1920x1080: 394 and 646, 1371 and 1647.  256x256, depth 4, 4 lights: 256 spheres
// 336 and 307, 1024: 823 and 663.
constexpr int kFlatSplit = 512;
inline bool flat_splits(const SceneSize& s) { return walked(s) >= kFlatSplit; }

// Whether a whole frame goes through k_path.
//
// Without a tree: at most kPathFlat triangles (1920x1080, depth 8, 1 light: 120 triangles 354 us and 527 through the
// queues, 255: 840 and 1037; 64x48: 255 triangles 255 and 270, 400: 474 and 413).  Shadow rays wait for the walks before
// theirs, so a small frame takes few spheres and planes, the fewer the more lights there are: 256x256, depth 4, 64
// spheres: 104 and 159 us with 1 light, 167 and 188 with 4; 256: 285 and 304, 467 and 339; 1024: 996 and 439 with 1.  A
// large one has waves to run meanwhile (1920x1080, depth 4: 256 spheres 2188 and 2420, 3351 and 3968; 1024: 9882 and
// 9986 with 1 light, 2029 and 3233 at depth 0).
//
// With a tree: as long as the rays, counted as paths x (1 + lights), are few for the tree's size.  Terrains, depth 4:
// 800x600 with 4 lights is 4.8 M: 13k triangles 453 us and 476 through the queues; 640x480 with 8 lights 5.5 M: 531 and
// 511; 212k triangles: 640x480 with 2 lights is 1.8 M: 407 and 453, with 4 3.1 M: 520 and 524.  Scattered triangles that
// are all mirrors cross earlier (depth 3, 4 lights: 30k triangles at 640x480 1166 and 911, 100k at 320x240 767 and 673),
// large images of few lights later (212k, 1280x960, 1 light, 4.9 M: 648 and 699).  Spheres and planes beside the tree
// count as without one (5k triangles, depth 3, 640x480: 63 spheres 493 and 507 with 1 light, 886 and 706 with 4; 255
// spheres 811 and 714, 1355 and 985; 1,023: 2216 and 1536; 64x48, 1,023 spheres: 1160 and 864).
constexpr int kPathFlat = 256;
constexpr int kPathWalk = 512;
constexpr int kPathTreeWalk = 128;
constexpr int64_t kPathMany = int64_t(1) << 21;
constexpr int kPathSmallTree = 32768;  // triangles; the nodes fit an XCD's L2 several times
inline bool path_wins(const SceneSize& s, int64_t paths) {
  const int64_t analytic = int64_t(s.S) + s.P;
  if (s.flat) return s.T <= kPathFlat && (paths >= kPathMany || analytic * std::max(s.L, 1) <= kPathWalk);
  if (analytic > kPathTreeWalk) return false;
  return paths * (1 + s.L) <= (s.T <= kPathSmallTree ? 5000000 : 2500000);
}

// How k_path's waves take a frame's paths: a batch of 64 a wave, or of fewer where that still leaves every wave of the
// full grid at most one.  With more batches than waves run at once, those take them one by one: in fixed shares, or left
// to the dispatcher, the last ones decide (641x479, 13k triangles: 251 us in fixed shares, 235 so; spheres at 1080p 134
// and 106).  Where each wave gets one batch of 64 and a few get two, batches of 32 are evener (480x360: 212 and 183 us);
// from 1.5 batches a wave on they no longer are (640x480: 222 and 239).
struct PathLaunch {
  int log2n;     // a wave's batch is 2^log2n paths
  bool dynamic;  // waves take one batch after another
  int64_t grid;  // workgroups
};

// `full` bounds the grid (each of its threads has a part of the traversal's spill area); `resident` workgroups run at
// once, by k_path's own occupancy and the limit of workgroups per CU.  Taken as 5/8 of the traversal's, that limit at 1
// left 96 of 256 CUs without work (641x479, 13k triangles: 755 us, 543 so; spheres at 1080p 520 and 376).
inline PathLaunch path_launch(bool flat, int64_t paths, int waves, int64_t full, int64_t resident) {
  PathLaunch l{6, false, 0};
  resident = std::max<int64_t>(1, std::min(resident, full));
  auto blocks = [&](int log2n) { return (paths + (int64_t(waves) << log2n) - 1) / (int64_t(waves) << log2n); };
  if (!flat) {
    while (l.log2n > min_rays_log2(false) && (paths >> (l.log2n - 1)) < full * waves) --l.log2n;
    if (l.log2n == 6 && blocks(6) > resident && 2 * blocks(6) < 3 * resident) l.log2n = 5;
  }
  l.dynamic = blocks(l.log2n) > full || (l.log2n >= 5 && blocks(l.log2n) > resident);
  l.grid = std::min(l.dynamic ? resident : full, blocks(l.log2n));
  return l;
}

}  // namespace srt
