// Linear BVH build on the device (gfx950).
//
// The paper (Section 3, Table 1) lists BVH trees as fast to construct, simple to
// traverse and well suited to GPUs.  The tree here is built from the Morton order:
//   1. per triangle: bounding box and centroid, input validation;
//   2. reduction of the centroid and scene bounds;
//   3. 63-bit Morton code of the centroid quantised to 2^21 cells per axis;
//   4. stable sort of (code, triangle id): LSD radix, 8 passes of 8 bits, or for
//      few triangles one launch that counts the codes before each;
//   5. binary tree over the sorted leaves: by default locally-ordered clustering
//      (PLOC: neighbours in the Morton order merge by smallest surface area, so
//      node boxes come with the merges); with RT_ACCEL_KARRAS, Karras (2012)
//      emission (split at the highest differing bit; equal codes split by index) and
//   6. a bottom-up box refit (an atomic arrival counter per node, the second
//      child to arrive unions both boxes and climbs on);
//   7. a bottom-up surface-area cost table that picks the cheapest way to cut the
//      binary tree into a 4-wide one (filled during the refit or as the clustering
//      makes the nodes);
//   8. top-down collapse into that 4-wide tree, level by level (the narrow levels
//      in one workgroup, two launches for each wide one), with the children's
//      boxes quantised to 8 bits on each node's own grid (64-byte nodes), and
//      48-byte triangle records in leaf order.
// Every step is deterministic, so a scene always builds the same tree.

#include <hip/hip_runtime.h>


#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

#include "cluster_plan.h"
#include "rt_internal.h"
#define SRT_HD __host__ __device__
#include "ploc_rule.h"


namespace srt {

int leaf_size() { return 1; }  // every leaf of the collapsed tree is one triangle

namespace {

constexpr int kBlock = 256;
constexpr int kSortItems = 16;                      // keys per thread of a sort tile (4,096 keys a block)
constexpr int kSortItemsFew = 4;                    // ... where that would leave most of the chip idle
constexpr int64_t kSortFew = 1 << 18;               // (fewer triangles than this)
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

__device__ inline bool finite3(float a, float b, float c) {
  return isfinite(a) && isfinite(b) && isfinite(c);
}

// ---------------------------------------------------------------------------------------------
// 1-2. Triangle boxes, validation, bounds
// ---------------------------------------------------------------------------------------------

struct Bounds6 {
  float clo[3], chi[3];  // centroid bounds
  float blo[3], bhi[3];  // scene box
};

__global__ __launch_bounds__(kBlock) void k_tri_prep(const float* __restrict__ tris,
                                                     const uint32_t* __restrict__ mat, int64_t T, int32_t M,
                                                     float4* __restrict__ lo_out, float4* __restrict__ hi_out,
                                                     Bounds6* __restrict__ partial, uint32_t* __restrict__ status) {
  __shared__ float red[12][kBlock];
  int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  float c[3] = {INFINITY, INFINITY, INFINITY}, cmax[3] = {-INFINITY, -INFINITY, -INFINITY};
  if (i < T) {
    const float* p = tris + 9 * i;
    float v[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = p[k];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 9; ++k) ok = ok && fabsf(v[k]) <= RT_MAX_COORD;  // false for NaN and inf too
    if (!ok) atomicOr(status, 1u);
    if (mat[i] >= uint32_t(M)) atomicOr(status, 2u);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(v[a], fminf(v[3 + a], v[6 + a]));
      hi[a] = fmaxf(v[a], fmaxf(v[3 + a], v[6 + a]));
      c[a] = 0.5f * lo[a] + 0.5f * hi[a];
      cmax[a] = c[a];
    }
    lo_out[i] = make_float4(lo[0], lo[1], lo[2], 0.f);
    hi_out[i] = make_float4(hi[0], hi[1], hi[2], 0.f);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    red[a][threadIdx.x] = c[a];
    red[3 + a][threadIdx.x] = cmax[a];
    red[6 + a][threadIdx.x] = lo[a];
    red[9 + a][threadIdx.x] = hi[a];
  }
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + s]);
        red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + s]);
        red[6 + a][threadIdx.x] = fminf(red[6 + a][threadIdx.x], red[6 + a][threadIdx.x + s]);
        red[9 + a][threadIdx.x] = fmaxf(red[9 + a][threadIdx.x], red[9 + a][threadIdx.x + s]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    Bounds6 b;
    for (int a = 0; a < 3; ++a) {
      b.clo[a] = red[a][0];
      b.chi[a] = red[3 + a][0];
      b.blo[a] = red[6 + a][0];
      b.bhi[a] = red[9 + a][0];
    }
    partial[blockIdx.x] = b;
  }
}

__global__ __launch_bounds__(kBlock) void k_reduce_bounds(const Bounds6* __restrict__ partial, int64_t n,
                                                          Bounds6* __restrict__ out) {
  __shared__ float red[12][kBlock];
  float v[12];
  for (int a = 0; a < 3; ++a) {
    v[a] = INFINITY;
    v[3 + a] = -INFINITY;
    v[6 + a] = INFINITY;
    v[9 + a] = -INFINITY;
  }
  for (int64_t i = threadIdx.x; i < n; i += kBlock) {
    Bounds6 b = partial[i];
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], b.clo[a]);
      v[3 + a] = fmaxf(v[3 + a], b.chi[a]);
      v[6 + a] = fminf(v[6 + a], b.blo[a]);
      v[9 + a] = fmaxf(v[9 + a], b.bhi[a]);
    }
  }
  for (int k = 0; k < 12; ++k) red[k][threadIdx.x] = v[k];
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      for (int a = 0; a < 3; ++a) {
        red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + s]);
        red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + s]);
        red[6 + a][threadIdx.x] = fminf(red[6 + a][threadIdx.x], red[6 + a][threadIdx.x + s]);
        red[9 + a][threadIdx.x] = fmaxf(red[9 + a][threadIdx.x], red[9 + a][threadIdx.x + s]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    Bounds6 b;
    for (int a = 0; a < 3; ++a) {
      b.clo[a] = red[a][0];
      b.chi[a] = red[3 + a][0];
      b.blo[a] = red[6 + a][0];
      b.bhi[a] = red[9 + a][0];
    }
    *out = b;
  }
}

__global__ __launch_bounds__(kBlock) void k_check_spheres_planes(const float* __restrict__ spheres,
                                                                 const uint32_t* __restrict__ smat, int32_t S,
                                                                 const float* __restrict__ planes,
                                                                 const uint32_t* __restrict__ pmat, int32_t P,
                                                                 int32_t M, uint32_t* __restrict__ status) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < S) {
    const float* s = spheres + 4 * i;
    if (!(finite3(s[0], s[1], s[2]) && isfinite(s[3]) && s[3] > 0.f) || smat[i] >= uint32_t(M)) atomicOr(status, 4u);
  } else if (i < S + P) {
    int k = i - S;
    const float* p = planes + 4 * k;
    bool ok = finite3(p[0], p[1], p[2]) && isfinite(p[3]) && (p[0] * p[0] + p[1] * p[1] + p[2] * p[2]) > 0.f;
    if (!ok || pmat[k] >= uint32_t(M)) atomicOr(status, 8u);
  }
}

// ---------------------------------------------------------------------------------------------
// 3. Morton codes
// ---------------------------------------------------------------------------------------------

__device__ inline uint64_t spread21(uint32_t x) {
  uint64_t v = x & 0x1fffffu;
  v = (v | (v << 32)) & 0x1f00000000ffffull;
  v = (v | (v << 16)) & 0x1f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

__global__ __launch_bounds__(kBlock) void k_morton(const float4* __restrict__ lo, const float4* __restrict__ hi,
                                                   const Bounds6* __restrict__ bounds, int64_t T,
                                                   uint64_t* __restrict__ keys, uint32_t* __restrict__ ids) {
  int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= T) return;
  Bounds6 b = bounds[0];
  float4 l = lo[i], h = hi[i];
  float c[3] = {0.5f * l.x + 0.5f * h.x, 0.5f * l.y + 0.5f * h.y, 0.5f * l.z + 0.5f * h.z};
  uint32_t q[3];
  const float cells = 2097152.0f;  // 2^21
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float ext = b.chi[a] - b.clo[a];
    float s = ext > 0.f ? (c[a] - b.clo[a]) / ext * cells : 0.f;
    s = fminf(fmaxf(s, 0.f), cells - 1.f);
    q[a] = uint32_t(s);
  }
  keys[i] = (spread21(q[0]) << 2) | (spread21(q[1]) << 1) | spread21(q[2]);
  ids[i] = uint32_t(i);
}

// ---------------------------------------------------------------------------------------------
// 4. Stable LSD radix sort, 8 bits per pass
// ---------------------------------------------------------------------------------------------

// A pass is bound by its traffic (12 bytes read and written a key, 8 read for the histogram) once its writes
// are runs: a block orders its tile in LDS first, so that a digit's keys leave it side by side.  Written one
// by one from the registers they took 60 us a pass for 3.4M keys; ordered, 28.  The prefix over the blocks is
// one launch with a workgroup a digit (three launches, 14 us, as a general prefix sum), or none: below
// kScanInScatter blocks each scatter block sums its own.
constexpr int kScanInScatter = 32;

// Per-block digit histogram, stored digit-major: hist[digit * nblocks + block].
template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_digit_hist(const uint64_t* __restrict__ keys, int64_t n, int shift,
                                                       uint32_t* __restrict__ hist, int64_t nblocks) {
  __shared__ uint32_t h[kRadix];
  h[threadIdx.x] = 0;
  __syncthreads();
  int64_t base = int64_t(blockIdx.x) * (ITEMS * kBlock);
#pragma unroll 4
  for (int k = 0; k < ITEMS; ++k) {
    int64_t i = base + int64_t(k) * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & (kRadix - 1)], 1u);
  }
  __syncthreads();
  hist[int64_t(threadIdx.x) * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Exclusive sum of v over the block's kBlock threads; the total in *total.  `tmp` holds one word per wave.
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* tmp, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(x, off);
    if (lane >= off) x += u;
  }
  __syncthreads();
  if (lane == 63) tmp[wave] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (int w = 0; w < kBlock / 64; ++w) {
    if (w < wave) before += tmp[w];
    all += tmp[w];
  }
  *total = all;
  return before + x - v;
}

// Block d: the exclusive prefix of digit d's counts over the blocks, in place; their sum to totals[d].
__global__ __launch_bounds__(kBlock) void k_digit_scan(uint32_t* __restrict__ hist, int64_t nblocks,
                                                       uint32_t* __restrict__ totals) {
  __shared__ uint32_t tmp[kBlock / 64];
  uint32_t* row = hist + int64_t(blockIdx.x) * nblocks;
  uint32_t run = 0;
  for (int64_t base = 0; base < nblocks; base += kBlock) {
    const int64_t i = base + threadIdx.x;
    const uint32_t v = i < nblocks ? row[i] : 0u;
    uint32_t total;
    const uint32_t x = block_scan(v, tmp, &total);
    if (i < nblocks) row[i] = run + x;
    run += total;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = run;
}

__device__ inline uint64_t lanemask_lt() {
  const int lane = threadIdx.x & 63;
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Stable scatter of one tile: wave w holds the tile's keys w * 64 * ITEMS on, 64 a round, so the order is
// (wave, round, lane).  SCAN: hist holds raw counts (k_digit_scan was not run).
template <int ITEMS, bool SCAN>
__global__ __launch_bounds__(kBlock) void k_scatter(const uint64_t* __restrict__ keys_in,
                                                    const uint32_t* __restrict__ ids_in, int64_t n, int shift,
                                                    const uint32_t* __restrict__ hist,
                                                    const uint32_t* __restrict__ totals, int64_t nblocks,
                                                    uint64_t* __restrict__ keys_out, uint32_t* __restrict__ ids_out) {
  constexpr int kTile = ITEMS * kBlock, kW = kBlock / 64;
  static_assert(kRadix == kBlock, "a thread a digit");
  __shared__ uint64_t s_key[kTile];
  __shared__ uint32_t s_id[kTile];
  __shared__ uint32_t cnt[kW][kRadix];     // keys of a digit in the wave's rounds so far, then those before the wave
  __shared__ uint32_t local[kRadix];       // a digit's first place in the ordered tile
  __shared__ uint32_t to_global[kRadix];   // ... and what a place of it adds to give the output position
  __shared__ uint32_t tmp[kW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = int64_t(blockIdx.x) * kTile;
  const int count = int(min(int64_t(kTile), n - base));
  for (int w = 0; w < kW; ++w) cnt[w][tid] = 0;
  uint64_t key[ITEMS];
  uint32_t id[ITEMS], rank[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int at = wave * 64 * ITEMS + k * 64 + lane;
    key[k] = at < count ? keys_in[base + at] : 0;
    id[k] = at < count ? ids_in[base + at] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const bool valid = wave * 64 * ITEMS + k * 64 + lane < count;
    const uint32_t digit = uint32_t(key[k] >> shift) & (kRadix - 1);
    uint64_t peers = __ballot(valid);  // lanes of this wave holding the same digit
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
      const uint64_t bal = __ballot((digit >> b) & 1u);
      peers &= ((digit >> b) & 1u) ? bal : ~bal;
    }
    const uint32_t below = __popcll(peers & lanemask_lt());
    // a wave's LDS operations keep their order: every lane reads before the digit's first lane adds
    const uint32_t before = valid ? __hip_atomic_load(&cnt[wave][digit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0u;
    if (valid && below == 0)
      __hip_atomic_store(&cnt[wave][digit], before + uint32_t(__popcll(peers)), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_WORKGROUP);
    rank[k] = before + below;
  }
  __syncthreads();
  uint32_t mine = 0, total;
  for (int w = 0; w < kW; ++w) {
    const uint32_t c = cnt[w][tid];
    cnt[w][tid] = mine;
    mine += c;
  }
  const uint32_t place = block_scan(mine, tmp, &total);
  uint32_t digit_total, before_block;  // digit tid: its keys in all blocks, and in the blocks before this one
  if (SCAN) {
    digit_total = before_block = 0;
    for (int64_t b = 0; b < nblocks; ++b) {
      const uint32_t c = hist[int64_t(tid) * nblocks + b];
      if (b < int64_t(blockIdx.x)) before_block += c;
      digit_total += c;
    }
  } else {
    digit_total = totals[tid];
    before_block = hist[int64_t(tid) * nblocks + blockIdx.x];
  }
  const uint32_t digit_base = block_scan(digit_total, tmp, &total);
  local[tid] = place;
  to_global[tid] = digit_base + before_block - place;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (wave * 64 * ITEMS + k * 64 + lane < count) {
      const uint32_t digit = uint32_t(key[k] >> shift) & (kRadix - 1);
      const uint32_t at = local[digit] + cnt[wave][digit] + rank[k];
      s_key[at] = key[k];
      s_id[at] = id[k];
    }
  }
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < count; i += kBlock) {
    const uint64_t v = s_key[i];
    const uint32_t pos = to_global[uint32_t(v >> shift) & (kRadix - 1)] + uint32_t(i);
    if (int64_t(pos) < n) {
      keys_out[pos] = v;
      ids_out[pos] = s_id[i];
    }
  }
}

// One stable pass by the digit at `shift`.
template <int ITEMS>
hipError_t sort_pass(const uint64_t* k0, const uint32_t* i0, int64_t n, int shift, uint32_t* hist, uint32_t* totals,
                     uint64_t* k1, uint32_t* i1, hipStream_t s) {
  const int64_t nb = (n + ITEMS * kBlock - 1) / (ITEMS * kBlock);
  k_digit_hist<ITEMS><<<unsigned(nb), kBlock, 0, s>>>(k0, n, shift, hist, nb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nb <= kScanInScatter) {
    k_scatter<ITEMS, true><<<unsigned(nb), kBlock, 0, s>>>(k0, i0, n, shift, hist, totals, nb, k1, i1);
    return hipGetLastError();
  }
  k_digit_scan<<<kRadix, kBlock, 0, s>>>(hist, nb, totals);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_scatter<ITEMS, false><<<unsigned(nb), kBlock, 0, s>>>(k0, i0, n, shift, hist, totals, nb, k1, i1);
  return hipGetLastError();
}

// Few keys in one launch: a key's place is the number of keys before it, counted over all pairs.  A pass of the
// radix sort is two launches that a small build spends waiting, 16 in all.  Lanes hold the keys of a tile of 64 and a
// workgroup's waves walk their shares of all keys, 64 at a time through LDS, where all lanes read the same word; it
// is bound by those reads.  10k triangles: 95 us for the passes, 17 this way (29 with the keys as scalar loads, eight
// a wait).  Builds of 2k / 15k / 30k / 53k triangles: 479 / 619 / 708 / 775 us by passes, 427 / 567 / 687 / 906 here.
constexpr int64_t kRankMost = 32768;
constexpr int kRankBlock = 1024;
__global__ __launch_bounds__(kRankBlock) void k_rank_sort(const uint64_t* __restrict__ keys, int n,
                                                          uint64_t* __restrict__ keys_out,
                                                          uint32_t* __restrict__ ids_out) {
  constexpr int kW = kRankBlock / 64;
  __shared__ uint64_t s_keys[kW][64];
  __shared__ uint32_t part[kW][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = int(blockIdx.x) * 64, i = tile + lane;
  const uint64_t key = i < n ? keys[i] : 0;  // keys have 63 bits
  const int share = ((n + 64 * kW - 1) / (64 * kW)) * 64, first = min(n, wave * share), last = min(n, first + share);
  uint32_t before = 0;
  for (int base = first; base < last; base += 64) {
    s_keys[wave][lane] = base + lane < last ? keys[base + lane] : ~uint64_t(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // equal keys keep their order: those of earlier tiles count, those of this and later ones do not
    const uint64_t bar = base < tile ? key + 1 : key;
#pragma unroll 16
    for (int k = 0; k < 64; ++k) before += s_keys[wave][k] < bar ? 1u : 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if (wave == 0)
    for (int j = tile; j < min(tile + 64, n); ++j) before += (keys[j] == key && j < i) ? 1u : 0u;
  part[wave][lane] = before;
  __syncthreads();
  if (wave != 0 || i >= n) return;
  uint32_t rank = 0;
  for (int w = 0; w < kW; ++w) rank += part[w][lane];
  keys_out[rank] = key;
  ids_out[rank] = uint32_t(i);
}

// ---------------------------------------------------------------------------------------------
// 5. Karras (2012) hierarchy emission
// ---------------------------------------------------------------------------------------------

__device__ inline int delta(const uint64_t* __restrict__ k, int64_t n, int64_t i, int64_t j) {
  if (j < 0 || j >= n) return -1;
  uint64_t a = k[i], b = k[j];
  if (a != b) return __clzll(a ^ b);
  return 64 + __clz(uint32_t(i) ^ uint32_t(j));
}

// made[i] = (left, right) references (and later the choice bits), parents of internal nodes at parent[0..T-2],
// parents of leaves at parent[T-1 + leaf]; range[i] = (first, last) sorted leaf indices.
__global__ __launch_bounds__(kBlock) void k_karras(const uint64_t* __restrict__ keys, int64_t n,
                                                   int4* __restrict__ made, int32_t* __restrict__ parent,
                                                   int2* __restrict__ range) {
  int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= n - 1) return;
  int d = (delta(keys, n, i, i + 1) - delta(keys, n, i, i - 1)) >= 0 ? 1 : -1;
  int dmin = delta(keys, n, i, i - d);
  int64_t lmax = 2;
  while (delta(keys, n, i, i + lmax * d) > dmin) lmax *= 2;
  int64_t l = 0;
  for (int64_t t = lmax / 2; t >= 1; t /= 2)
    if (delta(keys, n, i, i + (l + t) * d) > dmin) l += t;
  int64_t j = i + l * d;
  int dnode = delta(keys, n, i, j);
  int64_t s = 0, t = l;
  do {
    t = (t + 1) >> 1;
    if (delta(keys, n, i, i + (s + t) * d) > dnode) s += t;
  } while (t > 1);
  int64_t gamma = i + s * d + (d < 0 ? -1 : 0);
  int64_t first = i < j ? i : j, last = i < j ? j : i;
  int left = (first == gamma) ? ~int(gamma) : int(gamma);           // leaf refs as ~index here
  int right = (last == gamma + 1) ? ~int(gamma + 1) : int(gamma + 1);
  made[i] = make_int4(left, right, 0, 0);
  range[i] = make_int2(int(first), int(last));
  if (gamma < 0 || gamma + 1 >= n) return;  // cannot happen for a valid split; never write out of bounds
  if (left < 0) parent[n - 1 + ~left] = int(i); else parent[left] = int(i);
  if (right < 0) parent[n - 1 + ~right] = int(i); else parent[right] = int(i);
}

// ---------------------------------------------------------------------------------------------
// 6./7. Bottom-up refit and cost table
// ---------------------------------------------------------------------------------------------

__device__ inline float half_area(float4 lo, float4 hi) {
  return half_area_of(hi.x - lo.x, hi.y - lo.y, hi.z - lo.z);
}

#ifndef SRT_DP_TRI_COST
#define SRT_DP_TRI_COST 0.5f
#endif
// The cost of a leaf, rounded by itself
__device__ inline float leaf_cost(float4 lo, float4 hi) {
#pragma clang fp contract(off)
  return SRT_DP_TRI_COST * half_area(lo, hi);
}

// Cost-optimal cut of the binary tree into the 4-wide tree (surface-area model, as in Ylitie et al.
// 2017): C(n, j) is the least expected cost of binary subtree n when it may take j slots of its BVH4
// parent.  C(n, 1) = A(n) + D_n(4) (n becomes a BVH4 node whose four slots its two children share),
// D_n(j) = min over k of C(a, k) + C(b, j - k), and C(n, j) = min(C(n, 1), D_n(j)) for j > 1 (n kept
// whole, or opened across j slots).  A leaf costs its area times the relative cost of a triangle test,
// whatever its slot count.  Choice bits per node, for j = 2, 3, 4 at bit 3 (j - 2): the split k
// (2 bits) and whether opening wins.
__device__ inline void dp_child_costs(int r, const float4* dp_cost, const float4* leaf_lo, const float4* leaf_hi,
                                      const uint32_t* sorted_ids, float (&c)[4]) {
  if (r < 0) {
    const uint32_t id = sorted_ids[~r];
    const float a = leaf_cost(leaf_lo[id], leaf_hi[id]);
    c[0] = c[1] = c[2] = c[3] = a;
  } else {
    const float4 v = dp_cost[r];
    c[0] = v.x, c[1] = v.y, c[2] = v.z, c[3] = v.w;
  }
}

// The costs C(n, 1..4) and choice bits of a node of half area `area` whose children cost ca and cb.
__device__ inline float4 dp_costs(float area, const float (&ca)[4], const float (&cb)[4], uint32_t* choice_out) {
  float D[5];
  int K[5];
  for (int j = 2; j <= 4; ++j) {
    D[j] = INFINITY;
    K[j] = 1;
    for (int k = 1; k < j; ++k) {
      const float c = ca[k - 1] + cb[j - k - 1];
      if (c < D[j]) {
        D[j] = c;
        K[j] = k;
      }
    }
  }
  const float c1 = area + D[4];
  uint32_t choice = 0;
  for (int j = 2; j <= 4; ++j) choice |= (uint32_t(K[j]) | (D[j] < c1 ? 4u : 0u)) << (3 * (j - 2));
  *choice_out = choice;
  return make_float4(c1, fminf(c1, D[2]), fminf(c1, D[3]), fminf(c1, D[4]));
}

// Fills the cost table entry of binary node n, whose box and children's entries are final.
__device__ inline void dp_node(int64_t n, int4* made, const float4* nodebox, const float4* leaf_lo,
                               const float4* leaf_hi, const uint32_t* sorted_ids, float4* dp_cost) {
  const int4 ch = made[n];
  float ca[4], cb[4];
  dp_child_costs(ch.x, dp_cost, leaf_lo, leaf_hi, sorted_ids, ca);
  dp_child_costs(ch.y, dp_cost, leaf_lo, leaf_hi, sorted_ids, cb);
  uint32_t choice;
  dp_cost[n] = dp_costs(half_area(nodebox[2 * n], nodebox[2 * n + 1]), ca, cb, &choice);
  made[n].z = int(choice);
}

__global__ __launch_bounds__(kBlock) void k_refit(int4* made, const int32_t* __restrict__ parent,
                                                  const float4* __restrict__ leaf_lo, const float4* __restrict__ leaf_hi,
                                                  const uint32_t* __restrict__ sorted_ids, float4* nodebox,
                                                  uint32_t* flags, int64_t n, uint32_t* __restrict__ status,
                                                  float4* dp_cost) {
  int64_t leaf = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (leaf >= n) return;
  int node = parent[n - 1 + leaf];
  for (int guard = 0; guard < 256; ++guard) {
    if (node < 0 || node >= n - 1) {  // corrupt parent link: report instead of reading out of bounds
      atomicOr(status, 16u);
      return;
    }
    uint32_t old = __hip_atomic_fetch_add(&flags[node], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 0) break;  // the sibling subtree is still being built; its thread climbs on
    const int4 ch = made[node];
    float4 lo[2], hi[2];
    int c[2] = {ch.x, ch.y};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (c[k] < 0) {
        uint32_t id = sorted_ids[~c[k]];
        lo[k] = leaf_lo[id];
        hi[k] = leaf_hi[id];
      } else {
        lo[k] = nodebox[2 * c[k]];
        hi[k] = nodebox[2 * c[k] + 1];
      }
    }
    nodebox[2 * node] = make_float4(fminf(lo[0].x, lo[1].x), fminf(lo[0].y, lo[1].y), fminf(lo[0].z, lo[1].z), 0.f);
    nodebox[2 * node + 1] =
        make_float4(fmaxf(hi[0].x, hi[1].x), fmaxf(hi[0].y, hi[1].y), fmaxf(hi[0].z, hi[1].z), 0.f);
    dp_node(node, made, nodebox, leaf_lo, leaf_hi, sorted_ids, dp_cost);
    if (node == 0) break;
    node = parent[node];
  }
}

// ---------------------------------------------------------------------------------------------
// 5'-6'. PLOC: parallel locally-ordered clustering over the Morton order (Meister and Bittner
// 2018), an alternative to steps 5-6.  Clusters start as the sorted leaves.  Each round, every
// cluster finds the neighbour within kPlocRadius positions whose merged box has the smallest
// surface area (ties to the smaller position); mutual pairs merge into a new internal node, and
// the survivors are compacted in order.  The globally best pair is always mutual, so every round
// merges.  Node indices are handed out from T-2 downwards by prefix sums, so the root is node 0 and
// the tree is the same on every run.
//
// A build has 40 (10k triangles) to 65 (3.4M) rounds, each leaving about 0.8 of the clusters, so it is
// bound by the cost of a round that has little to do.  The number of clusters stays on the device: the
// host launches as many rounds as the decay suggests, two kernels each, without waiting for any of them,
// and one workgroup does every round from kPlocTail clusters down (about 30 of them) with the clusters in
// LDS.  A node's row of the cost table is made with the node.  With a host read, two prefix sums and five
// launches a round, and a launch a round for the cost table, building and showing a scene of 10k triangles took
// 2.99 ms and took 0.80 this way (3.4M triangles: 8.2 and 3.3 ms); 0.51 and 2.55 with the steps since.
// ---------------------------------------------------------------------------------------------

// Search radius: with the cost-table collapse, 32 gives the fewest node visits per frame on the
// benchmark scene (8, 16, 24, 48 and 64 were measured).
#ifndef SRT_PLOC_RADIUS
#define SRT_PLOC_RADIUS 32
#endif
constexpr int kPlocRadius = SRT_PLOC_RADIUS;

// What the build's kernels tell each other and, at its end, the host (the scratch's first words).
struct BuildState {
  uint32_t status;    // BuildResult::status_bits
  uint32_t error;     // a step that cannot happen: no merge in a round, more nodes than leaves
  uint32_t pad[2];
  struct Ploc {
    uint32_t n;     // clusters left; 1 when the tree is complete, 0 after an error
    uint32_t next;  // internal nodes not yet made: the next round's take the indices below this
    uint32_t buf;   // the buffer that holds the clusters
    uint32_t pad;
  } ploc[2];  // round k reads slot k & 1 and writes the other
  struct Wide {
    uint32_t m;          // BVH4 nodes of the level to come
    uint32_t allocated;  // BVH4 nodes down to that level
    uint32_t level;
    uint32_t pad;
  } wide[2];  // level launch k reads slot k & 1 and writes the other
  Bounds6 bounds;
};
static_assert(sizeof(BuildState) <= 256, "the plan sets 256 bytes aside");

// Clusters: the corners of the box, the reference (node, or ~position of a leaf) beside the lower one.  Buffer 0 holds
// the leaves and is kept: the collapse reads their boxes from it in leaf order.  The rounds write buffers 1 and 2 in
// turn.  What a cluster costs lies with its node and a leaf's follows from its box, so a round moves 32 bytes a cluster
// (with the costs carried along it was 48; 3.4M triangles, all rounds: 463 us of compaction then, 396 now).
struct Clusters {
  float4 *lo0, *lo1, *lo2, *hi0, *hi1, *hi2;
};
__device__ inline float4* buffer_of(uint32_t buf, float4* b0, float4* b1, float4* b2) {
  float4* b = b0;
  if (buf == 1) b = b1;
  if (buf == 2) b = b2;
  return b;
}
__device__ inline float4* lo_of(const Clusters& c, uint32_t buf) { return buffer_of(buf, c.lo0, c.lo1, c.lo2); }
__device__ inline float4* hi_of(const Clusters& c, uint32_t buf) { return buffer_of(buf, c.hi0, c.hi1, c.hi2); }

__global__ __launch_bounds__(kBlock) void k_ploc_init(const uint32_t* __restrict__ sorted_ids,
                                                      const float4* __restrict__ leaf_lo,
                                                      const float4* __restrict__ leaf_hi, int64_t n, Clusters c) {
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t id = sorted_ids[i];
  const float4 lo = leaf_lo[id], hi = leaf_hi[id];
  c.lo0[i] = make_float4(lo.x, lo.y, lo.z, __int_as_float(~int(i)));
  c.hi0[i] = make_float4(hi.x, hi.y, hi.z, 0.f);
}

constexpr int kPlocBlock = 512;    // threads of a search block ...
constexpr int kPlocLanes = 4;      // ... which share a position's search this many at a time
constexpr int kPlocFew = 65536;    // below this many, tiles of kPairOwn positions leave most of the chip idle
constexpr int kPackBlocks = 1024;  // workgroups that pack triangles beside it

// The positions that block `b` of `blocks` handles in a round of n clusters: whole tiles of `own`.
__device__ inline void ploc_range(uint32_t n, uint32_t own, uint32_t b, uint32_t blocks, uint32_t* begin,
                                  uint32_t* end) {
  const uint32_t tiles = (n + own - 1) / own, per = (tiles + blocks - 1) / blocks;
  *begin = min(uint64_t(b) * per * own, uint64_t(n));
  *end = min(uint64_t(b + 1) * per * own, uint64_t(n));
}

// Sum of v over the block (a multiple of 64 threads), in every thread; `tmp` holds one word per wave.
__device__ inline uint32_t block_sum(uint32_t v, uint32_t* tmp) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t t = 0;
  for (int w = 0; w < int(blockDim.x) / 64; ++w) t += tmp[w];
  return t;
}

// max and min without the instructions that quiet a signalling NaN first (12 of 87 in the search's loop; boxes of
// accepted input hold no NaN, and those of refused input are only ever written to the scratch).
__device__ inline float raw_max(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ inline float raw_min(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// merged_area for two boxes known to be no NaN
__device__ inline float merged_area_raw(float3 alo, float3 ahi, float3 blo, float3 bhi) {
  return half_area_of(raw_max(ahi.x, bhi.x) - raw_min(alo.x, blo.x), raw_max(ahi.y, bhi.y) - raw_min(alo.y, blo.y),
                      raw_max(ahi.z, bhi.z) - raw_min(alo.z, blo.z));
}

// v of another lane of the group of 2^(S + 1), of which each half holds one value throughout: with S = 0, 1, .. in turn
// a reduction over groups of up to 32 lanes, without the address and the trip through LDS of a shuffle.
template <int S>
__device__ inline uint32_t other_half(uint32_t v) {
  // pairs and quads exchanged, then mirrors of 8 and 16 lanes, then 16 lanes swapped
  constexpr int kDpp[4] = {0xb1, 0x4e, 0x141, 0x140};
  if (S < 4) return uint32_t(__builtin_amdgcn_mov_dpp(int(v), kDpp[S & 3], 0xf, 0xf, false));
  return uint32_t(__builtin_amdgcn_ds_swizzle(int(v), 0x401f));
}
template <int S>
__device__ inline void nearer_half(float* best, int* bk) {
  const float ob = __uint_as_float(other_half<S>(__float_as_uint(*best)));
  const int ok = int(other_half<S>(uint32_t(*bk)));
  if (ob < *best || (ob == *best && ok < *bk)) *best = ob, *bk = ok;
}

// counts[block] = (merges, absorbed) of a search block; `merges` and `absorbed` are each wave's own.
__device__ inline void store_counts(uint32_t merges, uint32_t absorbed, uint2* tmp, uint2* counts) {
  if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = make_uint2(merges, absorbed);
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < int(blockDim.x) / 64; ++w) merges += tmp[w].x, absorbed += tmp[w].y;
  counts[blockIdx.x] = make_uint2(merges, absorbed);
}

// partner[i] = the position cluster i merges with this round, or -1; counts[block] = (merges, absorbed
// clusters) of the block's positions.  A tile's mutual pairs need the choices of kPlocRadius positions on
// either side too, so a block makes those as well.  This is the search of a round with too few clusters to
// fill the chip: kPlocLanes lanes share a position's candidates.
__global__ __launch_bounds__(kPlocBlock) void k_ploc_nn(Clusters c, BuildState* state, int slot,
                                                        int32_t* __restrict__ partner, uint2* __restrict__ counts) {
  constexpr int R = kPlocRadius, LANES = kPlocLanes, kPos = kPlocBlock / LANES, kOwn = kPos - 2 * R;
  static_assert(kOwn > 0 && 2 * R % LANES == 0, "search split");
  __shared__ float4 s_lo[kPos + 2 * R], s_hi[kPos + 2 * R];
  __shared__ int s_nn[kPos];
  __shared__ uint2 tmp[kPlocBlock / 64];
  const uint32_t n = state->ploc[slot].n, buf = state->ploc[slot].buf;
  if (n <= kPlocTail) return;
  const float4 *__restrict__ lo = lo_of(c, buf), *__restrict__ hi = hi_of(c, buf);
  uint32_t begin, end, merges = 0, absorbed = 0;
  ploc_range(n, kOwn, blockIdx.x, gridDim.x, &begin, &end);
  const int p = threadIdx.x / LANES, sub = threadIdx.x % LANES;
  for (uint32_t base = begin; base < end; base += kOwn) {
    __syncthreads();
    for (int k = threadIdx.x; k < kPos + 2 * R; k += kPlocBlock) {
      const int64_t g = int64_t(base) - 2 * R + k;
      const bool in = g >= 0 && g < int64_t(n);
      // a box at +inf: any merge with it has an infinite area and is never chosen
      s_lo[k] = in ? lo[g] : make_float4(INFINITY, INFINITY, INFINITY, 0.f);
      s_hi[k] = in ? hi[g] : make_float4(INFINITY, INFINITY, INFINITY, 0.f);
    }
    __syncthreads();
    const int64_t g = int64_t(base) - R + p;  // this thread's position, at p + R in LDS
    const bool valid = g >= 0 && g < int64_t(n);
    const float4 alo = s_lo[p + R], ahi = s_hi[p + R];
    auto area = [&](int k) {
      auto f3 = [](float4 v) { return make_float3(v.x, v.y, v.z); };
      return merged_area_raw(f3(alo), f3(ahi), f3(s_lo[p + R + k]), f3(s_hi[p + R + k]));
    };
    float best = INFINITY;
    int bk = 0;
    // ascending positions: ties keep the smaller one
#pragma unroll 8
    for (int q = 0; q < R / LANES; ++q) {
      const int k = -R + q * LANES + sub;
      const float ar = area(k);
      if (ar < best) best = ar, bk = k;
    }
#pragma unroll 8
    for (int q = 0; q < R / LANES; ++q) {
      const int k = 1 + q * LANES + sub;
      const float ar = area(k);
      if (ar < best) best = ar, bk = k;
    }
    static_assert(LANES == 4, "two halvings");
    nearer_half<0>(&best, &bk);
    nearer_half<1>(&best, &bk);
    if (valid) {
      if (!(best < INFINITY)) bk = g > 0 ? -1 : 1;  // boxes of refused input only: keep the rounds well formed
      const int toward = (g & 1) ? -1 : 1;  // g ^ 1
      if (g + toward < int64_t(n) && ploc_takes_parity(best, alo, ahi, s_lo[p + R + toward], s_hi[p + R + toward]))
        bk = toward;
    }
    if (sub == 0) s_nn[p] = valid ? p + bk : -1;
    __syncthreads();
    int j = p;
    if (sub == 0 && p >= R && p < kPos - R && valid) {
      j = s_nn[p];
      const bool mutual = s_nn[j] == p;  // j lies within R of p
      partner[g] = mutual ? int32_t(g + j - p) : -1;
      if (!mutual) j = p;
    }
    merges += uint32_t(__popcll(__ballot(j > p)));    // the lower position of a mutual pair makes the node
    absorbed += uint32_t(__popcll(__ballot(j < p)));  // the higher one goes
  }
  store_counts(merges, absorbed, tmp, counts);
}

// The search of a round with many clusters, bound by the VALU (18 instructions a candidate, 64 candidates a
// position).  An area is the same from both sides, so it is computed once: a thread holds two neighbouring
// positions and walks the kPlocRadius positions above them; the better of its two areas with each goes to that
// position's word in LDS, (area bits << 32 | position), whose minimum is the best partner below, ties to the
// smaller position.  Even and odd positions lie in arrays of their own, so a wave's reads are consecutive.
// First round of 3.4M triangles: 166 us with all of a position's candidates in one thread, 86 us this way.
constexpr int kPairBlock = 256;
constexpr int kPairOwn = 2 * kPairBlock - 3 * kPlocRadius;

__global__ __launch_bounds__(kPairBlock) void k_ploc_nn_pairs(Clusters c, BuildState* state, int slot,
                                                              int32_t* __restrict__ partner,
                                                              uint2* __restrict__ counts) {
  constexpr int R = kPlocRadius, H = R / 2, kPos = 2 * kPairBlock, kHalf = kPairBlock + H;
  static_assert(R % 2 == 0 && kPairOwn > 0 && kPairOwn % 2 == 0, "positions come in pairs");
  __shared__ float4 s_lo[2][kHalf], s_hi[2][kHalf];  // position base - 2R + k at [k & 1][k / 2]
  __shared__ unsigned long long s_below[2][kHalf];   // its best partner below
  __shared__ int s_nn[kPos];
  __shared__ uint2 tmp[kPairBlock / 64];
  const uint32_t n = state->ploc[slot].n, buf = state->ploc[slot].buf;
  if (n <= kPlocTail) return;
  const float4 *__restrict__ lo = lo_of(c, buf), *__restrict__ hi = hi_of(c, buf);
  uint32_t begin, end, merges = 0, absorbed = 0;
  ploc_range(n, kPairOwn, blockIdx.x, gridDim.x, &begin, &end);
  const int q = threadIdx.x;
  for (uint32_t base = begin; base < end; base += kPairOwn) {
    __syncthreads();
    for (int k = threadIdx.x; k < 2 * kHalf; k += kPairBlock) {
      const int64_t g = int64_t(base) - 2 * R + k;
      const bool in = g >= 0 && g < int64_t(n);
      // a box at +inf: any merge with it has an infinite area and is never chosen
      s_lo[k & 1][k >> 1] = in ? lo[g] : make_float4(INFINITY, INFINITY, INFINITY, 0.f);
      s_hi[k & 1][k >> 1] = in ? hi[g] : make_float4(INFINITY, INFINITY, INFINITY, 0.f);
      s_below[k & 1][k >> 1] = ~0ull;
    }
    __syncthreads();
    const int64_t g0 = int64_t(base) - 2 * R + 2 * q;  // even, as tiles and R are; its parity partner is g0 + 1
    auto f3 = [](float4 v) { return make_float3(v.x, v.y, v.z); };
    const float3 lo0 = f3(s_lo[0][q]), hi0 = f3(s_hi[0][q]), lo1 = f3(s_lo[1][q]), hi1 = f3(s_hi[1][q]);
    float best0 = INFINITY, best1 = INFINITY;  // over the positions above
    int bk0 = 0, bk1 = 0;
    auto tell = [&](unsigned long long* word, float ar, int from) {
      __hip_atomic_fetch_min(word, (static_cast<unsigned long long>(__float_as_uint(ar)) << 32) | uint32_t(from),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // the box at LDS position j = 2q + k with both of the thread's
    auto both = [&](int odd, int at, int k) {
      const float3 l = f3(s_lo[odd][at]), h = f3(s_hi[odd][at]);
      const float a0 = merged_area_raw(lo0, hi0, l, h), a1 = merged_area_raw(lo1, hi1, l, h);
      if (a0 < best0) best0 = a0, bk0 = k;
      if (a1 < best1) best1 = a1, bk1 = k - 1;
      tell(&s_below[odd][at], a1 < a0 ? a1 : a0, a1 < a0 ? 2 * q + 1 : 2 * q);
    };
    {
      const float ar = merged_area_raw(lo0, hi0, lo1, hi1);
      best0 = ar, bk0 = 1;
      tell(&s_below[1][q], ar, 2 * q);
    }
#pragma unroll 3
    for (int kk = 1; kk < H; ++kk) {
      both(0, q + kk, 2 * kk);
      both(1, q + kk, 2 * kk + 1);
    }
    both(0, q + H, R);
    {  // R + 1 above the lower position: only the upper one reaches it
      const float ar = merged_area_raw(lo1, hi1, f3(s_lo[1][q + H]), f3(s_hi[1][q + H]));
      if (ar < best1) best1 = ar, bk1 = R;
      tell(&s_below[1][q + H], ar, 2 * q + 1);
    }
    __syncthreads();
    const bool v0 = g0 >= 0 && g0 < int64_t(n), v1 = g0 + 1 >= 0 && g0 + 1 < int64_t(n);
    auto choose = [&](int odd, float best, int bk, int64_t g) {
      const int p = 2 * q + odd;
      const unsigned long long w = s_below[odd][q];
      const float below = __uint_as_float(uint32_t(w >> 32));
      if (below < INFINITY && below <= best) {  // the partner below is the smaller position
        best = below;
        bk = int(uint32_t(w)) - p;
      }
      if (!(best < INFINITY)) bk = g > 0 ? -1 : 1;  // boxes of refused input only: keep the rounds well formed
      const float4 lo4 = s_lo[odd][q], hi4 = s_hi[odd][q], olo = s_lo[odd ^ 1][q], ohi = s_hi[odd ^ 1][q];
      if (v0 && v1 && ploc_takes_parity(best, lo4, hi4, olo, ohi)) bk = odd ? -1 : 1;
      return p + bk;
    };
    s_nn[2 * q] = v0 ? choose(0, best0, bk0, g0) : -1;
    s_nn[2 * q + 1] = v1 ? choose(1, best1, bk1, g0 + 1) : -1;
    __syncthreads();
    for (int k = 0; k < 2; ++k) {
      // positions from 2R to kPos - R are the tile's own; those from R on have seen every candidate
      const int p = 2 * q + k;
      int j = p;
      if (p >= 2 * R && p < kPos - R && (k ? v1 : v0)) {
        j = s_nn[p];
        const bool mutual = s_nn[j] == p;  // j lies within R of p
        partner[g0 + k] = mutual ? int32_t(g0 + k + j - p) : -1;
        if (!mutual) j = p;
      }
      merges += uint32_t(__popcll(__ballot(j > p)));    // the lower position of a mutual pair makes the node
      absorbed += uint32_t(__popcll(__ballot(j < p)));  // the higher one goes
    }
  }
  store_counts(merges, absorbed, tmp, counts);
}

struct PlocNodes {
  int4* made;      // (children, choice bits, 0)
  float4* nodebox;
  float4* cost;    // C(1..4)
};

__device__ inline float4 ploc_cost(const PlocNodes& out, float4 lo, float4 hi) {
  const int ref = __float_as_int(lo.w);
  if (ref >= 0) return out.cost[ref];
  const float c = leaf_cost(lo, hi);
  return make_float4(c, c, c, c);
}

// Merges clusters a (lower position) and b, which cost ca and cb, into node `node`.
__device__ inline float4 ploc_merge(const PlocNodes& out, int node, float4 alo, float4 ahi, float4 ca4, float4 blo,
                                    float4 bhi, float4 cb4, float4* lo, float4* hi) {
  const float4 ulo = make_float4(fminf(alo.x, blo.x), fminf(alo.y, blo.y), fminf(alo.z, blo.z), 0.f);
  const float4 uhi = make_float4(fmaxf(ahi.x, bhi.x), fmaxf(ahi.y, bhi.y), fmaxf(ahi.z, bhi.z), 0.f);
  const float ca[4] = {ca4.x, ca4.y, ca4.z, ca4.w}, cb[4] = {cb4.x, cb4.y, cb4.z, cb4.w};
  uint32_t choice;
  const float4 cost = dp_costs(half_area(ulo, uhi), ca, cb, &choice);
  out.made[node] = make_int4(__float_as_int(alo.w), __float_as_int(blo.w), int(choice), 0);
  out.nodebox[2 * int64_t(node)] = ulo;
  out.nodebox[2 * int64_t(node) + 1] = uhi;
  *lo = make_float4(ulo.x, ulo.y, ulo.z, __int_as_float(node));
  *hi = uhi;
  return cost;
}

// Makes the round's nodes and compacts the survivors into the other buffer.  `own` and the grid are those of
// the round's search, whose counts place each block's output.  A tile's loads are issued before the tile ahead of it
// is stored, and the first tile's before the counts are summed: a round is a chain of such waits.
__global__ __launch_bounds__(kBlock) void k_ploc_compact(Clusters c, BuildState* state, int slot,
                                                         const int32_t* __restrict__ partner,
                                                         const uint2* __restrict__ counts, uint32_t own,
                                                         PlocNodes out) {
  constexpr int kW = kBlock / 64;
  __shared__ uint4 wsum[kW];
  __shared__ uint32_t wkeep[2][kW], wmerge[2][kW];
  const BuildState::Ploc st = state->ploc[slot];
  BuildState::Ploc* next = &state->ploc[slot ^ 1];
  if (st.n <= kPlocTail) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *next = st;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t dst = st.buf == 1 ? 2u : 1u;
  const float4 *ilo = lo_of(c, st.buf), *ihi = hi_of(c, st.buf);
  float4 *olo = lo_of(c, dst), *ohi = hi_of(c, dst);
  uint32_t begin, end;
  ploc_range(st.n, own, blockIdx.x, gridDim.x, &begin, &end);
  int32_t j = -1;
  float4 lo, hi;
  auto fetch = [&](uint32_t i) {
    j = -1;
    if (i < end) j = partner[i], lo = ilo[i], hi = ihi[i];
  };
  fetch(begin + threadIdx.x);
  uint4 sum = make_uint4(0u, 0u, 0u, 0u);  // merges and absorbed clusters, of the blocks before and of all
  for (uint32_t k = threadIdx.x; k < gridDim.x; k += kBlock) {
    const uint2 v = counts[k];
    sum.z += v.x, sum.w += v.y;
    if (k < blockIdx.x) sum.x += v.x, sum.y += v.y;
  }
  for (int off = 32; off > 0; off >>= 1) {
    sum.x += __shfl_xor(sum.x, off), sum.y += __shfl_xor(sum.y, off);
    sum.z += __shfl_xor(sum.z, off), sum.w += __shfl_xor(sum.w, off);
  }
  if (lane == 0) wsum[wave] = sum;
  __syncthreads();
  uint32_t m0 = 0, a0 = 0, mall = 0, aall = 0;
  for (int w = 0; w < kW; ++w) m0 += wsum[w].x, a0 += wsum[w].y, mall += wsum[w].z, aall += wsum[w].w;
  // every round merges a pair, each pair absorbs one cluster, and T - 1 nodes are made in all
  const bool bad = mall == 0 || mall != aall || mall > st.next;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (bad) atomicOr(&state->error, 1u);
    *next = BuildState::Ploc{bad ? 0u : st.n - mall, bad ? 0u : st.next - mall, dst, 0u};
  }
  if (bad) return;
  uint32_t pos0 = begin - a0, node0 = st.next - mall + m0;
  int par = 0;
  for (uint32_t base = begin; base < end; base += kBlock, par ^= 1) {
    const uint32_t i = base + threadIdx.x;
    const bool merge = j > int32_t(i), keep = i < end && (j < 0 || merge);
    const uint64_t bk = __ballot(keep), bm = __ballot(merge);
    if (lane == 0) wkeep[par][wave] = uint32_t(__popcll(bk)), wmerge[par][wave] = uint32_t(__popcll(bm));
    float4 tlo = lo, thi = hi, blo, bhi, ca, cb;
    if (merge) {
      blo = ilo[j], bhi = ihi[j];
      ca = ploc_cost(out, tlo, thi);
      cb = ploc_cost(out, blo, bhi);
    }
    fetch(i + kBlock);
    __syncthreads();
    uint32_t kb = 0, mb = 0, kt = 0, mt = 0;
    for (int w = 0; w < kW; ++w) {
      const uint32_t x = wkeep[par][w], y = wmerge[par][w];
      if (w < wave) kb += x, mb += y;
      kt += x, mt += y;
    }
    const uint64_t lt = lanemask_lt();
    if (merge) {
      const uint32_t node = node0 + mb + uint32_t(__popcll(bm & lt));
      out.cost[node] = ploc_merge(out, int(node), tlo, thi, ca, blo, bhi, cb, &tlo, &thi);
    }
    if (keep) {
      const uint32_t pos = pos0 + kb + uint32_t(__popcll(bk & lt));
      olo[pos] = tlo;
      ohi[pos] = thi;
    }
    pos0 += kt;
    node0 += mt;
  }
}

// Triangle records in leaf order, and zeros over the part of the node area that the tree may leave unused, so
// that every build of a scene stores the same bytes.
struct PackArgs {
  const float* tris;
  const uint32_t* mat;
  const uint32_t* order;  // null: input order
  int64_t T;
  float4* recs;
  float4* nodes;
  int64_t node_float4;
};

__device__ inline void pack_scene(const PackArgs& a, int64_t first, int64_t step) {
  for (int64_t i = first; i < a.T; i += step) {
    const uint32_t id = a.order ? a.order[i] : uint32_t(i);
    const float* p = a.tris + 9 * int64_t(id);
    const float v0x = p[0], v0y = p[1], v0z = p[2];
    a.recs[3 * i + 0] = make_float4(v0x, v0y, v0z, __int_as_float(int(id)));
    a.recs[3 * i + 1] = make_float4(p[3] - v0x, p[4] - v0y, p[5] - v0z, __int_as_float(int(a.mat[id])));
    a.recs[3 * i + 2] = make_float4(p[6] - v0x, p[7] - v0y, p[8] - v0z, 0.f);
  }
  for (int64_t i = first; i < a.node_float4; i += step) a.nodes[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ __launch_bounds__(kBlock) void k_pack(PackArgs a) {
  pack_scene(a, int64_t(blockIdx.x) * kBlock + threadIdx.x, int64_t(gridDim.x) * kBlock);
}

// A workgroup's barrier for what passes through LDS.  __syncthreads also waits until memory has taken the
// stores so far, which nothing in the launch reads back.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The searches of positions i0 and i0 + 1 among the kPlocRadius positions above each, by lane `sub` of the 2^LOG2 that
// share them, ties to the first; `below` takes what they find for those positions (see k_ploc_nn_pairs).
template <int LOG2>
__device__ __attribute__((always_inline)) inline void search_pair(const float4* lo, const float4* hi,
                                                                  unsigned long long* below, int i0, int sub, float* best0,
                                                                  int* bk0, float* best1, int* bk1) {
  constexpr int R = kPlocRadius, kSteps = (R + 1 + (1 << LOG2) - 1) >> LOG2;
  auto f3 = [](float4 v) { return make_float3(v.x, v.y, v.z); };
  const float3 lo0 = f3(lo[i0]), hi0 = f3(hi[i0]), lo1 = f3(lo[i0 + 1]), hi1 = f3(hi[i0 + 1]);
#pragma unroll 4
  for (int k = 0; k < kSteps; ++k) {
    const int d = 1 + sub + (k << LOG2);
    if (d > R + 1) break;
    const float3 l = f3(lo[i0 + d]), h = f3(hi[i0 + d]);
    // i0 reaches d = 1 .. R, i0 + 1 reaches d = 2 .. R + 1
    const float a0 = d <= R ? merged_area_raw(lo0, hi0, l, h) : INFINITY;
    const float a1 = d >= 2 ? merged_area_raw(lo1, hi1, l, h) : INFINITY;
    if (a0 < *best0) *best0 = a0, *bk0 = d;
    if (a1 < *best1) *best1 = a1, *bk1 = d - 1;
    const unsigned long long word = (static_cast<unsigned long long>(__float_as_uint(a1 < a0 ? a1 : a0)) << 32) |
                                    uint32_t(a1 < a0 ? i0 + 1 : i0);
    __hip_atomic_fetch_min(&below[i0 + d], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// The remaining rounds of at most kPlocTail clusters, in one workgroup: a round costs a search whose candidates are
// split over as many lanes as there are to spare, and four barriers.  It is bound by the search, with one CU's VALU: each
// area is computed once, for both of its clusters, by lanes that hold two neighbours, with loads four candidates
// ahead.  10k triangles, 30 rounds: 136 us with a bounds check and a wait a candidate, shuffles through LDS and barriers
// that wait for stores; 115 without those; 101 with the areas shared.
// The launch's other workgroups pack the triangles meanwhile (77 us as a launch of its own, for 3.4M).
__global__ __launch_bounds__(kPlocTail) void k_ploc_tail(Clusters c, BuildState* state, int slot, PlocNodes out,
                                                         PackArgs pack) {
  constexpr int R = kPlocRadius, kW = kPlocTail / 64;
  __shared__ float4 p_lo[kPlocTail + 2 * R], p_hi[kPlocTail + 2 * R], s_cost[kPlocTail];
  __shared__ unsigned long long s_below[kPlocTail + 2 * R];  // a position's best partner below
  __shared__ int s_nn[kPlocTail];
  __shared__ uint32_t wkeep[kW], wmerge[kW];
  if (blockIdx.x > 0) {
    pack_scene(pack, int64_t(blockIdx.x - 1) * kPlocTail + threadIdx.x, int64_t(gridDim.x - 1) * kPlocTail);
    return;
  }
  BuildState::Ploc st = state->ploc[slot];
  if (st.n > kPlocTail || st.n < 2) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Boxes at +inf before the first cluster and after the last: any merge with them has an infinite area.
  const float4 nowhere = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
  float4 *const s_lo = p_lo + R, *const s_hi = p_hi + R;
  if (tid < R) p_lo[tid] = p_hi[tid] = s_lo[st.n + tid] = s_hi[st.n + tid] = nowhere;
  s_below[tid] = ~0ull;
  if (tid < int(st.n)) {
    const float4 lo = lo_of(c, st.buf)[tid], hi = hi_of(c, st.buf)[tid];
    s_lo[tid] = lo;
    s_hi[tid] = hi;
    s_cost[tid] = ploc_cost(out, lo, hi);
  }
  __syncthreads();
  bool bad = false;
  int n = int(st.n), next = int(st.next);
  while (n > 1) {  // every round merges a pair, or ends the loop
    int log2l = 1;  // lanes to a pair of positions
    while (log2l < 5 && (n + 1) << log2l <= kPlocTail) ++log2l;
    const int sub = tid & ((1 << log2l) - 1), i0 = (tid >> log2l) * 2;
    float best0 = INFINITY, best1 = INFINITY;
    int bk0 = 0, bk1 = 0;
    if (i0 < n) {
      switch (log2l) {
        case 1: search_pair<1>(s_lo, s_hi, s_below, i0, sub, &best0, &bk0, &best1, &bk1); break;
        case 2: search_pair<2>(s_lo, s_hi, s_below, i0, sub, &best0, &bk0, &best1, &bk1); break;
        case 3: search_pair<3>(s_lo, s_hi, s_below, i0, sub, &best0, &bk0, &best1, &bk1); break;
        case 4: search_pair<4>(s_lo, s_hi, s_below, i0, sub, &best0, &bk0, &best1, &bk1); break;
        default: search_pair<5>(s_lo, s_hi, s_below, i0, sub, &best0, &bk0, &best1, &bk1); break;
      }
    }
    nearer_half<0>(&best0, &bk0), nearer_half<0>(&best1, &bk1);
    if (log2l > 1) nearer_half<1>(&best0, &bk0), nearer_half<1>(&best1, &bk1);
    if (log2l > 2) nearer_half<2>(&best0, &bk0), nearer_half<2>(&best1, &bk1);
    if (log2l > 3) nearer_half<3>(&best0, &bk0), nearer_half<3>(&best1, &bk1);
    if (log2l > 4) nearer_half<4>(&best0, &bk0), nearer_half<4>(&best1, &bk1);
    lds_barrier();
    const int i = i0 + sub;
    if (sub < 2 && i < n) {
      float best = sub == 0 ? best0 : best1;
      int bk = sub == 0 ? bk0 : bk1;
      const unsigned long long w = s_below[i];
      const float area = __uint_as_float(uint32_t(w >> 32));
      if (area < INFINITY && area <= best) best = area, bk = int(uint32_t(w)) - i;  // the smaller position
      if (!(best < INFINITY)) bk = i > 0 ? -1 : 1;
      const int p = i ^ 1;
      if (p < n && ploc_takes_parity(best, s_lo[i], s_hi[i], s_lo[p], s_hi[p])) bk = p - i;
      s_nn[i] = i + bk;
    }
    lds_barrier();
    const int j = tid < n ? s_nn[tid] : -1;
    const bool mutual = tid < n && s_nn[j] == tid;
    const bool merge = mutual && j > tid, keep = tid < n && !(mutual && j < tid);
    const uint64_t bkeep = __ballot(keep), bmerge = __ballot(merge);
    if (lane == 0) wkeep[wave] = uint32_t(__popcll(bkeep)), wmerge[wave] = uint32_t(__popcll(bmerge));
    float4 lo, hi, cost, blo, bhi, bcost;
    if (keep) lo = s_lo[tid], hi = s_hi[tid], cost = s_cost[tid];
    if (merge) blo = s_lo[j], bhi = s_hi[j], bcost = s_cost[j];
    lds_barrier();
    int kb = 0, mb = 0, mt = 0;
    for (int w = 0; w < kW; ++w) {
      const int x = int(wkeep[w]), y = int(wmerge[w]);
      if (w < wave) kb += x, mb += y;
      mt += y;
    }
    if (mt == 0 || mt > next) {
      bad = true;
      break;
    }
    next -= mt;
    n -= mt;
    const uint64_t lt = lanemask_lt();
    if (merge) cost = ploc_merge(out, next + mb + __popcll(bmerge & lt), lo, hi, cost, blo, bhi, bcost, &lo, &hi);
    if (keep) {
      const int pos = kb + __popcll(bkeep & lt);
      s_lo[pos] = lo;
      s_hi[pos] = hi;
      s_cost[pos] = cost;
    }
    if (tid < R) s_lo[n + tid] = s_hi[n + tid] = nowhere;
    s_below[tid] = ~0ull;
    lds_barrier();
  }
  if (tid == 0) {
    bad = bad || next != 0;
    if (bad) atomicOr(&state->error, 1u);
    state->ploc[0].n = state->ploc[1].n = bad ? 0u : 1u;
  }
}

// ---------------------------------------------------------------------------------------------
// 8. Collapse into a 4-wide BVH, top-down one level at a time.  A BVH4 node takes a binary node's two
// children and opens some of them into their own children (keeping left-to-right order) where the
// cost table says, so it holds up to four.  Internal children become the next level's nodes; their
// indices come from a prefix sum, so the layout is deterministic and each level's nodes are
// contiguous.  A tree has 11 (10k triangles) to 17 levels (3.4M); their sizes stay on the device, as the
// clustering's do.
// ---------------------------------------------------------------------------------------------

constexpr int kWideEmpty = INT32_MIN;
constexpr int kWideBlocks = 1024;  // most blocks of a level: each sums the others' counts
constexpr int kWideTail = 1024;    // a level of at most this many nodes is done by the one-workgroup kernel,
constexpr int kWideSmall = 4096;   // of at most this many in a tree of at most kWideSmallTree triangles (2k / 10k /
                                   // 15k triangles: 499 / 587 / 615 us with launches a level, 478 / 573 / 620 without)
constexpr int64_t kWideSmallTree = 12288;

struct WideArgs {
  const int4* made;           // per binary node: children and the cost-optimal cut
  const float4* nodebox;
  const float4* leaf_lo;
  const float4* leaf_hi;
  const uint32_t* sorted_ids; // null: the leaf boxes are in leaf order
  int2* frontier[2];          // (binary node, BVH4 index) of level l's nodes in frontier[l & 1]
  int4* sel;                  // chosen binary-tree references per frontier item
  uint32_t* counts;           // internal children of a block's items
  float4* nodes;
  uint32_t max_nodes;         // T - 1
  uint32_t tail;              // kWideTail or kWideSmall
  BuildState* state;
};

// The up to four binary-tree references that BVH4 node of binary node `bin` holds; returns how many are
// internal.
__device__ inline uint32_t wide_select(const WideArgs& a, int bin, int (&out)[4]) {
  const int4 ch = a.made[bin];
  int r[4] = {ch.x, ch.y, kWideEmpty, kWideEmpty};
  int cnt = 2;
  // follow the cost-optimal cut: the node's four slots split k : 4 - k between its children, and a
  // child with j > 1 slots is opened when that is cheaper
  int js[4] = {int((uint32_t(ch.z) >> 6) & 3u), 0, 0, 0};
  js[1] = 4 - js[0];
  // (children, choice bits) of a reference that has slots to open into, read when it gets them: the reads of both
  // children overlap, and an opened one's children are there already
  auto record = [&](int ref, int slots) {
    return ref >= 0 && slots > 1 ? a.made[ref] : make_int4(0, 0, 0, 0);
  };
  int4 m[4] = {record(r[0], js[0]), record(r[1], js[1]), make_int4(0, 0, 0, 0), make_int4(0, 0, 0, 0)};
  for (int step = 0; step < 2; ++step) {
    int p = -1;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (p < 0 && k < cnt && r[k] >= 0 && js[k] > 1 && ((uint32_t(m[k].z) >> (3 * (js[k] - 2) + 2)) & 1u)) p = k;
    if (p < 0) break;
    int4 c = m[0];
    int jj = js[0];
#pragma unroll
    for (int k = 1; k < 4; ++k)
      if (k == p) c = m[k], jj = js[k];
    const int kk = int((uint32_t(c.z) >> (3 * (jj - 2))) & 3u);
    const int4 mx = step == 0 ? record(c.x, kk) : c, my = step == 0 ? record(c.y, jj - kk) : c;
#pragma unroll
    for (int k = 3; k > 0; --k)
      if (k > p + 1 && k <= cnt) {
        r[k] = r[k - 1];
        js[k] = js[k - 1];
        m[k] = m[k - 1];
      }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k == p) {
        r[k] = c.x;
        js[k] = kk;
        m[k] = mx;
      }
      if (k == p + 1) {
        r[k] = c.y;
        js[k] = jj - kk;
        m[k] = my;
      }
    }
    ++cnt;
  }
  uint32_t n = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    out[k] = r[k];
    n += (r[k] >= 0) ? 1u : 0u;
  }
  return n;
}

// The next FP64 value above x >= 0, and below x >= 0 (0 stays 0).
__device__ inline double next_double_up(double x) { return __longlong_as_double(__double_as_longlong(x) + 1); }
__device__ inline double next_double_down(double x) {
  return x == 0.0 ? 0.0 : __longlong_as_double(__double_as_longlong(x) - 1);
}

// The smallest e >= -126 with 255 * 2^e >= ext, for ext > 0: with ext = m 2^k, 1 <= m < 2, and
// 255 = 1.9921875 * 2^7, it is k - 7, or k - 6 where m > 1.9921875.
__device__ inline int grid_exponent(double ext) {
  const uint64_t bits = uint64_t(__double_as_longlong(ext));
  const int k = int(bits >> 52) - 1023;
  const int e = k - 7 + ((bits & 0xfffffffffffffull) > 0xfe00000000000ull ? 1 : 0);
  return e < -126 ? -126 : e;
}

// Writes BVH4 node `b4` with children r; its internal children are BVH4 nodes first, first + 1, ... and
// entries slot, slot + 1, ... of the next level, which put(entry, (binary node, BVH4 index)) takes.
template <class Put>
__device__ inline void wide_emit(const WideArgs& a, float p, int b4, const int (&r)[4], uint32_t first, uint32_t slot,
                                 Put put) {
  float lo[3][4], hi[3][4];
  int ref[4];
  uint32_t k_int = 0;
  
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float4 l, h;
    if (r[k] == kWideEmpty) {
      // an empty slot: a box at +inf on every axis misses every ray in the slab test
      l = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
      h = l;
      ref[k] = 0;
    } else if (r[k] < 0) {
      const uint32_t id = a.sorted_ids ? a.sorted_ids[~r[k]] : uint32_t(~r[k]);
      l = a.leaf_lo[id];
      h = a.leaf_hi[id];
      l = make_float4(l.x - p, l.y - p, l.z - p, 0.f);
      h = make_float4(h.x + p, h.y + p, h.z + p, 0.f);
      ref[k] = ~((~r[k]) << 2);
    } else {
      l = a.nodebox[2 * r[k]];
      h = a.nodebox[2 * r[k] + 1];
      l = make_float4(l.x - p, l.y - p, l.z - p, 0.f);
      h = make_float4(h.x + p, h.y + p, h.z + p, 0.f);
      const int idx = int(first + k_int);
      put(slot + k_int, make_int2(r[k], idx));
      ++k_int;
      ref[k] = idx;
    }
    lo[0][k] = l.x, lo[1][k] = l.y, lo[2][k] = l.z;
    hi[0][k] = h.x, hi[1][k] = h.y, hi[2][k] = h.z;
  }
#if SRT_QNODE
  // Quantise the children's boxes on the node's own grid: per axis a power-of-two step s with
  // 255 s >= the node's extent, lower corners rounded down and upper corners rounded up.  The
  // differences are formed in FP64 and nudged outwards by one FP64 ulp, so the exact grid box always
  // contains the padded FP32 box.  The node stores 2^24 s (the traversal reads each grid byte as the
  // FP16 value q 2^-24); s >= 2^-126 and, with vertices within RT_MAX_COORD, s <= 2^34, so 2^24 s
  // is a normal float.
  float plo[3], phi[3];
  for (int ax = 0; ax < 3; ++ax) {
    plo[ax] = INFINITY;
    phi[ax] = -INFINITY;
    for (int k = 0; k < 4; ++k)
      if (r[k] != kWideEmpty) {
        plo[ax] = fminf(plo[ax], lo[ax][k]);
        phi[ax] = fmaxf(phi[ax], hi[ax][k]);
      }
  }
  uint32_t qlo[3] = {0u, 0u, 0u}, qhi[3] = {0u, 0u, 0u};
  float steps[3];
  for (int ax = 0; ax < 3; ++ax) {
    const double base = double(plo[ax]);
    const double ext = next_double_up(double(phi[ax]) - base);
    const int e = grid_exponent(ext);
    steps[ax] = __uint_as_float(uint32_t(e + 24 + 127) << 23);  // 2^(e + 24)
    for (int k = 0; k < 4; ++k) {
      uint32_t ql = 255u, qh = 0u;
      if (r[k] != kWideEmpty) {
        const double dl = double(lo[ax][k]) - base, dh = double(hi[ax][k]) - base;  // both >= 0
        ql = uint32_t(fmin(floor(ldexp(next_double_down(dl), -e)), 255.0));
        qh = uint32_t(fmin(ceil(ldexp(next_double_up(dh), -e)), 255.0));
      }
      qlo[ax] |= ql << (8 * k);
      qhi[ax] |= qh << (8 * k);
    }
  }
  for (int k = 1; k < 4; ++k)
    if (r[k] == kWideEmpty) ref[k] = ref[0];
  float4* out = a.nodes + 4 * int64_t(b4);
  out[0] = make_float4(plo[0], plo[1], plo[2], steps[0]);
  out[1] = make_float4(__int_as_float(ref[0]), __int_as_float(ref[1]), __int_as_float(ref[2]), __int_as_float(ref[3]));
  out[2] = make_float4(__uint_as_float(qlo[0]), __uint_as_float(qhi[0]), __uint_as_float(qlo[1]), __uint_as_float(qhi[1]));
  out[3] = make_float4(__uint_as_float(qlo[2]), __uint_as_float(qhi[2]), steps[1], steps[2]);
#else
  float4* out = a.nodes + 8 * int64_t(b4);
  out[0] = make_float4(lo[0][0], lo[0][1], lo[0][2], lo[0][3]);
  out[1] = make_float4(hi[0][0], hi[0][1], hi[0][2], hi[0][3]);
  out[2] = make_float4(lo[1][0], lo[1][1], lo[1][2], lo[1][3]);
  out[3] = make_float4(hi[1][0], hi[1][1], hi[1][2], hi[1][3]);
  out[4] = make_float4(lo[2][0], lo[2][1], lo[2][2], lo[2][3]);
  out[5] = make_float4(hi[2][0], hi[2][1], hi[2][2], hi[2][3]);
  out[6] = make_float4(__int_as_float(ref[0]), __int_as_float(ref[1]), __int_as_float(ref[2]), __int_as_float(ref[3]));
  out[7] = make_float4(0.f, 0.f, 0.f, 0.f);
#endif
}

// Conservative box growth (slab and triangle-test rounding).
__device__ inline float wide_pad(const Bounds6& b) {
  float m = 0.f;
  for (int k = 0; k < 3; ++k) m = fmaxf(m, fmaxf(fabsf(b.blo[k]), fabsf(b.bhi[k])));
  return m * 0x1p-18f + 1e-20f;
}

// One level, first half: the cut of every node, and each block's count of the next level's nodes.
__global__ __launch_bounds__(kBlock) void k_wide_select(WideArgs a, int slot) {
  __shared__ uint32_t tmp[kBlock / 64];
  const BuildState::Wide st = a.state->wide[slot];
  if (st.m <= a.tail) return;
  const int2* frontier = (st.level & 1) ? a.frontier[1] : a.frontier[0];
  uint32_t begin, end, n = 0;
  ploc_range(st.m, kBlock, blockIdx.x, gridDim.x, &begin, &end);
  for (uint32_t i = begin + threadIdx.x; i < end; i += kBlock) {
    int r[4];
    n += wide_select(a, frontier[i].x, r);
    a.sel[i] = make_int4(r[0], r[1], r[2], r[3]);
  }
  n = block_sum(n, tmp);
  if (threadIdx.x == 0) a.counts[blockIdx.x] = n;
}

// Second half: the nodes, and the next level's entries.
__global__ __launch_bounds__(kBlock) void k_wide_emit(WideArgs a, int slot) {
  __shared__ uint32_t tmp[kBlock / 64];
  __shared__ uint32_t wcnt[2][kBlock / 64];
  const BuildState::Wide st = a.state->wide[slot];
  BuildState::Wide* out = &a.state->wide[slot ^ 1];
  if (st.m <= a.tail) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *out = st;
    return;
  }
  const int2* frontier = (st.level & 1) ? a.frontier[1] : a.frontier[0];
  int2* next = (st.level & 1) ? a.frontier[0] : a.frontier[1];
  uint32_t begin, end, before = 0, total = 0;
  ploc_range(st.m, kBlock, blockIdx.x, gridDim.x, &begin, &end);
  for (uint32_t k = threadIdx.x; k < gridDim.x; k += kBlock) {
    const uint32_t v = a.counts[k];
    total += v;
    if (k < blockIdx.x) before += v;
  }
  before = block_sum(before, tmp), total = block_sum(total, tmp);
  const bool bad = total > a.max_nodes - st.allocated;  // every level adds nodes: impossible for a valid tree
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (bad) atomicOr(&a.state->error, 2u);
    *out = BuildState::Wide{bad ? 0u : total, st.allocated + (bad ? 0u : total), st.level + 1u, 0u};
  }
  if (bad) return;
  const float pad = wide_pad(a.state->bounds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int par = 0;
  for (uint32_t base = begin; base < end; base += kBlock, par ^= 1) {
    const uint32_t i = base + threadIdx.x;
    const bool valid = i < end;
    int r[4] = {kWideEmpty, kWideEmpty, kWideEmpty, kWideEmpty};
    if (valid) {
      const int4 s4 = a.sel[i];
      r[0] = s4.x, r[1] = s4.y, r[2] = s4.z, r[3] = s4.w;
    }
    uint32_t n = 0;
    for (int k = 0; k < 4; ++k) n += r[k] >= 0 ? 1u : 0u;
    uint32_t scan = n;  // inclusive over the wave
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t u = __shfl_up(scan, off);
      if (lane >= off) scan += u;
    }
    if (lane == 63) wcnt[par][wave] = scan;
    __syncthreads();
    uint32_t wb = 0, all = 0;
    for (int w = 0; w < kBlock / 64; ++w) {
      if (w < wave) wb += wcnt[par][w];
      all += wcnt[par][w];
    }
    const uint32_t off = before + wb + scan - n;
    if (valid)
      wide_emit(a, pad, frontier[i].y, r, st.allocated + off, off, [&](uint32_t e, int2 v) { next[e] = v; });
    before += all;
  }
}

// Every level of at most a.tail nodes from the state's level on, in one workgroup: the top of the tree before the wide
// levels, and what is left after them.  A level is a chain of dependent reads (a node's record, its children's, the
// chosen children's boxes); its entries pass to the next one through LDS, also written to memory for the launch that
// takes over, and no barrier waits for a store.
__global__ __launch_bounds__(kWideTail) void k_wide_levels(WideArgs a, int slot) {
  constexpr int kW = kWideTail / 64;
  __shared__ int2 entries[2][kWideSmall];
  __shared__ uint32_t wcnt[kW];
  BuildState::Wide st = a.state->wide[slot];
  if (a.state->ploc[0].n != 1 || a.state->ploc[1].n != 1) return;  // the binary tree is not complete yet
  const float pad = wide_pad(a.state->bounds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool bad = false;
  if (st.m <= a.tail) {
    const int2* frontier = (st.level & 1) ? a.frontier[1] : a.frontier[0];
    for (uint32_t i = threadIdx.x; i < st.m; i += kWideTail) entries[st.level & 1][i] = frontier[i];
  }
  __syncthreads();
  while (st.m > 0 && st.m <= a.tail && !bad) {  // allocated grows with every level and is bounded
    int2* next = (st.level & 1) ? a.frontier[0] : a.frontier[1];
    int2* next_lds = entries[(st.level & 1) ^ 1];
    uint32_t total = 0;
    for (uint32_t base = 0; base < st.m && !bad; base += kWideTail) {
      const bool valid = base + threadIdx.x < st.m;
      int r[4] = {kWideEmpty, kWideEmpty, kWideEmpty, kWideEmpty};
      int2 item = make_int2(0, 0);
      uint32_t n = 0;
      if (valid) {
        item = entries[st.level & 1][base + threadIdx.x];
        n = wide_select(a, item.x, r);
      }
      uint32_t scan = n;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(scan, off);
        if (lane >= off) scan += u;
      }
      if (lane == 63) wcnt[wave] = scan;
      lds_barrier();
      uint32_t before = total;
      for (int w = 0; w < kW; ++w) {
        if (w < wave) before += wcnt[w];
        total += wcnt[w];
      }
      bad = total > a.max_nodes - st.allocated;
      const uint32_t off = before + scan - n;
      if (valid && !bad)
        wide_emit(a, pad, item.y, r, st.allocated + off, off, [&](uint32_t e, int2 v) {
          next[e] = v;
          if (e < uint32_t(kWideSmall)) next_lds[e] = v;
        });
      lds_barrier();  // the next level's entries are written, wcnt is free
    }
    if (bad) break;
    st.m = total;
    st.allocated += total;
    ++st.level;
  }
  if (threadIdx.x == 0) {
    if (bad) {
      atomicOr(&a.state->error, 2u);
      st.m = 0;
    }
    a.state->wide[slot] = st;
  }
}

// The state a build starts from.  ploc_clusters: 1 with the Karras tree, whose nodes are made elsewhere.
__global__ void k_build_init(BuildState* s, uint32_t ploc_clusters, int2* frontier0) {
  if (threadIdx.x != 0) return;
  s->status = 0;
  s->error = 0;
  for (int k = 0; k < 2; ++k) {
    s->ploc[k] = BuildState::Ploc{ploc_clusters, ploc_clusters - 1u, 0u, 0u};
    s->wide[k] = BuildState::Wide{1u, 1u, 0u, 0u};
  }
  for (int k = 0; k < 3; ++k) s->bounds.clo[k] = s->bounds.chi[k] = s->bounds.blo[k] = s->bounds.bhi[k] = 0.f;
  if (frontier0) *frontier0 = make_int2(0, 0);
}

template <typename T>
__global__ void k_fill(T* p, T v, int64_t n) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

inline unsigned blocks_for(int64_t n, int b = kBlock) { return unsigned((n + b - 1) / b); }

}  // namespace

BuildPlan plan_build(int64_t T, int64_t S, int64_t P, int64_t M, int64_t L, bool bvh, bool ploc) {
  BuildPlan p{};
  p.T = T;
  p.bvh = bvh && T >= 2;
  p.ploc = ploc;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  int64_t num_nodes = p.bvh ? T - 1 : 0;  // an upper bound for the 4-wide tree
  p.nodes_off = take(size_t(num_nodes) * kNodeBytes);
  p.tris_off = take(size_t(T) * 48);
  p.spheres_off = take(size_t(S) * 16);
  p.sphere_mat_off = take(size_t(S) * 4);
  p.planes_off = take(size_t(P) * 16);
  p.plane_mat_off = take(size_t(P) * 4);
  p.mats_off = take(size_t(M) * 48);
  p.lights_off = take(size_t(L) * 32 + 32);
  p.storage_bytes = off;

  off = 0;
  p.num_blocks_prep = (T + kBlock - 1) / kBlock;
  const int64_t sort_tile = int64_t(kBlock) * (T < kSortFew ? kSortItemsFew : kSortItems);
  p.num_sort_blocks = (T + sort_tile - 1) / sort_tile;
  p.status_off = take(256);
  p.partial_off = take(size_t(p.num_blocks_prep > 0 ? p.num_blocks_prep : 1) * sizeof(Bounds6));
  if (T > 0) {
    p.lo_off = take(size_t(T) * 16);
    p.hi_off = take(size_t(T) * 16);
  }
  if (p.bvh) {
    p.keys0_off = take(size_t(T) * 8);
    p.keys1_off = take(size_t(T) * 8);
    p.ids0_off = take(size_t(T) * 4);
    p.ids1_off = take(size_t(T) * 4);
    p.hist_off = take(size_t(p.num_sort_blocks) * kRadix * 4);
    p.made_off = take(size_t(T) * 16);
    p.nodebox_off = take(size_t(T) * 32);
    if (!ploc) {
      p.range_off = take(size_t(T) * 8);
      p.parent_off = take(size_t(2 * T) * 4);
      p.flags_off = take(size_t(T) * 4);
    }
    p.frontier_off[0] = take(size_t(T) * 8);
    p.frontier_off[1] = take(size_t(T) * 8);
    p.sel_off = take(size_t(T) * 16);
    p.dp_cost_off = p.sel_off;  // the costs are of no use to the collapse
    p.digit_totals_off = take(size_t(kRadix) * 4);
    p.counts_off = take(size_t(std::max(kPlocBlocks, kWideBlocks)) * 8);
    if (ploc) {
      for (int k = 0; k < 2; ++k) {
        p.ploc_lo_off[k] = take(size_t(T) * 16);
        p.ploc_hi_off[k] = take(size_t(T) * 16);
      }
      p.ploc_partner_off = take(size_t(T) * 4);
    }
  }
  p.scratch_bytes = off;
  return p;
}

hipError_t build_scene_device(const rt_scene_desc* desc, const BuildPlan& plan, char* storage, char* scratch,
                              hipStream_t stream, BuildResult* result) {
  const int64_t T = desc->num_triangles;
  const int S = desc->num_spheres, P = desc->num_planes, M = desc->num_materials, L = desc->num_lights;
  BuildState* state = reinterpret_cast<BuildState*>(scratch + plan.status_off);
  uint32_t* status = &state->status;
  hipError_t e;
#define SRT_CHECK(x)                   \
  do {                                 \
    e = (x);                           \
    if (e != hipSuccess) return e;     \
  } while (0)
#define SRT_LAUNCH_CHECK() SRT_CHECK(hipGetLastError())

  k_build_init<<<1, 64, 0, stream>>>(state, plan.bvh && plan.ploc ? uint32_t(T) : 1u,
                                     plan.bvh ? reinterpret_cast<int2*>(scratch + plan.frontier_off[0]) : nullptr);
  SRT_LAUNCH_CHECK();

  // spheres, planes, materials, lights
  if (S > 0) {
    SRT_CHECK(hipMemcpyAsync(storage + plan.spheres_off, desc->spheres, size_t(S) * 16, hipMemcpyDeviceToDevice, stream));
    SRT_CHECK(hipMemcpyAsync(storage + plan.sphere_mat_off, desc->sphere_material, size_t(S) * 4,
                             hipMemcpyDeviceToDevice, stream));
  }
  if (P > 0) {
    SRT_CHECK(hipMemcpyAsync(storage + plan.planes_off, desc->planes, size_t(P) * 16, hipMemcpyDeviceToDevice, stream));
    SRT_CHECK(hipMemcpyAsync(storage + plan.plane_mat_off, desc->plane_material, size_t(P) * 4,
                             hipMemcpyDeviceToDevice, stream));
  }
  if (S + P > 0) {
    k_check_spheres_planes<<<blocks_for(S + P), kBlock, 0, stream>>>(desc->spheres, desc->sphere_material, S,
                                                                     desc->planes, desc->plane_material, P, M, status);
    SRT_LAUNCH_CHECK();
  }
  {
    // materials: (kd, n), (ks, 0), (kr, 0); lights: (pos, 0), (I, 0)
    size_t mb = size_t(M) * 48, lb = size_t(L) * 32;
    float* host = static_cast<float*>(std::malloc(mb + lb + 16));
    if (!host) return hipErrorOutOfMemory;
    for (int i = 0; i < M; ++i) {
      const rt_material& m = desc->materials[i];
      float* o = host + 12 * i;
      o[0] = m.albedo[0], o[1] = m.albedo[1], o[2] = m.albedo[2], o[3] = m.shininess;
      o[4] = m.specular[0], o[5] = m.specular[1], o[6] = m.specular[2], o[7] = 0.f;
      o[8] = m.reflectance[0], o[9] = m.reflectance[1], o[10] = m.reflectance[2], o[11] = 0.f;
    }
    for (int i = 0; i < L; ++i) {
      const rt_light& l = desc->lights[i];
      float* o = host + 12 * M + 8 * i;
      o[0] = l.position[0], o[1] = l.position[1], o[2] = l.position[2], o[3] = 0.f;
      o[4] = l.intensity[0], o[5] = l.intensity[1], o[6] = l.intensity[2], o[7] = 0.f;
    }
    e = hipMemcpyAsync(storage + plan.mats_off, host, mb, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && lb)
      e = hipMemcpyAsync(storage + plan.lights_off, reinterpret_cast<char*>(host) + mb, lb, hipMemcpyHostToDevice,
                         stream);
    // pageable source: wait before freeing it
    hipError_t e2 = hipStreamSynchronize(stream);
    std::free(host);
    SRT_CHECK(e);
    SRT_CHECK(e2);
  }

  result->depth = 0;
  result->max_leaf = T > 0 ? 1 : 0;
  result->num_nodes = 0;
  result->root = 0;
  for (int a = 0; a < 3; ++a) result->lo[a] = result->hi[a] = 0.f;

  float4* recs = reinterpret_cast<float4*>(storage + plan.tris_off);
  BuildState done{};
  if (T > 0) {
    float4* lo = reinterpret_cast<float4*>(scratch + plan.lo_off);
    float4* hi = reinterpret_cast<float4*>(scratch + plan.hi_off);
    Bounds6* partial = reinterpret_cast<Bounds6*>(scratch + plan.partial_off);
    k_tri_prep<<<blocks_for(T), kBlock, 0, stream>>>(desc->triangles, desc->tri_material, T, M, lo, hi, partial,
                                                     status);
    SRT_LAUNCH_CHECK();
    PackArgs pack{desc->triangles, desc->tri_material, nullptr, T, recs, nullptr, 0};
    k_reduce_bounds<<<1, kBlock, 0, stream>>>(partial, plan.num_blocks_prep, &state->bounds);
    SRT_LAUNCH_CHECK();

    if (plan.bvh) {
      uint64_t* k0 = reinterpret_cast<uint64_t*>(scratch + plan.keys0_off);
      uint64_t* k1 = reinterpret_cast<uint64_t*>(scratch + plan.keys1_off);
      uint32_t* i0 = reinterpret_cast<uint32_t*>(scratch + plan.ids0_off);
      uint32_t* i1 = reinterpret_cast<uint32_t*>(scratch + plan.ids1_off);
      uint32_t* hist = reinterpret_cast<uint32_t*>(scratch + plan.hist_off);
      uint32_t* totals = reinterpret_cast<uint32_t*>(scratch + plan.digit_totals_off);
      k_morton<<<blocks_for(T), kBlock, 0, stream>>>(lo, hi, &state->bounds, T, k0, i0);
      SRT_LAUNCH_CHECK();
      if (T <= kRankMost) {
        k_rank_sort<<<unsigned((T + 63) / 64), kRankBlock, 0, stream>>>(k0, int(T), k1, i1);
        SRT_LAUNCH_CHECK();
        std::swap(k0, k1);
        std::swap(i0, i1);
      }
      for (int pass = T <= kRankMost ? 8 : 0; pass < 8; ++pass) {
        const int shift = pass * kRadixBits;
        SRT_CHECK(T < kSortFew ? sort_pass<kSortItemsFew>(k0, i0, T, shift, hist, totals, k1, i1, stream)
                               : sort_pass<kSortItems>(k0, i0, T, shift, hist, totals, k1, i1, stream));
        std::swap(k0, k1);
        std::swap(i0, i1);
      }
      pack.order = i0;
      // a node has at most four children, so the tree has at least (T - 1) / 3 of the T - 1 nodes
      const size_t zero_from = plan.nodes_off + size_t((T - 1) / 3) * kNodeBytes;
      pack.nodes = reinterpret_cast<float4*>(storage + zero_from);
      pack.node_float4 = int64_t((plan.tris_off - zero_from) / 16);
      int4* tree = reinterpret_cast<int4*>(scratch + plan.made_off);
      int2* range = reinterpret_cast<int2*>(scratch + plan.range_off);
      int32_t* parent = reinterpret_cast<int32_t*>(scratch + plan.parent_off);
      uint32_t* flags = reinterpret_cast<uint32_t*>(scratch + plan.flags_off);
      float4* nodebox = reinterpret_cast<float4*>(scratch + plan.nodebox_off);
      float4* dp_cost = reinterpret_cast<float4*>(scratch + plan.dp_cost_off);
      uint2* counts = reinterpret_cast<uint2*>(scratch + plan.counts_off);
      Clusters cl{};
      int32_t* partner = nullptr;
      const PlocNodes made{tree, nodebox, dp_cost};
      bool packed = false;
      ClusterPlan rounds(T);
      const int& round = rounds.rounds;
      // `count` clustering rounds and the one-workgroup rest.  A grid made for too few clusters takes more tiles a
      // block, and a round that finds at most kPlocTail clusters does nothing.
      auto cluster = [&](int count) -> hipError_t {
        for (int k = 0; k < count; ++k, rounds.next()) {
          const bool few = rounds.expected < kPlocFew;
          const unsigned own = few ? kPlocBlock / kPlocLanes - 2 * kPlocRadius : kPairOwn;
          const unsigned grid = unsigned(rounds.blocks(own));
          if (few)
            k_ploc_nn<<<grid, kPlocBlock, 0, stream>>>(cl, state, round & 1, partner, counts);
          else
            k_ploc_nn_pairs<<<grid, kPairBlock, 0, stream>>>(cl, state, round & 1, partner, counts);
          if ((e = hipGetLastError()) != hipSuccess) return e;
          k_ploc_compact<<<grid, kBlock, 0, stream>>>(cl, state, round & 1, partner, counts, own, made);
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        const int64_t blocks = packed ? 0 : std::min<int64_t>(kPackBlocks, (T + kPlocTail - 1) / kPlocTail);
        packed = true;
        k_ploc_tail<<<unsigned(1 + blocks), kPlocTail, 0, stream>>>(cl, state, round & 1, made, pack);
        return hipGetLastError();
      };
      if (plan.ploc) {
        cl.lo0 = reinterpret_cast<float4*>(scratch + plan.ploc_lo_off[0]);
        cl.hi0 = reinterpret_cast<float4*>(scratch + plan.ploc_hi_off[0]);
        cl.lo1 = reinterpret_cast<float4*>(scratch + plan.ploc_lo_off[1]);
        cl.hi1 = reinterpret_cast<float4*>(scratch + plan.ploc_hi_off[1]);
        cl.lo2 = lo;  // the boxes in input order, free once the leaves are in theirs
        cl.hi2 = hi;
        partner = reinterpret_cast<int32_t*>(scratch + plan.ploc_partner_off);
        k_ploc_init<<<blocks_for(T), kBlock, 0, stream>>>(i0, lo, hi, T, cl);
        SRT_LAUNCH_CHECK();
        SRT_CHECK(cluster(rounds.first()));
      } else {
        k_pack<<<blocks_for(T), kBlock, 0, stream>>>(pack);
        SRT_LAUNCH_CHECK();
        k_karras<<<blocks_for(T - 1), kBlock, 0, stream>>>(k0, T, tree, parent, range);
        SRT_LAUNCH_CHECK();
        k_fill<uint32_t><<<blocks_for(T - 1), kBlock, 0, stream>>>(flags, 0u, T - 1);
        SRT_LAUNCH_CHECK();
        k_refit<<<blocks_for(T), kBlock, 0, stream>>>(tree, parent, lo, hi, i0, nodebox, flags, T, status, dp_cost);
        SRT_LAUNCH_CHECK();
      }
      WideArgs wa{};
      wa.made = tree;
      wa.nodebox = nodebox;
      wa.leaf_lo = plan.ploc ? cl.lo0 : lo;
      wa.leaf_hi = plan.ploc ? cl.hi0 : hi;
      wa.sorted_ids = plan.ploc ? nullptr : i0;
      wa.sel = reinterpret_cast<int4*>(scratch + plan.sel_off);
      wa.counts = reinterpret_cast<uint32_t*>(counts);
      wa.nodes = reinterpret_cast<float4*>(storage + plan.nodes_off);
      wa.max_nodes = uint32_t(T - 1);
      wa.tail = T <= kWideSmallTree ? kWideSmall : kWideTail;
      wa.state = state;
      for (int k = 0; k < 2; ++k) wa.frontier[k] = reinterpret_cast<int2*>(scratch + plan.frontier_off[k]);
      int level = 0;
      // the top of the tree, `levels` wide levels and what is left
      auto collapse = [&](int levels) -> hipError_t {
        k_wide_levels<<<1, kWideTail, 0, stream>>>(wa, level & 1);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const unsigned grid = unsigned(std::min<int64_t>(kWideBlocks, (T + kBlock - 1) / kBlock));
        for (int k = 0; k < levels; ++k, ++level) {
          k_wide_select<<<grid, kBlock, 0, stream>>>(wa, level & 1);
          if ((e = hipGetLastError()) != hipSuccess) return e;
          k_wide_emit<<<grid, kBlock, 0, stream>>>(wa, level & 1);
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (levels > 0) k_wide_levels<<<1, kWideTail, 0, stream>>>(wa, level & 1);
        return hipGetLastError();
      };
      // levels of more than kWideTail nodes: none for a small tree, 10 of 17 for 3.4M triangles
      const int wide_levels = T <= kWideSmallTree ? 0 : 4 + int(std::ceil(std::log2(double(T) / kWideTail) / 2));
      SRT_CHECK(collapse(wide_levels));
      for (;;) {
        SRT_CHECK(hipMemcpyAsync(&done, state, sizeof(done), hipMemcpyDeviceToHost, stream));
        SRT_CHECK(hipStreamSynchronize(stream));
        if (done.status) break;  // refused input: its tree is of no use
        if (done.error) return hipErrorUnknown;
        const bool tree = done.ploc[round & 1].n == 1;
        if (tree && done.wide[level & 1].m == 0) break;
        // an unusual tree: more rounds or levels than the launches above.  Every round merges a pair and
        // every level adds a node, so this ends.
        if (!tree) SRT_CHECK(cluster(rounds.look(int64_t(done.ploc[round & 1].n))));
        SRT_CHECK(collapse(std::max(wide_levels, 4)));
      }
      result->num_nodes = done.wide[level & 1].allocated;
      result->depth = int32_t(done.wide[level & 1].level);
      result->root = 0;
    } else {
      k_pack<<<blocks_for(T), kBlock, 0, stream>>>(pack);
      SRT_LAUNCH_CHECK();
      result->root = ~0;  // a single leaf holding record 0 (used only when T == 1)
    }
  }
  if (!plan.bvh) {
    SRT_CHECK(hipMemcpyAsync(&done, state, sizeof(done), hipMemcpyDeviceToHost, stream));
    SRT_CHECK(hipStreamSynchronize(stream));
  }
  result->status_bits = done.status;
  for (int a = 0; a < 3; ++a) {
    result->lo[a] = T > 0 ? done.bounds.blo[a] : 0.f;
    result->hi[a] = T > 0 ? done.bounds.bhi[a] : 0.f;
  }
  return hipSuccess;
#undef SRT_CHECK
#undef SRT_LAUNCH_CHECK
}

}  // namespace srt
