// Stereo Whitted ray tracing on gfx950: wavefront-persistent kernels.
//
// A pass renders a range of paths (a path = one pixel of one eye; an 8x8 tile
// of the left eye is followed by the same tile of the right eye, so both of
// the paper's parallel levels -- the two channels and the pixels inside each
// -- share one queue and one launch).  With D mirror bounces, for d = 0..D+1:
//   k_trace(d)    persistent BVH traversal of the closest-hit rays of depth d
//                 (primary rays generated in-register, FP64 rounded once to
//                 FP32) together with the shadow rays spawned at depth d-1;
//                 the two ray kinds fill one grid, so neither leaves a tail.
//                 Its last batches add the unoccluded lights' terms of depth
//                 d-2 in light order
//   k_shade(d)    Phong shading of the depth-d hits: adds the ambient (or
//                 background) term, spawns one shadow ray per light with
//                 N.L > 0 into that light's queue and a mirror ray into the
//                 next depth's queue; queues are compacted with wave ballots
//                 and one atomic per block and queue
//   k_resolve(D)  adds the terms of the last depth (of every depth, with
//                 ray-tree signatures or the timer)
// Single scenes without a tree have a traversal kernel of their own
// (k_trace_flat), and small whole frames are one launch (k_path).
// Queues and per-depth buffers are double-buffered by depth parity.  Every
// pixel's radiance is accumulated by one thread at a time in a fixed order,
// so results do not depend on queue order, pass size or concurrent work.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <type_traits>
#include <vector>

#include "rt_internal.h"

#ifndef SRT_STACK_LDS
#define SRT_STACK_LDS 16
#endif
#ifndef SRT_TRACE_WAVES_PER_EU
#define SRT_TRACE_WAVES_PER_EU 8
#endif

#ifndef SRT_FLAT_STEP
#define SRT_FLAT_STEP 4
#endif

namespace srt {
namespace {

constexpr int kBlock = kTraceBlock;
constexpr int kFlatStep = SRT_FLAT_STEP;  // primitives that the kernels for scenes without a tree load at a time
constexpr int kWalkStep = 2;              // triangles that a batch's traversal does: 4 spill 8 more registers
constexpr int kWaves = kBlock / 64;
constexpr int kStackLds = SRT_STACK_LDS;       // traversal stack entries per lane kept in LDS (power of two)
constexpr int kStackGlobal = kStackMax - kStackLds;  // older entries spill to the workspace
constexpr int kMaxTraceBlocks = 2048;
static_assert(int64_t(kMaxTraceBlocks) * kBlock * kStackGlobal < (int64_t(1) << 32), "spill area index exceeds 32 bits");
// Shading blocks are large: queue slots are reserved with one device-scope atomic per block
// iteration and queue, and atomics on one address serialise.
#ifndef SRT_SHADE_BLOCK
#define SRT_SHADE_BLOCK 512
#endif
constexpr int kShadeBlock = SRT_SHADE_BLOCK;
constexpr int kShadeWaves = kShadeBlock / 64;
static_assert((kStackLds & (kStackLds - 1)) == 0, "LDS stack size must be a power of two");
#ifndef SRT_COOP_RAYS
#define SRT_COOP_RAYS 48
#endif
constexpr int kCoopRays = SRT_COOP_RAYS;  // a wave with at most this many rays left shares them between its lanes
static_assert(kCoopRays >= 0 && kCoopRays <= 64, "one slot per lane at most");
#ifndef SRT_COOP_SHARE
#define SRT_COOP_SHARE 8
#endif
constexpr int kCoopShare = SRT_COOP_SHARE;  // a hand-over needs at least 1/kCoopShare of the busy lanes in pairs

// ---------------------------------------------------------------------------------------------
// Small vector helpers
// ---------------------------------------------------------------------------------------------

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ inline float3 f3(float4 v) { return make_float3(v.x, v.y, v.z); }
__device__ inline float3 operator+(float3 a, float3 b) { return make_float3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ inline float3 operator-(float3 a, float3 b) { return make_float3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ inline float3 operator*(float s, float3 a) { return make_float3(s * a.x, s * a.y, s * a.z); }
__device__ inline float3 mul(float3 a, float3 b) { return make_float3(a.x * b.x, a.y * b.y, a.z * b.z); }
// Sums of products with their roundings written out: kernels that compute the same value get the same bits,
// however the compiler would contract each.
__device__ inline float fdot(float3 a, float3 b) { return fmaf(a.z, b.z, fmaf(a.x, b.x, a.y * b.y)); }
__device__ inline float3 fcross(float3 a, float3 b) {
  return make_float3(fmaf(a.y, b.z, -(a.z * b.y)), fmaf(a.z, b.x, -(a.x * b.z)), fmaf(a.x, b.y, -(a.y * b.x)));
}
// a + b rounded by itself, also where a or b is a product
__device__ inline float3 add_rn(float3 a, float3 b) {
#pragma clang fp contract(off)
  return make_float3(a.x + b.x, a.y + b.y, a.z + b.z);
}
// s * a + b
__device__ inline float3 fmad(float s, float3 a, float3 b) {
  return make_float3(fmaf(s, a.x, b.x), fmaf(s, a.y, b.y), fmaf(s, a.z, b.z));
}
__device__ inline float3 normalize(float3 a) { return (1.0f / sqrtf(fdot(a, a))) * a; }

// 1/d with exact zeros replaced by a tiny same-signed value, so that the slab
// products stay finite (no 0 * inf) for axis-parallel rays.
__device__ inline float safe_rcp(float x) {
  const float tiny = 1e-20f;
  if (fabsf(x) < tiny) x = copysignf(tiny, x);
  return 1.0f / x;
}

__device__ inline int lane_id() { return threadIdx.x & 63; }

// Number of lanes of `mask` below this one.
__device__ inline int lanes_below(uint64_t mask) {
  return int(__builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u)));
}

// A pointer to global memory held in scalar registers.  The empty asm hides where it came from, so that it
// is not loaded again, and the cast around it keeps accesses through it global ones (not flat).
template <class T>
__device__ __attribute__((always_inline)) inline T* global_scalar(T* p) {
  typedef __attribute__((address_space(1))) T global_t;
  global_t* g = (global_t*)p;
  asm("" : "+s"(g));
  return (T*)g;
}

// Next float above a non-negative x (+inf stays +inf): lets a `t < tmax` test admit t == x.
__device__ inline float next_up(float x) { return x == INFINITY ? x : __int_as_float(__float_as_int(x) + 1); }

// x rounded up to a multiple of 2^log2n
__device__ inline uint32_t round_up(uint32_t x, int log2n) { return ((x + (1u << log2n) - 1u) >> log2n) << log2n; }

// ---------------------------------------------------------------------------------------------
// Kernel arguments
// ---------------------------------------------------------------------------------------------

struct KArgs {
  DevItem one;            // single render (MULTI = false)
  const DevItem* items;   // batch table (MULTI = true)
  int32_t num_items;
  int32_t lstride;        // light queues (max lights over the items)
  int32_t dmax;           // max reflection depth over the items
  Counters* ctr;
  float4* ro[2];       // mirror-ray queue by depth parity: origin + pass-local path index bits
  float4* rd[2];       // direction + excluded primitive key bits; also of the primary rays
  float4* thr[2];      // throughput of a mirror ray
  float2* hit;         // (t, key bits) of the closest-hit rays of the current depth
  uint32_t* epath[2];  // [cap]: pass-local path index of a mirror-ray entry (at depth 0 the entry's own index)
  uint8_t* smask[2];   // [cap]: lights towards which the entry has a shadow ray
  float4* spos[2];     // [cap]: origin of an entry's shadow rays, excluded key bits; written where smask is not 0
  uint32_t* sowner[2]; // [light][cap]: entries with a shadow ray towards the light, in any order
  float* contrib[2];   // [light][cap][3]: the light's term times throughput
  uint8_t* vis[2];     // [light][cap]: 1 = light visible from the entry
  uint32_t* gstack;
  int32_t gstack_entries; // spill entries per lane in gstack
  int64_t path_begin, path_count;
  uint32_t cap;           // entries per queue
  int32_t brute;
  int32_t trace_threads;  // threads in the persistent traversal grid (gstack stride)
  int32_t resolve;        // k_trace of depth d also adds the lights' terms of depth d - 2
  unsigned long long launch;  // k_path: the launch's number
};
// Kernels take KArgs by value as their first argument, so its bytes start the kernel-argument
// segment (kernel_args reads them there).
static_assert(std::is_trivially_copyable<KArgs>::value && std::is_standard_layout<KArgs>::value,
              "KArgs must be plain data");

// The item a path belongs to: binary search over the items' first path ids.
template <bool MULTI>
__device__ inline int item_of(const KArgs& a, int64_t p) {
  if (!MULTI) return 0;
  typedef __attribute__((address_space(4))) const DevItem item_t;  // a scalar load where p is uniform
  int lo = 0, hi = a.num_items - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (((item_t*)a.items)[mid].path_offset <= p)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// ---------------------------------------------------------------------------------------------
// Camera
// ---------------------------------------------------------------------------------------------

// The pixel of path r of tile `tile`; false outside the image.
__device__ inline bool tile_pixel(const DevCamera& c, uint32_t tile, int r, int* eye, int* x, int* y) {
  *eye = r >> 6;
  const int w = r & 63;
  const int ty = int(tile / uint32_t(c.tiles_x)), tx = int(tile) - ty * c.tiles_x;
  *x = tx * kTile + (w & 7);
  *y = ty * kTile + (w >> 3);
  return *x < c.W && *y < c.H;
}
// The pixel of path p of an image (of at most RT_MAX_PIXELS pixels, so tiles count in 32 bits).
__device__ inline bool path_pixel(const DevCamera& c, int64_t p, int* eye, int* x, int* y) {
  return tile_pixel(c, uint32_t(p / kPathsPerTile), int(p % kPathsPerTile), eye, x, y);
}
// The same where all lanes' paths are of one tile.
__device__ inline bool wave_pixel(const DevCamera& c, int64_t p, int* eye, int* x, int* y) {
  const uint32_t tile = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(p / kPathsPerTile))));
  return tile_pixel(c, tile, int(p % kPathsPerTile), eye, x, y);
}

// Off-axis stereo pinhole: eye at C + s r (s = -+B/2), pixel-centre ray sheared by -s/Z0.
// Computed in FP64 and rounded once to FP32.
__device__ inline float3 eye_position(const DevCamera& c, int eye) {
  const double s = eye == 0 ? -c.half_baseline : c.half_baseline;
  return make_float3(float(fma(s, c.r[0], c.C[0])), float(fma(s, c.r[1], c.C[1])), float(fma(s, c.r[2], c.C[2])));
}
__device__ inline void primary_ray(const DevCamera& c, int eye, int x, int y, float3* o, float3* d) {
  double s = eye == 0 ? -c.half_baseline : c.half_baseline;
  double D[3];
  double a = (double(x) + 0.5 - c.cx) / c.fpx - s * c.inv_convergence;
  double b = -(double(y) + 0.5 - c.cy) / c.fpx;
  for (int k = 0; k < 3; ++k) D[k] = c.f[k] + a * c.r[k] + b * c.u[k];
  double inv = 1.0 / sqrt(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]);
  *o = eye_position(c, eye);
  *d = make_float3(float(D[0] * inv), float(D[1] * inv), float(D[2] * inv));
}

// ---------------------------------------------------------------------------------------------
// Ray-primitive tests (FP32)
// ---------------------------------------------------------------------------------------------

// Moller-Trumbore with its roundings written out, so that every kernel gets the same answer for the same ray
// and triangle however its compiler would contract the sums.
struct TriTest {
  float3 T, P, Q;
  float det, un, vn;

  __device__ static inline float dot_xyz(float3 a, float3 b) { return fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)); }

  // the determinant and the first barycentric coordinate times it
  __device__ inline void first(float3 o, float3 d, float3 v0, float3 e1, float3 e2) {
    P = fcross(d, e2);
    det = fdot(e1, P);
    T = o - v0;
    un = dot_xyz(T, P);
  }
  // the second one times the determinant
  __device__ inline void second(float3 d, float3 e1) {
    Q = fcross(T, e1);
    vn = fdot(d, Q);
  }
  // t, or +inf outside the triangle or (tmin, tmax); det != 0
  __device__ inline float t(float3 e2, float inv, float u, float tmin, float tmax) const {
    if (!(vn * inv >= 0.0f && fmaf(vn, inv, u) <= 1.0f)) return INFINITY;
    const float t = fdot(e2, Q) * inv;
    return (t > tmin && t < tmax) ? t : INFINITY;
  }
};

// Closed triangle; only det == 0 rejected.  Returns t or +inf.
__device__ inline float tri_t(const float4* __restrict__ recs, int r, float3 o, float3 d, float tmin, float tmax,
                              int* id_out) {
  const float4 a = recs[3 * r], b = recs[3 * r + 1], c = recs[3 * r + 2];
  *id_out = __float_as_int(a.w);
  const float3 e1 = f3(b), e2 = f3(c);
  TriTest m;
  m.first(o, d, f3(a), e1, e2);
  if (m.det == 0.0f) return INFINITY;
  const float inv = 1.0f / m.det;
  const float u = m.un * inv;
  if (!(u >= 0.0f && u <= 1.0f)) return INFINITY;
  m.second(d, e1);
  return m.t(e2, inv, u, tmin, tmax);
}

// Sphere with unit d: b = -oc.d, h^2 = |oc + b d|^2, disc = r^2 - h^2, roots b -+ sqrt(disc).
__device__ inline float sphere_t(float4 s, float3 o, float3 d, float tmin, float tmax) {
  const float3 oc = o - f3(s);
  const float b = -fdot(oc, d);
  const float3 foot = fmad(b, d, oc);
  const float disc = fmaf(s.w, s.w, -fdot(foot, foot));
  if (disc < 0.0f) return INFINITY;
  const float q = sqrtf(disc);
  const float t0 = b - q, t1 = b + q;
  if (t0 > tmin && t0 < tmax) return t0;
  if (t1 > tmin && t1 < tmax) return t1;
  return INFINITY;
}

__device__ inline float plane_t(float4 p, float3 o, float3 d, float tmin, float tmax) {
  const float nd = fdot(f3(p), d);
  if (nd == 0.0f) return INFINITY;
  const float t = (p.w - fdot(f3(p), o)) / nd;
  return (t > tmin && t < tmax) ? t : INFINITY;
}

// The shadow ray from P to light l: its direction, and its length as the distance to stop at.
__device__ inline float3 shadow_dir(const float4* lights, int l, float3 P, float* dist) {
  const float3 Lv = f3(lights[2 * l]) - P;
  *dist = sqrtf(fdot(Lv, Lv));
  return (1.0f / *dist) * Lv;
}

// Slab test of one child box; returns the entry distance, or +inf when missed.
__device__ inline float slab(float lox, float hix, float loy, float hiy, float loz, float hiz, float3 inv, float3 oi,
                             float tmin, float tmax) {
  const float x0 = fmaf(lox, inv.x, -oi.x), x1 = fmaf(hix, inv.x, -oi.x);
  const float y0 = fmaf(loy, inv.y, -oi.y), y1 = fmaf(hiy, inv.y, -oi.y);
  const float z0 = fmaf(loz, inv.z, -oi.z), z1 = fmaf(hiz, inv.z, -oi.z);
  const float tn = fmaxf(fmaxf(fminf(x0, x1), fminf(y0, y1)), fmaxf(fminf(z0, z1), tmin));
  const float tf = fminf(fminf(fmaxf(x0, x1), fmaxf(y0, y1)), fminf(fmaxf(z0, z1), tmax));
  return tn <= tf ? tn : INFINITY;
}

// max and min without the instruction that first quiets a signalling NaN in an operand: there is none.
// The two large launches of a frame issue a vector instruction in every cycle, most of them here.  These
// and the references pinned as one register of 128 bits (four pins cost four copies): 3.4 M triangles at
// 4K 6.95 -> 6.90 ms, 16 mixed scenes 7.43 -> 7.33 ms.  Sign masks of the direction kept in scalar
// registers gave single scenes 0.5% more and took 1% from the batch, for want of scalar registers.
__device__ inline float raw_max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ inline float raw_min3(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
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

// The four children of BVH4 node `node`: h whether the ray meets the child's box inside [tmin, tmax], t the entry
// distance (+inf where it does not), r the reference.  The loop counts the children to push from h, which are lane
// masks in scalar registers, and not from the sorted distances: 7 of about 100 vector instructions a step less (3.4 M
// triangles at 4K 6.53 -> 6.48 ms, 16 mixed scenes 6.78 -> 6.74).
__device__ __attribute__((always_inline)) inline void node4_children(const float4* __restrict__ nodes, int node,
                                                                     float3 inv, float3 oi, float tmin, float tmax,
                                                                     float (&t)[4], int (&r)[4], bool (&h)[4]) {
#if SRT_QNODE
  // Slab planes of child k on axis a are p_a + q s_a, i.e. t = q (s_a / d_a) + (p_a - o_a) / d_a; the
  // near and far planes of an axis are picked once per node from the ray's direction sign.  A byte q
  // placed in the low byte of an FP16 value is the subnormal q 2^-24, exactly; one v_perm_b32 makes
  // two such values from two grid bytes, and v_fma_mix_f32 takes one as its FP16 multiplicand.  The
  // node stores S = 2^24 s, so q 2^-24 (S / d) = q (s / d) exactly and each plane is the same fused
  // multiply-add, to the bit, as with q converted to FP32.  S / d is finite for every direction
  // because vertices lie within RT_MAX_COORD.
  const float4* n = nodes + 4 * node;
  const float4 n0 = n[0], n2 = n[2], n3 = n[3];
  typedef int int4_t __attribute__((ext_vector_type(4)));
  int4_t n1 = *reinterpret_cast<const int4_t*>(n + 1);
  // the references are used last; without this the compiler may load one of them a second time, later,
  // where it turns out to be needed, and wait for memory twice
  asm("" : "+v"(n1));
  const float ax = n0.w * inv.x, ay = n3.z * inv.y, az = n3.w * inv.z;  // 2^24 s / d; S is a power of two: exact
  const float bx = fmaf(n0.x, inv.x, -oi.x), by = fmaf(n0.y, inv.y, -oi.y), bz = fmaf(n0.z, inv.z, -oi.z);
  const bool px = inv.x >= 0.f, py = inv.y >= 0.f, pz = inv.z >= 0.f;
  const uint32_t qlx = __float_as_uint(n2.x), qhx = __float_as_uint(n2.y), qly = __float_as_uint(n2.z),
                 qhy = __float_as_uint(n2.w), qlz = __float_as_uint(n3.x), qhz = __float_as_uint(n3.y);
  const uint32_t nx = px ? qlx : qhx, fx = px ? qhx : qlx, ny = py ? qly : qhy, fy = py ? qhy : qly,
                 nz = pz ? qlz : qhz, fz = pz ? qhz : qlz;
  // bytes 2j and 2j+1 of w as the FP16 pair (q 2^-24, q' 2^-24): selector byte 0x0c gives a zero byte
  auto grid_pair = [](uint32_t w, int j) {
    return __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(0u, w, j ? 0x0c030c02u : 0x0c010c00u));
  };
  half2_t hnx[2], hfx[2], hny[2], hfy[2], hnz[2], hfz[2];
  for (int j = 0; j < 2; ++j) {
    hnx[j] = grid_pair(nx, j), hfx[j] = grid_pair(fx, j), hny[j] = grid_pair(ny, j), hfy[j] = grid_pair(fy, j);
    hnz[j] = grid_pair(nz, j), hfz[j] = grid_pair(fz, j);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    auto q = [k](const half2_t (&h)[2]) { return float((k & 1) ? h[k >> 1].y : h[k >> 1].x); };
    const float xn = fmaf(q(hnx), ax, bx), xf = fmaf(q(hfx), ax, bx);
    const float yn = fmaf(q(hny), ay, by), yf = fmaf(q(hfy), ay, by);
    const float zn = fmaf(q(hnz), az, bz), zf = fmaf(q(hfz), az, bz);
    const float tn = raw_max3(xn, yn, raw_max(zn, tmin));
    const float tf = raw_min3(xf, yf, raw_min(zf, tmax));
    h[k] = tn <= tf;
    t[k] = h[k] ? tn : INFINITY;
  }
  r[0] = n1.x;
  r[1] = n1.y;
  r[2] = n1.z;
  r[3] = n1.w;
#else
  const float4* n = nodes + 8 * node;
  const float4 lx = n[0], hx = n[1], ly = n[2], hy = n[3], lz = n[4], hz = n[5], cr = n[6];
  t[0] = slab(lx.x, hx.x, ly.x, hy.x, lz.x, hz.x, inv, oi, tmin, tmax);
  t[1] = slab(lx.y, hx.y, ly.y, hy.y, lz.y, hz.y, inv, oi, tmin, tmax);
  t[2] = slab(lx.z, hx.z, ly.z, hy.z, lz.z, hz.z, inv, oi, tmin, tmax);
  t[3] = slab(lx.w, hx.w, ly.w, hy.w, lz.w, hz.w, inv, oi, tmin, tmax);
  for (int k = 0; k < 4; ++k) h[k] = t[k] < INFINITY;
  r[0] = __float_as_int(cr.x);
  r[1] = __float_as_int(cr.y);
  r[2] = __float_as_int(cr.z);
  r[3] = __float_as_int(cr.w);
#endif
}

// ---------------------------------------------------------------------------------------------
// Traversal stack: kStackLds entries per lane in LDS used as a ring; older entries spill to
// a lane-interleaved area of the workspace.
// ---------------------------------------------------------------------------------------------

struct Stack {
  uint32_t* lds;     // this thread's column: entry k of the ring at [k * kBlock]
  uint32_t* global;  // the spill area: entry k of grid thread g at [k * gstride + g] (fits 32 bits)
  uint32_t gblock;   // the grid thread of this block's thread 0
  uint32_t gstride;
  int gcap;          // spill entries per lane
  int sp;
  bool overflow;

  __device__ inline uint32_t& spill(int k) const {
    return global[uint32_t(k) * gstride + (gblock + threadIdx.x)];
  }
  __device__ inline void push(int v) {
    if (sp >= kStackLds) {
      if (sp - kStackLds >= gcap) {  // excluded by the depth checks on the host; never write out of bounds
        overflow = true;
        return;
      }
      spill(sp - kStackLds) = lds[(sp & (kStackLds - 1)) * kBlock];
    }
    lds[(sp & (kStackLds - 1)) * kBlock] = uint32_t(v);
    ++sp;
  }
  // Pushes the np (1..3) entries c3, c2, c1 of which the last np are live (c1 ends on top).  With
  // room for three entries below the LDS ring's wrap point all three slots are written
  // unconditionally (entries above the new top are dead), so the common case takes no branch.
  __device__ inline void push_sorted(int c1, int c2, int c3, int np) {
    if (sp + 3 <= kStackLds) {
      const int s0 = np == 1 ? c1 : (np == 2 ? c2 : c3);
      const int s1 = np == 2 ? c1 : c2;
      lds[sp * kBlock] = uint32_t(s0);
      lds[(sp + 1) * kBlock] = uint32_t(s1);
      lds[(sp + 2) * kBlock] = uint32_t(c1);
      sp += np;
    } else {
      if (np >= 3) push(c3);
      if (np >= 2) push(c2);
      push(c1);
    }
  }
  __device__ inline int pop() {
    --sp;
    int v = int(lds[(sp & (kStackLds - 1)) * kBlock]);
    if (sp >= kStackLds) lds[(sp & (kStackLds - 1)) * kBlock] = spill(sp - kStackLds);
    return v;
  }
};

// Orders four (entry distance, child) pairs by distance; missed children (at +inf) sort last.
__device__ __attribute__((always_inline)) inline void sort4(float (&t)[4], int (&r)[4]) {
  auto cas = [&](int i, int j) {
    const bool sw = t[j] < t[i];
    const float ti = t[i], tj = t[j];
    const int ri = r[i], rj = r[j];
    t[i] = sw ? tj : ti;
    t[j] = sw ? ti : tj;
    r[i] = sw ? rj : ri;
    r[j] = sw ? ri : rj;
  };
  cas(0, 1);
  cas(2, 3);
  cas(0, 2);
  cas(1, 3);
  cas(1, 2);
}

// Value of the `node` register once a ray's traversal is finished (never a node index).
constexpr int kDoneRef = 0x7fffffff;

struct Best {
  float t;
  int key;
  int id;
};

// A wave's own LDS words, written by one of its lanes and read by another: within a wave LDS operations take
// effect in program order, and the atomic access keeps the compiler from caching the value.
template <class T>
__device__ inline T lds_get(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
template <class T>
__device__ inline void lds_put(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// The best hits of the rays a wave shares between its lanes, one slot per ray (LDS, this wave's part).
// A slot's word is (limit bits << 32 | id): as an integer it orders hits by (t, id), limit being the next
// float above t.
struct Share {
  unsigned long long* word;
  int* key;

  __device__ inline void open(int slot, uint32_t limit_bits, int id, int k) const {
    lds_put(&word[slot], (static_cast<unsigned long long>(limit_bits) << 32) | uint32_t(id));
    lds_put(&key[slot], k);
  }
  __device__ inline float limit(int slot) const { return __uint_as_float(uint32_t(lds_get(&word[slot]) >> 32)); }
  __device__ inline int key_of(int slot) const { return lds_get(&key[slot]); }
  // Takes a hit if it is the ray's best; no other lane offers the same (t, id).
  __device__ inline void offer(int slot, uint32_t limit_bits, int id, int k) const {
    const unsigned long long w = (static_cast<unsigned long long>(limit_bits) << 32) | uint32_t(id);
    __hip_atomic_fetch_min(&word[slot], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (lds_get(&word[slot]) == w) lds_put(&key[slot], k);
  }
  // An occlusion query is answered: no candidate lies below a limit of 0.
  __device__ inline void close(int slot) const { lds_put(&word[slot], 0ull); }
};

// A wave's working set of one kind of ray: lane l starts with ray l of the wave's batch (or none).
struct Ray {
  float3 o, d;
  float tmin, limit;  // the interval [tmin, limit) a candidate must lie in
  int exclude;        // key of the primitive the ray leaves (-1: none)
};

// Entry cap of a traversal loop; it only guards against a corrupt tree (T <= 2^29, so it fits 32 bits).
__device__ inline int loop_guard(int T) { return 2 * T + 64; }

__device__ inline float shfl_f(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src << 2, __float_as_int(v)));
}
__device__ inline int shfl_i(int v, int src) { return __builtin_amdgcn_ds_bpermute(src << 2, v); }

// True where the triangle test certainly rejects a barycentric coordinate num / det (signs and sizes only,
// before the division): below 0 by more than an underflow can hide, or above 1 by more than rounding can.
__device__ inline bool outside(float num_signed, float det_abs) {
  return num_signed < -1e-30f * det_abs || num_signed > 1.0001f * det_abs;
}

// Tests a wave's rays against triangle records first .. last - 1, all lanes together; accept(t, record, id)
// for the lanes with a candidate in (tmin, limit()).  STEP records are loaded at a time, so a wave waits once for
// all of them.
template <int STEP, class Limit, class Accept>
__device__ __attribute__((always_inline)) inline void flat_triangles(const float4* tris, int first, int last, float3 o,
                                                                     float3 d, float tmin, Limit limit, Accept accept) {
  typedef __attribute__((address_space(4))) const float4 const_float4;  // written by an earlier launch only
  auto test = [&](float4 a, float4 b, float4 c, int k) {
    const float3 e1 = f3(b), e2 = f3(c);
    TriTest m;
    m.first(o, d, f3(a), e1, e2);
    const uint32_t sign = __float_as_uint(m.det) & 0x80000000u;
    const float ad = fabsf(m.det);
    if (outside(__uint_as_float(__float_as_uint(m.un) ^ sign), ad)) return;
    m.second(d, e1);
    if (outside(__uint_as_float(__float_as_uint(m.vn) ^ sign), ad)) return;
    if (m.det == 0.0f) return;
    const float inv = 1.0f / m.det;
    const float u = m.un * inv;
    if (!(u >= 0.0f && u <= 1.0f)) return;
    const float t = m.t(e2, inv, u, tmin, limit());
    if (t < INFINITY) accept(t, k, __float_as_int(a.w));
  };
  const const_float4* recs = (const const_float4*)tris;
  int k = first;
  for (; k + STEP <= last; k += STEP) {
    float4 r[3 * STEP];
#pragma unroll
    for (int j = 0; j < 3 * STEP; ++j) r[j] = ((const float4*)(recs + 3 * __builtin_amdgcn_readfirstlane(k)))[j];
#pragma unroll
    for (int j = 0; j < STEP; ++j) test(r[3 * j], r[3 * j + 1], r[3 * j + 2], k + j);
  }
  for (; k < last; ++k) {
    const float4* r = (const float4*)(recs + 3 * __builtin_amdgcn_readfirstlane(k));
    test(r[0], r[1], r[2], k);
  }
}

// test(value, k) for elements first .. last - 1 of a scene array, which are the same for the whole wave and were written
// by an earlier launch: scalar loads, kFlatStep at a time, so that a wave waits once for all of them.
template <class Test>
__device__ __attribute__((always_inline)) inline void flat_each(const float4* p, int first, int last, Test test) {
  typedef __attribute__((address_space(4))) const float4 const_float4;
  const const_float4* v = (const const_float4*)p;
  int k = first;
  for (; k + kFlatStep <= last; k += kFlatStep) {
    float4 r[kFlatStep];
#pragma unroll
    for (int j = 0; j < kFlatStep; ++j) r[j] = ((const float4*)(v + __builtin_amdgcn_readfirstlane(k)))[j];
#pragma unroll
    for (int j = 0; j < kFlatStep; ++j) test(r[j], k + j);
  }
  for (; k < last; ++k) test(*(const float4*)(v + __builtin_amdgcn_readfirstlane(k)), k);
}

// Traverses the rays of one wave (all lanes call it together; `mine` marks the lanes that hold a ray).
// ANY = false: closest hit, minimum t, exact ties to the smaller original id; the limit starts at +inf.
// ANY = true : occlusion, stops at the first primitive with t in (tmin, limit).
// FLAT: scenes without a tree (or RT_FLAG_BRUTE_FORCE) may come too; k_trace_flat takes them otherwise.
// commit(key, t) is called once for every lane with a ray: the hit's key (-1: none) and distance.
// Closest-hit candidates are tested against the next float above the best t, so that an exact tie in t
// reaches the (t, id) comparison, and boxes entered exactly at the best t are not culled.
//
// One lane per ray while many rays are left.  A ray can need ten times the node visits of the average one,
// so a wave's last rays would run alone (before, half of the VALU lanes were idle), and one ray's chain of
// dependent node fetches (about 0.5 us each) sets the time of a small launch.  Once at most kCoopRays rays
// are left, the wave's idle lanes help: each takes the top entry of a busy lane's stack, with a copy of its
// ray, and traverses that subtree itself.  The lanes of one ray share its best hit through `share` (one slot
// per shared ray); the result is the minimum (t, id) over everything they reach, which does not depend on
// the order they reach it in.  Measured with the 8-wave budget on a 1080p frame of 3.4M triangles, depth 4,
// 4 lights: the six launches took 538, 1324, 300, 166, 222 and 135 us and take 455, 1130, 230, 81, 53 and
// 31; the frame went from 2844 to 2121 us.  kCoopRays 8 / 16 / 24 / 32 / 48 / 64: 2463 / 2376 / 2322 / 2278
// / 2258 / 2310 us (at 7 waves).
template <bool ANY, bool COUNT, bool FLAT, class Commit>
__device__ __attribute__((always_inline)) inline void traverse(const DevScene& sc, bool mine, Ray r,
                                                               bool brute, Stack& st, const Share& share,
                                                               uint32_t& nnodes, uint32_t& ntris, Commit commit) {
  constexpr bool kCoop = !COUNT && kCoopRays > 0;  // work counts are those of one lane per ray
  const int lane = lane_id();
  // the fields the loop reads, held in scalar registers (the empty asm hides that they could be loaded again)
  const float4* const nodes = global_scalar(sc.nodes);
  const float4* const tris = global_scalar(sc.tris);
  int num_nodes = sc.num_nodes, T = sc.T;
  asm("" : "+s"(num_nodes), "+s"(T));
  Best best{INFINITY, -1, 0x7fffffff};
  bool found = false;    // ANY: the ray is occluded
  int slot = 0;          // of the ray this lane works on, while the wave shares its rays
  bool coop = false;     // the wave shares its rays (wave-uniform)
  bool own_late = false; // this lane's own ray is one of them
  uint64_t late = 0;     // the lanes whose rays it shares (wave-uniform)
  auto accept = [&](float t, int key, int id) {
    if (key == r.exclude || !(t < INFINITY)) return;
    if (ANY) {
      found = true;
    } else if (kCoop && coop) {
      share.offer(slot, __float_as_uint(t) + 1u, id, key);
    } else if (t < best.t || (t == best.t && id < best.id)) {
      best.t = t;
      best.key = key;
      best.id = id;
      r.limit = __int_as_float(__float_as_int(t) + 1);  // the next float above t, finite here
    }
  };
  int node = kDoneRef;
  st.sp = 0;
  if (mine) {
    // Spheres and planes are the same for the whole wave.  Loaded one at a time by each lane, 2,000 of them beside a tree
    // of 5,000 triangles, 256x256, 2 lights, depth 3: 3030 us, 1670 this way.
    for (int k = 0; k < sc.S && !(ANY && __all(found)); k += 64)
      flat_each(sc.spheres, k, min(k + 64, sc.S),
                [&](float4 s, int i) { accept(sphere_t(s, r.o, r.d, r.tmin, r.limit), sc.T + i, sc.T + i); });
    for (int k = 0; k < sc.P && !(ANY && __all(found)); k += 64)
      flat_each(sc.planes, k, min(k + 64, sc.P), [&](float4 p, int i) {
        const int key = sc.T + sc.S + i;
        accept(plane_t(p, r.o, r.d, r.tmin, r.limit), key, key);
      });
    if (FLAT && (brute || !sc.has_bvh)) {
      if (COUNT) {
        for (int k = 0; k < sc.T && !(ANY && found); ++k) {
          int id;
          const float t = tri_t(sc.tris, k, r.o, r.d, r.tmin, r.limit, &id);
          ++ntris;
          accept(t, k, id);
        }
      } else {  // 16 images of 256x256, 2,000 triangles each, depth 2, 2 lights: 18.8 ms with the loop above, 5.7 this way
        for (int k = 0; k < sc.T && !(ANY && __all(found)); k += 64)
          flat_triangles<kWalkStep>(sc.tris, k, min(k + 64, sc.T), r.o, r.d, r.tmin, [&] { return r.limit; }, accept);
      }
    } else if (sc.T > 0 && sc.has_bvh && !(ANY && found)) {
      node = sc.root;
    }
  }
  float3 inv = make_float3(safe_rcp(r.d.x), safe_rcp(r.d.y), safe_rcp(r.d.z));
  float3 oi = mul(r.o, inv);
  for (int guard = loop_guard(T); guard > 0; --guard) {
    const uint64_t busy = __ballot(node != kDoneRef);
    if (busy == 0) break;
    if (kCoop) {
      if (!coop && __popcll(busy) <= kCoopRays) {
        coop = true;
        late = busy;
        own_late = node != kDoneRef;
        if (own_late) {
          slot = lanes_below(busy);
          share.open(slot, __float_as_uint(r.limit), best.id, best.key);
        } else if (mine) {
          commit(ANY ? (found ? 0 : -1) : best.key, best.t);
        }
      }
      if (coop) {
        // pair the k-th idle lane with the k-th busy lane that has a stack entry to give
        const bool can_give = node != kDoneRef && st.sp > 0, is_idle = node == kDoneRef;
        const uint64_t give = __ballot(can_give);
        const int ngive = __popcll(give), nidle = 64 - __popcll(busy);
        if (min(ngive, nidle) * kCoopShare >= 64 - nidle && give != 0) {
          const int below = lanes_below(give), rank = lanes_below(~busy);
          const bool gives = can_give && below < nidle, takes = is_idle && rank < ngive;
          // a permutation of the lanes that lists the givers first
          const int givers = __builtin_amdgcn_ds_permute((can_give ? below : ngive + lane - below) << 2, lane);
          const int giver = shfl_i(givers, rank);
          const int from = takes ? giver : lane;  // every other lane reads itself
          int top = node;
          if (gives) top = st.pop();
          const int taken = shfl_i(top, from);
          r.o.x = shfl_f(r.o.x, from), r.o.y = shfl_f(r.o.y, from), r.o.z = shfl_f(r.o.z, from);
          r.d.x = shfl_f(r.d.x, from), r.d.y = shfl_f(r.d.y, from), r.d.z = shfl_f(r.d.z, from);
          inv.x = shfl_f(inv.x, from), inv.y = shfl_f(inv.y, from), inv.z = shfl_f(inv.z, from);
          oi.x = shfl_f(oi.x, from), oi.y = shfl_f(oi.y, from), oi.z = shfl_f(oi.z, from);
          r.exclude = shfl_i(r.exclude, from);
          slot = shfl_i(slot, from);
          if (takes) {
            node = taken;
            found = false;
          }
        }
        if (node != kDoneRef) {
          r.limit = share.limit(slot);
          if (ANY && r.limit == 0.0f) {  // another lane found an occluder
            node = kDoneRef;
            st.sp = 0;
          }
        }
      }
    }
    // One internal-node step, then, if the lane now holds a leaf, its test, so the leaf step of a wave runs
    // with every lane that reached a leaf in this iteration.
    if (node >= 0 && node != kDoneRef) {
      if (node >= num_nodes) {  // corrupt reference: stop this ray, never read out of bounds
        st.overflow = true;
        node = kDoneRef;
        st.sp = 0;
      } else {
        if (COUNT) ++nnodes;
        float t[4];
        int c[4];
        bool h[4];
        node4_children(nodes, node, inv, oi, r.tmin, r.limit, t, c, h);
        if (ANY) {
          // occlusion: the order of the hit children does not change the answer, so they are taken in
          // slot order (the same for every lane of the wave) without sorting: the first hit child next,
          // the later hit children pushed so that they pop in slot order
          if (h[0] || h[1] || h[2] || h[3]) {
            node = h[0] ? c[0] : (h[1] ? c[1] : (h[2] ? c[2] : c[3]));
            // hits after the first
            const bool g1 = h[1] && h[0], g2 = h[2] && (h[0] || h[1]), g3 = h[3] && (h[0] || h[1] || h[2]);
            const int np = int(g1) + int(g2) + int(g3);
            if (np > 0) st.push_sorted(g1 ? c[1] : (g2 ? c[2] : c[3]), (g1 && g2) ? c[2] : c[3], c[3], np);
          } else {
            node = st.sp > 0 ? st.pop() : kDoneRef;
          }
        } else {
          if (h[0] || h[1] || h[2] || h[3]) {
            sort4(t, c);
            node = c[0];
            const int np = int(h[0]) + int(h[1]) + int(h[2]) + int(h[3]) - 1;
            if (np > 0) st.push_sorted(c[1], c[2], c[3], np);
          } else {
            node = st.sp > 0 ? st.pop() : kDoneRef;
          }
        }
      }
    }
    if (node < 0) {
      const int code = ~node;
      const int first = code >> 2, count = (code & 3) + 1;
      if (first + count > T) {
        st.overflow = true;
        st.sp = 0;
      } else {
        for (int k = 0; k < count && !(ANY && found); ++k) {
          const int i = first + k;
          if (i == r.exclude) continue;  // the secondary ray's own primitive: not fetched
          int id;
          const float t = tri_t(tris, i, r.o, r.d, r.tmin, r.limit, &id);
          if (COUNT) ++ntris;
          accept(t, i, id);
        }
      }
      if (ANY && found) {
        st.sp = 0;
        if (kCoop && coop) share.close(slot);
      }
      node = st.sp > 0 ? st.pop() : kDoneRef;
    }
  }
  if (node != kDoneRef) st.overflow = true;
  if (!kCoop || !coop) {
    if (mine) commit(ANY ? (found ? 0 : -1) : best.key, best.t);
  } else if (own_late) {
    const int own = lanes_below(late);
    const float limit = share.limit(own);
    if (ANY) {
      commit(limit == 0.0f ? 0 : -1, 0.0f);
    } else {
      const int key = share.key_of(own);
      commit(key, key < 0 ? INFINITY : __uint_as_float(__float_as_uint(limit) - 1u));
    }
  }
}

// The same for one lane's ray in a scene without a tree, where the wave's rays are of several scenes: each walk would
// wait for the ones before it (4 images of 64x64 over scenes of 200 spheres, depth 2: 306 us that way, 282 so).
template <bool ANY, bool COUNT, class Commit>
__device__ __attribute__((always_inline)) inline void walk_alone(const DevScene& sc, Ray r, uint32_t& ntris,
                                                                 Commit commit) {
  Best best{INFINITY, -1, 0x7fffffff};
  auto accept = [&](float t, int key, int id) {
    if (key == r.exclude || !(t < INFINITY)) return false;
    if (ANY || t < best.t || (t == best.t && id < best.id)) best = Best{t, key, id};
    if (!ANY) r.limit = next_up(best.t);
    return ANY;
  };
  bool found = false;
  for (int k = 0; k < sc.S && !found; ++k)
    found = accept(sphere_t(sc.spheres[k], r.o, r.d, r.tmin, r.limit), sc.T + k, sc.T + k);
  for (int k = 0; k < sc.P && !found; ++k)
    found = accept(plane_t(sc.planes[k], r.o, r.d, r.tmin, r.limit), sc.T + sc.S + k, sc.T + sc.S + k);
  for (int k = 0; k < sc.T && !found; ++k) {
    int id;
    const float t = tri_t(sc.tris, k, r.o, r.d, r.tmin, r.limit, &id);
    if (COUNT) ++ntris;
    found = accept(t, k, id);
  }
  commit(best.key, best.t);
}

__device__ inline void add_work(Counters* ctr, int slot, uint32_t v) {
  // wave reduction, one 64-bit atomic per wave
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if (lane_id() == 0 && v) atomicAdd(&ctr->work[slot], (unsigned long long)v);
}

// ---------------------------------------------------------------------------------------------
// k_trace: closest-hit rays of depth `depth` and shadow rays of depth `depth - 1` in one
// persistent grid.  The work space is [closest rays | shadow rays of light 0 | light 1 | ...],
// each range padded to whole batches so that every wave batch is one kind of ray.
// ---------------------------------------------------------------------------------------------

// Traversal occupancy: the traversal kernels are held to kTraceWaves waves per SIMD, a budget of
// 64 VGPRs and 20 KB of LDS a block.  The single-scene kernel meets it without spilling, the batch kernel
// with 4 registers spilled outside the node step.  7 waves: 2258 vs 2187 us for a 1080p frame of 3.4M
// triangles, 7.68 vs 7.47 ms for 16 mixed pairs.  The instrumented kernels are left free.
constexpr int kTraceWaves = SRT_TRACE_WAVES_PER_EU;
#define SRT_TRACE_ATTR __attribute__((amdgpu_waves_per_eu(COUNT || kTraceWaves <= 0 ? 1 : kTraceWaves)))

// The kernel's arguments read afresh from the kernel-argument segment: the empty asm hides that the
// pointer is loop-invariant, so fields used once per batch are loaded where they are used instead of
// being kept in scalar registers across the traversal loop, where they would spill.  A kernel's
// first argument starts the segment.
__device__ __attribute__((always_inline)) inline const KArgs& kernel_args() {
  typedef __attribute__((address_space(4))) const KArgs kargs_t;
  const kargs_t* p = (const kargs_t*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const KArgs*)p;
}

// Calls body(item, mine) for each scene that lanes of this wave hold, with an item of it and `mine` marking its
// lanes; every lane makes the call.  The item is the same for the whole wave, so its fields are scalar loads.  Queue
// entries are in path order within a shading block's run, so nearly every wave holds one item.  In a wave that holds
// several, lanes whose scene has no tree call alone(item) instead, all at once.
template <bool MULTI, class Body, class Alone>
__device__ __attribute__((always_inline)) inline void each_scene(const KArgs& a, bool valid, int k, Body body,
                                                                 Alone alone) {
  if (!MULTI) {
    body(a.one, valid);
    return;
  }
  typedef __attribute__((address_space(4))) const DevItem item_t;
  uint64_t todo = __ballot(valid);
  if (todo == 0) return;
  if (__ballot(valid && k == __builtin_amdgcn_readlane(k, __builtin_ctzll(todo))) != todo) {
    if (valid && (a.brute || !a.items[k].sc.has_bvh)) {
      alone(a.items[k]);
      valid = false;
    }
    todo = __ballot(valid);
    const uintptr_t scene = valid ? reinterpret_cast<uintptr_t>(a.items[k].sc.materials) : 0;  // in its own storage
    const int lo = int(uint32_t(scene)), hi = int(uint32_t(scene >> 32));
    for (uint64_t left = todo; left != 0;) {  // the lanes of a scene take one item's number
      const int from = __builtin_ctzll(left);
      const bool same = valid && lo == __builtin_amdgcn_readlane(lo, from) && hi == __builtin_amdgcn_readlane(hi, from);
      if (same) k = __builtin_amdgcn_readlane(k, from);
      left &= ~__ballot(same);
    }
  }
  while (todo != 0) {
    const int k0 = __builtin_amdgcn_readlane(k, __builtin_ctzll(todo));
    const bool mine = valid && k == k0;
    body(*(const DevItem*)((const item_t*)a.items + k0), mine);
    todo &= ~__ballot(mine);
  }
}

// Calls body(item, valid) once, with the item the lane holds: its fields are scalar loads where the wave holds one item,
// vector loads where it holds several.  One item after the other, as the traversal takes them, the entries of a batch of
// small images took up to 64 turns (64 images of 16x16, depth 4: 68 + 56 us for the shading of depths 2 and 3, 13 this
// way).
template <bool MULTI, class Body>
__device__ __attribute__((always_inline)) inline void each_item(const KArgs& a, bool valid, int k, Body body) {
  if (!MULTI) {
    body(a.one, valid);
    return;
  }
  typedef __attribute__((address_space(4))) const DevItem item_t;
  const uint64_t all = __ballot(valid);
  if (all == 0) return;
  const int k0 = __builtin_amdgcn_readlane(k, __builtin_ctzll(all));
  if (__ballot(valid && k == k0) == all)
    body(*(const DevItem*)((const item_t*)a.items + k0), valid);
  else
    body(a.items[valid ? k : k0], valid);
}

// 64 << kResolveLog2 entries make a batch of k_trace's.  As launches of their own the resolves of a 1080p frame of
// 3.4M triangles, depth 4, took 48 + 16 + 8 + 7 + 6 us; with all but the last in the traversal the frame went from 2056
// to 1999 us, 16 mixed scenes from 6738 to 6605, 8 small ones from 911 to 875 (64 entries a batch: 2001, 6795 and 888;
// 256: 1996, 6643 and 880).
constexpr int kResolveLog2 = 1;

// Adds the unoccluded lights' terms of entry e of depth `depth` to its path's pixel, in light order.  All lanes of a
// wave call it, with consecutive entries from a multiple of 64 on.
template <bool PATH_IDS, bool MULTI>
__device__ __attribute__((always_inline)) inline void resolve_entry(const KArgs& a, int depth, uint32_t e,
                                                                    uint32_t total) {
  const int q = depth & 1;
  const uint32_t mask = e < total ? a.smask[q][e] : 0u;  // 0: no shadow rays, also outside the image
  const uint32_t lp = depth == 0 || mask == 0 ? e : a.epath[q][e];
  int item = 0;
  if (MULTI) {
    if (depth == 0)
      item = item_of<MULTI>(a, a.path_begin + uint32_t(__builtin_amdgcn_readfirstlane(e)));  // one to a tile
    else if (mask)
      item = item_of<MULTI>(a, a.path_begin + lp);
  }
  each_item<MULTI>(a, mask != 0, item, [&](const DevItem& it, bool mine) {
    if (!mine) return;
    const int L = it.sc.L, D1 = it.cam.D + 1;
    int eye, x, y;
    const int64_t p = a.path_begin + lp - it.path_offset;
    if (depth == 0)
      wave_pixel(it.cam, p, &eye, &x, &y);
    else
      path_pixel(it.cam, p, &eye, &x, &y);
    const int64_t pix = int64_t(y) * it.cam.W + x;
    float3 sum = make_float3(0.f, 0.f, 0.f);
    for (int l = 0; l < L; ++l) {
      if (!((mask >> l) & 1u)) continue;
      const size_t k = size_t(l) * a.cap + e;
      const bool v = a.vis[q][k] != 0;
      if (v) sum = add_rn(sum, make_float3(a.contrib[q][3 * k], a.contrib[q][3 * k + 1], a.contrib[q][3 * k + 2]));
      if (PATH_IDS) it.out.shadow_state[eye][(pix * D1 + depth) * L + l] = v ? 2 : 1;
    }
    float* rad = it.out.radiance[eye] + 3 * pix;
    const float3 r = add_rn(make_float3(rad[0], rad[1], rad[2]), sum);
    rad[0] = r.x;
    rad[1] = r.y;
    rad[2] = r.z;
  });
}

template <bool COUNT, bool MULTI>
__global__ __launch_bounds__(kBlock) SRT_TRACE_ATTR void k_trace(KArgs a, int depth) {
  __shared__ uint32_t lstack[kStackLds * kBlock];
  __shared__ unsigned long long share_word[kWaves * std::max(kCoopRays, 1)];
  __shared__ int share_key[kWaves * std::max(kCoopRays, 1)];
  const int lane = lane_id();
  const Share share{&share_word[(threadIdx.x >> 6) * kCoopRays], &share_key[(threadIdx.x >> 6) * kCoopRays]};
  Stack st{&lstack[threadIdx.x], global_scalar(a.gstack), blockIdx.x * uint32_t(kBlock),
           uint32_t(a.trace_threads), a.gstack_entries, 0, false};
  const int LS = a.lstride;
  const bool closest = depth <= a.dmax;
  const bool shadows = depth >= 1;
  const int q = depth & 1;
  const int sq = (depth + 1) & 1;  // parity of depth - 1
  const uint32_t nc = closest ? (depth == 0 ? uint32_t(a.path_count) : a.ctr->refl_count[depth]) : 0u;
  uint32_t rays = nc;
  if (shadows)
    for (int l = 0; l < LS; ++l) rays += a.ctr->shadow_count[depth - 1][l];
  // Work comes in batches of 64 rays, one per lane, or fewer where that still gives every wave of the grid
  // at most one batch: the wave's other lanes then share its rays from the start (see traverse).  A 641x479
  // frame of 13k triangles takes 329 us that way and 436 us in batches of 64; batches of at least 4 or 16
  // rays instead of 8 are within 1%.  A batch of images goes down to one ray a wave: its last rays are of as many images,
  // whose traversals would wait for each other (256 images of 32x32 over 32 scenes, depth 4: 553 us with 8 rays at least,
  // 479 with one).
  const uint32_t nwaves = gridDim.x * uint32_t(kWaves);
  int blog = 6;
  if (!COUNT && kCoopRays > 0 && !a.brute)
    while (blog > min_rays_log2(MULTI) && (rays >> (blog - 1)) < nwaves) --blog;
  const uint32_t nc_pad = round_up(nc, blog);
  uint32_t total = nc_pad;
  if (shadows)
    for (int l = 0; l < LS; ++l) total += round_up(a.ctr->shadow_count[depth - 1][l], blog);
  uint32_t c_nodes = 0, c_tris = 0, s_nodes = 0, s_tris = 0;
  // Larger grabs than one batch unbalance the launch's end, and refilling single lanes stalls the wave on
  // every refill.  Device-scope atomics on one address serialise, so: wave w's first batch is batch w, with
  // no atomic (a launch whose work fits in the first round takes none); later batches b = nwaves + c + K k
  // come from counter c = w mod K of K = min(kWorkCounters, nwaves) interleaved counters, so K atomics
  // proceed at once.
  const uint32_t wid = blockIdx.x * uint32_t(kWaves) + uint32_t(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const uint32_t nbatches = total >> blog;
  // Last come the entries of depth - 2, whose lights' terms are still to be added: work that waits for memory, for
  // waves that would otherwise wait for the launch's last rays.
  const uint32_t nres = !COUNT && a.resolve && depth >= 2
                            ? (depth == 2 ? uint32_t(a.path_count) : a.ctr->refl_count[depth - 2])
                            : 0u;
  const uint32_t nall = nbatches + ((nres + (64u << kResolveLog2) - 1u) >> (6 + kResolveLog2));
  const uint32_t ncounters = nwaves < uint32_t(kWorkCounters) ? nwaves : uint32_t(kWorkCounters);  // each served
  const uint32_t home = wid % ncounters;
  uint32_t batch = wid;
  for (bool first = true;; first = false) {
    if (!first) {
      if (nwaves + home >= nall) break;  // no batch left for this counter
      uint32_t k = 0;
      if (lane == 0) k = atomicAdd(&a.ctr->trace_work[depth][home][0], 1u);
      batch = nwaves + home + ncounters * uint32_t(__builtin_amdgcn_readfirstlane(int(k)));
    }
    if (batch >= nall) break;
    const KArgs& a = kernel_args();  // the same values as the parameter, see kernel_args
    if (!COUNT && batch >= nbatches) {
      for (int k = 0; k < (1 << kResolveLog2); ++k)
        resolve_entry<false, MULTI>(a, depth - 2, ((((batch - nbatches) << kResolveLog2) + k) << 6) + lane, nres);
      continue;
    }
    const uint32_t base = batch << blog;
    const bool filled = lane < (1 << blog);
    if (base < nc_pad) {
      // ---- closest-hit batch
      const uint32_t e = base + lane;
      bool valid = filled && e < nc;
      int k = 0;
      if (MULTI && depth == 0)
        k = item_of<MULTI>(a, a.path_begin + base);  // a tile's paths belong to one item
      else if (MULTI && valid)
        k = item_of<MULTI>(a, a.path_begin + uint32_t(__float_as_int(a.ro[q][e].w)));
      auto ray = [&](const DevItem& it, bool& mine) {
        Ray r{};
        r.limit = INFINITY;
        r.tmin = depth == 0 ? 0.0f : kSecondaryTmin;
        r.exclude = -1;
        if (mine) {
          if (depth == 0) {
            int eye, x, y;
            mine = wave_pixel(it.cam, a.path_begin + e - it.path_offset, &eye, &x, &y);
            if (mine) {
              primary_ray(it.cam, eye, x, y, &r.o, &r.d);
              a.rd[q][e] = make_float4(r.d.x, r.d.y, r.d.z, __int_as_float(-1));
            }
          } else {
            const float4 ro = a.ro[q][e], rd = a.rd[q][e];
            r.o = f3(ro);
            r.d = f3(rd);
            r.exclude = __float_as_int(rd.w);
          }
        }
        return r;
      };
      auto commit = [&](int key, float t) {
        const uint32_t entry = e;
        global_scalar(a.hit)[entry] = make_float2(t, __int_as_float(key));
      };
      each_scene<MULTI>(
          a, valid, k,
          [&](const DevItem& it, bool mine) {
            const Ray r = ray(it, mine);
            traverse<false, COUNT, COUNT || MULTI>(it.sc, mine, r, a.brute != 0, st, share, c_nodes, c_tris, commit);
          },
          [&](const DevItem& it) {
            bool mine = true;
            walk_alone<false, COUNT>(it.sc, ray(it, mine), c_tris, commit);
          });
    } else {
      // ---- shadow batch: find the light whose (padded) range holds this batch
      uint32_t start = nc_pad;
      int l = 0;
      uint32_t cnt = a.ctr->shadow_count[depth - 1][0];
      while (l + 1 < LS && base >= start + round_up(cnt, blog)) {
        start += round_up(cnt, blog);
        ++l;
        cnt = a.ctr->shadow_count[depth - 1][l];
      }
      const uint32_t i = base - start + lane;
      const bool valid = filled && i < cnt;
      const uint32_t owner = valid ? a.sowner[sq][size_t(l) * a.cap + i] : 0u;
      int k = 0;
      if (MULTI && valid) k = item_of<MULTI>(a, a.path_begin + (depth == 1 ? owner : a.epath[sq][owner]));
      auto ray = [&](const DevItem& it, bool mine) {
        Ray r{};
        r.tmin = kSecondaryTmin;
        if (mine) {
          const float4 rec = a.spos[sq][owner];
          r.o = f3(rec);
          r.exclude = __float_as_int(rec.w);
          r.d = shadow_dir(it.sc.lights, l, r.o, &r.limit);
        }
        return r;
      };
      auto commit = [&](int key, float) {
        uint32_t o = owner;
        asm volatile("" : "+v"(o));  // the address is formed here, not before the loop
        global_scalar(a.vis[sq] + size_t(l) * a.cap)[o] = key < 0 ? 1 : 0;
      };
      each_scene<MULTI>(
          a, valid, k,
          [&](const DevItem& it, bool mine) {
            traverse<true, COUNT, COUNT || MULTI>(it.sc, mine, ray(it, mine), a.brute != 0, st, share, s_nodes, s_tris,
                                                  commit);
          },
          [&](const DevItem& it) { walk_alone<true, COUNT>(it.sc, ray(it, true), s_tris, commit); });
    }
  }
  if (st.overflow) atomicOr(&a.ctr->error, 1u);
  if (COUNT) {
    add_work(a.ctr, 0, c_nodes);
    add_work(a.ctr, 1, c_tris);
    add_work(a.ctr, 2, s_nodes);
    add_work(a.ctr, 3, s_tris);
  }
}

// ---------------------------------------------------------------------------------------------
// k_trace_flat: the same rays of a single scene without a tree (spheres and planes only, RT_ACCEL_NONE, one
// triangle) or under RT_FLAG_BRUTE_FORCE: every ray against every primitive.
//
// Primitives are the same for the whole wave, so they are scalar loads and a test is bound by the VALU: 45
// instructions a triangle, half of them behind the division.  Most waves find that no lane is inside a
// triangle's first edge pair long before that (24 instructions on average).  With many primitives, SEGS waves
// share a batch of 64 rays, each over its part of the spheres, planes and triangles: a frame of 131,072 paths is
// 2,048 batches, a quarter of the waves the chip holds, and a launch of few rays would last as long as one wave's
// walk over all of them (0.26 us a triangle, a dependent load, before).  256x256, 2,432 triangles, depth 1, 1
// light: 1815 us with the walk inside k_trace, 357 this way (390 with records loaded two at a time, 420 one at a
// time; 4 or 16 waves a batch: 463).  640x480, depth 4, 2 lights, 4,000 spheres and 520 triangles: 66.7 ms with all
// spheres in the first part, loaded one at a time, 9.1 this way; 256x256, 4 lights, 1,024 spheres: 2390 us through
// k_path, 663.
// ---------------------------------------------------------------------------------------------

constexpr int kFlatSegs = 8;        // waves that share a batch's walk
constexpr int kFlatWaves = 8192;    // waves of a full grid
template <int SEGS>
constexpr int kFlatBlock = SEGS > 1 ? 64 * SEGS : kBlock;

// One of `of` equal shares of a scene's primitives.
struct Part {
  int k, of;
  __device__ inline int first(int n) const { return int(int64_t(n) * k / of); }
  __device__ inline int last(int n) const { return int(int64_t(n) * (k + 1) / of); }
};

// The nearest hit among the primitives of a share.
__device__ __attribute__((always_inline)) inline Best flat_closest(const DevScene& sc, Part part, float3 o, float3 d,
                                                                   float tmin, int exclude) {
  Best best{INFINITY, -1, 0x7fffffff};
  auto accept = [&](float t, int key, int id) {
    if (key != exclude && t < INFINITY && (t < best.t || (t == best.t && id < best.id))) best = Best{t, key, id};
  };
  flat_each(sc.spheres, part.first(sc.S), part.last(sc.S),
            [&](float4 s, int k) { accept(sphere_t(s, o, d, tmin, next_up(best.t)), sc.T + k, sc.T + k); });
  flat_each(sc.planes, part.first(sc.P), part.last(sc.P), [&](float4 p, int k) {
    const int key = sc.T + sc.S + k;
    accept(plane_t(p, o, d, tmin, next_up(best.t)), key, key);
  });
  flat_triangles<kFlatStep>(sc.tris, part.first(sc.T), part.last(sc.T), o, d, tmin, [&] { return next_up(best.t); }, accept);
  return best;
}

// Whether any of them lies in (kSecondaryTmin, dist); in steps, so that a wave whose rays are all answered stops.
__device__ __attribute__((always_inline)) inline bool flat_occluded(const DevScene& sc, Part part, float3 o, float3 d,
                                                                    float dist, int exclude) {
  bool found = false;
  auto accept = [&](float t, int key, int) { found = found || (key != exclude && t < INFINITY); };
  auto steps = [&](int n, auto range) {
    const int last = part.last(n);
    for (int k = part.first(n); k < last && !__all(found); k += 64) range(k, min(k + 64, last));
  };
  steps(sc.S, [&](int first, int last) {
    flat_each(sc.spheres, first, last,
              [&](float4 s, int k) { accept(sphere_t(s, o, d, kSecondaryTmin, dist), sc.T + k, 0); });
  });
  steps(sc.P, [&](int first, int last) {
    flat_each(sc.planes, first, last,
              [&](float4 p, int k) { accept(plane_t(p, o, d, kSecondaryTmin, dist), sc.T + sc.S + k, 0); });
  });
  steps(sc.T, [&](int first, int last) {
    flat_triangles<kFlatStep>(sc.tris, first, last, o, d, kSecondaryTmin, [&] { return dist; }, accept);
  });
  return found;
}

template <int SEGS>
__global__ __launch_bounds__(kFlatBlock<SEGS>) void k_trace_flat(KArgs a, int depth) {
  __shared__ float s_t[SEGS > 1 ? SEGS * 64 : 1];
  __shared__ int s_key[SEGS > 1 ? SEGS * 64 : 1], s_id[SEGS > 1 ? SEGS * 64 : 1];
  __shared__ unsigned long long s_hit[SEGS > 1 ? SEGS : 1];
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int seg = SEGS > 1 ? wave : 0;
  const DevScene& sc = a.one.sc;
  const int LS = a.lstride;
  const int q = depth & 1, sq = (depth + 1) & 1;
  const uint32_t nc = depth > a.dmax ? 0u : (depth == 0 ? uint32_t(a.path_count) : a.ctr->refl_count[depth]);
  const uint32_t nc_pad = round_up(nc, 6);
  uint32_t total = nc_pad;
  if (depth >= 1)
    for (int l = 0; l < LS; ++l) total += round_up(a.ctr->shadow_count[depth - 1][l], 6);
  const Part part{seg, SEGS};
  constexpr uint32_t kPer = SEGS > 1 ? 1 : kFlatBlock<SEGS> / 64;  // batches a block holds at a time
  const uint32_t mine = blockIdx.x * kPer + (SEGS > 1 ? 0u : uint32_t(wave));
  for (uint32_t base = mine * 64u; base < total; base += gridDim.x * kPer * 64u) {  // block-uniform with SEGS > 1
    if (base < nc_pad) {
      // ---- closest-hit batch
      const uint32_t e = base + lane;
      bool valid = e < nc;
      float3 o = make_float3(0.f, 0.f, 0.f), d = o;
      int exclude = -1;
      if (valid) {
        if (depth == 0) {
          int eye, x, y;
          valid = wave_pixel(a.one.cam, a.path_begin + e, &eye, &x, &y);
          if (valid) {
            primary_ray(a.one.cam, eye, x, y, &o, &d);
            if (seg == 0) a.rd[q][e] = make_float4(d.x, d.y, d.z, __int_as_float(-1));
          }
        } else {
          const float4 ro = a.ro[q][e], rd = a.rd[q][e];
          o = f3(ro);
          d = f3(rd);
          exclude = __float_as_int(rd.w);
        }
      }
      Best best{INFINITY, -1, 0x7fffffff};
      if (valid)
        best = flat_closest(sc, part, o, d, depth == 0 ? 0.0f : kSecondaryTmin, exclude);
      if (SEGS > 1) {
        s_t[wave * 64 + lane] = best.t;
        s_id[wave * 64 + lane] = best.id;
        s_key[wave * 64 + lane] = best.key;
        __syncthreads();
        if (wave == 0) {
          for (int w = 1; w < SEGS; ++w) {
            const float t = s_t[w * 64 + lane];
            const int id = s_id[w * 64 + lane];
            if (t < best.t || (t == best.t && id < best.id)) best = Best{t, s_key[w * 64 + lane], id};
          }
        }
      }
      if (valid && seg == 0) a.hit[e] = make_float2(best.t, __int_as_float(best.key));
    } else {
      // ---- shadow batch: find the light whose (padded) range holds this batch
      uint32_t start = nc_pad;
      int l = 0;
      uint32_t cnt = a.ctr->shadow_count[depth - 1][0];
      while (l + 1 < LS && base >= start + round_up(cnt, 6)) {
        start += round_up(cnt, 6);
        ++l;
        cnt = a.ctr->shadow_count[depth - 1][l];
      }
      const uint32_t i = base - start + lane;
      const bool valid = i < cnt;
      uint32_t owner = 0;
      bool found = false;
      if (valid) {
        owner = a.sowner[sq][size_t(l) * a.cap + i];
        const float4 rec = a.spos[sq][owner];
        const float3 P = f3(rec);
        float dist;
        const float3 d = shadow_dir(sc.lights, l, P, &dist);
        found = flat_occluded(sc, part, P, d, dist, __float_as_int(rec.w));
      }
      uint64_t hits = __ballot(found);
      if (SEGS > 1) {
        if (lane == 0) s_hit[wave] = hits;
        __syncthreads();
        if (wave == 0)
          for (int w = 1; w < SEGS; ++w) hits |= s_hit[w];
      }
      if (valid && seg == 0) a.vis[sq][size_t(l) * a.cap + owner] = (hits >> lane) & 1 ? 0 : 1;
    }
    if (SEGS > 1) __syncthreads();  // the LDS results are reused by the next batch
  }
}

__device__ inline void material_of(const DevScene& sc, int key, float4* m0, float4* m1, float4* m2) {
  uint32_t mat;
  if (key < sc.T) {
    mat = uint32_t(__float_as_int(sc.tris[3 * key + 1].w));
  } else if (key < sc.T + sc.S) {
    mat = sc.sphere_mat[key - sc.T];
  } else {
    mat = sc.plane_mat[key - sc.T - sc.S];
  }
  *m0 = sc.materials[3 * mat];
  *m1 = sc.materials[3 * mat + 1];
  *m2 = sc.materials[3 * mat + 2];
}

__device__ inline float3 geometric_normal(const DevScene& sc, int key, float3 P) {
  if (key < sc.T) {
    const float3 e1 = f3(sc.tris[3 * key + 1]), e2 = f3(sc.tris[3 * key + 2]);
    return normalize(fcross(e1, e2));
  }
  if (key < sc.T + sc.S) {
    const float4 s = sc.spheres[key - sc.T];
    return (1.0f / s.w) * (P - f3(s));
  }
  const float4 p = sc.planes[key - sc.T - sc.S];
  return normalize(make_float3(p.x, p.y, p.z));
}

__device__ inline int32_t out_id(const DevScene& sc, int key) {
  if (key < 0) return -1;
  if (key < sc.T) return __float_as_int(sc.tris[3 * key].w);
  return key;
}

// The pieces of the shading, shared by the kernels that shade.

// The unit normal at P, turned towards the ray of direction d.
__device__ inline float3 facing_normal(const DevScene& sc, int key, float3 P, float3 d) {
  const float3 n = geometric_normal(sc, key, P);
  return fdot(n, d) > 0.0f ? -1.0f * n : n;
}

// The direction and distance from P to light l, and the cosine at the surface.
__device__ inline float light_at(const float4* lights, int l, float3 P, float3 N, float3* Ld, float* dist) {
  *Ld = shadow_dir(lights, l, P, dist);
  return fdot(N, *Ld);
}

// Light l's term (direction Ld, cosine ndl from light_at) times the path's throughput, for a surface of material
// (m0, m1) seen along d.
__device__ inline float3 light_term(const float4* lights, int l, float ndl, float3 Ld, float3 N, float3 d, float4 m0,
                                    float4 m1, float3 thr) {
  const float3 R = fmad(2.0f * ndl, N, -1.0f * Ld);
  const float spec = powf(fmaxf(0.0f, fdot(R, -1.0f * d)), m0.w);
  const float3 I = f3(lights[2 * l + 1]);
  return mul(mul(I, fmad(ndl, f3(m0), spec * f3(m1))), thr);
}

// The mirror direction of d at a surface of normal N.
__device__ inline float3 mirror_of(float3 d, float3 N) { return normalize(fmad(-(2.0f * fdot(d, N)), N, d)); }

// ---------------------------------------------------------------------------------------------
// k_shade: one thread per hit of depth `depth`.  Each block takes 512 consecutive entries per
// iteration; new shadow records (one queue per light) and mirror rays are compacted with wave
// ballots, a block prefix over the waves and one atomic per block and queue.
//
// The launches of depth 0 are bound by memory (3.8 TB/s, most of it written), so little is written: what all
// lights share (the hit point) once an entry, a light's queue holds entry numbers only, a term is 12 bytes in
// its light's own array (a batch's scenes with fewer lights than the most leave no gaps in it), a path's
// index is its entry at depth 0, and the origin of a primary ray is the eye.  Bytes a path with n lit lights
// at depth 0: 20 + 36 n before, 29 + 16 n now, and 24 instead of 40 from the traversal.  A light's direction and
// term are computed once, in one loop.  A batch's scene is the same for nearly every wave, see each_item.
// Depth-0 shading and resolve, before and now: 1920x1080, 4 lights 175 + 66 us, 122 + 48; 16 mixed scenes
// 1047 + 411 us, 744 + 255.
// Registers for 8 waves per SIMD; the batch's kernel would spill 8 of them (8 small scenes 970 us, 915 with 6).
// ---------------------------------------------------------------------------------------------

template <bool PATH_IDS, bool MULTI>
__global__ __launch_bounds__(kShadeBlock) __attribute__((amdgpu_waves_per_eu(MULTI ? 6 : 8))) void k_shade(
    KArgs a, int depth) {
  __shared__ uint32_t wcnt[kShadeWaves][RT_MAX_LIGHTS + 1];
  __shared__ uint32_t bbase[RT_MAX_LIGHTS + 1];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int q = depth & 1, nq = (depth + 1) & 1;
  const uint32_t total = depth == 0 ? uint32_t(a.path_count) : a.ctr->refl_count[depth];
  const int LS = a.lstride;
  uint32_t n_primary = 0;
  for (uint32_t base = blockIdx.x * kShadeBlock; base < total; base += gridDim.x * kShadeBlock) {  // block-uniform loop
    const uint32_t e = base + threadIdx.x;
    const bool active = e < total;
    uint32_t mask = 0, lp = e;
    bool spawn = false;
    float3 P = make_float3(0.f, 0.f, 0.f), rdir = P, next = P;
    int key = -1, item = 0;
    if (depth > 0 && active) lp = uint32_t(__float_as_int(a.ro[q][e].w));
    if (MULTI) {
      if (depth == 0)
        item = item_of<MULTI>(a, a.path_begin + uint32_t(__builtin_amdgcn_readfirstlane(e)));  // one to a tile
      else if (active)
        item = item_of<MULTI>(a, a.path_begin + lp);
    }
    each_item<MULTI>(a, active, item, [&](const DevItem& it, bool mine) {
      const DevScene& sc = it.sc;
      const int L = sc.L, D1 = it.cam.D + 1;
      int eye = 0, x = 0, y = 0;
      if (!mine) return;
      const int64_t p = a.path_begin + lp - it.path_offset;
      if (!(depth == 0 ? wave_pixel(it.cam, p, &eye, &x, &y) : path_pixel(it.cam, p, &eye, &x, &y))) return;
      const float4 rd = a.rd[q][e];
      const float2 hit = a.hit[e];
      float3 thr = make_float3(1.f, 1.f, 1.f);
      if (depth > 0) thr = f3(a.thr[q][e]);
      key = __float_as_int(hit.y);
      const int64_t pix = int64_t(y) * it.cam.W + x;
      float* rad = it.out.radiance[eye] + 3 * pix;
      const float3 o = depth == 0 ? eye_position(it.cam, eye) : f3(a.ro[q][e]), d = f3(rd);
      if (depth == 0) {
        ++n_primary;
        if (it.out.hit_t[eye]) it.out.hit_t[eye][pix] = hit.x;
        if (it.out.hit_prim[eye]) it.out.hit_prim[eye][pix] = out_id(sc, key);
        if (PATH_IDS) {
          for (int k = 0; k < D1; ++k) it.out.path_prims[eye][pix * D1 + k] = -2;
          for (int k = 0; k < D1 * L; ++k) it.out.shadow_state[eye][pix * D1 * L + k] = 0;
        }
      }
      if (PATH_IDS) it.out.path_prims[eye][pix * D1 + depth] = out_id(sc, key);
      float3 add;
      if (key < 0) {
        add = mul(thr, make_float3(sc.background[0], sc.background[1], sc.background[2]));
      } else {
        P = fmad(hit.x, d, o);
        const float3 N = facing_normal(sc, key, P, d);
        float4 m0, m1, m2;
        material_of(sc, key, &m0, &m1, &m2);
        add = mul(thr, mul(make_float3(sc.ambient[0], sc.ambient[1], sc.ambient[2]), f3(m0)));
        for (int l = 0; l < L; ++l) {
          float3 Ld;
          float dist;
          const float ndl = light_at(sc.lights, l, P, N, &Ld, &dist);
          if (dist > kSecondaryTmin && ndl > 0.0f) {
            mask |= 1u << l;
            const float3 term = light_term(sc.lights, l, ndl, Ld, N, d, m0, m1, thr);
            float* c = a.contrib[q] + 3 * (size_t(l) * a.cap + e);
            c[0] = term.x;
            c[1] = term.y;
            c[2] = term.z;
          }
        }
        if (depth < it.cam.D && (m2.x != 0.0f || m2.y != 0.0f || m2.z != 0.0f)) {
          spawn = true;
          rdir = mirror_of(d, N);
          next = mul(thr, f3(m2));
        }
      }
      if (depth > 0) add = add_rn(make_float3(rad[0], rad[1], rad[2]), add);
      rad[0] = add.x;
      rad[1] = add.y;
      rad[2] = add.z;
    });
    if (active) {
      a.smask[q][e] = uint8_t(mask);  // 0 too for paths outside the image
      if (depth > 0) a.epath[q][e] = lp;
      if (mask) a.spos[q][e] = make_float4(P.x, P.y, P.z, __int_as_float(key));
    }
    // per-wave counts of every queue (light queues 0..LS-1, mirror queue LS), then one atomic per
    // block and queue
    for (int l = 0; l <= LS; ++l) {
      const uint64_t bal = __ballot(l < LS ? ((mask >> l) & 1u) != 0 : spawn);
      if (lane == 0) wcnt[wave][l] = uint32_t(__popcll(bal));
    }
    __syncthreads();
    if (threadIdx.x <= uint32_t(LS)) {
      const int l = threadIdx.x;
      uint32_t run = 0;
      for (int w = 0; w < kShadeWaves; ++w) {
        const uint32_t c = wcnt[w][l];
        wcnt[w][l] = run;
        run += c;
      }
      uint32_t* ctr = l < LS ? &a.ctr->shadow_count[depth][l] : &a.ctr->refl_count[depth + 1];
      bbase[l] = run ? atomicAdd(ctr, run) : 0u;
    }
    __syncthreads();
    for (int l = 0; l < LS; ++l) {
      const bool mine = ((mask >> l) & 1u) != 0;
      const uint64_t bal = __ballot(mine);
      if (mine) {
        const uint32_t slot = bbase[l] + wcnt[wave][l] + uint32_t(lanes_below(bal));
        a.sowner[q][size_t(l) * a.cap + slot] = e;
      }
    }
    {
      const uint64_t bal = __ballot(spawn);
      if (spawn) {
        const uint32_t slot = bbase[LS] + wcnt[wave][LS] + uint32_t(lanes_below(bal));
        a.ro[nq][slot] = make_float4(P.x, P.y, P.z, __int_as_float(int(lp)));
        a.rd[nq][slot] = make_float4(rdir.x, rdir.y, rdir.z, __int_as_float(key));
        a.thr[nq][slot] = make_float4(next.x, next.y, next.z, 0.f);
      }
    }
    __syncthreads();  // wcnt / bbase are reused by the next iteration
  }
  if (depth == 0) {  // one atomic per block: device-scope atomics on one address serialise
    for (int off = 32; off > 0; off >>= 1) n_primary += __shfl_xor(n_primary, off);
    if (lane == 0) wcnt[wave][0] = n_primary;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t sum = 0;
      for (int w = 0; w < kShadeWaves; ++w) sum += wcnt[w][0];
      if (sum) atomicAdd(&a.ctr->primary, sum);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// k_path: a small frame in one launch.  A wave takes its paths through the whole recursion -- closest hit,
// shading, each light's shadow rays, the mirror ray -- with the pieces of the queue kernels, so each pixel
// gets the same operations in the same order and the same bits.  A small frame is bound by its launches: the
// queues cost 2 + 3 (D + 1) of them, each waiting for the last ray of the one before.  Here a wave waits only
// for its own rays, its idle lanes share them (see traverse), and nothing passes through memory but the
// result.  Larger frames gain more from the queues, which fill every wave with live rays.
// A hit's shadow rays are packed over the lights, so a wave makes as many rounds as its rays need and not one a
// light (641x479, 13k triangles, depth 4, 2 lights: 280 us a light at a time, 257 packed, 317 by queues).
// 256x256, depth 1, 1 light: spheres 46.3 -> 16.5 us, 100 triangles 68.4 -> 48.2.  5 waves per SIMD with 8
// spilled registers; 4 without spills or 6 with 37 take 5% longer on that frame, which now takes 235 us.
// ---------------------------------------------------------------------------------------------

#ifndef SRT_PATH_WAVES
#define SRT_PATH_WAVES 5
#endif

template <bool TREE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(SRT_PATH_WAVES))) void k_path(
    KArgs a, int blog, int dynamic, int64_t* out) {
  __shared__ uint32_t lstack[TREE ? kStackLds * kBlock : 1];
  __shared__ unsigned long long share_word[TREE ? kWaves * std::max(kCoopRays, 1) : 1];
  __shared__ int share_key[TREE ? kWaves * std::max(kCoopRays, 1) : 1];
  __shared__ uint32_t s_cnt[3][kWaves];
  __shared__ uint16_t s_ray[kWaves][64 * RT_MAX_LIGHTS];              // lane | light << 6
  __shared__ unsigned long long s_visible[kWaves][RT_MAX_LIGHTS];     // a bit a ray
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Share share{&share_word[TREE ? wave * kCoopRays : 0], &share_key[TREE ? wave * kCoopRays : 0]};
  Stack st{&lstack[TREE ? threadIdx.x : 0], global_scalar(a.gstack), blockIdx.x * uint32_t(kBlock),
           uint32_t(a.trace_threads), a.gstack_entries, 0, false};
  const DevScene& sc = a.one.sc;
  const uint32_t count = uint32_t(a.path_count), nwaves = gridDim.x * uint32_t(kWaves);
  uint32_t n_refl = 0, n_shadow = 0, unused = 0;
  // A wave takes its first batch by its number and, in a dynamic launch (whose counters were set to zero before), later
  // ones from interleaved counters, as k_trace does.
  const uint32_t wid = blockIdx.x * uint32_t(kWaves) + wave, ncounters = min(nwaves, uint32_t(kWorkCounters));
  auto later = [&] {
    uint32_t k = 0;
    if (lane == 0) k = atomicAdd(&kernel_args().ctr->trace_work[RT_MAX_DEPTH + 1][wid % ncounters][0], 1u);
    return nwaves + wid % ncounters + ncounters * uint32_t(__builtin_amdgcn_readfirstlane(int(k)));
  };
  for (uint32_t batch = wid; (uint64_t(batch) << blog) < count; batch = later()) {
    const uint32_t e = (batch << blog) + lane;
    float3 o = make_float3(0.f, 0.f, 0.f), d = o;
    int eye = 0, x = 0, y = 0;
    bool alive = lane < (1 << blog) && e < count && wave_pixel(a.one.cam, e, &eye, &x, &y);
    const bool inside = alive;
    if (alive) primary_ray(a.one.cam, eye, x, y, &o, &d);
    float3 thr = make_float3(1.f, 1.f, 1.f), rad = make_float3(0.f, 0.f, 0.f), sum = rad;
    bool lit = false;  // `sum` holds the lights' terms of the hit before, still to be added
    int exclude = -1;
    for (int depth = 0; __ballot(alive) != 0; ++depth) {
      // The arguments read afresh at every depth: kept from the start they spilled 79 scalar registers (641x479, 13k
      // triangles: 257 -> 255 us).
      const KArgs& a = kernel_args();  // the same values as the parameter, see kernel_args
      const DevScene& sc = a.one.sc;
      const float tmin = depth == 0 ? 0.0f : kSecondaryTmin;
      float t = INFINITY;
      int key = -1;
      if (TREE) {
        Ray r{o, d, tmin, INFINITY, exclude};
        traverse<false, false, false>(sc, alive, r, false, st, share, unused, unused, [&](int k, float tk) {
          key = k;
          t = tk;
        });
      } else if (alive) {
        const Best b = flat_closest(sc, Part{0, 1}, o, d, tmin, exclude);
        key = b.key;
        t = b.t;
      }
      float3 P = o, N = o;
      uint32_t mask = 0;
      bool spawn = false;
      if (alive) {
        if (depth == 0) {
          const int64_t pix = int64_t(y) * a.one.cam.W + x;
          if (a.one.out.hit_t[eye]) a.one.out.hit_t[eye][pix] = t;
          if (a.one.out.hit_prim[eye]) a.one.out.hit_prim[eye][pix] = out_id(sc, key);
        }
        float3 add;
        if (key < 0) {
          add = mul(thr, make_float3(sc.background[0], sc.background[1], sc.background[2]));
        } else {
          P = fmad(t, d, o);
          N = facing_normal(sc, key, P, d);
          float4 m0, m1, m2;
          material_of(sc, key, &m0, &m1, &m2);
          add = mul(thr, mul(make_float3(sc.ambient[0], sc.ambient[1], sc.ambient[2]), f3(m0)));
          for (int l = 0; l < sc.L; ++l) {
            float3 Ld;
            float dist;
            const float ndl = light_at(sc.lights, l, P, N, &Ld, &dist);
            if (dist > kSecondaryTmin && ndl > 0.0f) mask |= 1u << l;
          }
          spawn = depth < a.one.cam.D && (m2.x != 0.0f || m2.y != 0.0f || m2.z != 0.0f);
        }
        // the queue kernels' order: this depth's term, then the lights of the depth before
        rad = depth == 0 ? add : add_rn(rad, add);
        if (lit) rad = add_rn(rad, sum);
        sum = make_float3(0.f, 0.f, 0.f);
        lit = mask != 0;
      }
      // The shadow rays of all lights, packed: a wave traces them 64 at a time, whichever light they head for.
      uint32_t rays = 0;
      for (int l = 0; l < sc.L; ++l) {
        const bool cast = ((mask >> l) & 1u) != 0;
        const uint64_t b = __ballot(cast);
        if (cast) lds_put(&s_ray[wave][rays + lanes_below(b)], uint16_t(lane | (l << 6)));
        rays += uint32_t(__popcll(b));
      }
      for (uint32_t first = 0; first < rays; first += 64) {
        const bool cast = first + lane < rays;
        const uint32_t r = cast ? uint32_t(lds_get(&s_ray[wave][first + lane])) : uint32_t(lane);
        const int from = int(r & 63u);
        const float3 from_P = make_float3(shfl_f(P.x, from), shfl_f(P.y, from), shfl_f(P.z, from));
        const int from_key = shfl_i(key, from);
        bool visible = false;
        float dist = 0.0f;
        float3 Ld = from_P;
        if (cast) Ld = shadow_dir(sc.lights, int(r >> 6), from_P, &dist);
        if (TREE) {
          traverse<true, false, false>(sc, cast, Ray{from_P, Ld, kSecondaryTmin, dist, from_key}, false, st, share,
                                       unused, unused, [&](int k, float) { visible = k < 0; });
        } else if (cast) {
          visible = !flat_occluded(sc, Part{0, 1}, from_P, Ld, dist, from_key);
        }
        const uint64_t v = __ballot(visible);
        if (lane == 0) lds_put(&s_visible[wave][first >> 6], static_cast<unsigned long long>(v));
      }
      n_shadow += lane == 0 ? rays : 0u;
      rays = 0;
      for (int l = 0; l < sc.L; ++l) {
        const bool cast = ((mask >> l) & 1u) != 0;
        const uint64_t b = __ballot(cast);
        const uint32_t r = rays + lanes_below(b);
        rays += uint32_t(__popcll(b));
        if (cast && ((lds_get(&s_visible[wave][r >> 6]) >> (r & 63u)) & 1u)) {
          float4 m0, m1, m2;
          material_of(sc, key, &m0, &m1, &m2);
          float3 Ld;
          float dist;
          const float ndl = light_at(sc.lights, l, P, N, &Ld, &dist);
          sum = add_rn(sum, light_term(sc.lights, l, ndl, Ld, N, d, m0, m1, thr));
        }
      }
      if (spawn) {
        float4 m0, m1, m2;
        material_of(sc, key, &m0, &m1, &m2);
        d = mirror_of(d, N);
        o = P;
        thr = mul(thr, f3(m2));
        exclude = key;
        ++n_refl;
      }
      alive = spawn;
    }
    if (inside) {
      if (lit) rad = add_rn(rad, sum);
      wave_pixel(a.one.cam, e, &eye, &x, &y);
      float* pixel = a.one.out.radiance[eye] + 3 * (int64_t(y) * a.one.cam.W + x);
      pixel[0] = rad.x;
      pixel[1] = rad.y;
      pixel[2] = rad.z;
    }
    if (!dynamic) break;
  }
  for (int off = 32; off > 0; off >>= 1) {
    n_refl += __shfl_xor(n_refl, off);
    n_shadow += __shfl_xor(n_shadow, off);
  }
  const uint32_t broken = __ballot(st.overflow) != 0 ? 1u : 0u;
  if (lane == 0) s_cnt[0][wave] = n_refl, s_cnt[1][wave] = n_shadow, s_cnt[2][wave] = broken;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint4 c = make_uint4(0u, 0u, 0u, 0u);
    for (int w = 0; w < kWaves; ++w) c.x += s_cnt[0][w], c.y += s_cnt[1][w], c.z |= s_cnt[2][w];
    if (out) {
      unsigned long long* sum = reinterpret_cast<unsigned long long*>(out);
      if (blockIdx.x == 0) atomicAdd(&sum[RT_COUNT_PRIMARY], 2ull * a.one.cam.W * a.one.cam.H);
      if (c.x) atomicAdd(&sum[RT_COUNT_REFLECTION], c.x);
      if (c.y) atomicAdd(&sum[RT_COUNT_SHADOW], c.y);
      // one error a launch: the first block to leave the launch's number in the workspace adds it
      const KArgs& a = kernel_args();
      if (c.z && atomicExch(&a.ctr->stopped, a.launch) != a.launch) atomicAdd(&sum[RT_COUNT_ERRORS], 1ull);
    } else {
      reinterpret_cast<uint4*>(a.ctr)[blockIdx.x] = c;  // for k_path_finish, in the counters' bytes
    }
  }
}
static_assert(offsetof(Counters, trace_work) + sizeof(Counters::trace_work) / (RT_MAX_DEPTH + 2) * (RT_MAX_DEPTH + 1) >=
                  kMaxTraceBlocks * sizeof(uint4),
              "the blocks' counts end before the work counters in use");
static_assert(offsetof(Counters, stopped) >= kMaxTraceBlocks * sizeof(uint4), "... and before the launch's number");

// Adds the counts of k_path's blocks where they do not do it themselves.
__global__ __launch_bounds__(kBlock) void k_path_finish(const uint4* counts, int blocks, int64_t primary, int64_t* out) {
  __shared__ unsigned long long s_sum[2];
  __shared__ uint32_t s_err;
  if (threadIdx.x == 0) s_sum[0] = s_sum[1] = 0, s_err = 0;
  __syncthreads();
  unsigned long long refl = 0, shadow = 0;
  uint32_t err = 0;
  for (int i = threadIdx.x; i < blocks; i += kBlock) refl += counts[i].x, shadow += counts[i].y, err |= counts[i].z;
  for (int off = 32; off > 0; off >>= 1) {
    refl += __shfl_xor(refl, off);
    shadow += __shfl_xor(shadow, off);
    err |= __shfl_xor(err, off);
  }
  if (lane_id() == 0) {
    atomicAdd(&s_sum[0], refl);
    atomicAdd(&s_sum[1], shadow);
    atomicOr(&s_err, err);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    out[RT_COUNT_PRIMARY] += primary;
    out[RT_COUNT_REFLECTION] += int64_t(s_sum[0]);
    out[RT_COUNT_SHADOW] += int64_t(s_sum[1]);
    out[RT_COUNT_ERRORS] += s_err;
  }
}

// k_resolve: the lights' terms of one depth, see resolve_entry.
template <bool PATH_IDS, bool MULTI>
__global__ __launch_bounds__(kBlock) void k_resolve(KArgs a, int depth) {
  const uint32_t total = depth == 0 ? uint32_t(a.path_count) : a.ctr->refl_count[depth];
  for (uint32_t base = blockIdx.x * kBlock; base < total; base += gridDim.x * kBlock)
    resolve_entry<PATH_IDS, MULTI>(a, depth, base + threadIdx.x, total);
}

// One workgroup clears the counters (41 KB, most of it the spaced work cursors), 16 bytes a store.
constexpr int kResetBlock = 1024;
static_assert(sizeof(Counters) % 4 == 0, "Counters is cleared in words");
__global__ __launch_bounds__(kResetBlock) void k_reset(Counters* ctr) {
  constexpr int kQuads = int(sizeof(Counters) / 16), kWords = int(sizeof(Counters) / 4);
  uint4* q = reinterpret_cast<uint4*>(ctr);  // the workspace is 256-byte aligned and the counters come first
  for (int i = threadIdx.x; i < kQuads; i += kResetBlock) q[i] = make_uint4(0u, 0u, 0u, 0u);
  uint32_t* p = reinterpret_cast<uint32_t*>(ctr);
  for (int i = 4 * kQuads + threadIdx.x; i < kWords; i += kResetBlock) p[i] = 0;
}

__global__ void k_finish(const Counters* ctr, int D, int L, int64_t* out) {
  if (threadIdx.x != 0) return;
  int64_t refl = 0, shadow = 0;
  for (int d = 1; d <= D; ++d) refl += ctr->refl_count[d];
  for (int d = 0; d <= D; ++d)
    for (int l = 0; l < L; ++l) shadow += ctr->shadow_count[d][l];
  out[RT_COUNT_PRIMARY] += ctr->primary;
  out[RT_COUNT_REFLECTION] += refl;
  out[RT_COUNT_SHADOW] += shadow;
  out[RT_COUNT_CLOSEST_NODES] += int64_t(ctr->work[0]);
  out[RT_COUNT_CLOSEST_TRIS] += int64_t(ctr->work[1]);
  out[RT_COUNT_ANY_NODES] += int64_t(ctr->work[2]);
  out[RT_COUNT_ANY_TRIS] += int64_t(ctr->work[3]);
  out[RT_COUNT_ERRORS] += ctr->error;
}

// Readback: a grid of a few workgroups streams the radiance into mapped pinned host memory, so the
// copy leaves the compute units to the next frame's traversal.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void k_copy_to_host16(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                           size_t n) {
  for (size_t i = size_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += size_t(gridDim.x) * kBlock)
    __builtin_nontemporal_store(src[i], &dst[i]);
}

__global__ __launch_bounds__(kBlock) void k_copy_to_host4(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst,
                                                          size_t n) {
  for (size_t i = size_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += size_t(gridDim.x) * kBlock)
    __builtin_nontemporal_store(src[i], &dst[i]);
}

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// A number that no other launch has, of this process or of one that used the memory before; never 0.
unsigned long long launch_number() {
  static std::atomic<unsigned long long> next{
      static_cast<unsigned long long>(std::chrono::system_clock::now().time_since_epoch().count())};
  return (2 * next.fetch_add(1, std::memory_order_relaxed) + 1) * 0x9e3779b97f4a7c15ull;
}

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

template <typename K>
hipError_t launch(K kernel, unsigned grid, const KArgs& a, int depth, hipStream_t s, TimerImpl* timer, int stage,
                  int block = kBlock) {
  if (timer) timer_begin(timer, stage, s);
  kernel<<<grid, block, 0, s>>>(a, depth);
  hipError_t e = hipGetLastError();
  if (timer) timer_end(timer, stage, s);
  return e;
}

}  // namespace

hipError_t copy_to_host(const void* src, void* host_dst_device_view, size_t bytes, int blocks, hipStream_t s) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(src), b = reinterpret_cast<uintptr_t>(host_dst_device_view);
  if (((a | b) & 15u) == 0 && bytes % 16 == 0) {
    k_copy_to_host16<<<blocks, kBlock, 0, s>>>(static_cast<const u32x4*>(src),
                                               static_cast<u32x4*>(host_dst_device_view), bytes / 16);
  } else {
    k_copy_to_host4<<<blocks, kBlock, 0, s>>>(static_cast<const uint32_t*>(src),
                                              static_cast<uint32_t*>(host_dst_device_view), bytes / 4);
  }
  return hipGetLastError();
}

int resident_blocks(int device, int blocks_per_cu, GridOf kernel) {
  // per device (the current one, which the occupancy query reads): CUs and each kernel's workgroups per CU, looked up
  // once; renders may come from several threads
  static std::mutex lock;
  static int cached_cus[64] = {0}, cached_occ[64][4] = {{0}};
  if (device < 0 || device >= 64) return kMaxTraceBlocks;
  std::lock_guard<std::mutex> guard(lock);
  if (!cached_cus[device]) {
    hipDeviceProp_t prop;
    int cus = 256;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess) cus = prop.multiProcessorCount;
    auto look = [&](GridOf which, const void* f) {
      int occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, kBlock, 0) != hipSuccess || occ <= 0) occ = 4;
      cached_occ[device][int(which)] = occ;
    };
    look(GridOf::trace, reinterpret_cast<const void*>(k_trace<false, false>));
    look(GridOf::trace_batch, reinterpret_cast<const void*>(k_trace<false, true>));
    look(GridOf::path_flat, reinterpret_cast<const void*>(k_path<false>));
    look(GridOf::path_tree, reinterpret_cast<const void*>(k_path<true>));
    cached_cus[device] = cus;
  }
  int per_cu = cached_occ[device][int(kernel)];
  if (blocks_per_cu > 0) per_cu = std::min(per_cu, blocks_per_cu);
  return std::min(kMaxTraceBlocks, cached_cus[device] * per_cu);
}

int spill_entries_for_depth(int32_t bvh_depth) {
  // at most (width - 1) = 3 entries wait per level of the tree; the newest kStackLds stay in LDS
  return std::min(kStackGlobal, std::max(1, 3 * bvh_depth - kStackLds + 1));
}

size_t plan_render(int64_t chunk, int32_t L, int grid_trace, RenderPlan* p, int stack_entries, int stack_threads) {
  if (stack_entries <= 0 || stack_entries > kStackGlobal) stack_entries = kStackGlobal;
  if (stack_threads <= 0) stack_threads = kMaxTraceBlocks * kBlock;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  const size_t n = size_t(chunk);
  const size_t ns = n * size_t(std::max(L, 1));
  p->chunk_paths = chunk;
  p->grid_trace = grid_trace;
  p->counters_off = take(sizeof(Counters));
  for (int k = 0; k < 2; ++k) {
    p->ro_off[k] = take(n * 16);
    p->rd_off[k] = take(n * 16);
    p->thr_off[k] = take(n * 16);
    p->epath_off[k] = take(n * 4);
    p->smask_off[k] = take(n);
    p->spos_off[k] = take(n * 16);
    p->sowner_off[k] = take(ns * 4);
    p->contrib_off[k] = take(ns * 12);
    p->vis_off[k] = take(ns);
  }
  p->hit_off = take(n * 8);
  p->stack_entries = stack_entries;
  p->stack_threads = stack_threads;
  p->gstack_off = take(size_t(stack_threads) * size_t(stack_entries) * 4);
  p->bytes = off;
  return off;
}

hipError_t render_chunk(const RenderArgs& ra, hipStream_t s, TimerImpl* timer) {
  KArgs a{};
  const bool multi = ra.items != nullptr;
  a.one = ra.one;
  a.items = ra.items;
  a.num_items = multi ? ra.num_items : 1;
  a.lstride = std::max(ra.max_lights, 1);
  a.dmax = ra.max_depth;
  char* ws = ra.ws;
  const RenderPlan& p = ra.plan;
  a.ctr = reinterpret_cast<Counters*>(ws + p.counters_off);
  for (int k = 0; k < 2; ++k) {
    a.ro[k] = reinterpret_cast<float4*>(ws + p.ro_off[k]);
    a.rd[k] = reinterpret_cast<float4*>(ws + p.rd_off[k]);
    a.thr[k] = reinterpret_cast<float4*>(ws + p.thr_off[k]);
    a.epath[k] = reinterpret_cast<uint32_t*>(ws + p.epath_off[k]);
    a.smask[k] = reinterpret_cast<uint8_t*>(ws + p.smask_off[k]);
    a.spos[k] = reinterpret_cast<float4*>(ws + p.spos_off[k]);
    a.sowner[k] = reinterpret_cast<uint32_t*>(ws + p.sowner_off[k]);
    a.contrib[k] = reinterpret_cast<float*>(ws + p.contrib_off[k]);
    a.vis[k] = reinterpret_cast<uint8_t*>(ws + p.vis_off[k]);
  }
  a.hit = reinterpret_cast<float2*>(ws + p.hit_off);
  a.gstack = reinterpret_cast<uint32_t*>(ws + p.gstack_off);
  const bool ids = (ra.flags & RT_FLAG_PATH_IDS) != 0;
  const bool count = (ra.flags & RT_FLAG_COUNT_WORK) != 0;
  a.path_begin = ra.path_begin;
  a.path_count = ra.path_count;
  a.cap = uint32_t(p.chunk_paths);
  a.brute = (ra.flags & RT_FLAG_BRUTE_FORCE) ? 1 : 0;
  a.trace_threads = p.grid_trace * kBlock;
  a.gstack_entries = p.stack_entries;
  if (a.trace_threads > p.stack_threads) return hipErrorInvalidValue;  // the spill area is per grid thread

  // The persistent grid, cut where the launch cannot hold that many batches (small frames: a workgroup
  // without work still costs its dispatch).
  auto gtrace = [&](int d, int64_t rays_per_block, int64_t most) {
    const int64_t rays = ra.path_count * ((d <= ra.max_depth ? 1 : 0) + (d >= 1 ? ra.max_lights : 0) + (d >= 2 ? 1 : 0));
    return unsigned(std::max<int64_t>(1, std::min<int64_t>(most, (rays + rays_per_block - 1) / rays_per_block)));
  };
  // Single scenes without a tree to walk have kernels of their own (the work counters are k_trace's).
  const bool flat = !multi && !count && (a.brute || !ra.one.sc.has_bvh);
  SceneSize size = scene_size(ra.one.sc);
  size.flat = flat;
  const unsigned gstream =
      unsigned(std::max<int64_t>(1, std::min<int64_t>((ra.path_count + kBlock - 1) / kBlock, ra.stream_blocks)));
  const unsigned gshade = unsigned(std::max<int64_t>(
      1, std::min<int64_t>((ra.path_count + kShadeBlock - 1) / kShadeBlock, ra.stream_blocks * kBlock / kShadeBlock)));
  hipError_t e;
  // A small frame in one launch: whole frames only (the ray counts take the pixels as traced), and neither ray-tree
  // signatures nor the timer, whose stages are the queue kernels'.
  const bool whole = ra.path_begin == 0 && ra.path_count == ra.frame_paths;
  if (!multi && !count && !ids && !timer && whole && path_wins(size, ra.path_count)) {
    const PathLaunch l = path_launch(flat, ra.path_count, kWaves, p.grid_trace, p.grid_path[flat ? 0 : 1]);
    const int blog = l.log2n, dynamic = l.dynamic ? 1 : 0;
    const unsigned grid = unsigned(l.grid);
    // The workspace holds anything before the launch, but not its number.  A captured launch has one number for all its
    // replays, so those clear it.
    a.launch = launch_number();
    if (dynamic || (!flat && ra.ray_counts && capturing(s))) {
      k_reset<<<1, kResetBlock, 0, s>>>(a.ctr);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // The blocks add their ray counts to the caller's by themselves (256x256: spheres 18.7 us with a launch for it, 16.5
    // so; 100 triangles 51.9, 48.2; 641x479, 13k triangles 237, 234), but where all of them end at once and would wait
    // for each other's atomics: without a tree, one batch after another (spheres at 1080p 107 and 131 us).
    int64_t* direct = flat && dynamic ? nullptr : ra.ray_counts;
    if (flat)
      k_path<false><<<grid, kBlock, 0, s>>>(a, blog, dynamic, direct);
    else
      k_path<true><<<grid, kBlock, 0, s>>>(a, blog, dynamic, direct);
    e = hipGetLastError();
    if (e != hipSuccess || !ra.ray_counts || direct) return e;
    k_path_finish<<<1, kBlock, 0, s>>>(reinterpret_cast<const uint4*>(a.ctr), int(grid),
                                       2 * int64_t(ra.one.cam.W) * ra.one.cam.H, ra.ray_counts);
    return hipGetLastError();
  }
  if (timer) timer_begin(timer, RT_STAGE_SETUP, s);
  k_reset<<<1, kResetBlock, 0, s>>>(a.ctr);
  e = hipGetLastError();
  if (timer) timer_end(timer, RT_STAGE_SETUP, s);
  if (e != hipSuccess) return e;
  // The traversal takes the resolve of two depths before along, but for the ray-tree signatures, which k_resolve writes,
  // and the timer, whose stages are apart.
  a.resolve = !flat && !count && !ids && !timer ? 1 : 0;
  const int D = a.dmax;
  for (int d = 0; d <= D + 1; ++d) {
    if (flat) {
      if (flat_splits(size))
        e = launch(k_trace_flat<kFlatSegs>, gtrace(d, 64, kFlatWaves / kFlatSegs), a, d, s, timer, RT_STAGE_TRACE,
                   kFlatBlock<kFlatSegs>);
      else
        e = launch(k_trace_flat<1>, gtrace(d, kFlatBlock<1>, kFlatWaves * 64 / kFlatBlock<1>), a, d, s, timer,
                   RT_STAGE_TRACE, kFlatBlock<1>);
    } else {
      const unsigned grid = gtrace(d, int64_t(kWaves) << min_rays_log2(multi), p.grid_trace);
      if (multi)
        e = count ? launch(k_trace<true, true>, grid, a, d, s, timer, RT_STAGE_TRACE)
                  : launch(k_trace<false, true>, grid, a, d, s, timer, RT_STAGE_TRACE);
      else
        e = count ? launch(k_trace<true, false>, grid, a, d, s, timer, RT_STAGE_TRACE)
                  : launch(k_trace<false, false>, grid, a, d, s, timer, RT_STAGE_TRACE);
    }
    if (e != hipSuccess) return e;
    if (d <= D) {
      if (multi)
        e = ids ? launch(k_shade<true, true>, gshade, a, d, s, timer, RT_STAGE_SHADE, kShadeBlock)
                : launch(k_shade<false, true>, gshade, a, d, s, timer, RT_STAGE_SHADE, kShadeBlock);
      else
        e = ids ? launch(k_shade<true, false>, gshade, a, d, s, timer, RT_STAGE_SHADE, kShadeBlock)
                : launch(k_shade<false, false>, gshade, a, d, s, timer, RT_STAGE_SHADE, kShadeBlock);
      if (e != hipSuccess) return e;
    }
    if (d >= 1 && (!a.resolve || d == D + 1)) {
      if (multi)
        e = ids ? launch(k_resolve<true, true>, gstream, a, d - 1, s, timer, RT_STAGE_RESOLVE)
                : launch(k_resolve<false, true>, gstream, a, d - 1, s, timer, RT_STAGE_RESOLVE);
      else
        e = ids ? launch(k_resolve<true, false>, gstream, a, d - 1, s, timer, RT_STAGE_RESOLVE)
                : launch(k_resolve<false, false>, gstream, a, d - 1, s, timer, RT_STAGE_RESOLVE);
      if (e != hipSuccess) return e;
    }
  }
  if (ra.ray_counts) {
    k_finish<<<1, 64, 0, s>>>(a.ctr, D, a.lstride, ra.ray_counts);
    e = hipGetLastError();
  }
  return e;
}

// The item table is written by a kernel whose arguments carry up to kItemsPerUpload items, so a
// batch needs no host staging buffer and can be captured into a graph.
namespace {
constexpr int kItemsPerUpload = 8;
struct ItemUpload {
  DevItem items[kItemsPerUpload];
  int32_t n;
};
static_assert(sizeof(ItemUpload) <= 4000, "kernel argument block too large");
__global__ void k_upload_items(ItemUpload u, DevItem* dst) {
  const int i = threadIdx.x;
  if (i < u.n) dst[i] = u.items[i];
}
}  // namespace

hipError_t upload_items(const DevItem* items, int n, DevItem* dst, hipStream_t s) {
  for (int i = 0; i < n; i += kItemsPerUpload) {
    ItemUpload u{};
    u.n = std::min(kItemsPerUpload, n - i);
    for (int k = 0; k < u.n; ++k) u.items[k] = items[i + k];
    k_upload_items<<<1, kItemsPerUpload, 0, s>>>(u, dst + i);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace srt
