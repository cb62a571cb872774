// Stereo-pair building on the device: the paper's post-processing of the two
// channels for a display (Section 3, Fig. 2: e.g. an anaglyph).  Both modes
// write 8-bit RGBA:
//   red-cyan anaglyph: red from the left eye, green and blue from the right eye;
//   side by side: the left eye's image followed by the right eye's, 2W x H.
// Display encoding of a linear value x: code = floor(255 * sqrt(clamp(x * exposure, 0, 1)) + 0.5),
// every step a correctly rounded FP32 operation (no contraction), alpha 255.

#include <hip/hip_runtime.h>

#include "rt_internal.h"

namespace srt {
namespace {

__device__ inline uint32_t encode(float x, float exposure) {
  float v = __fmul_rn(x, exposure);
  v = fminf(fmaxf(v, 0.0f), 1.0f);
  const float g = __fsqrt_rn(v);
  return uint32_t(floorf(__fadd_rn(__fmul_rn(255.0f, g), 0.5f)));
}

__global__ __launch_bounds__(256) void k_compose(const float* __restrict__ left, const float* __restrict__ right,
                                                 int W, int H, int mode, float exposure, uint32_t* __restrict__ out) {
  const int64_t n = int64_t(W) * H;
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < (mode == RT_COMPOSE_SIDE_BY_SIDE ? 2 * n : n);
       i += int64_t(gridDim.x) * 256) {
    uint32_t r, g, b;
    int64_t o;
    if (mode == RT_COMPOSE_ANAGLYPH_RED_CYAN) {
      r = encode(left[3 * i + 0], exposure);
      g = encode(right[3 * i + 1], exposure);
      b = encode(right[3 * i + 2], exposure);
      o = i;
    } else {
      const int64_t row = i / (2 * W), col = i % (2 * W);
      const float* src = col < W ? left : right;
      const int64_t p = row * W + (col < W ? col : col - W);
      r = encode(src[3 * p + 0], exposure);
      g = encode(src[3 * p + 1], exposure);
      b = encode(src[3 * p + 2], exposure);
      o = i;
    }
    out[o] = r | (g << 8) | (b << 16) | (255u << 24);
  }
}

// Four pixels a thread: three 16-byte loads an eye and one 16-byte store, with one 64-bit division for four pixels
// of both eyes where there was one a pixel (side by side; the anaglyph needs none).  Needs 16-byte aligned pointers and, side by side, rows of whole groups (the
// output's and the eyes' groups then start together); other calls take k_compose.  Bound by memory: every
// line of both eyes is read, also for the channels an anaglyph leaves out.  3840x2160: anaglyph 41.1 -> 38.9 us
// (232 MB, 6.0 TB/s), side by side 57.5 -> 41.7; 2,048 or 4,096 workgroups 42.1 and 40.5, loads past the
// caches 51.1 (the pair was just rendered and is partly in the last-level cache).
__device__ inline uint32_t rgba(float r, float g, float b, float exposure) {
  return encode(r, exposure) | (encode(g, exposure) << 8) | (encode(b, exposure) << 16) | (255u << 24);
}

template <bool SIDE_BY_SIDE>
__global__ __launch_bounds__(256) void k_compose4(const float4* __restrict__ left, const float4* __restrict__ right,
                                                  int64_t groups, int row_groups, float exposure,
                                                  uint4* __restrict__ out) {
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < groups; i += int64_t(gridDim.x) * 256) {
    if (SIDE_BY_SIDE) {
      const int64_t row = i / row_groups, col = i - row * row_groups;
      for (int eye = 0; eye < 2; ++eye) {
        const float4* src = eye ? right : left;
        const float4 a = src[3 * i], b = src[3 * i + 1], c = src[3 * i + 2];
        out[2 * row * row_groups + eye * row_groups + col] =
            make_uint4(rgba(a.x, a.y, a.z, exposure), rgba(a.w, b.x, b.y, exposure), rgba(b.z, b.w, c.x, exposure),
                       rgba(c.y, c.z, c.w, exposure));
      }
    } else {
      const float4 a = left[3 * i], b = left[3 * i + 1], c = left[3 * i + 2];
      const float4 d = right[3 * i], e = right[3 * i + 1], f = right[3 * i + 2];
      out[i] = make_uint4(rgba(a.x, d.y, d.z, exposure), rgba(a.w, e.x, e.y, exposure),
                          rgba(b.z, e.w, f.x, exposure), rgba(c.y, f.z, f.w, exposure));
    }
  }
}

}  // namespace

hipError_t compose_stereo(const float* left, const float* right, int W, int H, int mode, float exposure,
                          uint8_t* out, hipStream_t s) {
  const bool sbs = mode == RT_COMPOSE_SIDE_BY_SIDE;
  const uintptr_t all = reinterpret_cast<uintptr_t>(left) | reinterpret_cast<uintptr_t>(right) | reinterpret_cast<uintptr_t>(out);
  if ((all & 15u) == 0 && (sbs ? W % 4 == 0 : (int64_t(W) * H) % 4 == 0)) {
    const int64_t groups = int64_t(W) * H / 4;
    const unsigned grid = unsigned(std::min<int64_t>((groups + 255) / 256, 8192));
    const float4 *l = reinterpret_cast<const float4*>(left), *r = reinterpret_cast<const float4*>(right);
    if (sbs)
      k_compose4<true><<<grid, 256, 0, s>>>(l, r, groups, W / 4, exposure, reinterpret_cast<uint4*>(out));
    else
      k_compose4<false><<<grid, 256, 0, s>>>(l, r, groups, 0, exposure, reinterpret_cast<uint4*>(out));
    return hipGetLastError();
  }
  const int64_t n = int64_t(W) * H * (mode == RT_COMPOSE_SIDE_BY_SIDE ? 2 : 1);
  const unsigned grid = unsigned(std::min<int64_t>((n + 255) / 256, 4096));
  k_compose<<<grid, 256, 0, s>>>(left, right, W, H, mode, exposure, reinterpret_cast<uint32_t*>(out));
  return hipGetLastError();
}

}  // namespace srt
