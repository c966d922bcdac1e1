// What the kernels of F(2x2, 3x3) share (wino_fwd.hip, wino_fwd_split.hip).
#pragma once
#include "wino_filter.h"

namespace nf {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct WinoAux {
  int TW, TPI, T;        // tiles per image row, per image, in all
  int nchunks, per;      // steps of channels; steps per reduction split
  int nblk;              // filter blocks
  FastDiv div_tpi, div_tw;
  uint32_t x_bytes, u_bytes;
  const float *U;
};

__device__ inline float4 bload(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  const floatx4 v = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline float el(const float4 &v, int k) { return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w; }
__device__ inline float4 add4(const float4 &a, const float4 &b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ inline float4 sub4(const float4 &a, const float4 &b) {
  return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
}
// a + s*b with s = +-1 (exact product)
__device__ inline float4 fma4(float s, const float4 &b, const float4 &a) {
  return make_float4(__builtin_fmaf(s, b.x, a.x), __builtin_fmaf(s, b.y, a.y), __builtin_fmaf(s, b.z, a.z),
                     __builtin_fmaf(s, b.w, a.w));
}
// bit e: component e is not finite
__device__ inline unsigned bad4(const float4 &v) {
  return (__builtin_isfinite(v.x) ? 0u : 1u) | (__builtin_isfinite(v.y) ? 0u : 2u) | (__builtin_isfinite(v.z) ? 0u : 4u) |
         (__builtin_isfinite(v.w) ? 0u : 8u);
}

// Four outputs (filters n .. n+3 of pixel (img, ho, wo)) by the direct sum over channels [c_lo, c_hi).
// Taps outside the image are left out, as in the direct kernel's position tiles: an infinite weight over the padding is not one of
// the sum's.  (Its other tiles multiply it by the zero they load.)
__device__ inline float4 direct4(const float *x, const float *w, int H, int W, int C, int img, int ho, int wo, int n,
                                 int c_lo, int c_hi, unsigned want) {
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  const long long ws = 9ll * C;
#pragma unroll 1
  for (int tap = 0; tap < 9; ++tap) {
    const int hi = ho + tap / 3 - 1, wi = wo + tap % 3 - 1;
    if (((unsigned)hi >= (unsigned)H) | ((unsigned)wi >= (unsigned)W)) continue;
    const float *xr = x + ((long long)(img * H + hi) * W + wi) * C;
    const float *wr = w + ((long long)n * 9 + tap) * C;
#pragma unroll 1
    for (int c = c_lo; c < c_hi; c += 4) {
      const float4 v = *reinterpret_cast<const float4 *>(xr + c);
      auto dot = [&](int k, float a) {
        const float4 g = *reinterpret_cast<const float4 *>(wr + k * ws + c);
        return __builtin_fmaf(v.w, g.w, __builtin_fmaf(v.z, g.z, __builtin_fmaf(v.y, g.y, __builtin_fmaf(v.x, g.x, a))));
      };
      s.x = dot(0, s.x), s.y = dot(1, s.y), s.z = dot(2, s.z), s.w = dot(3, s.w);
      // a NaN stays one: filters that have become NaN, as in a network that has diverged, cost a step of this
      const unsigned nan = (__builtin_isnan(s.x) ? 1u : 0u) | (__builtin_isnan(s.y) ? 2u : 0u) |
                           (__builtin_isnan(s.z) ? 4u : 0u) | (__builtin_isnan(s.w) ? 8u : 0u);
      if ((nan & want) == want) return s;
    }
  }
  return s;
}

// onto more than 32 filters (wino_fwd_split.hip); q: all but the grid's fields
// (small: 32 tiles per workgroup, where twice as many of them, each with a compute unit to itself, still fit the chip: a step takes
// 2.0 us then, 3.0 with 64 tiles)
inline bool wino_fwd_split_small(long long workgroups64) { return workgroups64 <= 128; }
hipError_t launch_wino_fwd_split(const FwdProblem &p, WinoAux q, int splits, hipStream_t st);

}  // namespace nf
