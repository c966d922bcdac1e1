// The weight gradient of first layers (stem.hip), for the launches that hold it.
#pragma once
#include "nf_internal.h"

namespace nf {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int STEM_THREADS = 256;  // threads per workgroup
constexpr int STEM_KS = 32;        // staged reduction length (R*S*C <= STEM_KS, zero padded)
constexpr int STEM_LDK = STEM_KS + 4;
constexpr int STEM_BP = 64, STEM_BR = 32;
constexpr int STEM_WGRAD_RED = 4 * 2 * 32 * 33;  // the waves' tiles, in the place of the staged rows
constexpr int STEM_WGRAD_LDS = STEM_WGRAD_RED + 16 * STEM_BP;
static_assert(STEM_BR * (STEM_BP + 4 + STEM_LDK) <= STEM_WGRAD_RED, "staged rows");

// element kg = (r, s, c) of the im2col row of output pixel (img, ho, wo); zero outside the image.
// Branch-free (the address is clamped into the tensor, the value selected afterwards) so that a
// thread's gathers are all in flight together instead of one behind each branch.
__device__ inline float col_tap(const float *__restrict__ x, int H, int W, int C, int stride, int pad, int img, int ho,
                                int wo, int r, int s, int c, bool live) {
  const int hi = ho * stride - pad + r, wi = wo * stride - pad + s;
  const bool ok = live & ((unsigned)hi < (unsigned)H) & ((unsigned)wi < (unsigned)W);
  const int hc = min(max(hi, 0), H - 1), wc = min(max(wi, 0), W - 1);
  const float v = x[((long long)(img * H + hc) * W + wc) * C + c];
  return ok ? v : 0.f;
}
__device__ inline float col_elem(const float *__restrict__ x, int H, int W, int C, int S, int RSC, int stride, int pad,
                                 int img, int ho, int wo, int kg, bool live) {
  const int k = min(kg, RSC - 1);
  const int tap = k / C, c = k - tap * C;
  const int r = tap / S, s = tap - r * S;
  return col_tap(x, H, W, C, stride, pad, img, ho, wo, r, s, c, live & (kg < RSC));
}

// part[z][pr][q] = sum over the rows m of split z of d[m][pr] * col[m][q]  (q < RSC <= 32), and
// part_b[z][pr] = sum of d[m][pr]: a 64 x 32 output tile per workgroup (by picks the 64
// output channels, bz the split).  Steps of 32 rows: d rows and im2col rows staged in LDS,
// each wave takes 8 of them (4 MFMA k-pairs x 2 tiles); the four waves' tiles are added in a
// fixed order at the end.
// lds: STEM_WGRAD_LDS floats.
template <bool VEC>
__device__ __forceinline__ void stem_wgrad_tile(const WgradProblem &p, int by, int bz, float *lds) {
  constexpr int BP = STEM_BP, BR = STEM_BR;  // output-channel tile, rows per step
  constexpr int LDP = BP + 4;
  float(*const Ds)[LDP] = reinterpret_cast<float(*)[LDP]>(lds);
  float(*const Xs)[STEM_LDK] = reinterpret_cast<float(*)[STEM_LDK]>(lds + BR * LDP);
  float(*const red)[2][32][33] = reinterpret_cast<float(*)[2][32][33]>(lds);
  float(*const redb)[BP] = reinterpret_cast<float(*)[BP]>(lds + STEM_WGRAD_RED);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int j = lane & 31, g = lane >> 5;
  const int p0 = by * BP, z = bz;
  const int m_begin = z * p.m_per_split, m_end = min(p.M, m_begin + p.m_per_split);

  floatx16 acc[2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[a][e] = 0.f;
  // d staging: thread -> (row = t / 16 (+16), 4 consecutive output channels); its column sums feed the bias gradient
  const int drow = t >> 4, dc = (t & 15) * 4;
  float4 bsum = make_float4(0.f, 0.f, 0.f, 0.f);
  // im2col staging: thread -> (row = t % 32, 4 consecutive kg)
  const int xrow = t & 31, xk = (t >> 5) * 4;

  for (int mb = m_begin; mb < m_end; mb += BR) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = drow + 16 * i, m = mb + r;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m < m_end) {
        const float *src = p.d + (long long)m * p.P + p0 + dc;
        if constexpr (VEC) {
          if (p0 + dc < p.P) v = *reinterpret_cast<const float4 *>(src);  // P % 4 == 0: whole group inside
        } else {
          if (p0 + dc + 0 < p.P) v.x = src[0];
          if (p0 + dc + 1 < p.P) v.y = src[1];
          if (p0 + dc + 2 < p.P) v.z = src[2];
          if (p0 + dc + 3 < p.P) v.w = src[3];
        }
      }
      *reinterpret_cast<float4 *>(&Ds[r][dc]) = v;
      bsum.x += v.x, bsum.y += v.y, bsum.z += v.z, bsum.w += v.w;
    }
    {
      const int m = mb + xrow;
      const bool live = m < m_end;
      const int mc = min(m, p.M - 1);
      const int img = (int)p.div_howo.div((uint32_t)mc);
      const int rem = mc - img * p.Ho * p.Wo;
      const int ho = (int)p.div_wo.div((uint32_t)rem);
      const int wo = rem - ho * p.Wo;
      float4 v;
      v.x = col_elem(p.x, p.H, p.W, p.C, p.S, p.RSC, p.stride, p.pad, img, ho, wo, xk + 0, live);
      v.y = col_elem(p.x, p.H, p.W, p.C, p.S, p.RSC, p.stride, p.pad, img, ho, wo, xk + 1, live);
      v.z = col_elem(p.x, p.H, p.W, p.C, p.S, p.RSC, p.stride, p.pad, img, ho, wo, xk + 2, live);
      v.w = col_elem(p.x, p.H, p.W, p.C, p.S, p.RSC, p.stride, p.pad, img, ho, wo, xk + 3, live);
      *reinterpret_cast<float4 *>(&Xs[xrow][xk]) = v;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = wave * 8 + 2 * i + g;
      const float xv = Xs[r][j];
#pragma unroll
      for (int a = 0; a < 2; ++a) acc[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(Ds[r][a * 32 + j], xv, acc[a], 0, 0, 0);
    }
    __syncthreads();
  }

  // ---- the four waves' tiles, added in a fixed order: (w0 + w1) + (w2 + w3) ----
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][a][8 * (e >> 2) + 4 * g + (e & 3)][j] = acc[a][e];
  *reinterpret_cast<float4 *>(&redb[drow][dc]) = bsum;
  __syncthreads();
  float *part = p.part + (long long)z * p.P * p.Qld;
  for (int i = t; i < BP * 32; i += STEM_THREADS) {
    const int pl = i >> 5, q = i & 31, a = pl >> 5, r = pl & 31;
    const int pr = p0 + pl;
    if (pr < p.P && q < p.Q) part[(long long)pr * p.Qld + q] = (red[0][a][r][q] + red[1][a][r][q]) + (red[2][a][r][q] + red[3][a][r][q]);
  }
  if (p.part_b && t < BP && p0 + t < p.P) {
    float s = 0.f;
    for (int r = 0; r < 16; ++r) s += redb[r][t];
    p.part_b[(long long)z * p.P + p0 + t] = s;
  }
}

}  // namespace
}  // namespace nf
