// First-layer ("stem") convolutions: few input channels, so the whole reduction R*S*C fits one
// 32-wide staging step (3x3x3 = 27 for RGB inputs).  NeuroFlux, arXiv 2402.14139: Eq. 1 for the
// first local layer (forward) and the gradient line of Algorithm 2 for its filter (weight gradient).
//
// These layers are bound by HBM, not by the MFMA pipe: the forward writes 64 output channels for 27
// multiply-adds each (arithmetic intensity ~13 flop/byte), the weight gradient reads them back.  The
// general-shape kernels spend their time in a pipelined reduction loop that here has one step;
// the kernels below stage the im2col rows once (scalar gathers: a channel count of 3 has no
// 16-byte groups), run the few MFMAs and stream the output / the dZ rows with 16-byte accesses.
#include "nf_internal.h"
#include "stem_wgrad.h"

namespace nf {
namespace {

constexpr int NT = STEM_THREADS, KS = STEM_KS, LDK = STEM_LDK;

// out[m][n] = act(bias[n] + sum_kg col[m][kg] * w[n][kg] (+ addsrc[m][n])), zeroed where mask <= 0.
// Tile: 128 output pixels x 64 output channels, 4 waves as 2 x 2, each 64 x 32 on 32x32x2 MFMAs.
// The reduction index of a gather is the same in every lane of a wave: its decode into (r, s, c) is
// scalar work, and all 24 loads of a thread are in flight together (with per-lane divisions, filter loads
// behind branches and an epilogue that tested for a shortcut at every element: 11.8 us where this takes
// 10.0; 8192 pixels, 16 filters: launch latency and one dependent chain of load, MFMA, store).
struct StemAux {
  FastDiv div_c, div_s;
};
__global__ __launch_bounds__(NT) void stem_fwd_kernel(FwdProblem p, StemAux q) {
  constexpr int BM = 128, BN = 64;
  __shared__ __attribute__((aligned(16))) float As[BM][LDK];
  __shared__ __attribute__((aligned(16))) float Bs[BN][LDK];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int j = lane & 31, g = lane >> 5;
  const int tiles_n = (p.N + BN - 1) / BN;
  const int tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x - tile_m * tiles_n;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  {  // im2col rows: thread -> (row, half of the reduction axis)
    const int row = t & (BM - 1), kh = __builtin_amdgcn_readfirstlane(t >> 7);
    const int m = m0 + row;
    int img = 0, ho = 0, wo = 0;
    const bool live = m < p.M;
    if (live) {
      img = (int)p.div_howo.div((uint32_t)m);
      const int rem = m - img * p.Ho * p.Wo;
      ho = (int)p.div_wo.div((uint32_t)rem);
      wo = rem - ho * p.Wo;
    }
    float v[KS / 2];
#pragma unroll
    for (int i = 0; i < KS / 2; ++i) {
      const int kg = kh * (KS / 2) + i, k = min(kg, p.RSC - 1);
      const int tap = (int)q.div_c.div((uint32_t)k), c = k - tap * p.C;
      const int r = (int)q.div_s.div((uint32_t)tap), s = tap - r * p.S;
      v[i] = col_tap(p.x, p.H, p.W, p.C, p.stride, p.pad, img, ho, wo, r, s, c, live & (kg < p.RSC));
    }
#pragma unroll
    for (int i = 0; i < KS / 2; i += 4)
      *reinterpret_cast<float4 *>(&As[row][kh * (KS / 2) + i]) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
  }
  {  // filter rows: thread -> (n, quarter of the reduction axis)
    const int nl = t & (BN - 1), kq = t >> 6;
    const int n = n0 + nl;
    const float *wr = p.w + (long long)min(n, p.N - 1) * p.RSC;
    float v[KS / 4];
#pragma unroll
    for (int i = 0; i < KS / 4; ++i) v[i] = wr[min(kq * (KS / 4) + i, p.RSC - 1)];
#pragma unroll
    for (int i = 0; i < KS / 4; ++i)
      Bs[nl][kq * (KS / 4) + i] = ((n < p.N) & (kq * (KS / 4) + i < p.RSC)) ? v[i] : 0.f;
  }
  __syncthreads();

  floatx16 acc[2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[a][e] = 0.f;
#pragma unroll
  for (int ks = 0; ks < KS / 8; ++ks) {
    const float4 b4 = *reinterpret_cast<const float4 *>(&Bs[wn * 32 + j][ks * 8 + g * 4]);
    const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const float4 a4 = *reinterpret_cast<const float4 *>(&As[wm * 64 + a * 32 + j][ks * 8 + g * 4]);
      const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc[a] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[kk], bv[kk], acc[a], 0, 0, 0);
    }
  }

  const int n = n0 + wn * 32 + j;
  if (n >= p.N) return;
  const float bias = p.bias ? p.bias[n] : 0.f;
  if (!p.addsrc && !p.mask) {  // a first layer without a shortcut: nothing but stores
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + wm * 64 + a * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
        float v = acc[a][e] + bias;
        v = (!p.relu | (v > 0.f)) ? v : 0.f;
        if (m < p.M) p.out[(long long)m * p.N + n] = v;
      }
    return;
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = m0 + wm * 64 + a * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
      if (m >= p.M) continue;
      const long long o = (long long)m * p.N + n;
      float v = acc[a][e] + bias;
      if (p.addsrc) v += p.addsrc[o];
      if (p.relu) v = v > 0.f ? v : 0.f;
      if (p.mask) v = p.mask[o] > 0.f ? v : 0.f;
      p.out[o] = v;
    }
}

template <bool VEC>
__global__ __launch_bounds__(NT) void stem_wgrad_kernel(WgradProblem p) {
  __shared__ __attribute__((aligned(16))) float lds[STEM_WGRAD_LDS];
  stem_wgrad_tile<VEC>(p, blockIdx.y, blockIdx.z, lds);
}

}  // namespace

bool stem_fwd_applicable(const FwdProblem &p) {
  // one staging step, no projection columns, no split; layers the 16-byte fast path can serve keep it
  if (p.RSC > KS || p.Cs != 0 || p.ksplits > 1 || p.Kg != p.RSC) return false;
  if (p.C % 4 == 0) return false;
  const long long B = p.M / ((long long)p.Ho * p.Wo);
  return B * p.H * p.W * p.C < (1ll << 31) && (long long)p.M * p.N < (1ll << 40);
}

hipError_t launch_stem_fwd(const FwdProblem &p, hipStream_t st, const char **kernel) {
  const int tiles = ((p.M + 127) / 128) * ((p.N + 63) / 64);
  *kernel = "stem_fwd";
  StemAux q;
  q.div_c = FastDiv(p.C), q.div_s = FastDiv(p.S);
  hipLaunchKernelGGL(stem_fwd_kernel, dim3((unsigned)tiles), dim3(NT), 0, st, p, q);
  return hipGetLastError();
}

bool stem_wgrad_applicable(const WgradProblem &p) {
  if (p.RSC > KS || p.Cs != 0 || p.Q != p.RSC) return false;
  if (p.C % 4 == 0) return false;
  const long long B = p.M / ((long long)p.Ho * p.Wo);
  return B * p.H * p.W * p.C < (1ll << 31);
}

hipError_t launch_stem_wgrad(const WgradProblem &p, hipStream_t st, const char **kernel) {
  const dim3 grid(1, (unsigned)((p.P + 63) / 64), (unsigned)p.splits);
  *kernel = "stem_wgrad";
  if (p.P % 4 == 0)
    hipLaunchKernelGGL(stem_wgrad_kernel<true>, grid, dim3(NT), 0, st, p);
  else
    hipLaunchKernelGGL(stem_wgrad_kernel<false>, grid, dim3(NT), 0, st, p);
  return hipGetLastError();
}

}  // namespace nf
