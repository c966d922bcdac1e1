// 3x3 / stride 1 / pad 1 convolution (Eq. 1, NeuroFlux, arXiv 2402.14139) through the minimal
// filtering algorithm F(2x2, 3x3) (S. Winograd, "Arithmetic Complexity of Computations", 1980;
// A. Lavin, S. Gray, arXiv 1509.09308), entirely in fp32: a 2x2 output tile is
//     Y = A^T [ (G g G^T) . (B^T d B) ] A
// with d the 4x4 input patch and g the 3x3 filter: 16 multiplications per channel where the direct
// sum takes 36.  The 16 positions of the transformed domain are 16 independent contractions over
// the channels, run on the fp32 matrix cores.
//
// What bounds it: the fp32 MFMA rate (16/36 of the direct kernel's MFMAs).  Layout of the work:
//   - a workgroup owns 32 output tiles (128 pixels) x 64 filters x all 16 positions, so the patches
//     are transformed on their way into the MFMA and the results on their way out: nothing of the
//     transformed domain but the filters (wino_filter_kernel) ever reaches memory;
//   - 4 waves = the 4 rows of the transformed domain.  A wave's row needs two rows of the patch (B^T
//     has two non-zeros per row), which it reads from LDS and combines in registers (32 additions
//     per 32 MFMAs); its filters come straight from memory in fragment order (no other wave of the
//     workgroup uses them, so LDS would only add a copy);
//   - 8 channels per step, one barrier per step; patches are loaded three steps ahead, written to
//     LDS two steps ahead, read and row-combined one step ahead; a filter fragment is re-loaded
//     for the next step right after its last MFMA;
//   - 128 accumulators per lane, two workgroups per CU: one's transforms, LDS traffic, loads and
//     stores fill in under the other's MFMAs (one workgroup of 64 tiles per CU: 101 us where this
//     takes 84, 64 channels on 56x56 maps, batch 64; equal where both fill the chip once).
// The reduction has C terms per position instead of 9 C: the rounding error against 64 bits is
// smaller than that of the direct sum (emitted activation, relative: 64 channels 1.7e-7 against 2.2e-7, four
// layers of 256 channels in a row 5.9e-7 against 7.1e-7).  That is a single result's: an average over pixels and samples keeps the
// rounding of the transformed filter (wino_fwd_pick_splits).
//
// Measured (us, the direct kernel / this with its filter launch of 5-8 us): 64 -> 64 channels, 65 536 pixels
// 50 / 32; 128 -> 128, 32 768 pixels 78 / 46; 256 -> 256, 8x8 pixels, batch 256 132 / 78; 512 -> 512, 4x4, batch 512 228 / 142 (the direct
// kernel without the padding there); a step of 8 channels takes 1.93 us on a CU with two workgroups, 0.87 of it MFMAs.
//
// The data gradient onto a layer of up to 32 filters runs through a variant of 32 per workgroup, half of whose columns
// would be padding otherwise: 64 accumulators, three workgroups per CU, the same patches and transforms for half of the
// MFMAs, so a step of 16 MFMAs takes 1.3 us with two workgroups on a CU where they alone take 0.9.  Measured (us, the direct kernel
// of 64x32 tiles / this, without the filter's launch): 64 channels, 65 536 pixels 30.2 / 19.5, 128 channels, 16 384 pixels 17.1 /
// 12.3.
//
// A value that is not finite anywhere in a tile makes neighbours of the transformed domain NaN that
// the direct sum would leave finite (or infinite): a thread that finds one among its results
// forms those results again by the direct sum.
#include <algorithm>

#include "wino_filter.h"

namespace nf {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int NTHREADS = 256;
constexpr int TB = 32;                   // output tiles per workgroup
constexpr int CH = WINO_CH;              // channels per step
constexpr int OOB = (int)0x80000000;     // offset no buffer of < 2 GiB contains
constexpr int RSRC_FLAGS = 0x00020000;   // raw buffer, 32-bit data format

struct WinoAux {
  int TW, TPI, T;        // tiles per image row, per image, in all
  int nchunks, per;      // steps of 8 channels; steps per reduction split
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

// One or two transformed filters, zero past the last filter and channel.  HBM-bound: 36 bytes read, 64 written per
// (filter, channel); 5-8 us, most of it the launch: the head's filter rides on its layer's (64 -> 64 channels, batch
// 64, 32-wide head: a launch of 4.5 us less).
struct FilterJobs {
  WinoFilter f[2];
  int nchunks[2], bx[2], blocks0;  // steps of 8 channels; blocks along the channels; blocks of job 0
};
__global__ __launch_bounds__(256) void wino_filter_kernel(FilterJobs js) {
  const int k = (int)blockIdx.x >= js.blocks0, b = blockIdx.x - (k ? js.blocks0 : 0);
  const WinoFilter f = js.f[k];
  const int nchunks = js.nchunks[k], bx = js.bx[k];
  const int t = threadIdx.x;
  const int c4 = b % bx * 8 + (t & 7), n = b / bx * 32 + (t >> 3);  // 8 lanes read 128 contiguous bytes
  if (c4 >= 2 * nchunks) return;
  float4 g[3][3];
  const bool ok = n < f.N && c4 * 4 < f.C;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s)
      g[r][s] = ok ? *reinterpret_cast<const float4 *>(f.w + ((long long)n * 9 + r * 3 + s) * f.C + c4 * 4)
                   : make_float4(0.f, 0.f, 0.f, 0.f);
  wino_filter_store(g, f.U, n, c4, nchunks, wino_nb(f.N));
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

// NF: MFMA columns of 32 filters per workgroup (2, or 1 for few filters).  POOL: the 2x2 max pooling of Eq. 1 follows in the
// epilogue: an output tile is a window, so the convolution's result never reaches memory (a quarter of its stores, and no pooling
// launch: 64 -> 128 channels, 65 536 pixels 53 + 8.2 us, so 50.8).
template <int NF, bool POOL>
__global__ __launch_bounds__(NTHREADS, NF == 2 ? 2 : 3) void wino_fwd_kernel(FwdProblem p, WinoAux q) {
  constexpr int NB = 32 * NF, UP = NB * CH, UB = 16 * UP;  // filters; words of U per position and per step
  constexpr int AW = 2 * 16 * TB * CH, CW = 4 * TB * 2 * NB;
  // main loop: As[2][16 patch pixels][32 tiles][8 channels]; epilogue: Cs[4 rows][32 tiles][2 columns][NB filters]
  __shared__ __attribute__((aligned(16))) float S[AW > CW ? AW : CW];

  const int t = threadIdx.x;
  const int lane = t & 63, row = t >> 6;  // a wave owns one row of the transformed domain
  const int j = lane & 31, h = lane >> 5;
  // XCD re-map (workgroups are dealt round-robin over 8 XCDs): each XCD gets a contiguous run with the
  // filter blocks fastest, so that the patches of a tile block are read into one L2 only
  const int nwg = gridDim.x, lin = blockIdx.x;
  const int wper = nwg >> 3, wrem = nwg & 7, xcd = lin & 7, slot = lin >> 3;
  const int id = xcd < wrem ? xcd * (wper + 1) + slot : wrem * (wper + 1) + (xcd - wrem) * wper + slot;
  const int nb = id % q.nblk, t0 = (id / q.nblk) * TB;
  const int s_lo = blockIdx.y * q.per, s_hi = min(q.nchunks, s_lo + q.per);

  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, q.x_bytes, RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t rsu = __builtin_amdgcn_make_buffer_rsrc((void *)q.U, 0, q.u_bytes, RSRC_FLAGS);

  // ---- staging: thread = (patch row, tile, channel half); its four loads are the row's pixels ----
  const int st_half = t & 1, st_tile = (t >> 1) & (TB - 1), st_row = t / (2 * TB);
  int xoff[4];
  {
    const int tile = t0 + st_tile;
    const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
    const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
    const int hi = 2 * ty - 1 + st_row, wi = 2 * tx - 1;
    const bool rok = (tile < q.T) & ((unsigned)hi < (unsigned)p.H);
    const int base = ((img * p.H + hi) * p.W + wi) * p.C * 4 + st_half * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      xoff[i] = (base + i * p.C * 4) | ((rok & ((unsigned)(wi + i) < (unsigned)p.W)) ? 0 : OOB);
  }
  // A load's offset is a lane's constant and a scalar that advances: no vector arithmetic beside the MFMAs (54 -> 35
  // vector instructions a step; 512 -> 512 channels, 8192 pixels: workgroups end after 162 / 154 us).  Steps past the
  // end load the last one again, which nothing reads.  The upper half of a last step of four channels is out of range.
  const int half_step = (p.C % CH) ? q.nchunks - 1 : -1;
  auto last = [&](int s) { return s < s_hi ? s : s_hi - 1; };
  auto halve = [&](int s) {  // in front of gload(s)
    if (last(s) == half_step) {
#pragma unroll
      for (int i = 0; i < 4; ++i) xoff[i] |= st_half ? OOB : 0;
    }
  };
  auto gload = [&](int s, float4 *sx) {
#pragma unroll
    for (int i = 0; i < 4; ++i) sx[i] = bload(rsx, xoff[i], last(s) * (CH * 4));
  };
  float *const st_base = S + (st_row * 4 * TB + st_tile) * CH + st_half * 4;
  auto lstore = [&](int buf, const float4 *sx) {
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<float4 *>(st_base + buf * (16 * TB * CH) + i * (TB * CH)) = sx[i];
  };

  // ---- this wave's row of B^T: d[ra] + sg * d[rb] ----
  const int ra = row == 0 ? 0 : row == 2 ? 2 : 1, rb = row == 0 ? 2 : row == 1 ? 2 : row == 2 ? 1 : 3;
  const float sg = row == 1 ? 1.f : -1.f;
  const float *const fa = S + (ra * 4 * TB + j) * CH + h * 4;
  const float *const fb = S + (rb * 4 * TB + j) * CH + h * 4;
  float4 tr[4];  // row-combined patch pixels of the step ahead
  auto lread = [&](int buf, int c) {
    const float4 u = *reinterpret_cast<const float4 *>(fa + buf * (16 * TB * CH) + c * (TB * CH));
    const float4 v = *reinterpret_cast<const float4 *>(fb + buf * (16 * TB * CH) + c * (TB * CH));
    tr[c] = fma4(sg, v, u);
  };

  const int ubase = ((nb * q.nchunks) * UB + row * 4 * UP + lane * 4) * 4;
  float4 uf[4][NF];  // fragments of column b: re-loaded one section after their last use
  auto uload = [&](int s, int b) {
#pragma unroll
    for (int n = 0; n < NF; ++n) uf[b][n] = bload(rsu, ubase + (b * UP + n * 256) * 4, last(s) * (UB * 4));
  };

  floatx16 acc[4][NF];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int n = 0; n < NF; ++n)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[b][n][e] = 0.f;

  // ---- prologue: steps s_lo, s_lo+1 in LDS, s_lo+2 in registers, row combination of s_lo ----
  float4 sx[4];
  {
    float4 sa[4], sb[4];
    halve(s_lo);
    gload(s_lo, sa);
    halve(s_lo + 1);
    gload(s_lo + 1, sb);
    halve(s_lo + 2);
    gload(s_lo + 2, sx);
#pragma unroll
    for (int b = 0; b < 3; ++b) uload(s_lo, b);
    lstore(0, sa);
    lstore(1, sb);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c) lread(0, c);

  // Four sections per step, one per column b of the transformed domain, each closed by a scheduling
  // fence: left alone the compiler gathers all loads at the end of the step, right in front of their use.
  int buf = 0;  // buffer of step s
  for (int s = s_lo; s < s_hi; ++s) {
    halve(s + 3);
    __syncthreads();  // step s+1 is in buffer buf^1; everybody has read step s out of buffer buf
    const float4 v[4] = {sub4(tr[0], tr[2]), add4(tr[1], tr[2]), sub4(tr[2], tr[1]), sub4(tr[1], tr[3])};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      lread(buf ^ 1, b);
      if (b == 0) {
        uload(s, 3);
        lstore(buf, sx);
      } else {
        uload(s + 1, b - 1);
      }
      if (b == 1) gload(s + 3, sx);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int n = 0; n < NF; ++n)
          acc[b][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(el(v[b], k), el(uf[b][n], k), acc[b][n], 0, 0, 0);
      if constexpr (NF == 2) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                // one MFMA
          if (i < 1) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);                     // + patch reads
          if (b == 0 && i >= 2 && i < 6) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0); // + an LDS write
          if (i < (b == 1 ? 6 : 2)) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);      // + a load
          if (i >= 3) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);                    // + address, row combination
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (i < 1) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          if (b == 0 && i >= 1 && i < 3) __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);
          if (b == 1 || i < 1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
          if (b == 1 && i == 3) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
          if (i >= 1) __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    buf ^= 1;
  }

  // ---- epilogue: this thread's results are filters n .. n+3 of NT (tile, column) x 2 rows ----
  constexpr int NG = NB / 4, NT = 64 * NG / NTHREADS;
  const bool split = gridDim.y > 1;
  float *const out = p.out + (split ? (long long)blockIdx.y * p.M * p.N : 0ll);
  const int n = nb * NB + (t % NG) * 4;
  // (POOL: a thread takes both columns of a tile)
  auto task_of = [&](int i) {
    if constexpr (POOL) return ((i >> 1) * (NTHREADS / NG) + t / NG) * 2 + (i & 1);
    return i * (NTHREADS / NG) + t / NG;
  };  // (tile, column)
  long long off[NT][2];  // -1: no such pixel or filter
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int task = task_of(i);
    const int tile = t0 + (task >> 1);
    const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
    const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
    const int wo = 2 * tx + (task & 1);
    const bool ok = (tile < q.T) & (wo < p.Wo) & (n < p.N);
#pragma unroll
    for (int k = 0; k < 2; ++k)
      off[i][k] = (ok & (2 * ty + k < p.Ho)) ? ((long long)(img * p.Ho + 2 * ty + k) * p.Wo + wo) * p.N + n : -1;
  }
  // shortcut or mask: fetched before the transform, so that the loads overlap it
  const float *const extra = split ? nullptr : p.addsrc ? p.addsrc : p.mask;
  float4 ex[NT][2];
  if (extra) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (off[i][k] >= 0) ex[i][k] = *reinterpret_cast<const float4 *>(extra + off[i][k]);
  }
  // output transform: columns in registers, rows through LDS
  __syncthreads();
  {
    float *const cw = S + row * (TB * 2 * NB) + NF * j;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = 8 * (e >> 2) + 4 * h + (e & 3);
      float y0[NF], y1[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const float pl = acc[1][f][e], mi = acc[2][f][e];
        y0[f] = acc[0][f][e] + pl + mi, y1[f] = pl - mi - acc[3][f][e];
      }
      if constexpr (NF == 2) {
        *reinterpret_cast<float2 *>(cw + (r * 2 + 0) * NB) = make_float2(y0[0], y0[1]);
        *reinterpret_cast<float2 *>(cw + (r * 2 + 1) * NB) = make_float2(y1[0], y1[1]);
      } else {
        cw[(r * 2 + 0) * NB] = y0[0], cw[(r * 2 + 1) * NB] = y1[0];
      }
    }
  }
  __syncthreads();
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  if (p.bias && !split && n < p.N) bias = *reinterpret_cast<const float4 *>(p.bias + n);
  // everything after the contraction for one result
  auto finish = [&](float4 v, float4 x, long long o) -> float4 {
    if (!split) {
      v = add4(v, bias);
      if (p.addsrc) v = add4(v, x);
      if (p.relu) v.x = v.x > 0.f ? v.x : 0.f, v.y = v.y > 0.f ? v.y : 0.f, v.z = v.z > 0.f ? v.z : 0.f, v.w = v.w > 0.f ? v.w : 0.f;
      if (p.mask) {
        const float4 m = p.addsrc ? *reinterpret_cast<const float4 *>(p.mask + o) : x;
        v.x = m.x > 0.f ? v.x : 0.f, v.y = m.y > 0.f ? v.y : 0.f, v.z = m.z > 0.f ? v.z : 0.f, v.w = m.w > 0.f ? v.w : 0.f;
      }
    }
    return v;
  };
  // results whose bits are not in `skip` (a projection's result, read as addsrc, may lie where they go)
  auto store = [&](const float4 &v, long long o, unsigned skip) {
    if (!skip) {
      *reinterpret_cast<float4 *>(out + o) = v;
      return;
    }
    if (!(skip & 1u)) out[o] = v.x;
    if (!(skip & 2u)) out[o + 1] = v.y;
    if (!(skip & 4u)) out[o + 2] = v.z;
    if (!(skip & 8u)) out[o + 3] = v.w;
  };
  if constexpr (POOL) {
    float4 y[NT][2];
    unsigned bad = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const float *c = S + task_of(i) * NB + (t % NG) * 4;
      constexpr int RS = TB * 2 * NB;
      const float4 r0 = *reinterpret_cast<const float4 *>(c), r1 = *reinterpret_cast<const float4 *>(c + RS);
      const float4 r2 = *reinterpret_cast<const float4 *>(c + 2 * RS), r3 = *reinterpret_cast<const float4 *>(c + 3 * RS);
      y[i][0] = add4(add4(r0, r1), r2), y[i][1] = sub4(sub4(r1, r2), r3);
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (off[i][k] >= 0) bad |= bad4(y[i][k]) << (4 * (2 * i + k));
    }
    if (bad) {
#pragma unroll 1
      for (int ik = 0; ik < 2 * NT; ++ik) {
        const unsigned want = bad >> (4 * ik) & 15u;
        if (!want) continue;
        const int task = task_of(ik >> 1), tile = t0 + (task >> 1);
        const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
        const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
        const float4 v = direct4(p.x, p.w, p.H, p.W, p.C, img, 2 * ty + (ik & 1), 2 * tx + (task & 1), n, s_lo * CH,
                                 min(p.C, s_hi * CH), want);
#pragma unroll
        for (int k = 0; k < 2 * NT; ++k)
          if (k == ik) {
            float4 &o = y[k >> 1][k & 1];
            if (want & 1u) o.x = v.x;
            if (want & 2u) o.y = v.y;
            if (want & 4u) o.z = v.z;
            if (want & 8u) o.w = v.w;
          }
      }
    }
#pragma unroll
    for (int i = 0; i < NT; i += 2) {
      const int tile = t0 + (task_of(i) >> 1);
      const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
      const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
      if ((tile >= q.T) | (ty >= p.Hp) | (tx >= p.Wp) | (n >= p.N)) continue;  // (else all four pixels exist)
      float best[4];
      unsigned at[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) best[e] = -INFINITY, at[e] = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {  // row-major, the first maximum wins
        const float4 v = finish(y[i + (w & 1)][w >> 1], ex[i + (w & 1)][w >> 1], off[i + (w & 1)][w >> 1]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (el(v, e) > best[e]) best[e] = el(v, e), at[e] = w;
      }
      const long long o = ((long long)(img * p.Hp + ty) * p.Wp + tx) * p.N + n;
      *reinterpret_cast<float4 *>(p.out + o) = make_float4(best[0], best[1], best[2], best[3]);
      *reinterpret_cast<unsigned *>(p.max_arg + o) = at[0] | at[1] << 8 | at[2] << 16 | at[3] << 24;
    }
    return;
  }
  unsigned bad = 0;  // four bits from 4*(2*i + k): which of those results are not finite
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int task = task_of(i), lt = task >> 1;
    const float *c = S + (lt * 2 + (task & 1)) * NB + (t % NG) * 4;
    constexpr int RS = TB * 2 * NB;  // next row of the transformed domain
    const float4 r0 = *reinterpret_cast<const float4 *>(c), r1 = *reinterpret_cast<const float4 *>(c + RS);
    const float4 r2 = *reinterpret_cast<const float4 *>(c + 2 * RS), r3 = *reinterpret_cast<const float4 *>(c + 3 * RS);
    const float4 y[2] = {add4(add4(r0, r1), r2), sub4(sub4(r1, r2), r3)};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (off[i][k] < 0) continue;
      const unsigned b = bad4(y[k]);
      bad |= b << (4 * (2 * i + k));
      store(finish(y[k], ex[i][k], off[i][k]), off[i][k], b);
    }
  }
  if (bad == 0) return;
#pragma unroll 1
  for (int ik = 0; ik < 2 * NT; ++ik) {
    const unsigned want = bad >> (4 * ik) & 15u;
    if (!want) continue;
    const int task = task_of(ik >> 1), tile = t0 + (task >> 1);
    const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
    const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
    const int ho = 2 * ty + (ik & 1), wo = 2 * tx + (task & 1);
    const long long o = ((long long)(img * p.Ho + ho) * p.Wo + wo) * p.N + n;
    const float4 v = direct4(p.x, p.w, p.H, p.W, p.C, img, ho, wo, n, s_lo * CH, min(p.C, s_hi * CH), want);
    float4 x = bias;
    if (extra) x = *reinterpret_cast<const float4 *>(extra + o);
    store(finish(v, x, o), o, ~want & 15u);
  }
}

}  // namespace

size_t wino_fwd_filter_floats(int N, int C) {
  const int nb = wino_nb(N);
  return (size_t)((N + nb - 1) / nb) * ((C + CH - 1) / CH) * (16 * nb * CH);
}

namespace {
bool applicable(const FwdProblem &p) {
  if (p.R != 3 || p.S != 3 || p.stride != 1 || p.pad != 1 || p.pool_part) return false;
  if (p.C % 4 || p.N % 4) return false;
  const long long lim = 0x7FFFFFF0ll, B = p.M / ((long long)p.Ho * p.Wo);
  return B * p.H * p.W * p.C * 4 <= lim && (long long)wino_fwd_filter_floats(p.N, p.C) * 4 <= lim;
}
}  // namespace

// Which kernel, and how many reduction splits: both times are estimated from the step times below and
// the smaller one wins.  Of 440 random shapes for which this kernel is chosen (16 ... 512 channels, 36 ... 512 filters) it
// takes 0.63 of the direct kernels' time in all, and is the slower one for 7, by 14 % at most (reductions split in two or
// four, whose direct form the estimate has a tenth too slow).  Examples (us, direct / this): 512 -> 512 channels,
// 8192 pixels 312 / 150; 128 -> 128, 16 384 pixels 45 / 30, 4096 pixels 20 / 22 (direct); 512 -> 512, 1024 pixels
// 52 / 40 (8 splits); 64 -> 64, 65 536 pixels 43 / 34.
// Two lines are drawn by accuracy, not by time.  Where the direct kernel splits its reduction its sums
// are short, and this one needs about as many splits to stay below their error (512 -> 512, 1024 pixels,
// 8 direct splits 2.7e-7: 4 splits here 3.4e-7, 8 splits 2.5e-7).  On maps narrower than 4 most taps
// multiply padding: the direct sum skips their rounding, the transforms do not (2x2 maps 1.5e-7
// against 1.9e-7 ... 2.9e-7).
namespace {
double finish_us(const FwdProblem &p, int s) {  // fwd_finish at 4 TB/s
  return s > 1 ? 3.5 + (double)p.M * p.N * 4.0 * (s + 1) / 4e6 : 0.0;
}
long long workgroups(const FwdProblem &p) {
  const int B = p.M / (p.Ho * p.Wo);
  const long long tiles = ((long long)B * ((p.Ho + 1) / 2) * ((p.Wo + 1) / 2) + TB - 1) / TB;
  const int nb = wino_nb(p.N);
  return tiles * ((p.N + nb - 1) / nb);
}
// this kernel: 1.13 us per step with one workgroup on a CU, 2.12 with two (before load offsets advanced in scalar registers; 1.03
// and 1.93 now, so that layers near the line keep the direct kernel), in rounds of 512 workgroups; 11 us of prologue, epilogue
// and launches, 3 us for each further round; the transformed filter written and read at 4 TB/s; a projection shortcut is a
// launch of its own whose result this kernel adds (enqueue_conv).  The pooling launch that a layer with 2x2 windows saves
// here (8 us) is not counted
double wino_us(const FwdProblem &p, int s) {
  const int nchunks = (p.C + CH - 1) / CH;
  const long long w = workgroups(p) * s;
  const long long full = w / 512, rest = w % 512;
  const double per = 2.12 * full + (rest > 256 ? 2.12 : rest > 0 ? 1.13 : 0.0), mn = (double)p.M * p.N;
  const double proj = p.Cs ? 8.0 + 2.0 * mn * p.Cs / 90e6 + 4.0 * mn / 4e6 : 0.0;
  return 11.0 + 3.0 * (full + (rest > 0) - 1) + (double)p.C * p.N * 100.0 / 4e6 + (nchunks + s - 1) / s * per +
         finish_us(p, s) + proj;
}
// its variant of 32 filters: 0.8, 1.4 and 2.1 us per step with one, two and three workgroups on a CU, 6 us of prologue,
// epilogue and launch, 3 us for a filter launch of its own in front of it (0.3 ... 5.3 us in backward calls of ten sizes: us a call, with
// it / direct: 8 -> 32 channels, 16x16, 64-wide head, batch 8 26.3 / 24.0, 64 35.8 / 35.8, 128 45.1 / 46.2; 28x28, 24 channels,
// 80-wide head, batch 50 72.4 / 77.5); the direct kernel of 64x32 tiles in its place 0.3 us per step and workgroup on a CU.  On 36 random shapes (17 ... 32 filters, 16 ... 512 channels) this one is chosen 10 times and is the
// faster one each time, by 3 to 33 % (us, direct / this with its filter launch: 64 -> 32, 204 800 pixels 72.5 / 50.1; 16 -> 28, 174 592
// pixels 29.2 / 22.6; 64 -> 32, 16 384 pixels 12.0 / 14.7, direct); the error of its single results is the smaller one on all 36 (64 -> 32
// 2.9e-7 / 2.1e-7)
double narrow_us(const FwdProblem &p, int s, bool ready) {
  const int nchunks = (p.C + CH - 1) / CH;
  const long long w = workgroups(p) * s, full = w / 768, rest = w % 768;
  const double per = 2.1 * full + (rest > 512 ? 2.1 : rest > 256 ? 1.4 : rest > 0 ? 0.8 : 0.0);
  return (ready ? 6.0 : 9.0) + 3.0 * (full + (rest > 0) - 1) + (nchunks + s - 1) / s * per + finish_us(p, s);
}
double narrow_direct_us(const FwdProblem &p, int ks) {
  const int nkb = (p.Kg + 31) / 32;
  const long long w = (long long)((p.M + 63) / 64) * ks;
  return 7.3 + (nkb + ks - 1) / ks * 0.3 * ((w + 255) / 256) + finish_us(p, ks);
}

int pick_splits(const FwdProblem &p, int ks, int most, bool ready) {
  // up to 16 filters half of a workgroup's columns would be padding; below 16 channels the result's own
  // traffic is all there is to either kernel (8 channels, 16 384 x 256 results: 17 / 14 + 5 for the filter launch)
  if (p.N <= 16 || p.C < 16 || p.Ho < 4 || p.Wo < 4 || !applicable(p)) return 0;
  const int nchunks = (p.C + CH - 1) / CH;
  const bool narrow = wino_nb(p.N) == 32;
  double best = 0.0;
  int splits = 0;
  for (int s = 1; s <= 16; s *= 2) {
    if (4 * s < 3 * ks) continue;
    if (s > most) break;
    if (s > 1 && (nchunks / s < 2 || workgroups(p) * s > 512)) break;
    const double us = narrow ? narrow_us(p, s, ready) : wino_us(p, s);
    if (!splits || us < best) best = us, splits = s;
  }
  if (narrow) return splits && best < 0.93 * narrow_direct_us(p, ks) ? splits : 0;
  // the direct kernel: steps of 32 products, 128x128 tiles one per CU, or 64x64 ones up to four, in rounds
  // of 1024 workgroups (2 us for each further one)
  const int nkb = (p.Kg + 31) / 32;
  const bool big = igemm_fwd_tile128(p.M, p.N, p.Kg, ks);
  const int bt = big ? 128 : 64;
  const long long w = (long long)((p.M + bt - 1) / bt) * ((p.N + bt - 1) / bt) * ks;
  const long long full = w / 1024, rest = w % 1024;
  const double per = big ? 2.06 * ((w + 255) / 256) : 2.2 * full + (rest > 0 ? std::max(0.56, 0.55 * rest / 256.0) : 0.0);
  const double direct = 8.0 + (big ? 0.0 : 2.0 * (full + (rest > 0) - 1)) + (nkb + ks - 1) / ks * per + finish_us(p, ks);
  return splits && best < 0.93 * direct ? splits : 0;
}
}  // namespace

// Up to 32 filters a layer and a head keep the direct sum.  The transformed filter is rounded once for all pixels and samples, which
// the head's pooling averages and its gradients sum: single results come out closer to 64 bits, these averages not.  Error of the
// 32-filter variant over the direct sum's, 24 inputs each: as a head's convolution (64 channels, 32x32, 32 filters) logits 1.11, dWf 1.32,
// dWa 1.11; as a layer's (64 -> 24, 24x24) its output 0.78, but dWf 1.12, dWa 1.10.  As a data gradient, whose every use is another
// contraction, it is the more exact one: 32 filters, 40x43, 80-wide head, dW 0.70, db 0.66; 16x16, 64-wide 0.89, 0.95.
int wino_fwd_pick_splits(const FwdProblem &p, int ks, int most) { return p.N <= 32 ? 0 : pick_splits(p, ks, most, false); }

int wino_dgrad_pick_splits(const FwdProblem &p, int ks, bool ready) { return pick_splits(p, ks, 16, ready); }

hipError_t launch_wino_fwd(const FwdProblem &p, float *U, bool filter_ready, const WinoFilter *also, hipStream_t st) {
  WinoAux q;
  const int TH = (p.Ho + 1) / 2, B = p.M / (p.Ho * p.Wo);
  q.TW = (p.Wo + 1) / 2, q.TPI = TH * q.TW, q.T = B * q.TPI;
  q.nchunks = (p.C + CH - 1) / CH;
  const int nb = wino_nb(p.N);
  q.nblk = (p.N + nb - 1) / nb;
  q.div_tpi = FastDiv(q.TPI), q.div_tw = FastDiv(q.TW);
  q.x_bytes = (uint32_t)((long long)B * p.H * p.W * p.C * 4);
  q.u_bytes = (uint32_t)(wino_fwd_filter_floats(p.N, p.C) * 4);
  q.U = U;
  const int splits = p.ksplits > 1 ? p.ksplits : 1;
  q.per = (q.nchunks + splits - 1) / splits;
  if (!filter_ready || also) {
    FilterJobs js;
    int blocks = js.blocks0 = 0, n = 0;
    for (int k = 0; k < 2; ++k) {
      if (k == 0 ? filter_ready : !also) continue;
      const WinoFilter f = k ? *also : WinoFilter{p.w, U, p.N, p.C};
      const int fnb = wino_nb(f.N);
      js.f[n] = f, js.nchunks[n] = (f.C + CH - 1) / CH, js.bx[n] = (2 * js.nchunks[n] + 7) / 8;
      blocks += js.bx[n] * ((f.N + fnb - 1) / fnb) * (fnb / 32);
      if (n++ == 0) js.blocks0 = blocks;
    }
    hipLaunchKernelGGL(wino_filter_kernel, dim3(blocks), dim3(256), 0, st, js);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const dim3 grid(q.nblk * ((q.T + TB - 1) / TB), splits);
#define NF_LAUNCH(NF_, POOL_) hipLaunchKernelGGL((wino_fwd_kernel<NF_, POOL_>), grid, dim3(NTHREADS), 0, st, p, q)
  if (nb == 32) NF_LAUNCH(1, false);
  else if (p.max_arg) NF_LAUNCH(2, true);
  else NF_LAUNCH(2, false);
#undef NF_LAUNCH
  return hipGetLastError();
}

}  // namespace nf
