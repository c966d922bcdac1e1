// Weight gradient of a 3x3 / stride 1 / pad 1 convolution (gradient line of Algorithm 2, NeuroFlux,
// arXiv 2402.14139) through the minimal filtering algorithm F(3x3, 2x2) (S. Winograd 1980; A. Lavin,
// S. Gray, arXiv 1509.09308), entirely in fp32.  Per 2x2 tile of output pixels, with d the 2x2
// gradient and x the 4x4 input patch,
//     dW (3x3) += A^T [ (G d G^T) . (B^T x B) ] A,
// 16 multiplications per (filter, channel) where the direct sum takes 36.  The sum over the tiles
// runs in the transformed domain: 16 contractions on the fp32 matrix cores, A^T . A once per sum.
//
// What bounds it: the fp32 MFMA rate (16/36 of the direct kernel's MFMAs).  Layout of the work:
//   - a workgroup owns 64 filters x 32 channels x all 16 positions over a range of tiles (a split of
//     the reduction); its 4 waves are the 4 rows of the transformed domain;
//   - a 16x16x4 MFMA takes four tiles, one per quarter of the wave.  A lane's operands are two
//     channels of a patch and four filters of a gradient tile: both tensors have channels innermost, so a
//     wave loads them in fragment order straight from memory (rows of 128 / 256 contiguous bytes, two
//     steps ahead), transforms them in registers and needs no barrier and no staged operand in its
//     loop.  A step is 32 MFMAs, 12 loads and 62 vector operations; the latter two are not free beside
//     fp32 MFMAs: two waves on a SIMD take about 3000 cycles for a step each, 2048 of them MFMAs (the vector operations in clumps,
//     see step; pipe busy 63 % of whole launches, 56 % with them spread singly);
//     (32x32x2 MFMAs, two tiles per step: half the operands per load, 24 loads for the same
//     MFMAs, 232 us where this took 216 before the clumps; 512 channels, 8192 pixels);
//   - the byte offsets of 64 tiles at a time stand in a table in LDS (one thread decodes a tile; what
//     is outside the image is an offset the hardware answers with zeros);
//   - every 64 tiles the accumulators go through A^T . A (columns in registers, in place and once per row, rows in
//     LDS, in a fixed order) and are added to the 3x3 result in LDS: 4.9 us beside the other workgroup's products, a
//     fifth of the time (5.5 us with the columns formed for each of the three additions of rows 1 and 2).  That keeps the sums in the transformed
//     domain short: its 9 terms per result would otherwise cost accuracy (relative error against 64 bits of
//     a 2048-tile sum, numpy model: direct 2.8e-7, this 2.2e-7, without the 64-tile sums 1.0e-6);
//   - 128 accumulators per lane, two workgroups per CU: one's transforms and LDS phases fill in under the
//     other's MFMAs.
//
// A value that is not finite makes NaN of neighbours that the direct sum would leave finite or
// infinite: a workgroup that finds one among its results forms them again by the direct sum.
#include <cmath>

#include "nf_internal.h"

namespace nf {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int NTHREADS = 256;
constexpr int PB = 64, QB = 32;          // filters, channels per workgroup
constexpr int PERIOD = 64;               // most tiles between additions to the result
constexpr int KT = 4;                    // tiles per step
constexpr int SETS = 2;                  // steps in flight
constexpr int NT = PERIOD + KT * (SETS + 1);  // table entries
static_assert(PERIOD % (KT * SETS) == 0 && SETS == 2 && NT <= 128, "whole rounds; two waves decode a table");
// Both tensors are smaller than 1 GiB: a table entry for "outside the image" and a lane's offset for
// "no such channel" are out of range each, and so is their sum.
constexpr int OOB_T = 0x40000000, OOB_L = (int)0x80000000;
constexpr int RSRC_FLAGS = 0x00020000;   // raw buffer, 32-bit data format

struct WinoWgradAux {
  int TW, TPI, T, tps;  // tiles per image row, per image, in all, per split (a multiple of 8)
  int period;           // tiles between additions to the result
  int nq, np;           // channel blocks, filter blocks
  FastDiv div_tpi, div_tw;
  uint32_t x_bytes, d_bytes;
};

typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ inline floatx2 bload2(__amdgpu_buffer_rsrc_t r, int voff) {
  return __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 0));
}
__device__ inline floatx4 bload4(__amdgpu_buffer_rsrc_t r, int voff) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
}

__global__ __launch_bounds__(NTHREADS, 2) void wino_wgrad_kernel(WgradProblem p, WinoWgradAux q) {
  // the 3x3 result [tap][channel][filter]; the 16 groups of 4 filters of a channel are stored at
  // group ^ (channel / 2), so that 16 lanes along the channel pairs touch all banks
  __shared__ __attribute__((aligned(16))) float R[9 * QB * PB];
  // per tile: byte offsets of the patch's 4x4 pixels, and of the gradient's 2x2 (a third row: none)
  __shared__ int4 Tx[4][NT];
  __shared__ int2 Td[3][NT];

  const int t = threadIdx.x;
  const int lane = t & 63, row = t >> 6;
  const int j = lane & 15, h = lane >> 4;  // channels q0 + 2j, +1; filters p0 + 4j .. +3; tile h of a step
  // XCD re-map: each XCD gets a contiguous run of (split, filter block, channel block), so that the
  // blocks of a split read its rows of x and d into one L2
  const int nwg = gridDim.x, lin = blockIdx.x;
  const int wper = nwg >> 3, wrem = nwg & 7, xcd = lin & 7, slot = lin >> 3;
  const int id = xcd < wrem ? xcd * (wper + 1) + slot : wrem * (wper + 1) + (xcd - wrem) * wper + slot;
  const int bq = id % q.nq, bpz = id / q.nq, bp = bpz % q.np, bz = bpz / q.np;
  const int p0 = bp * PB, q0 = bq * QB;
  const int t_lo = bz * q.tps, t_hi = min(q.T, t_lo + q.tps);

  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, q.x_bytes, RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t rsd = __builtin_amdgcn_make_buffer_rsrc((void *)p.d, 0, q.d_bytes, RSRC_FLAGS);

  auto table = [&](int base, int i) {  // entry i
    if (i < NT) {
      const int tile = base + i;
      const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
      const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
      const bool ok = tile < t_hi;
      const int wi = 2 * tx - 1, cs = p.C * 4, ps = p.P * 4;
      const bool c2 = wi + 2 < p.W;  // (also the gradient's second column)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int hi = 2 * ty - 1 + r;
        const bool rok = ok & ((unsigned)hi < (unsigned)p.H);
        const int o = ((img * p.H + hi) * p.W + wi) * cs;
        Tx[r][i] = make_int4((rok & (wi >= 0)) ? o : OOB_T, rok ? o + cs : OOB_T, (rok & c2) ? o + 2 * cs : OOB_T,
                             (rok & (wi + 3 < p.W)) ? o + 3 * cs : OOB_T);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const bool rok = ok & (2 * ty + k < p.Ho);
        const int o = ((img * p.Ho + 2 * ty + k) * p.Wo + 2 * tx) * ps;
        Td[k][i] = make_int2(rok ? o : OOB_T, (rok & c2) ? o + ps : OOB_T);
      }
      Td[2][i] = make_int2(OOB_T, OOB_T);
    }
  };

  // this wave's row of B^T: x[ra] + sg * x[rb]; of 2 G (rows 1, 2) or G (rows 0, 3): d[da] + sd * d[db]
  const int ra = row == 0 ? 0 : row == 2 ? 2 : 1, rb = row == 0 ? 2 : row == 1 ? 2 : row == 2 ? 1 : 3;
  const int da = row == 3 ? 1 : 0, db = (row == 0 || row == 3) ? 2 : 1;
  const float sg = row == 1 ? 1.f : -1.f, sd = row == 1 ? 1.f : row == 2 ? -1.f : 0.f;
  const int qoff = (q0 + 2 * j) * 4 + (q0 + 2 * j < p.C ? 0 : OOB_L);
  const int poff = (p0 + 4 * j) * 4 + (p0 + 4 * j < p.P ? 0 : OOB_L);

  floatx2 xr[SETS][2][4];  // [set][row ra, rb][column], two channels
  floatx4 dr[SETS][2][2];  // [set][row da, db][column], four filters
  int4 ea, eb;             // table entries of the step to load next
  int2 fa, fb;
  auto tread_x = [&](int i) { ea = Tx[ra][KT * i + h], eb = Tx[rb][KT * i + h]; };  // i: step within the table
  auto tread_d = [&](int i) { fa = Td[da][KT * i + h], fb = Td[db][KT * i + h]; };
  auto gload = [&](int set, int part) {  // a third of a step's twelve loads
    if (part == 0) {
      xr[set][0][0] = bload2(rsx, ea.x + qoff), xr[set][0][1] = bload2(rsx, ea.y + qoff);
      xr[set][0][2] = bload2(rsx, ea.z + qoff), xr[set][0][3] = bload2(rsx, ea.w + qoff);
    } else if (part == 1) {
      xr[set][1][0] = bload2(rsx, eb.x + qoff), xr[set][1][1] = bload2(rsx, eb.y + qoff);
      xr[set][1][2] = bload2(rsx, eb.z + qoff), xr[set][1][3] = bload2(rsx, eb.w + qoff);
    } else {
      dr[set][0][0] = bload4(rsd, fa.x + poff), dr[set][0][1] = bload4(rsd, fa.y + poff);
      dr[set][1][0] = bload4(rsd, fb.x + poff), dr[set][1][1] = bload4(rsd, fb.y + poff);
    }
  };

  floatx4 acc[4][4][2];  // [column of the transformed domain][filter][channel]
  floatx2 xc[4];  // row combination of the current step, [column]
  floatx4 u[2];
  floatx4 bs = (floatx4)(0.f);  // column sums of d (row 1)
  auto combine = [&](int set) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int n = 0; n < 2; ++n) xc[c][n] = __builtin_fmaf(sg, xr[set][1][c][n], xr[set][0][c][n]);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int a = 0; a < 4; ++a) u[c][a] = __builtin_fmaf(sd, dr[set][1][c][a], dr[set][0][c][a]);
  };

  // Step i, two sections of two columns of the transformed domain each: their operands, then their MFMAs, and the loads of step i+SETS
  // into set `cur`, whose rows step i already combined (one behind an MFMA: a burst of all twelve from four waves holds the waves
  // up at the address unit, 16 cycles a load); in the second also the row combination of step i+1.  The vector instructions stand
  // in two clumps a section: an fp32 MFMA and a vector instruction hold each other up, about 14 cycles for each change from the one
  // to the other and 2 (two waves on a SIMD) for each instruction, so that 62 of them spread singly behind 32 MFMAs add 550 cycles to
  // the 2048 of two waves' MFMAs and in four clumps half of that (512 channels, 8192 pixels 210 / 192 us; in two clumps, with more
  // registers held and spilled, 199).
  auto step = [&](int i, int cur, bool first) {  // first: the sums start at zero
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      floatx2 v[2];
      floatx4 g[2];
      if (half == 0) {
        v[0] = xc[0] - xc[2], v[1] = xc[1] + xc[2], g[0] = u[0], g[1] = u[0] + u[1];
        bs += g[1];
        gload(cur, 0), gload(cur, 1);
        tread_d(i + SETS);
      } else {
        v[0] = xc[2] - xc[1], v[1] = xc[1] - xc[3], g[0] = u[0] - u[1], g[1] = u[1];
        gload(cur, 2);
        combine((cur + 1) % SETS);
        tread_x(i + 1 + SETS);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int n = 0; n < 2; ++n)
            acc[2 * half + c][a][n] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(g[c][a], v[c][n], first ? (floatx4)(0.f) : acc[2 * half + c][a][n], 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 16, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 40, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                         // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                         // + a load
        if (k >= 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);             // + a table read
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // A^T on the columns, times s (a power of two): in place, three values of the four
  auto columns = [&](float s) {
    const float hs = 0.5f * s;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float m1 = acc[1][a][n][e], m2 = acc[2][a][n][e], t = hs * (m1 + m2);
          acc[0][a][n][e] = __builtin_fmaf(s, acc[0][a][n][e], t);
          acc[1][a][n][e] = hs * (m1 - m2);
          acc[2][a][n][e] = __builtin_fmaf(-s, acc[3][a][n][e], t);
        }
  };
  // adds s (+-1) times them to row r of the result, or stores them
  auto emit = [&](int r, float s, bool store) {
    int jj = j;
    asm volatile("" : "+v"(jj));  // keeps the addresses below from being held in registers over the main loop
    float *const base = R + (r * 3 * QB + 2 * jj) * PB;
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // six words at a time: all reads, then all writes
      const int n = k >> 1;
      floatx4 z[2][3];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int e = 2 * (k & 1) + i, grp = (4 * h + e) ^ jj;  // filters 16*h + 4*e .. +3 of channel 2j + n
#pragma unroll
        for (int c = 0; c < 3; ++c)
          z[i][c] = store ? (floatx4)(0.f) : *reinterpret_cast<const floatx4 *>(base + (c * QB + n) * PB + grp * 4);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int e = 2 * (k & 1) + i, grp = (4 * h + e) ^ jj;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma unroll
          for (int a = 0; a < 4; ++a) z[i][c][a] = __builtin_fmaf(s, acc[c][a][n][e], z[i][c][a]);
          *reinterpret_cast<floatx4 *>(base + (c * QB + n) * PB + grp * 4) = z[i][c];
        }
      }
    }
  };

  // ---- main loop ----
  table(t_lo, t);
  __syncthreads();
  // in this order, or the loop's waits are for the last of the loads
#pragma unroll
  for (int a = 0; a < SETS; ++a) {
    tread_x(a), tread_d(a);
    for (int k = 0; k < 3; ++k) gload(a, k);
    __builtin_amdgcn_sched_barrier(0);
  }
  combine(0);
  tread_x(SETS);
  __builtin_amdgcn_sched_barrier(0);
  for (int base = t_lo; base < t_hi; base += q.period) {
    const int nsteps = (min(q.period, t_hi - base) + KT * SETS - 1) / (KT * SETS) * SETS;
    step(0, 0, true);
    step(1, 1, false);
    for (int i = SETS; i < nsteps; i += SETS) {
#pragma unroll
      for (int a = 0; a < SETS; ++a) step(i + a, a, false);
    }
    __syncthreads();  // everybody has left the table and the previous additions
    // rows of A^T: 0 = +0 +1 +2, 1 = +1 -2, 2 = +1 +2 -3, with the factor 1/2 that rows 1 and 2 of G have
    // and sd leaves out; three phases without two waves on one row of the result, the waves that have
    // nothing to add in one decode the next tiles
    columns(row == 0 ? 1.f : row == 3 ? -1.f : 0.5f);
    if (row < 3) emit(row, 1.f, base == t_lo);
    else table(base + q.period, 64 + lane);
    __syncthreads();
    if (row == 0) table(base + q.period, lane);
    else emit(row == 3 ? 2 : row - 1, row == 2 ? -1.f : 1.f, false);
    __syncthreads();
    if (row == 1 || row == 2) emit(row == 2 ? 0 : 2, 1.f, false);
  }
  if (t_lo >= t_hi)  // an empty split
    for (int k = t; k < 9 * QB * PB / 4; k += NTHREADS) reinterpret_cast<float4 *>(R)[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();

  // ---- store: lanes along the channels ----
  float *const part = p.part + (long long)bz * p.P * p.Qld;
  bool bad = false;
  {
    const int c = t & 31;
#pragma unroll 2
    for (int k = t >> 5; k < 9 * 16; k += 8) {
      const int tap = k >> 4, grp = k & 15;
      const float4 v = *reinterpret_cast<const float4 *>(R + (tap * QB + c) * PB + (grp ^ (c >> 1)) * 4);
      bad |= !(__builtin_isfinite(v.x) & __builtin_isfinite(v.y) & __builtin_isfinite(v.z) & __builtin_isfinite(v.w));
      float *const o = part + (long long)(p0 + grp * 4) * p.Qld + tap * p.C + q0 + c;
      if (q0 + c < p.C && p0 + grp * 4 < p.P) o[0] = v.x, o[p.Qld] = v.y, o[2 * p.Qld] = v.z, o[3 * p.Qld] = v.w;
    }
  }
  if (bq == 0 && p.part_b && row == 1) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      bs[a] += __shfl_xor(bs[a], 16, 64);
      bs[a] += __shfl_xor(bs[a], 32, 64);
    }
    if (h == 0 && p0 + 4 * j < p.P) *reinterpret_cast<floatx4 *>(p.part_b + (long long)bz * p.P + p0 + 4 * j) = bs;
  }
  if (!__syncthreads_or(bad)) return;

  // ---- the direct sum: wave w forms taps w, w+4, w+8; a pixel outside the image takes no part, whatever its gradient ----
#pragma unroll 1
  for (int tap = row; tap < 9; tap += 4) {
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[0][a][0] = acc[0][a][1] = (floatx4)(0.f);
#pragma unroll 1
    for (int t4 = t_lo; t4 < t_hi; t4 += KT) {
      const int tile = t4 + h;
      const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
      const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ho = 2 * ty + (k >> 1), wo = 2 * tx + (k & 1), hi = ho + tap / 3 - 1, wi = wo + tap % 3 - 1;
        const bool ok = (tile < t_hi) & (ho < p.Ho) & (wo < p.Wo) & ((unsigned)hi < (unsigned)p.H) & ((unsigned)wi < (unsigned)p.W);
        const floatx4 d = bload4(rsd, poff + (ok ? ((img * p.Ho + ho) * p.Wo + wo) * p.P * 4 : OOB_T));
        const floatx2 x = bload2(rsx, qoff + (ok ? ((img * p.H + hi) * p.W + wi) * p.C * 4 : OOB_T));
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int n = 0; n < 2; ++n) acc[0][a][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[a], x[n], acc[0][a][n], 0, 0, 0);
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const int pr = p0 + 16 * h + 4 * e + a, c = q0 + 2 * j + n;
          if (pr < p.P && c < p.C) part[(long long)pr * p.Qld + tap * p.C + c] = acc[0][a][n][e];
        }
  }
}

}  // namespace

namespace {
bool applicable(const WgradProblem &p) {
  if (p.R != 3 || p.S != 3 || p.stride != 1 || p.pad != 1 || p.C % 4 || p.P % 4) return false;
  const long long lim = OOB_T, B = p.M / ((long long)p.Ho * p.Wo);
  return (long long)p.M * p.P * 4 <= lim && B * p.H * p.W * p.C * 4 <= lim;
}
long long num_tiles(const WgradProblem &p) {
  return (long long)(p.M / (p.Ho * p.Wo)) * ((p.Ho + 1) / 2) * ((p.Wo + 1) / 2);
}
int tiles_per_split(long long T, int splits) { return (int)(((T + splits - 1) / splits + 7) / 8 * 8); }
}  // namespace

// Which kernel, and how many splits: both times are estimated (this kernel and the direct one, each
// with the reading of its partial sums) and the smaller one wins.  Examples (us, direct / this, kernel +
// reduction): 512 -> 512 channels, 8192 pixels 328 + 19 / 216 + 17; 256 -> 256, 16 384 pixels 172 + 17 / 115 + 18;
// 128 -> 128, 16 384 pixels 55 + 14 / 40 + 14; 64 -> 64, 65 536 pixels 53 + 11 / 36 + 11; 16 384 pixels 20 + 10 / 22 + 12
// (direct).  (On 220 random shapes of 4 ... 512 channels it was chosen 118 times, 0.75 of the direct time on average, and
// once by mistake, 3 % slower; the 128x128 kernel is up to a tenth faster than its estimate, hence its larger margin.)  Left to the direct kernel whatever the time: up to 32 filters (half the tile would be
// padding); fewer than 8192 pixels and maps narrower than 4, where the direct sums are short and the
// transforms' own rounding would make this the less accurate one (relative error against 64 bits,
// direct / this: 256 channels, 4x4 maps, 4096 pixels 0.85e-7 / 0.93e-7, 2x2 maps 0.9e-7 / 1.8e-7; at 8192 and more
// pixels this one's is smaller: 1.5e-7 / 1.1e-7 with 512 channels, 1.1e-7 / 1.0e-7 with 128).
namespace {
double reduce_us(const WgradProblem &p, int s) { return s * (double)p.P * p.Q * 4.0 / 4e6; }  // at 4 TB/s
long long blocks_of(const WgradProblem &p) { return (long long)((p.C + QB - 1) / QB) * ((p.P + PB - 1) / PB); }
// a step of four tiles takes 1.0 us with one workgroup on a CU, 1.54 with two; the columns of a
// projection shortcut are a launch of their own (run_bwd)
double wino_us(const WgradProblem &p, int s) {
  const double w = (double)blocks_of(p) * s;
  const double proj = p.Cs ? 10.0 + 2.0 * p.M * p.P * p.Cs / 90e6 : 0.0;
  const double full = std::floor(w / 512), rest = w - 512 * full;  // rounds of two workgroups per CU
  const double rounds = 1.54 * full + (rest > 256 ? 1.54 : rest > 0 ? 1.0 : 0.0);
  return 11.0 + tiles_per_split(num_tiles(p), s) / KT * rounds + reduce_us(p, s) + proj;
}
// a direct kernel of 128x128 tiles: its padded contraction at the rate it reaches (flops per us), plus
// ramp-up and drain
double wide_us(const WgradProblem &p, double rate) {
  const double q128 = (p.Q + 127) / 128 * 128.0, p128 = (p.P + 127) / 128 * 128.0;
  return 14.0 + 2.0 * p.M * p128 * q128 / rate + reduce_us(p, wgrad_pick_splits(p.P, p.Q, p.M));
}
}  // namespace

int wino_wgrad_pick_splits(const WgradProblem &p, int most) {
  if (p.P <= 32 || p.M < 8192 || p.Ho < 4 || p.Wo < 4 || !applicable(p)) return 0;
  const long long T = num_tiles(p), blocks = blocks_of(p);
  double best = 0.0;
  int splits = 0;
  for (int wgs = 256; wgs <= 1024; wgs *= 2) {
    // (rounded down: 516 workgroups for 512 places take a second round of the chip)
    const int s = (int)(wgs > blocks ? wgs / blocks : 1);
    if (s > most || (s > 1 && T / s < 16)) break;
    const double us = wino_us(p, s);
    if (!splits || us < best) best = us, splits = s;
  }
  const int sd = wgrad_pick_splits(p.P, p.Q, p.M);
  const double p64 = (p.P + 63) / 64 * 64.0, q64 = (p.Q + 63) / 64 * 64.0;
  const bool wide = p.P > 64 && !igemm_wgrad_tile64(p.P, p.Q, sd);
  const double direct = wide ? wide_us(p, 118e6) : 8.0 + 2.0 * p.M * p64 * q64 / 104e6 + reduce_us(p, sd);
  return splits && best < (wide ? 0.95 : 0.975) * direct ? splits : 0;
}

// The split-operand kernel (six piece products) reaches 185 TFLOP/s.  Kernel alone, us (it / this): 512 -> 512
// channels, 8192 pixels 251 / 218, 256 -> 256, 16 384 pixels 129 / 116; error against 64 bits 1.7e-7 / 1.1e-7 and
// 1.4e-7 / 0.9e-7.
bool wino_wgrad_beats_split(const WgradProblem &p, int splits) { return wino_us(p, splits) < 0.95 * wide_us(p, 185e6); }

hipError_t launch_wino_wgrad(const WgradProblem &p, hipStream_t st) {
  WinoWgradAux q;
  const int B = p.M / (p.Ho * p.Wo);
  q.TW = (p.Wo + 1) / 2, q.TPI = (p.Ho + 1) / 2 * q.TW, q.T = (int)num_tiles(p);
  q.tps = tiles_per_split(q.T, p.splits);
  // short splits of a small problem compete with direct sums that are as short: 32 tiles at a time keep
  // the error below theirs (128 channels, 16 384 pixels: direct 1.09e-7, 64 tiles 1.13e-7, 32 tiles 0.97e-7; 4 us)
  q.period = q.tps <= PERIOD && q.T < 8192 ? PERIOD / 2 : PERIOD;
  q.nq = (p.C + QB - 1) / QB, q.np = (p.P + PB - 1) / PB;
  q.div_tpi = FastDiv(q.TPI), q.div_tw = FastDiv(q.TW);
  q.x_bytes = (uint32_t)((long long)B * p.H * p.W * p.C * 4);
  q.d_bytes = (uint32_t)((long long)p.M * p.P * 4);
  hipLaunchKernelGGL(wino_wgrad_kernel, dim3((unsigned)((long long)q.nq * q.np * p.splits)), dim3(NTHREADS), 0, st, p, q);
  return hipGetLastError();
}

}  // namespace nf
