// 3x3 / stride 1 / pad 1 convolution of more than 24 channels onto more than 32 filters (Eq. 1, NeuroFlux, arXiv 2402.14139) through
// F(2x2, 3x3) (wino_fwd.hip has the algorithm), its 16 contractions over the channels carried out on the bf16 matrix cores: operands and
// transforms are fp32, a transformed value is cut into three bf16 pieces that sum to it exactly (wino_filter.h), and of the nine
// piece products the six largest are accumulated in fp32.  The pieces are rounded to nearest, so that the three left out (2^-25
// of the product each, at most) have no common sign.  Per 16 channels of a 32x32 tile that is 192 cycles of the matrix pipe where fp32
// MFMAs take 512, and six roundings of the running sum where those make eight: the error against 64 bits is the smaller one (emitted
// activation and logits, relative, fp32 MFMAs / this: 64 channels 2.3e-7 / 1.9e-7, 256 4.4e-7 / 3.8e-7, 512 6.5e-7 / 5.7e-7, four layers of
// 128-256 channels in a row 5.2e-7 / 4.9e-7).  Averages over all pixels: bf16 MFMAs do not round their running sum to nearest but, on
// average, down; the positions with row + column odd are therefore formed negated, so that in the sum over a tile's outputs as many
// positions err up as down (512 channels, 8192 pixels 3.9e-8 / 4.0e-8, without it 4.7e-8; 64 to 256 channels equal).
//
// Layout of the work:
//   - a workgroup owns 64 output tiles (256 pixels) x 64 filters x all 16 positions, one per CU; its eight waves take two positions
//     each, half a row of the transformed domain, of all tiles and filters: every transformed patch is formed and cut once, every
//     filter fragment read once, and nothing but the patches passes through LDS;
//   - 16 channels per step.  Patches go from memory straight to LDS, a step ahead (buffer_load ... lds: no registers, no LDS
//     writes to issue); a wave reads the six pixels that its positions combine, forms and cuts them in registers, one group of 32
//     tiles ahead of its MFMAs.  Filters stand in memory as pieces in fragment order;
//   - 128 accumulators and 48 registers of filter fragments per lane, 256 registers in all, two waves per SIMD.
// What bounds it: up to five vector instructions behind an MFMA are free (two waves of such pairs on a SIMD: 68 cycles for two MFMAs
// of 32; six: 76, eight: 87); it needs 5.7, so a step's 3072 cycles of MFMAs are 3500 at best.  It takes 5200 of them, at 1.9 GHz:
// without the filter loads it would be a tenth faster, without the patch loads another.  Workgroups of one wave of the chip do
// not overlap their first loads and last stores: 9 us a launch with 65 536 pixels.
// Measured (us, kernel alone; the same with fp32 MFMAs, 32 tiles, two workgroups per CU / this): 512 -> 512 channels, 4x4, batch 512
// 144 / 100, 256 -> 256, 8x8, 256 82 / 55, 128 -> 128, 16x16, 128 46 / 37, 64 -> 64, 32x32, 64 29.0 / 25.7, 64 -> 128 with 2x2 pooling 51.3 / 43.6.
//
// A value that is not finite makes NaN of others in the transformed domain and of its own pieces: a thread that finds one among its
// results forms those again by the direct sum.
#include <algorithm>

#include "wino_common.h"

namespace nf {
namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));

constexpr int NTHREADS = 512;
constexpr int CH = WINO_CH64;            // channels per step
constexpr int NB = 64;                   // filters per workgroup
constexpr int OOB = (int)0x80000000;     // offset no buffer of < 2 GiB contains
constexpr int RSRC_FLAGS = 0x00020000;   // raw buffer, 32-bit data format

__device__ inline floatx16 mfma(const uint4 &a, const uint4 &b, const floatx16 &c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 16 bytes per lane from the buffer straight to LDS: lane l's go to lds + 16 l, zeros where its offset is out of range.
// The compiler does not know of these loads: the caller waits for them.
__device__ inline void dma16(intx4 rsrc, int voff, int soff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(soff), "s"(lds)
               : "memory");
}

// G: groups of 32 output tiles per workgroup (2; 1 where those would leave compute units idle).  POOL: the 2x2 max pooling of
// Eq. 1 follows in the epilogue.
template <int G, bool POOL>
__global__ __launch_bounds__(NTHREADS, 2) void wino_fwd_split_kernel(FwdProblem p, WinoAux q) {
  constexpr int TB = 32 * G;
  constexpr int PX = TB * CH, BUF = 16 * PX;     // words of a patch pixel, of a step
  constexpr int WS = 32 * 2 * NB;                // epilogue: words of a wave
  constexpr int UP = 2 * 3 * 1024, UB = 16 * UP; // bytes of U per position and per step
  // main loop: As[2][16 patch pixels][2 halves of 8 channels][TB tiles][8 channels], a tile's two 16-byte words at word ^ (tile / 8 % 2):
  // 16 lanes along the tiles read from all banks;
  // epilogue: Cs[8 waves][32 tiles][2 columns][64 filters]
  __shared__ __attribute__((aligned(16))) float S[2 * BUF > 8 * WS ? 2 * BUF : 8 * WS];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int row = wave >> 1, cb = wave & 1;  // positions (row, 2 cb) and (row, 2 cb + 1) of the transformed domain
  const int j = lane & 31, h = lane >> 5;
  // XCD re-map: each XCD gets a contiguous run with the filter blocks fastest, so that the patches of a tile block are read into one
  // L2 only (tile blocks fastest: 512 channels 126 us, 64 -> 128 54.5)
  const int nwg = gridDim.x, lin = blockIdx.x;
  const int wper = nwg >> 3, wrem = nwg & 7, xcd = lin & 7, slot = lin >> 3;
  const int id = xcd < wrem ? xcd * (wper + 1) + slot : wrem * (wper + 1) + (xcd - wrem) * wper + slot;
  const int nb = id % q.nblk, t0 = (id / q.nblk) * TB;
  const int s_lo = blockIdx.y * q.per, s_hi = min(q.nchunks, s_lo + q.per);

  const __amdgpu_buffer_rsrc_t rsu = __builtin_amdgcn_make_buffer_rsrc((void *)q.U, 0, q.u_bytes, RSRC_FLAGS);
  const uintptr_t xa = (uintptr_t)p.x;
  const intx4 rsx = {(int)(uint32_t)xa, (int)(uint32_t)(xa >> 32), (int)q.x_bytes, RSRC_FLAGS};

  // ---- staging: a wave takes pixels 2 wave and 2 wave + 1 of the patches, 32 tiles x 8 channels a load ----
  const int st_c = (lane & 1) ^ (lane >> 4 & 1);  // which four channels of the eight
  int xoff[G][2];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int tile = t0 + g * 32 + (lane >> 1);
    const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
    const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
    const int hi = 2 * ty - 1 + row, wi = 2 * tx - 1 + 2 * cb;
    const bool rok = (tile < q.T) & ((unsigned)hi < (unsigned)p.H);
    const int base = ((img * p.H + hi) * p.W + wi) * p.C * 4 + st_c * 16;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      xoff[g][i] = (base + i * p.C * 4) | ((rok & ((unsigned)(wi + i) < (unsigned)p.W)) ? 0 : OOB);
  }
  // channels past the last one: a whole half of the last step by its offset (a scalar), half of a half by a lane's
  const int tail = p.C % 8 ? p.C / 8 : -1;
  auto last = [&](int s) { return s < s_hi ? s : s_hi - 1; };
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float *)S;
  // load k of 4 G of step s; steps past the end load the last one again, which nothing reads
  auto stage = [&](int s, int buf, int k) {
    const int half = k & 1, i = k >> 1 & 1, g = k >> 2, c8 = 2 * last(s) + half;
    int off = xoff[g][i];
    if (c8 >= p.C / 8) off = (c8 == tail && !st_c) ? off : OOB;
    dma16(rsx, off, c8 * 32, lds0 + (buf * BUF + (2 * wave + i) * PX + half * (PX / 2) + g * 256) * 4);
  };

  // ---- operands ----
  // this wave's row of B^T: t = d[ra] + sg * d[rb]; its columns: t[0] - t[2], t[1] + t[2] | t[2] - t[1], t[1] - t[3], that is
  // t[c0] - t[c1] and t[c1] + sw * t[c2]
  const int ra = row == 0 ? 0 : row == 2 ? 2 : 1, rb = row == 0 ? 2 : row == 1 ? 2 : row == 2 ? 1 : 3;
  const float sg = row == 1 ? 1.f : -1.f, sw = cb ? -1.f : 1.f;
  int at[3][2];  // the bytes where a lane's channels of these pixels stand in the buffer of the patches to be read next
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int col = c == 0 ? (cb ? 2 : 0) : c == 1 ? (cb ? 1 : 2) : (cb ? 3 : 1);
    const int l = j * 8 + (h ^ (j >> 3 & 1)) * 4;
    at[c][0] = ((ra * 4 + col) * PX + l) * 4, at[c][1] = ((rb * 4 + col) * PX + l) * 4;
  }
  auto turn = [&] {
#pragma unroll
    for (int c = 0; c < 3; ++c) at[c][0] ^= BUF * 4, at[c][1] ^= BUF * 4;
  };

  const int ubase = (nb * q.nchunks) * UB + (row * 4 + 2 * cb) * UP + lane * 16;
  uint4 uf[2][2][3];  // [position][filter column][piece]
  auto uload = [&](int s, int b, int n, int k) {
    uf[b][n][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsu, ubase + b * UP + (n * 3 + k) * 1024, last(s) * UB, 0));
  };

  floatx16 acc[2][G][2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[b][g][n][e] = 0.f;

  unsigned pa[3][4], pb[3][4];  // pieces of the two positions' transformed patches: [piece][pair of channels]
  float v0[8], v1[8];           // transformed patches, still whole
  float4 ru[2], rv[2], tv;
  auto lread = [&](float4 (&r)[2], int c, int g, int half) {
#pragma unroll
    for (int k = 0; k < 2; ++k) r[k] = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(S) + at[c][k] + (half * (PX / 2) + g * 256) * 4);
  };
  // the five stages of cutting pair i of v into pieces, in place (wino_split2)
  auto cut = [&](float (&v)[8], unsigned (&o)[3][4], int i, int stage) {
    const bool back = stage & 1;
    if (!back) o[stage >> 1][i] = wino_pack(v[2 * i], v[2 * i + 1]);
    else v[2 * i] -= wino_low(o[stage >> 1][i]), v[2 * i + 1] -= wino_high(o[stage >> 1][i]);
  };
  auto rows = [&](const float4 (&r)[2]) { return fma4(sg, r[1], r[0]); };
  auto put = [&](float (&v)[8], const float4 &x, int half) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[half * 4 + e] = el(x, e);
  };

  // Tile group g of step s: the 24 MFMAs of its two positions, small products first.  Behind each MFMA stands a slice of what
  // the group `gn` that follows needs, four to eight vector instructions, closed by a scheduling fence (left alone the compiler
  // gathers them between the MFMAs): under the first twelve the second position's pieces and half of the next patches, under the
  // others the rest of them and the next first position's pieces.  `reload`: the step's last group, whose filter fragments are
  // loaded again for step s+1 after their last use.  Loads return in order, so that a wait for those is one for the patches sent
  // for before them: `bar`, which frees the buffer for the patches of step s+2, stands in the group before that.
  constexpr int KA[6] = {0, 1, 0, 2, 1, 0}, KB[6] = {2, 1, 1, 0, 0, 0};
  auto frag = [](const unsigned (&o)[3][4], int k) { return make_uint4(o[k][0], o[k][1], o[k][2], o[k][3]); };
  auto bar = [&] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    turn();
  };
  auto group = [&](int g, int gn, bool reload, int s, int buf) {
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const int k = i >> 1, n = i & 1;
      acc[0][g][n] = mfma(frag(pa, KA[k]), uf[0][n][KB[k]], acc[0][g][n]);
      if (G == 1 && i < 4) stage(s + 2, buf, i);
      if (reload && (k == 0 || k == 2 || k == 5)) uload(s + 1, 0, n, KB[k]);
      if (i == 0) lread(ru, 0, gn, 0), lread(rv, 1, gn, 0);
      if (i == 3) tv = rows(rv);
      if (i == 4) lread(rv, 2, gn, 0);
      if (i == 5) ru[0] = rows(ru);
      if (i == 6) put(v0, sub4(ru[0], tv), 0);
      if (i == 9) rv[0] = rows(rv);
      if (i == 11) put(v1, fma4(sw, rv[0], tv), 0);
      if (i % 5 == 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) cut(v1, pb, c, i / 5 * 2);
      } else if (i < 10) {
        cut(v1, pb, i % 5 - 1, i / 5 * 2 + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const int k = i >> 1, n = i & 1;
      acc[1][g][n] = mfma(frag(pb, KA[k]), uf[1][n][KB[k]], acc[1][g][n]);
      if (reload && (k == 0 || k == 2 || k == 5)) uload(s + 1, 1, n, KB[k]);
      if (i == 0) lread(ru, 0, gn, 1), lread(rv, 1, gn, 1), cut(v0, pa, 0, 0), cut(v0, pa, 1, 0);
      if (i == 1) cut(v0, pa, 0, 1);
      if (i == 2) cut(v0, pa, 1, 1);
      if (i == 3) cut(v0, pa, 0, 2), cut(v0, pa, 1, 2), tv = rows(rv), lread(rv, 2, gn, 1);
      if (i == 4) put(v0, sub4(rows(ru), tv), 1);
      if (i == 5) cut(v0, pa, 0, 3), cut(v0, pa, 2, 0), cut(v0, pa, 3, 0);
      if (i == 6) {
        cut(v0, pa, 1, 3);
        if (G == 2 && !reload) bar();
      }
      if (G == 2 && !reload && i > 6)
        for (int d = (i - 7) * 2; d < 8 && d < (i - 6) * 2; ++d) stage(s + 2, buf, d);
      if (i == 7) cut(v0, pa, 0, 4), cut(v0, pa, 1, 4), cut(v0, pa, 2, 1);
      if (i == 8) cut(v0, pa, 3, 1);
      if (i == 9) cut(v0, pa, 2, 2), cut(v0, pa, 3, 2), rv[0] = rows(rv);
      if (i == 10) cut(v0, pa, 2, 3), cut(v0, pa, 3, 3);
      if (i == 11) cut(v0, pa, 2, 4), cut(v0, pa, 3, 4), put(v1, fma4(sw, rv[0], tv), 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- prologue ----
#pragma unroll
  for (int k = 0; k < 4 * G; ++k) stage(s_lo, 0, k);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int n = 0; n < 2; ++n) uload(s_lo, b, n, 2 - k);
#pragma unroll
  for (int k = 0; k < 4 * G; ++k) stage(s_lo + 1, 1, k);
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(4 * G) : "memory");  // all but the last 4 G loads, those of step s_lo+1
  __syncthreads();
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    lread(ru, 0, 0, half), lread(rv, 1, 0, half);
    tv = rows(rv);
    put(v0, sub4(rows(ru), tv), half);
    lread(rv, 2, 0, half);
    put(v1, fma4(sw, rows(rv), tv), half);
  }
#pragma unroll
  for (int st = 0; st < 5; ++st)
#pragma unroll
    for (int c = 0; c < 4; ++c) cut(v0, pa, c, st);

  // At the bar everybody has read the step's patches, so that its buffer takes those of step s+2; those of step s+1, on their
  // way since the last bar, are waited for.
  int buf = 0;
  for (int s = s_lo; s < s_hi; ++s) {
    if constexpr (G == 2) group(0, 1, false, s, buf);
    else bar();
    __builtin_amdgcn_sched_barrier(0);
    group(G - 1, 0, true, s, buf);
    buf ^= 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // what is still on its way to LDS

  // ---- epilogue, a group of 32 tiles at a time: this thread's results are filters n .. n+3 of NT (tile, column) x 2 rows ----
  constexpr int NG = NB / 4, NT = 64 * NG / NTHREADS;
  const bool split = gridDim.y > 1;
  float *const out = p.out + (split ? (long long)blockIdx.y * p.M * p.N : 0ll);
  const int n = nb * NB + (t % NG) * 4;
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  if (p.bias && !split && n < p.N) bias = *reinterpret_cast<const float4 *>(p.bias + n);
  const float *const extra = split ? nullptr : p.addsrc ? p.addsrc : p.mask;
  // (POOL: a thread takes both columns of a tile)
  auto task_of = [&](int i) {
    if constexpr (POOL) return (t / NG) * 2 + i;
    return i * (NTHREADS / NG) + t / NG;
  };  // (tile, column)
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
  long long off[G][NT][2];  // -1: no such pixel or filter
  float4 ex[G][NT][2];      // shortcut or mask: fetched before the transform, so that the loads overlap it
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int task = task_of(i), tile = t0 + 32 * g + (task >> 1);
      const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
      const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
      const int wo = 2 * tx + (task & 1);
      const bool ok = (tile < q.T) & (wo < p.Wo) & (n < p.N);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        off[g][i][k] = (ok & (2 * ty + k < p.Ho)) ? ((long long)(img * p.Ho + 2 * ty + k) * p.Wo + wo) * p.N + n : -1;
        if (extra && off[g][i][k] >= 0) ex[g][i][k] = *reinterpret_cast<const float4 *>(extra + off[g][i][k]);
      }
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int tg = t0 + 32 * g;
    if (tg >= q.T) break;
    // output transform: a wave's part of the columns in registers, the rest through LDS (positions with row + column odd stand
    // negated: the columns here, the rows below)
    __syncthreads();
    {
      float *const cw = S + wave * WS + 2 * j;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = 8 * (e >> 2) + 4 * h + (e & 3);
        float y0[2], y1[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          const float m0 = acc[0][g][f][e], m1 = acc[1][g][f][e];
          y0[f] = cb ? m0 : m0 - m1, y1[f] = cb ? m1 - m0 : -m1;
        }
        *reinterpret_cast<float2 *>(cw + (r * 2 + 0) * NB) = make_float2(y0[0], y0[1]);
        *reinterpret_cast<float2 *>(cw + (r * 2 + 1) * NB) = make_float2(y1[0], y1[1]);
      }
    }
    __syncthreads();
    float4 y[NT][2];
    unsigned bad = 0;  // four bits from 4*(2*i + k): which of those results are not finite
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const float *c = S + task_of(i) * NB + (t % NG) * 4;
      float4 r[4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
        r[a] = add4(*reinterpret_cast<const float4 *>(c + 2 * a * WS), *reinterpret_cast<const float4 *>(c + (2 * a + 1) * WS));
      y[i][0] = add4(sub4(r[0], r[1]), r[2]), y[i][1] = sub4(r[3], add4(r[1], r[2]));
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (off[g][i][k] >= 0) bad |= bad4(y[i][k]) << (4 * (2 * i + k));
    }
    if (bad) {
#pragma unroll 1
      for (int ik = 0; ik < 2 * NT; ++ik) {
        const unsigned want = bad >> (4 * ik) & 15u;
        if (!want) continue;
        const int task = task_of(ik >> 1), tile = tg + (task >> 1);
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
    if constexpr (!POOL) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k)
          if (off[g][i][k] >= 0) *reinterpret_cast<float4 *>(out + off[g][i][k]) = finish(y[i][k], ex[g][i][k], off[g][i][k]);
    } else {
      const int tile = tg + (task_of(0) >> 1);
      const int img = (int)q.div_tpi.div((uint32_t)tile), rem = tile - img * q.TPI;
      const int ty = (int)q.div_tw.div((uint32_t)rem), tx = rem - ty * q.TW;
      if ((tile < q.T) & (ty < p.Hp) & (tx < p.Wp) & (n < p.N)) {  // (all four pixels exist)
        float best[4];
        unsigned at[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) best[e] = -INFINITY, at[e] = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {  // row-major, the first maximum wins
          const float4 v = finish(y[w & 1][w >> 1], ex[g][w & 1][w >> 1], off[g][w & 1][w >> 1]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (el(v, e) > best[e]) best[e] = el(v, e), at[e] = w;
        }
        const long long o = ((long long)(img * p.Hp + ty) * p.Wp + tx) * p.N + n;
        *reinterpret_cast<float4 *>(p.out + o) = make_float4(best[0], best[1], best[2], best[3]);
        *reinterpret_cast<unsigned *>(p.max_arg + o) = at[0] | at[1] << 8 | at[2] << 16 | at[3] << 24;
      }
    }
  }
}

}  // namespace

hipError_t launch_wino_fwd_split(const FwdProblem &p, WinoAux q, int splits, hipStream_t st) {
  int ntb = (q.T + 63) / 64;
  const bool one = wino_fwd_split_small((long long)ntb * q.nblk * splits);
  if (one) ntb = (q.T + 31) / 32;
  const dim3 grid(q.nblk * ntb, splits);
#define NF_LAUNCH(G_, POOL_) hipLaunchKernelGGL((wino_fwd_split_kernel<G_, POOL_>), grid, dim3(NTHREADS), 0, st, p, q)
  if (one && p.max_arg) NF_LAUNCH(1, true);
  else if (one) NF_LAUNCH(1, false);
  else if (p.max_arg) NF_LAUNCH(2, true);
  else NF_LAUNCH(2, false);
#undef NF_LAUNCH
  return hipGetLastError();
}

}  // namespace nf
