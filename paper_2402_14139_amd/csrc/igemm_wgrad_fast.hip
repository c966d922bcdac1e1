// Fast path of the implicit-GEMM weight gradient (see igemm_wgrad.hip for the GEMM view and the
// gradient line of Algorithm 2 it serves; NeuroFlux, arXiv 2402.14139).
//
// Requirements (checked by the launcher): channel counts and P multiples of 4, every operand
// smaller than 2 GiB.  What differs from the general kernel:
//   - all global reads are raw buffer loads with "no data here" (row past the split, tap outside
//     the image, column past P or Q) expressed as an out-of-range offset that the hardware answers
//     with zeros: the gather has no branches;
//   - global loads run two staging steps ahead of the MFMAs (two register sets), LDS fragment
//     reads one sub-step ahead (two fragment slots), one barrier per step;
//   - steps run in unconditional pairs, so the accumulators never leave the MFMA register file;
//   - columns of the 1x1 projection shortcut are fetched by a second load whose result is added
//     (one of the two is always zero), instead of a per-lane branch.
#include <type_traits>

#include "nf_internal.h"
#include "stem_wgrad.h"

namespace nf {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int BKM = 32;  // reduction rows staged per step
constexpr int NTHREADS = 256;
constexpr int OOB = (int)0x80000000;    // offset no buffer of < 2 GiB contains
constexpr int RSRC_FLAGS = 0x00020000;  // raw buffer, 32-bit data format

__device__ inline float4 bload(__amdgpu_buffer_rsrc_t r, int voff) {
  const floatx4 v = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
  return make_float4(v.x, v.y, v.z, v.w);
}

// LDS of a tile: two steps of both operands' rows and of the row table
constexpr int lds_floats(int bp, int bq) { return 2 * BKM * ((bp + 4) + (bq + 4) + 4); }

template <int N>
struct Frag;
template <>
struct Frag<1> {
  static __device__ inline void ld(const float *s, float *v) { v[0] = s[0]; }
};
template <>
struct Frag<2> {
  static __device__ inline void ld(const float *s, float *v) {
    const float2 t = *reinterpret_cast<const float2 *>(s);
    v[0] = t.x, v[1] = t.y;
  }
};
template <>
struct Frag<4> {
  static __device__ inline void ld(const float *s, float *v) {
    const float4 t = *reinterpret_cast<const float4 *>(s);
    v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
  }
};

// BP x BQ output tile, WP x WQ waves, each wave (32*PT) x (32*QT); LDS tiles [m][p], [m][q].
// PROJ 0: no projection columns.  1: a tile may hold taps and projection channels (RSC not a
// multiple of BQ): two loads per row, one of them out of range.  2: RSC is a multiple of BQ, a
// tile is all taps or all projection channels: one load, its source picked per workgroup.
// PM (no projection, channels a multiple of BQ: a tile is one tap): the reduction runs over the output positions whose window
// holds a pixel under that tap, all images of a position after the other; rows of padding are left out, 5 of 9 on 2x2 maps.  A
// split is a range of the rows that remain (a tap at the rim has shorter ones than the one in the centre, which forms the
// bias gradient).  (Padding contributes nothing: an infinite gradient beside it, of which the other tiles make a NaN by inf * 0, is not read.)
template <int BP, int BQ, int WP, int WQ, int PROJ, bool PM>
__device__ __forceinline__ void wgrad_tile(const WgradProblem &p, const PositionRows &q, const TileGrid &grid, int lin,
                                           float *lds) {
  static_assert(!PM || (PROJ == 0 && BP == BQ), "one table entry serves a row of both operands");
  constexpr int TP = BP / WP, TQ = BQ / WQ;
  constexpr int PT = TP / 32, QT = TQ / 32;
  static_assert(WP * WQ == 4 && (PT == 1 || PT == 2 || PT == 4) && (QT == 1 || QT == 2 || QT == 4), "tile");
  constexpr int LDP = BP + 4, LDQ = BQ + 4;
  constexpr int CP = BP / 4, CQ = BQ / 4;                // 16-byte chunks per staged row
  constexpr int RP = NTHREADS / CP, RQ = NTHREADS / CQ;  // rows covered per pass
  constexpr int NP = BKM / RP, NQ = BKM / RQ;            // passes per step
  static_assert(NP >= 1 && NQ >= 1 && RP * NP == BKM && RQ * NQ == BKM, "staging");
  constexpr int NSS = BKM / 4;  // sub-steps per step: two MFMA k-slices (4 reduction rows) each

  static_assert(lds_floats(BP, BQ) == 2 * BKM * (LDP + LDQ + 4), "staged rows and the table");
  float(*const Ds)[BKM][LDP] = reinterpret_cast<float(*)[BKM][LDP]>(lds);
  float(*const Xs)[BKM][LDQ] = reinterpret_cast<float(*)[BKM][LDQ]>(lds + 2 * BKM * LDP);
  int4(*const Rt)[BKM] = reinterpret_cast<int4(*)[BKM]>(lds + 2 * BKM * (LDP + LDQ));

  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int wp = wave / WQ, wq = wave % WQ;
  const int j = lane & 31, h = lane >> 5;
  // Workgroups are handed to the 8 XCDs (each with its own L2) round-robin by linear index.  The
  // index is re-mapped so that each XCD gets a contiguous run of (split, p-tile, q-tile) with the
  // tiles fastest: all tiles of one split read the same rows of D and X, which then come from that
  // XCD's L2 once instead of from every L2.
  const int gx = grid.x, gy = grid.y;
  const int nwg = gx * gy * grid.z;
  const int per = nwg >> 3, rem = nwg & 7, xcd = lin & 7, slot = lin >> 3;
  const int log_id = xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
  const int bx = log_id % gx, byz = log_id / gx, by = byz % gy, bz = byz / gy;
  const int p0 = by * BP, q0 = bx * BQ;
  int m_begin = bz * p.m_per_split;
  int m_end = min(p.M, m_begin + p.m_per_split);

  // D staging: this thread always loads columns p0 + chp*4 .. +3
  const int chp = t % CP, rowp = t / CP;
  const int pcol = p0 + chp * 4;
  // X staging: this thread always loads columns q0 + chq*4 .. +3, i.e. one fixed (r,s,c) or one
  // fixed projection channel
  const int chq = t % CQ, rowq = t / CQ;
  const int qcol = q0 + chq * 4;
  const bool is_tap = qcol < p.RSC, is_proj = PROJ != 0 && !is_tap && qcol < p.Q;
  const bool tile_proj = PROJ == 2 && q0 >= p.RSC;  // uniform
  int qr = 0, qs = 0, qc = 0;
  if (is_tap) {
    const int tap = qcol / p.C;
    qc = qcol - tap * p.C;
    qr = tap / p.S;
    qs = tap - qr * p.S;
  } else {
    qc = qcol - p.RSC;
  }
  // PM: output positions [ho0, ho0 + nh) x [wo0, wo0 + nw) see this tile's tap; rows are (position, image)
  int ho0 = 0, wo0 = 0, nw = 1, magic = 0;
  if constexpr (PM) {
    const int tap = q0 / p.C, tr = tap / p.S, ts = tap - tr * p.S;
    auto from = [&](int t) { return t < p.pad ? (p.pad - t + p.stride - 1) / p.stride : 0; };  // first output inside
    auto to = [&](int t, int in, int out) { return max(0, min(out, (in + p.pad - t + p.stride - 1) / p.stride)); };
    ho0 = from(tr), wo0 = from(ts);
    const int nh = max(0, to(tr, p.H, p.Ho) - ho0);
    nw = max(0, to(ts, p.W, p.Wo) - wo0);
    const int rows = nh * nw * (int)q.div_imgs.d;
    const int per = ((rows + grid.z - 1) / grid.z + BKM - 1) / BKM * BKM;
    m_begin = bz * per, m_end = min(rows, m_begin + per);
    magic = nw ? 65535 / nw + 1 : 0;  // i * magic >> 16 = i / nw for i, nw <= 64
  }
  const int dcol_off = pcol < p.P ? pcol * 4 : OOB;  // byte offset of this thread's D columns
  const int xtap_off = ((qr * p.W + qs) * p.C + qc) * 4;

  const __amdgpu_buffer_rsrc_t rsd = __builtin_amdgcn_make_buffer_rsrc((void *)p.d, 0, p.d_bytes, RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, p.x_bytes, RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t rsxs = __builtin_amdgcn_make_buffer_rsrc((void *)p.xs, 0, p.xs_bytes, RSRC_FLAGS);
  // PROJ == 2: the one source of this workgroup's X columns
  const __amdgpu_buffer_rsrc_t rs_sel = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(tile_proj ? p.xs : p.x), 0, tile_proj ? p.xs_bytes : p.x_bytes, RSRC_FLAGS);
  const int proj_mask = tile_proj ? -1 : 0;

  float4 rd[2][NP], rx[2][NQ];
  float4 bsum = make_float4(0.f, 0.f, 0.f, 0.f);
  const bool do_bias = (bx == (PM ? q.bias_tile : 0)) && (p.part_b != nullptr);
  const float bsel = do_bias ? 1.f : 0.f;

  // Row table: entry r of Rt[s & 1] describes reduction row m_begin + 32*s + r of staging step s:
  // {byte offset of its receptive field's corner in x, hi0, wi0, byte offset of its pixel in the
  // projection input}; hi0 is far negative for rows past the split.  Every thread decodes ONE row
  // per step (threads with equal t & 31 write the same entry) instead of its NQ rows.
  auto rt_make = [&](int s) {
    const int m = m_begin + s * BKM + (t & (BKM - 1));
    if constexpr (PM) {  // {offset in x, -, -, offset in d}
      const int at = (int)q.div_imgs.div((uint32_t)m), img = m - at * (int)q.div_imgs.d, r = (at * magic) >> 16;
      const int ho = ho0 + r, wo = wo0 + at - r * nw;
      const int bad = m < m_end ? 0 : OOB;
      const int xo = ((img * p.H + ho * p.stride - p.pad) * p.W + wo * p.stride - p.pad) * p.C * 4;
      Rt[s & 1][t & (BKM - 1)] = make_int4(bad ? OOB : xo, 0, 0, (((img * p.Ho + ho) * p.Wo + wo) * p.P * 4) | bad);
      return;
    }
    const int img = (int)p.div_howo.div((uint32_t)m);
    const int rem = m - img * p.Ho * p.Wo;
    const int ho = (int)p.div_wo.div((uint32_t)rem);
    const int wo = rem - ho * p.Wo;
    const int hi0 = ho * p.stride - p.pad, wi0 = wo * p.stride - p.pad;
    int4 e;
    e.x = ((img * p.H + hi0) * p.W + wi0) * p.C * 4;
    e.y = m < m_end ? hi0 : -(1 << 20);
    e.z = wi0;
    e.w = PROJ != 0 ? ((img * p.Hs + ho * p.ss) * p.Ws + wo * p.ss) * p.Cs * 4 : 0;
    Rt[s & 1][t & (BKM - 1)] = e;
  };

  // Branch-free gather of staging step `s` into register set `set` (the X rows go by the table entries
  // tread(s) fetched from Rt[s & 1]), one staged row per call so that the step can place the loads
  // between its MFMAs.
  int4 te[NQ];  // this thread's table entries of the step being loaded
  auto gload_d = [&](int s, int set, int i) {
    if constexpr (PM) {
      rd[set][i] = bload(rsd, (te[i].w + pcol * 4) | (pcol < p.P ? 0 : OOB));
      return;
    }
    const int m = m_begin + s * BKM + rowp + RP * i;
    const bool ok = (m < m_end) & (dcol_off != OOB);
    rd[set][i] = bload(rsd, (m * p.P * 4 + dcol_off) | (ok ? 0 : OOB));
  };
  auto tread = [&](int s) {
#pragma unroll
    for (int i = 0; i < NQ; ++i) te[i] = Rt[s & 1][rowq + RQ * i];
  };
  auto gload_x = [&](int set, int i) {
    const int4 e = te[i];
    if constexpr (PM) {  // (every column is a tap's: an offset of OOB and more stays out of range)
      rx[set][i] = bload(rsx, e.x + xtap_off);
      return;
    }
    const bool ok = is_tap & ((unsigned)(e.y + qr) < (unsigned)p.H) & ((unsigned)(e.z + qs) < (unsigned)p.W);
    // the offset is formed unconditionally and pushed out of range by its top bit: a select would
    // let the compiler sink the table read into a branch
    float4 v;
    if constexpr (PROJ == 2) {
      // bit selects with the workgroup-uniform mask: a ?: here would be turned into branches
      const int okp = (is_proj & (e.y > -(1 << 19))) ? 0 : OOB, okt = ok ? 0 : OOB;
      const int off = (((e.w + qc * 4) | okp) & proj_mask) | (((e.x + xtap_off) | okt) & ~proj_mask);
      v = bload(rs_sel, off);
    } else {
      v = bload(rsx, (e.x + xtap_off) | (ok ? 0 : OOB));
      if constexpr (PROJ == 1) {
        const bool okp = is_proj & (e.y > -(1 << 19));
        const float4 u = bload(rsxs, (e.w + qc * 4) | (okp ? 0 : OOB));
        v.x += u.x, v.y += u.y, v.z += u.z, v.w += u.w;  // one of the two is all zeros
      }
    }
    rx[set][i] = v;
  };
  auto gload = [&](int s, int set) {
    if (PM) tread(s);
#pragma unroll
    for (int i = 0; i < NP; ++i) gload_d(s, set, i);
    if (!PM) tread(s);
#pragma unroll
    for (int i = 0; i < NQ; ++i) gload_x(set, i);
  };

  auto lstore_d = [&](int buf, int set, int i) {
    *reinterpret_cast<float4 *>(&Ds[buf][rowp + RP * i][chp * 4]) = rd[set][i];
    bsum.x += bsel * rd[set][i].x, bsum.y += bsel * rd[set][i].y, bsum.z += bsel * rd[set][i].z,
        bsum.w += bsel * rd[set][i].w;
  };
  auto lstore_x = [&](int buf, int set, int i) {
    *reinterpret_cast<float4 *>(&Xs[buf][rowq + RQ * i][chq * 4]) = rx[set][i];
  };
  auto lstore = [&](int buf, int set) {
#pragma unroll
    for (int i = 0; i < NP; ++i) lstore_d(buf, set, i);
#pragma unroll
    for (int i = 0; i < NQ; ++i) lstore_x(buf, set, i);
  };

  floatx16 acc[PT][QT];
#pragma unroll
  for (int a = 0; a < PT; ++a)
#pragma unroll
    for (int b = 0; b < QT; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;

  // fragments of one sub-step: two k-slices (rows 4*ss + 2*k2 + h), PT / QT consecutive columns
  float df[2][2][PT], xf[2][2][QT];
  auto lfrag = [&](int buf, int ss, int slot) {
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      Frag<PT>::ld(&Ds[buf][4 * ss + 2 * k2 + h][wp * TP + PT * j], df[slot][k2]);
      Frag<QT>::ld(&Xs[buf][4 * ss + 2 * k2 + h][wq * TQ + QT * j], xf[slot][k2]);
    }
  };
  auto mma = [&](int slot) {
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
      for (int a = 0; a < PT; ++a)
#pragma unroll
        for (int b = 0; b < QT; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(df[slot][k2][a], xf[slot][k2][b], acc[a][b], 0, 0, 0);
  };

  // ---- software pipeline: step s uses LDS buffer s&1 ----
  //   sub-steps 0..NSS-2: fragment reads of sub-step ss+1 ride on the MFMAs of sub-step ss; the
  //     address arithmetic and buffer loads of step s+2 are spread over the first four sub-steps,
  //     the LDS writes of step s+1 (loaded one step ago) over the next three;
  //   barrier; first fragments of step s+1; MFMAs of the last sub-step.
  // Every sub-step is closed by a scheduling fence: without it the compiler moves fragment reads
  // between sub-steps and some end up right in front of the MFMA that needs them.
  constexpr int NM = 2 * PT * QT;  // MFMAs per sub-step
  constexpr int NW = NP + NQ;      // staged rows per thread and step (buffer loads, LDS writes)
  constexpr int LPS = (NW + 3) / 4;  // rows loaded per sub-step over sub-steps 0..3
  constexpr int WPS = (NW + 2) / 3;  // rows written per sub-step over sub-steps 4..6
  static_assert(NSS == 8, "placement of loads and writes");
  auto step = [&](int s, auto par_tag) {
    constexpr int par = decltype(par_tag)::value;
#pragma unroll
    for (int ss = 0; ss + 1 < NSS; ++ss) {
      lfrag(par, ss + 1, (ss + 1) & 1);
      mma(ss & 1);
      if (ss == 0) {
        tread(s + 2);     // table entries a sub-step or more ahead of the loads that need them
        rt_make(s + 3);   // the other table buffer
      }
      if (ss < 4) {                 // step s + 2 into set `par`, which held step s, already in LDS
#pragma unroll
        for (int it = ss * LPS; it < (ss + 1) * LPS && it < NW; ++it) {
          if (it < NP) gload_d(s + 2, par, it);
          else gload_x(par, it - NP);
        }
      } else {                      // step s + 1
#pragma unroll
        for (int it = (ss - 4) * WPS; it < (ss - 3) * WPS && it < NW; ++it) {
          if (it < NP) lstore_d(par ^ 1, par ^ 1, it);
          else lstore_x(par ^ 1, par ^ 1, it - NP);
        }
      }
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                          // one MFMA
        if (i < 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);              // + fragment reads
        if (ss < 4) __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);             // + address VALU
        if (ss < 4 && i < 2 * LPS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // + a buffer load
        if (ss >= 4 && i < WPS) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0); // + an LDS write
        if (ss >= 4) __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    lfrag(par ^ 1, 0, 0);
    mma((NSS - 1) & 1);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
      if (i < 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
    }
  };

  const int nsteps = max(0, m_end - m_begin + BKM - 1) / BKM;
  rt_make(0);
  rt_make(1);
  __syncthreads();
  gload(0, 0);
  lstore(0, 0);
  gload(1, 1);
  __syncthreads();  // table reads done
  rt_make(2);
  __syncthreads();
  lfrag(0, 0, 0);
  // unconditional pairs inside the loop (a conditional second step there makes the compiler move the
  // accumulators out of and back into the MFMA register file around every iteration); an odd count
  // ends with one step after the loop
  int s = 0;
  for (; s + 1 < nsteps; s += 2) {
    step(s, std::integral_constant<int, 0>{});
    step(s + 1, std::integral_constant<int, 1>{});
  }
  if (nsteps & 1) step(s, std::integral_constant<int, 0>{});

  // ---- store the partial tile: lane holds, per (a, e), QT consecutive q ----
  float *part = p.part + (long long)bz * p.P * p.Qld;
#pragma unroll
  for (int a = 0; a < PT; ++a) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = 8 * (e >> 2) + 4 * h + (e & 3);
      const int pr = p0 + wp * TP + PT * r + a;
      if (pr >= p.P) continue;
#pragma unroll
      for (int b = 0; b < QT; ++b) {
        const int q = q0 + wq * TQ + QT * j + b;
        if (q < p.Q) part[(long long)pr * p.Qld + q] = acc[a][b][e];
      }
    }
  }

  // ---- bias-gradient partials: sum the per-thread column sums over the RP staging rows ----
  if (do_bias) {  // uniform per workgroup
    __syncthreads();
    float *red = &Ds[0][0][0];  // reuse: [RP][BP]
    *reinterpret_cast<float4 *>(&red[rowp * BP + chp * 4]) = bsum;
    __syncthreads();
    if (t < BP && p0 + t < p.P) {
      float s = 0.f;
      for (int r = 0; r < RP; ++r) s += red[r * BP + t];
      p.part_b[(long long)bz * p.P + p0 + t] = s;
    }
  }
}

template <int BP, int BQ, int WP, int WQ, int PROJ, bool PM>
__global__ __launch_bounds__(NTHREADS, 2) void igemm_wgrad_fast_kernel(WgradProblem p, PositionRows q) {
  __shared__ __attribute__((aligned(16))) float lds[lds_floats(BP, BQ)];
  const TileGrid grid = {(int)gridDim.x, (int)gridDim.y, (int)gridDim.z};
  wgrad_tile<BP, BQ, WP, WQ, PROJ, PM>(p, q, grid, blockIdx.x + grid.x * (blockIdx.y + grid.y * blockIdx.z), lds);
}

// ---- a head's weight gradient and its layer's in one launch ----
// Both wait for the head (the layer's for the data gradient, too) and neither reads what the other writes.  In launches of their
// own each ramps up and drains a chip that it often leaves partly idle (a batch of small images: 1-100 workgroups of 7-14 us, 4-5 us of
// gap after each).  The layer's workgroups come first, the head's fill in beside and behind them: the same tiles, splits and sums.
// One kernel per pair of variants: each tile's loop is compiled as in its own kernel, and LDS and registers are the larger
// of two.  (One kernel that branches over all variants had 20-25 % more vector instructions in its loops, and three workgroups on a CU
// where these have four: 8 images of 32x32, 3 -> 16 channels, 41.6 us a step, but 3 -> 64 channels, 128 images 293.)  A step, two launches /
// one, us: 8 images 47.1 / 41.0; 512 -> 512 channels on 2x2 maps, 512 images, 64-wide head 166.3 / 156.5, batch 128, 256-wide head
// 139.3 / 133; 96 -> 48 channels, 5x5, 32x32, 64 images 448 / 437.
enum Form { F64, F64_POS, F32, F64_PROJ, F_STEM, F_NONE };  // 64x64, 32x128 (by PROJ, PM), stem_wgrad; a head's are the first three

constexpr int form_lds(int form) {
  return form == F_STEM ? STEM_WGRAD_LDS : form == F32 ? lds_floats(32, 128) : lds_floats(64, 64);
}
template <int FORM>
__device__ __forceinline__ void form_tile(const WgradProblem &p, const PositionRows &q, const TileGrid &g, int lin, float *lds) {
  if constexpr (FORM == F64) wgrad_tile<64, 64, 2, 2, 0, false>(p, q, g, lin, lds);
  if constexpr (FORM == F64_POS) wgrad_tile<64, 64, 2, 2, 0, true>(p, q, g, lin, lds);
  if constexpr (FORM == F32) wgrad_tile<32, 128, 1, 4, 0, false>(p, q, g, lin, lds);
  if constexpr (FORM == F64_PROJ) wgrad_tile<64, 64, 2, 2, 2, false>(p, q, g, lin, lds);
  if constexpr (FORM == F_STEM) stem_wgrad_tile<true>(p, lin % g.y, lin / g.y, lds);
}
template <int LAYER, int HEAD>
__global__ __launch_bounds__(NTHREADS, 2) void wgrad_pair_kernel(WgradPair a) {
  constexpr int FL = form_lds(LAYER), FH = form_lds(HEAD);
  __shared__ __attribute__((aligned(16))) float lds[FL > FH ? FL : FH];
  const int lin = blockIdx.x;
  if (lin >= a.head_at)
    form_tile<HEAD>(a.p[1], a.q[1], a.grid[1], lin - a.head_at, lds);
  else if (lin < a.grid[0].x * a.grid[0].y * a.grid[0].z)
    form_tile<LAYER>(a.p[0], a.q[0], a.grid[0], lin, lds);
}

void fill_bytes(WgradProblem *p) {
  const long long B = p->M / ((long long)p->Ho * p->Wo);
  p->d_bytes = (uint32_t)((long long)p->M * p->P * 4);
  p->x_bytes = (uint32_t)(B * p->H * p->W * p->C * 4);
  p->xs_bytes = p->Cs ? (uint32_t)(B * p->Hs * p->Ws * p->Cs * 4) : 0;
}

// Whether the rows of padding are left out (PM): at most 85 of 100 remain, and some tap sees every position.  Measured (us,
// with all rows / without), 128 images on 2x2 maps (4 of 9 remain): 512x4608 in three splits 34.4 / 24.4, 256x4608 in four 20.0 / 13.9.
bool position_rows(const WgradProblem &p, int bq, PositionRows *q) {
  if (p.Cs || p.C % bq || p.R * p.S == 1 || p.Ho * p.Wo > 64) return false;
  int all_r = -1, all_s = -1;
  auto inside = [&](int out, int in, int taps, int *all) {  // (output, tap) pairs inside the image, one direction
    int n = 0;
    for (int t = 0; t < taps; ++t) {
      int c = 0;
      for (int o = 0; o < out; ++o) c += (unsigned)(o * p.stride - p.pad + t) < (unsigned)in;
      if (c == out) *all = t;
      n += c;
    }
    return n;
  };
  const int nr = inside(p.Ho, p.H, p.R, &all_r), ns = inside(p.Wo, p.W, p.S, &all_s);
  if (all_r < 0 || all_s < 0) return false;
  q->div_imgs = FastDiv(p.M / (p.Ho * p.Wo)), q->bias_tile = (all_r * p.S + all_s) * (p.C / bq);
  return 100ll * nr * ns <= 85ll * p.Ho * p.Wo * p.R * p.S;
}

// which of a pair's variants serves a problem (F_NONE: another kernel), and its grid
int pair_form(WgradProblem *p, PositionRows *q, TileGrid *g) {
  q->bias_tile = 0;
  if (igemm_wgrad_small_applicable(*p)) return F_NONE;
  if (igemm_wgrad_fast_applicable(*p)) {
    if (contraction_mode() != NF_CONTRACT_F32 && igemm_wgrad_split_applicable(*p)) return F_NONE;
    if (p->P > 64 && !igemm_wgrad_tile64(p->P, p->Q, p->splits)) return F_NONE;
    const bool narrow = p->P <= 32;
    const int bp = narrow ? 32 : 64, bq = narrow ? 128 : 64;
    if (p->Cs && (narrow || p->RSC % bq)) return F_NONE;
    fill_bytes(p);
    *g = {(p->Q + bq - 1) / bq, (p->P + bp - 1) / bp, p->splits};
    return narrow ? F32 : position_rows(*p, bq, q) ? F64_POS : p->Cs ? F64_PROJ : F64;
  }
  if (!stem_wgrad_applicable(*p) || p->P % 4) return F_NONE;
  *g = {1, (p->P + 63) / 64, p->splits};
  return F_STEM;
}

long long tiles(const TileGrid &g) { return (long long)g.x * g.y * g.z; }

typedef void (*PairKernel)(WgradPair);
template <int LAYER>
PairKernel pair_kernel_of(int head) {
  return head == F64       ? wgrad_pair_kernel<LAYER, F64>
         : head == F64_POS ? wgrad_pair_kernel<LAYER, F64_POS>
         : head == F32     ? wgrad_pair_kernel<LAYER, F32>
                           : nullptr;
}

const char *pair_name(int layer, int head) {
#define NF_NAMES(L) {"igemm_wgrad_pair_" L "_64x64", "igemm_wgrad_pair_" L "_64x64_rows", "igemm_wgrad_pair_" L "_32x128"}
  static const char *const names[F_NONE][3] = {NF_NAMES("64x64"), NF_NAMES("64x64_rows"), NF_NAMES("32x128"),
                                               NF_NAMES("64x64_proj"), NF_NAMES("stem")};
#undef NF_NAMES
  return names[layer][head];
}

PairKernel make_pair(const WgradProblem &layer, const WgradProblem &head, WgradPair *a, const char **name) {
  a->p[0] = layer, a->p[1] = head;
  const int fl = pair_form(&a->p[0], &a->q[0], &a->grid[0]), fh = pair_form(&a->p[1], &a->q[1], &a->grid[1]);
  if (fl == F_NONE || fh > F32) return nullptr;
  a->head_at = (int)((tiles(a->grid[0]) + 7) / 8 * 8);
  // Of 64x64 tiles four reside on a CU, of the others (LDS, registers) three, and so of a pair that holds one.  A pair of those
  // that leaves a small second round of long tiles is no faster than two launches (step, us, two / one: 1020 workgroups of 14.5 GFLOP
  // 359 / 372, 1022 of 2.6 121.7 / 131.3, 1024 of 1.2 102.2 / 105.6, but 867 of 1.1 79.7 / 77.0, 1122 of 0.6 79.2 / 75.0).  Of
  // 82 random pairs all others gained, 2-11 us.
  const bool three = fl == F32 || fl == F64_PROJ || fh == F32;
  const double flops = 2.0 * ((double)layer.M * layer.P * layer.Q + (double)head.M * head.P * head.Q);
  if (three && tiles(a->grid[0]) + tiles(a->grid[1]) > 3 * 256 && flops > 1e9) return nullptr;
  *name = pair_name(fl, fh);
  return fl == F64       ? pair_kernel_of<F64>(fh)
         : fl == F64_POS ? pair_kernel_of<F64_POS>(fh)
         : fl == F32     ? pair_kernel_of<F32>(fh)
         : fl == F_STEM  ? pair_kernel_of<F_STEM>(fh)
                         : pair_kernel_of<F64_PROJ>(fh);
}

template <int BP, int BQ, int WP, int WQ>
hipError_t launch_cfg(const WgradProblem &p, hipStream_t st) {
  dim3 grid((p.Q + BQ - 1) / BQ, (p.P + BP - 1) / BP, p.splits);
  PositionRows q;
  q.bias_tile = 0;
  if constexpr (BP == BQ) {
    if (position_rows(p, BQ, &q)) {
      hipLaunchKernelGGL((igemm_wgrad_fast_kernel<BP, BQ, WP, WQ, 0, true>), grid, dim3(NTHREADS), 0, st, p, q);
      return hipGetLastError();
    }
  }
  if (p.Cs && p.RSC % BQ == 0)
    hipLaunchKernelGGL((igemm_wgrad_fast_kernel<BP, BQ, WP, WQ, 2, false>), grid, dim3(NTHREADS), 0, st, p, q);
  else if (p.Cs)
    hipLaunchKernelGGL((igemm_wgrad_fast_kernel<BP, BQ, WP, WQ, 1, false>), grid, dim3(NTHREADS), 0, st, p, q);
  else
    hipLaunchKernelGGL((igemm_wgrad_fast_kernel<BP, BQ, WP, WQ, 0, false>), grid, dim3(NTHREADS), 0, st, p, q);
  return hipGetLastError();
}

}  // namespace

bool igemm_wgrad_fast_applicable(const WgradProblem &p) {
  const long long lim = 0x7FFFFFF0ll, B = p.M / ((long long)p.Ho * p.Wo);
  if (p.C % 4 || p.Cs % 4 || p.P % 4) return false;
  if ((long long)p.M * p.P * 4 > lim || B * p.H * p.W * p.C * 4 > lim) return false;
  if (p.Cs && B * p.Hs * p.Ws * p.Cs * 4 > lim) return false;
  return true;
}

// 64x64 tiles (the same sums in the same order) where the 128x128 ones, two per CU, leave an eighth of the chip or
// more without work in their rounds, or pad the result by more than a tenth.  Measured, us, 128x128 / 64x64
// (workgroups of the former): 512x4608 over 256 rows (288) 31.0 / 24.5, 512 rows (432) 36.0 / 34.2, 128x1152 over 4096
// (288) 30.8 / 23.4, 256x256 over 2048 (64) 17.8 / 10.0; 160x4800 over 12 544 258 / 211; but 384x6400 over 288 (450)
// 26.8 / 27.3, 512x2304 over 1024 (504) 32.3 / 33.2, over 32 768 (504) 591 / 640.
bool igemm_wgrad_tile64(int P, int Q, int splits) {
  const auto up = [](long long n, long long m) { return (n + m - 1) / m; };
  const long long w = up(P, 128) * up(Q, 128) * splits, rounds = up(w, 512);
  return 8 * w < 7 * 512 * rounds || 10 * up(P, 64) * up(Q, 64) < 9 * 4 * up(P, 128) * up(Q, 128);
}

hipError_t launch_igemm_wgrad_fast(const WgradProblem &p0, hipStream_t st, const char **kernel) {
  if (contraction_mode() != NF_CONTRACT_F32 && igemm_wgrad_split_applicable(p0))
    return launch_igemm_wgrad_split(p0, contraction_mode() == NF_CONTRACT_BF16X9, st, kernel);
  WgradProblem p = p0;
  fill_bytes(&p);
  if (p.P > 64 && !igemm_wgrad_tile64(p.P, p.Q, p.splits)) {
    *kernel = "igemm_wgrad_fast_128x128";
    return launch_cfg<128, 128, 2, 2>(p, st);
  }
  if (p.P > 32) {
    *kernel = "igemm_wgrad_fast_64x64";
    return launch_cfg<64, 64, 2, 2>(p, st);
  }
  *kernel = "igemm_wgrad_fast_32x128";
  return launch_cfg<32, 128, 1, 4>(p, st);
}

WgradPairPlan plan_wgrad_pair(const WgradProblem &layer, const WgradProblem &head) {
  WgradPairPlan plan;
  plan.kernel = make_pair(layer, head, &plan.args, &plan.name);
  return plan;
}

hipError_t launch_wgrad_pair(const WgradPairPlan &plan, hipStream_t st) {
  const WgradPair &a = plan.args;
  hipLaunchKernelGGL(plan.kernel, dim3((unsigned)(a.head_at + tiles(a.grid[1]))), dim3(NTHREADS), 0, st, a);
  return hipGetLastError();
}

}  // namespace nf
