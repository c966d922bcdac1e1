// The auxiliary head after its convolution (NeuroFlux, arXiv 2402.14139, Eq. 2 and Eq. 3):
// adaptive average (or max) pooling F_n, the linear layer gamma_n, softmax cross-entropy (or
// mean squared error against the one-hot label) with the batch mean, and the backward of those
// three (gradient line of Algorithm 2).
// These steps are tiny next to the convolutions; they are written as fused wavefront /
// workgroup reductions with a fixed summation order (deterministic).
#include <algorithm>

#include "head_gamma.h"
#include "nf_internal.h"
#include "wino_filter.h"

namespace nf {
namespace {

constexpr int HT = 256;  // threads per workgroup in this file
static_assert(HT == GJ_T, "the batch-reducing jobs assume this workgroup size");

__device__ inline void adaptive_window(int i, int L, int O, int &lo, int &hi) {
  lo = (i * L) / O;
  hi = ((i + 1) * L + O - 1) / O;
}

// 1 / elements of the window that pooled feature f averages; 1 for max pooling
__device__ inline float pool_scale(const HeadShape &s, int f) {
  if (s.scale != 0.f) return s.scale;  // the same for all
  const int cell = (int)s.div_a.div((uint32_t)f), ci = (int)s.div_ow.div((uint32_t)cell), cj = cell - ci * s.ow;
  const int h0 = (int)s.div_oh.div((uint32_t)(ci * s.Hu)), h1 = (int)s.div_oh.div((uint32_t)((ci + 1) * s.Hu + s.oh - 1));
  const int w0 = (int)s.div_ow.div((uint32_t)(cj * s.Wu)), w1 = (int)s.div_ow.div((uint32_t)((cj + 1) * s.Wu + s.ow - 1));
  return 1.f / (float)((h1 - h0) * (w1 - w0));
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// V consecutive floats: channels of one element of the head's activation, features of a row of Wf
template <int V>
struct Chan {
  float v[V];
};
template <int V>
__device__ inline Chan<V> load_chan(const float *__restrict__ at) {
  Chan<V> c;
  if constexpr (V == 4) {
    const float4 x = *reinterpret_cast<const float4 *>(at);
    c.v[0] = x.x, c.v[1] = x.y, c.v[2] = x.z, c.v[3] = x.w;
  } else {
    c.v[0] = at[0];
  }
  return c;
}

// F_n: adaptive average pool (PMAX: adaptive max pool, which also records the flat position
// h*Wu+w of the first maximal element in row-major window order).  A workgroup serves G (sample,
// output cell) pairs; each pair has CA channel lanes (V channels each, 16-byte accesses when
// V == 4) x NS window-position slices, CA * NS * G = HT.  Slice results are combined in order
// through LDS.
// With splits > 0 the aux activation does not exist yet: it is formed here from the raw partial
// sums of the split aux convolution, U = act(sum_z part[z] + ba), and written out on the way.
// (all threads of a workgroup; pairs [pair0, pair0 + G) below pair_end; red / redi: HT*V entries of
// LDS; pq_lds / parg_lds, when given, also receive the results at index (pair - lds_pair0) * A + channel)
template <int V, bool PMAX>
__device__ inline void pool_pairs(const HeadShape &s, long long pair0, long long pair_end, float *__restrict__ U,
                                  const float *__restrict__ part, int splits, const float *__restrict__ ba,
                                  float *__restrict__ Pq, int32_t *__restrict__ parg, int CA, int NS, float *red,
                                  int *redi, float *pq_lds, int *parg_lds, long long lds_pair0) {
  const int t = threadIdx.x;
  const int per = CA * NS, G = HT / per;
  const int grp = t / per, tg = t - grp * per;
  const int lane = tg % CA, slice = tg / CA;
  const int cells = s.oh * s.ow;
  const long long pair = pair0 + grp;
  const bool live = grp < G && pair < pair_end;
  const int n = live ? (int)(pair / cells) : 0, cell = live ? (int)(pair - (long long)n * cells) : 0;
  const int ci = cell / s.ow, cj = cell - ci * s.ow;
  int h0, h1, w0, w1;
  adaptive_window(ci, s.Hu, s.oh, h0, h1);
  adaptive_window(cj, s.Wu, s.ow, w0, w1);
  const int ww = w1 - w0, npos = (h1 - h0) * ww;
  const int AV = s.A / V;
  const float inv = 1.f / (float)npos;
  const long long total = (long long)s.B * s.Hu * s.Wu * s.A;
  for (int c0 = 0; c0 < AV; c0 += CA) {
    const int col = c0 + lane;
    float acc[V];
    int bpos[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = PMAX ? -INFINITY : 0.f, bpos[e] = 0x7fffffff;
    if (live && col < AV) {
      float bias[V];
#pragma unroll
      for (int e = 0; e < V; ++e) bias[e] = (splits > 0 && ba) ? ba[col * V + e] : 0.f;
#pragma unroll 4
      for (int pos = slice; pos < npos; pos += NS) {
        const int hh = h0 + pos / ww, wx = w0 + pos % ww;
        const long long at = (((long long)n * s.Hu + hh) * s.Wu + wx) * s.A + col * V;
        float v[V];
        if (splits > 0) {
#pragma unroll
          for (int e = 0; e < V; ++e) v[e] = 0.f;
          for (int z = 0; z < splits; ++z) {
            const float *src = part + (long long)z * total + at;
            if constexpr (V == 4) {
              const float4 x = *reinterpret_cast<const float4 *>(src);
              v[0] += x.x, v[1] += x.y, v[2] += x.z, v[3] += x.w;
            } else {
              v[0] += src[0];
            }
          }
#pragma unroll
          for (int e = 0; e < V; ++e) {
            v[e] += bias[e];
            if (s.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
          }
          if constexpr (V == 4) {
            *reinterpret_cast<float4 *>(U + at) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
            U[at] = v[0];
          }
        } else {
          if constexpr (V == 4) {
            const float4 x = *reinterpret_cast<const float4 *>(U + at);
            v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
          } else {
            v[0] = U[at];
          }
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
          if constexpr (PMAX) {
            if (v[e] > acc[e]) acc[e] = v[e], bpos[e] = hh * s.Wu + wx;  // strict: first maximum of the slice
          } else {
            acc[e] += v[e];
          }
        }
      }
    }
    __syncthreads();  // previous round's reads of red are done
#pragma unroll
    for (int e = 0; e < V; ++e) {
      red[t * V + e] = acc[e];
      if constexpr (PMAX) redi[t * V + e] = bpos[e];
    }
    // the NS slices (a power of two) pairwise, a fixed tree: log2 NS dependent LDS reads instead of NS - 1
    // (head_pool, max pooling of 14x13 maps of 12 channels, batch 33: 14.9 -> 5.7 us)
    for (int half = NS >> 1; half > 0; half >>= 1) {
      __syncthreads();
      if (slice < half) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const int at = (t + half * CA) * V + e;
          const float cv = red[at];
          if constexpr (PMAX) {
            const int cp = redi[at];
            if (cv > acc[e] || (cv == acc[e] && cp < bpos[e])) acc[e] = cv, bpos[e] = cp;  // ties: earliest position
            redi[t * V + e] = bpos[e];
          } else {
            acc[e] += cv;
          }
          red[t * V + e] = acc[e];
        }
      }
    }
    if (live && slice == 0 && col < AV) {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const long long o = (long long)n * s.F + cell * s.A + col * V + e;
        const int li = (int)(pair - lds_pair0) * s.A + col * V + e;
        if constexpr (PMAX) {
          Pq[o] = acc[e];
          parg[o] = bpos[e];
          if (pq_lds) pq_lds[li] = acc[e], parg_lds[li] = bpos[e];
        } else {
          Pq[o] = acc[e] * inv;
          if (pq_lds) pq_lds[li] = acc[e] * inv;
        }
      }
    }
  }
}

template <int V, bool PMAX>
__global__ __launch_bounds__(HT) void head_pool_kernel(HeadShape s, float *__restrict__ U,
                                                       const float *__restrict__ part, int splits,
                                                       const float *__restrict__ ba, float *__restrict__ Pq,
                                                       int32_t *__restrict__ parg, int CA, int NS) {
  __shared__ float red[HT * V];
  __shared__ int redi[PMAX ? HT * V : 1];
  const int G = HT / (CA * NS);
  pool_pairs<V, PMAX>(s, (long long)blockIdx.x * G, (long long)s.B * s.oh * s.ow, U, part, splits, ba, Pq, parg, CA, NS,
                      red, redi, nullptr, nullptr, 0);
}

// Logits of one sample (all threads of a workgroup): z[q] = bf[q] + sum_f Wf[q][f] * pq[f], pq staged in LDS; ends
// with a barrier.  8 lanes per class with eight running sums each,
// added in a tree, so that a result is 64 sums of F / 64 products (relative error against 64 bits, 1024 features, 100
// classes: 1.0e-7; with two sums of 512 2.1e-7).  Four classes per thread at a time: their loads are
// in flight together (100 samples, 64 features, 100 classes: 17.0 us with one wavefront per class after the
// other, 5.5 so; logits_few took 4.8).  What bounds it is the latency of its loads and, with several workgroups on a CU, the
// lines they touch: 128 features, 100 classes, three workgroups on a CU 3.3 us, logits_few, whose lanes each read another row, 5.2.
__device__ inline void logits_lanes8(const HeadShape &s, const float *pq, float *z, const float *__restrict__ Wf,
                                     const float *__restrict__ bf) {
  constexpr int L = 8, NQ = 4, G = HT / L;  // lanes per class, classes per thread, classes side by side
  const int l = threadIdx.x & (L - 1), g = threadIdx.x / L;
  for (int q0 = 0; q0 < s.Cls; q0 += G * NQ) {
    float acc[NQ][8];
    const float *wr[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      wr[k] = Wf + (long long)min(q0 + k * G + g, s.Cls - 1) * s.F;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[k][e] = 0.f;
    }
    if ((s.F & 3) == 0) {
      for (int f0 = 4 * l; f0 < s.F; f0 += 8 * L)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int f = f0 + h * 4 * L;
          if (f >= s.F) break;
          float4 w[NQ];
#pragma unroll
          for (int k = 0; k < NQ; ++k) w[k] = *reinterpret_cast<const float4 *>(wr[k] + f);
#pragma unroll
          for (int k = 0; k < NQ; ++k) {
            acc[k][4 * h] += w[k].x * pq[f], acc[k][4 * h + 1] += w[k].y * pq[f + 1];
            acc[k][4 * h + 2] += w[k].z * pq[f + 2], acc[k][4 * h + 3] += w[k].w * pq[f + 3];
          }
        }
    } else {
      for (int f0 = l; f0 < s.F; f0 += 8 * L)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int f = f0 + e * L;
          if (f >= s.F) break;
#pragma unroll
          for (int k = 0; k < NQ; ++k) acc[k][e] += wr[k][f] * pq[f];
        }
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      float v = ((acc[k][0] + acc[k][1]) + (acc[k][2] + acc[k][3])) + ((acc[k][4] + acc[k][5]) + (acc[k][6] + acc[k][7]));
#pragma unroll
      for (int m = L / 2; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
      const int q = q0 + k * G + g;
      if (l == 0 && q < s.Cls) z[q] = v + (bf ? bf[q] : 0.f);
    }
  }
  __syncthreads();
}

// The same for up to 16 classes: 16 lanes and one class per thread, sixteen loads in flight (1024 features, 10 classes 2.8 us,
// logits_few 5.1).
__device__ inline void logits_lanes16(const HeadShape &s, const float *pq, float *z, const float *__restrict__ Wf,
                                      const float *__restrict__ bf) {
  constexpr int L = 16, NH = 16;
  const int l = threadIdx.x & (L - 1), q = threadIdx.x / L;
  const float *const wr = Wf + (long long)min(q, s.Cls - 1) * s.F;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  if ((s.F & 3) == 0) {
    for (int f1 = 0; f1 < s.F; f1 += 4 * L * NH) {
      float4 w[NH];
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int f = f1 + 4 * l + h * 4 * L;
        if (f1 + h * 4 * L < s.F) w[h] = *reinterpret_cast<const float4 *>(wr + (f < s.F ? f : 0));  // (all lanes or none)
      }
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int f = f1 + 4 * l + h * 4 * L, o = 4 * (h & 1);
        if (f1 + h * 4 * L >= s.F) break;
        const bool ok = f < s.F;
        const float4 x = *reinterpret_cast<const float4 *>(pq + (ok ? f : 0));
        acc[o] = ok ? acc[o] + w[h].x * x.x : acc[o], acc[o + 1] = ok ? acc[o + 1] + w[h].y * x.y : acc[o + 1];
        acc[o + 2] = ok ? acc[o + 2] + w[h].z * x.z : acc[o + 2], acc[o + 3] = ok ? acc[o + 3] + w[h].w * x.w : acc[o + 3];
      }
    }
  } else {
    for (int f = l, e = 0; f < s.F; f += L, e ^= 1) (e ? acc[1] : acc[0]) += wr[f] * pq[f];
  }
  float v = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
#pragma unroll
  for (int m = L / 2; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  if (l == 0 && q < s.Cls) z[q] = v + (bf ? bf[q] : 0.f);
  __syncthreads();
}

// The same for few features, whose rows are a line or two: fewer instructions, each run once (head_sample, 32 features, 100
// classes, with dpq_few: 10.6 us, 11.9 with the form above; the other one from 128 features on).  zp: HT floats of LDS.
__device__ inline void logits_few(const HeadShape &s, const float *pq, float *z, float *zp,
                                  const float *__restrict__ Wf, const float *__restrict__ bf) {
  const int t = threadIdx.x;
  // logits: P threads per class, each over a contiguous 1/P of the features (P a power of two with
  // P * Cls <= 256 and whole 16-byte groups per part), so that one batch of independent loads per
  // thread covers the row; the P partial sums are added in order through LDS
  int P = 1;
  if ((s.F & 3) == 0)
    while (P < 8 && 2 * P * s.Cls <= HT && ((s.F >> 2) % (2 * P)) == 0) P *= 2;
  if (s.Cls <= HT) {
    const int part = t / s.Cls, q = t - part * s.Cls;
    if (part < P) {
      const int fn = s.F / P, f0 = part * fn;
      const float *wr = Wf + (long long)q * s.F + f0;
      float acc = 0.f;
      if ((s.F & 3) == 0) {
#pragma unroll 8
        for (int f = 0; f < fn; f += 4) {
          const float4 w = *reinterpret_cast<const float4 *>(wr + f);
          acc += w.x * pq[f0 + f] + w.y * pq[f0 + f + 1] + w.z * pq[f0 + f + 2] + w.w * pq[f0 + f + 3];
        }
      } else {
        for (int f = 0; f < fn; ++f) acc += wr[f] * pq[f0 + f];
      }
      zp[t] = acc;
    }
    __syncthreads();
    if (t < s.Cls) {
      float acc = zp[t];
      for (int k = 1; k < P; ++k) acc += zp[k * s.Cls + t];
      z[t] = acc + (bf ? bf[t] : 0.f);
    }
  } else {
    for (int q = t; q < s.Cls; q += HT) {
      const float *wr = Wf + (long long)q * s.F;
      float acc = 0.f;
      if ((s.F & 3) == 0) {
#pragma unroll 8
        for (int f = 0; f < s.F; f += 4) {
          const float4 w = *reinterpret_cast<const float4 *>(wr + f);
          acc += w.x * pq[f] + w.y * pq[f + 1] + w.z * pq[f + 2] + w.w * pq[f + 3];
        }
      } else {
        for (int f = 0; f < s.F; ++f) acc += wr[f] * pq[f];
      }
      z[q] = acc + (bf ? bf[q] : 0.f);
    }
  }
  __syncthreads();
}

// FEW: launches of one workgroup per sample, about one on a CU, where the simple form is the faster one (head_fc, 128 features,
// 200 classes: 12.1 / 13.2 us).
template <bool FEW>
__device__ inline void logits_sample(const HeadShape &s, const float *pq, float *z, float *zp, const float *__restrict__ Wf,
                                     const float *__restrict__ bf) {
  if (FEW || s.F < 128) logits_few(s, pq, z, zp, Wf, bf);
  else if (s.Cls > 16) logits_lanes8(s, pq, z, Wf, bf);
  else logits_lanes16(s, pq, z, Wf, bf);
}

// out[f] = pool_scale(f) * sum_q dz[q] * Wf[q][f] (z holds dz; all threads of a workgroup).  With fewer features than
// threads the classes are cut into P ranges, one per group of F threads, and the P sums added in
// order through zp: a chain of Cls / P loads instead of Cls (head_sample, 16 features, 100 classes, with
// the pooling tree: 12.9 -> 10.7 us).
__device__ inline void dpq_few(const HeadShape &s, const float *z, float *zp, const float *__restrict__ Wf,
                               float *out) {
  const int t = threadIdx.x;
  int P = 1;
  while (2 * P * s.F <= HT && 32 * P <= s.Cls) P *= 2;  // at least 16 classes each
  if (P == 1) {
    for (int f = t; f < s.F; f += HT) {
      float acc = 0.f;
#pragma unroll 10
      for (int q = 0; q < s.Cls; ++q) acc += z[q] * Wf[(long long)q * s.F + f];
      out[f] = acc * pool_scale(s, f);
    }
    return;
  }
  const int part = t / s.F, f = t - part * s.F, qn = (s.Cls + P - 1) / P;
  if (part < P) {
    const int q1 = min(s.Cls, (part + 1) * qn);
    float acc = 0.f;
#pragma unroll 8
    for (int q = part * qn; q < q1; ++q) acc += z[q] * Wf[(long long)q * s.F + f];
    zp[t] = acc;
  }
  __syncthreads();
  if (t < s.F) {
    float acc = zp[t];
    for (int k = 1; k < P; ++k) acc += zp[k * s.F + t];
    out[t] = acc * pool_scale(s, t);
  }
}

// The same from 128 features on: V features per thread (4: 16-byte loads),
// and the classes cut into P ranges, one per group of F / V threads, their sums added in order through zp (HT * 4
// floats): a chain of Cls / P loads instead of Cls (128 features, 100 classes: 2.5 us with two ranges and single
// floats, 2.1 so).
__device__ inline void dpq_many(const HeadShape &s, const float *z, float *zp, const float *__restrict__ Wf,
                                float *out) {
  constexpr int V = 4, NB = 14;  // (a hundred classes in eight ranges are one batch)
  const int t = threadIdx.x, FG = s.F / V;
  int P = 1;
  while (P < 16 && 2 * P * FG <= HT && 8 * P <= s.Cls) P *= 2;  // at least 4 classes each
  const int qn = (s.Cls + P - 1) / P;
  for (int i = t; i < FG * P; i += HT) {  // (once where P > 1)
    const int part = i / FG, f = (i - part * FG) * V;
    const int q1 = min(s.Cls, (part + 1) * qn);
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    const float *const wf = Wf + f;
    for (int q0 = part * qn; q0 < q1; q0 += NB) {  // a batch of loads in flight, the last few of them repeated
      Chan<V> w[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) w[u] = load_chan<V>(wf + min(q0 + u, q1 - 1) * s.F);
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const float d = z[min(q0 + u, q1 - 1)];
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = q0 + u < q1 ? acc[e] + d * w[u].v[e] : acc[e];
      }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) (P == 1 ? out : zp + part * s.F)[f + e] = acc[e];
  }
  __syncthreads();
  for (int f = t; f < s.F; f += HT) {
    float acc = P == 1 ? out[f] : zp[f];
    for (int k = 1; k < P; ++k) acc += zp[k * s.F + f];
    out[f] = acc * pool_scale(s, f);
  }
}
template <bool FEW>
__device__ inline void dpq_sample(const HeadShape &s, const float *z, float *zp, const float *__restrict__ Wf,
                                  float *out) {
  if (FEW || s.F < 128 || (s.F & 3)) dpq_few(s, z, zp, Wf, out);
  else dpq_many(s, z, zp, Wf, out);
}

// gamma_n and Eq. 3 for one sample (all threads of a workgroup): logits (the pooled features pq[F]
// already staged in LDS), log-sum-exp, per-sample loss, dL/dz, and -- the
// sample's dz being at hand -- the gradient w.r.t. the pooled features
// dPq[f] = sum_q dz[q] * Wf[q][f], divided by the elements that f averages and stored to dPq_out (global row of the sample, or an LDS array).
// z: Cls floats of LDS, red: 8 floats of LDS.  write = false: dz and the loss are formed but not
// stored (a workgroup that only needs dPq of a sample another workgroup reports).
// after_logits is called once the linear layer has been read (loads that may run under the rest).
template <bool FEW, class Fn>
__device__ inline void fc_loss_sample(const HeadShape &s, int n, const float *pq, float *z, float *red,
                                      const int32_t *__restrict__ labels, const float *__restrict__ Wf,
                                      const float *__restrict__ bf, float *__restrict__ dz,
                                      float *__restrict__ loss_n, float *dPq_out, bool write, Fn after_logits) {
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  __shared__ __attribute__((aligned(16))) float zp[HT * 4];
  logits_sample<FEW>(s, pq, z, zp, Wf, bf);
  after_logits();

  if (s.mse) {
    // squared error against the one-hot label, mean over the classes (the batch mean follows)
    const int y = labels[n];
    const float sc = 2.f / ((float)s.B * (float)s.Cls);
    float se = 0.f;
    for (int q = t; q < s.Cls; q += HT) {
      const float e = z[q] - (q == y ? 1.f : 0.f);
      se += e * e;
      if (write) dz[(long long)n * s.Cls + q] = e * sc;
    }
    se = wave_sum(se);
    if (lane == 0) red[wave] = se;
    __syncthreads();
    if (t == 0 && write) loss_n[n] = ((red[0] + red[1]) + (red[2] + red[3])) / (float)s.Cls;
    for (int q = t; q < s.Cls; q += HT) z[q] = (z[q] - (q == y ? 1.f : 0.f)) * sc;
    __syncthreads();
    dpq_sample<FEW>(s, z, zp, Wf, dPq_out);
    return;
  }
  float m = -INFINITY;
  for (int q = t; q < s.Cls; q += HT) m = fmaxf(m, z[q]);
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float se = 0.f;
  for (int q = t; q < s.Cls; q += HT) se += expf(z[q] - m);
  se = wave_sum(se);
  if (lane == 0) red[4 + wave] = se;
  __syncthreads();
  se = (red[4] + red[5]) + (red[6] + red[7]);
  const float lse = m + logf(se);
  const int y = labels[n];
  const float invB = 1.f / (float)s.B;
  const float zy = (y >= 0 && y < s.Cls) ? z[y] : 0.f;
  __syncthreads();  // every read of the logits is done: z[] becomes dz[]
  for (int q = t; q < s.Cls; q += HT) {
    const float d = (expf(z[q] - lse) - (q == y ? 1.f : 0.f)) * invB;
    if (write) dz[(long long)n * s.Cls + q] = d;
    z[q] = d;
  }
  if (t == 0 && write) loss_n[n] = lse - zy;
  __syncthreads();
  dpq_sample<FEW>(s, z, zp, Wf, dPq_out);
}

// One sample per workgroup.  Dynamic LDS: F + Cls + 8 floats.
__global__ __launch_bounds__(HT) void head_fc_kernel(HeadShape s, const float *__restrict__ Pq,
                                                     const int32_t *__restrict__ labels,
                                                     const float *__restrict__ Wf, const float *__restrict__ bf,
                                                     float *__restrict__ dz, float *__restrict__ loss_n,
                                                     float *__restrict__ dPq) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float *pq = sm;           // [F]
  float *z = pq + s.F;      // [Cls]
  float *red = z + s.Cls;   // [8]
  const int n = blockIdx.x, t = threadIdx.x;
  for (int f = t; f < s.F; f += HT) pq[f] = Pq[(long long)n * s.F + f];
  __syncthreads();
  fc_loss_sample<true>(s, n, pq, z, red, labels, Wf, bf, dz, loss_n, dPq + (long long)n * s.F, true, [] {});
}

// The same step for wide heads (many pooled features): G samples per workgroup share every load
// of Wf, and the workgroup has WT = 1024 threads so that the chip still holds as many wavefronts
// as with one sample per 256 threads.  Logits: one wavefront per class, its lanes striding the
// features (coalesced float4 reads of the class's row), wavefront sum; softmax: one wavefront per
// sample; dPq: one thread per feature, the loop over classes unrolled so that many independent
// loads are in flight.  Needs F % 4 == 0.  Dynamic LDS: G * (F + Cls) floats.
constexpr int WT = 1024;
template <int G>
__global__ __launch_bounds__(WT) void head_fc_wide_kernel(HeadShape s, const float *__restrict__ Pq,
                                                          const int32_t *__restrict__ labels,
                                                          const float *__restrict__ Wf,
                                                          const float *__restrict__ bf, float *__restrict__ dz,
                                                          float *__restrict__ loss_n, float *__restrict__ dPq) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float *pq = sm;               // [G][F]
  float *z = pq + G * s.F;      // [G][Cls]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int n0 = blockIdx.x * G;
  const int ng = min(G, s.B - n0);
  for (int i = t * 4; i < G * s.F; i += WT * 4) {
    const int g = i / s.F;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (g < ng) v = *reinterpret_cast<const float4 *>(Pq + (long long)n0 * s.F + i);
    *reinterpret_cast<float4 *>(pq + i) = v;
  }
  __syncthreads();
  for (int q = wave; q < s.Cls; q += WT / 64) {
    const float *wr = Wf + (long long)q * s.F;
    float acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = 0.f;
#pragma unroll 4
    for (int f = lane * 4; f < s.F; f += 256) {
      const float4 w = *reinterpret_cast<const float4 *>(wr + f);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float4 x = *reinterpret_cast<const float4 *>(pq + g * s.F + f);
        acc[g] += w.x * x.x + w.y * x.y + w.z * x.z + w.w * x.w;
      }
    }
    const float bias = bf ? bf[q] : 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float v = wave_sum(acc[g]);
      if (lane == 0) z[g * s.Cls + q] = v + bias;
    }
  }
  __syncthreads();
  const float invB = 1.f / (float)s.B;
  if (wave < ng && s.mse) {
    const int g = wave;
    float *zg = z + g * s.Cls;
    const int y = labels[n0 + g];
    const float sc = 2.f / ((float)s.B * (float)s.Cls);
    float se = 0.f;
    for (int q = lane; q < s.Cls; q += 64) {
      const float e = zg[q] - (q == y ? 1.f : 0.f);
      se += e * e;
      dz[(long long)(n0 + g) * s.Cls + q] = e * sc;
      zg[q] = e * sc;
    }
    se = wave_sum(se);
    if (lane == 0) loss_n[n0 + g] = se / (float)s.Cls;
  } else if (wave < ng) {
    const int g = wave;
    float *zg = z + g * s.Cls;
    float m = -INFINITY;
    for (int q = lane; q < s.Cls; q += 64) m = fmaxf(m, zg[q]);
    m = wave_max(m);
    float se = 0.f;
    for (int q = lane; q < s.Cls; q += 64) se += expf(zg[q] - m);
    se = wave_sum(se);
    const float lse = m + logf(se);
    const int y = labels[n0 + g];
    const float zy = (y >= 0 && y < s.Cls) ? zg[y] : 0.f;
    // (one wavefront owns zg: its read of zg[y] above is issued before the stores below)
    for (int q = lane; q < s.Cls; q += 64) {
      const float d = (expf(zg[q] - lse) - (q == y ? 1.f : 0.f)) * invB;
      dz[(long long)(n0 + g) * s.Cls + q] = d;
      zg[q] = d;
    }
    if (lane == 0) loss_n[n0 + g] = lse - zy;
  }
  __syncthreads();
  for (int f = t; f < s.F; f += WT) {
    const float scale = pool_scale(s, f);
    float acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = 0.f;
#pragma unroll 20
    for (int q = 0; q < s.Cls; ++q) {
      const float w = Wf[(long long)q * s.F + f];
#pragma unroll
      for (int g = 0; g < G; ++g) acc[g] += z[g * s.Cls + q] * w;
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (g < ng) dPq[(long long)(n0 + g) * s.F + f] = acc[g] * scale;
  }
}

// Forward-only head for early-exit evaluation: one sample per workgroup; logits, then the arg-max
// over the classes with the lowest index winning among equal maxima.  Dynamic LDS: F + Cls floats.
__global__ __launch_bounds__(HT) void head_predict_kernel(HeadShape s, const float *__restrict__ Pq,
                                                          const int32_t *__restrict__ labels,
                                                          const float *__restrict__ Wf,
                                                          const float *__restrict__ bf,
                                                          float *__restrict__ logits_out, int32_t *__restrict__ pred,
                                                          int32_t *__restrict__ hit) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float rv[HT];
  __shared__ int ri[HT];
  float *pq = sm;          // [F]
  float *z = pq + s.F;     // [Cls]
  const int n = blockIdx.x, t = threadIdx.x;
  for (int f = t; f < s.F; f += HT) pq[f] = Pq[(long long)n * s.F + f];
  __syncthreads();
  logits_lanes8(s, pq, z, Wf, bf);
  if (logits_out)
    for (int q = t; q < s.Cls; q += HT) logits_out[(long long)n * s.Cls + q] = z[q];
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int q = t; q < s.Cls; q += HT)
    if (z[q] > best) best = z[q], bi = q;  // ascending q, strict: lowest index of this thread's maxima
  rv[t] = best, ri[t] = bi;
  __syncthreads();
  for (int o = HT / 2; o > 0; o >>= 1) {
    if (t < o) {
      const float cv = rv[t + o];
      const int ci = ri[t + o];
      if (cv > rv[t] || (cv == rv[t] && ci < ri[t])) rv[t] = cv, ri[t] = ci;
    }
    __syncthreads();
  }
  if (t == 0) {
    const int p = ri[0] == 0x7fffffff ? 0 : ri[0];  // no logit compared greater than -inf (all NaN): class 0
    pred[n] = p;
    if (labels) hit[n] = p == labels[n] ? 1 : 0;
  }
}

__global__ __launch_bounds__(HT) void count_hits_kernel(const int32_t *__restrict__ hit, int B,
                                                        int32_t *__restrict__ out, int accumulate) {
  __shared__ int red[HT];
  int acc = 0;
  for (int i = threadIdx.x; i < B; i += HT) acc += hit[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = HT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (accumulate ? *out : 0) + red[0];
}

__global__ __launch_bounds__(HT) void loss_mean_kernel(const float *__restrict__ loss_n, int B,
                                                       float *__restrict__ out) {
  __shared__ float red[HT];
  loss_mean_block(loss_n, B, out, red);
}

// dU for V consecutive channels u of one element (n, hh, w, av): F_n backward + aux ReLU mask.
// dpq points at the sample's dPq[F] (global or LDS), pargn at its selection record (max pooling).
template <int V>
__device__ inline void du_element(const HeadShape &s, int hh, int w, int av, const Chan<V> &u, const float *dpq,
                                  const int32_t *pargn, float *__restrict__ du_at) {
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  // the windows that hold row hh and column w: floor(i L / O) <= hh < ceil((i + 1) L / O)
  const int ci0 = (int)s.div_hu.div((uint32_t)(hh * s.oh)), ci1 = (int)s.div_hu.div((uint32_t)((hh + 1) * s.oh - 1));
  const int cj0 = (int)s.div_wu.div((uint32_t)(w * s.ow)), cj1 = (int)s.div_wu.div((uint32_t)((w + 1) * s.ow - 1));
  for (int ci = ci0; ci <= ci1; ++ci)
    for (int cj = cj0; cj <= cj1; ++cj) {
      const int fo = (ci * s.ow + cj) * s.A + av * V;
      if (s.pmax) {  // max pooling hands the gradient to the element it selected
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (pargn[fo + e] == hh * s.Wu + w) acc[e] += dpq[fo + e];
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += dpq[fo + e];
      }
    }
#pragma unroll
  for (int e = 0; e < V; ++e)
    if (s.relu && !(u.v[e] > 0.f)) acc[e] = 0.f;
  if constexpr (V == 4) {
    *reinterpret_cast<float4 *>(du_at) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  } else {
    du_at[0] = acc[0];
  }
}

// The whole per-sample chain of a head with a small activation map in one launch: workgroup n
// (n < B) runs F_n, gamma_n, the loss and dL/dz, dPq and the backward through F_n and the aux ReLU
// for sample n; the pooled features, dPq and the max-pooling selection stay in LDS between the
// stages.  With splits > 0 the aux activation is first formed from the raw partial sums of the
// split aux convolution (see pool_pairs).  Workgroups from B on re-lay the aux filter for the
// data gradient.
// Dynamic LDS: 2*F + Cls + 8 floats, + F ints for max pooling.
template <int V, bool PMAX>
__global__ __launch_bounds__(HT) void head_sample_kernel(HeadShape s, float *__restrict__ U,
                                                         const float *__restrict__ part, int splits,
                                                         const float *__restrict__ ba,
                                                         const int32_t *__restrict__ labels,
                                                         const float *__restrict__ Wf, const float *__restrict__ bf,
                                                         float *__restrict__ Pq, int32_t *__restrict__ parg,
                                                         float *__restrict__ dz, float *__restrict__ loss_n,
                                                         float *__restrict__ dU, RelayJob rj, int CA, int NS) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float red[HT * V];
  __shared__ int redi[PMAX ? HT * V : 1];
  const int t = threadIdx.x;
  if ((int)blockIdx.x >= s.B) {
    relay_block(rj, (int)blockIdx.x - s.B);
    return;
  }
  float *pq = sm;            // [F]
  float *dpq = pq + s.F;     // [F]
  float *z = dpq + s.F;      // [Cls]
  float *red8 = z + s.Cls;   // [8]
  int *pargl = reinterpret_cast<int *>(red8 + 8);  // [F] (max pooling)
  const int n = blockIdx.x;
  const int cells = s.oh * s.ow, G = HT / (CA * NS);
  for (int c0 = 0; c0 < cells; c0 += G)
    pool_pairs<V, PMAX>(s, (long long)n * cells + c0, (long long)(n + 1) * cells, U, part, splits, ba, Pq, parg, CA,
                        NS, red, redi, pq, PMAX ? pargl : nullptr, (long long)n * cells);
  __syncthreads();  // (with splits > 0 the sample's U was formed and written on the way: visible to the workgroup)
  fc_loss_sample<true>(s, n, pq, z, red8, labels, Wf, bf, dz, loss_n, dpq, true, [] {});
  __syncthreads();
  const int AV = s.A / V, per_n = s.Hu * s.Wu * AV;
  const long long base = (long long)n * per_n;
  for (int i = t; i < per_n; i += HT) {
    const int r = (int)s.div_av.div((uint32_t)i), av = i - r * AV;
    const int hh = (int)s.div_wu.div((uint32_t)r), w = r - hh * s.Wu;
    du_element<V>(s, hh, w, av, load_chan<V>(U + (base + i) * V), dpq, PMAX ? pargl : nullptr, dU + (base + i) * V);
  }
}

// Everything of the head after F_n for a LARGE activation map in one launch: gamma_n, the loss and
// dL/dz, dPq, and the backward through F_n and the aux ReLU (dU).  A sample's map is cut into NS
// slices, one workgroup each, so that the launch has enough workgroups to stream dU; every one of
// them recomputes the sample's tiny linear layer (F * Cls products, Wf from L2) instead of reading
// dPq from an earlier launch, and slice 0 stores dz and the per-sample loss.  Workgroups from
// B * NS on re-lay the aux filter for the data gradient.  With `ppart` given, F_n itself is formed
// here too (and Pq stored by slice 0) from the column sums the aux convolution's epilogue left.
// Dynamic LDS: 2*F + Cls + 8 floats.
template <int V>
__global__ __launch_bounds__(HT, 3) void head_wide_kernel(HeadShape s, int NS, const float *__restrict__ U,
                                                       float *__restrict__ Pq, const float *__restrict__ ppart,
                                                       const int32_t *__restrict__ labels,
                                                       const float *__restrict__ Wf, const float *__restrict__ bf,
                                                       float *__restrict__ dz, float *__restrict__ loss_n,
                                                       const int32_t *__restrict__ parg, float *__restrict__ dU,
                                                       RelayJob rj) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int t = threadIdx.x;
  if ((int)blockIdx.x >= s.B * NS) {
    relay_block(rj, (int)blockIdx.x - s.B * NS);
    return;
  }
  float *pq = sm;            // [F]
  float *dpq = pq + s.F;     // [F]
  float *z = dpq + s.F;      // [Cls]
  float *red8 = z + s.Cls;   // [8]
  const int n = blockIdx.x / NS, sl = blockIdx.x - n * NS;
  if (ppart) {
    // F_n (2x2 average pooling of an even-sized map) from the column sums the aux convolution left
    // per 16 consecutive pixels: image rows of 16 pixels carry both halves in two slots, wider rows
    // are whole 16-pixel groups per half.  Rows ascending, groups ascending: a fixed order.
    const bool split = s.Wu == 16;
    const int gpr = s.Wu >> 4;                // 16-pixel groups per image row
    const int gph = split ? 1 : (gpr >> 1);   // ... per half row
    const float inv = 1.f / (float)((s.Hu >> 1) * (s.Wu >> 1));
    // The partials of a feature go to P threads (one batch of loads each where that many threads are left); their sums
    // are added in order.
    __shared__ float pp[HT];
    const int np = (s.Hu >> 1) * gph;
    int P = 1;
    while (P < 8 && 2 * P * s.F <= HT && 4 * P <= np) P *= 2;
    const int ni = (np + P - 1) / P;
    for (int k = t; k < s.F * P; k += HT) {  // (once where P > 1)
      const int part = k / s.F, f = k - part * s.F;
      const int cell = f / s.A, a = f - cell * s.A;
      const int ci = cell >> 1, cj = cell & 1;
      // partial i of the cell: image row ci*Hu/2 + i / gph, group i % gph of the half row; loaded
      // eight at a time (independent loads), added in order
      const float *src = ppart + (split ? cj : 0) * s.A + a;
      const int e1 = min(np, (part + 1) * ni);
      float acc = 0.f;
      for (int e0 = part * ni; e0 < e1; e0 += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = e0 + u, hr = i / gph;
          const long long r16 = ((long long)n * s.Hu + ci * (s.Hu >> 1) + hr) * gpr + (split ? 0 : cj * gph + (i - hr * gph));
          v[u] = i < e1 ? src[r16 * 2 * s.A] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
      }
      (P == 1 ? pq : pp)[k] = acc;
    }
    if (P > 1) __syncthreads();
    for (int f = t; f < s.F; f += HT) {  // (without parts each thread reads what it wrote)
      float acc = P == 1 ? pq[f] : pp[f];
      for (int k = 1; k < P; ++k) acc += pp[k * s.F + f];
      pq[f] = acc * inv;
      if (sl == 0) Pq[(long long)n * s.F + f] = acc * inv;
    }
  } else {
    for (int f = t; f < s.F; f += HT) pq[f] = Pq[(long long)n * s.F + f];
  }
  __syncthreads();
  // the slice's first elements of U: their loads run under the softmax
  constexpr int AHEAD = 4;
  const int AV = s.A / V, per_n = s.Hu * s.Wu * AV;
  const int per_sl = (per_n + NS - 1) / NS;
  const int i0 = sl * per_sl + t, i1 = min(per_n, (sl + 1) * per_sl);
  const long long base = (long long)n * per_n;
  const float *const un = U + base * V;
  Chan<V> ahead[AHEAD];
  auto prefetch = [&] {
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) ahead[k] = load_chan<V>(un + min(i0 + k * HT, per_n - 1) * V);
  };
  fc_loss_sample<false>(s, n, pq, z, red8, labels, Wf, bf, dz, loss_n, dpq, sl == 0, prefetch);
  __syncthreads();
  auto element = [&](int i, const Chan<V> &u) {
    const int r = (int)s.div_av.div((uint32_t)i), av = i - r * AV;
    const int hh = (int)s.div_wu.div((uint32_t)r), w = r - hh * s.Wu;
    du_element<V>(s, hh, w, av, u, dpq, s.pmax ? parg + (long long)n * s.F : nullptr, dU + (base + i) * V);
  };
#pragma unroll
  for (int k = 0; k < AHEAD; ++k)
    if (i0 + k * HT < i1) element(i0 + k * HT, ahead[k]);
  for (int c = i0 + AHEAD * HT; c < i1; c += AHEAD * HT) {  // as many loads in flight, or each waits for the store before it
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) ahead[k] = load_chan<V>(un + min(c + k * HT, per_n - 1) * V);
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
      if (c + k * HT < i1) element(c + k * HT, ahead[k]);
  }
}

// Backward of the head after the softmax in one launch (gradient line of Algorithm 2); the
// workgroup index selects the job:
//   [0, nb_w)   gamma_n: one class q and one chunk of `fch` features; the 256 threads are fch
//               feature lanes x (256/fch) batch slices, slice sums added in order through LDS.
//               dWf[q][f] = sum_n dz[n][q] * Pq[n][f]; chunk 0 also forms dbf[q] = sum_n dz[n][q].
//   then nb_u   F_n backward + aux ReLU mask: dU = [U > 0] * sum over windows containing (h,w)
//               of dPq / |window| (max pooling: of dPq where the window selected (h,w)), V
//               channels per thread;
//   then nb_t   re-lay of the aux filter for the data gradient: WaT[k][r][s][a] = Wa[a][R-1-r][S-1-s][k];
//   then 0/1    batch mean of the per-sample losses (when loss_out is given).
struct HeadBwdJobs {
  int nb_w, nb_u, nb_t, fch, nchunks;
};
template <int V>
__global__ __launch_bounds__(HT) void head_bwd_kernel(HeadShape s, HeadBwdJobs jb, const float *__restrict__ Pq,
                                                      const float *__restrict__ dz, float *__restrict__ dWf,
                                                      float *__restrict__ dbf, const float *__restrict__ U,
                                                      const float *__restrict__ dPq, float *__restrict__ dU,
                                                      RelayJob rj, const float *__restrict__ loss_n,
                                                      float *__restrict__ loss_out,
                                                      const int32_t *__restrict__ parg) {
  __shared__ float red[HT];
  __shared__ float redb[HT];
  int b = blockIdx.x;
  const int t = threadIdx.x;
  if (b < jb.nb_w) {
    GammaJob g;
    g.B = s.B, g.F = s.F, g.Cls = s.Cls, g.Pq = Pq, g.dz = dz, g.dWf = dWf, g.dbf = dbf;
    g.Wf = g.bf = g.vWf = g.vbf = nullptr, g.lr = g.mu = 0.f;
    g.fch = jb.fch, g.nchunks = jb.nchunks;
    gamma_block(g, b, red, redb);
    return;
  }
  b -= jb.nb_w;
  if (b < jb.nb_u) {
    const int AV = s.A / V;
    const long long total = (long long)s.B * s.Hu * s.Wu * AV;
    const long long i = (long long)b * HT + t;
    if (i >= total) return;
    // pixels of all samples fit 31 bits, channel groups of all of them may not
    long long r0 = i / AV;
    if (total <= 0x7FFFFFFFll) r0 = s.div_av.div((uint32_t)i);
    const int r = (int)r0, av = (int)(i - r0 * AV), row = (int)s.div_wu.div((uint32_t)r), w = r - row * s.Wu;
    const int n = (int)s.div_hu.div((uint32_t)row), hh = row - n * s.Hu;
    du_element<V>(s, hh, w, av, load_chan<V>(U + i * V), dPq + (long long)n * s.F, s.pmax ? parg + (long long)n * s.F : nullptr,
                  dU + i * V);
    return;
  }
  b -= jb.nb_u;
  if (b < jb.nb_t) {
    relay_block(rj, b);
    return;
  }
  loss_mean_block(loss_n, s.B, loss_out, red);
}

}  // namespace

// pooling decomposition of a workgroup (see pool_pairs): channel lanes CA, position slices NS
static void pool_lanes(const HeadShape &h, int V, int *CA_out, int *NS_out) {
  const int AV = h.A / V;
  int CA = 1;
  while (CA < AV && CA < HT) CA *= 2;  // channel lanes: power of two covering A / V (or all threads)
  // largest pooling window -> position slices (power of two, at most what the workgroup has left)
  const int wh = (h.Hu + h.oh - 1) / h.oh + (h.Hu % h.oh ? 1 : 0), wwid = (h.Wu + h.ow - 1) / h.ow + (h.Wu % h.ow ? 1 : 0);
  int NS = 1;
  while (NS * 2 <= wh * wwid && CA * NS * 2 <= HT) NS *= 2;
  *CA_out = CA, *NS_out = NS;
}

hipError_t launch_head_pool(const HeadShape &h, float *U, const float *part, int splits, const float *ba, float *Pq,
                            int32_t *parg, hipStream_t st) {
  const int V = h.A % 4 == 0 ? 4 : 1;
  int CA, NS;
  pool_lanes(h, V, &CA, &NS);
  const int G = HT / (CA * NS);
  const long long pairs = (long long)h.B * h.oh * h.ow;
  const dim3 grid((unsigned)((pairs + G - 1) / G));
  if (h.pmax) {
    if (V == 4)
      hipLaunchKernelGGL((head_pool_kernel<4, true>), grid, dim3(HT), 0, st, h, U, part, splits, ba, Pq, parg, CA, NS);
    else
      hipLaunchKernelGGL((head_pool_kernel<1, true>), grid, dim3(HT), 0, st, h, U, part, splits, ba, Pq, parg, CA, NS);
  } else if (V == 4) {
    hipLaunchKernelGGL((head_pool_kernel<4, false>), grid, dim3(HT), 0, st, h, U, part, splits, ba, Pq, parg, CA, NS);
  } else {
    hipLaunchKernelGGL((head_pool_kernel<1, false>), grid, dim3(HT), 0, st, h, U, part, splits, ba, Pq, parg, CA, NS);
  }
  return hipGetLastError();
}

hipError_t launch_head_fc(const HeadShape &h, const float *Pq, const int32_t *labels, const float *Wf,
                          const float *bf, float *dz, float *loss_n, float *dPq, hipStream_t st) {
  constexpr int G = 4;
  const size_t lds_wide = (size_t)G * (h.F + h.Cls) * sizeof(float);
  if (h.F >= 256 && h.F % 4 == 0 && lds_wide <= 48 * 1024) {
    hipLaunchKernelGGL(head_fc_wide_kernel<G>, dim3((h.B + G - 1) / G), dim3(WT), lds_wide, st, h, Pq, labels, Wf, bf,
                       dz, loss_n, dPq);
    return hipGetLastError();
  }
  const size_t lds = (size_t)(h.F + h.Cls + 8) * sizeof(float);
  hipLaunchKernelGGL(head_fc_kernel, dim3(h.B), dim3(HT), lds, st, h, Pq, labels, Wf, bf, dz, loss_n, dPq);
  return hipGetLastError();
}

RelayJob relay_job(const float *Wa, float *WaT, float *U, int A, int R, int S, int K) {
  static_assert(HT == 256, "relay_block");
  RelayJob j;
  j.Wa = Wa, j.WaT = WaT, j.U = U, j.A = A, j.R = R, j.S = S, j.K = K;
  j.nchunks = (A + WINO_CH - 1) / WINO_CH;
  j.nb_t = (int)(((long long)A * R * S * K + HT - 1) / HT);
  const int nb = wino_nb(K);
  j.nb_u = U ? ((K + nb - 1) / nb * nb * 2 * j.nchunks + HT - 1) / HT : 0;
  return j;
}

bool head_sample_applicable(const HeadShape &h) {
  // a sample's activation map of at most 4 KiB (measured: at 16 KiB per sample and 128 samples the
  // three chip-wide launches are faster than 128 workgroups doing a sample each), the linear layer
  // narrow enough that sharing its weights between samples (head_fc_wide_kernel) does not pay
  return (long long)h.Hu * h.Wu * h.A <= 1024 && h.F <= 256 && h.Cls <= 1024;
}

hipError_t launch_head_sample(const HeadShape &h, float *U, const float *part, int splits, const float *ba,
                              const int32_t *labels, const float *Wf, const float *bf, float *Pq, int32_t *parg,
                              float *dz, float *loss_n, float *dU, const RelayJob &rj, hipStream_t st) {
  const int V = h.A % 4 == 0 ? 4 : 1;
  int CA, NS;
  pool_lanes(h, V, &CA, &NS);
  const unsigned nb_t = (unsigned)(rj.nb_t + rj.nb_u);
  const dim3 grid((unsigned)h.B + nb_t);
  const size_t lds = (size_t)(2 * h.F + h.Cls + 8) * sizeof(float) + (h.pmax ? (size_t)h.F * sizeof(int) : 0);
#define NF_HS(V_, P_)                                                                                              \
  hipLaunchKernelGGL((head_sample_kernel<V_, P_>), grid, dim3(HT), lds, st, h, U, part, splits, ba, labels, Wf, bf, Pq, \
                     parg, dz, loss_n, dU, rj, CA, NS)
  if (h.pmax) {
    if (V == 4) NF_HS(4, true);
    else NF_HS(1, true);
  } else {
    if (V == 4) NF_HS(4, false);
    else NF_HS(1, false);
  }
#undef NF_HS
  return hipGetLastError();
}

// slices per sample of head_wide_kernel: about 512 workgroups in all (768: 13.7 us for 64 samples of 32x32 pixels, 32 filters, 512:
// 13.0, 384: 14.2), at least 1024 values of dU each
static int wide_slices(const HeadShape &h) {
  const long long per_sample = (long long)h.Hu * h.Wu * h.A;
  return (int)std::max(1ll, std::min((511ll + h.B) / h.B, per_sample / 1024));
}

// One launch after the pooling (head_wide_kernel: the linear layer is recomputed by every slice of a sample, its weights read from
// L2 by every workgroup) or two (the linear layer, then head_bwd_kernel).
bool head_wide_applicable(const HeadShape &h) {
  if (head_sample_applicable(h) || h.F > 1024 || h.Cls > 1024) return false;
  // the other side is head_fc_kernel: the same sums, without the slices
  if (h.F < 256 || h.F % 4) return (long long)h.F * h.Cls <= 16384;
  // The other side is head_fc_wide_kernel, which shares the weights between four samples, so that 1024 samples are a round of the
  // chip; a chain over the classes bounds it.  Against that, per workgroup on a CU, the weights read twice (the logits in
  // passes of 16 or 128 classes), and the few workgroups that store dU.  us, fitted to 335 random heads of 256 ... 1024 features, 10
  // ... 880 classes, 1 ... 5800 samples of up to 48x48 pixels (means of a step and of the separate calls): of the 1924 us that the
  // better side of each is ahead in one launch, this choice takes 1840, 16384 weights as the line -75; of 200 more, with 2 ... 37
  // classes, 59 of 114.  Two launches / one, a step: 64 filters, 100 classes, 1 of 6x6 60 / 52; 72, 200, 509 of 21x21 364 / 349; 68,
  // 815, 87 of 16x16 297 / 255; 100, 599, 2 of 33x33 198 / 154.  And the other way: 140, 37, 465 of 6x6 167 / 175; 252, 162, 259 of
  // 5x5 116 / 125.  On a fifth of the heads neither is ahead by 1 us.
  const int pass = h.Cls <= 16 ? 16 : 128, padded = (h.Cls + pass - 1) / pass * pass;
  const double chain = 0.073 * h.Cls * std::max(1.0, h.B / 1024.0);
  const double weights = 0.3e-4 * h.F * 0.5 * (padded + h.Cls) * std::max(1.0, (double)h.B * wide_slices(h) / 256);
  const double stores = 0.19e-6 * h.B * h.Hu * h.Wu * h.A;
  return chain - weights - stores > 0.1;
}

bool head_pool_partials_applicable(const HeadShape &h) {
  // 2x2 average pooling of an even-sized map whose rows are whole groups of 16 pixels per half (or
  // exactly 16 pixels: the two halves are the two 8-pixel sums of a group)
  return !h.pmax && h.oh == 2 && h.ow == 2 && h.Hu % 2 == 0 && (h.Wu == 16 || h.Wu % 32 == 0);
}

hipError_t launch_head_wide(const HeadShape &h, const float *U, float *Pq, const float *ppart, const int32_t *labels,
                            const float *Wf, const float *bf, float *dz, float *loss_n, const int32_t *parg,
                            float *dU, const RelayJob &rj, hipStream_t st) {
  const int V = h.A % 4 == 0 ? 4 : 1;
  const int NS = wide_slices(h);
  const unsigned nb_t = (unsigned)(rj.nb_t + rj.nb_u);
  const dim3 grid((unsigned)(h.B * NS) + nb_t);
  const size_t lds = (size_t)(2 * h.F + h.Cls + 8) * sizeof(float);
  if (V == 4)
    hipLaunchKernelGGL(head_wide_kernel<4>, grid, dim3(HT), lds, st, h, NS, U, Pq, ppart, labels, Wf, bf, dz, loss_n, parg, dU,
                       rj);
  else
    hipLaunchKernelGGL(head_wide_kernel<1>, grid, dim3(HT), lds, st, h, NS, U, Pq, ppart, labels, Wf, bf, dz, loss_n, parg, dU,
                       rj);
  return hipGetLastError();
}

int gamma_job_plan(GammaJob &g) {
  // feature lanes per workgroup: few, so that many batch slices share the reduction over n
  g.fch = 8;
  while (g.fch < 32 && g.fch * 2 <= g.F) g.fch *= 2;
  g.nchunks = (g.F + g.fch - 1) / g.fch;
  g.nb_w = g.Cls * g.nchunks;
  g.nb_l = g.loss_out ? 1 : 0;
  return g.nb_w + g.nb_l;
}

hipError_t launch_head_predict(const HeadShape &h, const float *Pq, const int32_t *labels, const float *Wf,
                               const float *bf, float *logits_out, int32_t *pred, int32_t *hit, hipStream_t st) {
  const size_t lds = (size_t)(h.F + h.Cls) * sizeof(float);
  hipLaunchKernelGGL(head_predict_kernel, dim3(h.B), dim3(HT), lds, st, h, Pq, labels, Wf, bf, logits_out, pred, hit);
  return hipGetLastError();
}

hipError_t launch_count_hits(const int32_t *hit, int B, int32_t *out, bool accumulate, hipStream_t st) {
  hipLaunchKernelGGL(count_hits_kernel, dim3(1), dim3(HT), 0, st, hit, B, out, accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_loss_mean(const float *loss_n, int B, float *loss_out, hipStream_t st) {
  hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(HT), 0, st, loss_n, B, loss_out);
  return hipGetLastError();
}

hipError_t launch_head_bwd(const HeadShape &h, const float *Pq, const float *dz, float *dWf, float *dbf,
                           const float *U, const float *dPq, float *dU, const RelayJob &rj, const float *loss_n,
                           float *loss_out, const int32_t *parg, hipStream_t st) {
  HeadBwdJobs jb;
  GammaJob gj;
  gj.F = h.F, gj.Cls = h.Cls, gj.loss_out = nullptr;
  gamma_job_plan(gj);
  jb.fch = gj.fch, jb.nchunks = gj.nchunks, jb.nb_w = gj.nb_w;
  const int V = h.A % 4 == 0 ? 4 : 1;
  const long long total = (long long)h.B * h.Hu * h.Wu * (h.A / V);
  jb.nb_u = (int)((total + HT - 1) / HT);
  jb.nb_t = rj.nb_t + rj.nb_u;
  const dim3 grid((unsigned)(jb.nb_w + jb.nb_u + jb.nb_t + (loss_out ? 1 : 0)));
  if (V == 4)
    hipLaunchKernelGGL(head_bwd_kernel<4>, grid, dim3(HT), 0, st, h, jb, Pq, dz, dWf, dbf, U, dPq, dU, rj,
                       loss_n, loss_out, parg);
  else
    hipLaunchKernelGGL(head_bwd_kernel<1>, grid, dim3(HT), 0, st, h, jb, Pq, dz, dWf, dbf, U, dPq, dU, rj,
                       loss_n, loss_out, parg);
  return hipGetLastError();
}

}  // namespace nf
