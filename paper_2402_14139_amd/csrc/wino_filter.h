// Transformed filters of F(2x2, 3x3) in the fragment order of wino_fwd_kernel (wino_fwd.hip), and the
// job of extra workgroups that re-lays the head's filter for the data gradient (head.hip).
#pragma once
#include "nf_internal.h"

namespace nf {

// U[filter block of nb][step of 8 channels][position a*4+b][n][lane][4], nb = 64: the word of lane (j, h), element
// k is filter 64*block + 2*j + n, channel 8*step + 4*h + k, i.e. the B fragment of one MFMA group; nb = 32: one
// fragment (no n), filter 32*block + j.
constexpr int WINO_CH = 8;
// Filters per workgroup of wino_fwd: 64, or 32 where those would be half padding (wino_fwd.hip)
__host__ __device__ inline int wino_nb(int N) { return N <= 32 ? 32 : 64; }

// U = G g G^T for four consecutive channels 4*c4 .. +3 of filter n, g[r][s] holding their taps
__device__ inline void wino_filter_store(const float4 (&g)[3][3], float *U, int n, int c4, int nchunks, int nb) {
  auto add = [](const float4 &a, const float4 &b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
  auto sub = [](const float4 &a, const float4 &b) { return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w); };
  auto half = [](const float4 &a) { return make_float4(0.5f * a.x, 0.5f * a.y, 0.5f * a.z, 0.5f * a.w); };
  const int in = n & (nb - 1), two = nb >> 6, pos = nb * WINO_CH;  // words per position
  float *o = U + ((long long)(n / nb) * nchunks + (c4 >> 1)) * (16 * pos) + (in & two) * 256 + ((c4 & 1) * 32 + (in >> two)) * 4;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    float4 q[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      if (a == 0) q[s] = g[0][s];
      else if (a == 3) q[s] = g[2][s];
      else q[s] = half(a == 1 ? add(add(g[0][s], g[2][s]), g[1][s]) : sub(add(g[0][s], g[2][s]), g[1][s]));
    }
    const float4 e = add(q[0], q[2]);
    const float4 v[4] = {q[0], half(add(e, q[1])), half(sub(e, q[1])), q[2]};
#pragma unroll
    for (int b = 0; b < 4; ++b) *reinterpret_cast<float4 *>(o + (a * 4 + b) * pos) = v[b];
  }
}

// What block b (256 threads) of a RelayJob does: the first nb_t blocks re-lay, one element per thread,
// WaT[k][r][s][a] = Wa[a][R-1-r][S-1-s][k]; the other nb_u form the transformed filter of that (R = S = 3), four
// channels a of one filter k per thread, lanes along k (coalesced reads of Wa).  Independent of the head's
// samples, so it fills compute units that those leave idle; as a launch of its own in front of wino_fwd it
// took 4-5 us of a step (64 channels, batch 128: step 178 -> 173.5 us).
__device__ inline void relay_block(const RelayJob &j, int b) {
  if (b < j.nb_t) {
    const long long i = (long long)b * 256 + threadIdx.x;
    if (i >= (long long)j.A * j.R * j.S * j.K) return;
    const int a = (int)(i % j.A);
    long long r = i / j.A;
    const int ss = (int)(r % j.S);
    r /= j.S;
    const int rr = (int)(r % j.R), k = (int)(r / j.R);
    j.WaT[i] = j.Wa[(((long long)a * j.R + (j.R - 1 - rr)) * j.S + (j.S - 1 - ss)) * j.K + k];
    return;
  }
  const int nb = wino_nb(j.K), i = (b - j.nb_t) * 256 + threadIdx.x, nk = (j.K + nb - 1) / nb * nb;
  const int k = i % nk, c4 = i / nk;
  if (c4 >= 2 * j.nchunks) return;
  float4 g[3][3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int a = c4 * 4 + e, ac = a < j.A ? a : 0, kc = k < j.K ? k : 0;
        const float x = j.Wa[((long long)ac * 9 + (2 - r) * 3 + (2 - s)) * j.K + kc];
        v[e] = ((a < j.A) & (k < j.K)) ? x : 0.f;
      }
      g[r][s] = make_float4(v[0], v[1], v[2], v[3]);
    }
  wino_filter_store(g, j.U, k, c4, j.nchunks, nb);
}

}  // namespace nf
