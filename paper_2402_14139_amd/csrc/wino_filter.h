// Transformed filters of F(2x2, 3x3) in the fragment order of wino_fwd_kernel (wino_fwd.hip), and the
// job of extra workgroups that re-lays the head's filter for the data gradient (head.hip).
#pragma once
#include "nf_internal.h"

namespace nf {

// As pieces (more than 32 filters and 24 channels: wino_fwd_split.hip): U[filter block of 64][step of 16 channels][position
// a*4+b][n][piece][lane][8 bf16], the words of lane (j, h), element k being the three pieces (wino_split2) of filter 64*block + 2*j + n,
// channel 16*step + 8*(k/4) + 4*h + k%4.  In fp32 (wino_fwd.hip): U[filter block of nb][step of 8 channels][position][n][lane][4], nb = 64:
// the word of lane (j, h), element k is filter 64*block + 2*j + n, channel 8*step + 4*h + k; nb = 32: no n, filter 32*block + j.  Either
// is the B fragment of one MFMA or group of MFMAs.
constexpr int WINO_CH = 8, WINO_CH64 = 16;
__host__ __device__ inline int wino_nb(int N) { return N <= 32 ? 32 : 64; }                                   // filters per block
__host__ __device__ inline bool wino_pieces(int N, int C) { return N > 32 && C > 24; }
__host__ __device__ inline int wino_ch(int N, int C) { return wino_pieces(N, C) ? WINO_CH64 : WINO_CH; }      // channels per step
__host__ __device__ constexpr int wino_step_words(int nb, bool pieces) { return 16 * (pieces ? 6 * 256 : nb * WINO_CH); }  // of U, per block

// An fp32 number is the sum of three bf16 numbers, x = h + m + l: h = x to the nearest, m the rest to the nearest, l what is
// then left.  Both remainders are exact and so is l (24 significant bits are three times eight).  (v_dot2_f32_bf16 would take a
// piece off in one instruction, but costs 34 cycles of the matrix pipe beside MFMAs, measured, where four others cost 4.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ inline unsigned wino_pack(float a, float b) {
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2){a, b}, bf16x2));
}
__device__ inline float wino_low(unsigned pair) { return __uint_as_float(pair << 16); }
__device__ inline float wino_high(unsigned pair) { return __uint_as_float(pair & 0xffff0000u); }
// of two numbers, packed
__device__ inline void wino_split2(float x0, float x1, unsigned &h, unsigned &m, unsigned &l) {
  h = wino_pack(x0, x1);
  x0 -= wino_low(h), x1 -= wino_high(h);
  m = wino_pack(x0, x1);
  l = wino_pack(x0 - wino_low(m), x1 - wino_high(m));
}

__device__ inline float4 wino_add4(const float4 &a, const float4 &b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
__device__ inline float4 wino_sub4(const float4 &a, const float4 &b) { return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w); }
__device__ inline float4 wino_half4(const float4 &a) { return make_float4(0.5f * a.x, 0.5f * a.y, 0.5f * a.z, 0.5f * a.w); }
// G on the rows (row a of four, of taps g0 .. g2 of a column), then on the columns (q: that row's three)
__device__ inline float4 wino_filter_row(int a, const float4 &g0, const float4 &g1, const float4 &g2) {
  if (a == 0) return g0;
  if (a == 3) return g2;
  const float4 e = wino_add4(g0, g2);
  return wino_half4(a == 1 ? wino_add4(e, g1) : wino_sub4(e, g1));
}
__device__ inline void wino_filter_columns(const float4 (&q)[3], float4 (&v)[4]) {
  const float4 e = wino_add4(q[0], q[2]);
  v[0] = q[0], v[1] = wino_half4(wino_add4(e, q[1])), v[2] = wino_half4(wino_sub4(e, q[1])), v[3] = q[2];
}
// the pieces of four channels at word o of piece 0, the positions with a + b odd (`odd`) negated: bf16 MFMAs round their running sum
// down, not to nearest, and with every other position's sum of the other sign that cancels in the output transform (wino_fwd_split.hip)
__device__ inline void wino_store_pieces(float *o, const float4 &v, bool odd) {
  const float s = odd ? -1.f : 1.f;
  unsigned w[3][2];
  wino_split2(s * v.x, s * v.y, w[0][0], w[1][0], w[2][0]);
  wino_split2(s * v.z, s * v.w, w[0][1], w[1][1], w[2][1]);
#pragma unroll
  for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2 *>(o + k * 256) = make_uint2(w[k][0], w[k][1]);
}
// where the pieces of row a of the transformed domain, channels 4*c4 .. +3 of filter n begin
__device__ inline float *wino_pieces_at(float *U, int n, int c4, int nchunks, int a) {
  constexpr int words = wino_step_words(64, true);
  return U + ((long long)(n / 64) * nchunks + (c4 >> 2)) * words + a * (words / 4) + (n & 1) * 768 + ((c4 & 1) * 32 + (n & 63) / 2) * 4 +
         (c4 >> 1 & 1) * 2;
}
// the four positions of row a, its three columns of taps in q
__device__ inline void wino_store_row(float *o, const float4 (&q)[3], int a) {
  float4 v[4];
  wino_filter_columns(q, v);
#pragma unroll
  for (int b = 0; b < 4; ++b) wino_store_pieces(o + b * (wino_step_words(64, true) / 16), v[b], (a + b) & 1);
}
// the fp32 form of U = G g G^T for four consecutive channels 4*c4 .. +3 of filter n, g[r][s] holding their taps
__device__ inline void wino_filter_store(const float4 (&g)[3][3], float *U, int n, int c4, int nchunks, int nb) {
  const int in = n & (nb - 1), two = nb >> 6, words = wino_step_words(nb, false);
  float *const o = U + ((long long)(n / nb) * nchunks + (c4 >> 1)) * words + (in & two) * 256 + ((c4 & 1) * 32 + (in >> two)) * 4;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    float4 q[3], v[4];
#pragma unroll
    for (int s = 0; s < 3; ++s) q[s] = wino_filter_row(a, g[0][s], g[1][s], g[2][s]);
    wino_filter_columns(q, v);
#pragma unroll
    for (int b = 0; b < 4; ++b) *reinterpret_cast<float4 *>(o + (a * 4 + b) * (words / 16)) = v[b];
  }
}

// What block b (256 threads) of a RelayJob does: the first nb_t blocks re-lay, one element per thread,
// WaT[k][r][s][a] = Wa[a][R-1-r][S-1-s][k]; the other nb_u form the transformed filter of that (R = S = 3), four
// channels a of one filter k per thread (as pieces: one row of the transformed domain of them; all four in a thread took a head_bwd launch
// of 64 samples, 128 filters, 32-wide head from 5.2 to 6.8 us), lanes along k (coalesced reads of Wa).  Independent of the head's
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
  const int c4s = wino_ch(j.K, j.A) / 4 * j.nchunks, k = i % nk, c4 = i / nk % c4s, row = i / nk / c4s;
  const bool pieces = wino_pieces(j.K, j.A);
  if (row >= (pieces ? 4 : 1)) return;
  auto tap = [&](int r, int s) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int a = c4 * 4 + e, ac = a < j.A ? a : 0, kc = k < j.K ? k : 0;
      const float x = j.Wa[((long long)ac * 9 + (2 - r) * 3 + (2 - s)) * j.K + kc];
      v[e] = ((a < j.A) & (k < j.K)) ? x : 0.f;
    }
    return make_float4(v[0], v[1], v[2], v[3]);
  };
  if (pieces && (row == 0 || row == 3)) {  // (one row of taps)
    float4 q[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) q[s] = tap(row == 0 ? 0 : 2, s);
    wino_store_row(wino_pieces_at(j.U, k, c4, j.nchunks, row), q, row);
    return;
  }
  float4 g[3][3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s) g[r][s] = tap(r, s);
  if (!pieces) {
    wino_filter_store(g, j.U, k, c4, j.nchunks, nb);
    return;
  }
  float4 q[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) q[s] = wino_filter_row(row, g[0][s], g[1][s], g[2][s]);
  wino_store_row(wino_pieces_at(j.U, k, c4, j.nchunks, row), q, row);
}

}  // namespace nf
