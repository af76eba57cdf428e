// mlp_tile.h -- device pieces shared by the network kernels (mlp.hip,
// net_rows.hip): the 16x16x32 MFMA of either half type, rounding helpers, the
// fragment-major weight order and the extended-precision tail layers.
#pragma once

#include "cold_internal.h"

namespace cold {

template <typename TS> struct Mfma;
template <> struct Mfma<__bf16> {
  typedef bf16x8 frag;
  __device__ static inline f32x4 mac(const frag &a, const frag &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma<_Float16> {
  typedef f16x8 frag;
  __device__ static inline f32x4 mac(const frag &a, const frag &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

template <typename TS> struct Pair;
template <> struct Pair<__bf16> {
  typedef __bf16 v2 __attribute__((ext_vector_type(2)));
};
template <> struct Pair<_Float16> {
  typedef _Float16 v2 __attribute__((ext_vector_type(2)));
};

__device__ __forceinline__ uint32_t relu_bits2(uint32_t v) {
  typedef short s2 __attribute__((ext_vector_type(2)));
  const s2 r = __builtin_elementwise_max(__builtin_bit_cast(s2, v), (s2){0, 0});
  return __builtin_bit_cast(uint32_t, r);
}

template <typename TS>
__device__ __forceinline__ uint32_t round2(float lo, float hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  const typename Pair<TS>::v2 h = __builtin_convertvector((f2){lo, hi}, typename Pair<TS>::v2);
  return __builtin_bit_cast(uint32_t, h);
}

// Fragment-major weights of the fused tail: a [N][K] matrix (N % 16 == 0,
// K % 32 == 0) stored as one 1 KB block per (16-feature block fb, 32-deep K
// step k), in MFMA operand order: lane l holds features fb*16 + l % 16, K
// elements 32 k + 8 (l / 16) .. + 8.  A wave then loads a fragment as one
// contiguous 1 KB block instead of 16 half-used cache lines.
__host__ __device__ inline int64_t frag_offset(int fb, int k, int ksteps, int lane) {
  return ((int64_t)(fb * ksteps + k) * 64 + lane) * 8;
}

// the two storage-type values packed in one 32-bit word, widened to fp32
template <typename TS> __device__ __forceinline__ void unpack2(uint32_t w, float &a, float &b);
template <> __device__ __forceinline__ void unpack2<__bf16>(uint32_t w, float &a, float &b) {
  a = __uint_as_float(w << 16);
  b = __uint_as_float(w & 0xFFFF0000u);
}
template <> __device__ __forceinline__ void unpack2<_Float16>(uint32_t w, float &a, float &b) {
  a = static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)(w & 0xFFFFu)));
  b = static_cast<float>(__builtin_bit_cast(_Float16, (uint16_t)(w >> 16)));
}

// hi/lo pairs of two fp32 values (see above); a value whose hi is not finite
// (beyond the storage range) gets lo = 0
template <typename TS>
__device__ __forceinline__ void split2(float v0, float v1, uint32_t &hi, uint32_t &lo) {
  hi = round2<TS>(v0, v1);
  float h0, h1;
  unpack2<TS>(hi, h0, h1);
  const float d0 = __builtin_isfinite(h0) ? v0 - h0 : 0.0f;
  const float d1 = __builtin_isfinite(h1) ? v1 - h1 : 0.0f;
  lo = round2<TS>(d0, d1);
}

// MFMA sums of one tail layer on rows held in LDS: acc[i][j] = sum over K of
// W[n][k] in[r][k] for the 16-row blocks jb0 .. jb0 + JB - 1 and the
// NB 16-feature blocks of wf, from zero, K steps in order. in_at(row, c) is
// the LDS address of 16-byte chunk c of an input row; with EXT the low halves
// of the input sit lo_bytes after the high halves, and each K step adds
// W hi, then W lo. wf[k][i] is the weight fragment of feature block i and K
// step k.
template <typename TS, int KS, int NB, int JB, bool EXT, typename InAt>
__device__ __forceinline__ void tail_mma(const InAt &in_at, int lo_bytes,
                                         const typename Mfma<TS>::frag (&wf)[KS][NB], int jb0,
                                         int lane, f32x4 (&acc)[NB][JB]) {
  typedef typename Mfma<TS>::frag frag;
  const int frow = lane & 15, fq = lane >> 4;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < KS; ++k) {
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const TS *p = in_at((jb0 + j) * 16 + frow, 4 * k + fq);
      const frag fb = *reinterpret_cast<const frag *>(p);
      frag fl;
      if constexpr (EXT) fl = *reinterpret_cast<const frag *>(reinterpret_cast<const char *>(p) + lo_bytes);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        acc[i][j] = Mfma<TS>::mac(wf[k][i], fb, acc[i][j]);
        if constexpr (EXT) acc[i][j] = Mfma<TS>::mac(wf[k][i], fl, acc[i][j]);
      }
    }
  }
}

// bias (bg[i]: this lane's four features of block i), ReLU, then the hi/lo
// pair of every output: row (jb0 + j) * 16 + lane % 16,
// features (nb0 + i) * 16 + 4 (lane / 16) .. + 3; the low halves go lo_elems
// elements after the high halves
template <typename TS, int NB, int JB>
__device__ __forceinline__ void tail_store_ext(const f32x4 (&acc)[NB][JB], const float4 (&bg)[NB],
                                               TS *out, int stride, int lo_elems, int nb0, int jb0,
                                               int lane) {
  const int dn = (lane >> 4) * 4, dr = lane & 15;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int n = (nb0 + i) * 16 + dn;
    const float bv[4] = {bg[i].x, bg[i].y, bg[i].z, bg[i].w};
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = acc[i][j][e] + bv[e];
        v[e] = t > 0.0f ? t : 0.0f;
      }
      uint2 hi, lo;
      split2<TS>(v[0], v[1], hi.x, lo.x);
      split2<TS>(v[2], v[3], hi.y, lo.y);
      TS *o = out + ((jb0 + j) * 16 + dr) * stride + n;
      *reinterpret_cast<uint2 *>(o) = hi;
      *reinterpret_cast<uint2 *>(o + lo_elems) = lo;
    }
  }
}

// bias and ReLU in fp32, stored as fp32 (the last hidden layer)
template <int NB, int JB>
__device__ __forceinline__ void tail_store_f32(const f32x4 (&acc)[NB][JB], const float *__restrict__ bg,
                                               float *out, int stride, int nb0, int jb0, int lane) {
  const int dn = (lane >> 4) * 4, dr = lane & 15;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int n = (nb0 + i) * 16 + dn;
    float bv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) bv[e] = bg[n + e];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      float4 v;
      v.x = acc[i][j][0] + bv[0];
      v.y = acc[i][j][1] + bv[1];
      v.z = acc[i][j][2] + bv[2];
      v.w = acc[i][j][3] + bv[3];
      v.x = v.x > 0.0f ? v.x : 0.0f;
      v.y = v.y > 0.0f ? v.y : 0.0f;
      v.z = v.z > 0.0f ? v.z : 0.0f;
      v.w = v.w > 0.0f ? v.w : 0.0f;
      *reinterpret_cast<float4 *>(out + ((jb0 + j) * 16 + dr) * stride + n) = v;
    }
  }
}

// ---- the tail after a 256-wide layer whose output rows are in the LDS as
// hi/lo pairs: 512-byte rows, 16-byte chunk c of row r at slot c ^ (r & 7),
// the low halves after all PR rows of high halves
constexpr int kTailK = 256, kTailN1 = 128, kTailN2 = 64;
constexpr int kTailHRow = kTailK * 2;
constexpr int kTailS1 = kTailN1 + 8;          // padded LDS row of the first tail layer's output

constexpr int tail_lds_bytes(int PR) {        // first tail layer's pairs, then the head's partial sums
  return 2 * PR * kTailS1 * 2 + PR * (kTailN2 + 4) * 4;
}

// four consecutive features n .. n + 3 of row r: ReLU in fp32, hi/lo pairs
template <typename TS, int PR>
__device__ __forceinline__ void tail_put_pair(const f32x4 &a, unsigned char *hl, int n, int r) {
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = a[e] > 0.0f ? a[e] : 0.0f;
  uint2 hi, lo;
  split2<TS>(v[0], v[1], hi.x, lo.x);
  split2<TS>(v[2], v[3], hi.y, lo.y);
  unsigned char *o = hl + r * kTailHRow + (((n >> 3) ^ (r & 7)) << 4) + (n & 7) * 2;
  *reinterpret_cast<uint2 *>(o) = hi;
  *reinterpret_cast<uint2 *>(o + PR * kTailHRow) = lo;
}

// A wave's tail weights: feature blocks 2 (w % 4) and 2 (w % 4) + 1 of the
// first tail layer, feature block w % 4 of the second, and one head weight
// and bias per thread.
template <typename TS> struct TailWeights {
  typedef typename Mfma<TS>::frag frag;
  static constexpr int KS1 = kTailK / 32, KS2 = kTailN1 / 32;
  frag w1[KS1][2], w2[KS2][1];
  float4 b1[2], b2;      // the biases of this lane's features
  float whv, bhv;
  static __device__ __forceinline__ frag w1_frag(const TailArgs &t, int wave, int lane, int k, int i) {
    return *reinterpret_cast<const frag *>(static_cast<const TS *>(t.w1) +
                                           frag_offset(2 * (wave % 4) + i, k, KS1, lane));
  }
  __device__ __forceinline__ void load_w2(const TailArgs &t, int wave, int lane) {
    const TS *W2 = static_cast<const TS *>(t.w2);
#pragma unroll
    for (int k = 0; k < KS2; ++k)
      w2[k][0] = *reinterpret_cast<const frag *>(W2 + frag_offset(wave % 4, k, KS2, lane));
  }
  __device__ __forceinline__ void load(const TailArgs &t, int wave, int lane, int tid) {
#pragma unroll
    for (int k = 0; k < KS1; ++k)
#pragma unroll
      for (int i = 0; i < 2; ++i) w1[k][i] = w1_frag(t, wave, lane, k, i);
    load_w2(t, wave, lane);
    whv = Elem<TS>::to_f32(static_cast<const TS *>(t.wh)[tid < t.n_out * kTailN2 ? tid : 0]);
    bhv = t.bh[tid < t.n_out ? tid : 0];
  }
  __device__ __forceinline__ void bias_from(const float *v1, const float *v2, int wave, int lane) {
    const int dn = (lane >> 4) * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      b1[i] = *reinterpret_cast<const float4 *>(v1 + (2 * (wave % 4) + i) * 16 + dn);
    b2 = *reinterpret_cast<const float4 *>(v2 + (wave % 4) * 16 + dn);
  }
  __device__ __forceinline__ void load_bias(const TailArgs &t, int wave, int lane) {
    bias_from(t.b1, t.b2, wave, lane);
  }
  // head weights [2][kTailN2], then the two biases
  __device__ __forceinline__ void put_head(float *s_wh, int n_out, int tid) const {
    if (tid < n_out * kTailN2) s_wh[tid] = whv;
    if (tid < n_out) s_wh[2 * kTailN2 + tid] = bhv;
  }
};

// The tail's two layers and the head on PR rows of pairs at hl (complete:
// the caller has passed a barrier); waves split 4 (features) x NW / 4 (rows,
// JB 16-row blocks each). The layers' outputs go to `out` (tail_lds_bytes),
// which is hl's own place with ALIAS. row_of(lr) is the batch row of LDS row
// lr; rows at or past R are not stored. Each wave reads its row group once
// for its two feature blocks of the first layer. The head's sums over a
// block's 16 features come straight from the accumulators: lane (c, q) holds
// features 16 fb + 4 q + e of row c; its four products are added in e order,
// the four quarters by two shuffles, the four blocks in order from LDS.
// LATE: the biases are loaded here (the caller's registers are full before).
// mid() runs once the first layer's weights are dead.
template <typename TS, int PR, int JB, bool ALIAS, bool LATE, typename RowOf, typename Mid>
__device__ __forceinline__ void tail_rows(unsigned char *hl, unsigned char *out,
                                          TailWeights<TS> &tw, const TailArgs &t,
                                          const float *s_wh, float *__restrict__ scores,
                                          const RowOf &row_of, int64_t R, int tid, int lane, int wave,
                                          const Mid &mid) {
  constexpr int KS1 = TailWeights<TS>::KS1, KS2 = TailWeights<TS>::KS2, N2 = kTailN2, S1 = kTailS1;
  TS *s_h1 = reinterpret_cast<TS *>(out);
  float *s_h2 = reinterpret_cast<float *>(out + 2 * PR * S1 * 2);
  const float *s_bh = s_wh + 2 * N2;
  const int n_out = t.n_out, dr = lane & 15;
  auto in0 = [&](int row, int c) {
    return reinterpret_cast<const TS *>(hl + row * kTailHRow + ((c ^ (row & 7)) << 4));
  };
  f32x4 a1[2][JB];
  tail_mma<TS, KS1, 2, JB, true>(in0, PR * kTailHRow, tw.w1, (wave / 4) * JB, lane, a1);
  if (ALIAS) __syncthreads();   // the pairs are dead once every wave has its sums
  if constexpr (LATE) tw.load_bias(t, wave, lane);
  mid();
  tail_store_ext<TS, 2, JB>(a1, tw.b1, s_h1, S1, PR * S1, 2 * (wave % 4), (wave / 4) * JB, lane);
  __syncthreads();
  auto in1 = [&](int row, int c) { return s_h1 + row * S1 + c * 8; };
  f32x4 a2[1][JB];
  tail_mma<TS, KS2, 1, JB, true>(in1, PR * S1 * 2, tw.w2, (wave / 4) * JB, lane, a2);
  {
    const int fb = wave % 4, q4 = lane >> 4;
    const float bb[4] = {tw.b2.x, tw.b2.y, tw.b2.z, tw.b2.w};
    float wz0[4], wz1[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 16 * fb + 4 * q4 + e;
      wz0[e] = s_wh[k];
      wz1[e] = n_out > 1 ? s_wh[N2 + k] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      float z0 = 0.0f, z1 = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = a2[0][j][e] + bb[e];
        v = v > 0.0f ? v : 0.0f;
        z0 += wz0[e] * v;
        z1 += wz1[e] * v;
      }
      z0 += __shfl_xor(z0, 16);
      z0 += __shfl_xor(z0, 32);
      z1 += __shfl_xor(z1, 16);
      z1 += __shfl_xor(z1, 32);
      if (q4 == 0) {
        const int lr = ((wave / 4) * JB + j) * 16 + dr;
        s_h2[(fb * PR + lr) * 2] = z0;
        s_h2[(fb * PR + lr) * 2 + 1] = z1;
      }
    }
  }
  __syncthreads();
  if (tid < PR) {
    const int lr = tid;
    float z0 = s_h2[lr * 2], z1 = s_h2[lr * 2 + 1];
#pragma unroll
    for (int fb = 1; fb < 4; ++fb) {
      z0 += s_h2[(fb * PR + lr) * 2];
      z1 += s_h2[(fb * PR + lr) * 2 + 1];
    }
    const int64_t r = row_of(lr);
    if (r < R) {
      z0 += s_bh[0];
      if (n_out > 1) z1 += s_bh[1];
      scores[r] = n_out == 1 ? 1.0f / (1.0f + expf(-z0)) : 1.0f / (1.0f + expf(z0 - z1));
    }
  }
}

}  // namespace cold
