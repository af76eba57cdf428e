// se_literal.hip -- Eq. 2 of Section 3.2 as printed, s = sigmoid(W e + b) with
// e the concatenated embedding of a row, on the half-precision matrix cores
// at fp32 precision.
//
// The gathered rows are exact in the storage type, so only W needs more than
// it: each fp32 weight is the sum of three storage-type values (8 bits each
// in bf16, 11 in fp16 after scaling the row of W to the top of the fp16
// range), and a product of one of them with a stored value is exact in
// fp32. Three MFMAs of 32 products take the place of eight of 4 in fp32 and
// the rows are read as they are stored: 64,000 rows x 768 x 48 125 -> 42 us
// (2.6 TB/s of rows read and weights written), the gather before it writes
// 98 MB instead of 197 MB (88 -> 54 us), and the gather after it is gone (60 us):
// large batches weigh the rows as the network reads them (net_rows.hip, 4 us
// more there), smaller ones in this kernel. Whole call 429 -> 256 us, one
// 2,000-ad request 53 -> 39 us. The sum has an eighth of the fp32 kernel's
// roundings (24 K steps of three parts against 192); the weights are off from 64
// bits by 6.6e-8 in the mean square against 1.1e-7 before (fp16 6.5e-8
// against 1.2e-7, 3,200 values 1.3e-7 against 2.2e-7).
#include "cold_internal.h"
#include "gather_tile.h"
#include "mlp_tile.h"

namespace cold {

namespace {

constexpr int kParts = 3;
constexpr int kRB = 4;          // 16-row blocks of a wave

// One workgroup per 16 features: row n of W [N][K] as kParts fragment-major
// matrices (zeros past N and K) and the factor that undoes its scaling.
template <typename TS>
__global__ __launch_bounds__(256) void pack_literal_kernel(const float *__restrict__ W, int32_t N,
                                                           int32_t K, TS *__restrict__ out,
                                                           float *__restrict__ unscale) {
  __shared__ float s_max[4];
  const int n = blockIdx.x, tid = threadIdx.x, ks = (K + 31) / 32, nfb = (N + 15) / 16;
  float scale = 1.0f;
  if constexpr (__is_same(TS, _Float16)) {
    float m = 0.0f;
    if (n < N)
      for (int k = tid; k < K; k += 256) m = fmaxf(m, fabsf(W[(int64_t)n * K + k]));
    for (int o = 32; o; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((tid & 63) == 0) s_max[tid >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    // a power of two that puts the largest magnitude in [2^14, 2^15)
    if (m > 0.0f && m < INFINITY) {
      int e = 14 - (int)((__float_as_uint(m) >> 23) & 0xFF) + 127;
      e = e > 126 ? 126 : (e < -126 ? -126 : e);
      scale = __uint_as_float((uint32_t)(e + 127) << 23);
    }
  }
  if (tid == 0) unscale[n] = 1.0f / scale;
  for (int k = tid; k < ks * 32; k += 256) {
    const float w = n < N && k < K ? W[(int64_t)n * K + k] * scale : 0.0f;
    TS p[kParts];
    float rest = w;
#pragma unroll
    for (int i = 0; i < kParts; ++i) {
      if constexpr (__is_same(TS, __bf16)) {
        // the top 8 bits, cut: three cuts hold all 24
        p[i] = __builtin_bit_cast(__bf16, (uint16_t)(__float_as_uint(rest) >> 16));
      } else {
        p[i] = static_cast<_Float16>(rest);
      }
      const float h = Elem<TS>::to_f32(p[i]);
      rest = __builtin_isfinite(h) ? rest - h : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < kParts; ++i)
      out[(int64_t)i * nfb * ks * 512 + frag_offset(n >> 4, k >> 5, ks, ((k & 31) >> 3) * 16 + (n & 15)) + (k & 7)] = p[i];
  }
}

// w . x in fp32, 8 values a step: the sum where the split one is not finite.
// An infinite value times a zero part of a weight, or parts of opposite signs,
// would make a NaN of what is an infinity.
template <typename TS, typename Chunk>
__device__ __forceinline__ float whole_dot(const float *__restrict__ w, int nch, const Chunk &chunk) {
  float t = 0.0f;
#pragma unroll 1
  for (int ch = 0; ch < nch; ++ch) {
    float v[8];
    Elem<TS>::unpack(chunk(ch), v);
#pragma unroll
    for (int e = 0; e < 8; ++e) t = fmaf(w[8 * ch + e], v[e], t);
  }
  return t;
}

// Rows of at most kTileMaxK values: a workgroup of four waves holds 16 RB
// whole rows in LDS, so the layer has one barrier; wave w takes the feature
// blocks w, w + 4, ..., its weights streaming from L2 four K steps ahead. Two
// row blocks (three workgroups a CU at 768 values) halve the weight traffic;
// one while that would leave CUs without a workgroup. With APPLY the rows are
// then weighted, normalised (Eq. 3) and rounded in place from the LDS.
constexpr int kTileMaxK = 1024;

template <typename TS, int RB, bool APPLY>
__global__ __launch_bounds__(256) void se_literal_tile_kernel(TS *__restrict__ X, const float *__restrict__ W,
                                                              const TS *__restrict__ Wp,
                                                              const float *__restrict__ unscale,
                                                              const float *__restrict__ bias,
                                                              float *__restrict__ s, int64_t R, int32_t M,
                                                              int32_t K, int lcpg, int linear_log_on) {
  typedef typename Mfma<TS>::frag frag;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = (K + 31) / 32, nfb = (M + 15) / 16, nch = K / 8, nu = (nch + 15) / 16;
  const int row_bytes = nu * 256, ss = M + 1;              // LDS row strides: bytes; floats
  float *s_s = reinterpret_cast<float *>(smem + 16 * RB * row_bytes);
  const int64_t r0 = (int64_t)blockIdx.x * (16 * RB);
  // 16-byte chunk ch of row r of the tile: permuted within 16 chunks by the row
  auto at = [&](int r, int ch) { return smem + r * row_bytes + ((ch ^ (r & 15)) << 4); };
  const int64_t part = (int64_t)nfb * ks * 512;
  constexpr int D = 4;                                     // K steps of weights in flight
  frag w[D][kParts];
  auto load_w = [&](int fb, int k, frag (&v)[kParts]) {
    const TS *p = Wp + ((int64_t)fb * ks + (k < ks ? k : ks - 1)) * 512 + lane * 8;
#pragma unroll
    for (int i = 0; i < kParts; ++i) v[i] = *reinterpret_cast<const frag *>(p + i * part);
  };
  const int trow = tid >> 4, tch = tid & 15;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int64_t r = r0 + 16 * b + trow;
    const TS *xp = X + (r < R ? r : R - 1) * K;            // clamped: loaded, never stored
    uint4 v[kTileMaxK / 128];
#pragma unroll
    for (int u = 0; u < kTileMaxK / 128; ++u)
      if (u < nu) {
        const int ch = tch + 16 * u;
        v[u] = *reinterpret_cast<const uint4 *>(xp + (ch < nch ? ch : nch - 1) * 8);
        if (ch >= nch) v[u] = make_uint4(0, 0, 0, 0);      // past the row's end
      }
    if (b == 0 && wave < nfb)
#pragma unroll
      for (int d = 0; d < D; ++d) load_w(wave, d, w[d]);
#pragma unroll
    for (int u = 0; u < kTileMaxK / 128; ++u)
      if (u < nu) *reinterpret_cast<uint4 *>(at(16 * b + trow, tch + 16 * u)) = v[u];
  }
  __syncthreads();
  for (int fb = wave; fb < nfb; fb += 4) {
    if (fb != wave)
#pragma unroll
      for (int d = 0; d < D; ++d) load_w(fb, d, w[d]);
    f32x4 acc[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < ks; k0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (k0 + d < ks) {                                 // small parts first
          frag x[RB];
#pragma unroll
          for (int j = 0; j < RB; ++j) x[j] = *reinterpret_cast<const frag *>(at(16 * j + c, 4 * (k0 + d) + q));
#pragma unroll
          for (int p = kParts - 1; p >= 0; --p)
#pragma unroll
            for (int j = 0; j < RB; ++j) acc[j] = Mfma<TS>::mac(w[d][p], x[j], acc[j]);
        }
        load_w(fb, k0 + d + D, w[d]);
      }
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      const int64_t r = r0 + 16 * j + c;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = fb * 16 + 4 * q + e;
        if (n < M) {
          float t = acc[j][e] * unscale[n] + bias[n];
          if (!__builtin_isfinite(acc[j][e]))
            t = whole_dot<TS>(W + (int64_t)n * K, nch, [&](int ch) {
                  return *reinterpret_cast<const uint4 *>(at(16 * j + c, ch));
                }) + bias[n];
          const float sv = 1.0f / (1.0f + expf(-t));
          if (r < R) s[r * M + n] = sv;
          if (APPLY) s_s[(16 * j + c) * ss + n] = sv;
        }
      }
    }
  }
  if constexpr (APPLY) {
    __syncthreads();
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const int t = 16 * b + trow;
      const int64_t r = r0 + t;
      if (r < R)
        for (int ch = tch; ch < nch; ch += 16) {
          const float sv = s_s[t * ss + (ch >> lcpg)];
          float v[8];
          Elem<TS>::unpack(*reinterpret_cast<const uint4 *>(at(t, ch)), v);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = sv * v[e];
          if (linear_log_on)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = linear_log(v[e]);
          *reinterpret_cast<uint4 *>(X + r * K + ch * 8) = Elem<TS>::pack(v);
        }
    }
  }
}

// Longer rows: a wave takes 64 rows and 16 features straight from global
// memory; the waves of a workgroup take the features of the same rows first.
template <typename TS>
__global__ __launch_bounds__(256) void se_literal_kernel(const TS *__restrict__ X, const float *__restrict__ W,
                                                         const TS *__restrict__ Wp,
                                                         const float *__restrict__ unscale,
                                                         const float *__restrict__ bias,
                                                         float *__restrict__ s, int64_t R, int32_t M,
                                                         int32_t K, int64_t n_waves) {
  typedef typename Mfma<TS>::frag frag;
  const int lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ks = (K + 31) / 32, nfb = (M + 15) / 16, nch = K / 8;
  const int64_t gw = (int64_t)blockIdx.x * 4 + wave;
  if (gw >= n_waves) return;
  const int fb = (int)(gw % nfb);
  const int64_t r0 = gw / nfb * (16 * kRB);
  const TS *xp[kRB];
#pragma unroll
  for (int j = 0; j < kRB; ++j) {
    const int64_t r = r0 + 16 * j + c;
    xp[j] = X + (r < R ? r : R - 1) * K;         // clamped: loaded, never stored
  }
  const TS *wp = Wp + (int64_t)fb * ks * 512 + lane * 8;
  const int64_t part = (int64_t)nfb * ks * 512;
  auto load = [&](int k, frag (&x)[kRB], frag (&w)[kParts]) {
    const int ch = 4 * k + q;
#pragma unroll
    for (int j = 0; j < kRB; ++j) {
      uint4 v = *reinterpret_cast<const uint4 *>(xp[j] + (ch < nch ? ch : nch - 1) * 8);
      if (ch >= nch) v = make_uint4(0, 0, 0, 0);   // past the row's end
      x[j] = __builtin_bit_cast(frag, v);
    }
#pragma unroll
    for (int p = 0; p < kParts; ++p) w[p] = *reinterpret_cast<const frag *>(wp + p * part + k * 512);
  };
  f32x4 acc[kRB];
#pragma unroll
  for (int j = 0; j < kRB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int D = 4;                            // K steps in flight
  frag x[D][kRB], w[D][kParts];
#pragma unroll
  for (int d = 0; d < D; ++d) load(d < ks ? d : ks - 1, x[d], w[d]);
  for (int k0 = 0; k0 < ks; k0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (k0 + d < ks) {                          // small parts first
#pragma unroll
        for (int p = kParts - 1; p >= 0; --p)
#pragma unroll
          for (int j = 0; j < kRB; ++j) acc[j] = Mfma<TS>::mac(w[d][p], x[d][j], acc[j]);
      }
      load(k0 + d + D < ks ? k0 + d + D : ks - 1, x[d], w[d]);
    }
  }
#pragma unroll
  for (int j = 0; j < kRB; ++j) {
    const int64_t r = r0 + 16 * j + c;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = fb * 16 + 4 * q + e;
      if (r < R && n < M) {
        float t = acc[j][e] * unscale[n] + bias[n];
        if (!__builtin_isfinite(acc[j][e]))
          t = whole_dot<TS>(W + (int64_t)n * K, nch, [&](int ch) {
                return *reinterpret_cast<const uint4 *>(xp[j] + 8 * ch);
              }) + bias[n];
        s[r * M + n] = 1.0f / (1.0f + expf(-t));
      }
    }
  }
}

}  // namespace

// storage-type elements of the packed weights, and features with scale factors
size_t literal_packed_elems(int32_t M, int32_t K) {
  return (size_t)kParts * ((M + 15) / 16) * ((K + 31) / 32) * 512;
}
int32_t literal_features(int32_t M) { return (M + 15) / 16 * 16; }

hipError_t launch_pack_literal(int dtype, const float *w, int32_t M, int32_t K, void *wp, float *unscale,
                               hipStream_t s) {
  const dim3 grid((unsigned)literal_features(M));
  if (dtype == kBF16)
    hipLaunchKernelGGL(pack_literal_kernel<__bf16>, grid, dim3(256), 0, s, w, M, K, static_cast<__bf16 *>(wp), unscale);
  else if (dtype == kF16)
    hipLaunchKernelGGL(pack_literal_kernel<_Float16>, grid, dim3(256), 0, s, w, M, K, static_cast<_Float16 *>(wp), unscale);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <typename TS>
static hipError_t se_literal_t(void *x, const float *w, const void *wp, const float *unscale, const float *b, float *s_out,
                               int64_t R, int32_t M, int32_t K, int32_t d, bool apply, bool ll, hipStream_t s) {
  TS *X = static_cast<TS *>(x);
  const TS *Wp = static_cast<const TS *>(wp);
  if (K > kTileMaxK) {
    if (apply) return hipErrorInvalidValue;
    const int64_t n_waves = (R + 16 * kRB - 1) / (16 * kRB) * ((M + 15) / 16);
    if (n_waves > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(se_literal_kernel<TS>, dim3((unsigned)((n_waves + 3) / 4)), dim3(256), 0, s, X, w, Wp,
                       unscale, b, s_out, R, M, K, n_waves);
    return hipGetLastError();
  }
  const int64_t cus = device_cus() > 0 ? device_cus() : 256;
  const int rb = (R + 31) / 32 >= 2 * cus ? 2 : 1;
  const int64_t blocks = (R + 16 * rb - 1) / (16 * rb);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const size_t shmem = (size_t)16 * rb * ((K / 8 + 15) / 16 * 256) + (apply ? sizeof(float) * 16 * rb * (M + 1) : 0);
  const int lcpg = __builtin_ctz(d / 8);
  const dim3 grid((unsigned)blocks);
  if (rb == 2 && apply)
    hipLaunchKernelGGL((se_literal_tile_kernel<TS, 2, true>), grid, dim3(256), shmem, s, X, w, Wp, unscale, b, s_out, R, M, K, lcpg, ll);
  else if (rb == 2)
    hipLaunchKernelGGL((se_literal_tile_kernel<TS, 2, false>), grid, dim3(256), shmem, s, X, w, Wp, unscale, b, s_out, R, M, K, lcpg, ll);
  else if (apply)
    hipLaunchKernelGGL((se_literal_tile_kernel<TS, 1, true>), grid, dim3(256), shmem, s, X, w, Wp, unscale, b, s_out, R, M, K, lcpg, ll);
  else
    hipLaunchKernelGGL((se_literal_tile_kernel<TS, 1, false>), grid, dim3(256), shmem, s, X, w, Wp, unscale, b, s_out, R, M, K, lcpg, ll);
  return hipGetLastError();
}

bool se_literal_applies(int32_t K) { return K <= kTileMaxK; }

hipError_t launch_se_literal(int dtype, void *x, const float *w, const void *wp, const float *unscale, const float *b,
                             float *s_out, int64_t R, int32_t M, int32_t K, int32_t d, bool apply, bool ll,
                             hipStream_t s) {
  if (R <= 0) return hipSuccess;
  if (K % 8 != 0 || d < 8 || (d & (d - 1)) != 0 || M * d != K) return hipErrorInvalidValue;
  if (dtype == kBF16) return se_literal_t<__bf16>(x, w, wp, unscale, b, s_out, R, M, K, d, apply, ll, s);
  if (dtype == kF16) return se_literal_t<_Float16>(x, w, wp, unscale, b, s_out, R, M, K, d, apply, ll, s);
  return hipErrorInvalidValue;
}

}  // namespace cold
