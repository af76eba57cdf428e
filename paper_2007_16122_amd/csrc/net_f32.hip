// net_f32.hip -- a small fp32 model (Section 3.1-3.2 and 4.1 at the tiny
// workload's size: at most 64 groups of 8 values, two hidden layers of at
// most 64) from the ids to the CTR in one kernel.
//
// A call of such a model is latency: 512 rows are 0.6 MFLOP each way and a
// few hundred KB, but a gather, two dense layers and a head as kernels of
// their own are four launches and twelve dependent memory round trips
// (19.4 us for 512 rows). Here a workgroup of four waves takes 16 rows
// through everything: ids, table rows, squeeze, SE, reweighting, both layers
// and the head, with three memory round trips (offsets, ids, rows; the
// weights are on their way from the start) and the activations in LDS:
// 6.8 us. It stays ahead to the largest batches (8 x 4,096 rows of 16 groups
// 47.3 -> 22.5 us, of 32 groups 64.7 -> 49.3 us), since the input never goes
// to HBM, so every batch of such a model takes it.
#include "cold_internal.h"
#include "gather_tile.h"

namespace cold {

namespace {

constexpr int kTile = 16;        // rows
constexpr int kStride = 68;      // floats of an LDS row of up to 64 values

// NG: groups per thread (16 threads a row): models of up to 16 NG groups
template <int NG>
__global__ __launch_bounds__(256) void net_f32_kernel(GatherArgs a, NetF32Args n) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(1))) const f4 gl_f4;
  constexpr int KC = NG * 8;                  // 16-deep K chunks of the widest input
  constexpr int XS = KC * 16 + 4;             // floats of an input row in LDS
  __shared__ __align__(16) float s_x[kTile * XS];
  __shared__ __align__(16) float s_z[kTile * kStride], s_s[kTile * kStride];
  __shared__ __align__(16) float s_h1[kTile * kStride], s_h2[kTile * kStride];
  __shared__ int32_t s_req[kGatherMaxReqLds + 1];

  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.M, H = a.H, nu = a.n_user, K0 = M * 8, N1 = n.n1, N2 = n.n2;
  const int64_t R = a.R, Q = a.Q;
  const bool gpu_cross = a.cross_pairs != nullptr, req_lds = Q <= kGatherMaxReqLds;
  // this thread's groups: table, rows, divisor magic (clamped past the model's)
  const int trow = tid >> 4, tg = tid & 15;
  uint64_t tab[NG], magic[NG];
  int32_t nrows[NG], pair[NG];
#pragma unroll
  for (int u = 0; u < NG; ++u) {
    const int g = tg + 16 * u, gc = g < M ? g : 0;
    tab[u] = reinterpret_cast<uint64_t>(a.tables[gc]);
    magic[u] = a.table_magic[gc];
    nrows[u] = (int32_t)a.table_rows[gc];
    const int f = gc - nu - a.n_ad;
    pair[u] = gpu_cross && f >= 0 ? a.cross_pairs[2 * f] | (a.cross_pairs[2 * f + 1] << 16) : 0;
  }
  if (req_lds && Q > 1)
    for (int64_t i = tid; i <= Q; i += 256) s_req[i] = a.req_off[i];
  // request offsets sanity (reported in validate mode)
  for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < Q; i += (int64_t)gridDim.x * 256) {
    bool bad = a.req_off[i + 1] < a.req_off[i];
    if (i == 0) bad |= a.req_off[0] != 0;
    if (i == Q - 1) bad |= (int64_t)a.req_off[Q] != R;
    if (bad) atomicOr(a.err, 2);
  }
  if (req_lds && Q > 1) __syncthreads();

  // operands of the whole launch: SE (packed order, see pack_se_full_kernel)
  // and this wave's 16 features of both layers; zeros past the widths
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  f4 sw1[NG], sw2 = zero, sb1, sb2, w1[KC], w2[4], lb1, lb2;
  auto weights = [&]() {
#pragma unroll
    for (int u = 0; u < NG; ++u) sw1[u] = reinterpret_cast<const f4 *>(a.w1f)[u * 64 + lane];
    sw2 = reinterpret_cast<const f4 *>(a.w2f)[wave * 64 + lane];
    const int f1 = 16 * wave + c;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int kk = 16 * k + 4 * q;
      const bool in = f1 < N1 && kk < K0;
      const f4 v = *reinterpret_cast<const f4 *>(n.w1 + (in ? f1 * K0 + kk : 0));
      w1[k] = in ? v : zero;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int kk = 16 * k + 4 * q;
      const bool in = f1 < N2 && kk < N1;
      const f4 v = *reinterpret_cast<const f4 *>(n.w2 + (in ? f1 * N1 + kk : 0));
      w2[k] = in ? v : zero;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int f = 16 * wave + 4 * q + e, g = 16 * wave + 4 * e + q;
      sb1[e] = 4 * q + e < H ? a.b1[4 * q + e] : 0.0f;
      sb2[e] = g < M ? a.b2[g] : 0.0f;
      lb1[e] = f < N1 ? n.b1[f] : 0.0f;
      lb2[e] = f < N2 ? n.b2[f] : 0.0f;
    }
  };
  bool have_weights = false;

  const int64_t tiles = (R + kTile - 1) / kTile;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t r = tile * kTile + trow;
    const bool row_ok = r < R;
    const int64_t rr = row_ok ? r : R - 1;    // clamped: loaded, never stored
    int64_t rq = 0;
    if (Q > 1) rq = req_lds ? request_of_row(s_req, Q, rr) : request_of_row(a.req_off, Q, rr);
    // ---- ids (int32 ids zero-extended), all in flight together
    uint64_t id[NG], uid[NG];
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      const int g = tg + 16 * u, f = g - nu;
      const bool is_cross = f >= a.n_ad;
      const void *base = f < 0 ? a.user_ids : is_cross && !gpu_cross ? a.cross_ids : a.ad_ids;
      // a cross field built here starts from its ad field's id
      const int fc = is_cross ? (gpu_cross ? pair[u] >> 16 : f - a.n_ad) : f;
      const int64_t at = f < 0 ? (int64_t)g * Q + rq : (int64_t)fc * R + rr;
      id[u] = uid[u] = 0;
      if (g < M) {
        id[u] = a.hashed ? static_cast<const uint64_t *>(base)[at] : static_cast<const uint32_t *>(base)[at];
        if (is_cross && gpu_cross) {
          const int64_t ua = (int64_t)(pair[u] & 0xFFFF) * Q + rq;
          uid[u] = a.hashed ? static_cast<const uint64_t *>(a.user_ids)[ua]
                            : static_cast<const uint32_t *>(a.user_ids)[ua];
        }
      }
    }
    if (!have_weights) {      // behind the first ids, ahead of the rows
      weights();
      have_weights = true;
    }
    // ---- table rows; an absent one reads row 0 and is zeroed
    f4 e0[NG], e1[NG];
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      const int g = tg + 16 * u;
      const bool built = gpu_cross && g - nu >= a.n_ad;   // key = mix64(user id) ^ ad id
      const uint64_t key = built ? mix64(uid[u]) ^ id[u] : id[u];
      const uint64_t salt = (uint64_t)(g + 1) * 0x9e3779b97f4a7c15ull;
      int32_t row = (int32_t)(uint32_t)id[u];
      if (a.hashed || built) row = (int32_t)mod_barrett(mix64(key ^ salt), (uint64_t)nrows[u], magic[u]);
      const bool ok = row >= 0 && row < nrows[u];
      if (g < M && !ok) atomicOr(a.err, 1);
      if (a.rows_out && g < M && row_ok) a.rows_out[(int64_t)g * R + r] = ok ? row : -1;
      const uint64_t at = tab[u] + (uint64_t)(ok ? row : 0) * 32;
      const f4 v0 = *reinterpret_cast<gl_f4 *>(at), v1 = *reinterpret_cast<gl_f4 *>(at + 16);
      const bool there = g < M && ok;
      e0[u] = there ? v0 : zero;
      e1[u] = there ? v1 : zero;
    }
    // ---- squeeze
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      float t = 0.0f;
#pragma unroll
      for (int e = 0; e < 4; ++e) t += e0[u][e];
#pragma unroll
      for (int e = 0; e < 4; ++e) t += e1[u][e];
      s_z[trow * kStride + tg + 16 * u] = t * 0.125f;
    }
    __syncthreads();
    // ---- SE: every wave forms layer 1 of the 16 rows (lane (c, q): units
    // 4 q + e of row c), wave w the weights of groups 16 w + 4 e + q
    {
      f4 h = sb1;
#pragma unroll
      for (int u = 0; u < NG; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          h = __builtin_amdgcn_mfma_f32_16x16x4f32(sw1[u][e], s_z[c * kStride + 4 * (4 * u + e) + q], h, 0, 0, 0);
      if (wave < NG) {
        f4 o = sb2;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o = __builtin_amdgcn_mfma_f32_16x16x4f32(sw2[e], h[e] > 0.0f ? h[e] : 0.0f, o, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) s_s[c * kStride + 16 * wave + 4 * e + q] = 1.0f / (1.0f + expf(-o[e]));
      }
    }
    __syncthreads();
    // ---- reweight, linear_log; groups past the model's hold zeros
    float *X = static_cast<float *>(a.X);
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      const int g = tg + 16 * u;
      const float sw = s_s[trow * kStride + g];
      f4 x0 = sw * e0[u], x1 = sw * e1[u];
      if (a.linear_log) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x0[e] = linear_log(x0[e]);
          x1[e] = linear_log(x1[e]);
        }
      }
      x0 = g < M ? x0 : zero;
      x1 = g < M ? x1 : zero;
      *reinterpret_cast<f4 *>(s_x + trow * XS + 8 * g) = x0;
      *reinterpret_cast<f4 *>(s_x + trow * XS + 8 * g + 4) = x1;
      if (g < M && row_ok) {
        if (X) {
          *reinterpret_cast<f4 *>(X + (r * M + g) * 8) = x0;
          *reinterpret_cast<f4 *>(X + (r * M + g) * 8 + 4) = x1;
        }
        if (a.s_buf) a.s_buf[r * M + g] = sw;
      }
    }
    __syncthreads();
    // ---- hidden layers: wave w the 16 features from 16 w; in a 16-deep
    // chunk lane (c, q) holds k = 4 q .. 4 q + 3 of both operands
    {
      f4 acc = lb1;
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const f4 xv = *reinterpret_cast<const f4 *>(s_x + c * XS + 16 * k + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[k][e], xv[e], acc, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = acc[e] > 0.0f ? acc[e] : 0.0f;
      *reinterpret_cast<f4 *>(s_h1 + c * kStride + 16 * wave + 4 * q) = acc;
    }
    __syncthreads();
    {
      f4 acc = lb2;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f4 xv = *reinterpret_cast<const f4 *>(s_h1 + c * kStride + 16 * k + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[k][e], xv[e], acc, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = acc[e] > 0.0f ? acc[e] : 0.0f;
      *reinterpret_cast<f4 *>(s_h2 + c * kStride + 16 * wave + 4 * q) = acc;
    }
    __syncthreads();
    // ---- head: 16 threads a row, each a sixteenth of the inputs, then four
    // shuffle steps
    float z0 = 0.0f, z1 = 0.0f;
    for (int k = tg; k < N2; k += 16) {
      const float x = s_h2[trow * kStride + k];
      z0 += n.wh[k] * x;
      if (n.n_out > 1) z1 += n.wh[N2 + k] * x;
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      z0 += __shfl_xor(z0, o);
      z1 += __shfl_xor(z1, o);
    }
    if (tg == 0 && row_ok) {
      z0 += n.bh[0];
      if (n.n_out > 1) z1 += n.bh[1];
      n.scores[r] = n.n_out == 1 ? 1.0f / (1.0f + expf(-z0)) : 1.0f / (1.0f + expf(z0 - z1));
    }
    // the next tile's squeeze overwrites s_z, last read two barriers ago; its
    // later arrays are each a barrier or more behind their last readers
  }
}

}  // namespace

bool net_f32_shape(int32_t M, int32_t H, int32_t row_bytes, int32_t n_seq, const int32_t *w, int32_t L) {
  return gather_full_shape(M, H, row_bytes, n_seq) && row_bytes == 32 && n_seq == 0 && L == 3 && w[1] % 4 == 0 && w[1] <= 64 &&
         w[2] <= 64 && (w[3] == 1 || w[3] == 2);
}

template <int NG>
static void net_f32_go(const GatherArgs &g, const NetF32Args &n, hipStream_t s) {
  const int64_t cus = device_cus() > 0 ? device_cus() : 256;
  const int64_t tiles = (g.R + kTile - 1) / kTile;
  // two workgroups per CU, each walking its tiles with the weights in registers
  const unsigned grid = (unsigned)(tiles < 2 * cus ? tiles : 2 * cus);
  hipLaunchKernelGGL((net_f32_kernel<NG>), dim3(grid), dim3(256), 0, s, g, n);
}

hipError_t launch_net_f32(const GatherArgs &g, const NetF32Args &n, hipStream_t s) {
  if (g.R <= 0) return hipSuccess;
  if (!g.w1f || !g.w2f || g.d != 8 || g.M > kFullMaxM || g.H > kFullMaxH || g.n_seq != 0 || n.n1 % 4 != 0 ||
      n.n1 > 64 || n.n2 > 64)
    return hipErrorNotSupported;
  if (g.M <= 16) net_f32_go<1>(g, n, s);
  else if (g.M <= 32) net_f32_go<2>(g, n, s);
  else net_f32_go<4>(g, n, s);
  return hipGetLastError();
}

}  // namespace cold
