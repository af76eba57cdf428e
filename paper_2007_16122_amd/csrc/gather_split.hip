// gather_split.hip -- the register-resident gather with one wave per 16 groups
// of a 16-row tile: models of at most 64 groups and 16 hidden SE units whose
// group rows are 16 or 32 bytes, with or without pooled sequence groups.
//
// Lane l = 16 q + c of wave w owns row c and the groups 16 w + 4 j + q of its
// four slots, as in gather_full_kernel: the squeeze of a group is a sum inside
// one lane. The squeeze of the tile goes to LDS (double-buffered by tile parity,
// one barrier a tile); every wave then forms the whole of layer 1 on the fp32
// MFMAs, its steps in the one-wave form's order, and wave w forms layer 2's
// block w, whose weights land in the lanes that hold the values. So both forms
// give the same bits and the batch may choose between them. A pooled group
// takes its squeeze from the pooling pass and its fp32 values from there when
// it is weighted (one cache line for all rows of a request). The next tile's
// ids load while this tile's rows do.
//   Bound by the random row reads: the 1.28 M-row workload's 64 groups move
// 8.8 GB at 5.0 TB/s, the rate of a large copy. Against the general gather
// (stage events): 64,000 rows of 54 groups, 6 of them pooled, with linear_log
// 97 -> 67 us (a 2,000-ad request 17.2 -> 12.6 us), 9,000 rows of 39 groups
// 23.4 -> 17.1 us, 64,000 rows of 48 groups of 16 bytes 58 -> 46 us, 2,500 rows
// of them 15.9 -> 11.2 us; 60 hashed groups with linear_log 93 -> 81 us (the
// logarithms skipped). Groups of 64 bytes stay with the general gather, which is
// faster on large batches of them (64,000 rows 105 against 120 us).
#include "cold_internal.h"
#include "gather_tile.h"

namespace cold {

namespace {

// floats of a row's squeeze: the MFMA operand reads (16 rows x 4 groups) hit
// 64 banks
constexpr int kZStride = 68;

template <typename TS, int CPG, bool ULDS>
__global__ __launch_bounds__(256, 3) void gather_split_kernel(GatherArgs a) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(1))) const u32x4 gl_u32x4;
  constexpr int EPC = Elem<TS>::kPerChunk;   // elements per 16-byte chunk
  constexpr int EPG = CPG * EPC;             // elements per group (d)
  __shared__ uint64_t s_tab[kFullMaxM];
  __shared__ uint64_t s_magic[kFullMaxM];
  __shared__ int32_t s_rows[kFullMaxM];
  __shared__ int32_t s_pair[kFullMaxM];
  __shared__ int32_t s_req[kGatherMaxReqLds + 1];
  __shared__ float s_z[2][16 * kZStride];   // the tile's squeeze, by tile parity
  extern __shared__ __align__(16) unsigned char s_users[];   // [Q][nu][CPG] chunks, then [nu][Q] rows
  const int M = a.M, H = a.H, nu = a.n_user, ns = a.n_seq, nus = nu + ns, n_ad = a.n_ad;
  const int64_t R = a.R, Q = a.Q;
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = blockDim.x, GB = nt >> 6;   // one wave per 16 groups
  const bool gpu_cross = a.cross_pairs != nullptr;
  for (int g = tid; g < M; g += nt) {
    s_tab[g] = reinterpret_cast<uint64_t>(a.tables[g]);
    s_magic[g] = a.table_magic[g];
    s_rows[g] = (int32_t)a.table_rows[g];
  }
  if (gpu_cross)
    for (int f = tid; f < a.n_cross; f += nt) s_pair[f] = a.cross_pairs[2 * f] | (a.cross_pairs[2 * f + 1] << 16);
  const bool req_in_lds = Q <= kGatherMaxReqLds;
  if (req_in_lds)
    for (int64_t i = tid; i <= Q; i += nt) s_req[i] = a.req_off[i];
  // few requests: their users' rows resolved and staged here (no pooling pass)
  uint4 *s_uval = reinterpret_cast<uint4 *>(s_users);
  int32_t *s_urow = reinterpret_cast<int32_t *>(s_users + (size_t)Q * nu * CPG * 16);
  if (ULDS) {
    for (int64_t i = tid; i < Q * nu * CPG; i += nt) {
      const int p = (int)(i & (CPG - 1));
      const int64_t qq = i / CPG / nu;
      const int f = (int)(i / CPG - qq * nu);
      const int32_t row = a.hashed ? resolve_row<true>(a.user_ids, (int64_t)f * Q + qq, f, a.table_rows[f],
                                                       a.table_magic[f], a.err)
                                   : resolve_row<false>(a.user_ids, (int64_t)f * Q + qq, f, a.table_rows[f],
                                                        a.table_magic[f], a.err);
      uint4 v = make_uint4(0, 0, 0, 0);
      if (row >= 0) v = reinterpret_cast<const uint4 *>(static_cast<const TS *>(a.tables[f]) + (int64_t)row * EPG)[p];
      s_uval[i] = v;
      if (p == 0) s_urow[(int64_t)f * Q + qq] = row;
    }
    // request offsets sanity (the pooling pass checks them otherwise)
    for (int64_t qq = (int64_t)blockIdx.x * nt + tid; qq < Q; qq += (int64_t)gridDim.x * nt) {
      bool bad = a.req_off[qq + 1] < a.req_off[qq];
      if (qq == 0) bad |= a.req_off[0] != 0;
      if (qq == Q - 1) bad |= (int64_t)a.req_off[Q] != R;
      if (bad) atomicOr(a.err, 2);
    }
  }
  // the wave's SE operands
  float4 w1v[kFullMaxM / 16];
#pragma unroll
  for (int u = 0; u < kFullMaxM / 16; ++u) w1v[u] = reinterpret_cast<const float4 *>(a.w1f)[u * 64 + lane];
  const float4 w2v = reinterpret_cast<const float4 *>(a.w2f)[wave * 64 + lane];
  const float w2s[4] = {w2v.x, w2v.y, w2v.z, w2v.w};
  float b1v[4], b2v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    b1v[e] = 4 * q + e < H ? a.b1[4 * q + e] : 0.0f;
    const int g2 = 16 * wave + 4 * e + q;
    b2v[e] = g2 < M ? a.b2[g2] : 0.0f;
  }
  __syncthreads();

  const float inv_d = 1.0f / (float)EPG;             // exact: EPG is a power of two
  const TS *Uh = static_cast<const TS *>(a.Uh);
  TS *X = static_cast<TS *>(a.X);
  const int64_t n_tiles = (R + 15) >> 4;
  // ids of the lane's ad and cross groups, all in flight together (int32 ids
  // zero-extended); a cross field built here starts from its ad field's id
  uint64_t idv[4];
  auto load_ids = [&](int64_t wt) {
    const int64_t r = wt * 16 + c, rr = r < R ? r : R - 1;   // clamped: loaded, never stored
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int g = 16 * wave + 4 * j + q;
      idv[j] = 0;
      if (g >= nus && g < M) {
        const int f = g - nus;
        const bool is_ad = f < n_ad;
        const int fa = is_ad ? f : (gpu_cross ? s_pair[f - n_ad] >> 16 : f - n_ad);
        const void *ids = is_ad || gpu_cross ? a.ad_ids : a.cross_ids;
        const int64_t at = (int64_t)fa * R + rr;
        if (a.hashed) idv[j] = static_cast<const uint64_t *>(ids)[at];
        else idv[j] = static_cast<const uint32_t *>(ids)[at];
      }
    }
  };
  const uint64_t dummy = s_tab[0];                   // row 0 of a table: always present
  auto unpack = [](const u32x4 &u, float *v) { Elem<TS>::unpack(make_uint4(u.x, u.y, u.z, u.w), v); };
  if ((int64_t)blockIdx.x < n_tiles) load_ids(blockIdx.x);
  int parity = 0;
  for (int64_t wt = blockIdx.x; wt < n_tiles; wt += gridDim.x, parity ^= 1) {
    const int64_t r = wt * 16 + c;
    const bool row_ok = r < R;
    const int64_t rr = row_ok ? r : R - 1;
    int64_t rq = 0;
    if (Q > 1 && (nus > 0 || gpu_cross))
      rq = req_in_lds ? request_of_row(s_req, Q, rr) : request_of_row(a.req_off, Q, rr);
    // every chunk of the lane's groups (loads of absent rows read row 0 of a
    // table and are zeroed), and the squeeze of the pooled ones
    u32x4 raw[4][CPG];
    float zs[4];
    uint32_t absent = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int g = 16 * wave + 4 * j + q;
      uint64_t addr = 0;
      zs[j] = 0.0f;
      if (g < M) {
        if (g < nu) {
          if (!ULDS) addr = reinterpret_cast<uint64_t>(Uh + (rq * nu + g) * EPG);
          if (a.rows_out && row_ok)
            a.rows_out[(int64_t)g * R + r] = ULDS ? s_urow[(int64_t)g * Q + rq] : a.urow[rq * nu + g];
        } else if (g < nus) {
          zs[j] = a.zU[rq * nus + g];
          if (a.rows_out && row_ok) a.rows_out[(int64_t)g * R + r] = -1;
        } else {
          int32_t row;
          const int f = g - nus;
          const uint64_t salt = (uint64_t)(g + 1) * 0x9e3779b97f4a7c15ull;
          if (gpu_cross && f >= n_ad) {
            // user x ad cross value: key = mix64(user id) ^ ad id, hashed into
            // the group's table (ids as their unsigned bit patterns)
            const int64_t ua = (int64_t)(s_pair[f - n_ad] & 0xFFFF) * Q + rq;
            const uint64_t uid = a.hashed ? static_cast<const uint64_t *>(a.user_ids)[ua]
                                          : (uint64_t)static_cast<const uint32_t *>(a.user_ids)[ua];
            row = (int32_t)mod_barrett(mix64((mix64(uid) ^ idv[j]) ^ salt), (uint64_t)s_rows[g], s_magic[g]);
          } else if (a.hashed) {
            row = (int32_t)mod_barrett(mix64(idv[j] ^ salt), (uint64_t)s_rows[g], s_magic[g]);
          } else {
            row = (int32_t)(uint32_t)idv[j];
            if (row < 0 || row >= s_rows[g]) {
              atomicOr(a.err, 1);
              row = -1;
            }
          }
          if (a.rows_out && row_ok) a.rows_out[(int64_t)g * R + r] = row;
          if (row >= 0) addr = s_tab[g] + (uint64_t)row * (EPG * sizeof(TS));
        }
      }
      absent |= addr ? 0u : 1u << j;
      const uint64_t at = addr ? addr : dummy;
#pragma unroll
      for (int p = 0; p < CPG; ++p) raw[j][p] = *reinterpret_cast<gl_u32x4 *>(at + 16 * p);
    }
    if (wt + gridDim.x < n_tiles) load_ids(wt + gridDim.x);
    // squeeze
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int g = 16 * wave + 4 * j + q;
      if (absent >> j & 1) {
#pragma unroll
        for (int p = 0; p < CPG; ++p)
          raw[j][p] = ULDS && g < nu ? reinterpret_cast<const u32x4 *>(s_uval)[(rq * nu + g) * CPG + p]
                                     : u32x4{0, 0, 0, 0};
      }
      float t = 0.0f;
#pragma unroll
      for (int p = 0; p < CPG; ++p) {
        float v[EPC];
        unpack(raw[j][p], v);
#pragma unroll
        for (int e = 0; e < EPC; ++e) t += v[e];
      }
      s_z[parity][c * kZStride + g] = g >= nu && g < nus ? zs[j] : t * inv_d;
    }
    __syncthreads();
    // the rows are unpacked again below: their fp32 values are not kept
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int p = 0; p < CPG; ++p) asm volatile("" : "+v"(raw[j][p]));
    // layer 1, whole, by every wave, its steps in gather_full_kernel's order
    // (slots past the model's groups: zero weights, and the waves that would
    // write their squeeze may not exist)
    f32x4 h;
    h[0] = b1v[0]; h[1] = b1v[1]; h[2] = b1v[2]; h[3] = b1v[3];
#pragma unroll
    for (int u = 0; u < kFullMaxM / 16; ++u)
      if (u < GB) {
        const float w[4] = {w1v[u].x, w1v[u].y, w1v[u].z, w1v[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          h = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], s_z[parity][c * kZStride + 4 * (4 * u + e) + q], h, 0, 0, 0);
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = h[e] > 0.0f ? h[e] : 0.0f;
    // layer 2, block gb = wave: the weight of slot j in element j
    f32x4 o;
    o[0] = b2v[0]; o[1] = b2v[1]; o[2] = b2v[2]; o[3] = b2v[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) o = __builtin_amdgcn_mfma_f32_16x16x4f32(w2s[e], h[e], o, 0, 0, 0);
    // reweight, linear_log, round once, store the group's chunks
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int g = 16 * wave + 4 * j + q;
      const float sw = 1.0f / (1.0f + expf(-o[j]));
      float v[EPG];
#pragma unroll
      for (int p = 0; p < CPG; ++p) unpack(raw[j][p], v + p * EPC);
      if (ns > 0 && g >= nu && g < nus) {
        const float4 *src = reinterpret_cast<const float4 *>(a.U + (rq * nus + g) * EPG);
#pragma unroll
        for (int i = 0; i < EPG / 4; ++i) {
          const float4 u = src[i];
          v[4 * i] = u.x; v[4 * i + 1] = u.y; v[4 * i + 2] = u.z; v[4 * i + 3] = u.w;
        }
      }
#pragma unroll
      for (int e = 0; e < EPG; ++e) v[e] = sw * v[e];
      if (a.linear_log) linear_log_all(v);
      if (row_ok && g < M) {
        uint4 *dst = reinterpret_cast<uint4 *>(X + (r * M + g) * EPG);
#pragma unroll
        for (int p = 0; p < CPG; ++p) dst[p] = Elem<TS>::pack(v + p * EPC);
        if (a.s_buf) a.s_buf[r * M + g] = sw;
      }
    }
  }
}

template <typename TS, int CPG>
hipError_t gather_split_c(bool ulds, const GatherArgs &a, hipStream_t s) {
  const void *k = ulds ? reinterpret_cast<const void *>(&gather_split_kernel<TS, CPG, true>)
                       : reinterpret_cast<const void *>(&gather_split_kernel<TS, CPG, false>);
  const size_t shmem = ulds ? (size_t)a.Q * a.n_user * (CPG * 16 + 4) : 0;
  const int threads = 64 * ((a.M + 15) / 16);
  const int64_t resident = resident_blocks(k, threads, shmem);
  int64_t nb = (a.R + 15) / 16;
  if (resident > 0 && nb > resident) nb = resident;
  if (ulds) hipLaunchKernelGGL((gather_split_kernel<TS, CPG, true>), dim3((unsigned)nb), dim3(threads), shmem, s, a);
  else hipLaunchKernelGGL((gather_split_kernel<TS, CPG, false>), dim3((unsigned)nb), dim3(threads), shmem, s, a);
  return hipGetLastError();
}

template <typename TS>
hipError_t gather_split_t(bool ulds, const GatherArgs &a, hipStream_t s) {
  switch (a.d / Elem<TS>::kPerChunk) {
    case 1: return gather_split_c<TS, 1>(ulds, a, s);
    case 2: return gather_split_c<TS, 2>(ulds, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// users' rows in LDS when the pooling pass does not run
hipError_t launch_gather_split(int dtype, const GatherArgs &a, hipStream_t s) {
  if (a.R <= 0) return hipSuccess;
  if (!gather_full_supported(dtype, a)) return hipErrorInvalidValue;
  const bool ulds = !user_pool_needed(dtype, a);
  switch (dtype) {
    case kF32: return gather_split_t<float>(ulds, a, s);
    case kBF16: return gather_split_t<__bf16>(ulds, a, s);
    default: return gather_split_t<_Float16>(ulds, a, s);
  }
}

}  // namespace cold
