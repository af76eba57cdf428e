// net_rows.hip -- the whole network of the COLD model (Section 4.1) over row
// tiles: D_in x 1024 x 512 x 256 x 128 x 64 x {1, 2} (and the lighter D_in x
// 512 x 256 x 128 x 64 x {1, 2}) in one kernel, for batches of many rows.
//
// A workgroup (8 waves, one per CU, persistent) takes 64 rows through every
// layer. The activations never leave the LDS: 64 rows of the 1024-wide layer
// are 128 KB, which is what fixes the tile height. The waves split a layer's
// features; each streams its own weight fragments from L2 straight into
// registers (fragment-major, 1 KB per load, 16 in flight), so a layer has no
// barrier in its K loop, only one on either side of writing its output. A
// layer's last K steps load the next layer's first fragments, and the next
// tile's input rows and first fragments load under the tail.
//   What bounds it: every weight byte enters the CU once per 64 rows, 64 bytes
// per MFMA cycle, which is what a CU's vector L1 delivers; a tile takes 73,000
// cycles against 47,000 of MFMAs alone. With all CUs busy the clock then
// falls (1.9-2.1 GHz), so the sustained rate is near the library's large
// matrix product on the same card (1,200-1,290 TFLOP/s). Without the weight
// loads it would run at 1,510, without the LDS reads at 1,270 TFLOP/s.
//   Measured against the layer-by-layer path (stage events): 64,000 rows of
// D_in 768 203 -> 157 us (1,210 TFLOP/s), D_in 1024 230 -> 187 us; 16,500
// rows 102 -> 79 us; 8,000 rows 57 -> 40 us. Fewer than 96 tiles leave too
// many CUs idle: see net_rows_chosen.
//   Every sum runs over the same 32-deep K blocks in the same order as the
// layer-by-layer path, so a score does not depend on which one computed it.
#include "cold_internal.h"
#include "gather_tile.h"
#include "mlp_tile.h"

namespace cold {

namespace {

constexpr int kRows = 64;        // rows of a tile
constexpr int kWaves = 8;
constexpr int kNetRowsMaxK = 1024;   // widest input: a tile's rows stay in the LDS

// LDS writes of this wave done, then the workgroup's barrier; loads from
// global memory stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  compiler_fence();
  wait_vm<63>();
  __builtin_amdgcn_s_barrier();
  compiler_fence();
}

// 16-byte chunk c of row r of a tile held with STRIDE bytes per row: chunks
// permuted by the row, so that 16 rows' reads of one chunk hit 16 slots
template <int STRIDE>
__device__ __forceinline__ int row_slot(int r, int c) {
  return r * STRIDE + ((c ^ (r & 15)) << 4);
}

// A layer's fragment-major weights as seen by one wave, from its first
// feature block: fragment (i, k) is one buffer load whose lane offset is
// fixed and whose place is scalar.
template <typename TS> struct WaveWeights {
  typedef typename Mfma<TS>::frag frag;
  __amdgpu_buffer_rsrc_t rsrc;
  int voff, ksteps;
  __device__ __forceinline__ WaveWeights(const void *w, int n_blocks, int first_block, int ks, int lane)
      : voff(lane * 16), ksteps(ks) {
    const char *base = static_cast<const char *>(w) + (int64_t)first_block * ks * 1024;
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), (short)0,
                                             (n_blocks - first_block) * ks * 1024, 0x00020000);
  }
  __device__ __forceinline__ frag load(int i, int k) const {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, (i * ksteps + k) * 1024, 0);
    return __builtin_bit_cast(frag, v);
  }
};

// The weight fragments in flight: kQueue of them per wave, D = kQueue / NI K
// steps of a layer with NI feature blocks. Fragment (step s, block i) of the
// current round is wq[(s NI + i + OFF) % kQueue].
constexpr int kQueue = 16;

// One K step: NI x RJ MFMAs; each weight fragment, once used, is replaced by
// refill(its index in the round)
template <typename TS, int NI, int RJ, int OFF, typename Refill>
__device__ __forceinline__ void k_step(int s, typename Mfma<TS>::frag (&wq)[kQueue],
                                       const typename Mfma<TS>::frag (&xf)[RJ], f32x4 (&acc)[NI][RJ],
                                       const Refill &refill) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    typename Mfma<TS>::frag &w = wq[(s * NI + i + OFF) % kQueue];
#pragma unroll
    for (int j = 0; j < RJ; ++j) acc[i][j] = Mfma<TS>::mac(w, xf[j], acc[i][j]);
    w = refill(i);
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, RJ, 0);   // MFMAs
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);    // the load
  }
}

// One layer whose input rows are in LDS: acc += W in^T over ks K steps, a
// wave's NI feature blocks over RJ row blocks. wq holds the layer's first D
// steps on entry; the last ones are replaced by next(0), next(1), ..., the
// following layer's first fragments, so that its loads run under this
// layer's MFMAs. ks is a multiple of D, or one more (ODD, D = 2): then the
// next layer's fragments start at wq[(OFF + NI) % kQueue].
template <typename TS, int NI, int RJ, int D, int OFF, bool ODD, typename InAt, typename Next>
__device__ __forceinline__ void lds_layer(const WaveWeights<TS> &w, int ks, const InAt &in_at,
                                          typename Mfma<TS>::frag (&wq)[kQueue], f32x4 (&acc)[NI][RJ],
                                          const Next &next) {
  typedef typename Mfma<TS>::frag frag;
  static_assert(D % 2 == 0 && D * NI <= kQueue && (!ODD || D == 2), "rounds of the queue");
  frag xf[2][RJ];
  auto read = [&](int k, frag (&x)[RJ]) {
#pragma unroll
    for (int j = 0; j < RJ; ++j) x[j] = *reinterpret_cast<const frag *>(in_at(j, k));
    __builtin_amdgcn_sched_group_barrier(0x100, RJ, 0);
  };
  read(0, xf[0]);
  int k0 = 0;
#pragma unroll 1
  for (; k0 < ks - D - (ODD ? 1 : 0); k0 += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      read(k0 + s + 1, xf[(s + 1) & 1]);
      k_step<TS, NI, RJ, OFF>(s, wq, xf[s & 1], acc, [&](int i) { return w.load(i, k0 + s + D); });
    }
  }
  if constexpr (ODD) {
    read(k0 + 1, xf[1]);
    k_step<TS, NI, RJ, OFF>(0, wq, xf[0], acc, [&](int i) { return w.load(i, k0 + 2); });
    read(k0 + 2, xf[0]);
    k_step<TS, NI, RJ, OFF>(1, wq, xf[1], acc, [&](int i) { return next(i); });
    k_step<TS, NI, RJ, OFF>(0, wq, xf[0], acc, [&](int i) { return next(kQueue - NI + i); });
  } else {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      if (s + 1 < D) read(k0 + s + 1, xf[(s + 1) & 1]);
      k_step<TS, NI, RJ, OFF>(s, wq, xf[s & 1], acc, [&](int i) { return next(s * NI + i); });
    }
  }
}

// accumulators start at the biases of the lane's features (b: in LDS)
template <int NI, int RJ>
__device__ __forceinline__ void start_at(const float *b, f32x4 (&acc)[NI][RJ]) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const float4 v = *reinterpret_cast<const float4 *>(b + i * 16);
#pragma unroll
    for (int j = 0; j < RJ; ++j) acc[i][j] = f32x4{v.x, v.y, v.z, v.w};
  }
}

// nothing moves across: keeps the next phase's registers out of this one's
__device__ __forceinline__ void phase_end() {
  compiler_fence();
  __builtin_amdgcn_sched_barrier(0);
}
// the same once the sums are formed (a product is no memory operation, so a
// fence alone does not hold it back)
template <int NI, int RJ> __device__ __forceinline__ void phase_end(f32x4 (&acc)[NI][RJ]) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < RJ; ++j) asm volatile("" : "+v"(acc[i][j]));
  phase_end();
}

// ReLU and one rounding to the storage type, into rows of STRIDE bytes
template <typename TS, int NI, int RJ, int STRIDE>
__device__ __forceinline__ void store_act(const f32x4 (&acc)[NI][RJ], unsigned char *out, int n0, int r0) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int n = n0 + i * 16;
#pragma unroll
    for (int j = 0; j < RJ; ++j) {
      uint2 p;
      p.x = relu_bits2(round2<TS>(acc[i][j][0], acc[i][j][1]));
      p.y = relu_bits2(round2<TS>(acc[i][j][2], acc[i][j][3]));
      *reinterpret_cast<uint2 *>(out + row_slot<STRIDE>(r0 + j * 16, n >> 3) + (n & 7) * 2) = p;
    }
  }
}

}  // namespace

template <typename TS, int N0, int N1, int NX, bool ODD, bool WEIGH>
__global__ __launch_bounds__(64 * kWaves, 1) void net_rows_kernel(NetRowsArgs a) {
  typedef typename Mfma<TS>::frag frag;
  constexpr int NI0 = N0 / kWaves / 16;                 // first layer: 16-wide blocks of a wave
  constexpr int RJ = kRows / 16;
  constexpr int NL = N1 > 0 ? N1 : N0;                  // width before the 256-wide layer
  constexpr int XROW = kNetRowsMaxK * 2;                // bytes of an input row's place
  // LDS: the input rows; over them the first layer's output; then the next
  // layer's in its first part and the tail's pairs after that
  constexpr int MAIN = kRows * XROW;
  static_assert(kRows * N0 * 2 <= MAIN && kRows * NL * 2 + 2 * kRows * kTailHRow <= MAIN, "LDS plan");
  static_assert(tail_lds_bytes(kRows) <= kRows * NL * 2, "the tail's tiles take the 256-wide layer's input");
  __shared__ __align__(16) unsigned char smem[MAIN];
  // biases of every hidden layer, then the head's weights and biases
  constexpr int BO1 = N0, BO2 = BO1 + N1, BO3 = BO2 + kTailK, BO4 = BO3 + kTailN1, BOH = BO4 + kTailN2;
  __shared__ __align__(16) float s_b[BOH + 2 * kTailN2 + 2];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K0 = a.K0, ksteps = (K0 + 31) >> 5, nch = K0 >> 3;
  const TS *X = static_cast<const TS *>(a.x);

  {
    auto put = [&](const float *src, int at, int n) {
      for (int i = threadIdx.x; i < n; i += 64 * kWaves) s_b[at + i] = src[i];
    };
    put(a.b0, 0, N0);
    if constexpr (N1 > 0) put(a.b1, BO1, N1);
    put(a.b2, BO2, kTailK);
    put(a.tail.b1, BO3, kTailN1);
    put(a.tail.b2, BO4, kTailN2);
    for (int i = threadIdx.x; i < a.tail.n_out * kTailN2; i += 64 * kWaves)
      s_b[BOH + i] = Elem<TS>::to_f32(static_cast<const TS *>(a.tail.wh)[i]);
    put(a.tail.bh, BOH + 2 * kTailN2, a.tail.n_out);
  }
  // a tile's input rows in registers: thread t holds chunks t % 8 + 8 u of
  // row t / 8 (u < NX covers K0; loads past the row's end repeat its last
  // chunk); WEIGH: and the weight of each chunk's group
  uint4 xv[NX];
  float sv[WEIGH ? NX : 1];
  const int lcpg = WEIGH ? __builtin_ctz(a.d / 8) : 0, groups = WEIGH ? a.K0 / a.d : 0;
  auto load_x = [&](int64_t tile, int tid) {
    const int64_t rt = tile * kRows + (tid >> 3), r = rt < a.R ? rt : a.R - 1;
    const TS *xp = X + r * a.K0;
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      const int ch = u * 8 + (tid & 7);
      xv[u] = *reinterpret_cast<const uint4 *>(xp + (ch < nch ? ch : nch - 1) * 8);
      if constexpr (WEIGH) sv[u] = a.weights[r * groups + ((ch < nch ? ch : nch - 1) >> lcpg)];
    }
  };
  // and the first layer's first weight fragments
  constexpr int D0 = 2;
  frag wq[kQueue];
  auto load_w0 = [&](const WaveWeights<TS> &w0) {
#pragma unroll
    for (int f = 0; f < D0 * NI0; ++f) wq[f] = w0.load(f % NI0, f / NI0);
  };
  load_x(blockIdx.x, threadIdx.x);
  load_w0(WaveWeights<TS>(a.w0, N0 / 16, wave * NI0, ksteps, threadIdx.x & 63));

  for (int64_t tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
    const int64_t r0 = tile * kRows;
    // opaque to the compiler, so that no address derived from it is kept in
    // a register across the tile loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, c = lane & 15, q = lane >> 4, dn = q * 4;
    const WaveWeights<TS> w0(a.w0, N0 / 16, wave * NI0, ksteps, lane);
    constexpr int KS2 = NL / 32, NI2 = kTailK / kWaves / 16, D2 = kQueue / NI2;
    const WaveWeights<TS> w2(a.w2, kTailK / 16, wave * NI2, KS2, lane);
    auto next2 = [&](int f) { return w2.load(f % NI2, f / NI2); };
    // ---- the input rows to LDS (past the row's end, to a whole K step: zeros)
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      const int ch = u * 8 + (tid & 7);
      if constexpr (WEIGH) {
        float v[8];
        Elem<TS>::unpack(xv[u], v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = sv[u] * v[e];
        if (a.linear_log)
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = linear_log(v[e]);
        xv[u] = Elem<TS>::pack(v);
      }
      *reinterpret_cast<uint4 *>(smem + row_slot<XROW>(tid >> 3, ch)) =
          ch < nch ? xv[u] : make_uint4(0, 0, 0, 0);
    }
    lds_barrier();
    phase_end();
    f32x4 acc[NI0][RJ];
    start_at<NI0, RJ>(s_b + wave * NI0 * 16 + dn, acc);
    auto in0 = [&](int j, int k) { return smem + row_slot<XROW>(j * 16 + c, 4 * k + q); };
    constexpr int OFF = ODD ? NI0 : 0;   // where the queue starts after the first layer
    if constexpr (N1 > 0) {
      constexpr int NI1 = N1 / kWaves / 16, KS1 = N0 / 32, D1 = kQueue / NI1;
      const WaveWeights<TS> w1(a.w1, N1 / 16, wave * NI1, KS1, lane);
      static_assert(D0 * NI0 == kQueue, "the queue is whole");
      lds_layer<TS, NI0, RJ, D0, 0, ODD>(w0, ksteps, in0, wq, acc,
                                         [&](int f) { return w1.load(f % NI1, f / NI1); });
      phase_end(acc);
      lds_barrier();   // every wave has read the input rows
      store_act<TS, NI0, RJ, N0 * 2>(acc, smem, wave * NI0 * 16 + dn, c);
      lds_barrier();
      phase_end();
      f32x4 acc1[NI1][RJ];
      start_at<NI1, RJ>(s_b + BO1 + wave * NI1 * 16 + dn, acc1);
      auto in1 = [&](int j, int k) { return smem + row_slot<N0 * 2>(j * 16 + c, 4 * k + q); };
      lds_layer<TS, NI1, RJ, D1, OFF, false>(w1, KS1, in1, wq, acc1, next2);
      phase_end(acc1);
      lds_barrier();   // every wave has read the first layer's output
      phase_end();
      store_act<TS, NI1, RJ, N1 * 2>(acc1, smem, wave * NI1 * 16 + dn, c);
    } else {
      // the first layer fills half of the queue; the other half is the next
      // layer's from the start
      static_assert(2 * D0 * NI0 == kQueue, "the queue is half full");
#pragma unroll
      for (int u = 0; u < kQueue / 2; ++u) wq[kQueue / 2 + u] = next2(kQueue / 2 + u - OFF);
      lds_layer<TS, NI0, RJ, D0, 0, ODD>(w0, ksteps, in0, wq, acc, next2);
      phase_end(acc);
      lds_barrier();
      store_act<TS, NI0, RJ, N0 * 2>(acc, smem, wave * NI0 * 16 + dn, c);
    }
    // ---- the 256-wide layer, then the tail
    f32x4 acc2[NI2][RJ];
    start_at<NI2, RJ>(s_b + BO2 + wave * NI2 * 16 + dn, acc2);
    lds_barrier();
    phase_end();
    TailWeights<TS> tw;
    {
      auto in2 = [&](int j, int k) { return smem + row_slot<NL * 2>(j * 16 + c, 4 * k + q); };
      lds_layer<TS, NI2, RJ, D2, OFF, false>(w2, KS2, in2, wq, acc2,
                                             [&](int f) { return tw.w1_frag(a.tail, wave, lane, f / 2, f % 2); });
#pragma unroll
      for (int f = 0; f < kQueue; ++f) tw.w1[f / 2][f % 2] = wq[(f + OFF) % kQueue];
    }
    phase_end(acc2);
    tw.load_w2(a.tail, wave, lane);
    // the next tile's input rows, on their way during the tail
    load_x(tile + gridDim.x < a.tiles ? tile + gridDim.x : tile, tid);
    unsigned char *hl = smem + kRows * NL * 2;
#pragma unroll
    for (int i = 0; i < NI2; ++i)
#pragma unroll
      for (int j = 0; j < RJ; ++j)
        tail_put_pair<TS, kRows>(acc2[i][j], hl, (wave * NI2 + i) * 16 + dn, j * 16 + c);
    lds_barrier();
    phase_end();
    tw.bias_from(s_b + BO3, s_b + BO4, wave, lane);
    tail_rows<TS, kRows, 2, false, false>(hl, smem, tw, a.tail, s_b + BOH, a.scores, [&](int lr) { return r0 + lr; },
                                          a.R, tid, lane, wave, [&]() { load_w0(w0); });
    lds_barrier();   // the next tile's rows take the place of the tail's
  }
}

// widths D_in x 1024 x 512 x 256 x 128 x 64 x n_out, or the same without the
// 1024-wide layer
bool net_rows_shape(int dtype, const int32_t *w, int32_t L) {
  if (dtype == kF32 || w[0] % 8 != 0 || w[0] <= 64 || w[0] > kNetRowsMaxK) return false;
  if (L == 6) return w[1] == 1024 && w[2] == 512 && tail_supported(dtype, w[3], w[4], w[5], w[6]);
  if (L == 5) return w[1] == 512 && tail_supported(dtype, w[2], w[3], w[4], w[5]);
  return false;
}

// A tile costs 39 us however few there are, the layer-by-layer path grows
// with the rows; they meet at three eighths of a tile per CU (6,144 rows; D_in
// 768: 6,000 rows 49.2 against 46.5 us for the whole call, 6,500 rows 49.6
// against 51.4 us; without the 1024-wide layer 31.1 against 30.9 and 31.6
// against 33.2 us).
bool net_rows_chosen(int64_t R) {
  const int64_t cus = device_cus() > 0 ? device_cus() : 256;
  return (R + kRows - 1) / kRows * 8 >= 3 * cus;
}

template <typename TS, int N0, int N1, int NX, bool WEIGH>
static void net_rows_k(const NetRowsArgs &a, unsigned grid, hipStream_t s) {
  if (((a.K0 + 31) / 32) % 2)
    hipLaunchKernelGGL((net_rows_kernel<TS, N0, N1, NX, true, WEIGH>), dim3(grid), dim3(64 * kWaves), 0, s, a);
  else
    hipLaunchKernelGGL((net_rows_kernel<TS, N0, N1, NX, false, WEIGH>), dim3(grid), dim3(64 * kWaves), 0, s, a);
}

template <typename TS, bool WEIGH>
static hipError_t net_rows_t(int32_t n0, const NetRowsArgs &a, hipStream_t s) {
  const int cus = device_cus() > 0 ? device_cus() : 256;
  const unsigned grid = (unsigned)(a.tiles < cus ? a.tiles : cus);
  if (n0 == 1024 && a.K0 <= 768) net_rows_k<TS, 1024, 512, 12, WEIGH>(a, grid, s);
  else if (n0 == 1024) net_rows_k<TS, 1024, 512, 16, WEIGH>(a, grid, s);
  else if (a.K0 <= 768) net_rows_k<TS, 512, 0, 12, WEIGH>(a, grid, s);
  else net_rows_k<TS, 512, 0, 16, WEIGH>(a, grid, s);
  return hipGetLastError();
}

hipError_t launch_net_rows(int dtype, int32_t n0, int32_t n1, NetRowsArgs a, hipStream_t s) {
  if (a.R <= 0) return hipSuccess;
  if (dtype == kF32 || a.K0 <= 64 || a.K0 > kNetRowsMaxK || a.K0 % 8 != 0 ||
      (n0 == 1024 ? n1 != 512 : n0 != 512 || n1 != 0) ||
      (a.weights && (a.d < 8 || (a.d & (a.d - 1)) || a.K0 % a.d)))
    return hipErrorNotSupported;
  a.tiles = (a.R + kRows - 1) / kRows;
  if (a.weights)
    return dtype == kBF16 ? net_rows_t<__bf16, true>(n0, a, s) : net_rows_t<_Float16, true>(n0, a, s);
  return dtype == kBF16 ? net_rows_t<__bf16, false>(n0, a, s) : net_rows_t<_Float16, false>(n0, a, s);
}

}  // namespace cold
