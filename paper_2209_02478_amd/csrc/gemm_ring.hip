// bf16 GEMM for products with few output tiles: small block tiles, a deep ring of direct loads.
//
// C[M,N] = sum_k A(m,k) B(n,k).  A product of a few hundred rows has a handful of 128 x 128 tiles,
// and each walks the whole reduction on one compute unit with two k tiles in flight: it runs at the
// memory latency of its k tiles (T = 74, 768 columns, K = 3072: 6 tiles, 46 us), while most of the chip idles.
// Smaller tiles put more compute units on it, and the ring (NS stages of 64 reduction indices) keeps
// most of a unit's share of the reduction on its way.  The reduction is not cut: every element is the
// same chain of MFMAs over ascending k as in the kernels with larger tiles, so which
// kernel a product gets does not change a bit of it.
//
// All four layouts in all four tile sizes: forward, data gradients, and through the kernel-level entry point products with
// both operands m-major that are no weight gradient (768 x 768, K = 20480 in bf16: 66 us, 228 on 128 x 256 tiles).
// Weight gradients that nothing runs beside come in 128 x 128, with parts and row sums (ring_wgrad in gemm.hip).
//
// LDS tiles: a k-major tile
// [rows][64 k] keeps chunk kc of row r at kc ^ ((r >> 1) & 7); an m-major tile [64 k][R rows] keeps
// chunk mc of k row q at mc ^ s(q), with s so that four k rows read together meet different banks:
// 256 bytes hold 128/R k rows, so s(q) = 4 * ((q & 3) / (128/R)).
#include "gemm_device.h"

#include <type_traits>

namespace mk {

namespace {

constexpr int RBK = 64;
constexpr int RGROUP_M = 4;

__device__ __attribute__((aligned(16))) uint32_t g_zero16r[4] = {0u, 0u, 0u, 0u};

typedef __attribute__((address_space(3))) void lds_void_r;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4_r;

// One wave-level direct load, its waits placed by hand.  The s_nop is the wait state between a write of M0 and
// the load that reads it, which the hardware leaves to the program.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // m0 is a reserved register: named as clobbered on purpose
__device__ __forceinline__ void r_direct_load(const bf16_t* g, uint32_t lds_byte_address) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(lds_byte_address) : "memory", "m0");
}
#pragma clang diagnostic pop
// at most n loads in flight, no LDS operation pending
constexpr int r_wait(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }

template <bool KM, int R>
struct RTile {
  static constexpr int LOADS = R / 8;                 // 1 KB direct loads of a tile
  static constexpr int ELEMS = R * RBK;
  static __device__ __forceinline__ int swizzle(int q) { return 4 * ((q & 3) / (128 / R)); }
  // source of direct load j of the tile at rows r0, reduction index k0: the lane's 16 bytes
  static __device__ __forceinline__ const bf16_t* src(const bf16_t* X, int64_t ldx, int rows, int r0, int k0, int j, int lane,
                                                      int& k_in_tile) {
    if (KM) {
      const int r = 8 * j + (lane >> 3), kc = (lane & 7) ^ ((r >> 1) & 7);
      k_in_tile = kc * 8;
      return X + (int64_t)(r0 + r < rows ? r0 + r : r0) * ldx + k0 + kc * 8;   // outside: any row (never stored)
    }
    constexpr int RC = R / 8;
    const int q = j * (64 / RC) + lane / RC, mc = (lane % RC) ^ swizzle(q), row = r0 + mc * 8;
    k_in_tile = q;
    return X + (int64_t)(k0 + q) * ldx + (row < rows ? row : r0);
  }
  // fragment of the 32 rows from `block` on, k step ks: element offset of its (first) read
  static __device__ __forceinline__ int frag_at(int block, int ks, int lane) {
    if (KM) return (block + (lane & 31)) * RBK + (((2 * ks + (lane >> 5)) ^ ((lane >> 1) & 7)) << 3);
    const int kq = (lane & 15) >> 2, q = 16 * ks + 8 * (lane >> 5) + kq;
    const int mc = (block >> 3) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    return q * R + ((mc ^ swizzle(kq)) << 3) + (lane & 1) * 4;
  }
  static __device__ __forceinline__ bf16x8 read(const bf16_t* at) {
    if (KM) return *(const bf16x8*)at;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_r*)at);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_r*)(at + 4 * R));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

}  // namespace

// WM x WN waves, each TM x TN MFMA tiles of 32 x 32; NS stages in the ring.
template <bool AK, bool BKM, bool KTAIL, int WM, int WN, int TM, int TN, int NS>
__global__ __launch_bounds__(64 * WM * WN) void bgemm_ring_kernel(GemmDev p, int tiles_n, int total, int per_xcd) {
  constexpr int W = WM * WN, BM = 32 * WM * TM, BN = 32 * WN * TN;
  typedef RTile<AK, BM> TA;
  typedef RTile<BKM, BN> TB;
  static_assert(TA::LOADS % W == 0 && TB::LOADS % W == 0, "loads divide evenly among the waves");
  constexpr int LA = TA::LOADS / W, LB = TB::LOADS / W, STAGE = TA::ELEMS + TB::ELEMS;
  static_assert(NS * STAGE * 2 >= W * 4096, "4 KB per wave for the store");
  extern __shared__ __attribute__((aligned(1024))) unsigned char r_smem[];
  bf16_t* ring = (bf16_t*)r_smem;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= total) return;
  // weight gradients alone cut their reduction (units run part by part, see gemm_dma.hip) and carry
  // the row sums of A
  constexpr bool WG = !AK && !BKM;
  const int n_tiles = WG ? total / p.splits : total;
  const int split = WG ? unit / n_tiles : 0, t = unit - split * n_tiles;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int group = t / (RGROUP_M * tiles_n), first_m = group * RGROUP_M;
  const int gsize = min(tiles_m - first_m, RGROUP_M);
  const int in_group = t - group * RGROUP_M * tiles_n;
  const int tile_m = first_m + in_group % gsize, tile_n = in_group / gsize;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int k_begin = WG ? p.kb[split] : 0, k_end = WG ? p.kb[split + 1] : p.K;
  const int nk = (k_end - k_begin + RBK - 1) / RBK;
  const bool do_rowsum = WG && p.a_rowsum && tile_n == 0;
  float rs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const bf16_t *pa[LA], *pb[LB];
  int ka[LA], kb[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) pa[j] = TA::src((const bf16_t*)p.A, p.lda, p.M, m0, k_begin, wave * LA + j, lane, ka[j]);
#pragma unroll
  for (int j = 0; j < LB; ++j) pb[j] = TB::src((const bf16_t*)p.B, p.ldb, p.N, n0, k_begin, wave * LB + j, lane, kb[j]);
  const int64_t step_a = AK ? RBK : (int64_t)RBK * p.lda, step_b = BKM ? RBK : (int64_t)RBK * p.ldb;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_r*)ring);
  int k_issue = k_begin;
  // behind the last stage its loads are issued again, into slots that are not read any more: the loop
  // then has no end cases (a constant number of loads in flight, no branches)
  auto issue = [&](int stage) {
    const bool more = k_issue + RBK < k_end;
    const uint32_t la = lds0 + (uint32_t)(stage * STAGE * 2) + (uint32_t)(wave * LA) * 1024u;
    const uint32_t lb = lds0 + (uint32_t)(stage * STAGE * 2 + TA::ELEMS * 2) + (uint32_t)(wave * LB) * 1024u;
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const bf16_t* g = pa[j];
      if (KTAIL && k_issue + ka[j] >= k_end) g = (const bf16_t*)g_zero16r;      // chunks past the end read zeros
      r_direct_load(g, la + j * 1024u);
      pa[j] += more ? step_a : 0;
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const bf16_t* g = pb[j];
      if (KTAIL && k_issue + kb[j] >= k_end) g = (const bf16_t*)g_zero16r;
      r_direct_load(g, lb + j * 1024u);
      pb[j] += more ? step_b : 0;
    }
    k_issue += more ? RBK : 0;
  };
  int fa[TM][4], fb[TN][4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i][ks] = TA::frag_at((wm * TM + i) * 32, ks, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j][ks] = TA::ELEMS + TB::frag_at((wn * TN + j) * 32, ks, lane);
  }
  // Fragments of a stage are read one stage ahead of the MFMAs that use them (two register sets), so
  // neither the LDS latency nor the meeting of the waves stands between two stages' MFMAs.
  bf16x8 af[2][4][TM], bfr[2][4][TN];
  auto fragments = [&](auto set, int stage) {
    constexpr int S = decltype(set)::value;
    const bf16_t* at = ring + stage * STAGE;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[S][ks][i] = TA::read(at + fa[i][ks]);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[S][ks][j] = TB::read(at + fb[j][ks]);
    }
  };
  auto mfmas = [&](auto set) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[S][ks][j], af[S][ks][i], acc[i][j], 0, 0, 0);
  };
  // Row sums of the A tile: a thread owns 8 rows and every 16th reduction index, whatever the tile or
  // stage size (the sums' order is that of the other kernels).
  constexpr int RC = BM / 8;
  auto rowsum_acc = [&](const bf16_t* at) {
    if (RC * 16 < 64 * W && tid >= RC * 16) return;
#pragma unroll
    for (int j = 0; j < RBK / 16; ++j) {
      const int q = tid / RC + 16 * j;
      const bf16x8 v = *(const bf16x8*)(at + q * BM + (((tid % RC) ^ TA::swizzle(q)) << 3));
#pragma unroll
      for (int e = 0; e < 8; ++e) rs[e] += (float)v[e];
    }
  };
  constexpr int PER = LA + LB;
  static_assert(NS >= 3 && (NS - 2) * PER < 64, "loads in flight fit the counter");
#pragma unroll
  for (int i = 0; i < NS - 1; ++i) issue(i);
  int cur = 0, fill = NS - 1;                         // slots of the next stage to read and to fill
  // Own loads of the next stage have landed (the younger NS - 2 stages stay in flight), own fragment
  // reads are done, all waves meet; its fragments are read, and the slot read a turn ago is refilled.
  int sums_left = nk;                                 // an even count of stages ends with a turn behind the last
  auto turn = [&](auto set) {
    __builtin_amdgcn_sched_barrier(0);                // the other set's MFMAs stay behind the meeting
    __builtin_amdgcn_s_waitcnt(r_wait((NS - 2) * PER));
    if (W > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    fragments(set, cur);
    if (WG && do_rowsum && sums_left > 0) { rowsum_acc(ring + cur * STAGE); --sums_left; }
    issue(fill);
    fill = cur;
    cur = cur == NS - 1 ? 0 : cur + 1;
  };
  typedef std::integral_constant<int, 0> S0;
  typedef std::integral_constant<int, 1> S1;
  turn(S0());
  for (int pair = nk >> 1; pair > 0; --pair) {
    turn(S1());
    mfmas(S0());
    turn(S0());
    mfmas(S1());
  }
  if (nk & 1) mfmas(S0());
  __builtin_amdgcn_s_waitcnt(r_wait(0));
  // all residuals of the wave's tiles at once (one tile's after another's store cost a memory latency each)
  u32x4 resid[TM][TN][2];
  if (!WG && resid_ahead(p))
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int m = m0 + (wm * TM + i) * 32 + it * 16 + (lane >> 2), n = n0 + (wn * TN + j) * 32 + (lane & 3) * 8;
          if (m < p.M && n + 8 <= p.N) resid[i][j][it] = *(const u32x4*)((const bf16_t*)p.resid + (int64_t)m * p.ldr + n);
        }

  // 32 x 32 tiles through LDS, so that the stores are rows: register r of a lane is row lane%32,
  // column 8*(r/4) + 4*(lane/32) + r%4; float4 chunk c of row r sits at c ^ (r & 7)
  GemmDev q = p;
  if (WG) {
    float* rowsum = p.a_rowsum;
    if (p.splits > 1) {                               // raw tile and row sums of this part, see gemm_dma.hip
      q.C = p.partial + (int64_t)split * p.M * p.N;
      q.ldc = p.N; q.c_f32 = 1; q.bias = nullptr; q.resid = nullptr; q.gelu = GELU_NONE;
      q.vec = (p.N & 3) == 0;
      rowsum = p.partial + (int64_t)p.splits * p.M * p.N + (int64_t)split * p.M;
    }
    if (do_rowsum) {                                  // sixteen threads hold parts of every row
      float* red = (float*)ring;                      // [16][BM]
      __syncthreads();
      if (tid < RC * 16)
#pragma unroll
        for (int e = 0; e < 8; ++e) red[(tid / RC) * BM + (tid % RC) * 8 + e] = rs[e];
      __syncthreads();
      if (tid < BM && m0 + tid < p.M) {
        float tot = 0.f;
#pragma unroll
        for (int g = 0; g < 16; ++g) tot += red[g * BM + tid];
        rowsum[m0 + tid] = tot;
      }
    }
  }
  __syncthreads();
  float* ws = (float*)ring + wave * 1024;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int row = lane & 31, c = 2 * g + (lane >> 5);
        *(float4*)&ws[row * 32 + ((c ^ (row & 7)) << 2)] =
            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
      }
      __builtin_amdgcn_wave_barrier();
      const int mb = m0 + (wm * TM + i) * 32, nb = n0 + (wn * TN + j) * 32;
      const int n = nb + (lane & 3) * 8, c0 = 2 * (lane & 3);
      float cb[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (q.vec && q.bias && n + 8 <= p.N) unpack_bf16x8(*(const u32x4*)((const bf16_t*)q.bias + n), cb);
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int row = it * 16 + (lane >> 2), m = mb + row;
        const float4 lo = *(const float4*)&ws[row * 32 + ((c0 ^ (row & 7)) << 2)];
        const float4 hi = *(const float4*)&ws[row * 32 + (((c0 + 1) ^ (row & 7)) << 2)];
        float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        if (m >= p.M || n >= p.N) continue;
        if (!WG && resid_ahead(p) && n + 8 <= p.N) {
          float f[8];
          unpack_bf16x8(resid[i][j][it], f);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = v[e] + cb[e] + f[e];
          put8(p, m, n, v);
        } else if (q.vec) finish8(q, m, n, v, cb);
        else
          for (int e = 0; e < 8; ++e) epilogue<bf16_t>(q, m, n + e, v[e]);
      }
      __builtin_amdgcn_wave_barrier();
    }
}

template <bool AK, bool BKM, int WM, int WN, int TM, int TN, int NS>
static void launch_ring_t(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN, SMEM = NS * (BM + BN) * RBK * 2;
  static const bool configured = [] {
    (void)hipFuncSetAttribute((const void*)bgemm_ring_kernel<AK, BKM, false, WM, WN, TM, TN, NS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    (void)hipFuncSetAttribute((const void*)bgemm_ring_kernel<AK, BKM, true, WM, WN, TM, TN, NS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    return true;
  }();
  (void)configured;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN, total = tiles_m * tiles_n * p.splits, per = (total + 7) / 8;
  const dim3 grid(per * 8), block(64 * WM * WN);
  bool ktail = false;
  for (int i = 0; i < p.splits; ++i) ktail |= (p.kb[i + 1] - p.kb[i]) % RBK != 0 || p.kb[i + 1] == p.kb[i];
  if (ktail)
    launch_marked((bgemm_ring_kernel<AK, BKM, true, WM, WN, TM, TN, NS>), grid, block, SMEM, st, t0, t1, p, tiles_n, total, per);
  else
    launch_marked((bgemm_ring_kernel<AK, BKM, false, WM, WN, TM, TN, NS>), grid, block, SMEM, st, t0, t1, p, tiles_n, total, per);
}
template <bool AK, bool BKM>
static void launch_ring(const GemmDev& p, int which, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  switch (which) {
    case 0: launch_ring_t<AK, BKM, 2, 1, 1, 1, 6>(p, st, t0, t1); break;
    case 1: launch_ring_t<AK, BKM, 2, 2, 1, 1, 4>(p, st, t0, t1); break;
    case 2: launch_ring_t<AK, BKM, 2, 2, 2, 1, 5>(p, st, t0, t1); break;
    default: launch_ring_t<AK, BKM, 2, 4, 2, 1, 5>(p, st, t0, t1); break;
  }
}

bool launch_bgemm_ring(const GemmDev& p, int which, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  auto up8 = [](int64_t v) { return (v + 7) / 8 * 8; };
  if ((p.a_rowsum || p.splits > 1) && (p.a_k || p.b_k)) return false;
  if ((p.a_k || p.b_k) && (p.K & 7) && !(p.a_tail_zero && p.a_k && !p.b_k && p.lda >= up8(p.K))) return false;
  if (!p.a_k && p.lda < up8(p.M)) return false;
  if (!p.b_k && p.ldb < up8(p.N)) return false;
  if (p.a_k && p.b_k) launch_ring<true, true>(p, which, st, t0, t1);
  else if (p.a_k) launch_ring<true, false>(p, which, st, t0, t1);
  else if (p.b_k) launch_ring<false, true>(p, which, st, t0, t1);
  else launch_ring<false, false>(p, which, st, t0, t1);
  return true;
}

}  // namespace mk
