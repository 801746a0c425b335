// bf16 GEMM for long reductions behind few rows, A k-major (forward, data gradients): small block tiles of
// 16 x 16 x 32 MFMAs, a ring of direct loads.
//
// C[M,N] = sum_k A(m,k) B(n,k).  A product of a few hundred rows has fewer tiles than the chip has compute units,
// and a block that walks a whole reduction alone on its unit runs at the latency of a k step: the meeting of its
// waves, the reads behind it, a chain of MFMAs.  Against the ring kernel (gemm_ring.hip) a step is shorter:
// 16 x 16 x 32 MFMAs have a quarter of the latency of 32 x 32 x 16, loads are one instruction behind a fixed per-lane offset and a
// scalar base, 32 x 32 tiles put twice the units on a product, and the larger ones meet once in 128 indices.
// The reduction is not cut: every element is the same chain of MFMAs over ascending k as in the other
// kernels, so which kernel a product gets does not change a bit of it.  us, ring kernel -> here, operands from
// memory: 74, 150, 300 x 768, K = 3072 11.0 -> 8.5-9.0 (data gradient 11.2-11.7 -> 9.3-10.5), 74 x 768,
// K = 30528 94 -> 63 (119 -> 98); 1500 x 1024, K = 4096 on 96 x 64 29.1 -> 23.3 (27.9 -> 23.6); 2048 x 768, K = 3072 on
// 128 x 64 20.0 -> 17.8; 700 x 1024, K = 4096 on 64 x 64 16.3 -> 15.4 (both with a k-major B alone, see tiles_variant).
//
// LDS tiles: a k-major tile [rows][64 k] keeps chunk kc of row r at kc ^ ((r >> 1) & 7); an m-major tile
// [64 k][R rows] keeps chunk mc of k row q at mc ^ f(q), with f so that the four k rows and two groups of
// eight that transposing reads touch together meet different banks.  Both are filled by buffer loads with
// a fixed per-lane offset and a scalar base that moves along k.
#include "gemm_device.h"

#include <type_traits>

namespace mk {

namespace {

constexpr int TBK = 64;
constexpr int TGROUP_M = 4;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// at most n loads in flight, no LDS operation pending
constexpr int t_wait(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }

template <bool KM, int R>
struct TTile {
  static constexpr int LOADS = R / 8;                 // 1 KB direct loads of 64 indices
  static constexpr int ELEMS = R * TBK;
  static __device__ __forceinline__ int turn(int q) {
    return R >= 128 ? 4 * (q & 3) + 2 * ((q >> 3) & 1) : R == 64 ? 4 * ((q >> 3) & 1) + 2 * ((q >> 1) & 1) : 2 * ((q >> 3) & 1);
  }
  // first reduction index of the lane's 16 bytes of load j
  static __device__ __forceinline__ int index(int j, int lane) {
    if (KM) return ((lane & 7) ^ ((4 * j + (lane >> 4)) & 7)) * 8;
    return j * (64 / (R / 8)) + lane / (R / 8);
  }
  // their byte offset from the tile's first element
  static __device__ __forceinline__ uint32_t offset(int64_t ld, int rows, int j, int lane) {
    if (KM) return (uint32_t)((8 * j + (lane >> 3)) * (int)ld + index(j, lane)) * 2u;   // rows outside: behind the buffer's end
    constexpr int RC = R / 8;
    const int q = index(j, lane), mc = (lane % RC) ^ turn(q);
    return mc * 8 < rows ? (uint32_t)(q * (int)ld + mc * 8) * 2u : kOutside;
  }
  static __device__ __forceinline__ uint32_t bytes(int64_t ld, int rows) {
    return KM ? (uint32_t)min(rows, R) * (uint32_t)ld * 2u : kOutside;
  }
  // fragment of the 16 rows from `row` on, indices 32 h ..: element offset of its (first) read
  static __device__ __forceinline__ int frag_at(int row, int h, int lane) {
    if (KM) return (row + (lane & 15)) * TBK + (((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) << 3);
    const int g = lane >> 4, kq = (lane & 15) >> 2, q = 32 * h + 8 * g + kq;
    return q * R + ((((row >> 3) + ((lane & 3) >> 1)) ^ turn(q)) << 3) + (lane & 1) * 4;
  }
  static __device__ __forceinline__ bf16x8 read(const bf16_t* at) {
    if (KM) return *(const bf16x8*)at;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_l*)at);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_l*)(at + 4 * R));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

}  // namespace

// WM x WN waves, each TM x TN MFMA tiles of 16 x 16; NS stages of KB x 64 indices in the ring.
template <bool BKM, bool KTAIL, int WM, int WN, int TM, int TN, int KB, int NS>
__global__ __launch_bounds__(64 * WM * WN) void bgemm_tiles_kernel(GemmDev p, int tiles_n, int total, int per_xcd) {
  constexpr int W = WM * WN, BM = 16 * WM * TM, BN = 16 * WN * TN;
  typedef TTile<true, BM> TA;
  typedef TTile<BKM, BN> TB;
  static_assert(KB * TA::LOADS % W == 0 && KB * TB::LOADS % W == 0 && TN % 2 == 0, "loads divide evenly among the waves");
  constexpr int LA = KB * TA::LOADS / W, LB = KB * TB::LOADS / W, PER = LA + LB;
  constexpr int STAGE = KB * (TA::ELEMS + TB::ELEMS);                  // elements: KB tiles of A, KB of B
  static_assert(NS >= 3 && (NS - 2) * PER < 64 && NS * STAGE * 2 <= 160 * 1024, "ring in LDS, loads in flight in the counter");
  extern __shared__ __attribute__((aligned(1024))) unsigned char t_smem[];
  bf16_t* ring = (bf16_t*)t_smem;
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= total) return;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int group = t / (TGROUP_M * tiles_n), first_m = group * TGROUP_M;
  const int gsize = min(tiles_m - first_m, TGROUP_M);
  const int in_group = t - group * TGROUP_M * tiles_n;
  const int m0 = (first_m + in_group % gsize) * BM, n0 = in_group / gsize * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // ---- loads
  uint64_t base_a, base_b;
  uint32_t bytes_a, bytes_b, off_a[LA], off_b[LB];
  l_descriptor((const bf16_t*)p.A + (int64_t)m0 * p.lda, TA::bytes(p.lda, p.M - m0), base_a, bytes_a);
  l_descriptor((const bf16_t*)p.B + (BKM ? (int64_t)n0 * p.ldb : n0), TB::bytes(p.ldb, p.N - n0), base_b, bytes_b);
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int i = wave * LA + j, sub = i / TA::LOADS;
    off_a[j] = TA::offset(p.lda, p.M - m0, i % TA::LOADS, lane) + (uint32_t)(sub * TBK * 2);
  }
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const int i = wave * LB + j, sub = i / TB::LOADS;
    off_b[j] = TB::offset(p.ldb, p.N - n0, i % TB::LOADS, lane);
    if (off_b[j] != kOutside) off_b[j] += (uint32_t)(sub * TBK * 2) * (BKM ? 1u : (uint32_t)p.ldb);
  }
  const int64_t step_a = KB * TBK * 2, step_b = BKM ? KB * TBK * 2 : (int64_t)KB * TBK * 2 * p.ldb;
  const uint32_t lds0 = l_lds_address(ring), lds_a = lds0 + (uint32_t)(wave * LA) * 1024u,
                 lds_b = lds0 + (uint32_t)(KB * TA::ELEMS * 2) + (uint32_t)(wave * LB) * 1024u;
  const int n_stages = (p.K + KB * TBK - 1) / (KB * TBK);
  int left = p.K;                                     // indices from the stage to request on
  // behind the last stage its loads are issued again, into slots that are not read any more: the loop
  // then has no end cases (a constant number of loads in flight, no branches)
  auto issue = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const int i = wave * LA + j;
      const bool behind = KTAIL && TA::index(i % TA::LOADS, lane) + i / TA::LOADS * TBK >= left;
      l_direct_load(base_a, bytes_a, behind ? kOutside : off_a[j], lds_a + (uint32_t)(stage * STAGE * 2) + j * 1024u);
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const int i = wave * LB + j;
      const bool behind = KTAIL && TB::index(i % TB::LOADS, lane) + i / TB::LOADS * TBK >= left;
      l_direct_load(base_b, bytes_b, behind ? kOutside : off_b[j], lds_b + (uint32_t)(stage * STAGE * 2) + j * 1024u);
    }
    const bool more = left > KB * TBK;
    base_a += more ? step_a : 0;
    base_b += more ? step_b : 0;
    left -= more ? KB * TBK : 0;
  };

  // ---- fragments: of 64 indices one step ahead of the MFMAs that use them (two register sets), so neither the LDS
  // latency nor the meeting of the waves stands between two steps' MFMAs
  int fa[2], fb[TN][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    fa[h] = TA::frag_at(wm * TM * 16, h, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j][h] = KB * TA::ELEMS + TB::frag_at((wn * TN + j) * 16, h, lane);
  }
  bf16x8 af[2][2][TM], bfr[2][2][TN];
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto fragments = [&](auto set, int stage, int sub) __attribute__((always_inline)) {
    constexpr int S = decltype(set)::value;
    const bf16_t* at = ring + stage * STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[S][h][j] = TB::read(at + sub * TB::ELEMS + fb[j][h]);
#pragma unroll
      for (int i = 0; i < TM; ++i) af[S][h][i] = TA::read(at + sub * TA::ELEMS + fa[h] + i * 16 * TBK);
    }
  };
  auto mfmas = [&](auto set) __attribute__((always_inline)) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[S][h][j], af[S][h][i], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < NS - 1; ++i) issue(i);
  int cur = 0, fill = NS - 1;                         // slots of the next stage to read and to fill
  // Own loads of the next stage have landed (the younger NS - 2 stages stay in flight), own fragment
  // reads are done, all waves meet; then the slot read a turn ago may be refilled.
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);                // the other set's MFMAs stay behind the meeting
    __builtin_amdgcn_s_waitcnt(t_wait((NS - 2) * PER));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto next = [&]() __attribute__((always_inline)) {
    issue(fill);
    fill = cur;
    cur = cur == NS - 1 ? 0 : cur + 1;
  };
  typedef std::integral_constant<int, 0> S0;
  typedef std::integral_constant<int, 1> S1;
  if constexpr (KB == 1) {
    auto turn = [&](auto set) __attribute__((always_inline)) {
      meet();
      fragments(set, cur, 0);
      next();
    };
    turn(S0());
    for (int pair = n_stages >> 1; pair > 0; --pair) {
      turn(S1());
      mfmas(S0());
      turn(S0());
      mfmas(S1());
    }
    if (n_stages & 1) mfmas(S0());
  } else {
    meet();
    fragments(S0(), cur, 0);
    for (int s = 1; s < n_stages; ++s) {
      fragments(S1(), cur, 1);
      next();
      mfmas(S0());
      meet();
      fragments(S0(), cur, 0);
      mfmas(S1());
    }
    fragments(S1(), cur, 1);
    mfmas(S0());
    if (!KTAIL || (p.K - 1) % (2 * TBK) >= TBK) mfmas(S1());
  }
  __builtin_amdgcn_s_waitcnt(t_wait(0));              // no direct load may land in LDS that is the store's, or another block's, by then

  // ---- store: 16 x 32 pieces through LDS, so that the stores are rows.  Register r of fragment (i, j): row lane % 16,
  // column 4 * (lane / 16) + r; float4 chunk c of row r sits at c ^ ((r >> 1) & 7)
  const int mw = m0 + wm * TM * 16 + (lane >> 2), nw = n0 + wn * TN * 16 + (lane & 3) * 8;
  // all residuals of the wave's tiles at once (one piece's after another's store cost a memory latency each)
  u32x4 resid[TM][TN / 2];
  if (resid_ahead(p))
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN / 2; ++j) {
        const int m = mw + i * 16, n = nw + j * 32;
        if (m < p.M && n + 8 <= p.N) resid[i][j] = *(const u32x4*)((const bf16_t*)p.resid + (int64_t)m * p.ldr + n);
      }
  __syncthreads();
  float* ws = (float*)ring + wave * 512;
#pragma unroll
  for (int j = 0; j < TN / 2; ++j) {
    const int n = nw + j * 32, c0 = 2 * (lane & 3), row = lane >> 2;
    float cb[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (p.vec && p.bias && n + 8 <= p.N) unpack_bf16x8(*(const u32x4*)((const bf16_t*)p.bias + n), cb);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const f32x4 v = acc[i][2 * j + jj];
        *(float4*)&ws[(lane & 15) * 32 + (((4 * jj + (lane >> 4)) ^ ((lane >> 1) & 7)) << 2)] = make_float4(v[0], v[1], v[2], v[3]);
      }
      __builtin_amdgcn_wave_barrier();
      const float4 lo = *(const float4*)&ws[row * 32 + ((c0 ^ ((row >> 1) & 7)) << 2)];
      const float4 hi = *(const float4*)&ws[row * 32 + (((c0 + 1) ^ ((row >> 1) & 7)) << 2)];
      __builtin_amdgcn_wave_barrier();
      float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      const int m = mw + i * 16;
      if (m >= p.M || n >= p.N) continue;
      if (resid_ahead(p) && n + 8 <= p.N) {
        float f[8];
        unpack_bf16x8(resid[i][j], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] + cb[e] + f[e];
        put8(p, m, n, v);
      } else if (p.vec) finish8(p, m, n, v, cb);
      else
        for (int e = 0; e < 8; ++e) epilogue<bf16_t>(p, m, n + e, v[e]);
    }
  }
}

template <bool BKM, int WM, int WN, int TM, int TN, int KB, int NS>
static void launch_tiles_t(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN, SMEM = NS * KB * (BM + BN) * TBK * 2;
  static const bool configured = [] {
    (void)hipFuncSetAttribute((const void*)bgemm_tiles_kernel<BKM, false, WM, WN, TM, TN, KB, NS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    (void)hipFuncSetAttribute((const void*)bgemm_tiles_kernel<BKM, true, WM, WN, TM, TN, KB, NS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    return true;
  }();
  (void)configured;
  const int tiles_n = (p.N + BN - 1) / BN, total = (p.M + BM - 1) / BM * tiles_n, per = (total + 7) / 8;
  const dim3 grid(per * 8), block(64 * WM * WN);
  if (p.K % (KB * TBK))
    launch_marked((bgemm_tiles_kernel<BKM, true, WM, WN, TM, TN, KB, NS>), grid, block, SMEM, st, t0, t1, p, tiles_n, total, per);
  else
    launch_marked((bgemm_tiles_kernel<BKM, false, WM, WN, TM, TN, KB, NS>), grid, block, SMEM, st, t0, t1, p, tiles_n, total, per);
}
template <bool BKM>
static void launch_tiles(const GemmDev& p, int which, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  if (which == 0) launch_tiles_t<BKM, 2, 1, 1, 2, 1, 8>(p, st, t0, t1);        // 32 x 32
  else if (which == 2) launch_tiles_t<BKM, 2, 2, 3, 2, 2, 4>(p, st, t0, t1);   // 96 x 64
  else if constexpr (BKM) {
    if (which == 1) launch_tiles_t<true, 2, 2, 2, 2, 2, 5>(p, st, t0, t1);     // 64 x 64
    else launch_tiles_t<true, 4, 2, 2, 2, 1, 6>(p, st, t0, t1);                // 128 x 64
  }
}

// Requirements: A k-major; K % 8 == 0 or zeros vouched for behind A's last column, with B m-major; the leading
// dimension of an m-major B covers N rounded up to 8; a tile's 128 rows or indices span 512 MB at most.
bool launch_bgemm_tiles(const GemmDev& p, int which, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  auto up8 = [](int64_t v) { return (v + 7) / 8 * 8; };
  if (!p.a_k || p.a_rowsum || p.splits > 1) return false;
  if ((p.K & 7) && !(p.a_tail_zero && !p.b_k && p.lda >= up8(p.K))) return false;
  if (!p.b_k && (p.ldb < up8(p.N) || which == 1 || which == 3)) return false;
  if (p.lda >= (1 << 21) || p.ldb >= (1 << 21)) return false;          // 128 of them: 512 MB
  if (p.b_k) launch_tiles<true>(p, which, st, t0, t1);
  else launch_tiles<false>(p, which, st, t0, t1);
  return true;
}

}  // namespace mk
