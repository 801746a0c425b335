// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: true fp32 products and sums).
//
// C[M,N] = sum_k A(m,k) B(n,k).  Every wave owns one 32 x 32 tile of MFMA accumulators; a block of
// four waves is WM x WN of them side by side times WK ways of sharing the reduction: wave w of a
// k group multiplies its BK / WK indices of every k tile, and the WK accumulators are added
// through LDS, in wave order, before the epilogue.
//   2 x 2 x 1, BK = 32: 64 x 64 block tiles, for products with many of them
//   1 x 1 x 4, BK = 64: 32 x 32 block tiles, for products that would leave compute units idle with
//     the larger ones: four times the blocks, and the reduction's chain of dependent MFMAs (64
//     clocks per two indices) is a quarter as long
// An MFMA takes 64 clocks for 32 x 32 x 2, so LDS and L2 rates are no limit at these tile sizes (32
// and 16..32 bytes per clock and compute unit); what counts is that every SIMD has a wave to run.
//
// LDS layouts, double-buffered through registers:
//   k-major operand [rows][BK + 4]  : a lane reads four consecutive indices (16 bytes), conflict-free
//   m-major operand [BK][rows + 8]  : as it comes; a lane reads one value per MFMA, and the two
//                                     half-waves (4 index rows apart) fall in different banks
// MFMA number j of a group of eight indices multiplies indices j (lanes 0..31) and 4 + j (lanes
// 32..63) for both operands.  The order of the additions is fixed by the shape.
#include "gemm_device.h"

#include <hip/hip_ext.h>

namespace mk {

namespace {

constexpr int FGROUP_M = 4;                      // row panels per tile group (L2 reuse)

// One operand tile of R rows: global -> registers -> LDS -> MFMA operands.
template <bool KM, int R, int BK>
struct FTile {
  static constexpr int LD = KM ? BK + 4 : R + 8;
  static constexpr int ELEMS = KM ? R * LD : BK * LD;
  static constexpr int NCH = R * BK / 4 / 256;   // 16-byte chunks per thread
  static constexpr int FAST = (KM ? BK : R) / 4; // chunks along the contiguous index

  // where this thread's chunks of k tile 0 are; rows outside the matrix are replaced by the tile's
  // first row (their products are never stored)
  const float* src[NCH];
  int64_t step;
  __device__ __forceinline__ void init(const float* __restrict__ X, int64_t ldx, int rows, int r0, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 256, a = c / FAST, f = (c % FAST) * 4;
      if (KM) src[i] = X + (int64_t)(r0 + a < rows ? r0 + a : r0) * ldx + f;
      else src[i] = X + (int64_t)a * ldx + r0 + f;
    }
    step = KM ? (int64_t)BK : (int64_t)BK * ldx;
  }
  // k tile with all its indices inside K, all chunks inside the rows
  __device__ __forceinline__ void load(float4 (&v)[NCH]) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) { v[i] = *(const float4*)src[i]; src[i] += step; }
  }
  // tile at the end of K or of the rows, or operands without 16-byte alignment: element by element
  __device__ __forceinline__ void load_edge(float4 (&v)[NCH], int rows, int K, int r0, int k0, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 256, a = c / FAST, f = (c % FAST) * 4;
      const int slow = KM ? r0 + a : k0 + a, fast = KM ? k0 + f : r0 + f;
      const int slow_end = KM ? rows : K, fast_end = KM ? K : rows;
      const bool in = slow < slow_end;
      v[i].x = in && fast < fast_end ? src[i][0] : 0.f;
      v[i].y = in && fast + 1 < fast_end ? src[i][1] : 0.f;
      v[i].z = in && fast + 2 < fast_end ? src[i][2] : 0.f;
      v[i].w = in && fast + 3 < fast_end ? src[i][3] : 0.f;
      src[i] += step;
    }
  }
  static __device__ __forceinline__ void store(const float4 (&v)[NCH], float* tile, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 256;
      *(float4*)&tile[(c / FAST) * LD + (c % FAST) * 4] = v[i];
    }
  }
  // this lane's values of row `row` for the four MFMAs of indices k .. k + 7 (h: which half-wave)
  static __device__ __forceinline__ void frag(const float* tile, int row, int k, int h, float (&f)[4]) {
    if (KM) {
      const float4 t = *(const float4*)&tile[row * LD + k + 4 * h];
      f[0] = t.x; f[1] = t.y; f[2] = t.z; f[3] = t.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = tile[(k + 4 * h + j) * LD + row];
    }
  }
  static __device__ __forceinline__ float at(const float* tile, int row, int k) {
    return KM ? tile[row * LD + k] : tile[k * LD + row];
  }
};

}  // namespace

template <bool AK, bool BKM, int WM, int WN, int WK, int BK>
__global__ __launch_bounds__(256) void sgemm_mfma_kernel(GemmDev p, int vec, int tiles_n, int total, int per_xcd) {
  static_assert(WM * WN * WK == 4, "four waves");
  constexpr int BM = 32 * WM, BN = 32 * WN;
  typedef FTile<AK, BM, BK> TA;
  typedef FTile<BKM, BN, BK> TB;
  constexpr int SMEM = 2 * (TA::ELEMS + TB::ELEMS);
  static_assert(SMEM >= WK * WM * WN * 1024 && SMEM >= 256, "space for the partial tiles and row sums");
  __shared__ __attribute__((aligned(16))) float smem[SMEM];
  float* As = smem;
  float* Bs = smem + 2 * TA::ELEMS;
  // block id -> XCD-contiguous runs of tiles, in groups of FGROUP_M row panels
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= total) return;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int group = t / (FGROUP_M * tiles_n), first_m = group * FGROUP_M;
  const int gsize = min(tiles_m - first_m, FGROUP_M);
  const int in_group = t - group * FGROUP_M * tiles_n;
  const int tile_m = first_m + in_group % gsize, tile_n = in_group / gsize;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  const float* A = (const float*)p.A;
  const float* B = (const float*)p.B;

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const bool do_rowsum = p.a_rowsum && tile_n == 0;
  constexpr int RSK = 256 / BM;                       // threads sharing a row's sum
  float rs = 0.f;

  float4 ra[TA::NCH], rb[TB::NCH];
  TA ta;
  TB tb;
  ta.init(A, p.lda, p.M, m0, tid);
  tb.init(B, p.ldb, p.N, n0, tid);
  // an m-major operand is read along its rows, so its tile has to be whole; a k-major one is not
  const bool whole = vec && (AK || m0 + BM <= p.M) && (BKM || n0 + BN <= p.N);
  auto fetch = [&](int k0) {
    if (whole && k0 + BK <= p.K) {
      ta.load(ra);
      tb.load(rb);
    } else {
      ta.load_edge(ra, p.M, p.K, m0, k0, tid);
      tb.load_edge(rb, p.N, p.K, n0, k0, tid);
    }
  };
  auto stash = [&](int buf) {
    TA::store(ra, As + buf * TA::ELEMS, tid);
    TB::store(rb, Bs + buf * TB::ELEMS, tid);
  };
  fetch(0);
  stash(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < p.K; k0 += BK) {
    const bool more = k0 + BK < p.K;
    if (more) fetch(k0 + BK);
    const float* at = As + buf * TA::ELEMS;
    const float* bt = Bs + buf * TB::ELEMS;
    constexpr int KW = BK / WK;
#pragma unroll
    for (int g = 0; g < KW / 8; ++g) {
      float fa[4], fb[4];
      TA::frag(at, wm * 32 + l32, wk * KW + 8 * g, h, fa);
      TB::frag(bt, wn * 32 + l32, wk * KW + 8 * g, h, fb);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], acc, 0, 0, 0);
    }
    if (do_rowsum) {
#pragma unroll 4
      for (int k = tid / BM; k < BK; k += RSK) rs += TA::at(at, tid % BM, k);
    }
    if (more) stash(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }

  if (do_rowsum) {                                    // the shares of a row, in order
    smem[tid] = rs;
    __syncthreads();
    if (tid < BM && m0 + tid < p.M) {
      float s = smem[tid];
#pragma unroll
      for (int i = 1; i < RSK; ++i) s += smem[tid + i * BM];
      p.a_rowsum[m0 + tid] = s;
    }
    __syncthreads();
  }
  // accumulator register r of a lane: row 8*(r/4) + 4*h + r%4, column lane%32 of the wave's tile
  if (WK == 1) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      epilogue<float>(p, m0 + wm * 32 + 8 * (r >> 2) + 4 * h + (r & 3), n0 + wn * 32 + l32, acc[r]);
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) smem[wave * 1024 + r * 64 + lane] = acc[r];
    __syncthreads();
    // wave w finishes registers w, w + 4, ... of the tile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + wave;
      float s = smem[r * 64 + lane];
#pragma unroll
      for (int w = 1; w < WK; ++w) s += smem[w * 1024 + r * 64 + lane];
      epilogue<float>(p, m0 + 8 * (r >> 2) + 4 * h + (r & 3), n0 + l32, s);
    }
  }
}

template <bool AK, bool BKM>
static void launch_f32(const GemmDev& p, bool small, int vec, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  const int b = small ? 32 : 64;
  const int tiles_m = (p.M + b - 1) / b, tiles_n = (p.N + b - 1) / b, total = tiles_m * tiles_n, per = (total + 7) / 8;
  if (small)
    hipExtLaunchKernelGGL((sgemm_mfma_kernel<AK, BKM, 1, 1, 4, 64>), dim3(per * 8), dim3(256), 0, st, t0, t1, 0, p, vec, tiles_n,
                          total, per);
  else
    hipExtLaunchKernelGGL((sgemm_mfma_kernel<AK, BKM, 2, 2, 1, 32>), dim3(per * 8), dim3(256), 0, st, t0, t1, 0, p, vec, tiles_n,
                          total, per);
}

// Which tile size: the time of either is about its number of rounds over the 256 compute units times
// a block's work, four units with 64 x 64 tiles and one with 32 x 32, which pay 15 % more per unit
// (twice the loads per product).  At T = 2256: 2304 and 3072 columns of the forward 105 and 123 us
// with the large tiles (110 and 134 with the small), weight gradients of 768 x 768 and 3072 x 768
// 46 and 125 us with the small ones (69 and 137).  The kernel on the vector units that this one
// replaces took 218 and 264 us, 412 and 506 us there.
// rows: the row count the choice is made from (a product run in two row ranges must sum in the
// same order as the whole)
void launch_sgemm(const GemmDev& p, int rows, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  auto aligned = [](const void* q, int64_t ld) { return (((uintptr_t)q) & 15) == 0 && (ld & 3) == 0; };
  const int vec = aligned(p.A, p.lda) && aligned(p.B, p.ldb) ? 1 : 0;
  auto rounds = [&](int64_t b) { return (((rows + b - 1) / b) * ((p.N + b - 1) / b) + 255) / 256; };
  const bool small = 115 * rounds(32) < 400 * rounds(64);
#define GO_(AKV, BKV) launch_f32<AKV, BKV>(p, small, vec, st, t0, t1)
  if (p.a_k && p.b_k) GO_(true, true);
  else if (p.a_k) GO_(true, false);
  else if (p.b_k) GO_(false, true);
  else GO_(false, false);
#undef GO_
}

}  // namespace mk
