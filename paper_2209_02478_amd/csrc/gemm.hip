// GEMM kernels: C[M,N] = sum_k A(m,k) B(n,k) with fused epilogues.
//
// One operand description serves the three products of a linear layer:
//   forward   Y[T,out]  = X[T,in]   W[out,in]^T     A k-major, B k-major
//   dgrad     dX[T,in]  = dY[T,out] W[out,in]       A k-major, B m-major
//   wgrad     dW[out,in]= dY[T,out]^T X[T,in]       A m-major, B m-major
// "k-major": the reduction index is the contiguous one in memory.
//
// bf16: 128x128x64 tiles, 4 waves (2x2), each wave 64x64 as 2x2 MFMA 32x32x16
// tiles with fp32 accumulators, LDS double-buffered through registers.  k-major
// operands are staged [row][k] and read 16 bytes per lane; m-major operands are
// staged as they come, [k][row], and read with the transposing LDS loads of
// gfx950, so no operand is ever transposed in memory or in registers.  The
// reduction order over k is fixed by the shape alone: results are reproducible
// bit for bit.
// fp32: gemm_f32.hip.
#include "device_common.h"
#include "gemm_device.h"

#include <algorithm>

#include "kernels.h"

namespace mk {

// ------------------------------------------------------------------ bf16 MFMA
constexpr int BM = 128, BN = 128, BK = 64;
constexpr int GROUP_M = 4;                      // row panels per tile group (4-6 measured best in the step, 8 and 1 about 0.5 % behind, 64 3 % behind)
constexpr int NCH = BK / 16;                    // 16-byte chunks per thread and operand tile
constexpr int KCH = BK / 8;                     // chunks along k of a k-major row
constexpr int LDK = BK + 8;        // row stride of a k-major tile [128 rows][64 k] (144 B: conflict-free 16 B reads)
constexpr int LDM = 128 + 32;      // row stride of an m-major tile [64 k][128 rows] (320 B: conflict-free transposing reads)
constexpr int TILE_K_ELEMS = 128 * LDK, TILE_M_ELEMS = BK * LDM;

// One operand tile: global -> registers -> LDS -> MFMA fragments.
//   k-major source (elem(r,k) = X[r*ld+k]) is stored [row][k]; a fragment is one 16-byte read.
//   m-major source (elem(r,k) = X[k*ld+r]) is stored as it comes, [k][row]; a fragment is two
//   transposing 8-byte reads (ds_read_b64_tr_b16: within 16 lanes, lane i receives element i%4
//   of the four lanes 4k + i/4, i.e. a 4(k) x 16(row) block is handed out one row index per lane).
template <bool KM>
struct Tile {
  static constexpr int ELEMS = KM ? TILE_K_ELEMS : TILE_M_ELEMS;

  static __device__ __forceinline__ void addr(int c, int r0, int k0, int& gr, int& gk) {
    const int a = KM ? (c / KCH) : (c >> 4);         // slow index within the tile
    const int f = KM ? (c % KCH) * 8 : (c & 15) * 8; // fast (contiguous) index
    gr = KM ? r0 + a : r0 + f;                       // row (m or n) of the first element
    gk = KM ? k0 + f : k0 + a;                       // reduction index of the first element
  }
  // tile fully inside the matrix: plain 16-byte loads
  static __device__ __forceinline__ void load(u32x4 (&v)[NCH], const bf16_t* __restrict__ X, int64_t ldx, int r0, int k0,
                                              int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int gr, gk;
      addr(tid + i * 256, r0, k0, gr, gk);
      v[i] = *(const u32x4*)(KM ? X + (int64_t)gr * ldx + gk : X + (int64_t)gk * ldx + gr);
    }
  }
  // tile crossing an edge: out-of-range elements read as zero
  struct Regs { u32x4 v[NCH]; };
  static __device__ __forceinline__ Regs load_edge(const bf16_t* __restrict__ X, int64_t ldx, int R, int K, int r0,
                                                int k0, int tid) {
    Regs out;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      int gr, gk;
      addr(tid + i * 256, r0, k0, gr, gk);
      const bf16_t* src = KM ? X + (int64_t)gr * ldx + gk : X + (int64_t)gk * ldx + gr;
      u32x4 t = {0u, 0u, 0u, 0u};
      const bool slow_ok = KM ? gr < R : gk < K;
      const int fast_pos = KM ? gk : gr, fast_end = KM ? K : R;
      if (slow_ok) {
        if (fast_pos + 8 <= fast_end) {
          t = *(const u32x4*)src;
        } else if (fast_pos < fast_end) {
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const uint32_t e = fast_pos + q < fast_end ? (uint32_t)src[q] : 0u;
            t[q >> 1] |= e << (16 * (q & 1));
          }
        }
      }
      out.v[i] = t;
    }
    return out;
  }
  static __device__ __forceinline__ void store(const u32x4 (&v)[NCH], bf16_t* tile, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 256;
      if (KM) *(u32x4*)&tile[(c / KCH) * LDK + (c % KCH) * 8] = v[i];
      else *(u32x4*)&tile[(c >> 4) * LDM + (c & 15) * 8] = v[i];
    }
  }
  // fragment for rows rbase + lane%32, reduction indices 16*ks + 8*(lane/32) .. +7
  static __device__ __forceinline__ bf16x8 frag(const bf16_t* tile, int rbase, int ks, int lane) {
    if (KM) return *(const bf16x8*)&tile[(rbase + (lane & 31)) * LDK + ks * 16 + (lane >> 5) * 8];
    const int krow = ks * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int col = rbase + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    struct { s16x4 lo, hi; } r;
    r.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)&tile[krow * LDM + col]);
    r.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)&tile[(krow + 4) * LDM + col]);
    return __builtin_bit_cast(bf16x8, r);
  }
  // sum over the tile's 64 reduction indices of row `row` (partial, see caller)
  static __device__ __forceinline__ float rowsum_part(const bf16_t* tile, int tid) {
    float s = 0.f;
    if (KM) {                       // two threads per row, half of the k range each
      const bf16_t* src = &tile[(tid >> 1) * LDK + (tid & 1) * (BK / 2)];
#pragma unroll
      for (int e = 0; e < BK / 2; ++e) s += bf16_to_f32(src[e]);
    } else {                        // two threads per row: lower / upper half of the k rows
      const bf16_t* src = &tile[(tid & 1) * (BK / 2) * LDM + (tid >> 1)];
#pragma unroll
      for (int e = 0; e < BK / 2; ++e) s += bf16_to_f32(src[e * LDM]);
    }
    return s;
  }
};

// k loop of one block.  Global loads run two k tiles ahead of the MFMAs (two register sets), LDS
// holds two tiles, one barrier per k tile.  EDGE: tile crosses a matrix edge or K has a tail.
template <bool AK, bool BKM, bool EDGE>
__device__ __forceinline__ void mainloop(const GemmDev& p, bf16_t* As, bf16_t* Bs, int m0, int n0, int k_begin, int k_end,
                                         int tid, int lane, int wm, int wn, bool do_rowsum, f32x16 (&acc)[2][2],
                                         float& rs) {
  typedef Tile<AK> TA;
  typedef Tile<BKM> TB;
  const bf16_t* A = (const bf16_t*)p.A;
  const bf16_t* B = (const bf16_t*)p.B;
  // two register sets (named, never indexed at run time, so they stay in registers)
  u32x4 ra0[NCH], rb0[NCH], ra1[NCH], rb1[NCH];
  auto fetch = [&](u32x4 (&xa)[NCH], u32x4 (&xb)[NCH], int kt) {      // k tile kt (relative) -> register set
    const int k0 = k_begin + kt * BK;
    if (!EDGE) {
      TA::load(xa, A, p.lda, m0, k0, tid);
      TB::load(xb, B, p.ldb, n0, k0, tid);
    } else {
      const typename TA::Regs ea = TA::load_edge(A, p.lda, p.M, k_end, m0, k0, tid);
      const typename TB::Regs eb = TB::load_edge(B, p.ldb, p.N, k_end, n0, k0, tid);
#pragma unroll
      for (int i = 0; i < NCH; ++i) { xa[i] = ea.v[i]; xb[i] = eb.v[i]; }
    }
  };
  auto stash = [&](const u32x4 (&xa)[NCH], const u32x4 (&xb)[NCH], int buf) {
    TA::store(xa, As + buf * TA::ELEMS, tid);
    TB::store(xb, Bs + buf * TB::ELEMS, tid);
  };
  auto compute = [&](int buf) {
    const bf16_t* at = As + buf * TA::ELEMS;
    const bf16_t* bt = Bs + buf * TB::ELEMS;
    if (do_rowsum) rs += TA::rowsum_part(at, tid);
    __builtin_amdgcn_iglp_opt(0);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 af[2], bfr[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = TA::frag(at, wm * 64 + i * 32, ks, lane);
        bfr[i] = TB::frag(bt, wn * 64 + i * 32, ks, lane);
      }
      // roles swapped (B tile rows feed the MFMA's A side): a lane then owns one output row m
      // and, per register group, four consecutive columns n
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
    }
  };
  const int nk = (k_end - k_begin + BK - 1) / BK;
  if (nk <= 0) return;
  fetch(ra0, rb0, 0);
  stash(ra0, rb0, 0);
  if (nk > 1) fetch(ra1, rb1, 1);
  __syncthreads();
  int kt = 0;
  // steady state: every fetch is unconditional, so the wait before a stash only covers the
  // older register set and the newer loads stay in flight across the MFMAs
  for (; kt + 3 < nk; kt += 2) {
    fetch(ra0, rb0, kt + 2);
    compute(0);
    stash(ra1, rb1, 1);
    __syncthreads();
    fetch(ra1, rb1, kt + 3);
    compute(1);
    stash(ra0, rb0, 0);
    __syncthreads();
  }
  // one to three tiles left: buffer 0 holds tile kt, set 1 holds tile kt+1 (if any)
  if (kt + 2 < nk) fetch(ra0, rb0, kt + 2);
  compute(0);
  if (kt + 1 < nk) {
    stash(ra1, rb1, 1);
    __syncthreads();
    compute(1);
    if (kt + 2 < nk) {
      stash(ra0, rb0, 0);
      __syncthreads();
      compute(0);
    }
  }
}

// Grid: one-dimensional, 8 * ceil(units/8) blocks, a unit being (tile, k split).  Hardware hands
// consecutive block ids to the 8 XCDs in turn, so block id -> (xcd, slot) -> unit xcd*per + slot
// gives every XCD (and its L2) a contiguous run of tiles that share A row panels.
//
// Pipeline: global loads run two k tiles ahead of the MFMAs (two register sets), LDS holds two
// tiles; one barrier per k tile.
template <bool AK, bool BKM>
__global__ __launch_bounds__(256, 2) void bgemm_kernel(GemmDev p, int tiles_n, int total, int per_xcd) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  typedef Tile<AK> TA;
  typedef Tile<BKM> TB;
  bf16_t* As = (bf16_t*)smem_raw;                    // two buffers of TA::ELEMS
  bf16_t* Bs = As + 2 * TA::ELEMS;                   // two buffers of TB::ELEMS
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= total) return;
  // units run part by part (all tiles of the first k range, then of the second, ...): an XCD's
  // contiguous run of units then shares one k range of both operands in its L2
  const int n_tiles = total / p.splits;
  const int split = unit / n_tiles, t = unit - split * n_tiles;
  // tiles run down groups of GROUP_M row panels, so the tiles in flight on one XCD cover a
  // squarish patch of C and share both A and B panels in its L2
  const int tiles_m = (p.M + BM - 1) / BM;
  const int group = t / (GROUP_M * tiles_n), first_m = group * GROUP_M;
  const int gsize = min(tiles_m - first_m, GROUP_M);
  const int in_group = t - group * GROUP_M * tiles_n;
  const int tile_m = first_m + in_group % gsize, tile_n = in_group / gsize;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const bf16_t* A = (const bf16_t*)p.A;
  const bf16_t* B = (const bf16_t*)p.B;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int k_begin = p.kb[split], k_end = p.kb[split + 1];
  const bool do_rowsum = p.a_rowsum && tile_n == 0;
  float rs = 0.f;
  // tiles fully inside the matrices take the loop without any bounds logic
  if (m0 + BM <= p.M && n0 + BN <= p.N && (k_end - k_begin) % BK == 0)
    mainloop<AK, BKM, false>(p, As, Bs, m0, n0, k_begin, k_end, tid, lane, wm, wn, do_rowsum, acc, rs);
  else
    mainloop<AK, BKM, true>(p, As, Bs, m0, n0, k_begin, k_end, tid, lane, wm, wn, do_rowsum, acc, rs);

  GemmDev q = p;
  float* rowsum = p.a_rowsum;
  if (p.splits > 1) {
    // raw fp32 tile and row sums of this k range, as a plain matrix [M][N] in the workspace (which
    // is 16-byte aligned); a second kernel adds the parts in order
    q.C = p.partial + (int64_t)split * p.M * p.N;
    q.ldc = p.N; q.c_f32 = 1; q.bias = nullptr; q.resid = nullptr; q.gelu = GELU_NONE;
    q.vec = (p.N & 3) == 0;
    rowsum = p.partial + (int64_t)p.splits * p.M * p.N + (int64_t)split * p.M;
  }
  if (do_rowsum) {
    const float tot = rs + __shfl_xor(rs, 1, 64);
    const int m = m0 + (tid >> 1);
    if ((tid & 1) == 0 && m < p.M) rowsum[m] = tot;
  }
  static_assert(2 * (TA::ELEMS + TB::ELEMS) * sizeof(bf16_t) >= 4 * 64 * 64 * sizeof(float), "staging needs 16 KB per wave");
  u32x4 resid[8];
  load_resid<1>(q, m0 + wm * 64, n0 + wn * 64, lane, resid);
  __syncthreads();                                    // the operand tiles are dead
  store_tile<1>(q, acc, m0 + wm * 64, n0 + wn * 64, lane, (float*)smem_raw + wave * 4096, resid);
}

// C[m][n] = sum over splits (in order) of partial tiles; row sums likewise.  C is fp32, or bf16
// (the sum rounded once) when OUT_BF16.
template <bool OUT_BF16>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, void* __restrict__ Cv,
                                                            int64_t ldc, float* __restrict__ rowsum, int M, int N,
                                                            int splits) {
  const int64_t MN = (int64_t)M * N;
  const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  auto put = [&](int64_t o, float v) {
    if (OUT_BF16) ((bf16_t*)Cv)[o] = f32_to_bf16(v); else ((float*)Cv)[o] = v;
  };
  if (idx < MN) {
    const int m = (int)(idx / N), n = (int)(idx - (int64_t)m * N);
    if ((N & 3) == 0) {
      float4 s = *(const float4*)(partial + idx);
      for (int k = 1; k < splits; ++k) {
        const float4 v = *(const float4*)(partial + k * MN + idx);
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
      const int64_t o = (int64_t)m * ldc + n;
      if (OUT_BF16 && (ldc & 3) == 0) {
        uint2 w;
        w.x = pack_bf16x2(s.x, s.y); w.y = pack_bf16x2(s.z, s.w);
        *(uint2*)((bf16_t*)Cv + o) = w;
      } else {
        put(o, s.x); put(o + 1, s.y); put(o + 2, s.z); put(o + 3, s.w);
      }
    } else {
      for (int e = 0; e < 4 && idx + e < MN; ++e) {
        const int64_t q = idx + e;
        float s2 = partial[q];
        for (int k = 1; k < splits; ++k) s2 += partial[k * MN + q];
        const int mm = (int)(q / N), nn = (int)(q - (int64_t)mm * N);
        put((int64_t)mm * ldc + nn, s2);
      }
    }
  }
  if (rowsum && idx < M) {       // the first M/4 threads also finish the row sums
    const float* rp = partial + (int64_t)splits * MN;
    for (int e = 0; e < 4 && idx + e < M; ++e) {
      float s2 = rp[idx + e];
      for (int k = 1; k < splits; ++k) s2 += rp[(int64_t)k * M + idx + e];
      rowsum[idx + e] = s2;
    }
  }
}

int gemm_splits(int M, int N) {
  const int tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  int s = (256 + tiles - 1) / tiles;
  return s < 1 ? 1 : (s > 8 ? 8 : s);
}

// persistent blocks on tiles of 256 x 256 and 128 x 256 (gemm_large.h); false when the operands do not meet
// its requirements
bool launch_bgemm_large(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1);
bool launch_bgemm_large128(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1);
static int tiles128(int M, int N) { return ((M + 127) / 128) * ((N + 255) / 256); }
static int rounds(int tiles) { return (tiles + 255) / 256; }
// Rows of the tiles (256 or 128) of a product that is not cut in parts, or 0: the kernels with 128 x 128.
// One block per compute unit, so the time is a whole number of rounds of 256 tiles; a round of the
// smaller tiles takes about two thirds of one of the larger (0.95 against 1.5 us per 64 reduction indices,
// and 6-8 us of start and store).  One round against two thirds: ahead by 20-28 % at 88-128 large tiles
// (8192 x 768, K = 3072: 74 -> 49 us; 6352 x 1024, K = 4096: 87 -> 57), three against two (320 large tiles)
// by 0-6 %; from there on the larger are ahead by up to a fifth.  Left to the kernels with 128 x 128, of which a
// compute unit holds two or three, times of the large tiles over theirs:
// - fewer than 66 large tiles
// - B m-major where a second round of large tiles has just begun: 0.91-1.10 for data gradients (257-280) and
//   0.95-1.14 for both operands m-major (257-300), K = 512-6400.  With B k-major the tiles of 128 rows are ahead there too,
//   0.70-0.97 from K = 768 on and 0.73-1.02 at 512
// - one round of their own, 512, where tiles of 128 rows have begun a second one (a last column tile at most half
//   full, as in 2816 x 2944 or 16391 x 257): 0.95-1.88 with B m-major; with B k-major 0.84-1.70 up to K = 1024, 1.2 in
//   the mean, 0.80-1.30 at 2048 and 0.78-1.14 at 4096
static int large_rows(int M, int N, int K, bool a_k, bool b_k) {
  if (M < 256 || N < 256 || K < 512) return 0;
  const int large = gemm_large_tiles(M, N), r = rounds(large), r128 = rounds(tiles128(M, N));
  if (large < 66 || (!b_k && large > 256 && large <= (a_k ? 280 : 300))) return 0;
  if (r == 1 && r128 == 2 && ((M + BM - 1) / BM) * ((N + BN - 1) / BN) <= 512 && (!b_k || K < 4096)) return 0;
  return 2 * r128 <= 3 * r ? 128 : 256;
}

// Data-gradient products with a very long reduction and few output tiles (the head's, whose
// reduction runs over the vocabulary): on the large tiles, the reduction cut in parts so that
// about 200 units exist; with K in the tens of thousands a tile's start and end vanish and the
// parts are small against the operands (T = 6400, K = 30528: 330 us in three parts, 535 us on
// 128 x 128 tiles; T = 2048: 117 against 341 us).  The parts' rows are capped so that the scratch
// is a constant of the model, not a function of the batch.
constexpr int kLongK = 8192;
constexpr int64_t kLongKRows = 24576;            // parts x M at most
size_t gemm_long_k_workspace_bytes(int N) { return (size_t)kLongKRows * N * 4; }
static int long_k_splits(int M, int N) {
  const int tiles = gemm_large_tiles(M, N);
  int s = (205 + tiles - 1) / tiles;
  const int cap = (int)(kLongKRows / M);
  if (s > cap) s = cap;
  return s < 1 ? 1 : (s > 8 ? 8 : s);
}

size_t gemm_workspace_bytes(int M, int N) {
  const int s = gemm_splits(M, N);
  return s > 1 ? ((size_t)s * M * N + (size_t)s * M) * 4 : 0;
}

// t1 (optional): event bound to the end of this kernel, which ends the product it belongs to
static void launch_splitk_reduce(const GemmDev& p, hipStream_t st, hipEvent_t t1) {
  const int64_t MN = (int64_t)p.M * p.N;
  const dim3 grid((unsigned)((MN / 4 + 256) / 256));
  if (p.c_f32)
    launch_marked(splitk_reduce_kernel<false>, grid, dim3(256), 0, st, nullptr, t1, p.partial, p.C, p.ldc,
                          p.a_rowsum, p.M, p.N, p.splits);
  else
    launch_marked(splitk_reduce_kernel<true>, grid, dim3(256), 0, st, nullptr, t1, p.partial, p.C, p.ldc,
                          p.a_rowsum, p.M, p.N, p.splits);
}

template <bool AK, bool BKM>
static void launch_bgemm(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  constexpr int smem = 2 * (Tile<AK>::ELEMS + Tile<BKM>::ELEMS) * 2;
  static bool configured = false;
  if (!configured) {
    (void)hipFuncSetAttribute((const void*)bgemm_kernel<AK, BKM>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    configured = true;
  }
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  const int total = tiles_m * tiles_n * p.splits, per = (total + 7) / 8;
  launch_marked((bgemm_kernel<AK, BKM>), dim3(per * 8), dim3(256), smem, st, t0, p.splits > 1 ? nullptr : t1, p,
                        tiles_n, total, per);
  if (p.splits > 1) launch_splitk_reduce(p, st, t1);
}

// direct-to-LDS pipeline (gemm_dma.hip); false when the operands do not meet its alignment rules
bool launch_bgemm_dma(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1);

// fp32 on the bf16 matrix cores (gemm_f32.hip)
void launch_sgemm(const GemmDev& p, int rows, hipStream_t st, hipEvent_t t0, hipEvent_t t1);

// small tiles, deep ring (gemm_ring.hip); false when the operands do not meet its alignment rules
bool launch_bgemm_ring(const GemmDev& p, int which, hipStream_t st, hipEvent_t t0, hipEvent_t t1);
// Its block tiles are 64 x 32, 64 x 64, 128 x 64 and 128 x 128 (variants 0..3), one block per compute
// unit; a product gets the smallest that covers it in one round of the 256 units: more blocks than
// that queue, fewer leave units idle and each with a longer tile.  Measured against the kernels below
// at 768 columns and K = 3072: 74 rows 46 -> 11 us, 600 rows 46 -> 11, 1600 rows 45 -> 18, 2816 rows
// 33 -> 26, 4400 rows 46 -> 33; level at 6400 rows (300 tiles of 128 x 128, two rounds: not taken).
static int ring_variant(int M, int N) {
  auto tiles = [&](int64_t bm, int64_t bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn); };
  if (tiles(64, 32) <= 256) return 0;
  if (tiles(64, 64) <= 256) return 1;
  if (tiles(128, 64) <= 256) return 2;
  return tiles(128, 128) <= 256 ? 3 : -1;
}

// small tiles behind long reductions (gemm_tiles.hip); false when the operands do not meet its rules
bool launch_bgemm_tiles(const GemmDev& p, int which, hipStream_t st, hipEvent_t t0, hipEvent_t t1);
constexpr int kLongSteps = 1536;
// From K = 1536 on its k steps pay (K = 768: level, the launch and the first loads are most of the time).  Its tiles are
// 32 x 32, 64 x 64, 96 x 64 and 128 x 64 (variants 0..3); 64 x 32 and 128 x 128 stay with the ring (350 x 768, K = 3072
// on 64 x 64 12.0 us, 11.3 there; 3312 x 768 on 128 x 128 level), and so do the second and fourth with an m-major B, whose
// fragments take two transposing reads each: of the ring's time, operands in the caches / from memory, k-major B 0.95-1.05 /
// 0.92-1.01 (64 x 64) and 0.94-0.99 / 0.96-1.03 (128 x 64), m-major 1.00-1.08 / 0.98-1.03 and 0.99-1.03 / 1.00-1.04
// (1000 x 768, K = 1536-3072 7.7-12.1 us in the ring, 8.3-12.8 here); 32 x 32 and 96 x 64 0.76-0.98 and 0.82-1.05 either way.
static int tiles_variant(int M, int N, int K, bool b_kmajor) {
  if (K < kLongSteps) return -1;
  auto tiles = [&](int64_t bm, int64_t bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn); };
  if (tiles(32, 32) <= 256) return 0;
  if (tiles(64, 32) <= 256) return -1;
  if (tiles(64, 64) <= 256) return b_kmajor ? 1 : -1;
  if (tiles(96, 64) <= 256) return 2;
  return b_kmajor && tiles(128, 64) <= 256 ? 3 : -1;
}

// Weight gradients that nothing runs beside keep the parts of their reduction (gemm_splits) and with them the
// number of units.  Where these fit one round the ring's 128 x 128 tiles are ahead of the 128 x 256 tiles, which
// leave half of it idle (256 units at 4096 x 1024: 208 us against 257 at K = 20480, 28.9 against 34.9 at K = 2000;
// 36 at 768 x 768 in one part 178 against 253), and of the 128 x 128 kernel without the ring (245, 35.6;
// 228).  From where a second round starts they are behind both (288 at 768 x 3072: 60 us against 52 and 54 at
// K = 6400).
static bool ring_wgrad(int M, int N, int splits) {
  return ((M + BM - 1) / BM) * ((N + BN - 1) / BN) * splits <= 256;
}

static bool aligned16(const void* p) { return (((uintptr_t)p) & 15) == 0; }

bool gemm(int dtype, const GemmArgs& g, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) {             // nothing to launch that could carry the events
    for (hipEvent_t e : {g.time_start, g.time_stop})
      if (e) note_marking(hipEventRecord(e, st));
    return true;
  }
  GemmDev p;
  p.A = g.A; p.B = g.B; p.C = g.C; p.bias = g.bias; p.resid = g.resid; p.gelu_out = g.gelu_out; p.a_rowsum = g.a_rowsum;
  p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc; p.ldr = g.ldr;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.a_k = g.a_kmajor; p.b_k = g.b_kmajor; p.c_f32 = g.c_f32; p.gelu = g.gelu;
  p.splits = 1; p.partial = nullptr;
  p.a_tail_zero = g.a_tail_zero ? 1 : 0;
  if (p.gelu && (p.c_f32 || !p.gelu_out)) return false;
  const int rule_rows = g.rule_rows > 0 ? g.rule_rows : g.M;
  if (dtype == F32) {
    launch_sgemm(p, rule_rows, st, g.time_start, g.time_stop);
    return true;
  }
  if ((g.lda & 7) || (g.ldb & 7) || !aligned16(g.A) || !aligned16(g.B)) return false;
  const bool may_split = g.workspace && g.c_f32 && !g.bias && !g.resid && !g.gelu && aligned16(g.workspace);
  const int rule_k = g.k_blocks ? g.k_padded : g.K;
  // the parts of the reduction, in whole steps of `unit` indices (of the padded batch)
  auto cut = [&](int splits, int unit) {
    const int steps = (rule_k + unit - 1) / unit, per = (steps + splits - 1) / splits;
    p.splits = splits;
    for (int i = 0; i <= splits; ++i) {
      int64_t at = std::min<int64_t>((int64_t)i * per * unit, rule_k);
      if (g.k_blocks && at < rule_k) at = (int64_t)g.k_blocks[at / kRowBlock] * kRowBlock;
      p.kb[i] = (int)std::min<int64_t>(at, g.K);
    }
  };
  cut(1, 64);
  auto splits_for = [&](int want) {
    const int by_k = (rule_k + 255) / 256;                                   // >= 256 reduction indices per part
    const int sp = want < by_k ? want : by_k;
    return may_split && sp > 1 && g.workspace_bytes >= ((size_t)sp * g.M * g.N + (size_t)sp * g.M) * 4 ? sp : 1;
  };
  // vector epilogue: eight consecutive columns (16 bytes of bf16, 32 of fp32) per access
  const bool vec = (g.ldc & (g.c_f32 ? 3 : 7)) == 0 && aligned16(g.C) &&
                   (!g.resid || ((g.ldr & 7) == 0 && aligned16(g.resid))) && (!g.bias || aligned16(g.bias)) &&
                   (!g.gelu_out || aligned16(g.gelu_out));
  p.vec = vec ? 1 : 0;
  // a very long reduction behind a k-major A and an m-major B (the head's data gradient)
  if (g.a_kmajor && !g.b_kmajor && g.K >= kLongK && rule_rows >= 256 && g.N >= 256 && !g.bias && !g.resid && !g.gelu &&
      !g.a_rowsum && rule_rows <= kLongKRows) {
    int sp = long_k_splits(rule_rows, g.N);
    if (sp > 1 && !(g.workspace && aligned16(g.workspace) && g.workspace_bytes >= (size_t)sp * g.M * g.N * 4)) sp = 1;
    cut(sp, 64);
    p.partial = sp > 1 ? (float*)g.workspace : nullptr;
    if (launch_bgemm_large(p, st, g.time_start, sp > 1 ? nullptr : g.time_stop)) {
      if (sp > 1) launch_splitk_reduce(p, st, g.time_stop);
      return true;
    }
    cut(1, 64); p.partial = nullptr;
  }
  // few output tiles and a long reduction (weight gradients): cut k so the whole chip works
  {
    const int sp = splits_for(gemm_splits(g.M, g.N));
    if (sp > 1) { cut(sp, 32); p.partial = (float*)g.workspace; }
  }
  // Weight gradients, which are what has parts or row sums, and those of the iteration without a bias; what is left
  // of products with both operands m-major goes by its output tiles as the others do
  const bool wgrad = !g.a_kmajor && !g.b_kmajor && rule_k >= 1024 && (g.beside || g.a_rowsum || p.splits > 1);
  if (wgrad && !g.beside && ring_wgrad(g.M, g.N, p.splits) &&
      launch_bgemm_ring(p, 3, st, g.time_start, p.splits > 1 ? nullptr : g.time_stop)) {
    if (p.splits > 1) launch_splitk_reduce(p, st, g.time_stop);
    return true;
  }
  // Weight gradients: 128 x 256 tiles, also where they leave compute units idle (128 units at 4096 x 1024,
  // whose reduction is not cut; 144 at 3072 x 768 in two parts).  Beside another product that pays although it
  // is slower alone (see ring_wgrad): a unit's time is a quarter less and the other stream's kernels have
  // the rest.  Iterations against the 128 x 128 kernels: bert_large_stress 256 x 512
  // 1.06 of the speed, bert_large 64 x 320 1.03, 16 x 256 1.02, 16 x 100 1.06, bert_base 32 x 512 1.01, 32 x 200
  // 1.01, 32 x 88 1.02, padded 12 x 397 1.02, gpt2_medium 16 x 1024 1.00, 4 x 400 1.05, 12 x 400 0.99.
  // Same parts and order of every sum, so the same bits.
  if (wgrad && g.M >= 256 && g.N >= 256 && tiles128(g.M, g.N) <= 256 &&
      launch_bgemm_large128(p, st, g.time_start, p.splits > 1 ? nullptr : g.time_stop)) {
    if (p.splits > 1) launch_splitk_reduce(p, st, g.time_stop);
    return true;
  }
  // Forward and data-gradient products that one round of smaller tiles covers, by the rows that are left of the batch;
  // of a product run in two halves on two streams by the whole batch's, so that the halves share the round,
  // and only where it has too many and the reduction is long, by the half's own.  No bit depends on it.  By the
  // padded batch's rows padded iterations take 1.02-1.11 of the time (bert_stages 32 x 332, bert_large 40 x 300,
  // bert_base 20 x 150, gpt2_medium 10 x 500).  Without the halves' own rows bert_large 32 x 150 takes 1.038,
  // bert_base 32 x 180 1.028, 32 x 200 and 32 x 256 1.011-1.013, gpt2_medium 16 x 397 1.020; with them for short
  // reductions too bert_stages 16 x 200 and gpt2_medium 8 x 300 1.014, bert_base 32 x 88 1.004; by them
  // alone bert_stages 16 x 200 1.006, bert_large 16 x 256 1.004.
  if (p.splits == 1 && !g.a_rowsum) {
    for (const int rows : {g.whole_rows > 0 ? g.whole_rows : g.M, g.M}) {
      if (rows < g.whole_rows && g.K < kLongSteps) break;
      const int small = tiles_variant(rows, g.N, g.K, g.b_kmajor), which = ring_variant(rows, g.N);
      if (small >= 0 && launch_bgemm_tiles(p, small, st, g.time_start, g.time_stop)) return true;
      if (which >= 0 && launch_bgemm_ring(p, which, st, g.time_start, g.time_stop)) return true;
    }
  }
  // large tiles (a choice made from the shape alone)
  if (p.splits == 1) {
    const int rows = large_rows(g.M, g.N, g.K, g.a_kmajor, g.b_kmajor);
    if (rows == 256 && launch_bgemm_large(p, st, g.time_start, g.time_stop)) return true;
    if (rows && launch_bgemm_large128(p, st, g.time_start, g.time_stop)) return true;   // (row sums of few columns too)
  }
  // B m-major (weight gradients, data gradients): the direct-to-LDS pipeline measures faster there;
  // the register-staged kernel below is ahead when both operands are k-major (forward)
  if (!g.b_kmajor && launch_bgemm_dma(p, st, g.time_start, p.splits > 1 ? nullptr : g.time_stop)) {
    if (p.splits > 1) launch_splitk_reduce(p, st, g.time_stop);
    return true;
  }
#define LAUNCH_(AKV, BKV) launch_bgemm<AKV, BKV>(p, st, g.time_start, g.time_stop)
  if (g.a_kmajor && g.b_kmajor) LAUNCH_(true, true);
  else if (g.a_kmajor && !g.b_kmajor) LAUNCH_(true, false);
  else if (!g.a_kmajor && g.b_kmajor) LAUNCH_(false, true);
  else LAUNCH_(false, false);
#undef LAUNCH_
  return true;
}

}  // namespace mk
