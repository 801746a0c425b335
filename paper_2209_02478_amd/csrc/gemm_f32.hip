// fp32 GEMM on the bf16 matrix cores: every operand value is the sum of three bf16 values.
//
// C[M,N] = sum_k A(m,k) B(n,k).  x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1:
// both differences are exact in fp32, |x1| <= 2^-9 |x|, |x2| <= 2^-18 |x|, and what x2's own rounding
// leaves is below 2^-27 |x|.  Of the nine products of a pair the six down to 2^-18 are multiplied
// (v_mfma_f32_16x16x32_bf16: products exact, sums in fp32); the other three are below 2^-26 of the
// product, under the 2^-24 that one fp32 rounding costs.  x0 y0 has accumulators of its own; the other five, 2^-8
// of it, share a second set, added at the end.  (In one set the small products lose their last bits against a large
// sum, 1.7 times the error of fp32 MFMAs.)  A single way's turn has two slices, each with its own sum of x0 y0: two
// sums of half the size and half the roundings have half the error, in the same time (the registers of the 128 x 128
// tiles do not hold them).  Errors against 64 bits, 2-norm over the result's, fp32 MFMAs -> here, on N(0,1) operands:
// 768 indices 2.5e-7 -> 1.1-1.6e-7, 3072 5.0-9.9e-7 -> 1.6-3.4e-7, 30522 1.6e-6 -> 0.8e-6.  With both operands of one
// sign, whose errors are a third to two thirds of those, there is no bias, and 0.2-0.75 times the error, or 1.3-1.4
// times it where the fp32 MFMAs had four partial sums and the 128 x 128 tiles have one (1408 x 2304, K = 768
// 1.0e-7 -> 1.4e-7; 4096 x 768, K = 3072 7.4e-7 -> 2.6e-7).
//
// What is split is the value times 2^16, and sums are times 2^32 until the end: every part is then a bf16 number, denormal
// ones included, for every fp32 value down to 2^-149.  (Unscaled, the third part loses bits from 2^-109 on and the
// second from 2^-118.  The scale costs 2-3 %, 5 % at K = 3072 on 96 x 64 tiles; to look for lost bits instead, an OR for
// every two values, and take such tiles again 1-3 %.)
// What the split cannot carry are values that are not finite or above 2^112, and sums above 2^96: they leave
// an output that is infinite or NaN.  A wave that finds one takes its tile again with fp32 MFMAs straight from memory,
// so infinities, NaN and large values come out as fp32 arithmetic has them (some 20 times slower).
//
// The matrix cores multiply bf16 at 16 times their fp32 rate, so six products leave 2.7; the split takes the rest.  On
// 128 x 128 tiles the matrix pipes are busy for 53-58 % of the time and vector instructions issue in 52-59 %, on 96 x 64
// (three waves to a SIMD) 34-38 and 48.  Against 64 x 64 and 32 x 32 tiles of fp32 MFMAs, us, without the scale: 1408 x 768,
// K = 768 27 -> 19, K = 3072 87 -> 57; 1408 x 3072 78 -> 54; weight gradients over 1408 rows, 3072 x 768 74 -> 51,
// 30528 x 768 926 -> 371; 4096 x 3072, K = 768 173 -> 105; 64 x 768, K = 3072 27 -> 19; 64 columns and indices level.
//
// Block tiles are BM x BN with one thread or more for 8 floats of a slice, and WK ways of sharing the reduction: k way
// g takes the 32-index slices g, g + WK, ... and the ways' accumulators are added in order at the end.
// A way's first 4 BM threads bring its A slice, the next 4 BN its B slice: 8 floats each, loaded ND slices ahead into
// registers, split there (13 vector instructions for two values) and stored as three bf16 planes into
// one of two buffers while the MFMAs work on the other; any that are left only multiply.  A wave issues one vector
// instruction in 8 clocks, a SIMD one in 4, and splitting takes two or more for each MFMA: hence many waves with small
// parts of the tile each, three or four on every SIMD.  128 x 128 tiles: 16 waves of 32 x 32; 64 x 64: 8 waves of
// 16 x 32 a way; 32 x 32: 4 waves of 16 x 16 a way; 96 x 64 and 128 x 64, 12 and 16 waves of 16 x 32, where the squares
// have just begun a second round or leave units idle (us, the squares' best -> these): 1408 x 768, K = 3072 77 -> 57;
// 1408 x 3072 58 -> 54; 360 x 3072 24.4 -> 18.9; data gradient 1408 x 768, K = 30522 722 -> 614; weight gradient
// 2304 x 768 over 2256 rows 69 -> 59.
//
// LDS plane of an operand slice: slots of 64 bytes (32 indices), their four 16-byte chunks turned
// against bank conflicts.  Which row a fragment's lane holds is free, as it only renames outputs: lane l of
// fragment f of a wave's group (F fragments of 16) holds row F l + f of it.  With F = 2 a lane of the
// accumulator tiles then holds neighbouring columns, and an operand stored with the rows contiguous is
// turned by the registers it is loaded to: a thread loads two rows of four indices and stores each
// row's four indices.
#include "gemm_device.h"

#include <algorithm>
#include <type_traits>

namespace mk {

namespace {

constexpr int SGROUP_M = 4;                       // row panels per tile group (L2 reuse)
constexpr int SK = 32;                            // reduction indices of a slice
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Lane l's row of a fragment of 16 lies in slot place<F>(l) of the fragment's 16, so that the rows that
// one store instruction of an m-major operand covers (2 u + e of a group, e fixed) are neighbouring slots.
template <int F> __device__ __forceinline__ int place(int l) { return F == 2 ? l : (l & 1) * 8 + (l >> 1); }
template <int F> __device__ __forceinline__ int lane_of(int s) { return F == 2 ? s : (s & 7) * 2 + (s >> 3); }
// Bytes from a plane's start to chunk k8 of a slot.  16-byte reads are served to lanes 0-3, 12-15, 20-23 and
// 24-27 at a time (then 4-11, 16-19, 28-31; the upper half alike): the turns keep these in different banks.
template <int F> __device__ __forceinline__ int slot_at(int slot, int k8) {
  const int b = (slot >> 2) & 3, turn = F == 2 ? (0x78 >> 2 * b) & 3 : (b >> 1) | (b & 1) << 1;   // 0 2 3 1, 0 2 1 3
  return slot * 64 + ((k8 ^ turn) << 4);
}

// Two values -> the three bf16 parts of each times kUp, a's in the low halves
constexpr float kUp = 0x1p16f, kDown = 0x1p-32f;
__device__ __forceinline__ void split2(float a, float b, uint32_t (&w)[3]) {
  a *= kUp;
  b *= kUp;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    w[p] = pack_bf16x2(a, b);
    a -= __uint_as_float(w[p] << 16);
    b -= __uint_as_float(w[p] & 0xFFFF0000u);
  }
}

// One thread's share of its operand's slice, two rows' four indices.  k-major: two loads of four floats;
// else four of two.
struct Share {
  const float* base;                                // the same for the wave: the tile's first row, first index of the slice
  int64_t step;                                     // to the next slice of this way
  uint32_t off[2];                                  // bytes from there (m-major: off[0], to the first index)
  int at[2];                                        // where the rows' indices are stored in a plane
  int row;                                          // m-major: the first of the rows
  int k;                                            // first index inside the slice
};

// k-major: the slot that load i of thread t goes to, and its row
template <int R> __device__ __forceinline__ int slot_of(int i, int t) { return i * (R / 2) + (t >> 3); }
template <int R, int F>
__device__ __forceinline__ int row_of(int i, int t) {
  const int slot = slot_of<R>(i, t), q = slot % (16 * F);
  return slot - q + F * lane_of<F>(q % 16) + q / 16;
}
// R rows from r0 on, of `rows` altogether; F: fragments of a wave's group in this operand; thread t of 4 R
template <bool KM, int R, int F>
__device__ __forceinline__ void init_share(Share& s, const float* X, int64_t ldx, int rows, int r0, int t, int k0, int stride) {
  if (KM) {
    s.base = X + (int64_t)r0 * ldx + k0;
    s.step = stride;
    s.k = (t & 7) * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int slot = slot_of<R>(i, t), row = row_of<R, F>(i, t);
      s.off[i] = 4u * ((uint32_t)(r0 + row < rows ? row : 0) * (uint32_t)ldx + (uint32_t)s.k);   // rows past the end: never stored
      s.at[i] = slot_at<F>(slot, s.k >> 3) + (s.k & 4) * 2;
    }
  } else {
    constexpr int U = 8 * F;                        // units of two rows in a group
    const int u = t % U, group = t / (8 * U), row = group * 16 * F + 2 * u;
    s.base = X + (int64_t)k0 * ldx + r0;
    s.step = (int64_t)stride * ldx;
    s.k = t / U % 8 * 4;
    s.row = r0 + row;
    s.off[0] = 4u * ((uint32_t)s.k * (uint32_t)ldx + (uint32_t)row);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 2 * u + i, slot = group * 16 * F + (r % F) * 16 + place<F>(r / F);
      s.at[i] = slot_at<F>(slot, s.k >> 3) + (s.k & 4) * 2;
    }
  }
}
__device__ __forceinline__ const float* at_bytes(const float* p, uint32_t off) { return (const float*)((const char*)p + off); }
// index e of row i among the loaded floats
template <bool KM> __device__ __forceinline__ float get(const float (&v)[8], int i, int e) { return v[KM ? 4 * i + e : 2 * e + i]; }

}  // namespace

// WM x WN waves of (16 TM) x (16 TN) a way, WK ways, ND slices of a way requested ahead of the one that is split
template <bool AK, bool BKM, int WM, int WN, int TM, int TN, int WK, int ND>
__global__ __launch_bounds__(64 * WM * WN * WK) void sgemm_split_kernel(GemmDev p, int vec_in, int vec_out, int tiles_n,
                                                                       int total, int per_xcd) {
  constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN, GT = 64 * WM * WN;
  constexpr int FIRST_B = 4 * BM, FIRST_IDLE = FIRST_B + 4 * BN;             // threads of a way: 8 floats of a slice each
  static_assert(FIRST_IDLE <= GT && BM % 16 == 0 && BN % 16 == 0, "enough threads, whole waves for either operand");
  constexpr int PLANE_A = BM * 64, PLANE_B = BN * 64, OPERAND = 3 * PLANE_A, SLICE = OPERAND + 3 * PLANE_B;   // bytes
  constexpr int SMEM = 2 * WK * SLICE;
  static_assert(SMEM >= (WK > 1 ? WK * BM * BN * 4 : 0) && SMEM >= WK * 8 * BM * 4, "space for the ways' accumulators and row sums");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  // block id -> XCD-contiguous runs of tiles, in groups of SGROUP_M row panels
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= total) return;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tgroup = tile / (SGROUP_M * tiles_n), first_m = tgroup * SGROUP_M;
  const int gsize = min(tiles_m - first_m, SGROUP_M);
  const int in_group = tile - tgroup * SGROUP_M * tiles_n;
  const int tile_m = first_m + in_group % gsize, tile_n = in_group / gsize;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int way = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  const int gt = tid % GT, l16 = lane & 15, q = lane >> 4;
  const bool mine_a = wave % (WM * WN) < FIRST_B / 64;               // this wave brings A, else B,
  const bool idle = wave % (WM * WN) >= FIRST_IDLE / 64;             // else nothing
  const float* A = (const float*)p.A;
  const float* B = (const float*)p.B;

  Share sh;
  float raw[ND][8];
  float rs[2] = {0.f, 0.f};
  const bool do_rowsum = p.a_rowsum && tile_n == 0 && mine_a;
  if (mine_a) init_share<AK, BM, TM>(sh, A, p.lda, p.M, m0, gt, way * SK, WK * SK);
  else if (!idle) init_share<BKM, BN, TN>(sh, B, p.ldb, p.N, n0, gt - FIRST_B, way * SK, WK * SK);
  const bool km = mine_a ? AK : BKM;
  const int rows = mine_a ? p.M : p.N;
  // an m-major operand is read along its rows, so its tile has to be whole; a k-major one is not
  const bool whole = vec_in && (km || (mine_a ? m0 + BM : n0 + BN) <= rows);
  const int64_t ld = mine_a ? p.lda : p.ldb;
  auto load = [&](float (&v)[8], auto kmajor) {      // a slice inside K, of a whole tile
    if (decltype(kmajor)::value) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float4 x = *(const float4*)at_bytes(sh.base, sh.off[i]);
        v[4 * i] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 x = *(const float2*)at_bytes(sh.base + i * ld, sh.off[0]);
        v[2 * i] = x.x; v[2 * i + 1] = x.y;
      }
    }
    sh.base += sh.step;
  };
  auto fetch = [&](int t, float (&v)[8], auto kmajor) {                // slice t of this way
    const int kb = (t * WK + way) * SK;
    if (whole && kb + SK <= p.K) { load(v, kmajor); return; }
    constexpr bool KM = decltype(kmajor)::value;     // the tile's or the reduction's end, or no 16-byte accesses: one by one
    const float* X = mine_a ? A : B;
    const int r0 = mine_a ? m0 : n0, kl = p.K - kb - sh.k;            // indices left from this share's first
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = KM ? r0 + (mine_a ? row_of<BM, TM>(i, gt) : row_of<BN, TN>(i, gt - FIRST_B)) : sh.row + i;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[KM ? 4 * i + e : 2 * e + i] =
            e < kl && row < rows ? X[KM ? (int64_t)row * ld + kb + sh.k + e : (int64_t)(kb + sh.k + e) * ld + row] : 0.f;
    }
    sh.base += sh.step;
  };
  char* mine = smem + way * SLICE;
  char* to = mine + (mine_a ? 0 : OPERAND);
  const int plane = mine_a ? PLANE_A : PLANE_B;
  // half a row split; behind the second half the row's indices are stored
  uint32_t lo[3], hi[3];
  auto split_half = [&](const float (&v)[8], int half, int buf, auto kmajor) {
    constexpr bool KM = decltype(kmajor)::value;
    const int i = half >> 1;
    if (half % 2 == 0) { split2(get<KM>(v, i, 0), get<KM>(v, i, 1), lo); return; }
    split2(get<KM>(v, i, 2), get<KM>(v, i, 3), hi);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *(uint2*)(to + buf * (WK * SLICE) + pl * plane + sh.at[i]) = make_uint2(lo[pl], hi[pl]);
  };
  auto add_rows = [&](const float (&v)[8], auto kmajor) {            // (weight gradients have row sums, others hardly ever)
    constexpr bool KM = decltype(kmajor)::value;
    if (!AK || do_rowsum) {
#pragma unroll
      for (int i = 0; i < 2; ++i) rs[i] += (get<KM>(v, i, 0) + get<KM>(v, i, 1)) + (get<KM>(v, i, 2) + get<KM>(v, i, 3));
    }
  };
  auto stash = [&](const float (&v)[8], int buf, auto kmajor) {
#pragma unroll
    for (int half = 0; half < 4; ++half) split_half(v, half, buf, kmajor);
    add_rows(v, kmajor);
  };
  // sums of the large products, of every ND-th slice where a way has the reduction to itself; and of the five others
  constexpr int SETS = WK == 1 ? ND : 1;
  f32x4 sums[SETS][TM][TN], low[TM][TN];
  f32x4 (&acc)[TM][TN] = sums[0];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      low[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < SETS; ++s) sums[s][i][j] = low[i][j];
    }

  const int a_at = slot_at<TM>(wm * 16 * TM + place<TM>(l16), q), b_at = OPERAND + slot_at<TN>(wn * 16 * TN + place<TN>(l16), q);
  bf16x8 fa[3][TM], fb[3][TN];
  auto read = [&](int buf) {
    const char* at = mine + buf * (WK * SLICE);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[pl][i] = *(const bf16x8*)(at + pl * PLANE_A + i * 1024 + a_at);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[pl][j] = *(const bf16x8*)(at + pl * PLANE_B + j * 1024 + b_at);
    }
  };
  auto multiply = [&](int x, int u) {               // one of the six products of a turn's slice u
    constexpr int PA[6] = {0, 1, 0, 1, 2, 0}, PB[6] = {0, 0, 1, 1, 0, 2};
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f32x4& sum = x ? low[i][j] : sums[u % SETS][i][j];
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[PA[x]][i], fb[PB[x]][j], sum, 0, 0, 0);
      }
  };
  // While slice t is multiplied, slice t + 1 is split and stored and slice t + 1 + ND requested, the
  // vector instructions of the split dealt out between the MFMAs.  Slice t waits in raw[t % ND].
  const int n_slices = (p.K + WK * SK - 1) / (WK * SK);
  const int n_whole = whole ? max(0, (p.K / SK - way + WK - 1) / WK) : 0;    // of this way, inside K
  auto work = [&](auto kmajor, auto loads) {
    constexpr bool LOADS = decltype(loads)::value;
    if (LOADS) {
      fetch(0, raw[0], kmajor);
      stash(raw[0], 0, kmajor);
#pragma unroll
      for (int u = 1; u <= ND; ++u)
        if (u < n_slices) fetch(u, raw[u % ND], kmajor);
    }
    __syncthreads();
    int t = 0;
    if (!AK || !p.a_rowsum)
      for (; t + 2 * ND < n_whole; t += ND) {
#pragma unroll
        for (int u = 0; u < ND; ++u) {
          float (&v)[8] = raw[(u + 1) % ND];
          const int buf = ND % 2 ? (t + u) & 1 : u & 1;
          read(buf);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < 6; ++x) {
            if (LOADS && x >= 1 && x <= 4) split_half(v, x - 1, buf ^ 1, kmajor);
            if (LOADS && x == 5) { add_rows(v, kmajor); load(v, kmajor); }
            multiply(x, u);
#pragma unroll
            for (int f = 0; f < TM * TN; ++f) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            // an MFMA
              __builtin_amdgcn_sched_group_barrier(0x002, 12 / (TM * TN), 0);               // vector instructions
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          __syncthreads();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    while (t < n_slices) {
#pragma unroll
      for (int u = 0; u < ND; ++u, ++t) {
        if (t >= n_slices) break;
        float (&v)[8] = raw[(u + 1) % ND];
        read(t & 1);
        if (LOADS && t + 1 < n_slices) {
          stash(v, (t + 1) & 1, kmajor);
          if (t + 1 + ND < n_slices) fetch(t + 1 + ND, v, kmajor);
        }
#pragma unroll
        for (int x = 0; x < 6; ++x) multiply(x, u);
        __syncthreads();
      }
    }
  };
  // every wave meets the others n_slices + 1 times, whichever of the two it runs
  if (FIRST_IDLE < GT && idle) work(std::true_type(), std::false_type());
  else if (AK == BKM || mine_a) work(std::integral_constant<bool, AK>(), std::true_type());
  else work(std::integral_constant<bool, BKM>(), std::true_type());

#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int s = 1; s < SETS; ++s) acc[i][j] += sums[s][i][j];
      acc[i][j] += low[i][j];
    }
  if (p.a_rowsum && tile_n == 0) {                    // the shares of a row, in order
    float* red = (float*)smem;                        // [8 WK shares][BM rows]
    if (mine_a) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        red[(way * 8 + sh.k / 4) * BM + (AK ? row_of<BM, TM>(i, gt) : sh.row - m0 + i)] = rs[i];
    }
    __syncthreads();
    if (tid < BM && m0 + tid < p.M) {
      float s = red[tid];
#pragma unroll
      for (int i = 1; i < 8 * WK; ++i) s += red[i * BM + tid];
      p.a_rowsum[m0 + tid] = s;
    }
    __syncthreads();
  }
  if (WK > 1) {                                       // every way finishes its share of a tile's rows: register 4 i + r
    f32x4* red = (f32x4*)smem;                        // [way][wave of the way][fragment][lane]
    constexpr int WAVE = TM * TN * 64;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) red[wave * WAVE + (i * TN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f32x4 s = red[(wave % (WM * WN)) * WAVE + (i * TN + j) * 64 + lane];
#pragma unroll
        for (int w = 1; w < WK; ++w) s += red[(w * WM * WN + wave % (WM * WN)) * WAVE + (i * TN + j) * 64 + lane];
        acc[i][j] = s;
      }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] *= kDown;  // (infinities stay what they are)
  // register r of fragment (i, j): row TM * (4 q + r) + i, column TN * l16 + j of the wave's part
  const int mw = m0 + wm * 16 * TM, nw = n0 + wn * 16 * TN;
  bool finite = true;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) finite = finite && fabsf(acc[i][j][r]) < INFINITY;
  if (__any(!finite)) {
#pragma unroll 1
    for (int f = 0; f < TM * TN; ++f) {
      const int i = f / TN, j = f % TN;
      const int m = min(mw + TM * l16 + i, p.M - 1), n = min(nw + TN * l16 + j, p.N - 1);   // (rows past the end: never stored)
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int k = q; k - q < p.K; k += 4) {
        const float a = k < p.K ? A[AK ? (int64_t)m * p.lda + k : (int64_t)k * p.lda + m] : 0.f;
        const float b = k < p.K ? B[BKM ? (int64_t)n * p.ldb + k : (int64_t)k * p.ldb + n] : 0.f;
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, s, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (WK == 1 || (i * 4 + r) % WK == way) epilogue<float>(p, mw + TM * (4 * q + r) + i, nw + TN * l16 + j, s[r]);
    }
    return;
  }
  const int n = nw + TN * l16, left = p.N - n;        // this lane's columns
  const bool vec = vec_out && left >= TN;
  typedef float vecn __attribute__((ext_vector_type(TN)));
  auto fetch_n = [&](const float* from) {
    vecn v = 0.f;
    if (vec) return *(const vecn*)from;
#pragma unroll
    for (int j = 0; j < TN; ++j) if (j < left) v[j] = from[j];
    return v;
  };
  auto put = [&](float* dst, vecn v) {
    if (vec) { *(vecn*)dst = v; return; }
#pragma unroll
    for (int j = 0; j < TN; ++j) if (j < left) dst[j] = v[j];
  };
  vecn bias = 0.f;
  if (p.bias) bias = fetch_n((const float*)p.bias + n);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (WK > 1 && (i * 4 + r) % WK != way) continue;
      const int m = mw + TM * (4 * q + r) + i;
      if (m >= p.M) continue;
      vecn v;
#pragma unroll
      for (int j = 0; j < TN; ++j) v[j] = acc[i][j][r];
      if (p.bias) v += bias;
      if (p.resid) v += fetch_n((const float*)p.resid + (int64_t)m * p.ldr + n);
      put((float*)p.C + (int64_t)m * p.ldc + n, v);
      if (p.gelu) {
#pragma unroll
        for (int j = 0; j < TN; ++j) v[j] = p.gelu == GELU_TANH ? gelu_tanh(v[j]) : gelu_erf(v[j]);
        put((float*)p.gelu_out + (int64_t)m * p.ldc + n, v);
      }
    }
}

// The block tiles and ways of the reduction a product may get, and about what it then takes in units of 10 ns:
// `rounds` of 256 tiles (one for each compute unit), each with a start and end and `slices` of 32 indices.
// The one-way 64 x 64 and the two-way 32 x 32 tiles leave room for others on their unit, so from the
// second round on rounds overlap; the 128 x 128 ones on all units get in each other's way.  Fitted to 16-4096 rows or
// indices of 768, 2304, 3072 and 30528 columns; where two are close the estimate may take the second by up to 10 %.
constexpr int kVariants = 7;
static int64_t estimate(int which, int64_t M, int64_t N, int64_t K) {
  constexpr int kM[kVariants] = {128, 64, 64, 32, 32, 96, 128}, kN[kVariants] = {128, 64, 64, 32, 32, 64, 64};
  constexpr int kAlone[kVariants] = {500, 460, 500, 460, 460, 520, 550}, kAloneSlice[kVariants] = {95, 46, 35, 19, 15, 54, 66};
  constexpr int kMany[kVariants] = {600, 230, 500, 240, 400, 480, 500}, kManySlice[kVariants] = {115, 40, 35, 16, 15, 56, 68};
  const int64_t m = kM[which], n = kN[which], rounds = ((M + m - 1) / m * ((N + n - 1) / n) + 255) / 256, slices = (K + SK - 1) / SK;
  return rounds == 1 ? kAlone[which] + slices * kAloneSlice[which] : rounds * (kMany[which] + slices * kManySlice[which]);
}

template <bool AK, bool BKM>
static void launch_f32(const GemmDev& p, int which, int vec_in, int vec_out, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
#define GO_(WM, WN, TM, TN, WK, ND)                                                                                       \
  {                                                                                                                       \
    constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN;                                                                   \
    const int tiles_n = (p.N + BN - 1) / BN, total = (p.M + BM - 1) / BM * tiles_n, per = (total + 7) / 8;                \
    launch_marked((sgemm_split_kernel<AK, BKM, WM, WN, TM, TN, WK, ND>), dim3(per * 8), dim3(64 * WM * WN * WK),  \
                          0, st, t0, t1, p, vec_in, vec_out, tiles_n, total, per);                                     \
  }
  switch (which) {
    case 0: GO_(4, 4, 2, 2, 1, 1) break;
    case 1: GO_(4, 2, 1, 2, 1, 2) break;
    case 2: GO_(4, 2, 1, 2, 2, 2) break;
    case 3: GO_(2, 2, 1, 1, 2, 3) break;
    case 4: GO_(2, 2, 1, 1, 4, 2) break;
    case 5: GO_(6, 2, 1, 2, 1, 2) break;
    default: GO_(8, 2, 1, 2, 1, 2) break;
  }
#undef GO_
}

// rows: the row count the choice is made from (a product run in two row ranges must sum in the same order
// as the whole)
void launch_sgemm(const GemmDev& p, int rows, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  auto aligned = [](const void* q, int64_t ld) { return (((uintptr_t)q) & 15) == 0 && (ld & 3) == 0; };
  // 16-byte loads at 32-bit offsets from a tile's start
  const int vec_in = aligned(p.A, p.lda) && aligned(p.B, p.ldb) && std::max(p.lda, p.ldb) < (int64_t)1 << 23 ? 1 : 0;
  const int vec_out = aligned(p.C, p.ldc) && (!p.resid || aligned(p.resid, p.ldr)) && (!p.bias || aligned(p.bias, 0)) &&
                      (!p.gelu || aligned(p.gelu_out, 0)) ? 1 : 0;
  int which = 0;
  for (int w = 1; w < kVariants; ++w)
    if (estimate(w, rows, p.N, p.K) < estimate(which, rows, p.N, p.K)) which = w;
#define GO_(AKV, BKV) launch_f32<AKV, BKV>(p, which, vec_in, vec_out, st, t0, t1)
  if (p.a_k && p.b_k) GO_(true, true);
  else if (p.a_k) GO_(true, false);
  else if (p.b_k) GO_(false, true);
  else GO_(false, false);
#undef GO_
}

}  // namespace mk
