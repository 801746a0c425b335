// Row-wise, HBM-bound kernels: LayerNorm forward/backward, GELU backward, softmax
// cross-entropy, embedding forward/backward, dtype conversion.
//
// One 64-lane wave owns one row; lane i holds columns i, i+64, ... in registers, so a
// wave load touches one contiguous run of the row and reductions are wave shuffles.
// Column reductions over rows (LayerNorm's dgamma/dbeta) are two-stage with a row ->
// chunk mapping fixed by the shape, so they are reproducible bit for bit (no atomics).
#include "device_common.h"
#include <initializer_list>

#include "kernels.h"
#include "philox.h"

namespace mk {

constexpr int kRowsPerChunk = 16;   // rows summed by one block of a two-stage column reduction
constexpr int kMaxNPL = 16;         // columns per lane: supports rows up to 1024 wide

// ---------------------------------------------------------------- LayerNorm forward
template <typename T, int NPL>
__device__ __forceinline__ void row_stats(const float (&v)[NPL], int H, int lane, float& mean, float& rstd,
                                          float eps) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NPL; ++i) if (lane + 64 * i < H) s += v[i];
  mean = wave_sum(s) / (float)H;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NPL; ++i) if (lane + 64 * i < H) { float d = v[i] - mean; q += d * d; }
  rstd = rsqrtf(wave_sum(q) / (float)H + eps);
}

template <typename TX, typename T, int NPL>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const TX* __restrict__ x, const T* __restrict__ gamma,
                                                     const T* __restrict__ beta, T* __restrict__ y, int Trows,
                                                     int H, float eps) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= Trows) return;
  const TX* xr = x + (int64_t)row * H;
  float v[NPL];
#pragma unroll
  for (int i = 0; i < NPL; ++i) { int c = lane + 64 * i; v[i] = c < H ? ld<TX>(xr + c) : 0.f; }
  float mean, rstd;
  row_stats<T, NPL>(v, H, lane, mean, rstd, eps);
  T* yr = y + (int64_t)row * H;
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    int c = lane + 64 * i;
    if (c < H) st<T>(yr + c, (v[i] - mean) * rstd * ld<T>(gamma + c) + ld<T>(beta + c));
  }
}

// ---------------------------------------------------------------- LayerNorm backward
// Block = 4 waves = kRowsPerChunk rows.  Statistics are recomputed from x; `add` (optional) is a
// residual-path gradient added to the result.  dx may alias dy; add must not alias dx.  Each wave keeps
// per-column sums of dy*xhat and dy over its rows; the four waves are combined through LDS
// in wave order and written as one partial row.
template <typename TD, typename TX, typename T, int NPL>
__global__ __launch_bounds__(256) void ln_bwd_kernel(const TD* __restrict__ dy, const TX* __restrict__ x,
                                                     const T* __restrict__ gamma, T* __restrict__ dx,
                                                     const T* __restrict__ add, float* __restrict__ partial,
                                                     int Trows, int H, float eps) {
  __shared__ float red[4][2][64 * NPL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float g[NPL], sg[NPL], sb[NPL];
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    int c = lane + 64 * i;
    g[i] = c < H ? ld<T>(gamma + c) : 0.f;
    sg[i] = 0.f; sb[i] = 0.f;
  }
  for (int rr = 0; rr < kRowsPerChunk / 4; ++rr) {
    int row = blockIdx.x * kRowsPerChunk + rr * 4 + wave;
    if (row >= Trows) break;
    const TX* xr = x + (int64_t)row * H;
    const TD* dr = dy + (int64_t)row * H;
    float v[NPL], d[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      int c = lane + 64 * i;
      v[i] = c < H ? ld<TX>(xr + c) : 0.f;
      d[i] = c < H ? ld<TD>(dr + c) : 0.f;
    }
    float mean, rstd;
    row_stats<T, NPL>(v, H, lane, mean, rstd, eps);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      float xh = (v[i] - mean) * rstd;
      v[i] = xh;
      sg[i] += d[i] * xh;
      sb[i] += d[i];
      float dxh = d[i] * g[i];
      d[i] = dxh;
      s1 += dxh;
      s2 += dxh * xh;
    }
    s1 = wave_sum(s1) / (float)H;
    s2 = wave_sum(s2) / (float)H;
    T* or_ = dx + (int64_t)row * H;
    const T* ar = add ? add + (int64_t)row * H : nullptr;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      int c = lane + 64 * i;
      if (c < H) st<T>(or_ + c, rstd * (d[i] - s1 - v[i] * s2) + (ar ? ld<T>(ar + c) : 0.f));
    }
  }
#pragma unroll
  for (int i = 0; i < NPL; ++i) { red[wave][0][lane + 64 * i] = sg[i]; red[wave][1][lane + 64 * i] = sb[i]; }
  __syncthreads();
  float* prow = partial + (int64_t)blockIdx.x * 2 * H;
  for (int c = threadIdx.x; c < 2 * H; c += 256) {
    int which = c / H, col = c - which * H;
    float s = red[0][which][col];
    s += red[1][which][col];
    s += red[2][which][col];
    s += red[3][which][col];
    prow[c] = s;
  }
}

// out[c] = sum over partial rows, c in [0, ncols): 16 row groups x 16 columns per block,
// each group adds its rows in order, groups are combined in order.  (Fallback for column counts
// or pointers that do not allow 16-byte accesses.)
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ partial,
                                                              const int32_t* __restrict__ chunk_at, int P,
                                                              int ncols, float* __restrict__ out0,
                                                              float* __restrict__ out1, int split) {
  __shared__ float red[16][17];
  const int cg = threadIdx.x & 15, rg = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + cg;
  float s = 0.f;
  if (c < ncols)
    for (int r = rg; r < P; r += 16) {
      const int at = chunk_at ? chunk_at[r] : r;
      if (at >= 0) s += partial[(int64_t)at * ncols + c];
    }
  red[rg][cg] = s;
  __syncthreads();
  if (rg == 0 && c < ncols) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[i][cg];
    if (c < split) out0[c] = t; else out1[c - split] = t;
  }
}

// The same sums with whole 128-byte lines: a block owns 32 columns, 32 row groups x 8 lanes of four
// columns; a group adds rows g, g + 32, ... in order, eight loads in flight at a time (a chain of
// dependent loads costs a memory latency per row), groups are combined in order.  MAPPED: partial row
// r is row chunk_at[r], or zeros.  No load hangs on a condition, that would put a wait between any two:
// rows past the end and left-out ones read row 0 instead (8192 rows of 2048 with a condition on the
// row 120 us, without 31; 400 rows of 1536 6.6 and 3.9).
template <bool MAPPED>
__global__ __launch_bounds__(256) void reduce_partials_vec_kernel(const float* __restrict__ partial,
                                                                  const int32_t* __restrict__ chunk_at, int P,
                                                                  int ncols, float* __restrict__ out0,
                                                                  float* __restrict__ out1, int split) {
  __shared__ float4 red[32][8];
  const int cq = threadIdx.x & 7, rg = threadIdx.x >> 3;
  const int c = blockIdx.x * 32 + cq * 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c < ncols)
    for (int r0 = rg; r0 < P; r0 += 32 * 8) {
      int at[8];
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = r0 + 32 * u;
        at[u] = MAPPED ? chunk_at[min(r, P - 1)] : r;
        if (r >= P) at[u] = -1;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *(const float4*)(partial + (int64_t)max(at[u], 0) * ncols + c);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool in = at[u] >= 0;
        s.x += in ? v[u].x : 0.f; s.y += in ? v[u].y : 0.f; s.z += in ? v[u].z : 0.f; s.w += in ? v[u].w : 0.f;
      }
    }
  red[rg][cq] = s;
  __syncthreads();
  if (rg == 0 && c < ncols) {
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 32; ++i) { const float4 q = red[i][cq]; t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w; }
    const float e[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { const int cc = c + k; if (cc < split) out0[cc] = e[k]; else out1[cc - split] = e[k]; }
  }
}

// ---------------------------------------------------------------- vectorised row access
// 16-byte chunks: 8 bf16 or 4 fp32 per lane and access; lane l owns chunks l, l+64, ...
template <typename T> struct Chunk;
template <> struct Chunk<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) {
    const uint4 u = *(const uint4*)p;
    v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xFFFF0000u);
    v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xFFFF0000u);
    v[4] = __uint_as_float(u.z << 16); v[5] = __uint_as_float(u.z & 0xFFFF0000u);
    v[6] = __uint_as_float(u.w << 16); v[7] = __uint_as_float(u.w & 0xFFFF0000u);
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    uint4 u;
    u.x = pack_bf16x2(v[0], v[1]);
    u.y = pack_bf16x2(v[2], v[3]);
    u.z = pack_bf16x2(v[4], v[5]);
    u.w = pack_bf16x2(v[6], v[7]);
    *(uint4*)p = u;
  }
};
template <> struct Chunk<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void load(const float* p, float (&v)[4]) {
    const float4 u = *(const float4*)p;
    v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
  }
  static __device__ __forceinline__ void store(float* p, const float (&v)[4]) {
    *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
  }
};

// E consecutive elements of type T as floats (E = Chunk<storage type>::N; fp32 sources of a bf16
// configuration take two 16-byte loads)
template <typename T, int E>
__device__ __forceinline__ void load_elems(const T* p, float (&v)[E]) {
  constexpr int N = Chunk<T>::N;
#pragma unroll
  for (int k = 0; k < E / N; ++k) {
    float t[N];
    Chunk<T>::load(p + k * N, t);
#pragma unroll
    for (int e = 0; e < N; ++e) v[k * N + e] = t[e];
  }
}

// mean and 1/std of a row held as NC chunks per lane (chunks >= nchunks hold zeros)
template <int NC, int E>
__device__ __forceinline__ void chunk_stats(const float (&v)[NC][E], int nchunks, int lane, int H, float eps,
                                            float& mean, float& rstd) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int e = 0; e < E; ++e) s += v[i][e];
  mean = wave_sum(s) / (float)H;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i)
    if (lane + 64 * i < nchunks)
#pragma unroll
      for (int e = 0; e < E; ++e) { const float d = v[i][e] - mean; q += d * d; }
  rstd = rsqrtf(wave_sum(q) / (float)H + eps);
}

// the masked and scaled elements of chunk c of a row: v = keep ? v * scale : 0
template <int E>
__device__ __forceinline__ void drop_chunk(const DropDesc& d, int64_t mask_row, int H, int c, float (&v)[E]) {
  const uint64_t blk = ((uint64_t)mask_row * H + (uint64_t)c * E) >> 2;
#pragma unroll
  for (int q = 0; q < E / 4; ++q) {
    const uint4 w = drop_words(d, blk + q);
    v[4 * q] = w.x >= d.thr ? v[4 * q] * d.scale : 0.f;
    v[4 * q + 1] = w.y >= d.thr ? v[4 * q + 1] * d.scale : 0.f;
    v[4 * q + 2] = w.z >= d.thr ? v[4 * q + 2] * d.scale : 0.f;
    v[4 * q + 3] = w.w >= d.thr ? v[4 * q + 3] * d.scale : 0.f;
  }
}
struct DropRows { DropDesc d; Rows rows; int B, L; };

// DROP: x = resid + dropout(x) first, written back (what LayerNorm's backward reads); the pass is
// bound by memory, so making the masks here instead of in a pass of their own saves that pass.
template <typename TX, typename T, int NC, bool DROP>
__global__ __launch_bounds__(256) void ln_fwd_vec_kernel(TX* __restrict__ x, const T* __restrict__ gamma,
                                                         const T* __restrict__ beta, T* __restrict__ y,
                                                         int Trows, int H, float eps, const T* __restrict__ resid,
                                                         DropRows dr) {
  constexpr int E = Chunk<T>::N;
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= Trows) return;
  const int nchunks = H / E;
  TX* xr = x + (int64_t)row * H;
  float v[NC][E];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunks) load_elems<TX, E>(xr + c * E, v[i]);
    else
#pragma unroll
      for (int e = 0; e < E; ++e) v[i][e] = 0.f;
  }
  if (DROP) {
    const int64_t mask_row = padded_row(dr.rows, row, dr.B, dr.L);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = lane + 64 * i;
      if (c >= nchunks) continue;
      float r[E];
      Chunk<T>::load(resid + (int64_t)row * H + c * E, r);
      drop_chunk<E>(dr.d, mask_row, H, c, v[i]);
#pragma unroll
      for (int e = 0; e < E; ++e) v[i][e] = rnd<TX>(v[i][e] + r[e]);
      constexpr int N = Chunk<TX>::N;
#pragma unroll
      for (int k = 0; k < E / N; ++k) {
        float t[N];
#pragma unroll
        for (int e = 0; e < N; ++e) t[e] = v[i][k * N + e];
        Chunk<TX>::store(xr + c * E + k * N, t);
      }
    }
  }
  if (DROP && !y) return;
  float mean, rstd;
  chunk_stats<NC, E>(v, nchunks, lane, H, eps, mean, rstd);
  T* yr = y + (int64_t)row * H;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunks) {
      float g[E], b[E], o[E];
      Chunk<T>::load(gamma + c * E, g);
      Chunk<T>::load(beta + c * E, b);
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = (v[i][e] - mean) * rstd * g[e] + b[e];
      Chunk<T>::store(yr + c * E, o);
    }
  }
}

// Backward: a block takes kRowsPerChunk rows, WAVES waves of it a row each in turn, with AHEAD rows' elements in registers.
// A row is a chain of four sums over its columns.  Up to 256 blocks, one to a compute unit, 16 waves take a row each instead
// of four rows one after the other (with the reduction, bf16: 74 x 768 10.4 -> 8.3 us, 3312 x 768 14.3 -> 10.6; fp32 rows
// 9.4 -> 8.6, 12.4 -> 11.1; 4096 x 1024 in fp32 15.6 -> 13.7).  A second block on a unit waits for memory while the first
// works, and 16 waves fall behind 4 (level at 4400-8192 rows, 10000 x 768 25.9 us against 21.3).
// Of 4 waves' rows two are ahead from the third block to a unit on: three waves then fit a SIMD, where four rows'
// elements leave two (bf16 16384 x 768 39.7 -> 36.5 us, 131072 x 1024 296 -> 241; fp32 rows 38.3 -> 35.5, 300 -> 296).
// Four for fewer blocks, which wait for memory and not for each other, and from 14 blocks to a unit on beside the weight
// gradients (layernorm_bwd_rows' `beside`), to which they leave more: iterations with two against four, ms: 16384 rows
// 19.05 / 19.12, 51200 160.1 / 160.4, 65536 198.5 / 196.6, 131072 388.2 / 386.6.  Alone two are ahead there too (with
// four -> two, us: bf16 65536 x 768 134 -> 107, x 1024 141 -> 113; fp32 rows 119 -> 110, 153 -> 150; up to 512 columns
// 1-7 %), and so are wide rows in fp32 (three chunks a lane and more), of which no step measured has that many:
// 57360 x 1024 160 -> 153, with a residual 229 -> 202, 131072 x 1024 351 -> 340, x 768 267 -> 263.
// All four rows' sums side by side gained nothing and lost up to half.  Same outputs as ln_bwd_kernel, and the same order
// of the sums over rows; the sums over a row's columns run over other columns per lane.
template <typename TD, typename TX, typename T, int NC, int AHEAD, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 16 ? 4 : AHEAD == 2 ? 3 : 2)
void ln_bwd_vec_kernel(const TD* __restrict__ dy, const TX* __restrict__ x, const T* __restrict__ gamma, T* __restrict__ dx,
                       const T* __restrict__ add, float* __restrict__ partial, T* __restrict__ masked, DropRows dr, int Trows,
                       int H, float eps) {
  constexpr int E = Chunk<T>::N;
  constexpr int R = kRowsPerChunk / WAVES, Q = E / 4, COLS = 64 * NC * E;
  static_assert((WAVES == 4 || R == 1) && AHEAD <= R, "rows of a wave");
  // a lane's four columns e, .. e + 3 of chunk c are at ((e / 4) (64 NC) + c) 4
  __shared__ __attribute__((aligned(16))) float red[4][2][COLS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nchunks = H / E;
  float g[NC][E], sg[NC][E], sb[NC][E];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunks) Chunk<T>::load(gamma + c * E, g[i]);
#pragma unroll
    for (int e = 0; e < E; ++e) { if (c >= nchunks) g[i][e] = 0.f; sg[i][e] = 0.f; sb[i][e] = 0.f; }
  }
  float v[AHEAD][NC][E], d[AHEAD][NC][E];
  auto fetch = [&](int rr) {
    const int row = blockIdx.x * kRowsPerChunk + rr * WAVES + wave;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = lane + 64 * i;
      if (row < Trows && c < nchunks) {
        load_elems<TX, E>(x + (int64_t)row * H + c * E, v[rr % AHEAD][i]);
        load_elems<TD, E>(dy + (int64_t)row * H + c * E, d[rr % AHEAD][i]);
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) { v[rr % AHEAD][i][e] = 0.f; d[rr % AHEAD][i][e] = 0.f; }
      }
    }
  };
#pragma unroll
  for (int rr = 0; rr < (AHEAD > 1 ? AHEAD - 1 : 1); ++rr) fetch(rr);
#pragma unroll
  for (int rr = 0; rr < R; ++rr) {
    const int row = blockIdx.x * kRowsPerChunk + rr * WAVES + wave;
    if (row >= Trows) break;
    if (AHEAD > 1 && rr + AHEAD - 1 < R) fetch(rr + AHEAD - 1);
    float mean, rstd;
    chunk_stats<NC, E>(v[rr % AHEAD], nchunks, lane, H, eps, mean, rstd);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if (lane + 64 * i < nchunks)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float xh = (v[rr % AHEAD][i][e] - mean) * rstd;
          v[rr % AHEAD][i][e] = xh;
          sg[i][e] += d[rr % AHEAD][i][e] * xh;
          sb[i][e] += d[rr % AHEAD][i][e];
          const float dxh = d[rr % AHEAD][i][e] * g[i][e];
          d[rr % AHEAD][i][e] = dxh;
          s1 += dxh;
          s2 += dxh * xh;
        }
    s1 = wave_sum(s1) / (float)H;
    s2 = wave_sum(s2) / (float)H;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = lane + 64 * i;
      if (c < nchunks) {
        float o[E];
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] = rstd * (d[rr % AHEAD][i][e] - s1 - v[rr % AHEAD][i][e] * s2);
        if (add) {
          float a[E];
          Chunk<T>::load(add + (int64_t)row * H + c * E, a);
#pragma unroll
          for (int e = 0; e < E; ++e) o[e] += a[e];
        }
        Chunk<T>::store(dx + (int64_t)row * H + c * E, o);
        if (masked) {
#pragma unroll
          for (int e = 0; e < E; ++e) o[e] = rnd<T>(o[e]);
          drop_chunk<E>(dr.d, padded_row(dr.rows, row, dr.B, dr.L), H, c, o);
          Chunk<T>::store(masked + (int64_t)row * H + c * E, o);
        }
      }
    }
  }
  // A wave's sums: four waves hold four rows' each; of sixteen, four at a time add their row's to those
  // of the four rows before, in the order in which one wave would.
  float4* mine[2] = {(float4*)red[wave & 3][0] + lane, (float4*)red[wave & 3][1] + lane};
  if (WAVES == 4 || wave < 4) {
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        mine[0][64 * (q * NC + i)] = make_float4(sg[i][4 * q], sg[i][4 * q + 1], sg[i][4 * q + 2], sg[i][4 * q + 3]);
        mine[1][64 * (q * NC + i)] = make_float4(sb[i][4 * q], sb[i][4 * q + 1], sb[i][4 * q + 2], sb[i][4 * q + 3]);
      }
  }
  __syncthreads();
  if (WAVES > 4) {
    for (int turn = 1; turn < WAVES / 4; ++turn) {
      if (wave >> 2 == turn) {
#pragma unroll
        for (int i = 0; i < NC; ++i)
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            float4 a = mine[0][64 * (q * NC + i)], b = mine[1][64 * (q * NC + i)];
            const float(&xh)[E] = v[0][i];
            a.x += sb[i][4 * q] * xh[4 * q]; a.y += sb[i][4 * q + 1] * xh[4 * q + 1];
            a.z += sb[i][4 * q + 2] * xh[4 * q + 2]; a.w += sb[i][4 * q + 3] * xh[4 * q + 3];
            b.x += sb[i][4 * q]; b.y += sb[i][4 * q + 1]; b.z += sb[i][4 * q + 2]; b.w += sb[i][4 * q + 3];
            mine[0][64 * (q * NC + i)] = a;
            mine[1][64 * (q * NC + i)] = b;
          }
      }
      __syncthreads();
    }
  }
  float* prow = partial + (int64_t)blockIdx.x * 2 * H;
  for (int t = threadIdx.x; t < 2 * COLS; t += 64 * WAVES) {
    const int which = t / COLS, at = t % COLS, col = at / 4 % (64 * NC) * E + at / (256 * NC) * 4 + at % 4;
    if (col >= H) continue;
    float s = red[0][which][at];
    s += red[1][which][at];
    s += red[2][which][at];
    s += red[3][which][at];
    prow[which * H + col] = s;
  }
}

// ---------------------------------------------------------------- GELU backward (in place)
// VEC: 16-byte accesses (n may still end inside one): 1408 x 3072 in 7.9 us, eight elements a thread with one
// access each took 30
template <bool VEC>
__global__ __launch_bounds__(256) void gelu_bwd_f32_kernel(float* __restrict__ d, const float* __restrict__ pre,
                                                           int64_t n, int tanh_form) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  if (VEC && i + 4 <= n) {
    float x[4], v[4];
    Chunk<float>::load(pre + i, x);
    Chunk<float>::load(d + i, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= tanh_form ? gelu_tanh_grad(x[e]) : gelu_erf_grad(x[e]);
    Chunk<float>::store(d + i, v);
  } else {
    for (int e = 0; e < 4 && i + e < n; ++e) d[i + e] *= tanh_form ? gelu_tanh_grad(pre[i + e]) : gelu_erf_grad(pre[i + e]);
  }
}
__global__ __launch_bounds__(256) void gelu_bwd_bf16_kernel(bf16_t* __restrict__ d,
                                                            const bf16_t* __restrict__ pre, int64_t n,
                                                            int tanh_form) {
  int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  if (i + 8 <= n) {
    uint4 dv = *(const uint4*)(d + i), pv = *(const uint4*)(pre + i);
    bf16_t* dp = (bf16_t*)&dv;
    const bf16_t* pp = (const bf16_t*)&pv;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = bf16_to_f32(pp[e]);
      float gp = tanh_form ? gelu_tanh_grad(x) : gelu_erf_grad_bf16(x);
      dp[e] = f32_to_bf16(bf16_to_f32(dp[e]) * gp);
    }
    *(uint4*)(d + i) = dv;
  } else {
    for (int e = 0; i + e < n; ++e) {
      float x = bf16_to_f32(pre[i + e]);
      float gp = tanh_form ? gelu_tanh_grad(x) : gelu_erf_grad_bf16(x);
      d[i + e] = f32_to_bf16(bf16_to_f32(d[i + e]) * gp);
    }
  }
}

// ---------------------------------------------------------------- softmax cross-entropy
// One block per row.  Pass 1: running (max, sum of exp) per thread, merged in a fixed tree.
// Pass 2: the row is overwritten with (softmax - onehot)/n_valid, zero for unscored rows and
// for the padding columns [V, ld).
template <typename T>
__global__ __launch_bounds__(256) void xent_kernel(T* __restrict__ logits, int64_t ldl,
                                                   const int32_t* __restrict__ labels,
                                                   float* __restrict__ row_loss, int V, float inv_n) {
  __shared__ float sm[4], ss[4];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  T* lr = logits + (int64_t)row * ldl;
  const int label = labels[row];
  float m = -INFINITY, s = 0.f;
  for (int c = tid; c < V; c += 256) {
    float v = ld<T>(lr + c);
    if (v > m) { s = s * __expf(m - v) + 1.f; m = v; } else { s += __expf(v - m); }
  }
  float wm = wave_max(m);
  s = wave_sum(m == -INFINITY ? 0.f : s * __expf(m - wm));   // threads or waves past a short row hold nothing
  if (lane == 0) { sm[wave] = wm; ss[wave] = s; }
  __syncthreads();
  float bm = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
  float bs = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) bs += sm[w] == -INFINITY ? 0.f : ss[w] * __expf(sm[w] - bm);
  const float lse = bm + __logf(bs);
  if (tid == 0) row_loss[row] = label >= 0 ? lse - ld<T>(lr + label) : 0.f;
  __syncthreads();   // the label's logit is read before the row is overwritten
  const float scale = label >= 0 ? inv_n : 0.f;
  for (int c = tid; c < ldl; c += 256) {
    float g = 0.f;
    if (c < V) g = (__expf(ld<T>(lr + c) - lse) - (c == label ? 1.f : 0.f)) * scale;
    st<T>(lr + c, g);
  }
}

// bf16 rows of up to NCH * THREADS 16-byte chunks: the row is read once, kept in registers as
// fp32, and written once.
template <int THREADS, int NCH>
__global__ __launch_bounds__(THREADS) void xent_bf16_kernel(bf16_t* __restrict__ logits, int64_t ldl,
                                                            const int32_t* __restrict__ labels,
                                                            float* __restrict__ row_loss, int V, float inv_n) {
  constexpr int NW = THREADS / 64;
  __shared__ float sm[NW], ss[NW];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  bf16_t* lr = logits + (int64_t)row * ldl;
  const int label = labels[row];
  const float picked = (tid == 0 && label >= 0) ? bf16_to_f32(lr[label]) : 0.f;
  const int nchunks = (int)(ldl / 8);
  float v[NCH][8];
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = tid + THREADS * i;
    if (c < nchunks) {
      Chunk<bf16_t>::load(lr + c * 8, v[i]);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (c * 8 + e >= V) v[i][e] = -INFINITY;
        m = fmaxf(m, v[i][e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[i][e] = -INFINITY;
    }
  }
  m = wave_max(m);
  if (lane == 0) sm[wave] = m;
  __syncthreads();
  float bm = sm[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) bm = fmaxf(bm, sm[w]);
  // the exponentials are kept (in place of the logits): the gradient is made from them, so each
  // element costs one exponential, not two
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) { v[i][e] = __expf(v[i][e] - bm); s += v[i][e]; }
  s = wave_sum(s);
  if (lane == 0) ss[wave] = s;
  __syncthreads();
  float bs = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) bs += ss[w];
  const float lse = bm + __logf(bs);
  if (tid == 0) row_loss[row] = label >= 0 ? lse - picked : 0.f;
  const float scale = label >= 0 ? inv_n : 0.f;
  const float pscale = scale / bs;                    // softmax = exp(v - max) / sum
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = tid + THREADS * i;
    if (c < nchunks) {
      float g[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int col = c * 8 + e;
        g[e] = v[i][e] * pscale - (col == label ? scale : 0.f);   // columns >= V hold exp(-inf) = 0
      }
      Chunk<bf16_t>::store(lr + c * 8, g);
    }
  }
}

__global__ __launch_bounds__(256) void loss_reduce_kernel(const float* __restrict__ row_loss, int n, float inv_n,
                                                          float* __restrict__ loss) {
  __shared__ float red[256];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) s += row_loss[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = red[0] * inv_n;
}

// ---------------------------------------------------------------- embedding
template <typename T, int NPL>
__global__ __launch_bounds__(256) void embed_fwd_kernel(const int32_t* __restrict__ ids, const T* __restrict__ tok,
                                                        const T* __restrict__ pos, const T* __restrict__ gamma,
                                                        const T* __restrict__ beta, T* __restrict__ sum_out,
                                                        T* __restrict__ y, Rows rows, int Trows, int B, int L, int H,
                                                        float eps, int has_ln) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= Trows) return;
  const T* tr = tok + (int64_t)ids[row] * H;
  const T* pr = pos + (int64_t)(padded_row(rows, row, B, L) % L) * H;
  float v[NPL];
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    int c = lane + 64 * i;
    // the sum is formed in the storage type so LayerNorm sees exactly what is saved
    v[i] = c < H ? rnd<T>(ld<T>(tr + c) + ld<T>(pr + c)) : 0.f;
  }
  if (sum_out) {
    T* sr = sum_out + (int64_t)row * H;
#pragma unroll
    for (int i = 0; i < NPL; ++i) { int c = lane + 64 * i; if (c < H) st<T>(sr + c, v[i]); }
  }
  T* yr = y + (int64_t)row * H;
  if (!has_ln) {
#pragma unroll
    for (int i = 0; i < NPL; ++i) { int c = lane + 64 * i; if (c < H) st<T>(yr + c, v[i]); }
    return;
  }
  float mean, rstd;
  row_stats<T, NPL>(v, H, lane, mean, rstd, eps);
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    int c = lane + 64 * i;
    if (c < H) st<T>(yr + c, (v[i] - mean) * rstd * ld<T>(gamma + c) + ld<T>(beta + c));
  }
}

// VEC (1 or 4) consecutive elements as floats, in one access
template <typename T, int VEC>
__device__ __forceinline__ void load_few(const T* p, float (&v)[VEC]) {
  if (VEC == 1) { v[0] = ld<T>(p); return; }
  if (sizeof(T) == 2) {
    const uint2 u = *(const uint2*)p;
    v[0] = __uint_as_float(u.x << 16); v[1 % VEC] = __uint_as_float(u.x & 0xFFFF0000u);
    v[2 % VEC] = __uint_as_float(u.y << 16); v[3 % VEC] = __uint_as_float(u.y & 0xFFFF0000u);
  } else {
    const float4 u = *(const float4*)p;
    v[0] = u.x; v[1 % VEC] = u.y; v[2 % VEC] = u.z; v[3 % VEC] = u.w;
  }
}

// dpos[p][c] = sum over samples b (in order) of d[row of b's token p][c]; rows p >= L are cleared.
template <typename T>
__global__ __launch_bounds__(256) void embed_bwd_pos_kernel(const T* __restrict__ d, float* __restrict__ dpos,
                                                            Rows rows, int B, int L, int H, int max_seq) {
  int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)max_seq * H) return;
  int p = (int)(idx / H), c = (int)(idx - (int64_t)p * H);
  float s = 0.f;
  if (p < L)
    for (int b = 0; b < B; ++b) {
      const Sample sm = sample_rows(rows, b, L);
      if (p < sm.n) s += ld<T>(d + (sm.first + p) * H + c);
    }
  dpos[idx] = s;
}

// Rows of d at each distinct token id's positions (ascending) are summed and added onto the id's
// gradient row.  A wave owns one id and a group of 64 * VEC columns, with eight rows in flight.
// Frequent ids (separators, articles) would leave one wave with a serial chain over thousands of
// rows: an id with more than kLongRun positions is shared out over its block's 16 waves, whose
// parts are added in order.  (One wave with one row in flight took 16.7 ms for an id at 4800
// positions, H = 768; a memory latency per row.)
constexpr int kLongRun = 64;
template <typename T, int VEC>
__global__ __launch_bounds__(1024) void embed_bwd_tok_kernel(const T* __restrict__ d, const int32_t* __restrict__ ids,
                                                             const int32_t* __restrict__ order,
                                                             const int32_t* __restrict__ seg, int n_seg,
                                                             float* __restrict__ dtok, int H) {
  __shared__ float red[16][64 * VEC];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = (blockIdx.y * 64 + lane) * VEC;
  const bool in = c < H;
  auto sum_rows = [&](int beg, int end, float (&acc)[VEC]) {
    for (int k0 = beg; k0 < end; k0 += 64) {
      const int n = min(64, end - k0);
      const int mine = lane < n ? order[k0 + lane] : 0;
      for (int j = 0; j < n; j += 8) {
        float v[8][VEC];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t row = __builtin_amdgcn_readlane(mine, (j + u) & 63);
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[u][e] = 0.f;
          if (j + u < n && in) load_few<T, VEC>(d + row * H + c, v[u]);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[e] += v[u][e];
      }
    }
  };
  auto add_to = [&](int id, const float (&acc)[VEC]) {
    float* out = dtok + (int64_t)id * H + c;
#pragma unroll
    for (int e = 0; e < VEC; ++e) out[e] += acc[e];
  };
  const int s0 = blockIdx.x * 16;
  bool any_long = false;                              // the same in every wave
  for (int q = 0; q < 16 && s0 + q < n_seg; ++q) any_long |= seg[s0 + q + 1] - seg[s0 + q] > kLongRun;
  if (s0 + wave < n_seg) {
    const int beg = seg[s0 + wave], end = seg[s0 + wave + 1];
    if (end - beg <= kLongRun) {
      float acc[VEC] = {};
      sum_rows(beg, end, acc);
      if (in) add_to(ids[order[beg]], acc);
    }
  }
  if (!any_long) return;
  for (int q = 0; q < 16 && s0 + q < n_seg; ++q) {
    const int beg = seg[s0 + q], end = seg[s0 + q + 1];
    if (end - beg <= kLongRun) continue;
    const int part = (end - beg + 15) / 16;
    float acc[VEC] = {};
    sum_rows(beg + wave * part, min(end, beg + (wave + 1) * part), acc);
#pragma unroll
    for (int e = 0; e < VEC; ++e) red[wave][lane * VEC + e] = acc[e];
    __syncthreads();
    if (wave == q && in) {
      float tot[VEC] = {};
      for (int w = 0; w < 16; ++w)
#pragma unroll
        for (int e = 0; e < VEC; ++e) tot[e] += red[w][lane * VEC + e];
      add_to(ids[order[beg]], tot);
    }
    __syncthreads();
  }
}

template <typename T>
__global__ __launch_bounds__(256) void convert_kernel(const float* __restrict__ src, T* __restrict__ dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) st<T>(dst + i, src[i]);
}

template <typename T>
__global__ __launch_bounds__(256) void widen_kernel(const T* __restrict__ src, float* __restrict__ dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = ld<T>(src + i);
}

// dst[i] = (resid ? resid[i] : 0) + keep(i) * scale * src[i]; element i reads word i % 4 of block
// i / 4.  Four elements per thread; dst may be src.
template <typename TIO, typename TR>
__global__ __launch_bounds__(256) void dropout_kernel(TIO* __restrict__ dst, const TIO* src, const TR* __restrict__ resid,
                                                      int64_t n, DropDesc d, Rows rows, int B, int L, int H) {
  const int64_t blk = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t i0 = 4 * blk;
  if (i0 >= n) return;
  uint64_t mask_blk = (uint64_t)blk;
  if (rows.ends) {
    const int row = (int)(i0 / H);
    mask_blk = ((uint64_t)padded_row(rows, row, B, L) * H + (uint64_t)(i0 - (int64_t)row * H)) >> 2;
  }
  const uint4 w4 = drop_words(d, mask_blk);
  const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
  const int cnt = (int)min((int64_t)4, n - i0);
  for (int e = 0; e < cnt; ++e) {
    float v = w[e] >= d.thr ? ld<TIO>(src + i0 + e) * d.scale : 0.f;
    if (resid) v += ld<TR>(resid + i0 + e);
    st<TIO>(dst + i0 + e, v);
  }
}

// Element-wise, fp32 arithmetic:
//   m = b1 m + (1-b1) g;  v = b2 v + (1-b2) g^2
//   p = p - lr * ( (m / c1) / (sqrt(v / c2) + eps) + wd p )      (decoupled weight decay)
// The low-precision copy, when there is one, is the new master value rounded to nearest-even.
// Bound by memory: 28 or 30 bytes an element in seven or eight streams, none of which fits a cache until it is
// touched again, so all but the low-precision copy, which the next forward reads, go past the caches (non-temporal
// loads and stores; either alone gains nothing).  kAdamBlocks blocks share a chunk of kAdamChunk elements of one
// tensor, four elements a thread and no loop: stretches of 8 KB that start together.  110 M parameters in bf16, call
// behind call: a block for a chunk, through the caches, 650 us (5.05 TB/s), so 616 (5.3); behind an iteration's
// backward, which leaves some of the gradients in the last cache, 645 and 550-570.
constexpr int kAdamThreads = 512, kAdamBlocks = kAdamChunk / (4 * kAdamThreads);
__global__ __launch_bounds__(kAdamThreads) void adamw_kernel(const AdamTensor* __restrict__ tensors,
                                                             const AdamChunk* __restrict__ chunks, AdamHyper h) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const AdamChunk ck = chunks[blockIdx.x / kAdamBlocks];
  const AdamTensor t = tensors[ck.tensor];
  const float wd = t.decay ? h.weight_decay : 0.f;
  bf16_t* lowp = (bf16_t*)t.lowp;
  const int64_t i = ck.start + 4 * ((int64_t)(blockIdx.x % kAdamBlocks) * kAdamThreads + threadIdx.x);
  if (i + 4 <= t.n) {                                 // (tensor starts are 256-byte aligned)
    const f32x4 g4 = __builtin_nontemporal_load((const f32x4*)(t.grad + i)), m4 = __builtin_nontemporal_load((const f32x4*)(t.m + i)),
                v4 = __builtin_nontemporal_load((const f32x4*)(t.v + i)), p4 = __builtin_nontemporal_load((const f32x4*)(t.master + i));
    const float gs[4] = {g4[0], g4[1], g4[2], g4[3]};
    float ms[4] = {m4[0], m4[1], m4[2], m4[3]}, vs[4] = {v4[0], v4[1], v4[2], v4[3]}, ps[4] = {p4[0], p4[1], p4[2], p4[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ms[e] = h.beta1 * ms[e] + (1.f - h.beta1) * gs[e];
      vs[e] = h.beta2 * vs[e] + (1.f - h.beta2) * gs[e] * gs[e];
      ps[e] -= h.lr * ((ms[e] * h.inv_c1) / (sqrtf(vs[e] * h.inv_c2) + h.eps) + wd * ps[e]);
    }
    const f32x4 m = {ms[0], ms[1], ms[2], ms[3]}, v = {vs[0], vs[1], vs[2], vs[3]}, p = {ps[0], ps[1], ps[2], ps[3]};
    __builtin_nontemporal_store(m, (f32x4*)(t.m + i));
    __builtin_nontemporal_store(v, (f32x4*)(t.v + i));
    if (lowp) {
      __builtin_nontemporal_store(p, (f32x4*)(t.master + i));
      uint2 w;
      w.x = pack_bf16x2(p[0], p[1]);
      w.y = pack_bf16x2(p[2], p[3]);
      *(uint2*)(lowp + i) = w;
    } else {
      *(f32x4*)(t.master + i) = p;                    // (fp32: the master is what the next forward reads)
    }
  } else {
    for (int64_t j = i; j < t.n; ++j) {
      const float g = t.grad[j];
      const float m = h.beta1 * t.m[j] + (1.f - h.beta1) * g;
      const float v = h.beta2 * t.v[j] + (1.f - h.beta2) * g * g;
      float pv = t.master[j];
      pv -= h.lr * ((m * h.inv_c1) / (sqrtf(v * h.inv_c2) + h.eps) + wd * pv);
      t.m[j] = m; t.v[j] = v; t.master[j] = pv;
      if (lowp) lowp[j] = f32_to_bf16(pv);
    }
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* __restrict__ p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------- launchers
#define DISPATCH_NPL(H, M)                      \
  do {                                          \
    int npl_ = ((H) + 63) / 64;                 \
    if (npl_ <= 1) { M(1); }                    \
    else if (npl_ <= 2) { M(2); }               \
    else if (npl_ <= 4) { M(4); }               \
    else if (npl_ <= 8) { M(8); }               \
    else if (npl_ <= 12) { M(12); }             \
    else { M(16); }                             \
  } while (0)

// rows whose length is a whole number of 16-byte chunks and whose storage is 16-byte aligned
template <typename T>
static bool vec_ok(int H, std::initializer_list<const void*> ptrs) {
  if (H % Chunk<T>::N) return false;
  for (const void* p : ptrs) if (p && (((uintptr_t)p) & 15)) return false;
  return true;
}

template <typename TX, typename T>
static void ln_fwd_t(const void* x, const void* g, const void* b, void* y, int T_, int H, float eps,
                     hipStream_t st) {
  dim3 grid((T_ + 3) / 4);
  if (vec_ok<T>(H, {x, g, b, y})) {
    const int nc = (H / Chunk<T>::N + 63) / 64;
#define V_(NC) hipLaunchKernelGGL((ln_fwd_vec_kernel<TX, T, NC, false>), grid, dim3(256), 0, st, (TX*)const_cast<void*>(x), \
                                   (const T*)g, (const T*)b, (T*)y, T_, H, eps, (const T*)nullptr, DropRows())
    if (nc <= 1) { V_(1); return; }
    if (nc <= 2) { V_(2); return; }
    if (nc <= 4) { V_(4); return; }
#undef V_
  }
#define M_(NPL) hipLaunchKernelGGL((ln_fwd_kernel<TX, T, NPL>), grid, dim3(256), 0, st, (const TX*)x, (const T*)g, \
                                   (const T*)b, (T*)y, T_, H, eps)
  DISPATCH_NPL(H, M_);
#undef M_
}
void layernorm_fwd(int dtype, const void* x, bool x_f32, const void* gamma, const void* beta, void* y, int T_,
                   int H, float eps, hipStream_t st) {
  if (T_ <= 0) return;
  if (dtype != BF16) ln_fwd_t<float, float>(x, gamma, beta, y, T_, H, eps, st);
  else if (x_f32) ln_fwd_t<float, bf16_t>(x, gamma, beta, y, T_, H, eps, st);
  else ln_fwd_t<bf16_t, bf16_t>(x, gamma, beta, y, T_, H, eps, st);
}

template <typename TX, typename T>
static void drop_ln_fwd_t(void* x, const void* resid, const void* g, const void* b, void* y, int T_, int H, float eps,
                          const DropRows& dr, hipStream_t st) {
  dim3 grid((T_ + 3) / 4);
  const int nc = (H / Chunk<T>::N + 63) / 64;
#define V_(NC) hipLaunchKernelGGL((ln_fwd_vec_kernel<TX, T, NC, true>), grid, dim3(256), 0, st, (TX*)x, (const T*)g, \
                                   (const T*)b, (T*)y, T_, H, eps, (const T*)resid, dr)
  if (nc <= 1) V_(1); else if (nc <= 2) V_(2); else V_(4);
#undef V_
}
void dropout_layernorm_fwd(int dtype, void* x, bool x_f32, const void* resid, const void* gamma, const void* beta,
                           void* y, int T_, int H, float eps, const DropDesc& d, const Rows& rows, int B, int L,
                           hipStream_t st) {
  if (T_ <= 0) return;
  const bool vec = dtype == BF16 ? vec_ok<bf16_t>(H, {x, resid, gamma, beta, y}) : vec_ok<float>(H, {x, resid, gamma, beta, y});
  if (!vec) {                                         // the same in two passes
    dropout_apply(dtype, x, x, x_f32, resid, (int64_t)T_ * H, d, rows, B, L, H, st);
    if (y) layernorm_fwd(dtype, x, x_f32, gamma, beta, y, T_, H, eps, st);
    return;
  }
  const DropRows dr{d, rows, B, L};
  if (dtype != BF16) drop_ln_fwd_t<float, float>(x, resid, gamma, beta, y, T_, H, eps, dr, st);
  else if (x_f32) drop_ln_fwd_t<float, bf16_t>(x, resid, gamma, beta, y, T_, H, eps, dr, st);
  else drop_ln_fwd_t<bf16_t, bf16_t>(x, resid, gamma, beta, y, T_, H, eps, dr, st);
}

template <typename TD, typename TX, typename T>
static void ln_bwd_t(const void* dy, const void* x, const void* g, void* dx, const void* add, float* partial,
                     int T_, int H, float eps, const LnBwdMasked& ex, hipStream_t st, hipEvent_t done, bool beside) {
  dim3 grid((T_ + kRowsPerChunk - 1) / kRowsPerChunk);
  if (vec_ok<T>(H, {dy, x, g, dx, add, ex.masked})) {
    const int nc = (H / Chunk<T>::N + 63) / 64;
    const bool few = grid.x <= 256, ahead2 = grid.x > 512 && (!beside || grid.x <= 3584 || nc > 2);
#define A_(NC, AHEAD, WAVES) LAUNCH_MARKED_((ln_bwd_vec_kernel<TD, TX, T, NC, AHEAD, WAVES>), grid, dim3(64 * WAVES), st, \
                                   done, (const TD*)dy, (const TX*)x, (const T*)g, (T*)dx, (const T*)add, partial, (T*)ex.masked, \
                                   DropRows{ex.d, ex.rows, ex.B, ex.L}, T_, H, eps)
#define V_(NC) do { if (few) A_(NC, 1, 16); else if (ahead2) A_(NC, 2, 4); else A_(NC, 4, 4); } while (0)
    if (nc <= 1) { V_(1); return; }
    if (nc <= 2) { V_(2); return; }
    if constexpr (sizeof(T) == 4) {                   // (bf16 rows of 1024 are two chunks a lane)
      // against the kernel below 600 x 768 with the reduction 16.1 -> 10.7 us, 6352 x 1024 30.7 -> 24.2
      if (nc <= 3) { V_(3); return; }
      V_(4);
      return;
    }
#undef V_
#undef A_
  }
#define M_(NPL) hipLaunchKernelGGL((ln_bwd_kernel<TD, TX, T, NPL>), grid, dim3(256), 0, st, (const TD*)dy,    \
                                   (const TX*)x, (const T*)g, (T*)dx, (const T*)add, partial, T_, H, eps)
  DISPATCH_NPL(H, M_);
#undef M_
  if (ex.masked)                                      // dx is stored: the mask in a pass of its own
    dropout_apply(sizeof(T) == 2 ? BF16 : F32, ex.masked, dx, false, nullptr, (int64_t)T_ * H, ex.d, ex.rows, ex.B, ex.L, H, st);
  if (done) note_marking(hipEventRecord(done, st));
}
void layernorm_bwd_rows(int dtype, const void* dy, bool dy_f32, const void* x, bool x_f32, const void* gamma, void* dx,
                        const void* add, float* partial, int T_, int H, float eps, const LnBwdMasked& ex, hipStream_t st,
                        hipEvent_t done, bool beside) {
  if (T_ <= 0) return;
  if (dtype != BF16) ln_bwd_t<float, float, float>(dy, x, gamma, dx, add, partial, T_, H, eps, ex, st, done, beside);
  else if (dy_f32 && x_f32) ln_bwd_t<float, float, bf16_t>(dy, x, gamma, dx, add, partial, T_, H, eps, ex, st, done, beside);
  else if (dy_f32) ln_bwd_t<float, bf16_t, bf16_t>(dy, x, gamma, dx, add, partial, T_, H, eps, ex, st, done, beside);
  else if (x_f32) ln_bwd_t<bf16_t, float, bf16_t>(dy, x, gamma, dx, add, partial, T_, H, eps, ex, st, done, beside);
  else ln_bwd_t<bf16_t, bf16_t, bf16_t>(dy, x, gamma, dx, add, partial, T_, H, eps, ex, st, done, beside);
}
static_assert(kRowsPerChunk == kRowBlock, "padding is left out in whole chunks");
void layernorm_bwd_reduce(const float* partial, float* dgamma, float* dbeta, const int32_t* chunk_at, int T_, int H,
                          hipStream_t st) {
  if (T_ <= 0) return;
  int P = (T_ + kRowsPerChunk - 1) / kRowsPerChunk;
  if ((H & 1) == 0 && (((uintptr_t)partial) & 15) == 0) {    // rows of 2H floats: every float4 inside a row, lines aligned
    const dim3 grid((2 * H + 31) / 32);
    if (chunk_at) hipLaunchKernelGGL(reduce_partials_vec_kernel<true>, grid, dim3(256), 0, st, partial, chunk_at, P, 2 * H, dgamma, dbeta, H);
    else hipLaunchKernelGGL(reduce_partials_vec_kernel<false>, grid, dim3(256), 0, st, partial, chunk_at, P, 2 * H, dgamma, dbeta, H);
  } else
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((2 * H + 15) / 16), dim3(256), 0, st, partial, chunk_at, P, 2 * H, dgamma,
                       dbeta, H);
}
void layernorm_bwd(int dtype, const void* dy, bool dy_f32, const void* x, bool x_f32, const void* gamma, void* dx,
                   const void* add, float* dgamma, float* dbeta, float* partial, int T_, int H, float eps,
                   hipStream_t st) {
  layernorm_bwd_rows(dtype, dy, dy_f32, x, x_f32, gamma, dx, add, partial, T_, H, eps, LnBwdMasked(), st);
  layernorm_bwd_reduce(partial, dgamma, dbeta, nullptr, T_, H, st);
}
int partial_rows(int T_) { return (T_ + kRowsPerChunk - 1) / kRowsPerChunk; }

// Scratch of the entry point that allocates nothing: the per-chunk partial sums of the LayerNorm
// backward.  Each device the library runs on holds its own copy until the process ends; host code
// never uses the array's name as an address, only what hipGetSymbolAddress returned for the
// device that was current.
static __device__ __align__(256) float scratch[kStaticPartialFloats];
static float* g_scratch_of_device[64];

int layernorm_bwd_static(int dtype, const void* dy, bool dy_f32, const void* x, bool x_f32, const void* gamma,
                         void* dx, const void* add, float* dgamma, float* dbeta, int T_, int H, float eps,
                         hipStream_t st) {
  if ((size_t)partial_rows(T_) * 2 * (size_t)H > kStaticPartialFloats) return -1;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -2;
  float* ptr = g_scratch_of_device[dev];
  if (!ptr) {
    if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return -2;
    g_scratch_of_device[dev] = ptr;
  }
  // every partial row that the reduction reads is written by the row pass first: nothing to clear
  layernorm_bwd(dtype, dy, dy_f32, x, x_f32, gamma, dx, add, dgamma, dbeta, ptr, T_, H, eps, st);
  return 0;
}

void gelu_bwd(int dtype, void* d, const void* pre, int64_t n, int tanh_form, hipStream_t st, hipEvent_t done) {
  if (n <= 0) return;
  dim3 grid((unsigned)((n + 2047) / 2048));
  if (dtype == BF16) LAUNCH_MARKED_(gelu_bwd_bf16_kernel, grid, dim3(256), st, done, (bf16_t*)d, (const bf16_t*)pre, n, tanh_form);
  else {
    const dim3 grid4((unsigned)((n + 1023) / 1024));
    if ((((uintptr_t)d | (uintptr_t)pre) & 15) == 0)
      LAUNCH_MARKED_(gelu_bwd_f32_kernel<true>, grid4, dim3(256), st, done, (float*)d, (const float*)pre, n, tanh_form);
    else LAUNCH_MARKED_(gelu_bwd_f32_kernel<false>, grid4, dim3(256), st, done, (float*)d, (const float*)pre, n, tanh_form);
  }
}

void softmax_xent(int dtype, void* logits, int64_t ldl, const int32_t* labels, float* row_loss, float* loss,
                  int T_, int V, int n_valid, hipStream_t st) {
  if (T_ <= 0) return;
  float inv_n = 1.0f / (float)(n_valid > 0 ? n_valid : 1);
  const int64_t nch = ldl / 8;
  if (dtype == BF16 && ldl % 8 == 0 && ((((uintptr_t)logits) & 15) == 0) && nch <= 16 * 1024) {
    bf16_t* lg = (bf16_t*)logits;
    // threads x chunks per thread: the fewest registers per thread that hold the row (more waves per SIMD)
#define X_(TH, NC) hipLaunchKernelGGL((xent_bf16_kernel<TH, NC>), dim3(T_), dim3(TH), 0, st, lg, ldl, labels, row_loss, V, inv_n)
    if (nch <= 4 * 256) X_(256, 4);
    else if (nch <= 8 * 256) X_(256, 8);
    else if (nch <= 4 * 1024) X_(1024, 4);
    else if (nch <= 8 * 512) X_(512, 8);
    else if (nch <= 8 * 1024) X_(1024, 8);
    else X_(1024, 16);
#undef X_
  } else if (dtype == BF16) hipLaunchKernelGGL(xent_kernel<bf16_t>, dim3(T_), dim3(256), 0, st, (bf16_t*)logits, ldl, labels, row_loss, V, inv_n);
  else hipLaunchKernelGGL(xent_kernel<float>, dim3(T_), dim3(256), 0, st, (float*)logits, ldl, labels, row_loss, V, inv_n);
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(256), 0, st, row_loss, T_, inv_n, loss);
}

template <typename T>
static void embed_fwd_t(const int32_t* ids, const void* tok, const void* pos, const void* g, const void* b,
                        void* sum_out, void* y, const Rows& rows, int T_, int B, int L, int H, float eps, int has_ln,
                        hipStream_t st) {
  dim3 grid((T_ + 3) / 4);
#define M_(NPL) hipLaunchKernelGGL((embed_fwd_kernel<T, NPL>), grid, dim3(256), 0, st, ids, (const T*)tok,     \
                                   (const T*)pos, (const T*)g, (const T*)b, (T*)sum_out, (T*)y, rows, T_, B, L, \
                                   H, eps, has_ln)
  DISPATCH_NPL(H, M_);
#undef M_
}
void embed_fwd(int dtype, const int32_t* ids, const void* tok, const void* pos, const void* gamma,
               const void* beta, void* sum_out, void* y, const Rows& rows, int T, int B, int L, int H, float eps,
               int has_ln, hipStream_t st) {
  if (T <= 0) return;
  if (dtype == BF16) embed_fwd_t<bf16_t>(ids, tok, pos, gamma, beta, sum_out, y, rows, T, B, L, H, eps, has_ln, st);
  else embed_fwd_t<float>(ids, tok, pos, gamma, beta, sum_out, y, rows, T, B, L, H, eps, has_ln, st);
}

template <typename T>
static void embed_bwd_t(const void* d, const int32_t* ids, const int32_t* order, const int32_t* seg, int n_seg,
                        float* dtok, float* dpos, const Rows& rows, int B, int L, int H, int max_seq, hipStream_t st) {
  hipLaunchKernelGGL(embed_bwd_pos_kernel<T>, dim3((unsigned)(((int64_t)max_seq * H + 255) / 256)), dim3(256), 0, st,
                     (const T*)d, dpos, rows, B, L, H, max_seq);
  if (n_seg <= 0) return;
  const unsigned gx = (unsigned)((n_seg + 15) / 16);
  if (H % 4 == 0 && (((uintptr_t)d) & 15) == 0)
    hipLaunchKernelGGL((embed_bwd_tok_kernel<T, 4>), dim3(gx, (H + 255) / 256), dim3(1024), 0, st, (const T*)d, ids, order,
                       seg, n_seg, dtok, H);
  else
    hipLaunchKernelGGL((embed_bwd_tok_kernel<T, 1>), dim3(gx, (H + 63) / 64), dim3(1024), 0, st, (const T*)d, ids, order,
                       seg, n_seg, dtok, H);
}
void embed_bwd(int dtype, const void* d, const int32_t* ids, const int32_t* order, const int32_t* seg,
               int n_seg, float* dtok, float* dpos, const Rows& rows, int B, int L, int H, int max_seq, hipStream_t st) {
  if (B * L <= 0) return;
  if (dtype == BF16) embed_bwd_t<bf16_t>(d, ids, order, seg, n_seg, dtok, dpos, rows, B, L, H, max_seq, st);
  else embed_bwd_t<float>(d, ids, order, seg, n_seg, dtok, dpos, rows, B, L, H, max_seq, st);
}

void convert_from_f32(int dtype, const float* src, void* dst, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  dim3 grid((unsigned)((n + 255) / 256));
  if (dtype == BF16) hipLaunchKernelGGL(convert_kernel<bf16_t>, grid, dim3(256), 0, st, src, (bf16_t*)dst, n);
  else hipLaunchKernelGGL(convert_kernel<float>, grid, dim3(256), 0, st, src, (float*)dst, n);
}

void convert_to_f32(int dtype, const void* src, float* dst, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  dim3 grid((unsigned)((n + 255) / 256));
  if (dtype == BF16) hipLaunchKernelGGL(widen_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)src, dst, n);
  else hipLaunchKernelGGL(widen_kernel<float>, grid, dim3(256), 0, st, (const float*)src, dst, n);
}

void dropout_apply(int dtype, void* dst, const void* src, bool io_f32, const void* resid, int64_t n, const DropDesc& d,
                   const Rows& rows, int B, int L, int H, hipStream_t st) {
  if (n <= 0) return;
  dim3 grid((unsigned)(((n + 3) / 4 + 255) / 256));
  if (dtype == BF16 && !io_f32)
    hipLaunchKernelGGL((dropout_kernel<bf16_t, bf16_t>), grid, dim3(256), 0, st, (bf16_t*)dst, (const bf16_t*)src,
                       (const bf16_t*)resid, n, d, rows, B, L, H);
  else if (dtype == BF16)
    hipLaunchKernelGGL((dropout_kernel<float, bf16_t>), grid, dim3(256), 0, st, (float*)dst, (const float*)src,
                       (const bf16_t*)resid, n, d, rows, B, L, H);
  else
    hipLaunchKernelGGL((dropout_kernel<float, float>), grid, dim3(256), 0, st, (float*)dst, (const float*)src,
                       (const float*)resid, n, d, rows, B, L, H);
}

void adamw_update(int lowp_dtype, const AdamTensor* tensors, const AdamChunk* chunks, int n_chunks, AdamHyper h,
                  hipStream_t st) {
  (void)lowp_dtype;                                  // the only low-precision storage type is bf16
  if (n_chunks <= 0) return;
  hipLaunchKernelGGL(adamw_kernel, dim3((unsigned)n_chunks * kAdamBlocks), dim3(kAdamThreads), 0, st, tensors, chunks, h);
}

static thread_local hipError_t first_marking_error = hipSuccess;
void note_marking(hipError_t e) { if (first_marking_error == hipSuccess) first_marking_error = e; }
hipError_t marking_error() { const hipError_t e = first_marking_error; first_marking_error = hipSuccess; return e; }

void fill_zero(void* p, int64_t bytes, hipStream_t st) {
  int64_t n = bytes / 4;
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (uint32_t*)p, n);
}

}  // namespace mk
