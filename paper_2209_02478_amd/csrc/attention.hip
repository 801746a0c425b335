// Fused attention, forward and backward, in fp32 arithmetic on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32), without materialising the L x L matrices.
//
// Head sizes 32 and 64; the fp32 configuration, and bf16 with head size 32 (bf16 with head size 64
// runs on the bf16 kernels of attention_mfma.hip).  A group of W waves (one, two or four; R groups to a block, see
// block_shape) owns 32 query rows (forward, dQ) or 32 key rows (dK/dV) and takes the 32-row tiles of the opposite rows
// in turn; their results are added in wave order at the end.  An MFMA of 32 x 32 x 2 takes 64 clocks, a tile 64-128 of
// them: a wave that walks all tiles of its rows is a chain of 3 us for each, while a short batch has fewer waves than
// the chip has SIMDs.  Nothing is shared but the own rows: a wave loads a tile's rows from memory straight into
// operands of the first products, the next tile's while it works, and passes them through its own LDS for the
// product that needs them by columns, without a barrier.
//
//   forward   O_i = sum_j softmax_j(q_i k_j / sqrt(d)) v_j,   lse_i = log sum_j exp(s_ij)
//   backward  P_ij = exp(s_ij - lse_i), dP_ij = dO_i v_j, dS_ij = P_ij (dP_ij - delta_i),
//             delta_i = dO_i O_i;  dQ = dS K / sqrt(d), dK = dS^T Q / sqrt(d), dV = P^T dO
//
// MFMA 32x32x2 register layout: A, B: lane holds row / column lane%32, index lane/32 of the pair;
// D: lane holds column lane%32, register r holds row 8*(r/4) + 4*(lane/32) + r%4.  Score tiles are
// computed with the wave's own rows as columns, so a lane's 16 registers belong to one of its rows,
// and register r is, as it stands, the B operand of the next product for the index pair
// (8*(r/4) + r%4, the same + 4): the probabilities never leave their registers.
// (One wave per row with a shuffle per key: 222, 407 and 391 us per layer for forward, dQ
// and dK/dV at B = 16, L = 141, 12 heads of 64.)
//
// Every output element is produced by one wave in a fixed order: reproducible bit for bit.
#include "device_common.h"
#include "kernels.h"
#include "philox.h"

namespace mk {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// bf16, head size 64
void attention_fwd_mfma(const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int causal,
                        const DropDesc& drop, hipStream_t st);
void attention_bwd_mfma(const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta, void* dqkv,
                        const Rows& rows, int B, int L, int nh, int causal, const DropDesc& drop, hipStream_t st, hipEvent_t done);

namespace {

constexpr int TR = 32;                 // own rows of a group of waves, and rows of a streamed tile

__device__ __forceinline__ float4 load4(const float* p) { return *(const float4*)p; }
__device__ __forceinline__ float4 load4(const bf16_t* p) {
  const uint2 u = *(const uint2*)p;
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xFFFF0000u));
}
__device__ __forceinline__ void store4(float* p, float4 v) { *(float4*)p = v; }
__device__ __forceinline__ void store4(bf16_t* p, float4 v) {
  *(uint2*)p = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
}

// A tile's row l32 (rows past `last` are read as `last`) as the MFMA takes it: element j of group g is column 8g + 4h + j
template <typename T, int D>
__device__ __forceinline__ void fetch_rows(const T* src, int64_t ld, int r0, int last, int l32, int h, float4 (&f)[D / 8]) {
  const T* p = src + (int64_t)min(r0 + l32, last) * ld + 4 * h;
#pragma unroll
  for (int g = 0; g < D / 8; ++g) f[g] = load4(p + 8 * g);
}
// the same rows as they lie, [row][D + 4], to be read by columns
template <int D>
__device__ __forceinline__ void stash(float* tile, int l32, int h, const float4 (&f)[D / 8]) {
#pragma unroll
  for (int g = 0; g < D / 8; ++g) *(float4*)&tile[l32 * (D + 4) + 8 * g + 4 * h] = f[g];
}
__device__ __forceinline__ void clear(f32x16& v) {
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = 0.f;
}
__device__ __forceinline__ void multiply4(const float4& a, const float4& b, f32x16& s) {
  s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, s, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, s, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, s, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, s, 0, 0, 0);
}
// s = tile rows (A) x own rows (B), which lie in LDS, over the D columns
template <int D>
__device__ __forceinline__ void scores(const float4 (&rows)[D / 8], const float* own, int l32, int h, f32x16& s) {
  clear(s);
#pragma unroll
  for (int g = 0; g < D / 8; ++g) multiply4(rows[g], *(const float4*)&own[l32 * (D + 4) + 8 * g + 4 * h], s);
}
// What the lanes of a wave have stored to LDS before, the others read after: the hardware keeps a wave's accesses
// in order, the compiler has to be told.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}
// acc (rows = head columns, columns = own rows) += tile^T x s
template <int D>
__device__ __forceinline__ void accumulate(const float* tile, int l32, int h, const f32x16& s, f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float* row = &tile[(8 * (r >> 2) + 4 * h + (r & 3)) * (D + 4) + l32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(row[32 * db], s[r], acc[db], 0, 0, 0);
  }
}
// A wave's part of a sum over the tiles goes into its own part of LDS (at least TR * (D + 4) floats) ...
template <int D>
__device__ __forceinline__ void put_part(float* part, int lane, const f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(float4*)&part[((4 * db + g) * 64 + lane) * 4] =
          make_float4(acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]);
}
// ... and behind a barrier wave w adds the n waves' parts of head columns 8 q + 4 h .., q = w, w + W, ..., in wave
// order, each times its own row's factor.
template <typename T, int D, int W>
__device__ __forceinline__ void store_sum(T* dst, const float* parts, int stride, int n, int wave, int lane, const float (&factor)[W]) {
#pragma unroll
  for (int i = 0; i < D / 8 / W; ++i) {
    const int q = wave + W * i;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      if (w >= n) break;
      const float4 v = *(const float4*)&parts[w * stride + (q * 64 + lane) * 4];
      s.x = fmaf(v.x, factor[w], s.x); s.y = fmaf(v.y, factor[w], s.y);
      s.z = fmaf(v.z, factor[w], s.z); s.w = fmaf(v.w, factor[w], s.w);
    }
    store4(dst + 8 * q + 4 * (lane >> 5), s);
  }
}
// a single wave's sums straight from its registers, times factor (zeros where there is none)
template <typename T, int D>
__device__ __forceinline__ void store_own(T* dst, int lane, const f32x16 (&acc)[D / 32], bool any, float factor) {
#pragma unroll
  for (int q = 0; q < D / 8; ++q) {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    const f32x16& a = acc[q / 4];
    const int r = 4 * (q % 4);
    if (any) s = make_float4(a[r] * factor, a[r + 1] * factor, a[r + 2] * factor, a[r + 3] * factor);
    store4(dst + 8 * q + 4 * (lane >> 5), s);
  }
}

// The grid is 8 x blocks of a pair x groups of 8 pairs, so that the blocks of a (sample, head) pair run on one XCD and
// its keys and values (or queries) reach that XCD's L2 once.
__device__ __forceinline__ int pair_of_block() { return blockIdx.z * 8 + blockIdx.x; }

}  // namespace

// qkv row stride is 3*H; head hh of token t: q at t*3H + hh*D, k at +H, v at +2H.
template <typename T, int D, int W, int R>
__global__ __launch_bounds__(64 * W * R, 3) void attn_fwd_kernel(const T* __restrict__ qkv, T* __restrict__ ctx,
                                                       float* __restrict__ lse, Rows rows, int L, int nh, int pairs, int causal,
                                                       DropDesc drop) {
  __shared__ __attribute__((aligned(16))) float own_q_of[R][TR * (D + 4)], tiles_of[R][W][TR * (D + 4)];
  __shared__ float ms_of[R][W][TR], ls_of[R][W][TR];
  const int lane = threadIdx.x & 63, wave_of_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave_of_block / W, wave = wave_of_block % W, ql = lane & 31, h = lane >> 5;
  float(&own_q)[TR * (D + 4)] = own_q_of[group], (&tiles)[W][TR * (D + 4)] = tiles_of[group];
  float(&ms)[W][TR] = ms_of[group], (&ls)[W][TR] = ls_of[group];
  const int i0 = (blockIdx.y * R + group) * TR, bh = pair_of_block();
  if (bh >= pairs) return;
  const int b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  if ((int)(blockIdx.y * R) * TR >= sm.n) return;     // (a group of the block may yet have no rows: no tiles, no stores)
  const T* base = qkv + sm.first * ld3 + hh * D;
  const int qi = i0 + ql, qc = min(qi, sm.n - 1);
  const float scale = rsqrtf((float)D);
  const int kend = i0 >= sm.n ? 0 : causal ? min(sm.keys, i0 + TR) : sm.keys;
  float4 k[D / 8], v[D / 8];
  auto fetch = [&](int k0) {
    fetch_rows<T, D>(base + H, ld3, k0, sm.n - 1, ql, h, k);
    fetch_rows<T, D>(base + 2 * H, ld3, k0, sm.n - 1, ql, h, v);
  };
  if (wave * TR < kend) fetch(wave * TR);
  if (wave == 0) {
    float4 own[D / 8];
    fetch_rows<T, D>(base, ld3, i0, sm.n - 1, ql, h, own);
    stash<D>(own_q, ql, h, own);
  }
  __syncthreads();
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) clear(o[db]);
  float m = -INFINITY, l = 0.f;
  for (int k0 = wave * TR; k0 < kend; k0 += W * TR) {
    f32x16 s;
    scores<D>(k, own_q, ql, h, s);
    stash<D>(tiles[wave], ql, h, v);
    wave_sync();
    if (k0 + W * TR < kend) fetch(k0 + W * TR);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r >> 2) + 4 * h + (r & 3);
      s[r] = key >= sm.keys || (causal && key > qi) ? -INFINITY : s[r] * scale;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx);
    const float at = mnew == -INFINITY ? 0.f : mnew;  // no key of this wave's tiles so far is visible to the query
    const float alpha = expf(m - at);
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = expf(s[r] - at); rs += s[r]; }
    l = l * alpha + (rs + __shfl_xor(rs, 32, 64));    // the normaliser counts every probability
    m = mnew;
    if (drop.thr) {                                   // dropped ones leave the P V product; the scale waits for the end
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint4 w = attn_drop_words(drop, (int64_t)bh * L + qc, (L + 3) >> 2, k0 + 8 * g + 4 * h);
        if (w.x < drop.thr) s[4 * g] = 0.f;
        if (w.y < drop.thr) s[4 * g + 1] = 0.f;
        if (w.z < drop.thr) s[4 * g + 2] = 0.f;
        if (w.w < drop.thr) s[4 * g + 3] = 0.f;
      }
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    accumulate<D>(tiles[wave], ql, h, s, o);
    wave_sync();
  }
  T* out = ctx + (sm.first + qi) * H + hh * D;
  if (W == 1) {
    if (qi < sm.n) {
      store_own<T, D>(out, lane, o, true, drop.scale / l);
      if (h == 0) lse[(int64_t)bh * L + qi] = m + logf(l);
    }
    return;
  }
  // the waves' results brought to the largest maximum and added in order
  put_part<D>(tiles[wave], lane, o);
  if (h == 0) { ms[wave][ql] = m; ls[wave][ql] = l; }
  __syncthreads();
  const int n = min(W, (kend + TR - 1) / TR);
  float mall = ms[0][ql], lall = 0.f, factor[W];      // finite: key 0 is visible to every query
#pragma unroll
  for (int w = 1; w < W; ++w) mall = fmaxf(mall, ms[w][ql]);
#pragma unroll
  for (int w = 0; w < W; ++w) { factor[w] = expf(ms[w][ql] - mall); lall += ls[w][ql] * factor[w]; }
#pragma unroll
  for (int w = 0; w < W; ++w) factor[w] *= drop.scale / lall;
  if (qi < sm.n) {
    store_sum<T, D, W>(out, tiles[0], TR * (D + 4), n, wave, lane, factor);
    if (wave == 0 && h == 0) lse[(int64_t)bh * L + qi] = mall + logf(lall);
  }
}

// also writes delta_i = dO_i O_i for the dK/dV kernel, which runs after this one
template <typename T, int D, int W, int R>
__global__ __launch_bounds__(64 * W * R, 3) void attn_bwd_dq_kernel(const T* __restrict__ qkv, const T* __restrict__ ctx,
                                                          const T* __restrict__ dctx, const float* __restrict__ lse,
                                                          float* __restrict__ delta, T* __restrict__ dqkv, Rows rows, int L,
                                                          int nh, int pairs, int causal, DropDesc drop) {
  __shared__ __attribute__((aligned(16))) float own_q_of[R][TR * (D + 4)], own_g_of[R][TR * (D + 4)], tiles_of[R][W][TR * (D + 4)];
  const int lane = threadIdx.x & 63, wave_of_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave_of_block / W, wave = wave_of_block % W, ql = lane & 31, h = lane >> 5;
  float(&own_q)[TR * (D + 4)] = own_q_of[group], (&own_g)[TR * (D + 4)] = own_g_of[group];
  float(&tiles)[W][TR * (D + 4)] = tiles_of[group];
  const int i0 = (blockIdx.y * R + group) * TR, bh = pair_of_block();
  if (bh >= pairs) return;
  const int b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  if ((int)(blockIdx.y * R) * TR >= sm.n) return;     // (a group of the block may yet have no rows: no tiles, no stores)
  const T* base = qkv + sm.first * ld3 + hh * D;
  const int qi = i0 + ql, qc = min(qi, sm.n - 1);
  const float scale = rsqrtf((float)D);
  float4 k[D / 8], v[D / 8];
  const int kend = i0 >= sm.n ? 0 : causal ? min(sm.keys, i0 + TR) : sm.keys;
  auto fetch = [&](int k0) {
    fetch_rows<T, D>(base + H, ld3, k0, sm.n - 1, ql, h, k);
    fetch_rows<T, D>(base + 2 * H, ld3, k0, sm.n - 1, ql, h, v);
  };
  if (wave * TR < kend) fetch(wave * TR);
  const float lse_q = lse[(int64_t)bh * L + qc];
  float delta_q = 0.f;
  {
    float4 go[D / 8], of[D / 8];
    fetch_rows<T, D>(dctx + sm.first * H + hh * D, H, i0, sm.n - 1, ql, h, go);
    fetch_rows<T, D>(ctx + sm.first * H + hh * D, H, i0, sm.n - 1, ql, h, of);
#pragma unroll
    for (int g = 0; g < D / 8; ++g) {
      delta_q = fmaf(of[g].x, go[g].x, delta_q);
      delta_q = fmaf(of[g].y, go[g].y, delta_q);
      delta_q = fmaf(of[g].z, go[g].z, delta_q);
      delta_q = fmaf(of[g].w, go[g].w, delta_q);
    }
    delta_q += __shfl_xor(delta_q, 32, 64);
    if (wave == (W > 1 ? 1 : 0)) stash<D>(own_g, ql, h, go);
    if (wave == 0) {
      if (h == 0 && qi < sm.n) delta[(int64_t)bh * L + qi] = delta_q;
      fetch_rows<T, D>(base, ld3, i0, sm.n - 1, ql, h, of);
      stash<D>(own_q, ql, h, of);
    }
  }
  __syncthreads();
  f32x16 dq[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) clear(dq[db]);
  for (int k0 = wave * TR; k0 < kend; k0 += W * TR) {
    f32x16 s, dp;
    scores<D>(k, own_q, ql, h, s);
    scores<D>(v, own_g, ql, h, dp);
    stash<D>(tiles[wave], ql, h, k);
    wave_sync();
    if (k0 + W * TR < kend) fetch(k0 + W * TR);
    if (drop.thr) {                                   // d(P) of a dropped probability is zero, of a kept one scaled
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint4 w = attn_drop_words(drop, (int64_t)bh * L + qc, (L + 3) >> 2, k0 + 8 * g + 4 * h);
        dp[4 * g] = w.x < drop.thr ? 0.f : dp[4 * g] * drop.scale;
        dp[4 * g + 1] = w.y < drop.thr ? 0.f : dp[4 * g + 1] * drop.scale;
        dp[4 * g + 2] = w.z < drop.thr ? 0.f : dp[4 * g + 2] * drop.scale;
        dp[4 * g + 3] = w.w < drop.thr ? 0.f : dp[4 * g + 3] * drop.scale;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r >> 2) + 4 * h + (r & 3);
      const bool out = key >= sm.keys || (causal && key > qi);
      s[r] = out ? 0.f : expf(s[r] * scale - lse_q) * (dp[r] - delta_q);
    }
    accumulate<D>(tiles[wave], ql, h, s, dq);
    wave_sync();
  }
  T* out = dqkv + (sm.first + qi) * ld3 + hh * D;
  if (W == 1) {
    if (qi < sm.n) store_own<T, D>(out, lane, dq, true, scale);
    return;
  }
  put_part<D>(tiles[wave], lane, dq);
  __syncthreads();
  float factor[W];
#pragma unroll
  for (int w = 0; w < W; ++w) factor[w] = scale;
  if (qi < sm.n) store_sum<T, D, W>(out, tiles[0], TR * (D + 4), min(W, (kend + TR - 1) / TR), wave, lane, factor);
}

template <typename T, int D, int W, int R>
__global__ __launch_bounds__(64 * W * R, 2) void attn_bwd_dkv_kernel(const T* __restrict__ qkv, const T* __restrict__ dctx,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           T* __restrict__ dqkv, Rows rows, int L, int nh, int pairs, int causal,
                                                           DropDesc drop) {
  __shared__ __attribute__((aligned(16))) float own_k_of[R][TR * (D + 4)], own_v_of[R][TR * (D + 4)], tiles_of[R][W][TR * (D + 4)];
  __shared__ __attribute__((aligned(16))) float stats_of[R][W][2][TR];      // lse and delta of the tile's queries
  const int lane = threadIdx.x & 63, wave_of_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave_of_block / W, wave = wave_of_block % W, kl = lane & 31, h = lane >> 5;
  float(&own_k)[TR * (D + 4)] = own_k_of[group], (&own_v)[TR * (D + 4)] = own_v_of[group];
  float(&tiles)[W][TR * (D + 4)] = tiles_of[group], (&stats)[W][2][TR] = stats_of[group];
  const int j0 = (blockIdx.y * R + group) * TR, bh = pair_of_block();
  if (bh >= pairs) return;
  const int b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  if ((int)(blockIdx.y * R) * TR >= sm.n) return;     // (a group of the block may yet have no rows: no tiles, no stores)
  const T* base = qkv + sm.first * ld3 + hh * D;
  const T* gbase = dctx + sm.first * H + hh * D;
  const int ki = j0 + kl;
  const float scale = rsqrtf((float)D);
  float4 q[D / 8], go[D / 8];
  const int qstart = causal ? j0 : 0;                 // earlier queries never see these keys
  const int qend = j0 >= sm.keys ? 0 : sm.n;          // a block of padded keys only writes zeros
  const int first = qstart + wave * TR;
  if (first < qend) {
    fetch_rows<T, D>(base, ld3, first, sm.n - 1, kl, h, q);
    fetch_rows<T, D>(gbase, H, first, sm.n - 1, kl, h, go);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (wave == (W > 1 ? i : 0)) {
      float4 own[D / 8];
      fetch_rows<T, D>(base + (i + 1) * H, ld3, j0, sm.n - 1, kl, h, own);
      stash<D>(i ? own_v : own_k, kl, h, own);
    }
  __syncthreads();
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) { clear(dk[db]); clear(dv[db]); }
  for (int q0 = first; q0 < qend; q0 += W * TR) {
    const int next = q0 + W * TR;
    const float stat = (h ? delta : lse)[(int64_t)bh * L + min(q0 + kl, sm.n - 1)];
    f32x16 s, dp;
    scores<D>(q, own_k, kl, h, s);
    scores<D>(go, own_v, kl, h, dp);
    stash<D>(tiles[wave], kl, h, go);
    stats[wave][h][kl] = stat;
    wave_sync();
    if (next < qend) fetch_rows<T, D>(gbase, H, next, sm.n - 1, kl, h, go);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int qq = 8 * g + 4 * h;
      const float4 ls = *(const float4*)&stats[wave][0][qq], dl = *(const float4*)&stats[wave][1][qq];
      const float lss[4] = {ls.x, ls.y, ls.z, ls.w}, dls[4] = {dl.x, dl.y, dl.z, dl.w};
      // Dropout: a lane holds one key and four queries, a generator block four keys of one query.
      // The four lanes of a quad (four neighbouring keys) each make the block of one of the four
      // queries and pass its decisions round.
      bool keep[4] = {true, true, true, true};
      if (drop.thr) {
        const int qmine = min(q0 + qq + (lane & 3), sm.n - 1);
        quad_keep(attn_drop_words(drop, (int64_t)bh * L + qmine, (L + 3) >> 2, ki & ~3), drop.thr, lane, keep);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * g + e, at = q0 + qq + e;
        const bool out = at >= sm.n || (causal && ki > at);
        const float p = out ? 0.f : expf(s[r] * scale - lss[e]);
        const float d = keep[e] ? dp[r] * drop.scale : 0.f;
        s[r] = keep[e] ? p * drop.scale : 0.f;        // what multiplied V in the forward
        dp[r] = p * (d - dls[e]);
      }
    }
    accumulate<D>(tiles[wave], kl, h, s, dv);
    wave_sync();
    stash<D>(tiles[wave], kl, h, q);
    wave_sync();
    if (next < qend) fetch_rows<T, D>(base, ld3, next, sm.n - 1, kl, h, q);
    accumulate<D>(tiles[wave], kl, h, dp, dk);
    wave_sync();
  }
  const bool in = ki < sm.n;
  const int n = ki < sm.keys ? min(W, max(0, qend - qstart + TR - 1) / TR) : 0;   // padded keys: zeros, whatever the lane's column held
  T* out = dqkv + (sm.first + ki) * ld3 + hh * D;
  if (W == 1) {
    if (in) {
      store_own<T, D>(out + H, lane, dk, n > 0, scale);
      store_own<T, D>(out + 2 * H, lane, dv, n > 0, 1.f);
    }
    return;
  }
  float factor[W];
#pragma unroll
  for (int w = 0; w < W; ++w) factor[w] = scale;
  put_part<D>(tiles[wave], lane, dk);
  __syncthreads();
  if (in) store_sum<T, D, W>(out + H, tiles[0], TR * (D + 4), n, wave, lane, factor);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < W; ++w) factor[w] = 1.f;
  put_part<D>(tiles[wave], lane, dv);
  __syncthreads();
  if (in) store_sum<T, D, W>(out + 2 * H, tiles[0], TR * (D + 4), n, wave, lane, factor);
}

// Shape of a block, by the tiles of a sample and the blocks of 32 rows that the rows of the batch make (without padding
// that was left out of them; of halves on two streams the whole batch's).  Four waves make the chain of a sample's
// tiles a quarter as long; a wave without a tile only takes LDS and a place, and every further one's sums have to be added.
// So four where the blocks alone do not fill the chip: up to 512 of them for each tile of a sample, and up to 768 where of
// four waves' last turn two or three would idle; one where a sample has two tiles or three and the blocks do fill it.
// Iterations go by it too (12 layers in fp32, 16 x 141 padded to 88 on average: 9.47 / 9.10 / 8.98 ms with one / two / four).
// Two tiles' two waves twice in a block, 64 rows, where that is at most a block to a unit and 32 rows' blocks were more
// (a second block on a unit costs 50 %, a second group in its block 20), and with head size 32 from 1536 blocks of 32 rows
// on.  The same sums either way.
// Forward + backward in us with one / two / twice two / four waves, 12 heads of 64 in fp32 (heads of 32 alike), against
// two waves of a block on 64 rows that share tiles in LDS:
//   512 x 32 tokens 180 / 213 / - / 279 against 231     128 x 64 126 / 136 / 133 / 182 against 135
//   8 x 64 35 / 26.4 / 31.5 / 27 against 36             12-20 x 64 38-39 / 39-41 / 32-34 / 41-42 against 36-38
//   32 x 96 90 / 93 / 101 / 96 against 98               8 x 128 63 / 61 / 48 / 47 against 63
//   32 x 128 113 / 126 / 109 / 114 against 123          32 x 141 188 / 171 / - / 196 against 204
//   64 x 256 682 / 629 / 615 / 645 against 643          16 x 512 causal 575 / 459 / - / 433 against 606
//   head size 32: 64 x 64 43.9 / 43.2 / 40.9 / 54 against 42.3, 128 x 64 71.4 / 71.5 / 68.6 / 92 against 72.0
// (One tile of 12-192 pairs with head size 64 stays 3-4 % behind that, a microsecond for the three kernels.)
struct BlockShape { int waves, groups; };
static BlockShape block_shape(int L, int nh, int d, int64_t rule_rows) {
  const int tiles = (L + TR - 1) / TR;
  const int64_t blocks = (rule_rows + L - 1) / L * nh * tiles;
  if (tiles == 2 && ((blocks > 256 && blocks <= 512) || (d == 32 && blocks >= 1536))) return {2, 2};
  if (tiles == 1 || (tiles <= 3 && blocks >= 768 * (tiles - 1))) return {1, 1};
  const bool idle = tiles == 3 || tiles == 5 || tiles == 6;   // (behind more turns the last weighs little)
  return {tiles == 2 || blocks >= (idle ? 768 : 512 * (int64_t)tiles) ? 2 : 4, 1};
}

template <typename T, int D, int W, int R>
static void fwd_w(const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int causal,
                  const DropDesc& drop, hipStream_t st) {
  const int pairs = B * nh;
  hipLaunchKernelGGL((attn_fwd_kernel<T, D, W, R>), dim3(8, (L + TR * R - 1) / (TR * R), (pairs + 7) / 8), dim3(64 * W * R), 0,
                     st, (const T*)qkv, (T*)ctx, lse, rows, L, nh, pairs, causal, drop);
}
template <typename T, int D>
static void fwd_t(const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int64_t rule_rows, int L, int nh, int causal,
                  const DropDesc& drop, hipStream_t st) {
  const BlockShape shape = block_shape(L, nh, D, rule_rows);
  if (shape.groups == 2) fwd_w<T, D, 2, 2>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else if (shape.waves == 1) fwd_w<T, D, 1, 1>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else if (shape.waves == 2) fwd_w<T, D, 2, 1>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else fwd_w<T, D, 4, 1>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
}
template <typename T, int D, int W, int R>
static void bwd_w(const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta, void* dqkv,
                  const Rows& rows, int B, int L, int nh, int causal, const DropDesc& drop, hipStream_t st, hipEvent_t done) {
  const int pairs = B * nh;
  const dim3 grid(8, (L + TR * R - 1) / (TR * R), (pairs + 7) / 8);
  hipLaunchKernelGGL((attn_bwd_dq_kernel<T, D, W, R>), grid, dim3(64 * W * R), 0, st, (const T*)qkv, (const T*)ctx,
                     (const T*)dctx, lse, delta, (T*)dqkv, rows, L, nh, pairs, causal, drop);
  LAUNCH_MARKED_((attn_bwd_dkv_kernel<T, D, W, R>), grid, dim3(64 * W * R), st, done, (const T*)qkv, (const T*)dctx, lse, delta,
                 (T*)dqkv, rows, L, nh, pairs, causal, drop);
}
template <typename T, int D>
static void bwd_t(const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta, void* dqkv, const Rows& rows,
                  int B, int64_t rule_rows, int L, int nh, int causal, const DropDesc& drop, hipStream_t st, hipEvent_t done) {
  const BlockShape shape = block_shape(L, nh, D, rule_rows);
  if (shape.groups == 2) bwd_w<T, D, 2, 2>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st, done);
  else if (shape.waves == 1) bwd_w<T, D, 1, 1>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st, done);
  else if (shape.waves == 2) bwd_w<T, D, 2, 1>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st, done);
  else bwd_w<T, D, 4, 1>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st, done);
}

void attention_fwd(int dtype, const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int d,
                   int causal, const DropDesc& drop, hipStream_t st, int64_t rule_rows) {
  if (B * L <= 0) return;
  if (rule_rows <= 0) rule_rows = (int64_t)B * L;
  if (dtype == BF16 && d == 64) attention_fwd_mfma(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else if (dtype == BF16) fwd_t<bf16_t, 32>(qkv, ctx, lse, rows, B, rule_rows, L, nh, causal, drop, st);
  else if (d == 32) fwd_t<float, 32>(qkv, ctx, lse, rows, B, rule_rows, L, nh, causal, drop, st);
  else fwd_t<float, 64>(qkv, ctx, lse, rows, B, rule_rows, L, nh, causal, drop, st);
}

void attention_bwd(int dtype, const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta,
                   void* dqkv, const Rows& rows, int B, int L, int nh, int d, int causal, const DropDesc& drop,
                   hipStream_t st, hipEvent_t done, int64_t rule_rows) {
  if (B * L <= 0) return;
  if (rule_rows <= 0) rule_rows = (int64_t)B * L;
  if (dtype == BF16 && d == 64) attention_bwd_mfma(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st, done);
  else if (dtype == BF16) bwd_t<bf16_t, 32>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, rule_rows, L, nh, causal, drop, st, done);
  else if (d == 32) bwd_t<float, 32>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, rule_rows, L, nh, causal, drop, st, done);
  else bwd_t<float, 64>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, rule_rows, L, nh, causal, drop, st, done);
}

}  // namespace mk
