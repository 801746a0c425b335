// Fused attention, forward and backward, in fp32 arithmetic on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32), without materialising the L x L matrices.
//
// Head sizes 32 and 64; the fp32 configuration, and bf16 with head size 32 (bf16 with head size 64
// runs on the bf16 kernels of attention_mfma.hip).  One wave owns 32 query rows (forward, dQ) or 32
// key rows (dK/dV); a block's two waves share tiles of 32 opposite rows in LDS.  An MFMA of 32 x 32
// x 2 takes 64 clocks, so the matrix pipe is the limit and everything else hides behind it.
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
// (One wave per row with a shuffle per key, as before: 222, 407 and 391 us per layer for forward, dQ
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
                        const Rows& rows, int B, int L, int nh, int causal, const DropDesc& drop, hipStream_t st);

namespace {

constexpr int TR = 32;                 // rows of a streamed tile
constexpr int BLOCK_ROWS = 64;         // 2 waves x 32 rows

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

// Tile of TR rows x D columns: global -> registers -> LDS [row][D + 4].  128 threads, 16 bytes each.
template <typename T, int D>
struct RowTile {
  static constexpr int LD = D + 4;
  static constexpr int NCH = TR * D / 4 / 128;
  float4 v[NCH];
  __device__ __forceinline__ void fetch(const T* src, int64_t ld, int r0, int last, int tid) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 128, r = min(r0 + c / (D / 4), last);
      v[i] = load4(src + (int64_t)r * ld + (c % (D / 4)) * 4);
    }
  }
  __device__ __forceinline__ void stash(float* tile, int tid) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * 128;
      *(float4*)&tile[(c / (D / 4)) * LD + (c % (D / 4)) * 4] = v[i];
    }
  }
};

// the wave's own row as B operand: element j of group g is column 8g + 4h + j
template <typename T, int D>
__device__ __forceinline__ void own_row(const T* p, int h, float4 (&f)[D / 8]) {
#pragma unroll
  for (int g = 0; g < D / 8; ++g) f[g] = load4(p + 8 * g + 4 * h);
}
__device__ __forceinline__ void clear(f32x16& v) {
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = 0.f;
}
// s = tile rows (A) x own rows (B) over the D columns
template <int D>
__device__ __forceinline__ void scores(const float* tile, int l32, int h, const float4 (&own)[D / 8], f32x16& s) {
  clear(s);
#pragma unroll
  for (int g = 0; g < D / 8; ++g) {
    const float4 a = *(const float4*)&tile[l32 * (D + 4) + 8 * g + 4 * h];
    s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, own[g].x, s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, own[g].y, s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, own[g].z, s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, own[g].w, s, 0, 0, 0);
  }
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
template <typename T, int D>
__device__ __forceinline__ void store_own(T* dst, const f32x16 (&acc)[D / 32], int h, float mul) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      store4(dst + 32 * db + 8 * g + 4 * h,
             make_float4(acc[db][4 * g] * mul, acc[db][4 * g + 1] * mul, acc[db][4 * g + 2] * mul, acc[db][4 * g + 3] * mul));
}

}  // namespace

// qkv row stride is 3*H; head hh of token t: q at t*3H + hh*D, k at +H, v at +2H.
template <typename T, int D>
__global__ __launch_bounds__(128) void attn_fwd_kernel(const T* __restrict__ qkv, T* __restrict__ ctx,
                                                       float* __restrict__ lse, Rows rows, int L, int nh, int causal,
                                                       DropDesc drop) {
  __shared__ __attribute__((aligned(16))) float Ks[TR * (D + 4)], Vs[TR * (D + 4)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ql = lane & 31, h = lane >> 5;
  const int bh = blockIdx.y, b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  const int i0 = blockIdx.x * BLOCK_ROWS;
  if (i0 >= sm.n) return;
  const T* base = qkv + sm.first * ld3 + hh * D;
  const int qi = i0 + wave * 32 + ql, qc = min(qi, sm.n - 1);
  const float scale = rsqrtf((float)D);
  float4 q[D / 8];
  own_row<T, D>(base + (int64_t)qc * ld3, h, q);
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) clear(o[db]);
  float m = -INFINITY, l = 0.f;
  const int kend = causal ? min(sm.keys, i0 + BLOCK_ROWS) : sm.keys;
  RowTile<T, D> tk, tv;
  tk.fetch(base + H, ld3, 0, sm.n - 1, tid);
  tv.fetch(base + 2 * H, ld3, 0, sm.n - 1, tid);
  for (int k0 = 0; k0 < kend; k0 += TR) {
    __syncthreads();
    tk.stash(Ks, tid);
    tv.stash(Vs, tid);
    __syncthreads();
    if (k0 + TR < kend) {
      tk.fetch(base + H, ld3, k0 + TR, sm.n - 1, tid);
      tv.fetch(base + 2 * H, ld3, k0 + TR, sm.n - 1, tid);
    }
    f32x16 s;
    scores<D>(Ks, ql, h, q, s);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r >> 2) + 4 * h + (r & 3);
      s[r] = key >= sm.keys || (causal && key > qi) ? -INFINITY : s[r] * scale;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx);                  // finite: key 0 is visible to every query
    const float alpha = expf(m - mnew);
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = expf(s[r] - mnew); rs += s[r]; }
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
    accumulate<D>(Vs, ql, h, s, o);
  }
  if (qi < sm.n) {
    store_own<T, D>(ctx + (sm.first + qi) * H + hh * D, o, h, drop.scale / l);
    if (h == 0) lse[(int64_t)bh * L + qi] = m + logf(l);
  }
}

// also writes delta_i = dO_i O_i for the dK/dV kernel, which runs after this one
template <typename T, int D>
__global__ __launch_bounds__(128) void attn_bwd_dq_kernel(const T* __restrict__ qkv, const T* __restrict__ ctx,
                                                          const T* __restrict__ dctx, const float* __restrict__ lse,
                                                          float* __restrict__ delta, T* __restrict__ dqkv, Rows rows, int L,
                                                          int nh, int causal, DropDesc drop) {
  __shared__ __attribute__((aligned(16))) float Ks[TR * (D + 4)], Vs[TR * (D + 4)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ql = lane & 31, h = lane >> 5;
  const int bh = blockIdx.y, b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  const int i0 = blockIdx.x * BLOCK_ROWS;
  if (i0 >= sm.n) return;
  const T* base = qkv + sm.first * ld3 + hh * D;
  const int qi = i0 + wave * 32 + ql, qc = min(qi, sm.n - 1);
  const float scale = rsqrtf((float)D);
  float4 q[D / 8], go[D / 8], of[D / 8];
  own_row<T, D>(base + (int64_t)qc * ld3, h, q);
  own_row<T, D>(dctx + (sm.first + qc) * H + hh * D, h, go);
  own_row<T, D>(ctx + (sm.first + qc) * H + hh * D, h, of);
  float delta_q = 0.f;
#pragma unroll
  for (int g = 0; g < D / 8; ++g) {
    delta_q = fmaf(of[g].x, go[g].x, delta_q);
    delta_q = fmaf(of[g].y, go[g].y, delta_q);
    delta_q = fmaf(of[g].z, go[g].z, delta_q);
    delta_q = fmaf(of[g].w, go[g].w, delta_q);
  }
  delta_q += __shfl_xor(delta_q, 32, 64);
  if (h == 0 && qi < sm.n) delta[(int64_t)bh * L + qi] = delta_q;
  const float lse_q = lse[(int64_t)bh * L + qc];
  f32x16 dq[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) clear(dq[db]);
  const int kend = causal ? min(sm.keys, i0 + BLOCK_ROWS) : sm.keys;
  RowTile<T, D> tk, tv;
  tk.fetch(base + H, ld3, 0, sm.n - 1, tid);
  tv.fetch(base + 2 * H, ld3, 0, sm.n - 1, tid);
  for (int k0 = 0; k0 < kend; k0 += TR) {
    __syncthreads();
    tk.stash(Ks, tid);
    tv.stash(Vs, tid);
    __syncthreads();
    if (k0 + TR < kend) {
      tk.fetch(base + H, ld3, k0 + TR, sm.n - 1, tid);
      tv.fetch(base + 2 * H, ld3, k0 + TR, sm.n - 1, tid);
    }
    f32x16 s, dp;
    scores<D>(Ks, ql, h, q, s);
    scores<D>(Vs, ql, h, go, dp);
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
    accumulate<D>(Ks, ql, h, s, dq);
  }
  if (qi < sm.n) store_own<T, D>(dqkv + (sm.first + qi) * ld3 + hh * D, dq, h, scale);
}

template <typename T, int D>
__global__ __launch_bounds__(128) void attn_bwd_dkv_kernel(const T* __restrict__ qkv, const T* __restrict__ dctx,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           T* __restrict__ dqkv, Rows rows, int L, int nh, int causal,
                                                           DropDesc drop) {
  __shared__ __attribute__((aligned(16))) float Qs[TR * (D + 4)], Gs[TR * (D + 4)], lse_s[TR], delta_s[TR];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kl = lane & 31, h = lane >> 5;
  const int bh = blockIdx.y, b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  const int j0 = blockIdx.x * BLOCK_ROWS;
  if (j0 >= sm.n) return;
  const T* base = qkv + sm.first * ld3 + hh * D;
  const T* gbase = dctx + sm.first * H + hh * D;
  const int ki = j0 + wave * 32 + kl, kc = min(ki, sm.n - 1);
  const float scale = rsqrtf((float)D);
  float4 k[D / 8], v[D / 8];
  own_row<T, D>(base + (int64_t)kc * ld3 + H, h, k);
  own_row<T, D>(base + (int64_t)kc * ld3 + 2 * H, h, v);
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) { clear(dk[db]); clear(dv[db]); }
  const int qstart = causal ? j0 : 0;                 // earlier queries never see these keys
  const int qend = j0 >= sm.keys ? 0 : sm.n;          // a block of padded keys only writes zeros
  RowTile<T, D> tq, tg;
  float pre_lse = 0.f, pre_delta = 0.f;
  auto fetch = [&](int q0) {
    tq.fetch(base, ld3, q0, sm.n - 1, tid);
    tg.fetch(gbase, H, q0, sm.n - 1, tid);
    if (tid < TR) {
      const int q = min(q0 + tid, sm.n - 1);
      pre_lse = lse[(int64_t)bh * L + q];
      pre_delta = delta[(int64_t)bh * L + q];
    }
  };
  if (qstart < qend) fetch(qstart);
  for (int q0 = qstart; q0 < qend; q0 += TR) {
    __syncthreads();
    tq.stash(Qs, tid);
    tg.stash(Gs, tid);
    if (tid < TR) { lse_s[tid] = pre_lse; delta_s[tid] = pre_delta; }
    __syncthreads();
    if (q0 + TR < qend) fetch(q0 + TR);
    f32x16 s, dp;
    scores<D>(Qs, kl, h, k, s);
    scores<D>(Gs, kl, h, v, dp);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int qq = 8 * g + 4 * h;
      const float4 ls = *(const float4*)&lse_s[qq], dl = *(const float4*)&delta_s[qq];
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
        const int r = 4 * g + e, q = q0 + qq + e;
        const bool out = q >= sm.n || (causal && ki > q);
        const float p = out ? 0.f : expf(s[r] * scale - lss[e]);
        const float d = keep[e] ? dp[r] * drop.scale : 0.f;
        s[r] = keep[e] ? p * drop.scale : 0.f;        // what multiplied V in the forward
        dp[r] = p * (d - dls[e]);
      }
    }
    accumulate<D>(Gs, kl, h, s, dv);
    accumulate<D>(Qs, kl, h, dp, dk);
  }
  if (ki < sm.n) {
    if (ki >= sm.keys) {                              // whatever the lane's column held
#pragma unroll
      for (int db = 0; db < D / 32; ++db) { clear(dk[db]); clear(dv[db]); }
    }
    T* out = dqkv + (sm.first + ki) * ld3 + hh * D;
    store_own<T, D>(out + H, dk, h, scale);
    store_own<T, D>(out + 2 * H, dv, h, 1.f);
  }
}

template <typename T, int D>
static void fwd_t(const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int causal,
                  const DropDesc& drop, hipStream_t st) {
  dim3 grid((L + BLOCK_ROWS - 1) / BLOCK_ROWS, B * nh);
  hipLaunchKernelGGL((attn_fwd_kernel<T, D>), grid, dim3(128), 0, st, (const T*)qkv, (T*)ctx, lse, rows, L, nh, causal, drop);
}
template <typename T, int D>
static void bwd_t(const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta, void* dqkv,
                  const Rows& rows, int B, int L, int nh, int causal, const DropDesc& drop, hipStream_t st) {
  dim3 grid((L + BLOCK_ROWS - 1) / BLOCK_ROWS, B * nh);
  hipLaunchKernelGGL((attn_bwd_dq_kernel<T, D>), grid, dim3(128), 0, st, (const T*)qkv, (const T*)ctx, (const T*)dctx, lse,
                     delta, (T*)dqkv, rows, L, nh, causal, drop);
  hipLaunchKernelGGL((attn_bwd_dkv_kernel<T, D>), grid, dim3(128), 0, st, (const T*)qkv, (const T*)dctx, lse, delta,
                     (T*)dqkv, rows, L, nh, causal, drop);
}

void attention_fwd(int dtype, const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int d,
                   int causal, const DropDesc& drop, hipStream_t st) {
  if (B * L <= 0) return;
  if (dtype == BF16 && d == 64) attention_fwd_mfma(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else if (dtype == BF16) fwd_t<bf16_t, 32>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else if (d == 32) fwd_t<float, 32>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
  else fwd_t<float, 64>(qkv, ctx, lse, rows, B, L, nh, causal, drop, st);
}

void attention_bwd(int dtype, const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta,
                   void* dqkv, const Rows& rows, int B, int L, int nh, int d, int causal, const DropDesc& drop,
                   hipStream_t st) {
  if (B * L <= 0) return;
  if (dtype == BF16 && d == 64) attention_bwd_mfma(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st);
  else if (dtype == BF16) bwd_t<bf16_t, 32>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st);
  else if (d == 32) bwd_t<float, 32>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st);
  else bwd_t<float, 64>(qkv, ctx, dctx, lse, delta, dqkv, rows, B, L, nh, causal, drop, st);
}

}  // namespace mk
