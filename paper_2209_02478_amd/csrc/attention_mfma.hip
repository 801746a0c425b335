// Fused attention for bf16, head size 64, on the MFMA units (v_mfma_f32_32x32x16_bf16).
//
// The loops are bound by the vector instructions per score (exponential, FMA, maximum, sum, rounding)
// beside the MFMAs: mask instructions run only in tiles that cross the mask's edge, sums and maxima
// cross the wave's halves by v_permlane32_swap, and accumulators are scaled only when a maximum moved
// (16 causal samples of 1024 tokens, 16 heads: forward 89 -> 77 us, backward 245 -> 210).
//
// All three kernels compute score tiles transposed, S^T = K Q^T, so that a lane's 32x32
// accumulator registers belong to ONE query (forward, dQ) or ONE key (dK/dV): the softmax
// statistics of a row are then reductions over a lane's own registers plus one exchange with
// lane^32, and a lane's probabilities, converted to bf16, are directly the B operand of the
// next product (P V, dS K, P^T dO, dS^T Q) without passing through LDS.  The operand that
// multiplies them is needed contiguous along the reduction index, which is the tile's row: the
// transposing LDS reads of gfx950 (ds_read_b64_tr_b16) hand it out from the tile as it lies, so a
// tile is in LDS once and comes there straight from memory (global_load_lds), into one of two
// buffers while the other is multiplied, with one barrier per tile (backward of 32 x 512 x 12 heads
// 151 -> 135 us against tiles carried through registers and stored twice, as they lie and transposed).
//
// MFMA 32x32x16 register layout used below (A: 32 x 16, B: 16 x 32, D: 32 x 32):
//   A, B: lane holds row/column lane%32 and reduction indices 8*(lane/32) .. +7
//   D:    lane holds column lane%32; register r holds row 8*(r/4) + 4*(lane/32) + r%4
// Feeding D registers 8c..8c+7 as a B operand therefore assigns reduction slot (lane/32, e) the
// row 16c + 8*(e/4) + 4*(lane/32) + e%4, and the A operand is gathered with the same map: two
// runs of 4 consecutive indices.
//
// No atomics: dQ comes from a kernel that owns query rows, dK/dV from one that owns key rows.
#include "device_common.h"
#include "kernels.h"
#include "philox.h"

namespace mk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int D = 64;          // head size
constexpr int TK = 64;         // rows of a streamed tile
constexpr int TILE = TK * D;   // elements of a tile in LDS: rows of 128 bytes, no padding (a direct load fills 1 KB in lane order)
constexpr int ROWS_PER_BLOCK = 128;

constexpr float LOG2E = 1.44269504088896340736f;
// 2^x on the transcendental unit (v_exp_f32), no range fix-ups: arguments here are <= ~0 or the
// result is multiplied by zero-gradient terms; -inf gives 0
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8 ld_frag(const bf16_t* p) { return *(const bf16x8*)p; }

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return pack_bf16x2(a, b);
}
// registers 8c .. 8c+7 of an accumulator as a bf16 operand
__device__ __forceinline__ bf16x8 regs_to_frag(const f32x16& v, int c) {
  uint4 u;
  u.x = pack2(v[8 * c + 0], v[8 * c + 1]);
  u.y = pack2(v[8 * c + 2], v[8 * c + 3]);
  u.z = pack2(v[8 * c + 4], v[8 * c + 5]);
  u.w = pack2(v[8 * c + 6], v[8 * c + 7]);
  return __builtin_bit_cast(bf16x8, u);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// 16-byte chunk c of a tile's row r lies at position c ^ swizzle(r).  A plain read (16 rows, one
// chunk) and a transposing read (4 rows, 4 chunks in 32 lanes) then both meet all 64 banks once:
// rows two apart differ in bit 2, rows four apart in the low bits.
__device__ __forceinline__ int swizzle(int r) { return ((r & 2) << 1) | ((r >> 2) & 3); }

// A wave's fragments of a tile, as element offsets computed once.
struct FragAt {
  int plain[4];      // row (lane % 32) of a 32-row block, head columns 16 kk + 8 h .. +7
  int turned[2];     // head column (lane % 32) of 32-column block db, rows 4 h + {0..3}; rows + 8: chunk position ^ 2
  __device__ __forceinline__ void init(int lane) {
    const int h = lane >> 5, r = lane & 31, q = (lane & 15) >> 2;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) plain[kk] = r * D + (((2 * kk + h) ^ swizzle(r)) << 3);
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
      turned[db] = (4 * h + q) * D + ((chunk ^ swizzle(4 * h + q)) << 3) + 4 * (lane & 1);
    }
  }
  // row 32 * block + lane % 32 of the tile, columns 16 kk + 8 h .. +7
  __device__ __forceinline__ bf16x8 row(const bf16_t* tile, int block, int kk) const {
    return ld_frag(tile + block * 32 * D + plain[kk]);
  }
  // head column 32 db + lane % 32, tile rows base + 4h + {0..3}, base + 8 + 4h + {0..3} (base % 16 == 0).
  // Within 16 lanes of a transposing read, lane i gets column i of the 4 x 16 block whose row k lies
  // at the four lanes 4k ..; 8 rows on, bit 1 of swizzle() flips.
  __device__ __forceinline__ bf16x8 column(const bf16_t* tile, int db, int base) const {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tile + base * D + turned[db]));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tile + (base + 8) * D + (turned[db] ^ 16)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// One wave-level direct load: lane i's 16 bytes at g land at lds + 16 * i.  Inline assembly, so the
// compiler does not track it: landed() waits by hand.  The s_nop is the wait state between a write of M0
// and the load that reads it, which the hardware leaves to the program.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // m0 is a reserved register: named as clobbered on purpose
__device__ __forceinline__ void direct_load(const bf16_t* g, uint32_t lds_byte_address) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(g), "s"(lds_byte_address) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void*)p);
}
// Every wave's direct loads so far are in LDS, and every wave is done reading what it read before.
__device__ __forceinline__ void landed() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// The block's share of bringing rows r0 .. r0 + 63 (row stride ld, rows past `last` are read as
// `last`) of one operand into a tile: each of the four waves loads 16 rows in two pieces.
struct TileLoad {
  int row, chunk;
  __device__ __forceinline__ void init(int wave, int lane) {
    row = 16 * wave + (lane >> 3);
    chunk = ((lane & 7) ^ swizzle(row)) << 3;         // swizzle(row + 8) = swizzle(row) ^ 2
  }
  __device__ __forceinline__ void issue(const bf16_t* src, int64_t ld, int r0, int last, int wave, uint32_t tile) const {
    direct_load(src + (int64_t)min(r0 + row, last) * ld + chunk, tile + (uint32_t)wave * 2048u);
    direct_load(src + (int64_t)min(r0 + row + 8, last) * ld + (chunk ^ 16), tile + (uint32_t)wave * 2048u + 1024u);
  }
};

// the value of lane ^ 32, without a trip through LDS
__device__ __forceinline__ float other_half(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // {low half twice, high half twice}
  return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

__device__ __forceinline__ void zero(f32x16& v) {
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = 0.f;
}

// store a transposed accumulator pair (rows = head columns, lane column = token) as bf16
__device__ __forceinline__ void store_rows(bf16_t* dst, const f32x16 (&acc)[2], int h, float mul) {
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint2 o;
      o.x = pack2(acc[db][4 * g] * mul, acc[db][4 * g + 1] * mul);
      o.y = pack2(acc[db][4 * g + 2] * mul, acc[db][4 * g + 3] * mul);
      *(uint2*)(dst + 32 * db + 8 * g + 4 * h) = o;
    }
}

// Which row block (of nb) of which sample and head a block works on; false: none.  Consecutive block
// ids go to the 8 XCDs in turn, so an id's low three bits pick the pair of sample and head: all row
// blocks of a pair run on one XCD, whose L2 then fetches the pair's rows once, and the heads of a
// sample, all equally long, spread over the XCDs.  (With the row block as the fastest index a causal
// batch of 8 row blocks gave one XCD every longest block and another every shortest.)
// longest_last: the row block with most work is the last one; it starts first.  16 causal samples of
// 1024 tokens, 16 heads: forward 111 -> 91 us, backward 337 -> 283; without a mask level or 4 % ahead.
__device__ __forceinline__ bool row_block(int nb, int pairs, bool longest_last, int& rb, int& bh) {
  const int slot = blockIdx.x >> 3, group = slot / nb, i = slot - group * nb;
  rb = longest_last ? nb - 1 - i : i;
  bh = group * 8 + (blockIdx.x & 7);
  return bh < pairs;
}

}  // namespace

// ------------------------------------------------------------------ forward
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256, 2) void fa_fwd_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx,
                                                     float* __restrict__ lse, Rows rows,
                                                     int L, int nh, int pairs, DropDesc drop) {
  __shared__ __attribute__((aligned(1024))) bf16_t tiles[2][2][TILE];   // [buffer][K, V][key][d]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), ql = lane & 31, h = lane >> 5;
  int rb, bh;
  if (!row_block((L + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK, pairs, true, rb, bh)) return;
  const int b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  if (rb * ROWS_PER_BLOCK >= sm.n) return;
  const bf16_t* base = qkv + sm.first * ld3 + hh * D;
  const int w0 = rb * ROWS_PER_BLOCK + wave * 32, qi = w0 + ql;
  const int qc = min(qi, sm.n - 1);
  const float scale = 0.125f, c2 = scale * LOG2E;    // exp(scale * s - x) == exp2(c2 * s - LOG2E * x)

  bf16x8 qf[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) qf[kk] = ld_frag(base + (int64_t)qc * ld3 + 16 * kk + 8 * h);
  f32x16 o[2];
  zero(o[0]); zero(o[1]);
  float m = -INFINITY, l = 0.f;                       // running maximum of the raw (unscaled) scores, sum of exps
  const int Lk = sm.keys;                             // keys from Lk on are padding (1 <= Lk)
  const int kend = CAUSAL ? min(Lk, (rb + 1) * ROWS_PER_BLOCK) : Lk;

  FragAt at;
  at.init(lane);
  TileLoad load;
  load.init(wave, lane);
  const uint32_t lds = lds_address(&tiles[0][0][0]);
  auto fetch = [&](int k0, int buf) {
    load.issue(base + H, ld3, k0, sm.n - 1, wave, lds + (uint32_t)buf * (4u * TILE));
    load.issue(base + 2 * H, ld3, k0, sm.n - 1, wave, lds + (uint32_t)buf * (4u * TILE) + 2u * TILE);
  };
  fetch(0, 0);
  for (int k0 = 0, buf = 0; k0 < kend; k0 += TK, buf ^= 1) {
    landed();
    if (k0 + TK < kend) fetch(k0 + TK, buf ^ 1);
    const bf16_t *Ks = tiles[buf][0], *Vs = tiles[buf][1];
    if (w0 >= sm.n || (CAUSAL && k0 > w0 + 31)) continue;   // none of this wave's queries sees the tile
    const bool edge = k0 + TK > Lk || (CAUSAL && k0 + TK - 1 > w0);
    f32x16 s[2];
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      zero(s[kb]);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.row(Ks, kb, kk), qf[kk], s[kb], 0, 0, 0);
      if (edge) {                                     // only tiles that touch the mask pay for it
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
          if (key >= Lk || (CAUSAL && key > qi)) s[kb][r] = -INFINITY;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
    }
    mx = fmaxf(mx, other_half(mx));
    const float mnew = fmaxf(m, mx);                  // finite: key 0 is visible to every query
    float alpha = 1.f;
    if (__any(mx > m)) {                              // else alpha is 1 in every lane: nothing to scale
      alpha = fast_exp2((m - mnew) * c2);
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m = mnew;
    }
    const float off = -mnew * c2;
    float rs = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(fmaf(s[kb][r], c2, off));
        s[kb][r] = p;
        rs += p;
      }
    rs += other_half(rs);
    l = fmaf(l, alpha, rs);                           // the normaliser counts every probability
    if (DROP) {                                       // dropped ones leave the P V product; the scale waits for the end
      const int64_t row = (int64_t)bh * L + qc;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint4 w = attn_drop_words(drop, row, (L + 3) >> 2, k0 + 32 * kb + 8 * g + 4 * h);
          if (w.x < drop.thr) s[kb][4 * g] = 0.f;
          if (w.y < drop.thr) s[kb][4 * g + 1] = 0.f;
          if (w.z < drop.thr) s[kb][4 * g + 2] = 0.f;
          if (w.w < drop.thr) s[kb][4 * g + 3] = 0.f;
        }
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 pf = regs_to_frag(s[kb], c);
#pragma unroll
        for (int db = 0; db < 2; ++db)
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.column(Vs, db, 32 * kb + 16 * c), pf, o[db], 0, 0, 0);
      }
  }
  if (qi < sm.n) {
    store_rows(ctx + (sm.first + qi) * H + hh * D, o, h, (DROP ? drop.scale : 1.f) / l);
    if (h == 0) lse[(int64_t)bh * L + qi] = m * scale + __logf(l);
  }
}

// ------------------------------------------------------------------ dQ
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256, 2) void fa_bwd_dq_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx,
                                                        const bf16_t* __restrict__ dctx,
                                                        const float* __restrict__ lse, float* __restrict__ delta,
                                                        bf16_t* __restrict__ dqkv, Rows rows, int L,
                                                        int nh, int pairs, DropDesc drop) {
  __shared__ __attribute__((aligned(1024))) bf16_t tiles[2][2][TILE];   // [buffer][K, V][key][d]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), ql = lane & 31, h = lane >> 5;
  int rb, bh;
  if (!row_block((L + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK, pairs, true, rb, bh)) return;
  const int b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  if (rb * ROWS_PER_BLOCK >= sm.n) return;
  const bf16_t* base = qkv + sm.first * ld3 + hh * D;
  const int w0 = rb * ROWS_PER_BLOCK + wave * 32, qi = w0 + ql;
  const int qc = min(qi, sm.n - 1);
  const float scale = 0.125f;

  // delta = sum over the head's columns of dO * O for this query: each half of the wave holds 32
  // of the 64 columns.  Written out for the dK/dV kernel, which runs after this one.
  bf16x8 qf[4], gf[4];
  float delta_q = 0.f;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    qf[kk] = ld_frag(base + (int64_t)qc * ld3 + 16 * kk + 8 * h);
    gf[kk] = ld_frag(dctx + (sm.first + qc) * H + hh * D + 16 * kk + 8 * h);
    const bf16x8 of = ld_frag(ctx + (sm.first + qc) * H + hh * D + 16 * kk + 8 * h);
#pragma unroll
    for (int e = 0; e < 8; ++e) delta_q = fmaf((float)of[e], (float)gf[kk][e], delta_q);
  }
  delta_q += other_half(delta_q);
  if (h == 0 && qi < sm.n) delta[(int64_t)bh * L + qi] = delta_q;
  const float c2 = scale * LOG2E;
  const float nlse_q = -LOG2E * lse[(int64_t)bh * L + qc];
  f32x16 dq[2];
  zero(dq[0]); zero(dq[1]);
  const int Lk = sm.keys;                             // keys from Lk on are padding (1 <= Lk)
  const int kend = CAUSAL ? min(Lk, (rb + 1) * ROWS_PER_BLOCK) : Lk;

  FragAt at;
  at.init(lane);
  TileLoad load;
  load.init(wave, lane);
  const uint32_t lds = lds_address(&tiles[0][0][0]);
  auto fetch = [&](int k0, int buf) {
    load.issue(base + H, ld3, k0, sm.n - 1, wave, lds + (uint32_t)buf * (4u * TILE));
    load.issue(base + 2 * H, ld3, k0, sm.n - 1, wave, lds + (uint32_t)buf * (4u * TILE) + 2u * TILE);
  };
  fetch(0, 0);
  for (int k0 = 0, buf = 0; k0 < kend; k0 += TK, buf ^= 1) {
    landed();
    if (k0 + TK < kend) fetch(k0 + TK, buf ^ 1);
    const bf16_t *Ks = tiles[buf][0], *Vs = tiles[buf][1];
    if (w0 >= sm.n || (CAUSAL && k0 > w0 + 31)) continue;   // none of this wave's queries sees the tile
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      f32x16 s, dp;
      zero(s); zero(dp);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.row(Ks, kb, kk), qf[kk], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.row(Vs, kb, kk), gf[kk], dp, 0, 0, 0);
      }
      if (DROP) {                                     // d(P) of a dropped probability is zero, of a kept one scaled
        const int64_t row = (int64_t)bh * L + qc;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint4 w = attn_drop_words(drop, row, (L + 3) >> 2, k0 + 32 * kb + 8 * g + 4 * h);
          dp[4 * g] = w.x < drop.thr ? 0.f : dp[4 * g] * drop.scale;
          dp[4 * g + 1] = w.y < drop.thr ? 0.f : dp[4 * g + 1] * drop.scale;
          dp[4 * g + 2] = w.z < drop.thr ? 0.f : dp[4 * g + 2] * drop.scale;
          dp[4 * g + 3] = w.w < drop.thr ? 0.f : dp[4 * g + 3] * drop.scale;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = fast_exp2(fmaf(s[r], c2, nlse_q)) * (dp[r] - delta_q);
      if (k0 + TK > Lk || (CAUSAL && k0 + TK - 1 > w0)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
          if (key >= Lk || (CAUSAL && key > qi)) s[r] = 0.f;
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 dsf = regs_to_frag(s, c);
#pragma unroll
        for (int db = 0; db < 2; ++db)
          dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.column(Ks, db, 32 * kb + 16 * c), dsf, dq[db], 0, 0, 0);
      }
    }
  }
  if (qi < sm.n) store_rows(dqkv + (sm.first + qi) * ld3 + hh * D, dq, h, scale);
}

// ------------------------------------------------------------------ dK, dV
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256, 2) void fa_bwd_dkv_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx,
                                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                                         bf16_t* __restrict__ dqkv, Rows rows, int L,
                                                        int nh, int pairs, DropDesc drop) {
  __shared__ __attribute__((aligned(1024))) bf16_t tiles[2][2][TILE];   // [buffer][Q, dO][query][d]
  __shared__ __attribute__((aligned(16))) float lse_s[2][TK], delta_s[2][TK];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kl = lane & 31, h = lane >> 5;
  int rb, bh;
  if (!row_block((L + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK, pairs, false, rb, bh)) return;
  const int b = bh / nh, hh = bh - b * nh;
  const int H = nh * D;
  const int64_t ld3 = 3 * (int64_t)H;
  const Sample sm = sample_rows(rows, b, L);
  if (rb * ROWS_PER_BLOCK >= sm.n) return;
  const bf16_t* base = qkv + sm.first * ld3 + hh * D;
  const bf16_t* gbase = dctx + sm.first * H + hh * D;
  const int w0 = rb * ROWS_PER_BLOCK + wave * 32, ki = w0 + kl;
  const int kc = min(ki, sm.n - 1);
  const float scale = 0.125f, c2 = scale * LOG2E;

  bf16x8 kf[4], vf[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    kf[kk] = ld_frag(base + (int64_t)kc * ld3 + H + 16 * kk + 8 * h);
    vf[kk] = ld_frag(base + (int64_t)kc * ld3 + 2 * H + 16 * kk + 8 * h);
  }
  f32x16 dk[2], dv[2];
  zero(dk[0]); zero(dk[1]); zero(dv[0]); zero(dv[1]);
  const int qstart = CAUSAL ? rb * ROWS_PER_BLOCK : 0;     // earlier queries never see these keys
  const int Lk = sm.keys;                                          // keys from Lk on are padding: their dK, dV are zero
  const int qend = rb * ROWS_PER_BLOCK >= Lk ? 0 : sm.n; // a block of padded keys only writes zeros

  FragAt at;
  at.init(lane);
  TileLoad load;
  load.init(wave, lane);
  const uint32_t lds = lds_address(&tiles[0][0][0]);
  float pre_lse = 0.f, pre_delta = 0.f;
  auto fetch = [&](int q0, int buf) {
    load.issue(base, ld3, q0, sm.n - 1, wave, lds + (uint32_t)buf * (4u * TILE));
    load.issue(gbase, H, q0, sm.n - 1, wave, lds + (uint32_t)buf * (4u * TILE) + 2u * TILE);
    if (tid < TK) {
      const int q = min(q0 + tid, sm.n - 1);
      pre_lse = lse[(int64_t)bh * L + q];
      pre_delta = delta[(int64_t)bh * L + q];
    }
  };
  if (qstart < qend) fetch(qstart, 0);
  for (int q0 = qstart, buf = 0; q0 < qend; q0 += TK, buf ^= 1) {
    // lse_s: ready for exp2.  This buffer was last read two tiles ago, before the last barrier.
    if (tid < TK) { lse_s[buf][tid] = -LOG2E * pre_lse; delta_s[buf][tid] = pre_delta; }
    landed();
    if (q0 + TK < qend) fetch(q0 + TK, buf ^ 1);
    if (w0 >= Lk || (CAUSAL && q0 + TK <= w0)) continue;   // no query of the tile sees this wave's keys
    const bf16_t *Qs = tiles[buf][0], *Gs = tiles[buf][1];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      f32x16 s, dp;
      zero(s); zero(dp);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.row(Qs, qb, kk), kf[kk], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.row(Gs, qb, kk), vf[kk], dp, 0, 0, 0);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int qq = 32 * qb + 8 * g + 4 * h;
        const float4 nl = *(const float4*)&lse_s[buf][qq], dl = *(const float4*)&delta_s[buf][qq];
        const float nls[4] = {nl.x, nl.y, nl.z, nl.w}, dls[4] = {dl.x, dl.y, dl.z, dl.w};
        // Dropout: this lane holds one key and four queries; a generator block covers four keys
        // of one query.  The four lanes of a quad (four neighbouring keys) each make the block of
        // one of the four queries and pass its decisions round.
        bool keep[4] = {true, true, true, true};
        if (DROP) {
          const int qmine = min(q0 + qq + (lane & 3), sm.n - 1);
          quad_keep(attn_drop_words(drop, (int64_t)bh * L + qmine, (L + 3) >> 2, ki & ~3), drop.thr, lane, keep);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * g + e;
          const float p = fast_exp2(fmaf(s[r], c2, nls[e]));
          if (DROP) {
            s[r] = keep[e] ? p * drop.scale : 0.f;                         // what multiplied V in the forward
            dp[r] = p * ((keep[e] ? dp[r] * drop.scale : 0.f) - dls[e]);
          } else {
            s[r] = p;
            dp[r] = p * (dp[r] - dls[e]);
          }
        }
      }
      if (q0 + TK > sm.n || (CAUSAL && q0 < w0 + 31)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int q = q0 + 32 * qb + 8 * (r >> 2) + 4 * h + (r & 3);
          if (q >= sm.n || (CAUSAL && ki > q)) { s[r] = 0.f; dp[r] = 0.f; }
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8 pf = regs_to_frag(s, c), dsf = regs_to_frag(dp, c);
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.column(Gs, db, 32 * qb + 16 * c), pf, dv[db], 0, 0, 0);
          dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at.column(Qs, db, 32 * qb + 16 * c), dsf, dk[db], 0, 0, 0);
        }
      }
    }
  }
  if (ki < sm.n) {
    if (ki >= Lk) { zero(dk[0]); zero(dk[1]); zero(dv[0]); zero(dv[1]); }   // whatever the lane's column held
    bf16_t* out = dqkv + (sm.first + ki) * ld3 + hh * D;
    store_rows(out + H, dk, h, scale);
    store_rows(out + 2 * H, dv, h, 1.f);
  }
}

void attention_fwd_mfma(const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int causal,
                        const DropDesc& drop, hipStream_t st) {
  const int pairs = B * nh;
  const dim3 grid((unsigned)((L + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK) * 8u * (unsigned)((pairs + 7) / 8));
#define FWD_(C, D) hipLaunchKernelGGL((fa_fwd_kernel<C, D>), grid, dim3(256), 0, st, (const bf16_t*)qkv, (bf16_t*)ctx, lse, rows, L, nh, pairs, drop)
  if (drop.thr) { if (causal) FWD_(true, true); else FWD_(false, true); }
  else { if (causal) FWD_(true, false); else FWD_(false, false); }
#undef FWD_
}

void attention_bwd_mfma(const void* qkv, const void* ctx, const void* dctx, const float* lse, float* delta, void* dqkv,
                        const Rows& rows, int B, int L, int nh, int causal, const DropDesc& drop, hipStream_t st, hipEvent_t done) {
  const int pairs = B * nh;
  const dim3 grid((unsigned)((L + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK) * 8u * (unsigned)((pairs + 7) / 8));
#define BWD_(C, D)                                                                                               \
  hipLaunchKernelGGL((fa_bwd_dq_kernel<C, D>), grid, dim3(256), 0, st, (const bf16_t*)qkv, (const bf16_t*)ctx,  \
                     (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, rows, L, nh, pairs, drop);                          \
  LAUNCH_MARKED_((fa_bwd_dkv_kernel<C, D>), grid, dim3(256), st, done, (const bf16_t*)qkv, (const bf16_t*)dctx, lse, \
                     delta, (bf16_t*)dqkv, rows, L, nh, pairs, drop)
  if (drop.thr) { if (causal) { BWD_(true, true); } else { BWD_(false, true); } }
  else { if (causal) { BWD_(true, false); } else { BWD_(false, false); } }
#undef BWD_
}

}  // namespace mk
