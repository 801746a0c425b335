// Device-side pieces shared by the GEMM kernels: argument block and fused epilogues.
#pragma once
#include "device_common.h"
#include "kernels.h"

namespace mk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers


// ---- direct loads from memory to LDS through buffer descriptors --------------------------------
typedef __attribute__((address_space(3))) void lds_void_l;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4_l;

// Offsets from a buffer's size on lie outside: such a lane's 16 bytes of LDS are written with zeros.  No
// buffer is larger than this.
constexpr uint32_t kOutside = 0x80000000u;

// One wave-level direct load: lane i's 16 bytes at base + offset land at lds + 16 * i.  Inline assembly,
// so the compiler does not track it: the waits are placed by hand in the loop, and so is the wait state
// between a write of M0 and the load that reads it (s_nop), which the hardware leaves to the program.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // m0 is a reserved register: named as clobbered on purpose
__device__ __forceinline__ void l_direct_load(uint64_t base, uint32_t bytes, uint32_t offset, uint32_t lds_byte_address) {
  const u32x4 r = {(uint32_t)base, (uint32_t)(base >> 32), bytes, 0x00020000u};                 // raw buffer
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" : : "v"(offset), "s"(r), "s"(lds_byte_address) : "memory", "m0");
}
// A descriptor's address and size, the same in all lanes, settled in scalar registers: a scalar register that
// a vector instruction (readfirstlane) wrote may be read by a load five wait states later, which the hardware
// does not wait for either.  What comes out of the assembly counts as scalar from here on: moved and added to
// by scalar instructions alone, which need no wait.
__device__ __forceinline__ void l_descriptor(const void* p, uint32_t size, uint64_t& base, uint32_t& bytes) {
  const uint64_t a = (uint64_t)p;
  uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)a), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32));
  bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)size);
  asm volatile("s_nop 4" : "+s"(lo), "+s"(hi), "+s"(bytes));
  base = (uint64_t)lo | (uint64_t)hi << 32;
}
// a / b, the same in all lanes: vector instructions compute it, and without this all that follows from it
__device__ __forceinline__ int l_div(int a, int b) { return __builtin_amdgcn_readfirstlane(a / b); }
__device__ __forceinline__ uint32_t l_lds_address(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_l*)p);
}
#pragma clang diagnostic pop

struct GemmDev {
  const void* A; const void* B; void* C;
  const void* bias; const void* resid; void* gelu_out; float* a_rowsum;
  int64_t lda, ldb, ldc, ldr;
  int M, N, K;
  int a_k, b_k, c_f32, gelu;
  int vec;               // C, bias, residual and GELU output allow 16-byte accesses at columns n % 8 == 0
  int a_tail_zero;       // A k-major, K % 8 != 0: the columns up to the next multiple of 8 exist and are zero
  int kb[9];             // part s of the reduction: indices kb[s] .. kb[s + 1] - 1
  int splits;            // > 1: k range cut in `splits` parts, raw fp32 tiles go to `partial`
  float* partial;        // [splits][M][N] followed by [splits][M] row sums
};

template <typename T>
__device__ __forceinline__ void epilogue(const GemmDev& p, int m, int n, float v) {
  if (m >= p.M || n >= p.N) return;
  if (p.bias) v += ld<T>((const T*)p.bias + n);
  if (p.resid) v += ld<T>((const T*)p.resid + (int64_t)m * p.ldr + n);
  int64_t o = (int64_t)m * p.ldc + n;
  if (p.c_f32) {
    ((float*)p.C)[o] = v;
  } else {
    st<T>((T*)p.C + o, v);
    if (p.gelu) st<T>((T*)p.gelu_out + o, p.gelu == GELU_TANH ? gelu_tanh(v) : gelu_erf(v));
  }
}

// ---- block tile -> C for the bf16 kernels -----------------------------------------------------
// A 128 x 128 block tile held by 4 waves (wave (wm, wn): rows wm*64.., columns wn*64..) as 2 x 2
// MFMA 32x32 accumulators with the operand roles swapped: accumulator (i, j), register r of a
// lane is row i*32 + lane%32, column j*32 + 8*(r/4) + 4*(lane/32) + r%4 of the wave's 64 x 64.
//
// In that layout a store instruction would touch 32 rows with 16 bytes each.  The tile is turned
// through LDS instead (the operand tiles are dead by then): every wave parks its 64 x 64 floats in
// 16 KB of its own, then walks them 8 rows at a time, 8 lanes per row with 8 consecutive columns
// each, so bias / residual loads and the C / GELU stores are whole 128-byte lines.  The walk is a
// rolled loop, which keeps the kernel's code small, except where the residuals were loaded ahead:
// they sit in registers that only an unrolled walk can name.  Float4 chunk c of row r sits at chunk
// position c ^ (r & 15): conflict-free for the accumulator writes (16 rows, one chunk) and for
// the row reads (two rows, all even or all odd chunks).

__device__ __forceinline__ void unpack_bf16x8(const u32x4 w, float (&f)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(w[e] << 16);
    f[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ u32x4 pack_bf16x8(const float (&f)[8]) {
  u32x4 w;
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(f[2 * e], f[2 * e + 1]);
  return w;
}

// eight finished values of row m, from column n on
__device__ __forceinline__ void put8(const GemmDev& p, int m, int n, const float (&v)[8]) {
  const int64_t o = (int64_t)m * p.ldc + n;
  if (p.c_f32) {
    *(float4*)((float*)p.C + o) = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)((float*)p.C + o + 4) = make_float4(v[4], v[5], v[6], v[7]);
  } else {
    *(u32x4*)((bf16_t*)p.C + o) = pack_bf16x8(v);
  }
}
// eight consecutive columns of row m, from column n on, through the epilogue (cb: their bias)
__device__ __forceinline__ void finish8(const GemmDev& p, int m, int n, float (&v)[8], const float (&cb)[8]) {
  if (n + 8 > p.N) {                                          // ragged end of the row
    for (int e = 0; e < 8; ++e) epilogue<bf16_t>(p, m, n + e, v[e]);
    return;
  }
  float f[8];
  if (p.bias) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += cb[e];
  }
  if (p.resid) {
    unpack_bf16x8(*(const u32x4*)((const bf16_t*)p.resid + (int64_t)m * p.ldr + n), f);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += f[e];
  }
  put8(p, m, n, v);
  const int64_t o = (int64_t)m * p.ldc + n;
  if (p.gelu == GELU_ERF) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = gelu_erf_bf16(v[e]);
    *(u32x4*)((bf16_t*)p.gelu_out + o) = pack_bf16x8(f);
  } else if (p.gelu == GELU_TANH) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = gelu_tanh_bf16(v[e]);
    *(u32x4*)((bf16_t*)p.gelu_out + o) = pack_bf16x8(f);
  }
}

// How a wave walks its 64 x 64 part, 32 (HALVES == 2) or 64 columns wide: every lane eight columns of
// a row, in eight steps altogether.
template <int HALVES>
struct Walk {
  static constexpr int COLS = 64 / HALVES, LPR = COLS / 8, RPI = 64 / LPR, STEPS = 64 / RPI;   // columns, lanes per row, rows per step, steps per half
  static __device__ __forceinline__ int row(int step, int lane) { return step * RPI + lane / LPR; }
  static __device__ __forceinline__ int col(int half, int lane) { return half * COLS + (lane % LPR) * 8; }
};

// The residuals of a wave's 64 x 64 part, all requested before the part is stored: requested one step
// of the walk at a time they cost a memory latency per step.  Products with a residual and fp32 output,
// 1024 columns: T = 16384, K = 1024 57 -> 48 us, K = 4096 (forward) 134 -> 124; T = 6352 92 -> 90; 768
// columns: T = 6400, K = 768 27 -> 23, K = 3072 62 -> 58.
__device__ __forceinline__ bool resid_ahead(const GemmDev& p) { return p.vec && p.resid && !p.gelu; }
template <int HALVES>
__device__ __forceinline__ void load_resid(const GemmDev& p, int m0w, int n0w, int lane, u32x4 (&r)[8]) {
  typedef Walk<HALVES> W;
  if (!resid_ahead(p)) return;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int m = m0w + W::row(q % W::STEPS, lane), n = n0w + W::col(q / W::STEPS, lane);
    if (m < p.M && n + 8 <= p.N) r[q] = *(const u32x4*)((const bf16_t*)p.resid + (int64_t)m * p.ldr + n);
  }
}

// m0w, n0w: first row / column of this wave's 64 x 64 part; wstage: 16 KB / HALVES of LDS that only
// this wave uses from here on (HALVES == 2: the two 32-column halves take turns in 8 KB); r: load_resid's.
template <int HALVES>
__device__ __forceinline__ void store_tile(const GemmDev& p, const f32x16 (&acc)[2][2], int m0w, int n0w, int lane,
                                           float* wstage, const u32x4 (&r)[8]) {
  typedef Walk<HALVES> W;
  constexpr int COLS = W::COLS, CHUNKS = COLS / 4;              // staged columns, float4 chunks
#pragma unroll
  for (int h = 0; h < HALVES; ++h) {
    __builtin_amdgcn_wave_barrier();                            // the previous half's reads stay before
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jj = 0; jj < 2 / HALVES; ++jj)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int j = HALVES == 2 ? h : jj;
          const int row = i * 32 + (lane & 31), c = jj * 8 + 2 * g + (lane >> 5);
          *(float4*)&wstage[row * COLS + ((c ^ (row & (CHUNKS - 1))) << 2)] =
              make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
        }
    __builtin_amdgcn_wave_barrier();
    if (!p.vec) {                                               // unaligned operands: one element at a time
      for (int idx = lane; idx < 64 * COLS; idx += 64) {
        const int row = idx / COLS, col = idx % COLS;
        epilogue<bf16_t>(p, m0w + row, n0w + h * COLS + col,
                         wstage[row * COLS + ((((col >> 2) ^ (row & (CHUNKS - 1))) << 2) | (col & 3))]);
      }
      continue;
    }
    const int n = n0w + W::col(h, lane), c0 = 2 * (lane % W::LPR);
    float cb[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};    // the columns' bias: the same for every row
    if (p.bias && n + 8 <= p.N) unpack_bf16x8(*(const u32x4*)((const bf16_t*)p.bias + n), cb);
    auto staged = [&](int row, float (&v)[8]) {
      const float4 lo = *(const float4*)&wstage[row * COLS + ((c0 ^ (row & (CHUNKS - 1))) << 2)];
      const float4 hi = *(const float4*)&wstage[row * COLS + (((c0 + 1) ^ (row & (CHUNKS - 1))) << 2)];
      v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w; v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
    };
    if (resid_ahead(p)) {
#pragma unroll
      for (int it = 0; it < W::STEPS; ++it) {
        const int row = W::row(it, lane), m = m0w + row;
        if (m >= p.M || n >= p.N) continue;
        float v[8];
        staged(row, v);
        if (n + 8 > p.N) {
          for (int e = 0; e < 8; ++e) epilogue<bf16_t>(p, m, n + e, v[e]);
          continue;
        }
        float f[8];
        unpack_bf16x8(r[h * W::STEPS + it], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] + cb[e] + f[e];
        put8(p, m, n, v);
      }
    } else {
      for (int it = 0; it < W::STEPS; ++it) {
        const int row = W::row(it, lane), m = m0w + row;
        if (m >= p.M || n >= p.N) continue;
        float v[8];
        staged(row, v);
        finish8(p, m, n, v, cb);
      }
    }
  }
}

}  // namespace mk
