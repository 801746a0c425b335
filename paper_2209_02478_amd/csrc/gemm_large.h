// bf16 GEMM, large block tiles walked by persistent blocks.
//
// C[M,N] = sum_k A(m,k) B(n,k).  One block of 8 waves on a compute unit takes tile after tile of 256 x 256
// (FM = 8) or 128 x 256 (FM = 4); a wave owns 16 * FM x 64 of it as MFMA tiles of 16 x 16 x 32.  Why these
// sizes on gfx950: a compute unit draws about 54 bytes per clock from the L2, a 128 x 128 tile needs
// 64 at full matrix rate, 128 x 256 needs 48, 256 x 256 needs 32; and under matrix load the clock follows
// the power drawn (2.4 GHz with the matrix cores idle, 1.7 in the loop below with all units at it), so
// bytes moved per MFMA cost time even where they are hidden.  16 x 16 x 32 draws a tenth less than
// 32 x 32 x 16 (2.03 against 1.85 PFLOP/s in a loop of MFMAs alone on N(0,0.25) operands) and gives the
// same bits as two of those in a row, so the 128 x 128 kernels and these agree bit for bit.
//
// Operand tiles (64 reduction indices) go global -> LDS directly into rings that fill the 160 KB: FM = 8
// three slots of A and two of B, FM = 4 four and three.  A is requested NB k tiles ahead half a turn
// earlier than B.  A load is one buffer instruction with a per-lane offset that is fixed for the tile
// and a scalar base that moves along k: its descriptor stays in scalar registers, so issuing it takes the write
// of M0, the wait state behind that and the load, and the loop has no branch around it (a wave that has to
// branch around its loads loses about 60 clocks for each).  The loads run through the tile boundary: while a tile's
// last MFMAs and its store run, the first k tiles of the block's next one are on their way, so only a block's first
// tile waits for memory.
//
// The eight waves run freely, two on each SIMD, and meet once per k tile; a fragment's register takes
// the next half's as soon as the MFMAs that use it are issued.  K tile t, a wave's view:
//     half 0 (32 indices)         :  MFMAs; reads of half 1; loads of A tile t + NB (slot of tile t - 1)
//     half 1, the first quarter   :  MFMAs
//     own loads of tile t + 1 have landed, own reads of tile t are done: all waves meet
//     half 1, the rest            :  MFMAs; reads of tile t + 1, half 0; loads of B tile t + NB (slot of tile t)
// FM = 8, before the descriptors stayed in scalar registers: 2450 clocks per k tile with everything in the L2, of which MFMAs alone take 2048, the meeting
// about 200 and the fragment reads 100.
//
// A tile's store: the MFMA's operand roles are swapped (rows of B feed its A side), so a lane holds 4
// consecutive columns of one row.  16 rows of 128 bytes at a time go through 2 KB of LDS of the wave's own
// (the part of the free ring slot that its next loads fill) and come back with 8 lanes along each row;
// residuals take the same way in.  Whole lines with the lanes across the rows, by exchanges between
// lanes, leave a unit at 31 bytes per clock, along the rows at 104.  Whole launches of 262144 x 1024, K = 512,
// the one against the other (us): bf16 312 -> 293, with residual 340 -> 331, fp32 370 -> 346, with
// residual 442 -> 424, data gradient 298 -> 277; between tiles 8.0 -> 6.6 us in bf16, 11.9 -> 10.2 in fp32.  The
// loads of the first turn after a store wait at its end, so that its MFMAs are not held up behind the
// stores on their way out (bert_base 32 x 200 iterations 0.5 %, 32 x 512 1.5, bert_stages 32 x 332 1.1).
//
// Measured with rotating operands in one run, against the tiles of 256 x 256 in 32 x 32 x 16 MFMAs with a
// block per tile that this replaced (us): 65536 x 3072, K = 1024, bf16 454 -> 387; 65536 x 4096, K = 1024,
// with GELU 746 -> 624; 65536 x 1024, K = 4096, fp32 with residual 488 -> 449; data gradients 65536 x 4096,
// K = 1024 545 -> 462, 65536 x 1024, K = 4096 454 -> 410; weight gradient 30528 x 1024, K = 20480 with row sums
// 1164 -> 1076.  1.45 us per 64 reduction indices, bound by power; between tiles 5-10 us, bound by the stores'
// way into the L2, 15 with residuals or GELU (starting some compute units or XCDs half a tile later, or
// streaming stores, changed nothing).
//
// LDS layouts (16-byte chunks permuted so that fragment reads are conflict-free although a direct
// load can only write 1 KB contiguously):
//   k-major tile [rows][64 k], 128-byte rows : chunk kc of row r sits at kc ^ ((r >> 1) & 7)
//   m-major tile [64 k][rows]               : chunk mc of k row q sits at mc ^ (4 * (q & 3) + 2 * ((q >> 3) & 1))
// k-major fragments are one 16-byte read, m-major fragments two transposing 8-byte reads.
// The reduction order over k is fixed by the shape alone (results reproducible bit for bit).
#pragma once
#include "gemm_device.h"

#include <type_traits>

namespace mk {

namespace large {

constexpr int LBN = 256;                         // tile columns
constexpr int LBK = 64;                          // reduction indices per k tile
constexpr int LGROUP_M = 4;                      // row panels per tile group (L2 reuse)
constexpr int FN = 4;                            // 16 x 16 tiles of a wave across; down: FM = 8 or 4

// Sizes of a variant: FM blocks of 16 rows per wave, tiles of 32 * FM rows.
template <int FM>
struct Sizes {
  static constexpr int BM = 32 * FM;
  static constexpr int NB = FM == 8 ? 2 : 3, NA = NB + 1;             // ring slots of B and A: 160 KB
  static constexpr int A_TILE = BM * LBK, B_TILE = LBN * LBK;         // elements
  static constexpr int A_LOADS = BM / 64, B_LOADS = LBN / 64;         // 1 KB direct loads per wave and operand tile
  static constexpr int SMEM = (NA * A_TILE + NB * B_TILE) * 2;
  static constexpr int MEET = FM / 4;                                 // rows of the second half multiplied before the waves meet
  // loads younger than those of the next k tile when the waves meet: NB - 2 whole k tiles and an A tile
  static constexpr int YOUNGER = (NB - 2) * (A_LOADS + B_LOADS) + A_LOADS;
  static constexpr int STORES = 2 * FM;                               // 16-byte stores of a bf16 tile per lane
};

constexpr int kLibrary = 4;                      // on top of the GELU's form

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// 16 and 8 bytes wherever an element may lie: the same instructions, at full speed where they are aligned
typedef uint32_t u32x4_at4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_at2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_at2 __attribute__((ext_vector_type(2), aligned(2)));

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14)
constexpr int kLdsDone = 15 | (7 << 4) | (0 << 8) | (3 << 14);      // LDS operations done, vector memory untouched
constexpr int in_flight(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }   // at most n vector memory operations

__device__ __forceinline__ void l_meet() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// R: rows of the operand's tiles
template <bool KM, int R>
struct LTileOf {
  // Direct load j of a wave (a wave's loads follow each other, an even number or two) brings 64 chunks.
  // Byte offset of the lane's from the tile's first element, j = 0 or 1; that of j + 2 is this and 2 * two(ld).
  static __device__ __forceinline__ uint32_t src(int64_t ld, int rows, int j, int lane) {
    if (KM) {
      const int r = 8 * j + (lane >> 3), kc = (lane & 7) ^ ((r >> 1) & 7);
      return (uint32_t)(r * (int)ld + kc * 8) * 2u;               // rows outside the matrix: behind the buffer's end
    }
    constexpr int RC = R / 8;                                     // chunks per k row
    const int q = j * (64 / RC) + lane / RC, mc = (lane % RC) ^ (4 * (q & 3) + 2 * ((q >> 3) & 1));
    return mc * 8 < rows ? (uint32_t)(q * (int)ld + mc * 8) * 2u : kOutside;
  }
  static __device__ __forceinline__ uint32_t two(int64_t ld) { return (uint32_t)(KM ? 16 : 2 * 64 / (R / 8)) * (uint32_t)ld * 2u; }
  // size of the buffer that starts at the tile's first row and this k tile: the rows that exist end it
  static __device__ __forceinline__ uint32_t bytes(int64_t ld, int rows) { return KM ? (uint32_t)min(rows, R) * (uint32_t)ld * 2u : kOutside; }
  // whether that chunk lies behind the last of `left` reduction indices
  static __device__ __forceinline__ bool behind(int left, int j, int lane) {
    if (KM) return (((lane & 7) ^ ((4 * j + (lane >> 4)) & 7)) << 3) >= left;
    return lane / (R / 8) >= left - j * (64 / (R / 8));
  }
  // this lane's place in the fragments of the 16-row blocks from first_block on (a multiple of 4)
  int at[2];
  __device__ __forceinline__ void init(int first_block, int lane) {
    if (KM) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        at[h] = (first_block * 16 + (lane & 15)) * LBK + (((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) << 3);
    } else {
      const int g = lane >> 4, kq = (lane & 15) >> 2;
      at[0] = (8 * g + kq) * R + (((2 * first_block) ^ (((lane & 3) >> 1) + 4 * kq + 2 * (g & 1))) << 3) + (lane & 1) * 4;
      at[1] = 0;
    }
  }
  // fragment of block i, half h (both compile-time after unrolling): row lane % 16, indices 8 * (lane / 16) .. +7
  __device__ __forceinline__ bf16x8 read(const bf16_t* ring, int slot, int i, int h) const {
    if (KM) return *(const bf16x8*)(ring + slot + at[h] + i * 16 * LBK);
    const bf16_t* p = ring + ((slot + at[0]) ^ (i * 16)) + h * 32 * R;      // block i: bits 1 .. 3 of the chunk number
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_l*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_l*)(p + 4 * R));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

}  // namespace large

// GE: GELU in the store (GELU_NONE, GELU_ERF, GELU_TANH), of the sum with bias and residual, by the C library's
// functions in every column with kLibrary on top (C not on 16 bytes, as in the other kernels); a product
// without it stores bf16 or fp32, with or without bias and residual.  SUMS: row sums with B k-major; a loop with and
// one without them do not fit the registers there, and reloads in the loop wait for its loads to LDS (10624 x 1024,
// K = 4096: 110 us and, without sums, 105; apart 86 and 80), so every tile takes them.
template <int FM, bool AK, bool BKM, bool KTAIL, int GE, bool SUMS>
__global__ __launch_bounds__(512) void bgemm_large_kernel(GemmDev p, int tiles_n, int total, int per_xcd) {
  using namespace large;
  typedef Sizes<FM> Z;
  typedef LTileOf<AK, Z::BM> TA;
  typedef LTileOf<BKM, LBN> TB;
  constexpr int LA = Z::A_LOADS, LB = Z::B_LOADS, MEET = Z::MEET;
  constexpr bool LIBRARY = GE & kLibrary;
  constexpr int FORM = GE & (kLibrary - 1);
  extern __shared__ __attribute__((aligned(1024))) unsigned char l_smem[];
  bf16_t* const ring = (bf16_t*)l_smem;
  bf16_t* const ring_b = ring + Z::NA * Z::A_TILE;
  // Block ids go to the 8 XCDs in turn: XCD x gets the run of per_xcd units from x * per_xcd on, each of its 32
  // blocks (one per compute unit) every 32nd of them.  Units run part by part (all tiles of
  // the first k range, then of the second, ...): a run then shares one k range of both operands in the L2.
  constexpr int stride = 32;
  int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  const int u_end = min((int)(blockIdx.x & 7) * per_xcd + per_xcd, total);
  if (unit >= u_end) return;
  const int n_tiles = total / p.splits, tiles_m = (p.M + Z::BM - 1) / Z::BM;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform: address arithmetic on it stays scalar
  const int wm = wave >> 2, wn = wave & 3;
  constexpr bool PARTS = !BKM, WG = !AK && !BKM;                  // reduction cut in parts; weight gradients: no bias, no residual

  // ---- the loads' position: unit, its tile, the k tile
  struct Place { int m0, n0, split; } cur, ahead;
  int c_unit = unit, c_left, c_k;                                 // k tiles left; reduction indices left (KTAIL)
  uint64_t base_a, base_b;
  int64_t step_a = AK ? LBK * 2 : (int64_t)LBK * 2 * p.lda, step_b = BKM ? LBK * 2 : (int64_t)LBK * 2 * p.ldb;
  uint32_t off_a[2], off_b[2], bytes_a, bytes_b;
  auto enter = [&]() __attribute__((always_inline)) {                                            // first k tile of unit c_unit
    const int split = PARTS ? l_div(c_unit, n_tiles) : 0, t = c_unit - split * n_tiles;
    const int group = l_div(t, LGROUP_M * tiles_n), first_m = group * LGROUP_M;
    const int gsize = min(tiles_m - first_m, LGROUP_M);
    const int in_group = t - group * LGROUP_M * tiles_n, across = l_div(in_group, gsize);
    ahead = {(first_m + in_group - across * gsize) * Z::BM, across * LBN, split};
    const int k0 = p.kb[split];
    c_k = p.kb[split + 1] - k0;
    c_left = (c_k + LBK - 1) / LBK;
    l_descriptor((const bf16_t*)p.A + (AK ? (int64_t)ahead.m0 * p.lda + k0 : (int64_t)k0 * p.lda + ahead.m0),
                 TA::bytes(p.lda, p.M - ahead.m0), base_a, bytes_a);
    l_descriptor((const bf16_t*)p.B + (BKM ? (int64_t)ahead.n0 * p.ldb + k0 : (int64_t)k0 * p.ldb + ahead.n0),
                 TB::bytes(p.ldb, p.N - ahead.n0), base_b, bytes_b);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      off_a[j] = TA::src(p.lda, p.M - ahead.m0, wave * LA + j, lane);
      off_b[j] = TB::src(p.ldb, p.N - ahead.n0, wave * LB + j, lane);
    }
  };
  enter();
  cur = ahead;
  const uint32_t lds_a = l_lds_address(ring) + (uint32_t)wave * LA * 1024u;
  const uint32_t lds_b = l_lds_address(ring_b) + (uint32_t)wave * LB * 1024u;
  uint32_t fill_a = 0, fill_b = 0;                                // slots to fill, in bytes
  const uint32_t two_a = TA::two(p.lda), two_b = TB::two(p.ldb);
  auto load_a = [&](int j) __attribute__((always_inline)) {
    const uint32_t at = off_a[j & 1] + (j >> 1) * two_a;
    l_direct_load(base_a, bytes_a, KTAIL && TA::behind(c_k, wave * LA + j, lane) ? kOutside : at, lds_a + fill_a + j * 1024u);
  };
  auto load_b = [&](int j) __attribute__((always_inline)) {
    const uint32_t at = off_b[j & 1] + (j >> 1) * two_b;
    l_direct_load(base_b, bytes_b, KTAIL && TB::behind(c_k, wave * LB + j, lane) ? kOutside : at, lds_b + fill_b + j * 1024u);
  };
  // On to the next k tile, or the next unit's first.  Behind the block's last the same k tile is
  // requested again, into slots that are not read any more.
  auto advance = [&]() __attribute__((always_inline)) {
    fill_a = fill_a == (Z::NA - 1) * Z::A_TILE * 2u ? 0 : fill_a + Z::A_TILE * 2u;
    fill_b = fill_b == (Z::NB - 1) * Z::B_TILE * 2u ? 0 : fill_b + Z::B_TILE * 2u;
    base_a += step_a; base_b += step_b;
    c_k -= KTAIL ? LBK : 0;
    if (--c_left == 0) {                                          // (no else: its merge would leave the sizes in vector registers)
      const bool more = c_unit + stride < u_end;
      base_a -= more ? 0 : step_a; base_b -= more ? 0 : step_b;
      step_a = more ? step_a : 0; step_b = more ? step_b : 0;
      c_left = 1 << 30; c_k = 0;                                  // (no reduction index is left: zeros where KTAIL)
      if (more) {
        c_unit += stride;
        enter();
      }
    }
  };

  // ---- fragments of the k tile being multiplied
  TA fa;
  TB fb;
  fa.init(wm * FM, lane);
  fb.init(wn * FN, lane);
  int slot_a = 0, slot_b = 0;                                     // in elements
  bf16x8 af[FM], bfr[2][FN];
  auto read_a = [&](int i, int h) __attribute__((always_inline)) { af[i] = fa.read(ring, slot_a, i, h); };
  auto read_b = [&](int j, int h) __attribute__((always_inline)) { bfr[h][j] = fb.read(ring_b, slot_b, j, h); };
  f32x4 acc[FM][FN];
  // Row sums of A (bias gradients): the first column tiles take 64 rows each; a lane sums two neighbouring rows,
  // for each every 16th reduction index (the order of these sums is that of the other kernels with direct loads, and leaving out
  // 16 rows of zeros does not change it).  All waves of such a tile do the same share, 4 reads and 16 operations
  // in a k tile, so that none is late where they meet.  All rows' sums in the first column tile, in half of the
  // lanes, took a sixth of its time, and the first two waves of each column tile a seventh of everyone's.
  // 20480 indices: 4096 x 1024 339 -> 303 us (without the sums 285), 1024 x 4096 314 -> 280, 30528 x 1024 1245 -> 1065.
  constexpr int SUM_TILES = Z::BM / 64;
  const int sum_pos = 2 * wave + (lane >> 5);
  int sum_at = 0;
  float rs[2];
  int stored = 0, young = 1;                                      // stores of the tile before, and for how many turns they are younger than the loads waited for

  auto k_tile = [&](auto first_, auto sums_) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_)::value, SUM = decltype(sums_)::value;
    auto row = [&](int i, int h) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[h][j], af[i], FIRST && h == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][j], 0, 0, 0);
    };
    uint32_t sf[4];
    if (SUM)
#pragma unroll
      for (int u = 0; u < 4; ++u) sf[u] = *(const uint32_t*)(ring + slot_a + sum_at + u * 16 * Z::BM);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      if (SUM && i >= FM - 4) {
        rs[0] += __uint_as_float(sf[i - (FM - 4)] << 16);
        rs[1] += __uint_as_float(sf[i - (FM - 4)] & 0xFFFF0000u);
      }
      row(i, 0);
      read_a(i, 1);
      if (i < FN) read_b(i, 1);
      if (!FIRST && i % (FM / LA) == 0) {
        __builtin_amdgcn_sched_barrier(0);
        load_a(i / (FM / LA));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < MEET; ++i) row(i, 1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kLdsDone);
    // all but the loads of later k tiles and, in a tile's first turns, the stores of the tile before
    constexpr int YOUNGER = Z::YOUNGER - (FIRST ? LA : 0);        // (a tile's first turn has issued none yet)
    if (stored == 2 * Z::STORES) __builtin_amdgcn_s_waitcnt(in_flight(YOUNGER + 2 * Z::STORES));
    else if (stored == Z::STORES) __builtin_amdgcn_s_waitcnt(in_flight(YOUNGER + Z::STORES));
    else __builtin_amdgcn_s_waitcnt(in_flight(YOUNGER));
    if (--young == 0) stored = 0;
    l_meet();
    slot_a = slot_a == (Z::NA - 1) * Z::A_TILE ? 0 : slot_a + Z::A_TILE;
    slot_b = slot_b == (Z::NB - 1) * Z::B_TILE ? 0 : slot_b + Z::B_TILE;
#pragma unroll
    for (int i = 0; i < MEET; ++i) read_a(i, 0);
#pragma unroll
    for (int i = MEET; i < FM; ++i) {
      row(i, 1);
      read_a(i, 0);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        if (j * (FM - MEET) / FN == i - MEET) {
          read_b(j, 0);
          if (!FIRST) {
            __builtin_amdgcn_sched_barrier(0);
            load_b(j);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
    }
    if (FIRST) {                                                  // behind the stores of the tile before
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < LA; ++j) load_a(j);
#pragma unroll
      for (int j = 0; j < LB; ++j) load_b(j);
      __builtin_amdgcn_sched_barrier(0);
    }
    advance();
  };

  // ---- a finished tile
  // C and its leading dimension are the workspace's where the reduction is cut in parts
  auto store = [&](auto edge_, auto f32_, auto resid_, auto bias_, void* C, int64_t ldc) __attribute__((always_inline)) {
    constexpr bool EDGE = decltype(edge_)::value, C32 = decltype(f32_)::value, RESID = decltype(resid_)::value, BIAS = decltype(bias_)::value;
    // from a copy of the lane that the compiler takes for new: what the store computes from it would be held
    // through the loop, which has no registers left
    int l = lane;
    asm volatile("" : "+v"(l));
    const int lr = l & 15, lq = l >> 4, sr = l >> 3, sc = l & 7;   // place in a fragment: row, group of 4 columns; in memory: row, 16 bytes
    const int nw = cur.n0 + wn * 64, mw = cur.m0 + wm * FM * 16 + sr;
    u32x2 cb[FN];                                                 // bias of the lane's columns (the sums are never -0: adding 0 is no change)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      cb[j] = u32x2{0u, 0u};
      const int n = nw + 4 * lq + j * 16;
      if (BIAS && p.bias) {
        if (!EDGE || n + 4 <= p.N) cb[j] = *(const u32x2_at2*)((const bf16_t*)p.bias + n);
        else
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < p.N) cb[j][e >> 1] |= (uint32_t)((const bf16_t*)p.bias)[n + e] << (16 * (e & 1));
      }
    }
    // From fragment order to memory order through LDS, 16 rows of 128 bytes at a time: a store then takes whole
    // rows with the lanes along them.  The place is what this wave's own loads of A fill in the next turn: nobody
    // reads it any more, and nothing is on its way there.  The 16-byte chunks of a row are permuted by the row.
    unsigned char* const turn = l_smem;
    const uint32_t own = fill_a + (uint32_t)wave * LA * 1024u;
    const uint32_t in16 = own + lr * 128 + (((lq >> 1) ^ (lr >> 1)) << 4) + (lq & 1) * 8;      // 4 columns of bf16; column tile j: ^ 32 j
    const uint32_t in32 = own + lr * 128 + ((lq ^ (lr >> 1)) << 4);                           // of fp32; second of two tiles: ^ 64
    const uint32_t out = own + sr * 128 + ((sc ^ (sr >> 1)) << 4);                            // rows 8 .. 15: + 1024 and ^ 64
    auto fence = [&]() __attribute__((always_inline)) { asm volatile("" ::: "memory"); };
    constexpr int DEPTH = 2;                                      // rows of residuals requested ahead (three spill)
    u32x4 r[FM][2];                                               // in memory order
    u32x2 rf[FN];                                                 // of one row, in fragment order
    auto load = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int m = mw + i * 16 + s * 8, n = nw + sc * 8;
        // where the row ends within these 8 columns, its last 8, shifted when they are used (an element at a time each
        // row waits for memory: 1300 x 6500, K = 1024 data gradient with residual 40 us against 28)
        const bf16_t* at = (const bf16_t*)p.resid + (int64_t)m * p.ldr + (EDGE && n + 8 > p.N ? p.N - 8 : n);
        r[i][s] = u32x4{0u, 0u, 0u, 0u};
        if (!EDGE || (m < p.M && n < p.N)) r[i][s] = *(const u32x4_at2*)at;
      }
    };
    // the last N & 7 of 8 columns, in front
    auto shift = [&](const u32x4& w) __attribute__((always_inline)) {
      const uint64_t lo = (uint64_t)w[1] << 32 | w[0], hi = (uint64_t)w[3] << 32 | w[2];
      const int bits = 16 * (8 - (p.N & 7));
      const uint64_t x = bits < 64 ? lo >> bits | hi << (64 - bits) : hi >> ((bits - 64) & 63), y = bits < 64 ? hi >> bits : 0;
      return u32x4{(uint32_t)x, (uint32_t)(x >> 32), (uint32_t)y, (uint32_t)(y >> 32)};
    };
    auto spread = [&](int i) __attribute__((always_inline)) {
      fence();
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (EDGE && nw + sc * 8 + 8 > p.N) r[i][s] = shift(r[i][s]);
        *(u32x4*)(turn + ((out + s * 1024) ^ (s * 64))) = r[i][s];
      }
      fence();
#pragma unroll
      for (int j = 0; j < FN; ++j) rf[j] = *(const u32x2*)(turn + (in16 ^ (j * 32)));
      fence();
    };
    // Step t (row i = t / PER of fragments; of it the left or right columns in fp32, C or the GELU output) is
    // read back when it is written, and stored a step later
    constexpr int PER = C32 || GE != GELU_NONE ? 2 : 1;
    u32x4 held[2];
    auto send = [&](int t) __attribute__((always_inline)) {
      const int n = C32 ? nw + (t % PER) * 32 + sc * 4 : nw + sc * 8;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int m = mw + t / PER * 16 + s * 8;
        if (C32) {
          float* to = (float*)C + (int64_t)m * ldc + n;
          if (!EDGE || (m < p.M && n + 4 <= p.N)) *(u32x4_at4*)to = held[s];
          else if (m < p.M)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n + e < p.N) to[e] = __uint_as_float(held[s][e]);
        } else {
          bf16_t* to = (bf16_t*)(t % PER ? p.gelu_out : C) + (int64_t)m * ldc + n;
          if (!EDGE || (m < p.M && n + 8 <= p.N)) *(u32x4_at2*)to = held[s];
          else if (m < p.M)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (n + e < p.N) to[e] = (bf16_t)(held[s][e >> 1] >> (16 * (e & 1)));
        }
      }
    };
    auto back = [&](int t) __attribute__((always_inline)) {
      fence();
      const u32x4 w0 = *(const u32x4*)(turn + out), w1 = *(const u32x4*)(turn + ((out + 1024) ^ 64));
      fence();
      if (t > 0) send(t - 1);
      held[0] = w0; held[1] = w1;
    };
    auto put_bf16 = [&](int t, const f32x4 (&v)[FN]) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
        *(u32x2*)(turn + (in16 ^ (j * 32))) = u32x2{pack_bf16x2(v[j][0], v[j][1]), pack_bf16x2(v[j][2], v[j][3])};
      back(t);
    };
    auto put_f32 = [&](int t, const f32x4& x, const f32x4& y) __attribute__((always_inline)) {
      *(f32x4*)(turn + in32) = x;
      *(f32x4*)(turn + (in32 ^ 64)) = y;
      back(t);
    };
    // the last N % 8 columns take the C library's erf and tanh, as in the other kernels (tail: the first of them,
    // from the wave's first column on)
    const int tail = (p.N & ~7) - nw;
    const bool ragged = EDGE && GE != GELU_NONE && !LIBRARY && (p.N & 7) && tail >= 0 && tail < 64;
    if (RESID) {
#pragma unroll
      for (int i = 0; i < DEPTH; ++i) load(i);
      spread(0);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      f32x4 v[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        v[j] = acc[i][j];
        if (BIAS) {
          v[j][0] += __uint_as_float(cb[j][0] << 16); v[j][1] += __uint_as_float(cb[j][0] & 0xFFFF0000u);
          v[j][2] += __uint_as_float(cb[j][1] << 16); v[j][3] += __uint_as_float(cb[j][1] & 0xFFFF0000u);
        }
        if (RESID) {
          v[j][0] += __uint_as_float(rf[j][0] << 16); v[j][1] += __uint_as_float(rf[j][0] & 0xFFFF0000u);
          v[j][2] += __uint_as_float(rf[j][1] << 16); v[j][3] += __uint_as_float(rf[j][1] & 0xFFFF0000u);
        }
      }
      if (C32) {
        put_f32(2 * i, v[0], v[1]);
        put_f32(2 * i + 1, v[2], v[3]);
      } else {
        put_bf16(PER * i, v);
        if (GE != GELU_NONE) {
          f32x4 x = v[0];
          if (ragged) {
#pragma unroll
            for (int j = 1; j < FN; ++j)
              if (tail >> 4 == j) x = v[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = FORM == GELU_ERF ? gelu_erf(x[e]) : gelu_tanh(x[e]);
          }
#pragma unroll
          for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (LIBRARY) v[j][e] = FORM == GELU_ERF ? gelu_erf(v[j][e]) : gelu_tanh(v[j][e]);
              else v[j][e] = FORM == GELU_ERF ? gelu_erf_bf16(v[j][e]) : gelu_tanh_bf16(v[j][e]);
            if (ragged && tail >> 4 == j && (tail >> 3 & 1) == lq >> 1) v[j] = x;
          }
          put_bf16(PER * i + 1, v);
        }
      }
      if (RESID && i + DEPTH < FM) load(i + DEPTH);
      if (RESID && i + 1 < FM) spread(i + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    send(PER * FM - 1);
    stored = EDGE ? 0 : (GE != GELU_NONE || C32) ? 2 * Z::STORES : Z::STORES;
    young = Z::NB - 1;
  };

  // ---- the block's tiles
#pragma unroll
  for (int t = 0; t < Z::NB; ++t) {
#pragma unroll
    for (int j = 0; j < LA; ++j) load_a(j);
#pragma unroll
    for (int j = 0; j < LB; ++j) load_b(j);
    advance();
  }
  __builtin_amdgcn_s_waitcnt(in_flight((Z::NB - 1) * (LA + LB)));
  l_meet();
  typedef std::true_type T;
  typedef std::false_type F;
  for (;;) {
    // (read again where the tile before has read them ahead: kept through its store they cost registers)
#pragma unroll
    for (int j = 0; j < FN; ++j) read_b(j, 0);
#pragma unroll
    for (int i = 0; i < FM; ++i) read_a(i, 0);
    const int nk = (p.kb[cur.split + 1] - p.kb[cur.split] + LBK - 1) / LBK;
    // raw fp32 tile and row sums of this k range, as a plain matrix [M][N] in the workspace; a
    // second kernel adds the parts in order
    const bool part = PARTS && p.splits > 1;
    float* const rowsum = part ? p.partial + (int64_t)p.splits * p.M * p.N + (int64_t)cur.split * p.M : p.a_rowsum;
    void* const C = part ? (void*)(p.partial + (int64_t)cur.split * p.M * p.N) : p.C;
    const int64_t ldc = part ? p.N : p.ldc;
    const bool c_f32 = part || p.c_f32;
    const bool sum_tile = (WG || SUMS) && p.a_rowsum && cur.n0 < SUM_TILES * LBN;
    if (SUMS || sum_tile) {
      const int chunk = (sum_tile ? cur.n0 / LBN * 8 : 0) + ((lane & 31) >> 2);
      sum_at = sum_pos * Z::BM + ((chunk ^ (4 * (sum_pos & 3) + 2 * ((sum_pos >> 3) & 1))) << 3) + 2 * (lane & 3);
      rs[0] = rs[1] = 0.f;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int kt = 0; kt < nk; ++kt) k_tile(F(), T());
      // the 16 sums of a row, in order, through the free slot of A (see the store)
      auto place = [&](int pos, int r) __attribute__((always_inline)) {
        return (float*)(l_smem + fill_a + (pos >> 1) * LA * 1024 + (pos & 1) * 256) + r;
      };
      if (sum_tile) {
        *(float2*)place(sum_pos, 2 * (lane & 31)) = make_float2(rs[0], rs[1]);
        __builtin_amdgcn_s_waitcnt(kLdsDone);
        l_meet();
        if (wave == 0) {
          float s = 0.f;
#pragma unroll
          for (int g = 0; g < 16; ++g) s += *place(g, lane);
          const int m = cur.m0 + cur.n0 / LBN * 64 + lane;
          if (m < p.M) rowsum[m] = s;
        }
        __builtin_amdgcn_s_waitcnt(kLdsDone);
        l_meet();
      }
    } else {
      k_tile(T(), F());
      for (int kt = 1; kt < nk; ++kt) k_tile(F(), F());
    }
    const bool inside = cur.m0 + Z::BM <= p.M && cur.n0 + LBN <= p.N, resid = !WG && p.resid;
    auto store_as = [&](auto f32_, auto resid_) __attribute__((always_inline)) {
      auto with = [&](auto bias_) __attribute__((always_inline)) {
        if (!LIBRARY && inside) store(F(), f32_, resid_, bias_, C, ldc);
        else store(T(), f32_, resid_, bias_, C, ldc);
      };
      if (WG || (!BKM && !p.bias)) with(F());                     // (data gradients)
      else with(T());
    };
    if (GE != GELU_NONE && resid) store_as(F(), T());
    else if (GE != GELU_NONE) store_as(F(), F());
    else if (WG && c_f32) store_as(T(), F());
    else if (c_f32 && resid) store_as(T(), T());
    else if (c_f32) store_as(T(), F());
    else if (resid) store_as(F(), T());
    else store_as(F(), F());
    unit += stride;
    if (unit >= u_end) break;
    cur = ahead;
  }
  __builtin_amdgcn_s_waitcnt(in_flight(0));           // no direct load may land in LDS that is another block's by then
}

template <int FM, bool AK, bool BKM, int GE, bool SUMS = false>
void launch_large_t(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  static const bool configured = [] {
    (void)hipFuncSetAttribute((const void*)bgemm_large_kernel<FM, AK, BKM, false, GE, SUMS>, hipFuncAttributeMaxDynamicSharedMemorySize, large::Sizes<FM>::SMEM);
    (void)hipFuncSetAttribute((const void*)bgemm_large_kernel<FM, AK, BKM, true, GE, SUMS>, hipFuncAttributeMaxDynamicSharedMemorySize, large::Sizes<FM>::SMEM);
    return true;
  }();
  (void)configured;
  constexpr int BM = large::Sizes<FM>::BM;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + large::LBN - 1) / large::LBN;
  const int total = tiles_m * tiles_n * p.splits, per = (total + 7) / 8;
  // A block takes all its tiles.  Two of a data gradient's to a block where each unit gets six or more (the weight
  // gradients on the other stream get their units sooner) are behind: alone 262144 x 1024, K = 512 277 -> 304 us,
  // iterations of bert_large 64 x 512 93.1 -> 93.9 ms, bert_large_stress 256 x 512 393.5 -> 394.5, 192 x 512 292.8 -> 294.4.
  const dim3 grid(8 * (per < 32 ? per : 32)), block(512);
  bool ktail = false;
  for (int i = 0; i < p.splits; ++i) ktail |= (p.kb[i + 1] - p.kb[i]) % large::LBK != 0;
  if (ktail) launch_marked((bgemm_large_kernel<FM, AK, BKM, true, GE, SUMS>), grid, block, large::Sizes<FM>::SMEM, st, t0, t1, p, tiles_n, total, per);
  else launch_marked((bgemm_large_kernel<FM, AK, BKM, false, GE, SUMS>), grid, block, large::Sizes<FM>::SMEM, st, t0, t1, p, tiles_n, total, per);
}

// Requirements: K % 8 == 0 when an operand is k-major (or zeros vouched for behind a k-major A's last column,
// with B m-major); the leading dimension of an m-major operand covers its row count rounded up to 8; GELU with
// both operands k-major; both operands m-major: no bias or residual; row sums with A m-major, shared by
// BM / 64 column tiles (fewer are refused); a reduction in parts with B m-major; parts of more k tiles than the
// loads run ahead (into the block's next unit at most); 2 GB for a tile's rows; N >= 8 with a residual.
template <int FM>
bool launch_large(const GemmDev& p, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  auto up8 = [](int64_t v) { return (v + 7) / 8 * 8; };
  // a chunk of a k-major operand that straddles K is moved whole: allowed only where the caller
  // vouches for zeros behind A's last column while B (m-major) reads zeros from row K on
  if ((p.a_k || p.b_k) && (p.K & 7) && !(p.a_tail_zero && p.a_k && !p.b_k && p.lda >= up8(p.K))) return false;
  if (!p.a_k && p.lda < up8(p.M)) return false;
  if (!p.b_k && p.ldb < up8(p.N)) return false;
  if (p.a_rowsum && (p.a_k || p.N <= (large::Sizes<FM>::BM / 64 - 1) * large::LBN)) return false;
  if (p.splits > 1 && (p.b_k || p.bias || p.resid)) return false;
  if (p.lda >= (1 << 21) || p.ldb >= (1 << 21) || (p.resid && p.N < 8)) return false;
  for (int i = 0; i < p.splits; ++i)
    if (p.kb[i + 1] - p.kb[i] <= large::Sizes<FM>::NB * large::LBK) return false;
  if (p.a_k && p.b_k) {
    if (p.gelu == GELU_ERF && !p.vec) launch_large_t<FM, true, true, GELU_ERF | large::kLibrary>(p, st, t0, t1);
    else if (p.gelu == GELU_TANH && !p.vec) launch_large_t<FM, true, true, GELU_TANH | large::kLibrary>(p, st, t0, t1);
    else if (p.gelu == GELU_ERF) launch_large_t<FM, true, true, GELU_ERF>(p, st, t0, t1);
    else if (p.gelu == GELU_TANH) launch_large_t<FM, true, true, GELU_TANH>(p, st, t0, t1);
    else launch_large_t<FM, true, true, GELU_NONE>(p, st, t0, t1);
  } else {
    if (p.gelu || (!p.a_k && !p.b_k && (p.bias || p.resid))) return false;
    if (p.b_k && p.a_rowsum) launch_large_t<FM, false, true, GELU_NONE, true>(p, st, t0, t1);
    else if (p.b_k) launch_large_t<FM, false, true, GELU_NONE>(p, st, t0, t1);
    else if (p.a_k) launch_large_t<FM, true, false, GELU_NONE>(p, st, t0, t1);
    else launch_large_t<FM, false, false, GELU_NONE>(p, st, t0, t1);
  }
  return true;
}

}  // namespace mk
