// Launchers of the gfx950 kernels the training step is made of.
// All pointers are device pointers; every launcher only enqueues work on `st`.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mk {

enum DType : int { F32 = 0, BF16 = 1 };
enum Gelu : int { GELU_NONE = 0, GELU_ERF = 1, GELU_TANH = 2 };

constexpr int kMaxRowWidth = 1024;  // widest row the row-wise kernels accept (hidden size)

// Launches take events that are bound to a kernel's start or end.  A launch that fails leaves its event where it was,
// and nothing may wait for it: the first such failure on this thread since the last call, or success.
hipError_t marking_error();

inline size_t elt_size(int dtype) { return dtype == BF16 ? 2 : 4; }

// Dropout mask descriptor, passed by value to kernels.  thr == 0: dropout off.
struct DropDesc {
  uint32_t thr = 0;      // an element is kept when its 32-bit word >= thr (thr = round(p * 2^32))
  float scale = 1.f;     // 1 / (1 - p), applied to kept elements
  uint32_t k0 = 0, k1 = 0;  // seed, low and high half
  uint32_t site = 0;     // which tensor of the model (embedding, layer l's projections ...)
  uint32_t step = 0;     // iteration number
};

// Where the samples of a batch of B x L tokens are.  Neither array: sample b fills rows b*L ..
// b*L + L - 1.  lens (device, [B]): of a sample's rows the first lens[b] are real, no query gives the
// others' keys weight.  ends (device, [B]): padding was left out of the rows and sample b has rows
// ends[b-1] .. ends[b] - 1, at least its real ones (lens is given too).  Indices inside a sample
// stay those of the padded batch everywhere (lse, delta, dropout masks).
// ends and lens may point at the entries of a later sample, with first the row that sample begins
// at: then row pointers are those of that row.
struct Rows {
  const int32_t* lens = nullptr;
  const int32_t* ends = nullptr;
  int32_t first = 0;
};

// Rows of a padded batch that are left out: whole blocks of kRowBlock rows of padding, whose
// gradients are zeros.  A kernel that sums over rows in groups (MFMA steps of 16 reduction indices,
// LayerNorm's chunks) then meets the groups of the whole batch, minus groups of zeros, so the sums
// are the same bit for bit.
constexpr int kRowBlock = 16;

struct GemmArgs {
  const void* A; int64_t lda; bool a_kmajor;
  const void* B; int64_t ldb; bool b_kmajor;
  void* C; int64_t ldc; bool c_f32;
  int M, N, K;
  const void* bias = nullptr;      // [N], storage dtype
  const void* resid = nullptr;     // [M, ldr], storage dtype
  int64_t ldr = 0;
  void* gelu_out = nullptr;        // [M, ldc], storage dtype
  int gelu = GELU_NONE;
  float* a_rowsum = nullptr;       // [M] fp32: sum_k A(m,k) (bias gradient of a weight-gradient product)
  // A k-major with K not a multiple of 8: its columns [K, K rounded up to 8) exist (lda covers
  // them) and hold zeros, so a kernel that moves whole 16-byte chunks may read them
  bool a_tail_zero = false;
  // rows the choice of kernel is made from where the choice orders the sums (0: M): a bf16 reduction long
  // enough to be cut in parts, fp32's tiles and ways.  A product issued in row ranges, or with padding left out
  // of its rows, names the whole padded batch here
  int rule_rows = 0;
  // rows of the whole that a product issued in row ranges is a part of (0: M), for choices that order no sum
  int whole_rows = 0;
  // reduction over the rows of a batch with padding left out: the padded row count, and for each of
  // its blocks of kRowBlock rows (and one past the last) how many kept blocks lie before it (host)
  int k_padded = 0;
  const int32_t* k_blocks = nullptr;
  // a weight gradient that other products run beside, on another stream: it may leave compute units to them
  bool beside = false;
  void* workspace = nullptr;       // optional scratch of gemm_workspace_bytes(M, N) for split reductions
  size_t workspace_bytes = 0;
  // optional: events bound to the start of the product's first kernel and to the end of its last (a split product's
  // reduction).  time_stop alone marks the end for another stream that waits for it, so every path has to bind
  // it; together they time the product by its kernels and not by markers around the launch.
  hipEvent_t time_start = nullptr, time_stop = nullptr;
};

// scratch that lets a bf16 product with fp32 output cut its reduction in parts (0: never splits);
// a function of the output shape alone
size_t gemm_workspace_bytes(int M, int N);
// scratch that lets a data-gradient product with a very long reduction and few output tiles (the
// vocabulary-long one of the head: A k-major, B m-major, no epilogue) cut its reduction in parts:
// a function of the column count alone, so that it is a constant of the model
size_t gemm_long_k_workspace_bytes(int N);

// 256 x 256 tiles of an M x N product: the large-tile kernel runs them one per compute unit, 256 at a time
int gemm_large_tiles(int M, int N);

// returns false when the arguments violate the kernel's alignment assumptions
bool gemm(int dtype, const GemmArgs& g, hipStream_t st);

// x_f32: in a bf16 configuration the input rows are fp32 (an unrounded residual sum)
void layernorm_fwd(int dtype, const void* x, bool x_f32, const void* gamma, const void* beta,
                   void* y, int T, int H, float eps, hipStream_t st);
// x = resid + dropout(x) in place, then y = LayerNorm(x) (left out when y is null).  resid: storage
// type; masks and rows as in dropout_apply.  One pass where H is a multiple of 8 (bf16) or 4 (fp32)
// and every pointer 16-byte aligned, else two.
void dropout_layernorm_fwd(int dtype, void* x, bool x_f32, const void* resid, const void* gamma, const void* beta,
                           void* y, int T, int H, float eps, const DropDesc& d, const Rows& rows, int B, int L,
                           hipStream_t st);
// partial: fp32 scratch of partial_rows(T) * 2 * H elements
// dx = LayerNorm backward (+ add when given); dx may alias dy when they have the same type;
// dy_f32 / x_f32: in a bf16 configuration those inputs are fp32
void layernorm_bwd(int dtype, const void* dy, bool dy_f32, const void* x, bool x_f32,
                   const void* gamma, void* dx, const void* add, float* dgamma, float* dbeta,
                   float* partial, int T, int H, float eps, hipStream_t st);
// the two halves of layernorm_bwd: dx and the per-chunk partial sums; then dgamma, dbeta from them
// masked (optional): dx as stored with the dropout mask of d applied, for the branch behind a
// dropped product; in the same pass under the conditions of dropout_layernorm_fwd, else in its own.
struct LnBwdMasked {
  void* masked = nullptr;
  DropDesc d;
  Rows rows;
  int B = 0, L = 0;
};
// done (optional; of gelu_bwd and attention_bwd too): an event for the end of the last kernel, bound to its launch.
// beside: other kernels run at the same time on another stream (as in GemmArgs)
void layernorm_bwd_rows(int dtype, const void* dy, bool dy_f32, const void* x, bool x_f32, const void* gamma, void* dx,
                        const void* add, float* partial, int T, int H, float eps, const LnBwdMasked& extra, hipStream_t st,
                        hipEvent_t done = nullptr, bool beside = false);
// chunk_at (optional, device): T is the padded row count, and chunk_at[c] says which of the partial
// rows belongs to its rows c * kRowBlock .. (-1: left out, they would add zeros)
void layernorm_bwd_reduce(const float* partial, float* dgamma, float* dbeta, const int32_t* chunk_at, int T, int H,
                          hipStream_t st);
int partial_rows(int T);
// layernorm_bwd with the partial sums in a fixed device array of the library (no allocation, no
// workspace argument).  Returns 0, -1 when partial_rows(T) * 2 * H exceeds
// kStaticPartialFloats, -2 when the array's address cannot be obtained.  One array per device,
// shared by every call on that device.
constexpr size_t kStaticPartialFloats = (size_t)2 << 20;   // 8 MiB
int layernorm_bwd_static(int dtype, const void* dy, bool dy_f32, const void* x, bool x_f32, const void* gamma,
                         void* dx, const void* add, float* dgamma, float* dbeta, int T, int H, float eps,
                         hipStream_t st);
void gelu_bwd(int dtype, void* d, const void* pre, int64_t n, int tanh_form, hipStream_t st, hipEvent_t done = nullptr);
// drop: dropout of the probabilities (the
// softmax normaliser counts all of them; ctx = (mask * scale * P) V).
// rule_rows: rows the order of fp32 sums is chosen by (0: B * L), as in GemmArgs
void attention_fwd(int dtype, const void* qkv, void* ctx, float* lse, const Rows& rows, int B, int L, int nh, int d,
                   int causal, const DropDesc& drop, hipStream_t st, int64_t rule_rows = 0);
void attention_bwd(int dtype, const void* qkv, const void* ctx, const void* dctx, const float* lse,
                   float* delta, void* dqkv, const Rows& rows, int B, int L, int nh, int d, int causal,
                   const DropDesc& drop, hipStream_t st, hipEvent_t done = nullptr, int64_t rule_rows = 0);
void softmax_xent(int dtype, void* logits, int64_t ld, const int32_t* labels, float* row_loss,
                  float* loss, int T, int V, int n_valid, hipStream_t st);
// T: rows (B * L, or the real ones when rows.ends is given)
void embed_fwd(int dtype, const int32_t* ids, const void* tok, const void* pos, const void* gamma,
               const void* beta, void* sum_out, void* y, const Rows& rows, int T, int B, int L, int H, float eps, int has_ln,
               hipStream_t st);
void embed_bwd(int dtype, const void* d, const int32_t* ids, const int32_t* order,
               const int32_t* seg, int n_seg, float* dtok, float* dpos, const Rows& rows, int B, int L, int H,
               int max_seq, hipStream_t st);
// dst (storage dtype) = round(src fp32)
void convert_from_f32(int dtype, const float* src, void* dst, int64_t n, hipStream_t st);
void fill_zero(void* p, int64_t bytes, hipStream_t st);

// AdamW over a list of tensors in one launch.  Device-resident tables, one entry per tensor
// (master fp32 values, optional low-precision copy, gradient, first and second moment, element
// count, whether weight decay applies) and one per chunk of kAdamChunk elements (tensor, start).
constexpr int kAdamChunk = 16384;
struct AdamTensor {
  float* master; void* lowp; const float* grad; float* m; float* v; int64_t n; int32_t decay; int32_t pad;
};
struct AdamChunk { int32_t tensor; int32_t pad; int64_t start; };
struct AdamHyper { float lr, beta1, beta2, eps, weight_decay, inv_c1, inv_c2; };   // inv_c = 1 / (1 - beta^t)
void adamw_update(int lowp_dtype, const AdamTensor* tensors, const AdamChunk* chunks, int n_chunks, AdamHyper h,
                  hipStream_t st);
// dst[n] = (resid ? resid[n] : 0) + mask * d.scale * src[n] with the mask of d (element i: word i % 4
// of block i / 4).  dst and src have the storage type, or fp32 when io_f32; resid has the storage
// type; dst may be src.  With rows.ends: element e of row r is the mask's element of that token in
// the padded batch of B x L rows of H (a multiple of 4); else B, L and H are not looked at.
void dropout_apply(int dtype, void* dst, const void* src, bool io_f32, const void* resid, int64_t n, const DropDesc& d,
                   const Rows& rows, int B, int L, int H, hipStream_t st);
// dst fp32 = src (storage dtype)
void convert_to_f32(int dtype, const void* src, float* dst, int64_t n, hipStream_t st);

}  // namespace mk
