// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

namespace mllm {

struct GemmArgs {
  const void* a;
  const void* b;
  void* c;
  int64_t m, n, k;
  int64_t lda, ldb, ldc;   // leading dimensions (elements) of the matrices as stored
  int a_layout;            // 0: A stored [M,K]; 1: A stored [K,M]
  int b_layout;            // 0: B stored [K,N]; 1: B stored [N,K]
  int out_fp32;            // 0: bf16 C; 1: fp32 C
  int accumulate;          // fp32 C only: C += product
  const void* bias;        // bf16 [N] or null
  const void* residual;    // bf16 [M,N] (ld = ldres) or null; bf16 C only
  int64_t ldres;
  void* splitk_ws;         // optional fp32 scratch for split-K partial products (null: never split)
  size_t splitk_ws_bytes;
  // SwiGLU fused into the product's epilogue: C = [gate | up] is [M, N] bf16 as usual and
  // swiglu_act [M, N/2] bf16 also receives silu(gate) * up.  Only where gemm_swiglu_fusable().
  void* swiglu_act = nullptr;
  // SwiGLU's gradient fused into the epilogue of dA = dY.W_d^T ([M, N], N = f): with
  // swiglu_pre = [gate | up] ([M, 2N] bf16) the product itself is not stored; swiglu_dpre
  // ([M, 2N] bf16) receives [d gate | d up].  C is unused.  Only where gemm_swiglu_bwd_fusable().
  const void* swiglu_pre = nullptr;
  void* swiglu_dpre = nullptr;
  // Rotary positions fused into the epilogue of a forward product Y = X.W (+ bias): the leading
  // rope_cols columns of Y are heads of rope_head_dim (64 or 128) whose half-split pairs are rotated,
  // on the fp32 accumulators, by the angles of row rope_pos[row] of rope_table (launch_rope_table).
  // Only where gemm_rope_fusable().
  const float* rope_table = nullptr;
  const int32_t* rope_pos = nullptr;   // device int32 [M]
  int64_t rope_cols = 0;
  int32_t rope_head_dim = 0;
};
// Whether launch_gemm can rotate the q and k columns of a forward product in its epilogue (large-tile
// kernel, K a multiple of 64, heads of 64 or 128: a wavefront owns 128 columns, 64 in the form on eight wavefronts, which
// therefore leaves heads of 128 to the other).
bool gemm_rope_fusable(int64_t m, int64_t n, int64_t k, int32_t head_dim);
bool gemm_swiglu_bwd_fusable(int64_t m, int64_t n, int64_t k);
// Whether launch_gemm can write the SwiGLU activation of a forward product X[M,K].W[K,N] along
// with it (large-tile kernel, N/2 a multiple of 128, K a multiple of 64).
bool gemm_swiglu_fusable(int64_t m, int64_t n, int64_t k);
// A and B are addressed through 32-bit byte offsets: each operand must stay below this size.
constexpr int64_t GEMM_MAX_OPERAND_BYTES = 0xFFFFFFF0ll - 16;
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);
// What launch_gemm runs for a product: output tile (256, 224 or 192 x 256, 128 x 128, 64 x 64; 0 x 0: the general kernel) and parts
// of the K loop.
struct GemmForm { int tile_rows, tile_cols, k_parts; };
GemmForm gemm_form(const GemmArgs& g);
// Both gradients of a linear map Y [t, n] = X [t, k] . W [k, n] in one launch: x the arguments of dX = dY . W^T (or of its SwiGLU form), w
// those of dW (+)= X^T . dY.  Both name the same scratch.  Where that does not pay, on operands that the tile kernel does not
// take and on those that do not start on 16 bytes, two launches.
hipError_t launch_linear_bwd(const GemmArgs& x, const GemmArgs& w, hipStream_t s);
struct LinearBwdForm { bool paired; GemmForm x, w; bool x_first; };
LinearBwdForm linear_bwd_form(const GemmArgs& x, const GemmArgs& w);
size_t linear_bwd_ws_bytes(int64_t t, int64_t k, int64_t n, bool swiglu);   // scratch that launch_linear_bwd wants
// Scratch bytes launch_gemm wants for a product of this shape (0: it will not split the K loop); a_t: A stored
// [K, M]; b_t: B stored [K, N].
size_t gemm_splitk_ws_bytes(int64_t m, int64_t n, int64_t k, bool a_t, bool b_t);
// C [M, N] (+)= sum over p of partial[p], p ascending, (+ bias) (+ residual); fp32 or bf16, N a multiple of 8.
hipError_t launch_splitk_reduce(const float* partial, void* c, int splits, int64_t m, int64_t n, int out_fp32,
                                int accumulate, const void* bias, const void* residual, int64_t ldres, hipStream_t s);

// One workgroup of an attention kernel: a tile of a segment and a head (query head for the forward
// and dQ passes, kv head for the dK/dV pass).  The lists are built on the host (attn_items.h).
struct AttnItem {
  int32_t seg_start;  // first packed row of the segment
  int32_t seg_len;
  int32_t tile0;      // first row of the tile inside the segment
  int32_t causal;
  int32_t head;
};
// Whether two ranges of memory share a byte (empty or absent ones share none).
inline bool ranges_overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes) {
  return a && b && a_bytes > 0 && b_bytes > 0 && (uintptr_t)a < (uintptr_t)b + (uintptr_t)b_bytes && (uintptr_t)b < (uintptr_t)a + (uintptr_t)a_bytes;
}
struct AttnArgs {
  const void* q; const void* k; const void* v; void* o; float* lse;
  const void* d_o; void* dq; void* dk; void* dv; float* delta;
  int64_t q_stride, kv_stride, o_stride;   // row strides in elements (dq/dk/dv/do share them)
  int32_t total_tokens, n_q_heads, n_kv_heads, head_dim;
  const void* q_list; int32_t q_grid;      // device work list of the forward / dQ passes and its grid size
  const void* kv_list; int32_t kv_grid;    // device work list of the dK/dV pass and its grid size
  // backward only: when set (launch_rope_table, head_dim floats per position, positions counted from
  // the start of each segment), dq and dk leave rotated by the negative rotary angle of their row,
  // i.e. as gradients of the q and k that entered the rotation
  const float* rope_table;
  // backward only: the dK/dV pass in kv_parts parts per key tile (attn_kv_parts; 0 or 1: undivided), their sums in
  // dkv_partial, fp32 [kv_parts][2][total_tokens][n_kv_heads * head_dim]; pos: device int32, every row's
  // position in its segment (needed with a rope_table)
  int32_t kv_parts; float* dkv_partial; const int32_t* pos;
  double fwd_flops;                               // algorithmic forward FLOPs of this call (for timing reports)
};
constexpr int ATTN_FWD_Q_TILE = 128;   // query rows per workgroup, forward and dQ pass
constexpr int ATTN_BWD_KV_TILE = 128;  // key rows per workgroup, dK/dV pass
// In how many parts the dK/dV pass should walk its key tiles.  A workgroup owns a (key tile, kv head) and meets
// every query tile of every query head of the group one after the other, so with few kv heads and few
// tokens most CUs have no workgroup while the heaviest one sets the time (28 / 4 heads, 2999 tokens: 100
// workgroups, 370 us).  heaviest, total: the largest and the summed number of 64-row query tiles that the
// (key tile, kv head) items meet; rows: rows of the k matrix times kv heads.  Constants (microseconds) measured on the kernels
// before the present ones and not fitted again: a query tile 2.2 at head_dim 128 (the present kernel 1.8 with every CU busy, 13255
// causal tokens), 1.1 at 64; the parts' sums go through memory at 4 TB/s and cost a launch.
int attn_kv_parts(int64_t heaviest, int64_t total, int64_t rows, int head_dim);
hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t s);
hipError_t launch_attn_bwd(const AttnArgs& a, hipStream_t s);

// kind 0 LayerNorm, 1 RMSNorm.  stats: [2][T] fp32 (rstd, mean).  ld = elements between rows of
// every [t, d] operand (d for dense matrices; more when they are column slices of a wider one).
hipError_t launch_norm_fwd(int kind, const void* x, const void* gamma, const void* beta, void* y,
                           float* stats, int64_t t, int64_t d, int64_t ld, float eps, hipStream_t s,
                           void* x_copy = nullptr);   // x_copy: also receives x (same layout)
// Sums over the tokens (norm and bias gradients) in two stages.  A kernel that forms partial sums takes room for
// them here, [rows][n] fp32 for each of `outs` one after the other (a NULL in it: that set is not reduced), and flush()
// adds up everything taken so far in one launch: out[c] (+)= sum over rows.  A stage's backward pass
// flushes when the scratch or the list is full and at its end, where each sum had a launch of its own before
// (launches of 2-5 us and the gaps in front of them; a stage of three small layers, two
// microbatches: 681 -> 646 us; one 576-token image through the ViT-L layer: 270 -> 263 us).
// take() flushes first when an output already waits in the list, so that two layers may share a gradient.
struct PartialSums {
  static constexpr int MAX_JOBS = 32;
  struct Job { const float* partial; float* out; int rows; int64_t n; };
  PartialSums(float* scratch, size_t bytes, int accumulate_) : base(scratch), capacity(bytes / 4), accumulate(accumulate_) {}
  hipError_t take(int64_t rows, int64_t n, std::initializer_list<float*> outs, hipStream_t s, float** partial);
  hipError_t flush(hipStream_t s);
  float* base;
  size_t capacity, used = 0;   // floats
  int accumulate, count = 0;
  Job jobs[MAX_JOBS];
};
int64_t norm_bwd_partial_rows(int64_t t);                // an upper bound of
int64_t norm_bwd_workgroups(int64_t t, int64_t d);       // the rows of partial sums that launch_norm_bwd takes
inline int norm_bwd_sets(int kind, bool dx_colsum) { return dx_colsum ? 3 : kind == 0 ? 2 : 1; }
hipError_t launch_norm_bwd(int kind, const void* dy, const void* x, const void* gamma,
                           const float* stats, const void* dres, void* dx, float* dgamma,
                           float* dbeta, PartialSums& sums, int64_t t, int64_t d,
                           int64_t ld, hipStream_t s, float* dx_colsum = nullptr);
// dx_colsum (optional, fp32 [d]): the column sums of dx, formed in the same pass; only for rows of at
// most 1024 elements (norm_bwd_colsum_fusable).  There are then three sets of partial sums.
bool norm_bwd_colsum_fusable(int64_t d);
hipError_t launch_rope(void* qk, const int32_t* pos, int64_t t, int64_t row_stride, int64_t col0,
                       int32_t n_heads, int32_t head_dim, float rope_base, int inverse,
                       hipStream_t s);
// The forward rotation of the leading n_heads heads, with the factors of launch_rope_table.
hipError_t launch_rope_from_table(void* qk, const int32_t* pos, const float* table, int64_t t, int64_t row_stride,
                                  int32_t n_heads, int32_t head_dim, hipStream_t s);
// What a stage's pass begins with, in one launch: the call's metadata from pinned host memory (its device address), the tables
// of the rotary angles, and a copy of rows that depends on nothing (all but the tables may be absent).
struct RopeTableSpec { float* table; int32_t head_dim; float base; };
constexpr int BEGIN_TABLES = 4;
hipError_t launch_begin(const void* meta_src, void* meta, size_t meta_bytes, const RopeTableSpec* tables, int n_tables, int64_t n_pos,
                        const void* copy_src, void* copy_dst, size_t copy_bytes, hipStream_t s);
// table [n_pos, head_dim] fp32: cos then sin of pos * rope_base^(-2i/head_dim), i < head_dim / 2.
hipError_t launch_rope_table(float* table, int64_t n_pos, int32_t head_dim, float rope_base, hipStream_t s);
hipError_t launch_act_fwd(int act, const void* pre, void* a, int64_t t, int64_t f, hipStream_t s);
hipError_t launch_act_bwd(int act, const void* da, const void* pre, void* dpre, int64_t t,
                          int64_t f, hipStream_t s);
// GELU backward that also leaves the column sums of dpre (the gradient of the bias in front of the
// activation) in colsum [f] fp32, by way of colsum_partial_rows(t) rows of partial sums.
hipError_t launch_gelu_bwd_colsum(int act, const void* da, const void* pre, void* dpre, float* colsum,
                                  PartialSums& sums, int64_t t, int64_t f, hipStream_t s);
int64_t colsum_partial_rows(int64_t t);
hipError_t launch_colsum(const void* x, int64_t ldx, float* out, PartialSums& sums, int64_t t, int64_t n, hipStream_t s);
// dst[rows[i], :] = src[i, :] (scatter) or dst[i, :] = src[rows[i], :] (gather); bf16 rows of d.
hipError_t launch_scatter_rows(const void* src, void* dst, const int32_t* rows, int64_t n_rows,
                               int64_t d, int gather, hipStream_t s);
// dst[j, :] = mean of src[first[j] .. first[j] + count[j]) (bf16 rows of d, fp32 sum).
hipError_t launch_pool_rows(const void* src, void* dst, const int32_t* first, const int32_t* count,
                            int64_t n_out, int64_t d, hipStream_t s);
// dst[i, :] = src[window[i], :] / count[window[i]]: the gradient of launch_pool_rows.
hipError_t launch_unpool_rows(const void* src, void* dst, const int32_t* window, const int32_t* count,
                              int64_t n_rows, int64_t d, hipStream_t s);
// Gradient of the scattered connector rows: dproj[j] = dy[rows[j]], and dx_seq = dy with those rows zero.  scattered: a bit for
// every row of dy.  dx_seq may be dy.
hipError_t launch_connector_grad(const void* dy, void* dproj, void* dx_seq, const int32_t* rows, const uint32_t* scattered, int64_t n_rows,
                                 int64_t n_seq, int64_t d, hipStream_t s);
hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s);

// Optional per-launch timing with HIP events on the launch stream (off by default).  Classes:
enum ProfClass { PROF_GEMM_FWD = 0, PROF_GEMM_DX = 1, PROF_GEMM_DW = 2, PROF_ATTN_FWD = 3,
                 PROF_ATTN_BWD = 4, PROF_ELEMENTWISE = 5, PROF_GEMM_SMALL = 6, PROF_GEMM_ROWS192 = 7,
                 PROF_N_CLASSES = 8 };
struct ProfScope {   // records a start event now and a stop event when it goes out of scope
  ProfScope(int cls, double work, hipStream_t s);
  ~ProfScope();
  int slot;
  hipStream_t stream;
};

}  // namespace mllm
