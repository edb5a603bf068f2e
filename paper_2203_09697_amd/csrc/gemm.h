// Dense fp32 building blocks used by the interaction block (internal, not part of the C ABI).
#pragma once
#include "common.h"

// What happens to an accumulator value v at (row, col) before it is stored.  Steps run in
// this order; null pointers / zero flags skip a step.  All matrices are [rows, n] row-major.
struct gp_epilogue {
  const float* bias = nullptr;      // v += bias[col]
  const float* add_pre = nullptr;   // v += add_pre[row,col]
  float* save_pre = nullptr;        // save_pre[row,col] = v            (pre-activation)
  int act = 0;                      // 1: v = silu(v); 2: v *= silu'(zsrc[row,col]); 3: see gp_gemm_nt_gate_bwd and gp_gemm_nt_w
  const float* zsrc = nullptr;
  const float* mul = nullptr;       // v *= mul[row,col]
  const float* add_post = nullptr;  // v += add_post[row,col]
  // v *= sum_{k < lr_k} lr_a[row, k] lr_b[k, col]: a factor of rank lr_k <= 16 evaluated in the epilogue (lr_a to 16
  // bits as two bf16 terms, lr_b rounded to bf16, fp32 sum, two matrix-core instructions per 32x32 block) instead of
  // read from an [rows, n] matrix.
  // Takes the place of `mul` in the order of steps; only where gp_gemm_nt_takes_lowrank says so.
  const float* lr_a = nullptr;      // fp32 [rows, lr_k]
  const float* lr_b = nullptr;      // fp32 [lr_k, n]
  int lr_k = 0;
  float scale = 1.0f;               // v *= scale
  float* out = nullptr;             // out[row,col] = v
  float* out2 = nullptr;            // out2[row,col] = v * silu'(z2src[row,col])
  const float* z2src = nullptr;
  // Storage type of the [rows, n] matrices above: a set bit means the pointer addresses bf16
  // elements (2 bytes, round-to-nearest-even on store) instead of fp32; bias is always fp32.
  // Only the bf16-operand GEMM kernels accept a non-zero mask.
  unsigned bf16 = 0;
};
enum : unsigned {
  EPI_BF_ADD_PRE = 1u, EPI_BF_SAVE_PRE = 2u, EPI_BF_ZSRC = 4u, EPI_BF_MUL = 8u, EPI_BF_ADD_POST = 16u,
  EPI_BF_OUT = 32u, EPI_BF_OUT2 = 64u, EPI_BF_Z2SRC = 128u
};

// C = A[M,K] @ B[K,N]
// a_bf16 (bf16-operand kernels only): A addresses bf16 elements instead of fp32
int gp_gemm_nn(gp_ctx* ctx, const float* A, const float* B, int64_t M, int N, int K, const gp_epilogue& epi, int a_bf16 = 0,
               int b_bf16 = 0);
// C = A[M,K] @ Bt[N,K]^T
int gp_gemm_nt(gp_ctx* ctx, const float* A, const float* Bt, int64_t M, int N, int K, const gp_epilogue& epi, int a_bf16 = 0,
               int b_bf16 = 0);
// whether gp_gemm_nt with these shapes and bf16 operands runs in the kernel whose epilogue evaluates lr_a, lr_b
bool gp_gemm_nt_takes_lowrank(const gp_ctx* ctx, int64_t M, int N, int K);
// out = A[M,K] @ Bt[N,K]^T + A2[M,K] @ B2t[N,K]^T (fp32 result, no other epilogue step).  With tall bf16 operands this is
// ONE launch of the global->LDS kernel whose contraction runs over both pairs, so the result is written once instead
// of written, read back and written again; otherwise two launches, the second adding to the first's result.
// out_bf16: the result is stored as bf16 (bf16-operand kernels only).
int gp_gemm_nt2(gp_ctx* ctx, const float* A, const float* Bt, const float* A2, const float* B2t, int64_t M, int N, int K,
                float* out, int a_bf16 = 0, int b_bf16 = 0, int out_bf16 = 0);
// Backward step of a gated activation y = silu(z) gate, gate[e, h] = sum_k f[e, k] Wg[k, h] of rank R <= 16, behind the product that
// gives dy = A Bt^T (bf16 operands, both k-contiguous): dz = dy gate silu'(z) and dgate = dy silu(z); z, dz, dgate bf16 [M, N],
// f, Wg fp32.  dy is not stored.
int gp_gemm_nt_gate_bwd(gp_ctx* ctx, const float* A, const float* Bt, int64_t M, int N, int K, const __bf16* z, const float* f,
                        const float* Wg, int R, __bf16* dz, __bf16* dgate);
// out[M,N] = A[rows,M]^T @ B[rows,N]; deterministic two-stage reduction through `part`.
// If colsum_out != NULL it also receives colsum_out[n] = sum_r B[r,n] (the bias gradient).
size_t gp_gemm_tn_scratch(int64_t rows, int M, int N);
int gp_gemm_tn(gp_ctx* ctx, const float* A, const float* B, int64_t rows, int M, int N, float* out,
               float* colsum_out, float* part, size_t part_bytes, int a_bf16 = 0, int b_bf16 = 0);
// out[n] = sum_r X[r,n]
size_t gp_colsum_scratch(int64_t rows, int N);
int gp_colsum(gp_ctx* ctx, const float* X, int64_t rows, int N, float* out, float* part, size_t part_bytes);

// elementwise helpers, n elements
int gp_ew_dsilu_mul(gp_ctx* ctx, const float* g, const float* z, float* out, int64_t n);   // out = g * silu'(z)
int gp_ew_gate_bwd(gp_ctx* ctx, const float* dxg, const float* z, const float* gate, float* dz, float* dgate,
                   int64_t n);   // dz = dxg*gate*silu'(z), dgate = dxg*silu(z)
int gp_ew_add3(gp_ctx* ctx, const float* a, const float* b, const float* c, float* out, int64_t n);  // c may be NULL
// bf16-operand kernels (gemm_bf16.hip); mode 0 NN, 1 NT, 2 TN; args is the fp32 path's argument block
int gp_gemm_bf16_launch(gp_ctx* ctx, int mode, void* args, int splits);
int gp_gemm_bf16_gate_launch(gp_ctx* ctx, void* args);
// fp32 operands and result on the bf16 matrix cores, each operand as three bf16 planes (gemm_bf16.hip); mode 0 NN, 1 NT
int gp_gemm_split_launch(gp_ctx* ctx, int mode, void* args, int splits);
// A^T B with both operands bf16 through global->LDS loads and LDS transpose reads: number of splits of its plan (0: the
// shape is not taken) and a bound on it that is no smaller for more rows, whether the filled argument block qualifies, launch
int gp_gemm_bf16_tn_dl_splits(int64_t rows, int M, int N);
int gp_gemm_bf16_tn_dl_most(int64_t rows, int M, int N);
bool gp_gemm_bf16_tn_dl_ok(const void* args);
int gp_gemm_bf16_tn_dl(gp_ctx* ctx, void* args, int splits);
// While alive, GEMMs issued on the context round their operands to bf16 if `on`.
struct gp_bf16_scope {
  gp_ctx* c;
  bool prev;
  gp_bf16_scope(gp_ctx* ctx, bool on) : c(ctx), prev(ctx->gemm_bf16) { c->gemm_bf16 = on; }
  ~gp_bf16_scope() { c->gemm_bf16 = prev; }
};
// out[i] = sum_z part[z*n + i], z < splits
int gp_reduce_parts(gp_ctx* ctx, const float* part, int splits, int64_t n, float* out);
// the same of two arrays (of either none where its n is 0)
int gp_reduce_parts2(gp_ctx* ctx, const float* part, int splits, int64_t n, float* out, const float* part2, int64_t n2, float* out2);
// Gradients of the two factors of W = W1 W2, [R, B] and [B, H], from that of W: dW1 = dW W2^T, dW2 = W1^T dW
int gp_factor_grads(gp_ctx* ctx, const float* dW, const float* W1, const float* W2, int R, int B, int H, float* dW1, float* dW2);

// ---- fp32 products A W and A W^T with fp32 operands as two fp16 numbers each; the weights are converted ahead (gemm_planes.hip)
constexpr int GP_PLANE_JOBS_MAX = 24;
struct gp_plane_job {
  const float* src;
  void* dst;      // gp_planes_bytes(N, K)
  int N, K;       // columns and contraction length of the product
  int k_rows;     // src is [K, N] (A W), else [N, K] (A W^T)
};
size_t gp_planes_bytes(int N, int K);
// whether a product of this shape is better off in that form (M rows of A)
bool gp_planes_take(const gp_ctx* ctx, int64_t M, int N, int K);

// The weights of a call, converted by one launch.
struct gp_weight_planes {
  gp_ctx* ctx;
  char* next;     // room for the planes: gp_planes_bytes of every matrix added, each rounded up to 256 (NULL: no planes)
  gp_plane_job jobs[GP_PLANE_JOBS_MAX];
  int n = 0;
  gp_weight_planes(gp_ctx* c, void* room) : ctx(c), next(static_cast<char*>(room)) {}
  // planes of W for products with M rows (NULL where the general kernels take them, as they do where the room is not 16-byte aligned)
  const void* add(const float* W, int64_t M, int N, int K, int k_rows) {
    if (!next || n == GP_PLANE_JOBS_MAX || ((uintptr_t)next & 15) != 0 || !gp_planes_take(ctx, M, N, K)) return nullptr;
    jobs[n++] = gp_plane_job{W, next, N, K, k_rows};
    void* p = next;
    next += gp_align(gp_planes_bytes(N, K));
    return p;
  }
  int run();
};
// gp_gemm_nn / gp_gemm_nt with the planes of the weight matrix at hand (NULL: the general kernels)
int gp_gemm_nn_w(gp_ctx* ctx, const float* A, const float* W, const void* planes, int64_t M, int N, int K, const gp_epilogue& epi);
// gp_gemm_nt_w also takes act = 3, the backward step of y = silu(z) gate behind the product dy: out = dy mul silu'(zsrc) and
// out2 = dy silu(zsrc), with mul the gate; only with planes at hand and every matrix 16-byte aligned, which the caller looks at.
int gp_gemm_nt_w(gp_ctx* ctx, const float* A, const float* W, const void* planes, int64_t M, int N, int K, const gp_epilogue& epi);
// A^T B over the rows with three bf16 parts per value (gemm_planes.hip): tiles and splits of the rows of one product, the splits that
// products of 128 x 128 tiles share, launch of several products with the same rows and tile shape
constexpr int GP_TN_JOBS_MAX = 24;
struct gp_tn_part_job {
  const float *A, *B;        // [rows, M], [rows, N]
  float *part, *colsum_part; // [splits, M, N]; [splits * tiles_m, N] or NULL
  int M, N, vec, first;      // vec: 16-byte stores to part are legal; first: set by the launch
};
struct gp_tn_parts_plan {
  bool big;       // 256 x 256 tiles instead of 128 x 128
  int tiles_m, splits, most;   // most: no smaller for more rows, and at least `splits`
  int64_t per;    // rows of a split
};
gp_tn_parts_plan gp_parts_tn_plan(int64_t rows, int M, int N);
int gp_parts_tn_splits(int64_t rows, int64_t tiles);
int gp_parts_tn_launch(gp_ctx* ctx, bool big, const gp_tn_part_job* jobs, int n, int64_t rows, int64_t per, int splits);

// Several A^T B over the same rows (the weight gradients of a block), fp32 operands.  Alone, a product of 256 x 256 is cut into 128
// runs of the rows to fill the chip, whose partial sums are as many bytes as its operands; together a few runs are enough, and small graphs need
// two launches for all of them.  Products of 256 x 256 tiles and those of the other forms are run one by one.
struct gp_tn_product {
  const float *A, *B;   // [rows, M], [rows, N]
  int M, N;
  float *out, *colsum;  // [M, N]; colsum (or NULL): column sums of B
};
// part for any of the products, in one or several calls; no smaller for more rows
size_t gp_gemm_tn_group_scratch(int64_t rows, const gp_tn_product* p, int n);
int gp_gemm_tn_group(gp_ctx* ctx, const gp_tn_product* p, int n, int64_t rows, float* part, size_t part_bytes);

// ---- chains of dense layers over the rows in one launch (dense_chain.hip), fp32, all pointers 16-byte aligned
constexpr int GP_CHAIN_MAX = 24;
struct gp_chain_step {
  const float* W = nullptr;         // [K, N] (k_rows) or [N, K]
  int N = 0, K = 0, k_rows = 0;     // multiples of 16, at most the width H of the chain
  // operand x [rows, K]: the value of the step before, or load, then times silu'(load_z) and stored to load_out where those are given
  const float *load = nullptr, *load_z = nullptr;
  float* load_out = nullptr;
  // v = x W; in this order, NULL pointers skip a step
  const float* bias = nullptr;      // v += bias[col]
  const float* add_pre = nullptr;   // v += add_pre
  float* save_pre = nullptr;        // save_pre = v
  int act = 0;                      // v = silu(v)
  // gate: out2 = v mul silu'(z), out3 = v silu(z), v = out2; in place of what follows
  int gate = 0;
  const float* mul = nullptr;       // v *= mul
  const float* add = nullptr;       // v += add
  float* out = nullptr;             // out = v
  const float* z = nullptr;         // v *= silu'(z), out2 = v
  float *out2 = nullptr, *out3 = nullptr;
  int keep = 0;                     // the next step takes this one's operand, not its value
};
// whether there is a chain for layers of width H that meet widths F (multiple of 16)
bool gp_chain_takes(int H, int F);
// room for the weights of a step
size_t gp_chain_parts_bytes(int H, int N, int K);
// converts the weights of all steps; then runs of consecutive steps, each beginning with a load
int gp_chain_prepare(gp_ctx* ctx, int H, const gp_chain_step* steps, int n, void* parts, size_t parts_bytes);
int gp_chain_run(gp_ctx* ctx, int H, const gp_chain_step* steps, int from, int to, int64_t rows, const void* parts);
