// Output block (paper Sec. 3.3: the updated messages are summed per target atom, EdgeAggr, and
// the sum is transformed by an MLP, NodeUpdate), forward and backward.
//
//   t_e = m_e * (rbf_e W_rbf)                       [E, emb]   radial weighting (not stored where there are at most 16 functions)
//   h_i = sum_{e: dst[e] = i} t_e                   [N, emb]   in-edges of an atom are contiguous rows
//   u   = h W_up;  u = act(u W_k + b_k), k < L      [N, out]
//   P_i = u_i . w_final;  energy[g] (+)= sum_{i in g} P_i
//
// Backward of sum_g grad_energy[g] energy[g]: the node MLP in reverse (N rows: small GEMMs), then
// per edge  dt_e = dh[dst[e]],  grad_m_e (+)= dt_e * (rbf_e W_rbf)  (the gate is recomputed by the
// same GEMM, not stored),  grad_W_rbf = rbf^T (dt * m).  No atomics: every sum follows sorted order.
#include <stdarg.h>

#include <algorithm>
#include <type_traits>

#include "gemm.h"

namespace {

constexpr int WPB = 4;

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }
inline unsigned wblk(int64_t n) { return (unsigned)((n + WPB - 1) / WPB); }

// h[i, f] = sum over the in-edge rows of atom i of t[e, f]; one wavefront per (atom, 64 features)
__global__ void __launch_bounds__(256)
out_atom_sum_kernel(const float* __restrict__ t, const int32_t* __restrict__ row_ptr, int64_t n_atoms, int H,
                    float* __restrict__ h) {
  const int chunks = (H + 63) / 64;
  const int64_t w = (int64_t)blockIdx.x * WPB + (threadIdx.x >> 6);
  const int64_t i = w / chunks;
  if (i >= n_atoms) return;
  const int f = (int)(w % chunks) * 64 + (threadIdx.x & 63);
  if (f >= H) return;
  const int e0 = row_ptr[i], e1 = row_ptr[i + 1];
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  int e = e0;
  for (; e + 3 < e1; e += 4) {
    s0 += t[(int64_t)e * H + f];
    s1 += t[(int64_t)(e + 1) * H + f];
    s2 += t[(int64_t)(e + 2) * H + f];
    s3 += t[(int64_t)(e + 3) * H + f];
  }
  for (; e < e1; ++e) s0 += t[(int64_t)e * H + f];
  h[i * H + f] = (s0 + s1) + (s2 + s3);
}

// Few radial functions (R <= RADIAL_MAX): the gate's column of W_rbf fits a lane's registers, and the edges' passes of the output block are one
// kernel each that reads every row once.  As a product with K = R, a pass that gathers, one that multiplies and A^T B: 26 us forward
// and 54 backward at 13230 edges x 256 x 6, so 20 and 23.  The gate is summed in fp64 in two chains, 5 us forward: in fp32 sums over five
// edges have 10 (6 functions) to 39 per cent (16) more error than with the product (6.0e-8), so 10 less, and the gradient of the messages 1 to 3.
constexpr int RADIAL_MAX = 16;
template <int RM>
struct gate_column {
  double w[RM];
  __device__ __forceinline__ void load(const float* __restrict__ W, int R, int H, int f) {
#pragma unroll
    for (int r = 0; r < RM; ++r) w[r] = r < R ? (double)W[(int64_t)r * H + f] : 0.0;
  }
  // value r of the R >= 1 of an edge (uniform in the wavefront), 0 beyond them: an infinite value stays its own column's.  Loaded either way, so
  // that the loads of an edge are issued together instead of a branch for each.
  static __device__ __forceinline__ float value(const float* __restrict__ rbf, int r, int R) {
    const float x = rbf[r < R ? r : 0];
    return r < R ? x : 0.f;
  }
  __device__ __forceinline__ float at(const float* __restrict__ rbf, int R) const {
    double g[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < RM; ++r) g[r & 1] = __builtin_fma((double)value(rbf, r, R), w[r], g[r & 1]);
    return (float)(g[0] + g[1]);
  }
};

// h[i, f] = sum over the in-edges e of atom i of m[e, f] (rbf_e W)[f]; one wavefront per (atom, 64 features)
template <int RM>
__global__ void __launch_bounds__(256)
out_edge_sum_kernel(const float* __restrict__ m, const float* __restrict__ rbf, const float* __restrict__ W, const int32_t* __restrict__ row_ptr,
                    int64_t n_atoms, int H, int R, float* __restrict__ h) {
  const int chunks = (H + 63) / 64;
  const int64_t w = (int64_t)blockIdx.x * WPB + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = w / chunks;
  if (i >= n_atoms) return;
  const int f = (int)(w % chunks) * 64 + (threadIdx.x & 63);
  if (f >= H) return;
  gate_column<RM> col;
  col.load(W, R, H, f);
  const int e0 = row_ptr[i], e1 = row_ptr[i + 1];
  constexpr int U = 4;   // edges at a time, each with a sum of its own
  float s[U];
#pragma unroll
  for (int u = 0; u < U; ++u) s[u] = 0.f;
  int e = e0;
  for (; e + U - 1 < e1; e += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = m[(int64_t)(e + u) * H + f];
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = __builtin_fmaf(v[u], col.at(rbf + (int64_t)(e + u) * R, R), s[u]);
  }
  for (; e < e1; ++e) s[0] = __builtin_fmaf(m[(int64_t)e * H + f], col.at(rbf + (int64_t)e * R, R), s[0]);
  h[i * H + f] = (s[0] + s[1]) + (s[2] + s[3]);
}

// grad_m[e, f] (+)= dh[dst[e], f] (rbf_e W)[f] and, with part, the sums of rbf[e, r] dh[dst[e], f] m[e, f] over a run of `per` edges; one
// wavefront per (run, 64 features)
template <int RM>
__global__ void __launch_bounds__(256)
out_edge_grad_kernel(const float* __restrict__ m, const float* __restrict__ rbf, const float* __restrict__ W, const float* __restrict__ dh,
                     const int32_t* __restrict__ dst, int64_t n_edges, int64_t per, int H, int R, int accumulate, float* __restrict__ grad_m,
                     float* __restrict__ part) {
  const int chunks = (H + 63) / 64;
  const int64_t w = (int64_t)blockIdx.x * WPB + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t run = w / chunks, e0 = run * per, e1 = e0 + per < n_edges ? e0 + per : n_edges;
  if (e0 >= n_edges) return;
  const int f = (int)(w % chunks) * 64 + (threadIdx.x & 63);
  if (f >= H) return;
  gate_column<RM> col;
  col.load(W, R, H, f);
  float dw[RM];
#pragma unroll
  for (int r = 0; r < RM; ++r) dw[r] = 0.f;
  auto edges = [&](auto count, int64_t e) __attribute__((always_inline)) {
    constexpr int U = decltype(count)::value;
    float d[U], v[U], g0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      d[u] = dh[(int64_t)dst[e + u] * H + f];
      v[u] = part ? m[(e + u) * H + f] : 0.f;
      g0[u] = accumulate ? grad_m[(e + u) * H + f] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float* q = rbf + (e + u) * R;
      grad_m[(e + u) * H + f] = __builtin_fmaf(d[u], col.at(q, R), g0[u]);
      const float dg = d[u] * v[u];
#pragma unroll
      for (int r = 0; r < RM; ++r) dw[r] = __builtin_fmaf(col.value(q, r, R), dg, dw[r]);
    }
  };
  int64_t e = e0;
  for (; e + 3 < e1; e += 4) edges(std::integral_constant<int, 4>(), e);
  for (; e < e1; ++e) edges(std::integral_constant<int, 1>(), e);
  if (part) {
#pragma unroll
    for (int r = 0; r < RM; ++r)
      if (r < R) part[(run * R + r) * H + f] = dw[r];
  }
}
// runs of the edges: of 32, at most 1024
int64_t edge_runs_most(int64_t E) { return std::min<int64_t>((E + 31) / 32, 1024); }

// p[i] = u[i, :] . w; one wavefront per atom
__global__ void __launch_bounds__(256)
out_atom_dot_kernel(const float* __restrict__ u, const float* __restrict__ w, int64_t n_atoms, int K,
                    float* __restrict__ p) {
  const int64_t i = (int64_t)blockIdx.x * WPB + (threadIdx.x >> 6);
  if (i >= n_atoms) return;
  float s = 0.f;
  for (int k = threadIdx.x & 63; k < K; k += 64) s += u[i * K + k] * w[k];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) p[i] = s;
}

// energy[g] (+)= sum of p over the atoms of structure g (fixed order); one wavefront per structure
__global__ void __launch_bounds__(256)
out_graph_sum_kernel(const float* __restrict__ p, const int32_t* __restrict__ graph_ptr, int n_graphs, int accumulate,
                     float* __restrict__ energy) {
  const int g = blockIdx.x * WPB + (threadIdx.x >> 6);
  if (g >= n_graphs) return;
  float s = 0.f;
  for (int i = graph_ptr[g] + (threadIdx.x & 63); i < graph_ptr[g + 1]; i += 64) s += p[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) energy[g] = accumulate ? energy[g] + s : s;
}

// ga[i] = grad_energy[structure of atom i];  du[i, k] = ga[i] w[k] silu'(z[i, k]) (z NULL: without it); a wavefront per atom, which
// looks its structure up (one per structure walked its atoms one after the other: 52 us at 62 atoms each, 4 us so)
__global__ void __launch_bounds__(256)
out_seed_kernel(const float* __restrict__ grad_energy, const int32_t* __restrict__ graph_ptr, int n_graphs, int64_t n_atoms,
                const float* __restrict__ w, const float* __restrict__ z, int K, float* __restrict__ ga, float* __restrict__ du) {
  const int64_t i = (int64_t)blockIdx.x * WPB + (threadIdx.x >> 6);
  if (i >= n_atoms) return;
  int lo = 0, hi = n_graphs;   // graph_ptr[lo] <= i < graph_ptr[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (graph_ptr[mid] <= i) lo = mid;
    else hi = mid;
  }
  const float ge = grad_energy[lo];
  if ((threadIdx.x & 63) == 0) ga[i] = ge;
  for (int k = threadIdx.x & 63; k < K; k += 64) {
    const float v = ge * w[k];
    du[i * K + k] = z ? v * dsilu_f(z[i * K + k]) : v;
  }
}

// dt[e, :] = dh[dst[e], :]
__global__ void out_gather_rows_kernel(const float* __restrict__ dh, const int32_t* __restrict__ dst, int64_t n_edges,
                                       int H, float* __restrict__ dt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_edges * H) return;
  dt[i] = dh[(int64_t)dst[i / H] * H + (i % H)];
}

// a[i] *= b[i]
__global__ void out_mul_inplace_kernel(float* __restrict__ a, const float* __restrict__ b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] *= b[i];
}

__global__ void out_zero_kernel(float* __restrict__ a, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0.f;
}

struct out_saved {
  float *h, *u0;
  float *z[GP_MAX_OUT_LAYERS], *u[GP_MAX_OUT_LAYERS];
};
size_t carve_out_saved(void* p, int64_t N, int H, int D, int L, out_saved* s) {
  gp_carver c(p);
  s->h = c.take<float>(N * H);
  s->u0 = c.take<float>(N * D);
  for (int k = 0; k < L; ++k) {
    s->z[k] = c.take<float>(N * D);
    s->u[k] = c.take<float>(N * D);
  }
  return c.off;
}
struct out_scratch {
  float *tE;          // [E, H]: t in the forward pass, dt (then dt * m) in the backward pass (only with more than RADIAL_MAX functions)
  float *p, *ga;      // [N]
  float* du[GP_MAX_OUT_LAYERS + 1];   // [N, D] each: the gradients between the layers, which their weight gradients wait for together
  float *dh;          // [N, H]
  float* part;
  size_t part_bytes;
  void* planes;       // the weights of a call as operand planes (gemm_planes.hip)
};
size_t carve_out_scratch(void* p, int64_t N, int64_t E, int H, int D, int R, int L, out_scratch* s) {
  gp_carver c(p);
  s->tE = R > RADIAL_MAX ? c.take<float>(E * H) : nullptr;
  s->p = c.take<float>(N);
  s->ga = c.take<float>(N);
  for (int k = 0; k <= L; ++k) s->du[k] = c.take<float>(N * D);
  s->dh = c.take<float>(N * H);
  size_t m = gp_gemm_tn_scratch(E, R, H);
  if (R <= RADIAL_MAX) m = std::max(m, (size_t)edge_runs_most(E) * R * H * sizeof(float));
  gp_tn_product all[GP_MAX_OUT_LAYERS + 2];
  for (int k = 0; k < L; ++k) all[k] = gp_tn_product{nullptr, nullptr, D, D, nullptr, nullptr};
  all[L] = gp_tn_product{nullptr, nullptr, H, D, nullptr, nullptr};
  all[L + 1] = gp_tn_product{nullptr, nullptr, D, 1, nullptr, nullptr};
  m = std::max(m, gp_gemm_tn_group_scratch(N, all, L + 2));
  s->part_bytes = m;
  s->part = (float*)c.take<char>(m);
  s->planes = c.take<char>((size_t)L * gp_align(gp_planes_bytes(D, D)) + gp_align(std::max(gp_planes_bytes(D, H), gp_planes_bytes(H, D))));
  return c.off;
}

int check_out_dims(gp_ctx* ctx, int H, int D, int R, int L) {
  if (H < 1 || H > 4096 || D < 1 || D > 4096 || R < 1 || R > 1024 || L < 0 || L > GP_MAX_OUT_LAYERS)
    return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "output block: emb=%d out_emb=%d num_radial=%d layers=%d unsupported", H, D, R, L);
  return GP_OK;
}
int check_out_weights(gp_ctx* ctx, const gp_weights_out* w, int L, const char* what) {
  GP_REQUIRE(ctx, w && w->W_rbf && w->W_up && w->w_final, "%s has a NULL member", what);
  for (int k = 0; k < L; ++k) GP_REQUIRE(ctx, w->W[k] && w->b[k], "%s: layer %d missing", what, k);
  return GP_OK;
}

}  // namespace

extern "C" {

int gp_output_workspace(int32_t emb, int32_t out_emb, int32_t num_radial, int32_t n_layers, int64_t n_atoms,
                        int64_t n_edges, size_t* saved_bytes, size_t* scratch_bytes) {
  if (!saved_bytes || !scratch_bytes || n_atoms < 0 || n_edges < 0 || emb < 1 || out_emb < 1 || num_radial < 1 ||
      n_layers < 0 || n_layers > GP_MAX_OUT_LAYERS)
    return GP_BAD_ARG;
  out_saved s;
  out_scratch sc;
  *saved_bytes = carve_out_saved(nullptr, n_atoms, emb, out_emb, n_layers, &s);
  *scratch_bytes = carve_out_scratch(nullptr, n_atoms, n_edges, emb, out_emb, num_radial, n_layers, &sc);
  return GP_OK;
}

int gp_output_forward(gp_ctx* ctx, int32_t emb, int32_t out_emb, int32_t num_radial, int32_t n_layers,
                      const gp_weights_out* w, const float* m, const float* rbf, const int32_t* row_ptr,
                      const int32_t* graph_ptr, int64_t n_atoms, int64_t n_edges, int32_t n_graphs, int32_t accumulate,
                      float* energy, void* saved, size_t saved_bytes, void* scratch, size_t scratch_bytes) {
  if (!ctx) return GP_BAD_ARG;
  const int H = emb, D = out_emb, R = num_radial, L = n_layers;
  GP_TRY(check_out_dims(ctx, H, D, R, L));
  GP_TRY(check_out_weights(ctx, w, L, "weights"));
  GP_REQUIRE(ctx, n_atoms >= 0 && n_edges >= 0 && n_graphs >= 0, "gp_output_forward: negative size");
  if (n_atoms == 0 || n_graphs == 0) return GP_OK;
  GP_REQUIRE(ctx, row_ptr && graph_ptr && energy && saved && scratch && (n_edges == 0 || (m && rbf)), "gp_output_forward: NULL pointer");
  out_saved s;
  out_scratch sc;
  if (saved_bytes < carve_out_saved(saved, n_atoms, H, D, L, &s)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_output_forward: saved buffer too small");
  if (scratch_bytes < carve_out_scratch(scratch, n_atoms, n_edges, H, D, R, L, &sc)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_output_forward: scratch too small");
  GP_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t st = ctx->stream;
  gp_epilogue e;
  if (n_edges > 0 && R <= RADIAL_MAX) {
    gp_prof_scope prof(ctx, "out_edge_sum", 2.0 * (double)n_edges * H * (R + 1), 4.0 * ((double)n_edges * (H + R) + (double)n_atoms * H));
    (R <= 8 ? out_edge_sum_kernel<8> : out_edge_sum_kernel<RADIAL_MAX>)<<<wblk(n_atoms * ((H + 63) / 64)), 256, 0, st>>>(
        m, rbf, w->W_rbf, row_ptr, n_atoms, H, R, s.h);
    GP_LAUNCH_CHECK(ctx, "out_edge_sum_kernel");
  } else {
    if (n_edges > 0) {
      e = gp_epilogue(); e.mul = m; e.out = sc.tE;
      GP_TRY(gp_gemm_nn(ctx, rbf, w->W_rbf, n_edges, H, R, e));                       // t = (rbf W_rbf) * m
    }
    gp_prof_scope prof(ctx, "out_atom_sum", (double)n_edges * H, 4.0 * ((double)n_edges * H + (double)n_atoms * H));
    out_atom_sum_kernel<<<wblk(n_atoms * ((H + 63) / 64)), 256, 0, st>>>(sc.tE, row_ptr, n_atoms, H, s.h);
    GP_LAUNCH_CHECK(ctx, "out_atom_sum_kernel");
  }
  gp_weight_planes wp(ctx, sc.planes);
  const void* p_up = wp.add(w->W_up, n_atoms, D, H, 1);
  const void* p_layer[GP_MAX_OUT_LAYERS] = {};
  for (int k = 0; k < L; ++k) p_layer[k] = wp.add(w->W[k], n_atoms, D, D, 1);
  GP_TRY(wp.run());
  e = gp_epilogue(); e.out = s.u0;
  GP_TRY(gp_gemm_nn_w(ctx, s.h, w->W_up, p_up, n_atoms, D, H, e));
  const float* u = s.u0;
  for (int k = 0; k < L; ++k) {
    e = gp_epilogue(); e.bias = w->b[k]; e.save_pre = s.z[k]; e.act = 1; e.out = s.u[k];
    GP_TRY(gp_gemm_nn_w(ctx, u, w->W[k], p_layer[k], n_atoms, D, D, e));
    u = s.u[k];
  }
  out_atom_dot_kernel<<<wblk(n_atoms), 256, 0, st>>>(u, w->w_final, n_atoms, D, sc.p);
  out_graph_sum_kernel<<<wblk(n_graphs), 256, 0, st>>>(sc.p, graph_ptr, n_graphs, accumulate, energy);
  GP_LAUNCH_CHECK(ctx, "output block reductions");
  return GP_OK;
}

int gp_output_backward(gp_ctx* ctx, int32_t emb, int32_t out_emb, int32_t num_radial, int32_t n_layers,
                       const gp_weights_out* w, const float* m, const float* rbf, const int32_t* dst,
                       const int32_t* graph_ptr, int64_t n_atoms, int64_t n_edges, int32_t n_graphs,
                       const float* grad_energy, const void* saved, size_t saved_bytes, int32_t accumulate_grad_m,
                       float* grad_m, gp_weights_out* grad_w, void* scratch, size_t scratch_bytes) {
  if (!ctx) return GP_BAD_ARG;
  const int H = emb, D = out_emb, R = num_radial, L = n_layers;
  GP_TRY(check_out_dims(ctx, H, D, R, L));
  GP_TRY(check_out_weights(ctx, w, L, "weights"));
  if (grad_w) GP_TRY(check_out_weights(ctx, grad_w, L, "grad_w"));
  GP_REQUIRE(ctx, n_atoms >= 0 && n_edges >= 0 && n_graphs >= 0, "gp_output_backward: negative size");
  if (n_atoms == 0 || n_graphs == 0) return GP_OK;
  GP_REQUIRE(ctx, graph_ptr && grad_energy && saved && scratch && (n_edges == 0 || (m && rbf && dst && grad_m)),
             "gp_output_backward: NULL pointer");
  out_saved s;
  out_scratch sc;
  if (saved_bytes < carve_out_saved(const_cast<void*>(saved), n_atoms, H, D, L, &s)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_output_backward: saved buffer too small");
  if (scratch_bytes < carve_out_scratch(scratch, n_atoms, n_edges, H, D, R, L, &sc)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_output_backward: scratch too small");
  GP_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t st = ctx->stream;
  gp_epilogue e;
  float* du = sc.du[L];   // dz of layer L - 1
  out_seed_kernel<<<wblk(n_atoms), 256, 0, st>>>(grad_energy, graph_ptr, n_graphs, n_atoms, w->w_final, L > 0 ? s.z[L - 1] : nullptr, D,
                                                 sc.ga, du);                              // du = dz_{L-1}
  GP_LAUNCH_CHECK(ctx, "out_seed_kernel");
  gp_weight_planes wp(ctx, sc.planes);
  const void* p_up = wp.add(w->W_up, n_atoms, H, D, 0);
  const void* p_layer[GP_MAX_OUT_LAYERS] = {};
  for (int k = 0; k < L; ++k) p_layer[k] = wp.add(w->W[k], n_atoms, D, D, 0);
  GP_TRY(wp.run());
  gp_tn_product wg[GP_MAX_OUT_LAYERS + 2];
  int n_wg = 0;
  wg[n_wg++] = gp_tn_product{L > 0 ? s.u[L - 1] : s.u0, sc.ga, D, 1, grad_w ? grad_w->w_final : nullptr, nullptr};
  for (int k = L - 1; k >= 0; --k) {
    wg[n_wg++] = gp_tn_product{k > 0 ? s.u[k - 1] : s.u0, du, D, D, grad_w ? grad_w->W[k] : nullptr, grad_w ? grad_w->b[k] : nullptr};
    e = gp_epilogue(); e.out = sc.du[k];
    if (k > 0) e.act = 2, e.zsrc = s.z[k - 1];
    GP_TRY(gp_gemm_nt_w(ctx, du, w->W[k], p_layer[k], n_atoms, D, D, e));               // dz_{k-1}, du_{-1} = du0
    du = sc.du[k];
  }
  wg[n_wg++] = gp_tn_product{s.h, du, H, D, grad_w ? grad_w->W_up : nullptr, nullptr};
  if (grad_w) GP_TRY(gp_gemm_tn_group(ctx, wg, n_wg, n_atoms, sc.part, sc.part_bytes));
  e = gp_epilogue(); e.out = sc.dh;
  GP_TRY(gp_gemm_nt_w(ctx, du, w->W_up, p_up, n_atoms, H, D, e));                       // dh
  if (n_edges > 0 && R <= RADIAL_MAX) {
    const int64_t per = (n_edges + edge_runs_most(n_edges) - 1) / edge_runs_most(n_edges), runs = (n_edges + per - 1) / per;
    {
      gp_prof_scope prof(ctx, "out_edge_grad", 4.0 * (double)n_edges * H * (R + 1), 4.0 * (double)n_edges * (3.0 * H + R));
      (R <= 8 ? out_edge_grad_kernel<8> : out_edge_grad_kernel<RADIAL_MAX>)<<<wblk(runs * ((H + 63) / 64)), 256, 0, st>>>(
          m, rbf, w->W_rbf, sc.dh, dst, n_edges, per, H, R, accumulate_grad_m, grad_m, grad_w ? sc.part : nullptr);
      GP_LAUNCH_CHECK(ctx, "out_edge_grad_kernel");
    }
    if (grad_w) GP_TRY(gp_reduce_parts(ctx, sc.part, (int)runs, (int64_t)R * H, grad_w->W_rbf));
  } else if (n_edges > 0) {
    {
      gp_prof_scope prof(ctx, "out_gather_rows", 0.0, 4.0 * ((double)n_edges * H + (double)n_atoms * H));
      out_gather_rows_kernel<<<nblk(n_edges * H), 256, 0, st>>>(sc.dh, dst, n_edges, H, sc.tE);   // dt
      GP_LAUNCH_CHECK(ctx, "out_gather_rows_kernel");
    }
    e = gp_epilogue(); e.mul = sc.tE; e.out = grad_m;
    if (accumulate_grad_m) e.add_post = grad_m;
    GP_TRY(gp_gemm_nn(ctx, rbf, w->W_rbf, n_edges, H, R, e));                           // grad_m (+)= dt * gate
    if (grad_w) {
      out_mul_inplace_kernel<<<nblk(n_edges * H), 256, 0, st>>>(sc.tE, m, n_edges * H);  // dgate = dt * m
      GP_LAUNCH_CHECK(ctx, "out_mul_inplace_kernel");
      GP_TRY(gp_gemm_tn(ctx, rbf, sc.tE, n_edges, R, H, grad_w->W_rbf, nullptr, sc.part, sc.part_bytes));
    }
  } else if (grad_w) {
    out_zero_kernel<<<nblk((int64_t)R * H), 256, 0, st>>>(grad_w->W_rbf, (int64_t)R * H);
    GP_LAUNCH_CHECK(ctx, "out_zero_kernel");
  }
  return GP_OK;
}

}  // extern "C"
