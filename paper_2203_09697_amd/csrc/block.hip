// Interaction block, variant D (paper Sec. 3.3): the EdgeUpdate MLPs around
// TripletUpdate/TripletAggr, forward and hand-derived backward.  Pure launch sequencing on the
// context's stream; every arithmetic step runs in the kernels of gemm.hip / triplet.hip.
//
//   x_ji = act(m W_ji + b_ji)
//   x_kj = act(m W_kj + b_kj) * (rbf (W_rbf1 W_rbf2));  x_kj = act(x_kj W_down)
//   a_e  = sum_{t in seg(e)} x_kj[kj(t)] * ((sbf_t W_sbf1) W_sbf2)
//   h    = x_ji + act(a W_up);  residual layers;  h = act(h W_lin + b_lin) + m;  residual layers
#include <stdarg.h>

#include <algorithm>
#include <initializer_list>

#include "aux_stream.h"
#include "gemm.h"
#include "triplet.h"

namespace {

struct res_saved {
  float *z1, *y1, *z2, *hout;
};

struct saved_D {
  float *z_ji, *z_kj, *gate, *xg, *z_dn, *x_kj, *Q, *Bacc, *a, *z_up, *h0, *z_lin, *h_lin, *Wrbf;
  res_saved before[GP_MAX_RES], after[GP_MAX_RES];
};

size_t carve_saved_D(void* p, const gp_dims* d, int64_t E, saved_D* s) {
  gp_carver c(p);
  const size_t H = d->emb, F = d->int_emb, B = d->basis_emb, S = d->num_spherical, R = d->num_radial;
  s->z_ji = c.take<float>(E * H);
  s->z_kj = c.take<float>(E * H);
  s->gate = c.take<float>(E * H);
  s->xg = c.take<float>(E * H);
  s->z_dn = c.take<float>(E * F);
  s->x_kj = c.take<float>(E * F);
  s->Q = c.take<float>(E * S * B);
  s->Bacc = c.take<float>(E * B * F);
  s->a = c.take<float>(E * F);
  s->z_up = c.take<float>(E * H);
  s->h0 = c.take<float>(E * H);
  s->z_lin = c.take<float>(E * H);
  s->h_lin = c.take<float>(E * H);
  s->Wrbf = c.take<float>(R * H);
  for (int r = 0; r < d->n_res_before; ++r) {
    s->before[r].z1 = c.take<float>(E * H);
    s->before[r].y1 = c.take<float>(E * H);
    s->before[r].z2 = c.take<float>(E * H);
    s->before[r].hout = c.take<float>(E * H);
  }
  for (int r = 0; r < d->n_res_after; ++r) {
    s->after[r].z1 = c.take<float>(E * H);
    s->after[r].y1 = c.take<float>(E * H);
    s->after[r].z2 = c.take<float>(E * H);
    s->after[r].hout = c.take<float>(E * H);   // the last one is unused: the block output goes to m_out
  }
  return c.off;
}

// Gradients of the pre-activations of a block, one per dense layer over the edges, one for dxg and one for the gate; where the weight
// gradients are formed together they all have to last, else four are used in turn.
constexpr int DZ_MOST = 6 + 4 * GP_MAX_RES, DZ_TURN = 4;
int dz_private_D(const gp_dims* d) { return 6 + 2 * (d->n_res_before + d->n_res_after); }
// The weight gradients of a block are formed by a few launches for all of them where a product by itself would be cut into many
// runs of the rows (gp_gemm_tn_group), i.e. below width 512, and while the buffers that have to last for it take no more than 2 GiB
// beyond the four: with three residual layers 262 thousand edges at width 256, a million at 64.  Training step of three blocks, one by
// one / together (ms): width 256, 43 380 edges 5.42 / 5.19, 130 140 13.3 / 13.4, 260 280 26.2 / 26.2; 192, 260 280 22.7 / 21.6; 128, 260 280
// 12.5 / 11.8, 515 137 24.4 / 23.7; 64, 260 280 7.65 / 7.10, 1 003 162 36.9 / 32.3 (up to 192 together with the chains below).
// The width, two blocks: 384, 398 edges 1.23 / 1.11, 1884 1.37 / 1.22, 8698 2.04 / 1.93, 17 398 2.83 / 2.75; 448, 1.33 / 1.20, 1.48 / 1.36,
// 2.38 / 2.35, 3.63 / 3.64; 512, 1.72 / 1.85, 2.07 / 2.14, 2.72 / 3.01, 4.10 / 4.38; 1024, 2.31 / 2.59, 2.79 / 3.17, 5.89 / 6.25, 10.5 / 11.0.
constexpr int64_t GROUP_ROOM = (int64_t)1 << 31;
int64_t group_rows_D(const gp_dims* d) { return d->emb >= 512 ? 0 : GROUP_ROOM / ((int64_t)sizeof(float) * d->emb * (dz_private_D(d) - DZ_TURN)); }
bool group_D(const gp_dims* d, int64_t E) { return d->emb < 512 && E <= group_rows_D(d); }
int dz_buffers_D(const gp_dims* d, int64_t E) { return group_D(d, E) ? dz_private_D(d) : DZ_TURN; }
int64_t dz_stride_D(const gp_dims* d, int64_t E) { return (E * d->emb + 63) / 64 * 64; }   // floats from one to the next

struct scratch_D {
  float* buf[3];     // [E,H] each: gradients of the messages between layers
  float* dz[DZ_MOST];   // [E,H] each
  float *dF1, *dF2;  // [E,F]
  float* dQ;         // [E,S*B]
  float* P;          // [E,S,F]: per-edge factor of the gradient with respect to cos(alpha) (basis gradients only)
  float* dWrbf;      // [R,H]
  float* part;       // partial sums of the main stream's reductions, one at a time
  float* part_aux;   // of those issued on the side stream, groups among them
  size_t part_bytes, part_aux_bytes;
  void* planes;      // the weights of a call as operand planes (gemm_planes.hip) or as parts for its chains
  size_t planes_bytes;
};

// partial sums of the reductions over the edges, one at a time
size_t part_bytes_one_D(const gp_dims* d, int64_t E) {
  const int H = d->emb, F = d->int_emb, B = d->basis_emb, S = d->num_spherical, R = d->num_radial;
  size_t m = gp_gemm_tn_scratch(E, H, H);
  m = std::max(m, gp_gemm_tn_scratch(E, F, H));
  m = std::max(m, gp_gemm_tn_scratch(E, H, F));
  m = std::max(m, gp_gemm_tn_scratch(E, R, H));
  m = std::max(m, gp_colsum_scratch(E, H));
  m = std::max(m, gp_tripD_wgrad_scratch(E, F, S, R, B));
  return m;
}

// ... of groups too; no smaller for more edges
size_t part_bytes_aux_D(const gp_dims* d, int64_t E) {
  size_t m = part_bytes_one_D(d, E);
  if (group_rows_D(d) > 0) {
    gp_tn_product all[GP_TN_JOBS_MAX];
    int n = 0;
    auto add = [&](int a, int b) { all[n++] = gp_tn_product{nullptr, nullptr, a, b, nullptr, nullptr}; };
    for (int i = 0; i < 3 + 2 * (d->n_res_before + d->n_res_after); ++i) add(d->emb, d->emb);
    add(d->num_radial, d->emb);
    add(d->int_emb, d->emb);
    add(d->emb, d->int_emb);
    m = std::max(m, gp_gemm_tn_group_scratch(std::min(E, group_rows_D(d)), all, n));
  }
  return m;
}

// The matrix-core backward kernel also yields the gradient of W_sbf2, so the forward pass need not keep Bacc
// (E x basis_emb x int_emb floats).  Forward and backward must take the same decision: it depends only on the
// context's switch, the widths and the graph.
bool bwd_mfma_D(const gp_ctx* ctx, const gp_dims* d, const gp_graph* g) {
  if (ctx->trip_mfma == 0) return false;
  const int F = d->int_emb, S = d->num_spherical, B = d->basis_emb;
  return gp_tripD_mfma_usable(g, F, S, B) && gp_tripD_mfma_bwd_usable(g, F, S, B) &&
         gp_tripD_mfma_bwd_scratch(g, F) <= part_bytes_one_D(d, g->n_edges);
}

// room for the planes of every weight matrix that meets the edges, for the products of either pass
size_t planes_bytes_D(const gp_dims* d) {
  const int H = d->emb, F = d->int_emb;
  auto both = [](int a, int b) { return std::max(gp_align(gp_planes_bytes(a, b)), gp_align(gp_planes_bytes(b, a))); };
  const size_t square = 3 + 2 * d->n_res_before + 2 * d->n_res_after;
  const size_t chain = gp_chain_takes(H, F) ? square * gp_chain_parts_bytes(H, H, H) + gp_chain_parts_bytes(H, H, F) + gp_chain_parts_bytes(H, F, H) : 0;
  return std::max(square * both(H, H) + 2 * both(H, F), chain);
}

// Whether the layers over E edges run as chains (dense_chain.hip) with these pointers.  Training step of three blocks, layer by layer / as
// chains (ms): width 64, 13 668 edges 1.35 / 0.93, 100 119 edges 3.53 / 3.09; 128, 1.67 / 1.25 and 5.72 / 5.12; 192, 2.27 / 1.80 and
// 9.51 / 8.87; 256, 13 668 edges 2.55 / 2.25, 27 028 3.68 / 3.63, 32 538 4.13 / 4.03, 43 380 5.16 / 5.36, 100 119 10.54 / 11.11: at that width
// two workgroups of 64 rows fill a compute unit, and where some would come in a second round the layers' own launches are faster.
bool chain_D(const gp_ctx* ctx, const gp_dims* d, const gp_weights_D* w, int64_t E, std::initializer_list<const void*> more) {
  if (!ctx->f32_split || ctx->gemm_bf16 || !gp_chain_takes(d->emb, d->int_emb) || (d->emb > 192 && E > 32768)) return false;
  uintptr_t a = (uintptr_t)w->b_ji | (uintptr_t)w->b_kj | (uintptr_t)w->b_lin;
  for (int r = 0; r < d->n_res_before; ++r) a |= (uintptr_t)w->res_before[r][1] | (uintptr_t)w->res_before[r][3];
  for (int r = 0; r < d->n_res_after; ++r) a |= (uintptr_t)w->res_after[r][1] | (uintptr_t)w->res_after[r][3];
  for (const void* p : more) a |= (uintptr_t)p;
  return (a & 15) == 0;
}

// the steps of a call
struct chain_list {
  gp_chain_step s[GP_CHAIN_MAX];
  int n = 0;
  gp_chain_step& add(const float* W, int N, int K, int k_rows) {
    gp_chain_step& q = s[n++];
    q.W = W; q.N = N; q.K = K; q.k_rows = k_rows;
    return q;
  }
};

size_t carve_scratch_D(void* p, const gp_dims* d, int64_t E, scratch_D* s) {
  gp_carver c(p);
  const size_t H = d->emb, F = d->int_emb, B = d->basis_emb, S = d->num_spherical, R = d->num_radial;
  for (int i = 0; i < 3; ++i) s->buf[i] = c.take<float>(E * H);
  // as many as are used at E, and no less room than a smaller graph's groups take
  const int64_t stride = dz_stride_D(d, E), grouped = dz_private_D(d) * dz_stride_D(d, std::min(E, group_rows_D(d)));
  float* const dz = c.take<float>(std::max(DZ_TURN * stride, grouped));
  for (int i = 0; i < dz_buffers_D(d, E); ++i) s->dz[i] = dz + i * stride;
  s->dF1 = c.take<float>(E * F);
  s->dF2 = c.take<float>(E * F);
  s->dQ = c.take<float>(E * S * B);
  s->P = c.take<float>(E * S * F);
  s->dWrbf = c.take<float>(R * H);
  s->part_bytes = part_bytes_one_D(d, E);
  s->part = (float*)c.take<char>(s->part_bytes);
  s->part_aux_bytes = part_bytes_aux_D(d, E);
  s->part_aux = (float*)c.take<char>(s->part_aux_bytes);
  s->planes_bytes = planes_bytes_D(d);
  s->planes = c.take<char>(s->planes_bytes);
  return c.off;
}

int check_dims_D(gp_ctx* ctx, const gp_dims* d) {
  GP_REQUIRE(ctx, d, "dims is NULL");
  if (d->variant != GP_VARIANT_D) return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "variant %d is not the Hadamard block", d->variant);
  if (d->dtype != GP_F32) return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "variant D is implemented in fp32 only");
  if (d->emb < 1 || d->emb > 4096 || d->int_emb < 1 || d->int_emb > 256 || d->basis_emb < 1 || d->basis_emb > 16 ||
      d->num_spherical < 1 || d->num_spherical > 8 || d->num_radial < 1 || d->num_radial > 16 ||
      d->n_res_before < 0 || d->n_res_before > GP_MAX_RES || d->n_res_after < 0 || d->n_res_after > GP_MAX_RES)
    return gp_fail(ctx, GP_UNSUPPORTED_DIMS,
                   "variant D supports emb<=4096, int_emb<=256, basis_emb<=16, num_spherical<=8, num_radial<=16, "
                   "residual layers<=%d (got %d,%d,%d,%d,%d,%d,%d)", GP_MAX_RES, d->emb, d->int_emb, d->basis_emb,
                   d->num_spherical, d->num_radial, d->n_res_before, d->n_res_after);
  return GP_OK;
}

int check_weights_D(gp_ctx* ctx, const gp_dims* d, const gp_weights_D* w, const char* what) {
  GP_REQUIRE(ctx, w, "%s is NULL", what);
  bool ok = w->W_ji && w->b_ji && w->W_kj && w->b_kj && w->W_rbf1 && w->W_rbf2 && w->W_down && w->W_sbf1 &&
            w->W_sbf2 && w->W_up && w->W_lin && w->b_lin;
  for (int r = 0; r < d->n_res_before; ++r)
    for (int q = 0; q < 4; ++q) ok = ok && w->res_before[r][q];
  for (int r = 0; r < d->n_res_after; ++r)
    for (int q = 0; q < 4; ++q) ok = ok && w->res_after[r][q];
  GP_REQUIRE(ctx, ok, "%s has a NULL member", what);
  return GP_OK;
}

// From that many edges on the forward pass cuts the layers after the triplet sum into two halves of the rows.
constexpr int64_t SPLIT_MIN_ROWS = 2048;
// Whether a block is worth the side stream: not where its kernels are as short as an event and its wait on another stream take to issue.
// Two blocks forward and backward, one stream / two (ms), 288 edges: width 64 0.31 / 0.48, 128 0.50 / 0.57, 256 1.00 / 1.05, 384 1.13 / 1.09,
// 448 1.25 / 1.19, 512 1.88 / 1.57, 1024 2.76 / 2.15, 2048 5.15 / 4.18; 1494 edges: 0.38 / 0.48, 0.58 / 0.65, 1.07 / 1.10, 1.25 / 1.19, 1.41 / 1.31,
// 2.27 / 1.91, 3.40 / 2.93, 7.05 / 6.02.
bool side_D(const gp_dims* d, int64_t E) { return d->emb > 256 || E >= 2048; }

// one residual layer forward: hout = hin + act(act(hin W1 + b1) W2 + b2); pl: the planes of W1 and W2
int res_forward(gp_ctx* ctx, const float* hin, float* const* w, const void* const* pl, const res_saved& s, float* hout, int64_t E, int H) {
  gp_epilogue e1;
  e1.bias = w[1]; e1.save_pre = s.z1; e1.act = 1; e1.out = s.y1;
  GP_TRY(gp_gemm_nn_w(ctx, hin, w[0], pl[0], E, H, H, e1));
  gp_epilogue e2;
  e2.bias = w[3]; e2.save_pre = s.z2; e2.act = 1; e2.add_post = hin; e2.out = hout;
  return gp_gemm_nn_w(ctx, s.y1, w[2], pl[1], E, H, H, e2);
}

// The weight gradients of a backward pass and the buffers of the gradients that enter them.
struct wgrads_D {
  gp_ctx* ctx;
  gp_aux& aux;
  scratch_D& sc;
  int64_t E;
  bool group;
  int n_dz, at = 0, n = 0;
  gp_tn_product p[GP_TN_JOBS_MAX];
  wgrads_D(gp_ctx* c, gp_aux& a, scratch_D& s, const gp_dims* d, int64_t rows) : ctx(c), aux(a), sc(s), E(rows), group(group_D(d, rows)), n_dz(dz_buffers_D(d, rows)) {}
  // Room for the next gradient.  Where the buffers are used in turn the side stream may still read what was in it, which a gradient that it
  // writes itself (on_side) need not wait for.
  int take(float** dz, bool on_side = false) {
    *dz = sc.dz[at];
    at = at + 1 == n_dz ? 0 : at + 1;
    return group || on_side ? GP_OK : aux.before_write(*dz);
  }
  // W = A^T dz, b its column sums
  int add(const float* A, const float* dz, int M, int N, float* W, float* b) {
    if (group) {
      p[n++] = gp_tn_product{A, dz, M, N, W, b};
      return GP_OK;
    }
    return aux.on_aux([&] { return gp_gemm_tn(ctx, A, dz, E, M, N, W, b, sc.part_aux, sc.part_aux_bytes); }, {dz});
  }
  // forms what has been added, on the side stream
  int run() {
    if (n == 0) return GP_OK;
    const int k = n;
    n = 0;
    return aux.on_aux([&] { return gp_gemm_tn_group(ctx, p, k, E, sc.part_aux, sc.part_aux_bytes); }, {});
  }
};

// One residual layer backward.  dz2 = dh * silu'(z2) is given (written by the producer of dh).
// dh_out = dh + d(hin through the layer), dz_next = dh_out * silu'(z_next).
int res_backward(gp_ctx* ctx, wgrads_D& wg, const float* hin, float* const* w, const void* const* pl, float* const* gw,
                 const res_saved& s, const float* dh, const float* dz2, float* dh_out, const float* z_next, float** dz_next, int64_t E, int H) {
  GP_TRY(wg.add(s.y1, dz2, H, H, gw[2], gw[3]));
  float* dz1;
  GP_TRY(wg.take(&dz1));
  gp_epilogue e;
  e.act = 2; e.zsrc = s.z1; e.out = dz1;
  GP_TRY(gp_gemm_nt_w(ctx, dz2, w[2], pl[1], E, H, H, e));
  GP_TRY(wg.add(hin, dz1, H, H, gw[0], gw[1]));
  GP_TRY(wg.take(dz_next));
  gp_epilogue e2;
  e2.add_post = dh; e2.out = dh_out; e2.out2 = *dz_next; e2.z2src = z_next;
  return gp_gemm_nt_w(ctx, dz1, w[0], pl[0], E, H, H, e2);
}

}  // namespace

extern "C" {

int gp_block_workspace(const gp_dims* dims, int64_t n_atoms, int64_t n_edges, int64_t n_triplets, size_t* saved_bytes,
                       size_t* scratch_bytes) {
  if (!dims || !saved_bytes || !scratch_bytes || n_atoms < 0 || n_edges < 0 || n_triplets < 0) return GP_BAD_ARG;
  if (dims->variant == GP_VARIANT_D) {
    saved_D s;
    scratch_D sc;
    *saved_bytes = carve_saved_D(nullptr, dims, n_edges, &s);
    *scratch_bytes = carve_scratch_D(nullptr, dims, n_edges, &sc);
    return GP_OK;
  }
  if (dims->variant == GP_VARIANT_G) {
    *saved_bytes = gp_block_G_saved_bytes(dims, n_edges);
    *scratch_bytes = gp_block_G_scratch_bytes(dims, n_atoms, n_edges, n_triplets);
    return GP_OK;
  }
  return GP_UNSUPPORTED_DIMS;
}

int gp_block_forward_D(gp_ctx* ctx, const gp_dims* dims, const gp_weights_D* w, const gp_graph* graph,
                       const gp_basis* basis, const float* m_in, float* m_out, void* saved, size_t saved_bytes,
                       void* scratch, size_t scratch_bytes) {
  if (!ctx) return GP_BAD_ARG;
  GP_TRY(check_dims_D(ctx, dims));
  GP_TRY(check_weights_D(ctx, dims, w, "weights"));
  GP_REQUIRE(ctx, graph && basis, "gp_block_forward_D: graph/basis is NULL");
  const int64_t E = graph->n_edges;
  GP_REQUIRE(ctx, E >= 0 && graph->n_triplets >= 0, "gp_block_forward_D: negative size");
  if (E == 0) return GP_OK;
  GP_REQUIRE(ctx, m_in && m_out && saved && scratch, "gp_block_forward_D: NULL pointer");
  GP_REQUIRE(ctx, basis->rbf && basis->rad && (graph->n_triplets == 0 || basis->cos_alpha), "gp_block_forward_D: basis arrays missing");
  GP_TRY(gp_take_deferred(ctx, "gp_block_forward_D"));
  saved_D s;
  scratch_D sc;
  if (saved_bytes < carve_saved_D(saved, dims, E, &s)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_block_forward_D: saved buffer too small");
  if (scratch_bytes < carve_scratch_D(scratch, dims, E, &sc)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_block_forward_D: scratch too small");
  GP_HIP(ctx, hipSetDevice(ctx->device));
  const int H = dims->emb, F = dims->int_emb, B = dims->basis_emb, S = dims->num_spherical, R = dims->num_radial;
  float* x_ji = sc.buf[0];

  const bool chain = chain_D(ctx, dims, w, E, {m_in, m_out, saved, scratch});
  chain_list ch;
  int pre = 0;   // steps before the triplet sum
  if (chain) {
    gp_chain_step& ji = ch.add(w->W_ji, H, H, 1);
    ji.load = m_in; ji.bias = w->b_ji; ji.save_pre = s.z_ji; ji.act = 1; ji.out = x_ji; ji.keep = 1;
    gp_chain_step& kj = ch.add(w->W_kj, H, H, 1);
    kj.bias = w->b_kj; kj.save_pre = s.z_kj; kj.act = 1; kj.mul = s.gate; kj.out = s.xg;
    gp_chain_step& dn = ch.add(w->W_down, F, H, 1);
    dn.save_pre = s.z_dn; dn.act = 1; dn.out = s.x_kj;
    pre = ch.n;
    gp_chain_step& up = ch.add(w->W_up, H, F, 1);
    up.load = s.a; up.save_pre = s.z_up; up.act = 1; up.add = x_ji; up.out = s.h0;
    const float* h = s.h0;
    auto residual = [&](const float* const* wr, const res_saved& q, float* out) {
      gp_chain_step& s1 = ch.add(wr[0], H, H, 1);
      s1.bias = wr[1]; s1.save_pre = q.z1; s1.act = 1; s1.out = q.y1;
      gp_chain_step& s2 = ch.add(wr[2], H, H, 1);
      s2.bias = wr[3]; s2.save_pre = q.z2; s2.act = 1; s2.add = h; s2.out = out;
      h = out;
    };
    for (int r = 0; r < dims->n_res_before; ++r) residual(w->res_before[r], s.before[r], s.before[r].hout);
    gp_chain_step& li = ch.add(w->W_lin, H, H, 1);
    li.bias = w->b_lin; li.save_pre = s.z_lin; li.act = 1; li.add = m_in; li.out = dims->n_res_after == 0 ? m_out : s.h_lin;
    h = li.out;
    for (int r = 0; r < dims->n_res_after; ++r)
      residual(w->res_after[r], s.after[r], r == dims->n_res_after - 1 ? m_out : s.after[r].hout);
    GP_TRY(gp_chain_prepare(ctx, H, ch.s, ch.n, sc.planes, sc.planes_bytes));
  }

  gp_weight_planes wp(ctx, chain ? nullptr : sc.planes);
  const void *p_ji = wp.add(w->W_ji, E, H, H, 1), *p_kj = wp.add(w->W_kj, E, H, H, 1), *p_down = wp.add(w->W_down, E, F, H, 1),
             *p_up = wp.add(w->W_up, E, H, F, 1), *p_lin = wp.add(w->W_lin, E, H, H, 1);
  const void *p_before[GP_MAX_RES][2] = {}, *p_after[GP_MAX_RES][2] = {};
  for (int r = 0; r < dims->n_res_before; ++r)
    for (int q = 0; q < 2; ++q) p_before[r][q] = wp.add(w->res_before[r][2 * q], E, H, H, 1);
  for (int r = 0; r < dims->n_res_after; ++r)
    for (int q = 0; q < 2; ++q) p_after[r][q] = wp.add(w->res_after[r][2 * q], E, H, H, 1);
  GP_TRY(wp.run());

  // Side stream, before the triplet sum: the projected radial table is needed only by the triplet kernel and the
  // projection of the target-edge message only by the epilogue of the up-projection, so both run next to the chain
  // that leads to the triplet sum.  After it: the layers act on every edge by itself, and a GEMM over all E rows at
  // these widths is one round of workgroups whose loading, multiplying and storing phases coincide; the rows are cut
  // in two and the halves run as two chains on the two streams, out of step with each other (configuration 2:
  // 9.70 -> 9.40 ms per step; cutting the chain before the triplet sum as well: 9.51 ms).
  gp_aux aux(ctx, side_D(dims, E));
  const int64_t half = ((E / 2 + 127) / 128) * 128;
  const bool split = aux.active() && E >= SPLIT_MIN_ROWS && half < E;
  gp_epilogue e;
  e.out = s.Wrbf;
  GP_TRY(gp_gemm_nn(ctx, w->W_rbf1, w->W_rbf2, R, H, B, e));
  auto project_radial = [&] { return gp_tripD_project_radial(ctx, basis->rad, w->W_sbf1, E, S, R, B, s.Q); };   // Q is [S*B, E]: not cut
  auto ji_rows = [&](int64_t r0, int64_t n) {
    const int64_t o = r0 * H;
    gp_epilogue q; q.bias = w->b_ji; q.save_pre = s.z_ji + o; q.act = 1; q.out = x_ji + o;
    return gp_gemm_nn_w(ctx, m_in + o, w->W_ji, p_ji, n, H, H, q);
  };
  auto kj_rows = [&](int64_t r0, int64_t n) -> int {
    const int64_t o = r0 * H;
    gp_epilogue q; q.out = s.gate + o;
    GP_TRY(gp_gemm_nn(ctx, basis->rbf + r0 * R, s.Wrbf, n, H, R, q));
    q = gp_epilogue(); q.bias = w->b_kj; q.save_pre = s.z_kj + o; q.act = 1; q.mul = s.gate + o; q.out = s.xg + o;
    GP_TRY(gp_gemm_nn_w(ctx, m_in + o, w->W_kj, p_kj, n, H, H, q));
    q = gp_epilogue(); q.save_pre = s.z_dn + r0 * F; q.act = 1; q.out = s.x_kj + r0 * F;
    return gp_gemm_nn_w(ctx, s.xg + o, w->W_down, p_down, n, F, H, q);
  };
  GP_TRY(aux.on_aux([&] { return project_radial(); }, {s.Q}));
  if (chain) {
    gp_epilogue q; q.out = s.gate;
    GP_TRY(gp_gemm_nn(ctx, basis->rbf, s.Wrbf, E, H, R, q));
    GP_TRY(gp_chain_run(ctx, H, ch.s, 0, pre, E, sc.planes));
  } else {
    GP_TRY(aux.on_aux([&] { return ji_rows(0, E); }, {}));
    GP_TRY(kj_rows(0, E));
  }
  GP_TRY(aux.before_write(s.Q));   // the projected radial table, written on the side stream
  const bool fwd_mfma = ctx->trip_mfma != 0 && gp_tripD_mfma_usable(graph, F, S, B);
  const bool keep_Bacc = !(fwd_mfma && bwd_mfma_D(ctx, dims, graph));
  ctx->fwd_flags[saved] = keep_Bacc ? 1u : 0u;   // the backward call must agree on whether Bacc was written
  if (fwd_mfma || bwd_mfma_D(ctx, dims, graph)) GP_TRY(gp_check_degrees(ctx, graph));
  if (fwd_mfma)
    GP_TRY(gp_tripD_forward_mfma(ctx, graph, basis->cos_alpha, s.x_kj, s.Q, w->W_sbf2, F, S, B, s.a, keep_Bacc ? s.Bacc : nullptr));
  else
    GP_TRY(gp_tripD_forward(ctx, graph, basis->cos_alpha, s.x_kj, s.Q, w->W_sbf2, F, S, B, s.a, s.Bacc));
  GP_TRY(aux.join());
  if (chain) return gp_chain_run(ctx, H, ch.s, pre, ch.n, E, sc.planes);

  // rows [r0, r0 + n) of the layers after the triplet sum
  auto rows_forward = [&](int64_t r0, int64_t n) -> int {
    const int64_t o = r0 * H;
    auto at = [&](const res_saved& q) { return res_saved{q.z1 + o, q.y1 + o, q.z2 + o, q.hout + o}; };
    gp_epilogue eu; eu.save_pre = s.z_up + o; eu.act = 1; eu.add_post = x_ji + o; eu.out = s.h0 + o;
    GP_TRY(gp_gemm_nn_w(ctx, s.a + r0 * F, w->W_up, p_up, n, H, F, eu));
    const float* h = s.h0 + o;
    for (int r = 0; r < dims->n_res_before; ++r) {
      const res_saved q = at(s.before[r]);
      GP_TRY(res_forward(ctx, h, w->res_before[r], p_before[r], q, q.hout, n, H));
      h = q.hout;
    }
    float* lin_out = (dims->n_res_after == 0 ? m_out : s.h_lin) + o;
    gp_epilogue el; el.bias = w->b_lin; el.save_pre = s.z_lin + o; el.act = 1; el.add_post = m_in + o; el.out = lin_out;
    GP_TRY(gp_gemm_nn_w(ctx, h, w->W_lin, p_lin, n, H, H, el));
    h = lin_out;
    for (int r = 0; r < dims->n_res_after; ++r) {
      const res_saved q = at(s.after[r]);
      float* out = (r == dims->n_res_after - 1) ? m_out + o : q.hout;
      GP_TRY(res_forward(ctx, h, w->res_after[r], p_after[r], q, out, n, H));
      h = out;
    }
    return GP_OK;
  };
  if (split) {
    GP_TRY(aux.on_aux([&] { return rows_forward(half, E - half); }, {}));
    GP_TRY(rows_forward(0, half));
    return aux.join();
  }
  return rows_forward(0, E);
}

}  // extern "C"

namespace {

// P[e, l, f] = x[e, f] sum_b W_sbf2[b, f] Q[e, l, b]: with it, dL/dcos(alpha_t) = sum_l Y_l0'(cos alpha_t) sum_f
// grad_a[ji(t), f] P[kj(t), l, f], the same contraction as the bilinear block's (U = P, dz = grad_a)
__global__ void cos_factor_kernel(const float* __restrict__ x, const float* __restrict__ W2, const float* __restrict__ Qt, int64_t E,
                                  int S, int B, int F, float* __restrict__ P) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // (e, l, f)
  if (i >= E * S * F) return;
  const int f = (int)(i % F), l = (int)((i / F) % S);
  const int64_t e = i / ((int64_t)F * S);
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += W2[b * F + f] * Qt[(int64_t)(l * B + b) * E + e];
  P[i] = x[e * F + f] * s;
}

// grad_rad[e, l, n] (+)= sum_b grad_Q[e, l, b] W_sbf1[(l, n), b]   (Q[e, l, b] = sum_n rad[e, l, n] W_sbf1[(l, n), b])
__global__ void grad_rad_kernel(const float* __restrict__ gQ, const float* __restrict__ W1, int64_t E, int S, int R, int B,
                                int accumulate, float* __restrict__ grad_rad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // (e, l, n)
  if (i >= E * S * R) return;
  const int n = (int)(i % R), l = (int)((i / R) % S);
  const int64_t e = i / ((int64_t)R * S);
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += gQ[(e * S + l) * B + b] * W1[(l * R + n) * B + b];
  grad_rad[i] = accumulate ? grad_rad[i] + s : s;
}

int backward_D(gp_ctx* ctx, const gp_dims* dims, const gp_weights_D* w, const gp_graph* graph, const gp_basis* basis,
               const float* m_in, const void* saved, size_t saved_bytes, const float* grad_m_out, float* grad_m_in,
               gp_weights_D* gw, float* grad_rbf, float* grad_rad, float* grad_cos_kj, int accumulate_basis_grads,
               void* scratch, size_t scratch_bytes) {
  if (!ctx) return GP_BAD_ARG;
  GP_TRY(check_dims_D(ctx, dims));
  GP_TRY(check_weights_D(ctx, dims, w, "weights"));
  GP_TRY(check_weights_D(ctx, dims, gw, "grad_w"));
  GP_REQUIRE(ctx, graph && basis, "gp_block_backward_D: graph/basis is NULL");
  const int64_t E = graph->n_edges;
  GP_REQUIRE(ctx, E >= 0 && graph->n_triplets >= 0, "gp_block_backward_D: negative size");
  GP_REQUIRE(ctx, E > 0, "gp_block_backward_D: empty edge list");
  GP_REQUIRE(ctx, m_in && grad_m_out && grad_m_in && saved && scratch, "gp_block_backward_D: NULL pointer");
  GP_REQUIRE(ctx, basis->rbf && basis->rad && (graph->n_triplets == 0 || basis->cos_alpha_kj), "gp_block_backward_D: basis arrays missing");
  saved_D s;
  scratch_D sc;
  if (saved_bytes < carve_saved_D(const_cast<void*>(saved), dims, E, &s)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_block_backward_D: saved buffer too small");
  if (scratch_bytes < carve_scratch_D(scratch, dims, E, &sc)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_block_backward_D: scratch too small");
  GP_HIP(ctx, hipSetDevice(ctx->device));
  const int H = dims->emb, F = dims->int_emb, B = dims->basis_emb, S = dims->num_spherical, R = dims->num_radial;
  const int64_t EH = E * H;
  // rotating buffers for dh; `keep` is a gradient that must survive (the skip into m)
  const float* dh = grad_m_out;
  const float* keep = nullptr;
  auto next_buf = [&]() -> float* {
    for (int i = 0; i < 3; ++i)
      if (sc.buf[i] != dh && sc.buf[i] != keep) return sc.buf[i];
    return nullptr;
  };

  // Small graphs are launches and nothing else: one stream, all weight gradients at the end.  Otherwise they are formed on the side stream, in
  // groups or one by one, each as soon as what enters it is there.
  gp_aux aux(ctx, side_D(dims, E));
  wgrads_D wg(ctx, aux, sc, dims, E);
  // dz of the last activation in the block
  const float* z_first = dims->n_res_after > 0 ? s.after[dims->n_res_after - 1].z2 : s.z_lin;
  const bool chain = wg.group && chain_D(ctx, dims, w, E, {m_in, grad_m_out, grad_m_in, saved, scratch});   // its gradients all last
  chain_list ch;
  int pre = 0;   // steps before the triplet sum's gradients
  float *dz_ji, *dz_kj, *dgate, *dm_ji;
  gp_weight_planes wp(ctx, chain ? nullptr : sc.planes);
  const void *p_ji = wp.add(w->W_ji, E, H, H, 0), *p_kj = wp.add(w->W_kj, E, H, H, 0), *p_down = wp.add(w->W_down, E, H, F, 0),
             *p_up = wp.add(w->W_up, E, F, H, 0), *p_lin = wp.add(w->W_lin, E, H, H, 0);
  const void *p_before[GP_MAX_RES][2] = {}, *p_after[GP_MAX_RES][2] = {};
  for (int r = 0; r < dims->n_res_before; ++r)
    for (int q = 0; q < 2; ++q) p_before[r][q] = wp.add(w->res_before[r][2 * q], E, H, H, 0);
  for (int r = 0; r < dims->n_res_after; ++r)
    for (int q = 0; q < 2; ++q) p_after[r][q] = wp.add(w->res_after[r][2 * q], E, H, H, 0);
  GP_TRY(wp.run());
  if (chain) {
    float *dz, *dz_next;
    GP_TRY(wg.take(&dz));
    const float* z_next = nullptr;
    // a step and the gradients that come with it; the first one's operand is made from the gradient that was handed in
    auto step = [&](const float* W) -> gp_chain_step& {
      gp_chain_step& q = ch.add(W, H, H, 0);
      if (ch.n == 1) q.load = grad_m_out, q.load_z = z_first, q.load_out = dz;
      return q;
    };
    auto residual = [&](const float* hin, const float* const* wr, float* const* g, const res_saved& r) -> int {
      GP_TRY(wg.add(r.y1, dz, H, H, g[2], g[3]));
      GP_TRY(wg.take(&dz_next));
      gp_chain_step& s2 = step(wr[2]);
      s2.z = r.z1; s2.out2 = dz_next;
      dz = dz_next;
      GP_TRY(wg.add(hin, dz, H, H, g[0], g[1]));
      GP_TRY(wg.take(&dz_next));
      gp_chain_step& s1 = step(wr[0]);
      s1.add = dh; s1.out = next_buf(); s1.z = z_next; s1.out2 = dz_next;
      dh = s1.out;
      dz = dz_next;
      return GP_OK;
    };
    for (int r = dims->n_res_after - 1; r >= 0; --r) {
      z_next = r > 0 ? s.after[r - 1].z2 : s.z_lin;
      GP_TRY(residual(r == 0 ? s.h_lin : s.after[r - 1].hout, w->res_after[r], gw->res_after[r], s.after[r]));
    }
    keep = dh;
    GP_TRY(wg.add(dims->n_res_before > 0 ? s.before[dims->n_res_before - 1].hout : s.h0, dz, H, H, gw->W_lin, gw->b_lin));
    GP_TRY(wg.take(&dz_next));
    gp_chain_step& li = step(w->W_lin);
    li.out = next_buf(); li.z = dims->n_res_before > 0 ? s.before[dims->n_res_before - 1].z2 : s.z_up; li.out2 = dz_next;
    dh = li.out;
    dz = dz_next;
    for (int r = dims->n_res_before - 1; r >= 0; --r) {
      z_next = r > 0 ? s.before[r - 1].z2 : s.z_up;
      GP_TRY(residual(r == 0 ? s.h0 : s.before[r - 1].hout, w->res_before[r], gw->res_before[r], s.before[r]));
    }
    // h0 = x_ji + act(a W_up);  dh = dh0, dz = dz_up
    GP_TRY(wg.add(s.a, dz, F, H, gw->W_up, nullptr));
    ch.add(w->W_up, F, H, 0).out = sc.dF1;                        // da
    GP_TRY(wg.take(&dz_ji));
    dm_ji = next_buf();
    gp_chain_step& ji = ch.add(w->W_ji, H, H, 0);
    ji.load = dh; ji.load_z = s.z_ji; ji.load_out = dz_ji; ji.out = dm_ji;
    GP_TRY(wg.add(m_in, dz_ji, H, H, gw->W_ji, gw->b_ji));
    pre = ch.n;
    GP_TRY(wg.take(&dz_kj));
    GP_TRY(wg.take(&dgate));
    gp_chain_step& dn = ch.add(w->W_down, H, F, 0);
    dn.load = sc.dF2; dn.gate = 1; dn.z = s.z_kj; dn.mul = s.gate; dn.out2 = dz_kj; dn.out3 = dgate;
    gp_chain_step& kj = ch.add(w->W_kj, H, H, 0);                 // dm = kj path + ji path + skip
    kj.add_pre = dm_ji; kj.add = keep; kj.out = grad_m_in;
    GP_TRY(gp_chain_prepare(ctx, H, ch.s, ch.n, sc.planes, sc.planes_bytes));
    GP_TRY(gp_chain_run(ctx, H, ch.s, 0, pre, E, sc.planes));
    if (aux.active()) GP_TRY(wg.run());
  } else {
    float *dzcur, *dznext;
    GP_TRY(wg.take(&dzcur));
    GP_TRY(gp_ew_dsilu_mul(ctx, dh, z_first, dzcur, EH));

    // residual layers after the skip, last to first
    for (int r = dims->n_res_after - 1; r >= 0; --r) {
      const float* hin = (r == 0) ? s.h_lin : s.after[r - 1].hout;
      const float* z_next = (r > 0) ? s.after[r - 1].z2 : s.z_lin;
      float* out = next_buf();
      GP_TRY(res_backward(ctx, wg, hin, w->res_after[r], p_after[r], gw->res_after[r], s.after[r], dh, dzcur, out, z_next, &dznext, E, H));
      dh = out;
      dzcur = dznext;
    }
    // h_lin = act(h W_lin + b_lin) + m;  dzcur = dz_lin
    keep = dh;
    {
      const float* hin = dims->n_res_before > 0 ? s.before[dims->n_res_before - 1].hout : s.h0;
      const float* z_next = dims->n_res_before > 0 ? s.before[dims->n_res_before - 1].z2 : s.z_up;
      GP_TRY(wg.add(hin, dzcur, H, H, gw->W_lin, gw->b_lin));
      if (aux.active()) GP_TRY(wg.run());
      float* out = next_buf();
      GP_TRY(wg.take(&dznext));
      gp_epilogue e; e.out = out; e.out2 = dznext; e.z2src = z_next;
      GP_TRY(gp_gemm_nt_w(ctx, dzcur, w->W_lin, p_lin, E, H, H, e));
      dh = out;
      dzcur = dznext;
    }
    for (int r = dims->n_res_before - 1; r >= 0; --r) {
      const float* hin = (r == 0) ? s.h0 : s.before[r - 1].hout;
      const float* z_next = (r > 0) ? s.before[r - 1].z2 : s.z_up;
      float* out = next_buf();
      GP_TRY(res_backward(ctx, wg, hin, w->res_before[r], p_before[r], gw->res_before[r], s.before[r], dh, dzcur, out, z_next, &dznext, E, H));
      dh = out;
      dzcur = dznext;
    }
    // h0 = x_ji + act(a W_up);  dh = dh0, dzcur = dz_up
    // The branch through x_ji = act(m W_ji + b_ji) needs dh0 only: all of it (dz_ji, both gradients) runs on the side
    // stream next to the chain through the triplet sum, whose kernels leave much of the chip idle; its input gradient
    // is added by the epilogue of the last GEMM below.  The weight gradient first where it does not join a group: with the input gradient
    // ahead of it two blocks of 4656 edges x 512 take 2.51 ms instead of 2.44, of 5514 x 2048 13.4 instead of 13.2, of 5844 14.2 instead of
    // 14.0, of 1884 6.6 instead of 6.7, and at width 1024 the same.
    GP_TRY(wg.add(s.a, dzcur, F, H, gw->W_up, nullptr));
    GP_TRY(wg.take(&dz_ji, true));
    dm_ji = next_buf();
    GP_TRY(aux.on_aux(
        [&] {
          GP_TRY(gp_ew_dsilu_mul(ctx, dh, s.z_ji, dz_ji, EH));
          if (!wg.group) GP_TRY(gp_gemm_tn(ctx, m_in, dz_ji, E, H, H, gw->W_ji, gw->b_ji, sc.part_aux, sc.part_aux_bytes));
          gp_epilogue e; e.out = dm_ji;
          return gp_gemm_nt_w(ctx, dz_ji, w->W_ji, p_ji, E, H, H, e);
        },
        {dz_ji, dm_ji}));
    if (wg.group) GP_TRY(wg.add(m_in, dz_ji, H, H, gw->W_ji, gw->b_ji));
    if (aux.active()) GP_TRY(wg.run());
    {
      gp_epilogue e; e.out = sc.dF1;
      GP_TRY(gp_gemm_nt_w(ctx, dzcur, w->W_up, p_up, E, F, H, e));                                     // da
    }
  }
  // triplet interaction
  const bool bwd_mfma = bwd_mfma_D(ctx, dims, graph);
  {
    // the matrix-core backward kernel does without Bacc; the per-edge one needs what the forward call stored
    const auto it = ctx->fwd_flags.find(saved);
    if (!bwd_mfma && it != ctx->fwd_flags.end() && it->second == 0u)
      return gp_fail(ctx, GP_BAD_ARG, "gp_block_backward_D: the forward call of this `saved` buffer ran with the matrix-core triplet "
                     "kernels and kept no accumulator; gp_set_triplet_mfma must not change between forward and backward");
  }
  if (bwd_mfma)
    GP_TRY(gp_tripD_backward_mfma(ctx, graph, basis->cos_alpha_kj, s.x_kj, s.Q, w->W_sbf2, sc.dF1, s.z_dn, F, S, B,
                                  sc.dF2, sc.dQ, gw->W_sbf2, sc.part, sc.part_bytes));        // dz_dn, dQ, dW_sbf2
  else
    GP_TRY(gp_tripD_backward(ctx, graph, basis->cos_alpha_kj, s.x_kj, s.Q, w->W_sbf2, sc.dF1, s.z_dn, F, S, B,
                             sc.dF2, sc.dQ));                                                 // dz_dn, dQ
  // weight gradients that nothing below waits for: side stream (its own split-K buffer; its kernels run in order)
  GP_TRY(aux.on_aux(
      [&] {
        return gp_tripD_weight_grads(ctx, sc.dF1, bwd_mfma ? nullptr : s.Bacc, basis->rad, sc.dQ, E, F, S, R, B, gw->W_sbf2,
                                     gw->W_sbf1, sc.part_aux, sc.part_aux_bytes);
      },
      {}));
  // gradients with respect to the basis (forces, Sec. 3.2): radial part of the spherical basis from grad_Q, cos(alpha)
  // through the per-edge factor P and the kernel the bilinear block uses for the same contraction
  if (grad_rad) {
    const int64_t n = E * S * R;
    grad_rad_kernel<<<(unsigned)((n + 255) / 256), 256, 0, ctx->stream>>>(sc.dQ, w->W_sbf1, E, S, R, B, accumulate_basis_grads, grad_rad);
    GP_LAUNCH_CHECK(ctx, "grad_rad_kernel");
  }
  if (grad_cos_kj && graph->n_triplets > 0) {
    const int64_t n = E * S * F;
    cos_factor_kernel<<<(unsigned)((n + 255) / 256), 256, 0, ctx->stream>>>(s.x_kj, w->W_sbf2, s.Q, E, S, B, F, sc.P);
    GP_LAUNCH_CHECK(ctx, "cos_factor_kernel");
    GP_TRY(gp_tripG_grad_cos(ctx, graph, basis->cos_alpha_kj, sc.P, sc.dF1, F, S, accumulate_basis_grads, grad_cos_kj));
  }
  GP_TRY(wg.add(s.xg, sc.dF2, H, F, gw->W_down, nullptr));
  if (chain) {
    GP_TRY(gp_chain_run(ctx, H, ch.s, pre, ch.n, E, sc.planes));   // dz_kj, dgate and the result
  } else {
    GP_TRY(wg.take(&dz_kj));
    GP_TRY(wg.take(&dgate));
    // dxg = dF2 W_down^T is not stored where its epilogue can take the gate apart (two launches: 26 + 48 us at 43380 x 256): planes, and
    // buffers that start on 16 bytes
    bool gate_fused = p_down != nullptr;
    for (const void* p : {(const void*)sc.dF2, (const void*)s.z_kj, (const void*)s.gate, (const void*)dz_kj, (const void*)dgate})
      gate_fused = gate_fused && ((uintptr_t)p & 15) == 0;
    if (gate_fused) {
      gp_epilogue e; e.act = 3; e.zsrc = s.z_kj; e.mul = s.gate; e.out = dz_kj; e.out2 = dgate;
      GP_TRY(gp_gemm_nt_w(ctx, sc.dF2, w->W_down, p_down, E, H, F, e));                        // dz_kj, dgate
    } else {
      float* dxg;
      GP_TRY(wg.take(&dxg));
      gp_epilogue e; e.out = dxg;
      GP_TRY(gp_gemm_nt(ctx, sc.dF2, w->W_down, E, H, F, e));
      GP_TRY(gp_ew_gate_bwd(ctx, dxg, s.z_kj, s.gate, dz_kj, dgate, EH));                      // dz_kj, dgate
    }
  }
  // The radial gate's gradients join the others of a group; one by one they stay on the main stream, which has less to do by then.
  auto factors = [&] { return gp_factor_grads(ctx, sc.dWrbf, w->W_rbf1, w->W_rbf2, R, B, H, gw->W_rbf1, gw->W_rbf2); };
  if (wg.group) {
    GP_TRY(wg.add(basis->rbf, dgate, R, H, sc.dWrbf, nullptr));
  } else {
    GP_TRY(gp_gemm_tn(ctx, basis->rbf, dgate, E, R, H, sc.dWrbf, nullptr, sc.part, sc.part_bytes));
    GP_TRY(factors());
  }
  if (grad_rbf) {   // dL/drbf = dgate W_rbf^T
    gp_epilogue e; e.out = grad_rbf;
    if (accumulate_basis_grads) e.add_post = grad_rbf;
    GP_TRY(gp_gemm_nt(ctx, dgate, s.Wrbf, E, R, H, e));
  }
  GP_TRY(wg.add(m_in, dz_kj, H, H, gw->W_kj, gw->b_kj));
  GP_TRY(wg.run());
  if (wg.group) GP_TRY(aux.on_aux(factors, {}));
  if (!chain) {
    GP_TRY(aux.before_write(dm_ji));   // the side stream's input gradient of the ji path
    gp_epilogue e; e.add_pre = dm_ji; e.add_post = keep; e.out = grad_m_in;
    GP_TRY(gp_gemm_nt_w(ctx, dz_kj, w->W_kj, p_kj, E, H, H, e));                                     // dm = kj path + ji path + skip
  }
  return aux.join();
}

}  // namespace

extern "C" {

int gp_block_backward_D(gp_ctx* ctx, const gp_dims* dims, const gp_weights_D* w, const gp_graph* graph,
                        const gp_basis* basis, const float* m_in, const void* saved, size_t saved_bytes,
                        const float* grad_m_out, float* grad_m_in, gp_weights_D* gw, void* scratch,
                        size_t scratch_bytes) {
  return backward_D(ctx, dims, w, graph, basis, m_in, saved, saved_bytes, grad_m_out, grad_m_in, gw, nullptr, nullptr, nullptr, 0,
                    scratch, scratch_bytes);
}

int gp_block_backward_D_basis(gp_ctx* ctx, const gp_dims* dims, const gp_weights_D* w, const gp_graph* graph,
                              const gp_basis* basis, const float* m_in, const void* saved, size_t saved_bytes,
                              const float* grad_m_out, float* grad_m_in, gp_weights_D* gw, float* grad_rbf, float* grad_rad,
                              float* grad_cos_kj, int32_t accumulate_basis_grads, void* scratch, size_t scratch_bytes) {
  return backward_D(ctx, dims, w, graph, basis, m_in, saved, saved_bytes, grad_m_out, grad_m_in, gw, grad_rbf, grad_rad,
                    grad_cos_kj, accumulate_basis_grads, scratch, scratch_bytes);
}

}  // extern "C"
