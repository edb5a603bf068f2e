// Radius-graph construction and triplet enumeration (paper Sec. 3.1; the index set
// N_j \ {i} of the update equation in Sec. 3.3).  Integer outputs are bit-exact and
// deterministic: positions are compared with an uncontracted fp32 expression, output
// slots come from wavefront ballots and prefix counts, never from atomics' arrival order.
#include <stdarg.h>

#include <atomic>
#include <chrono>

#include "common.h"

namespace {

// ------------------------------------------------------------------ exclusive scan
// One workgroup walks the array in chunks of its own size, carrying the running total.
// in[n] (int32) -> out[n+1] (int32, exclusive prefix, out[n] = total); host_total, a word of pinned host memory, gets the
// untruncated sum so the host can detect int32 overflow.
constexpr int SCAN_THREADS = 1024;
__global__ void __launch_bounds__(SCAN_THREADS)
scan_exclusive_kernel(const int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t n,
                      int64_t* __restrict__ host_total) {
  __shared__ int64_t wave_tot[SCAN_THREADS / WAVE];
  __shared__ int64_t carry_s;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) carry_s = 0;
  __syncthreads();
  for (int64_t base = 0; base < n; base += SCAN_THREADS) {
    int64_t i = base + tid;
    int64_t v = (i < n) ? (int64_t)in[i] : 0;
    int64_t incl = v;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      int64_t u = __shfl_up(incl, o, WAVE);
      if (lane >= o) incl += u;
    }
    if (lane == WAVE - 1) wave_tot[w] = incl;
    __syncthreads();
    int64_t before = carry_s;
    for (int k = 0; k < w; ++k) before += wave_tot[k];
    if (i < n) out[i] = (int32_t)(before + incl - v);
    __syncthreads();
    if (tid == SCAN_THREADS - 1) carry_s = before + incl;
    __syncthreads();
  }
  // The host goes on when it sees the total: by then all that this workgroup wrote is visible to every stream (the barrier orders the
  // workgroup's stores before the release), and nothing of the workspace is touched any more.
  if (tid == 0) {
    out[n] = (int32_t)carry_s;
    __hip_atomic_store(host_total, carry_s, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ------------------------------------------------------------------ edges
// The distance predicate: every operation rounded once to fp32, no fused multiply-add.
__device__ __forceinline__ float dist2_f32(float xi, float yi, float zi, float xj, float yj, float zj) {
#pragma clang fp contract(off)
  float dx = __fsub_rn(xi, xj), dy = __fsub_rn(yi, yj), dz = __fsub_rn(zi, zj);
  return __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
}

// Periodic images tested per source atom: n_a = -rep[a] .. rep[a]; image index img counts them in
// lexicographic order of (n0, n1, n2).  Without a cell there is the one image n = 0.
struct images_t {
  const float* cell;   // [G, 3, 3] rows = lattice vectors, or NULL
  int r0, r1, r2;
  __host__ __device__ int count() const { return cell ? (2 * r0 + 1) * (2 * r1 + 1) * (2 * r2 + 1) : 1; }
};

// shift of image (n0, n1, n2) of structure g: n0 a0 + n1 a1 + n2 a2, every product and sum rounded once
__device__ __forceinline__ void image_of(const images_t& im, int g, int img, int& n0, int& n1, int& n2, float& sx,
                                         float& sy, float& sz) {
#pragma clang fp contract(off)
  if (!im.cell) {
    n0 = n1 = n2 = 0;
    sx = sy = sz = 0.f;
    return;
  }
  const int w2 = 2 * im.r2 + 1, w1 = 2 * im.r1 + 1;
  n2 = img % w2 - im.r2;
  n1 = (img / w2) % w1 - im.r1;
  n0 = img / (w2 * w1) - im.r0;
  const float* c = im.cell + 9 * (int64_t)g;
  const float f0 = (float)n0, f1 = (float)n1, f2 = (float)n2;
  sx = __fadd_rn(__fadd_rn(__fmul_rn(f0, c[0]), __fmul_rn(f1, c[3])), __fmul_rn(f2, c[6]));
  sy = __fadd_rn(__fadd_rn(__fmul_rn(f0, c[1]), __fmul_rn(f1, c[4])), __fmul_rn(f2, c[7]));
  sz = __fadd_rn(__fadd_rn(__fmul_rn(f0, c[2]), __fmul_rn(f1, c[5])), __fmul_rn(f2, c[8]));
}

// One wavefront per target atom i; candidates are (source atom j, image) pairs in the order
// (j, image index), the atom itself (j = i, n = 0) left out.  FILL = false: deg[i] = number of kept
// candidates.  FILL = true: write them in that order at row_ptr[i].
//
// The cap keeps the max_nb smallest keys (bits(d2), candidate order).  bits(d2) of a non-negative float orders like the
// float, so the count pass finds the max_nb-th smallest value by bisection over the 31 bits and leaves it with the number of
// candidates of exactly that value that are kept, cap[i] = {value, how many}; the fill pass then only compares.  The values
// in range are collected in LDS in candidate order and counted from registers, CAP_LDS per wavefront; an atom with more of
// them evaluates its candidates again in every step of the bisection.  (Ranking every candidate against every other one,
// which this replaces, took 2.2 ms per pass for 5 periodic slabs of 61 atoms x 25 images; this takes 14 us to count and 10 to fill.)
constexpr int CAP_LDS = 512;
template <bool FILL>
__global__ void __launch_bounds__(256)
edges_kernel(const float* __restrict__ pos, const int32_t* __restrict__ graph_ptr, int n_atoms,
             int n_graphs, float c2, int max_nb, images_t im, int32_t* __restrict__ deg, uint2* __restrict__ cap,
             const int32_t* __restrict__ row_ptr, int32_t* __restrict__ row_out, int32_t* __restrict__ src,
             int32_t* __restrict__ dst, int32_t* __restrict__ offset, float* __restrict__ dist, float* __restrict__ unit) {
  __shared__ uint32_t near_s[FILL ? 1 : 256 / WAVE][FILL ? 1 : CAP_LDS];
  const int i = blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x >> 6);
  if (i >= n_atoms) return;
  const int lane = lane_id();
  // structure containing atom i: largest g with graph_ptr[g] <= i
  int lo_g = 0, hi_g = n_graphs;
  while (hi_g - lo_g > 1) {
    int mid = (lo_g + hi_g) >> 1;
    if (graph_ptr[mid] <= i) lo_g = mid; else hi_g = mid;
  }
  const int lo = graph_ptr[lo_g], hi = graph_ptr[lo_g + 1];
  const float xi = pos[3 * i], yi = pos[3 * i + 1], zi = pos[3 * i + 2];
  const int NI = im.count();
  const int centre = im.cell ? ((im.r0 * (2 * im.r1 + 1) + im.r1) * (2 * im.r2 + 1) + im.r2) : 0;
  const int n_cand = (hi - lo) * NI;
  const int self_q = (i - lo) * NI + centre;

  // squared distance from atom i to candidate q (and where that candidate sits)
  auto cand_d2 = [&](int q, int& j, int& n0, int& n1, int& n2, float& xs, float& ys, float& zs) -> float {
    j = lo + q / NI;
    float sx, sy, sz;
    image_of(im, lo_g, q % NI, n0, n1, n2, sx, sy, sz);
    xs = __fadd_rn(pos[3 * j], sx);
    ys = __fadd_rn(pos[3 * j + 1], sy);
    zs = __fadd_rn(pos[3 * j + 2], sz);
    return dist2_f32(xi, yi, zi, xs, ys, zs);
  };
  // the same for a candidate that may be past the end: evaluated at a valid one, so that the loads of several rounds stay in
  // flight together; in_range says whether it counts
  auto cand_in = [&](int q, float& d2) -> bool {
    int j, n0, n1, n2;
    float xs, ys, zs;
    d2 = cand_d2(q < n_cand ? q : n_cand - 1, j, n0, n1, n2, xs, ys, zs);
    return q < n_cand && q != self_q && d2 < c2;
  };

  if (!FILL) {
    uint32_t* near = near_s[threadIdx.x >> 6];
    int total = 0;
    for (int base = 0; base < n_cand; base += 4 * WAVE) {
      float d2[4];
      bool in[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) in[u] = cand_in(base + u * WAVE + lane, d2[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t mask = __ballot(in[u]);
        const int at = total + mbcnt(mask);
        if (max_nb > 0 && in[u] && at < CAP_LDS) near[at] = __float_as_uint(d2[u]);
        total += __popcll(mask);
      }
    }
    uint2 keep_below = make_uint2(0xffffffffu, 0u);
    if (max_nb > 0 && total > max_nb) {
      const bool listed = total <= CAP_LDS;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the list is this wavefront's own
      __builtin_amdgcn_wave_barrier();
      uint32_t v[CAP_LDS / WAVE];
#pragma unroll
      for (int k = 0; k < CAP_LDS / WAVE; ++k)   // slots past the end count nowhere
        v[k] = listed && k * WAVE + lane < total ? near[k * WAVE + lane] : 0xffffffffu;
      // number of candidates in range with bits(d2) <= t
      auto count_le = [&](uint32_t t) -> int {
        int c = 0;
        if (listed) {
#pragma unroll
          for (int k = 0; k < CAP_LDS / WAVE; ++k) c += __popcll(__ballot(v[k] <= t));
        } else {
          for (int base = 0; base < n_cand; base += WAVE) {
            float d2;
            const bool in = cand_in(base + lane, d2);
            c += __popcll(__ballot(in && __float_as_uint(d2) <= t));
          }
        }
        return c;
      };
      uint32_t a = 0, b = __float_as_uint(c2);   // the smallest t with count_le(t) >= max_nb lies in a .. b
      while (a < b) {
        const uint32_t mid = a + ((b - a) >> 1);
        if (count_le(mid) >= max_nb) b = mid; else a = mid + 1;
      }
      keep_below = make_uint2(a, (uint32_t)(max_nb - (a > 0 ? count_le(a - 1) : 0)));
      total = max_nb;
    }
    if (lane == 0) {
      deg[i] = total;
      if (max_nb > 0) cap[i] = keep_below;
    }
    return;
  }

  const uint2 keep_below = max_nb > 0 ? cap[i] : make_uint2(0xffffffffu, 0u);
  const int row = row_ptr[i];
  if (lane == 0) {
    row_out[i] = row;
    if (i == n_atoms - 1) row_out[n_atoms] = row_ptr[n_atoms];
  }
  int total = 0;
  uint32_t ties = 0;   // candidates of exactly the last kept value so far
  for (int base = 0; base < n_cand; base += WAVE) {
    const int q = base + lane;
    int j, n0, n1, n2;
    float xs, ys, zs;
    const float d2 = cand_d2(q < n_cand ? q : n_cand - 1, j, n0, n1, n2, xs, ys, zs);
    const bool in = q < n_cand && q != self_q && d2 < c2;
    const uint32_t bits = __float_as_uint(d2);
    const uint64_t tie = __ballot(in && bits == keep_below.x);
    const bool keep = in && (bits < keep_below.x || (bits == keep_below.x && ties + mbcnt(tie) < keep_below.y));
    ties += __popcll(tie);
    const uint64_t mask = __ballot(keep);
    if (keep) {
      const int slot = row + total + mbcnt(mask);
      src[slot] = j;
      dst[slot] = i;
      if (offset) {
        offset[3 * slot + 0] = n0;
        offset[3 * slot + 1] = n1;
        offset[3 * slot + 2] = n2;
      }
      if (dist || unit) {
        float d = sqrtf(d2);
        if (dist) dist[slot] = d;
        if (unit) {
          float inv = 1.0f / d;
          unit[3 * slot + 0] = (xi - xs) * inv;
          unit[3 * slot + 1] = (yi - ys) * inv;
          unit[3 * slot + 2] = (zi - zs) * inv;
        }
      }
    }
    total += __popcll(mask);
  }
}

// ------------------------------------------------------------------ triplets
// Position, inside rows b .. b+n of an edge list sorted by (source, cell offset), of the edge with
// source v and offset (t0, t1, t2); -1 if there is none.  off == NULL: open boundaries, all offsets zero.
__device__ __forceinline__ int find_edge(const int32_t* __restrict__ src, const int32_t* __restrict__ off, int b, int n,
                                         int v, int t0, int t1, int t2) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1, e = b + mid;
    bool less = src[e] < v;
    if (off && src[e] == v) {
      const int o0 = off[3 * e], o1 = off[3 * e + 1], o2 = off[3 * e + 2];
      less = o0 < t0 || (o0 == t0 && (o1 < t1 || (o1 == t1 && o2 < t2)));
    }
    if (less) lo = mid + 1; else hi = mid;
  }
  if (lo >= n || src[b + lo] != v) return -1;
  if (off && (off[3 * (b + lo)] != t0 || off[3 * (b + lo) + 1] != t1 || off[3 * (b + lo) + 2] != t2)) return -1;
  return lo;
}

// The lists of a graph.  For an edge e = (j->i) let opp(e) = id_swap[e] be the edge (i->j) with the negated cell offset, -1 if
// the list has none.  The triplets of target edge e are the in-edges of j minus opp(e); those of source edge e' = (k->j) are
// the out-edges of j minus opp(e').  Everything follows from opp: links_kernel finds it (and counts the out-edges of every
// atom), lists_sums / lists_mid / lists_apply turn the segment lengths into offsets for both orders at once, out_lists_kernel
// orders the out-edges of every atom, triplet_fill_kernel writes both orders.  (Each list used to be built by kernels of its
// own, with the opposite edge searched three times, five scans and four waits of the host: 27 launches where this takes 7.)

// id_swap[e] = opp(e); arrival[e] = how many edges of the same source came before (in the order the atomics happen to run)
__global__ void __launch_bounds__(256)
links_kernel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, const int32_t* __restrict__ off,
             const int32_t* __restrict__ row_ptr, int n_edges, int32_t* __restrict__ id_swap, int32_t* __restrict__ out_deg,
             int32_t* __restrict__ arrival) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_edges) return;
  const int j = src[e], i = dst[e];
  const int b = row_ptr[j], n = row_ptr[j + 1] - b;
  const int p = off ? find_edge(src, off, b, n, i, -off[3 * (int64_t)e], -off[3 * (int64_t)e + 1], -off[3 * (int64_t)e + 2])
                    : find_edge(src, nullptr, b, n, i, 0, 0, 0);
  id_swap[e] = p >= 0 ? b + p : -1;
  if (out_deg) arrival[e] = atomicAdd(&out_deg[j], 1);
}

// number of triplets of edge e as the target and, with KJ, as the source edge
template <bool KJ>
__device__ __forceinline__ int2 triplet_counts(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                               const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ id_swap,
                                               const int32_t* __restrict__ out_deg, int64_t e) {
  const int j = src[e], has = id_swap[e] >= 0 ? 1 : 0;
  return make_int2(row_ptr[j + 1] - row_ptr[j] - has, KJ ? out_deg[dst[e]] - has : 0);
}

// Sum over the 4 or 16 wavefronts of a workgroup; every thread must call it.  Returns the exclusive prefix of v over the
// threads and the total of the workgroup; lds holds one value per wavefront and is free again after the next barrier.
template <class T>
__device__ __forceinline__ T block_prefix(T v, T* lds, T* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  T incl = v;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const T u = __shfl_up(incl, o, WAVE);
    if (lane >= o) incl += u;
  }
  if (lane == WAVE - 1) lds[w] = incl;
  __syncthreads();
  T before = 0, all = 0;
  for (int k = 0; k < nw; ++k) {
    before += k < w ? lds[k] : 0;
    all += lds[k];
  }
  *total = all;
  return before + incl - v;
}

constexpr int CHUNK = 1024;   // edges per workgroup of the two edge-wide passes, 4 per thread
inline int64_t chunks_of(int64_t n) { return (n + CHUNK - 1) / CHUNK; }

template <bool KJ>
__global__ void __launch_bounds__(256)
lists_sums_kernel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, const int32_t* __restrict__ row_ptr,
                  const int32_t* __restrict__ id_swap, const int32_t* __restrict__ out_deg, int64_t n_edges,
                  int64_t* __restrict__ sums /*[chunks][2]*/) {
  __shared__ int64_t lds[2][4];
  int64_t a = 0, b = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t e = (int64_t)blockIdx.x * CHUNK + u * 256 + threadIdx.x;
    if (e < n_edges) {
      const int2 c = triplet_counts<KJ>(src, dst, row_ptr, id_swap, out_deg, e);
      a += c.x;
      b += c.y;
    }
  }
  int64_t ta, tb;
  block_prefix(a, lds[0], &ta);
  block_prefix(b, lds[1], &tb);
  if (threadIdx.x == 0) {
    sums[2 * (int64_t)blockIdx.x] = ta;
    sums[2 * (int64_t)blockIdx.x + 1] = tb;
  }
}

// One workgroup: out_ptr from out_deg and the largest degrees (not with n_atoms = 0), the chunks' offsets; host (pinned memory, or
// NULL) = {triplets, largest in-degree, largest out-degree}.
__global__ void __launch_bounds__(1024)
lists_mid_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ out_deg, int n_atoms, int64_t n_chunks,
                 int32_t* __restrict__ out_ptr, int64_t* __restrict__ sums, int64_t* __restrict__ total,
                 int64_t* __restrict__ host) {
  __shared__ int32_t lds_i[2][16];
  __shared__ int64_t lds_l[2][2][16];
  __shared__ int32_t red[2][16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int carry_out = 0, max_in = 0, max_out = 0, flip = 0;
  for (int base = 0; base < n_atoms; base += 1024, flip ^= 1) {   // two sets of LDS words: one barrier per scan
    const int j = base + tid;
    const int d = j < n_atoms ? row_ptr[j + 1] - row_ptr[j] : 0, o = j < n_atoms ? out_deg[j] : 0;
    max_in = max_in > d ? max_in : d;
    max_out = max_out > o ? max_out : o;
    int tot_o;
    const int po = carry_out + block_prefix(o, lds_i[flip], &tot_o);
    if (j < n_atoms) out_ptr[j] = po;
    carry_out += tot_o;
  }
  int64_t carry_a = 0, carry_b = 0;
  flip = 0;
  for (int64_t base = 0; base < n_chunks; base += 1024, flip ^= 1) {
    const int64_t c = base + tid;
    int64_t ta, tb;
    const int64_t pa = carry_a + block_prefix(c < n_chunks ? sums[2 * c] : (int64_t)0, lds_l[flip][0], &ta);
    const int64_t pb = carry_b + block_prefix(c < n_chunks ? sums[2 * c + 1] : (int64_t)0, lds_l[flip][1], &tb);
    if (c < n_chunks) {
      sums[2 * c] = pa;
      sums[2 * c + 1] = pb;
    }
    carry_a += ta;
    carry_b += tb;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int u = __shfl_xor(max_in, o, 64), v = __shfl_xor(max_out, o, 64);
    max_in = u > max_in ? u : max_in;
    max_out = v > max_out ? v : max_out;
  }
  if (lane == 0) { red[0][w] = max_in; red[1][w] = max_out; }
  __syncthreads();
  if (tid == 0) {
    for (int k = 1; k < 16; ++k) {
      max_in = red[0][k] > max_in ? red[0][k] : max_in;
      max_out = red[1][k] > max_out ? red[1][k] : max_out;
    }
    out_ptr[n_atoms] = carry_out;
    *total = carry_a;
    if (host) {
      host[0] = carry_a;
      host[1] = max_in;
      host[2] = max_out;
    }
  }
}

// seg_ji from the chunks' offsets; with KJ also seg_kj, and the out-edges of every atom in arrival order
template <bool KJ>
__global__ void __launch_bounds__(256)
lists_apply_kernel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, const int32_t* __restrict__ row_ptr,
                   const int32_t* __restrict__ id_swap, const int32_t* __restrict__ out_deg, const int32_t* __restrict__ out_ptr,
                   const int32_t* __restrict__ arrival, int64_t n_edges, const int64_t* __restrict__ sums,
                   const int64_t* __restrict__ total, int32_t* __restrict__ seg_ji, int32_t* __restrict__ seg_kj,
                   int32_t* __restrict__ out_tmp) {
  __shared__ int64_t lds[2][4];
  const int64_t e0 = (int64_t)blockIdx.x * CHUNK + 4 * (int64_t)threadIdx.x;
  int2 c[4];
  int64_t a = 0, b = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    c[u] = e0 + u < n_edges ? triplet_counts<KJ>(src, dst, row_ptr, id_swap, out_deg, e0 + u) : make_int2(0, 0);
    a += c[u].x;
    b += c[u].y;
  }
  int64_t ta, tb;
  int64_t pa = sums[2 * (int64_t)blockIdx.x] + block_prefix(a, lds[0], &ta);
  int64_t pb = sums[2 * (int64_t)blockIdx.x + 1] + block_prefix(b, lds[1], &tb);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t e = e0 + u;
    if (e < n_edges) {
      seg_ji[e] = (int32_t)pa;
      if (KJ) {
        seg_kj[e] = (int32_t)pb;
        out_tmp[out_ptr[src[e]] + arrival[e]] = (int32_t)e;
      }
    }
    pa += c[u].x;
    pb += c[u].y;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    seg_ji[n_edges] = (int32_t)*total;
    if (KJ) seg_kj[n_edges] = (int32_t)*total;
  }
}

// Out-edges of every atom in ascending edge id, one workgroup per atom.  With open boundaries the in-edges of j come sorted by
// their source k and the edges j->k by k as well: where every out-edge is the opposite of an in-edge (always so without a
// cap) the list is opp of the in-edges with the gaps closed, no sorting (74 -> 10 us for the lists of 300 on average of the
// 1000-atom box).
__global__ void __launch_bounds__(256)
out_lists_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ id_swap, const int32_t* __restrict__ out_ptr,
                 const int32_t* __restrict__ out_tmp, int periodic, int32_t* __restrict__ out_list) {
  __shared__ int32_t lds[SORT_LDS];
  __shared__ int32_t cnt[2][4];
  const int j = blockIdx.x;
  const int b = out_ptr[j], n = out_ptr[j + 1] - b;
  const int r0 = row_ptr[j], d = row_ptr[j + 1] - r0;
  if (!periodic) {
    int have = 0;
    for (int r = threadIdx.x; r < d; r += 256) have += id_swap[r0 + r] >= 0 ? 1 : 0;
    int all;
    block_prefix(have, cnt[0], &all);
    if (all == n) {
      int done = 0, flip = 1;
      for (int base = 0; base < d; base += 256, flip ^= 1) {
        const int e = base + (int)threadIdx.x < d ? id_swap[r0 + base + threadIdx.x] : -1;
        int tot;
        const int at = done + block_prefix(e >= 0 ? 1 : 0, cnt[flip], &tot);
        if (e >= 0) out_list[b + at] = e;
        done += tot;
      }
      return;
    }
  }
  sort_list_block(out_tmp + b, n, out_list + b, lds);
}

// Both orders of the triplets.  Workgroups [0, ji_blocks): LANES lanes per target edge e = (j->i), whose triplets are the in-edge
// rows of j minus opp(e).  The others: teams (see run_team) of in-edge rows e' = (k->j), whose triplets are the out-edges of j
// minus opp(e').  Bound by the 16 bytes written per triplet: 1e8 triplets in 0.40 ms, 4.0 TB/s.
template <bool LONG>
__global__ void __launch_bounds__(256)
triplet_fill_kernel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, const int32_t* __restrict__ row_ptr,
                    const int32_t* __restrict__ id_swap, const int32_t* __restrict__ out_ptr, const int32_t* __restrict__ out_list,
                    const int32_t* __restrict__ seg_ji, const int32_t* __restrict__ seg_kj, int n_edges, int ji_blocks,
                    int32_t* __restrict__ idx_kj, int32_t* __restrict__ idx_ji, int32_t* __restrict__ perm_kj,
                    int32_t* __restrict__ idx_ji_kj) {
  using R = run_team<LONG>;
  __shared__ __align__(16) int32_t t_e[R::TEAMS][R::CHUNK + 4], t_first[R::TEAMS][R::CHUNK + 4], t_back[R::TEAMS][R::CHUNK + 4];
  __shared__ int32_t t_gap[R::TEAMS][R::ROWS];
  const int lane = lane_id(), team = threadIdx.x / R::TEAM, tid = threadIdx.x % R::TEAM;
  const int par = tid / R::LANES, ln = tid % R::LANES;
  if ((int)blockIdx.x < ji_blocks) {
    const int e = blockIdx.x * (256 / R::LANES) + threadIdx.x / R::LANES;
    if (e >= n_edges) return;
    const int j = src[e], r0 = row_ptr[j], n = row_ptr[j + 1] - r0, opp = id_swap[e], seg = seg_ji[e];
    const int cnt = n - (opp >= 0 ? 1 : 0), gap = opp >= 0 ? opp - r0 : INT32_MAX;
    const int same[5] = {e, e, e, e, e};
    for (int s0 = 4 * ln; s0 < cnt; s0 += 4 * R::LANES) {
      const int row[5] = {r0 + s0, r0 + s0 + 1, r0 + s0 + 2, r0 + s0 + 3, r0 + s0 + 4};
      store_run4<int4u>(idx_kj + seg, s0, cnt, gap, row);
      store_run4<int4u>(idx_ji + seg, s0, cnt, gap, same);
    }
    return;
  }
  const int p0 = (((int)blockIdx.x - ji_blocks) * R::TEAMS + team) * R::ROWS;
  if (p0 >= n_edges) return;   // the whole team
  const int n_own = n_edges - p0 < R::ROWS ? n_edges - p0 : R::ROWS;
  // lane u holds row u of the team
  const int pl = p0 + (lane < n_own ? lane : 0), jl = dst[pl], oppl = id_swap[pl], segl = seg_kj[pl];
  for (int done = 0; done < n_own;) {
    const int atom = __builtin_amdgcn_readlane(jl, done);
    const int len = __popcll(__ballot(lane < n_own && lane >= done && jl == atom));
    const int r0 = row_ptr[atom], ob = out_ptr[atom], n = out_ptr[atom + 1] - ob;
    const int base = p0 + done;   // first row of the run of equal atoms
    for (int b0 = 0; b0 < n; b0 += R::CHUNK) {
      team_sync<LONG>();   // the previous chunk has been consumed
      if (b0 == 0)
        for (int u = tid; u < R::ROWS; u += R::TEAM) t_gap[team][u] = INT32_MAX;
      team_sync<LONG>();
      for (int q = tid; q < R::CHUNK + 4 && b0 + q < n; q += R::TEAM) {
        const int e = out_list[ob + b0 + q], back = id_swap[e];
        t_e[team][q] = e;
        t_first[team][q] = seg_ji[e] - r0;
        t_back[team][q] = back >= 0 ? back : INT32_MAX;
        if (back >= base && back < base + len) t_gap[team][back - base] = b0 + q;
      }
      team_sync<LONG>();
      for (int u = par; u < len; u += R::PAR) {
        const int opp = __shfl(oppl, done + u, WAVE), seg = __shfl(segl, done + u, WAVE), row = base + u, gap = t_gap[team][u];
        const int cnt = n - (opp >= 0 ? 1 : 0), end = cnt < b0 + R::CHUNK ? cnt : b0 + R::CHUNK;
        for (int s0 = b0 + 4 * ln; s0 < end; s0 += 4 * R::LANES) {
          const int q = s0 - b0;
          const int4 e4 = *reinterpret_cast<const int4*>(&t_e[team][q]), f4 = *reinterpret_cast<const int4*>(&t_first[team][q]),
                     k4 = *reinterpret_cast<const int4*>(&t_back[team][q]);
          const int oe[5] = {e4.x, e4.y, e4.z, e4.w, t_e[team][q + 4]};
          const int first[5] = {f4.x, f4.y, f4.z, f4.w, t_first[team][q + 4]}, back[5] = {k4.x, k4.y, k4.z, k4.w, t_back[team][q + 4]};
          int t[5];
#pragma unroll
          for (int i = 0; i < 5; ++i) t[i] = first[i] + row - (row > back[i] ? 1 : 0);
          store_run4<int4u>(perm_kj + seg, s0, cnt, gap, t);
          store_run4<int4u>(idx_ji_kj + seg, s0, cnt, gap, oe);
        }
      }
    }
    done += len;
  }
}

struct edges_ws {
  int32_t* deg;      // [N]
  int32_t* row_ptr;  // [N+1]
  uint2* cap;        // [N] largest kept squared distance of a capped atom and how many of that value are kept
};
inline size_t carve_edges(void* p, int64_t n_atoms, edges_ws* w) {
  gp_carver c(p);
  w->deg = c.take<int32_t>(n_atoms);
  w->row_ptr = c.take<int32_t>(n_atoms + 1);
  w->cap = c.take<uint2>(n_atoms);
  return c.off;
}

struct triplets_ws {
  int32_t *id_swap, *seg_ji, *seg_kj, *out_list, *out_ptr;   // the lists, for callers that do not take them
  int32_t *arrival, *out_tmp, *out_deg;
  int64_t *sums, *total;                                     // chunk sums of the two segment lengths, number of triplets
};
inline size_t carve_triplets(void* p, int64_t n_atoms, int64_t n_edges, triplets_ws* w) {
  gp_carver c(p);
  w->id_swap = c.take<int32_t>(n_edges);
  w->seg_ji = c.take<int32_t>(n_edges + 1);
  w->seg_kj = c.take<int32_t>(n_edges + 1);
  w->out_list = c.take<int32_t>(n_edges);
  w->out_ptr = c.take<int32_t>(n_atoms + 1);
  w->arrival = c.take<int32_t>(n_edges);
  w->out_tmp = c.take<int32_t>(n_edges);
  w->out_deg = c.take<int32_t>(n_atoms);
  w->sums = c.take<int64_t>(2 * (size_t)chunks_of(n_edges));
  w->total = c.take<int64_t>(1);
  return c.off;
}

inline int blocks_for(int64_t n, int per_block) { return (int)((n + per_block - 1) / per_block); }

// largest ptr[i+1] - ptr[i]; one workgroup
__global__ void __launch_bounds__(1024)
max_degree_kernel(const int32_t* __restrict__ ptr, int64_t n, int32_t* __restrict__ out) {
  __shared__ int red[16];
  int m = 0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
    const int d = ptr[i + 1] - ptr[i];
    m = d > m ? d : m;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int v = __shfl_xor(m, o, 64);
    m = v > m ? v : m;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = red[w] > m ? red[w] : m;
    *out = m;
  }
}

}  // namespace

extern "C" {

int gp_reverse_edges(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset,
                     const int32_t* row_ptr, int64_t n_atoms, int64_t n_edges, int32_t* id_swap) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, n_atoms >= 0 && n_edges >= 0, "gp_reverse_edges: negative size");
  if (n_edges > INT32_MAX - 1 || n_atoms > INT32_MAX - 1) return gp_fail(ctx, GP_INT32_OVERFLOW, "gp_reverse_edges: sizes exceed int32");
  if (n_edges == 0) return GP_OK;
  GP_REQUIRE(ctx, src && dst && row_ptr && id_swap, "gp_reverse_edges: NULL pointer");
  GP_HIP(ctx, hipSetDevice(ctx->device));
  links_kernel<<<blocks_for(n_edges, 256), 256, 0, ctx->stream>>>(src, dst, offset, row_ptr, (int)n_edges, id_swap, nullptr, nullptr);
  GP_LAUNCH_CHECK(ctx, "links_kernel");
  return GP_OK;
}

int gp_csr_max_degree(gp_ctx* ctx, const int32_t* ptr, int64_t n, void* ws, size_t ws_bytes, int32_t* max_degree) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, max_degree, "gp_csr_max_degree: max_degree is NULL");
  GP_REQUIRE(ctx, n >= 0, "gp_csr_max_degree: negative size");
  *max_degree = 0;
  if (n == 0) return GP_OK;
  GP_REQUIRE(ctx, ptr && ws, "gp_csr_max_degree: NULL pointer");
  if (ws_bytes < sizeof(int32_t)) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "gp_csr_max_degree: workspace below 4 bytes");
  GP_HIP(ctx, hipSetDevice(ctx->device));
  max_degree_kernel<<<1, 1024, 0, ctx->stream>>>(ptr, n, static_cast<int32_t*>(ws));
  GP_LAUNCH_CHECK(ctx, "max_degree_kernel");
  GP_HIP(ctx, hipMemcpyAsync(max_degree, ws, sizeof(int32_t), hipMemcpyDeviceToHost, ctx->stream));
  GP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return GP_OK;
}

int gp_edges_workspace(int64_t n_atoms, size_t* bytes) {
  if (!bytes || n_atoms < 0) return GP_BAD_ARG;
  edges_ws w;
  *bytes = carve_edges(nullptr, n_atoms, &w);
  return GP_OK;
}

}  // extern "C"

namespace {

int check_images(gp_ctx* ctx, const char* who, const float* cell, int r0, int r1, int r2, int64_t n_atoms, images_t* im) {
  GP_REQUIRE(ctx, cell, "%s: cell is NULL", who);
  GP_REQUIRE(ctx, r0 >= 0 && r1 >= 0 && r2 >= 0 && r0 <= 16 && r1 <= 16 && r2 <= 16, "%s: image range must be 0..16 per axis", who);
  *im = images_t{cell, r0, r1, r2};
  if ((int64_t)im->count() * n_atoms > INT32_MAX) return gp_fail(ctx, GP_INT32_OVERFLOW, "%s: atoms x images exceed int32", who);
  return GP_OK;
}

// Waits for the first n host words, which the kernel launched last writes and which the caller had set to -1 before (the counts are never
// negative): the words themselves are looked at, which shows them some microseconds before the stream's own wait would return.  After a
// quarter of a second, or where the launch went wrong, the stream is waited for, so a kernel that never writes ends in its error.
int wait_host_words(gp_ctx* ctx, int n) {
  volatile int64_t* h = ctx->hwords;
  const auto start = std::chrono::steady_clock::now();
  for (;;) {
    for (int spin = 0; spin < 256; ++spin) {
      bool there = true;
      for (int i = 0; i < n; ++i) there = there && h[i] >= 0;
      if (there) {
        std::atomic_thread_fence(std::memory_order_acquire);
        return GP_OK;
      }
      __builtin_ia32_pause();
    }
    if (std::chrono::steady_clock::now() - start > std::chrono::milliseconds(250)) break;
  }
  GP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int i = 0; i < n; ++i)
    if (h[i] < 0) return gp_fail(ctx, GP_HIP_ERROR, "a count did not arrive");
  return GP_OK;
}

int edges_count_impl(gp_ctx* ctx, const char* who, const float* pos, const int32_t* graph_ptr, images_t im, int64_t n_atoms,
                     int32_t n_graphs, float cutoff, int32_t max_neighbors, void* ws, size_t ws_bytes, int64_t* n_edges) {
  GP_REQUIRE(ctx, n_edges, "%s: n_edges is NULL", who);
  GP_REQUIRE(ctx, n_atoms >= 0 && n_graphs >= 0 && max_neighbors >= 0, "%s: negative size", who);
  GP_REQUIRE(ctx, cutoff > 0.f && cutoff == cutoff, "%s: cutoff must be positive", who);
  if (n_atoms > INT32_MAX - 1) return gp_fail(ctx, GP_INT32_OVERFLOW, "%s: too many atoms", who);
  *n_edges = 0;
  if (n_atoms == 0 || n_graphs == 0) return GP_OK;
  GP_REQUIRE(ctx, pos && graph_ptr && ws, "%s: NULL pointer", who);
  edges_ws w;
  size_t need = carve_edges(ws, n_atoms, &w);
  if (ws_bytes < need) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "%s: workspace %zu < %zu", who, ws_bytes, need);
  GP_HIP(ctx, hipSetDevice(ctx->device));
  const float c2 = cutoff * cutoff;
  edges_kernel<false><<<blocks_for(n_atoms, 4), 256, 0, ctx->stream>>>(
      pos, graph_ptr, (int)n_atoms, n_graphs, c2, max_neighbors, im, w.deg, w.cap, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
  GP_LAUNCH_CHECK(ctx, "edges_kernel<count>");
  GP_REQUIRE_HOST_WORDS(ctx, who);
  std::lock_guard<std::mutex> words(ctx->count_mutex);
  *(volatile int64_t*)ctx->hwords = -1;
  scan_exclusive_kernel<<<1, SCAN_THREADS, 0, ctx->stream>>>(w.deg, w.row_ptr, n_atoms, ctx->hwords_dev);
  GP_LAUNCH_CHECK(ctx, "scan_exclusive_kernel");
  GP_TRY(wait_host_words(ctx, 1));
  const int64_t total = *(volatile int64_t*)ctx->hwords;
  *n_edges = total;
  if (total <= INT32_MAX) return GP_OK;
  GP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return gp_fail(ctx, GP_INT32_OVERFLOW, "%s: %lld edges exceed int32", who, (long long)total);
}

int edges_fill_impl(gp_ctx* ctx, const char* who, const float* pos, const int32_t* graph_ptr, images_t im, int64_t n_atoms,
                    int32_t n_graphs, float cutoff, int32_t max_neighbors, const void* ws, size_t ws_bytes, int64_t n_edges,
                    int32_t* src, int32_t* dst, int32_t* offset, int32_t* row_ptr, float* dist, float* unit) {
  GP_REQUIRE(ctx, n_atoms >= 0 && n_graphs >= 0 && max_neighbors >= 0 && n_edges >= 0, "%s: negative size", who);
  GP_REQUIRE(ctx, cutoff > 0.f && cutoff == cutoff, "%s: cutoff must be positive", who);
  GP_REQUIRE(ctx, row_ptr, "%s: row_ptr is NULL", who);
  if (n_atoms > INT32_MAX - 1 || n_edges > INT32_MAX) return gp_fail(ctx, GP_INT32_OVERFLOW, "%s: sizes exceed int32", who);
  GP_HIP(ctx, hipSetDevice(ctx->device));
  if (n_atoms == 0 || n_graphs == 0) {
    GP_HIP(ctx, (hipError_t)gp_zero_async(ctx->stream, row_ptr, sizeof(int32_t) * (n_atoms + 1)));
    return GP_OK;
  }
  GP_REQUIRE(ctx, pos && graph_ptr && ws, "%s: NULL pointer", who);
  GP_REQUIRE(ctx, n_edges == 0 || (src && dst), "%s: src/dst is NULL", who);
  edges_ws w;
  size_t need = carve_edges(const_cast<void*>(ws), n_atoms, &w);
  if (ws_bytes < need) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "%s: workspace %zu < %zu", who, ws_bytes, need);
  if (n_edges == 0) {   // nothing to write but the offsets
    GP_HIP(ctx, hipMemcpyAsync(row_ptr, w.row_ptr, sizeof(int32_t) * (n_atoms + 1), hipMemcpyDeviceToDevice, ctx->stream));
    return GP_OK;
  }
  const float c2 = cutoff * cutoff;
  edges_kernel<true><<<blocks_for(n_atoms, 4), 256, 0, ctx->stream>>>(
      pos, graph_ptr, (int)n_atoms, n_graphs, c2, max_neighbors, im, nullptr, w.cap, w.row_ptr, row_ptr, src, dst, offset, dist, unit);
  GP_LAUNCH_CHECK(ctx, "edges_kernel<fill>");
  return GP_OK;
}

}  // namespace

extern "C" {

int gp_edges_count(gp_ctx* ctx, const float* pos, const int32_t* graph_ptr, int64_t n_atoms,
                   int32_t n_graphs, float cutoff, int32_t max_neighbors, void* ws, size_t ws_bytes,
                   int64_t* n_edges) {
  if (!ctx) return GP_BAD_ARG;
  return edges_count_impl(ctx, "gp_edges_count", pos, graph_ptr, images_t{nullptr, 0, 0, 0}, n_atoms, n_graphs, cutoff,
                          max_neighbors, ws, ws_bytes, n_edges);
}

int gp_edges_fill(gp_ctx* ctx, const float* pos, const int32_t* graph_ptr, int64_t n_atoms,
                  int32_t n_graphs, float cutoff, int32_t max_neighbors, const void* ws, size_t ws_bytes,
                  int64_t n_edges, int32_t* src, int32_t* dst, int32_t* row_ptr, float* dist, float* unit) {
  if (!ctx) return GP_BAD_ARG;
  return edges_fill_impl(ctx, "gp_edges_fill", pos, graph_ptr, images_t{nullptr, 0, 0, 0}, n_atoms, n_graphs, cutoff,
                         max_neighbors, ws, ws_bytes, n_edges, src, dst, nullptr, row_ptr, dist, unit);
}

int gp_edges_count_pbc(gp_ctx* ctx, const float* pos, const int32_t* graph_ptr, const float* cell, int64_t n_atoms,
                       int32_t n_graphs, float cutoff, int32_t max_neighbors, int32_t rep0, int32_t rep1, int32_t rep2,
                       void* ws, size_t ws_bytes, int64_t* n_edges) {
  if (!ctx) return GP_BAD_ARG;
  images_t im;
  GP_TRY(check_images(ctx, "gp_edges_count_pbc", cell, rep0, rep1, rep2, n_atoms, &im));
  return edges_count_impl(ctx, "gp_edges_count_pbc", pos, graph_ptr, im, n_atoms, n_graphs, cutoff, max_neighbors, ws,
                          ws_bytes, n_edges);
}

int gp_edges_fill_pbc(gp_ctx* ctx, const float* pos, const int32_t* graph_ptr, const float* cell, int64_t n_atoms,
                      int32_t n_graphs, float cutoff, int32_t max_neighbors, int32_t rep0, int32_t rep1, int32_t rep2,
                      const void* ws, size_t ws_bytes, int64_t n_edges, int32_t* src, int32_t* dst, int32_t* offset,
                      int32_t* row_ptr, float* dist, float* unit) {
  if (!ctx) return GP_BAD_ARG;
  images_t im;
  GP_TRY(check_images(ctx, "gp_edges_fill_pbc", cell, rep0, rep1, rep2, n_atoms, &im));
  GP_REQUIRE(ctx, n_edges == 0 || offset, "gp_edges_fill_pbc: offset is NULL");
  return edges_fill_impl(ctx, "gp_edges_fill_pbc", pos, graph_ptr, im, n_atoms, n_graphs, cutoff, max_neighbors, ws,
                         ws_bytes, n_edges, src, dst, offset, row_ptr, dist, unit);
}

int gp_triplets_workspace(int64_t n_atoms, int64_t n_edges, size_t* bytes) {
  if (!bytes || n_atoms < 0 || n_edges < 0) return GP_BAD_ARG;
  triplets_ws w;
  *bytes = carve_triplets(nullptr, n_atoms, n_edges, &w);
  return GP_OK;
}

}  // extern "C"

namespace {

int check_lists(gp_ctx* ctx, const char* who, int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, triplets_ws* w) {
  GP_REQUIRE(ctx, n_atoms >= 0 && n_edges >= 0, "%s: negative size", who);
  if (n_atoms > INT32_MAX - 1 || n_edges > INT32_MAX - 1) return gp_fail(ctx, GP_INT32_OVERFLOW, "%s: sizes exceed int32", who);
  if (n_edges == 0 || n_atoms == 0) return GP_OK;
  GP_REQUIRE(ctx, ws, "%s: NULL pointer", who);
  const size_t need = carve_triplets(ws, n_atoms, n_edges, w);
  if (ws_bytes < need) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "%s: workspace %zu < %zu", who, ws_bytes, need);
  GP_HIP(ctx, hipSetDevice(ctx->device));
  return GP_OK;
}

// Opposite edges and both segment orders with the out-edge offsets, or the ji-major order alone.  w.seg_ji, seg_kj, out_ptr, id_swap
// point where the results belong (the caller's arrays or the workspace's).
int lists_pass(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset, const int32_t* row_ptr, int64_t n_atoms,
               int64_t n_edges, const triplets_ws& w, bool with_kj, int64_t* host_words) {
  hipStream_t st = ctx->stream;
  int32_t* out_deg = with_kj ? w.out_deg : nullptr;
  if (with_kj) GP_HIP(ctx, (hipError_t)gp_zero_async(st, out_deg, sizeof(int32_t) * n_atoms));
  links_kernel<<<blocks_for(n_edges, 256), 256, 0, st>>>(src, dst, offset, row_ptr, (int)n_edges, w.id_swap, out_deg, w.arrival);
  const int64_t nc = chunks_of(n_edges);
  (with_kj ? lists_sums_kernel<true> : lists_sums_kernel<false>)<<<(unsigned)nc, 256, 0, st>>>(src, dst, row_ptr, w.id_swap, out_deg, n_edges, w.sums);
  lists_mid_kernel<<<1, 1024, 0, st>>>(row_ptr, out_deg, with_kj ? (int)n_atoms : 0, nc, w.out_ptr, w.sums, w.total, host_words);
  GP_LAUNCH_CHECK(ctx, "list kernels");
  (with_kj ? lists_apply_kernel<true> : lists_apply_kernel<false>)<<<(unsigned)nc, 256, 0, st>>>(
      src, dst, row_ptr, w.id_swap, out_deg, w.out_ptr, w.arrival, n_edges, w.sums, w.total, w.seg_ji, w.seg_kj, w.out_tmp);
  GP_LAUNCH_CHECK(ctx, "lists_apply_kernel");
  return GP_OK;
}

// with_kj: the counts are waited for alone, and the last pass runs while the caller allocates; without it, and after an overflow,
// the stream is idle on return
int lists_count(gp_ctx* ctx, const char* who, const int32_t* src, const int32_t* dst, const int32_t* offset, const int32_t* row_ptr,
                int64_t n_atoms, int64_t n_edges, const triplets_ws& w, bool with_kj, int64_t* n_triplets, int32_t* max_in,
                int32_t* max_out) {
  GP_REQUIRE_HOST_WORDS(ctx, who);
  std::lock_guard<std::mutex> words(ctx->count_mutex);
  volatile int64_t* h = ctx->hwords;
  h[0] = h[1] = h[2] = -1;
  GP_TRY(lists_pass(ctx, src, dst, offset, row_ptr, n_atoms, n_edges, w, with_kj, ctx->hwords_dev));
  if (with_kj) GP_TRY(wait_host_words(ctx, 3));
  else GP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  *n_triplets = h[0];
  if (max_in) *max_in = (int32_t)h[1];
  if (max_out) *max_out = (int32_t)h[2];
  if (*n_triplets <= INT32_MAX) return GP_OK;
  GP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return gp_fail(ctx, GP_INT32_OVERFLOW, "%s: %lld triplets exceed int32", who, (long long)*n_triplets);
}

// with_kj: the out-edges in order and both orders of the triplets, else the ji-major one alone
int lists_fill(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* row_ptr, int64_t n_atoms, int64_t n_edges, int64_t n_triplets,
               bool periodic, bool with_kj, const triplets_ws& w, int32_t* idx_kj, int32_t* idx_ji, int32_t* perm_kj, int32_t* idx_ji_kj) {
  hipStream_t st = ctx->stream;
  if (with_kj) {
    out_lists_kernel<<<(unsigned)n_atoms, 256, 0, st>>>(row_ptr, w.id_swap, w.out_ptr, w.out_tmp, periodic ? 1 : 0, w.out_list);
    GP_LAUNCH_CHECK(ctx, "out_lists_kernel");
  }
  if (n_triplets == 0) return GP_OK;
  const bool wide = n_triplets >= LONG_LISTS * n_edges;
  const int ji = blocks_for(n_edges, wide ? 4 : 16);
  const int kj = with_kj ? blocks_for(n_edges, 64) : 0;   // 64 rows per workgroup in both forms
  (wide ? triplet_fill_kernel<true> : triplet_fill_kernel<false>)<<<(unsigned)(ji + kj), 256, 0, st>>>(
      src, dst, row_ptr, w.id_swap, w.out_ptr, w.out_list, w.seg_ji, w.seg_kj, (int)n_edges, ji, idx_kj, idx_ji, perm_kj, idx_ji_kj);
  GP_LAUNCH_CHECK(ctx, "triplet_fill_kernel");
  return GP_OK;
}

int triplets_count_impl(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset, const int32_t* row_ptr,
                        int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, int64_t* n_triplets) {
  GP_REQUIRE(ctx, n_triplets, "gp_triplets_count: n_triplets is NULL");
  *n_triplets = 0;
  triplets_ws w;
  GP_TRY(check_lists(ctx, "gp_triplets_count", n_atoms, n_edges, ws, ws_bytes, &w));
  if (n_edges == 0 || n_atoms == 0) return GP_OK;
  GP_REQUIRE(ctx, src && dst && row_ptr, "gp_triplets_count: NULL pointer");
  return lists_count(ctx, "gp_triplets_count", src, dst, offset, row_ptr, n_atoms, n_edges, w, false, n_triplets, nullptr, nullptr);
}

int triplets_fill_impl(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset, const int32_t* row_ptr,
                       int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, int64_t n_triplets,
                       int32_t* idx_kj, int32_t* idx_ji, int32_t* seg_ptr_ji, int32_t* perm_kj,
                       int32_t* idx_ji_kj, int32_t* seg_ptr_kj) {
  GP_REQUIRE(ctx, n_triplets >= 0, "gp_triplets_fill: negative size");
  if (n_triplets > INT32_MAX) return gp_fail(ctx, GP_INT32_OVERFLOW, "gp_triplets_fill: sizes exceed int32");
  GP_REQUIRE(ctx, seg_ptr_ji, "gp_triplets_fill: seg_ptr_ji is NULL");
  const bool want_kj = perm_kj || idx_ji_kj || seg_ptr_kj;
  GP_REQUIRE(ctx, !want_kj || (seg_ptr_kj && (n_triplets == 0 || (perm_kj && idx_ji_kj))),
             "gp_triplets_fill: perm_kj, idx_ji_kj, seg_ptr_kj must be given together");
  triplets_ws w;
  GP_TRY(check_lists(ctx, "gp_triplets_fill", n_atoms, n_edges, ws, ws_bytes, &w));
  hipStream_t st = ctx->stream;
  if (n_edges == 0 || n_atoms == 0) {
    GP_HIP(ctx, hipSetDevice(ctx->device));
    GP_HIP(ctx, (hipError_t)gp_zero_async(st, seg_ptr_ji, sizeof(int32_t) * (n_edges + 1)));
    if (seg_ptr_kj) GP_HIP(ctx, (hipError_t)gp_zero_async(st, seg_ptr_kj, sizeof(int32_t) * (n_edges + 1)));
    return GP_OK;
  }
  GP_REQUIRE(ctx, src && dst && row_ptr, "gp_triplets_fill: NULL pointer");
  GP_REQUIRE(ctx, n_triplets == 0 || (idx_kj && idx_ji), "gp_triplets_fill: idx_kj/idx_ji is NULL");
  if (want_kj) {
    w.seg_ji = seg_ptr_ji; w.seg_kj = seg_ptr_kj;
    GP_TRY(lists_pass(ctx, src, dst, offset, row_ptr, n_atoms, n_edges, w, true, nullptr));
  } else {
    GP_HIP(ctx, hipMemcpyAsync(seg_ptr_ji, w.seg_ji, sizeof(int32_t) * (n_edges + 1), hipMemcpyDeviceToDevice, st));
  }
  return lists_fill(ctx, src, dst, row_ptr, n_atoms, n_edges, n_triplets, offset != nullptr, want_kj, w, idx_kj, idx_ji, perm_kj, idx_ji_kj);
}

}  // namespace

extern "C" {

int gp_triplets_count(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* row_ptr,
                      int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, int64_t* n_triplets) {
  if (!ctx) return GP_BAD_ARG;
  return triplets_count_impl(ctx, src, dst, nullptr, row_ptr, n_atoms, n_edges, ws, ws_bytes, n_triplets);
}

int gp_triplets_fill(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* row_ptr,
                     int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, int64_t n_triplets,
                     int32_t* idx_kj, int32_t* idx_ji, int32_t* seg_ptr_ji, int32_t* perm_kj,
                     int32_t* idx_ji_kj, int32_t* seg_ptr_kj) {
  if (!ctx) return GP_BAD_ARG;
  return triplets_fill_impl(ctx, src, dst, nullptr, row_ptr, n_atoms, n_edges, ws, ws_bytes, n_triplets, idx_kj, idx_ji,
                            seg_ptr_ji, perm_kj, idx_ji_kj, seg_ptr_kj);
}

int gp_triplets_count_pbc(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset,
                          const int32_t* row_ptr, int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes,
                          int64_t* n_triplets) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, n_edges == 0 || offset, "gp_triplets_count_pbc: offset is NULL");
  return triplets_count_impl(ctx, src, dst, offset, row_ptr, n_atoms, n_edges, ws, ws_bytes, n_triplets);
}

int gp_triplets_fill_pbc(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset,
                         const int32_t* row_ptr, int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes,
                         int64_t n_triplets, int32_t* idx_kj, int32_t* idx_ji, int32_t* seg_ptr_ji, int32_t* perm_kj,
                         int32_t* idx_ji_kj, int32_t* seg_ptr_kj) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, n_edges == 0 || offset, "gp_triplets_fill_pbc: offset is NULL");
  return triplets_fill_impl(ctx, src, dst, offset, row_ptr, n_atoms, n_edges, ws, ws_bytes, n_triplets, idx_kj, idx_ji,
                            seg_ptr_ji, perm_kj, idx_ji_kj, seg_ptr_kj);
}

int gp_graph_lists_count(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset, const int32_t* row_ptr,
                         int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, int32_t* seg_ptr_ji, int32_t* seg_ptr_kj,
                         int32_t* out_ptr, int32_t* id_swap, int64_t* n_triplets, int32_t* max_in_degree,
                         int32_t* max_out_degree) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, n_triplets && max_in_degree && max_out_degree, "gp_graph_lists_count: NULL pointer");
  GP_REQUIRE(ctx, n_atoms > 0 && n_edges > 0, "gp_graph_lists_count: empty graph");
  GP_REQUIRE(ctx, src && dst && row_ptr && seg_ptr_ji && seg_ptr_kj && out_ptr && id_swap, "gp_graph_lists_count: NULL pointer");
  *n_triplets = 0;
  triplets_ws w;
  GP_TRY(check_lists(ctx, "gp_graph_lists_count", n_atoms, n_edges, ws, ws_bytes, &w));
  w.seg_ji = seg_ptr_ji; w.seg_kj = seg_ptr_kj; w.out_ptr = out_ptr; w.id_swap = id_swap;
  return lists_count(ctx, "gp_graph_lists_count", src, dst, offset, row_ptr, n_atoms, n_edges, w, true, n_triplets, max_in_degree,
                     max_out_degree);
}

int gp_graph_lists_fill(gp_ctx* ctx, const int32_t* src, const int32_t* dst, const int32_t* offset, const int32_t* row_ptr,
                        int64_t n_atoms, int64_t n_edges, void* ws, size_t ws_bytes, const int32_t* seg_ptr_ji, const int32_t* seg_ptr_kj,
                        const int32_t* out_ptr, const int32_t* id_swap, int64_t n_triplets, int32_t* out_list, int32_t* idx_kj,
                        int32_t* idx_ji, int32_t* perm_kj, int32_t* idx_ji_kj) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, n_atoms > 0 && n_edges > 0 && n_triplets >= 0, "gp_graph_lists_fill: bad sizes");
  if (n_triplets > INT32_MAX) return gp_fail(ctx, GP_INT32_OVERFLOW, "gp_graph_lists_fill: sizes exceed int32");
  GP_REQUIRE(ctx, src && dst && row_ptr && seg_ptr_ji && seg_ptr_kj && out_ptr && id_swap && out_list, "gp_graph_lists_fill: NULL pointer");
  GP_REQUIRE(ctx, n_triplets == 0 || (idx_kj && idx_ji && perm_kj && idx_ji_kj), "gp_graph_lists_fill: NULL pointer");
  triplets_ws w;
  GP_TRY(check_lists(ctx, "gp_graph_lists_fill", n_atoms, n_edges, ws, ws_bytes, &w));
  w.seg_ji = const_cast<int32_t*>(seg_ptr_ji); w.seg_kj = const_cast<int32_t*>(seg_ptr_kj);
  w.out_ptr = const_cast<int32_t*>(out_ptr); w.id_swap = const_cast<int32_t*>(id_swap); w.out_list = out_list;
  return lists_fill(ctx, src, dst, row_ptr, n_atoms, n_edges, n_triplets, offset != nullptr, true, w, idx_kj, idx_ji, perm_kj, idx_ji_kj);
}

}  // extern "C"
