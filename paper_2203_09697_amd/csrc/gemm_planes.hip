// fp32 products A W, A W^T (edge and atom rows times a weight matrix) on the fp16 matrix cores, and A^T B (sums over the rows:
// weight gradients), which has a form of its own below.
// In A W and A W^T every element enters as the sum of two fp16 numbers, v 2^k = hi + lo, and three of the four products of the parts
// are formed (lo.lo is below 2^-22 of the product).  The power of two is chosen so that the largest of the values that share it
// lies in [2^15, 2^16): the values of a row of A over 32 consecutive k, and a column of W.  fp16's last place is 2^-24, so a value
// keeps 23 bits down to 2^-17 of the largest, 21 at 2^-19 (SPAN) and would lose one more with every power of two below that.  Values of A that
// are smaller still get a pass over the same k of their own, with a scale of their own, and so on until none is left; of W the 16 k of 32
// columns that hold one are left out and added from the matrix itself, in fp32.  So no value loses bits for what stands beside it.
// The 32 k are summed from zero and enter the result with their scale taken back: K / 32 additions into the fp32 sum.
//
// Against the form with three bf16 parts and six products (gemm_split_kernel: 24 bits, 6 K / 16 additions) that is half the
// matrix instructions and a smaller error, because the additions are what that form's error is made of.  Relative error
// against 64 bits, operands uniform in +-1 (three bf16 parts / two fp16 parts / fp32 matrix instruction): K = 64 1.1e-7 / 8.3e-8 /
// 1.5e-7, K = 128 1.6e-7 / 8.9e-8 / 2.0e-7, K = 256 2.4e-7 / 9.8e-8 / 2.9e-7, K = 1024 4.8e-7 / 1.3e-7 / 5.7e-7, K = 2048 6.9e-7 /
// 1.7e-7 / 8.1e-7.  Shorter contractions, where the two forms meet, stay with the other kernels (gp_planes_take).
//
// What bounds these products is power as much as anything: with random operands the matrix units of the whole chip sustain 1.87
// PFLOP/s in bf16 and 1.72 in fp16 from registers alone (2.47 with zeros), so fewer matrix instructions is what helps.
#include <stdarg.h>

#include <type_traits>

#include <algorithm>

#include "gemm_common.h"

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(1))) void* global_void_ptr;

constexpr int PL = 2;                   // planes: hi, lo
constexpr int FRAG_B = 1024;            // one operand fragment of a wavefront: 64 lanes x 8 fp16
constexpr int GROUP_B = PL * FRAG_B;    // both planes of 32 columns x 16 k

// v = hi + lo, both rounded to nearest
__device__ __forceinline__ void split8(const float* v, f16x8& hi, f16x8& lo) {
#pragma unroll
  for (int c = 0; c < 8; ++c) hi[c] = (_Float16)v[c];
#pragma unroll
  for (int c = 0; c < 8; ++c) lo[c] = (_Float16)(v[c] - (float)hi[c]);
}
// v = p[0] + p[1] + p[2], every part with its own exponent
__device__ __forceinline__ void parts8(const float* v, bf16x8 (&p)[3]) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    float r = v[c];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      p[q][c] = (__bf16)r;
      r -= (float)p[q][c];
    }
  }
}

// Of the values that share a scale: the largest absolute value, and twice the bits of the smallest that is not zero, less one
struct value_range {
  float top = 0.f;
  uint32_t least = ~0u;
  __device__ __forceinline__ void add(float a, float b) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(top) : "v"(a), "v"(b));
    add_least(a);
    add_least(b);
  }
  __device__ __forceinline__ void add_least(float v) {
    const uint32_t d = (__float_as_uint(v) << 1) - 1u;
    least = d < least ? d : least;
  }
  __device__ __forceinline__ uint32_t most() const { return __float_as_uint(top); }
};
__device__ __forceinline__ bool any_below(const value_range& r, uint32_t from) {   // zeros are not
  return r.least < (from ? 2u * from - 1u : 0u);
}
// The biased exponent by which some values are scaled, for the bits of the largest absolute one: the next where fp16 would round it up to 2^16
__device__ __forceinline__ int top_exp(uint32_t bits) { return (int)((bits + 0x1000u) >> 23); }
// The bits of the smallest absolute value that keeps 21 bits beside that one: hi is at least 2^-4, lo at most 2^-25 off
constexpr int SPAN = 19;
__device__ __forceinline__ uint32_t keeps_from(uint32_t most) {
  const int e = top_exp(most) - SPAN;
  return (most >> 23) != 255u && e > 0 ? (uint32_t)e << 23 : 0u;
}

// The power of two 2^k that brings the largest of some values into [2^15, 2^16): k = 0 where that is 0, an infinity or a NaN, and
// at most 112 (below 2^-97 not all of the way), so that the factors back are normal numbers.
__device__ __forceinline__ int scale_exp(uint32_t bits) {
  const int k = 142 - top_exp(bits);
  return bits >= 0x7F800000u || bits == 0u ? 0 : k < 112 ? k : 112;
}
__device__ __forceinline__ float pow2(int k) { return __int_as_float((k + 127) << 23); }   // -126 <= k <= 127
// The matrix instruction's sums come out low on average, by a part of the last place of their largest term and whatever their
// sign: over the rows of a bias gradient that adds up.  Half of the sums are therefore formed with the sign of one operand turned round
// (its scale is negative, and so is the factor back): four blocks of width 256 over 43380 edges 6e-7 off (a quarter turned 2.2e-5,
// three bf16 parts, whose sums run on, 3.4e-5), one of width 2048 4.3e-7 (none turned 2.3e-5, three bf16 parts 4.0e-5).
__device__ __forceinline__ float turned(float scale, bool turn) { return __int_as_float(__float_as_int(scale) ^ (turn ? 1 << 31 : 0)); }
// the larger of lanes l and l ^ 32
__device__ __forceinline__ uint32_t max_halves(uint32_t m) {
  const auto h = __builtin_amdgcn_permlane32_swap(m, m, false, false);
  return h[0] > h[1] ? h[0] : h[1];
}
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkmcnt0() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

struct plane_jobs {
  gp_plane_job j[GP_PLANE_JOBS_MAX];
};

// One workgroup per 32 columns n: the scales of the columns first (largest |w| over all k), then the planes, a wavefront per
// 16 k: lane (kh, n) takes 8 consecutive k of column n.  Behind the planes: the columns' factors back, 2^14 / scale; a word per block
// of 32 columns, whether one of its 16-k pieces holds a value that would lose bits; a word per piece, whether this one does.  The
// planes of such a piece are zero and the products take it from the matrix itself.
constexpr int PREP_WAVES = 16, PREP_KEEP = 8;   // 16-k pieces a wavefront keeps in registers between the two passes
__global__ void __launch_bounds__(64 * PREP_WAVES) make_planes_kernel(const plane_jobs jobs) {
  const gp_plane_job& q = jobs.j[blockIdx.y];
  const int k16 = (q.K + 31) / 32 * 2, nb = (q.N + 31) / 32;
  const int blk = blockIdx.x;
  if (blk >= nb) return;
  __shared__ uint32_t big[32], some;
  if (threadIdx.x < 32) big[threadIdx.x] = 0u;
  if (threadIdx.x == 0) some = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = blk * 32 + (lane & 31);
  auto load = [&](int u, float* v) __attribute__((always_inline)) {
    const int k = u * 16 + (lane >> 5) * 8;
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = 0.f;
    if (u >= k16 || n >= q.N || k >= q.K) return;   // K is a multiple of 16
    if (q.k_rows) {
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = q.src[(int64_t)(k + c) * q.N + n];
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = q.src[(int64_t)n * q.K + k + c];
    }
  };
  float keep[PREP_KEEP][8];
  uint32_t m = 0;
  auto most = [&](const float* v) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t b = __float_as_uint(v[c]) & 0x7FFFFFFFu;
      m = b > m ? b : m;
    }
  };
#pragma unroll
  for (int i = 0; i < PREP_KEEP; ++i) load(wave + i * PREP_WAVES, keep[i]);
#pragma unroll
  for (int i = 0; i < PREP_KEEP; ++i) most(keep[i]);
  for (int u = wave + PREP_KEEP * PREP_WAVES; u < k16; u += PREP_WAVES) {
    float v[8];
    load(u, v);
    most(v);
  }
  atomicMax(&big[lane & 31], m);
  __syncthreads();
  const int se = scale_exp(big[lane & 31]);
  const float s = pow2(se);
  const uint32_t from = keeps_from(big[lane & 31]);
  char* tail = static_cast<char*>(q.dst) + (int64_t)nb * k16 * GROUP_B;
  uint32_t* uneven = reinterpret_cast<uint32_t*>(tail + (int64_t)nb * 32 * sizeof(float));
  auto put = [&](int u, const float* v) __attribute__((always_inline)) {
    value_range r;
#pragma unroll
    for (int c = 0; c < 8; ++c) r.add_least(v[c]);
    const bool out = __any(any_below(r, from));
    if (lane == 0) {
      uneven[nb + (int64_t)blk * k16 + u] = out;
      if (out) some = 1u;
    }
    f16x8 hi = {}, lo = {};
    if (!out) {
      float t[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) t[c] = v[c] * s;
      split8(t, hi, lo);
    }
    char* dst = static_cast<char*>(q.dst) + ((int64_t)blk * k16 + u) * GROUP_B + lane * 16;
    *reinterpret_cast<f16x8*>(dst) = hi;
    *reinterpret_cast<f16x8*>(dst + FRAG_B) = lo;
  };
#pragma unroll
  for (int i = 0; i < PREP_KEEP; ++i)
    if (wave + i * PREP_WAVES < k16) put(wave + i * PREP_WAVES, keep[i]);
  for (int u = wave + PREP_KEEP * PREP_WAVES; u < k16; u += PREP_WAVES) {
    float v[8];
    load(u, v);
    put(u, v);
  }
  if (threadIdx.x < 32) reinterpret_cast<float*>(tail)[n] = pow2(14 - se);
  __syncthreads();
  if (threadIdx.x == 0) uneven[blk] = some;
}

// Epilogue of a wavefront's MB x NB blocks for the steps EMASK names (see tile_epilogue_f32 for the register layout and the
// order of steps).  The matrices it reads are requested one block ahead of the block that is stored: block by block, each
// block waited for its own loads.  Rows past M read row M - 1 and columns past N the last four; nothing is stored there.
template <unsigned M>
struct epi_in {
  f32x4 bias, pre[4], z[4], mul[4], post[4], z2[4];
  __device__ __forceinline__ void load(const gp_epilogue& e, const int64_t (&o)[4], int col) {
    if constexpr ((M & EM_BIAS) != 0) bias = ld4(e.bias + col);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      if constexpr ((M & EM_ADD_PRE) != 0) pre[it] = ld4(e.add_pre + o[it]);
      if constexpr ((M & (EM_ACT2 | EM_GATE)) != 0) z[it] = ld4(e.zsrc + o[it]);
      if constexpr ((M & EM_MUL) != 0) mul[it] = ld4(e.mul + o[it]);
      if constexpr ((M & EM_ADD_POST) != 0) post[it] = ld4(e.add_post + o[it]);
      if constexpr ((M & EM_OUT2) != 0 && (M & EM_GATE) == 0) z2[it] = ld4(e.z2src + o[it]);
    }
  }
};

template <int MB, int NB, unsigned M>
__device__ __forceinline__ void epilogue_blocks(const gemm_args& g, f32x16 (&acc)[MB][NB], float* stage, int64_t row0, int col0, const float* inv) {
  const int lane = threadIdx.x & 63;
  const int kh = lane >> 5, l32 = lane & 31, c4 = (lane & 7) * 4;
  epi_in<M> in[2];
  auto at = [&](int b, int64_t (&o)[4], int& col) __attribute__((always_inline)) {
    const int c = col0 + (b % NB) * 32 + c4;
    col = c < g.N ? c : g.N - 4;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int64_t r = row0 + (b / NB) * 32 + it * 8 + (lane >> 3);
      o[it] = (r < g.M ? r : g.M - 1) * g.N + col;
    }
  };
  int64_t o[4];
  int col;
  at(0, o, col);
  in[0].load(g.epi, o, col);
#pragma unroll
  for (int b = 0; b < MB * NB; ++b) {
    const int i = b / NB, j = b % NB;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *reinterpret_cast<f32x4*>(&stage[l32 * EPI_LD + q4 * 8 + kh * 4]) =
          f32x4{acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]};
    if (b + 1 < MB * NB) {
      int64_t o1[4];
      int col1;
      at(b + 1, o1, col1);
      in[(b + 1) & 1].load(g.epi, o1, col1);
    }
    wave_lds_sync();
    const epi_in<M>& q = in[b & 1];
    at(b, o, col);
    const bool col_in = col0 + j * 32 + c4 < g.N;
    const f32x4 inv4 = ld4(inv + col);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      f32x4 v = *reinterpret_cast<const f32x4*>(&stage[(it * 8 + (lane >> 3)) * EPI_LD + c4]);
      const bool in_m = col_in && row0 + i * 32 + it * 8 + (lane >> 3) < g.M;
      v *= inv4;
      if constexpr ((M & EM_BIAS) != 0) v += q.bias;
      if constexpr ((M & EM_ADD_PRE) != 0) v += q.pre[it];
      if constexpr ((M & EM_SAVE_PRE) != 0) {
        if (in_m) st4(g.epi.save_pre + o[it], v);
      }
      if constexpr ((M & EM_ACT1) != 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = silu_f(v[c]);
      }
      if constexpr ((M & EM_ACT2) != 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] *= dsilu_f(q.z[it][c]);
      }
      if constexpr ((M & EM_GATE) != 0) {
        f32x4 dz, dg;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          dz[c] = v[c] * q.mul[it][c] * dsilu_f(q.z[it][c]);
          dg[c] = v[c] * silu_f(q.z[it][c]);
        }
        if (in_m) {
          st4(g.epi.out + o[it], dz);
          st4(g.epi.out2 + o[it], dg);
        }
        continue;
      }
      if constexpr ((M & EM_MUL) != 0) v *= q.mul[it];
      if constexpr ((M & EM_ADD_POST) != 0) v += q.post[it];
      if constexpr ((M & EM_OUT) != 0) {
        if (in_m) st4(g.epi.out + o[it], v);
      }
      if constexpr ((M & EM_OUT2) != 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] *= dsilu_f(q.z2[it][c]);
        if (in_m) st4(g.epi.out2 + o[it], v);
      }
    }
    wave_lds_sync();
  }
}

// the combinations of gemm_common.h and the gate's backward step
#define GP_EM_LIST_PLANES(X) GP_EM_LIST(X) X(1824)
static_assert((EM_GATE | EM_MUL | EM_OUT | EM_OUT2) == 1824, "listed above");
bool epilogue_listed(unsigned mask) {
  switch (mask) {
#define GP_EM_CASE(M) case M:
    GP_EM_LIST_PLANES(GP_EM_CASE)
#undef GP_EM_CASE
    return true;
    default: return false;
  }
}

// WAVES wavefronts stacked along M, each with MB x NB blocks of 32x32.  A goes from memory straight into the registers of the
// wavefront that multiplies it, in operand order, and is split there: no LDS traffic, no barrier and no second split of the
// same values by another wavefront of the workgroup.  The planes of W, 4 KB per 32 columns and 32 k, come through LDS by
// global->LDS loads, NBUF chunks of them, and are read once per wavefront.  JB column blocks are multiplied together; TD and
// WD: whether the sums of a group (added to the result while the next group is multiplied) and its planes are double.
// Rows with values of their own pass (SPAN) take the chunk again: they are read once more (cached), the planes are still in LDS.  Of gradients,
// which are products, one 32 x 32 in 30 has such a value, of activations one in 300; looking for them costs 1 to 3 %, the passes as much
// again at 43380 x 2048 x 2048 (1.17 -> 1.25 ms, gradients 1.49 -> 1.66); 13230 x 256 x 256 20 -> 23 us.
// The activations of the next chunk are requested as soon as this one's are split.  (Splitting the next chunk beside the
// products of this one, or wavefronts of 64 x 128, ran out of registers: 1.41 -> 1.8 ms at 43380 x 2048 x 2048.)
template <int MB, int NB, int WAVES, int NBUF, int OCC, int JB, int TD, int WD>
__global__ void __launch_bounds__(64 * WAVES, OCC)
gemm_planes_kernel(const gemm_args g) {
  constexpr int BM = 32 * MB * WAVES, BN = 32 * NB, NG = NB / JB;   // NG groups of column blocks
  constexpr int CHUNK_B = NB * 2 * GROUP_B;             // bytes of a chunk
  constexpr int PB = CHUNK_B / 1024 / WAVES;            // global->LDS loads per wavefront and chunk
  static_assert(CHUNK_B % (1024 * WAVES) == 0, "the loads of a chunk are dealt evenly");
  extern __shared__ __attribute__((aligned(16))) float smem[];
  char* lds = reinterpret_cast<char*>(smem);

  const int tiles_n = (g.N + BN - 1) / BN;
  const int tiles_m = (int)((g.M + BM - 1) / BM);
  const int tile = xcd_remap(blockIdx.x, tiles_m * tiles_n);
  const int64_t m0 = (int64_t)(tile / tiles_n) * BM;
  const int n0 = (tile % tiles_n) * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm0 = wave * (32 * MB);
  const int kh = lane >> 5, l32 = lane & 31;
  const int n_ch = (g.K + 31) / 32, n_st = 2 * n_ch;   // the planes of a K that is no multiple of 32 end in zeros

  const char* baseA = reinterpret_cast<const char*>(g.A + m0 * g.lda);   // uniform, and a lane's offset
  uint32_t offA[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int row = wm0 + i * 32 + l32;
    offA[i] = (uint32_t)(m0 + row < g.M ? row : (int)(g.M - 1 - m0)) * (uint32_t)(g.lda * 4) + kh * 32u;
  }
  f32x4 ra[2][MB][2];   // [step][block][half]: a chunk on its way
  auto fetchA = [&](int c) __attribute__((always_inline)) {
    c = c < n_ch ? c : n_ch - 1;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int k = c * 32 + ks * 16 < g.K ? c * 32 + ks * 16 : 0;   // past the end: any values, their weights are zero
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) ra[ks][i][h] = *reinterpret_cast<const f32x4*>(baseA + (int64_t)k * 4 + h * 16 + offA[i]);
    }
  };
  // KB q of a chunk: column block q / 4, step (q % 4) / 2, plane q % 2
  const int nb = (g.N + 31) / 32;                       // column blocks of the planes; past the last: that one again, never stored
  const char* srcB = reinterpret_cast<const char*>(g.B);
  auto issueB = [&](int c, int buf) __attribute__((always_inline)) {
    c = c < n_ch ? c : n_ch - 1;
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int q = wave * PB + i;
      const int blk = n0 / 32 + q / 4 < nb ? n0 / 32 + q / 4 : nb - 1;
      __builtin_amdgcn_global_load_lds((global_void_ptr)(srcB + (((int64_t)blk * n_st + 2 * c) * GROUP_B + (q % 4) * FRAG_B) + (uint32_t)lane * 16u),
                                       (lds_void_ptr)(lds + buf * CHUNK_B + q * 1024), 16, 0, 0);
    }
  };

  // W takes the place of the first operand, so a lane's column of the result is one row of A, whose scale is then a lane's
  f16x8 hi[2][MB], lo[2][MB];   // [step][block]
  float inv[MB];
  uint32_t from[MB];   // smaller values of the row wait for a pass of their own
  auto splitA = [&](int c) __attribute__((always_inline)) {   // returns whether there are any
    bool below = false;
    uint32_t most[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      value_range r;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 4; q += 2) r.add(ra[ks][i][h][q], ra[ks][i][h][q + 1]);
      most[i] = max_halves(r.most());   // the other 8 k of the row's steps
      from[i] = keeps_from(most[i]);
      below |= any_below(r, from[i]);
    }
    const bool more = __any(below);
    if (more) {
      asm volatile("");   // a branch, which is rarely taken
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if ((__float_as_uint(ra[ks][i][h][q]) & 0x7FFFFFFFu) < from[i]) ra[ks][i][h][q] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int se = scale_exp(most[i]);
      const bool turn = ((c ^ l32) & 1) == 0;
      const float sc = turned(pow2(se), turn);
      inv[i] = turned(pow2(-14 - se), turn);   // the columns' factors carry 2^14 back: the sums stay where the products of the fp32 values are
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = ra[ks][i][0][q] * sc, v[4 + q] = ra[ks][i][1][q] * sc;
        split8(v, hi[ks][i], lo[ks][i]);
      }
    }
    return more;
  };
  auto restA = [&](int c) __attribute__((always_inline)) {   // the values that wait
    fetchA(c);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if ((__float_as_uint(ra[ks][i][h][q]) & 0x7FFFFFFFu) >= from[i]) ra[ks][i][h][q] = 0.f;
  };

  f32x16 acc[MB][NB], t[TD][MB][JB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  f16x8 w[WD][2][PL][JB];   // [parity of the group][step][plane][block]
  auto readW = [&](int buf, int q) __attribute__((always_inline)) {
    const char* sb = lds + buf * CHUNK_B + lane * 16 + q * JB * 2 * GROUP_B;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int jj = 0; jj < JB; ++jj)
#pragma unroll
        for (int p = 0; p < PL; ++p) w[q % WD][ks][p][jj] = *reinterpret_cast<const f16x8*>(sb + (jj * 2 + ks) * GROUP_B + p * FRAG_B);
  };
  auto products = [&](int q) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int jj = 0; jj < JB; ++jj)
#pragma unroll
        for (int v = 0; v < 16; ++v) t[q % TD][i][jj][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int jj = 0; jj < JB; ++jj)
            t[q % TD][i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[q % WD][ks][x == 1][jj], x == 0 ? lo[ks][i] : hi[ks][i],
                                                                     t[q % TD][i][jj], 0, 0, 0);
  };
  auto add = [&](int q) __attribute__((always_inline)) {   // a group's sums over the chunk
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int jj = 0; jj < JB; ++jj)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][q * JB + jj][v] = __builtin_fmaf(t[q % TD][i][jj][v], inv[i], acc[i][q * JB + jj][v]);
  };

  const float* inv_n = reinterpret_cast<const float*>(reinterpret_cast<const char*>(g.B) + (int64_t)nb * n_st * GROUP_B);
  const uint32_t* out = reinterpret_cast<const uint32_t*>(inv_n + nb * 32);
  const uint32_t out_l = lane < NB && n0 / 32 + lane < nb ? out[n0 / 32 + lane] : 0u;   // asked for here, looked at below
#pragma unroll
  for (int c = 0; c < NBUF - 1; ++c) issueB(c, c);
  __builtin_amdgcn_sched_barrier(0);
  fetchA(0);
  __builtin_amdgcn_sched_barrier(0);
  wait_vmcnt_lgkmcnt0<4 * MB>();
  const uint32_t cols_out = (uint32_t)__ballot(out_l != 0u);
  __syncthreads();
  int bb = 0;
  for (int c = 0; c < n_ch; ++c) {
    readW(bb, 0);
    bool more = splitA(c);
    issueB(c + NBUF - 1, bb == 0 ? NBUF - 1 : bb - 1);
    for (;;) {
      __builtin_amdgcn_sched_barrier(0);   // the wait at the end counts on this order of the loads
      fetchA(c + 1);
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        if (WD == 2 && q + 1 < NG) readW(bb, q + 1);
        __builtin_amdgcn_sched_barrier(0);
        products(q);
        if (WD == 1 && q + 1 < NG) readW(bb, q + 1);
        if (TD == 2 && q > 0) add(q - 1);   // while this group's products run
        if (TD == 1) add(q);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (TD == 2) add(NG - 1);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc[i][j]));   // the additions stay on this side of the branch
      if (!more) break;
      restA(c);   // every pass takes the largest of what is left, and SPAN powers of two below it
      readW(bb, 0);
      more = splitA(c);
    }
    wait_vmcnt_lgkmcnt0<4 * MB + (NBUF - 2) * (PB + 4 * MB)>();
    __syncthreads();
    bb = bb == NBUF - 1 ? 0 : bb + 1;
  }
  wait_vmcnt_lgkmcnt0<0>();

  // The 16 k that W's planes leave out: these rows of W times A's values, both from memory, two k an instruction (fp32).  The sums are in
  // units of the columns' factors.
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int blk = n0 / 32 + j;
    if (!(cols_out >> j & 1u)) continue;
    const int n = blk * 32 + l32 < g.N ? blk * 32 + l32 : g.N - 1;
    const int back = (int)(__float_as_uint(inv_n[n]) >> 23) - 127;
    const int64_t w_k = g.w_k_rows ? g.N : 1;
    const float* wn = g.W + n * (int64_t)(g.w_k_rows ? 1 : g.K) + 8 * kh * w_k;
#pragma unroll 1
    for (int s0 = 0; s0 < n_st; s0 += 64) {
      uint64_t steps = __ballot(s0 + lane < n_st && out[nb + (int64_t)blk * n_st + s0 + lane] != 0u);   // none past K
#pragma unroll 1
      for (; steps; steps &= steps - 1) {
        const int k = (s0 + __builtin_ctzll(steps)) * 16;
        float w[8], a[MB][8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          w[q] = __builtin_ldexpf(wn[(k + q) * w_k], -back);
#pragma unroll
          for (int i = 0; i < MB; ++i) a[i][q] = *reinterpret_cast<const float*>(baseA + (int64_t)(k + q) * 4 + offA[i]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int i = 0; i < MB; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[q], a[i][q], acc[i][j], 0, 0, 0);
      }
    }
  }
  __syncthreads();
  float* stage = smem + wave * (32 * EPI_LD);
  switch (g.epi_mask) {   // uniform
#define GP_EM_CASE(M) case M: epilogue_blocks<MB, NB, M>(g, acc, stage, m0 + wm0, n0, inv_n); break;
    GP_EM_LIST_PLANES(GP_EM_CASE)
#undef GP_EM_CASE
    default: break;   // not launched with any other mask
  }
}

// C = A^T B, the contraction running over the rows of both (the weight gradients: rows = edges), of several matrix pairs at once.  Every
// value enters as the sum of three bf16 numbers, each with its own exponent (24 bits), and the six of the nine products that are not
// below 2^-24 of the whole are formed: a column of A becomes a row of the result, next to columns of any other size, and rows of any
// size meet in a sum, so there is no scale that could be shared.
// A chunk is 16 rows.  The loads are those of an operand: lane (kh, x) takes 8 consecutive rows of column x, one value a load (256
// bytes of two rows per instruction), so the parts are written to LDS as fragments and nothing is transposed.  A wavefront loads
// LA + LB blocks of 32 columns a chunk ahead and splits them once for the whole workgroup.
// Two buffers, one barrier a chunk.  Workgroup = (split of the rows, product, tile); partial sums [split, M, N] of every product and column
// sums of B (bias gradients, from the fp32 values, each chunk by one of the tiles that share it).
// 256 x 256 with 8 wavefronts of 128 x 64 where that many columns exist, else 128 x 128 with 4 of 64 x 64 (two workgroups per
// compute unit).  43380 rows, 2048 x 2048 1.91 ms, 256 x 256 42 us, 6 x 256 25; 13230, 256 x 256 19; 434, 256 x 256 7.7; 336, 32 x 32 6.1.  Two fp16
// parts under shared scales take 1.38 ms, 39, 32, 19, 7.3 and 6.5, and lose what is 2^17 smaller than its neighbours; with every such
// value sought out and added in fp32 they took 1.7 ms, 46, - and 27.
// Sums are of few chunks (FOLD: not for lack of registers), every second one of them with the sign of A's values turned, and go to a second
// set by fp32 additions: the matrix instruction's sums come out low (above), and a run of a product that shares its launch has thousands of
// rows.  Column sums are formed in fp64, eight rows at a time.  How many chunks: few where a run has few of them, more where the additions
// to the second set would be many, and no fewer than the error asks for (4 in the place of 8 costs a training step of 43380 x 256 1 per
// cent).  Relative error against 64 bits (1e-7) of a block's products of 256 x 256 together, and of one by itself in sums of one sign that
// are as long as its runs: 434 rows 0.91 (1.04), 1500 1.26 (1.42), 7593 1.40 (1.62), 13230 1.47 (2.02), 22730 1.81 (2.42), 43380 1.82 (3.24),
// 120000 1.88 (5.50); column sums 0.47 (0.85) to 0.25 (0.66).  Sums of 16 chunks and one sign: 1.23, 1.94, 2.47, 2.56, 2.69, 2.83, 3.17.
constexpr int TN_ROWS = 16, TN_BLOCK_B = 3 * FRAG_B;   // rows of a chunk, bytes of its three parts for 32 columns
// chunks of a sum, for runs of `per` rows
inline int tn_fold(int64_t per) { return per <= 8 * TN_ROWS ? 2 : per <= 96 * TN_ROWS ? 4 : 8; }
template <int JOBS>
struct tn_args {
  gp_tn_part_job j[JOBS];   // tiles first, first + 1, ... of a split belong to a product
  int n, tiles, fold;       // fold: chunks of a sum
  int64_t rows, per;
};
template <int MB, int NB, int WAVES_M, int WAVES_N, int OCC, bool FOLD, int JOBS>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N, OCC)
gemm_parts_tn_kernel(const tn_args<JOBS> q) {
  constexpr int NW = WAVES_M * WAVES_N, BA = MB * WAVES_M, BB = NB * WAVES_N;   // 32-wide blocks of the operands
  constexpr int LA = BA / NW, LB = BB / NW;                                     // ... a wavefront loads
  static_assert(BA % NW == 0 && BB % NW == 0, "blocks are dealt evenly");
  constexpr int BUF_B = (BA + BB) * TN_BLOCK_B;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  char* lds = reinterpret_cast<char*>(smem);

  const int work = xcd_remap(blockIdx.x, gridDim.x);   // the tiles of a split (same rows) side by side
  const int split = work / q.tiles, t = work % q.tiles;
  int job = 0;
  if constexpr (JOBS > 1)
    while (job + 1 < q.n && t >= q.j[job + 1].first) ++job;
  const gp_tn_part_job& jb = q.j[job];
  const int M = jb.M, N = jb.N, tile = t - jb.first;
  const int tiles_n = (N + 32 * BB - 1) / (32 * BB), tiles_m = (M + 32 * BA - 1) / (32 * BA);
  const int tile_m = tile / tiles_n;
  const int m0 = tile_m * 32 * BA, n0 = (tile % tiles_n) * 32 * BB;
  const int64_t k_begin = (int64_t)split * q.per;
  const int64_t k_end = k_begin + q.per < q.rows ? k_begin + q.per : q.rows;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave / WAVES_N) * MB, wn = (wave % WAVES_N) * NB;             // first blocks of the wavefront's products
  const int kh = lane >> 5, l32 = lane & 31;
  const int n_ch = (int)((k_end - k_begin + TN_ROWS - 1) / TN_ROWS);

  // loads: lane (kh, x) takes column x of a block, rows 8 kh .. + 7: a uniform address that moves with the rows plus the lane's offset
  constexpr int NL = LA + LB;
  const char* base[NL];
  int64_t ldb[NL];       // bytes per row
  uint32_t off[NL];
#pragma unroll
  for (int b = 0; b < NL; ++b) {
    const bool is_a = b < LA;
    const int x0 = is_a ? m0 + (wave * LA + b) * 32 : n0 + (wave * LB + b - LA) * 32, width = is_a ? M : N;
    const int xb = x0 < width ? x0 : 0;   // a block past the matrix reads its first columns and is not stored
    ldb[b] = (int64_t)width * 4;
    base[b] = reinterpret_cast<const char*>((is_a ? jb.A : jb.B) + xb);
    off[b] = (uint32_t)(8 * kh * ldb[b]) + 4u * (uint32_t)(xb + l32 < width ? l32 : width - 1 - xb);
  }
  float raw[NL][8];
  auto fetch = [&](int c) __attribute__((always_inline)) {
    c = c < n_ch ? c : n_ch - 1;
    const int64_t k0 = k_begin + (int64_t)c * TN_ROWS;
    if (k0 + TN_ROWS <= k_end) {
#pragma unroll
      for (int b = 0; b < NL; ++b) {
        const char* p = base[b] + k0 * ldb[b];
#pragma unroll
        for (int r = 0; r < 8; ++r) raw[b][r] = *reinterpret_cast<const float*>(p + r * ldb[b] + off[b]);
      }
    } else {   // the last rows of the split: a valid row in the place of those past the end, then zero
#pragma unroll
      for (int b = 0; b < NL; ++b)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int64_t k = k0 + 8 * kh + r;
          const float v = *reinterpret_cast<const float*>(base[b] + ((k < k_end ? k : k_end - 1) - 8 * kh) * ldb[b] + off[b]);
          raw[b][r] = k < k_end ? v : 0.f;
        }
    }
  };
  double cs[LB];
#pragma unroll
  for (int b = 0; b < LB; ++b) cs[b] = 0.0;
  const bool want_cs = jb.colsum_part != nullptr;
  // chunk c of the loaders' registers goes to LDS buffer u
  auto store = [&](int c, int u, uint32_t turn) __attribute__((always_inline)) {
    const bool mine = want_cs && c % tiles_m == tile_m;
#pragma unroll
    for (int b = 0; b < NL; ++b) {
      const int blk = b < LA ? wave * LA + b : BA + wave * LB + b - LA;
      bf16x8 part[3];
      if (FOLD && b < LA) {
#pragma unroll
        for (int r = 0; r < 8; ++r) raw[b][r] = __uint_as_float(__float_as_uint(raw[b][r]) ^ turn);
      }
      parts8(raw[b], part);
      char* dst = lds + u * BUF_B + blk * TN_BLOCK_B + lane * 16;
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8*>(dst + p * FRAG_B) = part[p];
      if (b >= LA && mine) {
        const float* r = raw[b];
        cs[b - LA < 0 ? 0 : b - LA] += (double)(((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7])));
      }
    }
  };

  f32x16 acc[MB][NB], whole[FOLD ? MB : 1][FOLD ? NB : 1];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][j][v] = 0.f;
        if constexpr (FOLD) whole[i][j][v] = 0.f;
      }
  auto multiply = [&](int u, auto begin) __attribute__((always_inline)) {   // begin: of a sum
    const char* sa = lds + u * BUF_B + wm * TN_BLOCK_B + lane * 16;
    const char* sb = lds + u * BUF_B + (BA + wn) * TN_BLOCK_B + lane * 16;
    bf16x8 b[NB][3];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int p = 0; p < 3; ++p) b[j][p] = *reinterpret_cast<const bf16x8*>(sb + j * TN_BLOCK_B + p * FRAG_B);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      bf16x8 a[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) a[p] = *reinterpret_cast<const bf16x8*>(sa + i * TN_BLOCK_B + p * FRAG_B);
      constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};   // the smallest first
#pragma unroll
      for (int x = 0; x < 6; ++x)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[x]], b[j][PB[x]], decltype(begin)::value && x == 0 ? f32x16{} : acc[i][j], 0, 0, 0);
    }
  };
  auto fold = [&](float sign) __attribute__((always_inline)) {
    if constexpr (FOLD) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) whole[i][j][v] = __builtin_fmaf(acc[i][j][v], sign, whole[i][j][v]);
    }
  };

  if (n_ch > 0) {
    uint32_t turn = 0;         // of the values in the buffer that is filled next
    float sign = 1.f;          // of the sums in acc
    int left = q.fold, in = q.fold - 1;   // chunks until the next fold, and until the next turn of the loaders
    fetch(0);
    store(0, 0, turn);
    fetch(1);
    __syncthreads();
    for (int c = 0; c < n_ch; ++c) {
      const int u = c & 1;
      if (c + 1 < n_ch) {
        if (FOLD && in == 0) turn ^= 0x80000000u, in = q.fold;
        --in;
        store(c + 1, u ^ 1, turn);
        fetch(c + 2);
      }
      if (FOLD && left == q.fold) multiply(u, std::true_type());
      else multiply(u, std::false_type());
      if (FOLD && --left == 0) {
        fold(sign);
        sign = -sign;
        left = q.fold;
      }
      __syncthreads();
    }
    if (left < q.fold) fold(sign);
  }
  __syncthreads();
  if (want_cs) {
#pragma unroll
    for (int b = 0; b < LB; ++b) {
      const float sum = (float)(cs[b] + __shfl_xor(cs[b], 32, 64));
      const int n = n0 + (wave * LB + b) * 32 + l32;
      if (kh == 0 && n < N) jb.colsum_part[((int64_t)split * tiles_m + tile_m) * N + n] = sum;
    }
  }
  gemm_args g{};
  g.M = M; g.N = N; g.part = jb.part; g.vecC = jb.vec;
  if constexpr (FOLD) tile_epilogue_f32<MB, NB, MODE_TN>(g, whole, smem, m0, n0, wm * 32, wn * 32, split);
  else tile_epilogue_f32<MB, NB, MODE_TN>(g, acc, smem, m0, n0, wm * 32, wn * 32, split);
}

// JOBS: room for that many products in the launch's arguments (with room for 24, a launch takes a microsecond longer)
template <int MB, int NB, int WMS, int WNS, int OCC, bool FOLD, int JOBS>
int launch_parts_tn(gp_ctx* ctx, const gp_tn_part_job* jobs, int n, int64_t rows, int64_t per, int splits) {
  constexpr int BA = MB * WMS, BB = NB * WNS, NW = WMS * WNS;
  tn_args<JOBS> q;
  q.n = n; q.rows = rows; q.per = per; q.fold = tn_fold(per);
  int64_t tiles = 0;
  double flops = 0.0, bytes = 0.0;
  for (int i = 0; i < n; ++i) {
    q.j[i] = jobs[i];
    q.j[i].first = (int)tiles;
    tiles += (int64_t)((jobs[i].M + 32 * BA - 1) / (32 * BA)) * ((jobs[i].N + 32 * BB - 1) / (32 * BB));
    flops += 2.0 * (double)jobs[i].M * jobs[i].N * rows;
    bytes += 4.0 * ((double)(jobs[i].M + jobs[i].N) * rows + (double)jobs[i].M * jobs[i].N * splits);
  }
  if (tiles * splits > INT32_MAX) return gp_fail(ctx, GP_BAD_ARG, "gemm: too many tiles");
  q.tiles = (int)tiles;
  static char name[48];
  if (!name[0]) snprintf(name, sizeof(name), "gemm_f32x3_tn_%dx%d", 32 * BA, 32 * BB);
  gp_prof_scope prof(ctx, name, flops, bytes);
  constexpr size_t lds_main = 2 * (size_t)(BA + BB) * TN_BLOCK_B;
  constexpr size_t lds_epi = sizeof(float) * NW * 32 * EPI_LD;
  constexpr size_t lds = lds_main > lds_epi ? lds_main : lds_epi;
  static bool raised = false;
  if (!raised && lds > 64 * 1024) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_parts_tn_kernel<MB, NB, WMS, WNS, OCC, FOLD, JOBS>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return gp_fail(ctx, GP_HIP_ERROR, "gemm: cannot raise the dynamic LDS limit to %zu bytes", lds);
    raised = true;
  }
  gemm_parts_tn_kernel<MB, NB, WMS, WNS, OCC, FOLD, JOBS><<<dim3((unsigned)(tiles * splits)), 64 * NW, lds, ctx->stream>>>(q);
  GP_LAUNCH_CHECK(ctx, "gemm_parts_tn_kernel");
  return GP_OK;
}

template <int MB, int NB, int WAVES, int NBUF, int OCC, int JB, int TD, int WD>
int launch_planes(gp_ctx* ctx, gemm_args& g) {
  constexpr int BM = 32 * MB * WAVES, BN = 32 * NB;
  const int64_t tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  if (tiles > INT32_MAX) return gp_fail(ctx, GP_BAD_ARG, "gemm: too many tiles");
  static char name[48];
  if (!name[0]) snprintf(name, sizeof(name), "gemm_f32x2_%dx%d", BM, BN);
  const double mnk = (double)g.M * g.N * g.K;
  gp_prof_scope prof(ctx, name, 2.0 * mnk, 4.0 * ((double)g.M * g.K + (double)g.K * g.N + (double)g.M * g.N));
  constexpr size_t lds_main = (size_t)NBUF * NB * 2 * GROUP_B;
  constexpr size_t lds_epi = sizeof(float) * WAVES * 32 * EPI_LD;
  constexpr size_t lds = lds_main > lds_epi ? lds_main : lds_epi;
  static bool raised = false;
  if (!raised && lds > 64 * 1024) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_planes_kernel<MB, NB, WAVES, NBUF, OCC, JB, TD, WD>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return gp_fail(ctx, GP_HIP_ERROR, "gemm: cannot raise the dynamic LDS limit to %zu bytes", lds);
    raised = true;
  }
  gemm_planes_kernel<MB, NB, WAVES, NBUF, OCC, JB, TD, WD><<<dim3((unsigned)tiles), 64 * WAVES, lds, ctx->stream>>>(g);
  GP_LAUNCH_CHECK(ctx, "gemm_planes_kernel");
  return GP_OK;
}

inline bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

size_t gp_planes_bytes(int N, int K) {
  const size_t nb = (size_t)(N + 31) / 32, k16 = (size_t)((K + 31) / 32 * 2);
  return nb * k16 * GROUP_B + nb * (32 + 1 + k16) * sizeof(float);
}

// From K = 64 on the error is the smaller one (above).  At K = 64 a short product is launch and epilogue, which both forms have
// (13505 x 256 x 64: 14.9 us in 64 x 64 tiles, 17.2 in 128 x 128, three bf16 parts 16.2; 43045 x 256 x 64: 39.8, three bf16 parts 45.8;
// 5448 x 64 x 64: 7.7, 7.5; 5448 x 256 x 64: 10.1, 13.0); the conversion of all weights of a call is one launch (6.5 us at width 256, 88 at 2048).
bool gp_planes_take(const gp_ctx* ctx, int64_t M, int N, int K) {
  return ctx->f32_split && !ctx->gemm_bf16 && K % 16 == 0 && N % 4 == 0 && N >= 64 && N <= 8192 && K <= 8192 &&
         (K >= 128 || (K >= 64 && M >= 8192));
}

int gp_weight_planes::run() {
  if (n == 0) return GP_OK;
  plane_jobs pj{};
  int most = 0;
  double bytes = 0.0;
  for (int i = 0; i < n; ++i) {
    pj.j[i] = jobs[i];
    most = std::max(most, (jobs[i].N + 31) / 32);
    bytes += 8.0 * jobs[i].N * jobs[i].K;
  }
  gp_prof_scope prof(ctx, "make_planes", 0.0, bytes);
  make_planes_kernel<<<dim3((unsigned)most, (unsigned)n), 64 * PREP_WAVES, 0, ctx->stream>>>(pj);
  GP_LAUNCH_CHECK(ctx, "make_planes_kernel");
  return GP_OK;
}

namespace {

// GP_OK, an error, or 1: not taken
int gemm_planes(gp_ctx* ctx, const float* A, const float* W, int k_rows, const void* planes, int64_t M, int N, int K, const gp_epilogue& epi) {
  gemm_args g{};
  g.W = W; g.w_k_rows = k_rows;
  g.A = A; g.B = static_cast<const float*>(planes); g.M = M; g.N = N; g.K = K; g.lda = K;
  g.epi = epi;
  g.vecC = al16(epi.bias) && al16(epi.add_pre) && al16(epi.save_pre) && al16(epi.zsrc) && al16(epi.mul) && al16(epi.add_post) &&
           al16(epi.out) && al16(epi.out2) && al16(epi.z2src);
  g.epi_mask = gp_epilogue_mask(g.epi, g.vecC);
  if (!planes || !al16(A) || !epilogue_listed(g.epi_mask)) return 1;
  GP_REQUIRE(ctx, M >= 0 && gp_planes_take(ctx, 8192, N, K), "gemm: planes of a shape that has none");
  if (M == 0) return GP_OK;
  // Tiles: 128 x 256 where there are enough of them for several rounds of two per compute unit (43045 x 2048 x 2048: 1.24 ms, with
  // 128 x 128 1.37; 13505 x 1024 x 1024, 424 tiles: 0.128, 0.150; 21612 x 512 x 512, 338: 0.074, 0.069; 8131 x 1024 x 1024, 256: 0.085,
  // 0.080); 64 x 64 where a launch of 128 x 128 leaves compute units idle or the matrix has 64 columns (2667 x 256 x 256: 14.7 us,
  // 128 x 128 20.5; 18844 x 128 x 128, 148 tiles: 14.1, 16.8; 27036 x 256 x 256, 424: 43.5, 31.0; 10790 x 512 x 512, 340: 47, 43).  The two
  // meet between 250 and 340 tiles (13505 x 256 x 256, 212: 20.6, 22.5; 16180, 254: 22.5, 23.8; 21612, 338: 29.6, 30.2; 8131 x 512 x 512,
  // 256: 34.5, 35.5): the line stands where it was drawn for products without passes over small values (210 tiles: 16.2, 15.3).
  // The values of the result do not depend on the choice.
  const int64_t rows = (M + 127) / 128;
  if (N >= 512 && rows * ((N + 255) / 256) >= 400) return launch_planes<1, 8, 4, 2, 2, 1, 2, 1>(ctx, g);
  if (N > 64 && rows * ((N + 127) / 128) >= 192) return launch_planes<1, 4, 4, 2, 3, 1, 1, 1>(ctx, g);
  return launch_planes<1, 2, 2, 3, 3, 1, 2, 2>(ctx, g);
}

}  // namespace

int gp_gemm_nn_w(gp_ctx* ctx, const float* A, const float* W, const void* planes, int64_t M, int N, int K, const gp_epilogue& epi) {
  const int rc = gemm_planes(ctx, A, W, 1, planes, M, N, K, epi);
  return rc == 1 ? gp_gemm_nn(ctx, A, W, M, N, K, epi) : rc;
}
int gp_gemm_nt_w(gp_ctx* ctx, const float* A, const float* W, const void* planes, int64_t M, int N, int K, const gp_epilogue& epi) {
  const int rc = gemm_planes(ctx, A, W, 0, planes, M, N, K, epi);
  GP_REQUIRE(ctx, rc != 1 || epi.act != 3, "gemm: the gate's step needs planes and 16-byte aligned matrices");
  return rc == 1 ? gp_gemm_nt(ctx, A, W, M, N, K, epi) : rc;
}

// Products of small tiles in one launch share its splits: so many that the workgroups of all of them fill the chip once.
int gp_parts_tn_splits(int64_t rows, int64_t tiles) {
  const int64_t runs = std::max(std::min<int64_t>((rows + 31) / 32, 32), (rows + 63) / 64);
  return (int)std::max<int64_t>(std::min(512 / tiles, runs), 1);
}

// Tiles and splits.  About one or two workgroups per compute unit; few rows are cut into short runs, since a workgroup spends 1 us
// on a chunk by itself: of 32 rows up to 1024 rows, then 32 runs up to 2048, then of 64 rows.  `most` grows with the rows, `splits` (rounded
// to whole chunks) need not: scratch is sized by the former, so that what serves a graph serves every smaller one.
gp_tn_parts_plan gp_parts_tn_plan(int64_t rows, int M, int N) {
  gp_tn_parts_plan p;
  p.big = (int64_t)(M / 256) * (N / 256) >= 4;
  const int T = p.big ? 256 : 128;
  p.tiles_m = (M + T - 1) / T;
  const int64_t tiles = (int64_t)p.tiles_m * ((N + T - 1) / T);
  const int64_t s = p.big ? std::max<int64_t>(std::min(256 / tiles, (rows + 255) / 256), 1) : gp_parts_tn_splits(rows, tiles);
  p.most = (int)s;
  p.per = std::max<int64_t>(((rows + s - 1) / s + 31) / 32 * 32, 32);   // no rows: one empty split, for the size of its scratch
  p.splits = (int)((rows + p.per - 1) / p.per);
  return p;
}

int gp_parts_tn_launch(gp_ctx* ctx, bool big, const gp_tn_part_job* jobs, int n, int64_t rows, int64_t per, int splits) {
  GP_REQUIRE(ctx, n >= 1 && n <= (big ? 1 : GP_TN_JOBS_MAX), "gemm_tn: number of products");
  if (big) return launch_parts_tn<4, 2, 2, 4, 2, false, 1>(ctx, jobs, n, rows, per, splits);
  if (n == 1) return launch_parts_tn<2, 2, 2, 2, 2, true, 1>(ctx, jobs, n, rows, per, splits);
  return launch_parts_tn<2, 2, 2, 2, 2, true, GP_TN_JOBS_MAX>(ctx, jobs, n, rows, per, splits);
}
