// Chains of dense layers over the edges in one launch (fp32).  The layers of a block between two triplet sums act on every row by itself,
// and one after the other they are bound by what a short product cannot hide: its first loads, its epilogue, and the rows written
// and read back between two layers.  Here a wavefront takes 16 rows through all of them: the result of a layer is the operand of the
// next one without leaving the registers.
//
// Arithmetic: every value enters as the sum of three bf16 numbers, each with its own exponent (24 bits), and the six products of the
// parts that are not below 2^-24 of the whole are formed, smallest first.  The 32 k of a chunk are summed from zero, half of the sums with
// the sign of the row's values turned round (the matrix instruction's sums come out low on average, whatever their sign), and enter the
// result by an fp32 addition.  Relative error of three blocks against 64 bits, layer by layer / as chains: width 64, messages 2.2e-7 / 1.3e-7,
// input gradient 3.1e-7 / 1.9e-7; 128, 1.9e-7 / 1.3e-7 and 2.9e-7 / 2.0e-7; 256, 1.8e-7 / 1.4e-7 and 3.0e-7 / 2.2e-7.
//
// Layout: with the weights as first operand of v_mfma_f32_16x16x32_bf16, lane (q, r) = (lane / 16, lane % 16) holds of row r the columns
// 16 b + 4 q .. + 3 of every 16-column block b.  That is also how the lanes load and store rows (16 bytes a lane, 64 a row), and it is an
// operand fragment for the next product once the weights' k are dealt the same way: element i of lane q in chunk c is
// k = 32 c + 16 (i / 4) + 4 q + i % 4.
//
// The weights of all layers lie in the order in which they are used, as fragments of 16 columns x 32 k x 3 parts (3 KB), and stream through
// a ring of three LDS stages of half the columns by 32 k (global->LDS loads, two stages ahead, across the layers).
//
// A layer of width 256 takes a wavefront that has its SIMD for itself 15 us, of which the matrix unit is busy 5, the rest being its splitting, its
// epilogue and waits for LDS; two to a SIMD, which two workgroups of 64 rows per compute unit make, 24.  Eight layers with their
// stores: 336 rows x 32 14 us, 4000 x 128 54, 13230 x 256 147, 32768 x 256 274.  A ring of six stages makes no difference.
#include <stdarg.h>

#include <type_traits>

#include "gemm_common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(1))) void* global_void_ptr;

constexpr int CHAIN_ROWS = 64, CHAIN_WAVES = 4;        // rows and wavefronts of a workgroup
constexpr int PART_B = 1024, FRAG3_B = 3 * PART_B;     // one part of a fragment, a fragment
constexpr int blocks_per_stage(int nb) { return nb <= 8 ? nb : nb / 2; }
constexpr int stage_bytes(int nb) { return (blocks_per_stage(nb) * FRAG3_B + 4095) / 4096 * 4096; }

// LDS reads done and all but the last N loads and stores
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkmcnt0() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}
// The barrier alone: __syncthreads() also waits for every load in flight, those of the stages ahead among them.
__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---- the weights of a chain, converted by one launch
struct part_job {
  const float* src;
  int N, K, k_rows;   // k_rows: src is [K, N], else [N, K]
  int first;          // first stage
};
struct part_jobs {
  part_job j[GP_CHAIN_MAX];
  int n;
};
template <int NB>
__global__ void __launch_bounds__(256) make_parts_kernel(const part_jobs q, char* __restrict__ dst) {
  constexpr int NBS = blocks_per_stage(NB), HALVES = NB / NBS;
  const int stage = blockIdx.x;
  int job = 0;
  while (job + 1 < q.n && stage >= q.j[job + 1].first) ++job;
  const part_job& p = q.j[job];
  const int s = stage - p.first, halves = (p.N + 16 * NBS - 1) / (16 * NBS), c = s / halves;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  static_assert(HALVES <= 2, "stages hold half of the columns");
  for (int b = threadIdx.x >> 6; b < NBS; b += 4) {
    const int n = ((s % halves) * NBS + b) * 16 + (lane & 15);
    bf16x8 part[3];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 32 * c + 16 * (i / 4) + 4 * g + i % 4;
      float r = n < p.N && k < p.K ? p.src[p.k_rows ? (int64_t)k * p.N + n : (int64_t)n * p.K + k] : 0.f;
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        part[x][i] = (__bf16)r;
        r -= (float)part[x][i];
      }
    }
    char* d = dst + (int64_t)stage * stage_bytes(NB) + b * FRAG3_B + lane * 16;
#pragma unroll
    for (int x = 0; x < 3; ++x) *reinterpret_cast<bf16x8*>(d + x * PART_B) = part[x];
  }
}

// What a value meets in the epilogue.  The first operand's loads go out before the last products of the layer, into the registers of the
// layer's own operand, which are free by then; the second's in groups of blocks, one group ahead.
enum : uint32_t {
  CF_LOAD = 1, CF_LOAD_Z = 2, CF_BIAS = 4, CF_P1 = 8, CF_P2 = 16, CF_ADD_PRE = 32, CF_SAVE = 64, CF_ACT = 128, CF_GATE = 256, CF_MUL = 512,
  CF_ADD = 1024, CF_ADD2 = 2048, CF_OUT = 4096, CF_Z = 8192, CF_Z2 = 16384, CF_KEEP = 32768
};
// the steps behind the operand that belong together in one of a block's layers; a loop over the blocks is compiled for each (options tested
// block by block cost more branches than a layer of 128 columns has products: 16 000 of its 20 000 cycles)
constexpr uint32_t CF_STEPS = CF_P1 | CF_P2 | CF_ADD_PRE | CF_SAVE | CF_ACT | CF_GATE | CF_MUL | CF_ADD | CF_ADD2 | CF_OUT | CF_Z | CF_Z2;
#define GP_CHAIN_STEPS(X)                                                                                                            \
  X(CF_OUT) X(CF_SAVE | CF_ACT | CF_OUT) X(CF_SAVE | CF_ACT | CF_OUT | CF_P1 | CF_MUL) X(CF_SAVE | CF_ACT | CF_OUT | CF_P1 | CF_ADD) \
  X(CF_P1 | CF_Z) X(CF_OUT | CF_P1 | CF_Z) X(CF_OUT | CF_P1 | CF_ADD | CF_P2 | CF_Z2) X(CF_P1 | CF_P2 | CF_GATE)                     \
  X(CF_OUT | CF_P1 | CF_ADD_PRE | CF_P2 | CF_ADD2)
bool steps_listed(uint32_t flags) {
  switch (flags & CF_STEPS) {
#define GP_CASE(M) case M:
    GP_CHAIN_STEPS(GP_CASE)
#undef GP_CASE
    return true;
    default: return false;
  }
}
struct chain_step {
  const float *load, *load_z, *bias, *p1, *p2;
  float *load_out, *save_pre, *out, *out2, *out3;
  int N, K;
  uint32_t flags;
};
struct chain_args {
  chain_step s[GP_CHAIN_MAX];
  const char* W;
  int64_t rows;
  int n, stages;
};
// in a scalar register from here on: tested and used block by block, a field that is read again each time costs its latency each time
template <class T>
__device__ __forceinline__ T pinned(T v) {
  asm volatile("" : "+s"(v));
  return v;
}

template <int NB>
__global__ void __launch_bounds__(64 * CHAIN_WAVES, 2)
dense_chain_kernel(const chain_args q) {
  constexpr int NBS = blocks_per_stage(NB), HALVES = NB / NBS, STAGE_B = stage_bytes(NB), CH = NB / 2;
  constexpr int PER = STAGE_B / 1024 / CHAIN_WAVES;   // global->LDS loads of a wavefront per stage
  constexpr int GRP = NB < 4 ? NB : 4;                // blocks of a group in the epilogue
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * CHAIN_ROWS + wave * 16 + (lane & 15);
  const bool inside = row0 < q.rows;
  const int64_t row = inside ? row0 : q.rows - 1;

  int next = 0, fill = 0;   // the next stage to be asked for, and the buffer it goes to
  auto issue = [&]() __attribute__((always_inline)) {
    const char* src = q.W + (int64_t)(next < q.stages ? next : q.stages - 1) * STAGE_B + wave * PER * 1024 + lane * 16;
    char* dst = lds + fill * STAGE_B + wave * PER * 1024;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_global_load_lds((global_void_ptr)(src + i * 1024), (lds_void_ptr)(dst + i * 1024), 16, 0, 0);
    __builtin_amdgcn_sched_barrier(0);   // the waits below count on this order of the loads
    ++next;
    fill = fill == 2 ? 0 : fill + 1;
  };
  auto st = [&](float* p, int64_t o, f32x4 v) __attribute__((always_inline)) {
    if (inside) *reinterpret_cast<f32x4*>(p + o) = v;
  };

  f32x4 X[NB], acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) X[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  issue();
  issue();
  int buf = 0;
  // Two blocks at a time; the fragments of the next two are on their way while these are multiplied, and the sums of the two before enter
  // the result.
  bf16x8 f[2][2][3];
  auto read = [&](int b, int set) __attribute__((always_inline)) {
    const char* w = lds + buf * STAGE_B + lane * 16 + b * FRAG3_B;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int p = 0; p < 3; ++p) f[set][u][p] = *reinterpret_cast<const bf16x8*>(w + u * FRAG3_B + p * PART_B);
  };
  for (int step = 0; step < q.n; ++step) {
    const chain_step& s = q.s[step];
    const int N = pinned(s.N), K = pinned(s.K);
    const uint32_t flags = pinned(s.flags);
    const float *p1s = pinned(s.p1), *p2s = pinned(s.p2);
    float *save_pre = pinned(s.save_pre), *out = pinned(s.out), *out2 = pinned(s.out2), *out3 = pinned(s.out3);
    if (flags & CF_LOAD) {
      const int64_t o = row * K + 4 * g;
#pragma unroll
      for (int b = 0; b < NB; ++b) X[b] = 16 * b < K ? ld4(s.load + o + 16 * b) : f32x4{0.f, 0.f, 0.f, 0.f};
      if (flags & CF_LOAD_Z) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (16 * b < K) acc[b] = ld4(s.load_z + o + 16 * b);
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (16 * b < K) {
#pragma unroll
            for (int i = 0; i < 4; ++i) X[b][i] *= dsilu_f(acc[b][i]);
            st(s.load_out, o + 16 * b, X[b]);
          }
      }
    }
    if (step == 0) {
      wait_vmcnt_lgkmcnt0<0>();
      barrier();
      read(0, 0);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (flags & CF_BIAS) {
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[b] = ld4(s.bias + 4 * g + (16 * b < N ? 16 * b : 0));
    }
    const int64_t o = row * N + 4 * g;
    // Before the wavefront that shares the SIMD while there are products: the two then take turns instead of splitting and multiplying at the
    // same time (eight layers of 32768 x 256 276 -> 264 us, 60000 x 128 172 -> 162).
    __builtin_amdgcn_s_setprio(1);
    const int chunks = (K + 31) / 32, halves = (N + 16 * NBS - 1) / (16 * NBS);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      if (c < chunks) {
        // the operand of chunk c, the sign of every second row turned round
        const uint32_t turn = (uint32_t)((c ^ lane) & 1) << 31;
        const float sign = __int_as_float((int)(turn | 0x3F800000u));
        bf16x8 x[3];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float r = __uint_as_float(__float_as_uint(X[2 * c + i / 4][i % 4]) ^ turn);
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            x[p][i] = (__bf16)r;
            r -= (float)x[p][i];
          }
        }
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
          if (h < halves) {
            issue();
            if (h == 0 && c == CH - 1 && (flags & CF_P1)) {   // the operand's registers are free
#pragma unroll
              for (int b = 0; b < NB; ++b) X[b] = ld4(p1s + o + (16 * b < N ? 16 * b : 0));
              __builtin_amdgcn_sched_barrier(0);
            }
            f32x4 t[2][2];
            auto fold = [&](int b) __attribute__((always_inline)) {
#pragma unroll
              for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                  acc[h * NBS + b + u][i] = __builtin_fmaf(t[(b / 2) & 1][u][i], sign, acc[h * NBS + b + u][i]);
            };
#pragma unroll
            for (int b = 0; b < NBS; b += 2) {
              const int set = (b / 2) & 1;
              if (b + 2 < NBS) {
                read(b + 2, set ^ 1);
              } else {
                // All of this stage has been read.  The one after it has to have landed, of which the first stage of a layer is sure
                // (below); behind the barrier the wavefronts may overwrite this one, and the next one's first fragments are asked for.
                buf = buf == 2 ? 0 : buf + 1;
                if (c + h == 0) wait_vmcnt_lgkmcnt0<63>();
                else if (c == CH - 1 && (flags & CF_P1)) wait_vmcnt_lgkmcnt0<PER + NB>();
                else wait_vmcnt_lgkmcnt0<PER>();
                barrier();
                read(0, set ^ 1);
              }
              __builtin_amdgcn_sched_barrier(0);
              constexpr int PW[6] = {2, 0, 1, 1, 0, 0}, PX[6] = {0, 2, 1, 0, 1, 0};   // the smallest first
              t[set][0] = t[set][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int y = 0; y < 6; ++y)
#pragma unroll
                for (int u = 0; u < 2; ++u) t[set][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[set][u][PW[y]], x[PX[y]], t[set][u], 0, 0, 0);
              if (b > 0) fold(b - 2);
              __builtin_amdgcn_sched_barrier(0);
            }
            fold(NBS - 2);
            if constexpr (NBS / 2 % 2 == 1) {   // a stage begins with the first set
#pragma unroll
              for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int p = 0; p < 3; ++p) f[0][u][p] = f[1][u][p];
            }
          }
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    // All that was asked for is waited for here, so that the waits of the next layer do not stand behind this one's stores.
    wait_vmcnt_lgkmcnt0<0>();
    if ((flags & CF_P1) && chunks < CH) {
#pragma unroll
      for (int b = 0; b < NB; ++b) X[b] = ld4(p1s + o + (16 * b < N ? 16 * b : 0));
    }
    // epilogue; no LDS
    auto epilogue = [&](auto steps) __attribute__((always_inline)) {
      constexpr uint32_t F = decltype(steps)::value;
      f32x4 P[2][GRP];
      auto second = [&](int b0, f32x4* p) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < GRP; ++u) p[u] = ld4(p2s + o + (b0 + u < NB && 16 * (b0 + u) < N ? 16 * (b0 + u) : 0));
      };
      if constexpr ((F & CF_P2) != 0) second(0, P[0]);
#pragma unroll
      for (int b0 = 0; b0 < NB; b0 += GRP) {
        if constexpr ((F & CF_P2) != 0) second(b0 + GRP, P[(b0 / GRP + 1) & 1]);
#pragma unroll
        for (int u = 0; u < GRP; ++u) {
          const int b = b0 + u;
          const int64_t ob = o + 16 * b;
          const bool put = inside && 16 * b < N;
          auto st = [&](float* p, f32x4 v) __attribute__((always_inline)) {
            if (put) *reinterpret_cast<f32x4*>(p + ob) = v;
          };
          f32x4 v = acc[b];
          const f32x4 p1 = X[b], p2 = P[(b0 / GRP) & 1][u];
          if constexpr ((F & CF_ADD_PRE) != 0) v += p1;
          if constexpr ((F & CF_SAVE) != 0) st(save_pre, v);
          if constexpr ((F & CF_ACT) != 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = silu_f(v[i]);
          }
          if constexpr ((F & CF_GATE) != 0) {   // p1 = z, p2 = mul
            f32x4 dg;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              dg[i] = v[i] * silu_f(p1[i]);
              v[i] = v[i] * p2[i] * dsilu_f(p1[i]);
            }
            st(out2, v);
            st(out3, dg);
          }
          if constexpr ((F & CF_MUL) != 0) v *= p1;
          if constexpr ((F & CF_ADD) != 0) v += p1;
          if constexpr ((F & CF_ADD2) != 0) v += p2;
          if constexpr ((F & CF_OUT) != 0) st(out, v);
          if constexpr ((F & (CF_Z | CF_Z2)) != 0) {
            const f32x4 z = (F & CF_Z) != 0 ? p1 : p2;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] *= dsilu_f(z[i]);
            st(out2, v);
          }
          acc[b] = v;
        }
      }
    };
    switch (flags & CF_STEPS) {   // uniform
#define GP_CASE(M) case M: epilogue(std::integral_constant<uint32_t, (M)>()); break;
      GP_CHAIN_STEPS(GP_CASE)
#undef GP_CASE
      default: break;   // not launched with any other
    }
    if (!(flags & CF_KEEP)) {   // a narrower result leaves zeros behind it
#pragma unroll
      for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int i = 0; i < 4; ++i) X[b][i] = 16 * b < N ? acc[b][i] : 0.f;
      }
    }
  }
  wait_vmcnt_lgkmcnt0<0>();   // the loads past the end land before the workgroup's LDS goes to another
}

template <int NB>
int chain_stages(const gp_chain_step& s) {
  return (s.K + 31) / 32 * ((s.N + 16 * blocks_per_stage(NB) - 1) / (16 * blocks_per_stage(NB)));
}

template <int NB>
int prepare_chain(gp_ctx* ctx, const gp_chain_step* steps, int n, void* parts, size_t parts_bytes) {
  part_jobs pj;
  int stages = 0;
  double bytes = 0.0;
  for (int i = 0; i < n; ++i) {
    pj.j[i] = part_job{steps[i].W, steps[i].N, steps[i].K, steps[i].k_rows, stages};
    stages += chain_stages<NB>(steps[i]);
    bytes += 10.0 * steps[i].N * steps[i].K;
  }
  pj.n = n;
  if ((size_t)stages * stage_bytes(NB) > parts_bytes) return gp_fail(ctx, GP_BUFFER_TOO_SMALL, "dense chain: scratch too small");
  gp_prof_scope prof(ctx, "make_parts", 0.0, bytes);
  make_parts_kernel<NB><<<(unsigned)stages, 256, 0, ctx->stream>>>(pj, static_cast<char*>(parts));
  GP_LAUNCH_CHECK(ctx, "make_parts_kernel");
  return GP_OK;
}

template <int NB>
int run_chain(gp_ctx* ctx, const gp_chain_step* steps, int from, int to, int64_t rows, const void* parts) {
  chain_args q;
  int before = 0;
  for (int i = 0; i < from; ++i) before += chain_stages<NB>(steps[i]);
  q.stages = 0;
  double mnk = 0.0, bytes = 0.0;
  for (int i = from; i < to; ++i) {
    const gp_chain_step& s = steps[i];
    chain_step& t = q.s[i - from];
    t = chain_step{s.load, s.load_z, s.bias, nullptr, nullptr, s.load_out, s.save_pre, s.out, s.out2, s.out3, s.N, s.K, 0u};
    uint32_t& f = t.flags;
    f = (s.load ? CF_LOAD : 0u) | (s.load_z ? CF_LOAD_Z : 0u) | (s.bias ? CF_BIAS : 0u) | (s.save_pre ? CF_SAVE : 0u) | (s.act ? CF_ACT : 0u) |
        (s.gate ? CF_GATE : 0u) | (s.out ? CF_OUT : 0u) | (s.keep ? CF_KEEP : 0u);
    auto take = [&](const float* p, uint32_t first, uint32_t second) {
      if (!p) return true;
      if (!t.p1 && first) t.p1 = p, f |= CF_P1 | first;
      else if (!t.p2 && second) t.p2 = p, f |= CF_P2 | second;
      else return false;
      return true;
    };
    bool ok = take(s.add_pre, CF_ADD_PRE, 0u) && (!s.load_z || s.load_out);
    if (s.gate) ok = ok && s.z && s.mul && s.out2 && s.out3 && !s.add && !s.out && take(s.z, CF_GATE, 0u) && take(s.mul, 0u, CF_GATE);
    else ok = ok && take(s.mul, CF_MUL, 0u) && take(s.add, CF_ADD, CF_ADD2) && take(s.z, CF_Z, CF_Z2) && (!s.z || s.out2);
    GP_REQUIRE(ctx, ok && !(s.keep && t.p1) && steps_listed(f), "dense chain: operands of a step");
    q.stages += chain_stages<NB>(s);
    mnk += (double)rows * s.N * s.K;
    auto m = [&](const void* p, int w) { bytes += p ? 4.0 * (double)rows * w : 0.0; };
    m(s.load, s.K); m(s.load_z, s.K); m(s.load_out, s.K);
    for (const void* p : {(const void*)s.add_pre, (const void*)s.save_pre, (const void*)s.mul, (const void*)s.add, (const void*)s.out,
                          (const void*)s.z, (const void*)s.out2, (const void*)s.out3}) m(p, s.N);
  }
  q.n = to - from;
  q.W = static_cast<const char*>(parts) + (size_t)before * stage_bytes(NB);
  q.rows = rows;
  constexpr size_t lds = 3 * (size_t)stage_bytes(NB);
  static bool raised = false;
  if (!raised && lds > 64 * 1024) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&dense_chain_kernel<NB>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return gp_fail(ctx, GP_HIP_ERROR, "dense chain: cannot raise the dynamic LDS limit to %zu bytes", lds);
    raised = true;
  }
  static char name[32];
  if (!name[0]) snprintf(name, sizeof(name), "dense_chain_%d", 16 * NB);
  gp_prof_scope prof(ctx, name, 2.0 * mnk, bytes);
  dense_chain_kernel<NB><<<(unsigned)((rows + CHAIN_ROWS - 1) / CHAIN_ROWS), 64 * CHAIN_WAVES, lds, ctx->stream>>>(q);
  GP_LAUNCH_CHECK(ctx, "dense_chain_kernel");
  return GP_OK;
}

}  // namespace

bool gp_chain_takes(int H, int F) {
  return (H == 32 || H == 64 || H == 128 || H == 192 || H == 256) && F % 16 == 0 && F >= 16 && F <= H;
}

size_t gp_chain_parts_bytes(int H, int N, int K) {
  const int nb = H / 16, nbs = blocks_per_stage(nb);
  return (size_t)((K + 31) / 32) * ((N + 16 * nbs - 1) / (16 * nbs)) * stage_bytes(nb);
}

int gp_chain_prepare(gp_ctx* ctx, int H, const gp_chain_step* steps, int n, void* parts, size_t parts_bytes) {
  GP_REQUIRE(ctx, steps && n >= 1 && n <= GP_CHAIN_MAX && parts && ((uintptr_t)parts & 15) == 0, "dense chain: bad arguments");
  for (int i = 0; i < n; ++i) {
    const gp_chain_step& s = steps[i];
    GP_REQUIRE(ctx, s.W && s.N >= 16 && s.N % 16 == 0 && s.N <= H && s.K >= 16 && s.K % 16 == 0 && s.K <= H, "dense chain: bad step");
  }
  switch (H) {
    case 32: return prepare_chain<2>(ctx, steps, n, parts, parts_bytes);
    case 64: return prepare_chain<4>(ctx, steps, n, parts, parts_bytes);
    case 128: return prepare_chain<8>(ctx, steps, n, parts, parts_bytes);
    case 192: return prepare_chain<12>(ctx, steps, n, parts, parts_bytes);
    case 256: return prepare_chain<16>(ctx, steps, n, parts, parts_bytes);
  }
  return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "dense chain: width %d", H);
}

int gp_chain_run(gp_ctx* ctx, int H, const gp_chain_step* steps, int from, int to, int64_t rows, const void* parts) {
  GP_REQUIRE(ctx, steps && from >= 0 && from < to && to <= GP_CHAIN_MAX && rows >= 0 && parts && steps[from].load, "dense chain: bad arguments");
  if (rows == 0) return GP_OK;
  if ((rows + CHAIN_ROWS - 1) / CHAIN_ROWS > INT32_MAX) return gp_fail(ctx, GP_INT32_OVERFLOW, "dense chain: too many rows");
  switch (H) {
    case 32: return run_chain<2>(ctx, steps, from, to, rows, parts);
    case 64: return run_chain<4>(ctx, steps, from, to, rows, parts);
    case 128: return run_chain<8>(ctx, steps, from, to, rows, parts);
    case 192: return run_chain<12>(ctx, steps, from, to, rows, parts);
    case 256: return run_chain<16>(ctx, steps, from, to, rows, parts);
  }
  return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "dense chain: width %d", H);
}
