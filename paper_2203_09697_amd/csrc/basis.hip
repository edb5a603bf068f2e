// Radial / spherical basis functions (named in paper Sec. 3.3; standard definitions).
// Per-edge quantities are evaluated in fp64 and rounded once to fp32 (E values only, the cost is
// negligible); per-triplet quantities (cosines, Legendre factors) are fp32.
#include <math.h>
#include <stdarg.h>

#include "common.h"

namespace {

constexpr int MAX_S = 8;
constexpr int MAX_R_BESSEL = 16;

struct bessel_table {
  double z[MAX_S * MAX_R_BESSEL];      // z[l*R + n]  zeros of j_l
  double inv_z[MAX_S * MAX_R_BESSEL];  // 1 / z
  double norm[MAX_S * MAX_R_BESSEL];   // sqrt(2 / (c^3 j_{l+1}(z)^2))
  double inv_cutoff, root;             // 1 / c, sqrt(2 / c)
};

// j_l(x) on the host, where the zeros are found: ascending series below the turning point, upward recurrence above it.  The series
// stops when its terms no longer reach the sum.
inline double sph_bessel(int l, double x) {
  if (x < (double)l + 1.0 && l >= 2) {
    const double q = -0.5 * x * x;
    double term = 1.0, sum = 1.0;
    for (int k = 1; k <= 40 && fabs(term) > 1e-18 * fabs(sum); ++k) {
      term *= q / ((double)k * (double)(2 * l + 2 * k + 1));
      sum += term;
    }
    double num = 1.0, den = 1.0;   // x^l / (2l+1)!!
    for (int k = 1; k <= l; ++k) {
      num *= x;
      den *= (double)(2 * k + 1);
    }
    return num / den * sum;
  }
  const double s = sin(x), c = cos(x), inv = 1.0 / x;
  double j0 = s * inv;
  if (l == 0) return j0;
  double j1 = (s * inv - c) * inv;
  for (int k = 1; k < l; ++k) {
    const double j2 = (double)(2 * k + 1) * inv * j1 - j0;
    j0 = j1;
    j1 = j2;
  }
  return j1;
}

// sin and cos of the arguments of the Bessel functions: the multiple of pi/2 taken off (pi/2 as the double next to it, whose
// multiple leaves y without rounding, since both end at 2^-52 and what is left is below 1, and the rest of it), then the Taylor sums over [-pi/4, pi/4] to r^17 and r^16 (what follows is below 1e-19 and 2e-18).  About 30
// instructions, a third of the library's sincos, which takes the arguments that are larger, infinite or no number.
__device__ __forceinline__ void sincos_small(double y, double* s, double* c) {
  if (!(fabs(y) < 1e5)) {
    sincos(y, s, c);
    return;
  }
  const double n = rint(y * M_2_PI);
  const int q = (int)n;
  const double r = fma(-n, 6.123233995736766e-17, fma(-n, M_PI_2, y));
  const double r2 = r * r;
  double a = 1.0 / 355687428096000.0, b = 1.0 / 20922789888000.0;
  a = fma(a, r2, -1.0 / 1307674368000.0);
  b = fma(b, r2, -1.0 / 87178291200.0);
  a = fma(a, r2, 1.0 / 6227020800.0);
  b = fma(b, r2, 1.0 / 479001600.0);
  a = fma(a, r2, -1.0 / 39916800.0);
  b = fma(b, r2, -1.0 / 3628800.0);
  a = fma(a, r2, 1.0 / 362880.0);
  b = fma(b, r2, 1.0 / 40320.0);
  a = fma(a, r2, -1.0 / 5040.0);
  b = fma(b, r2, -1.0 / 720.0);
  a = fma(a, r2, 1.0 / 120.0);
  b = fma(b, r2, 1.0 / 24.0);
  a = fma(a, r2, -1.0 / 6.0);
  b = fma(b, r2, -0.5);
  const double sr = fma(a * r2, r, r), cr = fma(b, r2, 1.0);
  const double s0 = q & 1 ? cr : sr, c0 = q & 1 ? sr : cr;
  *s = q & 2 ? -s0 : s0;
  *c = (q + 1) & 2 ? -c0 : c0;
}

// x^l / (2l+1)!! times 1 + q a[l][0] (1 + q a[l][1] (1 + ...)), q = -x^2 / 2: the ascending series of j_l, 14 terms of it for x < 0.6 (l + 2)
constexpr int SERIES_TERMS = 14;
struct series_table {
  double a[MAX_S][SERIES_TERMS], lead[MAX_S];
  constexpr series_table() : a(), lead() {
    double f = 1.0;
    for (int l = 0; l < MAX_S; ++l) {
      f *= (double)(2 * l + 1);
      lead[l] = 1.0 / f;
      for (int k = 1; k <= SERIES_TERMS; ++k) a[l][k - 1] = 1.0 / ((double)k * (double)(2 * l + 2 * k + 1));
    }
  }
};
__constant__ const series_table SERIES = series_table();
__device__ __forceinline__ double series_j(int l, double x) {
  const double q = -0.5 * x * x;
  double t = 1.0;
#pragma unroll
  for (int k = SERIES_TERMS - 1; k >= 0; --k) t = fma(q * SERIES.a[l][k], t, 1.0);
  double p = SERIES.lead[l];
  for (int k = 0; k < l; ++k) p *= x;
  return p * t;
}
// j_l(y) and, where PAIR, j_{l-1}(y) (l >= 1), y > 0 and inv = 1/y: the series below 0.6 (l + 1), and from there on the upward recurrence,
// whose relative error is largest at that line: 5e-16 for l = 1, 7e-15 for l = 4, 6e-14 for l = 7, against 6e-8 of the rounding to fp32.
template <bool PAIR>
__device__ __forceinline__ double sph_bessel_dev(int l, double y, double inv, double* below) {
  if (l >= 1 && y < 0.6 * (double)(l + 1)) {
    if (PAIR) *below = series_j(l - 1, y);
    return series_j(l, y);
  }
  double s, c;
  sincos_small(y, &s, &c);
  double j0 = s * inv;
  if (l == 0) return j0;
  double j1 = (j0 - c) * inv;
  for (int k = 1; k < l; ++k) {
    const double j2 = fma((double)(2 * k + 1) * inv, j1, -j0);
    j0 = j1;
    j1 = j2;
  }
  if (PAIR) *below = j0;
  return j1;
}

__host__ __device__ inline double envelope_d(double x, int p) {
  double xp = 1.0;
  for (int k = 0; k < p; ++k) xp *= x;
  double a = -0.5 * (p + 1) * (p + 2), b = (double)p * (p + 2), c = -0.5 * p * (p + 1);
  return 1.0 + xp * (a + x * (b + x * c));
}

// The first MAX_R_BESSEL zeros z of j_l, l < MAX_S, by bisection between consecutive zeros of j_{l-1}, and j_{l+1}(z): numbers
// that depend on nothing, found once per process (a few thousand evaluations: 0.1 ms that every basis and force call paid).
struct bessel_zeros {
  double z[MAX_S][MAX_R_BESSEL], j_next[MAX_S][MAX_R_BESSEL];
  bessel_zeros() {
    constexpr int N0 = MAX_S + MAX_R_BESSEL;
    double prev[N0], cur[N0];
    for (int n = 0; n < N0; ++n) prev[n] = M_PI * (n + 1);
    for (int l = 0; l < MAX_S; ++l) {
      if (l > 0) {
        for (int n = 0; n < N0 - l; ++n) {
          double a = prev[n], b = prev[n + 1], fa = sph_bessel(l, a);
          for (int it = 0; it < 200 && (b - a) > 1e-15 * b; ++it) {
            double mid = 0.5 * (a + b), fm = sph_bessel(l, mid);
            if ((fm > 0) == (fa > 0)) { a = mid; fa = fm; } else { b = mid; }
          }
          cur[n] = 0.5 * (a + b);
        }
        for (int n = 0; n < N0 - l; ++n) prev[n] = cur[n];
      }
      for (int n = 0; n < MAX_R_BESSEL; ++n) {
        z[l][n] = prev[n];
        j_next[l][n] = sph_bessel(l + 1, prev[n]);
      }
    }
  }
};
void make_bessel_table(int S, int R, double cutoff, bessel_table* t) {
  static const bessel_zeros zeros;   // initialised once, also with several threads
  t->inv_cutoff = 1.0 / cutoff;
  t->root = sqrt(2.0 / cutoff);
  for (int l = 0; l < S; ++l)
    for (int n = 0; n < R; ++n) {
      const double j = zeros.j_next[l][n];
      t->z[l * R + n] = zeros.z[l][n];
      t->inv_z[l * R + n] = 1.0 / zeros.z[l][n];
      t->norm[l * R + n] = sqrt(2.0 / (cutoff * cutoff * cutoff * j * j));
    }
}

// variant D: rbf[E,R] and rad[E,S*R].  A workgroup evaluates all R + S*R functions of EB edges, lanes over edges first: a
// wavefront then follows one or two orders l (their loops differ) and the results leave through LDS as whole rows.  What depends on
// the edge alone, three divisions and the envelope, is found once per edge and read from LDS.  One thread per value: with
// one per (edge, l) a thread's six values came one after the other.  Bound by fp64 instructions.
template <int EB>
__device__ __forceinline__ void basis_edges_D(int block, const float* __restrict__ dist, int64_t n_edges, int S, int R, int p, const bessel_table& tab,
                                              float* __restrict__ rbf, float* __restrict__ rad) {
  extern __shared__ float rows_s[];   // [EB][F + 1]
  __shared__ double edge_s[3][EB];    // x = d / c, 1 / x, the envelope
  const int F = R + S * R, ld = F + 1;
  const int first = rbf ? 0 : R, last = rad ? F : R;   // the functions that are wanted
  const int64_t e0 = (int64_t)block * EB;
  const int ne = n_edges - e0 < EB ? (int)(n_edges - e0) : EB;
  if ((int)threadIdx.x < ne) {
    const double x = (double)dist[e0 + threadIdx.x] * tab.inv_cutoff;
    edge_s[0][threadIdx.x] = x;
    edge_s[1][threadIdx.x] = 1.0 / x;
    edge_s[2][threadIdx.x] = envelope_d(x, p);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < EB * (last - first); i += 256) {
    const int el = i % EB, f = first + i / EB;
    if (el >= ne) continue;
    const double x = edge_s[0][el], inv_x = edge_s[1][el], u = edge_s[2][el];
    double v;
    if (f < R) {
      double s, c;
      sincos_small((double)(f + 1) * M_PI * x, &s, &c);
      v = u * tab.root * (tab.inv_cutoff * inv_x) * s;
    } else {
      const int k = f - R;
      v = u * tab.norm[k] * sph_bessel_dev<false>(k / R, tab.z[k] * x, tab.inv_z[k] * inv_x, nullptr);
    }
    rows_s[el * ld + f] = (float)v;
  }
  __syncthreads();
  if (rbf)
    for (int i = threadIdx.x; i < ne * R; i += 256) rbf[e0 * R + i] = rows_s[(i / R) * ld + i % R];
  if (rad)
    for (int i = threadIdx.x; i < ne * S * R; i += 256) rad[e0 * S * R + i] = rows_s[(i / (S * R)) * ld + R + i % (S * R)];
}
template <int EB>
__global__ void __launch_bounds__(256)
basis_edge_D_kernel(const float* __restrict__ dist, int64_t n_edges, int S, int R, int p, const bessel_table tab, float* __restrict__ rbf,
                    float* __restrict__ rad) {
  basis_edges_D<EB>(blockIdx.x, dist, n_edges, S, R, p, tab, rbf, rad);
}

// variant D, for forces: gd[e] = sum_n grad_rbf[e,n] d rbf_n / dd + sum_{l,n} grad_rad[e,l,n] d rad_ln / dd with
//   rbf_n(d) = u(x) sqrt(2/c) sin(k x) / d,  k = (n+1) pi,  x = d / c
//   rad_ln(d) = u(x) N_ln j_l(z_ln x),  j_l'(y) = j_{l-1}(y) - (l+1)/y j_l(y)  (j_0' = -j_1)
// LANES lanes of a wavefront per edge, over the terms, summed in fp64.  Bound by the latency of a term's fp64 chain where edges
// are few, by the arithmetic of lanes that follow different orders l where they are many; see the rule at the launch.
template <int LANES>
__global__ void __launch_bounds__(256)
grad_dist_bessel_kernel(const float* __restrict__ dist, const float* __restrict__ grad_rbf,
                        const float* __restrict__ grad_rad, int64_t n_edges, int S, int R, int p,
                        const bessel_table tab, float* __restrict__ gd) {
  const int64_t e = (int64_t)blockIdx.x * (256 / LANES) + threadIdx.x / LANES;
  if (e >= n_edges) return;
  const int lane = threadIdx.x % LANES;
  const double inv_c = tab.inv_cutoff, x = (double)dist[e] * inv_c, inv_x = 1.0 / x, inv_d = inv_c * inv_x;
  double xp1 = 1.0;                       // x^(p-1)
  for (int k = 0; k < p - 1; ++k) xp1 *= x;
  const double a = -0.5 * (p + 1) * (p + 2), b = (double)p * (p + 2), c = -0.5 * p * (p + 1);
  const double u = 1.0 + xp1 * x * (a + x * (b + x * c));
  const double du = xp1 * (p * a + x * ((p + 1) * b + x * (p + 2) * c)) * inv_c;   // du/dd
  double s = 0.0;
  for (int f = lane; f < R + S * R; f += LANES) {
    if (f < R) {
      if (grad_rbf) {
        const double k = (double)(f + 1) * M_PI;
        double sn, cs;
        sincos_small(k * x, &sn, &cs);
        s += (double)grad_rbf[e * R + f] * tab.root * inv_d * (du * sn + u * (k * inv_c * cs - sn * inv_d));
      }
    } else if (grad_rad) {
      const int k = f - R, l = k / R;
      const double z = tab.z[k], y = z * x, inv_y = tab.inv_z[k] * inv_x;
      double below;
      const double j = sph_bessel_dev<true>(l == 0 ? 1 : l, y, inv_y, &below);
      const double jl = l == 0 ? below : j, djl = l == 0 ? -j : fma(-(double)(l + 1) * inv_y, j, below);
      s += (double)grad_rad[e * S * R + k] * tab.norm[k] * (du * jl + u * z * inv_c * djl);
    }
  }
  for (int o = LANES / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, WAVE);
  if (lane == 0) gd[e] = (float)s;
}

// variant G: g[E,R] Gaussian radial basis.  A thread owns 8 consecutive functions of an edge: with a = (x - mu_0)(R - 1) at the
// first of them, exp(-(a - 1)^2 / 2) = exp(-a^2 / 2) exp(a - 1/2) and the ratio falls by exp(-1) with every function, so two
// fp64 exponentials serve eight values (the error stays at a few fp64 roundings; where the first value underflows, and the
// ratio is cut off, all eight are far below the smallest fp32 number).  134 us with one exponential per value at 300 636 edges x 128.
constexpr int GAUSS_RUN = 8;
__global__ void __launch_bounds__(256)
basis_edge_G_kernel(const float* __restrict__ dist, int64_t n_edges, int R, int p, double cutoff, int aligned,
                    float* __restrict__ g) {
  const int runs = (R + GAUSS_RUN - 1) / GAUSS_RUN;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t e = idx / runs;
  if (e >= n_edges) return;
  const int n0 = (int)(idx % runs) * GAUSS_RUN;
  const double x = (double)dist[e] / cutoff;
  const double a = x * (double)(R - 1) - (double)n0;
  double v = envelope_d(x, p) * exp(-0.5 * a * a), ratio = exp(fmin(a, 60.0) - 0.5);
  float out[GAUSS_RUN];
#pragma unroll
  for (int k = 0; k < GAUSS_RUN; ++k) {
    out[k] = (float)v;
    v *= ratio;
    ratio *= 0.36787944117144233;   // exp(-1)
  }
  float* o = g + e * R + n0;
  if (aligned) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    *reinterpret_cast<f4*>(o) = f4{out[0], out[1], out[2], out[3]};
    *reinterpret_cast<f4*>(o + 4) = f4{out[4], out[5], out[6], out[7]};
  } else {
#pragma unroll
    for (int k = 0; k < GAUSS_RUN; ++k)
      if (n0 + k < R) o[k] = out[k];
  }
}

__device__ __forceinline__ float cos_of(float ax, float ay, float az, float bx, float by, float bz) {
  return fminf(1.0f, fmaxf(-1.0f, -fmaf(az, bz, fmaf(ax, bx, ay * by))));
}

__global__ void cos_alpha_kernel(const float* __restrict__ unit, const int32_t* __restrict__ idx_kj,
                                 const int32_t* __restrict__ idx_ji, int64_t n_triplets,
                                 float* __restrict__ cos_alpha) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_triplets) return;
  const float* a = unit + 3 * (int64_t)idx_ji[t];
  const float* b = unit + 3 * (int64_t)idx_kj[t];
  cos_alpha[t] = cos_of(a[0], a[1], a[2], b[0], b[1], b[2]);
}

// Both orders of the cosines of a graph with its lists by centre atom: they are the entries of the d_in x d_out matrix
// -unit[in-edge] . unit[out-edge] of every atom, left out where the two edges are opposite.  Teams (see run_team) of in-edge rows
// write the kj-major order from the out-edges' unit vectors in LDS, teams of consecutive positions of the out-edge lists the
// ji-major order from the in-edges'.  Bound by the 8 bytes written per triplet: 1e8 triplets in 0.22 ms (0.26 with the values of
// a run's edge fetched by LDS permutes instead of of_lane's scalar reads; from the index arrays, 12 bytes read per triplet, and
// the second order as a gathered copy of the first: 0.36 + 0.61 ms; every wavefront fetching its own list: 0.33 - 0.38 ms).
// A run that seg_ptr gives another length than the lists do (triplets were taken out of a finished graph) follows its index array
// other[n_triplets], the edge on the far side of every slot; no run is written past n_triplets.
template <bool LONG, bool KJ>
__device__ __forceinline__ void cos_runs(int block, const float* __restrict__ unit, const int32_t* __restrict__ centre,
                                         const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ out_ptr,
                                         const int32_t* __restrict__ out_list, const int32_t* __restrict__ id_swap,
                                         const int32_t* __restrict__ seg_ptr, const int32_t* __restrict__ other, int n_edges,
                                         int n_triplets, float* __restrict__ out) {
  using R = run_team<LONG>;
  __shared__ __align__(16) float t_x[R::TEAMS][R::CHUNK + 4], t_y[R::TEAMS][R::CHUNK + 4], t_z[R::TEAMS][R::CHUNK + 4];
  __shared__ int32_t t_gap[R::TEAMS][R::ROWS];
  const int lane = lane_id(), team = threadIdx.x / R::TEAM, tid = threadIdx.x % R::TEAM;
  const int par = tid / R::LANES, ln = tid % R::LANES;
  const int p0 = (block * R::TEAMS + team) * R::ROWS;
  if (p0 >= n_edges) return;   // the whole team
  const int n_own = n_edges - p0 < R::ROWS ? n_edges - p0 : R::ROWS;
  // lane u holds edge u of the team
  const int pl = p0 + (lane < n_own ? lane : 0), el = KJ ? pl : out_list[pl], jl = centre[el], oppl = id_swap[el], segl = seg_ptr[el];
  const int endl = seg_ptr[el + 1];
  const float uxl = unit[3 * (int64_t)el], uyl = unit[3 * (int64_t)el + 1], uzl = unit[3 * (int64_t)el + 2];
  for (int done = 0; done < n_own;) {
    const int atom = __builtin_amdgcn_readlane(jl, done);
    const int len = __popcll(__ballot(lane < n_own && lane >= done && jl == atom));
    const int sb = KJ ? out_ptr[atom] : row_ptr[atom], n = (KJ ? out_ptr[atom + 1] : row_ptr[atom + 1]) - sb;   // the list in LDS
    const int base = p0 + done;   // first edge of the run of equal atoms
    for (int b0 = 0; b0 < n; b0 += R::CHUNK) {
      team_sync<LONG>();   // the previous chunk has been consumed
      if (KJ && b0 == 0)
        for (int u = tid; u < R::ROWS; u += R::TEAM) t_gap[team][u] = INT32_MAX;
      if (KJ) team_sync<LONG>();
      for (int q = tid; q < R::CHUNK + 4 && b0 + q < n; q += R::TEAM) {
        const int64_t e = KJ ? out_list[sb + b0 + q] : sb + b0 + q;
        t_x[team][q] = unit[3 * e];
        t_y[team][q] = unit[3 * e + 1];
        t_z[team][q] = unit[3 * e + 2];
        if (KJ) {
          const int back = id_swap[e];
          if (back >= base && back < base + len) t_gap[team][back - base] = b0 + q;
        }
      }
      team_sync<LONG>();
      for (int u = par; u < len; u += R::PAR) {
        const int opp = of_lane<LONG>(oppl, done + u), seg = of_lane<LONG>(segl, done + u), stop = of_lane<LONG>(endl, done + u);
        const float ux = of_lane<LONG>(uxl, done + u), uy = of_lane<LONG>(uyl, done + u), uz = of_lane<LONG>(uzl, done + u);
        const int gap = KJ ? t_gap[team][u] : opp >= 0 ? opp - sb : INT32_MAX;
        const int cnt = (stop < n_triplets ? stop : n_triplets) - seg, end = cnt < b0 + R::CHUNK ? cnt : b0 + R::CHUNK;
        if (cnt != n - (opp >= 0 ? 1 : 0)) {
          for (int t = seg + ln; b0 == 0 && other && t < seg + cnt; t += R::LANES) {
            const float* v = unit + 3 * (int64_t)other[t];
            out[t] = cos_of(ux, uy, uz, v[0], v[1], v[2]);
          }
          continue;
        }
        for (int s0 = b0 + 4 * ln; s0 < end; s0 += 4 * R::LANES) {
          const int q = s0 - b0;
          const float4 x4 = *reinterpret_cast<const float4*>(&t_x[team][q]), y4 = *reinterpret_cast<const float4*>(&t_y[team][q]),
                       z4 = *reinterpret_cast<const float4*>(&t_z[team][q]);
          const float x[5] = {x4.x, x4.y, x4.z, x4.w, t_x[team][q + 4]}, y[5] = {y4.x, y4.y, y4.z, y4.w, t_y[team][q + 4]},
                      z[5] = {z4.x, z4.y, z4.z, z4.w, t_z[team][q + 4]};
          float c[5];
#pragma unroll
          for (int i = 0; i < 5; ++i) c[i] = KJ ? cos_of(x[i], y[i], z[i], ux, uy, uz) : cos_of(ux, uy, uz, x[i], y[i], z[i]);
          store_run4<float4u>(out + seg, s0, cnt, gap, c);
        }
      }
    }
    done += len;
  }
}
struct cos_args {
  const float* unit;
  const int32_t *src, *dst, *row_ptr, *out_ptr, *out_list, *id_swap, *seg_ji, *seg_kj, *idx_kj, *idx_ji_kj;
  int n_edges, n_triplets, n_blocks;
  float *cos_ji, *cos_kj;
};
template <bool LONG>
__device__ __forceinline__ void cos_graph(int b, const cos_args& q) {
  if (b < q.n_blocks)
    cos_runs<LONG, true>(b, q.unit, q.dst, q.row_ptr, q.out_ptr, q.out_list, q.id_swap, q.seg_kj, q.idx_ji_kj, q.n_edges, q.n_triplets, q.cos_kj);
  else
    cos_runs<LONG, false>(b - q.n_blocks, q.unit, q.src, q.row_ptr, q.out_ptr, q.out_list, q.id_swap, q.seg_ji, q.idx_kj, q.n_edges, q.n_triplets, q.cos_ji);
}
template <bool LONG>
__global__ void __launch_bounds__(256) cos_graph_kernel(const cos_args q) { cos_graph<LONG>(blockIdx.x, q); }
// Both parts of the basis of a small graph in one launch, the first `edge_blocks` workgroups on the edges: one is fp64 arithmetic, the other
// memory latency, and neither fills the chip (43380 edges, 590 k triplets: 16.4 + 10.2 us one after the other, 20.1 together).
template <bool LONG, int EB>
__global__ void __launch_bounds__(256)
basis_graph_D_kernel(const cos_args q, int edge_blocks, const float* __restrict__ dist, int S, int R, int p, const bessel_table tab,
                     float* __restrict__ rbf, float* __restrict__ rad) {
  if ((int)blockIdx.x < edge_blocks) basis_edges_D<EB>(blockIdx.x, dist, q.n_edges, S, R, p, tab, rbf, rad);
  else cos_graph<LONG>((int)blockIdx.x - edge_blocks, q);
}

// out[q] = in[perm[q]].  For the kj-major copy of cos alpha the gathered values of neighbouring q lie a whole in-degree apart
// (each its own 64-byte sector), but all rows of a centre atom gather from the same d_in x d_out block; workgroup ids are
// dealt round-robin to the 8 XCDs, so they are renumbered to give each XCD a contiguous range of q: the block of an atom
// is then fetched into one L2 and hit there by the atom's other rows (3.5 GB fetched for 0.4 GB used otherwise).
__global__ void permute_kernel(const float* __restrict__ in, const int32_t* __restrict__ perm, int64_t n,
                               float* __restrict__ out) {
  const int64_t nb = gridDim.x, per = nb >> 3, rem = nb & 7;
  const int64_t x = blockIdx.x & 7, i = blockIdx.x >> 3;
  const int64_t blk = x * per + (x < rem ? x : rem) + i;
  const int64_t q = blk * blockDim.x + threadIdx.x;
  if (q < n) out[q] = in[perm[q]];
}

// materialised spherical basis, one thread per (triplet, l)
__global__ void sbf_kernel(const float* __restrict__ rad, const float* __restrict__ cos_alpha,
                           const int32_t* __restrict__ idx_kj, int64_t n_triplets, int S, int R,
                           float* __restrict__ sbf) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_triplets * S) return;
  int64_t t = idx / S;
  int l = (int)(idx % S);
  float c = cos_alpha[t];
  float p0 = 1.0f, p1 = c;
  for (int k = 1; k < l; ++k) {
    float p2 = ((2 * k + 1) * c * p1 - k * p0) / (float)(k + 1);
    p0 = p1;
    p1 = p2;
  }
  float P = (l == 0) ? 1.0f : p1;
  float Y = sqrtf((float)(2 * l + 1) / (4.0f * (float)M_PI)) * P;
  const float* r = rad + ((int64_t)idx_kj[t] * S + l) * R;
  float* o = sbf + (t * S + l) * R;
  for (int n = 0; n < R; ++n) o[n] = r[n] * Y;
}

inline int nblk(int64_t n) { return (int)((n + 255) / 256); }

}  // namespace

// The per-edge part of the two entry points, and with cos the cosines of the graph; *cos_done: whether the same launch did those.
static int basis_edges(gp_ctx* ctx, const char* who, const gp_dims* dims, const float* dist, int64_t n_edges, float* rbf, float* rad,
                       const cos_args* cos = nullptr, bool* cos_done = nullptr) {
  GP_REQUIRE(ctx, dims->cutoff > 0.f, "%s: cutoff must be positive", who);
  const int S = dims->num_spherical, R = dims->num_radial, p = dims->envelope_p;
  if (S < 1 || S > MAX_S || R < 1 || p < 1 || p > 16)
    return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "%s: num_spherical=%d num_radial=%d p=%d unsupported", who, S, R, p);
  GP_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t st = ctx->stream;
  if (n_edges > 0 && (rbf || rad)) {
    GP_REQUIRE(ctx, dist, "%s: dist is NULL", who);
    if (dims->variant == GP_VARIANT_D) {
      if (R > MAX_R_BESSEL) return gp_fail(ctx, GP_UNSUPPORTED_DIMS, "%s: num_radial=%d > %d", who, R, MAX_R_BESSEL);
      bessel_table tab;
      make_bessel_table(S, R, (double)dims->cutoff, &tab);
      // 32 edges per workgroup share the factors of an edge and fill the chip from about 12 000 edges on; below that the time is one
      // value's latency, and 4 edges per workgroup leave one value to a thread.  4 / 32 edges, 48 values each: 4.8 / 8.3 us at 4000
      // edges, 7.5 / 8.6 at 8000, 9.7 / 9.7 at 12 000, 11.9 / 9.8 at 16 000, 20 / 14 at 32 000, 164 / 85 at 300 000
      const bool many = n_edges >= 12288;
      const size_t row = sizeof(float) * (R + S * R + 1);
      // In one launch with the cosines while those do not fill the chip for long by themselves (above).  Apart / together: slabs, 0.2e6
      // triplets 21.4 / 18.0 us, 1.6e6 26.5 / 20.3, 6.3e6 69 / 65, 12.5e6 122 / 120, 15.6e6 147 / 147, 24.9e6 259 / 267; boxes with long
      // lists, 0.3e6 20.1 / 16.8, 2.2e6 25.0 / 18.5, 6.7e6 38 / 31, 14.3e6 59 / 53, 23.8e6 83 / 80
      if (cos && cos->n_triplets < 16 * 1000 * 1000) {
        *cos_done = true;
        const bool wide = cos->n_triplets >= LONG_LISTS * n_edges;
        const int eb = many ? 32 : 4, blocks = (int)((n_edges + eb - 1) / eb);
        auto* kernel = wide ? (eb == 32 ? basis_graph_D_kernel<true, 32> : basis_graph_D_kernel<true, 4>)
                            : (eb == 32 ? basis_graph_D_kernel<false, 32> : basis_graph_D_kernel<false, 4>);
        kernel<<<(unsigned)(blocks + 2 * cos->n_blocks), 256, eb * row, st>>>(*cos, blocks, dist, S, R, p, tab, rbf, rad);
        GP_LAUNCH_CHECK(ctx, "basis_graph_D_kernel");
        return GP_OK;
      }
      if (many)
        basis_edge_D_kernel<32><<<(unsigned)((n_edges + 31) / 32), 256, 32 * row, st>>>(dist, n_edges, S, R, p, tab, rbf, rad);
      else
        basis_edge_D_kernel<4><<<(unsigned)((n_edges + 3) / 4), 256, 4 * row, st>>>(dist, n_edges, S, R, p, tab, rbf, rad);
      GP_LAUNCH_CHECK(ctx, "basis_edge_D_kernel");
    } else if (dims->variant == GP_VARIANT_G) {
      GP_REQUIRE(ctx, R >= 2, "%s: Gaussian basis needs num_radial >= 2", who);
      if (rbf) {
        const int runs = (R + GAUSS_RUN - 1) / GAUSS_RUN;
        const int aligned = R % GAUSS_RUN == 0 && (reinterpret_cast<uintptr_t>(rbf) & 15) == 0;
        basis_edge_G_kernel<<<nblk(n_edges * runs), 256, 0, st>>>(dist, n_edges, R, p, (double)dims->cutoff, aligned, rbf);
        GP_LAUNCH_CHECK(ctx, "basis_edge_G_kernel");
      }
    } else {
      return gp_fail(ctx, GP_BAD_ARG, "%s: unknown variant %d", who, dims->variant);
    }
  }
  return GP_OK;
}

extern "C" int gp_basis_forward(gp_ctx* ctx, const gp_dims* dims, const float* dist, const float* unit,
                                const int32_t* idx_kj, const int32_t* idx_ji, const int32_t* perm_kj,
                                int64_t n_edges, int64_t n_triplets, float* rbf, float* rad,
                                float* cos_alpha, float* cos_alpha_kj, float* sbf) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, dims, "gp_basis_forward: dims is NULL");
  GP_REQUIRE(ctx, n_edges >= 0 && n_triplets >= 0, "gp_basis_forward: negative size");
  GP_TRY(basis_edges(ctx, "gp_basis_forward", dims, dist, n_edges, rbf, rad));
  const int S = dims->num_spherical, R = dims->num_radial;
  hipStream_t st = ctx->stream;
  if (n_triplets > 0 && cos_alpha) {
    GP_REQUIRE(ctx, unit && idx_kj && idx_ji, "gp_basis_forward: unit/idx_kj/idx_ji is NULL");
    cos_alpha_kernel<<<nblk(n_triplets), 256, 0, st>>>(unit, idx_kj, idx_ji, n_triplets, cos_alpha);
    GP_LAUNCH_CHECK(ctx, "cos_alpha_kernel");
    if (cos_alpha_kj) {
      GP_REQUIRE(ctx, perm_kj, "gp_basis_forward: cos_alpha_kj needs perm_kj");
      permute_kernel<<<nblk(n_triplets), 256, 0, st>>>(cos_alpha, perm_kj, n_triplets, cos_alpha_kj);
      GP_LAUNCH_CHECK(ctx, "permute_kernel");
    }
    if (sbf) {
      GP_REQUIRE(ctx, rad && dims->variant == GP_VARIANT_D, "gp_basis_forward: sbf needs rad (variant D)");
      sbf_kernel<<<nblk(n_triplets * S), 256, 0, st>>>(rad, cos_alpha, idx_kj, n_triplets, S, R, sbf);
      GP_LAUNCH_CHECK(ctx, "sbf_kernel");
    }
  } else if (n_triplets > 0) {
    GP_REQUIRE(ctx, !cos_alpha_kj && !sbf, "gp_basis_forward: cos_alpha_kj/sbf need cos_alpha");
  }
  return GP_OK;
}

extern "C" int gp_basis_forward_graph(gp_ctx* ctx, const gp_dims* dims, const float* dist, const float* unit, const int32_t* src,
                                      const int32_t* dst, const gp_graph* graph, float* rbf, float* rad, float* cos_alpha,
                                      float* cos_alpha_kj) {
  if (!ctx) return GP_BAD_ARG;
  GP_REQUIRE(ctx, dims && graph, "gp_basis_forward_graph: NULL pointer");
  const int64_t E = graph->n_edges, T = graph->n_triplets;
  GP_REQUIRE(ctx, E >= 0 && T >= 0, "gp_basis_forward_graph: negative size");
  if (E > INT32_MAX - 1 || T > INT32_MAX) return gp_fail(ctx, GP_INT32_OVERFLOW, "gp_basis_forward_graph: sizes exceed int32");
  if (E == 0 || T == 0) return basis_edges(ctx, "gp_basis_forward_graph", dims, dist, E, rbf, rad);
  GP_REQUIRE(ctx, unit && src && dst && cos_alpha && cos_alpha_kj && graph->row_ptr && graph->out_ptr && graph->out_list &&
             graph->id_swap && graph->seg_ptr_ji && graph->seg_ptr_kj, "gp_basis_forward_graph: NULL pointer");
  const int blocks = (int)((E + 63) / 64);   // 64 edges per workgroup in both forms
  const cos_args q{unit, src, dst, graph->row_ptr, graph->out_ptr, graph->out_list, graph->id_swap, graph->seg_ptr_ji, graph->seg_ptr_kj,
                   graph->idx_kj, graph->idx_ji_kj, (int)E, (int)T, blocks, cos_alpha, cos_alpha_kj};
  bool done = false;
  GP_TRY(basis_edges(ctx, "gp_basis_forward_graph", dims, dist, E, rbf, rad, &q, &done));
  if (done) return GP_OK;
  (T >= LONG_LISTS * E ? cos_graph_kernel<true> : cos_graph_kernel<false>)<<<2 * (unsigned)blocks, 256, 0, ctx->stream>>>(q);
  GP_LAUNCH_CHECK(ctx, "cos_graph_kernel");
  return GP_OK;
}

// dL/dd per edge from the gradients with respect to the Bessel radial basis and the radial part of the spherical
// basis (either may be NULL)
int gp_grad_dist_bessel(gp_ctx* ctx, const gp_dims* dims, const float* dist, const float* grad_rbf, const float* grad_rad,
                        int64_t n_edges, float* gd) {
  if (n_edges == 0) return GP_OK;
  const int S = dims->num_spherical, R = dims->num_radial;
  GP_REQUIRE(ctx, S >= 1 && S <= MAX_S && R >= 1 && R <= MAX_R_BESSEL, "grad_dist_bessel: basis sizes out of range");
  bessel_table tab;
  make_bessel_table(S, R, (double)dims->cutoff, &tab);
  // Few terms: one thread per edge is not slower anywhere (9 terms: 7 us up to 16 000 edges; 36 us at 900 000, 77 with 4 lanes).
  // From 16 terms on the lanes that keep the chip busy, 48 terms with 64 / 16 / 4 lanes per edge: 5.3 / 7.1 / 17 us at 336 edges,
  // 7.4 / 7.0 / 16 at 4000, 18 / 13 / 16 at 16 000, 32 / 21 / 21 at 32 000, 61 / 36 / 36 at 64 000, 333 / 178 / 152 at 300 000.
  auto launch = [&](auto kernel, int lanes) {
    const int per = 256 / lanes;
    kernel<<<(unsigned)((n_edges + per - 1) / per), 256, 0, ctx->stream>>>(dist, grad_rbf, grad_rad, n_edges, S, R, dims->envelope_p, tab,
                                                                           gd);
  };
  if (R + S * R < 16) launch(grad_dist_bessel_kernel<1>, 1);
  else if (n_edges < 4096) launch(grad_dist_bessel_kernel<64>, 64);
  else if (n_edges < 32768) launch(grad_dist_bessel_kernel<16>, 16);
  else launch(grad_dist_bessel_kernel<4>, 4);
  GP_LAUNCH_CHECK(ctx, "grad_dist_bessel_kernel");
  return GP_OK;
}
