// The Kubo-Greenwood route (Sec. A.3, with Eqs. 8, A-1, A-2): from a
// conductivity sigma(w) in the optical limit to the scaled structure factor
// S* = v(q) S, on which the eta test, the attenuation and the way back to
// eps^{-1} and sigma (the dielectric step with q^2 = 4 pi) run unchanged;
// and the Kubo-Greenwood conductivity of the states that the route starts
// from.  FP64.
//
// The conductivity in two steps: per transition t = (k, n -> m) of the
// q = 0 list, W_t = (df / delta) (1/3) sum_a |<m|p_a|n>|^2 (by bands on the
// FP64 MFMA); then sigma(w) = 2 i / (Omega N_k)
// sum_t W_t / (w - delta_t + i eta) as fixed-size chunks of transitions per
// workgroup (one frequency per lane) and a fixed-order tree
// over the chunk partials, so the result does not depend on scheduling.
#include <algorithm>
#include <cmath>

#include "chi0_tile.h"
#include "internal.h"
#include "tables.h"

namespace tdx {
namespace {

// Im chi* = Im 1/eps with eps = 1 + 4 pi i sigma / w (w != 0):
// eps = (1 - 4 pi Im sigma / w) + i (4 pi Re sigma / w), Im 1/eps = -Im eps / |eps|^2.
__device__ inline double im_chi_star(double2 s, double w) {
  const double er = 1.0 - 4.0 * M_PI * s.y / w, ei = 4.0 * M_PI * s.x / w;
  return -ei / (er * er + ei * ei);
}

// S* = -Im chi* / (pi n (1 - e^{-beta w})), the normalisation of S; w = 0
// takes the limit from the next grid point, -Im chi*(w1) / (pi n beta w1).
__global__ void k_kg_dsf(const double2 *sig, const double *w, int n, double beta, double dens,
                         double *S) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double wi = w[i];
  double v;
  if (wi != 0.0) {
    v = -im_chi_star(sig[i], wi) / (M_PI * dens * (-expm1(-beta * wi)));
  } else if (i + 1 < n && w[i + 1] > 0.0) {
    v = -im_chi_star(sig[i + 1], w[i + 1]) / (M_PI * dens * beta * w[i + 1]);
  } else {
    v = NAN;  // w = 0 without a positive neighbour
  }
  S[i] = v;
}

constexpr int kKgChunk = 2048;  // transitions per partial

// ------------------------------------------------------------- weights
// W_t by k-point and band: the transitions of five bands n against 16 bands m
// are one complex product on the FP64 MFMA,
//   p[m][(n, a)] = sum_G conj(c_mk(G)) (k + G)_a c_nk(G),
// 15 of 16 columns, for the tiles of m that the rows (k, n) of the list hold.
// |p_mn|^2 is symmetric, so a workgroup takes the m from its own first band
// on and also writes the weights of the opposite transitions (m -> n); bands
// that pair with lower ones only have nothing left to do.  The five orbitals
// and k + G sit in LDS; a wave reads the 16 orbitals m from global memory, 64
// contiguous bytes per lane.  The workgroups of a k run on one XCD, whose L2
// then holds its orbitals.  One wavefront per transition, which reads both
// its orbitals each time, is bound by L2 (10 TB/s).  Measured for 1.32 million
// transitions of 125 k with up to 483 plane waves and 264 bands: 1165 us that
// way; here 436 us with a workgroup for every group of bands, most of which
// found after some dependent loads that a lower one does their work, 256 us
// with a list of those that have some.  The products alone are about 110 us at
// the FP64 rate; the rest is the latency of the 16 rows and of the list.

// First transitions of the rows (k, n) of the list, and n after the last row;
// flag[0] is set if the list is not ordered by k, then n, then m (the rows are
// then not used).  A wave that sees the order broken says so once and stops:
// every lane saying it, on one address, took 930 us for a list of 1.32 million
// in reverse, and the gaps between the rows of a shuffled one, filled for each
// of its transitions, 33 ms (7 us either way now, as for an ordered one).
__global__ void k_kg_rows(const int *tk, const int *tn, const int *tm, int n, int nb_max,
                          long n_rows, int *rows, int *flag) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
    const long r = (long)tk[t] * nb_max + tn[t];
    const long before = t > 0 ? (long)tk[t - 1] * nb_max + tn[t - 1] : -1;
    if (__any(before > r || (before == r && tm[t - 1] >= tm[t]))) {
      if ((threadIdx.x & 63) == 0 && !__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    for (long i = before + 1; i <= r; ++i) rows[i] = t;
    if (t == n - 1)
      for (long i = r + 1; i <= n_rows; ++i) rows[i] = n;
  }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kKgBands = 5;  // bands n per workgroup: 15 columns
constexpr int kKgWaves = 8;

// The transition (m -> n) of the k whose rows these are, -1 if the list does
// not hold it: one look where a row has no gaps (most have none).
__device__ inline int kg_opposite(const int *rows_k, const int *tm, int m, int n) {
  int lo = rows_k[m], hi = rows_k[m + 1];
  if (lo == hi) return -1;
  const int end = hi, guess = lo + n - tm[lo];
  if (guess >= lo && guess < hi && tm[guess] == n) return guess;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (tm[mid] < n)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo < end && tm[lo] == n ? lo : -1;
}

// The groups of five bands that form weights, as k * chunks + chunk in about
// that order (their number in *n_groups): those with a transition to a band
// from their own first on, or one whose opposite the list does not hold.
// One wavefront per group.
__global__ void __launch_bounds__(256)
    k_kg_groups(const int *rows, const int *flag, const int *tn, const int *tm, int nb_max,
                int chunks, int n, int *groups, int *n_groups) {
  if (*flag) return;
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c >= n) return;
  const int n0 = c % chunks * kKgBands, n1 = std::min(n0 + kKgBands, nb_max);
  const int *rows_k = rows + (size_t)(c / chunks) * nb_max;
  const int t1 = rows_k[n1];
  bool work = false;
  for (int t = rows_k[n0] + lane; !work && t < t1; t += 64) {
    const int m = tm[t];
    work = m >= n0 || kg_opposite(rows_k, tm, m, tn[t]) < 0;
  }
  work = __any(work);
  if (work && lane == 0) groups[atomicAdd(n_groups, 1)] = c;
}

inline size_t kg_lds_bytes(int npw_max, int nb_max) {
  const size_t st = npw_max;
  return sizeof(double2) * kKgBands * st + sizeof(double) * 3 * st +
         sizeof(double) * kKgBands * (size_t)nb_max + sizeof(int) * ((size_t)nb_max / 16 + 2);
}

// Two workgroups per CU take the groups in turn, those of one XCD a run of the
// list; where there are fewer groups than workgroups, the tiles of m are dealt
// to several (down to two each).
__global__ void __launch_bounds__(64 * kKgWaves)
    k_kg_bands(const int *rows, const int *flag, const int *groups, const int *n_groups,
               const int *tn, const int *tm, const double *delta, const double *df,
               const double2 *coef, const int *miller, const int *npw, int npw_max, int nb_max, int N0, int N1, int N2,
               double3 b0, double3 b1, double3 b2, double *W) {
  if (*flag) return;
  extern __shared__ double2 kg_lds[];
  double2 *cn = kg_lds;                                         // [5][npw_max]
  double *gv = (double *)(cn + kKgBands * (size_t)npw_max);  // [3][npw_max]
  double *p2 = gv + 3 * (size_t)npw_max;                    // [5][nb_max] |p|^2
  int *need = (int *)(p2 + kKgBands * (size_t)nb_max);       // tiles of 16 bands m
  const int chunks = (nb_max + kKgBands - 1) / kKgBands;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_tiles = (nb_max + 15) / 16, ng = *n_groups, wgs = gridDim.x;
  const int parts = std::max(1, std::min(wgs / std::max(ng, 1), (n_tiles + 1) / 2));
  // workgroup b runs on XCD b % 8: its eighth of the items
  const int xcds = wgs % 8 ? 1 : 8;
  const long items = (long)ng * parts;
  const int x = blockIdx.x % xcds;
  const long end = items * (x + 1) / xcds;
  for (long it = items * x / xcds + blockIdx.x / xcds; it < end; it += wgs / xcds) {
    const int c = groups[it / parts], part = (int)(it % parts);
    const int k = c / chunks, n0 = c % chunks * kKgBands;
    const int np = npw[k];
    const int count = std::min(kKgBands, nb_max - n0);
    const int *rows_k = rows + (size_t)k * nb_max;
    const int t0 = rows_k[n0], t1 = rows_k[n0 + count];
    // whether this workgroup forms (n -> m): of the workgroups of the lower band
    // the one that has m's tile, or of the other band where the list holds one
    // direction only
    auto mine = [&](int n, int m) {
      return (m >> 4) % parts == part && (m >= n0 || kg_opposite(rows_k, tm, m, n) < 0);
    };
    for (int i = tid; i < n_tiles; i += 64 * kKgWaves) need[i] = 0;
    __syncthreads();
    bool work = false;
    for (int t = t0 + tid; t < t1; t += 64 * kKgWaves) {
      const int m = tm[t];
      if (mine(tn[t], m)) {
        need[m >> 4] = 1;
        work = true;
      }
    }
    if (!__syncthreads_or(work)) continue;
    const double2 *ck = coef + (size_t)k * nb_max * npw_max;
    for (int i = 0; i < kKgBands; ++i)
      for (int g = tid; g < np; g += 64 * kKgWaves)
        cn[(size_t)i * npw_max + g] =
            i < count ? ck[(size_t)(n0 + i) * npw_max + g] : make_double2(0.0, 0.0);
    const int r0 = k / (N1 * N2), r1 = (k / N2) % N1, r2 = k % N2;
    const double kr0 = (2.0 * r0 + 1.0 - N0) / (2.0 * N0), kr1 = (2.0 * r1 + 1.0 - N1) / (2.0 * N1),
                 kr2 = (2.0 * r2 + 1.0 - N2) / (2.0 * N2);
    const int *mk = miller + (size_t)k * npw_max * 3;
    for (int g = tid; g < np; g += 64 * kKgWaves) {
      const double m0 = kr0 + mk[3 * g], m1 = kr1 + mk[3 * g + 1], m2 = kr2 + mk[3 * g + 2];
      gv[g] = m0 * b0.x + m1 * b1.x + m2 * b2.x;
      gv[npw_max + g] = m0 * b0.y + m1 * b1.y + m2 * b2.y;
      gv[2 * npw_max + g] = m0 * b0.z + m1 * b1.z + m2 * b2.z;
    }
    __syncthreads();
    const int c16 = lane & 15, kq = lane >> 4;
    const int band = std::min(c16 / 3, kKgBands - 1), axis = c16 % 3;
    const double live = c16 < 3 * kKgBands ? 1.0 : 0.0;
    const double2 *cb = cn + (size_t)band * npw_max;
    const double *ga = gv + (size_t)axis * npw_max;
    int turn = 0;
    for (int tile = 0; tile < n_tiles; ++tile) {
      if (!need[tile] || turn++ % kKgWaves != wave) continue;
      const double2 *cm = ck + (size_t)std::min(16 * tile + c16, nb_max - 1) * npw_max;
      // K-step d of 16 plane waves: lane group kq holds number 4 kq + d
      auto load = [&](double2 (&x)[4], int j0) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int j = j0 + 4 * kq + d;
          x[d] = j < np ? cm[j] : make_double2(0.0, 0.0);
        }
      };
      double2 a[4], nx[4];
      load(nx, 0);
      // every 32 plane waves are summed from zero: beside the large terms of p_mn
      // (those of the bands' own plane waves) the others lose bits within their
      // block only.  Error of W 4 to 5e-16 (one sum: 1.5 to 1.8e-15; 64 lanes and
      // a tree: 2.5 to 3.2e-16), at no measurable time
      f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = re, sre = re, sim = re;
      for (int j0 = 0; j0 < np; j0 += 16) {
        if (j0 % 32 == 0) {
          sre += re;
          sim += im;
          re = im = f64x4{0.0, 0.0, 0.0, 0.0};
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) a[d] = nx[d];
        if (j0 + 16 < np) load(nx, j0 + 16);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int j = std::min(j0 + 4 * kq + d, np - 1);  // past the end a is zero
          const double2 x = a[d], c = cb[j];
          const double g = ga[j] * live;
          const double br = g * c.x, bi = g * c.y;
          // conj(x) b
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, br, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, bi, im, 0, 0, 0);
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, bi, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, br, im, 0, 0, 0);
        }
      }
      re += sre;
      im += sim;
      // lane (row l/16 + 4 e, column l%16): the three axes of a band are
      // neighbouring lanes
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double v = re[e] * re[e] + im[e] * im[e];
        const double s = v + __shfl_down(v, 1) + __shfl_down(v, 2);
        const int m = 16 * tile + kq + 4 * e;
        if (axis == 0 && c16 < 3 * kKgBands && m < nb_max) p2[(size_t)band * nb_max + m] = s;
      }
    }
    __syncthreads();
    for (int t = t0 + tid; t < t1; t += 64 * kKgWaves) {
      const int n = tn[t], m = tm[t];
      if (!mine(n, m)) continue;
      const double p = p2[(size_t)(n - n0) * nb_max + m] / 3.0;
      W[t] = df[t] / delta[t] * p;
      const int o = m >= n0 + count ? kg_opposite(rows_k, tm, m, n) : -1;
      if (o >= 0) W[o] = df[o] / delta[o] * p;
    }
  }
}

// W_t for transitions [0, n), a wavefront per U of them, whose loads wait
// together: for bases that do not fit in LDS five bands at a time (U = 1, flag
// null, a workgroup per four) and for lists in another order (U = 2, only if the
// flag is set, by 2048 workgroups, as more would cost the ordered lists the time
// to start them).  Those of one XCD then take an eighth of the list, so that
// its L2 holds the orbitals of the k they are at.  1.32 million transitions in
// reverse: 1730 us, shuffled 2790 (one at a time, the whole list dealt to all in
// turn: 2040 us in reverse, and 1500 with a workgroup per four).
template <int U>
__global__ void __launch_bounds__(256)
    k_kg_weights(const int *flag, const int *tk, const int *tn, const int *tm, const double *delta,
                 const double *df, long long n, const double2 *coef, const int *miller,
                 const int *npw, int npw_max, int nb_max, int N0, int N1, int N2, double3 b0,
                 double3 b1, double3 b2, double *W) {
  if (flag && !*flag) return;
  const int lane = threadIdx.x & 63, xcds = flag ? 8 : 1, xcd = blockIdx.x % xcds;
  const long long end = n * (xcd + 1) / xcds, stride = 4LL * U * (gridDim.x / xcds);
  for (long long t0 = n * xcd / xcds + U * (4LL * (blockIdx.x / xcds) + (threadIdx.x >> 6));
       t0 < end; t0 += stride) {
    int np[U], most = 0;
    double kr[U][3];
    const double2 *cn[U], *cm[U];
    const int *mk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long t = std::min(t0 + u, end - 1);
      const int k = tk[t];
      const int r0 = k / (N1 * N2), r1 = (k / N2) % N1, r2 = k % N2;
      kr[u][0] = (2.0 * r0 + 1.0 - N0) / (2.0 * N0);
      kr[u][1] = (2.0 * r1 + 1.0 - N1) / (2.0 * N1);
      kr[u][2] = (2.0 * r2 + 1.0 - N2) / (2.0 * N2);
      np[u] = npw[k];
      most = std::max(most, np[u]);
      cn[u] = coef + ((size_t)k * nb_max + tn[t]) * npw_max;
      cm[u] = coef + ((size_t)k * nb_max + tm[t]) * npw_max;
      mk[u] = miller + (size_t)k * npw_max * 3;
    }
    double p[U][3][2] = {};
    for (int g = lane; g < most; g += 64) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = std::min(g, np[u] - 1);
        const double2 a = cm[u][i], b = cn[u][i];
        const double m0 = kr[u][0] + mk[u][3 * i], m1 = kr[u][1] + mk[u][3 * i + 1],
                     m2 = kr[u][2] + mk[u][3 * i + 2];
        if (g >= np[u]) continue;
        const double gx = m0 * b0.x + m1 * b1.x + m2 * b2.x;
        const double gy = m0 * b0.y + m1 * b1.y + m2 * b2.y;
        const double gz = m0 * b0.z + m1 * b1.z + m2 * b2.z;
        // conj(a) b
        const double zr = a.x * b.x + a.y * b.y, zi = a.x * b.y - a.y * b.x;
        p[u][0][0] += gx * zr; p[u][0][1] += gx * zi;
        p[u][1][0] += gy * zr; p[u][1][1] += gy * zi;
        p[u][2][0] += gz * zr; p[u][2][1] += gz * zi;
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          p[u][a][0] += __shfl_xor(p[u][a][0], off);
          p[u][a][1] += __shfl_xor(p[u][a][1], off);
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long t = t0 + u;
      if (lane > 0 || t >= end) continue;
      double s = 0.0;
#pragma unroll
      for (int a = 0; a < 3; ++a) s += p[u][a][0] * p[u][a][0] + p[u][a][1] * p[u][a][1];
      W[t] = df[t] / delta[t] * (s / 3.0);
    }
  }
}

// part[c][w] = sum over chunk c of W_t / (w - delta_t + i eta), one frequency
// per lane and a quarter of the chunk per wavefront, the quarters added in
// order (a whole chunk per wavefront leaves fewer than two blocks a CU for a
// short list, and an uneven tail for a long one: 272 us against 230 below).
// FP64 issue is the bound (154 us at 18 cycles a term).  Two transitions take one
// reciprocal, of the product of their q = |w - delta + i eta|^2 (1 / q1 =
// q2 / (q1 q2)), from the hardware's estimate by one cubic step (residual e of
// 2^-26 or less: e + e^2 leaves e^3); the transitions are the same for all
// lanes and come through scalar loads, eight ahead.  1.32 million transitions
// by 500 frequencies: 525 us with a division each and the transitions in LDS,
// 316 us with a reciprocal each, 230 us so.  Values outside the range of the
// product and the estimate take the division.
__global__ void __launch_bounds__(256)
    k_kg_partial(const double *__restrict__ W, const double *__restrict__ delta, long long n,
                 const double *__restrict__ omega, int n_w, double eta,
                 double2 *__restrict__ part) {
  __shared__ double2 sum[3][64];
  const long long t0 = (long long)blockIdx.y * kKgChunk;
  const int len = (int)std::min<long long>(kKgChunk, n - t0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wi = blockIdx.x * 64 + lane;
  const double w = omega[std::min(wi, n_w - 1)], e2 = eta * eta;
  const double *Wc = W + t0, *dc = delta + t0;
  bool wide = !(e2 > 1e-140 && e2 < 1e140 && fabs(w) < 1e70);
  for (int i = threadIdx.x; i < len; i += 256) wide = wide || !(fabs(dc[i]) < 1e70);
  wide = __syncthreads_or(wide);
  const int each = (len + 3) / 4;
  int i = wave * each;
  const int i1 = std::min(len, i + each);
  double sr = 0.0, sc = 0.0;
  if (!wide && i1 - i >= 8) {
    // eight at a time, the next eight on their way
    const double *pd = dc + i, *pw = Wc + i;
    const int groups = (i1 - i) / 8;
    double nd[8], nw[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) nd[j] = pd[j], nw[j] = pw[j];
    for (int g = 0; g < groups; ++g) {
      double d[8], v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = nd[j], v[j] = nw[j];
      const int step = g + 1 < groups ? 8 : 0;
      pd += step, pw += step;
#pragma unroll
      for (int j = 0; j < 8; ++j) nd[j] = pd[j], nw[j] = pw[j];
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        // W / (x + i eta) = W (x - i eta) / (x^2 + eta^2)
        const double x1 = w - d[j], x2 = w - d[j + 1];
        const double q1 = fma(x1, x1, e2), q2 = fma(x2, x2, e2), q = q1 * q2;
        const double r = __builtin_amdgcn_rcp(q), e = fma(-q, r, 1.0);
        const double inv = fma(r, fma(e, e, e), r);
        const double a1 = v[j] * q2, a2 = v[j + 1] * q1;
        sc = fma(inv, a1 + a2, sc);
        sr = fma(inv, fma(a1, x1, a2 * x2), sr);
      }
    }
    i += 8 * groups;
  }
  for (; i < i1; ++i) {
    const double x = w - dc[i], c = Wc[i] / fma(x, x, e2);
    sr = fma(c, x, sr);
    sc += c;
  }
  if (wave) sum[wave - 1][lane] = make_double2(sr, sc);
  __syncthreads();
  if (wave || wi >= n_w) return;
  for (int j = 0; j < 3; ++j) {
    sr += sum[j][lane].x;
    sc += sum[j][lane].y;
  }
  part[(size_t)blockIdx.y * n_w + wi] = make_double2(sr, -eta * sc);
}

// sigma[w] = i pref sum_c part[c][w]: a block per eight frequencies, 32
// threads each over the chunks in strides of 32, then a fixed-order tree (one
// thread per frequency walked all chunks in two blocks: 174 us for 567 of
// them, now a few).
__global__ void __launch_bounds__(256)
    k_kg_reduce(const double2 *part, int n_chunks, int n_w, double pref, double2 *sigma) {
  __shared__ double2 sh[32][8];
  const int f = threadIdx.x & 7, c0 = threadIdx.x >> 3, wi = blockIdx.x * 8 + f;
  double sr = 0.0, si = 0.0;
  if (wi < n_w)
    for (int c = c0; c < n_chunks; c += 32) {
      const double2 v = part[(size_t)c * n_w + wi];
      sr += v.x;
      si += v.y;
    }
  sh[c0][f] = make_double2(sr, si);
  __syncthreads();
  for (int o = 16; o >= 1; o >>= 1) {
    if (c0 < o) {
      sh[c0][f].x += sh[c0 + o][f].x;
      sh[c0][f].y += sh[c0 + o][f].y;
    }
    __syncthreads();
  }
  if (c0 == 0 && wi < n_w) sigma[wi] = make_double2(-pref * sh[0][f].y, pref * sh[0][f].x);
}

size_t kg_chunks(long long n_trans) { return (size_t)((n_trans + kKgChunk - 1) / kKgChunk); }

}  // namespace
}  // namespace tdx

using namespace tdx;

extern "C" {

int tdx_kg_dsf(tdx_ctx *ctx, const double *sigma, const double *omega, int n_w, double beta,
               double density, double *S_star, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && sigma && omega && S_star, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_w > 0, TDX_ERR_SHAPE, "n_w must be positive");
  TDX_REQUIRE(std::isfinite(beta) && beta > 0 && std::isfinite(density) && density > 0,
              TDX_ERR_INVALID_ARG, "bad beta or density");
  TDX_TRY(check_device(ctx));
  hipLaunchKernelGGL(k_kg_dsf, dim3((n_w + 255) / 256), dim3(256), 0, as_stream(stream),
                     (const double2 *)sigma, omega, n_w, beta, density, S_star);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

size_t tdx_kg_work_bytes(int64_t n_trans, int n_w) {
  if (n_trans < 0 || n_w < 0) return 0;
  const size_t w = ((size_t)n_trans * sizeof(double) + 255) / 256 * 256;
  return w + kg_chunks(n_trans) * (size_t)n_w * sizeof(double2);
}

int tdx_kg_conductivity(tdx_ctx *ctx, const tdx_states *st, const tdx_translist *tl,
                        int64_t n_trans, const double *omega, int n_w, double eta, double *sigma,
                        void *work, size_t work_bytes, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && st && tl && omega && sigma, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_w > 0 && n_trans >= 0, TDX_ERR_SHAPE, "n_w must be positive, n_trans >= 0");
  TDX_REQUIRE(!tl->paired, TDX_ERR_INVALID_ARG,
              "the conductivity takes the full q = 0 list, not a paired one");
  TDX_REQUIRE(std::isfinite(eta) && eta > 0, TDX_ERR_INVALID_ARG, "eta must be positive");
  TDX_REQUIRE(st->omega_cell > 0 && st->n_k > 0, TDX_ERR_INVALID_ARG,
              "states without a cell volume (build them first)");
  TDX_REQUIRE(n_trans <= tl->capacity, TDX_ERR_SHAPE, "n_trans %lld exceeds the list capacity",
              (long long)n_trans);
  TDX_TRY(check_device(ctx));
  hipStream_t s = as_stream(stream);
  const double pref = 2.0 / (st->omega_cell * st->n_k);
  if (n_trans == 0) {
    // sigma = 0 without a memset: one reduction over no chunks
    hipLaunchKernelGGL(k_kg_reduce, dim3((n_w + 7) / 8), dim3(256), 0, s, nullptr, 0, n_w,
                       pref, (double2 *)sigma);
    TDX_HIP(hipGetLastError());
    return TDX_OK;
  }
  TDX_REQUIRE(work && work_bytes >= tdx_kg_work_bytes(n_trans, n_w), TDX_ERR_SHAPE,
              "work needs %zu bytes", tdx_kg_work_bytes(n_trans, n_w));
  TDX_REQUIRE(tl->k && tl->n && tl->m && tl->delta && tl->df, TDX_ERR_INVALID_ARG,
              "transition arrays missing");
  const size_t n_chunks = kg_chunks(n_trans);
  TDX_REQUIRE(n_chunks <= 65535, TDX_ERR_SHAPE, "%lld transitions exceed %d chunks",
              (long long)n_trans, 65535);
  double *W = (double *)work;
  double2 *part = (double2 *)((char *)work + ((size_t)n_trans * sizeof(double) + 255) / 256 * 256);
  const double3 b0 = make_double3(st->bvec[0], st->bvec[1], st->bvec[2]);
  const double3 b1 = make_double3(st->bvec[3], st->bvec[4], st->bvec[5]);
  const double3 b2 = make_double3(st->bvec[6], st->bvec[7], st->bvec[8]);
  const long long nb4 = (n_trans + 3) / 4;
  TDX_REQUIRE(nb4 < (1LL << 31), TDX_ERR_SHAPE, "too many transitions");
  // the rows of the list and the groups with work in the partials' space,
  // which the weights precede
  const long n_rows = (long)st->n_k * st->nb_max;
  const int chunks = (st->nb_max + kKgBands - 1) / kKgBands;
  const long n_chunked = (long)st->n_k * chunks;
  const size_t lds = kg_lds_bytes(st->npw_max, st->nb_max);
  int *flag = (int *)part, *n_groups = flag + 1, *rows = flag + 2, *groups = rows + n_rows + 1;
  const bool by_band = lds <= 160 * 1024 && n_rows < (1L << 30) &&
                       sizeof(int) * (size_t)(3 + n_rows + n_chunked) <=
                           sizeof(double2) * n_chunks * n_w;
  if (by_band) {
    hipLaunchKernelGGL(k_fill<int>, dim3(1), dim3(64), 0, s, flag, 2LL, 0);
    TDX_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_kg_rows, dim3((unsigned)std::min<long long>((n_trans + 255) / 256, 4096)),
                       dim3(256), 0, s, tl->k, tl->n, tl->m, (int)n_trans, st->nb_max, n_rows, rows,
                       flag);
    TDX_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_kg_groups, dim3((unsigned)((n_chunked + 3) / 4)), dim3(256), 0, s, rows,
                       flag, tl->n, tl->m, st->nb_max, chunks, (int)n_chunked, groups, n_groups);
    TDX_HIP(hipGetLastError());
    TDX_HIP(hipFuncSetAttribute((const void *)k_kg_bands,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(k_kg_bands, dim3(2 * ctx->n_cu), dim3(64 * kKgWaves), lds, s, rows, flag,
                       groups, n_groups, tl->n, tl->m, tl->delta, tl->df,
                       (const double2 *)st->coef, st->miller, st->npw, st->npw_max, st->nb_max, st->kgrid[0], st->kgrid[1],
                       st->kgrid[2], b0, b1, b2, W);
    TDX_HIP(hipGetLastError());
  }
#define TDX_KGW(U, GRID, FLAG)                                                                    \
  hipLaunchKernelGGL(k_kg_weights<U>, dim3((unsigned)(GRID)), dim3(256), 0, s, FLAG, tl->k, tl->n, \
                     tl->m, tl->delta, tl->df, (long long)n_trans, (const double2 *)st->coef,      \
                     st->miller, st->npw, st->npw_max, st->nb_max, st->kgrid[0], st->kgrid[1],     \
                     st->kgrid[2], b0, b1, b2, W)
  if (by_band)
    TDX_KGW(2, 2048, flag);
  else
    TDX_KGW(1, nb4, (const int *)nullptr);
#undef TDX_KGW
  TDX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_kg_partial, dim3((n_w + 63) / 64, (unsigned)n_chunks), dim3(256), 0, s, W,
                     tl->delta, (long long)n_trans, omega, n_w, eta, part);
  TDX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_kg_reduce, dim3((n_w + 7) / 8), dim3(256), 0, s, part,
                     (int)n_chunks, n_w, pref, (double2 *)sigma);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

}  // extern "C"
