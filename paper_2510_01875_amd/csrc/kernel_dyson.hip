// Interaction kernel K = v + f_xc and the Dyson solve, both FP64.
//
// K_GG' = 4 pi / |q+G|^2 delta_GG' + f_xc(G - G').  The ALDA part uses the
// density on the real-space grid r_j = sum_i (j_i/N_i) a_i,
//   n(r_j) = 2/(N_k Omega) sum_kn f_nk |sum_G c_nk(G) e^{i G.r_j}|^2,
// the local kernel f_xc(n) = d^2(n eps_xc)/dn^2 (Slater exchange + PW92
// correlation, Phys. Rev. B 45, 13244 (1992)), and
//   f_xc(G) = (1/N_r) sum_j f_xc(r_j) e^{-i G.r_j}.
// Both transforms are separable DFTs (three passes of 1D pencil sums on the
// FP64 MFMA) on a box held in LDS.
//
// Dyson: chi = chi0 + chi0 K chi, column G0 by LU with partial pivoting of
// (1 - chi0 K), one workgroup per frequency.
#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace tdx {
namespace {

constexpr int kMaxSide = 32;
constexpr double kOccSkip = 1e-20;

// Places on an axis of N points: the first c of them are used, all (c = N) or
// the c = 2 M + 1 with |m| <= M, 0 .. M and then -M .. -1.
__device__ inline int dft_place(int i, int c, int N) {
  return c == N || i <= (c - 1) / 2 ? i : N - c + i;
}

// The pencils along one axis of a box: nin places to nout places, for the
// pencils at c_hi x c_lo places of the two other axes.
struct DftPass {
  int N, stride, nin, nout;
  int n_hi, s_hi, c_hi, n_lo, s_lo, c_lo;
  const double2 *tw;
};

typedef double dft_f64x4 __attribute__((ext_vector_type(4)));

// One pass, in place: y_j = sum_m x_m e^{sign 2 pi i m j / N}.  16 pencils are
// one product on the FP64 MFMA, its matrix the real one of (re, im) rows and
// columns (rows past 2 nout and columns past 2 nin are padding), built from the
// twiddle table as the sum goes; a wave reads its pencils whole before it
// writes them.  kRows = ceil(2 nout / 16) tiles of rows, two tiles of pencils
// at a time.
template <int kRows>
__device__ void dft_rows(double *box, const DftPass &d, double sign) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int col = lane & 15, quad = lane >> 4;
  const int pencils = d.c_hi * d.c_lo, steps = (d.nin + 1) / 2;
  const unsigned inv = (65536u + d.N - 1) / d.N;  // x / N for x < 1024
  int jo[kRows];
  bool live[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int i = (16 * r + col) >> 1;
    live[r] = i < d.nout;
    jo[r] = dft_place(std::min(i, d.nout - 1), d.nout, d.N);
  }
  const bool cross = (col ^ quad) & 1;  // re from im or im from re
  const double s = cross ? (col & 1 ? sign : -sign) : 1.0;
  for (int p0 = wave * 32; p0 < pencils; p0 += waves * 32) {
    int base[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int p = std::min(p0 + 16 * x + col, pencils - 1);
      base[x] = 2 * (dft_place(p / d.c_lo, d.c_hi, d.n_hi) * d.s_hi +
                     dft_place(p % d.c_lo, d.c_lo, d.n_lo) * d.s_lo);
    }
    const bool two = p0 + 16 < pencils;
    dft_f64x4 y[2][kRows];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < kRows; ++r) y[x][r] = dft_f64x4{0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < steps; ++k) {
      const int i = 2 * k + (quad >> 1);
      const bool in = i < d.nin;
      const int m = dft_place(std::min(i, d.nin - 1), d.nin, d.N);
      const int at = 2 * m * d.stride + (quad & 1);
      const double b0 = box[base[0] + at], b1 = box[base[1] + at];
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const unsigned mj = m * jo[r];
        const double2 t = d.tw[mj - (mj * inv >> 16) * d.N];
        const double a = in && live[r] ? s * (cross ? t.y : t.x) : 0.0;
        y[0][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b0, y[0][r], 0, 0, 0);
        if (two) y[1][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1, y[1][r], 0, 0, 0);
      }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = 16 * r + quad + 4 * e, i = row >> 1;
          if (i < d.nout && p0 + 16 * x + col < pencils)
            box[base[x] + 2 * dft_place(i, d.nout, d.N) * d.stride + (row & 1)] = y[x][r][e];
        }
  }
}

// DFT of a box in LDS (workgroup of whole waves): sign = +1 from the used
// places (act) of each axis to all, sign = -1 from all to the used ones.  A
// basis of plane waves with |m| <= M takes up (2 M + 1)^3 of the N^3 places, so
// the first pass has fewer pencils, and each a shorter sum.
__device__ void dft_box(double2 *box, const double2 *tw, const int (&N)[3], const int (&act)[3],
                        double sign) {
  for (int step = 0; step < 3; ++step) {
    const int axis = sign > 0 ? 2 - step : step;
    DftPass d;
    d.N = axis == 0 ? N[0] : axis == 1 ? N[1] : N[2];
    const int c = axis == 0 ? act[0] : axis == 1 ? act[1] : act[2];
    d.stride = axis == 0 ? N[1] * N[2] : axis == 1 ? N[2] : 1;
    d.nin = sign > 0 ? c : d.N;
    d.nout = sign > 0 ? d.N : c;
    d.n_hi = axis == 0 ? N[1] : N[0];
    d.s_hi = axis == 0 ? N[2] : N[1] * N[2];
    d.c_hi = axis == 0 ? N[1] : act[0];
    d.n_lo = axis == 2 ? N[1] : N[2];
    d.s_lo = axis == 2 ? N[2] : 1;
    d.c_lo = axis == 2 ? act[1] : N[2];
    d.tw = tw + (axis == 0 ? 0 : axis == 1 ? N[0] : N[0] + N[1]);
    if (d.nout <= 8)
      dft_rows<1>((double *)box, d, sign);
    else if (d.nout <= 16)
      dft_rows<2>((double *)box, d, sign);
    else if (d.nout <= 24)
      dft_rows<3>((double *)box, d, sign);
    else
      dft_rows<4>((double *)box, d, sign);
    __syncthreads();
  }
}

// Places that a basis uses on each axis (all where its reach wraps round);
// box: scratch in LDS.  Ends behind a barrier.
__device__ void dft_reach(const int *mk, int np, const int (&N)[3], int *box, int (&act)[3]) {
  if (threadIdx.x < 3) box[threadIdx.x] = 0;
  __syncthreads();
  int far[3] = {0, 0, 0};
  for (int i = threadIdx.x; i < np; i += blockDim.x)
#pragma unroll
    for (int a = 0; a < 3; ++a) far[a] = std::max(far[a], std::abs(mk[3 * i + a]));
#pragma unroll
  for (int a = 0; a < 3; ++a) atomicMax(&box[a], far[a]);
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 3; ++a) act[a] = 2 * (long)box[a] + 1 < N[a] ? 2 * box[a] + 1 : N[a];
  __syncthreads();
}

__device__ inline int dft_spot(const int *m, const int (&N)[3]) {
  const int a = ((m[0] % N[0]) + N[0]) % N[0];
  const int b = ((m[1] % N[1]) + N[1]) % N[1];
  const int d = ((m[2] % N[2]) + N[2]) % N[2];
  return (a * N[1] + b) * N[2] + d;
}

// The orbitals of a workgroup's bands (n0, n0 + by, .. < nb with occupation),
// one after the other as u(r) on the box: f(n, occupation).  The next one's
// coefficients are on their way meanwhile.
template <typename F>
__device__ void each_orbital(double2 *box, const double2 *tw, const int (&N)[3],
                             const int (&act)[3], const double2 *coef, const double *occ,
                             const int *mk, int n0, int by, int nb, int np, int npw_max, F f) {
  const int tid = threadIdx.x;
  auto first = [&](int n) {
    return n < nb && tid < np ? coef[(size_t)n * npw_max + tid] : make_double2(0.0, 0.0);
  };
  double o = n0 < nb ? occ[n0] : 0.0;
  double2 c = first(n0);
  const int spot = tid < np ? dft_spot(mk + 3 * tid, N) : 0;
  for (int n = n0; n < nb; n += by) {
    const double on = n + by < nb ? occ[n + by] : 0.0;
    const double2 cn = first(n + by);
    if (o >= kOccSkip) {
      for (int j = tid; j < act[0] * act[1] * act[2]; j += blockDim.x) {
        const int a = dft_place(j / (act[1] * act[2]), act[0], N[0]);
        const int b = dft_place(j / act[2] % act[1], act[1], N[1]);
        box[(a * N[1] + b) * N[2] + dft_place(j % act[2], act[2], N[2])] = make_double2(0.0, 0.0);
      }
      __syncthreads();
      if (tid < np) box[spot] = c;
      for (int i = tid + blockDim.x; i < np; i += blockDim.x)
        box[dft_spot(mk + 3 * i, N)] = coef[(size_t)n * npw_max + i];
      __syncthreads();
      dft_box(box, tw, N, act, 1.0);
      f(n, o);
      __syncthreads();
    }
    o = on;
    c = cn;
  }
}

// Twiddle tables for the three axes: tw + off[a], e^{2 pi i t / N_a}.
__device__ void make_twiddles(double2 *tw, int N0, int N1, int N2) {
  const int Ns[3] = {N0, N1, N2};
  int off = 0;
  for (int a = 0; a < 3; ++a) {
    for (int t = threadIdx.x; t < Ns[a]; t += blockDim.x) {
      double s, c;
      sincospi(2.0 * t / Ns[a], &s, &c);
      tw[off + t] = make_double2(c, s);
    }
    off += Ns[a];
  }
}

constexpr int kDensThreads = 512;
constexpr int kDensPoints = 160 * 1024 / 16 / kDensThreads;  // per thread, of what LDS holds

// Partial sums of a k: about four per CU in all, each a share of the bands.
inline int dens_slices(const tdx_ctx *ctx, int n_k) {
  return std::max(1, std::min(16, (4 * ctx->n_cu + n_k - 1) / std::max(n_k, 1)));
}

// Density partials: dens[k][y] = sum_n f_nk |u_nk(r_j)|^2 over the bands n = p,
// p + slices, .. for each p = y, y + gridDim.y, .., these sums added in order.
// Grid (n_k, slices), or (n_k, 1) where a partial per slice has no room.  FP64
// issue is the bound.  64 k of up to 480 plane waves (reach 5) on a 20^3 grid:
// 4928 us with one workgroup per k, a thread per pencil (its values in scratch
// memory) and all places summed; 267 us.
__global__ void __launch_bounds__(kDensThreads)
    k_density(const double2 *coef, const double *occ, const int *nb, const int *npw,
              const int *miller, int nb_max, int npw_max, int N0, int N1, int N2, int slices,
              double *dens) {
  extern __shared__ double2 sm[];
  const int N[3] = {N0, N1, N2}, Nr = N0 * N1 * N2;
  double2 *box = sm;
  double2 *tw = sm + Nr;
  const int k = blockIdx.x, np = npw[k];
  const int *mk = miller + (size_t)k * npw_max * 3;
  int act[3];
  make_twiddles(tw, N0, N1, N2);
  dft_reach(mk, np, N, (int *)box, act);
  double *out = dens + ((size_t)k * gridDim.y + blockIdx.y) * Nr;
  for (int p = blockIdx.y; p < slices; p += gridDim.y) {
    double sum[kDensPoints];
#pragma unroll
    for (int i = 0; i < kDensPoints; ++i) sum[i] = 0.0;
    each_orbital(box, tw, N, act, coef + (size_t)k * nb_max * npw_max, occ + (size_t)k * nb_max, mk,
                 p, slices, nb[k], np, npw_max, [&](int, double f) {
#pragma unroll
                   for (int i = 0; i < kDensPoints; ++i) {
                     const int j = threadIdx.x + i * kDensThreads;
                     if (j < Nr) {
                       const double2 u = box[j];
                       sum[i] = fma(f, u.x * u.x + u.y * u.y, sum[i]);
                     }
                   }
                 });
#pragma unroll
    for (int i = 0; i < kDensPoints; ++i) {
      const int j = threadIdx.x + i * kDensThreads;
      if (j < Nr) out[j] = p == (int)blockIdx.y ? sum[i] : out[j] + sum[i];
    }
  }
}

// Sum of the partials [n_k][per_k][Nr] at point j = 32 block + (thread & 31),
// for the first 32 of 256 threads: those of a k in order, the k in eight
// strided sums, then these in order.
__device__ double sum_partials(const double *dens, int n_k, int per_k, int Nr, int j) {
  __shared__ double part[8][32];
  const int lane = threadIdx.x & 31, row = threadIdx.x >> 5;
  double s = 0.0;
  if (j < Nr)
    for (int k = row; k < n_k; k += 8) {
      const double *of = dens + (size_t)k * per_k * Nr + j;
      double d = of[0];
#pragma unroll 4
      for (int p = 1; p < per_k; ++p) d += of[(size_t)p * Nr];
      s += d;
    }
  part[row][lane] = s;
  __syncthreads();
  for (int i = 1; i < 8; ++i) s += part[i][lane];  // row 0 holds its own
  return s;
}

// Where a call's density partials go: a partial per slice in a workspace of its
// own, which a workspace limit gives back (only the density calls use it, and
// they synchronise), or the one per k that `one` holds where there is a limit
// or no room.  The sums are the same bits either way.
double *dens_partials(tdx_ctx *ctx, int n_k, int slices, int Nr, double *one, int *per_k) {
  *per_k = 1;
  if (ctx->limit || slices == 1) return one;
  void *w;
  if (ws_get(ctx, WS_DENS_SLICES, sizeof(double) * (size_t)n_k * slices * Nr, &w) != TDX_OK) {
    (void)hipGetLastError();
    clear_error();
    return one;
  }
  *per_k = slices;
  return (double *)w;
}

__device__ void pw92(double rs, double *e, double *e1, double *e2) {
  const double A = 0.031091, a1 = 0.21370;
  const double b1 = 7.5957, b2 = 3.5876, b3 = 1.6382, b4 = 0.49294;
  const double s = sqrt(rs);
  const double Q = 2 * A * (b1 * s + b2 * rs + b3 * rs * s + b4 * rs * rs);
  const double Q1 = 2 * A * (0.5 * b1 / s + b2 + 1.5 * b3 * s + 2 * b4 * rs);
  const double Q2 = 2 * A * (-0.25 * b1 / (rs * s) + 0.75 * b3 / s + 2 * b4);
  const double L = log1p(1.0 / Q);
  const double D = Q + Q * Q;
  const double L1 = -Q1 / D;
  const double L2 = -Q2 / D + Q1 * Q1 * (1 + 2 * Q) / (D * D);
  const double g = -2 * A * (1 + a1 * rs);
  *e = g * L;
  *e1 = -2 * A * a1 * L + g * L1;
  *e2 = -4 * A * a1 * L1 + g * L2;
}

// Sum the density partials, scale, apply f_xc(n) pointwise; 32 points a block.
__global__ void __launch_bounds__(256)
    k_fxc_real(const double *dens, int n_k, int per_k, int Nr, double scale, double2 *fx) {
  const int j = blockIdx.x * 32 + (threadIdx.x & 31);
  const double s = sum_partials(dens, n_k, per_k, Nr, j);
  if (threadIdx.x >= 32 || j >= Nr) return;
  const double n = s * scale;
  const double fxv = -(1.0 / 3.0) * cbrt(3.0 / M_PI) * pow(n, -2.0 / 3.0);
  const double rs = cbrt(3.0 / (4.0 * M_PI * n));
  double e, e1, e2;
  pw92(rs, &e, &e1, &e2);
  const double fcv = (rs * rs * e2 - 2.0 * rs * e1) / (9.0 * n);
  fx[j] = make_double2(fxv + fcv, 0.0);
}

// Third derivative of the PW92 correlation in rs (for the kernel's density
// response): with eps = g L(Q), g = -2A(1 + a1 rs) linear in rs,
//   d3 eps = 3 g' L2 + g L3,
//   L3 = -Q3/D + 3 Q1 Q2 (1 + 2Q)/D^2 + 2 Q1^3/D^2 - 2 Q1^3 (1 + 2Q)^2/D^3,
// D = Q(1 + Q), Qj and Lj the j-th derivatives in rs.
__device__ double pw92_e3(double rs) {
  const double A = 0.031091, a1 = 0.21370;
  const double b1 = 7.5957, b2 = 3.5876, b3 = 1.6382, b4 = 0.49294;
  const double s = sqrt(rs);
  const double Q = 2 * A * (b1 * s + b2 * rs + b3 * rs * s + b4 * rs * rs);
  const double Q1 = 2 * A * (0.5 * b1 / s + b2 + 1.5 * b3 * s + 2 * b4 * rs);
  const double Q2 = 2 * A * (-0.25 * b1 / (rs * s) + 0.75 * b3 / s + 2 * b4);
  const double Q3 = 2 * A * (0.375 * b1 / (rs * rs * s) - 0.375 * b3 / (rs * s));
  const double D = Q + Q * Q, T = 1 + 2 * Q;
  const double L2 = -Q2 / D + Q1 * Q1 * T / (D * D);
  const double L3 = -Q3 / D + 3 * Q1 * Q2 * T / (D * D) + 2 * Q1 * Q1 * Q1 / (D * D) -
                    2 * Q1 * Q1 * Q1 * T * T / (D * D * D);
  const double g = -2 * A * (1 + a1 * rs), g1 = -2 * A * a1;
  return 3 * g1 * L2 + g * L3;
}

// d f_xc / dn = d^3(n eps_xc)/dn^3: exchange (2/9)(3/pi)^(1/3) n^(-5/3);
// correlation, with f_c = (rs^2 e2 - 2 rs e1)/(9n) and d rs/dn = -rs/(3n),
//   d f_c/dn = -(rs^3 e3/3 + rs^2 e2 - (8/3) rs e1) / (9 n^2).
__device__ double fxc_deriv(double n) {
  const double dx = (2.0 / 9.0) * cbrt(3.0 / M_PI) * pow(n, -5.0 / 3.0);
  const double rs = cbrt(3.0 / (4.0 * M_PI * n));
  double e, e1, e2;
  pw92(rs, &e, &e1, &e2);
  const double e3 = pw92_e3(rs);
  const double dc =
      -(rs * rs * rs * e3 / 3.0 + rs * rs * e2 - (8.0 / 3.0) * rs * e1) / (9.0 * n * n);
  return dx + dc;
}

// Forward transform of f_xc on the box (one workgroup), scaled by 1/N_r: 46 us
// at 20^3 (316 us with a thread per pencil).
__global__ void __launch_bounds__(kDensThreads)
    k_fxc_forward(double2 *fx, int N0, int N1, int N2) {
  extern __shared__ double2 sm[];
  const int N[3] = {N0, N1, N2}, Nr = N0 * N1 * N2;
  double2 *box = sm, *tw = sm + Nr;
  make_twiddles(tw, N0, N1, N2);
  for (int j = threadIdx.x; j < Nr; j += blockDim.x) box[j] = fx[j];
  __syncthreads();
  dft_box(box, tw, N, N, -1.0);
  const double inv = 1.0 / Nr;
  for (int j = threadIdx.x; j < Nr; j += blockDim.x)
    fx[j] = make_double2(box[j].x * inv, box[j].y * inv);
}

__global__ void k_assemble_k(const int *gb, int n_g, double3 q, double3 b0, double3 b1,
                             double3 b2, const double2 *fxg, int N0, int N1, int N2, int alda,
                             double2 *K) {
  const int i = blockIdx.y, j = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_g || j >= n_g) return;
  double2 v = make_double2(0.0, 0.0);
  if (alda) {
    const int a = (((gb[3 * i] - gb[3 * j]) % N0) + N0) % N0;
    const int b = (((gb[3 * i + 1] - gb[3 * j + 1]) % N1) + N1) % N1;
    const int c = (((gb[3 * i + 2] - gb[3 * j + 2]) % N2) + N2) % N2;
    v = fxg[(a * N1 + b) * N2 + c];
  }
  if (i == j) {
    const int *m = gb + 3 * i;
    const double px = q.x + m[0] * b0.x + m[1] * b1.x + m[2] * b2.x;
    const double py = q.y + m[0] * b0.y + m[1] * b1.y + m[2] * b2.y;
    const double pz = q.z + m[0] * b0.z + m[1] * b1.z + m[2] * b2.z;
    v.x += 4.0 * M_PI / (px * px + py * py + pz * pz);
  }
  K[(size_t)i * n_g + j] = v;
}

// ------------------------------------------------------------------ Dyson
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ inline f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// A_w = I - chi0_w K (row-major) for every w at once: the chi0 matrices form
// one [n_w n][n] left operand, so the product is a single tall one on the
// FP64 MFMA.  A wave owns 16 rows against CB blocks of 16 columns of K; its
// rows come straight from global memory (one 16-byte value per lane and
// K-step, a chunk ahead), chunks of 16 rows of K pass through LDS, double
// buffered, for the four waves of the workgroup.  Rows and columns past the
// end are clamped or zero and not stored.
// At most three column blocks per workgroup: with nine (the rows read once)
// the 1040 workgroups of the crystal's 500 matrices of 133 are two rounds and
// a bit of the chip, 264 us against 210 (484 us on the vector units).
constexpr int kOmCols = 3;

template <int CB>
__device__ __attribute__((always_inline)) void one_minus_tile(double2 *lds, const double2 *chi0,
                                                              const double2 *K, int n,
                                                              long long rows, long long r0, int c0,
                                                              double2 *A) {
  constexpr int kC = 16 * CB, kPer = CB;  // 16 kC values of K over 256 threads
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c16 = lane & 15, kq = lane >> 4;
  const long long r = std::min(r0 + 16 * wave + c16, rows - 1);
  const double2 *arow = chi0 + (size_t)r * n;
  double2 a[4], kv[kPer];
  auto load_a = [&](int k0) {
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = arow[std::min(k0 + 4 * s + kq, n - 1)];
  };
  auto load_k = [&](int k0) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = tid + 256 * i, k = k0 + e / kC, c = c0 + e % kC;
      const double2 v = K[(size_t)std::min(k, n - 1) * n + std::min(c, n - 1)];
      kv[i] = k < n && c < n ? v : make_double2(0.0, 0.0);
    }
  };
  auto store_k = [&](double2 *buf) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) buf[tid + 256 * i] = kv[i];
  };
  f64x4 cr[CB], ci[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) cr[b] = ci[b] = f64x4{0.0, 0.0, 0.0, 0.0};
  load_a(0);
  load_k(0);
  store_k(lds);
  __syncthreads();
  int cur = 0;
  for (int k0 = 0; k0 < n; k0 += 16) {
    const bool more = k0 + 16 < n;
    double2 x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = a[s];
    if (more) {
      load_a(k0 + 16);
      load_k(k0 + 16);
    }
    const double2 *buf = lds + cur * 16 * kC;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (k0 + 4 * s >= n) break;
#pragma unroll
      for (int b = 0; b < CB; ++b) {
        const double2 y = buf[(4 * s + kq) * kC + 16 * b + c16];
        cr[b] = mfma64(x[s].x, y.x, cr[b]);
        ci[b] = mfma64(x[s].x, y.y, ci[b]);
        cr[b] = mfma64(-x[s].y, y.y, cr[b]);
        ci[b] = mfma64(x[s].y, y.x, ci[b]);
      }
    }
    if (more) store_k(lds + (cur ^ 1) * 16 * kC);
    __syncthreads();
    cur ^= 1;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const long long ro = r0 + 16 * wave + kq + 4 * j;  // row l/16 + 4 j of the FP64 MFMA's output
    if (ro >= rows) continue;
    const int i = (int)(ro % n);
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int c = c0 + 16 * b + c16;
      if (c < n)
        A[(size_t)ro * n + c] = make_double2((i == c ? 1.0 : 0.0) - cr[b][j], -ci[b][j]);
    }
  }
}

template <int CB>
__device__ __attribute__((always_inline)) void one_minus_n(int cb, double2 *lds,
                                                           const double2 *chi0, const double2 *K,
                                                           int n, long long rows, long long r0,
                                                           int c0, double2 *A) {
  if constexpr (CB > 1) {
    if (cb < CB) {
      one_minus_n<CB - 1>(cb, lds, chi0, K, n, rows, r0, c0, A);
      return;
    }
  }
  one_minus_tile<CB>(lds, chi0, K, n, rows, r0, c0, A);
}

// Workgroup: 64 rows and one of the gridDim.y nearly equal column groups.
__global__ void __launch_bounds__(256, 2)
    k_one_minus(const double2 *chi0, const double2 *K, int n, long long rows, double2 *A) {
  extern __shared__ double2 om_lds[];
  const int nb = (n + 15) / 16, g = gridDim.y;
  const int b0 = nb * (int)blockIdx.y / g, b1 = nb * ((int)blockIdx.y + 1) / g;
  one_minus_n<kOmCols>(b1 - b0, om_lds, chi0, K, n, rows, 64LL * blockIdx.x, 16 * b0, A);
}

int one_minus(const double2 *chi0, const double2 *K, int n, int n_w, double2 *A, hipStream_t s) {
  const int nb = (n + 15) / 16, groups = (nb + kOmCols - 1) / kOmCols;
  const size_t lds = sizeof(double2) * 2 * 16 * 16 * ((nb + groups - 1) / groups);
  const long long rows = (long long)n_w * n;
  TDX_HIP(hipFuncSetAttribute((const void *)k_one_minus,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(k_one_minus, dim3((unsigned)((rows + 63) / 64), groups), dim3(256), lds, s,
                     chi0, K, n, rows, A);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

constexpr int kLuThreads = 256;

__device__ inline double cabs1(double2 a) { return fabs(a.x) + fabs(a.y); }

__device__ inline double2 cdiv(double2 a, double2 b) {
  // Smith's algorithm
  if (fabs(b.x) >= fabs(b.y)) {
    const double r = b.y / b.x, d = b.x + b.y * r;
    return make_double2((a.x + a.y * r) / d, (a.y - a.x * r) / d);
  }
  const double r = b.x / b.y, d = b.y + b.x * r;
  return make_double2((a.x * r + a.y) / d, (a.y * r - a.x) / d);
}

// ------------------------------------------------ blocked LU, one w per workgroup
// Right-looking LU with partial pivoting (largest |re|+|im|, lowest row on
// ties) in panels of 16 columns, for bases up to kLuMaxN vectors.  An
// unblocked elimination passes over the whole trailing matrix in global
// memory once per column, with three barriers and a tree reduction each time;
// here
//  - a thread holds one row (or two) of the panel in registers; each wave
//    offers its best pivot row through LDS, so a column takes one barrier;
//  - rows do not move during the panel: the chosen ones are moved to the top
//    and the displaced ones into their places as the columns to the right are
//    solved against the panel's unit triangle (a thread per column);
//  - the trailing matrix is updated once per panel on the FP64 MFMA from the
//    panel's multipliers and solved rows in LDS, whose products are summed from
//    zero: an entry is rounded at its own size once a panel.
// A panel is a serial chain (about 2800 cycles a column, of which the pivot
// search and the row's way through LDS take most), so two workgroups share a
// CU where LDS allows (n <= 144): one's panel runs beside the other's update.
// The matrix stays in global memory (L2).  500 matrices of 133: 2.36 ms
// unblocked, 0.40 ms here; with the product 1 - chi0 K, 40 of 305 unblocked:
// 16.6 ms, 80 of 304 here: 1.4 ms.
constexpr int kNb = 16;
// Above 304 vectors the two 16-row operands of an update exceed LDS: the
// unblocked kernels run.
constexpr int kLuMaxN = 304;

// Maximum over the wave, every lane (NaN is ignored).
template <int CTRL, int ROWS>
__device__ inline double dpp_max(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return fmax(x, __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false),
                                  __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false)));
}
__device__ inline double wave_max(double x) {
  x = dpp_max<0x111, 0xf>(x);  // row_shr:1
  x = dpp_max<0x112, 0xf>(x);  // row_shr:2
  x = dpp_max<0x114, 0xf>(x);  // row_shr:4
  x = dpp_max<0x118, 0xf>(x);  // row_shr:8
  x = dpp_max<0x142, 0xa>(x);  // row_bcast:15
  x = dpp_max<0x143, 0xc>(x);  // row_bcast:31
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                          __builtin_amdgcn_readlane(__double2loint(x), 63));
}

__device__ inline double lane_get(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// 1 / z for finite z != 0: z is scaled by a power of two to about one, so
// |z|^2 neither overflows nor vanishes; the reciprocal by two Newton steps.
__device__ inline double2 crecip(double2 z) {
  const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(z.x), fabs(z.y)));
  const double x = ldexp(z.x, -e), y = ldexp(z.y, -e);
  const double d = fma(x, x, y * y);
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  return make_double2(ldexp(x * r, -e), ldexp(-y * r, -e));
}

// LDS of a factorisation (sizes in double2): the multipliers [16][mp] and the
// solved rows [16][mp] of a panel, its 16 x 16 block, the waves' pivot rows,
// the right-hand side and the reciprocal pivots.
struct LuLds {
  double2 *L, *U, *D, *cand, *b, *rinv;
  double *key;                              // [2][4] the waves' pivot sizes
  int *crow, *src, *dst, *q, *perm, *info;  // info: row moves, failing column + 1
  int mp;
};
constexpr int kCand = kNb + 2;  // a pivot row, its right-hand side, its reciprocal pivot
__host__ __device__ inline int lu_mp(int n) { return std::max(16, (n - 1) / 16 * 16); }
__host__ __device__ inline size_t lu_lds_bytes(int n, bool keep) {
  return sizeof(double2) * ((size_t)2 * kNb * lu_mp(n) + kNb * kNb + 2 * (size_t)n) +
         sizeof(double) * 8 + sizeof(int) * (8 + 3 * kNb + 2 + (keep ? (size_t)n : 0));
}
__device__ inline LuLds lu_lds(double2 *sm, int n) {
  LuLds w;
  w.mp = lu_mp(n);
  w.L = sm;
  w.U = w.L + kNb * w.mp;
  w.D = w.U + kNb * w.mp;
  w.cand = w.U;  // a panel's candidates are read before its solved rows are written
  w.b = w.D + kNb * kNb;
  w.rinv = w.b + n;
  w.key = (double *)(w.rinv + n);
  w.crow = (int *)(w.key + 8);
  w.src = w.crow + 8;
  w.dst = w.src + kNb;
  w.q = w.dst + kNb;
  w.info = w.q + kNb;
  w.perm = w.info + 2;
  return w;
}

// f(0), f(1), ... with compile-time arguments.
template <class F, int... J>
__device__ __attribute__((always_inline)) void lu_steps(F &f, std::integer_sequence<int, J...>) {
  (f(std::integral_constant<int, J>{}), ...);
}

// One panel: columns k0 .. k0 + nb - 1, rows k0 .. n - 1 (at most NT RPL).
// The right-hand side rides along as a column of its own.
template <int NT, int RPL, bool KEEP, bool FULL>
__device__ __attribute__((always_inline)) void lu_panel(double2 *A, int n, int k0, int cols,
                                                        const LuLds &w) {
  const int nb = FULL ? kNb : cols;  // straight-line steps for whole panels
  constexpr int kWaves = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double2 a[RPL][kNb + 1];
  bool act[RPL];
  int at[RPL];  // panel step that chose the row
#pragma unroll
  for (int s = 0; s < RPL; ++s) {
    const int r = k0 + tid + NT * s, rc = std::min(r, n - 1);
    act[s] = r < n;
    at[s] = 0;
    const double2 *row = A + (size_t)rc * n + k0;
#pragma unroll
    for (int c = 0; c < kNb; ++c) a[s][c] = row[std::min(c, nb - 1)];
    a[s][kNb] = w.b[rc];
  }
  int dead = 0;  // first column without a usable pivot + 1 (the rest is garbage then)
  auto step = [&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j >= nb) return;
    // the thread's best row, then the wave's; its reciprocal pivot is formed
    // beside the search
    double best = -1.0;
    double2 piv = a[0][j];
    int slot = 0;
#pragma unroll
    for (int s = 0; s < RPL; ++s) {
      const double v = act[s] ? cabs1(a[s][j]) : -1.0;
      if (v > best) {
        best = v;
        piv = a[s][j];
        slot = s;
      }
    }
    const double2 rc = crecip(piv);
    const double mx = wave_max(best);
    // the lowest row of those: a lane's second row lies below all first ones
    unsigned long long at_most = __ballot(best == mx);
    if constexpr (RPL > 1) {
      const unsigned long long upper = __ballot(best == mx && slot == 0);
      if (upper) at_most = upper;
    }
    const int pl = __ffsll((long long)at_most) - 1;
    const int buf = (j & 1) * kWaves;
    if (lane == pl) {
      double2 *o = w.cand + (buf + wave) * kCand;
      o[0] = rc;
#pragma unroll
      for (int c = j; c <= kNb; ++c) {
        double2 x = a[0][c];
        if (RPL > 1 && slot == RPL - 1) x = a[RPL - 1][c];
        o[c + 1] = x;
      }
      w.key[buf + wave] = mx;
      w.crow[buf + wave] = tid + NT * slot;
    }
    __syncthreads();
    double pmax = w.key[buf];
    int row = w.crow[buf], from = 0;
#pragma unroll
    for (int v = 1; v < kWaves; ++v) {
      const double k = w.key[buf + v];
      const int r = w.crow[buf + v];
      if (k > pmax || (k == pmax && r < row)) {
        pmax = k;
        row = r;
        from = v;
      }
    }
    if (dead == 0 && !(pmax > 0.0 && pmax < INFINITY)) dead = k0 + j + 1;
    const double2 *uc = w.cand + (buf + from) * kCand;
    double2 u[kNb + 1];
    const double2 inv = uc[0];
#pragma unroll
    for (int c = j + 1; c <= kNb; ++c) u[c] = uc[c + 1];
    if (tid == 0) {
      w.q[j] = k0 + row;
      w.rinv[k0 + j] = inv;
    }
#pragma unroll
    for (int s = 0; s < RPL; ++s) {
      if (row == tid + NT * s) {
        act[s] = false;
        at[s] = j;
      }
      const double2 x = a[s][j];
      double2 l = make_double2(fma(x.x, inv.x, -(x.y * inv.y)), fma(x.x, inv.y, x.y * inv.x));
      if (act[s])
        a[s][j] = l;
      else
        l = make_double2(0.0, 0.0);
#pragma unroll
      for (int c = j + 1; c <= kNb; ++c) {
        a[s][c].x = fma(-l.x, u[c].x, fma(l.y, u[c].y, a[s][c].x));
        a[s][c].y = fma(-l.x, u[c].y, fma(-l.y, u[c].x, a[s][c].y));
      }
    }
  };
  lu_steps(step, std::make_integer_sequence<int, kNb>{});
  if (dead && tid == 0) w.info[1] = dead;
  __syncthreads();
  if (dead) return;
  // rows k0 .. k0 + nb - 1 that were not chosen take the places of the chosen
  // rows below them, in order (the first wave holds all of them)
  const bool displaced = act[0] && tid < nb;
  int rank = 0;
  if (wave == 0) {
    const unsigned long long dm = __ballot(displaced), below = (1ull << lane) - 1;
    const int qj = lane < nb ? w.q[lane] : 0;
    const bool vac = lane < nb && qj >= k0 + nb;
    const unsigned long long vm = __ballot(vac);
    if (vac) w.dst[__popcll(vm & below)] = qj;
    rank = __popcll(dm & below);
    if (displaced) w.src[rank] = k0 + lane;
    if (lane == 0) w.info[0] = __popcll(dm);
    __threadfence_block();
  }
#pragma unroll
  for (int s = 0; s < RPL; ++s) {
    const int r = k0 + tid + NT * s;
    if (r >= n) continue;
    if (act[s]) {
      const int p = s == 0 && displaced ? w.dst[rank] : r;
#pragma unroll
      for (int c = 0; c < kNb; ++c) {
        if (c >= nb) continue;
        w.L[c * w.mp + p - k0 - nb] = a[s][c];
        if constexpr (KEEP) A[(size_t)p * n + k0 + c] = a[s][c];
      }
      w.b[p] = a[s][kNb];
    } else {
#pragma unroll
      for (int c = 0; c < kNb; ++c) {
        w.D[at[s] * kNb + c] = a[s][c];
        if (c < nb) A[(size_t)(k0 + at[s]) * n + k0 + c] = a[s][c];
      }
      w.b[k0 + at[s]] = a[s][kNb];
    }
  }
}

// Factors A (in place; multipliers stored below the diagonal if KEEP) and
// applies the forward elimination to w.b.  Returns 0 or the failing column
// + 1 (uniform).
template <int NT, int RPL, bool KEEP>
__device__ __attribute__((always_inline)) int lu_factor(double2 *A, int n, const LuLds &w) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c16 = lane & 15, kq = lane >> 4;
  if (tid == 0) w.info[1] = 0;
  __syncthreads();
  for (int k0 = 0; k0 < n; k0 += kNb) {
    const int nb = std::min(kNb, n - k0), e = k0 + nb, m = n - e;
    if (nb < kNb)
      lu_panel<NT, 1, KEEP, false>(A, n, k0, nb, w);
    else if (RPL == 1 || n - k0 <= NT)
      lu_panel<NT, 1, KEEP, true>(A, n, k0, nb, w);
    else
      lu_panel<NT, RPL, KEEP, true>(A, n, k0, nb, w);
    __syncthreads();
    if (w.info[1]) return w.info[1];
    // columns right of the panel and, with KEEP, the finished ones left of it:
    // row moves, then U12 = L11^-1 A12 for those to the right (a partial panel
    // is the last one: nothing to its right)
    const int nmove = __builtin_amdgcn_readfirstlane(w.info[0]), left = KEEP ? k0 : 0;
    for (int t = tid; t < m + left; t += NT) {
      const bool right = t < m;
      const unsigned col = right ? e + t : t - m;
      double2 v[kNb], d[kNb];
#pragma unroll
      for (int i = 0; i < kNb; ++i)
        if (i < nb) {
          const double2 x = (A + (size_t)__builtin_amdgcn_readfirstlane(w.q[i]) * n)[col];
          v[i].x = x.x;
          v[i].y = x.y;
        }
#pragma unroll
      for (int i = 0; i < kNb; ++i)
        if (i < nmove) {
          const double2 x = (A + (size_t)__builtin_amdgcn_readfirstlane(w.src[i]) * n)[col];
          d[i].x = x.x;
          d[i].y = x.y;
        }
#pragma unroll
      for (int i = 0; i < kNb; ++i)
        if (i < nmove)
          (A + (size_t)__builtin_amdgcn_readfirstlane(w.dst[i]) * n)[col] =
              make_double2(d[i].x, d[i].y);
      if (right) {
#pragma unroll
        for (int i = 1; i < kNb; ++i) {
#pragma unroll
          for (int j = 0; j < i; ++j) {
            const double2 l = w.D[i * kNb + j];
            v[i].x = fma(-l.x, v[j].x, fma(l.y, v[j].y, v[i].x));
            v[i].y = fma(-l.x, v[j].y, fma(-l.y, v[j].x, v[i].y));
          }
          if (i % 3 == 0) __builtin_amdgcn_sched_barrier(0);  // else all of D is read at once
        }
#pragma unroll
        for (int i = 0; i < kNb; ++i) w.U[i * w.mp + t] = v[i];
      }
#pragma unroll
      for (int i = 0; i < kNb; ++i)
        if (i < nb) (A + (size_t)(k0 + i) * n)[col] = make_double2(v[i].x, v[i].y);
    }
    if constexpr (KEEP) {
      if (tid == NT - 1) {
        int v[kNb], d[kNb];
#pragma unroll
        for (int i = 0; i < kNb; ++i) {
          if (i < nb) v[i] = w.perm[w.q[i]];
          if (i < nmove) d[i] = w.perm[w.src[i]];
        }
#pragma unroll
        for (int i = 0; i < kNb; ++i) {
          if (i < nb) w.perm[k0 + i] = v[i];
          if (i < nmove) w.perm[w.dst[i]] = d[i];
        }
      }
    }
    __syncthreads();
    if (m == 0) break;
    // trailing update A22 -= L21 U12 in pieces of 16 x 32 dealt to the waves,
    // each piece's values loaded while the one before is updated
    const int mt = (m + 15) / 16, mg = (mt + 1) / 2, pieces = mt * mg;
    double2 *B = A + (size_t)e * n + e;
    double2 nx[2][4];
    auto load = [&](int t) {
      const int i0 = 16 * (t / mg), c0 = 32 * (t % mg) + c16;
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          nx[g][j] = B[(unsigned)(std::min(i0 + kq + 4 * j, m - 1) * n + std::min(c0 + 16 * g, m - 1))];
    };
    if (wave < pieces) load(wave);
    for (int t = wave; t < pieces; t += NT / 64) {
      const int i0 = 16 * (t / mg), c0 = 32 * (t % mg) + c16;
      const bool two = c0 - c16 + 16 < m;  // uniform
      f64x4 cr[2], ci[2];
      double2 old[2][4];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        cr[g] = ci[g] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 4; ++j) old[g][j] = nx[g][j];
      }
      if (t + NT / 64 < pieces) load(t + NT / 64);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        if (g == 1 && !two) break;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double2 l = w.L[(4 * s + kq) * w.mp + i0 + c16];
          const double2 u = w.U[(4 * s + kq) * w.mp + c0 + 16 * g];
          cr[g] = mfma64(l.x, u.x, cr[g]);
          ci[g] = mfma64(l.x, u.y, ci[g]);
          cr[g] = mfma64(-l.y, u.y, cr[g]);
          ci[g] = mfma64(l.y, u.x, ci[g]);
        }
      }
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = i0 + kq + 4 * j, c = c0 + 16 * g;
          if (r < m && c < m) 
            B[(unsigned)(r * n + c)] =
                make_double2(old[g][j].x - cr[g][j], old[g][j].y - ci[g][j]);
        }
    }
    __syncthreads();
  }
  return 0;
}

// Products with the rows already solved are summed from zero, a block of 16 at a
// time, and then subtracted: one at a time from the right-hand side each of
// them is rounded at its size (errors of chi_00 against extended precision, N_G
// 133: 1.07e-15 that way with the trailing update likewise, 7.9e-16 so; dot
// products in a tree over the unblocked matrix 9.0e-16; N_G 17: 4.2, 3.4 and
// 3.4e-16).

// s += a b
__device__ inline void cmadd(double2 &s, double2 a, double2 b) {
  s.x = fma(a.x, b.x, fma(-a.y, b.y, s.x));
  s.y = fma(a.x, b.y, fma(a.y, b.x, s.y));
}

// Lane c's (re, im) inv, in every lane.
__device__ inline double2 lane_quotient(double re, double im, double2 inv, int c) {
  const double x = fma(re, inv.x, -(im * inv.y)), y = fma(re, inv.y, im * inv.x);
  return make_double2(lane_get(x, c), lane_get(y, c));
}

// Back substitution U x = b in blocks of 16 rows, x overwrites w.b, down to
// the block that holds row `stop`.  The first wave solves a block's triangle
// while every thread's row of the columns above it is on its way.
template <int NT>
__device__ __attribute__((always_inline)) void lu_back(const double2 *A, int n, int stop,
                                                       const LuLds &w) {
  const int tid = threadIdx.x;
  for (int k0 = (n - 1) / kNb * kNb; k0 >= 0; k0 -= kNb) {
    const int nb = std::min(kNb, n - k0);
    double2 u[kNb], v[kNb];
    if (tid < 64) {
      const double2 *row = A + (size_t)(k0 + std::min(tid, nb - 1)) * n + k0;
#pragma unroll
      for (int c = 0; c < kNb; ++c) v[c] = row[std::min(c, nb - 1)];
    }
    if (tid < k0) {
      const double2 *row = A + (size_t)tid * n + k0;
#pragma unroll
      for (int c = 0; c < kNb; ++c) u[c] = row[std::min(c, nb - 1)];
    }
    if (tid < 64) {
      const int i = std::min(tid, nb - 1);
      const double2 b = w.b[k0 + i], inv = w.rinv[k0 + i];
      double2 sum = make_double2(0.0, 0.0);
#pragma unroll
      for (int c = kNb - 1; c >= 0; --c) {
        if (c >= nb) continue;
        const double2 xc = lane_quotient(b.x - sum.x, b.y - sum.y, inv, c);
        if (tid < c) cmadd(sum, v[c], xc);
        if (tid == c) w.b[k0 + c] = xc;
      }
    }
    __syncthreads();
    if (k0 <= stop) break;
    for (int r = tid; r < k0; r += NT) {
      if (r != tid) {
        const double2 *row = A + (size_t)r * n + k0;
#pragma unroll
        for (int c = 0; c < kNb; ++c) u[c] = row[std::min(c, nb - 1)];
      }
      double2 sum = make_double2(0.0, 0.0);
#pragma unroll
      for (int c = 0; c < kNb; ++c)
        if (c < nb) cmadd(sum, u[c], w.b[k0 + c]);
      w.b[r] = make_double2(w.b[r].x - sum.x, w.b[r].y - sum.y);
    }
    __syncthreads();
  }
}

// chi_00 of one frequency per workgroup: LU of A_w, right-hand side
// chi0_w[:, g0]; writes x[g0] and a status per frequency.
template <int NT, int RPL>
__global__ void __launch_bounds__(NT, NT == 256 && RPL == 1 ? 2 : 1)
    k_lu_blocked(double2 *Aall, const double2 *chi0, int n, int g0, double2 *out, int *info) {
  extern __shared__ double2 lu_sm[];
  const LuLds w = lu_lds(lu_sm, n);
  const int f = blockIdx.x, tid = threadIdx.x;
  double2 *A = Aall + (size_t)f * n * n;
  const double2 *C = chi0 + (size_t)f * n * n;
  for (int i = tid; i < n; i += NT) w.b[i] = C[(size_t)i * n + g0];
  const int fail = lu_factor<NT, RPL, false>(A, n, w);
  if (!fail) lu_back<NT>(A, n, g0, w);
  if (tid == 0) {
    info[f] = fail;
    out[f] = fail ? make_double2(NAN, NAN) : w.b[g0];
  }
}

// LU with partial pivoting (largest |re|+|im|, lowest index on ties) of A_w,
// right-hand side chi0_w[:, g0]; writes x[g0] and a status per frequency.
__global__ void __launch_bounds__(kLuThreads)
    k_lu_solve(double2 *Aall, const double2 *chi0, int n, int g0, double2 *out, int *info) {
  extern __shared__ double2 sm[];
  double2 *b = sm;              // [n]
  double2 *l = sm + n;          // [n] multipliers
  __shared__ double pv[kLuThreads];
  __shared__ int pi[kLuThreads];
  __shared__ int fail;
  const int w = blockIdx.x, t = threadIdx.x;
  double2 *A = Aall + (size_t)w * n * n;
  const double2 *C = chi0 + (size_t)w * n * n;
  for (int i = t; i < n; i += kLuThreads) b[i] = C[(size_t)i * n + g0];
  if (t == 0) fail = 0;
  __syncthreads();
  for (int c = 0; c < n; ++c) {
    double best = -1.0;
    int arg = n;
    for (int r = c + t; r < n; r += kLuThreads) {
      const double v = cabs1(A[(size_t)r * n + c]);
      if (v > best) {
        best = v;
        arg = r;
      }
    }
    pv[t] = best;
    pi[t] = arg;
    __syncthreads();
    for (int s = kLuThreads / 2; s > 0; s >>= 1) {
      if (t < s) {
        if (pv[t + s] > pv[t] || (pv[t + s] == pv[t] && pi[t + s] < pi[t])) {
          pv[t] = pv[t + s];
          pi[t] = pi[t + s];
        }
      }
      __syncthreads();
    }
    const int p = pi[0];
    const double pmax = pv[0];
    if (!(pmax > 0.0) || !isfinite(pmax)) {
      if (t == 0) fail = c + 1;
      __syncthreads();
      break;
    }
    if (p != c) {
      for (int j = c + t; j < n; j += kLuThreads) {
        const double2 x = A[(size_t)c * n + j];
        A[(size_t)c * n + j] = A[(size_t)p * n + j];
        A[(size_t)p * n + j] = x;
      }
      if (t == 0) {
        const double2 x = b[c];
        b[c] = b[p];
        b[p] = x;
      }
    }
    __syncthreads();
    const double2 piv = A[(size_t)c * n + c];
    for (int r = c + 1 + t; r < n; r += kLuThreads) l[r] = cdiv(A[(size_t)r * n + c], piv);
    __syncthreads();
    const int m = n - c - 1;
    for (long e = t; e < (long)m * (m + 1); e += kLuThreads) {
      const int r = c + 1 + (int)(e / (m + 1));
      const int j = c + 1 + (int)(e % (m + 1));  // j == n stands for the right-hand side
      const double2 lr = l[r];
      if (j < n) {
        const double2 u = A[(size_t)c * n + j];
        double2 &a = A[(size_t)r * n + j];
        a.x = fma(-lr.x, u.x, fma(lr.y, u.y, a.x));
        a.y = fma(-lr.x, u.y, fma(-lr.y, u.x, a.y));
      } else {
        const double2 u = b[c];
        double2 &a = b[r];
        a.x = fma(-lr.x, u.x, fma(lr.y, u.y, a.x));
        a.y = fma(-lr.x, u.y, fma(-lr.y, u.x, a.y));
      }
    }
    __syncthreads();
  }
  if (fail) {
    if (t == 0) {
      info[w] = fail;
      out[w] = make_double2(NAN, NAN);
    }
    return;
  }
  // back substitution, x overwrites b
  __shared__ double sr[kLuThreads], si[kLuThreads];
  for (int r = n - 1; r >= 0; --r) {
    double re = 0.0, im = 0.0;
    for (int j = r + 1 + t; j < n; j += kLuThreads) {
      const double2 a = A[(size_t)r * n + j], x = b[j];
      re = fma(a.x, x.x, fma(-a.y, x.y, re));
      im = fma(a.x, x.y, fma(a.y, x.x, im));
    }
    sr[t] = re;
    si[t] = im;
    __syncthreads();
    for (int s = kLuThreads / 2; s > 0; s >>= 1) {
      if (t < s) {
        sr[t] += sr[t + s];
        si[t] += si[t + s];
      }
      __syncthreads();
    }
    if (t == 0) b[r] = cdiv(make_double2(b[r].x - sr[0], b[r].y - si[0]), A[(size_t)r * n + r]);
    __syncthreads();
  }
  if (t == 0) {
    info[w] = 0;
    out[w] = b[g0];
  }
}


// The LU solves of n_w frequencies: blocked up to kLuMaxN vectors (one wave
// where it holds the panel's rows), above it the unblocked kernel.
int lu_solve(double2 *A, const double2 *chi0, int n, int n_w, int g0, double2 *out, int *info,
             hipStream_t s) {
  if (n > kLuMaxN) {
    hipLaunchKernelGGL(k_lu_solve, dim3(n_w), dim3(kLuThreads), sizeof(double2) * 2 * n, s, A, chi0,
                       n, g0, out, info);
    TDX_HIP(hipGetLastError());
    return TDX_OK;
  }
  const size_t lds = lu_lds_bytes(n, false);
#define TDX_LU(NT, RPL)                                                                        \
  TDX_HIP(hipFuncSetAttribute((const void *)k_lu_blocked<NT, RPL>,                             \
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));          \
  hipLaunchKernelGGL((k_lu_blocked<NT, RPL>), dim3(n_w), dim3(NT), lds, s, A, chi0, n, g0,     \
                     out, info)
  if (n <= 64) {
    TDX_LU(64, 1);
  } else if (n <= 256) {
    TDX_LU(256, 1);
  } else {
    TDX_LU(256, 2);
  }
#undef TDX_LU
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

// Reverse mode of the Dyson step.  chi_00 = e^T A^{-1} chi0 e with
// A = 1 - chi0 K (e = e_g0), so d chi_00 = a^T d chi0 b with
//   a = A^{-T} e            (row g0 of A^{-1}),
//   b = e + K x,  x = A^{-1} chi0 e   (column g0 of 1 + K chi).
// With the cotangent convention dL = Re(conj(cbar) d chi_00) the cotangent
// of chi0 is the rank-1 matrix u v^H, u = cbar conj(a), v = b.
// One workgroup per frequency: LU with partial pivoting of A in place (rows
// swapped whole, multipliers stored below the diagonal, pivot order kept),
// then U x = L^{-1} P chi0 e, and for a: U^T y = e, L^T z = y, a = P^T z.
__device__ inline void block_dot(double re, double im, double *sr, double *si) {
  const int t = threadIdx.x;
  sr[t] = re;
  si[t] = im;
  __syncthreads();
  for (int s = kLuThreads / 2; s > 0; s >>= 1) {
    if (t < s) {
      sr[t] += sr[t + s];
      si[t] += si[t + s];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kLuThreads)
    k_lu_vjp(double2 *Aall, const double2 *chi0, const double2 *K, int n, int g0,
             const double2 *cbar, double2 *u, double2 *v, int *info, double2 *xout) {
  extern __shared__ double2 sm[];
  double2 *x = sm;                   // [n]
  double2 *y = sm + n;               // [n]
  int *piv = (int *)(sm + 2 * n);    // [n]
  __shared__ double pv[kLuThreads];
  __shared__ int pi[kLuThreads];
  __shared__ double sr[kLuThreads], si[kLuThreads];
  __shared__ int fail;
  const int w = blockIdx.x, t = threadIdx.x;
  double2 *A = Aall + (size_t)w * n * n;
  const double2 *C = chi0 + (size_t)w * n * n;
  for (int i = t; i < n; i += kLuThreads) x[i] = C[(size_t)i * n + g0];
  if (t == 0) fail = 0;
  __syncthreads();
  for (int c = 0; c < n; ++c) {
    double best = -1.0;
    int arg = n;
    for (int r = c + t; r < n; r += kLuThreads) {
      const double a = cabs1(A[(size_t)r * n + c]);
      if (a > best) {
        best = a;
        arg = r;
      }
    }
    pv[t] = best;
    pi[t] = arg;
    __syncthreads();
    for (int s = kLuThreads / 2; s > 0; s >>= 1) {
      if (t < s && (pv[t + s] > pv[t] || (pv[t + s] == pv[t] && pi[t + s] < pi[t]))) {
        pv[t] = pv[t + s];
        pi[t] = pi[t + s];
      }
      __syncthreads();
    }
    const int p = pi[0];
    const double pmax = pv[0];
    if (!(pmax > 0.0) || !isfinite(pmax)) {
      if (t == 0) fail = c + 1;
      __syncthreads();
      break;
    }
    if (t == 0) piv[c] = p;
    if (p != c) {
      for (int j = t; j < n; j += kLuThreads) {
        const double2 e = A[(size_t)c * n + j];
        A[(size_t)c * n + j] = A[(size_t)p * n + j];
        A[(size_t)p * n + j] = e;
      }
      if (t == 0) {
        const double2 e = x[c];
        x[c] = x[p];
        x[p] = e;
      }
    }
    __syncthreads();
    const double2 d = A[(size_t)c * n + c];
    for (int r = c + 1 + t; r < n; r += kLuThreads) A[(size_t)r * n + c] = cdiv(A[(size_t)r * n + c], d);
    __syncthreads();
    const int m = n - c - 1;
    for (long e = t; e < (long)m * (m + 1); e += kLuThreads) {
      const int r = c + 1 + (int)(e / (m + 1));
      const int j = c + 1 + (int)(e % (m + 1));  // j == n: right-hand side
      const double2 l = A[(size_t)r * n + c];
      const double2 src = j < n ? A[(size_t)c * n + j] : x[c];
      double2 &dst = j < n ? A[(size_t)r * n + j] : x[r];
      dst.x = fma(-l.x, src.x, fma(l.y, src.y, dst.x));
      dst.y = fma(-l.x, src.y, fma(-l.y, src.x, dst.y));
    }
    __syncthreads();
  }
  double2 *uw = u + (size_t)w * n, *vw = v + (size_t)w * n;
  if (fail) {
    for (int i = t; i < n; i += kLuThreads) uw[i] = vw[i] = make_double2(NAN, NAN);
    if (t == 0) info[w] = fail;
    return;
  }
  // U x = (L^{-1} P chi0 e), x overwritten
  for (int r = n - 1; r >= 0; --r) {
    double re = 0.0, im = 0.0;
    for (int j = r + 1 + t; j < n; j += kLuThreads) {
      const double2 a = A[(size_t)r * n + j], b = x[j];
      re = fma(a.x, b.x, fma(-a.y, b.y, re));
      im = fma(a.x, b.y, fma(a.y, b.x, im));
    }
    block_dot(re, im, sr, si);
    if (t == 0) x[r] = cdiv(make_double2(x[r].x - sr[0], x[r].y - si[0]), A[(size_t)r * n + r]);
    __syncthreads();
  }
  if (xout)
    for (int i = t; i < n; i += kLuThreads) xout[(size_t)w * n + i] = x[i];
  // v = e + K x
  for (int i = t; i < n; i += kLuThreads) {
    double re = i == g0 ? 1.0 : 0.0, im = 0.0;
    const double2 *Ki = K + (size_t)i * n;
    for (int j = 0; j < n; ++j) {
      const double2 a = Ki[j], b = x[j];
      re = fma(a.x, b.x, fma(-a.y, b.y, re));
      im = fma(a.x, b.y, fma(a.y, b.x, im));
    }
    vw[i] = make_double2(re, im);
  }
  // U^T y = e (forward), entries of U^T are A[j][i], j <= i
  for (int i = 0; i < n; ++i) {
    double re = 0.0, im = 0.0;
    for (int j = t; j < i; j += kLuThreads) {
      const double2 a = A[(size_t)j * n + i], b = y[j];
      re = fma(a.x, b.x, fma(-a.y, b.y, re));
      im = fma(a.x, b.y, fma(a.y, b.x, im));
    }
    block_dot(re, im, sr, si);
    if (t == 0)
      y[i] = cdiv(make_double2((i == g0 ? 1.0 : 0.0) - sr[0], -si[0]), A[(size_t)i * n + i]);
    __syncthreads();
  }
  // L^T z = y (backward, unit diagonal), z overwrites y
  for (int i = n - 1; i >= 0; --i) {
    double re = 0.0, im = 0.0;
    for (int j = i + 1 + t; j < n; j += kLuThreads) {
      const double2 a = A[(size_t)j * n + i], b = y[j];
      re = fma(a.x, b.x, fma(-a.y, b.y, re));
      im = fma(a.x, b.y, fma(a.y, b.x, im));
    }
    block_dot(re, im, sr, si);
    if (t == 0) y[i] = make_double2(y[i].x - sr[0], y[i].y - si[0]);
    __syncthreads();
  }
  // a = P^T z: undo the row swaps last to first
  if (t == 0) {
    for (int c = n - 1; c >= 0; --c) {
      const int p = piv[c];
      const double2 e = y[c];
      y[c] = y[p];
      y[p] = e;
    }
    info[w] = 0;
  }
  __syncthreads();
  const double2 cb = cbar[w];
  for (int i = t; i < n; i += kLuThreads) {
    const double2 a = y[i];  // u = cbar conj(a)
    uw[i] = make_double2(cb.x * a.x + cb.y * a.y, cb.y * a.x - cb.x * a.y);
  }
}

// k_lu_vjp on the blocked factorisation (bases up to kLuMaxN vectors).
template <int NT, int RPL>
__global__ void __launch_bounds__(NT, NT == 256 && RPL == 1 ? 2 : 1)
    k_lu_vjp_blocked(double2 *Aall, const double2 *chi0, const double2 *K, int n, int g0,
                     const double2 *cbar, double2 *u, double2 *v, int *info, double2 *xout) {
  extern __shared__ double2 lu_sm[];
  const LuLds w = lu_lds(lu_sm, n);
  const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double2 *A = Aall + (size_t)f * n * n;
  const double2 *C = chi0 + (size_t)f * n * n;
  double2 *uw = u + (size_t)f * n, *vw = v + (size_t)f * n;
  for (int i = tid; i < n; i += NT) {
    w.b[i] = C[(size_t)i * n + g0];
    w.perm[i] = i;
  }
  const int fail = lu_factor<NT, RPL, true>(A, n, w);
  if (tid == 0) info[f] = fail;
  if (fail) {
    for (int i = tid; i < n; i += NT) uw[i] = vw[i] = make_double2(NAN, NAN);
    return;
  }
  lu_back<NT>(A, n, 0, w);
  __syncthreads();
  if (xout)
    for (int i = tid; i < n; i += NT) xout[(size_t)f * n + i] = w.b[i];
  // v = e + K x, a row per wave
  for (int i = wave; i < n; i += NT / 64) {
    double re = 0.0, im = 0.0;
    for (int j = lane; j < n; j += 64) {
      const double2 a = K[(size_t)i * n + j], b = w.b[j];
      re = fma(a.x, b.x, fma(-a.y, b.y, re));
      im = fma(a.x, b.y, fma(a.y, b.x, im));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      re += __shfl_xor(re, o);
      im += __shfl_xor(im, o);
    }
    if (lane == 0) vw[i] = make_double2(re + (i == g0 ? 1.0 : 0.0), im);
  }
  double2 *y = w.L;  // the panel operands are done with
  for (int i = tid; i < n; i += NT) y[i] = make_double2(i == g0 ? 1.0 : 0.0, 0.0);
  __syncthreads();
  // r[c] -= sum_i M[k0 + i][c] y[k0 + i] over the columns c0 <= c < c1
  auto apply = [&](int k0, int nb, int c0, int c1) {
    for (int c = c0 + tid; c < c1; c += NT) {
      double2 sum = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < kNb; ++i)
        if (i < nb) cmadd(sum, A[(size_t)(k0 + i) * n + c], y[k0 + i]);
      y[c] = make_double2(y[c].x - sum.x, y[c].y - sum.y);
    }
    __syncthreads();
  };
  // U^T y = e: forward, from the block of g0 (y is zero before it)
  for (int k0 = g0 / kNb * kNb; k0 < n; k0 += kNb) {
    const int nb = std::min(kNb, n - k0);
    if (tid < 64) {
      const int j = std::min(tid, nb - 1);
      double2 m[kNb], sum = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < kNb; ++i) m[i] = A[(size_t)(k0 + std::min(i, nb - 1)) * n + k0 + j];
      const double2 inv = w.rinv[k0 + j], r = y[k0 + j];
#pragma unroll
      for (int i = 0; i < kNb; ++i) {
        if (i >= nb) continue;
        const double2 yi = lane_quotient(r.x - sum.x, r.y - sum.y, inv, i);
        if (tid > i) cmadd(sum, m[i], yi);
        if (tid == i) y[k0 + i] = yi;
      }
    }
    __syncthreads();
    apply(k0, nb, k0 + nb, n);
  }
  // L^T z = y: backward, unit diagonal
  for (int k0 = (n - 1) / kNb * kNb; k0 >= 0; k0 -= kNb) {
    const int nb = std::min(kNb, n - k0);
    if (tid < 64) {
      const int j = std::min(tid, nb - 1);
      double2 m[kNb], sum = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < kNb; ++i) m[i] = A[(size_t)(k0 + std::min(i, nb - 1)) * n + k0 + j];
      const double2 r = y[k0 + j];
#pragma unroll
      for (int i = kNb - 1; i >= 0; --i) {
        if (i >= nb) continue;
        const double2 zi = make_double2(lane_get(r.x - sum.x, i), lane_get(r.y - sum.y, i));
        if (tid < i) cmadd(sum, m[i], zi);
        if (tid == i) y[k0 + i] = zi;
      }
    }
    __syncthreads();
    apply(k0, nb, 0, k0);
  }
  // a = P^T z, u = cbar conj(a)
  const double2 cb = cbar[f];
  for (int i = tid; i < n; i += NT) {
    const double2 a = y[i];
    uw[w.perm[i]] = make_double2(cb.x * a.x + cb.y * a.y, cb.y * a.x - cb.x * a.y);
  }
}

int lu_vjp(double2 *A, const double2 *chi0, const double2 *K, int n, int n_w, int g0,
           const double2 *cbar, double2 *u, double2 *v, int *info, double2 *xout, hipStream_t s) {
  if (n > kLuMaxN) {
    hipLaunchKernelGGL(k_lu_vjp, dim3(n_w), dim3(kLuThreads),
                       (sizeof(double2) * 2 + sizeof(int)) * (size_t)n, s, A, chi0, K, n, g0, cbar,
                       u, v, info, xout);
    TDX_HIP(hipGetLastError());
    return TDX_OK;
  }
  const size_t lds = lu_lds_bytes(n, true);
#define TDX_LU(NT, RPL)                                                                          \
  TDX_HIP(hipFuncSetAttribute((const void *)k_lu_vjp_blocked<NT, RPL>,                           \
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));            \
  hipLaunchKernelGGL((k_lu_vjp_blocked<NT, RPL>), dim3(n_w), dim3(NT), lds, s, A, chi0, K, n, g0, \
                     cbar, u, v, info, xout)
  if (n <= 64) {
    TDX_LU(64, 1);
  } else if (n <= 256) {
    TDX_LU(256, 1);
  } else {
    TDX_LU(256, 2);
  }
#undef TDX_LU
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

// ------------------------------------------------- ALDA kernel adjoint
// The cotangent of the kernel matrix from the Dyson solve, then of f_xc on
// the grid, then of the density and through it of the occupations and the
// orbitals.  With x = A^{-1} chi0 e, a = A^{-T} e and u = chi00_bar conj(a)
// (k_lu_vjp), d chi00 = (chi0^T a)^T dK x, so
//   Kbar[G][G'] = sum_w p_w[G] conj(x_w[G']),  p_w = chi0(w)^H u_w.

// p_w = chi0(w)^H u_w (row-major chi0: p[G] = sum_H conj(chi0[H][G]) u[H]).
__global__ void k_chi0h_u(const double2 *chi0, const double2 *u, int n, double2 *p) {
  const int w = blockIdx.y, g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const double2 *C = chi0 + (size_t)w * n * n;
  const double2 *uw = u + (size_t)w * n;
  double re = 0.0, im = 0.0;
  for (int h = 0; h < n; ++h) {
    const double2 c = C[(size_t)h * n + g], a = uw[h];
    re = fma(c.x, a.x, fma(c.y, a.y, re));
    im = fma(c.x, a.y, fma(-c.y, a.x, im));
  }
  p[(size_t)w * n + g] = make_double2(re, im);
}

// Kbar[G][G'] += sum_w p_w[G] conj(x_w[G']), frequencies in order.
__global__ void k_kbar(const double2 *p, const double2 *x, int n, int n_w, double2 *Kbar) {
  const int i = blockIdx.y, j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  double re = 0.0, im = 0.0;
  for (int w = 0; w < n_w; ++w) {
    const double2 a = p[(size_t)w * n + i], b = x[(size_t)w * n + j];
    re = fma(a.x, b.x, fma(a.y, b.y, re));
    im = fma(a.y, b.x, fma(-a.x, b.y, im));
  }
  double2 &o = Kbar[(size_t)i * n + j];
  o.x += re;
  o.y += im;
}

// Phi[j][b] = exp(i G_b . r_j) = exp(2 pi i m_b . (j_0/N0, j_1/N1, j_2/N2)),
// the phases of the forward transform (integer products reduced mod N).
__global__ void k_phi(const int *gb, int n_g, int N0, int N1, int N2, double2 *Phi) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
  if (b >= n_g) return;
  const int j0 = j / (N1 * N2), j1 = (j / N2) % N1, j2 = j % N2;
  const int p0 = ((gb[3 * b] * j0) % N0 + N0) % N0;
  const int p1 = ((gb[3 * b + 1] * j1) % N1 + N1) % N1;
  const int p2 = ((gb[3 * b + 2] * j2) % N2 + N2) % N2;
  double sn, cs;
  sincospi(2.0 * ((double)p0 / N0 + (double)p1 / N1 + (double)p2 / N2), &sn, &cs);
  Phi[(size_t)j * n_g + b] = make_double2(cs, sn);
}

// fbar[j] += (1/N_r) Re sum_a conj(Phi[j][a]) T[j][a], T[j][a] =
// sum_b conj(Kbar[a][b]) Phi[j][b]: the cotangent of f_xc(r_j) from
// K[a][b] = (1/N_r) sum_j f_xc(r_j) exp(-i (G_a - G_b) . r_j).
__global__ void k_fbar(const double2 *Phi, const double2 *T, int n_g, int Nr, double *fbar) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= Nr) return;
  double re = 0.0;
  for (int a = 0; a < n_g; ++a) {
    const double2 f = Phi[(size_t)j * n_g + a], t = T[(size_t)j * n_g + a];
    re = fma(f.x, t.x, fma(f.y, t.y, re));
  }
  fbar[j] += re / Nr;
}

// nbar[j] = fbar[j] f_xc'(n(r_j)), n from the density partials; 32 points a block.
__global__ void __launch_bounds__(256)
    k_nbar(const double *dens, int n_k, int per_k, int Nr, double scale, const double *fbar,
           double *nbar) {
  const int j = blockIdx.x * 32 + (threadIdx.x & 31);
  const double s = sum_partials(dens, n_k, per_k, Nr, j);
  if (threadIdx.x >= 32 || j >= Nr) return;
  nbar[j] = fbar[j] * fxc_deriv(s * scale);
}

// Density adjoint of the bands n = slice, slice + slices, .. of a k (those the
// forward density summed); grid (n_k, slices):
//   occ_bar[k][n] += scale sum_j nbar_j |u_nk(r_j)|^2,
//   coef_bar[k][n](G) += 2 scale f_nk sum_j nbar_j u_nk(r_j) e^{-i G.r_j}
// (the second a forward transform of nbar u on the box, read at the basis).
__global__ void __launch_bounds__(kDensThreads)
    k_density_vjp(const double2 *coef, const double *occ, const int *nb, const int *npw,
                  const int *miller, int nb_max, int npw_max, int N0, int N1, int N2,
                  double scale, const double *nbar, double *occ_bar, double2 *coef_bar) {
  extern __shared__ double2 sm[];
  __shared__ double red[kDensThreads / 64];
  const int N[3] = {N0, N1, N2}, Nr = N0 * N1 * N2;
  double2 *box = sm;
  double2 *tw = sm + Nr;
  const int k = blockIdx.x, np = npw[k];
  const int *mk = miller + (size_t)k * npw_max * 3;
  int act[3];
  make_twiddles(tw, N0, N1, N2);
  dft_reach(mk, np, N, (int *)box, act);
  each_orbital(
      box, tw, N, act, coef + (size_t)k * nb_max * npw_max, occ + (size_t)k * nb_max, mk,
      blockIdx.y, gridDim.y, nb[k], np, npw_max, [&](int n, double f) {
        double s = 0.0;
        for (int j = threadIdx.x; j < Nr; j += kDensThreads) {
          const double2 u = box[j];
          const double w = nbar[j];
          s = fma(w, u.x * u.x + u.y * u.y, s);
          box[j] = make_double2(w * u.x, w * u.y);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
          for (int i = 1; i < kDensThreads / 64; ++i) s += red[i];
          occ_bar[(size_t)k * nb_max + n] += scale * s;
        }
        if (!coef_bar) return;
        dft_box(box, tw, N, act, -1.0);
        double2 *cb = coef_bar + ((size_t)k * nb_max + n) * npw_max;
        const double g = 2.0 * scale * f;
        for (int i = threadIdx.x; i < np; i += kDensThreads) {
          const double2 v = box[dft_spot(mk + 3 * i, N)];
          cb[i].x += g * v.x;
          cb[i].y += g * v.y;
        }
      });
}

// First failing frequency of a chunk of LU solves folded into the running
// status {frequency, column + 1} (one block; status[0] = INT_MAX: none yet).
__global__ void k_fold_status(const int *info, int n, int w0, int *status) {
  __shared__ int best[256];
  int b = INT_MAX;
  for (int i = threadIdx.x; i < n; i += 256)
    if (info[i] != 0) b = min(b, i);
  best[threadIdx.x] = b;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) best[threadIdx.x] = min(best[threadIdx.x], best[threadIdx.x + st]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && best[0] != INT_MAX && w0 + best[0] < status[0]) {
    status[0] = w0 + best[0];
    status[1] = info[best[0]];
  }
}

__global__ void k_clear_status(int *status) {
  if (threadIdx.x == 0) {
    status[0] = INT_MAX;
    status[1] = 0;
  }
}

// Scratch of the no-allocation Dyson entry point: a file-scope device array
// of fixed size (every GPU the library runs on holds its own copy until the
// process ends), laid out as the status words (256 bytes), the per-frequency
// pivot status of one chunk (rounded to 256 bytes), then the chunk's
// matrices 1 - chi0 K.  Host code reaches it only through the per-device
// address resolved below.
constexpr size_t kDysonScratchBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;
__device__ __align__(256) unsigned char scratch[kDysonScratchBytes];
void *g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mu;

size_t round256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

// With `device` current: resolve that device's address of the scratch array
// (once per device; later calls return at once).
int dyson_scratch_init(int device) {
  TDX_REQUIRE(device >= 0 && device < kMaxDevices, TDX_ERR_UNSUPPORTED,
              "device %d beyond the %d the scratch table holds", device, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return TDX_OK;
  void *p = nullptr;
  TDX_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
  TDX_REQUIRE(p != nullptr, TDX_ERR_HIP, "no device address for the Dyson scratch");
  g_scratch_ptr[device] = p;
  return TDX_OK;
}

}  // namespace tdx

using namespace tdx;

extern "C" {

size_t tdx_dyson_noalloc_max_bytes(void) { return kDysonScratchBytes; }

int tdx_dyson_noalloc(tdx_ctx *ctx, const double *chi0, const double *K, int n_g, int n_w,
                      int i_g0, double *chi00, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && chi0 && K && chi00, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_g > 0 && n_w > 0 && i_g0 >= 0 && i_g0 < n_g, TDX_ERR_SHAPE, "bad sizes");
  TDX_REQUIRE((size_t)n_g * 2 * sizeof(double2) <= 64 * 1024, TDX_ERR_SHAPE,
              "n_g %d too large for the LU kernel", n_g);
  const size_t mat = sizeof(double2) * (size_t)n_g * n_g;
  // frequencies per pass: the status words, their pivot status and their
  // matrices must fit in the scratch
  long long cw = (long long)((kDysonScratchBytes - 512) / (mat + sizeof(int)));
  cw = std::min<long long>(std::min<long long>(cw, n_w), 65535);
  while (cw > 0 && 256 + round256(sizeof(int) * (size_t)cw) + mat * (size_t)cw > kDysonScratchBytes)
    --cw;
  TDX_REQUIRE(cw >= 1, TDX_ERR_SHAPE,
              "n_g %d: one %zu-byte matrix exceeds the %zu-byte scratch of this entry point", n_g,
              mat, kDysonScratchBytes);
  TDX_TRY(check_device(ctx));
  TDX_REQUIRE(ctx->device >= 0 && ctx->device < kMaxDevices && g_scratch_ptr[ctx->device],
              TDX_ERR_HIP, "scratch of device %d not set up", ctx->device);
  hipStream_t s = as_stream(stream);
  unsigned char *base = (unsigned char *)g_scratch_ptr[ctx->device];
  int *status = (int *)base;
  int *info = (int *)(base + 256);
  double2 *A = (double2 *)(base + 256 + round256(sizeof(int) * (size_t)cw));
  hipLaunchKernelGGL(k_clear_status, dim3(1), dim3(64), 0, s, status);
  TDX_HIP(hipGetLastError());
  const size_t n2 = (size_t)n_g * n_g;
  for (int w0 = 0; w0 < n_w; w0 += (int)cw) {
    const int nw = (int)std::min<long long>(cw, n_w - w0);
    const double2 *c = (const double2 *)chi0 + (size_t)w0 * n2;
    TDX_TRY(one_minus(c, (const double2 *)K, n_g, nw, A, s));
    TDX_TRY(lu_solve(A, c, n_g, nw, i_g0, (double2 *)chi00 + w0, info, s));
    hipLaunchKernelGGL(k_fold_status, dim3(1), dim3(256), 0, s, info, nw, w0, status);
    TDX_HIP(hipGetLastError());
  }
  int h[2] = {0, 0};
  TDX_HIP(hipMemcpyAsync(h, status, sizeof(h), hipMemcpyDeviceToHost, s));
  TDX_HIP(hipStreamSynchronize(s));
  TDX_REQUIRE(h[0] == INT_MAX, TDX_ERR_NUMERIC,
              "Dyson matrix singular at frequency %d (column %d)", h[0], h[1] - 1);
  return TDX_OK;
}


// Check the density grid against the states and the LDS of the density and
// FFT kernels.
static int check_grid(const tdx_states *st, const int dens_grid[3], int *Nr, size_t *lds) {
  TDX_REQUIRE(dens_grid, TDX_ERR_INVALID_ARG, "ALDA needs a density grid");
  for (int i = 0; i < 3; ++i)
    TDX_REQUIRE(dens_grid[i] >= 2 * st->mmax[i] + 1 && dens_grid[i] <= kMaxSide, TDX_ERR_SHAPE,
                "density grid side %d must lie in [%d, %d]", dens_grid[i], 2 * st->mmax[i] + 1,
                kMaxSide);
  *Nr = dens_grid[0] * dens_grid[1] * dens_grid[2];
  *lds = sizeof(double2) * (*Nr + dens_grid[0] + dens_grid[1] + dens_grid[2]);
  TDX_REQUIRE(*lds <= 160 * 1024, TDX_ERR_SHAPE, "density grid of %d points exceeds LDS", *Nr);
  return TDX_OK;
}

int tdx_xc_kernel_grid(tdx_ctx *ctx, const tdx_states *st, const int dens_grid[3], double *fxg,
                       tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && st && fxg, TDX_ERR_INVALID_ARG, "null argument");
  TDX_TRY(check_device(ctx));
  int Nr;
  size_t lds;
  TDX_TRY(check_grid(st, dens_grid, &Nr, &lds));
  hipStream_t s = as_stream(stream);
  const int N0 = dens_grid[0], N1 = dens_grid[1], N2 = dens_grid[2];
  void *w;
  const int slices = dens_slices(ctx, st->n_k);
  TDX_TRY(ws_get(ctx, WS_DENS, sizeof(double) * (size_t)st->n_k * Nr, &w));
  int per_k;
  double *dens = dens_partials(ctx, st->n_k, slices, Nr, (double *)w, &per_k);
  TDX_HIP(hipFuncSetAttribute((const void *)k_density, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds));
  TDX_HIP(hipFuncSetAttribute((const void *)k_fxc_forward,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(k_density, dim3(st->n_k, per_k), dim3(kDensThreads), lds, s,
                     (const double2 *)st->coef, st->occ, st->nb, st->npw, st->miller, st->nb_max,
                     st->npw_max, N0, N1, N2, slices, dens);
  TDX_HIP(hipGetLastError());
  const double scale = 2.0 / (st->n_k * st->omega_cell);
  hipLaunchKernelGGL(k_fxc_real, dim3((Nr + 31) / 32), dim3(256), 0, s, dens, st->n_k, per_k, Nr,
                     scale, (double2 *)fxg);
  TDX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_fxc_forward, dim3(1), dim3(kDensThreads), lds, s, (double2 *)fxg, N0, N1,
                     N2);
  TDX_HIP(hipGetLastError());
  TDX_HIP(hipStreamSynchronize(s));  // the density workspace may be reused after return
  return TDX_OK;
}

int tdx_kernel_matrix_from_grid(tdx_ctx *ctx, const tdx_states *st, const int qj[3],
                                const int *gbasis, int n_g, int xc, const int dens_grid[3],
                                const double *fxg, double *K, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && st && qj && gbasis && K, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(xc == TDX_XC_RPA || xc == TDX_XC_ALDA, TDX_ERR_INVALID_ARG, "bad xc");
  TDX_REQUIRE(n_g > 0, TDX_ERR_SHAPE, "n_g must be positive");
  TDX_TRY(check_device(ctx));
  int N0 = 1, N1 = 1, N2 = 1;
  if (xc == TDX_XC_ALDA) {
    TDX_REQUIRE(fxg, TDX_ERR_INVALID_ARG, "ALDA needs the kernel grid");
    int Nr;
    size_t lds;
    TDX_TRY(check_grid(st, dens_grid, &Nr, &lds));
    N0 = dens_grid[0];
    N1 = dens_grid[1];
    N2 = dens_grid[2];
  }
  hipStream_t s = as_stream(stream);
  const double *B = st->bvec;
  const double3 b0 = make_double3(B[0], B[1], B[2]), b1 = make_double3(B[3], B[4], B[5]),
                b2 = make_double3(B[6], B[7], B[8]);
  double qr[3];
  for (int i = 0; i < 3; ++i) qr[i] = (double)qj[i] / st->kgrid[i];
  const double3 q = make_double3(qr[0] * B[0] + qr[1] * B[3] + qr[2] * B[6],
                                 qr[0] * B[1] + qr[1] * B[4] + qr[2] * B[7],
                                 qr[0] * B[2] + qr[1] * B[5] + qr[2] * B[8]);
  hipLaunchKernelGGL(k_assemble_k, dim3((n_g + 63) / 64, n_g), dim3(64), 0, s, gbasis, n_g, q, b0,
                     b1, b2, xc == TDX_XC_ALDA ? (const double2 *)fxg : nullptr, N0, N1, N2,
                     xc == TDX_XC_ALDA ? 1 : 0, (double2 *)K);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

int tdx_kernel_matrix(tdx_ctx *ctx, const tdx_states *st, const int qj[3], const int *gbasis,
                      int n_g, int xc, const int dens_grid[3], double *K, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && st && qj && gbasis && K, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(xc == TDX_XC_RPA || xc == TDX_XC_ALDA, TDX_ERR_INVALID_ARG, "bad xc");
  if (xc == TDX_XC_RPA)
    return tdx_kernel_matrix_from_grid(ctx, st, qj, gbasis, n_g, xc, dens_grid, nullptr, K,
                                       stream);
  int Nr;
  size_t lds;
  TDX_TRY(check_grid(st, dens_grid, &Nr, &lds));
  void *w;
  TDX_TRY(ws_get(ctx, WS_FXC, sizeof(double2) * (size_t)Nr, &w));
  TDX_TRY(tdx_xc_kernel_grid(ctx, st, dens_grid, (double *)w, stream));
  TDX_TRY(tdx_kernel_matrix_from_grid(ctx, st, qj, gbasis, n_g, xc, dens_grid, (const double *)w,
                                      K, stream));
  TDX_HIP(hipStreamSynchronize(as_stream(stream)));
  return TDX_OK;
}

size_t tdx_dyson_work_bytes(int n_g, int n_w) {
  return sizeof(double2) * (size_t)n_w * n_g * n_g;
}

int tdx_dyson_async(tdx_ctx *ctx, const double *chi0, const double *K, int n_g, int n_w,
                    int i_g0, double *chi00, void *work, int *info, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && chi0 && K && chi00 && work && info, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_g > 0 && n_w > 0 && i_g0 >= 0 && i_g0 < n_g, TDX_ERR_SHAPE, "bad sizes");
  TDX_REQUIRE((size_t)n_g * 2 * sizeof(double2) <= 64 * 1024, TDX_ERR_SHAPE,
              "n_g %d too large for the LU kernel", n_g);
  TDX_REQUIRE(n_w <= 65535, TDX_ERR_SHAPE, "n_w %d above 65535", n_w);
  hipStream_t s = as_stream(stream);
  double2 *A = (double2 *)work;
  TDX_TRY(one_minus((const double2 *)chi0, (const double2 *)K, n_g, n_w, A, s));
  return lu_solve(A, (const double2 *)chi0, n_g, n_w, i_g0, (double2 *)chi00, info, s);
}

int tdx_dyson(tdx_ctx *ctx, const double *chi0, const double *K, int n_g, int n_w, int i_g0,
              double *chi00, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && chi0 && K && chi00, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_g > 0 && n_w > 0 && i_g0 >= 0 && i_g0 < n_g, TDX_ERR_SHAPE, "bad sizes");
  TDX_TRY(check_device(ctx));
  hipStream_t s = as_stream(stream);
  void *w;
  const size_t abytes = tdx_dyson_work_bytes(n_g, n_w);
  TDX_TRY(ws_get(ctx, WS_DYSON, abytes + sizeof(int) * n_w, &w));
  int *info = (int *)((char *)w + abytes);
  TDX_TRY(tdx_dyson_async(ctx, chi0, K, n_g, n_w, i_g0, chi00, w, info, stream));
  std::vector<int> h(n_w);
  TDX_HIP(hipMemcpyAsync(h.data(), info, sizeof(int) * n_w, hipMemcpyDeviceToHost, s));
  TDX_HIP(hipStreamSynchronize(s));
  for (int i = 0; i < n_w; ++i)
    TDX_REQUIRE(h[i] == 0, TDX_ERR_NUMERIC, "Dyson matrix singular at frequency %d (column %d)",
                i, h[i] - 1);
  return TDX_OK;
}

int tdx_dyson_vjp(tdx_ctx *ctx, const double *chi0, const double *K, int n_g, int n_w, int i_g0,
                  const double *chi00_bar, double *u, double *v, void *work, int *info,
                  tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && chi0 && K && chi00_bar && u && v && work && info, TDX_ERR_INVALID_ARG,
              "null argument");
  TDX_REQUIRE(n_g > 0 && n_w > 0 && i_g0 >= 0 && i_g0 < n_g, TDX_ERR_SHAPE, "bad sizes");
  const size_t lds = (sizeof(double2) * 2 + sizeof(int)) * (size_t)n_g;
  TDX_REQUIRE(lds <= 64 * 1024, TDX_ERR_SHAPE, "n_g %d too large for the LU kernel", n_g);
  TDX_REQUIRE(n_w <= 65535, TDX_ERR_SHAPE, "n_w %d above 65535", n_w);
  hipStream_t s = as_stream(stream);
  double2 *A = (double2 *)work;
  TDX_TRY(one_minus((const double2 *)chi0, (const double2 *)K, n_g, n_w, A, s));
  return lu_vjp(A, (const double2 *)chi0, (const double2 *)K, n_g, n_w, i_g0,
                (const double2 *)chi00_bar, (double2 *)u, (double2 *)v, info, nullptr, s);
}

int tdx_dyson_kernel_vjp(tdx_ctx *ctx, const double *chi0, const double *K, int n_g, int n_w,
                         int i_g0, const double *chi00_bar, double *K_bar, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && chi0 && K && chi00_bar && K_bar, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_g > 0 && n_w > 0 && i_g0 >= 0 && i_g0 < n_g, TDX_ERR_SHAPE, "bad sizes");
  const size_t lds = (sizeof(double2) * 2 + sizeof(int)) * (size_t)n_g;
  TDX_REQUIRE(lds <= 64 * 1024, TDX_ERR_SHAPE, "n_g %d too large for the LU kernel", n_g);
  TDX_REQUIRE(n_w <= 65535 && n_g <= 65535, TDX_ERR_SHAPE, "sizes above the grid");
  TDX_TRY(check_device(ctx));
  hipStream_t s = as_stream(stream);
  const size_t mat = sizeof(double2) * (size_t)n_w * n_g * n_g;
  const size_t vec = sizeof(double2) * (size_t)n_w * n_g;
  const size_t ints = (sizeof(int) * ((size_t)n_w + 2) + 255) / 256 * 256;
  void *w;
  TDX_TRY(ws_get(ctx, WS_DYSON, mat + 4 * vec + ints, &w));
  double2 *A = (double2 *)w;
  double2 *u = (double2 *)((char *)w + mat), *v = u + (size_t)n_w * n_g;
  double2 *x = v + (size_t)n_w * n_g, *p = x + (size_t)n_w * n_g;
  int *info = (int *)(p + (size_t)n_w * n_g), *status = info + n_w;
  TDX_TRY(one_minus((const double2 *)chi0, (const double2 *)K, n_g, n_w, A, s));
  TDX_TRY(lu_vjp(A, (const double2 *)chi0, (const double2 *)K, n_g, n_w, i_g0,
                 (const double2 *)chi00_bar, u, v, info, x, s));
  hipLaunchKernelGGL(k_clear_status, dim3(1), dim3(64), 0, s, status);
  hipLaunchKernelGGL(k_fold_status, dim3(1), dim3(256), 0, s, info, n_w, 0, status);
  TDX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_chi0h_u, dim3((n_g + 63) / 64, n_w), dim3(64), 0, s, (const double2 *)chi0,
                     u, n_g, p);
  TDX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_kbar, dim3((n_g + 63) / 64, n_g), dim3(64), 0, s, p, x, n_g, n_w,
                     (double2 *)K_bar);
  TDX_HIP(hipGetLastError());
  int h[2] = {0, 0};
  TDX_HIP(hipMemcpyAsync(h, status, sizeof(h), hipMemcpyDeviceToHost, s));
  TDX_HIP(hipStreamSynchronize(s));
  TDX_REQUIRE(h[0] == INT_MAX, TDX_ERR_NUMERIC,
              "Dyson matrix singular at frequency %d (column %d)", h[0], h[1] - 1);
  return TDX_OK;
}

int tdx_kernel_matrix_vjp(tdx_ctx *ctx, const tdx_states *st, const int *gbasis, int n_g,
                          const int dens_grid[3], const double *K_bar, double *fxc_bar,
                          tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && st && gbasis && K_bar && fxc_bar, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_g > 0 && n_g <= 65535, TDX_ERR_SHAPE, "bad n_g");
  TDX_TRY(check_device(ctx));
  int Nr;
  size_t lds;
  TDX_TRY(check_grid(st, dens_grid, &Nr, &lds));
  hipStream_t s = as_stream(stream);
  const int N0 = dens_grid[0], N1 = dens_grid[1], N2 = dens_grid[2];
  const size_t mat = sizeof(double2) * (size_t)Nr * n_g;
  void *w;
  TDX_TRY(ws_get(ctx, WS_ADJ2, 2 * mat, &w));
  double2 *Phi = (double2 *)w, *T = (double2 *)((char *)w + mat);
  hipLaunchKernelGGL(k_phi, dim3((n_g + 63) / 64, Nr), dim3(64), 0, s, gbasis, n_g, N0, N1, N2,
                     Phi);
  TDX_HIP(hipGetLastError());
  TDX_REQUIRE(rocblas_set_stream(ctx->blas, s) == rocblas_status_success, TDX_ERR_HIP,
              "rocblas_set_stream failed");
  const rocblas_double_complex one(1.0, 0.0), zero(0.0, 0.0);
  // T (column-major n_g x N_r) = Kbar_cm^H Phi_cm, Kbar_cm(b, a) = Kbar[a][b]
  const rocblas_status rs = rocblas_zgemm(
      ctx->blas, rocblas_operation_conjugate_transpose, rocblas_operation_none, n_g, Nr, n_g, &one,
      (const rocblas_double_complex *)K_bar, n_g, (const rocblas_double_complex *)Phi, n_g, &zero,
      (rocblas_double_complex *)T, n_g);
  TDX_REQUIRE(rs == rocblas_status_success, TDX_ERR_HIP, "rocblas_zgemm failed (%d)", (int)rs);
  hipLaunchKernelGGL(k_fbar, dim3((Nr + 255) / 256), dim3(256), 0, s, Phi, T, n_g, Nr, fxc_bar);
  TDX_HIP(hipGetLastError());
  TDX_HIP(hipStreamSynchronize(s));  // the workspace may be reused after return
  return TDX_OK;
}

int tdx_density_vjp(tdx_ctx *ctx, const tdx_states *st, const int dens_grid[3],
                    const double *fxc_bar, double *occ_bar, double *coef_bar,
                    tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && st && fxc_bar && occ_bar, TDX_ERR_INVALID_ARG, "null argument");
  TDX_TRY(check_device(ctx));
  int Nr;
  size_t lds;
  TDX_TRY(check_grid(st, dens_grid, &Nr, &lds));
  TDX_REQUIRE(lds + 256 * sizeof(double) <= 160 * 1024, TDX_ERR_SHAPE,
              "density grid of %d points exceeds LDS", Nr);
  hipStream_t s = as_stream(stream);
  const int N0 = dens_grid[0], N1 = dens_grid[1], N2 = dens_grid[2];
  void *w;
  const int slices = dens_slices(ctx, st->n_k);
  TDX_TRY(ws_get(ctx, WS_DENS, sizeof(double) * ((size_t)st->n_k + 1) * Nr, &w));
  int per_k;
  double *nbar = (double *)w + (size_t)st->n_k * Nr;
  double *dens = dens_partials(ctx, st->n_k, slices, Nr, (double *)w, &per_k);
  TDX_HIP(hipFuncSetAttribute((const void *)k_density, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds));
  TDX_HIP(hipFuncSetAttribute((const void *)k_density_vjp,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(k_density, dim3(st->n_k, per_k), dim3(kDensThreads), lds, s,
                     (const double2 *)st->coef, st->occ, st->nb, st->npw, st->miller, st->nb_max,
                     st->npw_max, N0, N1, N2, slices, dens);
  TDX_HIP(hipGetLastError());
  const double scale = 2.0 / (st->n_k * st->omega_cell);
  hipLaunchKernelGGL(k_nbar, dim3((Nr + 31) / 32), dim3(256), 0, s, dens, st->n_k, per_k, Nr,
                     scale, fxc_bar, nbar);
  TDX_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_density_vjp, dim3(st->n_k, slices), dim3(kDensThreads), lds, s, (const double2 *)st->coef,
                     st->occ, st->nb, st->npw, st->miller, st->nb_max, st->npw_max, N0, N1, N2,
                     scale, nbar, occ_bar, (double2 *)coef_bar);
  TDX_HIP(hipGetLastError());
  TDX_HIP(hipStreamSynchronize(s));  // the density workspace may be reused after return
  return TDX_OK;
}

}  // extern "C"
