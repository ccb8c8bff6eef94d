// Constraints-based attenuation of narrow-band fluctuations (Sec. 3,
// Eqs. 3-7, Figs. 3 and 4): a bank of Savitzky-Golay filters applied to S on
// the frequency grid, the scores of the window/degree grid search (AICc, a
// frequency-domain penalty at the fluctuations' frequencies found from the
// spectrum of dS/dw, a curvature penalty), the imaginary-time conditions on
// the residual F_n = F_TDDFT - F_p, and the selection.  All FP64; every
// reduction is a fixed-order tree, so results are bitwise reproducible.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace tdx {
namespace {

constexpr int kSgMaxDeg = 8;
constexpr int kRedThreads = 256;
constexpr int kMaxTargets = 16;

// Fixed-order sums of N values over the block (blockDim.x == kRedThreads):
// within each wave by shuffles, then the four waves in order; every thread
// gets the totals.  Two barriers for all N (a tree in LDS takes ten for each).
template <int N>
__device__ void block_sums(double (&v)[N], double *sh) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
    for (int x = 0; x < N; ++x) v[x] += __shfl_xor(v[x], o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int x = 0; x < N; ++x) sh[4 * x + (threadIdx.x >> 6)] = v[x];
  __syncthreads();
#pragma unroll
  for (int x = 0; x < N; ++x) v[x] = ((sh[4 * x] + sh[4 * x + 1]) + sh[4 * x + 2]) + sh[4 * x + 3];
}

// Output point i of the degree-P filter with w-point windows: the
// least-squares polynomial over the window centred on i (moved inside the
// grid at the edges) evaluated at i, and the weight of S_i in that value
// (diagonal of the smoother).  Coordinates t = (j - c) / a with c the window
// centre and a = max(c, 1) keep the Gram matrix well scaled; it is factored
// by Cholesky, value = u.v and weight = u.u with L u = phi(t_i), L v = rhs.
template <int P>
__device__ void sg_point(const double *S, int n, int w, int i, double *out, double *hii) {
  constexpr int M = P + 1;
  const int h = w / 2;
  const int s = min(max(i - h, 0), n - w);
  const double c = 0.5 * (w - 1), a = fmax(c, 1.0);
  double G[M][M], r[M];
#pragma unroll
  for (int x = 0; x < M; ++x) {
    r[x] = 0.0;
#pragma unroll
    for (int y = 0; y < M; ++y) G[x][y] = 0.0;
  }
  for (int j = 0; j < w; ++j) {
    const double t = (j - c) / a, yj = S[s + j];
    double ph[M];
    ph[0] = 1.0;
#pragma unroll
    for (int x = 1; x < M; ++x) ph[x] = ph[x - 1] * t;
#pragma unroll
    for (int x = 0; x < M; ++x) {
      r[x] += ph[x] * yj;
#pragma unroll
      for (int y = 0; y <= x; ++y) G[x][y] += ph[x] * ph[y];
    }
  }
  // Cholesky G = L L^T in the lower triangle
#pragma unroll
  for (int k = 0; k < M; ++k) {
    double d = G[k][k];
#pragma unroll
    for (int l = 0; l < k; ++l) d -= G[k][l] * G[k][l];
    const double lkk = sqrt(d);
    G[k][k] = lkk;
#pragma unroll
    for (int x = k + 1; x < M; ++x) {
      double e = G[x][k];
#pragma unroll
      for (int l = 0; l < k; ++l) e -= G[x][l] * G[k][l];
      G[x][k] = e / lkk;
    }
  }
  const double ti = (i - s - c) / a;
  double u[M], v[M];
  double p = 1.0;
#pragma unroll
  for (int x = 0; x < M; ++x) {
    double eu = p, ev = r[x];
#pragma unroll
    for (int l = 0; l < x; ++l) {
      eu -= G[x][l] * u[l];
      ev -= G[x][l] * v[l];
    }
    u[x] = eu / G[x][x];
    v[x] = ev / G[x][x];
    p *= ti;
  }
  double val = 0.0, hw = 0.0;
#pragma unroll
  for (int x = 0; x < M; ++x) {
    val += u[x] * v[x];
    hw += u[x] * u[x];
  }
  *out = val;
  *hii = hw;
}

// Windows and degrees of up to 256 filters, passed by value (two copies of
// the host lists on the stream cost more than the filters).
struct SgBank {
  int window[256];
  unsigned char degree[256];
};

// grid (ceil(n / 64), filters): filter f0 + blockIdx.y, point i.
__global__ void __launch_bounds__(64)
    k_sg_filter(const double *S, int n, SgBank bank, int f0, double *Sp, double *hdiag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int f = f0 + blockIdx.y, w = bank.window[blockIdx.y];
  double val = 0.0, hw = 0.0;
  switch (bank.degree[blockIdx.y]) {  // uniform over the block
    case 0: sg_point<0>(S, n, w, i, &val, &hw); break;
    case 1: sg_point<1>(S, n, w, i, &val, &hw); break;
    case 2: sg_point<2>(S, n, w, i, &val, &hw); break;
    case 3: sg_point<3>(S, n, w, i, &val, &hw); break;
    case 4: sg_point<4>(S, n, w, i, &val, &hw); break;
    case 5: sg_point<5>(S, n, w, i, &val, &hw); break;
    case 6: sg_point<6>(S, n, w, i, &val, &hw); break;
    case 7: sg_point<7>(S, n, w, i, &val, &hw); break;
    default: sg_point<8>(S, n, w, i, &val, &hw); break;
  }
  Sp[(size_t)f * n + i] = val;
  if (hdiag) hdiag[(size_t)f * n + i] = hw;
}

// Power of the central-difference derivative D_i = (y_{i+1} - y_{i-1}) /
// (w_{i+1} - w_{i-1}), i = 1..n-2, of N series at frequency nu (cycles per
// unit of w): |(1/(n-2)) sum_i D_i exp(-2 pi i nu w_i)|^2.  Block-wide.
template <int N>
__device__ void deriv_power(const double *const (&y)[N], const double *om, int n, double nu,
                            double *sh, double (&p)[N]) {
  double v[2 * N] = {};
  for (int i = 1 + threadIdx.x; i + 1 < n; i += kRedThreads) {
    double sn, cs;
    sincospi(-2.0 * nu * om[i], &sn, &cs);
    const double dw = om[i + 1] - om[i - 1];
#pragma unroll
    for (int x = 0; x < N; ++x) {
      const double d = (y[x][i + 1] - y[x][i - 1]) / dw;
      v[2 * x] += d * cs;
      v[2 * x + 1] += d * sn;
    }
  }
  block_sums(v, sh);
  const double m = (double)(n - 2);
#pragma unroll
  for (int x = 0; x < N; ++x) p[x] = (v[2 * x] * v[2 * x] + v[2 * x + 1] * v[2 * x + 1]) / (m * m);
}

// one block per (set, nu): psd[set][k]
__global__ void __launch_bounds__(kRedThreads)
    k_deriv_psd(const double *S, const double *om, int n, const double *nu, int n_nu,
                double *psd) {
  __shared__ double sh[16];
  const int k = blockIdx.x, set = blockIdx.y;
  const double *const y[1] = {S + (size_t)set * n};
  double p[1];
  deriv_power(y, om, n, nu[k], sh, p);
  if (threadIdx.x == 0) psd[(size_t)set * n_nu + k] = p[0];
}

// one block per filter: scores[f] = (RSS, k_eff, AICc, P_freq, P_curv)
__global__ void __launch_bounds__(kRedThreads)
    k_sg_scores(const double *S, const double *Sp, const double *hdiag, const double *om, int n,
                const double *nu, int n_nu, double *scores) {
  __shared__ double sh[16];
  const int f = blockIdx.x;
  const double *y = Sp + (size_t)f * n, *hd = hdiag + (size_t)f * n;
  double v[4] = {};  // RSS, sum of the diagonal, curvatures after and before
  for (int i = threadIdx.x; i < n; i += kRedThreads) {
    const double e = y[i] - S[i];
    v[0] += e * e;
    v[1] += hd[i];
    if (i > 0 && i + 1 < n) {
      const double a = y[i + 1] - 2.0 * y[i] + y[i - 1];
      const double b = S[i + 1] - 2.0 * S[i] + S[i - 1];
      v[2] += a * a;
      v[3] += b * b;
    }
  }
  block_sums(v, sh);
  const double *const ys[2] = {y, S};
  double pf = 0.0;
  for (int t = 0; t < n_nu; ++t) {
    double p[2];
    deriv_power(ys, om, n, nu[t], sh, p);
    pf += p[0] / p[1];
  }
  if (threadIdx.x == 0) {
    const double rss = v[0], k = v[1];
    const double dn = (double)n, den = dn - k - 1.0;
    const double aicc = den > 0.0 ? dn * log(rss / dn) + 2.0 * k + 2.0 * k * (k + 1.0) / den
                                  : INFINITY;
    double *o = scores + (size_t)f * 5;
    o[0] = rss;
    o[1] = k;
    o[2] = aicc;
    o[3] = n_nu > 0 ? pf / n_nu : 0.0;
    o[4] = v[3] > 0.0 ? v[2] / v[3] : NAN;
  }
}

// one block per set: out[set] = (max |F_n / F_ref|, Fbar_n / F_ref(beta/2),
// sigma_n / F_ref(beta/2)), F_n = F_ref - F_p[set]; NaN for a grid that does
// not start at 0, end at beta/2 or beta, and hold beta/2.
__global__ void __launch_bounds__(kRedThreads)
    k_residual_itcf(const double *Fr, const double *Fp, const double *tau, int n_tau,
                    double beta, double *out) {
  __shared__ double sh[8];
  __shared__ int mid;  // index of beta/2 (the last one, -1 if none)
  const int set = blockIdx.x;
  const double *fp = Fp + (size_t)set * n_tau;
  const double tol = 1e-12 * beta;
  const double t_end = tau[n_tau - 1];
  const bool half = fabs(t_end - 0.5 * beta) <= tol, full = fabs(t_end - beta) <= tol;
  if (threadIdx.x == 0) mid = -1;
  __syncthreads();
  // integrals over the grid; a grid ending at beta/2 covers half of [0, beta]
  // and F_n(tau) = F_n(beta - tau) for every S, so each doubles
  const double span = half ? 0.5 * beta : beta;
  double a[1] = {}, e = 0.0;
  for (int j = threadIdx.x; j < n_tau; j += kRedThreads) {
    const double d = Fr[j] - fp[j];
    e = fmax(e, fabs(d / Fr[j]));
    if (j + 1 < n_tau) a[0] += 0.5 * (tau[j + 1] - tau[j]) * (d + (Fr[j + 1] - fp[j + 1]));
    if (fabs(tau[j] - 0.5 * beta) <= tol) atomicMax(&mid, j);
  }
  block_sums(a, sh);
  const double mean = a[0] / span;
  double q[1] = {};
  for (int j = threadIdx.x; j + 1 < n_tau; j += kRedThreads) {
    const double d0 = Fr[j] - fp[j] - mean, d1 = Fr[j + 1] - fp[j + 1] - mean;
    q[0] += 0.5 * (tau[j + 1] - tau[j]) * (d0 * d0 + d1 * d1);
  }
  block_sums(q, sh);
  // max over the block (all values are >= 0)
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) e = fmax(e, __shfl_xor(e, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) {
    e = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    const bool ok = n_tau > 1 && tau[0] == 0.0 && (half || full) && mid >= 0;
    const double fm = ok ? Fr[mid] : NAN;
    // root-mean-square deviation over [0, beta]: the integral over the grid
    // is q * beta / span, its mean over [0, beta] q / span
    const double sigma = sqrt(q[0] / span);
    double *o = out + (size_t)set * 3;
    o[0] = ok ? e : NAN;
    o[1] = ok ? mean / fm : NAN;
    o[2] = ok ? sigma / fm : NAN;
  }
}

}  // namespace
}  // namespace tdx

using namespace tdx;

extern "C" {

int tdx_sg_filter(tdx_ctx *ctx, const double *S, int n_w, const int *windows,
                  const int *degrees, int n_filt, double *Sp, double *hdiag, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && S && (n_filt == 0 || (windows && degrees && Sp)), TDX_ERR_INVALID_ARG,
              "null argument");
  TDX_REQUIRE(n_w > 0 && n_filt >= 0, TDX_ERR_SHAPE, "bad sizes");
  for (int f = 0; f < n_filt; ++f) {
    const int w = windows[f], p = degrees[f];
    TDX_REQUIRE(p >= 0 && p <= kSgMaxDeg, TDX_ERR_INVALID_ARG,
                "filter %d: degree %d outside 0..%d", f, p, kSgMaxDeg);
    TDX_REQUIRE(w % 2 == 1 && w > p && w <= n_w, TDX_ERR_INVALID_ARG,
                "filter %d: window %d must be odd, above the degree %d and at most %d", f, w,
                p, n_w);
  }
  TDX_TRY(check_device(ctx));
  if (n_filt == 0) return TDX_OK;
  for (int f0 = 0; f0 < n_filt; f0 += 256) {
    SgBank bank;
    const int nf = std::min(256, n_filt - f0);
    for (int f = 0; f < nf; ++f) {
      bank.window[f] = windows[f0 + f];
      bank.degree[f] = (unsigned char)degrees[f0 + f];
    }
    hipLaunchKernelGGL(k_sg_filter, dim3((n_w + 63) / 64, nf), dim3(64), 0, as_stream(stream), S,
                       n_w, bank, f0, Sp, hdiag);
    TDX_HIP(hipGetLastError());
  }
  TDX_HIP(hipStreamSynchronize(as_stream(stream)));  // as the interface promises
  return TDX_OK;
}

int tdx_derivative_psd(tdx_ctx *ctx, const double *S, const double *omega, int n_w, int n_set,
                       const double *nu, int n_nu, double *psd, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && S && omega && ((n_set == 0 || n_nu == 0) || (nu && psd)),
              TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_w >= 3 && n_set >= 0 && n_nu >= 0, TDX_ERR_SHAPE, "bad sizes");
  TDX_TRY(check_device(ctx));
  if (n_set == 0 || n_nu == 0) return TDX_OK;
  hipLaunchKernelGGL(k_deriv_psd, dim3(n_nu, n_set), dim3(kRedThreads), 0, as_stream(stream), S,
                     omega, n_w, nu, n_nu, psd);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

int tdx_sg_scores(tdx_ctx *ctx, const double *S, const double *Sp, const double *hdiag,
                  const double *omega, int n_w, int n_filt, const double *nu, int n_nu,
                  double *scores, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && S && omega && (nu || n_nu == 0) && (n_filt == 0 || (Sp && hdiag && scores)),
              TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_w >= 3 && n_filt >= 0, TDX_ERR_SHAPE, "bad sizes");
  TDX_REQUIRE(n_nu >= 0 && n_nu <= kMaxTargets, TDX_ERR_SHAPE, "at most %d target frequencies",
              kMaxTargets);
  TDX_TRY(check_device(ctx));
  if (n_filt == 0) return TDX_OK;
  hipLaunchKernelGGL(k_sg_scores, dim3(n_filt), dim3(kRedThreads), 0, as_stream(stream), S, Sp,
                     hdiag, omega, n_w, nu, n_nu, scores);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

int tdx_residual_itcf(tdx_ctx *ctx, const double *F_ref, const double *F_p, int n_set,
                      const double *tau, int n_tau, double beta, double *out,
                      tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && F_ref && tau && (n_set == 0 || (F_p && out)), TDX_ERR_INVALID_ARG,
              "null argument");
  TDX_REQUIRE(n_tau > 1 && n_set >= 0, TDX_ERR_SHAPE, "bad sizes");
  TDX_REQUIRE(std::isfinite(beta) && beta > 0, TDX_ERR_INVALID_ARG, "bad beta");
  TDX_TRY(check_device(ctx));
  if (n_set == 0) return TDX_OK;
  hipLaunchKernelGGL(k_residual_itcf, dim3(n_set), dim3(kRedThreads), 0, as_stream(stream),
                     F_ref, F_p, tau, n_tau, beta, out);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

int tdx_sg_select(const double *scores, const double *resid, int n_filt, int n_w, double lam_f,
                  double lam_c, double mean_tol, double sigma_tol, int *best) {
  clear_error();
  TDX_REQUIRE(best && (scores || n_filt == 0), TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(n_filt >= 0 && n_w > 0, TDX_ERR_SHAPE, "bad sizes");
  TDX_REQUIRE(std::isfinite(lam_f) && lam_f >= 0 && std::isfinite(lam_c) && lam_c >= 0,
              TDX_ERR_INVALID_ARG, "penalty weights must be finite and non-negative");
  int b = -1;
  double jb = INFINITY;
  for (int f = 0; f < n_filt; ++f) {
    const double *o = scores + 5 * (size_t)f;
    const double J = o[2] / n_w + lam_f * o[3] + lam_c * o[4];
    if (!std::isfinite(J)) continue;
    if (resid) {
      const double *r = resid + 3 * (size_t)f;
      if (!(fabs(r[1]) <= mean_tol && r[2] <= sigma_tol)) continue;
    }
    if (J < jb) {
      jb = J;
      b = f;
    }
  }
  *best = b;
  return TDX_OK;
}

}  // extern "C"
