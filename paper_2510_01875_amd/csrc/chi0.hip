// chi0_GG'(q,w) = pref * sum_t df_t / (w - delta_t + i eta) rho_t(G) conj(rho_t(G'))
// (for a time-reversal-paired list each kept t carries its partner too, with
// the weight df_t [1/(w - delta_t + i eta) - 1/(w + delta_t + i eta)]).
//
// The entry point and the slice reduction.  The contraction kernels: FP32 and
// FP64 in chi0_fp.hip, split-BF16 in chi0_bf16x3.hip (with its batches in
// chi0_batch.hip).  The transition axis is cut into slices whose FP64
// partials are summed here in a fixed order (no atomics: bitwise
// reproducible).
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace tdx {
namespace {

__global__ void k_reduce_slices(const double2 *part, int n_slices, size_t per_slice, double pref,
                                double2 *out) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < per_slice;
       i += (size_t)gridDim.x * blockDim.x) {
    double re = 0.0, im = 0.0;
    for (int s = 0; s < n_slices; ++s) {
      const double2 v = part[(size_t)s * per_slice + i];
      re += v.x;
      im += v.y;
    }
    out[i] = make_double2(pref * re, pref * im);
  }
}

// Slices of an FP64 contraction: a slice is npt pair tiles times nft frequency
// tiles of about nfb / nft frequency blocks, run `slots` at a time.  Where all
// tiles are alike they run in whole rounds, and a count just past one leaves
// most of the chip idle in the last; where nft does not divide nfb some hold a
// block more, the slots fall out of step and end within about half a tile of
// each other (N_G 32, 200 frequencies, 13 blocks as 3 + 3 + 3 + 4: 42.8 TFLOP/s
// with the slices of equal tiles, 49.5 with these).  A tile's cost is its transitions plus the 64 or
// so that its start and end take, per block.  The count of least predicted
// time, the fewest within 1 % of the best, from 1 to `cap`.
long long slices_fp64(long long npt, int nft, int nfb, long long slots, long long n_trans,
                      int chunk, long long cap) {
  auto cost = [&](long long ns) {
    const double len = (double)(((n_trans + ns - 1) / ns + chunk - 1) / chunk * chunk) + 64.0;
    if (nfb % nft == 0) return (double)((npt * nft * ns + slots - 1) / slots) * len * (nfb / nft);
    return ((double)(npt * nfb * ns) / slots + 0.6 * (nfb / nft + 1)) * len;
  };
  double best = cost(1);
  for (long long ns = 2; ns <= cap; ++ns) best = std::min(best, cost(ns));
  long long ns = 1;
  while (cost(ns) > 1.01 * best) ++ns;
  return ns;
}

}  // namespace

// FP32 path (chi0_fp.hip).
int chi0_fp32_variant_count();
void chi0_fp32_shape(int v, int *wblock, int *cols, int *chunk);
int chi0_fp32_launch(int v, const void *P, int ld, const double *delta, const double *df,
                     int paired, long long n_trans, long long slice_len, int slices,
                     const double *omega, int n_w, double eta, int n_g, double2 *part,
                     hipStream_t s);

// FP64 path (chi0_fp64.hip).
int chi0_fp64_variant_count();
int chi0_fp64_default_variant(int n_g);
void chi0_fp64_tiles(int v, int n_w, int n_g, int *nft, int *npt, int *chunk, int *slots_per_cu);
int chi0_fp64_launch(int v, const void *P, int ld, const double *delta, const double *df,
                     int paired, long long n_trans, long long slice_len, int slices,
                     const double *omega, int n_w, double eta, int n_g, double pref,
                     double2 *part, double2 *out, hipStream_t s);

// Split-BF16 path (chi0_bf16x3.hip).
int chi0_bf16x3(tdx_ctx *ctx, const void *P, int ld, const double *delta, const double *df,
                int paired, long long n_trans, const double *omega, int n_w, double eta, int n_g,
                double pref, double2 *chi0, hipStream_t s);

}  // namespace tdx

using namespace tdx;

extern "C" int tdx_chi0(tdx_ctx *ctx, const tdx_translist *tl, int64_t n_trans, const void *P,
                        int n_g, int prec, const double *omega, int n_w, double eta, double pref,
                        double *chi0, tdx_stream stream) {
  clear_error();
  TDX_REQUIRE(ctx && tl && P && omega && chi0, TDX_ERR_INVALID_ARG, "null argument");
  TDX_REQUIRE(prec >= TDX_PREC_FP64 && prec <= TDX_PREC_BF16X3, TDX_ERR_INVALID_ARG, "bad prec");
  TDX_REQUIRE(n_g > 0 && n_w > 0 && n_trans >= 0 && n_trans <= tl->capacity, TDX_ERR_SHAPE,
              "bad sizes");
  TDX_REQUIRE(std::isfinite(eta) && eta > 0 && std::isfinite(pref), TDX_ERR_INVALID_ARG,
              "bad eta or prefactor");
  TDX_TRY(check_device(ctx));
  hipStream_t s = as_stream(stream);
  const int ld = (n_g + 15) / 16 * 16;
  const size_t out_elems = (size_t)n_w * n_g * n_g;
  if (n_trans == 0) {
    // a reduction over no slices writes zeros (a kernel, not a memset node,
    // so a caller may capture this call)
    const unsigned rb = (unsigned)std::min<size_t>((out_elems + 255) / 256, 8192);
    hipLaunchKernelGGL(k_reduce_slices, dim3(rb), dim3(256), 0, s, (const double2 *)nullptr, 0,
                       out_elems, pref, (double2 *)chi0);
    TDX_HIP(hipGetLastError());
    return TDX_OK;
  }
  if (prec == TDX_PREC_BF16X3)
    return chi0_bf16x3(ctx, P, ld, tl->delta, tl->df, tl->paired, n_trans, omega, n_w, eta, n_g,
                       pref,
                       (double2 *)chi0, s);
  const int nblk = ld / 16;
  const bool f64 = prec == TDX_PREC_FP64;
  const int tv = ctx->tune[prec][std::min(nblk, 63)].variant;
  const int n_var = f64 ? chi0_fp64_variant_count() : chi0_fp32_variant_count();
  const int v = tv >= 0 && tv < n_var ? tv : f64 ? chi0_fp64_default_variant(n_g) : 0;
  int chunk;
  long long slices;
  if (f64) {
    int nft, npt, per_cu;
    chi0_fp64_tiles(v, n_w, n_g, &nft, &npt, &chunk, &per_cu);
    // at most the slices (and so the workspace) that give 4096 tiles of
    // 8 x 16 x 48; without a workspace limit up to 4 times that within 1 GiB
    const long long base = (long long)((n_w + 7) / 8) * nblk * ((ld + 47) / 48);
    long long cap = std::max<long long>(1, (4096 + base - 1) / base);
    if (ctx->limit == 0)
      cap = std::max(cap, std::min<long long>(
                              4 * cap, (long long)(((size_t)1 << 30) / (sizeof(double2) * out_elems))));
    cap = std::min<long long>(std::min<long long>(cap, (n_trans + chunk - 1) / chunk), 512);
    slices = slices_fp64(npt, nft, (n_w + 15) / 16, (long long)per_cu * std::max(ctx->n_cu, 1),
                         n_trans, chunk, cap);
  } else {
    int wblock, cols;
    chi0_fp32_shape(v, &wblock, &cols, &chunk);
    const long long base =
        (long long)((n_w + wblock - 1) / wblock) * nblk * ((ld + cols - 1) / cols);
    // enough slices to fill the chip
    slices = std::max<long long>(1, (4096 + base - 1) / base);
    slices = std::min<long long>(slices, (n_trans + chunk - 1) / chunk);
    slices = std::min<long long>(slices, 512);
  }
  // equal slices, a multiple of the chunk long (or the context's fixed length)
  long long slice_len = (n_trans + slices - 1) / slices;
  if (ctx->slice_len > 0) slice_len = ctx->slice_len;
  slice_len = (slice_len + chunk - 1) / chunk * chunk;
  slices = (n_trans + slice_len - 1) / slice_len;
  TDX_REQUIRE(slices <= 65535, TDX_ERR_SHAPE, "%lld slices exceed the grid (slice length %lld)",
              slices, slice_len);
  void *w;
  TDX_TRY(ws_get(ctx, WS_PARTIAL, sizeof(double2) * out_elems * slices, &w));
  double2 *part = (double2 *)w;
  if (f64)
    return chi0_fp64_launch(v, P, ld, tl->delta, tl->df, (int)tl->paired, (long long)n_trans,
                            slice_len, (int)slices, omega, n_w, eta, n_g, pref, part,
                            (double2 *)chi0, s);
  TDX_TRY(chi0_fp32_launch(v, P, ld, tl->delta, tl->df, (int)tl->paired, (long long)n_trans,
                           slice_len, (int)slices, omega, n_w, eta, n_g, part, s));
  TDX_HIP(hipGetLastError());
  const unsigned rb = (unsigned)std::min<size_t>((out_elems + 255) / 256, 8192);
  hipLaunchKernelGGL(k_reduce_slices, dim3(rb), dim3(256), 0, s, part, (int)slices, out_elems,
                     pref, (double2 *)chi0);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}
