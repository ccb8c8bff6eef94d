// chi0_GG'(q,w) = pref * sum_t df_t / (w - delta_t + i eta) rho_t(G) conj(rho_t(G'))
// (for a time-reversal-paired list each kept t carries its partner too, with
// the weight df_t [1/(w - delta_t + i eta) - 1/(w + delta_t + i eta)]).
//
// The entry point and the slice reduction.  The contraction kernels: FP32
// in chi0_fp.hip, FP64 in chi0_fp64.hip (with its slice reduction), split-BF16
// in chi0_bf16x3.hip (with its batches in chi0_batch.hip).  The transition axis is cut into slices whose FP64
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

// Slice length of an FP64 contraction of at most `cap` slices, whose partials
// are the workspace.  A slice is `tiles` workgroup tiles of up to fb blocks of
// 16 frequencies, run `slots` at a time, longest first.
//  - Sums: a term of the pairs' form takes about half the roundings of the
//    complex product's, so that a sum's length and the slices added after it may
//    be 1.75 times those of `cap` equal slices; up to 128 their roundings are
//    fewer than those of the weights.  Errors against extended precision, N_G
//    94, 40 frequencies, 44838 transitions: 1.0 to 2.1e-15 with 69 slices of the
//    complex product, 0.9 to 1.6e-15 here (1.9 to 3.1e-15 with 7, which would
//    take 1.41 ms against 1.50); 144, 40, 1000: 4.0e-16 and 3.9e-16 (6.5e-16 in
//    one slice, 110 us against 150).
//  - Time, where all tiles are alike (nfb a multiple of nft): whole rounds of
//    equal slices leave most of the chip idle in the last, so the last slice
//    may be shorter: its tiles fill the places that the last round of the
//    others leaves empty (N_G 133, 500 frequencies, 50000 transitions, 560
//    tiles on 256 places, three slices: seven rounds of 16672 if equal; two of
//    20016 and one of 9968 take five rounds and one of the short ones, 6 % less,
//    and as long as five equal slices did with 1.7 times the workspace).
//  - Else some tiles hold a block more, the slots fall out of step and end
//    within about half a tile of each other (N_G 32, 200 frequencies, 13
//    blocks as 3 + 3 + 3 + 4).
// A tile's cost is its transitions plus the 64 or so that its start and end
// take, per block (53 ns each), a slice's the writing and reading of its
// partial of `out` values (at 4 TB/s).  The length of least predicted time, the
// longest within 1 % of it.
long long slice_len_fp64(long long tiles, int nft, int nfb, long long slots, long long n_trans,
                         int chunk, long long cap, double out) {
  const int fb = (nfb + nft - 1) / nft;
  const bool alike = nfb % nft == 0;
  const double ends = 64.0;
  auto cost = [&](long long len) {
    const long long ns = (n_trans + len - 1) / len;  // all but the last of `len`
    const double tile = (double)len + ends, rest = (double)(n_trans - (ns - 1) * len) + ends;
    const double partials = 1.5e-4 * (double)ns * out;
    if (!alike)
      return (double)(tiles * nfb) / nft * ((ns - 1) * tile + rest) / slots + 0.6 * fb * tile +
             partials;
    const long long full = (ns - 1) * tiles, rounds = (full + slots - 1) / slots;
    const long long idle = rounds * slots - full;  // places of the long tiles' last round
    const long long left = std::max<long long>(0, tiles - idle * (long long)(tile / rest));
    return fb * (rounds * tile + (double)((left + slots - 1) / slots) * rest) + partials;
  };
  // counts about 3 % apart, the last slice such that `fit` of its tiles run in
  // the time of one of the others
  const double most = std::max(128.0, 1.75 * ((double)n_trans / cap + (double)cap));
  auto each = [&](auto f) {
    for (long long ns = std::max<long long>(1, (long long)(n_trans / most)); ns <= cap;
         ns += 1 + ns / 32)
      for (int fit = 1; fit <= (alike && ns > 1 && ns <= 16 && ns * tiles > slots ? 8 : 1); ++fit) {
        const double len = (n_trans + ends * (1.0 - 1.0 / fit)) / (ns - 1 + 1.0 / fit);
        const long long whole = ((long long)std::ceil(len) + chunk - 1) / chunk * chunk;
        if ((double)(whole - chunk + ns) <= most) f(whole);
      }
  };
  double best = INFINITY;
  each([&](long long len) { best = std::min(best, cost(len)); });
  long long longest = 0;
  each([&](long long len) {
    if (cost(len) <= 1.01 * best) longest = std::max(longest, len);
  });
  return longest;
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
long long chi0_fp64_most_slices(int v, int n_w, int n_g);
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
  long long slice_len;
  if (f64) {
    int nft, npt, per_cu;
    chi0_fp64_tiles(v, n_w, n_g, &nft, &npt, &chunk, &per_cu);
    const long long cap = std::min<long long>(
        std::min<long long>(chi0_fp64_most_slices(tv < n_var ? tv : -1, n_w, n_g),
                            (n_trans + chunk - 1) / chunk), 512);
    slice_len = slice_len_fp64((long long)nft * npt, nft, (n_w + 15) / 16,
                               (long long)per_cu * std::max(ctx->n_cu, 1), n_trans, chunk, cap,
                               (double)out_elems);
  } else {
    int wblock, cols;
    chi0_fp32_shape(v, &wblock, &cols, &chunk);
    const long long base =
        (long long)((n_w + wblock - 1) / wblock) * nblk * ((ld + cols - 1) / cols);
    // enough equal slices to fill the chip
    long long n = std::max<long long>(1, (4096 + base - 1) / base);
    n = std::min<long long>(std::min<long long>(n, (n_trans + chunk - 1) / chunk), 512);
    slice_len = (n_trans + n - 1) / n;
  }
  // a multiple of the chunk (or the context's fixed length)
  if (ctx->slice_len > 0) slice_len = ctx->slice_len;
  slice_len = (slice_len + chunk - 1) / chunk * chunk;
  const long long slices = (n_trans + slice_len - 1) / slice_len;
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
