// FP64 chi0 contraction on the 16x16x4 FP64 MFMA of gfx950.
//
// With X_t = rho_t rho_t^H and w_t = wr_t + i wi_t,
//   chi0 = H_R + i H_A,  H_R = sum_t wr_t X_t,  H_A = sum_t wi_t X_t,
// and X_t is Hermitian, so its n_g^2 real numbers (re and im of the pairs
// G <= G') hold all of it.  The contraction is the real product
//   [2 n_w weights] x [t]  times  [t] x [n_g^2 components of X_t]:
// 2 n_w n_g^2 multiply-adds per transition, half of the 4 n_w n_g^2 that the
// complex product (w_t rho_t) rho_t^H takes.
//
// What bounds it: the FP64 MFMA.  A wave holds one block of 16 pairs against
// FB blocks of 16 frequencies: 4 FB accumulators (H_R and H_A, re and im).
//  - X needs no exchange between lanes: lane l of a B operand is transition
//    l/16 of the K-step and pair l%16, so each lane loads its rho(G) and
//    rho(G') (one chunk ahead, L1/L2 hits) and forms re and im of X with four
//    FP64 operations per 4 FB MFMAs of 64 cycles each.
//  - The weights (one division each) are formed once per workgroup and chunk,
//    double-buffered in LDS, and read as (wr, wi) pairs: both A operands of a
//    frequency block in one 16-byte read.
// Two waves per SIMD (one workgroup of eight waves, or two of four) cover each
// other's loads and barriers; FP64 VALU work shares the MFMA's issue time, so
// eight waves, which halve the weights formed per MFMA, come out ahead.
// Chunks are branch-free (the list's last, partial chunk has a body of its
// own): with a bounds check per load the same tiles ran 14 % slower.
//
// N_G 133, 500 frequencies, 50000 paired transitions: 28.0 ms (63.2 TFLOP/s
// on the MFMA, 87 % of what a large dgemm reaches on this card); the complex
// product (w_t rho_t) rho_t^H on the same MFMA took 68.9 ms.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "chi0_tile.h"
#include "internal.h"

namespace tdx {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kChunk64 = 16;  // transitions per chunk of weights
// Transitions in one sum: a longer slice adds the sums of equal runs in its
// partial.  A run's end costs about 30 us (its tile's partial read and
// written, the next loads not yet on their way).  N_G 133, 500 frequencies,
// 50000 transitions in slices of 20016: error against extended precision
// 5.0e-15 in one sum and 27.6 ms, 2.7e-15 and 28.0 in runs of at most 8192,
// 1.6e-15 and 28.1 of 4096, 1.6e-15 and 28.4 of 2048 (the complex product on
// slices of 16667: 6.0e-15, 69 ms).
constexpr int kRun64 = 6144;

// Pair p = 0 .. n (n + 1) / 2 - 1 of the upper triangle, rows first:
// row G starts at G n - G (G - 1) / 2 and holds G' = G .. n - 1.
__device__ inline void pair_of(long long p, int n, int *G, int *Gp) {
  const double b = 2.0 * n + 1.0;
  long long g = (long long)(0.5 * (b - sqrt(b * b - 8.0 * (double)p)));
  auto start = [n](long long x) { return x * n - x * (x - 1) / 2; };
  while (g > 0 && start(g) > p) --g;
  while (start(g + 1) <= p) ++g;
  *G = (int)g;
  *Gp = (int)(g + (p - start(g)));
}

// One tile: 16 FB frequencies from w0, 16 NW pairs from p0, transitions
// [t_lo, t_hi).  part is the slice's block: per frequency n (n + 1) / 2
// values chi0(G, G') of the pairs in order, then the n (n - 1) / 2 values
// chi0(G', G) of the pairs G < G' (pair p's is number p - G - 1).
template <int NW, int FB, bool PAIRED>
__device__ __attribute__((always_inline)) void tile64(
    double2 *lds, const double2 *P, int ld, const double *delta, const double *df, long long t_lo,
    long long t_hi, const double *omega, int n_w, double eta, int n_g, long long n_pairs, int w0,
    long long p0, double2 *part) {
  constexpr int kF = 16 * FB, kThreads = 64 * NW, kWeights = kChunk64 * kF;
  constexpr int kPer = (kWeights + kThreads - 1) / kThreads, kSteps = kChunk64 / 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c16 = lane & 15, kq = lane >> 4;
  const long long p = p0 + 16 * wave + c16;
  int G, Gp;
  pair_of(p < n_pairs ? p : n_pairs - 1, n_g, &G, &Gp);

  // this thread's weights of a chunk: e = tid + kThreads i is frequency
  // e % kF of transition e / kF (those past n_w take the last frequency's:
  // their rows are not stored)
  double om[kPer], wd[kPer], wf[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) om[i] = omega[std::min(w0 + (tid + kThreads * i) % kF, n_w - 1)];
  auto load_w = [&](long long tc, int last) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int r = std::min((tid + kThreads * i) / kF, last);
      wd[i] = (delta + tc)[r];
      wf[i] = (df + tc)[r];
    }
  };
  auto store_w = [&](double2 *buf, int last) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = tid + kThreads * i;
      if (kWeights % kThreads != 0 && e >= kWeights) break;
      double2 v;
      if constexpr (PAIRED) {
        // 2 df delta / D, D = (w - delta)(w + delta) - eta^2 + 2 i w eta
        const double dr = (om[i] - wd[i]) * (om[i] + wd[i]) - eta * eta, di = 2.0 * om[i] * eta;
        const double sc = 2.0 * wf[i] * wd[i] / fma(dr, dr, di * di);
        v = make_double2(sc * dr, -sc * di);
      } else {
        // df / (x + i eta) = df (x - i eta) / (x^2 + eta^2), x = w - delta
        const double x = om[i] - wd[i];
        const double sc = wf[i] / fma(x, x, eta * eta);
        v = make_double2(sc * x, -sc * eta);
      }
      buf[e] = e / kF <= last ? v : make_double2(0.0, 0.0);
    }
  };
  // rho(G) and rho(G') of this lane's transition in each K-step of a chunk,
  // rows past the list clamped to its last one (their weights are zero)
  double2 a[kSteps], b[kSteps];
  const unsigned row = 16u * (unsigned)ld, oa = 16u * (unsigned)G, ob = 16u * (unsigned)Gp;
  auto load_x = [&](int s, const char *chunk, int last) {
    const unsigned r = (unsigned)std::min(4 * s + kq, last) * row;
    a[s] = *(const double2 *)(chunk + (r + oa));
    b[s] = *(const double2 *)(chunk + (r + ob));
  };

  f64x4 acc[FB][4];
  // a run's sums into the slice's partial: the first run's stored, others added
  auto fold = [&](bool first) {
    const size_t per = (size_t)n_g * n_g;
    // this lane's place anew: else it and the addresses stay in registers over
    // the whole run
    unsigned at = threadIdx.x, g16 = oa;
    asm volatile("" : "+v"(at), "+v"(g16));
    const int row0 = w0 + ((at & 63) >> 4), G = (int)(g16 / 16);
    const long long p = p0 + 16 * (at >> 6) + (at & 15);
    const bool twice = ob != oa;  // G < G'
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int w = row0 + 16 * f + 4 * j;  // row l/16 + 4 j of the FP64 MFMA's output
        if (w >= n_w || p >= n_pairs) continue;
        double2 *o = part + (size_t)w * per;
        const double rr = acc[f][0][j], ri = acc[f][1][j], ar = acc[f][2][j], ai = acc[f][3][j];
        double2 x = make_double2(rr - ai, ri + ar), y = make_double2(rr + ai, ar - ri);
        if (!first) {
          const double2 u = o[p];
          x.x += u.x;
          x.y += u.y;
        }
        o[p] = x;
        if (!twice) continue;
        double2 *l = o + (n_pairs + p - G - 1);
        if (!first) {
          const double2 u = *l;
          y.x += u.x;
          y.y += u.y;
        }
        *l = y;
      }
  };

  // one chunk, its weights in buf, with the loads and weights of the next
  // one: NEXT 0 a whole chunk, 1 the list's last, partial one, 2 none
  const char *rows;
  long long t_end;  // of the run
  auto chunk = [&](auto next, const double2 *buf, double2 *nbuf, long long nx, int left) {
    constexpr int NEXT = decltype(next)::value;
    const int last = NEXT == 1 ? left - 1 : kChunk64 - 1;
    if constexpr (NEXT < 2) load_w(nx, last);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const double xr = fma(a[s].x, b[s].x, a[s].y * b[s].y);
      const double xi = fma(a[s].y, b[s].x, -(a[s].x * b[s].y));
      if constexpr (NEXT < 2) load_x(s, rows, last);
#pragma unroll
      for (int f = 0; f < FB; ++f) {
        const double2 w = buf[(4 * s + kq) * kF + 16 * f + c16];
        acc[f][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, xr, acc[f][0], 0, 0, 0);
        acc[f][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, xi, acc[f][1], 0, 0, 0);
        acc[f][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.y, xr, acc[f][2], 0, 0, 0);
        acc[f][3] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.y, xi, acc[f][3], 0, 0, 0);
      }
      if (NEXT < 2 && s == 1) store_w(nbuf, last);
    }
    __syncthreads();
  };
  // equal runs of whole chunks
  const long long runs = (t_hi - t_lo + kRun64 - 1) / kRun64;
  const long long each = ((t_hi - t_lo + runs - 1) / runs + kChunk64 - 1) / kChunk64 * kChunk64;
  for (long long t_run = t_lo; t_run < t_hi; t_run += each) {
    t_end = std::min(t_hi, t_run + each);
    rows = (const char *)P + (size_t)t_run * row;
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[f][x] = f64x4{0.0, 0.0, 0.0, 0.0};
    {
      const int last = (int)std::min<long long>(kChunk64, t_end - t_run) - 1;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) load_x(s, rows, last);
      load_w(t_run, last);
      store_w(lds, last);
    }
    __syncthreads();
    int cur = 0;
    long long tc = t_run;
    for (; tc + 2 * kChunk64 <= t_end; tc += kChunk64, cur ^= 1) {
      rows += (size_t)kChunk64 * row;
      chunk(std::integral_constant<int, 0>{}, lds + cur * kWeights, lds + (cur ^ 1) * kWeights,
            tc + kChunk64, 0);
    }
    if (tc + kChunk64 < t_end) {
      rows += (size_t)kChunk64 * row;
      chunk(std::integral_constant<int, 1>{}, lds + cur * kWeights, lds + (cur ^ 1) * kWeights,
            tc + kChunk64, (int)(t_end - tc - kChunk64));
      cur ^= 1;
    }
    chunk(std::integral_constant<int, 2>{}, lds + cur * kWeights, nullptr, 0, 0);
    fold(t_run == t_lo);
  }
}

template <int NW, int FB, bool PAIRED>
__device__ __attribute__((always_inline)) void tile64_n(
    int fb, double2 *lds, const double2 *P, int ld, const double *delta, const double *df,
    long long t_lo, long long t_hi, const double *omega, int n_w, double eta, int n_g,
    long long n_pairs, int w0, long long p0, double2 *part) {
  if constexpr (FB > 1) {
    if (fb < FB) {
      tile64_n<NW, FB - 1, PAIRED>(fb, lds, P, ld, delta, df, t_lo, t_hi, omega, n_w, eta, n_g,
                                   n_pairs, w0, p0, part);
      return;
    }
  }
  tile64<NW, FB, PAIRED>(lds, P, ld, delta, df, t_lo, t_hi, omega, n_w, eta, n_g, n_pairs, w0, p0,
                         part);
}

// One tile per workgroup; grid (tiles of a slice, slices), logical tile =
// (frequency tile fastest, then pair tile), contiguous ranges of a slice's
// tiles per XCD: the frequency tiles of a pair tile and the neighbouring pair
// tiles read the same rho rows, and a short last slice is spread over all
// XCDs.  The blocks of 16 frequencies are dealt evenly to the nft frequency
// tiles (at most FB each), so a ragged grid leaves no tile nearly empty.
template <int NW, int FB, bool PAIRED>
__global__ void __launch_bounds__(64 * NW, 2)
    k_chi0_fp64(const double2 *P, int ld, const double *delta, const double *df,
                long long n_trans, long long slice_len, const double *omega, int n_w, double eta,
                int n_g, long long n_pairs, int nft, double2 *part) {
  extern __shared__ double2 lds64[];
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int pt = L / nft, sl = blockIdx.y;
  // an XCD hands workgroups to its four shader engines in turn whatever their
  // load: with nft of 2 or 4 the tiles that hold a block more than the others
  // would all land on the same engine (N_G 133, 200 frequencies as 3 + 3 + 3 + 4
  // blocks: 50.3 TFLOP/s), so their place moves with the pair tile (55.7)
  const int ft = (L + (pt >> 1)) % nft;
  const int nfb = (n_w + 15) / 16;
  const int f0 = (int)((long long)nfb * ft / nft), f1 = (int)((long long)nfb * (ft + 1) / nft);
  const long long t_lo = sl * slice_len;
  const long long t_hi = std::min(n_trans, t_lo + slice_len);
  tile64_n<NW, FB, PAIRED>(f1 - f0, lds64, P, ld, delta, df, t_lo, t_hi, omega, n_w, eta, n_g,
                           n_pairs, 16 * f0, (long long)pt * 16 * NW,
                           part + (size_t)sl * n_w * n_g * n_g);
}

// chi0 = pref sum over the slices of both halves of each pair, 256 / LANES pairs
// a block: a lane sums every LANES-th slice in order, then the lanes' sums in a
// fixed tree.  One lane reads whole rows of 256 pairs, which a few slices of a
// large basis want; with many slices there are few pairs, and one lane's chain
// of loads is what they wait for (N_G 48, one frequency, 5000 transitions in
// 156 slices: 87 us, most of it that chain).
template <int LANES>
__global__ void __launch_bounds__(256)
    k_reduce_pairs(const double2 *part, int n_slices, int n_w, int n_g, long long n_pairs,
                   double pref, double2 *out) {
  constexpr int kPairs = 256 / LANES;
  __shared__ double2 sums[LANES > 1 ? 2 : 1][LANES][kPairs];
  const int x = threadIdx.x % kPairs, lane = threadIdx.x / kPairs;
  const long long p = blockIdx.x * (long long)kPairs + x;
  int G = 0, Gp = 0;
  if (p < n_pairs) pair_of(p, n_g, &G, &Gp);
  const size_t per = (size_t)n_g * n_g, slice = per * n_w;
  const bool twice = Gp > G;
  for (int w = blockIdx.y; w < n_w; w += gridDim.y) {
    const double2 *u = part + w * per + p;
    const double2 *l = twice ? part + w * per + n_pairs + p - G - 1 : u;
    double2 s = make_double2(0.0, 0.0), r = make_double2(0.0, 0.0);
    if (p < n_pairs) {
#pragma unroll 4
      for (int i = lane; i < n_slices; i += LANES) {
        const double2 a = u[i * slice], b = l[i * slice];
        s.x += a.x;
        s.y += a.y;
        r.x += b.x;
        r.y += b.y;
      }
    }
    if constexpr (LANES > 1) {
      sums[0][lane][x] = s;
      sums[1][lane][x] = r;
      for (int o = LANES / 2; o >= 1; o /= 2) {
        __syncthreads();
        if (lane >= o) continue;
        s.x += sums[0][lane + o][x].x;
        s.y += sums[0][lane + o][x].y;
        r.x += sums[1][lane + o][x].x;
        r.y += sums[1][lane + o][x].y;
        sums[0][lane][x] = s;
        sums[1][lane][x] = r;
      }
      __syncthreads();
    }
    if (lane > 0 || p >= n_pairs) continue;
    out[w * per + (size_t)G * n_g + Gp] = make_double2(pref * s.x, pref * s.y);
    if (twice) out[w * per + (size_t)Gp * n_g + G] = make_double2(pref * r.x, pref * r.y);
  }
}

// Tile variants: waves per workgroup (16 pairs each), blocks of 16
// frequencies, workgroups per CU (by registers); the frequencies x columns by
// which the variant's slices, and so its workspace, are counted (one of 4096
// such tiles of [w][G][G']).
struct Variant64 {
  int waves, fb, per_cu, slice_w, slice_cols;
  const void *fn[2];  // full list, paired list
};
#define TDX_V64(NW, FB, N, W, C)                                                         \
  Variant64 {                                                                            \
    NW, FB, N, W, C,                                                                     \
    {(const void *)k_chi0_fp64<NW, FB, false>, (const void *)k_chi0_fp64<NW, FB, true>}  \
  }
const Variant64 kVar64[] = {TDX_V64(8, 4, 1, 8, 48), TDX_V64(4, 2, 2, 8, 32),
                            TDX_V64(4, 3, 2, 8, 64), TDX_V64(4, 4, 2, 4, 48),
                            TDX_V64(8, 2, 1, 4, 96)};
#undef TDX_V64

}  // namespace

int chi0_fp64_variant_count() { return (int)(sizeof(kVar64) / sizeof(kVar64[0])); }

// Variant of a basis with no tuned entry: eight waves share a chunk's weights
// (64.3 TFLOP/s at N_G 133 and 192 frequencies, four waves 60.9) unless the
// last tile of 128 pairs would be so empty that tiles of 64 come out ahead
// (N_G 32, 528 pairs: 53.4 against 54.1).
int chi0_fp64_default_variant(int n_g) {
  const long long n_pairs = (long long)n_g * (n_g + 1) / 2;
  const double wide = (double)((n_pairs + 127) / 128 * 128), narrow = (double)((n_pairs + 63) / 64 * 64);
  return wide <= 1.055 * narrow ? 0 : 3;
}

// Most slices of a variant (v < 0: of the default): its partials take what
// 4096 tiles of 16 rows by the variant's columns and frequencies would.
long long chi0_fp64_most_slices(int v, int n_w, int n_g) {
  const Variant64 &V = kVar64[std::max(v, 0)];
  const int nblk = (n_g + 15) / 16;
  const long long tiles = (long long)((n_w + V.slice_w - 1) / V.slice_w) * nblk *
                          ((16 * nblk + V.slice_cols - 1) / V.slice_cols);
  return std::max<long long>(1, (4096 + tiles - 1) / tiles);
}

// Workgroup tiles of one slice (frequency tiles, pair tiles), transitions per
// chunk (slices are multiples of it) and workgroups per CU.
void chi0_fp64_tiles(int v, int n_w, int n_g, int *nft, int *npt, int *chunk, int *per_cu) {
  const Variant64 &V = kVar64[v];
  const long long n_pairs = (long long)n_g * (n_g + 1) / 2;
  *nft = ((n_w + 15) / 16 + V.fb - 1) / V.fb;
  *npt = (int)((n_pairs + 16 * V.waves - 1) / (16 * V.waves));
  *chunk = kChunk64;
  *per_cu = V.per_cu;
}

int chi0_fp64_launch(int v, const void *P, int ld, const double *delta, const double *df,
                     int paired, long long n_trans, long long slice_len, int slices,
                     const double *omega, int n_w, double eta, int n_g, double pref,
                     double2 *part, double2 *out, hipStream_t s) {
  const Variant64 &V = kVar64[v];
  const long long n_pairs = (long long)n_g * (n_g + 1) / 2;
  int nft, npt, chunk, per_cu;
  chi0_fp64_tiles(v, n_w, n_g, &nft, &npt, &chunk, &per_cu);
  TDX_REQUIRE((long long)nft * npt * 64 * V.waves < (1LL << 32), TDX_ERR_SHAPE, "%lld tiles",
              (long long)nft * npt);
  const size_t lds = sizeof(double2) * 2 * kChunk64 * 16 * V.fb;
  const double2 *Pd = (const double2 *)P;
  void *args[] = {(void *)&Pd,        (void *)&ld,    (void *)&delta, (void *)&df,
                  (void *)&n_trans,   (void *)&slice_len, (void *)&omega,
                  (void *)&n_w,       (void *)&eta,   (void *)&n_g,   (void *)&n_pairs,
                  (void *)&nft,       (void *)&part};
  TDX_HIP(hipLaunchKernel(V.fn[paired ? 1 : 0], dim3((unsigned)(nft * npt), (unsigned)slices),
                          dim3(64 * V.waves), args, lds, s));
  const unsigned ny = (unsigned)std::min(n_w, 65535);
  if (slices < 16)
    hipLaunchKernelGGL(k_reduce_pairs<1>, dim3((unsigned)((n_pairs + 255) / 256), ny), dim3(256), 0,
                       s, part, slices, n_w, n_g, n_pairs, pref, out);
  else
    hipLaunchKernelGGL(k_reduce_pairs<8>, dim3((unsigned)((n_pairs + 31) / 32), ny), dim3(256), 0,
                       s, part, slices, n_w, n_g, n_pairs, pref, out);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}

}  // namespace tdx
