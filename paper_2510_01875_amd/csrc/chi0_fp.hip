// FP32 chi0 contraction on the 16x16x4 FP32 MFMA of gfx950 (the FP64 form
// has a kernel of its own, chi0_fp64.hip).
//
// The complex contraction is one real GEMM as in the split-BF16 tile: one
// K-step of 4 covers 2 transitions with (re, im) interleaved.  With
// a = w_t(w) rho_t(G) and b = rho_t(G'):
//   A[G][2t + p]   = (Re a, Im a),   A_rot[G][2t + p] = (Im a, -Re a),
//   B[2t + p][G']  = (Re b, Im b),
// A B accumulates Re chi0 and A_rot B accumulates Im chi0 in FP32.  The
// accumulators are folded into the tile's FP64 partial every 128 chunks;
// slices are reduced in FP64 in a fixed order (bitwise reproducible).  The
// weights are taken in FP32 (w - delta in FP64 first).
//
// Lane l of an MFMA holds A[l%16][l/16] and B[l/16][l%16]: transition
// 2s + (l/16)/2, component (l/16)%2.  A is formed in registers from the rho
// row and the weight, once per K-step and frequency, and reused over every
// column block of the tile; an MFMA of this shape runs long enough that the
// formation costs nothing.  The pair-density rows ([T][ld] complex, no
// padding) are copied into LDS by global-to-LDS transfers of 16 bytes per
// lane: per chunk the tile's 16 rows (for A) and its 16 NSUB columns (for B)
// of CHUNK transitions, double-buffered; rows past the end of the list are
// clamped to the last one (their weights are zero).
#include <algorithm>
#include <cmath>

#include "chi0_tile.h"
#include "internal.h"

namespace tdx {
namespace {

template <int WPW, int SUB, int CHUNK>
struct CfgFp {
  static constexpr int kThreads = 256;
  static constexpr int kWBlock = 4 * WPW;           // frequencies per workgroup
  static constexpr int kSub = SUB;
  static constexpr int kCols = 16 * SUB;            // G' per tile
  static constexpr int kChunk = CHUNK;
  static constexpr int kSteps = CHUNK / 2;          // K-steps of two transitions
  static constexpr int kBWords = CHUNK * kCols * 2;  // [t][16 NSUB] complex
  static constexpr int kRhoWords = CHUNK * 16 * 2;   // [t][16] complex
  static constexpr int kWtWords = CHUNK * kWBlock * 2;
  static constexpr int kBufWords = kBWords + kRhoWords + kWtWords;
  static constexpr bool kWPart = CHUNK * kWBlock < 256;
  static constexpr int kNW = kWPart ? 1 : CHUNK * kWBlock / 256;
  static_assert(256 % kWBlock == 0 && CHUNK % 16 == 0, "tile must divide the block");
};

constexpr int kFpFoldChunks = 128;  // chunks summed in FP32 between folds

// LDS transfers of one chunk: the B rows (CHUNK x 16 NSUB complex, row
// stride 16 NSUB) and the rho rows (CHUNK x 16), in 1 KB pieces dealt to the
// waves in turn.  Lane l of piece j copies LDS bytes 1024 j + 16 l; its
// source row and byte within the row are fixed per slot.
template <class C, int NSUB>
struct DmaPlanFp {
  static constexpr int kRowB = 16 * NSUB * 8, kRowR = 16 * 8;  // bytes per row
  static constexpr int kB = C::kChunk * kRowB / 1024, kR = C::kChunk * kRowR / 1024;
  static constexpr int kT = kB + kR, kSlots = (kT + 3) / 4;
  int row[kSlots];       // row of the chunk the lane copies from
  unsigned col[kSlots];  // byte offset within that row (from col0 or row0)
  int dst[kSlots];       // word offset in a buffer
  bool is_r[kSlots], ok[kSlots];

  __device__ inline DmaPlanFp(int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      const int x = 4 * i + wave;  // uniform across the wave
      ok[i] = x < kT;
      is_r[i] = x >= kB;
      const int j = is_r[i] ? std::min(x, kT - 1) - kB : x;
      const int o = 1024 * j + 16 * lane;
      const int rb = is_r[i] ? kRowR : kRowB;
      row[i] = o / rb;
      col[i] = (unsigned)(o % rb);
      dst[i] = (is_r[i] ? C::kBWords : 0) + 256 * j;
    }
  }

  __device__ inline void issue(const unsigned char *P, int ld, int col0, int row0, long long tc,
                               long long t_max, unsigned int *buf) const {
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      if (!ok[i]) continue;  // uniform across the wave
      const long long t = std::min(tc + row[i], t_max);
      const unsigned char *src =
          P + ((size_t)t * ld + (is_r[i] ? row0 : col0)) * 8 + col[i];
      dma16(src, buf + dst[i]);
    }
  }
};

// One tile: rows row0..row0+15, columns col0..col0+16 NSUB-1, frequencies
// w0..w0+kWBlock-1, transitions [t_lo, t_hi).
template <int WPW, int SUB, int CHUNK, int NSUB>
__device__ __attribute__((always_inline)) void chi0_tile_fp(
    unsigned int *lds, const void *P, int ld, const double *delta, const double *df, int paired,
    long long n_trans, long long t_lo, long long t_hi, const double *omega, int n_w, double eta,
    int n_g, int w0, int row0, int col0, double2 *part) {
  typedef CfgFp<WPW, SUB, CHUNK> C;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tau = lane >> 5, comp = (lane >> 4) & 1, c16 = lane & 15;

  f32x4 ar[WPW][NSUB], ai[WPW][NSUB];
#pragma unroll
  for (int i = 0; i < WPW; ++i)
#pragma unroll
    for (int b = 0; b < NSUB; ++b) {
      ar[i][b] = f32x4{0, 0, 0, 0};
      ai[i][b] = f32x4{0, 0, 0, 0};
    }

  const unsigned char *Pb = (const unsigned char *)P;
  const long long t_max = n_trans - 1;
  const DmaPlanFp<C, NSUB> dma(wave, lane);
  Weights<C> pw;
  const int wi = w0 + tid % C::kWBlock;
  const bool w_ok = wi < n_w;
  const double om = omega[std::min(wi, n_w - 1)];
  auto store = [&](unsigned int *buf, long long tc) {
    unsigned int *w = buf + C::kBWords + C::kRhoWords;
    store_weights<C>(pw, (float2 *)w, om, w_ok, eta, paired, tid, tc, t_hi);
  };
  dma.issue(Pb, ld, col0, row0, t_lo, t_max, lds);
  load_weights<C>(pw, delta, df, t_lo, t_max, tid);
  store(lds, t_lo);
  wait_vm();
  __syncthreads();
  int cur = 0;
  bool first = true;
  constexpr long long kRun = (long long)kFpFoldChunks * CHUNK;
  for (long long rs = t_lo; rs < t_hi; rs += kRun) {
    const long long re = std::min(t_hi, rs + kRun);
    for (long long tc = rs; tc < re; tc += CHUNK) {
      const long long nx = tc + CHUNK;
      const bool more = nx < t_hi;
      if (more) {
        load_weights<C>(pw, delta, df, nx, t_max, tid);
        dma.issue(Pb, ld, col0, row0, nx, t_max, lds + (cur ^ 1) * C::kBufWords);
      }
      const unsigned int *buf = lds + cur * C::kBufWords;
      const float *bq = (const float *)buf;
      const float2 *rq = (const float2 *)(buf + C::kBWords);
      const float2 *wt = (const float2 *)(buf + C::kBWords + C::kRhoWords);
#pragma unroll 2
      for (int s = 0; s < C::kSteps; ++s) {
        const int tl = 2 * s + tau;
        const float2 rho = rq[tl * 16 + c16];
        float a[WPW], r[WPW];
#pragma unroll
        for (int i = 0; i < WPW; ++i) {
          const float2 w = wt[wt_index<C>(tl, wave * WPW + i)];
          const float are = w.x * rho.x - w.y * rho.y;
          const float aim = w.x * rho.y + w.y * rho.x;
          a[i] = comp ? aim : are;
          r[i] = comp ? -are : aim;
        }
#pragma unroll
        for (int b = 0; b < NSUB; ++b) {
          const float bv = bq[(tl * 16 * NSUB + b * 16 + c16) * 2 + comp];
#pragma unroll
          for (int i = 0; i < WPW; ++i) {
            ar[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], bv, ar[i][b], 0, 0, 0);
            ai[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[i], bv, ai[i][b], 0, 0, 0);
          }
        }
      }
      if (more) store(lds + (cur ^ 1) * C::kBufWords, nx);
      wait_vm();
      __syncthreads();
      cur ^= 1;
    }
    fold<WPW, NSUB>(ar, ai, part, n_w, n_g, w0, row0, col0, lane, wave, first);
    first = false;
  }
}

template <int WPW, int SUB, int CHUNK, int NSUB = SUB>
__device__ __attribute__((always_inline)) void chi0_tile_fp_n(
    int nsub, unsigned int *lds, const void *P, int ld, const double *delta, const double *df,
    int paired, long long n_trans, long long t_lo, long long t_hi, const double *omega, int n_w,
    double eta, int n_g, int w0, int row0, int col0, double2 *part) {
  if constexpr (NSUB > 1) {
    if (nsub < NSUB) {
      chi0_tile_fp_n<WPW, SUB, CHUNK, NSUB - 1>(nsub, lds, P, ld, delta, df, paired, n_trans,
                                                    t_lo, t_hi, omega, n_w, eta, n_g, w0, row0,
                                                    col0, part);
      return;
    }
  }
  chi0_tile_fp<WPW, SUB, CHUNK, NSUB>(lds, P, ld, delta, df, paired, n_trans, t_lo, t_hi,
                                         omega, n_w, eta, n_g, w0, row0, col0, part);
}

// One tile per workgroup; logical tile = (frequency block fastest, then
// (G block, G' block), then slice), XCD-aware as in the split-BF16 grid.
template <int WPW, int SUB, int CHUNK>
__global__ void __launch_bounds__(256, 2)
    k_chi0_fp(const void *P, int ld, const double *delta, const double *df, int paired,
              long long n_trans, long long slice_len, const double *omega, int n_w, double eta,
              int n_g, int ncb, double2 *part) {
  typedef CfgFp<WPW, SUB, CHUNK> C;
  extern __shared__ unsigned int lds[];
  const int nx = gridDim.x, ny = gridDim.y;
  const int id = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
  const int L = xcd_logical(id, nx * ny * gridDim.z);
  const int bx = L % nx, by = (L / nx) % ny, bz = L / (nx * ny);
  const int gb = by / ncb, gc = by % ncb;
  const long long t_lo = (long long)bz * slice_len;
  const long long t_hi = std::min(n_trans, t_lo + slice_len);
  const int col0 = gc * C::kCols;
  chi0_tile_fp_n<WPW, SUB, CHUNK>(std::min(SUB, (ld - col0) / 16), lds, P, ld, delta, df,
                                     paired, n_trans, t_lo, t_hi, omega, n_w, eta, n_g,
                                     bx * C::kWBlock, gb * 16, col0,
                                     part + (size_t)bz * n_w * n_g * n_g);
}

template <int WPW, int SUB, int CHUNK>
int launch_fp(const void *P, int ld, const double *delta, const double *df, int paired,
              long long n_trans, long long slice_len, int slices, const double *omega, int n_w,
              double eta, int n_g, double2 *part, hipStream_t s) {
  typedef CfgFp<WPW, SUB, CHUNK> C;
  const void *fn = (const void *)k_chi0_fp<WPW, SUB, CHUNK>;
  const size_t lds = (size_t)2 * C::kBufWords * 4;
  const int nblk = ld / 16, ncb = (ld + C::kCols - 1) / C::kCols;
  dim3 grid((n_w + C::kWBlock - 1) / C::kWBlock, nblk * ncb, (unsigned)slices);
  TDX_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL((k_chi0_fp<WPW, SUB, CHUNK>), grid, dim3(256), lds, s, P, ld, delta, df,
                     paired, n_trans, slice_len, omega, n_w, eta, n_g, ncb, part);
  TDX_HIP(hipGetLastError());
  return TDX_OK;
}


// ------------------------------------------------- all columns in one tile
// Bases of 17 to 29 and of 33 to 144 vectors, on lists long enough for them
// (rows_pay).  The rows (w, G) of w_t(w) rho_t(G) are one list
// of n_w n_g, dealt to the waves in tiles of 16 whatever frequencies these
// hold, against all columns G': no row is padding, one set of rho rows in LDS
// (contiguous in memory) serves rows and columns, and a tile of A is formed
// once for all columns.  The bound is the FP32 MFMA, with which the other
// vector instructions share the issue (they add to its time, whether or not
// they are placed between MFMAs): the K-steps of a chunk are unrolled so that
// LDS addresses cost none (not for 32 columns, whose six row tiles would
// spill).  The sums run over the same transitions in the same order as in the
// tiles above, so the results are bitwise those.  N_G 116, 500 frequencies,
// 100000 paired transitions: 55.9 to 44.8 ms (120 TFLOP/s without the padding
// of the columns, 133 with it; a large sgemm reaches 151); N_G 60, 200
// frequencies: 87 to 118 TFLOP/s; N_G 20, 300 frequencies: 40 to 65.  More
// columns leave a wave too few accumulators per row tile, and their padding
// is small.
constexpr int kFlatChunk = 32;
constexpr long long kRun = 4096;  // transitions summed in FP32 between folds

// Frequencies that 64 R rows (w, G), w n_g + G, of a workgroup touch, at most
// (n_g > 16 (NSUB - 1)).
template <int R, int NSUB>
constexpr int flat_freqs() {
  return (64 * R - 1) / (16 * (NSUB - 1) + 1) + 2;
}

template <int R, int NSUB, bool PAIRED>
__global__ void __launch_bounds__(256, 2)
    k_chi0_fp_rows(const void *P, const double *delta, const double *df, long long n_trans,
                   long long slice_len, const double *omega, int n_w, double eta, int n_g,
                   double2 *part) {
  constexpr int kF = flat_freqs<R, NSUB>(), kLd = 16 * NSUB, kSteps = kFlatChunk / 2;
  constexpr int kPer = (kF * kFlatChunk + 255) / 256, kBytes = kFlatChunk * kLd * 8;
  constexpr int kUnroll = NSUB > 2 ? kSteps : 2;
  extern __shared__ float2 flat_lds[];  // two chunks of rows, two of weights
  float2 *wts = flat_lds + 2 * kFlatChunk * kLd;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tau = lane >> 5, comp = (lane >> 4) & 1, c16 = lane & 15;
  const int L = xcd_logical(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const long long rows = (long long)n_w * n_g, row0 = (long long)(L % gridDim.x) * 64 * R;
  const int sl = L / gridDim.x;
  const long long t_lo = sl * slice_len, t_hi = std::min(n_trans, t_lo + slice_len);
  part += (size_t)sl * rows * n_g;
  const int wf = (int)(row0 / n_g);
  // this lane's row of each tile: its vector and its frequency's place
  int g[R], f[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const long long x = std::min(row0 + 16 * (wave * R + i) + c16, rows - 1);
    f[i] = (int)(x / n_g) - wf;
    g[i] = (int)(x % n_g);
  }
  // this thread's weights of a chunk: number e = tid + 256 i is frequency
  // e % kF of transition e / kF
  const double e2 = eta * eta;
  const float etaf = (float)eta;
  double om[kPer], wd[kPer], wv[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) om[i] = omega[std::min(wf + (tid + 256 * i) % kF, n_w - 1)];
  auto load_w = [&](long long tc) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const long long t = std::min(tc + std::min((tid + 256 * i) / kF, kFlatChunk - 1), n_trans - 1);
      wd[i] = delta[t];
      wv[i] = df[t];
    }
  };
  // the arithmetic of store_weights (chi0_tile.h)
  auto store_w = [&](float2 *w, long long tc) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = tid + 256 * i;
      if (e >= kF * kFlatChunk) break;
      float2 v;
      if constexpr (PAIRED) {
        const float dr = (float)fma(om[i] - wd[i], om[i] + wd[i], -e2);
        const float di = (float)(2.0 * om[i] * eta);
        const float sc =
            (float)(2.0 * wv[i] * wd[i]) * __builtin_amdgcn_rcpf(fmaf(dr, dr, di * di));
        v = make_float2(sc * dr, -sc * di);
      } else {
        const float x = (float)(om[i] - wd[i]);
        const float sc = (float)wv[i] * __builtin_amdgcn_rcpf(fmaf(x, x, etaf * etaf));
        v = make_float2(sc * x, -sc * etaf);
      }
      w[e] = tc + e / kF < t_hi ? v : make_float2(0.f, 0.f);
    }
  };
  // a chunk's rows are contiguous: 1 KB pieces dealt to the waves in turn.
  // Past the list the last row again, each vector in its own column: the
  // weights there are zero, and a value that is not finite spoils the sums of
  // its own row and column of chi0 only.
  const char *Pb = (const char *)P;
  auto copy = [&](float2 *dst, long long tc) {
    const char *src = Pb + tc * kLd * 8;
    const bool whole = tc + kFlatChunk <= n_trans;  // uniform
    const int last = (int)std::min<long long>(n_trans - tc, kFlatChunk) - 1;
#pragma unroll
    for (int i = 0; i < kBytes / 4096; ++i) {
      const int o = 4096 * i + 1024 * wave;
      int at = o + 16 * lane;
      if (!whole) at = std::min(at / (kLd * 8), last) * kLd * 8 + at % (kLd * 8);
      dma16(src + at, (unsigned int *)((char *)dst + o));
    }
  };
  f32x4 ar[R][NSUB], ai[R][NSUB];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int b = 0; b < NSUB; ++b) ar[i][b] = ai[i][b] = f32x4{0, 0, 0, 0};
  copy(flat_lds, t_lo);
  load_w(t_lo);
  store_w(wts, t_lo);
  wait_vm();
  __syncthreads();
  int cur = 0;
  bool first = true;
  for (long long rs = t_lo; rs < t_hi; rs += kRun) {
    const long long re = std::min(t_hi, rs + kRun);
    for (long long tc = rs; tc < re; tc += kFlatChunk) {
      const long long nx = tc + kFlatChunk;
      const bool more = nx < t_hi;
      if (more) {
        load_w(nx);
        copy(flat_lds + (cur ^ 1) * kFlatChunk * kLd, nx);
      }
      // K-step s: this lane's transition 2 s + tau
      const float2 *rq = flat_lds + cur * kFlatChunk * kLd + tau * kLd;
      const float2 *wq = wts + cur * kFlatChunk * kF + tau * kF;
      const float *bq = (const float *)rq + 2 * c16 + comp;
      float2 rho[R], w[R];
      float bv[NSUB];
      auto read = [&](int s) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
          rho[i] = rq[2 * s * kLd + g[i]];
          w[i] = wq[2 * s * kF + f[i]];
        }
#pragma unroll
        for (int b = 0; b < NSUB; ++b) bv[b] = bq[4 * s * kLd + 32 * b];
      };
      read(0);
#pragma unroll kUnroll
      for (int s = 0; s < kSteps; ++s) {
        // a = w rho: its component `comp` for Re chi0, and (Im a, -Re a)'s
        float a[R], q[R], x[NSUB];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const float u = comp ? rho[i].y : rho[i].x, v = comp ? -rho[i].x : rho[i].y;
          a[i] = fmaf(w[i].x, u, -(w[i].y * v));
          q[i] = fmaf(w[i].x, v, w[i].y * u);
        }
#pragma unroll
        for (int b = 0; b < NSUB; ++b) x[b] = bv[b];
        read((s + 1) % kSteps);
#pragma unroll
        for (int b = 0; b < NSUB; ++b)
#pragma unroll
          for (int i = 0; i < R; ++i) {
            ar[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], x[b], ar[i][b], 0, 0, 0);
            ai[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[i], x[b], ai[i][b], 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) store_w(wts + (cur ^ 1) * kFlatChunk * kF, nx);
      wait_vm();
      __syncthreads();
      cur ^= 1;
    }
    // into the slice's FP64 partial, [w][G][G'] = [row][G'] (element j of a
    // lane is row 4 (lane / 16) + j, column lane % 16)
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int b = 0; b < NSUB; ++b) {
        const int col = 16 * b + c16;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const long long row = row0 + 16 * (wave * R + i) + 4 * (lane >> 4) + j;
          if (row < rows && col < n_g) {
            double2 *d = part + row * n_g + col;
            double2 v = make_double2((double)ar[i][b][j], (double)ai[i][b][j]);
            if (!first) {
              const double2 o = *d;
              v.x += o.x;
              v.y += o.y;
            }
            *d = v;
          }
        }
        ar[i][b] = ai[i][b] = f32x4{0, 0, 0, 0};
      }
    first = false;
  }
}

template <int R, int NSUB>
int launch_rows(const void *P, const double *delta, const double *df, int paired,
                long long n_trans, long long slice_len, int slices, const double *omega, int n_w,
                double eta, int n_g, double2 *part, hipStream_t s) {
  const void *fn = paired ? (const void *)k_chi0_fp_rows<R, NSUB, true>
                          : (const void *)k_chi0_fp_rows<R, NSUB, false>;
  const size_t lds = 2 * sizeof(float2) * kFlatChunk * (16 * NSUB + flat_freqs<R, NSUB>());
  const long long tiles = ((long long)n_w * n_g + 64 * R - 1) / (64 * R);
  TDX_REQUIRE(tiles * slices < (1LL << 31), TDX_ERR_SHAPE, "too many tiles");
  TDX_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  void *args[] = {(void *)&P,     (void *)&delta, (void *)&df,  (void *)&n_trans, (void *)&slice_len,
                  (void *)&omega, (void *)&n_w,   (void *)&eta, (void *)&n_g,     (void *)&part};
  TDX_HIP(hipLaunchKernel(fn, dim3((unsigned)tiles, (unsigned)slices), dim3(256), args, lds, s));
  return TDX_OK;
}

// Tile variants: (frequencies per wave, column blocks, transitions per
// chunk); variant 0 is the default.
struct FpVariant {
  int wpw, sub, chunk;
  int (*launch)(const void *, int, const double *, const double *, int, long long, long long,
                int, const double *, int, double, int, double2 *, hipStream_t);
};

#define TDX_FPV(W, S, K) FpVariant{W, S, K, launch_fp<W, S, K>}
const FpVariant kVarF32[] = {TDX_FPV(4, 3, 32), TDX_FPV(4, 2, 32), TDX_FPV(4, 4, 32),
                             TDX_FPV(2, 3, 32), TDX_FPV(2, 6, 32)};
#undef TDX_FPV

}  // namespace

int chi0_fp32_variant_count() { return (int)(sizeof(kVarF32) / sizeof(kVarF32[0])); }

// Tile shape of variant v: frequencies and G' columns per workgroup,
// transitions per chunk (slices are multiples of it).
void chi0_fp32_shape(int v, int *wblock, int *cols, int *chunk) {
  const FpVariant &V = kVarF32[v];
  *wblock = 4 * V.wpw;
  *cols = 16 * V.sub;
  *chunk = V.chunk;
}

// Whether the tiles that hold all columns come out ahead of the variant's.  They
// do at 4, 6 and 7 column blocks.  Those of 2, 3, 5 and 9 spill around the run of
// a list, and at 2, 8 and 9 a workgroup's share is larger than the variant's, so
// that a list of few slices leaves CUs idle: steps pay that back, by the list's
// length or by that times the frequencies.
// Either side of the lines, all-column tiles over the variant's, mean over the
// bases: 2 columns 1.18 (80 frequencies, 700 transitions) and 0.90 (130, 1000);
// 3: 1.04 (20, 700) and 0.93 (40, 1000); 5: 1.07 (80, 100) and 0.95 (20, 700);
// 8: 1.04 (20, 100) and 0.93 (20, 300); 9: 1.13 (20, 100) and 0.82 (20, 300).
// 30 to 32 vectors have hardly any padding to save (N_G 32, 700 frequencies,
// 2000 transitions: 240 us, 231 in the tiles of the variant).
bool rows_pay(int n_g, int n_w, long long n_trans) {
  const long long work = n_trans * n_w;
  switch ((n_g + 15) / 16) {
    case 2: return n_g <= 29 && (n_trans >= 5000 || work >= 100000);
    case 3: return n_trans >= 5000 || work >= 40000;
    case 5: return n_trans >= 1000 || work >= 13000;
    case 8: return n_trans >= 700 || work >= 4000;
    case 9: return n_trans >= 300;
  }
  return true;
}

// The launch of a basis of 17 to 144 vectors does not depend on the variant
// where rows_pay; the variant still sets the slices (and so the order of the
// sums).
int chi0_fp32_launch(int v, const void *P, int ld, const double *delta, const double *df,
                     int paired, long long n_trans, long long slice_len, int slices,
                     const double *omega, int n_w, double eta, int n_g, double2 *part,
                     hipStream_t s) {
  switch (rows_pay(n_g, n_w, n_trans) ? ld / 16 : 0) {
#define TDX_ROWS(N, R)                                                                         \
  case N:                                                                                      \
    return launch_rows<R, N>(P, delta, df, paired, n_trans, slice_len, slices, omega, n_w, eta, \
                             n_g, part, s);
    TDX_ROWS(2, 6)
    TDX_ROWS(3, 4)
    TDX_ROWS(4, 3)
    TDX_ROWS(5, 3)
    TDX_ROWS(6, 2)
    TDX_ROWS(7, 2)
    TDX_ROWS(8, 2)
    TDX_ROWS(9, 2)
#undef TDX_ROWS
  }
  return kVarF32[v].launch(P, ld, delta, df, paired, n_trans, slice_len, slices, omega, n_w, eta,
                           n_g, part, s);
}

}  // namespace tdx
