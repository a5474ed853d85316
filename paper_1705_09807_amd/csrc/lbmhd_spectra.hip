// Energy spectra: the radially binned kinetic and magnetic energies compared in
// Sec. 4 of Flint & Vahala, arXiv 1705.09807.
//
// Two complex fields per state, z_u = u_x + i u_y and z_B = B_x + i B_y: over a
// bin that contains -k with every k, sum |Z(k)|^2 equals sum |A(k)|^2 + |B(k)|^2
// of the real fields' transforms.  Row transforms, then column transforms that
// bin |Z|^2 / n^4; all FP64, all sums in a fixed order.
//
// A transform of n = 2^LOGN points is held in registers, E = 16 points per thread
// (4 up to n = 128; Stockham form, radix E with one smaller pass at the end): in
// every pass thread t of T = n / E has the points t + T m, m < E, does its
// butterflies and exchanges the results through LDS, real parts first, then
// imaginary parts, so up to n = 16384 fit one workgroup.  Both the first read and
// the last write are in natural order and coalesced.  An LDS index i is padded
// to i + i / 16, which spreads every pass's stride over the banks.  Twiddles:
// w^m = w^(64 (m / 64)) w^(m % 64) from two tables in LDS, filled with sincospi
// by each workgroup.
//
// Bound by HBM: mom read once, the row transforms written and read once.  A
// column workgroup takes C adjacent columns at a time (C n = 8192); its neighbours
// take the rest of their cache lines at the same time.  Measured at 4096^2: radix-2 passes in LDS with a sincospi
// per butterfly and one thread adding up a column 702 (rows), 1988 (columns) and
// 134 us (final sum); this form 258, 433 and 19 us.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lbmhd_cell.h"
#include "lbmhd_internal.h"

namespace lbm {

template <int LOGN>
struct Fft {
  static constexpr int N = 1 << LOGN;
  // radix 4 where few transforms fill the chip (n = 128, diagnostics, moments and spectra:
  // 71 us a call against 76)
  static constexpr int LOGE = N <= 128 ? 2 : 4;
  static constexpr int E = 1 << LOGE;         // points per thread, the radix of the passes
  static constexpr int T = N / E;             // threads per transform
  // transforms per workgroup: 512 threads where n allows, few on small grids, whose
  // workgroups else leave most of the chip idle
  static constexpr int C = N >= 16384 ? 1 : (N >= 1024 ? 8192 / N : 4);
  static constexpr int ACTIVE = C * T;                          // threads that hold points
  static constexpr int THREADS = ACTIVE < 256 ? 256 : ACTIVE;   // the others fill tables and bins
  static constexpr int WAVES = THREADS >= 512 ? 4 : 1;  // per SIMD: two workgroups of 512 on a compute unit
  // Column pass: a workgroup takes ROUNDS times C columns; SET workgroups side by
  // side together take the eight columns of a cache line in the same round.
  static constexpr int SET = C < 8 && N >= 1024 ? 8 / C : 1;
  static constexpr int ROUNDS = N >= 8192 ? 16 : (N >= 2048 ? 4 : 1);
  static constexpr int GROUPS = N / (C * ROUNDS);
  static constexpr int PAD = N + N / 16 + (N < 16 ? 1 : 0);
  static constexpr int HI = N > 64 ? N / 64 : 1;  // entries of the coarse twiddle table
  static constexpr size_t lds_bytes() { return (size_t)C * PAD * sizeof(double); }
};

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// X[k] = sum_n x[n] exp(-2 pi i n k / R), in place.
__device__ __forceinline__ void dft(double2 (&v)[2]) {
  const double2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}
__device__ __forceinline__ void dft(double2 (&v)[4]) {
  const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = csub(v[1], v[3]);
  v[0] = cadd(a, c);
  v[2] = csub(a, c);
  v[1] = make_double2(b.x + d.y, b.y - d.x);  // b - i d
  v[3] = make_double2(b.x - d.y, b.y + d.x);
}
__device__ __forceinline__ void dft(double2 (&v)[8]) {
  constexpr double h = 0.70710678118654752440;
  double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
  dft(e);
  dft(o);
  o[1] = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));   // (1 - i) / sqrt 2
  o[2] = make_double2(o[2].y, -o[2].x);                                // -i
  o[3] = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));  // (-1 - i) / sqrt 2
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = cadd(e[k], o[k]);
    v[k + 4] = csub(e[k], o[k]);
  }
}
__device__ __forceinline__ void dft(double2 (&v)[16]) {
  // n = 4 n1 + n2, k = k1 + 4 k2
  constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
  double2 a[4][4];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < 4; ++n1) a[n2][n1] = v[4 * n1 + n2];
    dft(a[n2]);
  }
  // a[n2][k1] *= exp(-2 pi i n2 k1 / 16)
  a[1][1] = cmul(a[1][1], make_double2(c1, -s1));
  a[1][2] = make_double2(h * (a[1][2].x + a[1][2].y), h * (a[1][2].y - a[1][2].x));
  a[1][3] = cmul(a[1][3], make_double2(s1, -c1));
  a[2][1] = make_double2(h * (a[2][1].x + a[2][1].y), h * (a[2][1].y - a[2][1].x));
  a[2][2] = make_double2(a[2][2].y, -a[2][2].x);
  a[2][3] = make_double2(h * (a[2][3].y - a[2][3].x), -h * (a[2][3].x + a[2][3].y));
  a[3][1] = cmul(a[3][1], make_double2(s1, -c1));
  a[3][2] = make_double2(h * (a[3][2].y - a[3][2].x), -h * (a[3][2].x + a[3][2].y));
  a[3][3] = cmul(a[3][3], make_double2(-c1, s1));
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    double2 b[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
    dft(b);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = b[k2];
  }
}

template <int LOGN>
struct Twiddles {
  double2 hi[Fft<LOGN>::HI], lo[64];
};
template <int LOGN>
__device__ __forceinline__ void fill_twiddles(Twiddles<LOGN>& tw) {
  using F = Fft<LOGN>;
  for (int e = threadIdx.x; e < F::HI + 64; e += F::THREADS) {
    const int m = e < F::HI ? 64 * e : e - F::HI;
    double s, c;
    sincospi(-2.0 * double(m) / double(F::N), &s, &c);
    (e < F::HI ? tw.hi[e] : tw.lo[e - F::HI]) = make_double2(c, s);
  }
}

// One pass of radix R after passes of product NS.  at(i) is the LDS index of
// point i of this thread's transform; threads that hold no points (not active)
// only meet the barriers.
template <int LOGN, int NS, int R, bool LAST, typename At>
__device__ __forceinline__ void fft_pass(double2 (&x)[Fft<LOGN>::E], int t, bool active, const Twiddles<LOGN>& tw,
                                         double* lds, At at) {
  using F = Fft<LOGN>;
  constexpr int U = F::E / R;  // butterflies per thread
#pragma unroll
  for (int u = 0; u < U; ++u) {
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = x[u + r * U];
    if constexpr (NS > 1) {
      const int k = ((t + u * F::T) & (NS - 1)) * (F::N / (NS * R));
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const int m = k * r;
        v[r] = cmul(v[r], cmul(tw.hi[m >> 6], tw.lo[m & 63]));
      }
    }
    dft(v);
#pragma unroll
    for (int r = 0; r < R; ++r) x[u + r * U] = v[r];
  }
  if constexpr (!LAST) {
    auto out = [&](int u, int r) {
      const int j = t + u * F::T;
      return at((j / NS) * (NS * R) + (j & (NS - 1)) + r * NS);
    };
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      __syncthreads();  // the buffer's earlier contents are read
      if (active) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int r = 0; r < R; ++r) lds[out(u, r)] = part ? x[u + r * U].y : x[u + r * U].x;
      }
      __syncthreads();
      if (active) {
#pragma unroll
        for (int m = 0; m < F::E; ++m) (part ? x[m].y : x[m].x) = lds[at(t + F::T * m)];
      }
    }
  }
}

// Transform of the points t + T m held in x[m], natural order in and out.
template <int LOGN, typename At>
__device__ __forceinline__ void fft_points(double2 (&x)[Fft<LOGN>::E], int t, bool active, const Twiddles<LOGN>& tw,
                                           double* lds, At at) {
  constexpr int B = Fft<LOGN>::E, LB = Fft<LOGN>::LOGE, P = LOGN / LB, REM = 1 << (LOGN % LB);
  fft_pass<LOGN, 1, B, P == 1 && REM == 1>(x, t, active, tw, lds, at);
  if constexpr (P > 1) fft_pass<LOGN, B, B, P == 2 && REM == 1>(x, t, active, tw, lds, at);
  if constexpr (P > 2) fft_pass<LOGN, B * B, B, P == 3 && REM == 1>(x, t, active, tw, lds, at);
  static_assert(P <= 3, "three passes of the full radix at most");
  if constexpr (REM > 1) fft_pass<LOGN, 1 << (LB * P), REM, true>(x, t, active, tw, lds, at);
}

template <int LOGN>
__global__ void __launch_bounds__(Fft<LOGN>::THREADS, Fft<LOGN>::WAVES)
k_fft_rows(const double* __restrict__ mom, double2* __restrict__ work) {
  using F = Fft<LOGN>;
  extern __shared__ double lds[];
  __shared__ Twiddles<LOGN> tw;
  const int t = threadIdx.x % F::T, c = threadIdx.x / F::T, pair = blockIdx.y;
  const bool active = F::ACTIVE == F::THREADS || threadIdx.x < F::ACTIVE;
  const int64_t nn = (int64_t)F::N * F::N, row = ((int64_t)blockIdx.x * F::C + c) * F::N;
  double2 x[F::E];
#pragma unroll
  for (int m = 0; m < F::E; ++m) {
    x[m] = make_double2(0.0, 0.0);
    if (!active) continue;
    const int64_t i = row + t + F::T * m;
    if (pair == 0) {
      const double r = mom[i];
      x[m] = make_double2(mom[nn + i] / r, mom[2 * nn + i] / r);
    } else {
      x[m] = make_double2(mom[3 * nn + i], mom[4 * nn + i]);
    }
  }
  fill_twiddles(tw);
  __syncthreads();
  fft_points<LOGN>(x, t, active, tw, lds, [&](int i) { return c * F::PAD + i + (i >> 4); });
  if (!active) return;
#pragma unroll
  for (int m = 0; m < F::E; ++m) work[pair * nn + row + t + F::T * m] = x[m];
}

// ceil(sqrt(max(v, 0))), exact.
__device__ __forceinline__ int isqrt_ceil(int v) {
  if (v <= 0) return 0;
  int r = int(sqrtf(float(v)));
  while (r * r >= v) --r;
  while (r * r < v) ++r;
  return r;
}

constexpr int spectra_bins_of(int n) {
  // floor(sqrt(2) n / 2 + 1/2) + 1: bins of round(|k|), |k|^2 <= n^2 / 2
  int b = 0;
  while (int64_t(b) * b - b + 1 <= int64_t(n) * n / 2) ++b;
  return b;
}

// Column pass of pair blockIdx.y (workgroups numbered XCD-contiguously, so that
// those of a set share an L2): transforms, then the bins.  Bin b holds the k with
// floor(|k| + 1/2) = b, i.e. |k|^2 = 0 for b = 0 and b^2 - b + 1 <= |k|^2 <= b^2 + b
// for b >= 1 (exact in integers), so of column k_x it holds the |k_y| from
// ceil(sqrt(b^2 - b + 1 - k_x^2)) to one below the next bin's first.  One thread per
// bin and column walks that range; the columns' sums are added across lanes, the
// rounds' sums in order.
template <int LOGN>
__global__ void __launch_bounds__(Fft<LOGN>::THREADS, Fft<LOGN>::WAVES)
k_fft_cols(const double2* __restrict__ work, double* __restrict__ part, double* __restrict__ partx) {
  using F = Fft<LOGN>;
  constexpr int N = F::N, C = F::C, TH = F::THREADS, NB = spectra_bins_of(N), W = TH / 64;
  extern __shared__ double lds[];
  __shared__ Twiddles<LOGN> tw;
  __shared__ double red[W][C];
  const int tid = threadIdx.x, c = tid % C, t = tid / C, pair = blockIdx.y;
  const bool active = F::ACTIVE == TH || tid < F::ACTIVE;
  const int g = xcd_contiguous(blockIdx.x, gridDim.x);
  const int64_t nn = (int64_t)N * N;
  const double inv = 1.0 / (double(N) * double(N));
  double* out = part + ((int64_t)pair * gridDim.x + g) * NB;
  fill_twiddles(tw);
  for (int round = 0; round < F::ROUNDS; ++round) {
    const int col0 = (((g / F::SET) * F::ROUNDS + round) * F::SET + g % F::SET) * C;
    double2 x[F::E];
    const double2* src = work + pair * nn + (int64_t)t * N + col0 + c;
#pragma unroll
    for (int m = 0; m < F::E; ++m) x[m] = active ? src[(int64_t)m * F::T * N] : make_double2(0.0, 0.0);
    __syncthreads();  // tables filled; the powers of the columns before are read
    fft_points<LOGN>(x, t, active, tw, lds, [&](int i) { return (i + (i >> 4)) * C + c; });
    // scaled powers of the columns: lds[k_y * C + c]
    double sum = 0.0;
    __syncthreads();
    if (active) {
#pragma unroll
      for (int m = 0; m < F::E; ++m) {
        const double re = x[m].x * inv, im = x[m].y * inv, p = re * re + im * im;
        lds[(t + F::T * m) * C + c] = p;
        sum += p;
      }
    }
    // column sums: lanes of one column, then the waves in order
#pragma unroll
    for (int off = 32; off >= C; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if ((tid & 63) < C) red[tid >> 6][c] = sum;
    __syncthreads();
    if (pair == 0 && tid < C) {
      double a = red[0][tid];
      for (int w = 1; w < W; ++w) a += red[w][tid];
      partx[col0 + tid] = a;
    }
    const int kxi = col0 + c, kx = kxi < N / 2 ? kxi : N - kxi;  // |k_x| of this thread's column
    const double* P = lds + c;
    for (int b0 = 0; b0 < NB; b0 += TH / C) {
      const int b = b0 + t;
      double s = 0.0;
      const int hi = isqrt_ceil(b * b + b + 1 - kx * kx);  // first |k_y| of bin b + 1
      if (hi != 0 && b < NB) {
        const int a0 = b == 0 ? 0 : isqrt_ceil(b * b - b + 1 - kx * kx), a1 = min(hi - 1, N / 2);
        for (int ay = a0; ay <= a1; ++ay) {
          s += P[ay * C];
          if (ay != 0 && ay != N / 2) s += P[(N - ay) * C];
        }
      }
#pragma unroll
      for (int off = C / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (c == 0 && b < NB) out[b] = round == 0 ? s : out[b] + s;  // this thread's own value
    }
  }
}

// Sums of the column groups' bins in a fixed order: thread (bin, s) of a 64 x 16
// block adds the groups s, s + 16, s + 32, ... of its bin (consecutive bins
// are consecutive addresses), then the 16 partial sums are added in order of s.
__global__ void __launch_bounds__(1024)
k_spectra_final(const double* __restrict__ part, const double* __restrict__ partx, int n, int groups, int nbins,
                double* __restrict__ ek, double* __restrict__ em, double* __restrict__ ekx) {
  __shared__ double red[2][16][64];
  const int bl = threadIdx.x, sl = threadIdx.y;
  const int b = blockIdx.x * 64 + bl;
  double su = 0.0, sb = 0.0;
  if (b < nbins) {
    for (int k = sl; k < groups; k += 16) {
      su += part[(int64_t)k * nbins + b];
      sb += part[((int64_t)groups + k) * nbins + b];
    }
  }
  red[0][sl][bl] = su;
  red[1][sl][bl] = sb;
  __syncthreads();
  if (sl == 0 && b < nbins) {
    double tu = 0.0, tb = 0.0;
    for (int i = 0; i < 16; ++i) {
      tu += red[0][i][bl];
      tb += red[1][i][bl];
    }
    ek[b] = 0.5 * tu;
    em[b] = 0.5 * tb;
  }
  if (ekx && sl == 1 && b <= n / 2) {
    double x = partx[b];
    if (b != 0 && b != n / 2) x += partx[n - b];
    ekx[b] = 0.5 * x;
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
int spectra_bins(int n) { return (int)floor(sqrt(2.0) * double(n / 2) + 0.5) + 1; }

// f(std::integral_constant<int, LOGN>) for n = 8 .. 16384.
template <typename F>
static auto by_length(int n, F&& f) {
  switch (n) {
    case 8: return f(std::integral_constant<int, 3>{});
    case 16: return f(std::integral_constant<int, 4>{});
    case 32: return f(std::integral_constant<int, 5>{});
    case 64: return f(std::integral_constant<int, 6>{});
    case 128: return f(std::integral_constant<int, 7>{});
    case 256: return f(std::integral_constant<int, 8>{});
    case 512: return f(std::integral_constant<int, 9>{});
    case 1024: return f(std::integral_constant<int, 10>{});
    case 2048: return f(std::integral_constant<int, 11>{});
    case 4096: return f(std::integral_constant<int, 12>{});
    case 8192: return f(std::integral_constant<int, 13>{});
    default: return f(std::integral_constant<int, 14>{});
  }
}

// The row transforms, room for the bins of every column and for the column sums
// (and, beyond 4096 columns, as much again as their powers take): more than the
// kernels use, as callers have sized it.
size_t spectra_work_bytes(int n) {
  const size_t nn = (size_t)n * n;
  const size_t big = n > 4096 ? 2 * nn * sizeof(double) : 0;
  return 2 * nn * sizeof(double2) + big + (size_t)2 * n * spectra_bins(n) * sizeof(double) +
         (size_t)2 * n * sizeof(double);
}

template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

hipError_t launch_spectra(const double* mom, int n, double* ek, double* em, double* ekx, void* work, hipStream_t st) {
  const int nb = spectra_bins(n);
  double2* cw = static_cast<double2*>(work);
  double* part = reinterpret_cast<double*>(cw + (size_t)2 * n * n);
  return by_length(n, [&](auto l) {
    constexpr int LOGN = decltype(l)::value;
    using F = Fft<LOGN>;
    static_assert(F::GROUPS * F::C * F::ROUNDS == F::N && F::GROUPS % F::SET == 0, "column groups");
    const int groups = F::GROUPS;
    double* partx = part + (size_t)2 * groups * nb;
    hipError_t e;
    if ((e = allow_lds(&k_fft_rows<LOGN>, F::lds_bytes())) != hipSuccess) return e;
    if ((e = allow_lds(&k_fft_cols<LOGN>, F::lds_bytes())) != hipSuccess) return e;
    hipLaunchKernelGGL((k_fft_rows<LOGN>), dim3(F::N / F::C, 2), dim3(F::THREADS), F::lds_bytes(), st, mom, cw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_fft_cols<LOGN>), dim3(groups, 2), dim3(F::THREADS), F::lds_bytes(), st, cw, part, partx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int fin = nb > n / 2 + 1 ? nb : n / 2 + 1;
    hipLaunchKernelGGL(k_spectra_final, dim3((fin + 63) / 64), dim3(64, 16), 0, st, part, partx, n, groups, nb, ek, em,
                       ekx);
    return hipGetLastError();
  });
}

}  // namespace lbm
