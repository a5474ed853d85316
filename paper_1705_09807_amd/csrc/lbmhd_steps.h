// Sweeps that advance the fused schedule by several timesteps per launch
// (temporal blocking).
//
// A one-step sweep moves every population through HBM once per step and is
// bound by that: at 4096^2 FP32 its loads and stores alone take as long as the
// whole sweep (410 us closure off, 440 us on), while its arithmetic needs a
// fifth of the time.  The sweep here keeps the states between the steps on the
// chip: a workgroup marches up a column strip with one group of waves per step;
// each group collides a row a few rows behind the group before it and hands the
// post-collision populations on through LDS, so HBM sees one read and one write
// of the state per K steps.  Step s of a strip is valid on one column less at
// each side than step s - 1 (closure off), or two (one for the gradients, one for
// the streaming), so T columns of a group give T - 2 H stored ones and the outer
// H are recomputed by the neighbouring strip; likewise a segment of rows starts
// H rows early and ends H rows late.
//
// Values handed on are rounded to the storage type exactly as a store and a load
// would, and the arithmetic is the shared per-cell code, evaluated as written:
// the results equal those of one-step sweeps bit for bit.
//
// Measured, us per step over long runs (the first thirty launches or so of the sweeps
// that the arithmetic bounds are slower: 1024^2 FP32 closure on 77 us, then 52-57), one-step
// sweep -> K steps per launch: 4096^2 FP32 closure off 410 -> 131 (K = 4), on
// 445 -> 170 (K = 3); 8192^2 BF16 844 -> 379 and 951 -> 597, FP16 854 -> 377 and
// 960 -> 647; 4096^2 FP64 953 -> 344 and 851 -> 344; 1024^2 FP32 25.2 -> 9.7 and
// 27.3 -> 17.4; 4096^2 D2Q9 FP32 589 -> 250 and 624 -> 249; 1500 x 1001 D2Q9
// FP64 with density gradients 128 -> 51.  What bounds it now:
// at 4096^2 FP32 a launch moves its 2.55 GB at 4.9-5.0 TB/s with the closure and
// the vector ALUs busy about half the time; 16-bit storage is bound by the vector
// ALUs (8192^2 BF16: about 230 instructions a cell and step, 410 of the 597 us).
// The same steps evaluated one after another by one group of waves (each lane
// every step of its column) took 252 us at K = 2 and 224 at K = 3 (4096^2 FP32,
// closure on): a wave's arithmetic, its LDS and its loads then wait on each other.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lbmhd_cell.h"
#include "lbmhd_device.h"
#include "lbmhd_internal.h"

namespace lbm {

// Strip, segment and group of this thread (workgroups numbered XCD-contiguously: the
// strips of a segment run side by side on one XCD and share the lines at their
// edges in its L2).
struct MsTile {
  int step, lane;      // group, lane within it
  int x0, x1, y0, y1;  // cells the workgroup stores
};
__device__ __forceinline__ MsTile ms_tile(int nx, int ny, int w, int ry, int k) {
  MsTile t;
  const int T = blockDim.x / k;
  t.step = __builtin_amdgcn_readfirstlane(threadIdx.x / T);
  t.lane = threadIdx.x - t.step * T;
  const int nstrip = (nx + w - 1) / w;
  const int vb = xcd_contiguous(blockIdx.x, gridDim.x);
  t.x0 = (vb % nstrip) * w;
  t.x1 = min(t.x0 + w, nx);
  t.y0 = (vb / nstrip) * ry;
  t.y1 = min(t.y0 + ry, ny);
  return t;
}
// The lane's column, x0 - halo + lane (periodic; lanes past the right halo repeat its
// last column).
__device__ __forceinline__ int ms_column(const MsTile& t, int halo, int nx) {
  const int x = min(t.x0 - halo + t.lane, t.x1 - 1 + halo);
  return x < 0 ? x + nx : (x >= nx ? x - nx : x);
}
// Whether the lane stores its column.
__device__ __forceinline__ bool ms_owner(const MsTile& t, int halo) {
  return t.lane >= halo && t.lane < halo + (t.x1 - t.x0);
}
// Row y (within a grid height of the grid) of the state before the launch.
template <typename S, int QG>
__device__ __forceinline__ void ms_pull(const S* __restrict__ src, uint32_t pq, int y, int ny, const Cols& cx,
                                        RawCell<S, QG>& c) {
  auto wrapy = [&](int v) { return v < 0 ? v + ny : (v >= ny ? v - ny : v); };
  pull_raw<S, QG>(src, pq, wrapy(y - 1), wrapy(y), wrapy(y + 1), cx, c);
}
// Store of row y, dropped outside the workgroup's rows and columns.  Ordinary
// stores: the strips' edges share lines, which then meet in L2 (non-temporal
// stores took 370 against 297 us per step at 4096^2).
template <typename S, int QG>
__device__ __forceinline__ void ms_store(S* __restrict__ dst, uint32_t pq, const MsTile& t, int y, bool owner,
                                         const Cols& cx, const typename ComputeOf<S>::type* v) {
  const bool mine = y >= t.y0 && y < t.y1;
  const uint32_t rowb = uint32_t(kPop<QG>) * pq;
  const __amdgpu_buffer_rsrc_t d = row_rsrc(reinterpret_cast<char*>(dst) + int64_t(mine ? y : t.y0) * rowb, rowb);
  const uint32_t xo = owner && mine ? cx.c : kDropOffset;
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) buf_store<S, false>(narrow<S>(v[q]), d, xo, uint32_t(q) * pq);
}

// Closure off, K steps per launch.  A workgroup holds K groups of T = blockDim / K
// lanes, one per step, and marches up the rows of its strip; the lanes of a group own
// the same columns.  In iteration i group 0 collides row i (loaded an iteration
// earlier) and hands it on; group s > 0 reads the row that group s - 1 handed on in
// the iteration before, whose populations stream into the rows above, beside and
// below it: the row below it, i - 2 s, is then complete in registers and is
// collided and handed on or, in the last group, stored.  Rows are handed on
// through two LDS slots by parity, one barrier per iteration.  One wave of every
// group runs on every SIMD, so while one waits for its loads, LDS or the barrier the
// others' arithmetic fills in.  (Gathering a row from three LDS slots behind a second
// barrier: 512^2 FP32 5.5 against 4.5 us per step, 1024^2 11.7 against 9.7; the same
// at 4096^2, where HBM sets the pace.)
template <typename S, int QG, int K, int LN>
struct DnsLds {
  S pop[K - 1][2][kPop<QG>][LN + 2];  // step, parity, population, lane + 1
};

// `load` gets a row of the state before the launch, AHEAD (1 or 3) iterations before it is
// collided, `store` takes a row of the state after it.
template <typename S, int QG, int K, int LN, int AHEAD, typename Load, typename Store>
__device__ __forceinline__ void dns_march(DnsLds<S, QG, K, LN>& lds, const MsTile& t, bool swapped,
                                          const Rates<typename ComputeOf<S>::type>& r, Load&& load, Store&& store) {
  using C = typename ComputeOf<S>::type;
  constexpr int NP = kPop<QG>, H = K - 1;  // H: recomputed columns at each side, rows at each end
  const int l = t.lane + 1;
  const int first = t.y0 - H, last = t.y1 - 1 + H;  // rows of the first step
  const int end = t.y1 + 2 * (K - 1);               // iterations first .. end - 1
  const Closure<C> off = {C(0), C(0), C(0), C(0)};
  auto collide = [&](C* v) __attribute__((always_inline)) {
    const Mom<C> m = moments_of<QG, kUnits<S>>(v);
    collide_q<QG, false, false, kUnits<S>>(v, m, off, r, swapped);
  };
  auto hand_on = [&](int s, int par, const C* v) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NP; ++q) lds.pop[s][par][q][l] = narrow<S>(v[q]);
  };
  using N0 = std::integral_constant<int, 0>;
  using N1 = std::integral_constant<int, 1>;
  using N2 = std::integral_constant<int, 2>;
  using N3 = std::integral_constant<int, 3>;

  if (t.step == 0) {
    constexpr int NR = AHEAD + 1;  // rows in flight and the current one
    static_assert(4 % NR == 0, "the loop is unrolled by four");
    RawCell<S, QG> raw[NR];
    auto iter = [&](int i, auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      load(min(i + AHEAD, last), raw[(u + AHEAD) % NR]);
      __builtin_amdgcn_sched_barrier(0);
      C v[NP];
      widen_raw<S, C, QG>(raw[u % NR], v);
      collide(v);
      hand_on(0, u & 1, v);
      __syncthreads();
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) load(min(first + k, last), raw[k]);
    // small grids, of few iterations, leave at `end`; past it nothing is stored
    for (int i = first; i < end; i += 4) {
      iter(i, N0{});
      if (AHEAD > 1 && i + 1 >= end) break;
      iter(i + 1, N1{});
      if (AHEAD > 1 && i + 2 >= end) break;
      iter(i + 2, N2{});
      if (AHEAD > 1 && i + 3 >= end) break;
      iter(i + 3, N3{});
    }
  } else {
    C row[4][NP];  // rows being completed, by the iteration (mod 4) that completes them
    auto iter = [&](int i, auto uc, auto sc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value, st = decltype(sc)::value;
#pragma unroll
      for (int q = 0; q < NP; ++q)
        row[(u + 1 + qcy<QG>(q)) & 3][q] = widen<C>(lds.pop[st - 1][(u & 1) ^ 1][q][l - qcx<QG>(q)]);
      if constexpr (sizeof(S) == 8) __builtin_amdgcn_sched_barrier(0);  // registers: the reads before the collision
      C v[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) v[q] = row[u][q];
      collide(v);
      if constexpr (st + 1 < K)
        hand_on(st, u & 1, v);
      else
        store(i - 2 * st, v);
      __syncthreads();
    };
    auto loop = [&](auto sc) __attribute__((always_inline)) {
      for (int i = first; i < end; i += 4) {
        iter(i, N0{}, sc);
        if (AHEAD > 1 && i + 1 >= end) break;
        iter(i + 1, N1{}, sc);
        if (AHEAD > 1 && i + 2 >= end) break;
        iter(i + 2, N2{}, sc);
        if (AHEAD > 1 && i + 3 >= end) break;
        iter(i + 3, N3{}, sc);
      }
    };
    if (t.step == 1) loop(N1{});
    if constexpr (K > 2) {
      if (t.step == 2) loop(N2{});
    }
    if constexpr (K > 3) {
      if (t.step == 3) loop(N3{});
    }
  }
}

template <typename S, int QG, int K, int LN, int AHEAD>
__global__ void __launch_bounds__(LN* K)
k_dns_steps(const S* __restrict__ src, S* __restrict__ dst, int nx, int ny, int64_t pitch, int w, int ry,
            Rates<typename ComputeOf<S>::type> r) {
  using C = typename ComputeOf<S>::type;
  constexpr int H = K - 1;
  extern __shared__ __attribute__((aligned(16))) char ms_lds[];
  const MsTile t = ms_tile(nx, ny, w, ry, K);
  const int x = ms_column(t, H, nx);
  const Cols cx = cols_of<S>(x, nx);
  const bool owner = ms_owner(t, H);
  const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S));
  dns_march<S, QG, K, LN, AHEAD>(
      *reinterpret_cast<DnsLds<S, QG, K, LN>*>(ms_lds), t, swapped_rest<S>(x, nx), r,
      [&](int y, RawCell<S, QG>& c) __attribute__((always_inline)) { ms_pull<S, QG>(src, pq, y, ny, cx, c); },
      [&](int y, const C* v) __attribute__((always_inline)) { ms_store<S, QG>(dst, pq, t, y, owner, cx, v); });
}

// LDS rows that hand population q from one step to the next: a row written in
// iteration j is read in j + 1 by the populations that move down, j + 2 by those
// that stay in their row and j + 3 by those that move up, always before that
// iteration's write.
template <int QG>
constexpr int ms_slots(int q) { return qcy<QG>(q) < 0 ? 1 : (qcy<QG>(q) == 0 ? 2 : 3); }
template <int QG>
constexpr int ms_row(int q) {
  int k = 0;
  for (int p = 0; p < q; ++p) k += ms_slots<QG>(p);
  return k;
}
template <int QG>
constexpr int kMsRows = ms_row<QG>(kPop<QG>);

// LDS of k_les_steps for at most LN columns (and one pad column at each side).
template <typename S, int MODE, int QG, int K, int LN>
struct LesLds {
  using C = typename ComputeOf<S>::type;
  static constexpr bool FULL = MODE == kClosureFull;
  struct alignas(4 * sizeof(C)) Quad {
    C v[4];
  };
  Quad mom[K][3][LN + 2];  // m_x, m_y, B_x - B_ref, B_y - B_ref by step, row slot, lane + 1
  C rho[FULL ? K : 1][FULL ? 3 : 1][FULL ? LN + 2 : 1];
  S pop[K - 1][kMsRows<QG>][LN + 2];  // handed-on populations
};

// Closure on, K steps per launch, groups as in k_dns_steps.  In iteration i
//  first half:  group 0 has row i (loaded an iteration earlier), group s > 0 gathers
//               row i - 3 s of its step from the populations that group s - 1 handed
//               on; each puts the row's moments into its ring (three row slots);
//  second half: each group collides the row before it with the gradients from its
//               ring, and hands it on or, in the last group, stores it.
// A barrier after each half.  (One barrier per iteration, as in k_dns_steps, takes
// two more rows of registers and spills: 4096^2 FP32 201 against 178 us per step.)
template <typename S, int STENCIL, int MODE, int QG, int K, int LN, typename Load, typename Store>
__device__ __forceinline__ void les_march(LesLds<S, MODE, QG, K, LN>& lds, const MsTile& t,
                                          const Rates<typename ComputeOf<S>::type>& r, Load&& load, Store&& store) {
  using C = typename ComputeOf<S>::type;
  using Lds = LesLds<S, MODE, QG, K, LN>;
  using Quad = typename Lds::Quad;
  constexpr int NP = kPop<QG>, NF = Lds::FULL ? 5 : 4;
  constexpr bool LOCAL = STENCIL >= LBM_STENCIL_LOCAL_ISO9 && QG == 5 && MODE != kClosureFull;
  constexpr int H = 2 * K - 1;  // recomputed columns at each side, rows at each end
  const int l = t.lane + 1;
  const int first = t.y0 - H, last = t.y1 - 1 + H;  // rows of the first step's moments
  const int end = t.y1 + 3 * (K - 1) + 1;           // iterations first .. end - 1

  auto put = [&](int s, int sl, const C* v) __attribute__((always_inline)) {
    const Mom<C> m = moments_of<QG, kUnits<S>>(v);
    lds.mom[s][sl][l] = Quad{m.mx, m.my, m.dbx, m.dby};
    if constexpr (NF == 5) lds.rho[s][sl][l] = m.drho;
  };
  // closure and collision of a cell whose row sits in slot sc of step s's ring, its
  // southern and northern neighbours' rows in ss and sn
  auto collide = [&](int s, int ss, int sc, int sn, C* v) __attribute__((always_inline)) {
    const Mom<C> m = moments_of<QG, kUnits<S>>(v);
    const auto& q = lds.mom[s];
    C gr[NF][2];
    // FP64: two fields at a time, which the registers have room for
    constexpr int kAtOnce = sizeof(C) == 8 ? 2 : 4;
#pragma unroll
    for (int k0 = 0; k0 < 4; k0 += kAtOnce) {
#pragma unroll
      for (int k = k0; k < k0 + kAtOnce; ++k)
        grad3x3<C, STENCIL>(q[sc][l + 1].v[k], q[sc][l - 1].v[k], q[sn][l].v[k], q[ss][l].v[k], q[sn][l + 1].v[k],
                            q[sn][l - 1].v[k], q[ss][l + 1].v[k], q[ss][l - 1].v[k], gr[k][0], gr[k][1]);
      if constexpr (kAtOnce < 4) __builtin_amdgcn_sched_barrier(0);
    }
    const C ir = C(1) / (r.rho0 + m.drho);
    Closure<C> cl;
    if constexpr (Lds::FULL) {
      const auto& p = lds.rho[s];
      grad3x3<C, STENCIL>(p[sc][l + 1], p[sc][l - 1], p[sn][l], p[ss][l], p[sn][l + 1], p[sn][l - 1], p[ss][l + 1],
                          p[ss][l - 1], gr[4][0], gr[4][1]);
      cl = closure_terms_full(gr, m.mx, m.my, r.bx0 + m.dbx, r.by0 + m.dby, ir, r.k2);
    } else {
      if constexpr (LOCAL)
        local_gradients<kUnits<S>>(v, m, r, gr[1][0] - gr[0][1], gr);
      cl = closure_terms<LOCAL>(gr[0][0], gr[0][1], gr[1][0], gr[1][1], gr[2][0], gr[2][1], gr[3][0], gr[3][1], ir, r.k2);
    }
    collide_q<QG, true, LOCAL, kUnits<S>>(v, m, cl, r);
  };
  // slot of population q in iteration i: u = i mod 3, par = i mod 2
  auto slot = [](int q, int u, int par) { return ms_row<QG>(q) + (qcy<QG>(q) > 0 ? u : (qcy<QG>(q) == 0 ? par : 0)); };
  auto hand_on = [&](int s, int u, int par, const C* v) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NP; ++q) lds.pop[s][slot(q, u, par)][l] = narrow<S>(v[q]);
  };
  using N0 = std::integral_constant<int, 0>;
  using N1 = std::integral_constant<int, 1>;
  using N2 = std::integral_constant<int, 2>;

  if (t.step == 0) {
    RawCell<S, QG> raw[3];
    auto iter = [&](int i, int par, auto uc) __attribute__((always_inline)) {
      constexpr int u0 = decltype(uc)::value, u1 = (u0 + 2) % 3, u2 = (u0 + 1) % 3;  // rows i, i - 1, i - 2
      load(min(i + 1, last), raw[u2]);
      __builtin_amdgcn_sched_barrier(0);
      C v[NP];
      widen_raw<S, C, QG>(raw[u0], v);
      put(0, u0, v);
      __syncthreads();
      widen_raw<S, C, QG>(raw[u1], v);
      collide(0, u2, u1, u0, v);
      hand_on(0, u0, par, v);
      __syncthreads();
    };
    load(first, raw[0]);
    for (int i = first, par = 0; i < end; i += 3, par ^= 1) {  // past `end`: nothing is stored
      iter(i, par, N0{});
      iter(i + 1, par ^ 1, N1{});
      iter(i + 2, par, N2{});
    }
  } else {
    C vs[3][NP];  // rows gathered and not yet collided
    auto iter = [&](int i, int par, auto uc, auto sc) __attribute__((always_inline)) {
      constexpr int u0 = decltype(uc)::value, u1 = (u0 + 2) % 3, u2 = (u0 + 1) % 3, st = decltype(sc)::value;
#pragma unroll
      for (int q = 0; q < NP; ++q) vs[u0][q] = widen<C>(lds.pop[st - 1][slot(q, u0, par)][l - qcx<QG>(q)]);
      put(st, u0, vs[u0]);
      __syncthreads();
      C v[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) v[q] = vs[u1][q];
      collide(st, u2, u1, u0, v);
      if constexpr (st + 1 < K)
        hand_on(st, u0, par, v);
      else
        store(i - 3 * st - 1, v);
      __syncthreads();
    };
    auto loop = [&](auto sc) __attribute__((always_inline)) {
      for (int i = first, par = 0; i < end; i += 3, par ^= 1) {
        iter(i, par, N0{}, sc);
        iter(i + 1, par ^ 1, N1{}, sc);
        iter(i + 2, par, N2{}, sc);
      }
    };
    if (t.step == 1) loop(N1{});
    if constexpr (K > 2) {
      if (t.step == 2) loop(N2{});
    }
  }
}

template <typename S, int STENCIL, int MODE, int QG, int K, int LN>
__global__ void __launch_bounds__(LN* K)
k_les_steps(const S* __restrict__ src, S* __restrict__ dst, int nx, int ny, int64_t pitch, int w, int ry,
            Rates<typename ComputeOf<S>::type> r) {
  using C = typename ComputeOf<S>::type;
  constexpr int H = 2 * K - 1;
  extern __shared__ __attribute__((aligned(16))) char ms_lds[];
  const MsTile t = ms_tile(nx, ny, w, ry, K);
  const Cols cx = cols_of<S>(ms_column(t, H, nx), nx);
  const bool owner = ms_owner(t, H);
  const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S));
  les_march<S, STENCIL, MODE, QG, K, LN>(
      *reinterpret_cast<LesLds<S, MODE, QG, K, LN>*>(ms_lds), t, r,
      [&](int y, RawCell<S, QG>& c) __attribute__((always_inline)) { ms_pull<S, QG>(src, pq, y, ny, cx, c); },
      [&](int y, const C* v) __attribute__((always_inline)) { ms_store<S, QG>(dst, pq, t, y, owner, cx, v); });
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
constexpr int kClosureOff = 3;  // beside the closure variants

template <typename S, int STENCIL, int MODE, int QG, int K, int LN>
static hipError_t launch_k_steps(const Launch& L) {
  using C = typename ComputeOf<S>::type;
  using Lds = std::conditional_t<MODE == kClosureOff, DnsLds<S, QG, K, LN>, LesLds<S, MODE, QG, K, LN>>;
  static_assert(sizeof(Lds) <= 160 * 1024, "LDS of a compute unit");
  // as the time estimate of 16-bit sweeps assumes
  static_assert(sizeof(S) > 2 || MODE == kClosureOff || (160 * 1024 / sizeof(Lds) > 1) == (MODE != kClosureFull || K < 3),
                "workgroups per compute unit");
  const MsShape sh = ms_shape(L, MODE != kClosureOff ? 2 * K - 1 : K - 1, LN, 160 * 1024 / sizeof(Lds));
  const auto kernel = [] {
    if constexpr (MODE == kClosureOff)
      return &k_dns_steps<S, QG, K, LN, LN < 256 ? 3 : 1>;
    else
      return &k_les_steps<S, STENCIL, MODE, QG, K, LN>;
  }();
  if (sizeof(Lds) > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Lds));
    if (e != hipSuccess) return e;
  }
  char* base = static_cast<char*>(L.state);
  const size_t off = buffer_offset_bytes(L.nx, L.ny, L.dtype, L.qg);
  hipLaunchKernelGGL(kernel, dim3(sh.blocks), dim3(sh.lanes * K), sizeof(Lds), L.stream,
                     reinterpret_cast<const S*>(base + (L.cur ? off : 0)),
                     reinterpret_cast<S*>(base + (L.cur ? 0 : off)), L.nx, L.ny, L.pitch, sh.w, sh.ry,
                     make_rates<C>(L));
  return hipGetLastError();
}

// The instance for this run's closure, stencil and k (2 .. ms_most_steps).
template <typename S, int MODE, int QG, int K, int LN>
static hipError_t launch_k_stencil(const Launch& L) {
  if constexpr (MODE == kClosurePlain && QG == 5) {
    if (L.stencil == LBM_STENCIL_LOCAL_ISO9) return launch_k_steps<S, LBM_STENCIL_LOCAL_ISO9, MODE, QG, K, LN>(L);
    if (L.stencil == LBM_STENCIL_LOCAL_CENTRAL5)
      return launch_k_steps<S, LBM_STENCIL_LOCAL_CENTRAL5, MODE, QG, K, LN>(L);
  }
  if constexpr (MODE != kClosureOff) {
    if (L.stencil == LBM_STENCIL_CENTRAL5) return launch_k_steps<S, LBM_STENCIL_CENTRAL5, MODE, QG, K, LN>(L);
  }
  return launch_k_steps<S, LBM_STENCIL_ISO9, MODE, QG, K, LN>(L);
}

template <typename S, int MODE, int QG, int LN>
static hipError_t launch_k(const Launch& L, int k) {
  constexpr int most = ms_most_steps(sizeof(S), MODE != kClosureOff, QG);
  if constexpr (most >= 4) {
    if (k == 4) return launch_k_stencil<S, MODE, QG, 4, LN>(L);
  }
  if constexpr (most >= 3) {
    if (k == 3) return launch_k_stencil<S, MODE, QG, 3, LN>(L);
  }
  return k == 2 ? launch_k_stencil<S, MODE, QG, 2, LN>(L) : hipErrorInvalidValue;
}

// Closure off: rows loaded three ahead, by groups of 64 (FP64) or 128 columns whose
// waves have the registers for it, on small grids, where a few rows per workgroup wait
// for their loads (128^2 FP64 3.75 -> 2.8 us per step, 256^2 5.06 -> 3.98, 512^2
// 7.96 -> 6.9, FP32 256^2 3.6 -> 3.3, BF16 384^2 4.8 -> 4.25; 512^2 FP32 4.61
// against 4.88, 724^2 BF16 6.92 against 7.11).  The closure's rows wait for its arithmetic
// instead (64^2 FP32, three steps 6.0 us each either way).
template <typename S, int QG>
static hipError_t launch_dns(const Launch& L, int k) {
  if (int64_t(L.nx) * L.ny < dns_deep_cells(sizeof(S))) return launch_k<S, kClosureOff, QG, sizeof(S) == 8 ? 64 : 128>(L, k);
  return launch_k<S, kClosureOff, QG, 256>(L, k);
}

template <typename S>
static hipError_t launch_steps_typed(const Launch& L, int k) {
  constexpr int LN = sizeof(S) == 8 ? 128 : 256;  // closure on
  if constexpr (sizeof(S) >= 4) {
    if (L.qg == 9) {
      if (L.k2 == 0.0) return launch_dns<S, 9>(L, k);
      return L.full ? launch_k<S, kClosureFull, 9, LN>(L, k) : launch_k<S, kClosurePlain, 9, LN>(L, k);
    }
  }
  if (L.k2 == 0.0) return launch_dns<S, 5>(L, k);
  return L.full ? launch_k<S, kClosureFull, 5, LN>(L, k) : launch_k<S, kClosurePlain, 5, LN>(L, k);
}

}  // namespace lbm
