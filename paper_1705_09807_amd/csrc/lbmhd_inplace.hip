// In-place schedule (one buffer): sweeps that advance two or four timesteps per
// launch, from an even time.
//
// A one-step sweep of the in-place schedule reads and writes the state once per step
// (with synchronous gradients it reads it twice and moves the moment planes), and
// is bound by that.  At even times slot q of cell x holds f_q(x), so an even
// number of steps maps that layout to itself: the sweeps of lbmhd_steps.h keep the
// states between the steps on the chip here too.  What is left is that a
// workgroup reads, and recomputes, cells at the edges of its block that its neighbours
// overwrite in the same launch.  A small launch before the sweep copies those
// cells: 2 H columns at every boundary between strips and 2 H rows at every
// boundary between segments, H being the sweep's recomputed cells at each side.
// The sweep then reads from the buffer only cells at least one inside its own
// block, and writes slots of cells at most one outside it (the last step's
// streaming): no slot is read by one workgroup and written by another.  Within a
// workgroup a row is stored two or more iterations after the rows it touches were
// read, behind a barrier.  The copies lie in the work buffer, in the room of five
// FP64 planes that an in-place context has for them (one-step sweeps run where that
// is too little).
//
// The results equal those of one-step sweeps bit for bit.
#include <algorithm>

#include "lbmhd_steps.h"

namespace lbm {

// Copies of the cells at the edges of the blocks, for a field of NQ values per cell with
// element (x, y, q) of the buffer at y * row + q * plane + x:
//   rows: 2 H lattice rows of NQ x pitch elements per segment, from row y0 - H on;
//   cols: 2 H elements per strip, lattice row and q, from column x0 - H on.
struct EdgeShape {
  int nx, ny, w, ry, h;
  uint32_t strips, segs;
};

// One element of the copies per thread.
template <typename T, int NQ>
__device__ __forceinline__ void save_edges(const T* src, int64_t row, int64_t plane, T* rows, T* cols, int pitch,
                                           const EdgeShape& e, uint32_t i) {
  const uint32_t h2 = 2 * e.h, nx = e.nx, ny = e.ny;
  const uint32_t nc = e.strips * ny * NQ * h2;
  if (i < nc) {
    const uint32_t j = i % h2, a = i / h2, q = a % NQ, b = a / NQ, y = b % ny, s = b / ny;
    int x = int(s) * e.w - e.h + int(j);
    x = x < 0 ? x + e.nx : (x >= e.nx ? x - e.nx : x);
    cols[i] = src[y * row + q * plane + x];
    return;
  }
  i -= nc;
  const uint32_t x = i % nx, a = i / nx, q = a % NQ, b = a / NQ, j = b % h2, s = b / h2;
  if (s >= e.segs) return;
  int y = int(s) * e.ry - e.h + int(j);
  y = y < 0 ? y + e.ny : (y >= e.ny ? y - e.ny : y);
  rows[int64_t(b * NQ + q) * pitch + x] = src[y * row + q * plane + x];
}
static uint64_t edge_elems(const EdgeShape& e, int nq) {
  return uint64_t(2 * e.h) * nq * (uint64_t(e.strips) * e.ny + uint64_t(e.segs) * e.nx);
}

// Populations (blocks below `pb`) and, with lagged gradients, the moment planes.
template <typename S, bool LAGGED>
__global__ void __launch_bounds__(256)
k_aa_edges(const S* A, const typename ComputeOf<S>::type* mb, int pitch, EdgeShape e, S* prows, S* pcols,
           typename ComputeOf<S>::type* mrows, typename ComputeOf<S>::type* mcols, uint32_t pb) {
  if (!LAGGED || blockIdx.x < pb)
    save_edges<S, kQ>(A, int64_t(kQ) * pitch, pitch, prows, pcols, pitch, e, blockIdx.x * 256 + threadIdx.x);
  else
    save_edges<typename ComputeOf<S>::type, 4>(mb, e.nx, int64_t(e.nx) * e.ny, mrows, mcols, e.nx, e,
                                               (blockIdx.x - pb) * 256 + threadIdx.x);
}

// Where a lane finds its column of such a field: per-lane bases and strides, so that a
// row is NQ loads without a branch.
template <typename T, int NQ>
struct LaneField {
  const char* base;            // element (column, row 0, q 0): the buffer's, or a column copy's
  uint32_t row, plane;         // bytes to the next lattice row / q of `base`
  const char *below, *above;   // its element in the row copies, of rows y0 - H and y1 - H
  uint32_t crow, cplane;       // bytes to the next row / q of the row copies
  int y0, y1, h;

  __device__ __forceinline__ LaneField(const T* src, uint32_t row_, int64_t plane_, const T* rows, const T* cols,
                                       int pitch, const EdgeShape& e, const MsTile& t) {
    y0 = t.y0, y1 = t.y1, h = e.h;
    const int xl = min(t.x0 - h + t.lane, t.x1 - 1 + h);
    const int x = xl < 0 ? xl + e.nx : (xl >= e.nx ? xl - e.nx : xl);
    const bool left = xl <= t.x0, edge = left || xl >= t.x1 - 1;
    const uint32_t s = uint32_t(t.x0) / uint32_t(e.w);
    const uint32_t sb = left ? s : (s + 1 == e.strips ? 0 : s + 1);
    const int j = xl - ((left ? t.x0 : t.x1) - h);
    const uint32_t es = uint32_t(sizeof(T)), h2 = 2 * h;
    base = edge ? reinterpret_cast<const char*>(cols + (int64_t(sb) * e.ny * NQ * h2 + j))
                : reinterpret_cast<const char*>(src + x);
    row = edge ? NQ * h2 * es : row_ * es;
    plane = edge ? h2 * es : uint32_t(plane_) * es;
    const uint32_t g = uint32_t(t.y0) / uint32_t(e.ry), gn = g + 1 == e.segs ? 0 : g + 1;
    crow = uint32_t(NQ) * pitch * es;
    cplane = uint32_t(pitch) * es;
    below = reinterpret_cast<const char*>(rows + x) + int64_t(g * h2) * crow;
    above = reinterpret_cast<const char*>(rows + x) + int64_t(gn * h2) * crow;
  }
  // f(q, value) of row y, y0 - H <= y < y1 + H
  template <typename F>
  __device__ __forceinline__ void load(int y, F&& f) const {
    const bool lo = y <= y0, copy = lo || y >= y1 - 1;
    const char* p = copy ? (lo ? below : above) + int64_t(y - ((lo ? y0 : y1) - h)) * crow : base + int64_t(y) * row;
    const uint64_t step = copy ? cplane : plane;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      f(q, *reinterpret_cast<const T*>(p));
      p += step;
    }
  }
};

// Populations of row y after the last step, streamed: slot q of cell x + c_q.
template <typename S>
__device__ __forceinline__ void aa_scatter(S* A, uint32_t pq, const MsTile& t, int y, int ny, bool owner,
                                           const Cols& cx, const typename ComputeOf<S>::type* v) {
  const bool mine = y >= t.y0 && y < t.y1;
  const int yc = mine ? y : t.y0;
  const uint32_t rowb = uint32_t(kQ) * pq;
  char* b = reinterpret_cast<char*>(A);
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(b + int64_t(yc == 0 ? ny - 1 : yc - 1) * rowb, rowb);
  const __amdgpu_buffer_rsrc_t rc = row_rsrc(b + int64_t(yc) * rowb, rowb);
  const __amdgpu_buffer_rsrc_t rn = row_rsrc(b + int64_t(yc + 1 == ny ? 0 : yc + 1) * rowb, rowb);
  const bool st = owner && mine;
  const uint32_t xc = st ? cx.c : kDropOffset, xe = st ? cx.e : kDropOffset, xw = st ? cx.w : kDropOffset;
#pragma unroll
  for (int q = 0; q < kQ; ++q)
    buf_store<S, false>(narrow<S>(v[q]), qcy(q) > 0 ? rn : (qcy(q) < 0 ? rs : rc),
                        qcx(q) > 0 ? xe : (qcx(q) < 0 ? xw : xc), uint32_t(q) * pq);
}

// Closure off: dns_march.
template <typename S, int K, int LN>
__global__ void __launch_bounds__(LN* K)
k_aa_dns_steps(S* A, const S* rows, const S* cols, EdgeShape e, int pitch, Rates<typename ComputeOf<S>::type> r) {
  using C = typename ComputeOf<S>::type;
  constexpr int H = K - 1;
  extern __shared__ __attribute__((aligned(16))) char ms_lds[];
  const MsTile t = ms_tile(e.nx, e.ny, e.w, e.ry, K);
  const LaneField<S, kQ> f(A, kQ * pitch, pitch, rows, cols, pitch, e, t);
  const Cols cx = cols_of<S>(ms_column(t, H, e.nx), e.nx);
  const bool owner = ms_owner(t, H);
  const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S));
  dns_march<S, 5, K, LN, 1>(
      *reinterpret_cast<DnsLds<S, 5, K, LN>*>(ms_lds), t, false, r,
      [&](int y, RawCell<S, 5>& c) __attribute__((always_inline)) { f.load(y, [&](int q, S v) { c.v[q] = v; }); },
      [&](int y, const C* v) __attribute__((always_inline)) { aa_scatter<S>(A, pq, t, y, e.ny, owner, cx, v); });
}

// Closure on, gradients of the same step: les_march.
template <typename S, int STENCIL, int LN>
__global__ void __launch_bounds__(LN * 2)
k_aa_les_steps(S* A, const S* rows, const S* cols, EdgeShape e, int pitch, Rates<typename ComputeOf<S>::type> r) {
  using C = typename ComputeOf<S>::type;
  constexpr int H = 3;
  extern __shared__ __attribute__((aligned(16))) char ms_lds[];
  const MsTile t = ms_tile(e.nx, e.ny, e.w, e.ry, 2);
  const LaneField<S, kQ> f(A, kQ * pitch, pitch, rows, cols, pitch, e, t);
  const Cols cx = cols_of<S>(ms_column(t, H, e.nx), e.nx);
  const bool owner = ms_owner(t, H);
  const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S));
  les_march<S, STENCIL, kClosurePlain, 5, 2, LN>(
      *reinterpret_cast<LesLds<S, kClosurePlain, 5, 2, LN>*>(ms_lds), t, r,
      [&](int y, RawCell<S, 5>& c) __attribute__((always_inline)) { f.load(y, [&](int q, S v) { c.v[q] = v; }); },
      [&](int y, const C* v) __attribute__((always_inline)) { aa_scatter<S>(A, pq, t, y, e.ny, owner, cx, v); });
}

// Closure on, gradients of the step before (lagged): two steps, t and t + 1.  Group 0
// takes its gradients from the moment planes of t - 1 (a ring of three rows) and puts the
// moments of t into a ring of six, of which group 1, four rows behind, takes its
// gradients; group 1 writes the moments of t + 1 over the planes.  In iteration i
//  first half:  group 0 puts row i of both rings; group 1 gathers row i - 3 and
//               writes its moments;
//  second half: group 0 collides row i - 1 and hands it on, group 1 collides and
//               stores row i - 4.
// H = 2: one column for the streaming, one for the gradients of the first step.
template <typename S, int LN>
struct LaggedLds {
  using C = typename ComputeOf<S>::type;
  struct alignas(4 * sizeof(C)) Quad {
    C v[4];
  };
  Quad prev[3][LN + 2];  // moments of t - 1 by row mod 3
  Quad mom[6][LN + 2];   // moments of t by row mod 6
  S pop[kMsRows<5>][LN + 2];
};

//
// LATE: row i + 2 is loaded after the collision of row i - 1, into its registers,
// not row i + 1 at the start of iteration i, so that the loads run beside the
// other group's stores of populations and not of planes.
template <typename S, int STENCIL, bool LATE, int LN>
__global__ void __launch_bounds__(LN * 2)
k_aa_lagged_steps(S* A, typename ComputeOf<S>::type* mb, const S* rows, const S* cols,
                  const typename ComputeOf<S>::type* mrows, const typename ComputeOf<S>::type* mcols, EdgeShape e,
                  int pitch, Rates<typename ComputeOf<S>::type> r) {
  using C = typename ComputeOf<S>::type;
  using Lds = LaggedLds<S, LN>;
  using Quad = typename Lds::Quad;
  constexpr int H = 2;
  extern __shared__ __attribute__((aligned(16))) char ms_lds[];
  Lds& lds = *reinterpret_cast<Lds*>(ms_lds);
  const MsTile t = ms_tile(e.nx, e.ny, e.w, e.ry, 2);
  const int l = t.lane + 1;
  const int first = t.y0 - H, last = t.y1 - 1 + H;  // rows of the first step's gradients
  const int end = t.y1 + 4;                         // iterations first .. end - 1

  auto collide = [&](const Quad* ss, const Quad* sc, const Quad* sn, C* v) __attribute__((always_inline)) {
    const Mom<C> m = moments_of<5, kUnits<S>>(v);
    C gr[4][2];
    constexpr int kAtOnce = sizeof(C) == 8 ? 2 : 4;  // FP64: as many fields as there are registers
#pragma unroll
    for (int k0 = 0; k0 < 4; k0 += kAtOnce) {
#pragma unroll
      for (int k = k0; k < k0 + kAtOnce; ++k)
        grad3x3<C, STENCIL>(sc[l + 1].v[k], sc[l - 1].v[k], sn[l].v[k], ss[l].v[k], sn[l + 1].v[k], sn[l - 1].v[k],
                            ss[l + 1].v[k], ss[l - 1].v[k], gr[k][0], gr[k][1]);
      if constexpr (kAtOnce < 4) __builtin_amdgcn_sched_barrier(0);
    }
    const C ir = C(1) / (r.rho0 + m.drho);
    const Closure<C> cl =
        closure_terms(gr[0][0], gr[0][1], gr[1][0], gr[1][1], gr[2][0], gr[2][1], gr[3][0], gr[3][1], ir, r.k2);
    collide_q<5, true, false, kUnits<S>>(v, m, cl, r);
  };
  // slot of population q (i mod 3 = u, i mod 2 = par), and of row i in the ring of six
  auto slot = [](int q, int u, int par) { return ms_row<5>(q) + (qcy(q) > 0 ? u : (qcy(q) == 0 ? par : 0)); };
  auto six = [](int u, int par) { return u + 3 * par; };
  using N0 = std::integral_constant<int, 0>;
  using N1 = std::integral_constant<int, 1>;
  using N2 = std::integral_constant<int, 2>;

  if (t.step == 0) {
    const LaneField<S, kQ> f(A, kQ * pitch, pitch, rows, cols, pitch, e, t);
    const LaneField<C, 4> fm(mb, e.nx, int64_t(e.nx) * e.ny, mrows, mcols, e.nx, e, t);
    RawCell<S, 5> raw[3];
    Quad pm[3];
    auto load = [&](int y, RawCell<S, 5>& c, Quad& m) __attribute__((always_inline)) {
      f.load(y, [&](int q, S v) { c.v[q] = v; });
      fm.load(y, [&](int q, C v) { m.v[q] = v; });
    };
    auto iter = [&](int i, int par, auto uc) __attribute__((always_inline)) {
      constexpr int u0 = decltype(uc)::value, u1 = (u0 + 2) % 3, u2 = (u0 + 1) % 3;  // rows i, i - 1, i - 2
      if constexpr (!LATE) {
        load(min(i + 1, last), raw[u2], pm[u2]);
        __builtin_amdgcn_sched_barrier(0);
      }
      C v[kQ];
      widen_raw<S, C, 5>(raw[u0], v);
      const Mom<C> m = moments_of<5, kUnits<S>>(v);
      lds.prev[u0][l] = pm[u0];
      lds.mom[six(u0, par)][l] = Quad{m.mx, m.my, m.dbx, m.dby};
      __syncthreads();
      widen_raw<S, C, 5>(raw[u1], v);
      collide(lds.prev[u2], lds.prev[u1], lds.prev[u0], v);
      if constexpr (LATE) {
        __builtin_amdgcn_sched_barrier(0);
        load(min(i + 2, last), raw[u1], pm[u1]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < kQ; ++q) lds.pop[slot(q, u0, par)][l] = narrow<S>(v[q]);
      __syncthreads();
    };
    load(first, raw[0], pm[0]);
    if constexpr (LATE) load(first + 1, raw[1], pm[1]);
    for (int i = first, par = 0; i < end; i += 3, par ^= 1) {  // past `end`: nothing is stored
      iter(i, par, N0{});
      iter(i + 1, par ^ 1, N1{});
      iter(i + 2, par, N2{});
    }
  } else {
    const int x = ms_column(t, H, e.nx);
    const Cols cx = cols_of<S>(x, e.nx);
    const bool owner = ms_owner(t, H);
    const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S)), mrow = uint32_t(e.nx) * uint32_t(sizeof(C));
    const int64_t n = int64_t(e.nx) * e.ny;
    C vs[3][kQ];  // rows gathered and not yet collided
    auto iter = [&](int i, int par, auto uc) __attribute__((always_inline)) {
      constexpr int u0 = decltype(uc)::value, u1 = (u0 + 2) % 3, u2 = (u0 + 1) % 3;  // rows i - 3, i - 4, i - 5
#pragma unroll
      for (int q = 0; q < kQ; ++q) vs[u0][q] = widen<C>(lds.pop[slot(q, u0, par)][l - qcx(q)]);
      const Mom<C> m = moments_of<5, kUnits<S>>(vs[u0]);
      const int y = i - 3;
      const bool mine = y >= t.y0 && y < t.y1;
      const uint32_t xo = owner && mine ? uint32_t(x) * uint32_t(sizeof(C)) : kDropOffset;
      const C mv[4] = {m.mx, m.my, m.dbx, m.dby};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        buf_store<C, false>(mv[k], row_rsrc(mb + k * n + int64_t(mine ? y : t.y0) * e.nx, mrow), xo, 0);
      __syncthreads();
      C v[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) v[q] = vs[u1][q];
      collide(lds.mom[six(u2, par ^ 1)], lds.mom[six(u1, par)], lds.mom[six(u0, par ^ 1)], v);
      aa_scatter<S>(A, pq, t, i - 4, e.ny, owner, cx, v);
      __syncthreads();
    };
    for (int i = first, par = 0; i < end; i += 3, par ^= 1) {
      iter(i, par, N0{});
      iter(i + 1, par ^ 1, N1{});
      iter(i + 2, par, N2{});
    }
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// Blocks of the sweep, and the copies' places in the work buffer; false where the copies
// do not fit.
struct InplacePlan {
  EdgeShape e;
  int lanes, blocks;
  size_t prows, pcols, mrows, mcols;  // bytes from off_edges
};
static bool inplace_plan(const Launch& L, int k, InplacePlan& p) {
  const bool les = L.k2 != 0.0, lagged = les && L.schedule == LBM_SCHED_AA_LAGGED;
  const size_t es = storage_bytes(L.dtype), cs = es == 8 ? 8 : 4;
  const int h = !les ? k - 1 : (lagged ? 2 : 3);
  const MsShape s = ms_shape(L, h, es == 8 && les ? 128 : 256, 1);
  p.lanes = s.lanes;
  const int strips = (L.nx + s.w - 1) / s.w;
  // one workgroup per compute unit; two where the arithmetic of 16-bit storage is the bound
  // (BF16 4096^2 237 us per step against 306; FP32 346 against 303, FP64 693 against 616)
  for (int ry = es == 2 && les && !lagged ? (s.ry + 1) / 2 : s.ry;; ry *= 2) {
    ry = std::min(ry, L.ny);
    const int segs = (L.ny + ry - 1) / ry;
    p.e = EdgeShape{L.nx, L.ny, s.w, ry, h, uint32_t(strips), uint32_t(segs)};
    p.blocks = strips * segs;
    const size_t row = size_t(segs) * 2 * h, col = size_t(strips) * L.ny * 2 * h;
    p.prows = 0;
    p.pcols = p.prows + up256(row * kQ * size_t(L.pitch) * es);
    p.mrows = p.pcols + up256(col * kQ * es);
    p.mcols = p.mrows + (lagged ? up256(row * 4 * L.nx * cs) : 0);
    const size_t bytes = p.mcols + (lagged ? up256(col * 4 * cs) : 0);
    // the thread index and the offsets of a lane's field are 32-bit
    if (bytes <= L.off_part - L.off_edges && edge_elems(p.e, kQ) < (1ull << 31) &&
        uint64_t(L.nx) * L.ny * cs < (1ull << 32))
      return true;
    if (ry == L.ny) return false;
  }
}

// Below these sizes the one-step sweeps stay: the state then lives in the caches, few
// workgroups march and the copies are a launch of their own.  Measured, us per step,
// several steps against one (closure off / synchronous / lagged gradients): FP32
// 850^2 16.3/29.5/23.0 against 17.6/30.5/21.9, 1000^2 18.2/33.5/28.0 against 23.2/39.7/28.5,
// 1024^2 19.1/37.6/27.0 against 23.9/40.5/29.4, 1448^2 25.0/50.2/44.2 against
// 46.0/78.2/56.4, 4096^2 157/301/368 against 449/768/556; FP64 512^2 16.4/50.9/40.6
// against 12.8/23.0/16.7, 1024^2 32.0/52.6/43.7 against 45.7/78.6/57.1, 4096^2
// 555/617/787 against 898/1527/1111; 16-bit 2048^2 47.5/80.3/68.7 against 44.8/86.1/97.0
// (BF16), 2900^2 82.0/136.9/124.2 against 113.9/252.5/204, 4096^2 154/241/240 against
// 229/473/368.  Narrow strips, whose copied and recomputed columns are many to those
// stored, stay too: FP32 64 x 24000 42.0/89.8/61.9 against 33.2/61.7/44.0, 128 x 9000
// -/49.7/32.9 against -/45.0/31.8 (128 x 20000 41.2/89.5/72.9 against 55.0/93.7/91.9), FP64
// 64 x 16000 48.7/75.0/60.0 against 44.2/77.0/54.0, BF16 synchronous 128 x 32768 117 against
// 98 (200 x 32768 129 against 232).  Two steps with the closure off, where four would fit:
// FP32 1024^2 21.5 against 23.9, 128 x 20000 61.6 against 55.0; 16-bit 2900^2 123 against 113
// (FP16), 4096^2 236 against 229 (BF16).
InplaceSteps multi_steps_inplace(const Launch& L) {
  InplacePlan p;
  const int64_t cells = int64_t(L.nx) * L.ny;
  const size_t bytes = storage_bytes(L.dtype);
  const bool les = L.k2 != 0.0;
  const int64_t least = bytes >= 4 ? 1000000 : (les ? 4000000 : 8000000);
  if (cells < least || L.nx < 16 || L.ny < 16 || !inplace_plan(L, 2, p)) return {1, 1};
  const bool wide = p.e.w >= 160;
  if (bytes == 4 && cells < 1500000 && !wide) return {1, 1};
  if (bytes == 2 && les && L.schedule == LBM_SCHED_AA && !wide) return {1, 1};
  if (p.e.w < 80) return {1, 1};
  if (les || bytes == 8) return {2, 2};
  const int most = inplace_plan(L, 4, p) ? 4 : 2;
  return {bytes == 4 && wide ? 2 : most, most};
}

template <typename S, bool LAGGED, int K, int LN, typename Kernel>
static hipError_t launch_inplace(const Launch& L, Kernel kernel, size_t lds) {
  using C = typename ComputeOf<S>::type;
  InplacePlan p;
  if (!inplace_plan(L, K, p)) return hipErrorInvalidValue;
  char* w = static_cast<char*>(L.work) + L.off_edges;
  S* prows = reinterpret_cast<S*>(w + p.prows);
  S* pcols = reinterpret_cast<S*>(w + p.pcols);
  C* mrows = reinterpret_cast<C*>(w + p.mrows);
  C* mcols = reinterpret_cast<C*>(w + p.mcols);
  S* A = static_cast<S*>(L.state);
  C* mb = reinterpret_cast<C*>(static_cast<char*>(L.work) + L.off_mb);  // set 0: the sweep starts at an even time
  const uint32_t pb = uint32_t((edge_elems(p.e, kQ) + 255) / 256);
  const uint32_t mblk = LAGGED ? uint32_t((edge_elems(p.e, 4) + 255) / 256) : 0;
  hipLaunchKernelGGL((k_aa_edges<S, LAGGED>), dim3(pb + mblk), dim3(256), 0, L.stream, A, mb, int(L.pitch), p.e, prows,
                     pcols, mrows, mcols, pb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (lds > 64 * 1024) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            int(lds));
    if (e != hipSuccess) return e;
  }
  if constexpr (LAGGED)
    hipLaunchKernelGGL(kernel, dim3(p.blocks), dim3(p.lanes * K), lds, L.stream, A, mb, prows, pcols, mrows, mcols,
                       p.e, int(L.pitch), make_rates<C>(L));
  else
    hipLaunchKernelGGL(kernel, dim3(p.blocks), dim3(p.lanes * K), lds, L.stream, A, prows, pcols, p.e, int(L.pitch),
                       make_rates<C>(L));
  return hipGetLastError();
}

template <typename S>
static hipError_t launch_inplace_typed(const Launch& L, int k) {
  constexpr int LN = sizeof(S) == 8 ? 128 : 256;  // closure on
  if (L.k2 == 0.0) {
    if constexpr (sizeof(S) < 8) {  // FP64 does not fit the LDS
      constexpr size_t lds = sizeof(DnsLds<S, 5, 4, 256>);
      static_assert(lds <= 160 * 1024, "LDS of a compute unit");
      if (k == 4) return launch_inplace<S, false, 4, 256>(L, &k_aa_dns_steps<S, 4, 256>, lds);
    }
    return launch_inplace<S, false, 2, 256>(L, &k_aa_dns_steps<S, 2, 256>, sizeof(DnsLds<S, 5, 2, 256>));
  }
  if (L.schedule == LBM_SCHED_AA_LAGGED) {
    constexpr size_t lds = sizeof(LaggedLds<S, LN>);
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    // late loads beyond the caches, with storage of 4 and 8 bytes (4096^2 FP32 368 us per step
    // against 404, FP64 787 against 854, 3000^2 FP32 201 against 206; 2048^2 FP32 96
    // against 88, 4096^2 BF16 262 against 239)
    auto go = [&](auto late) {
      constexpr bool LATE = decltype(late)::value;
      if (L.stencil == LBM_STENCIL_ISO9)
        return launch_inplace<S, true, 2, LN>(L, &k_aa_lagged_steps<S, LBM_STENCIL_ISO9, LATE, LN>, lds);
      return launch_inplace<S, true, 2, LN>(L, &k_aa_lagged_steps<S, LBM_STENCIL_CENTRAL5, LATE, LN>, lds);
    };
    if constexpr (sizeof(S) >= 4) {
      if (int64_t(L.nx) * L.ny * kQ * int(sizeof(S)) >= (512 << 20)) return go(std::true_type{});
    }
    return go(std::false_type{});
  }
  constexpr size_t lds = sizeof(LesLds<S, kClosurePlain, 5, 2, LN>);
  switch (L.stencil) {
    case LBM_STENCIL_ISO9: return launch_inplace<S, false, 2, LN>(L, &k_aa_les_steps<S, LBM_STENCIL_ISO9, LN>, lds);
    case LBM_STENCIL_CENTRAL5:
      return launch_inplace<S, false, 2, LN>(L, &k_aa_les_steps<S, LBM_STENCIL_CENTRAL5, LN>, lds);
    case LBM_STENCIL_LOCAL_ISO9:
      return launch_inplace<S, false, 2, LN>(L, &k_aa_les_steps<S, LBM_STENCIL_LOCAL_ISO9, LN>, lds);
    default: return launch_inplace<S, false, 2, LN>(L, &k_aa_les_steps<S, LBM_STENCIL_LOCAL_CENTRAL5, LN>, lds);
  }
}

hipError_t launch_steps_inplace(const Launch& L, int k) {
  switch (L.dtype) {
    case LBM_FP64: return launch_inplace_typed<double>(L, k);
    case LBM_FP32: return launch_inplace_typed<float>(L, k);
    case LBM_FP16: return launch_inplace_typed<_Float16>(L, k);
    default: return launch_inplace_typed<__bf16>(L, k);
  }
}

}  // namespace lbm
