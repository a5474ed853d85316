// HIP kernels (gfx950) of the filtered lattice-Boltzmann MHD timestep.
//
// Method: Flint & Vahala, arXiv 1705.09807.  Sec. 2: kinetic equations
// (LBKinEqn, LBMagEqn), equilibria (feq, geq), moment transform
// (FluidTMatrix), equilibrium moments (KinMomentEq, MagMomentEq), transport
// coefficients; Sec. 2.1: filtered equilibrium moments built from the
// Delta-expansion FilterExampleSmall; Sec. 3: SRT runs, density gradients
// dropped (simplified M3).
//
// Storage: structure of arrays by lattice row.  Lattice row y holds the 19
// population rows f_0..f_8, g_x0..g_x4, g_y0..g_y4 (x fastest) one after
// another, each padded to a multiple of 64 elements.  FP32 stores f as the deviation
// f_i - w_i rho0 from the rest equilibrium, so that the small dynamic part
// keeps its digits; FP64 stores f itself (rho0 = 0 below); g is stored as is.
//
// Two schedules:
//  * fused (two buffers, pull streaming): a buffer holds post-collision
//    populations at their source cell; a sweep gathers f_q(x) from x - c_q
//    (loads shifted by at most one cell), collides and stores aligned rows.
//    With the closure on, one workgroup marches up a column strip and keeps
//    a 4-row ring of moments in LDS, so the 3x3 gradient stencil costs no
//    extra HBM pass.
//  * AA (one buffer, in place): even steps read and write the cell's own
//    slots (reversed), odd steps read from and write to the neighbours; the
//    read set of a cell equals its write set, so cells never race.  With the
//    closure on, a moment sweep writes m and B to four planes first.
//
// All arithmetic that defines the method (moments, closure, collision) lives
// in the __device__ functions of lbmhd_cell.h and lbmhd_device.h and is shared
// by every kernel, so all schedules with the same gradients compute identical values
// (but for the last bits of 16-bit runs without closure: swapped_rest).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "lbmhd_cell.h"
#include "lbmhd_device.h"
#include "lbmhd_internal.h"
#include "lbmhd_learned.h"
#include "lbmhd_mlp_device.h"

namespace lbm {

// Closure off (Delta = 0).  One row segment of 2 * 128 cells per workgroup,
// two cells per thread, aligned two-element stores.  Requires nx even.
// Measured against 64- and 256-thread segments and two rows per workgroup at
// 4096^2 and 8192^2 FP32: 0.4-4 % faster than each.
template <typename S, typename C, bool NT, int QG>
__global__ void __launch_bounds__(128)
k_fused_dns_pair(const S* __restrict__ src, S* __restrict__ dst, int nx, int ny, int64_t pitch, Rates<C> r) {
  using nv2 = Vec2<S>;
  const int x = (blockIdx.x * 128 + threadIdx.x) * 2;
  const int y = blockIdx.y;
  if (x >= nx) return;
  const Rows rw = rows_of<S, QG>(y, ny, pitch);
  C a[kPop<QG>], b[kPop<QG>];
  pull_pair<S, C, QG>(src, pitch, nx, rw, x, a, b);
  const Closure<C> cl = {C(0), C(0), C(0), C(0)};
  {
    const Mom<C> m = moments_of<QG, kUnits<S>>(a);
    collide_q<QG, false, false, kUnits<S>>(a, m, cl, r);
  }
  {
    const Mom<C> m = moments_of<QG, kUnits<S>>(b);
    collide_q<QG, false, false, kUnits<S>>(b, m, cl, r);
  }
  const uint32_t xo = uint32_t(x) * uint32_t(sizeof(S));
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) {
    nv2 t;
    t.x = narrow<S>(a[q]);
    t.y = narrow<S>(b[q]);
    store<NT>(reinterpret_cast<nv2*>(at(dst + q * pitch, rw.c, xo)), t);
  }
}


// Closure off, any nx: one cell per thread, row segments of 256 cells.
template <typename S, typename C, bool NT, int QG>
__global__ void __launch_bounds__(256)
k_fused_dns(const S* __restrict__ src, S* __restrict__ dst, int nx, int ny, int64_t pitch, Rates<C> r) {
  const int x = blockIdx.x * 256 + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= nx) return;
  const Rows rw = rows_of<S, QG>(y, ny, pitch);
  const Cols cl = cols_of<S>(x, nx);
  C v[kPop<QG>];
  pull_cell<S, C, QG>(src, pitch, rw, cl, v);
  const Mom<C> m = moments_of<QG, kUnits<S>>(v);
  const Closure<C> zero = {C(0), C(0), C(0), C(0)};
  collide_q<QG, false, false, kUnits<S>>(v, m, zero, r);
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) store<NT>(at(dst + q * pitch, rw.c, cl.c), narrow<S>(v[q]));
}

// Closure off, 16-bit storage, nx a multiple of 4: four cells per thread, so
// every population moves in one aligned 8-byte load and store per thread (plus
// one 2-byte load of the neighbour column for those that stream along x),
// addressed through a resource per lattice row.  Measured 7-9 % faster than
// two cells per thread at 8192^2 with FP16 and BF16 storage (slower with FP32,
// whose pair loads are already 8 bytes), and the buffer form 0-4 % faster
// than per-lane addresses (BF16 8192^2 884-893 against 901-916 us; for the
// FP32 pair kernel it measured up to 3 % slower, so that one keeps them).
template <typename S, typename C, bool NT>
__global__ void __launch_bounds__(64)
k_fused_dns_quad(const S* __restrict__ src, S* __restrict__ dst, int nx, int ny, int64_t pitch, Rates<C> r) {
  using V4 = Vec4<S>;
  const int nseg = (nx + 255) / 256;  // row segments of 256 cells
  const int vb = xcd_contiguous(blockIdx.x, gridDim.x);
  const int x = ((vb % nseg) * 64 + threadIdx.x) * 4;
  const int y = vb / nseg;
  if (x >= nx) return;
  const uint32_t es = uint32_t(sizeof(S)), pq = uint32_t(pitch) * es, rowb = uint32_t(kQ) * pq;
  const char* b = reinterpret_cast<const char*>(src);
  const int ys = y == 0 ? ny - 1 : y - 1, yn = y + 1 == ny ? 0 : y + 1;
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(b + int64_t(ys) * rowb, rowb);
  const __amdgpu_buffer_rsrc_t rc = row_rsrc(b + int64_t(y) * rowb, rowb);
  const __amdgpu_buffer_rsrc_t rn = row_rsrc(b + int64_t(yn) * rowb, rowb);
  const uint32_t x0 = uint32_t(x) * es;
  const uint32_t xw = uint32_t(x == 0 ? nx - 1 : x - 1) * es;
  const uint32_t x4 = uint32_t(x + 4 == nx ? 0 : x + 4) * es;
  V4 in[kQ];
  S edge[kQ];  // the neighbour column's value of the populations that stream along x
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const __amdgpu_buffer_rsrc_t rr = qcy(q) > 0 ? rs : (qcy(q) < 0 ? rn : rc);
    const uint32_t so = uint32_t(q) * pq;
    in[q] = buf_load_v<V4>(rr, x0, so);
    if (qcx(q) != 0) edge[q] = buf_load<S>(rr, qcx(q) > 0 ? xw : x4, so);
  }
  C v[4][kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    // BF16: no value used before the last load is issued (a third of the loads are
    // otherwise moved behind the waits for the others: 1024^2 13.56 us, with them first
    // 13.14, 1500 x 1001 18.8 and 18.05, 600^2 7.1 and 6.8; FP16 12.9 as it is, 13.4 so)
    if constexpr (kUnits<S> == 1) {
      asm volatile("" : "+v"(in[q]));
      if (qcx(q) != 0) asm volatile("" : "+v"(edge[q]));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = k - qcx(q);
      v[k][q] = widen<C>(j < 0 || j > 3 ? edge[q] : in[q][j & 3]);
    }
  }
  const Closure<C> cl = {C(0), C(0), C(0), C(0)};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const Mom<C> m = moments19<kUnits<S>>(v[k]);
    collide19<false, false, kUnits<S>>(v[k], m, cl, r, swapped_rest<S>(k, 4));
  }
  const __amdgpu_buffer_rsrc_t d = row_rsrc(reinterpret_cast<char*>(dst) + int64_t(y) * rowb, rowb);
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    V4 t;
    t.x = narrow<S>(v[0][q]);
    t.y = narrow<S>(v[1][q]);
    t.z = narrow<S>(v[2][q]);
    t.w = narrow<S>(v[3][q]);
    buf_store_v<V4, NT>(t, d, x0, uint32_t(q) * pq);
  }
}

// Closure on.  A workgroup of W + 64 lanes owns the columns x0 .. x0+W-1 (W a
// multiple of 64, so every wave stores whole aligned cache lines) and marches up
// the rows y0 .. y1-1; the moment fields (m_x, m_y, B_x - B_ref, B_y - B_ref) of
// rows y-1 .. y+2 live in a 4-slot LDS ring indexed by column - x0 + 1.  Per row a
// collision lane issues the loads of row y + 2, collides and stores row y from
// the ring, puts row y + 2's moments into the ring and meets the others at the
// row's barrier (which waits for LDS only).  A ring slot is rewritten only after
// the barrier that follows its last read.  The row body has no branch around a
// memory operation: a lane past the last column loads the last column, drops its
// stores (kDropOffset) and puts its moments into a spare ring column (W + 2), so
// the compiler waits on each batch of loads alone; three register sets rotate the
// rows without copies.  The last wave gathers the two halo columns (x0 - 1 and the
// column after the strip's last cell) two rows ahead, in a loop of its own with
// the same barrier per row.  FP64 64^2 (one row per workgroup): with per-lane
// addresses, branches and the three first rows loaded one after another 5.3 us per
// step, this form 4.5; 4096^2 961 and 881, with D2Q9 and
// the density-gradient closure 1692 and 1273.
//
// MODE kClosureCorr: four FP32 planes (tau_xx, tau_xy, tau_yy, eps) of a
// learned correction are added to the analytic subgrid terms of every cell.
// MODE kClosureFull: the ring carries rho - rho0 as a fifth field and the
// closure keeps the filtered-density gradient terms.
template <typename S, int W, int STENCIL, bool NT, int MODE, int QG>
__global__ void __launch_bounds__(W + 64)
k_fused_les_f(const S* __restrict__ src, S* __restrict__ dst, int nx, int ny, int64_t pitch, int ry,
              Rates<typename ComputeOf<S>::type> r, const float* __restrict__ corr) {
  using C = typename ComputeOf<S>::type;
  constexpr int NF = MODE == kClosureFull ? 5 : 4;
  constexpr int NP = kPop<QG>;
  constexpr bool LOCAL = STENCIL >= LBM_STENCIL_LOCAL_ISO9 && QG == 5 && MODE != kClosureFull;
  __shared__ C ring[4][NF][W + 3];
  const int tid = threadIdx.x;
  const int nstrip = (nx + W - 1) / W;
  const int vb = xcd_contiguous(blockIdx.x, gridDim.x);  // strip vb % nstrip of segment vb / nstrip
  const int x0 = (vb % nstrip) * W;
  const int last = min(x0 + W, nx) - 1;  // last column of this strip
  const int y0 = (vb / nstrip) * ry;
  const int y1 = min(y0 + ry, ny);
  const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S));  // bytes between population rows
  const uint32_t rowb = uint32_t(NP) * pq;                    // bytes of a lattice row
  auto wrapy = [&](int y) { return y < 0 ? y + ny : (y >= ny ? y - ny : y); };
  auto slot = [&](int y) { return (y - y0 + 1) & 3; };  // ring slot of row y
  auto pull = [&](int y, const Cols& cx, RawCell<S, QG>& c) __attribute__((always_inline)) {
    pull_raw<S, QG>(src, pq, wrapy(y - 1), y, wrapy(y + 1), cx, c);
  };
  auto put = [&](int sl, int widx, const RawCell<S, QG>& c) __attribute__((always_inline)) {
    C v[NP];
    widen_raw<S, C, QG>(c, v);
    const Mom<C> m = moments_of<QG, kUnits<S>>(v);
    ring[sl][0][widx] = m.mx;
    ring[sl][1][widx] = m.my;
    ring[sl][2][widx] = m.dbx;
    ring[sl][3][widx] = m.dby;
    if constexpr (NF == 5) ring[sl][4][widx] = m.drho;
  };

  if (tid >= W) {
    // halo wave: lane 0 gathers the column left of the strip, the others the
    // column right of it (only lanes 0 and 1 put theirs into the ring)
    const int hl = tid - W;
    const int xc = hl == 0 ? (x0 == 0 ? nx - 1 : x0 - 1) : (last + 1 == nx ? 0 : last + 1);
    const int widx = hl == 0 ? 0 : (hl == 1 ? last - x0 + 2 : W + 2);
    const Cols cx = cols_of<S>(xc, nx);
    auto ahead = [&](int y) { return wrapy(y <= y1 ? y : y1); };  // rows past y1 are not needed
    RawCell<S, QG> ca, cb, cc;
    pull(wrapy(y0 - 1), cx, ca);
    pull(y0, cx, cb);
    pull(wrapy(y0 + 1), cx, cc);
    __builtin_amdgcn_sched_barrier(0);  // all three rows on their way first
    put(0, widx, ca);
    put(1, widx, cb);
    put(2, widx, cc);
    pull(ahead(y0 + 2), cx, ca);
    __syncthreads();
    int y = y0;
    for (; y + 2 <= y1; y += 2) {  // rows y, y + 1: put rows y + 2 and y + 3
      pull(ahead(y + 3), cx, cb);
      put(slot(y + 2), widx, ca);
      __syncthreads();
      pull(ahead(y + 4), cx, ca);
      if (y + 3 <= y1) put(slot(y + 3), widx, cb);
      __syncthreads();
    }
    if (y < y1) __syncthreads();  // row y1 - 1 needs no further row
    return;
  }

  const bool valid = x0 + tid <= last;
  const int xc = valid ? x0 + tid : last;  // idle lanes address a valid cell, never stored
  const Cols cx = cols_of<S>(xc, nx);
  const int widx = valid ? tid + 1 : W + 2;
  const uint32_t xo_store = valid ? cx.c : kDropOffset;
  const int64_t n = (int64_t)nx * ny;
  float cc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, cn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  auto load_corr = [&](int y, float (&c)[4]) __attribute__((always_inline)) {
    const int64_t ci = (int64_t)y * nx + xc;
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = corr[k * n + ci];
  };

  // Row y: rcur holds it as stored, rt receives row y + 2 (row y + 1 again
  // for the segment's last row, whose ring slot is then never read).
  auto row = [&](const RawCell<S, QG>& rcur, RawCell<S, QG>& rt, int y) __attribute__((always_inline)) {
    const bool more = y + 1 < y1;
    pull(wrapy(more ? y + 2 : y + 1), cx, rt);
    if constexpr (MODE == kClosureCorr) load_corr(more ? y + 1 : y, cn);
    // the loads stay ahead of the collision (the scheduler would otherwise
    // sink them to their use to save registers)
    __builtin_amdgcn_sched_barrier(0);
    const int sc = slot(y), sn = slot(y + 1), ss = slot(y - 1), l = tid + 1;
    C gr[NF][2];
#pragma unroll
    for (int k = 0; k < NF; ++k)
      grad3x3<C, STENCIL>(ring[sc][k][l + 1], ring[sc][k][l - 1], ring[sn][k][l], ring[ss][k][l], ring[sn][k][l + 1],
                          ring[sn][k][l - 1], ring[ss][k][l + 1], ring[ss][k][l - 1], gr[k][0], gr[k][1]);
    C cur[NP];
    widen_raw<S, C, QG>(rcur, cur);
    const Mom<C> m = moments_of<QG, kUnits<S>>(cur);
    const C ir = C(1) / (r.rho0 + m.drho);
    Closure<C> cl;
    if constexpr (MODE == kClosureFull) {
      cl = closure_terms_full(gr, m.mx, m.my, r.bx0 + m.dbx, r.by0 + m.dby, ir, r.k2);
    } else {
      if constexpr (LOCAL)
        local_gradients<kUnits<S>>(cur, m, r, gr[1][0] - gr[0][1], gr);
      cl = closure_terms<LOCAL>(gr[0][0], gr[0][1], gr[1][0], gr[1][1], gr[2][0], gr[2][1], gr[3][0], gr[3][1], ir, r.k2);
    }
    if constexpr (MODE == kClosureCorr) {
      const C txx = C(cc[0]), tyy = C(cc[2]);
      cl.tau_xy += C(cc[1]);
      cl.tau_d += txx - tyy;
      cl.tau_s += txx + tyy;
      cl.eps += C(cc[3]);
    }
    collide_q<QG, true, LOCAL, kUnits<S>>(cur, m, cl, r);
    const __amdgpu_buffer_rsrc_t d = row_rsrc(reinterpret_cast<char*>(dst) + int64_t(y) * rowb, rowb);
#pragma unroll
    for (int q = 0; q < NP; ++q) buf_store<S, NT>(narrow<S>(cur[q]), d, xo_store, uint32_t(q) * pq);
    __builtin_amdgcn_sched_barrier(0);
    put(slot(y + 2), widx, rt);
    if constexpr (MODE == kClosureCorr) {
#pragma unroll
      for (int k = 0; k < 4; ++k) cc[k] = cn[k];
    }
    __syncthreads();
  };

  RawCell<S, QG> ra, rb, rc;
  pull(wrapy(y0 - 1), cx, ra);
  pull(y0, cx, rb);
  pull(wrapy(y0 + 1), cx, rc);
  if constexpr (MODE == kClosureCorr) load_corr(y0, cc);
  __builtin_amdgcn_sched_barrier(0);  // all three rows on their way first
  put(0, widx, ra);
  put(1, widx, rb);
  put(2, widx, rc);
  __syncthreads();
  int y = y0;
  for (; y + 3 <= y1; y += 3) {  // one straight-line block of three rows
    row(rb, ra, y);
    row(rc, rb, y + 1);
    row(ra, rc, y + 2);
  }
  if (y < y1) row(rb, ra, y);
  if (y + 1 < y1) row(rc, rb, y + 1);
}

// ---------------------------------------------------------------------------
// AA schedule (one buffer, in place).
//  even t: load A[q][x],             store f*_q to A[opp q][x]
//  odd  t: load A[opp q][x - c_q],   store f*_q to A[q][x + c_q]
// Every kernel of the schedule runs one row segment of kAARow cells per
// workgroup (1-D row blocks keep each wave's accesses within DRAM rows;
// measured 1.1-1.25x faster than 64 x 4 tiles at 4096^2) and addresses a
// population row by its wave-uniform base plus a 32-bit byte offset.
// ---------------------------------------------------------------------------
constexpr int kAARow = 256;

// Row segment x0 .. x0 + kAARow - 1 of row y for this workgroup, from a
// one-dimensional grid numbered XCD-contiguously.
__device__ __forceinline__ void aa_segment(int nx, int& x0, int& y) {
  const int nseg = (nx + kAARow - 1) / kAARow;
  const int vb = xcd_contiguous(blockIdx.x, gridDim.x);
  x0 = (vb % nseg) * kAARow;
  y = vb / nseg;
}

// DECODED: in natural units, not in stored ones (for sums alone, which take the decode
// into their additions).  ORDERED: widened after the last load is issued (with 16-bit
// storage the lagged sweep's loads are otherwise moved behind the waits for the others:
// FP16 1024^2 20.8 us, ordered 19.8; BF16 64^2 4.57 and 4.06, 1024^2 21.4 and 19.7, 4096^2 443
// and 368; FP32 and FP64 the same either way).
template <typename S, typename C, bool ODD, bool DECODED = false, bool ORDERED = false>
__device__ __forceinline__ void aa_load(const S* __restrict__ A, int64_t pitch, const Rows& rw, const Cols& cl,
                                        C v[kQ]) {
  S raw[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if (!ODD) {
      raw[q] = *at(A + q * pitch, rw.c, cl.c);
    } else {
      const uint32_t xo = qcx(q) > 0 ? cl.w : (qcx(q) < 0 ? cl.e : cl.c);  // x - c_q
      const int64_t yo = qcy(q) > 0 ? rw.s : (qcy(q) < 0 ? rw.n : rw.c);
      raw[q] = *at(A + qopp(q) * pitch, yo, xo);
    }
    if (!ORDERED) v[q] = DECODED ? decode<C>(raw[q]) : widen<C>(raw[q]);
  }
  if constexpr (ORDERED) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      asm volatile("" : "+v"(raw[q]));
      v[q] = widen<C>(raw[q]);
    }
  }
}

template <typename S, typename C, bool ODD>
__device__ __forceinline__ void aa_store(S* __restrict__ A, int64_t pitch, const Rows& rw, const Cols& cl,
                                         const C v[kQ]) {
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if (!ODD) {
      *at(A + qopp(q) * pitch, rw.c, cl.c) = narrow<S>(v[q]);
    } else {
      const uint32_t xo = qcx(q) > 0 ? cl.e : (qcx(q) < 0 ? cl.w : cl.c);  // x + c_q
      const int64_t yo = qcy(q) > 0 ? rw.n : (qcy(q) < 0 ? rw.s : rw.c);
      *at(A + q * pitch, yo, xo) = narrow<S>(v[q]);
    }
  }
}

template <typename S, typename C, bool ODD>
__global__ void __launch_bounds__(kAARow) k_aa_dns(S* __restrict__ A, int nx, int ny, int64_t pitch, Rates<C> r) {
  int x0, y;
  aa_segment(nx, x0, y);
  const int x = x0 + threadIdx.x;
  if (x >= nx) return;
  const Rows rw = rows_of<S>(y, ny, pitch);
  const Cols cl = cols_of<S>(x, nx);
  C v[kQ];
  aa_load<S, C, ODD>(A, pitch, rw, cl, v);
  const Mom<C> m = moments19<kUnits<S>>(v);
  const Closure<C> zero = {C(0), C(0), C(0), C(0)};
  collide19<false, false, kUnits<S>>(v, m, zero, r);
  aa_store<S, C, ODD>(A, pitch, rw, cl, v);
}

// Moment sweep of the in-place closure schedule: m_x, m_y, B_x, B_y of the
// state at time t into four dense planes of the compute type.
template <typename S, typename C, bool ODD>
__global__ void __launch_bounds__(kAARow)
k_aa_moments(const S* __restrict__ A, C* __restrict__ mb, int nx, int ny, int64_t pitch) {
  int x0, y;
  aa_segment(nx, x0, y);
  const int x = x0 + threadIdx.x;
  if (x >= nx) return;
  const Rows rw = rows_of<S>(y, ny, pitch);
  const Cols cl = cols_of<S>(x, nx);
  C v[kQ];
  aa_load<S, C, ODD, true>(A, pitch, rw, cl, v);
  const Mom<C> m = moments19(v);
  const int64_t n = (int64_t)nx * ny, c0 = (int64_t)y * nx + x;
  mb[c0] = m.mx;
  mb[n + c0] = m.my;
  mb[2 * n + c0] = m.dbx;
  mb[3 * n + c0] = m.dby;
}

// The (kAARow + 2) x 3 halo tile of four moment planes (rows y - 1 .. y + 1)
// for the gradient stencil of one row segment.  Columns beyond the first halo
// column of a ragged last segment are not needed and not loaded.
template <typename C>
__device__ __forceinline__ void stage_tile(C (&tile)[4][3][kAARow + 2], const C* __restrict__ mb, int nx, int ny,
                                           int x0, int y) {
  const int64_t n = (int64_t)nx * ny;
  for (int idx = threadIdx.x; idx < 3 * (kAARow + 2); idx += kAARow) {
    const int ly = idx / (kAARow + 2), lx = idx - ly * (kAARow + 2);
    const int gx0 = x0 + lx - 1;
    if (gx0 > nx) continue;
    const int gx = gx0 < 0 ? gx0 + nx : (gx0 == nx ? 0 : gx0);
    const int gy = wrap1(y + ly - 1, ny);
    const int64_t c = (int64_t)gy * nx + gx;
#pragma unroll
    for (int k = 0; k < 4; ++k) tile[k][ly][lx] = mb[k * n + c];
  }
}

template <typename C, int STENCIL>
__device__ __forceinline__ void tile_gradients(const C (&tile)[4][3][kAARow + 2], int lx, C gr[4][2]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    grad3x3<C, STENCIL>(tile[k][1][lx + 1], tile[k][1][lx - 1], tile[k][2][lx], tile[k][0][lx], tile[k][2][lx + 1],
                        tile[k][2][lx - 1], tile[k][0][lx + 1], tile[k][0][lx - 1], gr[k][0], gr[k][1]);
  }
}

// Collide sweep of the in-place closure schedule (synchronous gradients of
// the moment planes written by k_aa_moments).
template <typename S, typename C, bool ODD, int STENCIL>
__global__ void __launch_bounds__(kAARow)
k_aa_les(S* __restrict__ A, const C* __restrict__ mb, int nx, int ny, int64_t pitch, Rates<C> r) {
  __shared__ C tile[4][3][kAARow + 2];
  int x0, y;
  aa_segment(nx, x0, y);
  stage_tile(tile, mb, nx, ny, x0, y);
  __syncthreads();
  const int x = x0 + threadIdx.x;
  if (x >= nx) return;
  const Rows rw = rows_of<S>(y, ny, pitch);
  const Cols cl = cols_of<S>(x, nx);
  C v[kQ];
  aa_load<S, C, ODD>(A, pitch, rw, cl, v);
  const Mom<C> m = moments19<kUnits<S>>(v);
  C gr[4][2];
  tile_gradients<C, STENCIL>(tile, threadIdx.x + 1, gr);
  const C ir = C(1) / (r.rho0 + m.drho);
  constexpr bool LOCAL = STENCIL >= LBM_STENCIL_LOCAL_ISO9;
  if constexpr (LOCAL) local_gradients<kUnits<S>>(v, m, r, gr[1][0] - gr[0][1], gr);
  const Closure<C> cls = closure_terms<LOCAL>(gr[0][0], gr[0][1], gr[1][0], gr[1][1], gr[2][0], gr[2][1], gr[3][0],
                                       gr[3][1], ir, r.k2);
  collide19<true, LOCAL, kUnits<S>>(v, m, cls, r);
  aa_store<S, C, ODD>(A, pitch, rw, cl, v);
}

// Single-sweep in-place closure schedule (lagged gradients): the halo tile
// comes from the previous step's moment planes mb_prev, while the cell's own
// moments go to mb_next for the next step.  19 + 4 values read, 19 + 4
// written per cell.
template <typename S, typename C, bool ODD, int STENCIL>
__global__ void __launch_bounds__(kAARow)
k_aa_les_lagged(S* __restrict__ A, const C* __restrict__ mb_prev, C* __restrict__ mb_next, int nx, int ny,
                int64_t pitch, Rates<C> r) {
  __shared__ C tile[4][3][kAARow + 2];
  int x0, y;
  aa_segment(nx, x0, y);
  stage_tile(tile, mb_prev, nx, ny, x0, y);
  __syncthreads();
  const int x = x0 + threadIdx.x;
  if (x >= nx) return;
  const Rows rw = rows_of<S>(y, ny, pitch);
  const Cols cl = cols_of<S>(x, nx);
  C v[kQ];
  aa_load<S, C, ODD, false, sizeof(S) == 2>(A, pitch, rw, cl, v);
  const Mom<C> m = moments19<kUnits<S>>(v);
  const int64_t n = (int64_t)nx * ny, c0 = (int64_t)y * nx + x;
  mb_next[c0] = m.mx;
  mb_next[n + c0] = m.my;
  mb_next[2 * n + c0] = m.dbx;
  mb_next[3 * n + c0] = m.dby;
  C gr[4][2];
  tile_gradients<C, STENCIL>(tile, threadIdx.x + 1, gr);
  const C ir = C(1) / (r.rho0 + m.drho);
  const Closure<C> cls = closure_terms(gr[0][0], gr[0][1], gr[1][0], gr[1][1], gr[2][0], gr[2][1], gr[3][0],
                                       gr[3][1], ir, r.k2);
  collide19<true, false, kUnits<S>>(v, m, cls, r);
  aa_store<S, C, ODD>(A, pitch, rw, cl, v);
}

// ---------------------------------------------------------------------------
// Natural-layout access for initial state, state IO, moments and diagnostics.
// `base` is the buffer holding the state at time t and `layout` says where
// population q of cell x sits in it:
//   kLayoutNatural: slot q of cell x                (AA buffer, even t)
//   kLayoutAAOdd:   slot opp(q) of cell x - c_q     (AA buffer, odd t)
//   kLayoutPull:    slot q of cell x - c_q          (fused buffers, any t)
// ---------------------------------------------------------------------------
constexpr int kLayoutNatural = 0;
constexpr int kLayoutAAOdd = 1;
constexpr int kLayoutPull = 2;

template <int QG = 5>
__device__ __forceinline__ int64_t natural_index(int q, int x, int y, int nx, int ny, int64_t pitch, int layout) {
  if (layout == kLayoutNatural) return ((int64_t)y * kPop<QG> + q) * pitch + x;
  const int xs = wrap1(x - qcx<QG>(q), nx), ys = wrap1(y - qcy<QG>(q), ny);
  return ((int64_t)ys * kPop<QG> + (layout == kLayoutAAOdd ? qopp<QG>(q) : q)) * pitch + xs;
}

// Rest values subtracted from the stored populations: w_q rho0 for f,
// w'_i B_ref for g (all zero for FP64 storage).
struct RestRef {
  double rho0, bx0, by0;
};

template <int QG = 5>
__device__ __forceinline__ double rest_value(int q, const RestRef& ref) {
  return q < 9 ? w9(q) * ref.rho0 : (q < 9 + QG ? wg<QG>(q - 9) * ref.bx0 : wg<QG>(q - 9 - QG) * ref.by0);
}

// SplitMix64 (Steele, Lea & Flood, OOPSLA 2014): output number counter + 1 of
// the sequence started at `seed`.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t counter) {
  uint64_t z = seed + (counter + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Unfiltered equilibria feq / geq (Sec. 2) of one cell's fields, evaluated in
// FP64 and rounded to the storage type.
template <typename S, int QG = 5>
__device__ __forceinline__ void write_equilibrium(S* __restrict__ base, int x, int y, int nx, int ny, int64_t pitch,
                                                  int layout, const RestRef& ref, double rho, double ux, double uy,
                                                  double bx, double by) {
  const double usq = ux * ux + uy * uy, bsq = bx * bx + by * by;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const double cu = cx9(i) * ux + cy9(i) * uy;
    const double cb = cx9(i) * bx + cy9(i) * by;
    const double c2 = double(cx9(i) * cx9(i) + cy9(i) * cy9(i));
    const double feq = w9(i) * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq) + 4.5 * w9(i) * (0.5 * bsq * c2 - cb * cb);
    base[natural_index<QG>(i, x, y, nx, ny, pitch, layout)] = encode<S>(feq - rest_value<QG>(i, ref));
  }
#pragma unroll
  for (int i = 0; i < QG; ++i) {
    const double cu = cx9(i) * ux + cy9(i) * uy;
    const double cb = cx9(i) * bx + cy9(i) * by;
    const double gx = wg<QG>(i) * (bx + 3.0 * (cu * bx - cb * ux));
    const double gy = wg<QG>(i) * (by + 3.0 * (cu * by - cb * uy));
    base[natural_index<QG>(9 + i, x, y, nx, ny, pitch, layout)] = encode<S>(gx - rest_value<QG>(9 + i, ref));
    base[natural_index<QG>(9 + QG + i, x, y, nx, ny, pitch, layout)] =
        encode<S>(gy - rest_value<QG>(9 + QG + i, ref));
  }
}

// Kelvin-Helmholtz double shear layer at the unfiltered equilibria.
template <typename S, int QG>
__global__ void __launch_bounds__(256)
k_init_kh(S* __restrict__ base, int nx, int ny, int64_t pitch, int layout, RestRef ref, lbm_kh_params kh) {
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  if (x >= nx || y >= ny) return;
  const double L = double(ny), d = kh.delta_over_L * L;
  const double yy = double(y), xx = double(x);
  const double ux = kh.U0 * (tanh((yy - 0.25 * L) / d) - tanh((yy - 0.75 * L) / d) - 1.0);
  const uint64_t z = splitmix64_at(kh.seed, (uint64_t)y * (uint64_t)nx + (uint64_t)x);
  const double xi = 2.0 * (double(z >> 11) * 0x1.0p-53) - 1.0;
  const double uy = kh.pert_amp_over_U0 * kh.U0 * sin(2.0 * M_PI * xx / double(nx)) + kh.noise_amp * xi;
  write_equilibrium<S, QG>(base, x, y, nx, ny, pitch, layout, ref, kh.rho0, ux, uy, kh.B0, 0.0);
}

// The magnetized jet of Sec. 4 at the unfiltered equilibria.
template <typename S, int QG>
__global__ void __launch_bounds__(256)
k_init_sech2(S* __restrict__ base, int nx, int ny, int64_t pitch, int layout, RestRef ref, lbm_sech2_params jet) {
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  if (x >= nx || y >= ny) return;
  const double xf = double(x), yf = double(y), d = fmin(xf, double(nx) - xf);
  const double kx = 2.0 * M_PI * double(jet.k) / double(nx), ky = 2.0 * M_PI * double(jet.k) / double(ny);
  const double ch = cosh(kx * d);
  const double uy = jet.U0 / (ch * ch) + jet.pert * jet.U0 * sin(kx * xf);
  const double ux = jet.pert * jet.U0 * sin(ky * yf);
  const double bx = jet.pert * jet.B0 * sin(ky * yf);
  const double by = jet.B0 + jet.pert * jet.B0 * sin(kx * xf);
  write_equilibrium<S, QG>(base, x, y, nx, ny, pitch, layout, ref, jet.rho0, ux, uy, bx, by);
}

// Equilibria of given fields: 5 FP64 planes rho, m_x, m_y, B_x, B_y.
template <typename S, int QG>
__global__ void __launch_bounds__(256)
k_init_moments(S* __restrict__ base, const double* __restrict__ mom, int nx, int ny, int64_t pitch, int layout,
               RestRef ref) {
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  if (x >= nx || y >= ny) return;
  const int64_t n = (int64_t)nx * ny, c = (int64_t)y * nx + x;
  const double rho = mom[c];
  write_equilibrium<S, QG>(base, x, y, nx, ny, pitch, layout, ref, rho, mom[n + c] / rho, mom[2 * n + c] / rho,
                       mom[3 * n + c], mom[4 * n + c]);
}

template <typename S, int QG>
__global__ void __launch_bounds__(256)
k_get_state(const S* __restrict__ base, double* __restrict__ out, int nx, int ny, int64_t pitch, int layout,
            RestRef ref) {
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  if (x >= nx || y >= ny) return;
  const int64_t n = (int64_t)nx * ny, c0 = (int64_t)y * nx + x;
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) {
    const double v = decode<double>(base[natural_index<QG>(q, x, y, nx, ny, pitch, layout)]);
    out[q * n + c0] = v + rest_value<QG>(q, ref);
  }
}

template <typename S, int QG>
__global__ void __launch_bounds__(256)
k_set_state(S* __restrict__ base, const double* __restrict__ in, int nx, int ny, int64_t pitch, int layout,
            RestRef ref) {
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  if (x >= nx || y >= ny) return;
  const int64_t n = (int64_t)nx * ny, c0 = (int64_t)y * nx + x;
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) {
    const double v = in[q * n + c0];
    base[natural_index<QG>(q, x, y, nx, ny, pitch, layout)] = encode<S>(v - rest_value<QG>(q, ref));
  }
}

// rho, m_x, m_y, B_x, B_y in FP64 (5 dense planes).  256-cell row segments (measured 1.2-1.4x faster than 64 x 4 tiles for the moment
// gathers).
template <typename S, int QG>
__global__ void __launch_bounds__(256)
k_moments_out(const S* __restrict__ base, double* __restrict__ out, int nx, int ny, int64_t pitch, int layout,
              RestRef ref) {
  const int x = blockIdx.x * 256 + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= nx) return;
  double v[kPop<QG>];
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) v[q] = decode<double>(base[natural_index<QG>(q, x, y, nx, ny, pitch, layout)]);
  const Mom<double> m = moments_of<QG>(v);
  const int64_t n = (int64_t)nx * ny, c0 = (int64_t)y * nx + x;
  out[c0] = ref.rho0 + m.drho;
  out[n + c0] = m.mx;
  out[2 * n + c0] = m.my;
  out[3 * n + c0] = ref.bx0 + m.dbx;
  out[4 * n + c0] = ref.by0 + m.dby;
}

// Input vectors of the learned correction (first stage; the network kernel is
// the second).  For every cell of a fused-schedule state (layout kLayoutPull):
// rho, m, B in FP32 from the gathered populations, u = m / rho, the central-
// difference vorticity and current, the seven fields normalised (FP32) and
// rounded to bfloat16, and the out-of-range flag (CellIn, 16 bytes).  Each
// wave walks its own strip of 64 columns down a segment of kCellInRows rows,
// independently of the other waves (no workgroup barrier): each lane gathers
// one column per row, u_x, u_y, B_x, B_y go to the wave's four-row LDS ring,
// and the row above the newest one is finished from the ring.  The strip's
// outer two columns and the rows just outside the segment are gathered for
// their neighbours only: 62 output columns per strip.  FP64 storage runs this
// kernel; FP32 compute runs k_cell_inputs_f below, whose aligned strips store
// whole lines (16384^2 BF16: 2.73 ms against 2.94 ms for this form, whose
// 62-column strips split the lines they store with their neighbours).
constexpr int kCellInW = 64, kCellInRows = 8;

__host__ __device__ constexpr int cell_input_strips(int nx) { return (nx + kCellInW - 3) / (kCellInW - 2); }

template <typename S>
__global__ void __launch_bounds__(256)
k_cell_inputs(const S* __restrict__ src, int nx, int ny, int64_t pitch, RestRef ref, int nstrips,
              const char* __restrict__ pk, CellIn* __restrict__ out) {
  using C = typename ComputeOf<S>::type;
  __shared__ float ring_all[4][4][4][kCellInW];  // wave, row slot, field (u_x, u_y, B_x, B_y), column
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int strip = blockIdx.x * 4 + wid;
  if (strip >= nstrips) return;
  float(*ring)[4][kCellInW] = ring_all[wid];
  const int xu = strip * (kCellInW - 2) - 1 + lane;  // unwrapped column, >= -1
  const int x = xu < 0 ? nx - 1 : xu % nx;
  const bool out_col = lane >= 1 && lane < kCellInW - 1 && xu < nx;
  const int y0 = blockIdx.y * kCellInRows;
  const int nrow = (y0 + kCellInRows <= ny ? kCellInRows : ny - y0);
  const lbm_mlp_norm* nm = reinterpret_cast<const lbm_mlp_norm*>(pk + kPkNorm);
  const Cols cl = cols_of<S>(x, nx);
  float pr = 0.0f, pux = 0.0f, puy = 0.0f, pbx = 0.0f, pby = 0.0f;  // own column, previous row
  for (int k = 0; k < nrow + 2; ++k) {
    int yk = y0 - 1 + k;
    yk = yk < 0 ? yk + ny : (yk >= ny ? yk - ny : yk);
    C v[kQ];
    pull_cell<S, C, 5>(src, pitch, rows_of<S>(yk, ny, pitch), cl, v);
    const Mom<C> m = moments19<kUnits<S>>(v);
    const float r = float(C(ref.rho0) + m.drho);
    const float ux = float(m.mx) / r, uy = float(m.my) / r;
    const float bx = float(C(ref.bx0) + m.dbx), by = float(C(ref.by0) + m.dby);
    const int sl = k & 3;
    ring[sl][0][lane] = ux;
    ring[sl][1][lane] = uy;
    ring[sl][2][lane] = bx;
    ring[sl][3][lane] = by;
    // the wave's own LDS writes, visible to all its lanes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (k >= 2 && out_col) {
      // row yk - 1 (slot k - 1), between rows yk - 2 and yk
      const int sm = (k - 2) & 3, s0 = (k - 1) & 3;
      const float om = 0.5f * (ring[s0][1][lane + 1] - ring[s0][1][lane - 1]) - 0.5f * (ring[sl][0][lane] - ring[sm][0][lane]);
      const float jz = 0.5f * (ring[s0][3][lane + 1] - ring[s0][3][lane - 1]) - 0.5f * (ring[sl][2][lane] - ring[sm][2][lane]);
      const float f[7] = {pr, pux, puy, pbx, pby, om, jz};
      bool bad = false;
      f32x8 z;
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        z[i] = (f[i] - nm->shift[i]) * nm->scale[i];
        bad = bad || !(fabsf(z[i]) <= kOodLimit);  // NaN counts as out of range
      }
      z[7] = 0.0f;
      u32x4 w = __builtin_bit_cast(u32x4, to_bf16x8(z));
      w[3] = (w[3] & 0xFFFFu) | (bad ? unsigned(kCellOutOfRange) << 16 : 0u);
      out[(int64_t)(y0 + k - 2) * nx + x] = __builtin_bit_cast(CellIn, w);
    }
    pr = r;
    pux = ux;
    puy = uy;
    pbx = bx;
    pby = by;
  }
}

// Input vectors with FP32 compute (FP32, FP16, BF16 storage): the strip
// schedule of k_fused_les_f.  A workgroup of W + 64 lanes owns the columns
// x0 .. x0+W-1 (so each row's input vectors are whole aligned lines) and walks
// the rows y0 .. y1-1.  A lane keeps rho, u, B of the rows y-1, y, y+1 of its
// own column in registers and reads u_y, B_y of its two neighbour columns from
// an LDS row (two slots by row parity, one barrier per row); the last wave
// gathers the two halo columns.  Rows are gathered two ahead of their use with
// buffer loads, three register sets rotate through a three-times unrolled
// loop, and lanes past the strip's last column drop their stores through
// kDropOffset, so the row body has no branch around a memory operation.  The
// arithmetic is k_cell_inputs' (same expressions, same results).
struct CellFields {
  float r, ux, uy, bx, by;
};

template <typename S, int W>
__global__ void __launch_bounds__(W + 64)
k_cell_inputs_f(const S* __restrict__ src, int nx, int ny, int64_t pitch, int ry, RestRef ref,
                const char* __restrict__ pk, CellIn* __restrict__ out) {
  using C = float;
  constexpr int NP = kPop<5>;
  __shared__ float rowbuf[2][2][W + 3];  // row parity, field (u_y, B_y), column - x0 + 1 (W + 2: spare)
  const int tid = threadIdx.x;
  const int nstrip = (nx + W - 1) / W;
  const int vb = xcd_contiguous(blockIdx.x, gridDim.x);  // strip vb % nstrip of segment vb / nstrip
  const int x0 = (vb % nstrip) * W;
  const int last = min(x0 + W, nx) - 1;
  const int y0 = (vb / nstrip) * ry;
  const int y1 = min(y0 + ry, ny);
  const uint32_t pq = uint32_t(pitch) * uint32_t(sizeof(S));
  const lbm_mlp_norm* nm = reinterpret_cast<const lbm_mlp_norm*>(pk + kPkNorm);
  auto wrapy = [&](int y) { return y < 0 ? y + ny : (y >= ny ? y - ny : y); };
  auto ahead = [&](int y) { return wrapy(y <= y1 ? y : y1); };  // rows past y1 are not needed

  const bool halo = tid >= W;
  const int hl = tid - W;
  const bool valid = !halo && x0 + tid <= last;
  const int xc = halo ? (hl == 0 ? (x0 == 0 ? nx - 1 : x0 - 1) : (last + 1 == nx ? 0 : last + 1))
                      : (valid ? x0 + tid : last);
  const int widx = halo ? (hl == 0 ? 0 : (hl == 1 ? last - x0 + 2 : W + 2)) : (valid ? tid + 1 : W + 2);
  const Cols cx = cols_of<S>(xc, nx);
  const uint32_t xo_store = valid ? uint32_t(x0 + tid) * uint32_t(sizeof(CellIn)) : kDropOffset;
  const uint32_t orow = uint32_t(nx) * uint32_t(sizeof(CellIn));

  auto pull = [&](int y, RawCell<S, 5>& c) __attribute__((always_inline)) {
    pull_raw<S, 5>(src, pq, wrapy(y - 1), y, wrapy(y + 1), cx, c);
  };
  auto fields = [&](const RawCell<S, 5>& c, CellFields& f) __attribute__((always_inline)) {
    C v[NP];
    decode_raw<S, C, 5>(c, v);
    const Mom<C> m = moments19(v);
    f.r = float(C(ref.rho0) + m.drho);
    f.ux = float(m.mx) / f.r;
    f.uy = float(m.my) / f.r;
    f.bx = float(C(ref.bx0) + m.dbx);
    f.by = float(C(ref.by0) + m.dby);
  };
  auto share = [&](int y, const CellFields& f) __attribute__((always_inline)) {
    rowbuf[y & 1][0][widx] = f.uy;
    rowbuf[y & 1][1][widx] = f.by;
  };

  // Row y: fm, fc hold rows y - 1 and y, fn receives row y + 1 from rn (loaded
  // two rows ago); rt receives row y + 3.
  auto row = [&](const CellFields& fm, const CellFields& fc, CellFields& fn, const RawCell<S, 5>& rn,
                 RawCell<S, 5>& rt, int y) __attribute__((always_inline)) {
    pull(ahead(y + 3), rt);
    __builtin_amdgcn_sched_barrier(0);
    fields(rn, fn);
    share(y + 1, fn);
    {
      // the halo wave runs the same body on column 1 and drops its stores
      const int l = halo ? 1 : tid + 1;
      const float om = 0.5f * (rowbuf[y & 1][0][l + 1] - rowbuf[y & 1][0][l - 1]) - 0.5f * (fn.ux - fm.ux);
      const float jz = 0.5f * (rowbuf[y & 1][1][l + 1] - rowbuf[y & 1][1][l - 1]) - 0.5f * (fn.bx - fm.bx);
      const float f[7] = {fc.r, fc.ux, fc.uy, fc.bx, fc.by, om, jz};
      bool bad = false;
      f32x8 z;
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        z[i] = (f[i] - nm->shift[i]) * nm->scale[i];
        bad = bad || !(fabsf(z[i]) <= kOodLimit);  // NaN counts as out of range
      }
      z[7] = 0.0f;
      u32x4 w = __builtin_bit_cast(u32x4, to_bf16x8(z));
      w[3] = (w[3] & 0xFFFFu) | (bad ? unsigned(kCellOutOfRange) << 16 : 0u);
      const __amdgpu_buffer_rsrc_t d = row_rsrc(reinterpret_cast<char*>(out) + int64_t(y) * orow, orow);
      // non-temporal: the network kernel reads the vectors back after the
      // whole grid is written (16384^2 learned step 0.5-1 % faster, 1024^2 no slower)
      __builtin_amdgcn_raw_buffer_store_b128(w, d, int(xo_store), 0, 2);
    }
    __syncthreads();
  };

  CellFields fa, fb, fc;
  RawCell<S, 5> ra, rb, rc;
  pull(wrapy(y0 - 1), ra);
  fields(ra, fa);
  pull(y0, rb);
  fields(rb, fb);
  share(y0, fb);
  pull(ahead(y0 + 1), ra);
  pull(ahead(y0 + 2), rb);
  __syncthreads();
  int y = y0;
  for (; y + 3 <= y1; y += 3) {  // one straight-line block of three rows
    row(fa, fb, fc, ra, rc, y);
    row(fb, fc, fa, rb, ra, y + 1);
    row(fc, fa, fb, rc, rb, y + 2);
  }
  if (y < y1) row(fa, fb, fc, ra, rc, y);
  if (y + 1 < y1) row(fb, fc, fa, rb, ra, y + 1);
}

// ---------------------------------------------------------------------------
// Diagnostics: FP64 terms of every cell straight from the populations, summed
// per thread in a fixed order, wave and block reductions into one partial per
// workgroup, then a single-workgroup fixed-order final pass.
// Accumulators: 0 mass, 1-2 momentum, 3-4 sum B, 5 kinetic energy, 6 magnetic
// energy, 7 enstrophy, 8 J_z^2, 9 (div B)^2, 10 max |div B|, 11 non-finite.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void diag_combine(double* a, const double* b) {
#pragma unroll
  for (int k = 0; k < kDiagVals; ++k) a[k] = (k == 10) ? fmax(a[k], b[k]) : a[k] + b[k];
}

__device__ void block_reduce_diag(double* acc, double* out) {
  __shared__ double red[4][kDiagVals];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    double o[kDiagVals];
#pragma unroll
    for (int k = 0; k < kDiagVals; ++k) o[k] = __shfl_down(acc[k], off, 64);
    diag_combine(acc, o);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kDiagVals; ++k) red[wid][k] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t[kDiagVals];
#pragma unroll
    for (int k = 0; k < kDiagVals; ++k) t[k] = red[0][k];
    for (int w = 1; w < int(blockDim.x >> 6); ++w) diag_combine(t, red[w]);
#pragma unroll
    for (int k = 0; k < kDiagVals; ++k) out[k] = t[k];
  }
}

// A workgroup of at most kDiagLanes lanes walks a strip of two columns less (the
// outer lanes serve the neighbours' values) up a segment of rows: a lane keeps the fields of rows
// y - 1, y, y + 1 of its column in registers and takes u_y, B_x, B_y of its
// neighbour columns from an LDS row (two slots by row parity, one barrier per
// row); the row after next is being loaded meanwhile.  Reads the populations
// once and writes nothing else: HBM bound.  Measured 4096^2 FP32: through five
// FP64 moment planes in memory 337 + 264 us, this form 251 us (1.28 GB), with the final pass 258 against 621 a call.
constexpr int kDiagLanes = 256;
struct DiagCell {
  double r, mx, my, bx, by, ux, uy;
};

template <typename S, int QG, int LAYOUT>
__global__ void __launch_bounds__(kDiagLanes)
k_diag_partial(const S* __restrict__ base, double* __restrict__ partial, int nx, int ny, int64_t pitch, int ry,
               RestRef ref) {
  constexpr int NP = kPop<QG>;
  const int W = int(blockDim.x) - 2;
  __shared__ double rowbuf[2][3][kDiagLanes + 2];  // row parity, field (u_y, B_x, B_y), lane + 1
  const int tid = threadIdx.x, l = tid + 1;
  const int nstrip = (nx + W - 1) / W;
  const int vb = xcd_contiguous(blockIdx.x, gridDim.x);
  const int x0 = (vb % nstrip) * W, x1 = min(x0 + W, nx);
  const int y0 = (vb / nstrip) * ry, y1 = min(y0 + ry, ny);
  const bool owner = tid >= 1 && tid <= x1 - x0;
  int x = min(x0 - 1 + tid, x1);
  x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
  const Cols cl = cols_of<S>(x, nx);
  auto pull = [&](int y, RawCell<S, QG>& c) __attribute__((always_inline)) {
    const int yw = min(y, y1);  // rows past y1 are not needed
    const Rows rw = rows_of<S, QG>(yw < 0 ? yw + ny : (yw >= ny ? yw - ny : yw), ny, pitch);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int slot = LAYOUT == kLayoutAAOdd ? qopp<QG>(q) : q;
      const bool own = LAYOUT == kLayoutNatural;
      const uint32_t xo = own || qcx<QG>(q) == 0 ? cl.c : (qcx<QG>(q) > 0 ? cl.w : cl.e);
      const int64_t yo = own || qcy<QG>(q) == 0 ? rw.c : (qcy<QG>(q) > 0 ? rw.s : rw.n);
      c.v[q] = *at(base + slot * pitch, yo, xo);
    }
  };
  // a cell with a non-finite population has no density: it shows in every sum
  auto fields = [&](const RawCell<S, QG>& c, DiagCell& f) __attribute__((always_inline)) {
    double v[NP];
    bool finite = true;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      v[q] = decode<double>(c.v[q]);
      finite = finite && isfinite(v[q]);
    }
    const Mom<double> m = moments_of<QG>(v);
    f.r = finite ? ref.rho0 + m.drho : __builtin_nan("");
    f.mx = m.mx;
    f.my = m.my;
    f.bx = ref.bx0 + m.dbx;
    f.by = ref.by0 + m.dby;
    f.ux = f.mx / f.r;
    f.uy = f.my / f.r;
  };
  auto share = [&](int y, const DiagCell& f) __attribute__((always_inline)) {
    rowbuf[y & 1][0][l] = f.uy;
    rowbuf[y & 1][1][l] = f.bx;
    rowbuf[y & 1][2][l] = f.by;
  };
  double acc[kDiagVals];
#pragma unroll
  for (int k = 0; k < kDiagVals; ++k) acc[k] = 0.0;

  DiagCell fs, fc, fn;  // rows y - 1, y, y + 1
  RawCell<S, QG> raw;
  pull(y0 - 1, raw);
  fields(raw, fs);
  pull(y0, raw);
  fields(raw, fc);
  share(y0, fc);
  pull(y0 + 1, raw);
  __syncthreads();
  for (int y = y0; y < y1; ++y) {
    fields(raw, fn);
    pull(y + 2, raw);
    share(y + 1, fn);
    const auto& row = rowbuf[y & 1];
    if (owner) {
      const double w = (row[0][l + 1] - row[0][l - 1]) / 2.0 - (fn.ux - fs.ux) / 2.0;
      const double jz = (row[2][l + 1] - row[2][l - 1]) / 2.0 - (fn.bx - fs.bx) / 2.0;
      const double dv = (row[1][l + 1] - row[1][l - 1]) / 2.0 + (fn.by - fs.by) / 2.0;
      acc[0] += fc.r;
      acc[1] += fc.mx;
      acc[2] += fc.my;
      acc[3] += fc.bx;
      acc[4] += fc.by;
      acc[5] += 0.5 * (fc.mx * fc.mx + fc.my * fc.my) / fc.r;
      acc[6] += 0.5 * (fc.bx * fc.bx + fc.by * fc.by);
      acc[7] += 0.5 * w * w;
      acc[8] += jz * jz;
      acc[9] += dv * dv;
      acc[10] = fmax(acc[10], fabs(dv));
      acc[11] += isfinite(fc.r) ? 0.0 : 1.0;
    }
    fs = fc;
    fc = fn;
    __syncthreads();
  }
  block_reduce_diag(acc, partial + (int64_t)blockIdx.x * kDiagVals);
}

__global__ void __launch_bounds__(256) k_diag_final(const double* __restrict__ partial, double* __restrict__ out,
                                                    int nparts) {
  double acc[kDiagVals];
#pragma unroll
  for (int k = 0; k < kDiagVals; ++k) acc[k] = 0.0;
  for (int p = threadIdx.x; p < nparts; p += blockDim.x) diag_combine(acc, partial + (int64_t)p * kDiagVals);
  block_reduce_diag(acc, out);
}

// ---------------------------------------------------------------------------
// Host side: layout and launchers
// ---------------------------------------------------------------------------
size_t storage_bytes(int dtype) {
  return dtype == LBM_FP64 ? 8 : (dtype == LBM_FP32 ? 4 : 2);
}

int64_t row_pitch(int nx) {
  // Population rows padded to a multiple of 64 elements (whole cache lines);
  // no padding at the power-of-two sizes of the benchmarks, where measured
  // paddings of 64 and 256 elements were slower.
  return ((int64_t)nx + 63) / 64 * 64;
}

int64_t buffer_elems(int nx, int ny, int qg) {
  // ny lattice rows of 9 + 2 qg population rows; rounded to 256 elements.
  const int64_t e = (int64_t)ny * (9 + 2 * qg) * row_pitch(nx);
  return (e + 255) / 256 * 256;
}

size_t buffer_offset_bytes(int nx, int ny, int dtype, int qg) {
  // The second buffer of the fused schedule starts 4 KB past a 64 KB boundary
  // after the first.  The closure sweep reads rows of one buffer while it
  // writes rows of the other; measured at 4096^2 and 8192^2 (FP32), offsets
  // that are multiples of 64 KB put both streams on the same memory channels
  // and cost 10-20 % (8192^2: 2164 us against 1757 us at 4 KB past them).
  const size_t one = (size_t)buffer_elems(nx, ny, qg) * storage_bytes(dtype);
  return (one + 65535) / 65536 * 65536 + 4096;
}

size_t state_bytes(int nx, int ny, int dtype, int schedule, int qg) {
  const size_t one = (size_t)buffer_elems(nx, ny, qg) * storage_bytes(dtype);
  return schedule == LBM_SCHED_FUSED ? buffer_offset_bytes(nx, ny, dtype, qg) + one : one;
}

static size_t align256(size_t v) { return (v + 255) / 256 * 256; }

size_t work_layout(Launch& L) {
  const size_t n = (size_t)L.nx * (size_t)L.ny;
  const size_t cbytes = L.dtype == LBM_FP64 ? 8 : 4;  // compute type of the moment planes
  size_t off = 0;
  L.off_mb = off;
  if (L.schedule == LBM_SCHED_AA) off += align256(4 * n * cbytes);
  if (L.schedule == LBM_SCHED_AA_LAGGED) off += 2 * align256(4 * n * cbytes);
  L.off_edges = off;
  if (L.schedule != LBM_SCHED_FUSED) off += align256(5 * n * sizeof(double));
  const int64_t want = ((int64_t)n + 255) / 256;
  L.diag_blocks = (int)(want < kDiagBlocksMax ? (want < 1 ? 1 : want) : kDiagBlocksMax);
  L.off_part = off;
  off += align256((size_t)L.diag_blocks * kDiagVals * sizeof(double));
  L.off_final = off;
  off += align256(kDiagVals * sizeof(double));
  if (L.learned) {
    L.off_cellin = off;
    off += align256(16 * n);
    L.off_corr = off;
    off += align256(4 * n * sizeof(float));
    L.off_mlp = off;
    off += align256(LBM_MLP_PACKED_BYTES);
  }
  return off;
}

static dim3 tile_grid(int nx, int ny) { return dim3((nx + 63) / 64, (ny + 3) / 4); }

// Magnetic-lattice dispatch: f(std::integral_constant<int, QG>).  The D2Q9
// vector distribution is built for FP64 and FP32 storage (the ABI rejects
// the 16-bit types with it), so 16-bit storage instantiates D2Q5 only.
template <typename S, typename F>
static hipError_t by_lattice(const Launch& L, F&& f) {
  if constexpr (sizeof(S) >= 4) {
    if (L.qg == 9) return f(std::integral_constant<int, 9>{});
  }
  return f(std::integral_constant<int, 5>{});
}
static const dim3 kTile(64, 4);

// Row segments of the in-place schedule's kernels (one-dimensional grid, see
// aa_segment).
static dim3 aa_grid(const Launch& L) { return dim3((L.nx + kAARow - 1) / kAARow * L.ny); }

// The buffer that holds the current state (fused schedule: buffer L.cur), and
// the one the next sweep of the fused schedule writes.
template <typename S>
static S* buffer_index(const Launch& L, int b) {
  char* base = static_cast<char*>(L.state);
  if (L.schedule == LBM_SCHED_FUSED && b) base += buffer_offset_bytes(L.nx, L.ny, L.dtype, L.qg);
  return reinterpret_cast<S*>(base);
}
template <typename S>
static S* current_buffer(const Launch& L) {
  return buffer_index<S>(L, L.cur);
}

static RestRef rest_ref(const Launch& L) { return RestRef{L.rho0, L.bref[0], L.bref[1]}; }

static int layout_at(const Launch& L, int64_t t) {
  if (L.schedule == LBM_SCHED_FUSED) return kLayoutPull;
  return (t & 1) ? kLayoutAAOdd : kLayoutNatural;
}

// Moment set k (0 or 1) of the lagged schedule.
template <typename C>
static C* moment_set(const Launch& L, int k) {
  const size_t n = (size_t)L.nx * (size_t)L.ny;
  const size_t stride = (4 * n * sizeof(C) + 255) / 256 * 256;
  return reinterpret_cast<C*>(static_cast<char*>(L.work) + L.off_mb + (size_t)k * stride);
}

template <typename S, typename C, int W, bool NT, int MODE, int QG, int STENCIL>
static void launch_les_s(const Launch& L, const S* src, S* dst, const Rates<C>& r, const float* corr) {
  const int ry = les_rows(L, W);
  const int strips = (L.nx + W - 1) / W, segs = (L.ny + ry - 1) / ry;
  // one-dimensional grid, numbered XCD-contiguously in the kernel
  hipLaunchKernelGGL((k_fused_les_f<S, W, STENCIL, NT, MODE, QG>), dim3(strips * segs), dim3(W + 64), 0, L.stream,
                     src, dst, L.nx, L.ny, L.pitch, ry, r, corr);
}

template <typename S, typename C, int W, bool NT, int MODE, int QG>
static void launch_les_k(const Launch& L, const S* src, S* dst, const Rates<C>& r, const float* corr) {
  // the density-gradient closure and the D2Q9 vector distribution take
  // stencil gradients only
  if constexpr (MODE != kClosureFull && QG == 5) {
    if (L.stencil == LBM_STENCIL_LOCAL_ISO9) {
      launch_les_s<S, C, W, NT, MODE, QG, LBM_STENCIL_LOCAL_ISO9>(L, src, dst, r, corr);
      return;
    }
    if (L.stencil == LBM_STENCIL_LOCAL_CENTRAL5) {
      launch_les_s<S, C, W, NT, MODE, QG, LBM_STENCIL_LOCAL_CENTRAL5>(L, src, dst, r, corr);
      return;
    }
  }
  if (L.stencil == LBM_STENCIL_CENTRAL5)
    launch_les_s<S, C, W, NT, MODE, QG, LBM_STENCIL_CENTRAL5>(L, src, dst, r, corr);
  else
    launch_les_s<S, C, W, NT, MODE, QG, LBM_STENCIL_ISO9>(L, src, dst, r, corr);
}

template <typename S, typename C, int W, bool NT, int QG>
static void launch_les(const Launch& L, const S* src, S* dst, const Rates<C>& r, const float* corr) {
  if constexpr (QG == 5) {  // the learned correction is built for D2Q5
    if (corr) {
      launch_les_k<S, C, W, NT, kClosureCorr, QG>(L, src, dst, r, corr);
      return;
    }
  }
  if (L.full)
    launch_les_k<S, C, W, NT, kClosureFull, QG>(L, src, dst, r, nullptr);
  else
    launch_les_k<S, C, W, NT, kClosurePlain, QG>(L, src, dst, r, nullptr);
}

template <typename S, typename C, bool NT, int QG>
static void launch_fused(const Launch& L, const S* src, S* dst, const Rates<C>& r, const float* corr) {
  if (L.k2 == 0.0 && !corr) {
    if constexpr (sizeof(S) == 2 && QG == 5) {
      if ((L.nx & 3) == 0) {
        hipLaunchKernelGGL((k_fused_dns_quad<S, C, NT>), dim3((L.nx + 255) / 256 * L.ny), dim3(64), 0, L.stream, src,
                           dst, L.nx, L.ny, L.pitch, r);
        return;
      }
    }
    if ((L.nx & 1) == 0)
      hipLaunchKernelGGL((k_fused_dns_pair<S, C, NT, QG>), dim3((L.nx + 255) / 256, L.ny), dim3(128), 0, L.stream,
                         src, dst, L.nx, L.ny, L.pitch, r);
    else
      hipLaunchKernelGGL((k_fused_dns<S, C, NT, QG>), dim3((L.nx + 255) / 256, L.ny), dim3(256), 0, L.stream, src,
                         dst, L.nx, L.ny, L.pitch, r);
    return;
  }
  // Strips of 512 lanes for wide grids (the LDS ring of a 512-lane FP64 strip would
  // exceed 64 KB).  Measured with the lattice-row layout and XCD-contiguous numbering:
  // 256-lane strips (two or four workgroups per compute unit) against 512 take
  // 0-10 % longer with FP32 storage at 4096^2 and 8192^2 and 16-18 % longer
  // with FP16 at 8192^2 (with the earlier two-dimensional grids: up to 1.6x).
  const int W = strip_width(L.nx, sizeof(C) == 4);
  if constexpr (sizeof(C) == 4) {
    if (W == 512) {
      launch_les<S, C, 512, NT, QG>(L, src, dst, r, corr);
      return;
    }
  }
  if (W == 256)
    launch_les<S, C, 256, NT, QG>(L, src, dst, r, corr);
  else
    launch_les<S, C, 64, NT, QG>(L, src, dst, r, corr);
}

template <typename S>
// The learned closure runs in the fused schedule only (checked at creation),
// so the state is always in the pull layout here.
static hipError_t cell_inputs_typed(const Launch& L, int64_t t, CellIn* out) {
  if (layout_at(L, t) != kLayoutPull) return hipErrorInvalidValue;
  const char* pk = static_cast<const char*>(L.work) + L.off_mlp;
  if constexpr (sizeof(typename ComputeOf<S>::type) == 4) {
    const int W = strip_width(L.nx, true);
    const int ry = fused_rows(L.nx, L.ny, W, W == 64 ? 4 * L.cus : L.cus, 128);
    const dim3 g(((L.nx + W - 1) / W) * ((L.ny + ry - 1) / ry));  // numbered XCD-contiguously in the kernel
    if (W == 512)
      hipLaunchKernelGGL((k_cell_inputs_f<S, 512>), g, dim3(512 + 64), 0, L.stream, current_buffer<S>(L), L.nx, L.ny,
                         L.pitch, ry, rest_ref(L), pk, out);
    else if (W == 256)
      hipLaunchKernelGGL((k_cell_inputs_f<S, 256>), g, dim3(256 + 64), 0, L.stream, current_buffer<S>(L), L.nx, L.ny,
                         L.pitch, ry, rest_ref(L), pk, out);
    else
      hipLaunchKernelGGL((k_cell_inputs_f<S, 64>), g, dim3(64 + 64), 0, L.stream, current_buffer<S>(L), L.nx, L.ny,
                         L.pitch, ry, rest_ref(L), pk, out);
  } else {
    const int strips = cell_input_strips(L.nx);
    hipLaunchKernelGGL((k_cell_inputs<S>), dim3((strips + 3) / 4, (L.ny + kCellInRows - 1) / kCellInRows),
                       dim3(256), 0, L.stream, current_buffer<S>(L), L.nx, L.ny, L.pitch, rest_ref(L), strips, pk, out);
  }
  return hipGetLastError();
}

hipError_t launch_correction(const Launch& L, int64_t t, float* out) {
  CellIn* in = reinterpret_cast<CellIn*>(static_cast<char*>(L.work) + L.off_cellin);
  hipError_t e;
  switch (L.dtype) {
    case LBM_FP64: e = cell_inputs_typed<double>(L, t, in); break;
    case LBM_FP32: e = cell_inputs_typed<float>(L, t, in); break;
    case LBM_FP16: e = cell_inputs_typed<_Float16>(L, t, in); break;
    default: e = cell_inputs_typed<__bf16>(L, t, in); break;
  }
  if (e != hipSuccess) return e;
  return launch_mlp_correct(in, static_cast<char*>(L.work) + L.off_mlp, out, L.nx, L.ny, L.stream);
}

template <typename S, typename C, int STENCIL>
static void launch_aa_les(const Launch& L, S* A, const C* mb, const Rates<C>& r, bool odd) {
  if (odd)
    hipLaunchKernelGGL((k_aa_les<S, C, true, STENCIL>), aa_grid(L), dim3(kAARow), 0, L.stream, A, mb, L.nx, L.ny,
                       L.pitch, r);
  else
    hipLaunchKernelGGL((k_aa_les<S, C, false, STENCIL>), aa_grid(L), dim3(kAARow), 0, L.stream, A, mb, L.nx,
                       L.ny, L.pitch, r);
}

template <typename S>
static hipError_t step_typed(const Launch& L, int64_t t, bool corr_refresh) {
  using C = typename ComputeOf<S>::type;
  const Rates<C> r = make_rates<C>(L);
  const dim3 grid = aa_grid(L);
  const bool les = L.k2 != 0.0;
  if (L.schedule == LBM_SCHED_FUSED) {
    const S* src = current_buffer<S>(L);
    S* dst = buffer_index<S>(L, L.cur ^ 1);
    const float* corr = nullptr;
    if (L.learned) {
      float* c = reinterpret_cast<float*>(static_cast<char*>(L.work) + L.off_corr);
      if (corr_refresh) {
        const hipError_t e = launch_correction(L, t, c);
        if (e != hipSuccess) return e;
      }
      corr = c;
    }
    return by_lattice<S>(L, [&](auto qg) {
      constexpr int QG = decltype(qg)::value;
      if (streaming_stores(L))
        launch_fused<S, C, true, QG>(L, src, dst, r, corr);
      else
        launch_fused<S, C, false, QG>(L, src, dst, r, corr);
      return hipGetLastError();
    });
  }
  S* A = static_cast<S*>(L.state);
  const bool odd = t & 1;
  if (les && L.schedule == LBM_SCHED_AA_LAGGED) {
    const C* prev = moment_set<C>(L, int(t & 1));
    C* next = moment_set<C>(L, int((t + 1) & 1));
    if (L.stencil == LBM_STENCIL_ISO9) {
      if (odd)
        hipLaunchKernelGGL((k_aa_les_lagged<S, C, true, LBM_STENCIL_ISO9>), grid, dim3(kAARow), 0, L.stream, A, prev, next,
                           L.nx, L.ny, L.pitch, r);
      else
        hipLaunchKernelGGL((k_aa_les_lagged<S, C, false, LBM_STENCIL_ISO9>), grid, dim3(kAARow), 0, L.stream, A, prev, next,
                           L.nx, L.ny, L.pitch, r);
    } else {
      if (odd)
        hipLaunchKernelGGL((k_aa_les_lagged<S, C, true, LBM_STENCIL_CENTRAL5>), grid, dim3(kAARow), 0, L.stream, A, prev,
                           next, L.nx, L.ny, L.pitch, r);
      else
        hipLaunchKernelGGL((k_aa_les_lagged<S, C, false, LBM_STENCIL_CENTRAL5>), grid, dim3(kAARow), 0, L.stream, A, prev,
                           next, L.nx, L.ny, L.pitch, r);
    }
    return hipGetLastError();
  }
  if (!les) {
    if (odd)
      hipLaunchKernelGGL((k_aa_dns<S, C, true>), grid, dim3(kAARow), 0, L.stream, A, L.nx, L.ny, L.pitch, r);
    else
      hipLaunchKernelGGL((k_aa_dns<S, C, false>), grid, dim3(kAARow), 0, L.stream, A, L.nx, L.ny, L.pitch, r);
    return hipGetLastError();
  }
  C* mb = reinterpret_cast<C*>(static_cast<char*>(L.work) + L.off_mb);
  if (odd)
    hipLaunchKernelGGL((k_aa_moments<S, C, true>), grid, dim3(kAARow), 0, L.stream, A, mb, L.nx, L.ny, L.pitch);
  else
    hipLaunchKernelGGL((k_aa_moments<S, C, false>), grid, dim3(kAARow), 0, L.stream, A, mb, L.nx, L.ny, L.pitch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (L.stencil) {
    case LBM_STENCIL_ISO9: launch_aa_les<S, C, LBM_STENCIL_ISO9>(L, A, mb, r, odd); break;
    case LBM_STENCIL_CENTRAL5: launch_aa_les<S, C, LBM_STENCIL_CENTRAL5>(L, A, mb, r, odd); break;
    case LBM_STENCIL_LOCAL_ISO9: launch_aa_les<S, C, LBM_STENCIL_LOCAL_ISO9>(L, A, mb, r, odd); break;
    default: launch_aa_les<S, C, LBM_STENCIL_LOCAL_CENTRAL5>(L, A, mb, r, odd);
  }
  return hipGetLastError();
}

template <typename S>
static hipError_t lag_prime_typed(const Launch& L, int64_t t) {
  using C = typename ComputeOf<S>::type;
  S* A = static_cast<S*>(L.state);
  C* mb = moment_set<C>(L, int(t & 1));
  if (t & 1)
    hipLaunchKernelGGL((k_aa_moments<S, C, true>), aa_grid(L), dim3(kAARow), 0, L.stream, A, mb, L.nx, L.ny,
                       L.pitch);
  else
    hipLaunchKernelGGL((k_aa_moments<S, C, false>), aa_grid(L), dim3(kAARow), 0, L.stream, A, mb, L.nx, L.ny,
                       L.pitch);
  return hipGetLastError();
}

hipError_t launch_lag_prime(const Launch& L, int64_t t) {
  switch (L.dtype) {
    case LBM_FP64: return lag_prime_typed<double>(L, t);
    case LBM_FP32: return lag_prime_typed<float>(L, t);
    case LBM_FP16: return lag_prime_typed<_Float16>(L, t);
    default: return lag_prime_typed<__bf16>(L, t);
  }
}

hipError_t launch_step(const Launch& L, int64_t t, bool corr_refresh) {
  switch (L.dtype) {
    case LBM_FP64: return step_typed<double>(L, t, corr_refresh);
    case LBM_FP32: return step_typed<float>(L, t, corr_refresh);
    case LBM_FP16: return step_typed<_Float16>(L, t, corr_refresh);
    default: return step_typed<__bf16>(L, t, corr_refresh);
  }
}

template <typename S>
static hipError_t init_typed(const Launch& L, const lbm_kh_params& kh) {
  return by_lattice<S>(L, [&](auto qg) {
    hipLaunchKernelGGL((k_init_kh<S, decltype(qg)::value>), tile_grid(L.nx, L.ny), kTile, 0, L.stream,
                       current_buffer<S>(L), L.nx, L.ny, L.pitch, layout_at(L, 0), rest_ref(L), kh);
    return hipGetLastError();
  });
}

hipError_t launch_init_kh(const Launch& L, const lbm_kh_params& kh) {
  switch (L.dtype) {
    case LBM_FP64: return init_typed<double>(L, kh);
    case LBM_FP32: return init_typed<float>(L, kh);
    case LBM_FP16: return init_typed<_Float16>(L, kh);
    default: return init_typed<__bf16>(L, kh);
  }
}

template <typename S>
static hipError_t init_sech2_typed(const Launch& L, const lbm_sech2_params& jet) {
  return by_lattice<S>(L, [&](auto qg) {
    hipLaunchKernelGGL((k_init_sech2<S, decltype(qg)::value>), tile_grid(L.nx, L.ny), kTile, 0, L.stream,
                       current_buffer<S>(L), L.nx, L.ny, L.pitch, layout_at(L, 0), rest_ref(L), jet);
    return hipGetLastError();
  });
}

hipError_t launch_init_sech2(const Launch& L, const lbm_sech2_params& jet) {
  switch (L.dtype) {
    case LBM_FP64: return init_sech2_typed<double>(L, jet);
    case LBM_FP32: return init_sech2_typed<float>(L, jet);
    case LBM_FP16: return init_sech2_typed<_Float16>(L, jet);
    default: return init_sech2_typed<__bf16>(L, jet);
  }
}

template <typename S>
static hipError_t init_moments_typed(const Launch& L, int64_t t, const double* mom) {
  return by_lattice<S>(L, [&](auto qg) {
    hipLaunchKernelGGL((k_init_moments<S, decltype(qg)::value>), tile_grid(L.nx, L.ny), kTile, 0, L.stream,
                       current_buffer<S>(L), mom, L.nx, L.ny, L.pitch, layout_at(L, t), rest_ref(L));
    return hipGetLastError();
  });
}

hipError_t launch_init_moments(const Launch& L, int64_t t, const double* mom) {
  switch (L.dtype) {
    case LBM_FP64: return init_moments_typed<double>(L, t, mom);
    case LBM_FP32: return init_moments_typed<float>(L, t, mom);
    case LBM_FP16: return init_moments_typed<_Float16>(L, t, mom);
    default: return init_moments_typed<__bf16>(L, t, mom);
  }
}

template <typename S>
static hipError_t get_typed(const Launch& L, int64_t t, double* out) {
  return by_lattice<S>(L, [&](auto qg) {
    hipLaunchKernelGGL((k_get_state<S, decltype(qg)::value>), tile_grid(L.nx, L.ny), kTile, 0, L.stream,
                       current_buffer<S>(L), out, L.nx, L.ny, L.pitch, layout_at(L, t), rest_ref(L));
    return hipGetLastError();
  });
}

hipError_t launch_get_state(const Launch& L, int64_t t, double* out) {
  switch (L.dtype) {
    case LBM_FP64: return get_typed<double>(L, t, out);
    case LBM_FP32: return get_typed<float>(L, t, out);
    case LBM_FP16: return get_typed<_Float16>(L, t, out);
    default: return get_typed<__bf16>(L, t, out);
  }
}

template <typename S>
static hipError_t set_typed(const Launch& L, int64_t t, const double* in) {
  return by_lattice<S>(L, [&](auto qg) {
    hipLaunchKernelGGL((k_set_state<S, decltype(qg)::value>), tile_grid(L.nx, L.ny), kTile, 0, L.stream,
                       current_buffer<S>(L), in, L.nx, L.ny, L.pitch, layout_at(L, t), rest_ref(L));
    return hipGetLastError();
  });
}

hipError_t launch_set_state(const Launch& L, int64_t t, const double* in) {
  switch (L.dtype) {
    case LBM_FP64: return set_typed<double>(L, t, in);
    case LBM_FP32: return set_typed<float>(L, t, in);
    case LBM_FP16: return set_typed<_Float16>(L, t, in);
    default: return set_typed<__bf16>(L, t, in);
  }
}

template <typename S>
static hipError_t moments_typed(const Launch& L, int64_t t, double* out) {
  return by_lattice<S>(L, [&](auto qg) {
    hipLaunchKernelGGL((k_moments_out<S, decltype(qg)::value>), dim3((L.nx + 255) / 256, L.ny), dim3(256), 0,
                       L.stream, current_buffer<S>(L), out, L.nx, L.ny, L.pitch, layout_at(L, t), rest_ref(L));
    return hipGetLastError();
  });
}

hipError_t launch_moments(const Launch& L, int64_t t, double* out) {
  switch (L.dtype) {
    case LBM_FP64: return moments_typed<double>(L, t, out);
    case LBM_FP32: return moments_typed<float>(L, t, out);
    case LBM_FP16: return moments_typed<_Float16>(L, t, out);
    default: return moments_typed<__bf16>(L, t, out);
  }
}

// Partial sums of the diagnostics; *blocks receives their number, at most
// L.diag_blocks (the room for them).
template <typename S>
static hipError_t diag_typed(const Launch& L, int64_t t, double* part, int* blocks) {
  const int lanes = std::min(kDiagLanes, (L.nx + 2 + 63) / 64 * 64);
  const int strips = (L.nx + lanes - 3) / (lanes - 2);
  // about four waves' worth of workgroups per SIMD, segments of at least two rows
  const int segs = std::min({1024 * (kDiagLanes / lanes) / strips, (L.ny + 1) / 2, L.diag_blocks / strips});
  if (segs < 1) return hipErrorInvalidValue;  // 1024 >= strips and diag_blocks >= strips for every grid
  const int ry = (L.ny + segs - 1) / segs;
  *blocks = strips * ((L.ny + ry - 1) / ry);
  const auto go = [&](auto qg, auto layout) {
    hipLaunchKernelGGL((k_diag_partial<S, decltype(qg)::value, decltype(layout)::value>), dim3(*blocks),
                       dim3(lanes), 0, L.stream, current_buffer<S>(L), part, L.nx, L.ny, L.pitch, ry, rest_ref(L));
    return hipGetLastError();
  };
  using D2Q5 = std::integral_constant<int, 5>;
  switch (layout_at(L, t)) {
    case kLayoutPull:
      return by_lattice<S>(L, [&](auto qg) { return go(qg, std::integral_constant<int, kLayoutPull>{}); });
    case kLayoutAAOdd: return go(D2Q5{}, std::integral_constant<int, kLayoutAAOdd>{});
    default: return go(D2Q5{}, std::integral_constant<int, kLayoutNatural>{});
  }
}

hipError_t launch_diagnostics(const Launch& L, int64_t t, double* vals_host) {
  char* w = static_cast<char*>(L.work);
  double* part = reinterpret_cast<double*>(w + L.off_part);
  double* fin = reinterpret_cast<double*>(w + L.off_final);
  hipError_t e;
  int blocks = 0;
  switch (L.dtype) {
    case LBM_FP64: e = diag_typed<double>(L, t, part, &blocks); break;
    case LBM_FP32: e = diag_typed<float>(L, t, part, &blocks); break;
    case LBM_FP16: e = diag_typed<_Float16>(L, t, part, &blocks); break;
    default: e = diag_typed<__bf16>(L, t, part, &blocks); break;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(256), 0, L.stream, part, fin, blocks);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(vals_host, fin, kDiagVals * sizeof(double), hipMemcpyDeviceToHost, L.stream)) !=
      hipSuccess)
    return e;
  return hipStreamSynchronize(L.stream);
}

}  // namespace lbm
