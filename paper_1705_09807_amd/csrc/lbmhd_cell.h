// Per-cell arithmetic of the timestep and the addressing of the population
// buffers, shared by every timestep kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lbmhd_device.h"
#include "lbmhd_internal.h"

namespace lbm {

// ---------------------------------------------------------------------------
// Lattice (Sec. 2): D2Q9 velocities; the vector distribution uses the first
// QG of them: five (D2Q5, the default) or all nine (D2Q9, Sec. 2's own
// lattice for g).  Population q: f_q (q < 9), g_x,q-9 (9 .. 8+QG),
// g_y,q-9-QG (9+QG .. 8+2QG); NPOP = 9 + 2 QG populations per cell.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int cx9(int i) {
  return (i == 1 || i == 5 || i == 8) ? 1 : ((i == 3 || i == 6 || i == 7) ? -1 : 0);
}
__host__ __device__ constexpr int cy9(int i) {
  return (i == 2 || i == 5 || i == 6) ? 1 : ((i == 4 || i == 7 || i == 8) ? -1 : 0);
}
__host__ __device__ constexpr int opp9(int i) {
  return i == 0 ? 0 : (i < 5 ? ((i + 1) % 4) + 1 : ((i - 3) % 4) + 5);
}
template <int QG> constexpr int kPop = 9 + 2 * QG;
template <int QG = 5>
__host__ __device__ constexpr int qbase(int q) { return q < 9 ? q : (q < 9 + QG ? q - 9 : q - 9 - QG); }
template <int QG = 5>
__host__ __device__ constexpr int qcx(int q) { return cx9(qbase<QG>(q)); }
template <int QG = 5>
__host__ __device__ constexpr int qcy(int q) { return cy9(qbase<QG>(q)); }
template <int QG = 5>
__host__ __device__ constexpr int qopp(int q) {
  return q < 9 ? opp9(q) : (q < 9 + QG ? 9 + opp9(q - 9) : 9 + QG + opp9(q - 9 - QG));
}
// D2Q9 weights (rest deviation of f, and g on D2Q9) and D2Q5 weights of the
// vector distribution.
__host__ __device__ constexpr double w9(int i) { return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0); }
__host__ __device__ constexpr double w5(int i) { return i == 0 ? 1.0 / 3.0 : 1.0 / 6.0; }
template <int QG>
__host__ __device__ constexpr double wg(int i) { return QG == 5 ? w5(i) : w9(i); }

static_assert(opp9(1) == 3 && opp9(2) == 4 && opp9(3) == 1 && opp9(4) == 2, "opposites");
static_assert(opp9(5) == 7 && opp9(6) == 8 && opp9(7) == 5 && opp9(8) == 6, "opposites");
static_assert(qcx(10) == 1 && qcy(16) == 1 && qopp(15) == 17, "vector planes");
static_assert(qcx<9>(14) == 1 && qcy<9>(20) == 1 && qopp<9>(23) == 25 && qopp<9>(14) == 16, "D2Q9 vector planes");
static_assert(kPop<5> == kQ, "D2Q5 population count");

template <typename S> struct ComputeOf { using type = float; };
template <> struct ComputeOf<double> { using type = double; };

// Storage codecs.  FP64 and FP32 store values as they are.  The 16-bit
// storage types hold the deviations (see below) for FP32 arithmetic: FP16
// scaled by 2^8, which lifts the small deviations out of the FP16 subnormal
// range (normal values start at 6.1e-5) while the largest ones (~0.1) stay
// far below 65504; BF16 unscaled (it has the FP32 exponent range).  All
// conversions round to nearest even.
template <typename S> struct Codec {
  static constexpr float kScale = 1.0f;
};
template <> struct Codec<_Float16> {
  static constexpr float kScale = 256.0f;
};
// Stored units per unit of a value: the timestep kernels widen and narrow the stored
// numbers as they are and work on populations in stored units, scaling the few sums
// of a cell instead of its 38 values (a power of two: the same bits).  FP16 1024^2, one
// step per launch: closure off 13.8 -> 12.9 us, on 19.5 -> 18.4, lagged in place
// 21.5 -> 19.8.
template <typename S> constexpr int kUnits = int(Codec<S>::kScale);
template <typename C, typename S>
__device__ __forceinline__ C widen(S v) {
  if constexpr (sizeof(S) == 2)
    return C(float(v));
  else
    return C(v);
}
template <typename S, typename C>
__device__ __forceinline__ S narrow(C v) {
  if constexpr (sizeof(S) == 2) {
    // FP16: the FP32 result is rounded once more, as a value that is stored and loaded
    // would be (the compiler would else round a multiply-add straight to FP16)
    float x = float(v);
    if constexpr (kUnits<S> != 1) asm("" : "+v"(x));
    return S(x);
  } else {
    return S(v);
  }
}
template <typename C, typename S>
__device__ __forceinline__ C decode(S v) {
  if constexpr (sizeof(S) == 2)
    return C(float(v) * (1.0f / Codec<S>::kScale));
  else
    return C(v);
}
template <typename S, typename C>
__device__ __forceinline__ S encode(C v) {
  if constexpr (sizeof(S) == 2)
    return S(float(v) * Codec<S>::kScale);
  else
    return S(v);
}

__device__ __forceinline__ int wrap1(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Rates in the compute type, with the 1/|row|^2 of T^-1 = T^T diag(1/|row|^2)
// folded in: |row|^2 = 9, 6, 6, 4, 4, 12, 12, 180, 20 for M0..M8.
template <typename C>
struct Rates {
  C s3q, s4q, s5q, s6q, s7q, s8q;
  C sm, k2, rho0;
  C bx0, by0;  // reference field of the stored g deviations
};

template <typename C>
static Rates<C> make_rates(const Launch& L) {
  Rates<C> r;
  r.s3q = C(L.rate[3] / 4.0);
  r.s4q = C(L.rate[4] / 4.0);
  r.s5q = C(L.rate[5] / 12.0);
  r.s6q = C(L.rate[6] / 12.0);
  r.s7q = C(L.rate[7] / 180.0);
  r.s8q = C(L.rate[8] / 20.0);
  r.sm = C(L.sm);
  r.k2 = C(L.k2);
  r.rho0 = C(L.rho0);
  r.bx0 = C(L.bref[0]);
  r.by0 = C(L.bref[1]);
  return r;
}

// ---------------------------------------------------------------------------
// Per-cell arithmetic of the method.  The expressions are evaluated as
// written: contraction is off and every fused multiply-add is spelled out, so
// a cell's result does not depend on the kernel, or on the copy of an unrolled
// body, that evaluates it.  Sweeps of one and of several steps can then be mixed freely
// with the same bits, and the schedules give the same; one exception: 16-bit storage with
// the closure off and a width of whole quads, where the two-buffer schedule sums the rest
// population of one column in four in another order than the in-place one (swapped_rest),
// so that these states differ in last bits and are not the same shifted along x.
// ---------------------------------------------------------------------------
template <typename C>
struct Mom {
  C drho, mx, my, dbx, dby;  // rho - rho0, rho u, B - B_ref
};

// rho = sum f_i, rho u = sum c_i f_i, B = sum g_i (Sec. 2), from the stored
// deviations f_i - w_i rho0 and g_i - w'_i B_ref (sum_i w_i = sum_i w'_i = 1,
// sum_i w_i c_i = 0).  Fixed summation order: every kernel gets bit-identical
// moments for a cell.  U: v is in units of 1 / U (see kUnits).
template <int QG, int U = 1, typename C>
__device__ __forceinline__ Mom<C> moments_of(const C* v) {
  Mom<C> m;
  m.drho = (((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]))) + v[8];
  m.mx = ((v[1] - v[3]) + (v[5] - v[6])) + (v[8] - v[7]);
  m.my = ((v[2] - v[4]) + (v[5] - v[7])) + (v[6] - v[8]);
  if constexpr (QG == 5) {
    m.dbx = ((v[9] + v[10]) + (v[11] + v[12])) + v[13];
    m.dby = ((v[14] + v[15]) + (v[16] + v[17])) + v[18];
  } else {
    m.dbx = (((v[9] + v[10]) + (v[11] + v[12])) + ((v[13] + v[14]) + (v[15] + v[16]))) + v[17];
    m.dby = (((v[18] + v[19]) + (v[20] + v[21])) + ((v[22] + v[23]) + (v[24] + v[25]))) + v[26];
  }
  if constexpr (U != 1) {
    constexpr C u = C(1) / U;
    m.drho *= u;
    m.mx *= u;
    m.my *= u;
    m.dbx *= u;
    m.dby *= u;
  }
  return m;
}

template <int U = 1, typename C>
__device__ __forceinline__ Mom<C> moments19(const C v[kQ]) {
  return moments_of<5, U>(v);
}

// a / U + b and a - U b (a in units of 1 / U), one rounding each.
template <int U, typename C>
__device__ __forceinline__ C plus_units(C a, C b) {
  if constexpr (U == 1)
    return a + b;
  else
    return fmadd(a, C(1) / U, b);
}
template <int U, typename C>
__device__ __forceinline__ C minus_units(C a, C b) {
  if constexpr (U == 1)
    return a - b;
  else
    return fmadd(C(-U), b, a);
}

// One collision of the 19 populations of a cell (Sec. 2, Sec. 3).
//  f: the collision term of LBKinEqn with rate tensor s' = T^-1 S T, i.e.
//     f* = f - T^-1 S (M - M_eq), M = T f, M_eq the filtered KinMomentEq table
//     (rho u_x rho u_y / rho - B_x B_y + tau_xy, ...).  Conserved M0..M2 have
//     rate 0, so only rows 3..8 are formed, and T^-1 = T^T diag(1/|row|^2).
//     In deviation storage M(w rho0) = (rho0, 0, ..., 0, 5 rho0 / 3) shifts
//     only M8's equilibrium.
//  g: g* = g - s_m (g - g_eq), g_eq_i = w'_i (B + 3 [(c.u) B - (c.B) u]) on D2Q5
//     or D2Q9, which is g_eq_ix = w'_i (B_x - 3 c_iy E), g_eq_iy = w'_i (B_y +
//     3 c_ix E) with E = (m_x B_y - m_y B_x) / rho + eps.  On D2Q9 this is the
//     moment-space SRT of MagTMatrix / MagMomentEq: with one rate for every
//     moment, relaxing T_m g towards N^eq and mapping back is relaxing g
//     towards T_m^-1 N^eq, the D2Q9 geq.
// LES false: the closure is off (cl is not read).  LOCAL: after local_gradients, whose
// unfused equilibria are shared.  swapped: the rest population sums its two products
// in the other order (see swapped_rest).  U: v is in units of 1 / U; everything but v
// and the rows of T applied to it is in natural units.
template <int QG, bool LES, bool LOCAL = false, int U = 1, typename C>
__device__ __forceinline__ void collide_q(C* v, const Mom<C>& m, const Closure<C>& cl, const Rates<C>& r,
                                          bool swapped = false) {
#pragma clang fp contract(off)
  const C rho = r.rho0 + m.drho;
  const C ir = C(1) / rho;
  const C mx = m.mx, my = m.my, bx = r.bx0 + m.dbx, by = r.by0 + m.dby;
  // rows 3..8 of T applied to the stored deviations
  const C d56 = v[5] - v[6], d78 = v[7] - v[8], s56 = v[5] + v[6], s78 = v[7] + v[8];
  const C s14 = (v[1] + v[2]) + (v[3] + v[4]);
  const C s58 = s56 + s78;
  const C M3 = d56 + d78;
  const C M4 = (v[1] + v[3]) - (v[2] + v[4]);
  const C M5 = fmadd(C(2), v[3] - v[1], d56) - d78;
  const C M6 = fmadd(C(2), v[4] - v[2], s56) - s78;
  const C M7 = fmadd(C(4), s58, fmadd(C(4), v[0], C(-5) * s14));
  const C M8 = fmadd(C(4), v[0], -s58);
  // filtered equilibrium moments (deviation form for M8)
  const C q2 = (LOCAL ? mx * mx + my * my : fmadd(mx, mx, my * my)) * ir;
  C e3 = LOCAL ? mx * my * ir - bx * by : fmadd(mx * my, ir, -(bx * by));
  C e4 = LOCAL ? (mx * mx - my * my) * ir - (bx * bx - by * by)
               : fmadd(fmadd(mx, mx, -(my * my)), ir, -fmadd(bx, bx, -(by * by)));
  if constexpr (LES) {
    e3 += cl.tau_xy;
    e4 += cl.tau_d;
  }
  const C e7 = LES ? fmadd(C(-3), q2, C(-3) * cl.tau_s) : C(-3) * q2;
  const C m7 = LES ? plus_units<U>(M7, -e7) : fmadd(C(3), q2, U == 1 ? M7 : M7 * (C(1) / U));
  const C m3 = plus_units<U>(M3, -e3), m5 = plus_units<U>(M5, mx), m6 = plus_units<U>(M6, my);
  const C m8 = plus_units<U>(M8, -fmadd(C(5.0 / 3.0), m.drho, e7));
  const C d4 = r.s4q * plus_units<U>(M4, -e4), d5 = r.s5q * m5, d6 = r.s6q * m6, d7 = r.s7q * m7, d8 = r.s8q * m8;
  const C h = fmadd(C(4), d7, -d8);
  v[0] = fmadd(C(-4 * U), swapped ? fmadd(r.s7q, m7, d8) : fmadd(r.s8q, m8, d7), v[0]);
  v[1] = minus_units<U>(v[1], fmadd(C(-5), d7, fmadd(C(-2), d5, d4)));
  v[2] = minus_units<U>(v[2], fmadd(C(-5), d7, fmadd(C(-2), d6, -d4)));
  v[3] = minus_units<U>(v[3], fmadd(C(-5), d7, fmadd(C(2), d5, d4)));
  v[4] = minus_units<U>(v[4], fmadd(C(-5), d7, fmadd(C(2), d6, -d4)));
  v[5] = minus_units<U>(v[5], fmadd(r.s6q, m6, fmadd(r.s3q, m3, d5)) + h);
  v[6] = minus_units<U>(v[6], fmadd(-r.s5q, m5, fmadd(-r.s3q, m3, d6)) + h);
  v[7] = minus_units<U>(v[7], fmadd(-r.s6q, m6, fmadd(r.s3q, m3, -d5)) + h);
  v[8] = minus_units<U>(v[8], fmadd(-r.s6q, m6, fmadd(-r.s3q, m3, d5)) + h);
  // vector distribution, SRT; the w'_i B_ref part of the stored deviation
  // cancels against that of g_eq
  const C n = LOCAL ? mx * by - my * bx : fmadd(mx, by, -(my * bx));
  const C E = !LES ? n * ir : (LOCAL ? n * ir + cl.eps : fmadd(n, ir, cl.eps));
  const C bxp = fmadd(C(3), E, m.dbx), bxm = fmadd(C(-3), E, m.dbx);
  const C byp = fmadd(C(3), E, m.dby), bym = fmadd(C(-3), E, m.dby);
#pragma unroll
  for (int i = 0; i < QG; ++i) {
    const C wi = C(wg<QG>(i)) * C(U);
    C& x = v[9 + i];
    C& y = v[9 + QG + i];
    x = fmadd(-r.sm, fmadd(-wi, cy9(i) == 0 ? m.dbx : (cy9(i) > 0 ? bxm : bxp), x), x);
    y = fmadd(-r.sm, fmadd(-wi, cx9(i) == 0 ? m.dby : (cx9(i) > 0 ? byp : bym), y), y);
  }
}

template <bool LES, bool LOCAL = false, int U = 1, typename C>
__device__ __forceinline__ void collide19(C v[kQ], const Mom<C>& m, const Closure<C>& cl, const Rates<C>& r,
                                          bool swapped = false) {
  collide_q<5, LES, LOCAL, U>(v, m, cl, r, swapped);
}

// 16-bit storage, closure off, nx a multiple of 4, two-buffer schedule: one column in four
// rounds its rest population from the two products in the other order (FP16 the third, BF16
// the second), as the sweep of four columns a thread always has.  A difference in the last
// bit of FP32 would now and then become one of a stored 16-bit value, so every sweep of
// that schedule keeps it: runs and saved states continue with the same bits.  In sweeps of
// several steps it costs a multiply-add and a select per cell and step.
template <typename S>
__device__ __forceinline__ bool swapped_rest(int x, int nx) {
  if constexpr (sizeof(S) == 2) return (nx & 3) == 0 && (x & 3) == (std::is_same_v<S, __bf16> ? 1 : 2);
  return false;
}

// Closure gradients from local non-equilibrium moments (LOCAL stencils),
// with the stencil vorticity wm = D_x m_y - D_y m_x.  First-order
// Chapman-Enskog of the pre-collision populations: M3 - M3^eq =
// -(2 rho / (3 s3)) S_xy, M4 - M4^eq = -(2 rho / (3 s4)) (S_xx - S_yy) with the
// unfiltered equilibria, S_xx = -S_yy (incompressible), D m = rho D u; and
// D_b B_a = -3 s_m (Lam_ba - Lam^eq_ba), Lam_ba = sum_i c_ib g_ia, Lam^eq_xy =
// E, Lam^eq_yx = -E.  The stored deviations have the same M3, M4 and Lam
// (the rest state has none).  gr[k] = (D_x, D_y) of m_x, m_y, B_x, B_y.
// U: v is in units of 1 / U.
template <int U = 1, typename C>
__device__ __forceinline__ void local_gradients(const C v[kQ], const Mom<C>& m, const Rates<C>& r, C wm,
                                                C gr[4][2]) {
  // evaluated as written (no contraction into FMAs), so every copy of an
  // unrolled row body gives the same bits
#pragma clang fp contract(off)
  const C rho = r.rho0 + m.drho;
  const C ir = C(1) / rho;
  const C bx = r.bx0 + m.dbx, by = r.by0 + m.dby;
  const C M3 = (v[5] - v[6]) + (v[7] - v[8]);
  const C M4 = (v[1] + v[3]) - (v[2] + v[4]);
  const C e3 = m.mx * m.my * ir - bx * by;
  const C e4 = (m.mx * m.mx - m.my * m.my) * ir - (bx * bx - by * by);
  // rho S: s3 = 4 s3q and s4 = 4 s4q exactly
  const C rsxy = C(-6) * r.s3q * plus_units<U>(M3, -e3);
  const C rsxx = C(-3) * r.s4q * plus_units<U>(M4, -e4);
  gr[0][0] = rsxx;
  gr[0][1] = rsxy - C(0.5) * wm;
  gr[1][0] = rsxy + C(0.5) * wm;
  gr[1][1] = -rsxx;
  const C E = (m.mx * by - m.my * bx) * ir;
  const C k = C(-3) * r.sm;
  const C ku = U == 1 ? k : k * (C(1) / U);
  gr[2][0] = ku * (v[10] - v[12]);
  gr[2][1] = k * plus_units<U>(v[11] - v[13], E);
  gr[3][0] = k * plus_units<U>(v[15] - v[17], -E);
  gr[3][1] = ku * (v[16] - v[18]);
}

// ---------------------------------------------------------------------------
// Fused schedule (two buffers, pull streaming).  A buffer holds the
// post-collision populations of the previous step at their source cell, so
// the state at time t is f_q(x) = buf[q][x - c_q]: every sweep gathers with
// loads shifted by at most one cell and stores aligned, coalesced rows.
// ---------------------------------------------------------------------------

// Two consecutive stored values (one aligned load or store).
template <typename S> using Vec2 = S __attribute__((ext_vector_type(2)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

// Addressing.  A buffer is ny lattice rows, each holding the NPOP population
// rows of that lattice row one after another, `pitch` elements apart:
// element (q, x, y) at (y * NPOP + q) * pitch + x.  Keeping the populations
// of a lattice row together means the workgroups that run at the same time
// read and write a few contiguous stretches of memory instead of one stretch
// per population plane.  An access is a wave-uniform row base (the lattice
// row's offset, 64-bit, plus q * pitch, in scalar registers) plus a 32-bit
// byte offset of the column, the scalar-base + vector-offset form of global
// loads and stores.
template <typename S>
__device__ __forceinline__ const S* at(const S* __restrict__ base, int64_t row_off, uint32_t col_off) {
  return reinterpret_cast<const S*>(reinterpret_cast<const char*>(base) + row_off + col_off);
}
template <typename S>
__device__ __forceinline__ S* at(S* __restrict__ base, int64_t row_off, uint32_t col_off) {
  return reinterpret_cast<S*>(reinterpret_cast<char*>(base) + row_off + col_off);
}

// Streaming store: non-temporal when the working set exceeds the caches.
template <bool NT, typename T>
__device__ __forceinline__ void store(T* p, T v) {
  if (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// Byte offsets of the lattice rows y - 1, y, y + 1 (periodic) and of the
// columns x - 1, x, x + 1 of a cell.
struct Rows {
  int64_t s, c, n;
};
template <typename S, int QG = 5>
__device__ __forceinline__ Rows rows_of(int y, int ny, int64_t pitch) {
  const int64_t rb = int64_t(kPop<QG>) * pitch * int64_t(sizeof(S));
  Rows r;
  r.c = int64_t(y) * rb;
  r.s = int64_t(y == 0 ? ny - 1 : y - 1) * rb;
  r.n = int64_t(y + 1 == ny ? 0 : y + 1) * rb;
  return r;
}
struct Cols {
  uint32_t w, c, e;
};
template <typename S>
__device__ __forceinline__ Cols cols_of(int x, int nx) {
  Cols c;
  c.c = uint32_t(x) * uint32_t(sizeof(S));
  c.w = uint32_t(x == 0 ? nx - 1 : x - 1) * uint32_t(sizeof(S));
  c.e = uint32_t(x + 1 == nx ? 0 : x + 1) * uint32_t(sizeof(S));
  return c;
}

// f_q(x, y) = src[q][x - c_q][y - c_q] for one cell, in stored units.
template <typename S, typename C, int QG = 5>
__device__ __forceinline__ void pull_cell(const S* __restrict__ src, int64_t pitch, const Rows& rw, const Cols& cl,
                                          C* v) {
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) {
    const uint32_t xo = qcx<QG>(q) > 0 ? cl.w : (qcx<QG>(q) < 0 ? cl.e : cl.c);
    const int64_t yo = qcy<QG>(q) > 0 ? rw.s : (qcy<QG>(q) < 0 ? rw.n : rw.c);
    v[q] = widen<C>(*at(src + q * pitch, yo, xo));
  }
}

// Two horizontally adjacent cells x, x + 1 (x even, nx even): the c_x = 0
// populations come in one aligned two-element load.
template <typename S, typename C, int QG = 5>
__device__ __forceinline__ void pull_pair(const S* __restrict__ src, int64_t pitch, int nx, const Rows& rw, int x,
                                          C* a, C* b) {
  using V2 = Vec2<S>;
  const uint32_t es = uint32_t(sizeof(S));
  const uint32_t xw = uint32_t(x == 0 ? nx - 1 : x - 1) * es, x0 = uint32_t(x) * es, x1 = x0 + es;
  const uint32_t x2 = uint32_t(x + 2 == nx ? 0 : x + 2) * es;
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) {
    const int64_t yo = qcy<QG>(q) > 0 ? rw.s : (qcy<QG>(q) < 0 ? rw.n : rw.c);
    const S* pq = src + q * pitch;
    if (qcx<QG>(q) == 0) {
      const V2 t = *reinterpret_cast<const V2*>(at(pq, yo, x0));
      a[q] = widen<C>(t.x);
      b[q] = widen<C>(t.y);
    } else if (qcx<QG>(q) > 0) {
      a[q] = widen<C>(*at(pq, yo, xw));
      b[q] = widen<C>(*at(pq, yo, x0));
    } else {
      a[q] = widen<C>(*at(pq, yo, x1));
      b[q] = widen<C>(*at(pq, yo, x2));
    }
  }
}

template <typename S> using Vec4 = S __attribute__((ext_vector_type(4)));

// Closure variants of the fused sweeps: see k_fused_les_f.
enum { kClosurePlain = 0, kClosureCorr = 1, kClosureFull = 2 };

// A cell's populations as stored (16-bit values widened where they are used).
template <typename S, int QG>
struct RawCell {
  S v[kPop<QG>];
};
template <typename S, typename C, int QG>
__device__ __forceinline__ void widen_raw(const RawCell<S, QG>& c, C* v) {
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) v[q] = widen<C>(c.v[q]);
}
template <typename S, typename C, int QG>
__device__ __forceinline__ void decode_raw(const RawCell<S, QG>& c, C* v) {
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) v[q] = decode<C>(c.v[q]);
}

// Buffer addressing of the wave-strip sweep: a buffer resource per lattice
// row (its base held in scalar registers), the population's row offset as
// the scalar offset and the column's byte offset as the per-lane offset, so a
// load or store costs no per-lane address arithmetic.  Raw resources
// (stride 0) of num_records = the lattice row's bytes; every access of a row
// lies inside it, except the stores of lanes that own no output column,
// which take an offset past num_records: the hardware's range check drops
// them, so the row body has no branch around its stores.  (nx <= 32768, as
// lbm_create requires, keeps a lattice row below 27 * 32768 * 8 B = 7 MB
// and a row of input vectors at 512 KB, far below kDropOffset.)
constexpr uint32_t kDropOffset = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), 0x00020000);
}
template <typename S>
__device__ __forceinline__ S buf_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(S) == 2)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(r, int(voff), int(soff), 0));
  else if constexpr (sizeof(S) == 4)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, int(voff), int(soff), 0));
  else
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, int(voff), int(soff), 0));
}
template <typename S, bool NT>
__device__ __forceinline__ void buf_store(S v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  constexpr int aux = NT ? 2 : 0;  // non-temporal
  if constexpr (sizeof(S) == 2)
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, int(voff), int(soff), aux);
  else if constexpr (sizeof(S) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, int(voff), int(soff), aux);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, int(voff), int(soff), aux);
}

// Buffer loads and stores of T (4, 8 or 16 bytes: one, two or four stored values).
template <typename T>
__device__ __forceinline__ T buf_load_v(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, int(voff), int(soff), 0));
  else if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, int(voff), int(soff), 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, int(voff), int(soff), 0));
}
template <typename T, bool NT>
__device__ __forceinline__ void buf_store_v(T v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  constexpr int aux = NT ? 2 : 0;
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, int(voff), int(soff), aux);
  else if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, int(voff), int(soff), aux);
  else
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), r, int(voff), int(soff), aux);
}

// f_q(x, y) = src[q][x - c_q][y - c_q] of one cell, as stored; ys, yc, yn
// are the (periodic) rows y - 1, y, y + 1, pq the bytes between population
// rows.
template <typename S, int QG>
__device__ __forceinline__ void pull_raw(const S* __restrict__ src, uint32_t pq, int ys, int yc, int yn,
                                         const Cols& cl, RawCell<S, QG>& c) {
  const uint32_t rowb = uint32_t(kPop<QG>) * pq;
  const char* b = reinterpret_cast<const char*>(src);
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(b + int64_t(ys) * rowb, rowb);
  const __amdgpu_buffer_rsrc_t rc = row_rsrc(b + int64_t(yc) * rowb, rowb);
  const __amdgpu_buffer_rsrc_t rn = row_rsrc(b + int64_t(yn) * rowb, rowb);
#pragma unroll
  for (int q = 0; q < kPop<QG>; ++q) {
    const uint32_t xo = qcx<QG>(q) > 0 ? cl.w : (qcx<QG>(q) < 0 ? cl.e : cl.c);
    const __amdgpu_buffer_rsrc_t rr = qcy<QG>(q) > 0 ? rs : (qcy<QG>(q) < 0 ? rn : rc);
    c.v[q] = buf_load<S>(rr, xo, uint32_t(q) * pq);
  }
}

// Workgroups go to the XCDs in turn: workgroup b of a one-dimensional grid
// runs on XCD b % 8.  xcd_contiguous renumbers the nb workgroups so that each
// XCD takes one contiguous range of work items, so neighbouring row segments
// (or strips) run side by side on one XCD and the cache lines at their common
// edge, which both read, come from that XCD's L2 instead of two.  A bijection
// of 0 .. nb-1 for any nb, so results do not depend on the XCD count of the
// device or partition; only the cache benefit assumes eight.  Measured with the same results: the closure sweep
// at 8192^2 FP32 1701-1750 against 1761-1782 us (its reads 1.03x instead of
// 1.12x the algorithmic bytes at 4096^2), the 16-bit DNS sweep at 8192^2
// 844-862 against 916-918 us (FP16); the FP32 pair kernel was 3 % slower with
// it and keeps its two-dimensional grid.
__device__ __forceinline__ int xcd_contiguous(int b, int nb) {
  const int xcd = b & 7, k = b >> 3, q = nb >> 3, rm = nb & 7;
  return xcd < rm ? xcd * (q + 1) + k : rm * (q + 1) + (xcd - rm) * q + k;
}

}  // namespace lbm
