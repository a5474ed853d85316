// HIP kernels (gfx950) of the learned subgrid closure and the filtered-DNS
// pipeline that trains it.
//
// Method: Flint & Vahala, arXiv 1705.09807.  The analytic closure (Sec. 2.1
// FilterExampleSmall, Sec. 3) keeps the Delta^2/12 term of the filtered
// products; the learned closure adds a per-cell correction of the same four
// subgrid terms (tau_xx, tau_xy, tau_yy, eps), predicted by a 63-64-64-4 ReLU
// network trained on filtered DNS (the convolution of Sec. 1, VelFilter, with
// a Gaussian of variance Delta^2/12).
//
// Network on the matrix cores.  One wave evaluates 32 cells at a time in the
// transposed form H^T = W^T X^T, so that every layer's output (rows = hidden
// units, columns = cells) is directly the B operand of the next layer:
// v_mfma_f32_32x32x16_bf16 with A = 32 rows of W^T x 16 inputs, B = 16
// inputs x 32 cells, D = 32 x 32 FP32 (lane l holds column l % 32 and, in
// register i, row (i/4)*8 + (l/32)*4 + i%4).  The 16-input blocks of layers 2
// and 3 take their B operand from eight consecutive accumulator registers,
// which hold hidden rows (2 b + j/4) * 8 + (l/32) * 4 + j % 4; the packed A
// operands use the same permutation of the contraction index.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "lbmhd_device.h"
#include "lbmhd_internal.h"
#include "lbmhd_learned.h"
#include "lbmhd_mlp_device.h"

namespace lbm {

// ---------------------------------------------------------------------------
// Packing
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_mlp_pack(const float* __restrict__ p, const lbm_mlp_norm* __restrict__ norm, char* __restrict__ pk) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  __bf16* a = reinterpret_cast<__bf16*>(pk);
  if (e < 4096) {  // A1: W1^T rows
    const int ot = e / 2048, kb = (e / 512) % 4, l = (e / 8) % 64, j = e % 8;
    const int hid = ot * 32 + l % 32, k = kb * 16 + (l / 32) * 8 + j;
    a[kPkA1 / 2 + e] = __bf16(k < 63 ? p[LBM_MLP_OFF_W1 + k * 64 + hid] : 0.0f);
  } else if (e < 8192) {  // A2: W2^T rows, chained contraction order
    const int f = e - 4096;
    const int ot = f / 2048, kb = (f / 512) % 4, l = (f / 8) % 64, j = f % 8;
    const int out = ot * 32 + l % 32, k = chained_k(kb, l / 32, j);
    a[kPkA2 / 2 + f] = __bf16(p[LBM_MLP_OFF_W2 + k * 64 + out]);
  } else if (e < 10240) {  // A3: W3^T rows 0..3, rest zero
    const int f = e - 8192;
    const int kb = f / 512, l = (f / 8) % 64, j = f % 8;
    const int o = l % 32, k = chained_k(kb, l / 32, j);
    a[kPkA3 / 2 + f] = __bf16(o < 4 ? p[LBM_MLP_OFF_W3 + k * 4 + o] : 0.0f);
  } else if (e < 10240 + 64) {
    const int i = e - 10240;
    reinterpret_cast<float*>(pk + kPkB1)[i] = p[LBM_MLP_OFF_B1 + i];
    reinterpret_cast<float*>(pk + kPkB2)[i] = p[LBM_MLP_OFF_B2 + i];
    reinterpret_cast<float*>(pk + kPkB3)[i] = i < 4 ? p[LBM_MLP_OFF_B3 + i] : 0.0f;
  } else if (e < 10240 + 64 + 32) {
    const int i = e - 10240 - 64;
    reinterpret_cast<float*>(pk + kPkNorm)[i] = reinterpret_cast<const float*>(norm)[i];
  } else if (e < 10240 + 64 + 32 + 4096) {  // A1n: W1^T rows, patch-ordered inputs
    const int f = e - (10240 + 64 + 32);
    const int ot = f / 2048, kb = (f / 512) % 4, l = (f / 8) % 64, j = f % 8;
    const int hid = ot * 32 + l % 32, pos = kb * 2 + l / 32;
    // element j < 7: field j at pos; element 7: field pos at position 8
    const int k = j < 7 ? j * 9 + pos : (pos < 7 ? pos * 9 + 8 : -1);
    __bf16* c = reinterpret_cast<__bf16*>(pk + kPkA1n);
    c[f] = __bf16(k >= 0 ? p[LBM_MLP_OFF_W1 + k * 64 + hid] : 0.0f);
  }
}

// ---------------------------------------------------------------------------
// Forward on feature rows (inference of given inputs; also the parity probe
// of the matrix-core network)
// ---------------------------------------------------------------------------

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void global_void;

// Layer-1 operand kb of lane half h from the eight features u, v at kb*16 + h*8
// (FP32): z = (x - shift) * scale per field, pad 0, rounded to bfloat16.  Sets
// *ood when any |z| exceeds the limit.
__device__ __forceinline__ void feature_operands(const f32x4& u, const f32x4& v, int kb, int h, const lbm_mlp_norm* nm,
                                                 bf16x8& zb, bool* ood) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = kb * 16 + h * 8 + j;
    const float xv = j < 4 ? u[j] : v[j - 4];
    float z = 0.0f;
    if (k < 63) {
      const int f = feat_field(k);
      z = (xv - nm->shift[f]) * nm->scale[f];
    }
    *ood = *ood || !(fabsf(z) <= kOodLimit);  // NaN counts as out of range
    zb[j] = __bf16(z);
  }
}

// A wave takes 32 rows at a time, 8 KB in one stretch, loaded straight into LDS
// (16 bytes a lane).  The 16-byte piece c of row r goes to place c ^ (r % 16) of
// that row, so the lanes that then read the same piece of 32 rows spread over the
// banks.  The next rows are on their way while the network runs.  Measured 2^20 rows: operands read from memory with a
// row's stride between lanes 96 us, this form 66 us.
__global__ void __launch_bounds__(256)
k_mlp_forward(const char* __restrict__ pk, const float* __restrict__ x, int64_t n, float* __restrict__ y,
              int32_t* __restrict__ ood_out) {
  __shared__ f32x4 rows[4][32 * 16];
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t wave = (int64_t)blockIdx.x * 4 + wid;
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  const lbm_mlp_norm* nm = reinterpret_cast<const lbm_mlp_norm*>(pk + kPkNorm);
  MlpA w;
  load_mlp(pk, lane, w);
  auto fetch = [&](int64_t g) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = i * 4 + (lane >> 4), c = (lane & 15) ^ (r & 15);
      const int64_t src = g * 32 + r < n ? g * 32 + r : n - 1;
      __builtin_amdgcn_global_load_lds((global_void*)(x + src * 64 + c * 4), (lds_void*)(&rows[wid][i * 64]), 16, 0, 0);
    }
  };
  if (wave * 32 < n) fetch(wave);
  for (int64_t g = wave; g * 32 < n; g += nwaves) {
    __builtin_amdgcn_s_waitcnt(0);  // the loads into LDS are complete
    const int64_t row = g * 32 + (lane & 31);
    f32x4 in[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int r = lane & 31, j = (k >> 1) * 4 + h * 2 + (k & 1);
      in[k] = rows[wid][r * 16 + (j ^ (r & 15))];
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): read, so the next rows may arrive
    __builtin_amdgcn_sched_barrier(0);
    if ((g + nwaves) * 32 < n) fetch(g + nwaves);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 zb[4];
    bool o = false;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) feature_operands(in[2 * kb], in[2 * kb + 1], kb, h, nm, zb[kb], &o);
    const f32x4 v = mlp_wave(w, zb, reinterpret_cast<const float*>(pk + kPkB1), lane, nullptr, nullptr);
    // every lane takes part in the exchange (a short-circuit would leave the
    // flagged lane inactive and its partner would read nothing from it)
    const int partner = __shfl_xor(int(o), 32, 64);
    const bool oo = o || partner != 0;
    if (h == 0 && row < n) {
      *reinterpret_cast<f32x4*>(y + row * 4) = v;
      if (ood_out) ood_out[row] = oo ? 1 : 0;
    }
  }
}

// ---------------------------------------------------------------------------
// Correction of a simulation state, second stage: the network on the per-cell
// input vectors (CellIn, 16 bytes per cell) that the first stage wrote from
// the state.  A workgroup loads the vectors of a 64 x 16 tile and its
// one-cell halo straight into LDS (one 16-byte load per cell, no register
// staging), then evaluates the network for its 1024 cells (each wave 8 groups
// of 32).  Layer 1 contracts over four 16-input blocks of patch positions
// (kPkA1n): a lane's operand of a block is one 16-byte LDS read whose last
// element is replaced by a field of position 8.  A cell is out of
// distribution when a flagged cell lies in its 3x3 neighbourhood (its 63
// inputs are exactly the seven fields there).  Output: four FP32 planes
// tau_xx, tau_xy, tau_yy, eps = out_scale * y, 0 for out-of-distribution cells
// and cells whose output is not finite.
// ---------------------------------------------------------------------------
constexpr int kCorrTX = 64, kCorrTY = 16;
constexpr int kCorrLX = kCorrTX + 2, kCorrLY = kCorrTY + 2, kCorrPL = kCorrLX * kCorrLY;

// LDS cell offset of patch position pos (< 9: row pos / 3, column pos % 3)
// of tile cell (ty, tx) from ty * LX + tx: the patch corner is at (ty, tx)
// in the tile with its one-cell halo.
__host__ __device__ constexpr int corr_patch_offset(int pos) { return (pos / 3) * kCorrLX + pos % 3; }

// Periodic wrap of v in [-1, n + kCorrLX) into [0, n).
__device__ __forceinline__ int wrap_halo(int v, int n, bool wide) {
  if (wide) {
    v = v < 0 ? v + n : v;
    return v >= n ? v - n : v;
  }
  v %= n;
  return v < 0 ? v + n : v;
}

__global__ void __launch_bounds__(256, 2)
k_mlp_correct(const CellIn* __restrict__ in, const char* __restrict__ pk, float* __restrict__ corr, int nx, int ny) {
  constexpr int LX = kCorrLX, PL = kCorrPL, PER = (PL + 255) / 256;
  __shared__ CellIn zt[PER * 256];
  __shared__ __attribute__((aligned(16))) float bias[132];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, h = lane >> 5;
  const int x0 = blockIdx.x * kCorrTX, y0 = blockIdx.y * kCorrTY;
  const int64_t n = (int64_t)nx * ny;
  const bool wide_x = nx >= LX, wide_y = ny >= kCorrLY;
  // each wave fills 64 consecutive entries per pass (entry base + lane)
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = tid + 256 * i;
    if (e < PL) {
      const int ly = e / LX, lx = e - ly * LX;
      const int gx = wrap_halo(x0 + lx - 1, nx, wide_x), gy = wrap_halo(y0 + ly - 1, ny, wide_y);
      __builtin_amdgcn_global_load_lds((global_void*)(in + ((int64_t)gy * nx + gx)),
                                       (lds_void*)(zt + 256 * i + 64 * wid), 16, 0, 0);
    }
  }
  if (tid < 132) bias[tid] = reinterpret_cast<const float*>(pk + kPkB1)[tid];
  const lbm_mlp_norm* nm = reinterpret_cast<const lbm_mlp_norm*>(pk + kPkNorm);
  MlpA w;
  load_mlp_n(pk, lane, w);
  const float os0 = nm->out_scale[0], os1 = nm->out_scale[1], os2 = nm->out_scale[2], os3 = nm->out_scale[3];
  __builtin_amdgcn_s_waitcnt(0);  // the loads into LDS are complete
  __syncthreads();
  for (int g = wid; g < kCorrTX * kCorrTY / 32; g += 4) {
    const int ty = g >> 1, tx = (g & 1) * 32 + (lane & 31), base = ty * LX + tx;
    CellIn v[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) v[kb] = zt[base + (h ? corr_patch_offset(2 * kb + 1) : corr_patch_offset(2 * kb))];
    const CellIn v8 = zt[base + corr_patch_offset(8)];
    bf16x8 zb[4];
    bool bad;
    patch_operands(v, v8, h, zb, &bad);
    // the two halves of a cell see complementary patch positions.  Every lane
    // takes part in the exchange: under a short-circuit only the lanes with
    // bad == false would run it, the value they send would be known to be 0,
    // and the compiler drops the exchange altogether.
    const int partner = __shfl_xor(int(bad), 32, 64);
    const bool pb = bad || partner != 0;
    const f32x4 y = mlp_wave(w, zb, bias, lane, nullptr, nullptr);
    const bool o = pb || !(isfinite(y[0]) && isfinite(y[1]) && isfinite(y[2]) && isfinite(y[3]));
    const int gx = x0 + tx, gy = y0 + ty;
    if (h == 0 && gx < nx && gy < ny) {
      float* cp = corr + ((int64_t)gy * nx + gx);
      // non-temporal stores: the planes are read by the next sweep, after the
      // whole grid is written (measured together with the input vectors'
      // non-temporal stores: the 16384^2 learned step 0.5-1 % faster)
      __builtin_nontemporal_store(o ? 0.0f : y[0] * os0, cp);
      __builtin_nontemporal_store(o ? 0.0f : y[1] * os1, cp + n);
      __builtin_nontemporal_store(o ? 0.0f : y[2] * os2, cp + 2 * n);
      __builtin_nontemporal_store(o ? 0.0f : y[3] * os3, cp + 3 * n);
    }
  }
}

// ---------------------------------------------------------------------------
// Training: forward and backward on the matrix cores.  A workgroup takes chunks
// of 64 batch rows (32 per wave in the forward).  With the
// batch row r, the loss L = sum (y - t)^2 / (4 batch) and straight-through
// gradients of the bfloat16 roundings:
//   d3 = dL/dy,  d2 = (d3 W3^T) [h2 > 0],  d1 = (d2 W2^T) [h1 > 0],
//   G3 = h2^T d3, G2 = h1^T d2, G1 = z^T d1, biases: column sums of d.
// d3 and d2 are formed in FP32 on the vector ALU (contraction over the four
// outputs).  d1^T = W2 d2^T is one matrix-core product in the transposed
// form of the forward (hidden units x rows, d2 in the accumulator layout of
// h2, so it is directly the B operand), and G2, G1 are products over the 64
// rows of the chunk from feature-major LDS tiles.  A delta enters the matrix
// cores as three bfloat16 terms, d = hi + mid + lo + O(2^-25 |d|), so the
// products carry the FP32 delta; activations and weights are bfloat16
// already.  (Two terms, 16 bits, left 1e-4 relative errors in G1 over 5000
// rows, where the row sums cancel.)  Each wave owns half of a weight gradient and
// accumulates it over its workgroup's chunks in a fixed order; per-workgroup
// partials are summed in a fixed order by k_mlp_reduce.
// ---------------------------------------------------------------------------
constexpr int kTrainChunk = 64;
constexpr int kTrainBlocksMax = 1024;
constexpr int kGradStride = 8704;  // floats per partial (>= LBM_MLP_PARAMS, 256-byte multiple)
constexpr int kTs = 72;            // bfloat16 per feature row of an LDS tile (64 rows + pad)

struct TrainLds {
  __bf16 z[64][kTs], h1[64][kTs], h2[64][kTs];     // [feature][chunk row]
  __bf16 d2h[64][kTs], d2m[64][kTs], d2l[64][kTs], d1h[64][kTs], d1m[64][kTs], d1l[64][kTs];
  bf16x8 a1[2][4][64], a2[2][4][64], a3[4][64];    // A operands of the forward
  bf16x8 a2b[2][4][64];                            // A operands of d1^T = W2 d2^T
  float d3[4][kTrainChunk];
  float w3[64 * 4];                                // bfloat16-rounded W3
  float bias[64 + 64 + 4];
  double loss[64];
};

// hi + mid + lo bfloat16 split of eight floats (each remainder is exact in
// FP32, so the three terms carry 24 bits).
__device__ __forceinline__ void split_bf16x8(const float* v, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
  f32x8 a, b, c;
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = v[j];
  hi = to_bf16x8(a);
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = v[j] - float(hi[j]);
  mid = to_bf16x8(b);
#pragma unroll
  for (int j = 0; j < 8; ++j) c[j] = b[j] - float(mid[j]);
  lo = to_bf16x8(c);
}

// One 32 x 32 tile of sum_r A[m][r] B[n][r] over the 64 rows of the chunk,
// from feature-major LDS tiles (operands: 8 consecutive rows per lane); the
// B tile is split hi + mid + lo.
__device__ __forceinline__ f32x16 rows_product(f32x16 acc, const __bf16 (*a)[kTs], const __bf16 (*bh)[kTs],
                                               const __bf16 (*bm)[kTs], const __bf16 (*bl)[kTs], int ma, int nb,
                                               int lane) {
  const int r0 = (lane >> 5) * 8, la = lane & 31;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    const bf16x8 av = *reinterpret_cast<const bf16x8*>(&a[ma + la][kb * 16 + r0]);
    const bf16x8 hv = *reinterpret_cast<const bf16x8*>(&bh[nb + la][kb * 16 + r0]);
    const bf16x8 mv = *reinterpret_cast<const bf16x8*>(&bm[nb + la][kb * 16 + r0]);
    const bf16x8 lv = *reinterpret_cast<const bf16x8*>(&bl[nb + la][kb * 16 + r0]);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, hv, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, mv, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, lv, acc, 0, 0, 0);
  }
  return acc;
}

// ReLU'd bfloat16 activations of two accumulator tiles (as activate()), stored
// feature-major for chunk row sl; also returned as the next layer's B operands.
__device__ __forceinline__ void activate_to_lds(const f32x16 acc[2], bf16x8 hb[4], __bf16 (*dst)[kTs], int h,
                                                int sl) {
  activate(acc, hb, nullptr);
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int j = 0; j < 8; ++j) dst[chained_k(kb, h, j)][sl] = hb[kb][j];
}

__device__ __forceinline__ void adam_update(int i, float g, float* __restrict__ p, float* __restrict__ m,
                                            float* __restrict__ v, float lr, float bc1, float bc2) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mi = b1 * m[i] + (1.0f - b1) * g;
  const float vi = b2 * v[i] + (1.0f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// Four waves per workgroup: all of them round the weights into operands (straight
// from the FP32 parameters); waves 0 and 1 run the forward pass of 32 rows each
// while 2 and 3 prepare the backward operands; in the backward pass wave w forms
// half w / 2 of d1 for the rows of half w % 2, and then two 32 x 32 tiles of one weight
// gradient.  A chain of dependent phases, too short for the chip to fill: bound by
// their latencies.  Measured, batch 4096 (64 workgroups): two waves reading
// operands packed by a launch of their own, 3.7 + 17.9 us; this form 16.1 us.
__global__ void __launch_bounds__(256)
k_mlp_train(const float* __restrict__ p, const lbm_mlp_norm* __restrict__ nm, const float* __restrict__ x,
            const float* __restrict__ t, const int32_t* __restrict__ idx, int batch, float* __restrict__ partial,
            double* __restrict__ loss_part) {
  __shared__ TrainLds s;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *b1 = s.bias, *b2 = s.bias + 64, *b3 = s.bias + 128;
  const int half = wid & 1, part = wid >> 1;       // rows and work of this wave
  const int sl = half * 32 + (lane & 31);          // chunk row of this lane
  const int chunks = (batch + kTrainChunk - 1) / kTrainChunk;
  // this lane's eight 16-byte pieces of its row of a chunk and the row's targets,
  // asked for before anything else needs them (the first chunk's during the weights)
  f32x4 in[8], tv;
  auto fetch = [&](int c) __attribute__((always_inline)) {
    const int64_t row = idx[min(c * kTrainChunk + sl, batch - 1)];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      in[k] = *reinterpret_cast<const f32x4*>(x + row * 64 + (k >> 1) * 16 + h * 8 + (k & 1) * 4);
    tv = *reinterpret_cast<const f32x4*>(t + row * 4);
  };
  if (part == 0) fetch(blockIdx.x);
  if (tid >= 128 && tid < 192) s.bias[tid - 128] = p[LBM_MLP_OFF_B1 + tid - 128];
  if (tid >= 192) s.bias[tid - 128] = p[LBM_MLP_OFF_B2 + tid - 192];
  if (tid >= 128 && tid < 132) s.bias[tid] = p[LBM_MLP_OFF_B3 + tid - 128];
  // A operands of the forward (the order of lbm_mlp_pack): W1^T, W2^T in the chained
  // contraction order, W3^T rows 0 .. 3
  for (int e = wid; e < 20; e += 4) {
    bf16x8 v;
    if (e < 8) {
      const int ot = e >> 2, kb = e & 3;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = kb * 16 + h * 8 + j;
        v[j] = __bf16(k < 63 ? p[LBM_MLP_OFF_W1 + k * 64 + ot * 32 + (lane & 31)] : 0.0f);
      }
      s.a1[ot][kb][lane] = v;
    } else if (e < 16) {
      const int ot = (e - 8) >> 2, kb = e & 3;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = __bf16(p[LBM_MLP_OFF_W2 + chained_k(kb, h, j) * 64 + ot * 32 + (lane & 31)]);
      s.a2[ot][kb][lane] = v;
    } else {
      const int kb = e - 16, o = lane & 31;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = __bf16(o < 4 ? p[LBM_MLP_OFF_W3 + chained_k(kb, h, j) * 4 + (o & 3)] : 0.0f);
      s.a3[kb][lane] = v;
    }
  }
  // gradient accumulators: waves 0 and 1 own rows [32 half, 32 half + 32) of G2,
  // waves 2 and 3 those of G1 (two 32 x 32 tiles each, columns 0..31 and 32..63);
  // thread tid owns an entry of G3, threads 0..63 one of b2's, 64..127 one of b1's
  // and 128..131 one of b3's bias gradients
  f32x16 gw[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int e = 0; e < 16; ++e) gw[c][e] = 0.0f;
  float g3 = 0.0f, gb = 0.0f;
  double loss = 0.0;
  const float inv = 2.0f / (float(batch) * 4.0f);
  __syncthreads();
  for (int c = blockIdx.x; c < chunks; c += gridDim.x) {
    if (part == 0) {
      // forward (the operations of mlp_wave), activations to LDS
      const bool valid = c * kTrainChunk + sl < batch;
      bf16x8 zb[4];
      bool o = false;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) feature_operands(in[2 * kb], in[2 * kb + 1], kb, h, nm, zb[kb], &o);
      const f32x4 target = tv;
      if (c + int(gridDim.x) < chunks) fetch(c + gridDim.x);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int j = 0; j < 8; ++j) s.z[kb * 16 + h * 8 + j][sl] = zb[kb][j];
      f32x16 acc[2];
      bf16x8 hb[4];
#pragma unroll
      for (int ot = 0; ot < 2; ++ot) {
        acc[ot] = bias_tile(b1, ot, h);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
          acc[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.a1[ot][kb][lane], zb[kb], acc[ot], 0, 0, 0);
      }
      activate_to_lds(acc, hb, s.h1, h, sl);
#pragma unroll
      for (int ot = 0; ot < 2; ++ot) {
        acc[ot] = bias_tile(b2, ot, h);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
          acc[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.a2[ot][kb][lane], hb[kb], acc[ot], 0, 0, 0);
      }
      activate_to_lds(acc, hb, s.h2, h, sl);
      f32x16 out;
#pragma unroll
      for (int i = 0; i < 16; ++i) out[i] = 0.0f;
      if (h == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = b3[i];
      }
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
        out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.a3[kb][lane], hb[kb], out, 0, 0, 0);
      if (h == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float r = out[q] - target[q] / nm->out_scale[q];
          s.d3[q][sl] = valid ? inv * r : 0.0f;
          if (valid) loss += double(r) * double(r);
        }
      }
    } else if (c == blockIdx.x) {
      // A operands of d1^T = W2 d2^T: row i = ot*32 + lane%32 of W2, contraction
      // index j in the chained order of the accumulator layout
      for (int e = half; e < 8; e += 2) {
        const int ot = e >> 2, kb = e & 3;
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          v[j] = __bf16(p[LBM_MLP_OFF_W2 + (ot * 32 + (lane & 31)) * 64 + chained_k(kb, h, j)]);
        s.a2b[ot][kb][lane] = v;
      }
      for (int e = tid - 128; e < 256; e += 128) s.w3[e] = bf16_round(p[LBM_MLP_OFF_W3 + e]);
    }
    __syncthreads();
    // d2 in the accumulator layout of h2 (element kb*8 + j: hidden
    // chained_k(kb, h, j)), then half `part` of d1^T = W2 d2^T
    {
      float d3v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) d3v[q] = s.d3[q][sl];
      bf16x8 dh[4], dm[4], dl[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        float d2[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int ck = chained_k(kb, h, j);
          const float* w3 = &s.w3[ck * 4];
          const float a = w3[0] * d3v[0] + w3[1] * d3v[1] + w3[2] * d3v[2] + w3[3] * d3v[3];
          d2[j] = float(s.h2[ck][sl]) > 0.0f ? a : 0.0f;
        }
        split_bf16x8(d2, dh[kb], dm[kb], dl[kb]);
        if ((kb >> 1) == part) {  // both waves of these rows have it: each stores half
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int ck = chained_k(kb, h, j);
            s.d2h[ck][sl] = dh[kb][j];
            s.d2m[ck][sl] = dm[kb][j];
            s.d2l[ck][sl] = dl[kb][j];
          }
        }
      }
      const int ot = part;
      f32x16 acc;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        const bf16x8 a = s.a2b[ot][kb][lane];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dh[kb], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dm[kb], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dl[kb], acc, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float d1[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int hid = ot * 32 + acc_row(q * 8 + j, h);
          d1[j] = float(s.h1[hid][sl]) > 0.0f ? acc[q * 8 + j] : 0.0f;
        }
        bf16x8 hi, mi, lo;
        split_bf16x8(d1, hi, mi, lo);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int hid = ot * 32 + acc_row(q * 8 + j, h);
          s.d1h[hid][sl] = hi[j];
          s.d1m[hid][sl] = mi[j];
          s.d1l[hid][sl] = lo[j];
        }
      }
    }
    __syncthreads();
    // weight gradients over the chunk's rows
#pragma unroll
    for (int cn = 0; cn < 2; ++cn)
      gw[cn] = part == 0 ? rows_product(gw[cn], s.h1, s.d2h, s.d2m, s.d2l, half * 32, cn * 32, lane)
                         : rows_product(gw[cn], s.z, s.d1h, s.d1m, s.d1l, half * 32, cn * 32, lane);
    {
      // G3[tid / 4][tid % 4]; biases
      const bf16x8* hv = reinterpret_cast<const bf16x8*>(s.h2[tid >> 2]);
      const f32x4* dv = reinterpret_cast<const f32x4*>(s.d3[tid & 3]);
#pragma unroll
      for (int r = 0; r < kTrainChunk / 8; ++r) {
        const bf16x8 a = hv[r];
        const f32x4 u = dv[2 * r], v = dv[2 * r + 1];
#pragma unroll
        for (int j = 0; j < 8; ++j) g3 += float(a[j]) * (j < 4 ? u[j & 3] : v[j & 3]);
      }
    }
    if (part == 0) {
      const int bh = lane;
      const bf16x8* ph = reinterpret_cast<const bf16x8*>(half == 0 ? s.d2h[bh] : s.d1h[bh]);
      const bf16x8* pm = reinterpret_cast<const bf16x8*>(half == 0 ? s.d2m[bh] : s.d1m[bh]);
      const bf16x8* pl = reinterpret_cast<const bf16x8*>(half == 0 ? s.d2l[bh] : s.d1l[bh]);
#pragma unroll
      for (int r = 0; r < kTrainChunk / 8; ++r) {
        const bf16x8 a = ph[r], m = pm[r], l = pl[r];
#pragma unroll
        for (int j = 0; j < 8; ++j) gb += (float(a[j]) + float(m[j])) + float(l[j]);
      }
    } else if (tid < 132) {
      const f32x4* dv = reinterpret_cast<const f32x4*>(s.d3[tid - 128]);
#pragma unroll
      for (int r = 0; r < kTrainChunk / 4; ++r) {
        const f32x4 v = dv[r];
#pragma unroll
        for (int j = 0; j < 4; ++j) gb += v[j];
      }
    }
    __syncthreads();
  }
  float* out = partial + (int64_t)blockIdx.x * kGradStride;
#pragma unroll
  for (int cn = 0; cn < 2; ++cn)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = half * 32 + acc_row(e, h), n = cn * 32 + (lane & 31);
      out[(part == 0 ? LBM_MLP_OFF_W2 : LBM_MLP_OFF_W1) + m * 64 + n] = gw[cn][e];
    }
  out[LBM_MLP_OFF_W3 + tid] = g3;
  if (part == 0)
    out[(half == 0 ? LBM_MLP_OFF_B2 : LBM_MLP_OFF_B1) + lane] = gb;
  else if (tid < 132)
    out[LBM_MLP_OFF_B3 + tid - 128] = gb;
  // loss: fixed-order sum over the lanes that hold outputs
  if (part == 0 && h == 0) s.loss[sl] = loss;
  __syncthreads();
  if (tid == 0) {
    double a = 0.0;
    for (int k = 0; k < 64; ++k) a += s.loss[k];
    loss_part[blockIdx.x] = a;
  }
}

// Sum of the partial gradients (and of the loss partials) in a fixed order: each
// run of kReduceGroup consecutive partials in order, then the runs' sums in order;
// with ADAM the update follows (Kingma & Ba 2015, bias corrections bc1 = 1 -
// beta1^t, bc2 = 1 - beta2^t).  A workgroup takes 64 parameters, a wave a run at a
// time, so the loads of many partials are in flight at once.  Measured, 64 partials: three
// launches (runs, their sum, the update) 4.1 + 3.0 + 2.3 us, this one 3.9 us.
constexpr int kReduceGroup = 16;

template <bool ADAM>
__global__ void __launch_bounds__(256)
k_mlp_reduce(const float* __restrict__ partial, int nparts, float* __restrict__ grad,
             const double* __restrict__ loss_part, float* __restrict__ loss_out, float loss_norm,
             float* __restrict__ p, float* __restrict__ m, float* __restrict__ v, float lr, float bc1, float bc2) {
  constexpr int kRuns = kTrainBlocksMax / kReduceGroup;
  __shared__ float run[kRuns][64];
  __shared__ double loss_run[kRuns];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const int runs = (nparts + kReduceGroup - 1) / kReduceGroup;
  for (int g = wid; g < runs; g += 4) {
    const int b0 = g * kReduceGroup, nb = min(kReduceGroup, nparts - b0);
    if (i < LBM_MLP_PARAMS) {
      float q[kReduceGroup];
#pragma unroll
      for (int k = 0; k < kReduceGroup; ++k) q[k] = k < nb ? partial[(int64_t)(b0 + k) * kGradStride + i] : 0.0f;
      float a = q[0];
#pragma unroll
      for (int k = 1; k < kReduceGroup; ++k)
        if (k < nb) a += q[k];
      run[g][lane] = a;
    }
  }
  const bool with_loss = blockIdx.x == 0 && loss_out;
  if (with_loss && int(threadIdx.x) < runs) {
    const int b0 = threadIdx.x * kReduceGroup, nb = min(kReduceGroup, nparts - b0);
    double a = loss_part[b0];
    for (int k = 1; k < nb; ++k) a += loss_part[b0 + k];
    loss_run[threadIdx.x] = a;
  }
  __syncthreads();
  if (wid == 0 && i < LBM_MLP_PARAMS) {
    float g = 0.0f;
    for (int k = 0; k < runs; ++k) g += run[k][lane];
    if constexpr (ADAM) {
      adam_update(i, g, p, m, v, lr, bc1, bc2);
    } else {
      grad[i] = g;
    }
  }
  if (with_loss && threadIdx.x == 64) {
    double a = 0.0;
    for (int k = 0; k < runs; ++k) a += loss_run[k];
    *loss_out = float(a * double(loss_norm));
  }
}

__global__ void __launch_bounds__(256)
k_mlp_adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v, const float* __restrict__ grad,
           float lr, float bc1, float bc2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < LBM_MLP_PARAMS) adam_update(i, grad[i], p, m, v, lr, bc1, bc2);
}

// ---------------------------------------------------------------------------
// Normalisation statistics, FP64, one pass over the rows: counts, sums, and sums
// of squared deviations from the mean, combined pairwise (Chan, Golub & LeVeque
// 1983: M2 = M2_a + M2_b + (mean_b - mean_a)^2 n_a n_b / n) from threads to waves,
// workgroups and, in a second kernel, the whole, always in the same order.  A
// thread takes the deviations of its rows from its first row, so nothing cancels
// beyond its few rows.  Bound by HBM (the centre features touch every line of a
// row).  Measured 2^20 rows: two passes and two one-thread final sums 2 x 53 + 2 x
// 65 us, this form 51 + 9 us.
// ---------------------------------------------------------------------------
constexpr int kStatBlocks = 256;
constexpr int kStatVals = 26;  // count, 7 sums, 7 means, 7 M2, 4 sums of squared targets

struct Stats {
  double n, sum[7], mean[7], m2[7], t2[4];
};

__device__ __forceinline__ void stats_add(Stats& a, const Stats& b) {
  const double n = a.n + b.n;
  if (b.n != 0.0) {
    const double wb = b.n / n, w = a.n * wb;
#pragma unroll
    for (int f = 0; f < 7; ++f) {
      const double d = b.mean[f] - a.mean[f];
      a.mean[f] = a.n == 0.0 ? b.mean[f] : a.mean[f] + d * wb;
      a.m2[f] = a.n == 0.0 ? b.m2[f] : a.m2[f] + b.m2[f] + d * d * w;
    }
  }
#pragma unroll
  for (int f = 0; f < 7; ++f) a.sum[f] += b.sum[f];
#pragma unroll
  for (int o = 0; o < 4; ++o) a.t2[o] += b.t2[o];
  a.n = n;
}

// Sum over a workgroup of 256 threads; the result is in thread 0's s.
__device__ void block_stats(Stats& s) {
  static_assert(sizeof(Stats) == kStatVals * sizeof(double), "layout");
  __shared__ Stats red[4];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    Stats o;
    const double* src = reinterpret_cast<const double*>(&s);
    double* dst = reinterpret_cast<double*>(&o);
#pragma unroll
    for (int k = 0; k < kStatVals; ++k) dst[k] = __shfl_down(src[k], off, 64);
    if ((threadIdx.x & 63) + off >= 64) o.n = 0.0;  // no such lane
    if ((threadIdx.x & (2 * off - 1)) == 0) stats_add(s, o);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < 4; ++w) stats_add(s, red[w]);
}

__global__ void __launch_bounds__(256)
k_stats_pass(const float* __restrict__ x, const float* __restrict__ t, int64_t n, Stats* __restrict__ part) {
  Stats s;
  double ref[7], dev[7];
  s.n = 0.0;
#pragma unroll
  for (int f = 0; f < 7; ++f) s.sum[f] = s.mean[f] = s.m2[f] = ref[f] = dev[f] = 0.0;
#pragma unroll
  for (int o = 0; o < 4; ++o) s.t2[o] = 0.0;
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t r0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t r = r0; r < n; r += stride) {
    const f32x4 tv = *reinterpret_cast<const f32x4*>(t + r * 4);
#pragma unroll
    for (int f = 0; f < 7; ++f) {
      const double v = x[r * 64 + f * 9 + 4];
      if (r == r0) ref[f] = isfinite(v) ? v : 0.0;
      const double d = v - ref[f];
      s.sum[f] += v;
      dev[f] += d;
      s.m2[f] += d * d;
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) s.t2[o] += double(tv[o]) * double(tv[o]);
    s.n += 1.0;
  }
  if (s.n != 0.0) {
#pragma unroll
    for (int f = 0; f < 7; ++f) {
      const double d = dev[f] / s.n;
      s.mean[f] = ref[f] + d;
      s.m2[f] -= dev[f] * d;
    }
  }
  block_stats(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Statistics of the whole -> normalisation.
__global__ void __launch_bounds__(256)
k_stats_final(const Stats* __restrict__ part, int nparts, lbm_mlp_norm* __restrict__ norm) {
  Stats s;
  if (threadIdx.x < nparts) {
    s = part[threadIdx.x];
  } else {
    double* z = reinterpret_cast<double*>(&s);
#pragma unroll
    for (int k = 0; k < kStatVals; ++k) z[k] = 0.0;
  }
  block_stats(s);
  if (threadIdx.x != 0) return;
  lbm_mlp_norm nm;
  for (int k = 0; k < 8; ++k) {
    nm.shift[k] = 0.0f;
    nm.scale[k] = 1.0f;
  }
#pragma unroll
  for (int f = 0; f < 7; ++f) {
    const double sd = sqrt(s.m2[f] / s.n);
    nm.shift[f] = float(s.sum[f] / s.n);
    nm.scale[f] = sd > 0.0 ? float(1.0 / sd) : 1.0f;
  }
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const double rms = sqrt(s.t2[o] / s.n);
    nm.out_scale[o] = rms > 0.0 ? float(rms) : 1.0f;
  }
  for (int k = 0; k < 12; ++k) nm.pad[k] = 0.0f;
  *norm = nm;
}

// ---------------------------------------------------------------------------
// Filtered DNS: Gaussian taps, x pass (12 products, subsampled columns), y
// pass (subsampled rows).  FP64 throughout.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_gauss_taps(double sigma2, int R, double* __restrict__ taps) {
  __shared__ double wv[256];
  const int r = threadIdx.x;
  if (r <= 2 * R) {
    const double d = double(r - R);
    wv[r] = exp(-d * d / (2.0 * sigma2));
  }
  __syncthreads();
  if (r == 0) {
    double s = 0.0;
    for (int k = 0; k <= 2 * R; ++k) s += wv[k];
    wv[255] = s;
  }
  __syncthreads();
  if (r <= 2 * R) taps[r] = wv[r] / wv[255];
}

// x pass.  A workgroup forms the 12 products of one row's fine cells once (they are
// used by 2 R / FACTOR + 1 outputs), in LDS, and each of its four waves
// filters three of them: a lane computes B adjacent outputs, so a value read from LDS
// serves up to B of them.  A fine cell x of the segment sits at [x % (B FACTOR)][x /
// (B FACTOR)], so the lanes of a wave, B FACTOR cells apart, read consecutive
// doubles.  Taps are uniform (scalar loads).  Bound by HBM (40 B read, 96 B /
// FACTOR written per fine cell) and the LDS reads.  A workgroup takes several rows, the
// next one's cells on their way during the filter, and SMALL (2 R at most 6 P) lets
// three workgroups share a compute unit.  Measured 4096^2, FACTOR 4, R = 24: one
// thread per output forming its own products (and three divisions) per tap 1502 us,
// one row per workgroup 441 us; the whole filter with that 685 us, in this form 580
// (FACTOR 8, R = 35: 545 and 510; FACTOR 16, R = 70: 667 and 552).
template <int FACTOR, bool SMALL>
struct FilterX {
  static constexpr int B = FACTOR <= 4 ? 2 : 1;       // outputs per lane
  static constexpr int P = B * FACTOR;                // fine cells between lanes
  static constexpr int E = SMALL ? 6 * P : 2 * 127;   // most fine cells past the lanes' own
  static constexpr int N0 = 64 + (E + P - 1) / P;
  static constexpr int NI = N0 + (N0 % 16 == 0);       // neighbouring cells in different banks
  static constexpr int NE = (64 * P + E + 255) / 256;  // fine cells per thread
};

// The three products at `v` of one row at the lane's outputs: out(product, output, value).
template <int FACTOR, bool SMALL, typename Out>
__device__ __forceinline__ void filter_row(const double* v, int R, const double* __restrict__ taps, Out&& out) {
  constexpr int B = FilterX<FACTOR, SMALL>::B, P = FilterX<FACTOR, SMALL>::P, NI = FilterX<FACTOR, SMALL>::NI;
  double acc[3][B];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[k][b] = 0.0;
  // position t of a lane's window is tap t - b FACTOR of its output b
  const int end = 2 * R + (B - 1) * FACTOR;
  for (int t0 = 0; t0 <= end; t0 += P) {
    const double* vq = v + t0 / P;
    if (t0 >= (B - 1) * FACTOR && t0 + P - 1 <= 2 * R) {  // every tap of the body exists
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double a = vq[(k * P + p) * NI];
#pragma unroll
          for (int b = 0; b < B; ++b) acc[k][b] += taps[t0 + p - b * FACTOR] * a;
        }
    } else {
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          const int r = t0 + p - b * FACTOR;
          if (r < 0 || r > 2 * R) continue;  // uniform
          const double w = taps[r];
#pragma unroll
          for (int k = 0; k < 3; ++k) acc[k][b] += w * vq[(k * P + p) * NI];
        }
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int b = 0; b < B; ++b) out(k, b, acc[k][b]);
}

template <int FACTOR, bool SMALL>
__global__ void __launch_bounds__(256)
k_filter_x(const double* __restrict__ mom, int nx, int ny, int R, int rows, const double* __restrict__ taps,
           double* __restrict__ tmp) {
  using F = FilterX<FACTOR, SMALL>;
  constexpr int B = F::B, P = F::P, NI = F::NI, NE = F::NE;
  extern __shared__ double prod[];  // [12][P][NI]
  const int tid = threadIdx.x, lane = tid & 63;
  const int k0 = 3 * __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cx = nx / FACTOR;
  const int X0 = blockIdx.x * 64 * B;
  // fine cells of the segment's outputs: few on narrow grids and at a ragged end (lanes past
  // the last output read cells that are not there; their sums are dropped)
  const int count = min(64 * P, (cx - X0) * FACTOR) + 2 * R;
  const int y0 = blockIdx.y * rows, y1 = min(y0 + rows, ny);
  const int64_t n = (int64_t)nx * ny, cn = (int64_t)cx * ny;
  const double* v = prod + k0 * P * NI + lane;
  int xs[NE];
  double f[NE][5];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    int xx = (X0 * FACTOR - R + min(tid + 256 * i, count - 1)) % nx;
    xs[i] = xx < 0 ? xx + nx : xx;
  }
  auto load = [&](int y) __attribute__((always_inline)) {
    const double* row = mom + (int64_t)y * nx;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      if (256 * i >= count) break;  // uniform
#pragma unroll
      for (int k = 0; k < 5; ++k) f[i][k] = row[k * n + xs[i]];
    }
  };
  load(y0);
  for (int y = y0; y < y1; ++y) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = tid + 256 * i;
      if (e >= count) break;
      const double rho = f[i][0], mx = f[i][1], my = f[i][2], bx = f[i][3], by = f[i][4];
      const double p[12] = {rho, mx, my, bx, by, mx * mx / rho, mx * my / rho, my * my / rho,
                            bx * bx, bx * by, by * by, (mx * by - my * bx) / rho};
#pragma unroll
      for (int k = 0; k < 12; ++k) prod[(k * P + e % P) * NI + e / P] = p[k];
    }
    __syncthreads();
    if (y + 1 < y1) load(y + 1);
    filter_row<FACTOR, SMALL>(v, R, taps, [&](int k, int b, double a) __attribute__((always_inline)) {
      const int X = X0 + lane * B + b;
      if (X < cx) tmp[(k0 + k) * cn + (int64_t)y * cx + X] = a;
    });
    __syncthreads();  // the row's products are read
  }
}

// y pass: a lane computes B outputs of one column, so a row it reads serves several of them,
// where that leaves enough waves to hide the loads' latency (filter_y_outputs).  Measured
// 4096^2 by 4, R = 24: 503 us with one output per thread, 202 us with four.
template <int B>
__global__ void __launch_bounds__(64)
k_filter_y(const double* __restrict__ tmp, int nx, int ny, int factor, int R, const double* __restrict__ taps,
           double* __restrict__ out) {
  constexpr int U = B == 1 ? 8 : 4;  // rows in flight
  const int cx = nx / factor, cy = ny / factor;
  const int X = blockIdx.x * 64 + threadIdx.x, Y = blockIdx.y * B, k = blockIdx.z;
  if (X >= cx) return;
  const int64_t cn = (int64_t)cx * ny;
  const double* col = tmp + k * cn + X;
  double acc[B];
#pragma unroll
  for (int b = 0; b < B; ++b) acc[b] = 0.0;
  const int end = 2 * R + (B - 1) * factor;
  int yy = (Y * factor - R) % ny;
  if (yy < 0) yy += ny;
  auto next = [&]() __attribute__((always_inline)) {
    const double a = col[(int64_t)yy * cx];
    yy = yy + 1 == ny ? 0 : yy + 1;
    return a;
  };
  auto some = [&](int t) __attribute__((always_inline)) {
    const double a = next();
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int r = t - b * factor;
      if (r >= 0 && r <= 2 * R) acc[b] += taps[r] * a;  // uniform
    }
  };
  int t = 0;
  for (; t < (B - 1) * factor && t <= end; ++t) some(t);
  for (; t + U - 1 <= 2 * R; t += U) {  // every tap exists
    double a[U];
#pragma unroll
    for (int j = 0; j < U; ++j) a[j] = next();
#pragma unroll
    for (int j = 0; j < U; ++j)
#pragma unroll
      for (int b = 0; b < B; ++b) acc[b] += taps[t + j - b * factor] * a[j];
  }
  for (; t <= end; ++t) some(t);
#pragma unroll
  for (int b = 0; b < B; ++b)
    if (Y + b < cy) out[(int64_t)k * cx * cy + (int64_t)(Y + b) * cx + X] = acc[b];
}

// ---------------------------------------------------------------------------
// Training samples on the coarse grid: inputs and exact-minus-analytic
// targets of every cell (FP64 arithmetic, FP32 output).  A workgroup takes a
// tile of cells: velocities (one division per component and cell) and B of the
// tile with a two-cell halo in LDS, from them the seven FP32 input fields with a
// one-cell halo, and from those the rows, 16 lanes per cell with 16-byte stores.
// Bound by the 272 B written per cell.  Measured 1024^2: one thread per cell
// recomputing every neighbour's fields 842 us, 98 us.
// ---------------------------------------------------------------------------
constexpr int kSampX = 32, kSampY = 8;

template <int STENCIL>
__global__ void __launch_bounds__(256)
k_closure_samples(const double* __restrict__ c12, int nx, int ny, double k2, float* __restrict__ xo,
                  float* __restrict__ to) {
  constexpr int DX = kSampX + 4, DY = kSampY + 4, FX = kSampX + 2, FY = kSampY + 2;
  __shared__ double uv[4][DY][DX];     // u_x, u_y, B_x, B_y
  __shared__ float fld[7 * FY * FX + 1];  // input fields; the last entry is the zero pad
  const int tid = threadIdx.x;
  const int x0 = blockIdx.x * kSampX, y0 = blockIdx.y * kSampY;
  const int64_t n = (int64_t)nx * ny;
  auto wrap = [](int v, int m) {
    v %= m;
    return v < 0 ? v + m : v;
  };
  for (int e = tid; e < DY * DX; e += 256) {
    const int ly = e / DX, lx = e - ly * DX;
    const int64_t c = (int64_t)wrap(y0 + ly - 2, ny) * nx + wrap(x0 + lx - 2, nx);
    const double rho = c12[c];
    uv[0][ly][lx] = c12[n + c] / rho;
    uv[1][ly][lx] = c12[2 * n + c] / rho;
    uv[2][ly][lx] = c12[3 * n + c];
    uv[3][ly][lx] = c12[4 * n + c];
    if (ly >= 1 && ly <= FY && lx >= 1 && lx <= FX) fld[(ly - 1) * FX + lx - 1] = float(rho);
  }
  if (tid == 0) fld[7 * FY * FX] = 0.0f;
  __syncthreads();
  for (int e = tid; e < FY * FX; e += 256) {
    const int fy = e / FX, fx = e - fy * FX, ly = fy + 1, lx = fx + 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) fld[(k + 1) * FY * FX + e] = float(uv[k][ly][lx]);
    // w: (u_y, u_x); J_z: (B_y, B_x)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const auto& p = uv[2 * k + 1];
      const auto& q = uv[2 * k];
      fld[(5 + k) * FY * FX + e] =
          float(0.5 * (p[ly][lx + 1] - p[ly][lx - 1]) - 0.5 * (q[ly + 1][lx] - q[ly - 1][lx]));
    }
  }
  __syncthreads();
  {
    // features 4 q .. 4 q + 3 of a cell from its corner's entry
    const int q = tid & 15;
    int off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 4 * q + j, f = k / 9, d = k - 9 * f;
      off[j] = k < 63 ? f * FY * FX + (d / 3) * FX + d % 3 : -1;
    }
    for (int c = tid >> 4; c < kSampX * kSampY; c += 16) {
      const int cy = c / kSampX, cxl = c - cy * kSampX;
      if (x0 + cxl >= nx || y0 + cy >= ny) continue;
      const int base = cy * FX + cxl;
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = fld[off[j] < 0 ? 7 * FY * FX : base + off[j]];
      *reinterpret_cast<f32x4*>(xo + ((int64_t)(y0 + cy) * nx + x0 + cxl) * 64 + 4 * q) = v;
    }
  }
  const int x = x0 + (tid & (kSampX - 1)), y = y0 + tid / kSampX;
  if (x >= nx || y >= ny) return;
  const int xe = x + 1 == nx ? 0 : x + 1, xw = x == 0 ? nx - 1 : x - 1;
  const int64_t rc = (int64_t)y * nx, rn = (int64_t)(y + 1 == ny ? 0 : y + 1) * nx,
                rs = (int64_t)(y == 0 ? ny - 1 : y - 1) * nx, c = rc + x;
  auto at = [&](int k) { return c12[k * n + c]; };
  // exact subgrid terms of the filtered products
  const double rho = at(0), mx = at(1), my = at(2), bx = at(3), by = at(4);
  const double rxx = at(5) - mx * mx / rho, rxy = at(6) - mx * my / rho, ryy = at(7) - my * my / rho;
  const double qxx = at(8) - bx * bx, qxy = at(9) - bx * by, qyy = at(10) - by * by;
  const double eps = at(11) - (mx * by - my * bx) / rho;
  // analytic closure of the filtered fields
  double g[4][2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double* f = c12 + (1 + k) * n;
    grad3x3<double, STENCIL>(f[rc + xe], f[rc + xw], f[rn + x], f[rs + x], f[rn + xe], f[rn + xw], f[rs + xe],
                             f[rs + xw], g[k][0], g[k][1]);
  }
  const Closure<double> cl =
      closure_terms(g[0][0], g[0][1], g[1][0], g[1][1], g[2][0], g[2][1], g[3][0], g[3][1], 1.0 / rho, k2);
  const double a_xx = 0.5 * (cl.tau_s + cl.tau_d), a_yy = 0.5 * (cl.tau_s - cl.tau_d);
  f32x4 v;
  v[0] = float((rxx + 0.5 * (qyy - qxx)) - a_xx);
  v[1] = float((rxy - qxy) - cl.tau_xy);
  v[2] = float((ryy + 0.5 * (qxx - qyy)) - a_yy);
  v[3] = float(eps - cl.eps);
  *reinterpret_cast<f32x4*>(to + c * 4) = v;
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
static int train_blocks(int batch) {
  const int chunks = (batch + kTrainChunk - 1) / kTrainChunk;
  return chunks < kTrainBlocksMax ? chunks : kTrainBlocksMax;
}

// Work of a training step: per-workgroup partial gradients and loss partials (with
// room for a packed network before and a reduced gradient after them, as callers
// have sized it).
size_t mlp_train_work_bytes(int batch) {
  const int blocks = train_blocks(batch);
  return (size_t)LBM_MLP_PACKED_BYTES + (size_t)blocks * kGradStride * sizeof(float) +
         ((size_t)blocks * sizeof(double) + 255) / 256 * 256 + (size_t)kGradStride * sizeof(float);
}

hipError_t launch_mlp_pack(const float* params, const lbm_mlp_norm* norm, void* packed, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_pack, dim3((10240 + 64 + 32 + 4096 + 255) / 256), dim3(256), 0, st, params, norm,
                     static_cast<char*>(packed));
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const void* packed, const float* x, int64_t n, float* y, int32_t* ood, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int64_t groups = (n + 31) / 32;
  // two workgroups fit a compute unit (its registers hold the weights); more
  // would only load the weights again
  int64_t blocks = (groups + 3) / 4;
  if (blocks > 512) blocks = 512;
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const char*>(packed), x, n,
                     y, ood);
  return hipGetLastError();
}

struct AdamArgs {
  float *p = nullptr, *m = nullptr, *v = nullptr;
  float lr = 0, bc1 = 1, bc2 = 1;
};
static AdamArgs adam_args(float* params, float* m, float* v, int64_t step, double lr) {
  return AdamArgs{params, m, v, float(lr), float(1.0 - pow(0.9, double(step))), float(1.0 - pow(0.999, double(step)))};
}

// Batch gradient into grad, or the Adam step with it.
template <bool ADAM>
static hipError_t launch_batch(const float* params, const lbm_mlp_norm* norm, const float* x, const float* t,
                               const int32_t* idx, int batch, void* work, float* grad, float* loss, const AdamArgs& ad,
                               hipStream_t st) {
  char* w = static_cast<char*>(work);
  const int blocks = train_blocks(batch);
  float* partial = reinterpret_cast<float*>(w + LBM_MLP_PACKED_BYTES);
  double* lpart = reinterpret_cast<double*>(w + LBM_MLP_PACKED_BYTES + (size_t)blocks * kGradStride * sizeof(float));
  hipLaunchKernelGGL(k_mlp_train, dim3(blocks), dim3(256), 0, st, params, norm, x, t, idx, batch, partial, lpart);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_reduce<ADAM>, dim3((LBM_MLP_PARAMS + 63) / 64), dim3(256), 0, st, partial, blocks, grad,
                     lpart, loss, float(1.0 / (double(batch) * 4.0)), ad.p, ad.m, ad.v, ad.lr, ad.bc1, ad.bc2);
  return hipGetLastError();
}

hipError_t launch_mlp_gradient(const float* params, const lbm_mlp_norm* norm, const float* x, const float* t,
                               const int32_t* idx, int batch, void* work, float* grad, float* loss, hipStream_t st) {
  return launch_batch<false>(params, norm, x, t, idx, batch, work, grad, loss, AdamArgs{}, st);
}

hipError_t launch_mlp_adam(float* params, float* m, float* v, const float* grad, int64_t step, double lr,
                           hipStream_t st) {
  const AdamArgs ad = adam_args(params, m, v, step, lr);
  hipLaunchKernelGGL(k_mlp_adam, dim3((LBM_MLP_PARAMS + 255) / 256), dim3(256), 0, st, params, m, v, grad, ad.lr,
                     ad.bc1, ad.bc2);
  return hipGetLastError();
}

hipError_t launch_mlp_train(float* params, float* m, float* v, int64_t step, double lr, const lbm_mlp_norm* norm,
                            const float* x, const float* t, const int32_t* idx, int batch, void* work,
                            float* loss, hipStream_t st) {
  return launch_batch<true>(params, norm, x, t, idx, batch, work, nullptr, loss, adam_args(params, m, v, step, lr), st);
}

// Training step without a caller-provided work buffer.  Its work (per-workgroup
// partial gradients, loss partials; every byte the kernels read is written earlier in the same step, so nothing
// needs clearing) lives in this fixed device array, one copy per GPU that the
// library runs on, held until the process ends.  In host code `scratch` names
// a host-side stand-in, not device memory: kernels get the address that
// hipGetSymbolAddress returns on the current device, looked up once per device
// at the first call there.
static __device__ __align__(256) char scratch[LBM_MLP_TRAIN_NOALLOC_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

hipError_t scratch_on_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

bool mlp_train_noalloc_limit_ok(int batch) {
  return batch >= 1 && batch <= LBM_MLP_TRAIN_NOALLOC_BATCH && mlp_train_work_bytes(batch) <= sizeof(scratch);
}

hipError_t launch_mlp_train_noalloc(float* params, float* m, float* v, int64_t step, double lr,
                                    const lbm_mlp_norm* norm, const float* x, const float* t, const int32_t* idx,
                                    int batch, float* loss, hipStream_t st) {
  if (!mlp_train_noalloc_limit_ok(batch)) return hipErrorInvalidValue;
  void* work = nullptr;
  const hipError_t e = scratch_on_current_device(&work);
  if (e != hipSuccess) return e;
  return launch_mlp_train(params, m, v, step, lr, norm, x, t, idx, batch, work, loss, st);
}

size_t mlp_stats_work_bytes() { return kStatBlocks * sizeof(Stats); }

hipError_t launch_mlp_stats(const float* x, const float* t, int64_t n, lbm_mlp_norm* norm, void* work,
                            hipStream_t st) {
  Stats* part = static_cast<Stats*>(work);
  const int64_t want = (n + 255) / 256;
  const int blocks = int(want < kStatBlocks ? want : kStatBlocks);
  hipLaunchKernelGGL(k_stats_pass, dim3(blocks), dim3(256), 0, st, x, t, n, part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(256), 0, st, part, blocks, norm);
  return hipGetLastError();
}

int filter_radius(double delta) { return (int)ceil(5.0 * (delta / sqrt(12.0))); }

size_t filter_work_bytes(int nx, int ny, int factor) {
  return 256 * sizeof(double) + (size_t)12 * (size_t)(nx / factor) * (size_t)ny * sizeof(double);
}

template <int FACTOR, bool SMALL>
static hipError_t launch_filter_x(const double* mom, int nx, int ny, int R, const double* taps, double* tmp,
                                  hipStream_t st) {
  using F = FilterX<FACTOR, SMALL>;
  if constexpr (!SMALL) {
    if (2 * R <= 6 * F::P) return launch_filter_x<FACTOR, true>(mom, nx, ny, R, taps, tmp, st);
  }
  const size_t lds = (size_t)12 * F::P * F::NI * sizeof(double);
  const auto kernel = &k_filter_x<FACTOR, SMALL>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int per = 64 * F::B, across = (nx / FACTOR + per - 1) / per;
  // rows per workgroup: up to 8, while there are 1024 workgroups
  const int rows = (int)std::min<int64_t>(8, std::max<int64_t>(1, (int64_t)across * ny / 1024));
  hipLaunchKernelGGL(kernel, dim3(across, (ny + rows - 1) / rows), dim3(256), lds, st, mom, nx, ny, R, rows, taps,
                     tmp);
  return hipGetLastError();
}

// Outputs per lane of the y pass: fewer where its waves are too few to hide a lane's chain
// of loads.  Measured, the whole filter with one, two and four: 256^2 by 4 (768 waves of
// one output) 32.0, 32.6 and 37.6 us, 256^2 by 16 45, 59 and 82, 1024^2 by 8 (3072) 47.5, 49.4 and
// 60.2, 1536^2 by 8 (6912) 66.6, 65.6 and 74.7, 1536^2 by 4 (27648) 122, 125 and 109 with R = 24
// and 85.8, 77.8 and 80.0 with R = 6, 4096^2 by 2 1067, 842 and 777.
static int filter_y_outputs(int cx, int cy) {
  const int64_t waves = (int64_t)12 * ((cx + 63) / 64) * cy;  // of one output per lane
  return waves >= 12288 ? 4 : (waves >= 6144 ? 2 : 1);
}

hipError_t launch_filter(const double* mom, int nx, int ny, int factor, double delta, double* out, void* work,
                         hipStream_t st) {
  const int R = filter_radius(delta);
  double* taps = static_cast<double*>(work);
  double* tmp = taps + 256;
  hipLaunchKernelGGL(k_gauss_taps, dim3(1), dim3(256), 0, st, delta * delta / 12.0, R, taps);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int cx = nx / factor, cy = ny / factor;
  switch (factor) {
    case 1: e = launch_filter_x<1, false>(mom, nx, ny, R, taps, tmp, st); break;
    case 2: e = launch_filter_x<2, false>(mom, nx, ny, R, taps, tmp, st); break;
    case 4: e = launch_filter_x<4, false>(mom, nx, ny, R, taps, tmp, st); break;
    case 8: e = launch_filter_x<8, false>(mom, nx, ny, R, taps, tmp, st); break;
    default: e = launch_filter_x<16, false>(mom, nx, ny, R, taps, tmp, st);
  }
  if (e != hipSuccess) return e;
  const auto y_pass = [&](auto b) {
    constexpr int B = decltype(b)::value;
    hipLaunchKernelGGL(k_filter_y<B>, dim3((cx + 63) / 64, (cy + B - 1) / B, 12), dim3(64), 0, st, tmp, nx, ny, factor,
                       R, taps, out);
    return hipGetLastError();
  };
  switch (filter_y_outputs(cx, cy)) {
    case 1: return y_pass(std::integral_constant<int, 1>{});
    case 2: return y_pass(std::integral_constant<int, 2>{});
    default: return y_pass(std::integral_constant<int, 4>{});
  }
}

hipError_t launch_closure_samples(const double* c12, int nx, int ny, double delta, int stencil, float* x, float* t,
                                  hipStream_t st) {
  const dim3 g((nx + kSampX - 1) / kSampX, (ny + kSampY - 1) / kSampY), b(256);
  const double k2 = delta * delta / 12.0;
  if (stencil == LBM_STENCIL_ISO9)
    hipLaunchKernelGGL(k_closure_samples<LBM_STENCIL_ISO9>, g, b, 0, st, c12, nx, ny, k2, x, t);
  else
    hipLaunchKernelGGL(k_closure_samples<LBM_STENCIL_CENTRAL5>, g, b, 0, st, c12, nx, ny, k2, x, t);
  return hipGetLastError();
}

hipError_t launch_mlp_correct(const void* cell_in, const void* packed, float* corr, int nx, int ny, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_correct, dim3((nx + kCorrTX - 1) / kCorrTX, (ny + kCorrTY - 1) / kCorrTY), dim3(256), 0, st,
                     static_cast<const CellIn*>(cell_in), static_cast<const char*>(packed), corr, nx, ny);
  return hipGetLastError();
}

}  // namespace lbm
