// Multi-step sweeps (lbmhd_steps.h) for FP16 and BF16 storage, and their
// dispatch.
#include <algorithm>

#include "lbmhd_steps.h"

namespace lbm {

// Measured on MI355X, 256^2 .. 8192^2, microseconds per step:
//  * groups of 256 columns, of 128 with the closure off on small grids, where
//    more and narrower strips fill the chip (512^2 FP32 5.4 against 7.2, 2048^2 36.8
//    against 34.1);
//  * one workgroup per compute unit: few, tall segments keep few rows of the
//    state open and recompute least (4096^2 FP32 closure on 175 against 180 with
//    two, 2048^2 51 against 59); two for 16-bit storage on tall segments, where
//    the arithmetic of two hides each other's barriers (8192^2 BF16 588 against
//    620, 4096^2 161 against 157);
//  * on large grids strips of whole 64-byte sectors where that takes at most 1/32
//    more strips (8192^2 FP32 closure off 503 against 544, on 665 against 708),
//    with D2Q9, whose rows are longest, whole 128-byte lines for at most 1/8 more
//    (4096^2 closure off 240 against 318, on 249 against 299); 16-bit storage is
//    bound by its arithmetic and takes the fewest strips.
MsShape ms_shape(const Launch& L, int halo, int max_lanes, int per_cu_lds) {
  const int64_t cells = int64_t(L.nx) * L.ny;
  const int bytes = int(storage_bytes(L.dtype));
  MsShape s;
  s.lanes = std::min(L.k2 == 0.0 && cells < 800000 ? 128 : max_lanes, max_lanes);
  s.lanes = std::min(s.lanes, (L.nx + 2 * halo + 63) / 64 * 64);
  const int most = s.lanes - 2 * halo;
  int strips = (L.nx + most - 1) / most;
  s.w = (L.nx + strips - 1) / strips;
  if (bytes > 2 && cells >= (1 << 23)) {
    const int unit = (L.qg == 9 ? 128 : 64) / bytes, part = L.qg == 9 ? 8 : 32;
    const int up = (s.w + unit - 1) / unit * unit, w = up <= most ? up : most / unit * unit;
    const int n = (L.nx + w - 1) / w;
    if (part * n <= (part + 1) * strips) {
      s.w = w;
      strips = n;
    }
  }
  int segs = std::max(1, L.cus / strips);
  if (bytes == 2 && per_cu_lds > 1 && L.ny / segs >= 512) segs = std::max(1, 2 * L.cus / strips);
  s.ry = (L.ny + segs - 1) / segs;
  s.blocks = strips * ((L.ny + s.ry - 1) / s.ry);
  return s;
}

// Grids below these sizes take one-step sweeps: the rows and columns that a
// sweep of several steps recomputes, and its longer pipeline, then cost more than
// the traffic it saves.  Measured (several steps against one): closure on, FP32
// 512^2 11.2 against 9.3 us and 700^2 11.4 against 15.4; BF16 512^2 12.7 against
// 9.6, 600^2 12.8 against 14.5; FP64 two steps 384^2 10.8 against 10.5, 512^2 12.6
// against 16.3 (three: 13.7), three steps 1024^2 30.3 against 37.8 for two; D2Q9
// FP64 256^2 10.3 against 8.9, 384^2 12.5 against 14.8; closure off, FP32 256^2 3.3
// against 4.6 and 64^2 2.5 against 3.3, FP64 64^2 2.5 against 3.5, 256^2 4.0 against
// 6.3, BF16 64^2 2.9 against 4.4, 256^2 3.7 against 4.1, 512^2 5.4 against 5.8.  Flat
// grids of 16-bit storage, whose few rows per segment are mostly recomputed, stay
// too (8000 x 64 closure on 14.3 against 12.1, 32768 x 20 off 14.0 against 10.7;
// FP32 8000 x 64 13.7 against 15.6), and FP16 near 1024^2, whose conversions
// outweigh what the caches leave to save there (closure off 15.6 against 13.7, on 21.9
// against 21.1; 724^2 8.3 against 10.4, 1448^2 21.1 against 26.1).
int multi_steps(const Launch& L) {
  if (L.schedule != LBM_SCHED_FUSED || L.learned || L.nx < 16 || L.ny < 16) return 1;
  const int64_t cells = int64_t(L.nx) * L.ny;
  const size_t bytes = storage_bytes(L.dtype);
  const bool les = L.k2 != 0.0;
  const int most = ms_most_steps(bytes, les, L.qg);
  if (L.dtype == LBM_FP16 && L.nx >= 1024 && cells >= 800000 && cells < 1300000) return 1;
  if (!les) return bytes == 2 && cells >= 300000 && L.ny < 64 ? 1 : most;
  if (bytes <= 4) return cells >= 360000 && (bytes == 4 || L.ny >= 128) ? most : 1;
  return cells >= 400000 ? most : (cells >= (L.qg == 9 ? 140000 : 160000) ? 2 : 1);
}

hipError_t launch_steps_fp64(const Launch& L, int k);
hipError_t launch_steps_fp32(const Launch& L, int k);

hipError_t launch_steps(const Launch& L, int k) {
  switch (L.dtype) {
    case LBM_FP64: return launch_steps_fp64(L, k);
    case LBM_FP32: return launch_steps_fp32(L, k);
    case LBM_FP16: return launch_steps_typed<_Float16>(L, k);
    default: return launch_steps_typed<__bf16>(L, k);
  }
}

}  // namespace lbm
