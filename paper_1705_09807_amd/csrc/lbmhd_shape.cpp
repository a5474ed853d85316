// Strips, segments and rows of the fused schedule's sweeps (host).
#include <algorithm>

#include "lbmhd_internal.h"

namespace lbm {

// Measured on MI355X, 256^2 .. 8192^2, microseconds per step over long runs:
//  * groups of 256 columns, of 128 with the closure off on small grids, where
//    more and narrower strips fill the chip (FP32 512^2 4.1 against 5.1, 700^2 5.4 against
//    6.2; 2048^2 39.8 against 33.0, though 1024^2 8.5 against 9.7);
//  * one workgroup per compute unit: few, tall segments keep few rows of the
//    state open and recompute least (FP32 closure on 4096^2 170.5 against 178.1 with
//    two, 2048^2 49.8 against 56.8, 1024^2 17.4 against 25.0); two for 16-bit storage on
//    tall segments, where the arithmetic of two hides each other's barriers (BF16 8192^2
//    597 against 630, on the shorter segments of 4096^2 161.6 against 154.1);
//  * on large grids strips of whole 64-byte sectors where that takes at most 1/32
//    more strips (FP32 closure on 16384 x 4096 860 against 892, 8192^2 690 against 693,
//    off 3100 x 4096 95.4 against 101.4; most widths within 1 %), with D2Q9, whose
//    rows are longest, whole 128-byte lines for at most 1/8 more (4096^2 closure off
//    248 against 318, on 247 against 301); 16-bit storage is bound by its arithmetic and
//    takes the fewest strips.
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

// Non-temporal stores pay off once the two population buffers no longer fit
// in the 256 MB Infinity Cache; below that the next step re-reads them from it.
bool streaming_stores(const Launch& L) {
  return 2.0 * double(9 + 2 * L.qg) * double(L.nx) * double(L.ny) * double(storage_bytes(L.dtype)) > 256.0e6;
}

// Strip width of the fused closure kernel and of the input vectors: 512 lanes for wide
// grids with FP32 compute, 256 otherwise, 64 for narrow grids and where 256 would leave
// more than 0.3 of their lanes idle (300 x 1000 FP32 11.2 against 13.7 us, 332 x 145 5.5
// against 5.9; 400^2 8.5 against 8.8, 500^2 10.1 against 9.7).
int strip_width(int nx, bool fp32) {
  if (fp32 && nx >= 1024) return 512;
  return nx >= 256 && 10 * (int64_t)nx >= 7 * ((nx + 255) / 256 * 256) ? 256 : 64;
}

// Rows per workgroup of the fused closure kernel.  Measured on MI355X over
// 1024^2 .. 16384^2 (512-lane FP32 strips): one workgroup per compute unit is
// fastest (every strip segment runs concurrently from start to end, and the
// two halo rows re-read per segment are amortised over many rows) as long as
// a segment then holds at most 128 rows (FP32) or 64 rows (FP64); larger
// grids run more, 64-row segments (4096^2: 440 us at 128 rows = one per
// compute unit, 444 us at 64; 8192^2: 1764 us at 64 rows, 1781 us at 512).
int fused_rows(int nx, int ny, int strip, int cus, int cap) {
  const int64_t strips = (nx + strip - 1) / strip;
  const int64_t blocks = cus / strips > 1 ? cus / strips : 1;  // segments per strip column
  int64_t ry = (ny + blocks - 1) / blocks;
  if (ry > cap) ry = 64;
  return (int)(ry < 1 ? 1 : ry);
}

// Segments sized for one workgroup per compute unit, two for k_fused_les_f
// beyond the Infinity Cache (two fit a compute unit; measured 4096^2 FP32
// 448 against 466 us, 8192^2 within 1 % either way, while the cache-resident
// 1024^2 sweep prefers one: 28.7 against 31.4 us).  64-lane strips, of two waves, march
// four to a compute unit (FP64 two where one would have six rows), so that each has fewer
// rows to wait for: 97 x 2675 FP16 26.0 -> 13.4 us, 200 x 1500 FP32 24.2 -> 12.3,
// 200^2 BF16 6.9 -> 5.1, 100 x 1000 FP64 12.2 -> 10.4 (180^2 FP64 6.9 against 7.2).
int les_rows(const Launch& L, int strip) {
  const bool fp32 = L.dtype != LBM_FP64;
  const bool two64 = (int64_t)L.ny * ((L.nx + strip - 1) / strip) >= 6 * (int64_t)L.cus;
  const int per_cu = strip == 64 ? (fp32 ? 4 : (two64 ? 2 : 1)) : (fp32 && streaming_stores(L) ? 2 : 1);
  return fused_rows(L.nx, L.ny, strip, L.cus * per_cu, fp32 ? 128 : 64);
}

}  // namespace lbm
