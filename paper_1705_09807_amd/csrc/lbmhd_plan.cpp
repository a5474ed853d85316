// How many timesteps each launch of a step call advances (host).
#include <algorithm>
#include <limits>

#include "lbmhd_internal.h"

namespace lbm {

constexpr double kNever = std::numeric_limits<double>::infinity();

// Estimated times of a launch of k steps, microseconds, with 16-bit storage, whose sweeps
// are bound by their rows' arithmetic and latencies while the state fits the caches: rows
// marched times the time of a row.  Within 8 % of the measured times (12 % on strips of
// 128 lanes and fewer) from 256^2 to 2048^2 and on flat and tall grids.  FP32 and FP64
// sweeps are bound by the caches' bandwidth instead, which the sizes below describe.

// Closure on.
static double les16_time(const Launch& L, int k) {
  const bool local = L.stencil >= LBM_STENCIL_LOCAL_ISO9;
  if (k == 1) {
    const int W = strip_width(L.nx, true), ry = les_rows(L, W), strips = (L.nx + W - 1) / W;
    const int per_cu = W == 64 ? 4 : (streaming_stores(L) ? 2 : 1);
    const int64_t blocks = int64_t(strips) * ((L.ny + ry - 1) / ry);
    const int64_t waves = (blocks + L.cus * per_cu - 1) / (L.cus * per_cu);
    const double base = W == 512 ? 5.4 : (W == 256 ? 3.5 : 2.6), row = W == 512 ? 1.58 : (W == 256 ? 1.28 : 1.40);
    const double t = base + row * (L.full ? 1.06 : (local ? 0.92 : 1.0)) * double(ry) * double(waves);
    // beyond the caches no faster than its loads and stores
    return streaming_stores(L) ? std::max(t, 76.0 * L.nx * L.ny / 5.0e6) : t;
  }
  const int halo = 2 * k - 1;
  const bool two = !(L.full && k == 3);  // workgroups per compute unit that the LDS holds (checked in launch_k_steps)
  const MsShape s = ms_shape(L, halo, 256, two ? 2 : 1);
  const int rows = (s.ry + halo + 3 * (k - 1) + 1 + 2) / 3 * 3;
  double base, row;
  if (k == 2) {
    base = s.lanes <= 128 ? 2.7 : 2.0;
    row = s.lanes <= 128 ? 0.97 : 1.45;
  } else {
    base = s.lanes <= 128 ? 5.2 : 1.4;
    row = (s.lanes <= 128 ? 1.03 : (L.dtype == LBM_BF16 ? 1.65 : 1.80)) * (L.full && L.dtype == LBM_BF16 ? 1.33 : 1.0);
  }
  // one strip of at most 192 lanes
  if (s.lanes > 128 && s.lanes <= 192 && s.w == L.nx) row *= 0.88;
  // two workgroups on a compute unit against one (8192^2 BF16 three steps 1780 us; two 1415,
  // FP16 1590)
  const double share = s.blocks > L.cus ? (k == 2 ? 1.85 : 1.94) : 1.0;
  return base + row * share * rows;
}

// Closure off, in the caches.
static double off16_time(const Launch& L, int k) {
  const double cells = double(L.nx) * L.ny;
  if (k == 1) {
    // row segments of 256 cells, whole or not
    const double segments = double((L.nx + 255) / 256) * L.ny;
    return std::max(3.9, 2.4 + 1.2e-3 * segments + 6.25e-6 * cells) + (L.nx % 4 ? 0.8 : 0.0);
  }
  const bool deep = cells < dns_deep_cells(2);
  const MsShape s = ms_shape(L, k - 1, deep ? 128 : 256, 1);
  const int march = s.ry + 3 * (k - 1), rows = deep ? march : (march + 3) / 4 * 4;
  // base, per row, per million cells; by k - 2
  constexpr double kDeep[3][3] = {{2.1, 0.79, 0.0}, {1.5, 0.96, 0.0}, {0.8, 1.005, 0.0}};
  constexpr double k128[3][3] = {{2.8, 0.57, 5.5}, {2.1, 0.60, 14.5}, {3.0, 0.56, 16.7}};
  constexpr double k256[3][3] = {{4.0, 0.81, 0.75}, {4.25, 1.05, 0.57}, {4.65, 1.23, 0.80}};
  const double(&c)[3] = (deep ? kDeep : (s.lanes <= 128 ? k128 : k256))[k - 2];
  return (c[0] + c[1] * rows + c[2] * 1e-6 * cells) * (s.blocks > L.cus ? 1.35 : 1.0);
}

// cost[k]: weight of a launch of k steps, kNever where it is not taken.  Sweeps of several
// steps pay where the traffic they save outweighs the rows and columns that they
// recompute and their longer pipeline.  Measured, us per step, several steps (their
// number) against one:
//  * closure off, FP32 and FP64: always (FP32 64^2 2.5 against 3.3, 256^2 3.3 against 4.6,
//    FP64 64^2 2.5 against 3.5, 256^2 4.0 against 6.3); 16-bit beyond the caches always
//    (2048^2 two 45, three 32, four 29 against 60), in them by off16_time: BF16 64^2 four
//    2.7 against 3.9; 512^2 two 6.6, three 5.9, four 5.1 against 5.4; 1024^2 two 11.8, four
//    11.2 against 13.1 (FP16 12.6, 11.2 against 12.9); 32768 x 20 four 11.1 against 9.4;
//  * closure on, FP32: 512^2 11.2 against 9.1, 600^2 11.3 (two) and 11.6 against 13.6;
//    not on grids of one 64-column strip, whose one-step workgroups march four to a
//    compute unit (64 x 8000 16.2 against 15.2, 20 x 32768 40 against 37; D2Q9 three
//    steps 17.6 against 20.0, two 21.1); FP64 two 384^2 10.8 against 10.5, 512^2 13.0 against
//    16.2 (three: 13.7), three 1024^2 29.7 against 35.0 for two; D2Q9 FP64 256^2 10.3
//    against 8.9, 384^2 12.5 against 14.8; below 24 rows, ten of which three steps recompute,
//    two (FP64 32768 x 20 28.7, three 34.7, one 33.1);
//  * closure on, 16-bit: les16_time.  1024^2 BF16 22.7 (two) and 18.9 (three) against
//    18.4, FP16 20.4 against 18.5: its strips of 512 lanes are full and its rows few;
//    1000 x 1048, in strips of 256 lanes, 18.8 and 18.9 against 25.0, 1200^2 20.6 against
//    28.4, 64 x 8000 18.3 against 15.0.
//
// apart: extra time of one-step launches among others.  16-bit storage, closure off, rows not
// of whole quads: their one-step sweeps leave a row on another XCD than the sweeps of
// several steps, which then read it through the Infinity Cache (6.4 us after a launch at
// 97 x 2675, 5.5 at 509 x 512, 3.4 at 725 x 724, 0.5 at 1021 x 1030; none for whole quads).
static void launch_costs(const Launch& L, double (&cost)[kMostSteps + 1], double& apart) {
  const int64_t cells = int64_t(L.nx) * L.ny;
  const size_t bytes = storage_bytes(L.dtype);
  const bool les = L.k2 != 0.0;
  const int most = ms_most_steps(bytes, les, L.qg);
  for (double& c : cost) c = kNever;
  apart = 0.0;
  // fewest launches, of nearly equal numbers of steps
  auto take = [&](int k) { cost[k] = 1.0 + 0.001 * k * k; };
  take(1);
  if (L.learned || L.nx < 16 || L.ny < 16) return;
  if (bytes == 2 && (les || !streaming_stores(L))) {
    // several steps have to gain more than the estimate may be off by; of equals, the fewest launches
    for (int k = 1; k <= most; ++k)
      cost[k] = (k == 1 ? 1.0 : 1.03) * (les ? les16_time(L, k) : off16_time(L, k)) + 0.5;
    if (!les && L.nx % 4) apart = std::max(0.0, 8.0 - 8.0e-6 * cells);
    return;
  }
  for (int k = 2; k <= most; ++k) {
    bool pays = true;
    if (les && bytes == 4) {
      pays = cells >= 360000 && (L.nx > 64 || (L.qg == 9 && k == 3));
      if (k == 3 && L.ny < 24 && L.full) pays = false;
    } else if (les) {
      pays = k == 2 ? cells >= (L.qg == 9 ? 140000 : 160000) : cells >= 400000 && L.ny >= 24;
    }
    if (pays) take(k);
  }
}

StepPlan::StepPlan(const Launch& L, int64_t n, bool keep_parity) {
  fused = L.schedule == LBM_SCHED_FUSED;
  if (n <= 1) {
    one = true;
    return;
  }
  if (!fused) {
    const InplaceSteps s = multi_steps_inplace(L);
    least_steps = s.least;
    most = s.most;
    one = most == 1;
    return;
  }
  double cost[kMostSteps + 1], apart;
  launch_costs(L, cost, apart);
  best = 1;
  for (int k = 2; k <= kMostSteps; ++k)
    if (cost[k] < kNever) most = k;
  for (int k = 2; k <= most; ++k)
    if (cost[k] / k < cost[best] / best) best = k;
  one = most == 1;
  if (one) return;
  const double ones = cost[1];
  cost[1] += apart;
  // least[p][m]: m steps by launches that together advance an even (p = 0) or odd number
  // of steps more than there are launches
  double least[2][kTail + 1];
  for (int m = 0; m <= kTail; ++m)
    for (int p = 0; p < 2; ++p) {
      least[p][m] = m == 0 && p == 0 ? 0.0 : kNever;
      next_of[p][m] = 0;
      for (int k = 1; k <= std::min(m, most); ++k) {
        const double c = cost[k] + least[p ^ ((k - 1) & 1)][m - k];
        if (c < least[p][m]) {
          least[p][m] = c;
          next_of[p][m] = int8_t(k);
        }
      }
    }
  // the steps before the last few go by `best`
  const int64_t lead = n > kTail ? (n - kTail + best - 1) / best : 0;
  const int tail = int(n - lead * best);
  const int lead_parity = int(lead & 1) & ((best - 1) & 1);
  parity = keep_parity ? lead_parity : (least[1][tail] < least[0][tail] ? 1 : 0);
  leading = lead;
  one = double(n) * ones <= double(lead) * cost[best] + least[parity][tail];
}

int StepPlan::next(int64_t left, int64_t t) {
  if (one) return 1;
  if (!fused) {
    // an even number of steps from even times
    const int k = t % 2 ? 1 : int(std::min<int64_t>(left, most)) & ~1;
    return k >= least_steps ? k : 1;
  }
  if (leading > 0) {
    --leading;
    return best;
  }
  const int k = next_of[parity][left];
  parity ^= (k - 1) & 1;
  return k;
}

}  // namespace lbm

// Steps of the launches of lbm_step(n) at time t with `cus` compute units: their number,
// the first `room` of them in `steps` (for the tests: which sweeps a call takes).
extern "C" int64_t lbm_internal_launch_plan(const lbm_params* p, int32_t cus, int64_t n, int64_t t,
                                            int32_t recorded, int32_t* steps, int64_t room) {
  lbm::Launch L;
  if (!lbm::launch_of(p, &L) || cus < 1 || n < 0) return -1;
  lbm::work_layout(L);
  L.cus = cus;
  lbm::StepPlan plan(L, n, recorded != 0);
  int64_t count = 0;
  for (int64_t left = n; left > 0; ++count) {
    const int k = plan.next(left, t);
    if (count < room) steps[count] = k;
    left -= k;
    t += k;
  }
  return count;
}
