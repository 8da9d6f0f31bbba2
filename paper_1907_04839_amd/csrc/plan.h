// Host-side planning shared by the C-ABI layer and the kernels' launchers:
// the work decomposition of the pair sums, the scale factors, and the byte
// layout of a problem's workspace.  Plain C++ (no HIP), so the host tests
// build it with the sanitizers.
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdlib>

#include "lddmm.h"

namespace lddmm {

// Precision of the pair sums (the FP64 state, loss and optimiser are FP64 in
// every mode).
enum Mode : int { kFP32 = 0, kFP32Comp = 1, kFP64 = 2 };

// Pairs in an FP32 sum, at most, before it is added in FP64 (compensated mode): a
// multiple of the split loops' unroll depths (6 and 3), so that no tile of theirs
// ends in a partial iteration.
constexpr int kTile = 72;

// Launch of a row kernel: a workgroup of ig x jg waves takes ig groups of m
// landmarks i against every j (each wave one group and every jg-th tile of 64
// j), so a step needs no partial sums in memory and no second launch.
struct RowPlan {
  int m;        // landmarks i per wave (0: no row kernel)
  int ig, jg;   // waves per workgroup: i-groups times shares of the j tiles
  int groups;   // workgroups
};
constexpr int kRowGroups = 2;   // i-groups of a row plan's workgroup at most

// Work decomposition of one N x N pair sum.  Landmark i is owned by lane
// (i mod 64) of a wave of i-block ib = i / 64; the j range is split into S
// chunks (one workgroup each) and, inside a workgroup, over W waves.
// Partial sums of different chunks are combined in chunk order.
struct Plan {
  int n;        // landmarks
  int nb;       // i-blocks of 64
  int S;        // j-chunks (workgroups) per i-block
  int W;        // waves per workgroup of the forward pair kernel
  int chunk;    // j per workgroup
  int wchunk;   // j per wave of the forward pair kernel
  int Wa;       // waves per workgroup of the adjoint pair kernel
  int wchunk_a; // j per wave of the adjoint pair kernel
  RowPlan row;  // m > 0: the row kernels take the step instead
  bool chain;   // one launch takes all steps (then row is set too)
};

// Coordinates enter the pair kernels pre-scaled by k = sqrt(log2(e) / (2 sigma^2)),
// so that the kernel value is exp2(-|k q_i - k q_j|^2).
struct Scales {
  double k;         // coordinate pre-scale
  double hq;        // Hq = hq * sum g s (kq_i - kq_j)           = -(c / k)
  double adj_a;     // A  = adj_a * (A1 / kappa - A2)            =  c / k
  double kappa;     // 2 ln 2 = c / k^2 (independent of sigma)
  double bscale;    // adjoint record stores b_hat = bscale * b = kappa k b
  double dt;
};

inline Plan make_plan(int n, int target_waves) {
  Plan p{};
  p.n = n;
  p.nb = (n + 63) / 64;
  // Waves per i-block: enough to give the chip ~target_waves waves, at most
  // 64 and at least 16 pairs per wave.  Workgroups of at most 8 waves:
  // measured on N = 4096, 16384 and 65536, 8-wave workgroups with up to 4x
  // more waves beat 16-wave ones by 3 %, 22 % and 17 % (shorter LDS combine
  // and barriers, two workgroups per CU interleaving their phases); 64 waves
  // per i-block was the best split at N = 4096 and 16384.
  int per_i = (target_waves + p.nb - 1) / p.nb;
  if (per_i > 64) per_i = 64;
  const int max_per_i = n / 16 > 1 ? n / 16 : 1;
  if (per_i > max_per_i) per_i = max_per_i;
  if (per_i < 1) per_i = 1;
  static const int max_w = [] {
    const char* e = std::getenv("LDDMM_MAX_WG_WAVES");
    const int v = e ? std::atoi(e) : 0;
    return (v == 1 || v == 2 || v == 4 || v == 8 || v == 16) ? v : 8;
  }();
  int W = 1;
  while (W * 2 <= per_i && W * 2 <= max_w) W *= 2;
  p.W = W;
  int S = (per_i + W - 1) / W;
  // the combine kernel keeps all S loads in flight for S in {2, 3, 4, 8, 16}
  if (S > 4 && S < 8) S = 4;
  else if (S > 8 && S < 16) S = 8;
  p.S = S < 1 ? 1 : S;
  p.chunk = (n + p.S - 1) / p.S;
  p.wchunk = (p.chunk + W - 1) / W;
  p.Wa = W;
  p.wchunk_a = p.wchunk;
  return p;
}

// Wider workgroups for the plans of 8 waves and 8, 4, 3 or 2 j-chunks.  The
// best width depends on the kernel instance's registers and LDS and on how
// many workgroups share a CU.  Measured per precision mode and kind of step
// (ms per loss+gradient evaluation; widths forward/adjoint 12/12, 8/8, 16/16;
// Euler unless marked; the smaller sizes stand for the shape of a step, the row
// kernels take those up to 5120 in FP32 and 3072 in FP64):
//   FP32-compensated: N = 4096 1.298, 1.351, 1.451; 16384 (T = 4) 1.298,
//     1.322, 1.585; 65536 (T = 3) 14.38, 14.78, 17.35; Runge-Kutta N = 4096
//     (T = 10) 1.317, 1.378, 1.469 -> 12/12 everywhere.  Its 16-wave workgroups,
//     like the FP64 ones, hold 72 KiB of LDS for the wave combine and were slow
//     wherever workgroups share a CU.
//   FP32 (16/16 first): N = 4096 1.213, 1.241, 1.296; 32768 (T = 2) 2.384,
//     2.438, 2.446; 65536 13.93, 14.17, 14.33 -> 16/16; Runge-Kutta N = 4096
//     1.288, 1.269, 1.320 -> 12/12.
//   FP64: N = 4096 2.314, 2.415, 2.694; 16384 2.845, 2.913, 3.310; 65536
//     33.58, 34.43, 41.39 -> 12/12; Runge-Kutta N = 4096 8/8 2.356 against 2.573
//     (12/12) -> unwidened.
// Widths 10 and 14 leave the four SIMDs unevenly loaded (measured slower).
// The sum order within a workgroup follows the width, so results change at
// rounding level.
inline void widen_plan(Plan& p, int mode, bool rk) {
  if (p.W != 8) return;
  if (p.S != 8 && p.S != 4 && p.S != 3 && p.S != 2) return;
  // make_plan also gives 8 x 2 plans at N = 144-271, where 12 or 16 waves
  // would leave fewer than 8 (or no) j per wave: the 8 x 2 widths were
  // measured at N = 65536 only, so they apply where every wave keeps >= 16 j.
  if (p.S == 2 && (p.chunk + 15) / 16 < 16) return;
  if (rk && mode == kFP64) return;
  const int w = mode == kFP32 && !rk ? 16 : 12;
  p.W = p.Wa = w;
  p.wchunk = p.wchunk_a = (p.chunk + w - 1) / w;
}

// The row kernels take the sizes where a step is bound by its launches rather
// than by its pair sums: n <= 5120 with FP32 sums, n <= 3072 in FP64.  Measured
// per loss+gradient evaluation (us, T = 20; split kernels against row kernels):
//   FP32-compensated: n = 200 293 -> 157; 1000 298 -> 187; 1847 339 -> 256;
//     2500 494 -> 353; 3001 550 -> 412; 4096 658 -> 606; 5000 994 -> 907; 6000
//     1133 -> 1150, 8192 1819 -> 1913, 16384 6211 -> 6937, where the split kernels'
//     loops, which have no loads and masks per pair, are the faster ones.
//   FP64: n = 64 222 -> 140 (the split plan's one launch per step runs one
//     workgroup); 500 375 -> 176; 1000 354 -> 233; 1847 475 -> 418; 2500 809 ->
//     722; 3001 933 -> 839; 4096 1188 -> 1340.
// m is chosen for the fullest CU's work, ceil(groups / 256) (m + 1): m rows and
// about one row's time for a wave's loads, the larger m of equals.  At n = 1300
// m = 3, 4, 5 took 219, 234, 260 us, at n = 2500 390, 372, 353; FP64 at n = 2500
// (adjoint step) 25.7 us for m = 2 and 21.8 for m = 4.  One workgroup per CU gets
// 8 waves; with up to two, both are merged into one, whose i-groups share their j
// records in the CU's cache (n = 1847: 266 -> 256 us; FP64 475 -> 418).  FP64 waves
// hold twice the registers: 8 per workgroup at most.  In FP32 workgroups of four
// waves are the better ones from n = 3073 on, where several share a CU and a wave
// still has 12 tiles or more (n = 4096 624 -> 605; but 3001 410 -> 442, 2500 341 ->
// 387).  They end at 72 tiles: the FP32 sums are those of four lanes, of a quarter
// of the tiles each, and cover kTile pairs at most (T = 12, four | eight waves: n =
// 4608 469 | 496, 5000 517 | 532).
inline RowPlan row_plan(int n, int mode) {
  constexpr int kCUs = 256;   // MI355X
  const bool f64 = mode == kFP64;
  RowPlan r{};
  if (n > (f64 ? 3072 : 5120)) return r;
  const int lo = f64 ? 2 : 3, hi = f64 ? 4 : 5;
  const auto groups = [&](int rows) { return (n + rows - 1) / rows; };
  int best = 0;
  for (int m = lo; m <= hi; ++m) {
    const int load = (groups(m) + kCUs - 1) / kCUs * (m + 1);
    if (r.m == 0 || load <= best) {
      best = load;
      r.m = m;
    }
  }
  const int g = groups(r.m), tiles = (n + 63) / 64;
  r.ig = g > kCUs && g <= 2 * kCUs ? 2 : 1;
  r.jg = (f64 ? g > kCUs : n > 3072 && tiles <= kTile) ? 4 : 8;
  if (r.jg > tiles) r.jg = tiles;
  r.groups = groups(r.m * r.ig);
  return r;
}

// The chain kernels take the sizes that one landmark per lane of a wave holds; their
// comment has the figures on both sides of the line.
constexpr int kChainMax = 64;

// Kernels of a server's batches.  Row items are short, so a few jobs of uneven size,
// or one alone, still fill the chip evenly; i-blocks of 64 landmarks run the split
// kernels' faster loops (165 cycles per forward + adjoint pair against about 200)
// but need many workgroups of them: one of n = 8000 keeps a CU for 46 us (forward),
// more than the CU's share of such a batch.  How many jobs share the chip is what a
// server's configuration says, and a job's result must not follow from what else
// runs, so the configuration alone decides.  Time of a solve with rows over blocks,
// all slots full, of jobs of max_n | of max_n / 16 to max_n (Euler, 3D):
//   FP32-compensated  500: 8 slots 0.76 | 0.70, 16 0.95 | 0.75, 32 1.31 | 0.87
//     1000: 8 0.78 | 0.54, 12 0.99 | 0.60, 16 1.13 | 0.67, 32 1.31 | 0.86
//     2000: 1 0.37, 8 0.94 | 0.50, 12 0.91 | 0.60, 16 1.07 | 0.68, 32 1.2 | 0.95
//     4096: 1 0.46, 8 0.95 | 0.60, 12 1.02 | 0.74, 16 1.05 | 0.84
//     8000: 1 0.67, 4 1.01 | 0.70, 8 1.00 to 1.08 | 0.78 (0.74 of 500 to 8000), 12
//       1.08 | 0.88;  12000: 1 0.78, 5 1.02 | 0.78;  15000: 1 0.87, 2 0.97, 4 0.97 | 0.87
//     15500 (from here one job's blocks fill the 256 CUs): 1 0.97, 2 1.05, 4 1.02 | 0.91
//     16000: 1 1.01, 4 1.07 | 0.93;  16384: 1 1.15, 2 1.10;  65536: 1 1.11
//   Runge-Kutta stages the same within 0.04; planar never above 0.96 up to 16000.
//   FP64  1000: 16 slots 0.85 | 0.51, 24 0.95 | 0.57, 32 1.29 | 0.64;  4096: 16 0.95 |
//     0.66;  8000: 8 0.92 | 0.64, 12 1.02 | 0.75, 16 1.06;  16384: 4 0.93;  65536: 0.97
// Both sides of the lines lose something: eight equal jobs of 8000, whose blocks
// happen to fill two rounds, against uneven ones there (5400: 12 slots 1.04 | 0.78).
inline bool batch_blocks(int max_slots, int max_n, int mode) {
  const bool f64 = mode == kFP64;
  return max_slots > (f64 ? 24 : 12) || (!f64 && max_n > 15000) ||
         (long long)max_slots * ((max_n + 63) / 64) > 1024;
}

// Row plans of the batched kernels: four waves of five rows per workgroup.
// Measured (ms; eight jobs of 500 to 8000 landmarks, one of 2000, four of 1500; T = 40,
// 4 iterations; 8-wave items before the loops' later steps):
//   8 waves, m = 5                         43.6   4.22  8.36
//   2 waves, m = 5                         41.6   5.84  7.18
//   4 waves, m = 4, 5, 6, 8                36.6, 34.4, 39.7, 41.2;  3.82, 4.12, 4.76,
//                                          4.82;  6.12, 6.38, 6.80, 7.27
// and FP64 (T = 10) blocks 38.1, 8.90, 9.05, rows 22.2, 1.77, 3.41 (m = 4).
// The waves share the j tiles (jg = 4), which a job alone on the chip needs (one of
// 2000 with jg = 1: 9.5 ms); more i-groups, whose waves share their j records and
// whose workgroups end less often, are the better ones where there are rows enough
// for them (jg = 4 | 2, T = 16: 12 of 4096 29.9 | 28.9, eight of 8000 56.1 | 53.9, one
// of 8000 10.0 | 10.2, one of 4096 (T = 20) 4.65 | 4.63).
// Workgroups of a launch: up to 4096 an item each, so that the hardware balances them
// (2048, 4096, 65536: 12 of 2000 15.2, 14.0, 14.1; eight of 8000 56.1, 53.9, 53.9).
constexpr int kBatchWaves = 4;
constexpr int kBatchRows = 5;
constexpr int kBatchGrid = 4096;

inline RowPlan batch_plan(int n) {
  RowPlan r{};
  r.m = kBatchRows;
  r.jg = n < 3072 ? 4 : n < 16384 ? 2 : 1;
  r.ig = kBatchWaves / r.jg;
  r.groups = (n + r.m * r.ig - 1) / (r.m * r.ig);
  return r;
}

// The most workgroups that a job of at most max_n landmarks has.
inline int batch_groups(int max_n) {
  int g = batch_plan(max_n).groups;
  const int last[2] = {3071, 16383};   // of the plans with more i-groups after them
  for (int k = 0; k < 2; ++k)
    if (last[k] < max_n && batch_plan(last[k]).groups > g) g = batch_plan(last[k]).groups;
  return g;
}

// Tiles that a wave of a batched row kernel sums before it adds them in FP64.  In FP32
// the sums of four lanes are added first, so a lane takes a quarter of kTile.  The rms
// error of A1 / kappa - A2 is 0.85 to 0.91 of the block kernels' (8000 to 32000
// landmarks; 1.0 to 1.5 with kTile tiles, and both terms share a sum here).  It costs
// nothing up to 4096 landmarks and 1 to 3 % above (ms, rounds of 72 | 18: eight jobs of
// 500 to 8000 35.3 | 34.9, eight of 8000 at T = 20 68.2 | 70.2).
constexpr int batch_round(bool f64) { return f64 ? kTile : kTile / 4; }

// Landmark (before the clamp to n - 1) whose state lane `lane` of the wave that ends a
// row workgroup's step loads: its own row, or the workgroup's last one for the
// lanes beyond the workgroup's `rows`.  Other workgroups store the other rows'
// state in the same launch, so none of those may be read.
constexpr int row_state(int row0, int rows, int lane) {
  return row0 + (lane < rows ? lane : rows - 1);
}

// The point flow's cut of the landmarks, by their number alone: eight pairs of equal
// chunks from 1024 landmarks on, before that chunks of 64 landmarks or more.
// Chunks of whole 64-landmark tiles left waves idle just above multiples of 1024 and
// made small sets run mostly padding (us, eight steps of 262144 points, FP32-compensated
// n = 10 64 -> 33, 129 154 -> 114, 1025 625 -> 553; FP64 n = 300 642 -> 522, 4097 6975 ->
// 6410).
struct FlowPlan { int pairs, clen; };

inline FlowPlan flow_plan(int n) {
  FlowPlan f{1, 0};
  while (f.pairs < 8 && f.pairs * 2 * 128 <= n) f.pairs *= 2;
  f.clen = (n + 2 * f.pairs - 1) / (2 * f.pairs);
  return f;
}

inline Scales make_scales(double sigma, int T) {
  Scales s{};
  const double log2e = 1.4426950408889634;
  const double c = 1.0 / (sigma * sigma);
  s.k = std::sqrt(log2e / (2.0 * sigma * sigma));
  s.hq = -c / s.k;
  s.adj_a = c / s.k;
  s.kappa = c / (s.k * s.k);
  s.bscale = s.kappa * s.k;
  s.dt = 1.0 / T;
  return s;
}

// Size in bytes of one point record ((k q, 0, p, 0) or (a, 0, b_hat, 0): eight
// values) and of one partial-sum element.
inline size_t rec_bytes(int mode) { return mode == kFP64 ? 64 : 32; }
inline size_t acc_bytes(int mode) { return mode == kFP32 ? sizeof(float) : sizeof(double); }


inline size_t a256(size_t b) { return (b + 255) & ~size_t(255); }

// Byte offsets of the workspace buffers of one problem.
struct Layout {
  size_t st, ad, hp0, hq0, xc, cen, h0p, out3, traj, arec, ckpt, partial;
  size_t hpT, hqT, hTp, stT, recT;   // energy at t = 1 only (else empty)
  size_t rk_acc, rk_lam;             // Runge-Kutta steps only (else empty)
  size_t total;
  int slots;   // trajectory slots (records: 1 per Euler step, 4 per Runge-Kutta step)
  int nseg;    // checkpoint segments (0 = full trajectory)
};

inline Layout make_layout(const lddmm_params& p, const Plan& plan) {
  Layout L{};
  const size_t n = (size_t)p.n, rb = rec_bytes(p.precision), ab = acc_bytes(p.precision);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += a256(bytes); return o; };
  L.st = take(6 * n * 8);
  L.ad = take(6 * n * 8);
  L.hp0 = take(3 * n * 8);
  L.hq0 = take(3 * n * 8);
  L.xc = take(3 * n * 8);
  L.cen = take(4 * 8);
  L.h0p = take((size_t)plan.nb * 8);
  L.out3 = take(4 * 8);
  const int s = p.ckpt_every;
  const bool ck = s > 0 && s < p.T;
  const int spt = p.integrator == LDDMM_RK4 ? 4 : 1;   // records per step
  L.slots = spt * (ck ? s : p.T) + 1;
  L.nseg = ck ? (p.T + s - 1) / s : 0;
  L.traj = take((size_t)L.slots * n * rb);
  L.arec = take(2 * n * rb);
  L.ckpt = take((size_t)L.nseg * 6 * n * 8);
  L.partial = take(plan.S > 1 ? (size_t)plan.S * 9 * n * ab : 0);
  const bool fin = p.energy == LDDMM_ENERGY_FINAL;
  L.hpT = take(fin ? 3 * n * 8 : 0);
  L.hqT = take(fin ? 3 * n * 8 : 0);
  L.hTp = take(fin ? (size_t)plan.nb * 8 : 0);
  L.stT = take(fin ? 6 * n * 8 : 0);
  L.recT = take(fin ? n * rb : 0);
  L.rk_acc = take(spt == 4 ? 6 * n * 8 : 0);
  L.rk_lam = take(spt == 4 ? 6 * n * 8 : 0);
  L.total = off;
  return L;
}

}  // namespace lddmm
