// HIP kernels for landmark geodesic shooting on gfx950 (CDNA4).
//
// The hot path is the all-pairs Gaussian-kernel sums of one explicit Euler
// step of the Hamiltonian flow (eq. 2 with H = 1/2 <p, K(q) p>, eq. 1) and of
// its exact discrete adjoint, which together give dL/dp0 for the loss of
// eq. 3.  The paper streams pair terms through on-chip memory instead of
// materialising the N x N kernel matrix (Sec. 2.5); this file keeps that idea
// and re-plans it for wave64 hardware:
//
//  * Large problems (split kernels): lane l of a wave owns landmark i = 64 ib + l
//    and keeps its data and its running sums in VGPRs.  The j landmarks are
//    wave-uniform, so their records arrive through scalar loads into SGPRs and
//    every VALU instruction of the pair term reads at most one SGPR operand;
//    there is no LDS traffic and no barrier inside the j loop.
//  * A few thousand landmarks (row kernels, and the batched kernels of the
//    server): lanes own the j, a wave's few rows i are uniform, a workgroup sees
//    every j of its rows and ends the step in the same launch.  Up to 64
//    landmarks (chain kernels) one launch takes all steps.
//  * Coordinates are stored pre-scaled by k = sqrt(log2(e) / (2 sigma^2)), so
//    g_ij = exp2(-|k q_i - k q_j|^2) is one v_exp_f32 with a negate modifier.
//    A forward pair costs 16 VALU + 1 exp, an adjoint pair 35 to 37 VALU + 1 exp.
//  * The split kernels' j range is cut over the W waves of a workgroup and, when
//    one workgroup per i-block would not fill the chip, over S workgroups.
//    Partials are combined in a fixed order (waves through LDS, workgroups
//    through a [S][C][N] buffer): no float atomics, so results are
//    bit-reproducible and depend only on N and the precision (a served job's also on
//    its server's configuration), never on what else is running.
//  * Precision modes: FP32 with one running FP32 sum per wave ("naive", in the
//    split kernels); FP32 with FP32 sums of at most 72 pairs folded into FP64
//    ("compensated", and both FP32 modes of the other kernels); or everything in
//    FP64 (with an own 2^x).  The live state (q, p, a, b), the Euler updates, the
//    Hamiltonian and the loss are FP64 in every mode.
//  * Planar problems instantiate the same loops without the z terms, and
//    the flow of arbitrary points (eq. 4) carries its points through all steps of
//    the stored trajectory in a single launch.
//  * Classical Runge-Kutta steps (an option beside the paper's Euler steps)
//    reuse the pair loops stage by stage; separate compile-time instances
//    (RKS) hold the stage bookkeeping so that the Euler kernels carry none.
#include "shoot_internal.h"

#include <hip/hip_ext.h>

#include <cstdlib>
#include <type_traits>

namespace lddmm {

namespace {

constexpr int kLossThreads = 1024;

// Point record: (k q, 0, p, 0) for the trajectory, (a, 0, b_hat, 0) for the
// adjoint.  Eight scalars so that one record is one 32-byte (FP32) or
// 64-byte (FP64) scalar load.
template <typename R>
struct alignas(8 * sizeof(R)) Rec {
  R x, y, z, u, px, py, pz, w;
};

// Pointers that arrive through a descriptor in memory carry no address
// space; the pair loops read records through a global (address space 1)
// pointer so that wave-uniform loads can become scalar loads.
template <typename T>
using GlobalPtr = const __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ GlobalPtr<T> global_ptr(const T* p) {
  return (GlobalPtr<T>)p;
}

template <typename R, bool COMP>
struct AccOf { using type = double; };

template <typename R>
struct Rec;

// Record j as one 8-wide vector load (an address-space-qualified struct
// cannot be copied as a whole): a wave-uniform j gives one s_load_dwordx8
// (FP32) or s_load_dwordx16 (FP64) that the compiler issues ahead of use.
template <typename R>
using Vec8 = R __attribute__((ext_vector_type(8)));

template <typename R>
__device__ __forceinline__ Rec<R> load_rec(GlobalPtr<Rec<R>> p, int j) {
  const Vec8<R> v = *reinterpret_cast<GlobalPtr<Vec8<R>>>(p + j);
  Rec<R> r;
  r.x = v[0]; r.y = v[1]; r.z = v[2]; r.u = v[3];
  r.px = v[4]; r.py = v[5]; r.pz = v[6]; r.w = v[7];
  return r;
}
template <>
struct AccOf<float, false> { using type = float; };

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// 2^x in FP64 for the pair kernels (x = -|k dq|^2 <= 0).  Reduction x = n + f
// with n = rint(x), |f| <= 1/2 (exact), then 2^f from the degree-11
// polynomial below (monomial form of the Chebyshev interpolant of 2^f on
// [-1/2, 1/2]; interpolation error < 5e-18, evaluated error < 1 ulp) and the
// scale 2^n by ldexp.  x is clamped at -1100, where 2^x underflows to 0
// anyway, so that n always fits an int.  Table generated by gen_exp2.py.
constexpr double kExp2Poly[12] = {
    1.0,
    0.6931471805599453,
    0.24022650695910158,
    0.055504108664821625,
    0.009618129107587256,
    0.001333355814640647,
    0.00015403530463724353,
    1.5252733841556773e-05,
    1.3215432535912375e-06,
    1.0178057087733941e-07,
    7.074194297288521e-09,
    4.4558179083360645e-10};

__device__ __forceinline__ double ex2(double x) {
  x = fmax(x, -1100.0);
  const double n = rint(x);
  const double f = x - n;
  double p = kExp2Poly[11];
#pragma unroll
  for (int k = 10; k >= 0; --k) p = fma(p, f, kExp2Poly[k]);
  return ldexp(p, (int)n);
}

template <typename R>
__device__ __forceinline__ Rec<R> make_rec(double x, double y, double z, double a, double b,
                                           double c) {
  Rec<R> r;
  r.x = (R)x; r.y = (R)y; r.z = (R)z; r.u = (R)0;
  r.px = (R)a; r.py = (R)b; r.pz = (R)c; r.w = (R)0;
  return r;
}

// ---------------------------------------------------------------------------
// forward pair sums over j in [j0, j1) for the lane's landmark i:
//   h[0..2] += sum_j g_ij p_j                      (Hp)
//   h[3..5] += sum_j g_ij (p_i . p_j) (kq_i - kq_j)  (Hq up to the factor -c/k)
// D = 2 is the planar specialisation: the z terms are left out (every z is 0
// there), which leaves 11 VALU + 1 exp per pair.  On planar data the two
// forms give bitwise the same sums: each z term the 3D loop adds is an exact 0.
// ---------------------------------------------------------------------------
// U: j landmarks per unrolled iteration (see kFwdUnroll).
template <typename R, int D, int U>
__device__ __forceinline__ void fwd_range(const Rec<R>* __restrict__ Xp, const Rec<R>& ri, int j0,
                                          int j1, R h[6]) {
  const GlobalPtr<Rec<R>> X = global_ptr(Xp);
  R hp0 = h[0], hp1 = h[1], hp2 = h[2], hq0 = h[3], hq1 = h[4], hq2 = h[5];
#pragma unroll U
  for (int j = j0; j < j1; ++j) {
    const Rec<R> rj = load_rec<R>(X, j);
    const R dx = ri.x - rj.x, dy = ri.y - rj.y;
    R r2 = dx * dx;
    r2 = fma(dy, dy, r2);
    R dz = (R)0;
    if constexpr (D == 3) {
      dz = ri.z - rj.z;
      r2 = fma(dz, dz, r2);
    }
    const R g = ex2(-r2);
    hp0 = fma(g, rj.px, hp0);
    hp1 = fma(g, rj.py, hp1);
    if constexpr (D == 3) hp2 = fma(g, rj.pz, hp2);
    R s = ri.px * rj.px;
    s = fma(ri.py, rj.py, s);
    if constexpr (D == 3) s = fma(ri.pz, rj.pz, s);
    const R gs = g * s;
    hq0 = fma(gs, dx, hq0);
    hq1 = fma(gs, dy, hq1);
    if constexpr (D == 3) hq2 = fma(gs, dz, hq2);
  }
  h[0] = hp0; h[1] = hp1; h[2] = hp2; h[3] = hq0; h[4] = hq1; h[5] = hq2;
}

// ---------------------------------------------------------------------------
// adjoint pair sums over j in [j0, j1).  With D = kq_i - kq_j, db = b^_i - b^_j
// (b^ = kappa k b), e = D.db, s = p_i.p_j, pi = a_i.p_j + p_i.a_j:
//   h[0..2] += sum_j g s db                (A1)
//   h[3..5] += sum_j g (pi + s e) D        (A2)
//   h[6..8] += sum_j g (a_j + e p_j)       (B)
// and A = (c/k)(A1/kappa - A2).
// ---------------------------------------------------------------------------
// U: j landmarks per unrolled iteration (see kAdjUnroll).
template <typename R, int D, int U>
__device__ __forceinline__ void adj_range(const Rec<R>* __restrict__ Xp,
                                          const Rec<R>* __restrict__ Yp, const Rec<R>& ri,
                                          const Rec<R>& yi, int j0, int j1, R h[9]) {
  const GlobalPtr<Rec<R>> X = global_ptr(Xp);
  const GlobalPtr<Rec<R>> Y = global_ptr(Yp);
  R a10 = h[0], a11 = h[1], a12 = h[2], a20 = h[3], a21 = h[4], a22 = h[5];
  R b0 = h[6], b1 = h[7], b2 = h[8];
  constexpr bool Z = D == 3;   // planar (D = 2): the z terms are all 0 and left out
#pragma unroll U
  for (int j = j0; j < j1; ++j) {
    const Rec<R> rj = load_rec<R>(X, j);
    const Rec<R> yj = load_rec<R>(Y, j);
    const R dx = ri.x - rj.x, dy = ri.y - rj.y;
    const R dz = Z ? ri.z - rj.z : (R)0;
    R r2 = dx * dx;
    r2 = fma(dy, dy, r2);
    if constexpr (Z) r2 = fma(dz, dz, r2);
    const R g = ex2(-r2);
    const R ex = yi.px - yj.px, ey = yi.py - yj.py;
    const R ez = Z ? yi.pz - yj.pz : (R)0;
    R e = dx * ex;
    e = fma(dy, ey, e);
    if constexpr (Z) e = fma(dz, ez, e);
    R s = ri.px * rj.px;
    s = fma(ri.py, rj.py, s);
    if constexpr (Z) s = fma(ri.pz, rj.pz, s);
    R pi = yi.x * rj.px;
    pi = fma(yi.y, rj.py, pi);
    if constexpr (Z) pi = fma(yi.z, rj.pz, pi);
    pi = fma(ri.px, yj.x, pi);
    pi = fma(ri.py, yj.y, pi);
    if constexpr (Z) pi = fma(ri.pz, yj.z, pi);
    const R gs = g * s;
    const R v = g * fma(s, e, pi);
    a10 = fma(gs, ex, a10);
    a11 = fma(gs, ey, a11);
    if constexpr (Z) a12 = fma(gs, ez, a12);
    a20 = fma(v, dx, a20);
    a21 = fma(v, dy, a21);
    if constexpr (Z) a22 = fma(v, dz, a22);
    const R ge = g * e;
    b0 = fma(g, yj.x, b0);
    b1 = fma(g, yj.y, b1);
    if constexpr (Z) b2 = fma(g, yj.z, b2);
    b0 = fma(ge, rj.px, b0);
    b1 = fma(ge, rj.py, b1);
    if constexpr (Z) b2 = fma(ge, rj.pz, b2);
  }
  h[0] = a10; h[1] = a11; h[2] = a12; h[3] = a20; h[4] = a21; h[5] = a22;
  h[6] = b0; h[7] = b1; h[8] = b2;
}

// One wave's share of the j range, in the precision of the mode.
template <typename R, bool COMP, int NC, typename F>
__device__ __forceinline__ void wave_sums(int j0, int j1, typename AccOf<R, COMP>::type o[NC],
                                          F&& range) {
  if constexpr (std::is_same<R, float>::value && COMP) {
    for (int c = 0; c < NC; ++c) o[c] = 0.0;
    for (int t0 = j0; t0 < j1; t0 += kTile) {
      float h[NC];
      for (int c = 0; c < NC; ++c) h[c] = 0.0f;
      range(t0, min(j1, t0 + kTile), h);
      for (int c = 0; c < NC; ++c) o[c] += (double)h[c];
    }
  } else {
    R h[NC];
    for (int c = 0; c < NC; ++c) h[c] = (R)0;
    range(j0, j1, h);
    for (int c = 0; c < NC; ++c) o[c] = h[c];
  }
}

// Depth of the unrolled j loops.  Unrolling interleaves independent pairs and
// leaves each running sum's order alone (the sums are bitwise the same at any
// depth).  FP32-compensated: 6 (forward) and 3 (adjoint), measured 2.5 % and
// 0.3-0.7 % faster per launch than 4 and 2 at N = 16384 and 65536 (8 and 1 or
// 4 no better); those depths made the FP32-naive kernels 15-19 % slower, and
// FP64 loses waves to them (adjoint 75 -> 99 VGPRs), so both keep 4 and 2.
template <typename R, bool COMP>
constexpr int kFwdUnroll = std::is_same<R, float>::value && COMP ? 6 : 4;
template <typename R, bool COMP>
constexpr int kAdjUnroll = std::is_same<R, float>::value && COMP ? 3 : 2;

// Combine the W waves' sums of a workgroup in wave order; afterwards red[c*64+l]
// holds the workgroup's sum of component c for lane l.
template <typename Acc, int NC, int W>
__device__ __forceinline__ void block_combine(Acc* red, const Acc o[NC], int w, int lane) {
  for (int c = 0; c < NC; ++c) red[(w * NC + c) * 64 + lane] = o[c];
  __syncthreads();
  for (int idx = threadIdx.x; idx < NC * 64; idx += 64 * W) {
    Acc sum = red[idx];
    for (int v = 1; v < W; ++v) sum += red[v * NC * 64 + idx];
    red[idx] = sum;
  }
  __syncthreads();
}

// The split path's version: the same sums in the same order, each stored
// straight to the workgroup's partial [S][NC][n] instead of back to LDS (one
// barrier and one LDS pass fewer).
template <typename Acc, int NC, int W>
__device__ __forceinline__ void block_combine_store(Acc* red, const Acc o[NC], int w, int lane,
                                                    Acc* P, int s, int ib, int n) {
  for (int c = 0; c < NC; ++c) red[(w * NC + c) * 64 + lane] = o[c];
  __syncthreads();
  for (int idx = threadIdx.x; idx < NC * 64; idx += 64 * W) {
    Acc sum = red[idx];
    for (int v = 1; v < W; ++v) sum += red[v * NC * 64 + idx];
    const int c = idx >> 6, i = ib * 64 + (idx & 63);
    if (i < n) P[((size_t)s * NC + c) * n + i] = sum;
  }
}

// ---------------------------------------------------------------------------
// per-landmark Euler updates (FP64), shared by the fused and the split path
// ---------------------------------------------------------------------------
// FP64 state of one landmark, loaded before the sums it is combined with so
// that its memory latency overlaps them.
struct FwdState { double q[3], p[3], acc[6]; };
struct AdjState { double a[3], b[3], hp0[3], hq0[3], lam[6]; };

// (i is clamped: lanes without a landmark load the last one's state.  No lane may ask
// for a landmark that another workgroup of the launch updates.)
template <bool RKS>
__device__ __forceinline__ FwdState load_fwd_state(const FwdArgs& A, int i) {
  FwdState v;
  const int ic = min(i, A.n - 1);
  for (int c = 0; c < 3; ++c) { v.q[c] = A.st[c * A.n + ic]; v.p[c] = A.st[(3 + c) * A.n + ic]; }
  if constexpr (RKS)
    for (int c = 0; c < 6; ++c) v.acc[c] = A.rk >= 2 ? A.rk_acc[c * A.n + ic] : 0.0;
  return v;
}

template <bool RKS>
__device__ __forceinline__ AdjState load_adj_state(const AdjArgs& A, int i) {
  AdjState v;
  const int ic = min(i, A.n - 1);
  for (int c = 0; c < 3; ++c) {
    v.a[c] = A.ad[c * A.n + ic];
    v.b[c] = A.ad[(3 + c) * A.n + ic];
    v.hp0[c] = (A.grad && A.hp0) ? A.hp0[c * A.n + ic] : 0.0;
    v.hq0[c] = (A.grad_q0 && A.hq0) ? A.hq0[c * A.n + ic] : 0.0;
  }
  if constexpr (RKS)
    for (int c = 0; c < 6; ++c) v.lam[c] = A.rk <= 3 ? A.rk_lam[c * A.n + ic] : 0.0;
  return v;
}

// Landmark i of this lane (own: it has one); part: index of the wave's H0 partial.
// The whole wave calls it.  v becomes the state after the step (or stage); returns
// the record written.
template <typename R, bool RKS>
__device__ __forceinline__ Rec<R> fwd_finish(const FwdArgs& A, int i, bool own, int part, int lane,
                                             FwdState& v, const double hp[3],
                                             const double hqs[3]) {
  const int n = A.n;
  double h0 = 0.0;
  Rec<R> out{};
  if (own) {
    if (A.hp0) {
      for (int c = 0; c < 3; ++c) A.hp0[c * n + i] = hp[c];
      h0 = v.p[0] * hp[0] + v.p[1] * hp[1] + v.p[2] * hp[2];
    }
    bool stage_out = false;   // a Runge-Kutta stage 1-3 writes a stage record, not a state
    if constexpr (!RKS) {
      for (int c = 0; c < 3; ++c) {
        const double hq = A.sc.hq * hqs[c];
        if (A.hq0) A.hq0[c * n + i] = hq;
        v.q[c] = v.q[c] + A.sc.dt * hp[c];
        v.p[c] = v.p[c] - A.sc.dt * hq;
      }
    } else {
      // Runge-Kutta stage rk: k = (Hp, -Hq) at the stage state.  Stages 1-3
      // accumulate k1 + 2 k2 + 2 k3 and write the next stage state y + c k
      // (c = dt/2, dt/2, dt) as the record the next stage's pair sums read;
      // stage 4 takes y' = y + dt/6 (k1 + 2 k2 + 2 k3 + k4).
      double hq[3];
      for (int c = 0; c < 3; ++c) {
        hq[c] = A.sc.hq * hqs[c];
        if (A.hq0) A.hq0[c * n + i] = hq[c];
      }
      if (A.rk <= 3) {
        stage_out = true;
        const double w = A.rk == 1 ? 1.0 : 2.0, cs = A.rk == 3 ? A.sc.dt : 0.5 * A.sc.dt;
        double y[6];
        for (int c = 0; c < 3; ++c) {
          v.acc[c] = A.rk == 1 ? hp[c] : v.acc[c] + w * hp[c];
          v.acc[3 + c] = A.rk == 1 ? -hq[c] : v.acc[3 + c] + w * -hq[c];
          A.rk_acc[c * n + i] = v.acc[c];
          A.rk_acc[(3 + c) * n + i] = v.acc[3 + c];
          y[c] = v.q[c] + cs * hp[c];
          y[3 + c] = v.p[c] - cs * hq[c];
        }
        const double k = A.sc.k;
        out = make_rec<R>(k * y[0], k * y[1], k * y[2], y[3], y[4], y[5]);
      } else {
        for (int c = 0; c < 3; ++c) {
          v.q[c] = v.q[c] + A.sc.dt / 6.0 * (v.acc[c] + hp[c]);
          v.p[c] = v.p[c] + A.sc.dt / 6.0 * (v.acc[3 + c] + -hq[c]);
        }
      }
    }
    if (!stage_out) {
      for (int c = 0; c < 3; ++c) { A.st[c * n + i] = v.q[c]; A.st[(3 + c) * n + i] = v.p[c]; }
      if (A.ckpt)
        for (int c = 0; c < 3; ++c) { A.ckpt[c * n + i] = v.q[c]; A.ckpt[(3 + c) * n + i] = v.p[c]; }
      const double k = A.sc.k;
      out = make_rec<R>(k * v.q[0], k * v.q[1], k * v.q[2], v.p[0], v.p[1], v.p[2]);
    }
    static_cast<Rec<R>*>(A.rec_t1)[i] = out;
  }
  if (A.h0_part) {          // whole wave takes part: fixed butterfly order
    for (int off = 32; off > 0; off >>= 1) h0 += __shfl_xor(h0, off, 64);
    if (lane == 0) A.h0_part[part] = h0;
  }
  return out;
}

// sa = A1 / kappa - A2 and sb = B of landmark i.  v becomes the adjoint after the
// step (or stage); returns the record written.
template <typename R, bool RKS>
__device__ __forceinline__ Rec<R> adj_finish(const AdjArgs& A, int i, AdjState& v,
                                             const double sa[3], const double sb[3]) {
  const int n = A.n;
  Rec<R> out;
  if constexpr (!RKS) {
    for (int c = 0; c < 3; ++c) {
      const double Ac = A.sc.adj_a * sa[c];
      v.a[c] = v.a[c] + A.sc.dt * Ac;
      v.b[c] = v.b[c] + A.sc.dt * sb[c];
    }
    for (int c = 0; c < 3; ++c) { A.ad[c * n + i] = v.a[c]; A.ad[(3 + c) * n + i] = v.b[c]; }
    const double bs = A.sc.bscale;
    out = make_rec<R>(v.a[0], v.a[1], v.a[2], bs * v.b[0], bs * v.b[1], bs * v.b[2]);
  } else {
    // Runge-Kutta stage rk (4 down to 1): w = J(Y_rk)^T u from the pair sums;
    // lambda' + the w so far accumulates in rk_lam, and the next stage's
    // adjoint u = cl lambda' + cw w goes out as its record.  Stage 1 ends the
    // step: the accumulated lambda is the adjoint at step t, and the record
    // is dt/6 lambda for stage 4 of step t - 1.
    const double bs = A.sc.bscale;
    const double dt = A.sc.dt;
    const double cl = A.rk == 4 ? dt / 3.0 : A.rk == 3 ? dt / 3.0 : dt / 6.0;
    const double cw = A.rk == 4 ? dt : 0.5 * dt;
    double lam[6], u[6];
    for (int c = 0; c < 3; ++c) {
      const double wa = A.sc.adj_a * sa[c], wb = sb[c];
      const double la = A.rk == 4 ? v.a[c] : v.lam[c], lb = A.rk == 4 ? v.b[c] : v.lam[3 + c];
      lam[c] = la + wa;
      lam[3 + c] = lb + wb;
      u[c] = cl * v.a[c] + cw * wa;
      u[3 + c] = cl * v.b[c] + cw * wb;
    }
    if (A.rk > 1) {
      for (int c = 0; c < 6; ++c) A.rk_lam[c * n + i] = v.lam[c] = lam[c];
    } else {
      for (int c = 0; c < 3; ++c) {
        v.a[c] = lam[c];
        v.b[c] = lam[3 + c];
        A.ad[c * n + i] = v.a[c];
        A.ad[(3 + c) * n + i] = v.b[c];
        u[c] = dt / 6.0 * v.a[c];
        u[3 + c] = dt / 6.0 * v.b[c];
      }
    }
    out = make_rec<R>(u[0], u[1], u[2], bs * u[3], bs * u[4], bs * u[5]);
  }
  static_cast<Rec<R>*>(A.arec_next)[i] = out;
  if (A.grad)
    for (int c = 0; c < 3; ++c) A.grad[3 * i + c] = v.b[c] + v.hp0[c];
  if (A.grad_q0)
    for (int c = 0; c < 3; ++c) A.grad_q0[3 * i + c] = v.a[c] + v.hq0[c];
  return out;
}

// The same for the lane's landmark of i-block ib from the nine sums A1, A2, B.
template <typename R, bool RKS>
__device__ __forceinline__ void adj_finish9(const AdjArgs& A, int ib, int lane, AdjState& v,
                                            const double s[9]) {
  const int i = ib * 64 + lane;
  if (i >= A.n) return;
  const double inv_kappa = 1.0 / A.sc.kappa;
  double sa[3];
  for (int c = 0; c < 3; ++c) sa[c] = s[c] * inv_kappa - s[3 + c];
  adj_finish<R, RKS>(A, i, v, sa, s + 6);
}

// ---------------------------------------------------------------------------
// pair kernels
// ---------------------------------------------------------------------------
// One workgroup's share of a pair-sum step: i-block ib (64 landmarks, one
// per lane) against j-chunk s, split over the W waves.  With S == 1 the sums
// are final and wave 0 applies the Euler update; otherwise the workgroup
// writes its partial for the combine kernel.  red: W*C*64 accumulators of LDS.
template <typename R, bool COMP, bool RKS, int W, int D>
__device__ __forceinline__ void fwd_block(const FwdArgs& A, int ib, int s,
                                          typename AccOf<R, COMP>::type* red) {
  using Acc = typename AccOf<R, COMP>::type;
  constexpr int NC = 6;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const Rec<R>* __restrict__ X = static_cast<const Rec<R>*>(A.rec_t);
  const Rec<R> ri = X[min(ib * 64 + lane, A.n - 1)];
  const int jb = s * A.chunk;
  const int je = min(A.n, jb + A.chunk);
  const int j0 = min(je, jb + w * A.wchunk);
  const int j1 = min(je, j0 + A.wchunk);
  // With FP32 sums the fused path's state is loaded after the j loop, so that
  // its registers are not held through it (the split path, which never loads
  // it, would pay them too) and the LDS combine covers the load's latency.
  // The FP64 forward keeps the early load: loaded late, its Euler update
  // spills to scratch.
  constexpr bool late = std::is_same<R, float>::value;
  FwdState v{};
  if (!late && A.S == 1 && w == 0) v = load_fwd_state<RKS>(A, ib * 64 + lane);
  Acc o[NC];
  wave_sums<R, COMP, NC>(j0, j1, o,
                         [&](int a, int b, auto* h) {
                           fwd_range<R, D, kFwdUnroll<R, COMP>>(X, ri, a, b, h);
                         });
  if (A.S == 1) {
    if (late && w == 0) v = load_fwd_state<RKS>(A, ib * 64 + lane);
    block_combine<Acc, NC, W>(red, o, w, lane);
    if (w == 0) {
      double h[NC];
      for (int c = 0; c < NC; ++c) h[c] = red[c * 64 + lane];
      fwd_finish<R, RKS>(A, ib * 64 + lane, ib * 64 + lane < A.n, ib, lane, v, h, h + 3);
    }
  } else {
    block_combine_store<Acc, NC, W>(red, o, w, lane, static_cast<Acc*>(A.partial), s, ib, A.n);
  }
}

template <typename R, bool COMP, bool RKS, int W, int D>
__device__ __forceinline__ void adj_block(const AdjArgs& A, int ib, int s,
                                          typename AccOf<R, COMP>::type* red) {
  using Acc = typename AccOf<R, COMP>::type;
  constexpr int NC = 9;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const Rec<R>* __restrict__ X = static_cast<const Rec<R>*>(A.rec_t);
  const Rec<R>* __restrict__ Y = static_cast<const Rec<R>*>(A.arec);
  const int ic = min(ib * 64 + lane, A.n - 1);
  const Rec<R> ri = X[ic];
  const Rec<R> yi = Y[ic];
  const int jb = s * A.chunk;
  const int je = min(A.n, jb + A.chunk);
  const int j0 = min(je, jb + w * A.wchunk);
  const int j1 = min(je, j0 + A.wchunk);
  Acc o[NC];
  wave_sums<R, COMP, NC>(j0, j1, o,
                         [&](int a, int b, auto* h) {
                           adj_range<R, D, kAdjUnroll<R, COMP>>(X, Y, ri, yi, a, b, h);
                         });
  if (A.S == 1) {
    // the state is loaded after the j loop, so that its registers are not
    // held through it (the split path, which never loads it, would pay them
    // too: with 2-deep loops 77 instead of 64 VGPRs in the FP32-compensated
    // kernel, 94 instead of 75 in FP64); the LDS combine covers the load's
    // latency
    AdjState v{};
    if (w == 0) v = load_adj_state<RKS>(A, ib * 64 + lane);
    block_combine<Acc, NC, W>(red, o, w, lane);
    if (w == 0) {
      double h[NC];
      for (int c = 0; c < NC; ++c) h[c] = red[c * 64 + lane];
      adj_finish9<R, RKS>(A, ib, lane, v, h);
    }
  } else {
    block_combine_store<Acc, NC, W>(red, o, w, lane, static_cast<Acc*>(A.partial), s, ib, A.n);
  }
}

// RKS: the launch is a Runge-Kutta stage (its own instances, so that the
// Euler kernels carry none of the stage bookkeeping).
template <typename R, bool COMP, bool RKS, int W, int D>
__global__ __launch_bounds__(64 * W) void k_fwd(FwdArgs A) {
  __shared__ typename AccOf<R, COMP>::type red[W * 6 * 64];
  fwd_block<R, COMP, RKS, W, D>(A, blockIdx.x / A.S, blockIdx.x % A.S, red);
}

template <typename R, bool COMP, bool RKS, int W, int D>
__global__ __launch_bounds__(64 * W) void k_adj(AdjArgs A) {
  __shared__ typename AccOf<R, COMP>::type red[W * 9 * 64];
  adj_block<R, COMP, RKS, W, D>(A, blockIdx.x / A.S, blockIdx.x % A.S, red);
}

// ---------------------------------------------------------------------------
// row kernels: one launch per step
// ---------------------------------------------------------------------------
// Below a few thousand landmarks a step of the split kernels is two dependent
// launches of 3 to 4 us whose pair sums take 1 to 3 us.  Here a workgroup holds
// every j of its rows and ends the step itself.  The roles of the split
// kernels' operands are swapped: lane l of a wave owns landmark j = 64 t + l of
// tile t (loaded once per tile, coalesced, no LDS staging) and M landmarks i are
// wave-uniform, so a workgroup can be as small as M rows and the chip fills from
// n = 256 M on.  Each lane's M x 2D sums are added across the wave at the end:
// two half-exchanges leave a quarter of the values per lane, the rest of the
// sum (16 lanes x waves) is FP64 in every mode.  A lane adds n / (64 jg) <= 18 pairs
// (row_plan), so an FP32 sum covers kTile at most and needs no tiles; both FP32
// modes run the same code.
// The adjoint is written on w = a_j + e p_j: pi + s e = a_i.p_j + p_i.w and B's
// term is g w, and A1 / kappa and -A2 share one accumulator (p_j / kappa is formed
// once per tile): 35 VALU + 1 exp per pair and 6 sums per row instead of 37 + 1
// and 9.  The rounding of p_j / kappa costs less than the shorter sums gain: rms error
// of dL/dq0 0.78 of the split kernels', of dL/dp0 0.72 (means over n = 4 to 5120, both
// FP32 modes, planar and 3D, Euler and Runge-Kutta; no case above 1.1).
// What bounds them: at n = 1000 a step takes 4.7 us, of which 3.6 are a
// dependent launch that loads, combines and stores (n = 64 takes as long); at n =
// 4096 the loops (10.7 and 18.3 us per step, 6.0 and 12.0 at the rate of the
// 65536-landmark kernels: a tile's addresses and masks, four waves per SIMD).
template <typename R>
using Vec3 = R __attribute__((ext_vector_type(3)));

// 2^(-x) with an s_nop behind the transcendental.  FP32 instructions of two waves
// issue together on a SIMD, but after a v_exp_f32 with only vector
// instructions around it they stop doing so for some 20 cycles (issue probe, one
// v_exp_f32 per 15 v_fmac_f32: 4.1 cycles per instruction, 2.8 with the s_nop);
// it took 8 to 15 % off these loops.  The s_nop also covers the wait state
// between a transcendental and its use.
__device__ __forceinline__ float ex2n(float x) {
  float g;
  asm("v_exp_f32 %0, -%1\n\ts_nop 0" : "=v"(g) : "v"(x));
  return g;
}
__device__ __forceinline__ double ex2n(double x) { return ex2(-x); }

// Half-wave exchanges: a + b of the two halves, the low half of the result
// holding a's sums and the high half b's (rows of 16 likewise in swap16_add).
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double swap32_add(double a, double b) {
  const unsigned al = __double2loint(a), ah = __double2hiint(a);
  const unsigned bl = __double2loint(b), bh = __double2hiint(b);
  const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ __forceinline__ double swap16_add(double a, double b) {
  const unsigned al = __double2loint(a), ah = __double2hiint(a);
  const unsigned bl = __double2loint(b), bh = __double2hiint(b);
  const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}

// v plus v of the lane CTRL (a row_ror) away within its row of 16.
template <int CTRL>
__device__ __forceinline__ double row_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}

template <typename R>
constexpr int kRowWaves = std::is_same<R, double>::value ? 8 : 16;   // waves of a row workgroup at most

// A wave-uniform value held in a vector register: the FP64 adjoint's rows do not
// fit the scalar registers beside the exponential's constants (spilled, its
// loops took 20 % longer).
__device__ __forceinline__ double in_vgpr(double s) {
  int lo, hi;
  asm("v_mov_b32 %0, %1" : "=v"(lo) : "s"(__double2loint(s)));
  asm("v_mov_b32 %0, %1" : "=v"(hi) : "s"(__double2hiint(s)));
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float in_vgpr(float s) { return s; }

// Sums of M rows, padded to a multiple of four (the combine halves them twice),
// and where row k of a workgroup starts in its combined sums.
template <int D, int M>
constexpr int row_pad = (M * 2 * D + 3) / 4 * 4;
template <int D, int M>
__device__ __forceinline__ int row_at(int k) {
  return (k / M) * row_pad<D, M> + (k % M) * 2 * D;
}

template <typename R, bool CONST>
__device__ __forceinline__ Rec<R> load_row(GlobalPtr<Rec<R>> p, int i) {
  if constexpr (!CONST) return load_rec<R>(p, i);
  using ConstVec = const __attribute__((address_space(4))) Vec8<R>*;
  const Vec8<R> v = ((ConstVec)(unsigned long long)p)[i];
  return {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
}

// One pair's terms of landmark i's sums, added to h; x: q_i, p_i; y: a_i, b^_i.
// Forward: h = {Hp, Hq's sums} (D components each).
template <typename R, int D>
__device__ __forceinline__ void fwd_term(const R* x, Vec3<R> q, Vec3<R> p, R* h) {
  R d[3];
  R r2 = (R)0, s = (R)0;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    d[c] = x[c] - q[c];
    r2 = c == 0 ? d[c] * d[c] : fma(d[c], d[c], r2);
  }
  const R g = ex2n(r2);
#pragma unroll
  for (int c = 0; c < D; ++c) s = c == 0 ? x[3 + c] * p[c] : fma(x[3 + c], p[c], s);
  const R gs = g * s;
#pragma unroll
  for (int c = 0; c < D; ++c) h[c] = fma(g, p[c], h[c]);
#pragma unroll
  for (int c = 0; c < D; ++c) h[D + c] = fma(gs, d[c], h[D + c]);
}

// Adjoint: h = {A1 / kappa - A2, B}; pi . pj = p_i . p_j / kappa (either side scaled).
template <typename R, int D>
__device__ __forceinline__ void adj_term(const R* x, const R* y, const R* pi, Vec3<R> q, Vec3<R> p,
                                         Vec3<R> pj, Vec3<R> a, Vec3<R> b, R* h) {
  R d[3], ex[3], w[3];
  R r2 = (R)0, s = (R)0, e = (R)0, v = (R)0;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    d[c] = x[c] - q[c];
    r2 = c == 0 ? d[c] * d[c] : fma(d[c], d[c], r2);
  }
  const R g = ex2n(r2);
#pragma unroll
  for (int c = 0; c < D; ++c) s = c == 0 ? pi[c] * pj[c] : fma(pi[c], pj[c], s);
  const R gs = g * s;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    ex[c] = y[3 + c] - b[c];
    e = c == 0 ? d[c] * ex[c] : fma(d[c], ex[c], e);
  }
#pragma unroll
  for (int c = 0; c < D; ++c) w[c] = fma(e, p[c], a[c]);
#pragma unroll
  for (int c = 0; c < D; ++c) v = c == 0 ? y[c] * p[c] : fma(y[c], p[c], v);
#pragma unroll
  for (int c = 0; c < D; ++c) v = fma(x[3 + c], w[c], v);
  const R gv = g * v;
#pragma unroll
  for (int c = 0; c < D; ++c) h[c] = fma(gs, ex[c], h[c]);
#pragma unroll
  for (int c = 0; c < D; ++c) h[c] = fma(-gv, d[c], h[c]);
#pragma unroll
  for (int c = 0; c < D; ++c) h[D + c] = fma(g, w[c], h[D + c]);
}

// Adds the four quarters of a wave: lanes 16 g .. 16 g + 15 of h[k] then hold value
// k + Q g (Q = row_pad / 4).  In FP32 an entry is the sum of four lanes' terms.
template <typename R, int D, int M>
__device__ __forceinline__ void row_exchange(R h[row_pad<D, M>]) {
  constexpr int NV = row_pad<D, M>, Q = NV / 4;
#pragma unroll
  for (int k = 0; k < NV / 2; ++k) h[k] = swap32_add(h[k], h[k + NV / 2]);
#pragma unroll
  for (int k = 0; k < Q; ++k) h[k] = swap16_add(h[k], h[k + Q]);
}

// What a row workgroup keeps of its waves' sums: the values themselves, or, in the
// batched kernels, their FP64 sums over the rounds.
template <typename R, bool BATCH>
using RowRed = typename std::conditional<BATCH, double, R>::type;

// Sums of one wave: rows i0 .. i0 + M - 1 over the tiles t = t0, t0 + JG, ... < t1,
// exchanged and stored to the lane's slots own[64 k].
// ADJ: h[m] = {A1 / kappa - A2 (D components), B (D)}, else {Hp (D), Hq's sums (D)}.
// BATCH: n may be large, so the tiles are taken batch_round at a time and each round's
// sums are added to the slots in FP64 (no barrier: a lane reads back what it wrote),
// which keeps an FP32 sum to kTile pairs.  The row plans end before that, and with
// the loop around them their adjoint took 10 % longer (n = 1847).
// The batched pointers come from a descriptor in memory, and the compiler would hold
// the rows in vector registers for fear of the stores; through the constant address
// space (records of the step are not written by its launch) they become scalar
// loads (eight jobs of 500 to 8000: 38.9 -> 37.1 ms, FP64 24.2 -> 22.2).
template <typename R, bool ADJ, int D, int M, bool BATCH>
__device__ __forceinline__ void row_sums(const void* Xv, const void* Yv, int n, int i0, int t0,
                                         int t1, int JG, int lane, R inv_kappa,
                                         RowRed<R, BATCH>* own) {
  const GlobalPtr<Rec<R>> X = global_ptr(static_cast<const Rec<R>*>(Xv));
  const GlobalPtr<Rec<R>> Y = global_ptr(static_cast<const Rec<R>*>(Yv));
  R xi[M][6], yi[M][6];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int i = min(i0 + m, n - 1);
    const Rec<R> a = load_row<R, BATCH>(X, i);
    xi[m][0] = a.x; xi[m][1] = a.y; xi[m][2] = a.z;
    xi[m][3] = a.px; xi[m][4] = a.py; xi[m][5] = a.pz;
    if constexpr (ADJ) {
      const Rec<R> b = load_row<R, BATCH>(Y, i);
      yi[m][0] = in_vgpr(b.x); yi[m][1] = in_vgpr(b.y); yi[m][2] = in_vgpr(b.z);
      yi[m][3] = in_vgpr(b.px); yi[m][4] = in_vgpr(b.py); yi[m][5] = in_vgpr(b.pz);
    }
  }
  struct Tile { Vec3<R> q, p, a, b; };
  // 32-bit byte offsets from a scalar base: an address is one instruction (with the
  // narrower mask below 2-4 % of a step, FP64 n = 2500 forward 14.1 -> 12.8 us)
  const auto load = [&](unsigned o) {
    Tile r;
    const GlobalPtr<Rec<R>> x = (GlobalPtr<Rec<R>>)((GlobalPtr<char>)X + o);
    r.q = *reinterpret_cast<GlobalPtr<Vec3<R>>>(&x->x);
    r.p = *reinterpret_cast<GlobalPtr<Vec3<R>>>(&x->px);
    if constexpr (ADJ) {
      const GlobalPtr<Rec<R>> y = (GlobalPtr<Rec<R>>)((GlobalPtr<char>)Y + o);
      r.a = *reinterpret_cast<GlobalPtr<Vec3<R>>>(&y->x);
      r.b = *reinterpret_cast<GlobalPtr<Vec3<R>>>(&y->px);
    }
    return r;
  };
  // one tile ahead (the last one twice): with few waves per SIMD the loads'
  // latency shows (FP64, n = 2500: adjoint 21.6 us per step without, 19.9 with)
  constexpr unsigned kRec = sizeof(Rec<R>);
  const unsigned end = (unsigned)(n - 1) * kRec;
  unsigned o = (unsigned)(t0 * 64 + lane) * kRec;
  Tile next = load(min(o, end));
  int t = t0;
  bool first = true;
  do {
    const int te = BATCH ? min(t1, t + batch_round(std::is_same<R, double>::value) * JG) : t1;
    R h[row_pad<D, M>];
#pragma unroll
    for (int k = 0; k < row_pad<D, M>; ++k) h[k] = (R)0;
    for (; t < te; t += JG) {
      const bool in = o <= end;
      const Tile cur = next;
      o += 64 * kRec * (unsigned)JG;
      next = load(min(o, end));
      Vec3<R> q = cur.q, p = cur.p, a = (R)0, b = (R)0;
      if constexpr (ADJ) { a = cur.a; b = cur.b; }
      // Lanes beyond n add an exact 0 to every sum with p_j = a_j = 0.  In the batched
      // kernels a branch keeps that to the ragged tile (eight jobs of 500 to 8000: 36.0
      // -> 34.4 ms); in the others the adjoint's loop comes out slower then (n = 2500
      // 9.7 -> 11.7 us per step), and slower too when it does not zero q and b (2D n = 3000
      // 9.8 -> 10.8).
      if constexpr (BATCH) {
        if (t * 64 + 64 > n && !in) { p = (R)0; a = (R)0; }
      } else {
        if (!in) p = (R)0;
        if (ADJ && !in) { q = (R)0; a = (R)0; b = (R)0; }
      }
      Vec3<R> ps = p;
      if constexpr (ADJ) ps = p * inv_kappa;
#pragma unroll
      for (int m = 0; m < M; ++m) {
        if constexpr (ADJ) adj_term<R, D>(xi[m], yi[m], &xi[m][3], q, p, ps, a, b, h + 2 * D * m);
        else fwd_term<R, D>(xi[m], q, p, h + 2 * D * m);
      }
    }
    row_exchange<R, D, M>(h);
#pragma unroll
    for (int k = 0; k < row_pad<D, M> / 4; ++k) {
      if (BATCH && !first) own[k * 64] += (RowRed<R, BATCH>)h[k];
      else own[k * 64] = (RowRed<R, BATCH>)h[k];
    }
    first = false;
  } while (BATCH && t < t1);
}

// The workgroup's sums of rows [0, M ig) in fin (row_at), from every wave's
// exchanged values in red.
template <typename T, int D, int M>
__device__ __forceinline__ void row_combine(const T* red, double* fin, int ig, int jg, int w,
                                            int lane) {
  constexpr int NV = row_pad<D, M>, Q = NV / 4;
  __syncthreads();
  for (int kk = w; kk < Q * ig; kk += ig * jg) {
    const int k = kk % Q, g = kk / Q;
    double s = (double)red[(g * Q + k) * 64 + lane];
    for (int v = 1; v < jg; ++v) s += (double)red[((v * ig + g) * Q + k) * 64 + lane];
    s = row_add<0x121>(s);
    s = row_add<0x122>(s);
    s = row_add<0x124>(s);
    s = row_add<0x128>(s);
    if ((lane & 15) == 0) fin[g * NV + k + Q * (lane >> 4)] = s;
  }
  __syncthreads();
}

// Combined sums (fin) of the rows of a workgroup item, in ig x jg waves.
template <typename R, bool ADJ, int D, int M, bool BATCH>
__device__ __forceinline__ void row_step(const void* X, const void* Y, int n, int ig, int jg,
                                         int row0, R inv_kappa, RowRed<R, BATCH>* red, double* fin,
                                         int w, int lane) {
  row_sums<R, ADJ, D, M, BATCH>(X, Y, n, row0 + (w % ig) * M, w / ig, (n + 63) >> 6, jg, lane,
                                inv_kappa, red + w * (row_pad<D, M> / 4) * 64 + lane);
  row_combine<RowRed<R, BATCH>, D, M>(red, fin, ig, jg, w, lane);
}

template <typename R, bool RKS, int D, int M, bool BATCH = false>
__device__ __forceinline__ void fwd_rows(const FwdArgs& A, int g, RowRed<R, BATCH>* red,
                                         double* fin) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row0 = g * A.ig * M;
  FwdState v{};
  if (!BATCH && w == 0)   // its latency under the sums
    v = load_fwd_state<RKS>(A, row_state(row0, A.ig * M, lane));
  row_step<R, false, D, M, BATCH>(A.rec_t, nullptr, A.n, A.ig, A.jg, row0, (R)0, red, fin, w, lane);
  if (w == 0) {
    if (BATCH) v = load_fwd_state<RKS>(A, row_state(row0, A.ig * M, lane));
    const bool own = lane < A.ig * M && row0 + lane < A.n;
    double hp[3] = {0.0, 0.0, 0.0}, hq[3] = {0.0, 0.0, 0.0};
    if (own)
      for (int c = 0; c < D; ++c) {
        hp[c] = fin[row_at<D, M>(lane) + c];
        hq[c] = fin[row_at<D, M>(lane) + D + c];
      }
    fwd_finish<R, RKS>(A, row0 + lane, own, g, lane, v, hp, hq);
  }
}

template <typename R, bool RKS, int D, int M, bool BATCH = false>
__device__ __forceinline__ void adj_rows(const AdjArgs& A, int g, RowRed<R, BATCH>* red,
                                         double* fin) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row0 = g * A.ig * M;
  AdjState v{};
  if (!BATCH && w == 0)   // its latency under the sums
    v = load_adj_state<RKS>(A, row_state(row0, A.ig * M, lane));
  row_step<R, true, D, M, BATCH>(A.rec_t, A.arec, A.n, A.ig, A.jg, row0, (R)(1.0 / A.sc.kappa), red,
                                 fin, w, lane);
  if (w == 0 && lane < A.ig * M && row0 + lane < A.n) {
    if (BATCH) v = load_adj_state<RKS>(A, row_state(row0, A.ig * M, lane));
    double sa[3] = {0.0, 0.0, 0.0}, sb[3] = {0.0, 0.0, 0.0};
    for (int c = 0; c < D; ++c) {
      sa[c] = fin[row_at<D, M>(lane) + c];
      sb[c] = fin[row_at<D, M>(lane) + D + c];
    }
    adj_finish<R, RKS>(A, row0 + lane, v, sa, sb);
  }
}

template <typename R, bool RKS, int D, int M>
__global__ __launch_bounds__(64 * kRowWaves<R>) void k_fwd_rows(FwdArgs A) {
  __shared__ R red[kRowWaves<R> * (row_pad<D, M> / 4) * 64];
  __shared__ double fin[kRowGroups * row_pad<D, M>];
  fwd_rows<R, RKS, D, M>(A, blockIdx.x, red, fin);
}

template <typename R, bool RKS, int D, int M>
__global__ __launch_bounds__(64 * kRowWaves<R>) void k_adj_rows(AdjArgs A) {
  __shared__ R red[kRowWaves<R> * (row_pad<D, M> / 4) * 64];
  __shared__ double fin[kRowGroups * row_pad<D, M>];
  adj_rows<R, RKS, D, M>(A, blockIdx.x, red, fin);
}

// ---------------------------------------------------------------------------
// chain kernels: all steps of a few landmarks in one launch
// ---------------------------------------------------------------------------
// Up to 64 landmarks a step's pair sums take a microsecond on one CU, less than the
// launch that a step of the row kernels is.  One workgroup takes all steps:
// records and sums stay in LDS, the FP64 state in the registers of the wave whose
// lanes own the landmarks, and a step is three barriers.  Every wave holds all
// landmarks i, one per lane, and takes every eighth j, whose record is an LDS
// broadcast.  Records, state and checkpoints are stored to memory for the adjoint
// and later launches, but no store is read back: the barriers wait for the LDS
// alone.
// What bounds them: barriers and LDS latency (1.2 us per step at n = 16), then the
// pairs of one CU.  A loss+gradient evaluation of 20 Euler steps took (us, row
// kernels -> chain): FP64 n = 16 157 -> 69, 64 160 -> 121; FP32 143 -> 56, 146 ->
// 81; beyond 64, two landmarks per lane of the wave: FP64 n = 80 162 -> 231, FP32 96
// 144 -> 130, 128 144 -> 157.  With 4 waves FP32 n = 64 takes 109, with 16 the same
// 84 (FP64 spills).
// Barrier for data in LDS (__syncthreads would wait for the stores to memory).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr int kChainWaves = 8;

template <typename R>
struct alignas(16) LdsRec { R v[sizeof(R) == 8 ? 6 : 8]; };   // q (p), p; or a, b^

template <typename R>
__device__ __forceinline__ void lds_put(LdsRec<R>* r, const Rec<R>& x) {
  r->v[0] = x.x; r->v[1] = x.y; r->v[2] = x.z;
  r->v[3] = x.px; r->v[4] = x.py; r->v[5] = x.pz;
}

// Sums over the waves, in their order: red[w][c][64] -> fin[c][64].
template <typename R, int D>
__device__ __forceinline__ void chain_combine(const R h[2 * D], R* red, double* fin, int w,
                                              int lane) {
#pragma unroll
  for (int c = 0; c < 2 * D; ++c) red[(w * 2 * D + c) * 64 + lane] = h[c];
  lds_barrier();
  if (w < 2 * D) {
    double s = (double)red[w * 64 + lane];
    for (int v = 1; v < kChainWaves; ++v) s += (double)red[(v * 2 * D + w) * 64 + lane];
    fin[w * 64 + lane] = s;
  }
  lds_barrier();
}
static_assert(kChainWaves >= 6, "a wave per sum");

template <typename R, bool RKS, int D>
__global__ __launch_bounds__(64 * kChainWaves) void k_fwd_chain(ChainArgs C, FwdArgs A) {
  __shared__ LdsRec<R> X[64];
  __shared__ R red[2 * D * 64 * kChainWaves];
  __shared__ double fin[2 * D * 64];
  const int i = threadIdx.x & 63, n = A.n, ic = min(i, n - 1);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  double* const hp0 = A.hp0;
  double* const hq0 = A.hq0;
  FwdState v{};
  if (w == 0) {
    A.rk = RKS ? 1 : 0;   // (no sums to load yet)
    v = load_fwd_state<RKS>(A, i);
    lds_put<R>(&X[i], static_cast<const Rec<R>*>(C.rec(C.t0, 0, n, sizeof(Rec<R>)))[ic]);
  }
  lds_barrier();
  for (int t = C.t0; t < C.t1; ++t)
    for (int st = 0; st < (RKS ? 4 : 1); ++st) {
      const bool last = st == (RKS ? 3 : 0);
      R h[2 * D], x[6];
#pragma unroll
      for (int c = 0; c < 2 * D; ++c) h[c] = (R)0;
#pragma unroll
      for (int c = 0; c < 6; ++c) x[c] = X[ic].v[c];
      for (int j = w; j < n; j += kChainWaves) {
        const LdsRec<R> r = X[j];
        fwd_term<R, D>(x, Vec3<R>{r.v[0], r.v[1], r.v[2]}, Vec3<R>{r.v[3], r.v[4], r.v[5]}, h);
      }
      chain_combine<R, D>(h, red, fin, w, i);
      if (w == 0) {
        double hp[3] = {0.0, 0.0, 0.0}, hq[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < D; ++c) {
          hp[c] = fin[c * 64 + i];
          hq[c] = fin[(D + c) * 64 + i];
        }
        const bool field = C.first && t == 0 && st == 0;   // the field at (q0, p0)
        A.rk = RKS ? st + 1 : 0;
        A.rec_t1 = last ? C.rec(t + 1, 0, n, sizeof(Rec<R>)) : C.rec(t, st + 1, n, sizeof(Rec<R>));
        A.hp0 = field ? hp0 : nullptr;
        A.hq0 = field ? hq0 : nullptr;
        A.h0_part = field ? C.h0_part : nullptr;
        A.ckpt = last ? C.ckpt_of(t + 1, n) : nullptr;
        const Rec<R> r = fwd_finish<R, RKS>(A, i, i < n, 0, i, v, hp, hq);
        if (field && i > 0 && i < C.nh) C.h0_part[i] = 0.0;   // all of H0 is in partial 0
        lds_put<R>(&X[i], r);
      }
      lds_barrier();
    }
}

template <typename R, bool RKS, int D>
__global__ __launch_bounds__(64 * kChainWaves) void k_adj_chain(ChainArgs C, AdjArgs A) {
  __shared__ LdsRec<R> X[64], Y[64];
  __shared__ R red[2 * D * 64 * kChainWaves];
  __shared__ double fin[2 * D * 64];
  constexpr int S = RKS ? 4 : 1;
  const int i = threadIdx.x & 63, n = A.n, ic = min(i, n - 1);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  double* const grad = A.grad;
  double* const grad_q0 = A.grad_q0;
  void* const buf[2] = {A.arec_next, const_cast<void*>(A.arec)};   // written in turn
  const R inv_kappa = (R)(1.0 / A.sc.kappa);
  const auto rec = [&](int t, int st) {
    return static_cast<const Rec<R>*>(C.rec(t, st, n, sizeof(Rec<R>)))[ic];
  };
  AdjState v{};
  Rec<R> next{};   // the record of the coming stage, loaded a stage ahead
  if (w == 0) {
    if (C.t0 > 0) { A.grad = nullptr; A.grad_q0 = nullptr; }
    A.rk = RKS ? 4 : 0;   // (no sums to load yet)
    v = load_adj_state<RKS>(A, i);
    lds_put<R>(&Y[i], static_cast<const Rec<R>*>(A.arec)[ic]);
    next = rec(C.t1 - 1, S - 1);
  }
  int k = 0;
  for (int t = C.t1 - 1; t >= C.t0; --t)
    for (int st = S - 1; st >= 0; --st, ++k) {
      if (w == 0) {
        lds_put<R>(&X[i], next);
        if (st > 0) next = rec(t, st - 1);
        else if (t > C.t0) next = rec(t - 1, S - 1);
      }
      lds_barrier();
      R h[2 * D], x[6], y[6], pi[3];
#pragma unroll
      for (int c = 0; c < 2 * D; ++c) h[c] = (R)0;
#pragma unroll
      for (int c = 0; c < 6; ++c) { x[c] = X[ic].v[c]; y[c] = Y[ic].v[c]; }
#pragma unroll
      for (int c = 0; c < 3; ++c) pi[c] = x[3 + c] * inv_kappa;
      for (int j = w; j < n; j += kChainWaves) {
        const LdsRec<R> r = X[j], z = Y[j];
        const Vec3<R> p{r.v[3], r.v[4], r.v[5]};
        adj_term<R, D>(x, y, pi, Vec3<R>{r.v[0], r.v[1], r.v[2]}, p, p,
                       Vec3<R>{z.v[0], z.v[1], z.v[2]}, Vec3<R>{z.v[3], z.v[4], z.v[5]}, h);
      }
      chain_combine<R, D>(h, red, fin, w, i);
      if (w == 0 && i < n) {
        double sa[3] = {0.0, 0.0, 0.0}, sb[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < D; ++c) {
          sa[c] = fin[c * 64 + i];
          sb[c] = fin[(D + c) * 64 + i];
        }
        const bool end = t == 0 && st == 0;
        A.rk = RKS ? st + 1 : 0;
        A.arec_next = buf[k & 1];
        A.grad = end ? grad : nullptr;
        A.grad_q0 = end ? grad_q0 : nullptr;
        lds_put<R>(&Y[i], adj_finish<R, RKS>(A, i, v, sa, sb));
      }
    }
}

// ---------------------------------------------------------------------------
// flow of arbitrary points (eq. 4)
// ---------------------------------------------------------------------------
// Lane l owns RP points.  With FP32 sums a wave copies its landmarks to its own
// LDS tile, 64 at a time, and reads them back as broadcasts, so that every
// operand of a pair is a vector register: an FP32 instruction with a scalar
// operand issues beside one without, not beside another with, and with the
// landmark in scalar registers 6 of the pair's 9 have one.  9 VALU + 1 exp per
// pair; two points per lane halve the LDS reads per pair (25 cycles of a SIMD's
// share of the LDS with one, against 37 of issue).  What bounds it is issue: on
// the 64^3 grid around 4096 landmarks a step takes 240 us, 35 cycles per pair and
// wave, against 30 if every instruction found a partner and 40 (276 us) with
// scalar operands.
constexpr int kFlowTile = 64;

template <int D>
struct FlowTile;
template <>
struct alignas(16) FlowTile<3> {
  float4 a[kFlowTile];
  float2 b[kFlowTile];
  __device__ void put(int l, const Rec<float>& r) {
    a[l] = make_float4(r.x, r.y, r.z, r.px);
    b[l] = make_float2(r.py, r.pz);
  }
  __device__ void get(int j, float q[3], float p[3]) const {
    const float4 u = a[j];
    const float2 v = b[j];
    q[0] = u.x; q[1] = u.y; q[2] = u.z; p[0] = u.w; p[1] = v.x; p[2] = v.y;
  }
};
template <>
struct alignas(16) FlowTile<2> {
  float4 a[kFlowTile];
  __device__ void put(int l, const Rec<float>& r) { a[l] = make_float4(r.x, r.y, r.px, r.py); }
  __device__ void get(int j, float q[3], float p[3]) const {
    const float4 u = a[j];
    q[0] = u.x; q[1] = u.y; p[0] = u.z; p[1] = u.w;
  }
};
// A wave's LDS: its tile, and over it (between the sums) its sums for the combine.
template <int RP>
constexpr int kFlowWaveLds = RP * 3 * 64 * 8;
static_assert(sizeof(FlowTile<3>) <= kFlowWaveLds<1>, "a tile fits its wave's sums");

// v += the first cnt landmarks of the tile for the lane's pre-scaled points xs.  FULL:
// cnt is kFlowTile (a constant count takes 3 to 10 % less, n = 10007, m = 100000).
template <int D, int RP, bool FULL>
__device__ __forceinline__ void flow_tile(const FlowTile<D>& tile, const float xs[RP][3], int cnt,
                                          float v[RP][3]) {
#pragma unroll 2
  for (int j = 0; j < (FULL ? kFlowTile : cnt); ++j) {
    float q[3], p[3];
    tile.get(j, q, p);
#pragma unroll
    for (int r = 0; r < RP; ++r) {
      float r2 = 0.0f;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const float d = xs[r][c] - q[c];
        r2 = c == 0 ? d * d : fma(d, d, r2);
      }
      const float g = ex2n(r2);
#pragma unroll
      for (int c = 0; c < D; ++c) v[r][c] = fma(g, p[c], v[r][c]);
    }
  }
}

// o += sum over landmarks [c0, c1) of g(x, q_j) p_j for the lane's pre-scaled
// points xs.  FP32: tiles of 64 terms through the wave's LDS, each folded into FP64.
template <int D, int RP>
__device__ __forceinline__ void flow_chunk(const Rec<float>* __restrict__ X, void* lds,
                                           const float xs[RP][3], int c0, int c1, int lane,
                                           double o[RP][3]) {
  FlowTile<D>& tile = *static_cast<FlowTile<D>*>(lds);
  for (int s = c0; s < c1; s += kFlowTile) {
    const int cnt = min(kFlowTile, c1 - s);
    tile.put(lane, X[min(s + lane, c1 - 1)]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float v[RP][3];
#pragma unroll
    for (int r = 0; r < RP; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) v[r][c] = 0.0f;
    if (cnt == kFlowTile) flow_tile<D, RP, true>(tile, xs, cnt, v);
    else flow_tile<D, RP, false>(tile, xs, cnt, v);
#pragma unroll
    for (int r = 0; r < RP; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) o[r][c] += (double)v[r][c];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// FP64: no co-issue to gain, so the landmarks come as scalar operands.  The
// records do not change while the kernel runs, which the constant address space
// states: behind the barriers and stores of the loop over the steps the compiler
// would load them per lane otherwise (2.2 times slower).
using ConstRec = const __attribute__((address_space(4))) Vec8<double>*;

template <int D, int RP>
__device__ __forceinline__ void flow_chunk(const Rec<double>* __restrict__ Xp, void*,
                                           const double xs[RP][3], int c0, int c1, int,
                                           double o[RP][3]) {
  const ConstRec X = (ConstRec)(uintptr_t)Xp;
#pragma unroll 4
  for (int j = c0; j < c1; ++j) {
    const Vec8<double> rj = X[j];
    const double q[3] = {rj[0], rj[1], rj[2]}, p[3] = {rj[4], rj[5], rj[6]};
#pragma unroll
    for (int r = 0; r < RP; ++r) {
      double r2 = 0.0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const double d = xs[r][c] - q[c];
        r2 = c == 0 ? d * d : fma(d, d, r2);
      }
      const double g = ex2(-r2);
#pragma unroll
      for (int c = 0; c < D; ++c) o[r][c] = fma(g, p[c], o[r][c]);
    }
  }
}

// One workgroup: 64 RP points through all steps [t0, t1).  Wave w sums its chunk
// (half) or pair of chunks; the sums are combined pair by pair in order.  Row k =
// 3 r + c of the points' state (component c of point r of each lane) belongs to
// wave k mod W, which combines and advances it; the positions go to the other
// waves through LDS, so that no wave holds FP64 state through its sums.
template <typename R, bool RKS, int D, int RP>
__global__ __launch_bounds__(1024) void k_flow(FlowArgs A) {
  extern __shared__ __align__(16) unsigned char flow_lds[];
  __shared__ double xl[RP * 3][64];                   // positions
  __shared__ R yl[RP * 3][64];                        // positions of the sums, pre-scaled
  __shared__ double al[RKS ? RP * 3 : 1][64];         // k1 + 2 k2 + 2 k3
  constexpr int kWave = kFlowWaveLds<RP>;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int W = blockDim.x >> 6;
  const auto red = [&](int v) { return reinterpret_cast<double*>(flow_lds + v * kWave); };
  const auto point = [&](int k) { return (int)(blockIdx.x * RP + k / 3) * 64 + lane; };
  for (int k = w; k < RP * 3; k += W) {
    const int c = k % 3, ic = min(point(k), A.m - 1);
    const double x = A.x_in ? A.x_in[3 * (size_t)ic + c] - A.cen[c] : A.xs[(size_t)c * A.m + ic];
    xl[k][lane] = x;
    yl[k][lane] = (R)(A.k * x);
  }
  const bool split = gridDim.y > 1;   // the pairs are spread over workgroups
  const int ch0 = A.half ? (int)blockIdx.y * W + w : 2 * w;
  const int stages = RKS ? 4 : 1;
  for (int t = stages * A.t0; t < stages * A.t1; ++t) {   // records: steps or their stages
    __syncthreads();   // yl is written; the sums of the last record are read
    const Rec<R>* X = static_cast<const Rec<R>*>(A.traj) + (size_t)(t % A.slots) * A.n;
    R ys[RP][3];
    double o[RP][3], o2[RP][3];
#pragma unroll
    for (int r = 0; r < RP; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ys[r][c] = yl[3 * r + c][lane];
        o[r][c] = o2[r][c] = 0.0;
      }
    const auto chunk = [&](int ch, double s[RP][3]) {
      flow_chunk<D, RP>(X, red(w), ys, min(A.n, ch * A.clen), min(A.n, (ch + 1) * A.clen), lane, s);
    };
    chunk(ch0, o);
    if (!A.half) chunk(ch0 + 1, o2);
#pragma unroll
    for (int r = 0; r < RP; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) {
        if (!A.half) o[r][c] += o2[r][c];
        red(w)[(3 * r + c) * 64 + lane] = o[r][c];
      }
    __syncthreads();
    if (split) break;
    for (int k = w; k < RP * 3; k += W) {
      double v = 0.0;
      if (k % 3 < D) {
        const int e = k * 64 + lane;
        if (A.half) {
          v = red(0)[e] + red(1)[e];
          for (int u = 2; u < W; u += 2) v += red(u)[e] + red(u + 1)[e];
        } else {
          v = red(0)[e];
          for (int u = 1; u < W; ++u) v += red(u)[e];
        }
      }
      if (A.v_out) {   // one record: stored below
        xl[k][lane] = v;
        continue;
      }
      const double x = xl[k][lane];
      double y;
      if constexpr (RKS) {
        // stage positions x + c v (c = dt/2, dt/2, dt), then x + dt/6 (v1 + 2 v2 + 2 v3 + v4)
        const int st = t & 3;
        const double acc = st == 0 ? 0.0 : al[k][lane];
        if (st < 3) {
          al[k][lane] = st == 0 ? v : acc + 2.0 * v;
          y = x + (st == 2 ? A.dt : 0.5 * A.dt) * v;
        } else {
          y = x + A.dt / 6.0 * (acc + v);
          xl[k][lane] = y;
        }
      } else {
        y = x + A.dt * v;
        xl[k][lane] = y;
      }
      yl[k][lane] = (R)(A.k * y);
    }
  }
  if (split) {   // wave u writes the sum of the workgroup's pair u
    if (w >= W / 2) return;
    const int pair = (int)blockIdx.y * (W / 2) + w;
    for (int r = 0; r < RP; ++r)
      for (int c = 0; c < D; ++c) {
        const int e = (3 * r + c) * 64 + lane;
        if (point(3 * r) < A.m)
          A.v_part[((size_t)pair * 3 + c) * A.m + point(3 * r)] = red(2 * w)[e] + red(2 * w + 1)[e];
      }
    return;
  }
  for (int k = w; k < RP * 3; k += W) {
    const int c = k % 3, i = point(k);
    if (i >= A.m) continue;
    if (A.v_out) A.v_out[3 * (size_t)i + c] = xl[k][lane];
    else if (A.x_out) A.x_out[3 * (size_t)i + c] = xl[k][lane] + A.cen[c];
    else A.xs[(size_t)c * A.m + i] = xl[k][lane];
  }
}

// v = sum over the pairs in order (planar: z is 0).
__global__ __launch_bounds__(256) void k_flow_sum(int m, int pairs, int dim,
                                                  const double* __restrict__ part,
                                                  double* __restrict__ v) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  for (int c = 0; c < 3; ++c) {
    double s = 0.0;
    if (c < dim) {
      s = part[(size_t)c * m + i];
      for (int u = 1; u < pairs; ++u) s += part[((size_t)u * 3 + c) * m + i];
    }
    v[3 * (size_t)i + c] = s;
  }
}

// Launch `kernel` on grid x threads.  With timing events (ev non-null) the
// launch goes through hipExtLaunchKernelGGL, which ties ev[0] and ev[1] to the
// start and the end of the kernel's own execution, so the elapsed time is
// the kernel's, without the stream's dispatch gap before it.
template <typename A>
inline void launch_timed(void (*kernel)(A), dim3 grid, unsigned threads, hipStream_t s,
                         const A& args, hipEvent_t* ev) {
  if (ev)
    hipExtLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, ev[0], ev[1], 0, args);
  else
    kernel<<<grid, threads, 0, s>>>(args);
}

// Launch KERNEL<targs..., W, D> with W waves per workgroup (1, 2, 4, 8 or 16)
// for planar (D = 2) or 3D (D = 3) problems; other W: invalid value.
#define LDDMM_LAUNCH_WD(W, D, grid, s, args, ev, KERNEL, ...)                                \
  switch ((D) == 2 ? (W) : -(W)) {                                                           \
    case 1: launch_timed(KERNEL<__VA_ARGS__, 1, 2>, grid, 64, s, args, ev); break;           \
    case 2: launch_timed(KERNEL<__VA_ARGS__, 2, 2>, grid, 128, s, args, ev); break;          \
    case 4: launch_timed(KERNEL<__VA_ARGS__, 4, 2>, grid, 256, s, args, ev); break;          \
    case 8: launch_timed(KERNEL<__VA_ARGS__, 8, 2>, grid, 512, s, args, ev); break;          \
    case 12: launch_timed(KERNEL<__VA_ARGS__, 12, 2>, grid, 768, s, args, ev); break;        \
    case 16: launch_timed(KERNEL<__VA_ARGS__, 16, 2>, grid, 1024, s, args, ev); break;       \
    case -1: launch_timed(KERNEL<__VA_ARGS__, 1, 3>, grid, 64, s, args, ev); break;          \
    case -2: launch_timed(KERNEL<__VA_ARGS__, 2, 3>, grid, 128, s, args, ev); break;         \
    case -4: launch_timed(KERNEL<__VA_ARGS__, 4, 3>, grid, 256, s, args, ev); break;         \
    case -8: launch_timed(KERNEL<__VA_ARGS__, 8, 3>, grid, 512, s, args, ev); break;         \
    case -12: launch_timed(KERNEL<__VA_ARGS__, 12, 3>, grid, 768, s, args, ev); break;       \
    case -16: launch_timed(KERNEL<__VA_ARGS__, 16, 3>, grid, 1024, s, args, ev); break;      \
    default: return hipErrorInvalidValue;                                                    \
  }

template <typename R, bool RKS, int D>
hipError_t flow_run(const FlowArgs& a, dim3 grid, int W, int rp, hipStream_t s, hipEvent_t* ev) {
  const unsigned lds = (unsigned)(W * (rp == 2 ? kFlowWaveLds<2> : kFlowWaveLds<1>));
  auto kernel = k_flow<R, RKS, D, 1>;
  if constexpr (std::is_same<R, float>::value)
    if (rp == 2) kernel = k_flow<R, RKS, D, 2>;
  if (ev)
    hipExtLaunchKernelGGL(kernel, grid, dim3(64u * W), lds, s, ev[0], ev[1], 0, a);
  else
    kernel<<<grid, 64 * W, lds, s>>>(a);
  return hipGetLastError();
}

template <typename R>
hipError_t flow_dispatch(const FlowArgs& a, dim3 grid, int W, int rp, hipStream_t s,
                         hipEvent_t* ev) {
  if (a.spt == 4)
    return a.dim == 2 ? flow_run<R, true, 2>(a, grid, W, rp, s, ev)
                      : flow_run<R, true, 3>(a, grid, W, rp, s, ev);
  return a.dim == 2 ? flow_run<R, false, 2>(a, grid, W, rp, s, ev)
                    : flow_run<R, false, 3>(a, grid, W, rp, s, ev);
}

// Split path (S > 1): combine the S workgroup partials in chunk order, then
// update.  A separate launch: combining through memory inside the pair
// kernel needs agent-scope release/acquire per workgroup, whose L2
// write-back and invalidate cost more than this launch.  The partials were
// written by workgroups on other XCDs, so every load is a memory round
// trip: with the chunk count SC known at compile time all of them are in
// flight at once (SC = 0: any S, loaded chunk by chunk).
// Components [C0, C1) of NC (all of them by default); h is indexed by component.
template <typename Acc, int NC, int SC, int C0 = 0, int C1 = NC>
__device__ __forceinline__ void gather_partials(const Acc* __restrict__ P, int n, int S, int ic,
                                                double h[NC]) {
  if constexpr (SC > 0) {
    Acc v[SC][C1 - C0];
#pragma unroll
    for (int s = 0; s < SC; ++s)
#pragma unroll
      for (int c = C0; c < C1; ++c) v[s][c - C0] = P[((size_t)s * NC + c) * n + ic];
#pragma unroll
    for (int c = C0; c < C1; ++c) {
      Acc sum = v[0][c - C0];
#pragma unroll
      for (int s = 1; s < SC; ++s) sum += v[s][c - C0];
      h[c] = sum;
    }
  } else {
    Acc sum[NC];
    for (int c = 0; c < NC; ++c) sum[c] = P[(size_t)c * n + ic];
    for (int s = 1; s < S; ++s)
      for (int c = 0; c < NC; ++c) sum[c] += P[((size_t)s * NC + c) * n + ic];
    for (int c = 0; c < NC; ++c) h[c] = sum[c];
  }
}

// One wave per i-block and latency-bound: let the scheduler spend registers
// on loads in flight rather than on occupancy.
#define LDDMM_LATENCY_BOUND __attribute__((amdgpu_waves_per_eu(1, 2)))

template <typename R, bool COMP, int SC, bool RKS>
__global__ __launch_bounds__(64) LDDMM_LATENCY_BOUND void k_fwd_update(FwdArgs A) {
  using Acc = typename AccOf<R, COMP>::type;
  const int ib = blockIdx.x, lane = threadIdx.x;
  FwdState v = load_fwd_state<RKS>(A, ib * 64 + lane);
  double h[6];
  gather_partials<Acc, 6, SC>(static_cast<const Acc*>(A.partial), A.n, A.S,
                              min(ib * 64 + lane, A.n - 1), h);
  fwd_finish<R, RKS>(A, ib * 64 + lane, ib * 64 + lane < A.n, ib, lane, v, h, h + 3);
}

template <typename R, bool COMP, int SC, bool RKS>
__global__ __launch_bounds__(64) LDDMM_LATENCY_BOUND void k_adj_update(AdjArgs A) {
  using Acc = typename AccOf<R, COMP>::type;
  const int ib = blockIdx.x, lane = threadIdx.x;
  AdjState v = load_adj_state<RKS>(A, ib * 64 + lane);
  double h[9];
  gather_partials<Acc, 9, SC>(static_cast<const Acc*>(A.partial), A.n, A.S,
                              min(ib * 64 + lane, A.n - 1), h);
  adj_finish9<R, RKS>(A, ib, lane, v, h);
}

// The same with two waves per i-block, for SC >= 8: one lane's 9 SC partial
// loads would exceed the 63 vector loads a wave can keep in flight and cost a
// second memory round trip.  Wave 1 sums components 5-8 (in chunk order, as
// above) and hands them over through LDS; wave 0 sums 0-4 and finishes.
template <typename R, bool COMP, int SC, bool RKS>
__global__ __launch_bounds__(128) LDDMM_LATENCY_BOUND void k_adj_update2(AdjArgs A) {
  using Acc = typename AccOf<R, COMP>::type;
  __shared__ double red[4 * 64];
  const int ib = blockIdx.x, lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ic = min(ib * 64 + lane, A.n - 1);
  const Acc* P = static_cast<const Acc*>(A.partial);
  double h[9];
  if (w == 1) {
    gather_partials<Acc, 9, SC, 5, 9>(P, A.n, A.S, ic, h);
    for (int c = 5; c < 9; ++c) red[(c - 5) * 64 + lane] = h[c];
  }
  AdjState v{};
  if (w == 0) {
    v = load_adj_state<RKS>(A, ib * 64 + lane);
    gather_partials<Acc, 9, SC, 0, 5>(P, A.n, A.S, ic, h);
  }
  __syncthreads();
  if (w == 0) {
    for (int c = 5; c < 9; ++c) h[c] = red[(c - 5) * 64 + lane];
    adj_finish9<R, RKS>(A, ib, lane, v, h);
  }
}

// ---------------------------------------------------------------------------
// O(N) kernels: centroid, staging, checkpoint restore, loss, outputs
// ---------------------------------------------------------------------------

// Fixed-order block tree sum over kLossThreads values (result in red[0]).
__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int off = kLossThreads / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// K block sums at once: each is the same fixed-order tree as block_sum, so
// every result is bitwise what K separate calls give, for one set of barriers.
// red holds K * kLossThreads values.
template <int K>
__device__ __forceinline__ void block_sums(double v[K], double* red) {
  for (int k = 0; k < K; ++k) red[k * kLossThreads + threadIdx.x] = v[k];
  __syncthreads();
  for (int off = kLossThreads / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off)
      for (int k = 0; k < K; ++k)
        red[k * kLossThreads + threadIdx.x] += red[k * kLossThreads + threadIdx.x + off];
    __syncthreads();
  }
  for (int k = 0; k < K; ++k) v[k] = red[k * kLossThreads];
  __syncthreads();
}

// Sum of part b (kCenPart landmarks) of q0: per thread the points i = t, t +
// kLossThreads, ... in increasing i (two points' loads in flight at a time), then
// one tree per coordinate.  The centroid is the sum of the parts in order.
constexpr int kCenPart = 4096;

__device__ __forceinline__ void center_part(const double* __restrict__ q0, int n, int b,
                                            double s[3], double* red) {
  const int end = min(n, (b + 1) * kCenPart);
  for (int c = 0; c < 3; ++c) s[c] = 0.0;
  for (int i0 = b * kCenPart + threadIdx.x; i0 < end; i0 += 2 * kLossThreads) {
    double v[2][3];
    for (int u = 0; u < 2; ++u) {
      const int i = min(i0 + u * kLossThreads, end - 1);
      for (int c = 0; c < 3; ++c) v[u][c] = q0[3 * i + c];
    }
    for (int u = 0; u < 2; ++u)
      if (i0 + u * kLossThreads < end)
        for (int c = 0; c < 3; ++c) s[c] += v[u][c];
  }
  block_sums<3>(s, red);
}

__global__ __launch_bounds__(kLossThreads) void k_center_parts(const double* __restrict__ q0, int n,
                                                               double* __restrict__ part) {
  __shared__ double red[3 * kLossThreads];
  double s[3];
  center_part(q0, n, blockIdx.x, s, red);
  if (threadIdx.x < 3) part[3 * blockIdx.x + threadIdx.x] = s[threadIdx.x];
}

// Staging.  Every workgroup forms the centroid for itself: up to 4096 landmarks (98 KB)
// from the points (part null: a launch less, 3.6 us), else from the parts, in
// workgroups of 256 (of 1024: 2.3 us more, n = 4097).
template <typename R>
__global__ __launch_bounds__(kLossThreads) void k_stage(
    int n, const double* __restrict__ q0, const double* __restrict__ p0,
    const double* __restrict__ x, double* __restrict__ cen, const double* __restrict__ part,
    double k, double* __restrict__ st, double* __restrict__ xc, Rec<R>* __restrict__ rec0) {
  __shared__ double red[3 * kLossThreads];
  double s[3];
  if (!part) {
    center_part(q0, n, 0, s, red);
  } else {
    const int np = (n + kCenPart - 1) / kCenPart;
    for (int c = 0; c < 3; ++c) {
      s[c] = part[c];
      for (int b = 1; b < np; ++b) s[c] += part[3 * b + c];
    }
  }
  for (int c = 0; c < 3; ++c) s[c] = s[c] / n;
  if (blockIdx.x == 0 && threadIdx.x < 3) cen[threadIdx.x] = s[threadIdx.x];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double q[3], p[3];
  for (int c = 0; c < 3; ++c) {
    q[c] = q0[3 * i + c] - s[c];
    p[c] = p0[3 * i + c];
    st[c * n + i] = q[c];
    st[(3 + c) * n + i] = p[c];
    if (x) xc[c * n + i] = x[3 * i + c] - s[c];
  }
  rec0[i] = make_rec<R>(k * q[0], k * q[1], k * q[2], p[0], p[1], p[2]);
}

template <typename R>
__global__ __launch_bounds__(256) void k_restore(int n, const double* __restrict__ ck, double k,
                                                 double* __restrict__ st, Rec<R>* __restrict__ rec) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double v[6];
  for (int c = 0; c < 6; ++c) { v[c] = ck[c * n + i]; st[c * n + i] = v[c]; }
  rec[i] = make_rec<R>(k * v[0], k * v[1], k * v[2], v[3], v[4], v[5]);
}

__device__ __forceinline__ double sum_h0(const double* __restrict__ h0_part, int nb, double* red) {
  double h = 0.0;
  for (int b = threadIdx.x; b < nb; b += kLossThreads) h += h0_part[b];
  return 0.5 * block_sum(h, red);
}

template <typename R>
__device__ __forceinline__ void loss_body(int n, int nb, double lambda, const double* __restrict__ st,
                                          const double* __restrict__ xc,
                                          const double* __restrict__ cen,
                                          const double* __restrict__ h0_part,
                                          double* __restrict__ ad, Rec<R>* __restrict__ arec0,
                                          double* __restrict__ out3, double* __restrict__ q1,
                                          double* __restrict__ p1, int* __restrict__ flag,
                                          double* __restrict__ grad_x,
                                          const double* __restrict__ hqT,
                                          const double* __restrict__ hpT, double bscale,
                                          double rscale, double* red) {
  // Landmarks i = t, t + kLossThreads, ... in increasing i, two at a time with
  // every input loaded before any output is stored (all loads in flight).
  double mis = 0.0;
  for (int i0 = threadIdx.x; i0 < n; i0 += 2 * kLossThreads) {
    double qv[2][3], xv[2][3], hq[2][3], hp[2][3], pv[2][3];
    for (int u = 0; u < 2; ++u) {
      const int i = min(i0 + u * kLossThreads, n - 1);
      for (int c = 0; c < 3; ++c) {
        qv[u][c] = st[c * n + i];
        xv[u][c] = xc[c * n + i];
        hq[u][c] = hqT ? hqT[c * n + i] : 0.0;
        hp[u][c] = hqT ? hpT[c * n + i] : 0.0;
        pv[u][c] = p1 ? st[(3 + c) * n + i] : 0.0;
      }
    }
    for (int u = 0; u < 2; ++u) {
      const int i = i0 + u * kLossThreads;
      if (i >= n) break;
      double a[3], b[3];
      for (int c = 0; c < 3; ++c) {
        const double q = qv[u][c];
        const double r = q - xv[u][c];
        mis += r * r;
        a[c] = 2.0 * lambda * r;           // dL/dq(1) of the mismatch
        b[c] = 0.0;                        // dL/dp(1)
        if (grad_x) grad_x[3 * i + c] = -a[c];
        if (hqT) {                         // energy term H(q(1), p(1))
          a[c] += hq[u][c];
          b[c] = hp[u][c];
        }
        ad[c * n + i] = a[c];
        ad[(3 + c) * n + i] = b[c];
        if (q1) q1[3 * i + c] = q + cen[c];
        if (p1) p1[3 * i + c] = pv[u][c];
      }
      if (rscale != 1.0)                   // the first Runge-Kutta stage adjoint is dt/6 lambda
        for (int c = 0; c < 3; ++c) { a[c] = rscale * a[c]; b[c] = rscale * b[c]; }
      arec0[i] = make_rec<R>(a[0], a[1], a[2], bscale * b[0], bscale * b[1], bscale * b[2]);
    }
  }
  double h = 0.0;
  for (int b = threadIdx.x; b < nb; b += kLossThreads) h += h0_part[b];
  double sums[2] = {mis, h};
  block_sums<2>(sums, red);                // red: 2 kLossThreads values
  const double m = sums[0];
  const double H0 = 0.5 * sums[1];
  if (threadIdx.x == 0) {
    const double L = H0 + lambda * m;
    out3[0] = L;
    out3[1] = H0;
    out3[2] = m;
    if (!isfinite(L)) atomicOr(flag, 1);
  }
}

template <typename R>
__global__ __launch_bounds__(kLossThreads) void k_loss(
    int n, int nb, double lambda, const double* __restrict__ st, const double* __restrict__ xc,
    const double* __restrict__ cen, const double* __restrict__ h0_part, double* __restrict__ ad,
    Rec<R>* __restrict__ arec0, double* __restrict__ out3, double* __restrict__ q1,
    double* __restrict__ p1, int* __restrict__ flag, double* __restrict__ grad_x,
    const double* __restrict__ hqT, const double* __restrict__ hpT, double bscale,
    double rscale) {
  __shared__ double red[2 * kLossThreads];
  loss_body<R>(n, nb, lambda, st, xc, cen, h0_part, ad, arec0, out3, q1, p1, flag, grad_x, hqT,
               hpT, bscale, rscale, red);
}

__global__ __launch_bounds__(kLossThreads) void k_forward_out(
    int n, int nb, const double* __restrict__ st, const double* __restrict__ cen,
    const double* __restrict__ h0_part, double* __restrict__ H0, double* __restrict__ q1,
    double* __restrict__ p1) {
  __shared__ double red[kLossThreads];
  for (int i = threadIdx.x; i < n; i += kLossThreads)
    for (int c = 0; c < 3; ++c) {
      if (q1) q1[3 * i + c] = st[c * n + i] + cen[c];
      if (p1) p1[3 * i + c] = st[(3 + c) * n + i];
    }
  const double h = sum_h0(h0_part, nb, red);
  if (threadIdx.x == 0 && H0) *H0 = h;
}

// ---------------------------------------------------------------------------
// batched kernels: several registrations per launch
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool job_live(const BatchJob& b) { return b.active && *b.done == 0; }

template <typename R>
__global__ __launch_bounds__(256) void k_stage_batch(const BatchJob* __restrict__ J) {
  const BatchJob& b = J[blockIdx.y];
  if (!job_live(b)) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= b.n) return;
  const int n = b.n;
  double q[3], p[3];
  for (int c = 0; c < 3; ++c) {
    q[c] = b.q0[3 * i + c] - b.cen[c];
    p[c] = b.p0[3 * i + c];
    b.st[c * n + i] = q[c];
    b.st[(3 + c) * n + i] = p[c];
  }
  const double k = b.sc.k;
  static_cast<Rec<R>*>(b.traj)[i] = make_rec<R>(k * q[0], k * q[1], k * q[2], p[0], p[1], p[2]);
}

// stage: 0 for an Euler step, else Runge-Kutta stage 1..4 of step t.  Record
// r = spt t + stage - 1 (stage 0: r = t) is read, record r + 1 written (the
// next stage's state, or after the last stage the state of step t + 1).
// (BW: waves per workgroup of the block kernels.)
template <typename R, int D, int BW = 1>
__device__ __forceinline__ FwdArgs batch_fwd_args(const BatchJob& b, int t, int stage) {
  FwdArgs A{};
  A.n = b.n; A.ig = b.row.ig; A.jg = b.row.jg;
  A.nb = b.nb; A.S = 1; A.chunk = b.n; A.wchunk = (b.n + BW - 1) / BW;
  A.dim = D;
  A.rk = stage;
  A.rk_acc = b.rk_acc;
  A.sc = b.sc;
  const int r = b.spt * t + (stage > 0 ? stage - 1 : 0);
  A.rec_t = static_cast<const Rec<R>*>(b.traj) + (size_t)r * b.n;
  A.rec_t1 = static_cast<Rec<R>*>(b.traj) + (size_t)(r + 1) * b.n;
  A.st = b.st;
  const bool first = t == 0 && stage <= 1;   // the field at (q0, p0)
  A.hp0 = first ? b.hp0 : nullptr;
  A.h0_part = first ? b.h0p : nullptr;
  return A;
}

// Adjoint launches run t = T-1 .. 0 (and stages 4 .. 1 within a Runge-Kutta
// step); the loss kernel fills adjoint record buffer 0 for the first of them,
// and each launch reads buffer (launch index & 1) and writes the other.
template <typename R, int D, int BW = 1>
__device__ __forceinline__ AdjArgs batch_adj_args(const BatchJob& b, int t, int stage, int T) {
  AdjArgs A{};
  A.n = b.n; A.ig = b.row.ig; A.jg = b.row.jg;
  A.nb = b.nb; A.S = 1; A.chunk = b.n; A.wchunk = (b.n + BW - 1) / BW;
  A.dim = D;
  A.rk = stage;
  A.rk_lam = b.rk_lam;
  A.sc = b.sc;
  const int launch = stage > 0 ? (T - 1 - t) * 4 + (4 - stage) : T - 1 - t;
  const int cur = launch & 1;
  const int r = b.spt * t + (stage > 0 ? stage - 1 : 0);
  A.rec_t = static_cast<const Rec<R>*>(b.traj) + (size_t)r * b.n;
  A.arec = static_cast<const Rec<R>*>(b.arec) + (size_t)cur * b.n;
  A.arec_next = static_cast<Rec<R>*>(b.arec) + (size_t)(cur ^ 1) * b.n;
  A.ad = b.ad;
  A.hp0 = b.hp0;
  A.grad = t == 0 && stage <= 1 ? b.grad : nullptr;
  return A;
}

// Work items: nitems[0] items of 3D jobs, then nitems[1] items of planar jobs;
// the D = 3 instance takes the first group, the D = 2 instance the second.  An
// item is one workgroup's rows of a job (row kernels); workgroup b of G takes the
// items b, b + G, ... (one each, up to kBatchGrid of them).  The items come with the
// largest jobs first, so what is left to balance at the end are short ones; the state
// is loaded after the sums (other workgroups cover its latency, and the registers are
// worth more).  FP32's occupancy is what its registers allow without spills.  What
// bounds it: issue.
template <typename R, int D, bool ADJ, bool RKS>
__global__ __launch_bounds__(64 * kBatchWaves,
                             sizeof(R) == 8 ? 1 : ADJ ? 4 : 5) void k_batch(const BatchJob* __restrict__ J,
                                                            const int2* __restrict__ items,
                                                            const int* __restrict__ nitems, int t,
                                                            int stage, int T) {
  constexpr int M = kBatchRows;
  __shared__ double red[kBatchWaves * (row_pad<D, M> / 4) * 64];
  __shared__ double fin[kBatchWaves * row_pad<D, M>];
  const int2* it = items + (D == 2 ? nitems[0] : 0);
  const int count = nitems[D == 2 ? 1 : 0];
  for (int k = blockIdx.x; k < count; k += gridDim.x) {
    const BatchJob& b = J[it[k].x];
    if (!job_live(b)) continue;
    if constexpr (ADJ) adj_rows<R, RKS, D, M, true>(batch_adj_args<R, D>(b, t, stage, T), it[k].y, red, fin);
    else fwd_rows<R, RKS, D, M, true>(batch_fwd_args<R, D>(b, t, stage), it[k].y, red, fin);
  }
}

// The block kernels (batch_blocks): an item is one i-block of 64 landmarks, a
// workgroup of BW waves that splits the j.  Their loops are the split kernels', in
// FP32 the compensated ones for both modes: a job's accuracy must not follow from the
// server's size, and 12 waves of them are the faster ones too (solves of 2 to 64 jobs
// in 0.53 to 1.03 of the time of the 8-wave running sums, most below 0.95).
template <typename R, bool COMP, int D, bool ADJ, bool RKS>
__global__ __launch_bounds__(64 * batch_waves(COMP)) void k_batch_blocks(
    const BatchJob* __restrict__ J, const int2* __restrict__ items, const int* __restrict__ nitems,
    int t, int stage, int T) {
  constexpr int BW = batch_waves(COMP);
  __shared__ typename AccOf<R, COMP>::type red[BW * (ADJ ? 9 : 6) * 64];
  if ((int)blockIdx.x >= nitems[D == 2 ? 1 : 0]) return;
  const int2 it = items[(D == 2 ? nitems[0] : 0) + (int)blockIdx.x];
  const BatchJob& b = J[it.x];
  if (!job_live(b)) return;
  if constexpr (ADJ)
    adj_block<R, COMP, RKS, BW, D>(batch_adj_args<R, D, BW>(b, t, stage, T), it.y, 0, red);
  else fwd_block<R, COMP, RKS, BW, D>(batch_fwd_args<R, D, BW>(b, t, stage), it.y, 0, red);
}

template <typename R>
__global__ __launch_bounds__(kLossThreads) void k_loss_batch(const BatchJob* __restrict__ J) {
  __shared__ double red[2 * kLossThreads];
  const BatchJob& b = J[blockIdx.x];
  if (!job_live(b)) return;
  loss_body<R>(b.n, b.nh, b.lambda, b.st, b.xc, b.cen, b.h0p, b.ad, static_cast<Rec<R>*>(b.arec),
               b.out3, b.q1, nullptr, b.flag, nullptr, nullptr, nullptr, 0.0,
               b.spt == 4 ? b.sc.dt / 6.0 : 1.0, red);
}

// ---------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------
template <typename R, bool COMP, bool RKS>
hipError_t fwd_dispatch(const Plan& p, const FwdArgs& a, hipStream_t s, hipEvent_t* ev) {
  const dim3 grid(p.nb * p.S);
  LDDMM_LAUNCH_WD(p.W, a.dim, grid, s, a, ev, k_fwd, R, COMP, RKS)
  switch (p.S) {
    case 1: break;
    case 2: k_fwd_update<R, COMP, 2, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 3: k_fwd_update<R, COMP, 3, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 4: k_fwd_update<R, COMP, 4, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 8: k_fwd_update<R, COMP, 8, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 16: k_fwd_update<R, COMP, 16, RKS><<<p.nb, 64, 0, s>>>(a); break;
    default: k_fwd_update<R, COMP, 0, RKS><<<p.nb, 64, 0, s>>>(a); break;
  }
  return hipGetLastError();
}

template <typename R, bool COMP, bool RKS>
hipError_t adj_dispatch(const Plan& p, const AdjArgs& a, hipStream_t s, hipEvent_t* ev) {
  const dim3 grid(p.nb * p.S);
  LDDMM_LAUNCH_WD(p.Wa, a.dim, grid, s, a, ev, k_adj, R, COMP, RKS)
  switch (p.S) {
    case 1: break;
    case 2: k_adj_update<R, COMP, 2, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 3: k_adj_update<R, COMP, 3, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 4: k_adj_update<R, COMP, 4, RKS><<<p.nb, 64, 0, s>>>(a); break;
    case 8: k_adj_update2<R, COMP, 8, RKS><<<p.nb, 128, 0, s>>>(a); break;
    case 16: k_adj_update2<R, COMP, 16, RKS><<<p.nb, 128, 0, s>>>(a); break;
    default: k_adj_update<R, COMP, 0, RKS><<<p.nb, 64, 0, s>>>(a); break;
  }
  return hipGetLastError();
}

// Row kernels (RowPlan): the whole step in one launch.
template <typename R, bool RKS, int M>
hipError_t fwd_rows_launch(const RowPlan& p, const FwdArgs& a, hipStream_t s, hipEvent_t* ev) {
  launch_timed(a.dim == 2 ? k_fwd_rows<R, RKS, 2, M> : k_fwd_rows<R, RKS, 3, M>,
               dim3((unsigned)p.groups), 64u * (unsigned)(p.ig * p.jg), s, a, ev);
  return hipGetLastError();
}
template <typename R, bool RKS, int M>
hipError_t adj_rows_launch(const RowPlan& p, const AdjArgs& a, hipStream_t s, hipEvent_t* ev) {
  launch_timed(a.dim == 2 ? k_adj_rows<R, RKS, 2, M> : k_adj_rows<R, RKS, 3, M>,
               dim3((unsigned)p.groups), 64u * (unsigned)(p.ig * p.jg), s, a, ev);
  return hipGetLastError();
}

template <bool RKS>
hipError_t fwd_rows_dispatch(int mode, const RowPlan& p, const FwdArgs& a, hipStream_t s,
                             hipEvent_t* ev) {
  if (mode == kFP64) {
    switch (p.m) {
      case 2: return fwd_rows_launch<double, RKS, 2>(p, a, s, ev);
      case 3: return fwd_rows_launch<double, RKS, 3>(p, a, s, ev);
      case 4: return fwd_rows_launch<double, RKS, 4>(p, a, s, ev);
    }
  } else {
    switch (p.m) {
      case 3: return fwd_rows_launch<float, RKS, 3>(p, a, s, ev);
      case 4: return fwd_rows_launch<float, RKS, 4>(p, a, s, ev);
      case 5: return fwd_rows_launch<float, RKS, 5>(p, a, s, ev);
    }
  }
  return hipErrorInvalidValue;
}

template <bool RKS>
hipError_t adj_rows_dispatch(int mode, const RowPlan& p, const AdjArgs& a, hipStream_t s,
                             hipEvent_t* ev) {
  if (mode == kFP64) {
    switch (p.m) {
      case 2: return adj_rows_launch<double, RKS, 2>(p, a, s, ev);
      case 3: return adj_rows_launch<double, RKS, 3>(p, a, s, ev);
      case 4: return adj_rows_launch<double, RKS, 4>(p, a, s, ev);
    }
  } else {
    switch (p.m) {
      case 3: return adj_rows_launch<float, RKS, 3>(p, a, s, ev);
      case 4: return adj_rows_launch<float, RKS, 4>(p, a, s, ev);
      case 5: return adj_rows_launch<float, RKS, 5>(p, a, s, ev);
    }
  }
  return hipErrorInvalidValue;
}

inline unsigned blocks256(int n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// The point record's size is what the workspace layout (plan.h) assumes.
static_assert(sizeof(Rec<float>) == 32 && sizeof(Rec<double>) == 64, "record size");

hipError_t launch_stage(int mode, int n, const double* q0, const double* p0, const double* x,
                        double* cen, double* part, double k, double* st, double* xc, void* rec0,
                        hipStream_t s) {
  const bool fused = n <= kCenPart;
  const int threads = fused ? kLossThreads : 256;
  if (fused) part = nullptr;
  else k_center_parts<<<(n + kCenPart - 1) / kCenPart, kLossThreads, 0, s>>>(q0, n, part);
  const unsigned grid = (unsigned)((n + threads - 1) / threads);
  if (mode == kFP64)
    k_stage<double><<<grid, threads, 0, s>>>(n, q0, p0, x, cen, part, k, st, xc,
                                             static_cast<Rec<double>*>(rec0));
  else
    k_stage<float><<<grid, threads, 0, s>>>(n, q0, p0, x, cen, part, k, st, xc,
                                            static_cast<Rec<float>*>(rec0));
  return hipGetLastError();
}

hipError_t launch_restore(int mode, int n, const double* ckpt, double k, double* st, void* rec,
                          hipStream_t s) {
  if (mode == kFP64)
    k_restore<double><<<blocks256(n), 256, 0, s>>>(n, ckpt, k, st, static_cast<Rec<double>*>(rec));
  else
    k_restore<float><<<blocks256(n), 256, 0, s>>>(n, ckpt, k, st, static_cast<Rec<float>*>(rec));
  return hipGetLastError();
}

template <typename R>
void fwd_chain_dispatch(const ChainArgs& c, const FwdArgs& a, hipStream_t s, hipEvent_t* ev) {
  auto* k = c.spt == 4 ? (a.dim == 2 ? k_fwd_chain<R, true, 2> : k_fwd_chain<R, true, 3>)
                       : (a.dim == 2 ? k_fwd_chain<R, false, 2> : k_fwd_chain<R, false, 3>);
  const dim3 threads(64 * kChainWaves);
  if (ev) hipExtLaunchKernelGGL(k, dim3(1), threads, 0, s, ev[0], ev[1], 0, c, a);
  else k<<<1, threads, 0, s>>>(c, a);
}
template <typename R>
void adj_chain_dispatch(const ChainArgs& c, const AdjArgs& a, hipStream_t s, hipEvent_t* ev) {
  auto* k = c.spt == 4 ? (a.dim == 2 ? k_adj_chain<R, true, 2> : k_adj_chain<R, true, 3>)
                       : (a.dim == 2 ? k_adj_chain<R, false, 2> : k_adj_chain<R, false, 3>);
  const dim3 threads(64 * kChainWaves);
  if (ev) hipExtLaunchKernelGGL(k, dim3(1), threads, 0, s, ev[0], ev[1], 0, c, a);
  else k<<<1, threads, 0, s>>>(c, a);
}

hipError_t launch_fwd_chain(int mode, const ChainArgs& c, const FwdArgs& a, hipStream_t s,
                            hipEvent_t* ev) {
  if (a.n > kChainMax) return hipErrorInvalidValue;
  if (mode == kFP64) fwd_chain_dispatch<double>(c, a, s, ev);
  else fwd_chain_dispatch<float>(c, a, s, ev);
  return hipGetLastError();
}

hipError_t launch_adj_chain(int mode, const ChainArgs& c, const AdjArgs& a, hipStream_t s,
                            hipEvent_t* ev) {
  if (a.n > kChainMax) return hipErrorInvalidValue;
  if (mode == kFP64) adj_chain_dispatch<double>(c, a, s, ev);
  else adj_chain_dispatch<float>(c, a, s, ev);
  return hipGetLastError();
}

hipError_t launch_fwd_step(int mode, const Plan& p, const FwdArgs& a, hipStream_t s,
                           hipEvent_t* ev) {
  const bool rk = a.rk != 0;
  if (p.row.m > 0) {
    if (mode != kFP32 && mode != kFP32Comp && mode != kFP64) return hipErrorInvalidValue;
    return rk ? fwd_rows_dispatch<true>(mode, p.row, a, s, ev)
              : fwd_rows_dispatch<false>(mode, p.row, a, s, ev);
  }
  switch (mode) {
    case kFP32:
      return rk ? fwd_dispatch<float, false, true>(p, a, s, ev)
                : fwd_dispatch<float, false, false>(p, a, s, ev);
    case kFP32Comp:
      return rk ? fwd_dispatch<float, true, true>(p, a, s, ev)
                : fwd_dispatch<float, true, false>(p, a, s, ev);
    case kFP64:
      return rk ? fwd_dispatch<double, false, true>(p, a, s, ev)
                : fwd_dispatch<double, false, false>(p, a, s, ev);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_adj_step(int mode, const Plan& p, const AdjArgs& a, hipStream_t s,
                           hipEvent_t* ev) {
  const bool rk = a.rk != 0;
  if (p.row.m > 0) {
    if (mode != kFP32 && mode != kFP32Comp && mode != kFP64) return hipErrorInvalidValue;
    return rk ? adj_rows_dispatch<true>(mode, p.row, a, s, ev)
              : adj_rows_dispatch<false>(mode, p.row, a, s, ev);
  }
  switch (mode) {
    case kFP32:
      return rk ? adj_dispatch<float, false, true>(p, a, s, ev)
                : adj_dispatch<float, false, false>(p, a, s, ev);
    case kFP32Comp:
      return rk ? adj_dispatch<float, true, true>(p, a, s, ev)
                : adj_dispatch<float, true, false>(p, a, s, ev);
    case kFP64:
      return rk ? adj_dispatch<double, false, true>(p, a, s, ev)
                : adj_dispatch<double, false, false>(p, a, s, ev);
  }
  return hipErrorInvalidValue;
}

// A wave per chunk while the points leave room for it (us per step at n = 4096:
// m = 5003 47 -> 18, 20000 48 -> 32, 100000 129 -> 112; with a wave per pair of
// chunks and two points per lane 41, 42, 124); two points per lane where that
// fills its rounds of 1024 workgroups at least 0.94 as well as one per lane fills
// its rounds of 512 (m = 262144: 275 -> 242, one per lane 258).  FP64: a wave
// per pair from 2048 such waves on (velocity at n = 4096, m = 262144 779 us, per chunk
// 842; Runge-Kutta flow at n = 10007, m = 20000, two steps, 2950 and 3120, where 16
// waves leave a CU one workgroup).
// A velocity of fewer than 512 workgroups is also spread by the pairs (n =
// 4096, m = 5003 86 -> 29 us; n = 20000, m = 1000 136 -> 81, 105 without).
hipError_t launch_flow(int mode, const FlowArgs& args, hipStream_t s, hipEvent_t* ev) {
  FlowArgs a = args;
  if (a.m <= 0 || a.n <= 0 || a.t1 <= a.t0 || a.slots <= 0) return hipErrorInvalidValue;
  if (a.v_out && a.t1 != a.t0 + 1) return hipErrorInvalidValue;
  if (mode != kFP32 && mode != kFP32Comp && mode != kFP64) return hipErrorInvalidValue;
  const auto filled = [](int b, int round) { return (double)b / ((b + round - 1) / round * round); };
  const int b1 = (a.m + 63) / 64, b2 = (a.m + 127) / 128;
  const bool two = mode != kFP64 && a.pairs == 8 && b2 >= 1024 &&
                   filled(b2, 1024) >= 0.94 * filled(b1, 512);
  a.half = two || (mode == kFP64 && b1 * a.pairs >= 2048) ? 0 : 1;
  int W = a.half ? 2 * a.pairs : a.pairs;
  dim3 grid((unsigned)(two ? b2 : b1));
  const bool split = a.v_part && a.v_out && a.half && W > 4 && b1 < 512;
  if (split) {
    grid.y = (unsigned)(W / 4);
    W = 4;
  }
  const int rp = two ? 2 : 1;
  const hipError_t e = mode == kFP64 ? flow_dispatch<double>(a, grid, W, rp, s, ev)
                                     : flow_dispatch<float>(a, grid, W, rp, s, ev);
  if (e != hipSuccess || !split) return e;
  k_flow_sum<<<blocks256(a.m), 256, 0, s>>>(a.m, a.pairs, a.dim == 2 ? 2 : 3, a.v_part, a.v_out);
  return hipGetLastError();
}

hipError_t launch_loss(int mode, int n, int nb, double lambda, double bscale, double rscale,
                       const double* st, const double* xc, const double* cen,
                       const double* h0_part, double* ad, void* arec0, double* out3, double* q1,
                       double* p1, int* flag, double* grad_x, const double* hqT,
                       const double* hpT, hipStream_t s) {
  if (mode == kFP64)
    k_loss<double><<<1, kLossThreads, 0, s>>>(n, nb, lambda, st, xc, cen, h0_part, ad,
                                              static_cast<Rec<double>*>(arec0), out3, q1, p1, flag,
                                              grad_x, hqT, hpT, bscale, rscale);
  else
    k_loss<float><<<1, kLossThreads, 0, s>>>(n, nb, lambda, st, xc, cen, h0_part, ad,
                                             static_cast<Rec<float>*>(arec0), out3, q1, p1, flag,
                                             grad_x, hqT, hpT, bscale, rscale);
  return hipGetLastError();
}

hipError_t launch_forward_out(int n, int nb, const double* st, const double* cen,
                              const double* h0_part, double* H0, double* q1, double* p1,
                              hipStream_t s) {
  k_forward_out<<<1, kLossThreads, 0, s>>>(n, nb, st, cen, h0_part, H0, q1, p1);
  return hipGetLastError();
}

hipError_t launch_stage_batch(int mode, const BatchJob* jobs, int max_slots, int max_n,
                              hipStream_t s) {
  const dim3 grid((max_n + 255) / 256, max_slots);
  if (mode == kFP64) k_stage_batch<double><<<grid, 256, 0, s>>>(jobs);
  else k_stage_batch<float><<<grid, 256, 0, s>>>(jobs);
  return hipGetLastError();
}

template <typename R, bool COMP, int D, bool ADJ>
void batch_dispatch(bool blocks, const BatchJob* jobs, const int2* items, const int* nitems,
                    int capacity, int t, int stage, int T, hipStream_t s) {
  const auto launch = [&](auto* k, int grid, int waves) {
    k<<<grid, 64 * waves, 0, s>>>(jobs, items, nitems, t, stage, T);
  };
  const int rows = min(capacity, kBatchGrid);
  if (blocks && stage > 0)
    launch(k_batch_blocks<R, COMP, D, ADJ, true>, capacity, batch_waves(COMP));
  else if (blocks) launch(k_batch_blocks<R, COMP, D, ADJ, false>, capacity, batch_waves(COMP));
  else if (stage > 0) launch(k_batch<R, D, ADJ, true>, rows, kBatchWaves);
  else launch(k_batch<R, D, ADJ, false>, rows, kBatchWaves);
}

template <bool ADJ, int D>
hipError_t batch_mode(int mode, bool blocks, const BatchJob* jobs, const int2* items,
                      const int* nitems, int capacity, int t, int stage, int T, hipStream_t s) {
  switch (mode) {
    case kFP32:   // the same sums as kFP32Comp
    case kFP32Comp: batch_dispatch<float, true, D, ADJ>(blocks, jobs, items, nitems, capacity, t, stage, T, s); break;
    case kFP64: batch_dispatch<double, false, D, ADJ>(blocks, jobs, items, nitems, capacity, t, stage, T, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fwd_batch(int mode, int dim, bool blocks, const BatchJob* jobs, const int2* items,
                            const int* nitems, int capacity, int t, int stage, hipStream_t s) {
  if (dim == 2) return batch_mode<false, 2>(mode, blocks, jobs, items, nitems, capacity, t, stage, 0, s);
  if (dim == 3) return batch_mode<false, 3>(mode, blocks, jobs, items, nitems, capacity, t, stage, 0, s);
  return hipErrorInvalidValue;
}

hipError_t launch_adj_batch(int mode, int dim, bool blocks, const BatchJob* jobs, const int2* items,
                            const int* nitems, int capacity, int t, int stage, int T,
                            hipStream_t s) {
  if (dim == 2) return batch_mode<true, 2>(mode, blocks, jobs, items, nitems, capacity, t, stage, T, s);
  if (dim == 3) return batch_mode<true, 3>(mode, blocks, jobs, items, nitems, capacity, t, stage, T, s);
  return hipErrorInvalidValue;
}

hipError_t launch_loss_batch(int mode, const BatchJob* jobs, int max_slots, hipStream_t s) {
  if (mode == kFP64) k_loss_batch<double><<<max_slots, kLossThreads, 0, s>>>(jobs);
  else k_loss_batch<float><<<max_slots, kLossThreads, 0, s>>>(jobs);
  return hipGetLastError();
}

}  // namespace lddmm
