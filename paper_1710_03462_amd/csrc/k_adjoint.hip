// k_adjoint.hip -- gfx950 kernels for differentiating RK2 advection in the
// ABC field: forward with checkpoints, the discrete adjoint with
// recomputation, and a squared-distance loss.
//
// One thread owns one particle (in small sets a quad of lanes does, see below)
// for the whole time loop; the state stays in registers.  The adjoint walks
// the checkpoint segments backwards; for each segment it recomputes the states
// from the checkpoint, keeping every state's
// sines and cosines (in registers, indexed by compile-time constants through
// fully unrolled loops so that they never touch scratch memory, and in LDS),
// and sweeps them backwards.  Segments longer than what is kept are split
// into sub-segments, each recomputed from the checkpoint.  When k and nsteps
// are multiples of the renewal interval below, the forward and the adjoint
// run their steps in blocks of straight-line code without a branch per step.
// Parameter gradients are summed per particle in reverse step order, then
// over particles by a fixed-shape tree (per workgroup, then one final
// workgroup), so results are deterministic and do not depend on k.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_math.h"
#include "launch.h"

namespace soax {

namespace {

constexpr int kRedBlock = kAdjointBlock;  // workgroup size of every reducing kernel but the quads'

// Rows of one checkpoint on the tape: the position and the sines and cosines
// the forward evaluated at it.
constexpr int kTapeRows = 9;

// Sines and cosines of the state of step s (its global index) in the loops
// over many steps of one particle.  With every shift proven at most 1/8 (TIER
// kTierSmall or kTierMid) they come from the previous state's by rotation over
// the step's displacement, renewed by a full reduction at every step index
// that is a multiple of kAnchor, so each value depends on the step index
// alone (not on the checkpoint interval) and carries at most kAnchor - 1
// rotations (half an ulp of 1 to one ulp each).  Larger steps (kTierAny)
// reduce every state in full.  kAnchor equals the register block of the usual
// checkpoint interval (20), so that a block that starts at a multiple of it
// has no renewal inside: such blocks run as straight-line code
// (rk2_ckpt_blocks_kernel, adjoint_blocks_kernel).
constexpr int64_t kAnchor = 20;

// One explicit-midpoint step from (x, y, z) with sines and cosines t, no
// wrap; on return (x, y, z) is the next state and t its sines and cosines,
// reduced in full (RENEW, and every step of kTierAny) or carried: rotated by
// the step's displacement before the position is rounded, which is closer to
// the step as written than a rotation between the two rounded positions.
template <int TIER, bool RENEW>
__device__ __forceinline__ void rk2_advance_to(const StepAbc& p, double& x, double& y, double& z,
                                               Trig3& t) {
  double m0, m1, m2;
  field_of(p.h, t, m0, m1, m2);
  const Trig3 tm = trig3_shift<TIER>(t, x, y, z, m0, m1, m2);
  field_of(p.d, tm, m0, m1, m2);
  const double x1 = x + m0, y1 = y + m1, z1 = z + m2;
  if (RENEW || TIER == kTierAny)
    t = trig3(x1, y1, z1);
  else
    t = trig3_shift<TIER>(t, x, y, z, m0, m1, m2);
  x = x1;
  y = y1;
  z = z1;
}

// The same with the choice at run time: renew, the next state's index is a
// multiple of kAnchor.
template <int TIER>
__device__ __forceinline__ void rk2_advance(const StepAbc& p, bool renew, double& x, double& y,
                                            double& z, Trig3& t) {
  if (renew)
    rk2_advance_to<TIER, true>(p, x, y, z, t);
  else
    rk2_advance_to<TIER, false>(p, x, y, z, t);
}

// A checkpoint (x, y, z, t) at tp, rows n apart.  The tape is written once
// and read back much later.
__device__ __forceinline__ void store_ckpt(double* tp, int64_t n, double x, double y, double z,
                                           const Trig3& t) {
  st1<true>(tp, x);
  st1<true>(tp + n, y);
  st1<true>(tp + 2 * n, z);
  st1<true>(tp + 3 * n, t.sx);
  st1<true>(tp + 4 * n, t.cx);
  st1<true>(tp + 5 * n, t.sy);
  st1<true>(tp + 6 * n, t.cy);
  st1<true>(tp + 7 * n, t.sz);
  st1<true>(tp + 8 * n, t.cz);
}

__device__ __forceinline__ void load_ckpt(const double* cp, int64_t n, double& x, double& y,
                                          double& z, Trig3& t) {
  x = cp[0];
  y = cp[n];
  z = cp[2 * n];
  t = Trig3{cp[3 * n], cp[4 * n], cp[5 * n], cp[6 * n], cp[7 * n], cp[8 * n]};
}

template <int TIER>
__global__ __launch_bounds__(256) void rk2_ckpt_kernel(CkptArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const StepAbc& p = a.step;
  const int64_t e = i * a.stride;
  double x = a.x0[0][e], y = a.x0[1][e], z = a.x0[2][e];
  Trig3 t = trig3(x, y, z);
  double* tp = a.tape + i;
  const int64_t n = a.n;
  int64_t until_ckpt = 0;
  int r = 1;  // (s + 1) mod kAnchor, kept by counting
  for (int64_t s = 0; s < a.nsteps; ++s) {
    if (until_ckpt == 0) {
      store_ckpt(tp, n, x, y, z, t);
      tp += kTapeRows * n;
      until_ckpt = a.k;
    }
    --until_ckpt;
    rk2_advance<TIER>(p, r == 0, x, y, z, t);
    r = r + 1 == kAnchor ? 0 : r + 1;
  }
  st1<true>(a.xT[0] + e, x);
  st1<true>(a.xT[1] + e, y);
  st1<true>(a.xT[2] + e, z);
}

// rk2_ckpt_kernel when k and nsteps are multiples of kAnchor: the steps run
// in blocks of kAnchor that start at renewal points, each kAnchor - 1 carried
// steps and one renewed step as straight-line code (the same values; without
// a branch per step the compiler overlaps consecutive steps).  Every
// checkpoint falls on a block's start.
template <int TIER>
__global__ __launch_bounds__(256) void rk2_ckpt_blocks_kernel(CkptArgs a) {
  constexpr int KB = static_cast<int>(kAnchor);
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const StepAbc& p = a.step;
  const int64_t e = i * a.stride;
  double x = a.x0[0][e], y = a.x0[1][e], z = a.x0[2][e];
  Trig3 t = trig3(x, y, z);
  double* tp = a.tape + i;
  const int64_t n = a.n;
  for (int64_t s0 = 0; s0 < a.nsteps; s0 += KB) {
    if (s0 % a.k == 0) {
      store_ckpt(tp, n, x, y, z, t);
      tp += kTapeRows * n;
    }
#pragma unroll
    for (int j = 0; j < KB - 1; ++j) {
      rk2_advance_to<TIER, false>(p, x, y, z, t);
      // keep the sums of displacements where they arise: put off to the end
      // of the block they would hold a register pair per step
      asm volatile("" : "+v"(x), "+v"(y), "+v"(z));
    }
    rk2_advance_to<TIER, true>(p, x, y, z, t);
  }
  st1<true>(a.xT[0] + e, x);
  st1<true>(a.xT[1] + e, y);
  st1<true>(a.xT[2] + e, z);
}

// Reverse one midpoint step taken from state (x, y, z), whose sines and
// cosines are t.  With xm = x + (dt/2) u(x) and x+ = x + dt u(xm):
//   mu  = dt J(xm)^T lam+
//   g  += dt G(xm)^T lam+ + (dt/2) G(x)^T mu
//   lam = lam+ + mu + (dt/2) J(x)^T mu
// where J = du/dx and G = du/d(A,B,C).  Each row of J^T is one amplitude
// times a difference, (J^T v)_0 = B (cos x v_1 - sin x v_2) and so on; with r
// those differences at xm, m = (dt/2) J(xm)^T lam+ = mu/2, and g kept without
// its factor dt (the caller multiplies by it at the end):
//   r = (cos x_m lam_1 - sin x_m lam_2, ...),  m = (dt/2) (B, C, A) r,
//   g/dt += G(xm)^T lam+ + G(x)^T m,
//   lam  = lam+ + dt (B, C, A) (r + (cos x m_1 - sin x m_2, ...))
// so that every sum is a chain of fused multiply-adds.  A step's four terms of
// g are summed by themselves, smallest first, and added with one rounding of
// g's size: taken into g one by one they round it four times a step.
// (x, y, z) is read by kTierAny alone.
template <int TIER>
__device__ __forceinline__ void rk2_reverse(const StepAbc& p, const Trig3& t, double x, double y,
                                            double z, double& l0, double& l1, double& l2,
                                            double& g0, double& g1, double& g2) {
  double h0, h1, h2;  // (dt/2) u(x), as in the forward step
  field_of(p.h, t, h0, h1, h2);
  const Trig3 m = trig3_shift<TIER>(t, x, y, z, h0, h1, h2);  // at xm
  const double r0 = fma(m.cx, l1, -(m.sx * l2));
  const double r1 = fma(m.cy, l2, -(m.sy * l0));
  const double r2 = fma(m.cz, l0, -(m.sz * l1));
  const double m0 = p.h.B * r0, m1 = p.h.C * r1, m2 = p.h.A * r2;
  g0 += fma(m.sz, l0, fma(m.cz, l1, fma(t.sz, m0, t.cz * m1)));
  g1 += fma(m.sx, l1, fma(m.cx, l2, fma(t.sx, m1, t.cx * m2)));
  g2 += fma(m.sy, l2, fma(m.cy, l0, fma(t.sy, m2, t.cy * m0)));
  l0 = fma(p.d.B, fma(t.cx, m1, fma(-t.sx, m2, r0)), l0);
  l1 = fma(p.d.C, fma(t.cy, m2, fma(-t.sy, m0, r1)), l1);
  l2 = fma(p.d.A, fma(t.cz, m0, fma(-t.sz, m1, r2)), l2);
}

// Sum v over the workgroup (BLOCK threads) in a fixed tree order.
template <int BLOCK = kRedBlock>
__device__ __forceinline__ void block_sum3(double v0, double v1, double v2, double* out3) {
  __shared__ double red[3][BLOCK];
  const int t = threadIdx.x;
  red[0][t] = v0;
  red[1][t] = v1;
  red[2][t] = v2;
  __syncthreads();
  for (int s = BLOCK / 2; s > 0; s >>= 1) {
    if (t < s) {
      red[0][t] += red[0][t + s];
      red[1][t] += red[1][t + s];
      red[2][t] += red[2][t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    out3[0] = red[0][0];
    out3[1] = red[1][0];
    out3[2] = red[2][0];
  }
}

// A point the compiler may not see through: the values are read and written
// there, as far as it knows.
__device__ __forceinline__ void opaque(Trig3& t) {
  asm volatile("" : "+v"(t.sx), "+v"(t.cx), "+v"(t.sy), "+v"(t.cy), "+v"(t.sz), "+v"(t.cz));
}

// The sines and cosines of the states 0 .. K - 1 of a (sub-)segment, written
// by the recomputation and read by the reverse sweep with compile-time
// indices (the sweep used to carry them back from state to state, 36 more
// instructions a step): the first L states in LDS, one 16-byte pair per
// coordinate and thread, the others in registers.
//
// The reverse sweep also needs each step's midpoint values, which the
// recomputation has had, and the compiler would rather keep those too than
// repeat them: twelve more registers a state, which it then spills.  get()
// is opaque below state `reuse`, so that the midpoint is evaluated again
// there, and the last few states, whose midpoints are wanted first and for
// which registers are left, keep theirs.
template <int K, int L>
struct KeptTrig {
  double2 (*lds)[3][kRedBlock];
  Trig3 reg[K - L];

  __device__ __forceinline__ void put(int j, const Trig3& t) {
    if (j < L) {
      lds[j][0][threadIdx.x] = make_double2(t.sx, t.cx);
      lds[j][1][threadIdx.x] = make_double2(t.sy, t.cy);
      lds[j][2][threadIdx.x] = make_double2(t.sz, t.cz);
    } else {
      reg[j - L] = t;
    }
  }
  __device__ __forceinline__ Trig3 get(int j, int reuse) const {
    Trig3 t;
    if (j < L) {
      const double2 a = lds[j][0][threadIdx.x], b = lds[j][1][threadIdx.x],
                    c = lds[j][2][threadIdx.x];
      t = Trig3{a.x, a.y, b.x, b.y, c.x, c.y};
    } else {
      t = reg[j - L];
    }
    if (j < reuse) opaque(t);
    return t;
  }
};

// States of a 20-state segment kept in LDS: 6 x 48 bytes a thread, and 24 for
// block_sum3, for each of the two workgroups of 256 threads that share a
// compute unit (156 of its 160 KB); the others' 168 registers leave two waves
// per SIMD.
constexpr int kLdsStates = 6;
static_assert(2 * kRedBlock * (kLdsStates * sizeof(Trig3) + 3 * sizeof(double)) <= 160 * 1024,
              "two workgroups must share a compute unit's LDS");

// The adjoint for any k and nsteps (shifts of at most 1/8).  4e6 particles x
// 160 steps, forward and loss included, before -> now: k = 16 7.28 -> 5.71 ms,
// k = 10 7.68 -> 5.24, k = 5 7.86 -> 5.69, k = 32 9.14 -> 6.18, and with
// shifts beyond 1/64, which used to reduce every state in full, 11.7 -> 5.9.
// A segment is cut into pieces of at most KM states that do not cross a renewal point, so that
// a piece's recomputation only carries; the steps from the checkpoint to a
// later piece's first state are taken one by one.  KM: states kept, the first
// L of them in LDS; REUSE: as in KeptTrig.
template <int KM, int L, int REUSE, int TIER>
__global__ __launch_bounds__(kRedBlock, 2) void adjoint_kernel(AdjointArgs a) {
  static_assert(KM <= kAnchor && kAnchor % KM == 0, "a piece must not cross a renewal point");
  constexpr int kPrefetchAt = KM < 8 ? KM : 8;
  __shared__ double2 kept_lds[L > 0 ? L : 1][3][kRedBlock];
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const StepAbc& p = a.step;
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;
  if (i < a.n) {
    const int64_t n = a.n;
    const int64_t e = i * a.stride;
    double l0 = a.lam[0][e], l1 = a.lam[1][e], l2 = a.lam[2][e];
    int64_t end = a.nsteps;                               // the piece is [begin, end)
    int64_t c = (a.nsteps + a.k - 1) / a.k - 1;           // its segment
    double x = 0.0, y = 0.0, z = 0.0;
    Trig3 t{};
    if (a.nsteps > 0) load_ckpt(a.tape + (c * kTapeRows) * n + i, n, x, y, z, t);
    while (end > 0) {
      const int64_t ck = c * a.k;
      const int64_t cut = (end - 1) / KM * KM;  // KM divides kAnchor
      const int64_t begin = cut > ck ? cut : ck;
      for (int64_t s = ck; s < begin; ++s)
        rk2_advance<TIER>(p, (s + 1) % kAnchor == 0, x, y, z, t);
      const int m = static_cast<int>(end - begin);
      end = begin;
      c = begin == ck && c > 0 ? c - 1 : c;
      KeptTrig<KM, L> kept;
      kept.lds = kept_lds;
#pragma unroll
      for (int j = 0; j < KM; ++j) {
        if (j < m) {
          if (j > 0) rk2_advance_to<TIER, false>(p, x, y, z, t);
          opaque(t);
          kept.put(j, t);
        }
      }
#pragma unroll
      for (int j = KM - 1; j >= kPrefetchAt; --j)
        if (j < m) rk2_reverse<TIER>(p, kept.get(j, REUSE), 0.0, 0.0, 0.0, l0, l1, l2, g0, g1, g2);
      load_ckpt(a.tape + (c * kTapeRows) * n + i, n, x, y, z, t);  // the next piece's
#pragma unroll
      for (int j = kPrefetchAt - 1; j >= 0; --j)
        if (j < m) rk2_reverse<TIER>(p, kept.get(j, REUSE), 0.0, 0.0, 0.0, l0, l1, l2, g0, g1, g2);
    }
    a.gx[0][e] = l0;
    a.gx[1][e] = l1;
    a.gx[2][e] = l2;
  }
  block_sum3(a.dt * g0, a.dt * g1, a.dt * g2, a.partial + 3 * static_cast<int64_t>(blockIdx.x));
}

// The adjoint for shifts that may exceed 1/8 (kTierAny): the states'
// positions are kept, KM of them in registers, and every state's sines and
// cosines are reduced in full, in the recomputation and in the reverse sweep.
template <int KM>
__global__ __launch_bounds__(kRedBlock) void adjoint_any_kernel(AdjointArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const StepAbc& p = a.step;
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;
  if (i < a.n) {
    const int64_t n = a.n;
    const int64_t e = i * a.stride;
    double l0 = a.lam[0][e], l1 = a.lam[1][e], l2 = a.lam[2][e];
    const int64_t nseg = (a.nsteps + a.k - 1) / a.k;
    for (int64_t c = nseg - 1; c >= 0; --c) {
      const int64_t len = min(a.k, a.nsteps - c * a.k);
      const double* cp = a.tape + (c * kTapeRows) * n + i;
      const int64_t nsub = (len + KM - 1) / KM;
      for (int64_t q = nsub - 1; q >= 0; --q) {
        double x, y, z;
        Trig3 t;
        load_ckpt(cp, n, x, y, z, t);
        for (int64_t s = 0; s < q * KM; ++s) rk2_advance_to<kTierAny, true>(p, x, y, z, t);
        const int m = static_cast<int>(min(static_cast<int64_t>(KM), len - q * KM));
        double sx[KM], sy[KM], sz[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) {
          if (j < m) {
            sx[j] = x;
            sy[j] = y;
            sz[j] = z;
            if (j + 1 < m) rk2_advance_to<kTierAny, true>(p, x, y, z, t);
          }
        }
#pragma unroll
        for (int j = KM - 1; j >= 0; --j) {
          if (j < m)
            rk2_reverse<kTierAny>(p, trig3(sx[j], sy[j], sz[j]), sx[j], sy[j], sz[j], l0, l1, l2,
                                  g0, g1, g2);
        }
      }
    }
    a.gx[0][e] = l0;
    a.gx[1][e] = l1;
    a.gx[2][e] = l2;
  }
  block_sum3(a.dt * g0, a.dt * g1, a.dt * g2, a.partial + 3 * static_cast<int64_t>(blockIdx.x));
}

// Bound by fp64 issue: 95% of the issue slots (counters) at the 1.9 GHz the
// clock falls to under this load, so its time is its instruction count.
// 1e7 particles x 200 steps, k = 20, with the loss and the forward: 18.2 ms
// before the states' sines were kept, the sums fused and the carried
// displacement left unrounded, 14.6 ms with them (adjoint 13.3 -> 9.0 ms;
// 136 instructions per particle-step, 203 before), and 14.7 with a step's
// gradient terms summed before they reach the running sum (three more).  One
// wave per SIMD with 512 registers and more midpoints kept: 15.0 ms against
// the 14.6.  Errors against an 80-bit reference, before -> now: grad_x0
// 1.8e-15 -> 1.6e-15 and xT 7.2e-16 -> 7.2e-16 of 2e4 particles,
// dL/d(A,B,C) of 24 sets of 64 particles 8.8e-16 -> 8.1e-16 (130 steps of
// 1e-2: 6.3e-16 -> 5.3e-16), of 3 sets of 33000 1.2e-16 -> 0.9e-16.
//
// adjoint_kernel when k and nsteps are multiples of kAnchor: every segment's
// length is then a multiple of kAnchor too, and every block of kAnchor states
// starts at a renewal point (its first state's index is a multiple of
// kAnchor), so its recomputation only carries.  These are adjoint_kernel's
// values bit for bit, as straight-line code without a branch per step, which
// lets the compiler overlap consecutive steps (adjoint_kernel's per-step
// branches split the code into blocks it does not schedule across).  The
// next block's checkpoint is loaded inside the reverse sweep, whose kept
// states leave their registers one by one.
template <int TIER>
__global__ __launch_bounds__(kRedBlock, 2) void adjoint_blocks_kernel(AdjointArgs a) {
  constexpr int KB = static_cast<int>(kAnchor);
  constexpr int kReuse = 18;  // states from here on keep their midpoints
  constexpr int kPrefetchAt = 8;  // states still to reverse when the next checkpoint is asked for
  __shared__ double2 kept_lds[kLdsStates][3][kRedBlock];
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const StepAbc& p = a.step;
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;
  if (i < a.n) {
    const int64_t n = a.n;
    const int64_t e = i * a.stride;
    double l0 = a.lam[0][e], l1 = a.lam[1][e], l2 = a.lam[2][e];
    const int64_t per_seg = a.k / KB;  // blocks of a whole segment
    int64_t c = (a.nsteps + a.k - 1) / a.k - 1;      // segment of the current block
    int64_t q = (a.nsteps - c * a.k) / KB - 1;       // its index in the segment
    double x = 0.0, y = 0.0, z = 0.0;
    Trig3 t{};
    if (a.nsteps > 0) load_ckpt(a.tape + (c * kTapeRows) * n + i, n, x, y, z, t);
    for (int64_t left = a.nsteps / KB; left > 0; --left) {
      for (int64_t s = 0; s < q; ++s) {  // up to the block's first state
#pragma unroll 1
        for (int j = 0; j < KB - 1; ++j) rk2_advance_to<TIER, false>(p, x, y, z, t);
        rk2_advance_to<TIER, true>(p, x, y, z, t);
      }
      // the next block: the one before in this segment, or the last of the
      // segment before (this one again when none is left)
      const bool same = q > 0 || c == 0;
      c = same ? c : c - 1;
      q = q > 0 ? q - 1 : per_seg - 1;
      KeptTrig<KB, kLdsStates> kept;
      kept.lds = kept_lds;
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        kept.put(j, t);
        if (j + 1 < KB) rk2_advance_to<TIER, false>(p, x, y, z, t);
        opaque(t);
      }
#pragma unroll
      for (int j = KB - 1; j >= kPrefetchAt; --j)
        rk2_reverse<TIER>(p, kept.get(j, kReuse), 0.0, 0.0, 0.0, l0, l1, l2, g0, g1, g2);
      load_ckpt(a.tape + (c * kTapeRows) * n + i, n, x, y, z, t);
#pragma unroll
      for (int j = kPrefetchAt - 1; j >= 0; --j)
        rk2_reverse<TIER>(p, kept.get(j, kReuse), 0.0, 0.0, 0.0, l0, l1, l2, g0, g1, g2);
    }
    a.gx[0][e] = l0;
    a.gx[1][e] = l1;
    a.gx[2][e] = l2;
  }
  block_sum3(a.dt * g0, a.dt * g1, a.dt * g2, a.partial + 3 * static_cast<int64_t>(blockIdx.x));
}

// ------------------------------------------- small sets: a quad per particle
//
// Up to kQuadMax particles the kernels above leave the machine short of
// waves: a wave is alone on its SIMD, and its time is its instruction count.
// Here a particle's three coordinates go to three lanes of a quad (the fourth
// repeats the first and stores nothing), which halves the instructions of a
// step and quadruples the waves.  The field and its transpose couple the
// coordinates cyclically,
//   u_d = alpha_d sin x_(d+2) + beta_d cos x_(d+1),
//   alpha = (A, B, C), beta = (C, A, B), indices modulo 3,
// so every lane runs the same code on its own coordinate and its two
// neighbours' values, moved within the quad.  Each component is evaluated in
// the same order as above: the results are the same, bit for bit, but for the
// order in which particles' parameter gradients are summed.

// Lane d's value from lanes (d+1) mod 3 and (d+2) mod 3 of its quad.
constexpr int kQuadNext = 1 | (2 << 2) | (0 << 4) | (1 << 6);
constexpr int kQuadPrev = 2 | (0 << 2) | (1 << 4) | (2 << 6);

template <int CTRL>
__device__ __forceinline__ double quad_move(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp(static_cast<int>(b), CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_mov_dpp(static_cast<int>(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ double quad_next(double v) { return quad_move<kQuadNext>(v); }
__device__ __forceinline__ double quad_prev(double v) { return quad_move<kQuadPrev>(v); }

template <typename T>
__device__ __forceinline__ T pick3(int d, T a, T b, T c) {
  return d == 0 ? a : (d == 1 ? b : c);
}

// One coordinate's share of the field's coefficients, times dt/2 and dt.
struct QuadAbc {
  double ah, bh, ad, bd;  // alpha and beta
  double ch, cd;          // (B, C, A): the rows of the transposed Jacobian
  __device__ __forceinline__ QuadAbc(const StepAbc& p, int d)
      : ah(pick3(d, p.h.A, p.h.B, p.h.C)), bh(pick3(d, p.h.C, p.h.A, p.h.B)),
        ad(pick3(d, p.d.A, p.d.B, p.d.C)), bd(pick3(d, p.d.C, p.d.A, p.d.B)),
        ch(pick3(d, p.h.B, p.h.C, p.h.A)), cd(pick3(d, p.d.B, p.d.C, p.d.A)) {}
};

struct Trig1 {
  double s, c;
};

__device__ __forceinline__ double quad_field(double a, double b, const Trig1& t) {
  return fma(a, quad_prev(t.s), b * quad_next(t.c));
}

template <int TIER>
__device__ __forceinline__ Trig1 shift1(const Trig1& t, double d) {
  Trig1 r;
  trig::sincos_shift<TIER>(0.0, t.s, t.c, d, &r.s, &r.c);
  return r;
}

// rk2_advance_to on one coordinate.
template <int TIER, bool RENEW>
__device__ __forceinline__ void quad_advance(const QuadAbc& p, double& x, Trig1& t) {
  static_assert(TIER != kTierAny, "the quad kernels carry");
  const Trig1 tm = shift1<TIER>(t, quad_field(p.ah, p.bh, t));
  const double m = quad_field(p.ad, p.bd, tm);
  x = x + m;
  if (RENEW)
    trig::sincos_fast(x, &t.s, &t.c);
  else
    t = shift1<TIER>(t, m);
}

// rk2_reverse on one coordinate; lane d's g is the gradient of (B, C, A)[d].
template <int TIER>
__device__ __forceinline__ void quad_reverse(const QuadAbc& p, const Trig1& t, double& l,
                                             double& g) {
  const Trig1 tm = shift1<TIER>(t, quad_field(p.ah, p.bh, t));
  const double l1 = quad_next(l), l2 = quad_prev(l);
  const double r = fma(tm.c, l1, -(tm.s * l2));
  const double m = p.ch * r;
  const double m1 = quad_next(m), m2 = quad_prev(m);
  g += fma(tm.s, l1, fma(tm.c, l2, fma(t.s, m1, t.c * m2)));
  l = fma(p.cd, fma(t.c, m1, fma(-t.s, m2, r)), l);
}

constexpr int kQuadBlock = 256;
constexpr int kQuadParticles = kQuadBlock / 4;

template <int TIER>
__global__ __launch_bounds__(kQuadBlock) void rk2_ckpt_quad_kernel(CkptArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kQuadParticles + (threadIdx.x >> 2);
  if (i >= a.n) return;
  const int lane = static_cast<int>(threadIdx.x) & 3;
  const int d = lane == 3 ? 0 : lane;
  const bool stores = lane != 3;
  const QuadAbc p(a.step, d);
  const int64_t e = i * a.stride, n = a.n;
  double x = pick3(d, a.x0[0], a.x0[1], a.x0[2])[e];
  Trig1 t;
  trig::sincos_fast(x, &t.s, &t.c);
  double* tp = a.tape + i;
  int64_t to_ckpt = 0, to_renew = kAnchor;  // steps until the next of each
  for (int64_t left = a.nsteps; left > 0;) {
    if (to_ckpt == 0) {
      if (stores) {
        st1<true>(tp + d * n, x);
        st1<true>(tp + (3 + 2 * d) * n, t.s);
        st1<true>(tp + (4 + 2 * d) * n, t.c);
      }
      tp += kTapeRows * n;
      to_ckpt = a.k;
    }
    // steps up to the next checkpoint, renewal or end: all but the last carry
    int64_t run = to_ckpt < to_renew ? to_ckpt : to_renew;
    run = run < left ? run : left;
    left -= run;
    to_ckpt -= run;
    to_renew -= run;
    const int carried = static_cast<int>(run) - 1;  // run <= kAnchor
    int j = 0;
    for (; j + 4 <= carried; j += 4) {
      quad_advance<TIER, false>(p, x, t);
      quad_advance<TIER, false>(p, x, t);
      quad_advance<TIER, false>(p, x, t);
      quad_advance<TIER, false>(p, x, t);
    }
    for (; j < carried; ++j) quad_advance<TIER, false>(p, x, t);
    if (to_renew == 0) {
      quad_advance<TIER, true>(p, x, t);
      to_renew = kAnchor;
    } else {
      quad_advance<TIER, false>(p, x, t);
    }
  }
  if (stores) st1<true>(pick3(d, a.xT[0], a.xT[1], a.xT[2]) + e, x);
}

// adjoint_kernel with a quad per particle.  A whole piece of 20 states runs as
// straight-line code, in which the compiler also keeps the midpoints' sines
// and cosines (a lane keeps one coordinate's, 80 registers each way).
template <int TIER>
__global__ __launch_bounds__(kQuadBlock, 2) void adjoint_quad_kernel(AdjointArgs a) {
  constexpr int KM = static_cast<int>(kAnchor);
  __shared__ double red[3][kQuadParticles];
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kQuadParticles + (threadIdx.x >> 2);
  const int lane = static_cast<int>(threadIdx.x) & 3;
  const int d = lane == 3 ? 0 : lane;
  const QuadAbc p(a.step, d);
  double g = 0.0;
  if (i < a.n) {
    const int64_t n = a.n;
    const int64_t e = i * a.stride;
    double l = pick3(d, a.lam[0], a.lam[1], a.lam[2])[e];
    const double* tape = a.tape + i;
    int64_t end = a.nsteps;                      // the piece is [begin, end)
    int64_t c = (a.nsteps + a.k - 1) / a.k - 1;  // its segment
    double x = 0.0;
    Trig1 t{};
    const auto load = [&]() {
      const double* cp = tape + c * kTapeRows * n;
      x = cp[d * n];
      t = Trig1{cp[(3 + 2 * d) * n], cp[(4 + 2 * d) * n]};
    };
    if (a.nsteps > 0) load();
    while (end > 0) {
      const int64_t ck = c * a.k;
      const int64_t cut = (end - 1) / kAnchor * kAnchor;
      const int64_t begin = cut > ck ? cut : ck;
      int r = static_cast<int>(ck % kAnchor);
      for (int64_t s = ck; s < begin; ++s) {
        r = r + 1 == KM ? 0 : r + 1;
        if (r == 0) quad_advance<TIER, true>(p, x, t);
        else quad_advance<TIER, false>(p, x, t);
      }
      const int m = static_cast<int>(end - begin);
      end = begin;
      c = begin == ck && c > 0 ? c - 1 : c;
      Trig1 kept[KM];
      if (m == KM) {
#pragma unroll
        for (int j = 0; j < KM; ++j) {
          if (j > 0) quad_advance<TIER, false>(p, x, t);
          kept[j] = t;
        }
        load();  // the next piece's checkpoint
#pragma unroll
        for (int j = KM - 1; j >= 0; --j) quad_reverse<TIER>(p, kept[j], l, g);
      } else {
#pragma unroll
        for (int j = 0; j < KM; ++j) {
          if (j < m) {
            if (j > 0) quad_advance<TIER, false>(p, x, t);
            kept[j] = t;
          }
        }
        load();
#pragma unroll
        for (int j = KM - 1; j >= 0; --j)
          if (j < m) quad_reverse<TIER>(p, kept[j], l, g);
      }
    }
    if (lane != 3) pick3(d, a.gx[0], a.gx[1], a.gx[2])[e] = l;
  }
  // the workgroup's sums in a fixed tree order: lane 0 holds B's gradient,
  // lane 1 C's and lane 2 A's
  const int q = static_cast<int>(threadIdx.x) >> 2;
  if (lane != 3) red[pick3(lane, 1, 2, 0)][q] = a.dt * g;
  __syncthreads();
  for (int s = kQuadParticles / 2; s > 0; s >>= 1) {
    if (q < s && lane != 3) red[lane][q] += red[lane][q + s];
    __syncthreads();
  }
  if (threadIdx.x < 3) a.partial[3 * static_cast<int64_t>(blockIdx.x) + threadIdx.x] = red[threadIdx.x][0];
}

// One thread's share of the partial sums (every kSumBlock-th triple), in
// ascending order.  The loads of kSumBatch triples leave before the first
// addition: one workgroup does the whole sum, which otherwise waits out one
// memory latency per triple (39063 triples, 1e7 particles: 69 -> 13 us with
// 1024 threads in place of 256).
constexpr int kSumBlock = 1024;
constexpr int kSumBatch = 8;

__device__ __forceinline__ void sum_partials(const double* __restrict__ partial, int64_t nparts,
                                             double& v0, double& v1, double& v2) {
  int64_t b = threadIdx.x;
  for (; b + (kSumBatch - 1) * kSumBlock < nparts; b += kSumBatch * kSumBlock) {
    double w[kSumBatch][3];
#pragma unroll
    for (int j = 0; j < kSumBatch; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) w[j][d] = partial[3 * (b + j * kSumBlock) + d];
#pragma unroll
    for (int j = 0; j < kSumBatch; ++j) {
      v0 += w[j][0];
      v1 += w[j][1];
      v2 += w[j][2];
    }
  }
  for (; b < nparts; b += kSumBlock) {
    v0 += partial[3 * b];
    v1 += partial[3 * b + 1];
    v2 += partial[3 * b + 2];
  }
}

// One workgroup: out[d] = sum_b partial[3b + d], each thread summing a fixed
// strided slice in order, then the fixed tree.
__global__ __launch_bounds__(kSumBlock) void final_sum3_kernel(const double* __restrict__ partial,
                                                               int64_t nparts,
                                                               double* __restrict__ out) {
  double v0 = 0.0, v1 = 0.0, v2 = 0.0;
  sum_partials(partial, nparts, v0, v1, v2);
  block_sum3<kSumBlock>(v0, v1, v2, out);
}

// Like final_sum3_kernel but the sum of the three components goes to out[0].
__global__ __launch_bounds__(kSumBlock) void final_sum1_kernel(const double* __restrict__ partial,
                                                               int64_t nparts,
                                                               double* __restrict__ out) {
  __shared__ double tot[3];
  double v0 = 0.0, v1 = 0.0, v2 = 0.0;
  sum_partials(partial, nparts, v0, v1, v2);
  block_sum3<kSumBlock>(v0, v1, v2, tot);
  __syncthreads();
  if (threadIdx.x == 0) out[0] = (tot[0] + tot[1]) + tot[2];
}

__global__ __launch_bounds__(kRedBlock) void sqdist_kernel(LossArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  double e0 = 0.0, e1 = 0.0, e2 = 0.0;
  if (i < a.n) {
    const int64_t e = i * a.stride;
    e0 = a.xT[0][e] - a.target[0][i];
    e1 = a.xT[1][e] - a.target[1][i];
    e2 = a.xT[2][e] - a.target[2][i];
    if (a.lam[0]) {
      a.lam[0][e] = 2.0 * e0;
      a.lam[1][e] = 2.0 * e1;
      a.lam[2][e] = 2.0 * e2;
    }
  }
  block_sum3(e0 * e0, e1 * e1, e2 * e2, a.partial + 3 * static_cast<int64_t>(blockIdx.x));
}

}  // namespace

namespace {

// Particles up to which a quad of lanes takes each (steps whose shifts are
// at most 1/8): up to 2^15 the quads' waves are at most two to a SIMD.  us for
// forward, loss and adjoint of 160 steps, k = 20, and of 130 steps with
// dt = 1e-2, k = 16, one lane per particle -> quads: 1000 particles 86 -> 49
// and 122 -> 68, 16000 88 -> 51 and 126 -> 71, 32000 90 -> 72 and 128 -> 97;
// 50000 91 -> 116 and 129 -> 161.
constexpr int64_t kQuadMax = 1 << 15;

bool quad_case(int64_t n, int tier) { return n <= kQuadMax && tier != kTierAny; }

int64_t quad_blocks(int64_t n) { return (n + kQuadParticles - 1) / kQuadParticles; }

template <int TIER>
void forward_launch(const CkptArgs& a, hipStream_t s) {
  const int64_t grid = (a.n + 255) / 256;
  if constexpr (TIER != kTierAny) {
    if (quad_case(a.n, TIER)) {
      hipLaunchKernelGGL(rk2_ckpt_quad_kernel<TIER>, dim3(quad_blocks(a.n)), dim3(kQuadBlock), 0, s,
                         a);
      return;
    }
    if (a.k % kAnchor == 0 && a.nsteps % kAnchor == 0) {
      hipLaunchKernelGGL(rk2_ckpt_blocks_kernel<TIER>, dim3(grid), dim3(256), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL(rk2_ckpt_kernel<TIER>, dim3(grid), dim3(256), 0, s, a);
}

template <int TIER>
void adjoint_launch(const AdjointArgs& a, int64_t grid, hipStream_t s) {
  if (quad_case(a.n, TIER))
    hipLaunchKernelGGL(adjoint_quad_kernel<TIER>, dim3(grid), dim3(kQuadBlock), 0, s, a);
  else if (a.k % kAnchor == 0 && a.nsteps % kAnchor == 0)
    hipLaunchKernelGGL(adjoint_blocks_kernel<TIER>, dim3(grid), dim3(kRedBlock), 0, s, a);
  else if (a.k <= 10)
    hipLaunchKernelGGL((adjoint_kernel<10, 0, 10, TIER>), dim3(grid), dim3(kRedBlock), 0, s, a);
  else
    hipLaunchKernelGGL((adjoint_kernel<20, kLdsStates, 20, TIER>), dim3(grid), dim3(kRedBlock), 0,
                       s, a);
}

}  // namespace

hipError_t launch_rk2_forward_ckpt(const CkptArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  switch (a.tier) {
    case kTierSmall: forward_launch<kTierSmall>(a, s); break;
    case kTierMid: forward_launch<kTierMid>(a, s); break;
    default: forward_launch<kTierAny>(a, s); break;
  }
  return hipGetLastError();
}

int64_t adjoint_partials(int64_t n, int tier) {
  return quad_case(n, tier) ? quad_blocks(n) : (n + kRedBlock - 1) / kRedBlock;
}

hipError_t launch_adjoint(const AdjointArgs& a, hipStream_t s) {
  const int64_t grid = adjoint_partials(a.n, a.tier);
  if (grid > 0) {
    switch (a.tier) {
      case kTierSmall: adjoint_launch<kTierSmall>(a, grid, s); break;
      case kTierMid: adjoint_launch<kTierMid>(a, grid, s); break;
      default:
        if (a.k <= 8)
          hipLaunchKernelGGL(adjoint_any_kernel<8>, dim3(grid), dim3(kRedBlock), 0, s, a);
        else if (a.k <= 20)
          hipLaunchKernelGGL(adjoint_any_kernel<20>, dim3(grid), dim3(kRedBlock), 0, s, a);
        else
          hipLaunchKernelGGL(adjoint_any_kernel<32>, dim3(grid), dim3(kRedBlock), 0, s, a);
        break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(final_sum3_kernel, dim3(1), dim3(kSumBlock), 0, s, a.partial, grid,
                     a.grad_abc);
  return hipGetLastError();
}

int64_t loss_partials(int64_t n) { return (n + kRedBlock - 1) / kRedBlock; }

hipError_t launch_sqdist_loss(const LossArgs& a, hipStream_t s) {
  const int64_t grid = loss_partials(a.n);
  if (grid > 0) {
    hipLaunchKernelGGL(sqdist_kernel, dim3(grid), dim3(kRedBlock), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(final_sum1_kernel, dim3(1), dim3(kSumBlock), 0, s, a.partial, grid, a.loss);
  return hipGetLastError();
}

}  // namespace soax
