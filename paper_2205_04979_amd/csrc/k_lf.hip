// One-dimensional Eulerian deposition model (Appendix B): particle momentum
// equation with turbophoresis, image-charge and wall-cohesion forces, and the
// constant-flux equation that gives V_dep+, for many particle classes at once.
//
// The momentum equation is marched from the pipe centre (V = 0) to the wall with
// implicit drag; the flux equation J = D drho/dy + V rho, rho(centre) = 1,
// J = rho_w h_w, is carried along the SAME inward pass: over each cell the exact
// solution with V, D frozen at the cell means maps rho linearly, so
// rho(y) = alpha(y) + J beta(y) and only two scaled coefficients travel with the
// march (s = 1/alpha, b = beta/alpha; both stay bounded where alpha itself would
// overflow).  At the wall the kinetic wall condition closes J = h_w / (s_0 - h_w b_0).
//
// Mapping: a workgroup takes C classes through the nodes in chunks.  Only the speed (the root of
// a quadratic per node) and the two flux coefficients (two products) depend on the node before;
// everything else of a node -- the closure's power and quotient, the potentials, the exponential
// of the flux cell, about nine tenths of the arithmetic -- is independent from node to node.  One
// wave, lane = class, runs the two short chains; the others take one node and class per lane, one
// chunk ahead of the chains and one behind, with one barrier per chunk.  With few classes the
// speed chain bounds the time (about 17 dependent operations a node), with many the FP64 rate.
// One lane per class, each marching alone through every node, took 1.61 ms for 480 classes x
// 1,600 nodes and 1.62 ms for 25,920 (0.4 waves per SIMD, every latency exposed); now 0.18 and
// 0.46 ms.  Error of the result against 80-bit arithmetic over 1,000 random classes: relative rms
// 1.00e-15, as with the library's pow, exp, expm1, sqrt and divisions (1.00e-15).
//
// Closures (the paper defers them to other publications; these are stated
// substitutes): tau_1+ = tau_p+; V'_fy+ = 0.005 y^2 / (1 + 0.002923 y^2.128);
// Rr = 1 / (1 + tau_p+ / tau_L+), tau_L+ = 10; eps/nu = tau_L+ Rr V'_fy+^2;
// D_B/nu by Stokes-Einstein at 293 K; wall velocity variance
// Rr V'_fy+^2 + k_B T / (m u*^2); half-Maxwellian wall flux.
// Grid: gaps y+ - d+/2 geometric from 1e-12 m to 1 wall unit (n_wall nodes),
// then uniform to the centre (n_core more nodes).

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "launch.hpp"

namespace depo {

namespace {

constexpr double kBoltzmann = 1.380649e-23;
constexpr double kTempLF = 293.0;
constexpr double kTauLPlus = 10.0;
constexpr double kGapMin = 1e-12;

// Quotient of normal numbers: Newton's iteration on the hardware's reciprocal, then one residual
// correction of the quotient.
__device__ __forceinline__ double quot(double a, double b) {
  double y = __builtin_amdgcn_rcp(b);
  y = fma(y, fma(-b, y, 1.0), y);
  y = fma(y, fma(-b, y, 1.0), y);
  const double q = a * y;
  return fma(fma(-b, q, a), y, q);
}

constexpr double kLn2Hi = 0.693147180559945309, kLn2Lo = 2.3190468138462996e-17;   // ln 2 to 106 bits

// e^x = two_k (1 + p): x = k ln 2 + r, |r| <= ln 2 / 2, p = e^r - 1 by its Taylor series
// (the term left out is r^14 / 14! < 5e-18).
__device__ __forceinline__ double exp_split(double x, double &two_k) {
  x = fmax(x, -1100.0);   // e^x is 0 long before
  const double k = __builtin_rint(x * 1.4426950408889634);
  const double r = fma(-k, kLn2Lo, fma(-k, kLn2Hi, x));
  double t = 1.0 / 6227020800.0;
  t = fma(t, r, 1.0 / 479001600.0);
  t = fma(t, r, 1.0 / 39916800.0);
  t = fma(t, r, 1.0 / 3628800.0);
  t = fma(t, r, 1.0 / 362880.0);
  t = fma(t, r, 1.0 / 40320.0);
  t = fma(t, r, 1.0 / 5040.0);
  t = fma(t, r, 1.0 / 720.0);
  t = fma(t, r, 1.0 / 120.0);
  t = fma(t, r, 1.0 / 24.0);
  t = fma(t, r, 1.0 / 6.0);
  t = fma(t, r, 0.5);
  two_k = __builtin_amdgcn_ldexp(1.0, (int)k);
  return fma(t * r, r, r);
}

// Natural logarithm of a positive normal number: y = 2^e m, sqrt(1/2) <= m < sqrt(2),
// ln m = 2 artanh(s), s = (m - 1) / (m + 1), by its series (s^2 < 0.0295; the term left out is
// below 1e-18).
__device__ __forceinline__ double log_pos(double y) {
  double m = __builtin_amdgcn_frexp_mant(y);
  int e = __builtin_amdgcn_frexp_exp(y);
  if (m < 0.70710678118654752) {
    m *= 2.0;
    e -= 1;
  }
  const double s = quot(m - 1.0, m + 1.0), z = s * s;
  double t = 1.0 / 23.0;
  t = fma(t, z, 1.0 / 21.0);
  t = fma(t, z, 1.0 / 19.0);
  t = fma(t, z, 1.0 / 17.0);
  t = fma(t, z, 1.0 / 15.0);
  t = fma(t, z, 1.0 / 13.0);
  t = fma(t, z, 1.0 / 11.0);
  t = fma(t, z, 1.0 / 9.0);
  t = fma(t, z, 1.0 / 7.0);
  t = fma(t, z, 1.0 / 5.0);
  t = fma(t, z, 1.0 / 3.0);
  return fma((double)e, kLn2Hi, fma((double)e, kLn2Lo, 2.0 * fma(s * z, t, s)));
}

// V'_fy+ = 0.005 y^2 / (1 + 0.002923 y^2.128); y^2.128 = y^2 y^0.128: the small exponent keeps the
// logarithm's rounding out of the result (and is the exact difference 2.128 - 2 of the constants).
__device__ __forceinline__ double rms_fluid_plus(double y) {
  const double y2 = y * y;
  double two_k;
  const double p = exp_split((2.128 - 2.0) * log_pos(y), two_k);
  return quot(0.005 * y2, fma(0.002923 * y2, fma(two_k, p, two_k), 1.0));
}

// Positive root V of V^2 / 2 + a V = w, 0 for w <= 0.  The hardware's FP32 reciprocal root
// and reciprocal give V and the slope's inverse 1 / (V + a) = 1 / sqrt(a^2 + 2 w) to about 2^-21; two
// Newton steps in FP64 take V to its last digit: a shorter chain than an FP64 root and quotient.
// For a >= 0: sqrt(a^2 + 2 w) + a cancels otherwise, and FP32 may keep no digit of it.
// far: set where FP32's range does not hold the operands (the caller then takes speed_far).
__device__ __forceinline__ double speed(double a, double w, bool &far) {
  w = fmax(w, 0.0);
  const float af = (float)a, wf = (float)w;
  const float qf = fmaf(af, af, 2.0f * wf);
  far |= !(qf > 1e-30f && qf < 1e30f) || (w > 0.0 && wf < 1e-30f);
  const float y = __builtin_amdgcn_rsqf(qf);
  double V = (double)(2.0f * wf * __builtin_amdgcn_rcpf(fmaf(qf, y, af)));
  const double yd = (double)y;
  V = fma(fma(-V, fma(0.5, V, a), w), yd, V);
  return fma(fma(-V, fma(0.5, V, a), w), yd, V);
}
__device__ __forceinline__ double speed_far(double a, double w) {
  return w > 0.0 ? 2.0 * w / (a + sqrt(fma(a, a, 2.0 * w))) : 0.0;
}

constexpr int kLfThreads = 512;
constexpr int kLfPar = kLfThreads - 64;        // threads of the node waves; the last wave runs the chains

// C classes (a power of two, at most 64) per workgroup, n_wall + n_core nodes from the wall (0) to
// the centre; cell c spans the nodes nn - 1 - c (up) and nn - 2 - c (lo), NC cells per chunk.
// In interval t (between two barriers) the node waves take chunk t's nodes, chunk t - 1's cells
// (differences of neighbouring nodes) and chunk t - 3's flux exponentials, the chain wave chunk
// t - 2's speeds and chunk t - 4's flux coefficients: every array below is written one interval
// before it is read, into the half its reader does not hold.
template <int C>
__global__ void __launch_bounds__(kLfThreads) __attribute__((amdgpu_waves_per_eu(C > 16 ? 4 : 2)))
k_lf(LfConst c, int64_t n, const double *__restrict__ d_diam, const double *__restrict__ d_q,
     const double *__restrict__ d_A, double *__restrict__ out) {
  constexpr int NC = kLfPar / C, S = NC * C;   // cells per chunk, cell slots (cell x class)
  constexpr int NB = 7;                        // cells per register block of the chains
  static_assert(NC % NB == 0, "whole register blocks");
  __shared__ double gap[2][S], igap[2][S];     // class-independent part of the next S nodes
  __shared__ double phi[2][S], pot[2][S], last_phi[3][C], last_pot[3][C];
  __shared__ double cw[2][S], ca[2][S];        // per cell: work, h / tau
  __shared__ double cv[2][S + C];              // speeds at the cells' lo nodes; row NC: at the chunk's first up node
  __shared__ double ce[2][S], cf[2][S];        // flux over the cell: e^-x and (1 - e^-x) / V
  const bool chain = threadIdx.x >= kLfPar;    // wave-uniform
  const int id = chain ? (int)threadIdx.x - kLfPar : (int)threadIdx.x;
  const int cl = id % C, slot = id / C;
  const int64_t i = (int64_t)blockIdx.x * C + cl;
  const bool has = i < n;
  const double d = has ? d_diam[i] : 1e-6, q = has ? d_q[i] : 0.0, A = has ? d_A[i] : 0.0;
  const double us = c.re_tau * c.nu / c.R;
  const double lw = c.nu / us;
  const double taup_plus = c.rho_p * d * d / (18.0 * c.rho_f * c.nu) * us * us / c.nu;
  const double m = c.rho_p * M_PI * d * d * d / 6.0;
  const double rr = 1.0 / (1.0 + taup_plus / kTauLPlus);
  const double yw = 0.5 * d / lw;
  const int nw = c.n_wall, nn = c.n_wall + c.n_core;
  const int cells = nn - 1, chunks = (cells + NC - 1) / NC;

  if (!chain) {
    const double db_plus = kBoltzmann * kTempLF / (3.0 * M_PI * c.rho_f * c.nu * c.nu * d);
    const double inv_us2 = 1.0 / (us * us);
    const double e_img = q * q / (16.0 * M_PI * c.eps0 * m) * inv_us2;  // image potential times y
    const double c_vdw = A * d / (12.0 * m) * inv_us2;                  // wall cohesion potential times gap
    const double lg0 = log(kGapMin / lw);
    const double gap_c = c.R / lw - yw, core_step = (gap_c - 1.0) / c.n_core;
    const bool act = slot < NC;                // kLfPar need not be a multiple of C
    // lo nodes of the S cells from cell c0 on: gap in wall units and 1 / gap near the wall, the number
    // of core steps beyond
    auto fill = [&](int c0, double *g_, double *ig_) {
      if (!act) return;
      const int k = nn - 2 - (c0 + id);
      double g, ig = 0.0;
      if (k <= 0) {
        g = kGapMin / lw;
      } else if (k < nw - 1) {
        double two_k;
        const double p = exp_split(lg0 * (1.0 - (double)k / (double)(nw - 1)), two_k);
        g = fma(two_k, p, two_k);
      } else {
        g = k == nw - 1 ? 1.0 : (double)(k - nw + 1);
      }
      if (k < nw) ig = 1.0 / (g * lw);
      g_[id] = g;
      ig_[id] = ig;
    };
    auto node = [&](int k, double g, double ig, double &y, double &f, double &u) {
      if (k >= nw) {
        g = k == nn - 1 ? gap_c : 1.0 + g * core_step;
        ig = quot(1.0, g * lw);
      }
      y = yw + g;
      const double v = rms_fluid_plus(y);
      f = rr * v * v;
      u = e_img * quot(1.0, y * lw) + c_vdw * ig;
    };
    fill(0, gap[0], igap[0]);
    if (slot == 0) {                           // the centre node
      double y, f, u;
      node(nn - 1, 0.0, 0.0, y, f, u);
      last_phi[2][cl] = f;
      last_pot[2][cl] = u;
    }
    __syncthreads();
    // own node of the chunk taken last, and h / D of the cells of the two chunks before it
    double y0 = 0.0, f0 = 0.0, u0 = 0.0, hd1 = 0.0, hd2 = 0.0;
    double yu = 0.0;                           // y of the own cell's up node
    for (int t = 0; t < chunks + 4; ++t) {
      if ((t + 1) % C == 0) fill((t + 1) * NC, gap[((t + 1) / C) & 1], igap[((t + 1) / C) & 1]);
      // chunk t - 3: flux over the cell: rho_up = rho_lo e^-x + J (h / Dm) (1 - e^-x) / x, x = Vm h / Dm; inverted
      if (act && t >= 3) {
        double e = 1.0, f = 0.0;               // beyond the last cell: nothing
        if ((t - 3) * NC + slot < cells) {
          const double *v = cv[(t - 3) & 1];
          const double vm = 0.5 * (v[(slot ? slot - 1 : NC) * C + cl] + v[slot * C + cl]);
          const double x = vm * hd2;
          f = hd2;
          if (x > 0.0) {
            double two_k;
            const double p = exp_split(-x, two_k);
            e = fma(two_k, p, two_k);
            f = -quot(fma(two_k, p, two_k - 1.0), vm);
          }
        }
        ce[(t - 3) & 1][id] = e;
        cf[(t - 3) & 1][id] = f;
      }
      hd2 = hd1;
      // chunk t - 1: the momentum's driving term and drag over the cell, and h / D
      if (act && t >= 1 && (t - 1) * NC + slot < cells) {
        const double fu = slot ? phi[(t - 1) & 1][id - C] : last_phi[(t + 1) % 3][cl];
        const double uu = slot ? pot[(t - 1) & 1][id - C] : last_pot[(t + 1) % 3][cl];
        const double h = yu - y0;
        cw[(t - 1) & 1][id] = (fu - f0) + (u0 - uu);
        ca[(t - 1) & 1][id] = quot(h, taup_plus);
        hd1 = quot(h, db_plus + kTauLPlus * (0.5 * (fu + f0)));   // D / nu = db + tau_L Phi at both ends
      }
      // chunk t: the lo node
      if (act && t * NC + slot < cells) {
        const int k = nn - 2 - (t * NC + slot), e = (t % C) * NC + slot, tb = (t / C) & 1;
        node(k, gap[tb][e], igap[tb][e], y0, f0, u0);
        phi[t & 1][id] = f0;
        pot[t & 1][id] = u0;
        if (slot == NC - 1) {
          last_phi[t % 3][cl] = f0;
          last_pot[t % 3][cl] = u0;
        }
        // the up node's y: the table's entry before, or (the table's first entry) from its own formula
        const int ku = k + 1;
        double gu;
        if (ku >= nw) {
          gu = ku == nn - 1 ? gap_c : 1.0 + (double)(ku - nw + 1) * core_step;
        } else if (e > 0) {
          gu = gap[tb][e - 1];
        } else {
          gu = gap[tb ^ 1][S - 1];
        }
        yu = yw + gu;
      }
      __syncthreads();
    }
    return;
  }

  // the chain wave: issues ahead of the node waves that share its SIMD
  __builtin_amdgcn_s_setprio(3);
  const bool lane = id < C;
  // A pipe of less than a wall unit beyond the particle makes the core's cells run backwards (a < 0), a wall
  // unit below the smallest gap the wall's: such a class takes speed_far throughout.
  const bool back = !(c.R / lw - yw > 1.001) || !(kGapMin < lw);
  double V = 0.0, Vwall = 0.0;   // speed toward the wall at the last node; at the wall
  double s = 1.0, b = 0.0;       // flux coefficients at the last node
  __syncthreads();
  for (int t = 0; t < chunks + 4; ++t) {
    if (lane) {
      // chunk t - 2: K_lo = K_up + (Phi_up - Phi_lo) + work - h V_lo / tau_1, drag implicit, and beside it
      // chunk t - 4's flux coefficients.  NB cells at a time from registers, each reloaded for the
      // next block as soon as it is used, so that no step of the chain waits for the LDS.  Cells
      // beyond the last one (and the chunks before 0 and after the last) are computed and not used.
      const double *w_ = cw[t & 1], *a_ = ca[t & 1], *e_ = ce[t & 1], *f_ = cf[t & 1];
      double *v_ = cv[t & 1];
      const int left = cells - 1 - (t - 2) * NC;   // the chunk's cell at the wall
      const bool flux = t >= 4;
      if (t <= 2) V = 0.0;         // at the centre
      v_[S + cl] = V;
      double w[NB], a[NB], e[NB], f[NB], v[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        w[k] = w_[k * C + cl];
        a[k] = a_[k * C + cl];
        e[k] = e_[k * C + cl];
        f[k] = f_[k * C + cl];
      }
      for (int k0 = 0; k0 < NC; k0 += NB) {
        const int kn = k0 + NB < NC ? k0 + NB : 0;
        bool far = back;
        const double K0 = 0.5 * V * V;
        double K = K0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
          v[k] = speed(a[k], K + w[k], far);
          K = 0.5 * v[k] * v[k];
          if (flux) {
            b = fma(-f[k], s, b);
            s *= e[k];
          }
          w[k] = w_[(kn + k) * C + cl];
          a[k] = a_[(kn + k) * C + cl];
          e[k] = e_[(kn + k) * C + cl];
          f[k] = f_[(kn + k) * C + cl];
        }
        if (far) {
          K = K0;
          for (int k = 0; k < NB; ++k) {
            const double x = speed_far(a_[(k0 + k) * C + cl], K + w_[(k0 + k) * C + cl]);
            v_[(k0 + k) * C + cl] = x;
            K = 0.5 * x * x;
          }
#pragma unroll
          for (int k = 0; k < NB; ++k) v[k] = v_[(k0 + k) * C + cl];
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
          v_[(k0 + k) * C + cl] = v[k];
          if (k0 + k == left) Vwall = v[k];
        }
        V = v[NB - 1];
      }
    }
    __syncthreads();
  }
  if (!lane || !has) return;
  if (!(d > 0.0) || !isfinite(d) || !isfinite(q) || !isfinite(A)) {
    out[i] = NAN;
    return;
  }
  // kinetic wall condition: flux of a half-Maxwellian with mean V_w and rms vp; the wall is node 0
  const double vfw = rms_fluid_plus(yw + kGapMin / lw);
  const double vp = sqrt(rr * vfw * vfw + kBoltzmann * kTempLF / (m * us * us));
  const double M = Vwall / (M_SQRT2 * vp);
  const double hw = vp * exp(-M * M) / sqrt(2.0 * M_PI) + Vwall * (1.0 + erf(M)) * 0.5;
  out[i] = hw / (s - hw * b);
}

}  // namespace

void launch_lf(const LfConst &c, int64_t n, const double *d, const double *q, const double *A, double *out,
               hipStream_t s) {
  if (n <= 0) return;
  // The fewer classes a workgroup takes, the more of the chip a small call uses, until there are more
  // workgroups than CUs: 16 up to 4,096 classes (a workgroup per CU; 172 us at 3,000 classes x 1,600
  // nodes, 213 with 32, 279 with 64), 32 up to 8,192 (225 us at 8,000; 333 with 16, 278 with 64), then
  // 64, where the node waves' lanes all share a node and the chains' wave is full (460 us at 25,920;
  // 572 with 32).
  auto go = [&](auto kernel, int C) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + C - 1) / C)), dim3(kLfThreads), 0, s, c, n, d, q, A, out);
  };
  if (n <= 4096)
    go(k_lf<16>, 16);
  else if (n <= 8192)
    go(k_lf<32>, 32);
  else
    go(k_lf<64>, 64);
}

}  // namespace depo
