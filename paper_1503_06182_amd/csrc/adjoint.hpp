// adjoint.hpp -- hand-written adjoint of the Drell-Yan VEGAS estimator with
// respect to theta = (M_Z, Gamma_Z, sin^2 theta_W, PDF exponent a, PDF exponent b).
//
// sigma(theta) = (1/N) sum_i w_i(theta) at a fixed grid and a fixed random stream
// (common random numbers for every parameter point).  The proposal -- grid map,
// Breit-Wigner and tau mappings -- stays at the nominal parameters of the handle,
// so only |M|^2 and the PDFs carry theta, and the pathwise gradient of the
// estimator is (1/N) sum_i dw_i/dtheta.
//
// |M|^2 summed over flavours and helicities is, with s = m_ll^2, d = s - M_Z^2 and
// D = d^2 + (M_Z G_Z)^2, proportional to c0 + (c1 s d + c2 s^2) / D, where c0 = 4 sum (Q_q
// Q_l)^2 and c1, c2 are sums of the couplings of the point alone.  So the reverse sweep of
// an event needs no sweep over the eight amplitudes: with K the theta-independent weight,
// E = exp(a ln tau + b ln((1-x1)(1-x2))) and v = K E s / D, a point accumulates
//   w = c0 K E + v (c1 d + c2 s),  v,  v d,  v s,  q = v (c1 d + c2 s) / D,  q d,
//   w ln tau,  w ln((1-x1)(1-x2)),
// and its derivatives are combinations of these sums with the point's constants, formed
// once per row.
//
// Work split: one wave owns a row of consecutive 64-event tiles (rows from the number of
// events alone).  Phase 1, lane = event: K, s and the two logarithms go to LDS.  Phase 2,
// lane = (event group, parameter point): with B points the wave holds floor(64 / B)
// groups, and group g takes events g, g + G, ... of the tile in order.  The groups' sums
// are added in group order, the rows by a fixed tree, so the result does not depend on
// the launch.
//
// Bound: FP64 VALU issue, 46 instructions per (event, point) instead of the 208 of a sweep
// over the amplitudes with the library's exp: 64 points x 1e6 events 445 -> 136 us a call.
// Few points: with one event at a time 9 of 64 lanes worked for 9 points; the groups take
// the kernel from 61 to 12 us at 9 points x 1e5 events.
#pragma once
#include <hip/hip_runtime.h>

#include "device_common.hpp"
#include "integrands.hpp"

namespace vg {

constexpr int kGradMaxPoints = 64;
constexpr int kGradVals = 6;  // w, dw/dMZ, dw/dGZ, dw/dsw2, dw/da, dw/db
constexpr int kTreeRows = 256;

// tiles per row of partials: at most 4096 rows, one for each wave of a full GPU (four waves
// per SIMD on 256 CUs), as long as the tiles allow: one tile a row writes 48 MB of partials
// for 64 points x 1e6 events, and each wave pays the couplings of its point once per row.
// A function of the number of events alone.
constexpr int64_t kGradRows = 4096;
// A lane's sums are set aside every kGradStretch events of the lane, so that the chains of
// additions do not grow with the row: at most kGradStretch events, then one addition per
// stretch (2048 of them at the largest call, 2^31 - 1 events and 64 points, where a row has
// 8192 tiles and a lane would add 524,288 events one by one; 1e8 events 10.35 ms either way)
constexpr int kGradStretch = 256;
inline int64_t grad_tiles_per_row(int64_t ntiles) { return (ntiles + kGradRows - 1) / kGradRows; }

struct GradArgs {
  PhysConst pc;          // nominal constants of the handle (mappings)
  const double* edges;   // grid [3][nbins+1]
  const double* theta;   // [B][5]
  double* rows_out;      // [nrows][6][B]
  uint64_t seed;
  int64_t nev;
  int64_t ntiles, nrows, tiles_per_row;
  uint32_t iter;
  int nbins, B;
  double e4_12;          // e^4 / 12 (alpha fixed)
};

// a b + c with c in a scalar register pair as the instruction's operand (left to itself the
// compiler copies each coefficient into the accumulating form's destination first)
__device__ __forceinline__ double fma_coef(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// exp(t) for |t| up to about 1e9 (0 and inf where it leaves the range), exp_fin's polynomial in
// the form that suits this loop (k rounded and converted, the additions by fma_coef).  No
// branches; NaN stays NaN
__device__ __forceinline__ double exp_core(double t) {
  const double k = rint(t * 1.4426950408889634);
  const double r = __fma_rn(-k, kLn2Lo, __fma_rn(-k, kLn2, t));
  double q = fma_coef(kExpQ[9], r, kExpQ[8]);
  q = fma_coef(q, r, kExpQ[7]);
  q = fma_coef(q, r, kExpQ[6]);
  q = fma_coef(q, r, kExpQ[5]);
  q = fma_coef(q, r, kExpQ[4]);
  q = fma_coef(q, r, kExpQ[3]);
  q = fma_coef(q, r, kExpQ[2]);
  q = fma_coef(q, r, kExpQ[1]);
  q = fma_coef(q, r, kExpQ[0]);
  return ldexp(__fma_rn(r * r, q, r) + 1.0, static_cast<int>(k));
}

// Z couplings g_L = (T3 - Q x)/sqrt(x(1-x)), g_R = -Q sqrt(x/(1-x)), x = sin^2 theta_W,
// and their derivatives in x
__device__ __forceinline__ void zcoup(double T3, double Q, double x, double& gL, double& gR, double& dgL,
                                      double& dgR) {
  const double sc = sqrt(x * (1.0 - x));
  gL = (T3 - Q * x) / sc;
  gR = -Q * sqrt(x / (1.0 - x));
  dgL = -Q / sc - (T3 - Q * x) * (1.0 - 2.0 * x) / (2.0 * sc * x * (1.0 - x));
  dgR = -Q / (2.0 * sqrt(x) * (1.0 - x) * sqrt(1.0 - x));
}

// phase 2 of one tile: lane's events e = g, g + G, ... (row 64 is a row of weight 0)
template <bool FAST>
__device__ __forceinline__ void grad_points(const double* ev, int g, int G, double M2, double MG2, double pa, double pb,
                                            double c0, double c1, double c2, double S[8]) {
  for (int e0 = 0; e0 < 64; e0 += G) {
    const double* r = ev + 4 * (e0 + g < 64 ? e0 + g : 64);
    const double K = r[0], s = r[1], ls = r[2], Ls = r[3];
    const double t = __fma_rn(pa, ls, pb * Ls);
    const double KE = K * (FAST ? exp_core(t) : exp(t));
    const double d = s - M2, iD = rcp_nr(__fma_rn(d, d, MG2));
    const double v = KE * iD * s, f = __fma_rn(c1, d, c2 * s);
    const double vf = v * f, w = __fma_rn(c0, KE, vf), q = vf * iD;
    S[0] += w;
    S[1] += v;
    S[2] = __fma_rn(v, d, S[2]);
    S[3] = __fma_rn(v, s, S[3]);
    S[4] += q;
    S[5] = __fma_rn(q, d, S[5]);
    S[6] = __fma_rn(w, ls, S[6]);
    S[7] = __fma_rn(w, Ls, S[7]);
  }
}

constexpr int kGradSums = 8;
constexpr int kGradLds = 65 * 4 + kGradSums * 64;  // doubles of LDS per wave: the tile's rows, the groups' sums

__global__ __launch_bounds__(256, 4) void k_dy_grad(GradArgs a) {
  extern __shared__ double sm[];
  const int n = a.nbins;
  double* e_lds = sm;                                    // [3][n+1]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  double* ev = sm + 3 * (n + 1) + wave * kGradLds;       // [65][4]
  double* gs = ev + 65 * 4;                              // [8][64]: stretches, then groups
  for (int i = threadIdx.x; i < 3 * (n + 1); i += blockDim.x) e_lds[i] = a.edges[i];
  if (lane < 4) ev[64 * 4 + lane] = lane == 1 ? -1.0 : 0.0;

  // this lane's group and parameter point: couplings and their sw2-derivatives
  const int G = 64 / a.B, g = lane / a.B, b = lane - g * a.B;
  const bool mine = g < G;
  const double* th = a.theta + 5 * (mine ? b : 0);
  const double M = th[0], GZ = th[1], x = th[2], pa = th[3], pb = th[4];
  // exp_core's range: ln tau and the clamped logarithm are at most 1e4 in size
  const bool fast = __all(fabs(pa) <= 1e4 && fabs(pb) <= 1e4);
  double c0 = 0.0, c1 = 0.0, c2 = 0.0, dc1 = 0.0, dc2 = 0.0;
  {
    double lL, lR, dlL, dlR;
    zcoup(-0.5, -1.0, x, lL, lR, dlL, dlR);
    const double gl[2] = {lL, lR}, dgl[2] = {dlL, dlR};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const double qql = q == 0 ? -2.0 / 3.0 : 1.0 / 3.0;  // Q_q Q_l, Q_l = -1
      double qL, qR, dqL, dqR;
      zcoup(q == 0 ? 0.5 : -0.5, q == 0 ? 2.0 / 3.0 : -1.0 / 3.0, x, qL, qR, dqL, dqR);
      const double gq[2] = {qL, qR}, dgq[2] = {dqL, dqR};
      c0 += 4.0 * qql * qql;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int hp = 0; hp < 2; ++hp) {
          const double gg = gq[h] * gl[hp], dgg = dgq[h] * gl[hp] + gq[h] * dgl[hp];
          c1 += 2.0 * qql * gg;
          dc1 += 2.0 * qql * dgg;
          c2 += gg * gg;
          dc2 += 2.0 * gg * dgg;
        }
    }
  }
  const double M2 = M * M, MG2 = (M * GZ) * (M * GZ);
  const double kc = a.pc.conv * a.pc.pdfA * a.pc.pdfA * a.e4_12;
  __syncthreads();

  for (int64_t row = static_cast<int64_t>(blockIdx.x) * wpb + wave; row < a.nrows;
       row += static_cast<int64_t>(gridDim.x) * wpb) {
    const int64_t t1 = min(a.ntiles, (row + 1) * a.tiles_per_row);
    double S[kGradSums] = {0, 0, 0, 0, 0, 0, 0, 0};
    bool aside = false;  // gs holds the sums of the stretches before
    int left = kGradStretch / 64 * G;  // tiles, of ceil(64 / G) events per lane each
    for (int64_t tile = row * a.tiles_per_row; tile < t1; ++tile) {
      if (--left < 0) {
#pragma unroll
        for (int k = 0; k < kGradSums; ++k) {
          double* const q = gs + k * 64 + lane;
          *q = aside ? *q + S[k] : S[k];
          S[k] = 0.0;
        }
        aside = true;
        left += kGradStretch / 64 * G;
      }
      // wave priorities: phase 1 (uniforms, grid map, kinematics) at the base priority,
      // phase 2 (the parameter points' sums) raised, so that the waves of a SIMD drift
      // apart in phase
      __builtin_amdgcn_s_setprio(0);
      // ---- phase 1: lane = event, theta-independent part at the nominal proposal
      const int64_t i = tile * 64 + lane;
      double K = 0.0, m2 = -1.0, ls = 0.0, Ls = 0.0;
      if (i < a.nev) {
        double u[3], xx[3];
        event_uniforms<3>(a.seed, a.iter, static_cast<uint64_t>(i), 3, u);
        double J = 1.0;
        {
#pragma clang fp contract(off)
          const double dn = static_cast<double>(n);
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            const double t = u[d] * dn;
            int k = static_cast<int>(t);
            k = k > n - 1 ? n - 1 : k;
            const double delta = t - static_cast<double>(k);
            const double* e = e_lds + d * (n + 1);
            const double h = e[k + 1] - e[k];
            xx[d] = __fma_rn(delta, h, e[k]);
            J *= dn * h;
          }
        }
        const double s = bw_mass(a.pc, xx[0], a.pc.rho_rng), dm = s - a.pc.M2;
        const double jbw = a.pc.rho_rng * __fma_rn(dm, dm, a.pc.MG2) * a.pc.invMG;
        double L, l1, l2;
        {
#pragma clang fp contract(off)
          L = log_pos(s * a.pc.invS);
          l1 = xx[1] * L;
          l2 = L - l1;
        }
        const double jtau = -L * a.pc.invS;
        const double cs = 2.0 * xx[2] - 1.0;
        // conv J_grid J_bw J_tau 2 / (2 s) / (16 pi) times e^4 / 12 s^2 2 (1 + cos^2) / s^2
        K = kc * J * jbw * jtau * (2.0 * rcp_nr(s)) * (1.0 / (16.0 * kPi)) * (1.0 + cs * cs);
        if (K != 0.0) {
          m2 = s;
          ls = L;
          const double P = expm1_fin(l1) * expm1_fin(l2);
          Ls = P > 0.0 ? log_pos(P) : -1e4;
        }
      }
      ev[lane * 4 + 0] = K;
      ev[lane * 4 + 1] = m2;
      ev[lane * 4 + 2] = ls;
      ev[lane * 4 + 3] = Ls;
      // the wave reads what its own lanes wrote (LDS operations of a wave are in order)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_s_setprio(3);
      // ---- phase 2: lane = (event group, parameter point)
      if (fast) grad_points<true>(ev, mine ? g : 0, G, M2, MG2, pa, pb, c0, c1, c2, S);
      else grad_points<false>(ev, mine ? g : 0, G, M2, MG2, pa, pb, c0, c1, c2, S);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (aside)
#pragma unroll
      for (int k = 0; k < kGradSums; ++k) S[k] += gs[k * 64 + lane];
    // the groups' sums in group order
    if (G > 1) {
#pragma unroll
      for (int k = 0; k < kGradSums; ++k) gs[k * 64 + lane] = S[k];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (lane < a.B)
        for (int gg = 1; gg < G; ++gg)
#pragma unroll
          for (int k = 0; k < kGradSums; ++k) S[k] += gs[k * 64 + gg * a.B + lane];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (lane < a.B) {
      double* o = a.rows_out + row * kGradVals * a.B + lane;
      o[0] = S[0];
      o[a.B] = -2.0 * M * (c1 * S[1] + GZ * GZ * S[4] - 2.0 * S[5]);
      o[2 * a.B] = -2.0 * M2 * GZ * S[4];
      o[3 * a.B] = dc1 * S[2] + dc2 * S[3];
      o[4 * a.B] = S[6];
      o[5 * a.B] = S[7];
    }
  }
}

// one level of the fixed tree: rows [256 c, 256 c + 256) of every column -> row c
// (stride-halving pairwise sums over a zero-padded chunk; blockDim must be 256).
// Block (c, y) stages the chunk's rows of 16 columns at a time in LDS -- each row's
// 16 doubles are one contiguous 128-byte load -- and then adds, per column, exactly
// the pairs the stride-halving order prescribes.
constexpr int kTreeCols = 16;
__global__ __launch_bounds__(256) void k_tree_level(const double* in, double* out, int64_t rows, int cols) {
  __shared__ double s[kTreeRows][kTreeCols + 1];  // +1: the column sums read across rows
  const int64_t chunk = blockIdx.x;
  const int tid = threadIdx.x, cc = tid % kTreeCols, rr = tid / kTreeCols;
  for (int c0 = blockIdx.y * kTreeCols; c0 < cols; c0 += gridDim.y * kTreeCols) {
    const int c = c0 + cc;
#pragma unroll 4
    for (int r = rr; r < kTreeRows; r += kTreeRows / kTreeCols) {
      const int64_t row = chunk * kTreeRows + r;
      s[r][cc] = row < rows && c < cols ? in[row * cols + c] : 0.0;
    }
    __syncthreads();
    for (int stride = kTreeRows / 2; stride > 0; stride >>= 1) {
      for (int i = tid; i < stride * kTreeCols; i += kTreeRows) {
        const int r = i / kTreeCols, q = i % kTreeCols;
        s[r][q] += s[r + stride][q];
      }
      __syncthreads();
    }
    if (tid < kTreeCols && c0 + tid < cols) out[chunk * cols + c0 + tid] = s[0][tid];
    __syncthreads();
  }
}

// the tree's last rows (at most kGradLast) added in order -> sigma[B], dsigma[B][5]
constexpr int kGradLast = 16;
__global__ __launch_bounds__(384) void k_grad_out(const double* in, int64_t rows, int B, int64_t nev, double* sigma,
                                                  double* dsigma) {
  const int c = threadIdx.x, cols = kGradVals * B;
  if (c >= cols) return;
  double v[kGradLast], t = 0.0;
#pragma unroll
  for (int r = 0; r < kGradLast; ++r) v[r] = r < rows ? in[r * cols + c] : 0.0;
#pragma unroll
  for (int r = 0; r < kGradLast; ++r) t += v[r];
  t *= 1.0 / static_cast<double>(nev);
  const int k = c / B, b = c - k * B;
  if (k == 0) sigma[b] = t;
  else dsigma[5 * b + k - 1] = t;
}

}  // namespace vg
