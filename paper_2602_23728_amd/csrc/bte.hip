// Full scattering matrix of the linearised BTE and its two solutions
// (paper: "Boltzmann Transport Equation": Eq. BTE, Eq. gamma1, Eq. invBTE,
// Eq. kappa_general, Eq. sc_iter, Eq. inverse).
//
// Rows of Gamma~ = diag(Gamma0) + Gamma1, one per mode mu = (q, s).  For each
// ordered candidate (q s; q1 s'; q2 s''), q + q1 + q2 = G, passing the 2-sigma
// cut of the linewidths, with the coalescence and decay rates
//   d+ = 2 P |V|^2 (n1 - n2) g(x+) / (w w1 w2),
//   d- = 2 P |V|^2 1/2 (n1 + n2 + 1) g(x-) / (w w1 w2),   P = pi hbar U^3/(8 N_q),
// row mu receives Gamma0 += d+ + d- (= 2 Gamma of Eq. gamma), and
//   column (q1, s')       +d+ w1/w          (absorbed partner)
//   column tr(q1, s')     -d- w1/w          (emitted partner of the decay)
//   column tr(q2, s'')    -(d+ + d-) w2/w   (emitted partner of both)
// tr(q', s') is the time-reversal partner of a mode: the mode at -q' whose
// eigenvector overlaps eta(q', s')* most (the vertex holds eta(q2); the
// emitted phonon is the mode at -q2 with the conjugate eigenvector).  These
// rows make Eq. sc_iter the iterative scheme of the adaptive-smearing
// reference the paper cites.  Modes without RTA conductivity (nu < nu_min,
// Gamma0 <= 1e-8 max Gamma0) are decoupled: zero row and column, unit
// diagonal, zero right-hand side.
//
// Kernels:
//   bte_tr_map     time-reversal partner of every mode (largest overlap)
//   bte_zero       clears the n x n matrix
//   bte_rows<NB3>  one workgroup per q, three waves each over a third of
//                  the branches of q: A~_q (FP64, LDS, by atom block), then
//                  the partners q1 in rounds of 64 (one per lane): an FP32
//                  test against the widest cut, the near pairs queued in LDS
//                  for the exact FP64 cut, the passing ones for their vertices
//                  (64 lanes each), sums per column kind and partner in LDS,
//                  written in three passes whose columns are a bijection of q1
//                  (no two lanes of a pass touch one element), Gamma0 reduced
//                  in a fixed order and added to the diagonal.  Latency of few
//                  waves bounds it (the sums leave two workgroups a CU);
//                  diamond 15^3: 18.3 ms with the exact cut of every pair in
//                  every lane and each term taken back by its own lane in
//                  turn, now 5.7
//   bte_gmax, bte_flags, bte_decouple   the RTA selection
//   bte_compact_index, bte_compact_cols, bte_gather3, bte_scatter3   the
//                  solve's restriction to the coupled modes (row map, coupled
//                  columns moved to the front of each coupled row)
//   lu_left, lu_panels, lu_gemm   blocked LU without pivoting of
//                  the coupled block (64 x 64 blocks, panels of eight; the
//                  panels and updates on the FP64 matrix cores)
//   lu_solve<FORWARD>, lu_solve_rest   the two triangular sweeps for the 3 RHS, panel by panel
//   bte_gemv, bte_sc_init, bte_sc_update   the iteration of Eq. sc_iter
//   bte_kappa      Eq. kappa_general, fixed-order reduction
// Every reduction and every sequence of additions into one matrix element
// runs in a fixed order: results are bitwise reproducible.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "lw_common.h"

namespace kaldo {

constexpr int kLuB = 64;     // LU block edge
constexpr int kLuPanel = 8;  // blocks per panel of the blocked LU

typedef __attribute__((__vector_size__(4 * sizeof(double)))) double d4;
typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// ------------------------------------------------------------------ tables

__global__ void bte_tr_map(int nq, int nb3, int N0, int N1, int N2,
                           const double* __restrict__ evec, int32_t* __restrict__ tr) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nq * nb3) return;
  const int q = m / nb3, s = m - q * nb3;
  const int a0 = q / (N1 * N2), a1 = (q / N2) % N1, a2 = q % N2;
  const int mq = (((N0 - a0) % N0) * N1 + (N1 - a1) % N1) * N2 + (N2 - a2) % N2;
  const double* x = evec + (size_t)q * nb3 * nb3 * 2;
  const double* y = evec + (size_t)mq * nb3 * nb3 * 2;
  int best = 0;
  double bo = -1.0;
  for (int t = 0; t < nb3; ++t) {
    double re = 0.0, im = 0.0;
    for (int i = 0; i < nb3; ++i) {
      const double xr = x[(i * nb3 + s) * 2], xi = x[(i * nb3 + s) * 2 + 1];
      const double yr = y[(i * nb3 + t) * 2], yi = y[(i * nb3 + t) * 2 + 1];
      re += yr * xr - yi * xi;  // eta_i(-q, t) eta_i(q, s), no conjugate
      im += yr * xi + yi * xr;
    }
    const double o = re * re + im * im;
    if (o > bo) {
      bo = o;
      best = t;
    }
  }
  tr[m] = mq * nb3 + best;
}

__global__ void bte_zero(size_t n, double* __restrict__ x) {
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (size_t)gridDim.x * blockDim.x)
    x[k] = 0.0;
}

// Per-process rates of one candidate without |V|^2 and the prefactor:
// dp = (n1 - n2) g(x+) / (w w1 w2), dm = 1/2 (n1 + n2 + 1) g(x-) / (w w1 w2),
// each 0 unless its own |x| < 2 sigma.
__device__ __forceinline__ void process_rates(const LwParams& p, double w, double w1, double w2,
                                              double n1, double n2, double sp, double sm,
                                              double& dp, double& dm) {
  const double xp = (w + w1) - w2, xm = (w - w1) - w2;
  const double den = w * (w1 * w2);
  dp = fabs(xp) < 2.0 * sp ? (n1 - n2) * smear(p.shape, xp, sp) / den : 0.0;
  dm = fabs(xm) < 2.0 * sm ? 0.5 * (n1 + n2 + 1.0) * smear(p.shape, xm, sm) / den : 0.0;
}

// ------------------------------------------------------------------ rows

constexpr int kRowWaves = 3;    // waves per row workgroup, each over a third of the branches s
constexpr int kRowQueue = 128;  // slots of a wave's two queues, which are worked off 64 at a time

template <int NB3>
__global__ __launch_bounds__(64 * kRowWaves) void bte_rows(
    LwParams p, int n_rep, const int32_t* __restrict__ rep, const double* __restrict__ omega,
    const double* __restrict__ vel, const double* __restrict__ occ,
    const uint8_t* __restrict__ phys, const double* __restrict__ evec,
    const float2* __restrict__ near_tab, const double2* __restrict__ phase_tab, int n_blk, const int32_t* __restrict__ e_blk,
    const int32_t* __restrict__ e_bg, const int32_t* __restrict__ blk_d,
    const int32_t* __restrict__ pair_ptr, const int32_t* __restrict__ t_ptr,
    const int32_t* __restrict__ t_i, const int32_t* __restrict__ t_l2,
    const double* __restrict__ t_coef, const int32_t* __restrict__ tr, double pref,
    double* __restrict__ mat, double* __restrict__ gamma0) {
  // [n_blk][9][NB3]: A~_q by atom block (jb, kb, d) and Cartesian pair
  // (beta, gamma), phases e^{+i q.R''} folded in
  extern __shared__ double2 at[];
  constexpr int NB = NB3 / 3;
  static_assert(NB3 % kRowWaves == 0, "the branches of q split evenly over the waves");
  constexpr int SPW = NB3 / kRowWaves;  // branches s per wave
  constexpr int BS = 64 * kRowWaves;
  __shared__ double acc[3][NB3][NB3][64];  // [kind][s][s' or s''][lane]
  __shared__ double2 phq[64];
  __shared__ double red[NB3][64];
  // lane | s1 << 6 | s2 << 9 | s << 12 of the pairs near the cut, and of those
  // that pass it with their rates
  static_assert(NB3 <= 8, "three bits a branch");
  __shared__ uint16_t near_w[kRowWaves][kRowQueue], pass_w[kRowWaves][kRowQueue];
  __shared__ double dp_w[kRowWaves][kRowQueue], dm_w[kRowWaves][kRowQueue];
  __shared__ double wq[NB3];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s_lo = wv * SPW;  // this wave's branches of q: [s_lo, s_lo + SPW)
  uint16_t *near_q = near_w[wv], *pass_q = pass_w[wv];
  double *dp_q = dp_w[wv], *dm_q = dm_w[wv];
  const int q = blockIdx.x;
  const int nq = p.nq;
  const size_t n = (size_t)nq * NB3;
  const int N0 = p.N[0], N1 = p.N[1], N2 = p.N[2];
  const int a0 = q / (N1 * N2), a1 = (q / N2) % N1, a2 = q % N2;
  bool any = false;
  for (int s = 0; s < NB3; ++s) any = any || phys[q * NB3 + s];
  if (!any) {
    if (tid < NB3) gamma0[q * NB3 + tid] = 0.0;
    return;
  }
  if (tid < NB3) wq[tid] = omega[q * NB3 + tid];
  for (int l = tid; l < n_rep; l += BS) {
    const int32_t* r = rep + 3 * l;
    const int m0 = ((a0 * r[0]) % N0 + N0) % N0, m1 = ((a1 * r[1]) % N1 + N1) % N1,
              m2 = ((a2 * r[2]) % N2 + N2) % N2;
    const double f = (double)m0 / N0 + (double)m1 / N1 + (double)m2 / N2;
    double sn, cs;
    sincospi(2.0 * f, &sn, &cs);
    phq[l] = make_double2(cs, sn);
  }
  for (int k = tid; k < n_blk * 9 * NB3; k += BS) at[k] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int k = tid; k < p.n_e * NB3; k += BS) {
    const int e = k / NB3, s = k % NB3;
    double re = 0.0, im = 0.0;
    for (int t = t_ptr[e]; t < t_ptr[e + 1]; ++t) {
      const size_t o = (((size_t)q * NB3 + t_i[t]) * NB3 + s) * 2;
      const double ex = evec[o], ey = evec[o + 1];
      const double2 f = phq[t_l2[t]];
      const double c = t_coef[t];
      re += c * (ex * f.x - ey * f.y);
      im += c * (ex * f.y + ey * f.x);
    }
    at[(e_blk[e] * 9 + e_bg[e]) * NB3 + s] = make_double2(re, im);
  }
  __syncthreads();
  double g0[SPW];  // Gamma0 of the wave's branches, from the terms this lane computed
  float ws[SPW];   // their FP32 frequencies, NaN below nu_min
  float w_max = 0.0f;
#pragma unroll
  for (int k = 0; k < SPW; ++k) {
    g0[k] = 0.0;
    const float w = (float)omega[q * NB3 + s_lo + k];
    ws[k] = phys[q * NB3 + s_lo + k] ? w : __builtin_nanf("");
    w_max = fmaxf(w_max, fabsf(w));
  }
  const int t0 = (N0 - a0) % N0, t1 = (N1 - a1) % N1, t2 = (N2 - a2) % N2;
  auto partner = [&](int q1) {
    const int b0 = q1 / (N1 * N2), b1 = (q1 / N2) % N1, b2 = q1 % N2;
    return (wrap_sub(t0, b0, N0) * N1 + wrap_sub(t1, b1, N1)) * N2 + wrap_sub(t2, b2, N2);
  };
  // |V|^2 of one (q1, s1, q2, s2, s) with the prefactor:
  // V = sum_blk e^{-i q1.R_d(blk)} sum_{beta gamma} A~[blk][beta gamma][s]
  //     eta_{3 jb + beta}(q1, s1) eta_{3 kb + gamma}(q2, s2),
  // the two eigenvector rows in registers, complex multiply-adds as fused
  // multiply-adds into the sums
  auto vertex2 = [&](int q1, int s1, int q2, int s2, int s) {
    double2 x[NB3], y[NB3];
#pragma unroll
    for (int i = 0; i < NB3; ++i) {
      const double* ex = evec + (((size_t)q1 * NB3 + i) * NB3 + s1) * 2;
      const double* ey = evec + (((size_t)q2 * NB3 + i) * NB3 + s2) * 2;
      x[i] = make_double2(ex[0], ex[1]);
      y[i] = make_double2(ey[0], ey[1]);
    }
    const double2* ph = phase_tab + (size_t)q1 * p.n_d;
    double vr = 0.0, vi = 0.0;
#pragma unroll
    for (int jb = 0; jb < NB; ++jb) {
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) {
        for (int blk = pair_ptr[jb * NB + kb]; blk < pair_ptr[jb * NB + kb + 1]; ++blk) {
          const double2* ab = at + (size_t)blk * 9 * NB3 + s;
          double ur = 0.0, ui = 0.0;
#pragma unroll
          for (int be = 0; be < 3; ++be) {
            double tr_ = 0.0, ti = 0.0;
#pragma unroll
            for (int ga = 0; ga < 3; ++ga) {
              const double2 a = ab[(be * 3 + ga) * NB3], v = y[3 * kb + ga];
              tr_ = fma(a.x, v.x, tr_);
              tr_ = fma(-a.y, v.y, tr_);
              ti = fma(a.x, v.y, ti);
              ti = fma(a.y, v.x, ti);
            }
            const double2 u = x[3 * jb + be];
            ur = fma(u.x, tr_, ur);
            ur = fma(-u.y, ti, ur);
            ui = fma(u.x, ti, ui);
            ui = fma(u.y, tr_, ui);
          }
          const double2 f = ph[blk_d[blk]];
          vr = fma(f.x, ur, vr);
          vr = fma(-f.y, ui, vr);
          vi = fma(f.x, ui, vi);
          vi = fma(f.y, ur, vi);
        }
      }
    }
    return pref * (vr * vr + vi * vi);
  };
  // A round takes 64 partners q1, one per lane of every wave; wave w takes
  // the branches s of q in [w SPW, (w + 1) SPW).  Each lane tests its
  // (s1, s2, s) in that order against the widest cut the pair's FP32 speeds
  // allow (what passes its own cut passes here: 2 sigma <= 2 max(floor,
  // (|v1| + |v2|) h / sqrt(12)), with slack for the rounding of the test);
  // the near ones go to the wave's queue in LDS (slots by ballot: candidate
  // order, lanes ascending), 64 of them at a time take the exact FP64 cut and
  // rates, and those that pass the second queue, of which 64 at a time are
  // projected.  A projected term belongs to the element of its kind, branches
  // and lane: the terms of one s2 (kinds 0 and 1), of one s1 (kind 2) all have
  // different ones, so they are added in NB3 + NB3 steps, always in this order.
  // A wave's queues and elements are its own: a wave-level fence and barrier
  // order its steps.
  const unsigned long long below = (1ull << lane) - 1ull;
  auto wave_sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };
  const float hr = p.adaptive ? 2.008f : 0.0f;
  const float r_min = 2.0f * (float)(p.adaptive ? p.sig_floor : p.sig_fixed) * 1.00001f;
  for (int base = 0; base < nq; base += 64) {
    const int q1 = base + lane;
    const bool ok = q1 < nq;
    for (int k = 0; k < 3; ++k)
      for (int s = s_lo; s < s_lo + SPW; ++s)
        for (int u = 0; u < NB3; ++u) acc[k][s][u][lane] = 0.0;
    const int q2 = ok ? partner(q1) : 0;
    int n_near = 0, n_pass = 0;  // entries of the queues (the same in every lane)
    auto project = [&](int n) {
      wave_sync();
      const bool on = lane < n;
      const int code = on ? pass_q[lane] : 0;
      const int o = code & 63, s1 = (code >> 6) & 7, s2 = (code >> 9) & 7, s = code >> 12;
      const int e1 = base + o, e2 = __shfl(q2, o, 64);
      double a = 0.0, b = 0.0, c = 0.0, g = 0.0;
      if (on) {
        const double w = wq[s], w1 = omega[e1 * NB3 + s1], w2 = omega[e2 * NB3 + s2];
        const double v2 = vertex2(e1, s1, e2, s2, s);
        const double dp = dp_q[lane] * v2, dm = dm_q[lane] * v2;
        g = dp + dm;
        a = dp * (w1 / w);
        b = dm * (w1 / w);
        c = g * (w2 / w);
      }
#pragma unroll
      for (int k = 0; k < SPW; ++k) g0[k] += on && s == s_lo + k ? g : 0.0;
      // (the barriers keep the steps apart: to one lane they are one)
      for (int u = 0; u < NB3; ++u) {
        if (on && s2 == u) {
          acc[0][s][s1][o] += a;
          acc[1][s][s1][o] += b;
        }
        wave_sync();
      }
      for (int u = 0; u < NB3; ++u) {
        if (on && s1 == u) acc[2][s][s2][o] += c;
        wave_sync();
      }
    };
    auto classify = [&](int n, bool last) {
      wave_sync();
      const bool on = lane < n;
      const int code = on ? near_q[lane] : 0;
      const int o = code & 63, s1 = (code >> 6) & 7, s2 = (code >> 9) & 7, s = code >> 12;
      const int m1 = (base + o) * NB3 + s1, m2 = __shfl(q2, o, 64) * NB3 + s2;
      bool pass = false;
      double dp = 0.0, dm = 0.0;
      if (on) {
        const double w = wq[s], w1 = omega[m1], w2 = omega[m2];
        double sp, sm;
        widths(p, vel, m1, m2, sp, sm);
        // the cut first, then the rates
        if (fabs((w + w1) - w2) < 2.0 * sp || fabs((w - w1) - w2) < 2.0 * sm) {
          process_rates(p, w, w1, w2, occ[m1], occ[m2], sp, sm, dp, dm);
          pass = !(dp == 0.0 && dm == 0.0);
        }
      }
      const unsigned long long mask = __ballot(pass);
      if (pass) {
        const int r = n_pass + __popcll(mask & below);
        pass_q[r] = (uint16_t)code;
        dp_q[r] = dp;
        dm_q[r] = dm;
      }
      n_pass += __popcll(mask);
      while (n_pass >= 64 || (last && n_pass > 0)) {
        project(min(n_pass, 64));
        // the rest, fewer than 64, moves to the front
        n_pass = max(n_pass - 64, 0);
        const uint16_t mc = pass_q[64 + lane];
        const double mp = dp_q[64 + lane], mm = dm_q[64 + lane];
        wave_sync();
        pass_q[lane] = mc;
        dp_q[lane] = mp;
        dm_q[lane] = mm;
      }
      // what the near queue holds past the first 64 moves to the front
      wave_sync();
      const uint16_t mn = near_q[64 + lane];
      wave_sync();
      near_q[lane] = mn;
      n_near = max(n_near - 64, 0);
    };
    for (int s1 = 0; s1 < NB3; ++s1) {
      float2 f1 = near_tab[(size_t)s1 * nq + (ok ? q1 : 0)];
      if (!ok) f1.x = __builtin_nanf("");
#pragma unroll
      for (int s2 = 0; s2 < NB3; ++s2) {
        const float2 f2 = near_tab[(size_t)s2 * nq + q2];
        const float reach =
            fmaxf(r_min, hr * (f1.y + f2.y)) + 1e-6f * (w_max + fabsf(f1.x) + fabsf(f2.x)) + 1e-8f;
        const float cp = f1.x - f2.x, cm = -f1.x - f2.x;  // NaN below nu_min: fails every comparison
        unsigned hit = 0;
#pragma unroll
        for (int k = 0; k < SPW; ++k)
          hit |= fabsf(ws[k] + cp) < reach || fabsf(ws[k] + cm) < reach ? 1u << k : 0u;
        if (!__ballot(hit != 0)) continue;
#pragma unroll 1
        for (int k = 0; k < SPW; ++k) {
          const unsigned long long mask = __ballot(hit >> k & 1);
          if (hit >> k & 1)
            near_q[n_near + __popcll(mask & below)] =
                (uint16_t)(lane | s1 << 6 | s2 << 9 | (s_lo + k) << 12);
          n_near += __popcll(mask);
          if (n_near >= 64) classify(64, false);
        }
      }
    }
    classify(n_near, true);
    __syncthreads();
    // three passes; within each the columns of different lanes differ
    if (ok) {
      for (int s = s_lo; s < s_lo + SPW; ++s) {
        double* row = mat + (size_t)(q * NB3 + s) * n;
        for (int u = 0; u < NB3; ++u) {
          const double x = acc[0][s][u][lane];
          if (x != 0.0) row[q1 * NB3 + u] += x;
        }
      }
    }
    __syncthreads();
    if (ok) {
      for (int s = s_lo; s < s_lo + SPW; ++s) {
        double* row = mat + (size_t)(q * NB3 + s) * n;
        for (int u = 0; u < NB3; ++u) {
          const double x = acc[1][s][u][lane];
          if (x != 0.0) row[tr[q1 * NB3 + u]] -= x;
        }
      }
    }
    __syncthreads();
    if (ok) {
      for (int s = s_lo; s < s_lo + SPW; ++s) {
        double* row = mat + (size_t)(q * NB3 + s) * n;
        for (int u = 0; u < NB3; ++u) {
          const double x = acc[2][s][u][lane];
          if (x != 0.0) row[tr[q2 * NB3 + u]] -= x;
        }
      }
    }
    __syncthreads();
  }
  // Gamma0: fixed-order tree over the lanes, then onto the diagonal
#pragma unroll
  for (int k = 0; k < SPW; ++k) red[s_lo + k][lane] = g0[k];
  __syncthreads();
  for (int w = 32; w > 0; w >>= 1) {
    if (lane < w)
      for (int s = s_lo; s < s_lo + SPW; ++s) red[s][lane] += red[s][lane + w];
    __syncthreads();
  }
  if (lane < SPW) {
    const int s = s_lo + lane, mu = q * NB3 + s;
    const double g = phys[mu] ? red[s][0] : 0.0;
    gamma0[mu] = g;
    mat[(size_t)mu * n + mu] += g;
  }
}

// Largest Gamma0 (order-independent), one workgroup.
__global__ __launch_bounds__(1024) void bte_gmax(long n, const double* __restrict__ g0,
                                                 double* __restrict__ out) {
  __shared__ double red[1024];
  double m = 0.0;
  for (long k = threadIdx.x; k < n; k += 1024) m = fmax(m, g0[k]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

__device__ __forceinline__ bool bte_active(double w, double g, double gmax, double nu_min) {
  return (w / kTwoPi >= nu_min) && (g > kGammaFloorRel * gmax) && (g > 0.0);
}

// Which modes keep their RTA conductivity (1) or are decoupled (0).
__global__ void bte_flags(long n, const double* __restrict__ omega, const double* __restrict__ g0,
                          const double* __restrict__ gmax, double nu_min,
                          uint8_t* __restrict__ act) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) act[i] = bte_active(omega[i], g0[i], *gmax, nu_min) ? 1 : 0;
}

// Decoupled modes: zero row and column, unit diagonal.  One workgroup per
// row j, its threads along the row: a decoupled row is written whole, the
// row of a kept mode only at the decoupled columns (coalesced either way).
__global__ __launch_bounds__(256) void bte_decouple(long n, const uint8_t* __restrict__ act,
                                                    double* __restrict__ mat) {
  const long j = blockIdx.x;
  if (j >= n) return;
  double* row = mat + j * n;
  if (!act[j]) {
    for (long i = threadIdx.x; i < n; i += 256) row[i] = (i == j) ? 1.0 : 0.0;
  } else {
    for (long i = threadIdx.x; i < n; i += 256)
      if (!act[i]) row[i] = 0.0;
  }
}

// Right-hand side: v on active modes, 0 elsewhere; rhs[i][3].
// The coupled modes in order: rows[a] = the a-th mode with act = 1, *count =
// their number.  One workgroup; each thread counts a contiguous run of
// modes, a block-wide scan places the runs.
__global__ __launch_bounds__(1024) void bte_compact_index(long n, const uint8_t* __restrict__ act,
                                                          int32_t* __restrict__ rows,
                                                          int32_t* __restrict__ count) {
  __shared__ int sums[1024];
  const int tid = threadIdx.x;
  const long per = (n + 1023) / 1024;
  const long lo = tid * per < n ? tid * per : n, hi = lo + per < n ? lo + per : n;
  int c = 0;
  for (long i = lo; i < hi; ++i) c += act[i];
  sums[tid] = c;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int v = tid >= off ? sums[tid - off] : 0;
    __syncthreads();
    sums[tid] += v;
    __syncthreads();
  }
  int r = sums[tid] - c;
  for (long i = lo; i < hi; ++i)
    if (act[i]) rows[r++] = (int32_t)i;
  if (tid == 1023) *count = sums[1023];
}

// Moves the coupled columns of a coupled row to its front: row rows[a]
// becomes (A[rows[a]][rows[0]], ..., A[rows[a]][rows[na - 1]], ...).  One
// workgroup per row, in slices of 256 columns: a slice's values are all read
// before any is written, and its targets lie before the sources of every
// later slice (rows[b] >= b).
__global__ __launch_bounds__(256) void bte_compact_cols(long na, long ld,
                                                        const int32_t* __restrict__ rows,
                                                        double* __restrict__ mat) {
  const long a = blockIdx.x;
  if (a >= na) return;
  double* row = mat + (long)rows[a] * ld;
  for (long b0 = 0; b0 < na; b0 += 256) {
    const long b = b0 + threadIdx.x;
    const double v = b < na ? row[rows[b]] : 0.0;
    __syncthreads();
    if (b < na) row[b] = v;
    __syncthreads();
  }
}

// dst[a] = src[rows[a]] (three components), and back: dst[rows[a]] = src[a]
// over a zeroed dst.
__global__ void bte_gather3(long na, const int32_t* __restrict__ rows,
                            const double* __restrict__ src, double* __restrict__ dst) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < 3 * na) dst[k] = src[3 * (long)rows[k / 3] + k % 3];
}
__global__ void bte_scatter3(long na, const int32_t* __restrict__ rows,
                             const double* __restrict__ src, double* __restrict__ dst) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < 3 * na) dst[3 * (long)rows[k / 3] + k % 3] = src[k];
}

__global__ void bte_rhs(long n, const double* __restrict__ omega, const double* __restrict__ vel,
                        const double* __restrict__ g0, const double* __restrict__ gmax,
                        double nu_min, double* __restrict__ rhs) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const bool a = bte_active(omega[i], g0[i], *gmax, nu_min);
  for (int c = 0; c < 3; ++c) rhs[3 * i + c] = a ? vel[3 * i + c] : 0.0;
}

// kappa_ab = scale sum_i c_i v_ia lambda_ib over active modes; one workgroup.
__global__ __launch_bounds__(1024) void bte_kappa(long n, const double* __restrict__ omega,
                                                  const double* __restrict__ vel,
                                                  const double* __restrict__ lam,
                                                  const double* __restrict__ g0,
                                                  const double* __restrict__ gmax,
                                                  double inv_kt_hbar, double nu_min,
                                                  double scale, double* __restrict__ kappa) {
  __shared__ double red[1024][9];
  const int t = threadIdx.x;
  double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const double gm = *gmax;
  for (long i = t; i < n; i += 1024) {
    const double w = omega[i];
    if (!bte_active(w, g0[i], gm, nu_min)) continue;
    const double x = w * inv_kt_hbar;
    const double em = expm1(x);
    const double c = x * x * (em + 1.0) / (em * em);
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) acc[3 * a + b] += c * vel[3 * i + a] * lam[3 * i + b];
  }
  for (int k = 0; k < 9; ++k) red[t][k] = acc[k];
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (t < w)
      for (int k = 0; k < 9; ++k) red[t][k] += red[t + w][k];
    __syncthreads();
  }
  if (t < 9) kappa[t] = scale * red[0][t];
}

// ------------------------------------------------------------------ LU

// The coupled block of the matrix as the LU sees it: element (i, j) of the
// n x n coupled system sits at row rows[i] of the stored matrix (leading
// dimension ld), column j (the coupled columns of each stored row are moved
// to its front by bte_compact_cols).
struct MatRows {
  double* mat;
  const int32_t* rows;
  long ld;
  __device__ double* row(long i) const { return mat + (long)rows[i] * ld; }
};

// 64 x 64 x 64 product P Q from two LDS blocks, four waves of 32 x 32 on
// v_mfma_f64_16x16x4f64; wave wv holds rows wm = 32 (wv / 2) and columns
// wn = 32 (wv % 2) of the result in acc[a][b] (16 x 16 tiles).
struct BlockProduct {
  int wm, wn, lr, lg;
  d4 acc[2][2];
  __device__ void clear(int tid) {
    const int lane = tid & 63, wv = tid >> 6;
    wm = (wv >> 1) * 32;
    wn = (wv & 1) * 32;
    lr = lane & 15;
    lg = lane >> 4;
    for (int a = 0; a < 2; ++a)
      for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  }
  __device__ void add(const double (*P)[kLuB + 1], const double (*Q)[kLuB + 1]) {
    for (int kk = 0; kk < kLuB; kk += 4) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const double av = P[wm + 16 * a + lr][kk + lg];  // A[row = lane % 16][k = lane / 16]
          const double bv = Q[kk + lg][wn + 16 * b + lr];  // B[k = lane / 16][col = lane % 16]
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[a][b], 0, 0, 0);
        }
    }
  }
  // FP64 16 x 16 accumulator: item r of lane l is row 4 r + l / 16, column l % 16
  __device__ int row(int a, int r) const { return wm + 16 * a + 4 * r + lg; }
  __device__ int col(int b) const { return wn + 16 * b + lr; }
};

// Panels of step k: row blocks A_kj <- Linv A_kj (j > k, first nb - k - 1
// workgroups), column blocks A_ik <- A_ik Uinv (i > k, the rest).
__global__ __launch_bounds__(256) void lu_panels(long n, int nb, int k, MatRows A,
                                                 const double* __restrict__ linv,
                                                 const double* __restrict__ uinv) {
  constexpr int B = kLuB;
  __shared__ double M[B][B + 1];
  __shared__ double T[B][B + 1];
  const int tid = threadIdx.x;
  const int m = nb - k - 1;
  const bool row = (int)blockIdx.x < m;
  const int other = k + 1 + (row ? blockIdx.x : blockIdx.x - m);
  const long bi = row ? k : other, bj = row ? other : k;
  const int pc = 2 * (tid & 31), pr = tid >> 5;  // pair tid % 32 of the rows tid / 32 + 8 i
  const double* inv = (row ? linv : uinv) + pr * B + pc;
  const long c = bj * B + pc;
  d2 pm[8], pt[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const double* r = A.row(min(bi * B + pr + 8 * i, n - 1));
    if (c + 1 < n)
      pm[i] = *reinterpret_cast<const d2u*>(r + c);
    else
      pm[i] = d2{c < n ? r[c] : 0.0, 0.0};
    pt[i] = *reinterpret_cast<const d2*>(inv + 8 * i * B);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    M[pr + 8 * i][pc] = pm[i].x;
    M[pr + 8 * i][pc + 1] = pm[i].y;
    T[pr + 8 * i][pc] = pt[i].x;
    T[pr + 8 * i][pc + 1] = pt[i].y;
  }
  __syncthreads();
  BlockProduct bp;
  bp.clear(tid);
  if (row)
    bp.add(T, M);
  else
    bp.add(M, T);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long gi = bi * B + bp.row(a, r), gj = bj * B + bp.col(b);
        if (gi < n && gj < n) A.row(gi)[gj] = bp.acc[a][b][r];
      }
}

// The factorisation (no pivoting) of a 64 x 64 block D in LDS to L\U, and the
// inverses of the unit lower L (strictly lower part of X) and of the upper U
// (the rest of X).  Wave w keeps columns 16 w .. 16 w + 15 in registers, a lane
// per row.  In turn each wave factors its own columns, every row, and
// publishes the multipliers, which the waves to the right apply; the pivot
// row is read lane to scalar, so a step has no barrier and no LDS round trip.
// Then the inverses: of each 16 x 16 diagonal block by its wave (L in sixteen
// lanes, U turned about in sixteen others: the same substitution), and the
// other blocks X_ij = -X_ii sum_t L_it X_tj (and U alike) by distance from the
// diagonal, a wave per block, on the matrix cores: an accumulator's items are
// the next product's second operand as they lie.
// One workgroup is the serial part of every step, so this is latency alone:
// 64 steps over the whole block with a barrier each took a launch of 51 us,
// this 33.
typedef double (*Block)[kLuB + 1];
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __builtin_bit_cast(long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, (long long)((unsigned long long)hi << 32 | lo));
}
__device__ __forceinline__ void factor_block(Block D, Block X, int tid, int32_t* flags) {
  constexpr int Q = 16;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  double a[Q];
#pragma unroll
  for (int c = 0; c < Q; ++c) a[c] = D[lane][Q * wv + c];
  bool singular = false;
#pragma unroll 1
  for (int w = 0; w < kLuB / Q; ++w) {
    const int o = Q * w;
    Block mul = X + (w & 1) * Q;  // the multipliers l_i of its 16 steps, in two places in turn
    if (wv == w) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const double piv = lane_value(a[j], o + j);
        singular |= !(fabs(piv) > 1e-300);
        const double r = 1.0 / piv, q = a[j] * r;
        const bool below = lane > o + j;
        const double l = below ? q : 0.0;
        a[j] = below ? q : a[j];
        mul[j][lane] = l;
#pragma unroll
        for (int c = j + 1; c < Q; ++c) a[c] = fma(-l, lane_value(a[c], o + j), a[c]);
      }
    }
    __syncthreads();
    if (wv > w) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const double l = mul[j][lane];
#pragma unroll
        for (int c = 0; c < Q; ++c) a[c] = fma(-l, lane_value(a[c], o + j), a[c]);
      }
    }
  }
  if (singular && lane == 0) raise_flag(flags, kFlagSingular);
#pragma unroll
  for (int c = 0; c < Q; ++c) D[lane][Q * wv + c] = a[c];
  __syncthreads();
  {
    const int o = Q * wv;
    const bool up = lane & Q;
    const double* corner = &D[o + (up ? Q - 1 : 0)][o + (up ? Q - 1 : 0)];
    const int dir = up ? -1 : 1;
    auto at = [&](int i, int j) { return corner[dir * (i * (kLuB + 1) + j)]; };
    const double own = up ? 1.0 / at(lr, lr) : 1.0;
    double x[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) x[i] = i == lr ? 1.0 : 0.0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      x[j] *= __shfl(own, (lane & Q) + j, 64);
#pragma unroll
      for (int i = j + 1; i < Q; ++i) x[i] = fma(-at(i, j), x[j], x[i]);
      if (j % 4 == 3) asm volatile("" ::: "memory");  // the reads of four columns in flight, not of all
    }
    if (lane < 2 * Q) {
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        if (up && i >= lr) X[o + Q - 1 - i][o + Q - 1 - lr] = x[i];
        if (!up && i > lr) X[o + i][o + lr] = x[i];
      }
    }
  }
  __syncthreads();
  // element (i, j) of the inverse of L, of U
  auto inv_l = [&](int i, int j) { return i > j ? X[i][j] : i == j ? 1.0 : 0.0; };
  auto inv_u = [&](int i, int j) { return i <= j ? X[i][j] : 0.0; };
  for (int dist = 1; dist < kLuB / Q; ++dist) {
    const int per = kLuB / Q - dist;
    for (int t = wv; t < 2 * per; t += 4) {
      const bool low = t < per;
      const int lo = low ? t : t - per, hi = lo + dist;  // L: block (hi, lo); U: (lo, hi)
      const int bi = low ? hi : lo, bj = low ? lo : hi;
      d4 sum = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
      for (int b = low ? lo : lo + 1; b < (low ? hi : hi + 1); ++b)
#pragma unroll
        for (int k = 0; k < Q; k += 4) {
          const int kk = Q * b + k + lg, c = Q * bj + lr;
          sum = __builtin_amdgcn_mfma_f64_16x16x4f64(-D[Q * bi + lr][kk], low ? inv_l(kk, c) : inv_u(kk, c), sum,
                                                     0, 0, 0);
        }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = Q * bi + lr, kk = Q * bi + 4 * k + lg;
        x = __builtin_amdgcn_mfma_f64_16x16x4f64(low ? inv_l(i, kk) : inv_u(i, kk), sum[k], x, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) X[Q * bi + 4 * r + lg][Q * bj + lr] = x[r];
    }
    __syncthreads();
  }
}

// Step k of a panel that starts at block k0: the blocks of row and column k
// take the panel's earlier steps, A_ij -= sum_{k0 <= t < k} A_it A_tj (one
// product over all of them, so that a block is read and written once), and
// workgroup 0, which has the diagonal block, factors it meanwhile; its L\U is
// written back, the inverses of L and U to linv / uinv [64][64].  Workgroups 1
// .. m have the blocks (k + 1 ..., k), the next m the blocks (k, k + 1 ...).
// Rows and columns past n read as others' and are not written; the diagonal
// block's act as identity.  Updating every block of the panel at every step, as
// a third launch, the factorisation's steps took 26.9 ms of 13,500 equations,
// now 13.4.  Panels of four and six blocks: 9.4 and 10.2 ms here against 10.0,
// but 32.6 and 30.2 in the product against 28.7.
__global__ __launch_bounds__(256) void lu_left(long n, int nb, int k0, int k, MatRows A,
                                               double* __restrict__ linv, double* __restrict__ uinv,
                                               int32_t* __restrict__ flags) {
  constexpr int B = kLuB;
  __shared__ double L[B][B + 1];
  __shared__ double U[B][B + 1];
  const int tid = threadIdx.x, m = nb - k - 1, wb = (int)blockIdx.x;
  const int bi = wb <= m ? k + wb : k, bj = wb <= m ? k : k + wb - m;
  // pair tid % 32 of the rows tid / 32 + 8 i of a block
  const int pc = 2 * (tid & 31), pr = tid >> 5;
  BlockProduct bp;
  bp.clear(tid);
  const bool whole = (long)bj * B + B <= n;
  // (the rows' places in the matrix one block ahead of their elements)
  d2 pl[8], pu[8];
  int rl[8], ru[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    rl[i] = A.rows[min((long)bi * B + pr + 8 * i, n - 1)];
    ru[i] = A.rows[min((long)k0 * B + pr + 8 * i, n - 1)];
  }
  auto fetch = [&](int t) {
    const long c = (long)bj * B + pc;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pl[i] = *reinterpret_cast<const d2u*>(A.mat + rl[i] * A.ld + (long)t * B + pc);
      const double* u = A.mat + ru[i] * A.ld;
      if (whole)
        pu[i] = *reinterpret_cast<const d2u*>(u + c);
      else
        pu[i] = d2{u[min(c, n - 1)], u[min(c + 1, n - 1)]};
      ru[i] = A.rows[min((long)(t + 1) * B + pr + 8 * i, n - 1)];
    }
  };
  if (k0 < k) fetch(k0);
  for (int t = k0; t < k; ++t) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      L[pr + 8 * i][pc] = pl[i].x;
      L[pr + 8 * i][pc + 1] = pl[i].y;
      U[pr + 8 * i][pc] = pu[i].x;
      U[pr + 8 * i][pc + 1] = pu[i].y;
    }
    __syncthreads();
    if (t + 1 < k) fetch(t + 1);
    bp.add(L, U);
    __syncthreads();
  }
  // the block itself, every load unconditional (rows and columns past n read
  // the last one): under conditions they would wait for each other
  double* row[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) row[a][r] = A.row(min((long)bi * B + bp.row(a, r), n - 1));
  double old[2][2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) old[a][b][r] = row[a][r][min((long)bj * B + bp.col(b), n - 1)];
  auto each = [&](auto f) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = bp.row(a, r), j = bp.col(b);
          const long gj = (long)bj * B + j;
          f(i, j, (long)bi * B + i < n && gj < n, row[a][r] + gj, old[a][b][r] - bp.acc[a][b][r]);
        }
  };
  if (wb != 0) {
    each([&](int, int, bool in, double* to, double v) {
      if (in) *to = v;
    });
    return;
  }
  each([&](int i, int j, bool in, double*, double v) { L[i][j] = in ? v : (i == j ? 1.0 : 0.0); });
  __syncthreads();
  factor_block(L, U, tid, flags);
  each([&](int i, int j, bool in, double* to, double) {
    if (in) *to = L[i][j];
  });
  for (int idx = tid; idx < B * B; idx += 256) {
    const int i = idx / B, j = idx % B;
    linv[idx] = i > j ? U[i][j] : i == j ? 1.0 : 0.0;
    uinv[idx] = i <= j ? U[i][j] : 0.0;
  }
}

// Deferred update of a panel: A_ij -= sum_k A_ik A_kj over the panel's
// columns k in [kc, kc + kw) for the trailing elements i, j >= r0 (blocked
// LU: the panel's own steps update only the panel's columns and rows, this one
// product the rest).  128 x 128 tile per workgroup, four waves of 64 x 64 as
// 4 x 4 v_mfma_f64_16x16x4f64 accumulators, which start as the tile itself
// (the rows are staged negated); K in slices of 16 staged in LDS (two buffers,
// the next slice fetched into registers while the current one is multiplied).
// Every load is 16 bytes without a condition: rows past n repeat the last one
// and are not written, the last tile of columns is moved back to end at n and
// writes its own columns only (n >= 128 wherever a panel is full, and the
// panel's columns are all below n).  Rows are read by pairs of k: lane group
// lg of an instruction holds k = 2 lg (+ 1 for the next instruction) of both
// operands.  Bound by the matrix cores, with conditions on every element of a
// fetch 50 % busy: the products of 13,500 equations took 41.1 ms, now 28.7 (52
// TFLOP/s).  Workgroups in 2 x 2 to 8 x 8 groups per XCD measured 29.0 to 31.1.
constexpr int kLgT = 128;        // tile edge
constexpr int kLgK = 16;         // K slice
constexpr int kLgLd = kLgT + 8;  // LDS stride of a k (doubles): the rows two lane groups read, 2 k apart, share no bank
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void lu_gemm(
    long n, long r0, long kc, int kw, int ntl, MatRows A) {
  __shared__ d2 As[2][kLgT * 8];        // row r, pair p at 8 r + (p ^ (r / 2 % 8)): conflict-free
  __shared__ double Bs[2][kLgK][kLgLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long row0 = r0 + (long)(blockIdx.x / ntl) * kLgT, col0 = r0 + (long)(blockIdx.x % ntl) * kLgT;
  if (row0 >= n || col0 >= n) return;
  const long cs = min(col0, n - kLgT);
  // staging: pair tid % 8 of the rows tid / 8 + 32 i; k = wv + 4 i, columns 2 lane, + 1
  const int ap = tid & 7, ar = tid >> 3;
  const double* arow[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) arow[i] = A.row(min(row0 + ar + 32 * i, n - 1)) + 2 * ap;
  d2 pa[4], pb[4];
  auto fetch = [&](long k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) pa[i] = *reinterpret_cast<const d2u*>(arow[i] + k0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      pb[i] = *reinterpret_cast<const d2u*>(A.row(k0 + wv + 4 * i) + cs + 2 * lane);
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ar + 32 * i;
      As[buf][r * 8 + (ap ^ ((r >> 1) & 7))] = -pa[i];
      *reinterpret_cast<d2*>(&Bs[buf][wv + 4 * i][2 * lane]) = pb[i];
    }
  };
  const int wm = (wv >> 1) * 64, wn = (wv & 1) * 64;
  const int lr = lane & 15, lg = lane >> 4;
  fetch(kc);
  // item r of lane l of an accumulator is row 4 r + l / 16, column l % 16
  d4 acc[4][4];
  auto each_row = [&](auto f) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long gi = row0 + wm + 16 * a + 4 * r + lg;
        f(a, r, gi < n, A.row(min(gi, n - 1)) + cs + wn + lr);
      }
  };
  each_row([&](int a, int r, bool, const double* row) {
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b][r] = row[16 * b];
  });
  stage(0);
  __syncthreads();
  int cur = 0;
  for (long k0 = kc; k0 < kc + kw; k0 += kLgK) {
    const bool more = k0 + kLgK < kc + kw;
    if (more) fetch(k0 + kLgK);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      d2 av[4];
      double b0[4], b1[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = wm + 16 * t + lr;
        av[t] = As[cur][r * 8 + ((4 * h + lg) ^ ((r >> 1) & 7))];
        b0[t] = Bs[cur][8 * h + 2 * lg][wn + 16 * t + lr];
        b1[t] = Bs[cur][8 * h + 2 * lg + 1][wn + 16 * t + lr];
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].x, b0[b], acc[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].y, b1[b], acc[a][b], 0, 0, 0);
    }
    if (more) stage(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
  each_row([&](int a, int r, bool in, const double* row) {
    if (in) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (cs + wn + 16 * b + lr >= col0) const_cast<double*>(row)[16 * b] = acc[a][b][r];
    }
  });
}

// Triangular sweeps with 3 right-hand sides, right-looking by the panels of
// the factorisation: the residual r starts as the right-hand side; a panel's
// blocks are solved in turn by one workgroup, x_k = Tinv_k r_k, r_i -= A_ik x_k
// for the panel's blocks still to solve (lu_solve), then one product with all
// its columns updates the rows past it (lu_solve_rest; forward the rows below
// with the L blocks, backward the rows above with the U blocks).  Fixed-order
// sums.  With a launch per block that updated every row, every workgroup
// forming x_k for itself, the two sweeps of 13,500 rows took 8.7 ms, now 4.6.
constexpr int kPanelRows = kLuPanel * kLuB;

// Sum over a lane's row of 16 by rotations of the row: vector instructions
// (through LDS the reductions took most of lu_solve).
template <int ROT>
__device__ __forceinline__ double add_rotated(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const unsigned lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + ROT, 0xf, 0xf, false),
                 hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + ROT, 0xf, 0xf, false);
  return v + __builtin_bit_cast(double, (long long)((unsigned long long)hi << 32 | lo));
}
__device__ __forceinline__ double sum16(double v) {
  return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(v))));
}
template <bool FORWARD>
__global__ __launch_bounds__(1024) void lu_solve(long n, int k0, int k1, const double* __restrict__ tinv,
                                                 MatRows A, double* __restrict__ x,
                                                 const double* __restrict__ r) {
  constexpr int B = kLuB;
  __shared__ double rs[kPanelRows][3];
  __shared__ double xk[B][3];
  const int tid = threadIdx.x, row = tid >> 4, sub = 4 * (tid & 15);
  const long g0 = (long)k0 * B;
  for (int i = tid; i < kPanelRows * 3; i += 1024) rs[i / 3][i % 3] = g0 + i / 3 < n ? r[3 * g0 + i] : 0.0;
  // rows and columns past n read the last one: their x is zero, their r not stored
  const double* at[kLuPanel];
#pragma unroll
  for (int b = 0; b < kLuPanel; ++b) at[b] = A.row(min(g0 + (long)b * B + row, n - 1));
  // four elements of a row of 64, sixteen lanes a row
  auto dot = [&](const double* a, const double (*v)[3], double* s) {
    for (int c = 0; c < 3; ++c) s[c] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < 3; ++c) s[c] = fma(a[u], v[sub + u][c], s[c]);
    for (int c = 0; c < 3; ++c) s[c] = sum16(s[c]);
  };
  for (int step = 0; step < k1 - k0; ++step) {
    const int kb = FORWARD ? step : k1 - k0 - 1 - step;
    const long col = g0 + (long)kb * B;
    // what the step reads from memory, all before its first barrier
    double t[4], a[kLuPanel][4], s[3];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = tinv[(size_t)(k0 + kb) * B * B + row * B + sub + u];
#pragma unroll
    for (int b = 0; b < kLuPanel; ++b)
#pragma unroll
      for (int u = 0; u < 4; ++u) a[b][u] = at[b][min(col + sub + u, n - 1)];
    __syncthreads();
    dot(t, rs + kb * B, s);
    if (sub == 0) {
      for (int c = 0; c < 3; ++c) {
        xk[row][c] = s[c];
        if (col + row < n) x[3 * (col + row) + c] = s[c];
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kLuPanel; ++b) {
      if (FORWARD ? b <= kb : b >= kb) continue;
      dot(a[b], xk, s);
      if (sub == 0)
        for (int c = 0; c < 3; ++c) rs[b * B + row][c] -= s[c];
    }
  }
}

// r_i -= sum over the panel's columns [c0, c1) of A_ic x_c for the rows [i0, i1);
// a wave per row, four rows in turn.
__global__ __launch_bounds__(256) void lu_solve_rest(long i0, long i1, long c0, long c1, MatRows A,
                                                     const double* __restrict__ x, double* __restrict__ r) {
  __shared__ double xs[kPanelRows][3];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < kPanelRows * 3; i += 256) xs[i / 3][i % 3] = c0 + i / 3 < c1 ? x[3 * c0 + i] : 0.0;
  __syncthreads();
  for (int k = 0; k < 4; ++k) {
    const long gi = i0 + (long)blockIdx.x * 16 + (tid >> 6) * 4 + k;
    if (gi >= i1) return;
    const double* row = A.row(gi) + c0;
    double a[8], s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = 2 * lane + 128 * u;
      d2u v = {0.0, 0.0};
      if (c0 + c + 1 < c1)
        v = *reinterpret_cast<const d2u*>(row + c);
      else if (c0 + c < c1)
        v.x = row[c];
      a[2 * u] = v.x;
      a[2 * u + 1] = v.y;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) s[q] = fma(a[u], xs[2 * lane + 128 * (u >> 1) + (u & 1)][q], s[q]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double v = wave_sum_fixed(s[q]);
      if (lane == q) r[3 * gi + q] -= v;
    }
  }
}

__global__ void bte_copy3(long n, const double* __restrict__ src, double* __restrict__ dst) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 3 * n) dst[i] = src[i];
}

// ------------------------------------------------------------------ iteration

// y = A x for 3 right-hand sides, one workgroup per row, fixed-order sums.
__global__ __launch_bounds__(256) void bte_gemv(long n, const double* __restrict__ mat,
                                                const double* __restrict__ x,
                                                double* __restrict__ y) {
  __shared__ double red[256][3];
  const long i = blockIdx.x;
  const int t = threadIdx.x;
  const double* a = mat + i * n;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  for (long c = t; c < n; c += 256) {
    const double v = a[c];
    s0 += v * x[3 * c];
    s1 += v * x[3 * c + 1];
    s2 += v * x[3 * c + 2];
  }
  red[t][0] = s0;
  red[t][1] = s1;
  red[t][2] = s2;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w)
      for (int c = 0; c < 3; ++c) red[t][c] += red[t + w][c];
    __syncthreads();
  }
  if (t < 3) y[3 * i + t] = red[0][t];
}

// lambda0 = v / Gamma0 on active modes (Eq. sc_iter's start, the RTA).
__global__ void bte_sc_init(long n, const double* __restrict__ rhs, const double* __restrict__ g0,
                            double* __restrict__ lam) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const bool a = rhs[3 * i] != 0.0 || rhs[3 * i + 1] != 0.0 || rhs[3 * i + 2] != 0.0;
  for (int c = 0; c < 3; ++c) lam[3 * i + c] = a ? rhs[3 * i + c] / g0[i] : 0.0;
}

// lambda <- (v - Gamma1 lambda) / Gamma0 = lambda + (v - Gamma~ lambda) / Gamma0
// (y = Gamma~ lambda); decoupled modes keep lambda = 0.
__global__ void bte_sc_update(long n, const double* __restrict__ rhs,
                              const double* __restrict__ g0, const double* __restrict__ omega,
                              const double* __restrict__ gmax, double nu_min,
                              const double* __restrict__ y, double* __restrict__ lam) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (!bte_active(omega[i], g0[i], *gmax, nu_min)) return;
  for (int c = 0; c < 3; ++c) lam[3 * i + c] += (rhs[3 * i + c] - y[3 * i + c]) / g0[i];
}

// ------------------------------------------------------------------ host

struct BteWs {
  size_t off_occ, off_phys, off_act, off_rows, off_count, off_tr, off_phase, off_gmax, off_rhs,
      off_lam, off_y, off_y2,
      off_linv, off_uinv, off_kappa, total;
};

static BteWs bte_ws(const kaldo_crystal* c, long nq) {
  const long n = nq * c->nb3;
  const long nb = (n + kLuB - 1) / kLuB;
  BteWs w;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t r = o;
    o += (bytes + 255) / 256 * 256;
    return r;
  };
  w.off_occ = take(8 * n);
  w.off_phys = take(n);
  w.off_act = take(n);
  w.off_rows = take(4 * n);
  w.off_count = take(4);
  w.off_tr = take(4 * n);
  w.off_phase = take(16 * nq * (size_t)std::max(1, c->bloch.n_d));
  w.off_gmax = take(8);
  w.off_rhs = take(24 * n);
  w.off_lam = take(24 * n);
  w.off_y = take(24 * n);
  w.off_y2 = take(24 * n);
  w.off_linv = take(8 * kLuB * kLuB * nb);
  w.off_uinv = take(8 * kLuB * kLuB * nb);
  w.off_kappa = take(8 * 9);
  w.total = o;
  return w;
}

static bool bte_supported(const kaldo_crystal* c) {
  if (c->nb3 != 3 && c->nb3 != 6) return false;
  return (size_t)c->bloch.n_blk * 9 * c->nb3 * 16 <= 64 * 1024 && c->n_rep <= 64;
}

// near_tab [branch][q]: the FP32 frequency (NaN below nu_min) and an upper
// bound of |v| h / sqrt(12), the mode's share of an adaptive width.
__global__ void bte_prepare(int nq, int nb3, const double* __restrict__ omega,
                            const double* __restrict__ vel, double inv_kt_hbar, double nu_min,
                            float hs, double* __restrict__ occ, uint8_t* __restrict__ phys,
                            float2* __restrict__ near_tab, int32_t* __restrict__ flags) {
  const int n_modes = nq * nb3;
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_modes) return;
  const double w = omega[m];
  const bool p = (w / kTwoPi) >= nu_min;
  phys[m] = p;
  occ[m] = p ? 1.0 / expm1(w * inv_kt_hbar) : 0.0;
  const double* v = vel + 3 * (size_t)m;
  const float speed = (float)sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  near_tab[(size_t)(m % nb3) * nq + m / nb3] =
      make_float2(p ? (float)w : __builtin_nanf(""), speed * hs * 1.000001f);
  if (!(w - w == 0.0)) raise_flag(flags, kFlagNonFinite);
  if (w < 0.0 && (-w / kTwoPi) >= nu_min) raise_flag(flags, kFlagImaginary);
}

static int check_common(const kaldo_crystal* c, const int32_t* mesh, double T, long* nq_out) {
  KALDO_REQUIRE(c && mesh, "bte: NULL argument");
  KALDO_REQUIRE(mesh[0] >= 1 && mesh[1] >= 1 && mesh[2] >= 1, "bte: mesh must be >= 1");
  KALDO_REQUIRE(std::isfinite(T) && T > 0, "bte: temperature <= 0");
  const long nq = (long)mesh[0] * mesh[1] * mesh[2];
  KALDO_REQUIRE(nq <= 65535L, "bte: mesh too large (N_q > 65535)");
  *nq_out = nq;
  return KALDO_OK;
}

}  // namespace kaldo

using namespace kaldo;

extern "C" size_t kaldo_bte_workspace(const kaldo_crystal* c, const int32_t* mesh) {
  if (!c || !mesh || mesh[0] < 1 || mesh[1] < 1 || mesh[2] < 1) return 0;
  return bte_ws(c, (long)mesh[0] * mesh[1] * mesh[2]).total;
}

extern "C" int kaldo_scattering_matrix(const kaldo_crystal* c, const int32_t* mesh,
                                       const double* omega, const double* evec, const double* vel,
                                       double temperature, const kaldo_broadening* b,
                                       void* workspace, size_t workspace_bytes, double* matrix,
                                       double* gamma0, void* stream) {
  long nq = 0;
  int rc = check_common(c, mesh, temperature, &nq);
  if (rc) return rc;
  KALDO_REQUIRE(omega && evec && vel && b && matrix && gamma0, "kaldo_scattering_matrix: NULL argument");
  rc = check_broadening(b, true);
  if (rc) return rc;
  if (!bte_supported(c)) {
    set_error("kaldo_scattering_matrix: implemented for cells of 1 or 2 atoms whose folded FC3 fits 64 KB of LDS");
    return KALDO_EUNSUPPORTED;
  }
  const BteWs w = bte_ws(c, nq);
  KALDO_REQUIRE(workspace && workspace_bytes >= w.total, "kaldo_scattering_matrix: workspace too small");
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto* ws = static_cast<unsigned char*>(workspace);
  const int nb3 = c->nb3;
  const long n = nq * nb3;
  double* occ = reinterpret_cast<double*>(ws + w.off_occ);
  uint8_t* phys = ws + w.off_phys;
  uint8_t* act = ws + w.off_act;
  int32_t* tr = reinterpret_cast<int32_t*>(ws + w.off_tr);
  double2* phase = reinterpret_cast<double2*>(ws + w.off_phase);
  // in the place of the solve's right-hand sides (24 bytes a mode)
  float2* near_tab = reinterpret_cast<float2*>(ws + w.off_rhs);
  double* gmax = reinterpret_cast<double*>(ws + w.off_gmax);
  LwParams p = make_params(c, mesh, temperature, b);
  KALDO_LAUNCH("bte_prepare", bte_prepare, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
               (int)nq, nb3, omega, vel, kHbar / (kKb * temperature), b->nu_min_thz,
               p.adaptive ? (float)std::sqrt(p.h2 / 12.0) : 0.0f, occ, phys, near_tab, c->d_flags);
  KALDO_LAUNCH("bte_tr_map", bte_tr_map, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
               (int)nq, nb3, mesh[0], mesh[1], mesh[2], evec, tr);
  const long nph = nq * std::max(1, p.n_d);
  KALDO_LAUNCH("lw_phase_table", lw_phase_table<double>, dim3((unsigned)((nph + 255) / 256)),
               dim3(256), 0, st, (int)nq, p.n_d, mesh[0], mesh[1], mesh[2], c->bloch.dvec, phase);
  const size_t n2 = (size_t)n * n;
  KALDO_LAUNCH("bte_zero", bte_zero, dim3((unsigned)std::min<size_t>((n2 + 255) / 256, 1u << 20)),
               dim3(256), 0, st, n2, matrix);
  const size_t lds = (size_t)c->bloch.n_blk * 9 * nb3 * sizeof(double2);
  const double pref = 2.0 * kPrefactor / (double)nq;
  const Fc3Bloch& bl = c->bloch;
  if (nb3 == 6)
    KALDO_LAUNCH("bte_rows", bte_rows<6>, dim3((unsigned)nq), dim3(64 * kRowWaves), lds, st, p, c->n_rep,
                 c->d_rep, omega, vel, occ, phys, evec, near_tab, phase, bl.n_blk, bl.e_blk, bl.e_bg,
                 bl.blk_d, bl.pair_ptr, bl.t_ptr, bl.t_i, bl.t_l2, bl.t_coef, tr, pref, matrix,
                 gamma0);
  else
    KALDO_LAUNCH("bte_rows", bte_rows<3>, dim3((unsigned)nq), dim3(64 * kRowWaves), lds, st, p, c->n_rep,
                 c->d_rep, omega, vel, occ, phys, evec, near_tab, phase, bl.n_blk, bl.e_blk, bl.e_bg,
                 bl.blk_d, bl.pair_ptr, bl.t_ptr, bl.t_i, bl.t_l2, bl.t_coef, tr, pref, matrix,
                 gamma0);
  KALDO_LAUNCH("bte_gmax", bte_gmax, dim3(1), dim3(1024), 0, st, n, gamma0, gmax);
  KALDO_LAUNCH("bte_flags", bte_flags, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n,
               omega, gamma0, gmax, b->nu_min_thz, act);
  KALDO_LAUNCH("bte_decouple", bte_decouple, dim3((unsigned)n), dim3(256), 0, st, n, act, matrix);
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}

static int bte_solve_common(const kaldo_crystal* c, const int32_t* mesh, const double* omega,
                            const double* vel, const double* gamma0, double T, double nu_min,
                            void* workspace, size_t workspace_bytes, const BteWs& w, long nq,
                            hipStream_t st) {
  KALDO_REQUIRE(omega && vel && gamma0, "bte: NULL argument");
  KALDO_REQUIRE(std::isfinite(nu_min) && nu_min >= 0, "bte: nu_min_thz < 0");
  KALDO_REQUIRE(workspace && workspace_bytes >= w.total, "bte: workspace too small");
  auto* ws = static_cast<unsigned char*>(workspace);
  const long n = nq * c->nb3;
  double* gmax = reinterpret_cast<double*>(ws + w.off_gmax);
  double* rhs = reinterpret_cast<double*>(ws + w.off_rhs);
  (void)mesh;
  (void)T;
  KALDO_LAUNCH("bte_gmax", bte_gmax, dim3(1), dim3(1024), 0, st, n, gamma0, gmax);
  KALDO_LAUNCH("bte_rhs", bte_rhs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, omega,
               vel, gamma0, gmax, nu_min, rhs);
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}

extern "C" int kaldo_bte_solve(const kaldo_crystal* c, const int32_t* mesh, const double* omega,
                               const double* vel, const double* gamma0, double temperature,
                               double nu_min_thz, double* matrix, void* workspace,
                               size_t workspace_bytes, double* lambda, double* kappa,
                               void* stream) {
  long nq = 0;
  int rc = check_common(c, mesh, temperature, &nq);
  if (rc) return rc;
  KALDO_REQUIRE(matrix && lambda && kappa, "kaldo_bte_solve: NULL argument");
  const BteWs w = bte_ws(c, nq);
  hipStream_t st = static_cast<hipStream_t>(stream);
  rc = bte_solve_common(c, mesh, omega, vel, gamma0, temperature, nu_min_thz, workspace,
                        workspace_bytes, w, nq, st);
  if (rc) return rc;
  auto* ws = static_cast<unsigned char*>(workspace);
  const long n_all = nq * c->nb3;
  double* linv = reinterpret_cast<double*>(ws + w.off_linv);
  double* uinv = reinterpret_cast<double*>(ws + w.off_uinv);
  double* rhs = reinterpret_cast<double*>(ws + w.off_rhs);
  double* lam_c = reinterpret_cast<double*>(ws + w.off_lam);
  double* y = reinterpret_cast<double*>(ws + w.off_y);
  double* gmax = reinterpret_cast<double*>(ws + w.off_gmax);
  uint8_t* act = ws + w.off_act;
  int32_t* rows = reinterpret_cast<int32_t*>(ws + w.off_rows);
  int32_t* count = reinterpret_cast<int32_t*>(ws + w.off_count);
  const size_t blk = (size_t)kLuB * kLuB;
  // The decoupled modes (unit diagonal, zero row and column, lambda = 0)
  // drop out: the factorisation runs on the coupled block only, reached
  // through the row map and with its columns moved to the front of each
  // row.  The host learns the coupled count (one synchronisation).
  KALDO_LAUNCH("bte_flags", bte_flags, dim3((unsigned)((n_all + 255) / 256)), dim3(256), 0, st,
               n_all, omega, gamma0, gmax, nu_min_thz, act);
  KALDO_LAUNCH("bte_compact_index", bte_compact_index, dim3(1), dim3(1024), 0, st, n_all, act,
               rows, count);
  int32_t n_coupled = 0;
  KALDO_HIP(hipMemcpyAsync(&n_coupled, count, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  KALDO_HIP(hipStreamSynchronize(st));
  const long n = n_coupled;
  const dim3 g3all((unsigned)((3 * n_all + 255) / 256));
  KALDO_LAUNCH("bte_zero", bte_zero, g3all, dim3(256), 0, st, (size_t)(3 * n_all), lambda);
  if (n > 0) {
    const MatRows A{matrix, rows, n_all};
    KALDO_LAUNCH("bte_compact_cols", bte_compact_cols, dim3((unsigned)n), dim3(256), 0, st, n,
                 n_all, rows, matrix);
    const int nb = (int)((n + kLuB - 1) / kLuB);
    // Blocked LU in panels of kLuPanel blocks: inside a panel left-looking, a
    // step's row and column of blocks take the panel's earlier steps when
    // their turn comes; the rest of the trailing matrix takes one
    // rank-(64 kLuPanel) product per panel (lu_gemm).
    for (int k0 = 0; k0 < nb; k0 += kLuPanel) {
      const int k1 = std::min(nb, k0 + kLuPanel);
      for (int k = k0; k < k1; ++k) {
        const int m = nb - k - 1;
        KALDO_LAUNCH("lu_left", lu_left, dim3(k > k0 ? 2 * m + 1 : 1), dim3(256), 0, st, n, nb, k0, k, A,
                     linv + k * blk, uinv + k * blk, c->d_flags);
        if (m > 0)
          KALDO_LAUNCH("lu_panels", lu_panels, dim3(2 * m), dim3(256), 0, st, n, nb, k, A,
                       linv + k * blk, uinv + k * blk);
      }
      if (k1 < nb) {
        const long r0 = (long)k1 * kLuB;
        const int ntl = (int)((n - r0 + kLgT - 1) / kLgT);
        KALDO_LAUNCH("lu_gemm", lu_gemm, dim3((unsigned)(ntl * ntl)), dim3(256), 0, st, n, r0,
                     (long)k0 * kLuB, (k1 - k0) * kLuB, ntl, A);
      }
    }
    // the coupled right-hand sides, then forward: y = L^-1 b, the residual in
    // y2 (starting as b)
    double* r = reinterpret_cast<double*>(ws + w.off_y2);
    const dim3 g3((unsigned)((3 * n + 255) / 256));
    KALDO_LAUNCH("bte_gather3", bte_gather3, g3, dim3(256), 0, st, n, rows, rhs, r);
    auto rest = [&](long i0, long i1, long c0, long c1, double* sol) {
      if (i1 > i0)
        KALDO_LAUNCH("lu_solve_rest", lu_solve_rest, dim3((unsigned)((i1 - i0 + 15) / 16)), dim3(256), 0, st,
                     i0, i1, c0, c1, A, sol, r);
    };
    const int last = (nb - 1) / kLuPanel * kLuPanel;
    for (int k0 = 0; k0 < nb; k0 += kLuPanel) {
      const int k1 = std::min(nb, k0 + kLuPanel);
      KALDO_LAUNCH("lu_solve", lu_solve<true>, dim3(1), dim3(1024), 0, st, n, k0, k1, linv, A, y, r);
      rest((long)k1 * kLuB, n, (long)k0 * kLuB, std::min(n, (long)k1 * kLuB), y);
    }
    // backward: lambda = U^-1 y, the residual in y2 (starting as y)
    KALDO_LAUNCH("bte_copy3", bte_copy3, g3, dim3(256), 0, st, n, y, r);
    for (int k0 = last; k0 >= 0; k0 -= kLuPanel) {
      const int k1 = std::min(nb, k0 + kLuPanel);
      KALDO_LAUNCH("lu_solve", lu_solve<false>, dim3(1), dim3(1024), 0, st, n, k0, k1, uinv, A, lam_c, r);
      rest(0, (long)k0 * kLuB, (long)k0 * kLuB, std::min(n, (long)k1 * kLuB), lam_c);
    }
    KALDO_LAUNCH("bte_scatter3", bte_scatter3, g3, dim3(256), 0, st, n, rows, lam_c, lambda);
  }
  const double scale = kKappaUnit / ((double)nq * c->volume);
  KALDO_LAUNCH("bte_kappa", bte_kappa, dim3(1), dim3(1024), 0, st, n_all, omega, vel, lambda, gamma0,
               gmax, kHbar / (kKb * temperature), nu_min_thz, scale, kappa);
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}

extern "C" int kaldo_bte_iterate(const kaldo_crystal* c, const int32_t* mesh, const double* omega,
                                 const double* vel, const double* gamma0, double temperature,
                                 double nu_min_thz, const double* matrix, int32_t n_iterations,
                                 double tolerance, void* workspace, size_t workspace_bytes,
                                 double* lambda, double* kappa, int32_t* iterations,
                                 void* stream) {
  long nq = 0;
  int rc = check_common(c, mesh, temperature, &nq);
  if (rc) return rc;
  KALDO_REQUIRE(matrix && lambda && kappa, "kaldo_bte_iterate: NULL argument");
  KALDO_REQUIRE(n_iterations >= 0 && std::isfinite(tolerance) && tolerance >= 0,
                "kaldo_bte_iterate: bad n_iterations or tolerance");
  const BteWs w = bte_ws(c, nq);
  hipStream_t st = static_cast<hipStream_t>(stream);
  rc = bte_solve_common(c, mesh, omega, vel, gamma0, temperature, nu_min_thz, workspace,
                        workspace_bytes, w, nq, st);
  if (rc) return rc;
  auto* ws = static_cast<unsigned char*>(workspace);
  const long n = nq * c->nb3;
  double* rhs = reinterpret_cast<double*>(ws + w.off_rhs);
  double* y = reinterpret_cast<double*>(ws + w.off_y);
  double* gmax = reinterpret_cast<double*>(ws + w.off_gmax);
  double* kap_ws = reinterpret_cast<double*>(ws + w.off_kappa);
  const double scale = kKappaUnit / ((double)nq * c->volume);
  const double ikt = kHbar / (kKb * temperature);
  const dim3 g1((unsigned)((n + 255) / 256));
  KALDO_LAUNCH("bte_sc_init", bte_sc_init, g1, dim3(256), 0, st, n, rhs, gamma0, lambda);
  KALDO_LAUNCH("bte_kappa", bte_kappa, dim3(1), dim3(1024), 0, st, n, omega, vel, lambda, gamma0,
               gmax, ikt, nu_min_thz, scale, kap_ws);
  double kh[9];
  KALDO_HIP(hipMemcpyAsync(kh, kap_ws, sizeof(kh), hipMemcpyDeviceToHost, st));
  KALDO_HIP(hipStreamSynchronize(st));
  double k_prev = (kh[0] + kh[4] + kh[8]) / 3.0;
  int it = 0;
  bool conv = false;
  while (it < n_iterations) {
    KALDO_LAUNCH("bte_gemv", bte_gemv, dim3((unsigned)n), dim3(256), 0, st, n, matrix, lambda, y);
    KALDO_LAUNCH("bte_sc_update", bte_sc_update, g1, dim3(256), 0, st, n, rhs, gamma0, omega, gmax,
                 nu_min_thz, y, lambda);
    KALDO_LAUNCH("bte_kappa", bte_kappa, dim3(1), dim3(1024), 0, st, n, omega, vel, lambda, gamma0,
                 gmax, ikt, nu_min_thz, scale, kap_ws);
    KALDO_HIP(hipMemcpyAsync(kh, kap_ws, sizeof(kh), hipMemcpyDeviceToHost, st));
    KALDO_HIP(hipStreamSynchronize(st));
    ++it;
    const double k_new = (kh[0] + kh[4] + kh[8]) / 3.0;
    const bool stop = std::fabs(k_new - k_prev) <= tolerance * std::fabs(k_prev);
    k_prev = k_new;
    if (stop) {
      conv = true;
      break;
    }
  }
  KALDO_HIP(hipMemcpyAsync(kappa, kap_ws, sizeof(kh), hipMemcpyDeviceToDevice, st));
  KALDO_HIP(hipStreamSynchronize(st));
  if (iterations) *iterations = it;
  if (!conv || !std::isfinite(k_prev)) {
    set_error("kaldo_bte_iterate: no convergence within n_iterations (the iteration contracts only "
              "when the off-diagonal part is small against the diagonal); kappa is the last iterate's");
    return KALDO_ENUMERIC;
  }
  return KALDO_OK;
}
