// Isotope (mass-disorder) scattering of a crystal on a Gamma-centred mesh.
//
// Paper: Eq. isotope (Tamura's perturbation theory):
//   gamma_iso(q,s) = pi/(2 N_q) w^2 sum_{q' s'} delta(w - w')
//                    sum_i g_i |sum_a eta*_{ia}(q,s) eta_{ia}(q',s')|^2
// with the Cartesian sum inside the modulus (the form that does not depend on
// the orientation of the Cartesian axes), delta the smearing of Eq.
// broadening with its 2 sigma cut, partners and modes below nu_min excluded,
// and for the adaptive width sigma = max(floor, |v(q',s')| h / sqrt(12)) (the
// rate at which w - w' varies with the summed q').  gamma_iso is a linewidth
// in the convention of Eq. gamma, to which it adds (Eq. lifetime).
//
//   iso_order    per branch the q-points in order of frequency, by rank (how
//                many keys are smaller), and everything the sum reads of a
//                mode stored at its place in that order: w (NaN below
//                nu_min), sigma, its factors, the eigenvector by component;
//                input checks
//   iso_ranges   per (tile of partners in that order, branch): the frequency
//                range of its physical modes and their largest sigma, a wave
//                per tile
//   iso_kernel   one workgroup per four modes of a branch adjacent in that order
//                (nearly equal frequencies: they share each partner's loads):
//                first which tiles can meet the cut, a lane per tile, then
//                those tiles dealt to the waves in turn: lanes over the tile's
//                partners, exact FP64 cut per mode and partner, overlap and
//                smearing in FP64, per-lane sums in tile order, fixed wave
//                reduction per mode
//
// What bounds the sum: FP64 arithmetic, 84 % of the vector ALU's issue slots
// (diamond 24^3: 2.16 ms, 2.49 with the live tiles of each branch searched and
// dealt by themselves, 3.2 with a wave per group of modes and the vectors kept
// in registers).  A bitonic sort of the keys in one workgroup per branch, the
// ranges one thread per tile and a launch for the largest sigma' took 105 us
// on the diamond 15^3 mesh, the ranks and ranges 31.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "lw_common.h"

namespace kaldo {

constexpr int kIsoMaxBasis = 5;          // 3 N_b <= 16
constexpr size_t kIsoRanges = 48 << 10;  // bytes of the range table: 24 a tile of a branch
constexpr int kIsoWords = kIsoRanges / 24 / 64;  // and its tiles in words of 64, short of one a branch

struct IsoParams {
  int nq, nb3, nb, blk, nblk;  // blk: partner q-points per tile (a multiple of 64)
  int shape, adaptive;
  double sig_fixed, sig_floor, h2, nu_min, scale;  // scale = pi / (2 N_q)
  double g[kIsoMaxBasis];
};

// Place i of branch s holds the mode of q-point perm[s][i]: physical modes in
// ascending frequency (keys: the FP32 rounding of w, whose bits order like the
// values for w > 0, then q), the others last.  A workgroup ranks 64 modes of a
// branch, each wave against a quarter of the keys, which pass through LDS.
constexpr int kIsoKeys = 2048;

__global__ __launch_bounds__(256) void iso_order(IsoParams p, const double* __restrict__ omega,
                                                 const double* __restrict__ vel,
                                                 const double* __restrict__ evec,
                                                 double2* __restrict__ rec, double2* __restrict__ inv,
                                                 double2* __restrict__ eta, int32_t* __restrict__ perm,
                                                 int32_t* __restrict__ flags) {
  __shared__ unsigned long long keys[kIsoKeys];
  __shared__ int part[4][64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, s = blockIdx.y;
  const int q = blockIdx.x * 64 + lane;
  const bool in = q < p.nq;
  auto key = [&](int i) {
    const double w = omega[(size_t)i * p.nb3 + s];
    const bool first = (w / kTwoPi) >= p.nu_min && w > 0.0;
    return ((unsigned long long)(first ? __float_as_uint((float)w) : 0xffffffffu) << 32) | (unsigned)i;
  };
  const unsigned long long own = key(in ? q : 0);
  int below = 0;
  for (int base = 0; base < p.nq; base += kIsoKeys) {
    __syncthreads();
    for (int i = tid; i < kIsoKeys; i += 256) keys[i] = base + i < p.nq ? key(base + i) : ~0ull;
    __syncthreads();
    const int quarter = kIsoKeys / 4, n = min(quarter, max(0, p.nq - base - wv * quarter));
#pragma unroll 8
    for (int i = 0; i < (n + 7) / 8 * 8; ++i) below += keys[wv * quarter + i] < own ? 1 : 0;
  }
  part[wv][lane] = below;
  __syncthreads();
  if (!in) return;
  const int at = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
  const size_t row = (size_t)s * p.nq + at, m = (size_t)q * p.nb3 + s;
  double chk = 0.0;
  for (int j = wv; j < p.nb3; j += 4) {
    const size_t src = (((size_t)q * p.nb3 + j) * p.nb3 + s) * 2;
    const double re = evec[src], im = evec[src + 1];
    chk += (re - re) + (im - im);
    eta[((size_t)s * p.nb3 + j) * p.nq + at] = make_double2(re, im);
  }
  if (wv == 0) {
    const double w = omega[m], v0 = vel[3 * m], v1 = vel[3 * m + 1], v2 = vel[3 * m + 2];
    const bool phys = (w / kTwoPi) >= p.nu_min;
    double sig = p.sig_fixed;
    if (p.adaptive) sig = fmax(sqrt((v0 * v0 + v1 * v1 + v2 * v2) * p.h2 / 12.0), p.sig_floor);
    perm[row] = q;
    rec[row] = make_double2(phys ? w : __builtin_nan(""), sig);
    // 1/sigma and 1/(sqrt(pi) sigma) of the partner, once per mode
    inv[row] = make_double2(1.0 / sig, 1.0 / (kSqrtPi * sig));
    chk += (w - w) + (v0 - v0) + (v1 - v1) + (v2 - v2);
    if (w < 0.0 && (-w / kTwoPi) >= p.nu_min) raise_flag(flags, kFlagImaginary);
  }
  if (!(chk == 0.0)) raise_flag(flags, kFlagNonFinite);
}

// range[(s' * nblk + b)] = (lowest w, highest w, largest sigma) of the
// physical modes of branch s' in tile b of its order; an empty tile gets
// (+inf, -inf, 0).  Tiles run in frequency order, so lowest w does not
// decrease with b.
__global__ __launch_bounds__(256) void iso_ranges(IsoParams p, const double2* __restrict__ rec,
                                                  double* __restrict__ range) {
  const int lane = threadIdx.x & 63, k = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= p.nblk * p.nb3) return;
  const int s = k / p.nblk, b = k - s * p.nblk;
  double lo = INFINITY, hi = -INFINITY, smax = 0.0;
  for (int i = b * p.blk + lane; i < min(p.nq, (b + 1) * p.blk); i += 64) {
    const double2 r = rec[(size_t)s * p.nq + i];
    if (r.x == r.x) {  // physical (not NaN)
      lo = fmin(lo, r.x);
      hi = fmax(hi, r.x);
      smax = fmax(smax, r.y);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
    smax = fmax(smax, __shfl_xor(smax, off, 64));
  }
  if (lane == 0) {
    range[3 * (size_t)k] = lo;
    range[3 * (size_t)k + 1] = hi;
    range[3 * (size_t)k + 2] = smax;
  }
}

// Modes per workgroup: MPW modes of one branch at consecutive places of its
// order (nearly the same frequency, so nearly the same live tiles and passing
// partners) share every partner's record and eigenvector load (the diamond 15^3
// sum with the tiles of each branch dealt from the first wave on: two 296 us,
// three 253, four 234, six 226 with more registers than the larger cells have,
// eight 239).
constexpr int kIsoMpw = 4;

template <int NB3>
__global__ __launch_bounds__(256) void iso_kernel(IsoParams p, const double2* __restrict__ rec,
                                                  const double2* __restrict__ inv,
                                                  const double2* __restrict__ eta,
                                                  const double* __restrict__ range,
                                                  const int32_t* __restrict__ perm,
                                                  int accumulate, double* __restrict__ gamma) {
  constexpr int NB = NB3 / 3;
  constexpr int MPW = kIsoMpw;
  __shared__ unsigned long long live_lds[kIsoWords + NB3];  // bit b of word [s'][b/64]: tile b is live
  __shared__ double2 e0s[MPW][NB3];  // the modes' eigenvectors
  __shared__ double sums[4][MPW];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup -> (branch s, first position in the branch's frequency order):
  // neighbouring workgroups scan similar tiles.  Its waves take the tiles in
  // turn: with a group of modes per wave the groups of many partners left the
  // chip a quarter full (1.3 waves a SIMD on the diamond 15^3 mesh, 302 us)
  const int groups = (p.nq + MPW - 1) / MPW;
  const int s = blockIdx.x / groups;
  const int i0 = (blockIdx.x - s * groups) * MPW;
  double w[MPW];
  bool live_m[MPW];
  int qm[MPW];
#pragma unroll
  for (int k = 0; k < MPW; ++k) {
    const bool in = i0 + k < p.nq;
    qm[k] = in ? perm[(size_t)s * p.nq + i0 + k] : 0;
    const double2 r = in ? rec[(size_t)s * p.nq + i0 + k] : make_double2(__builtin_nan(""), 0.0);
    w[k] = r.x;
    live_m[k] = in && (r.x == r.x);
    if (in && wv == 0 && lane < NB3) e0s[k][lane] = eta[((size_t)s * NB3 + lane) * p.nq + i0 + k];
  }
  // the tiles that can hold a partner of one of the modes, |w - w'| < 2 sigma':
  // one lane tests one tile, each wave every fourth 64 of them, and the live
  // tiles are dealt to the waves in turn across the branches.  (With each wave
  // searching the run of live tiles of every branch in a copy of the table in
  // LDS, and the tiles of each branch dealt from the first wave on, calls of
  // three atoms and narrow cuts took 222 us on 15^3 and 1,170 on 24^3, now 136
  // and 838; the diamond 15^3 call 251, now 195.  Whole branches to the waves:
  // up to three times the time, the waves end far apart.)
  const int words = (p.nblk + 63) / 64;
  for (int t = wv; t < NB3 * words; t += 4) {
    const int s1 = t / words, b = (t - s1 * words) * 64 + lane;
    bool tile = false;
    if (b < p.nblk) {
      const double* r = range + 3 * ((size_t)s1 * p.nblk + b);
      const double lo = r[0], hi = r[1], reach = 2.0 * r[2] * (1.0 + 1e-12);
#pragma unroll
      for (int k = 0; k < MPW; ++k) tile |= live_m[k] && w[k] > lo - reach && w[k] < hi + reach;
    }
    const unsigned long long mask = __ballot(tile);
    if (lane == 0) live_lds[t] = mask;
  }
  __syncthreads();
  double acc[MPW];
#pragma unroll
  for (int k = 0; k < MPW; ++k) acc[k] = 0.0;
  int turn = 0;
  for (int s1 = 0; s1 < NB3; ++s1) {
    for (int word = 0; word < words; ++word) {
      const unsigned long long mask = live_lds[s1 * words + word];
      unsigned long long left =
          (unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(mask >> 32)) << 32 |
          (unsigned)__builtin_amdgcn_readfirstlane((unsigned)mask);
      while (left) {
        const int b = word * 64 + __builtin_ctzll(left);
        left &= left - 1;
        if ((turn++ & 3) != wv) continue;
        for (int i1 = b * p.blk + lane; i1 < min(p.nq, (b + 1) * p.blk); i1 += 64) {
          const size_t m1 = (size_t)s1 * p.nq + i1;
          asm volatile("" ::: "memory");  // the modes' vectors from LDS again: kept in registers they cost a wave a SIMD
          // every load of the partner at once, whether it passes or not
          const double2 o = rec[m1], iv = inv[m1];
          double2 e1[NB3];
#pragma unroll
          for (int j = 0; j < NB3; ++j) e1[j] = eta[((size_t)s1 * NB3 + j) * p.nq + i1];
          bool pass[MPW];
          bool any = false;
#pragma unroll
          for (int k = 0; k < MPW; ++k) {
            pass[k] = live_m[k] && fabs(w[k] - o.x) < 2.0 * o.y;  // fails for partners below nu_min (NaN)
            any |= pass[k];
          }
          if (!any) continue;
#pragma unroll
          for (int k = 0; k < MPW; ++k) {
            if (!pass[k]) continue;
            double ov = 0.0;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              double dr = 0.0, di = 0.0;
#pragma unroll
              for (int a = 0; a < 3; ++a) {
                const double2 u = e0s[k][3 * i + a], v = e1[3 * i + a];
                // conj(u) v, as fused multiply-adds into the sums
                dr = fma(u.x, v.x, dr);
                dr = fma(u.y, v.y, dr);
                di = fma(u.x, v.y, di);
                di = fma(-u.y, v.x, di);
              }
              ov += p.g[i] * (dr * dr + di * di);
            }
            const double x = w[k] - o.x;
            double d;
            if (p.shape == KALDO_GAUSS) {
              const double u = x * iv.x;
              d = exp(-(u * u)) * iv.y;
            } else {
              d = smear(p.shape, x, o.y);
            }
            acc[k] += d * ov;
          }
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < MPW; ++k) {
    const double v = wave_sum_fixed(acc[k]);
    if (lane == 0) sums[wv][k] = v;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < MPW; ++k) {
    if ((int)threadIdx.x != k || i0 + k >= p.nq) continue;
    const double v = ((sums[0][k] + sums[1][k]) + sums[2][k]) + sums[3][k];
    const size_t m = (size_t)qm[k] * NB3 + s;
    if (live_m[k]) {
      const double gi = p.scale * w[k] * w[k] * v;
      gamma[m] = accumulate ? gamma[m] + gi : gi;
    } else if (!accumulate) {
      gamma[m] = 0.0;  // below nu_min: no linewidth
    }
  }
}

struct IsoWs {
  int blk, nblk;
  size_t off_rec, off_inv, off_eta, off_range, off_perm, total;
};

static IsoWs iso_ws(long nq, int nb3) {
  IsoWs w{};
  // tiles of 64 q-points, widened until the range table and the words of live
  // tiles stay small
  int blk = 64;
  while (((nq + blk - 1) / blk) * (size_t)nb3 * 3 * sizeof(double) > kIsoRanges) blk += 64;
  w.blk = blk;
  w.nblk = (int)((nq + blk - 1) / blk);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t r = o;
    o += (bytes + 255) / 256 * 256;
    return r;
  };
  w.off_rec = take(sizeof(double2) * nq * nb3);
  w.off_inv = take(sizeof(double2) * nq * nb3);
  w.off_eta = take(sizeof(double2) * nq * nb3 * nb3);
  w.off_range = take(sizeof(double) * 3 * (size_t)w.nblk * nb3);
  w.off_perm = take(sizeof(int32_t) * (size_t)nq * nb3);
  w.total = o;
  return w;
}

}  // namespace kaldo

using namespace kaldo;

extern "C" size_t kaldo_isotope_workspace(const kaldo_crystal* c, const int32_t* mesh) {
  if (!c || !mesh || mesh[0] < 1 || mesh[1] < 1 || mesh[2] < 1) return 0;
  return iso_ws((long)mesh[0] * mesh[1] * mesh[2], c->nb3).total;
}

extern "C" int kaldo_isotope_linewidths(const kaldo_crystal* c, const int32_t* mesh,
                                        const double* omega, const double* evec,
                                        const double* vel, const double* g_factor,
                                        const kaldo_broadening* b, int32_t accumulate,
                                        void* workspace, size_t workspace_bytes, double* gamma,
                                        void* stream) {
  KALDO_REQUIRE(c && mesh && omega && evec && vel && g_factor && b && gamma,
                "kaldo_isotope_linewidths: NULL argument");
  KALDO_REQUIRE(mesh[0] >= 1 && mesh[1] >= 1 && mesh[2] >= 1,
                "kaldo_isotope_linewidths: mesh must be >= 1");
  KALDO_REQUIRE(c->nb <= kIsoMaxBasis, "kaldo_isotope_linewidths: more than 5 basis atoms");
  KALDO_REQUIRE(accumulate == 0 || accumulate == 1, "kaldo_isotope_linewidths: accumulate must be 0 or 1");
  int rc = check_broadening(b, true);
  if (rc) return rc;
  for (int i = 0; i < c->nb; ++i)
    KALDO_REQUIRE(std::isfinite(g_factor[i]) && g_factor[i] >= 0,
                  "kaldo_isotope_linewidths: g_factor must be finite and >= 0");
  const long nq = (long)mesh[0] * mesh[1] * mesh[2];
  KALDO_REQUIRE(nq <= 65535L, "kaldo_isotope_linewidths: mesh too large (N_q > 65535)");
  const IsoWs w = iso_ws(nq, c->nb3);
  KALDO_REQUIRE(workspace && workspace_bytes >= w.total,
                "kaldo_isotope_linewidths: workspace too small");
  hipStream_t st = static_cast<hipStream_t>(stream);
  IsoParams p{};
  p.nq = (int)nq;
  p.nb3 = c->nb3;
  p.nb = c->nb;
  p.blk = w.blk;
  p.nblk = w.nblk;
  p.shape = b->shape;
  p.adaptive = b->adaptive;
  p.sig_fixed = kTwoPi * b->sigma_thz;
  p.sig_floor = kTwoPi * b->sigma_floor_thz;
  p.nu_min = b->nu_min_thz;
  p.scale = kPi / (2.0 * (double)nq);
  {
    double rc9[9];
    reciprocal(c->lattice, rc9);
    double h2 = 0.0;
    for (int r = 0; r < 3; ++r)
      for (int k = 0; k < 3; ++k) {
        const double x = rc9[3 * r + k] / mesh[r];
        h2 += x * x;
      }
    p.h2 = h2 / 3.0;
  }
  for (int i = 0; i < c->nb; ++i) p.g[i] = g_factor[i];
  auto* ws = static_cast<unsigned char*>(workspace);
  auto* rec = reinterpret_cast<double2*>(ws + w.off_rec);
  auto* inv = reinterpret_cast<double2*>(ws + w.off_inv);
  auto* eta = reinterpret_cast<double2*>(ws + w.off_eta);
  auto* range = reinterpret_cast<double*>(ws + w.off_range);
  auto* perm = reinterpret_cast<int32_t*>(ws + w.off_perm);
  KALDO_LAUNCH("iso_order", iso_order, dim3((unsigned)((nq + 63) / 64), (unsigned)c->nb3), dim3(256), 0, st,
               p, omega, vel, evec, rec, inv, eta, perm, c->d_flags);
  KALDO_LAUNCH("iso_ranges", iso_ranges, dim3((p.nblk * p.nb3 + 3) / 4), dim3(256), 0, st, p, rec, range);
  const long n_groups = (long)c->nb3 * ((nq + kIsoMpw - 1) / kIsoMpw);
  const dim3 grid((unsigned)n_groups);
#define KALDO_ISO_CASE(NB3V)                                                                   \
  case NB3V:                                                                                   \
    KALDO_LAUNCH("iso_kernel", iso_kernel<NB3V>, grid, dim3(256), 0, st, p, rec, inv, eta, range, \
                 perm, accumulate, gamma);                                                     \
    break;
  switch (c->nb3) {
    KALDO_ISO_CASE(3)
    KALDO_ISO_CASE(6)
    KALDO_ISO_CASE(9)
    KALDO_ISO_CASE(12)
    KALDO_ISO_CASE(15)
    default:
      set_error("kaldo_isotope_linewidths: unsupported branch count");
      return KALDO_EUNSUPPORTED;
  }
#undef KALDO_ISO_CASE
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}
