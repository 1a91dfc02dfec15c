// Crystal linewidths with the dense per-(q, q1) eigenvector contractions on
// the matrix cores (cells with up to 16 branches, zero-padded to 16).
//
// Paper: Eq. phi3_proj evaluated as in its "Computational Implementation":
// the home-cell contraction with eta(q) first (A~_q, in LDS), then for every
// partner q1 and branch s the two dense products
//     T_s = B_s eta(q2),   V_s = eta(q1)^T T_s,
//     B_s[jc][kc] = sum_d e^{-i q1.R_d} A~_q[d][jc][kc][s],
// followed by Eq. gamma / Eq. broadening / Eq. bose for all (s', s'') in FP64.
//
// A complex 16x16x16 product is two real products with the complex parts
// stacked along K (K = 32):  Re C = [Re A | -Im A][Re B ; Im B] and
// Im C = [Im A | Re A][Re B ; Im B].
//   FP64 form:  v_mfma_f64_16x16x4_f64, FP32 form: v_mfma_f32_16x16x4_f32,
//               8 per real product.
//   BF16x3:     v_mfma_f32_16x16x32_bf16 on x = hi + lo splits,
//               hi*hi + hi*lo + lo*hi per real product, FP32 accumulation.
// One workgroup per (q, group of branches), one workgroup a CU; each wave
// takes its own partners q1.  With Phi3 symmetric in its last two slots the
// tile of the mirrored partner (q2, q1) is V^T, so only q1 <_lex q2 is swept
// (q1 == q2 once) and each candidate carries the terms of both orderings.
//
// What bounds it: the FP64 and FP32 matrix instructions run at the vector
// rate and hold the vector unit while they do (a wave of MFMAs beside a wave
// of fused multiply-adds takes the sum of both times), so a (partner, branch)
// costs its 32 MFMAs (1024 cycles in FP32, 2048 in FP64) plus every vector
// instruction around them.  Hence B_s is built in operand order with the
// table's values loaded a branch ahead and no masks (16 steps of four fused
// multiply-adds; a padded slot meets a zero phase), partners are decoded 64
// at a time one per lane, nothing is projected for a branch without a
// candidate, and the candidates of a partner's branches are weighted together,
// one exponential a loop trip.  Measured, abx3 cell (15 branches):
//   FP32, 12^3 mesh:        33.5 -> 21.2 ms (8 waves and a work item per q before);
//   BF16x3, 11x9x7 mesh:    5.4 -> 4.0 ms;
//   FP64, 7x6x5 mesh:       126 ms (generic kernel, per-lane gathers) -> 0.78 ms.
// FP32 runs 12 waves (three a SIMD; 22.7 ms with eight, phases in registers),
// FP64 and the split form eight (their registers).
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "common.h"
#include "lw_common.h"

namespace kaldo {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4;

enum DenseForm { kF64 = 0, kF32 = 1, kSplit = 2 };
constexpr int kAccSlots = 16;   // sums a wave keeps per branch: lanes l, l + 16, ... share one in turn
constexpr int kTileCand = 256;  // queue slots of a wave: one branch's candidates always fit

typedef __attribute__((__vector_size__(4 * sizeof(double)))) double d4;
__device__ __forceinline__ d4 mma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mma(bf16x8 a, bf16x8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// x = hi + lo in bf16, rounded two values an instruction.
typedef float f8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void split8(f8 x, bf16x8& hi, bf16x8& lo) {
  const bf16v8 h = __builtin_convertvector(x, bf16v8);
  const bf16v8 l = __builtin_convertvector(x - __builtin_convertvector(h, f8), bf16v8);
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}
// kWaves: waves of a workgroup, of which a CU holds one
template <int FORM>
struct Dense {
  using T = float;
  using V4 = f4;
  static constexpr int kWaves = FORM == kF32 ? 12 : 8;
};
template <>
struct Dense<kF64> {
  using T = double;
  using V4 = d4;
  static constexpr int kWaves = 8;
};

// Steps of a B_s entry: the blocks of an atom pair, padded to a multiple of
// four.  With four (nearest-neighbour tables; the FOUR kernels) a partner's
// phases are kept per pair, zero past its blocks; otherwise per block, with
// one zero phase after the last.
__host__ __device__ inline int tile_slots(int max_pair_blk) { return (max_pair_blk + 3) / 4 * 4; }
__host__ __device__ inline int tile_phases(int nb, int n_blk, int n_slot) {
  return n_slot == 4 ? nb * nb * 4 : n_blk + 1;
}

// LDS of lw_tiles besides the A~ table, in bytes.  Per wave: the phases of
// the current partner, the mode data of its two q-points, the candidate queue, the sums
// [branch][kAccSlots] and, in the split form, a B_s tile.
template <int FORM>
__host__ __device__ inline size_t tile_wave_lds(int group, int n_ph) {
  const size_t cs = sizeof(typename Cx<typename Dense<FORM>::T>::type);
  return n_ph * cs + 2 * 16 * 5 * 8 + kTileCand * (cs + 2) + group * kAccSlots * 8 +
         (FORM == kSplit ? (16 * 17 + 1) * cs : 0);
}

template <int FORM, bool FOUR>
__global__ __launch_bounds__(64 * Dense<FORM>::kWaves)
__attribute__((amdgpu_waves_per_eu(Dense<FORM>::kWaves / 4))) void lw_tiles(
    LwParams p, int n_rep, int group, int n_group, int n_slot, const int32_t* __restrict__ rep,
    const double* __restrict__ omega, const double* __restrict__ vel,
    const float4* __restrict__ modef, const double* __restrict__ occ,
    const uint8_t* __restrict__ phys, const uint8_t* __restrict__ sel,
    const double* __restrict__ evec, const typename Cx<typename Dense<FORM>::T>::type* __restrict__ phase_tab,
    const int32_t* __restrict__ t_ptr, const int32_t* __restrict__ t_i,
    const int32_t* __restrict__ t_l2, const double* __restrict__ t_coef,
    const int32_t* __restrict__ e_blk, const int32_t* __restrict__ e_bg,
    const int32_t* __restrict__ blk_d, const int32_t* __restrict__ pair_ptr,
    const int32_t* __restrict__ bwork, double scale, double* __restrict__ gamma) {
  using T = typename Dense<FORM>::T;
  using V4 = typename Dense<FORM>::V4;
  using C = typename Cx<T>::type;
  constexpr int kTileWaves = Dense<FORM>::kWaves, kTileThreads = 64 * kTileWaves;
  constexpr bool kSpl = FORM == kSplit;
  constexpr bool kAhead = FOUR && !kSpl;  // the split form has no registers to load ahead
  const int NB3 = p.nb3, NB = NB3 / 3;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: partner indices stay scalar
  const int lr = lane & 15, lg = lane >> 4;
  const int q = blockIdx.x / n_group, s_lo = (blockIdx.x - q * n_group) * group;
  const int n_s = min(group, NB3 - s_lo);
  const int N0 = p.N[0], N1 = p.N[1], N2 = p.N[2];
  const int a0 = q / (N1 * N2), a1 = (q / N2) % N1, a2 = q % N2;

  extern __shared__ double2 smem[];
  const int at_s = p.n_blk * 9;                  // entries of one branch
  const int at_n = group * at_s + 9 * n_slot;    // and a zero tail a padded range may read
  const int n_ph = tile_phases(NB, p.n_blk, n_slot);
  C* at = reinterpret_cast<C*>(smem);            // [branch of the group][n_blk][9]
  unsigned char* wave_lds = reinterpret_cast<unsigned char*>(smem) +
                            ((size_t)at_n * sizeof(C) + 15) / 16 * 16 +
                            wv * tile_wave_lds<FORM>(group, n_ph);
  C* phb = reinterpret_cast<C*>(wave_lds);       // e^{-i q1.R_d} per phase slot
  double(*md)[16][5] =
      reinterpret_cast<double(*)[16][5]>(wave_lds + n_ph * sizeof(C));  // (w, n, v) of q1's and q2's modes
  C* cq_v = reinterpret_cast<C*>(md + 2);                     // queued candidates: V,
  double* acc = reinterpret_cast<double*>(cq_v + kTileCand);  // sums [branch of the group][kAccSlots]
  uint16_t* cq_code = reinterpret_cast<uint16_t*>(acc + group * kAccSlots);  // s - s_lo | s' << 4 | s'' << 8
  C* bt = reinterpret_cast<C*>(cq_code + kTileCand);  // split form: B_s tile [row jc][17: column kc]
  int* slot_d = reinterpret_cast<int*>(
      reinterpret_cast<unsigned char*>(smem) + ((size_t)at_n * sizeof(C) + 15) / 16 * 16 +
      kTileWaves * tile_wave_lds<FORM>(group, n_ph));           // d of each phase slot, -1: none
  __shared__ double2 phq[64];
  __shared__ double wq64[16];
  __shared__ unsigned bad_lds;  // branches of the group whose table is not finite

  unsigned live = 0, any_sel = 0;  // branches of the group, bit s - s_lo
  float wq_abs_max = 0.0f;
  for (int s = 0; s < n_s; ++s) {
    const int m = q * NB3 + s_lo + s;
    const bool ph = phys[m], se = sel[m];
    live |= (ph && se) ? (1u << s) : 0u;
    any_sel |= se ? (1u << s) : 0u;
    wq_abs_max = fmaxf(wq_abs_max, fabsf((float)omega[m]));
  }
  if (live == 0) {
    if (tid < n_s && (any_sel >> tid & 1u)) gamma[q * NB3 + s_lo + tid] = 0.0;
    return;
  }
  if (tid < n_s) wq64[tid] = omega[q * NB3 + s_lo + tid];
  if (tid == 0) bad_lds = 0;
  for (int k = lane; k < n_s * kAccSlots; k += 64) acc[k] = 0.0;
  if constexpr (kSpl)
    for (int k = lane; k < 16 * 17; k += 64) bt[k] = Cx<T>::make((T)0, (T)0);
  for (int l = tid; l < n_rep; l += kTileThreads) {
    const int32_t* r = rep + 3 * l;
    int m0 = ((a0 * r[0]) % N0 + N0) % N0, m1 = ((a1 * r[1]) % N1 + N1) % N1,
        m2 = ((a2 * r[2]) % N2 + N2) % N2;
    double f = (double)m0 / N0 + (double)m1 / N1 + (double)m2 / N2;
    double sn, cs;
    sincospi(2.0 * f, &sn, &cs);
    phq[l] = make_double2(cs, sn);
  }
  for (int k = tid; k < at_n; k += kTileThreads) at[k] = Cx<T>::make((T)0, (T)0);
  for (int k = tid; k < n_ph; k += kTileThreads) {
    const int blk = FOUR ? pair_ptr[k >> 2] + (k & 3) : k;
    slot_d[k] = blk < (FOUR ? pair_ptr[(k >> 2) + 1] : p.n_blk) ? blk_d[blk] : -1;
  }
  __syncthreads();
  for (int k = tid; k < p.n_e * n_s; k += kTileThreads) {
    const int e = k / n_s, s = k - e * n_s;
    double re = 0.0, im = 0.0;
    for (int t = t_ptr[e]; t < t_ptr[e + 1]; ++t) {
      const size_t o = (((size_t)q * NB3 + t_i[t]) * NB3 + s_lo + s) * 2;
      const double ex = evec[o], ey = evec[o + 1];
      const double2 f = phq[t_l2[t]];
      const double c = t_coef[t];
      re += c * (ex * f.x - ey * f.y);
      im += c * (ex * f.y + ey * f.x);
    }
    // a padded range may read into the next branch's table, and a zero phase
    // hides nothing that is not finite: such a branch keeps zeros there, and its
    // terms are NaN where they are weighted
    T x = (T)re, y = (T)im;
    if (!((x - x) + (y - y) == (T)0)) {
      x = y = (T)0;
      atomicOr(&bad_lds, 1u << s);
    }
    at[s * at_s + e_blk[e] * 9 + e_bg[e]] = Cx<T>::make(x, y);
  }
  __syncthreads();
  const unsigned bad = __builtin_amdgcn_readfirstlane(bad_lds);

  // Accumulator item r of a lane is row row_of(r) of its column lr; K slot
  // (MFMA t, lane group lg) of the first product is column 4 (t % 4) + lg of
  // B_s (part t / 4 of the stacked complex K), of the second row row_of(t % 4)
  // of T, so that T goes from the accumulators straight into the next product.
  // The split form's products take element i of lane group lg as column
  // 8 (lg % 2) + i of part lg / 2, and row 4 lg + i % 4 of part i / 4.
  auto row_of = [&](int r) { return FORM == kF64 ? 4 * r + lg : 4 * lg + r; };
  // this lane's four B_s entries: first table entry and first phase of their
  // atom pair.  In operand order (row jc = lr, columns kc = 4 i + lg; an entry
  // outside the cell takes entry 0 and is dropped); in the split form, where
  // two lanes read each entry, the balanced work list's, handed round through
  // the tile at position b_pos (no entry: the spare one).
  int b_at[4], b_ph[4], b_cnt[4], b_pos[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int jc = lr, kc = 4 * i + lg;
    if constexpr (kSpl) {
      b_pos[i] = bwork[i * 64 + lane];
      if (b_pos[i] < 0) b_pos[i] = 16 * 17;
      jc = b_pos[i] / 17;
      kc = b_pos[i] - 17 * jc;
    }
    const bool in = kSpl ? b_pos[i] < 16 * 17 : lr < NB3 && kc < NB3;
    const int pr = in ? (jc / 3) * NB + kc / 3 : 0;
    b_at[i] = in ? pair_ptr[pr] * 9 + (jc % 3) * 3 + kc % 3 : 0;
    b_ph[i] = FOUR ? 4 * pr : pair_ptr[pr];
    b_cnt[i] = pair_ptr[pr + 1] - pair_ptr[pr];
  }
  // Steps the wave takes for each of the four.  The split form's list is sorted
  // by length: its later entries are fewer and shorter, or none (random three
  // atoms on 7^3, adaptive: 843 us, 1,105 with all sixteen steps for each).
  int b_end[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int n = n_slot;
    if constexpr (kSpl && !FOUR) {
      n = b_pos[i] < 16 * 17 ? b_cnt[i] : 0;
      for (int off = 1; off < 64; off <<= 1) n = max(n, __shfl_xor(n, off, 64));
      n = __builtin_amdgcn_readfirstlane(n);
    }
    b_end[i] = n;
  }

  // Exact FP64 cut and weight of queued candidates, one per lane, in queue
  // order, from the partner's mode data staged in LDS (the queue only ever
  // holds candidates of the current partner); the contribution goes to this
  // lane's sum of the candidate's branch.
  int n_cand = 0;  // wave-uniform
  auto resolve = [&](int dbl) {
    for (int base = 0; base < n_cand; base += 64) {
      const int e = base + lane;
      double c = 0.0;
      int cs_ = 0;
      if (e < n_cand) {
        const int code = cq_code[e];
        cs_ = code & 15;
        const double* d1 = md[0][(code >> 4) & 15];
        const double* d2 = md[1][code >> 8];
        double sp, sm;
        widths_v(p, d1 + 2, d2 + 2, sp, sm);
        const C v = cq_v[e];
        c = pair_weight_both(p, dbl, wq64[cs_], d1[0], d2[0], d1[1], d2[1], sp, sm) *
            ((double)v.x * (double)v.x + (double)v.y * (double)v.y);
        if (bad >> cs_ & 1u) c = __builtin_nan("");
      }
      double* a = acc + cs_ * kAccSlots + (lane & (kAccSlots - 1));
#pragma unroll
      for (int k = 0; k < 64; k += kAccSlots) {  // the lanes of one slot in turn
        if (lane >= k && lane < k + kAccSlots && e < n_cand) *a += c;
        lds_wave_sync();
      }
    }
    n_cand = 0;
  };

  // the group's next live branch after s, n_s when there is none (the next of
  // all in the split form of few blocks, whose loop then is 1 % shorter)
  constexpr bool kJump = !(kSpl && FOUR);
  auto next_live = [&](int s) {
    const unsigned m = live >> (s + 1);
    return !kJump ? s + 1 : m ? s + __ffs(m) : n_s;
  };
  const Partners prt(p.half != 0, a0, a1, a2, N0, N1, N2);
  const float w_lane = lane < n_s ? (float)wq64[lane] : 0.0f;  // branch frequencies, read by readlane
  unsigned partner = 0;  // lane k: q1 | q2 << 16 of the wave's k-th partner of 64
  unsigned long long dbl_mask = 0;
  for (int pi = wv, n_done = 0; pi < prt.n; pi += kTileWaves, ++n_done) {
    if ((n_done & 63) == 0) {  // the next 64 partners, decoded one per lane
      const int mine = pi + lane * kTileWaves;
      int b0 = 0, b1 = 0, b2 = 0, twice = 0;
      if (mine < prt.n) twice = prt.get(mine, N1, N2, b0, b1, b2);
      const unsigned c0 = wrap_sub(prt.h[0].t, b0, N0), c1 = wrap_sub(prt.h[1].t, b1, N1),
                     c2 = wrap_sub(prt.h[2].t, b2, N2);
      partner = (unsigned)((b0 * N1 + b1) * N2 + b2) | ((c0 * N1 + c1) * N2 + c2) << 16;
      dbl_mask = __ballot(twice);
    }
    const unsigned pk = __builtin_amdgcn_readlane(partner, n_done & 63);
    const int dbl = (int)(dbl_mask >> (n_done & 63) & 1ull);  // all wave-uniform
    const int q1 = pk & 0xffff, q2 = pk >> 16;
    lds_wave_sync();
    for (int k = lane; k < n_ph; k += 64) {
      const int d = slot_d[k];
      phb[k] = d >= 0 ? phase_tab[(size_t)q1 * p.n_d + d] : Cx<T>::make((T)0, (T)0);
    }
    if ((lane & 15) < NB3 && lane < 32) {
      const int m = (lane < 16 ? q1 : q2) * NB3 + (lane & 15);
      double* d = md[lane >> 4][lane & 15];
      d[0] = omega[m];
      d[1] = occ[m];
      d[2] = vel[3 * (size_t)m];
      d[3] = vel[3 * (size_t)m + 1];
      d[4] = vel[3 * (size_t)m + 2];
    }
    lds_wave_sync();
    // The branches of the group, in runs as long as the queue takes whole
    // branches (one run, as a rule): a run ends with its candidates resolved,
    // where none of its operand registers is live.
    int s = next_live(-1);
    do {
      // eta(q2)[kc][s''] as the B operand of T = B_s eta2 (column n = lr) and
      // eta(q1)[jc][s'] as A = eta1^T (row m = lr) of V = eta1^T T; zero
      // outside the cell, which also drops what B_s and T hold there
      const double* v2 = evec + (size_t)q2 * NB3 * NB3 * 2;
      const double* v1 = evec + (size_t)q1 * NB3 * NB3 * 2;
      C e2[4], e1[4];
      bf16x8 e2h, e2l, e1ah, e1al, e1bh, e1bl;  // split form: x = hi + lo
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned k2 = 4 * i + lg, k1 = row_of(i);
        e2[i] = e1[i] = Cx<T>::make((T)0, (T)0);
        if (!kSpl && k2 < (unsigned)NB3 && lr < NB3) {
          const unsigned o = (k2 * NB3 + lr) * 2;
          e2[i] = Cx<T>::make((T)v2[o], (T)v2[o + 1]);
        }
        if (k1 < (unsigned)NB3 && lr < NB3) {
          const unsigned o = (k1 * NB3 + lr) * 2;
          e1[i] = Cx<T>::make((T)v1[o], (T)v1[o + 1]);
        }
      }
      if constexpr (kSpl) {
        f8 b, a1, a2;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          // B' = [Re eta2 ; Im eta2]; A'(eta1^T) = [Re | -Im], A'' = [Im | Re]
          const unsigned k = 8 * (lg & 1) + i;
          b[i] = 0.0f;
          if (k < (unsigned)NB3 && lr < NB3) b[i] = (float)v2[(k * NB3 + lr) * 2 + (lg < 2 ? 0 : 1)];
          a1[i] = (i < 4) ? e1[i & 3].x : -e1[i & 3].y;
          a2[i] = (i < 4) ? e1[i & 3].y : e1[i & 3].x;
        }
        split8(b, e2h, e2l);
        split8(a1, e1ah, e1al);
        split8(a2, e1bh, e1bl);
      }
      // this lane's epilogue pairs: s' = row_of(r), s'' = lr.  FP32
      // pre-classification from the mode copies (a mode below the floor carries
      // a NaN frequency and fails every comparison); the exact FP64 decision
      // and weight are the queue's.
      float bhi_p[4], bhi_m[4], cpv[4], cmv[4];
      const float4 none = make_float4(0.f, 0.f, 0.f, __builtin_nanf(""));
      const float4 f2 = lr < NB3 ? modef[q2 * NB3 + lr] : none;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float4 f1 = row_of(r) < NB3 ? modef[q1 * NB3 + row_of(r)] : none;
        float s2p, s2m, e_sig;
        widths2_f(p, f1, f2, s2p, s2m, e_sig);
        const float scl = wq_abs_max + fabsf(f1.w) + fabsf(f2.w);
        bhi_p[r] = make_band_f(s2p, scl, e_sig).hi;
        bhi_m[r] = make_band_f(s2m, scl, e_sig).hi;
        // with the mirrored ordering, |w + cp| and |w - cp| share the edge
        // bhi_p, and for w >= 0 the smaller is |w - |cp|| (bitwise in FP32):
        // one test covers both
        const float cp = f1.w - f2.w;
        cpv[r] = dbl ? -fabsf(cp) : cp;
        cmv[r] = -f1.w - f2.w;
      }
      // the A~ values of a branch, loaded while the branch before is projected
      C an[kAhead ? 16 : 1];
      auto fetch = [&](int sb) {
        const C* as = at + min(sb, n_s - 1) * at_s;
#pragma unroll
        for (int k = 0; k < 16; ++k) an[k] = as[b_at[k >> 2] + 9 * (k & 3)];
      };
      if constexpr (kAhead) fetch(s);
#pragma unroll 1
      for (; s < n_s; s = next_live(s)) {
        // the candidates of this branch, before anything is projected:
        // coalescence of either ordering, or decay (w > 0: s is live)
        const float wsf = __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w_lane), s));
        bool near[4];
        unsigned long long mask[4];
        int n_new = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool np = fabsf(wsf + cpv[r]) < bhi_p[r], nm = fabsf(wsf + cmv[r]) < bhi_m[r];
          near[r] = np || nm;
          mask[r] = __ballot(np) | __ballot(nm);
          n_new += __popcll(mask[r]);
        }
        const bool skip = n_new == 0 || (!kJump && !(live >> s & 1u));  // uniform
        if (!skip && n_cand + n_new > kTileCand) break;  // uniform: n_new <= 256 fits an empty queue
        if (skip) {
          if constexpr (kAhead) fetch(next_live(s));
          continue;
        }
        // B_s in operand order; a pair's slots past its blocks have a zero phase
        T br[4] = {0, 0, 0, 0}, bi[4] = {0, 0, 0, 0};
        auto quad = [&](int i, const C* a, const C* f) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            br[i] = fma(f[j].x, a[j].x, br[i]);
            br[i] = fma(-f[j].y, a[j].y, br[i]);
            bi[i] = fma(f[j].x, a[j].y, bi[i]);
            bi[i] = fma(f[j].y, a[j].x, bi[i]);
          }
        };
        if constexpr (kAhead) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            C f[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = phb[b_ph[i] + j];
            quad(i, an + 4 * i, f);
          }
          fetch(next_live(s));
        } else {
          const C* as = at + s * at_s;
          for (int j0 = 0; j0 < (FOUR ? 4 : n_slot); j0 += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (!FOUR && kSpl && j0 >= b_end[i]) continue;  // uniform
              C a[4], f[4];
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                a[j] = as[b_at[i] + 9 * (j0 + j)];
                f[j] = phb[FOUR || j0 + j < b_cnt[i] ? b_ph[i] + j0 + j : p.n_blk];
              }
              quad(i, a, f);
            }
          }
        }
        // T (rows row_of(r) of column lr, in registers) is the B operand of V
        V4 tr = {0, 0, 0, 0}, ti = {0, 0, 0, 0}, vr = {0, 0, 0, 0}, vi = {0, 0, 0, 0};
        if constexpr (kSpl) {
          lds_wave_sync();
#pragma unroll
          for (int i = 0; i < 4; ++i)
            bt[b_pos[i]] = Cx<T>::make(br[i], bi[i]);
          lds_wave_sync();
          f8 a1, a2;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const C b = bt[lr * 17 + 8 * (lg & 1) + i];
            a1[i] = (lg < 2) ? b.x : -b.y;
            a2[i] = (lg < 2) ? b.y : b.x;
          }
          bf16x8 a1h, a1l, a2h, a2l;
          split8(a1, a1h, a1l);
          split8(a2, a2h, a2l);
          tr = mma(a1l, e2h, tr);
          ti = mma(a2l, e2h, ti);
          tr = mma(a1h, e2l, tr);
          ti = mma(a2h, e2l, ti);
          tr = mma(a1h, e2h, tr);
          ti = mma(a2h, e2h, ti);
          f8 b;
#pragma unroll
          for (int i = 0; i < 8; ++i) b[i] = (i < 4) ? tr[i & 3] : ti[i & 3];
          bf16x8 th, tl;
          split8(b, th, tl);
          vr = mma(e1al, th, vr);
          vi = mma(e1bl, th, vi);
          vr = mma(e1ah, tl, vr);
          vi = mma(e1bh, tl, vi);
          vr = mma(e1ah, th, vr);
          vi = mma(e1bh, th, vi);
        } else {
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int i = t & 3;
            const T x = (t < 4) ? br[i] : -bi[i];
            const T y = (t < 4) ? bi[i] : br[i];
            const T e = (t < 4) ? e2[i].x : e2[i].y;
            tr = mma(x, e, tr);
            ti = mma(y, e, ti);
          }
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int i = t & 3;
            const T x = (t < 4) ? e1[i].x : -e1[i].y;
            const T y = (t < 4) ? e1[i].y : e1[i].x;
            const T b = (t < 4) ? tr[i] : ti[i];
            vr = mma(x, b, vr);
            vi = mma(y, b, vi);
          }
        }
        // the candidates' V[s' = row_of(r)][s'' = lr], queued for the exact FP64
        // decision and weight
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (near[r]) {
            const unsigned lo = (unsigned)mask[r], hi = (unsigned)(mask[r] >> 32);
            const int slot = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, n_cand));
            cq_code[slot] = (uint16_t)(s | (row_of(r) << 4) | (lr << 8));
            cq_v[slot] = Cx<T>::make(vr[r], vi[r]);
          }
          n_cand += __popcll(mask[r]);
        }
      }
      lds_wave_sync();
      resolve(dbl);  // the queue never carries candidates past their partner
    } while (s < n_s);
  }
  // fixed order: a branch's sixteen sums of every wave in turn, then a butterfly
  __syncthreads();
  for (int s = wv; s < n_s; s += kTileWaves) {
    double sum = 0.0;
    if (lane < kAccSlots)
      for (int w = 0; w < kTileWaves; ++w)
        sum += reinterpret_cast<const double*>(
            reinterpret_cast<const unsigned char*>(acc + s * kAccSlots + lane) +
            (ptrdiff_t)(w - wv) * (ptrdiff_t)tile_wave_lds<FORM>(group, n_ph))[0];
    sum = wave_sum_fixed(sum);
    if (lane == 0 && (any_sel >> s & 1u))
      gamma[q * NB3 + s_lo + s] = (live >> s & 1u) ? scale * sum : 0.0;
  }
}

// Static LDS of lw_tiles, and the dynamic part with `group` branches a workgroup.
constexpr size_t kTileStatic = 64 * 16 + 16 * 8 + 16;
template <int FORM>
static size_t tile_lds(const kaldo_crystal* c, int group) {
  const size_t cs = sizeof(typename Cx<typename Dense<FORM>::T>::type);
  const int n_slot = tile_slots(c->bloch.max_pair_blk);
  const int n_ph = tile_phases(c->nb, c->bloch.n_blk, n_slot);
  const size_t at_n = (size_t)group * c->bloch.n_blk * 9 + 9 * n_slot;
  return (at_n * cs + 15) / 16 * 16 + Dense<FORM>::kWaves * tile_wave_lds<FORM>(group, n_ph) + sizeof(int) * n_ph;
}

// Branches a workgroup of lw_tiles takes, 0 when the tables of one branch do
// not fit.  A CU holds one workgroup, which per partner pays a set-up of
// about half a branch's projection, with pairs of more than four blocks of
// several (random three atoms on a 7^3 mesh, fixed width, all nine branches
// against five and four: FP32 803 and 898 us, split 884 and 988): the group
// count that minimises rounds of 256 workgroups x (set-up + branches).
template <int FORM>
static int tile_group(const kaldo_crystal* c, int nq) {
  int best = 0;
  double cost = 0.0;
  const double setup = tile_slots(c->bloch.max_pair_blk) == 4 ? 0.5 : 4.0;
  for (int n = 1; n <= c->nb3; ++n) {
    const int g = (c->nb3 + n - 1) / n;
    if (tile_lds<FORM>(c, g) + kTileStatic > c->lds_max) continue;
    const double t = std::ceil((double)nq * n / 256.0) * (g + setup);
    if (!best || t < cost) best = g, cost = t;
  }
  return best;
}

bool mfma64_supported(const kaldo_crystal* c) {
  return c->nb3 <= 16 && c->n_rep <= 64 && tile_group<kF64>(c, 1) > 0;
}

template <int FORM>
static int launch_tiles(const char* name, const kaldo_crystal* c, const LwParams& p,
                        const double* omega, const double* vel, const float4* modef,
                        const double* occ, const uint8_t* phys, const uint8_t* sel,
                        const double* evec, void* phase_ws, double scale, double* gamma,
                        hipStream_t st) {
  using T = typename Dense<FORM>::T;
  using C = typename Cx<T>::type;
  C* phase_tab = static_cast<C*>(phase_ws);
  const int nq = p.nq;
  const long nph = (long)nq * std::max(1, p.n_d);
  KALDO_LAUNCH("lw_phase_table", lw_phase_table<T>, dim3((nph + 255) / 256), dim3(256), 0, st, nq,
               p.n_d, p.N[0], p.N[1], p.N[2], c->bloch.dvec, phase_tab);
  const Fc3Bloch& b = c->bloch;
  const int group = tile_group<FORM>(c, nq), n_group = (c->nb3 + group - 1) / group;
  const int n_slot = tile_slots(b.max_pair_blk);
  auto run = [&](auto kernel) {
    KALDO_LAUNCH(name, kernel, dim3((unsigned)nq * n_group),
                 dim3(64 * Dense<FORM>::kWaves),
                 tile_lds<FORM>(c, group), st, p, c->n_rep, group, n_group, n_slot, c->d_rep, omega,
                 vel, modef, occ, phys, sel, evec, phase_tab, b.t_ptr, b.t_i, b.t_l2, b.t_coef,
                 b.e_blk, b.e_bg, b.blk_d, b.pair_ptr, b.bwork, scale, gamma);
  };
  if (n_slot == 4)
    run(lw_tiles<FORM, true>);
  else
    run(lw_tiles<FORM, false>);
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}

// The FP32 and split forms serve the cells whose A~ tables of all branches
// fit the LDS with kMfmaBeside bytes to spare (the FP32 form leaves larger
// cells to the pruned kernel).
constexpr int kMfmaMaxBlocks = 128;
constexpr size_t kMfmaBeside = 53376;
bool mfma_supported(const kaldo_crystal* c) {
  if (c->nb3 > 16 || c->n_rep > 64 || c->bloch.n_blk > kMfmaMaxBlocks) return false;
  return (size_t)c->bloch.n_blk * 9 * c->nb3 * 8 + kMfmaBeside <= c->lds_max &&
         tile_group<kF32>(c, 1) > 0 && tile_group<kSplit>(c, 1) > 0;
}

int launch_mfma(const kaldo_crystal* c, const LwParams& p, int prec, const double* omega,
                const double* vel, const float4* modef, const double* occ, const uint8_t* phys,
                const uint8_t* sel, const double* evec, void* phase_ws, double scale,
                double* gamma, hipStream_t st) {
  if (prec == KALDO_FP64)
    return launch_tiles<kF64>("lw_mfma_fp64", c, p, omega, vel, modef, occ, phys, sel, evec,
                              phase_ws, scale, gamma, st);
  if (prec == KALDO_BF16X3)
    return launch_tiles<kSplit>("lw_mfma_bf16x3", c, p, omega, vel, modef, occ, phys, sel, evec,
                                phase_ws, scale, gamma, st);
  return launch_tiles<kF32>("lw_mfma_fp32", c, p, omega, vel, modef, occ, phys, sel, evec, phase_ws,
                            scale, gamma, st);
}

}  // namespace kaldo
