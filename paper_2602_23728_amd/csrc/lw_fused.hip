// Fused crystal linewidth kernel of the small cells (fused_boxes; the others'
// is lw_rounds.hip): one workgroup per (q-point, share of its partners).
//
// Paper: Eq. phi3_proj (projection on three Bloch eigenvectors), Eq. gamma
// with its Delta terms, Eq. broadening (only pairs with |x| < 2 sigma are
// projected, as the paper's implementation does), Eq. bose.
//
// Work of one workgroup (q fixed, all branches s at once):
//  1. A~_q (the FC3 COO contracted on its home-cell index with eta(q), with
//     the phase e^{+i q.R''} folded in) built in FP64 and stored in LDS in an
//     atom-block layout [block (jb, kb, d)][beta gamma][s].
//  2. Each wave sweeps tiles of at most 64 partners q1, compact in q-space (a
//     box of d0 x d1 x d2 mesh points, a lane per point); q2 = -q - q1 then
//     runs over a box of the same shape.  The frequency ranges of both boxes,
//     kept for every box position and branch (lw_tables), tell which (s', s'')
//     and which s of them can hold a pair inside the cut: 12 % of the (s', s'')
//     and 4 % of the triples on the diamond 24^3 mesh with boxes of 4 x 4 x 4.
//     Of those the pairs nearer than the boxes' widest cut, from the two
//     frequencies alone, join the wave's first queue in LDS; a queue of 192 is
//     classified in FP32 against a conservative band from the FP32 mode
//     copies, 64 at a time, and the candidates join the second, in the same
//     fixed order.  When Phi3 is symmetric in its last two slots the ordered
//     pair (q1 s', q2 s'') and its mirror (q2 s'', q1 s') have the same V, so
//     only q1 <_lex q2 is swept (and q1 == q2 once) and an entry carries the
//     terms of both orderings, each with its own cut.
//  3. Full batches of 64 candidates are weighted (exact FP64 cut) and
//     projected, one per lane: V = sum_blocks e^{-i q1.R_d} sum_{beta,gamma}
//     A~[blk][beta gamma][s] eta_{3jb+beta}(q1,s') eta_{3kb+gamma}(q2,s''),
//     in the contraction type T, and w |V|^2 (FP64) added to the lane's
//     per-branch sum.  A batch's records and phases come through LDS (pull_rows).
//  4. A fixed butterfly per wave and the waves in order give this work item's
//     partial sum; lw_fused_finish adds the chunks of a q in order.
// Every order above depends on the inputs only, so results are bitwise
// reproducible.  Waves never wait for each other between 1 and 4.
//
// What bounds it: the return path of the vector memory, 90 % busy, and beside it
// the vector ALU, 62 % (diamond 24^3, FP64).  Of 5.6 ms there the projection
// takes 3.4, the sweep 1.8, the classification 0.3, A~ 0.1.  One partner q1 per
// lane in mesh order without ranges took 14.2 ms, boxes with ranges 8.4 (28
// divergent loads a batch, and the classification at full (s', s'') cost);
// records and phases through LDS, one phase per +-d and the two queues
// 5.6 (FP32, diamond 15^3: 1.02, 0.69 and 0.57 ms).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <initializer_list>

#include "common.h"
#include "lw_common.h"

namespace kaldo {

constexpr int kFusedThreads = 256;
constexpr int kFusedWaves = kFusedThreads / 64;
constexpr int kQueue = 256;           // slots of a wave's queue of near pairs
constexpr int kFlush = kQueue - 64;   // classified when it holds at least that many
constexpr int kPairs = 128;           // slots of its queue of candidates, projected 64 at a time
constexpr int kFusedItems = 2048;     // (q, chunk) work items a launch aims for

// Waves per SIMD the register allocation targets: four for the small FP32
// cells (three 671 us against 565 on the diamond 15^3 mesh), three for the
// FP64 cells (two 8.1 ms against 6.3 on 24^3, four spill the vectors).
template <int NB, typename T>
constexpr int fused_waves_per_eu() {
  return sizeof(T) == 4 ? 4 : 3;
}

// Partner boxes of a mesh: extents and numbers per axis.
struct Boxes {
  int d[3], n[3];
};

// The box shape of a mesh: at most 64 points, the fewest boxes weighed with
// their size, since a longer box spans wider frequency ranges and prunes less.
// Measured on the diamond cell: about 140 instructions a box and 85 for each
// (s', s'') that survives, 5 % of them plus 13 % of the box's share of the
// mesh's edges.  The boxes of a q are dealt over the four waves of its
// workgroup, or of two on meshes small enough for a second, so what counts is
// their number rounded up to that: one box of 4 x 4 x 4 for that mesh left
// three waves idle (FP32, adaptive: 45.8 us against 33.2 with eight boxes).
static int n_boxes(const Boxes& b) { return b.n[0] * b.n[1] * b.n[2]; }
static Boxes choose_boxes(const int* N) {
  const int nq = N[0] * N[1] * N[2];
  const int deal = nq >= 64 && nq < kFusedItems ? 2 * kFusedWaves : kFusedWaves;
  int num[3][9];
  double part[3][9];
  for (int x = 0; x < 3; ++x)
    for (int a = 1; a <= std::min(N[x], 8); ++a) {
      num[x][a] = (N[x] + a - 1) / a;
      part[x][a] = 0.13 * a / N[x];
    }
  Boxes best{};
  double cost = 0.0;
  for (int a = 1; a <= std::min(N[0], 8); ++a)
    for (int b = 1; b <= std::min(N[1], 8); ++b)
      for (int c = 1; c <= std::min({N[2], 8, 64 / (a * b)}); ++c) {
        const int boxes = num[0][a] * num[1][b] * num[2][c], dealt = (boxes + deal - 1) / deal * deal;
        const double t = dealt * (140.0 + 85.0 * 36.0 * std::min(1.0, 0.05 + part[0][a] + part[1][b] + part[2][c]));
        if (!best.d[0] || t < cost) best = {{a, b, c}, {num[0][a], num[1][b], num[2][c]}}, cost = t;
      }
  return best;
}

// Gamma of the selected modes: the chunk sums of their q in chunk order.
__global__ void lw_fused_finish(int n_modes, int nb3, const uint8_t* __restrict__ phys,
                                const uint8_t* __restrict__ sel, const int32_t* __restrict__ idx_of_q,
                                int n_chunk, const double* __restrict__ part, double scale,
                                double* __restrict__ gamma) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_modes || !sel[m]) return;
  const int q = m / nb3, s = m - q * nb3, k = idx_of_q[q];
  if (!phys[m] || k < 0) {
    gamma[m] = 0.0;
    return;
  }
  double acc = 0.0;
  for (int c = 0; c < n_chunk; ++c) acc += part[((size_t)k * n_chunk + c) * nb3 + s];
  gamma[m] = scale * acc;
}

// Record of a mode: FP64 w, n, v_x, v_y, v_z, then its eigenvector.  An FP64
// eigenvector is turned so that its first component is real (|V| does not
// depend on it) and that component takes eight bytes; so does the first
// component of an FP32 one.  The record of a two-atom cell is then 128 bytes
// in FP64, one cache line, and 88 in FP32, kept in one.
template <int NB, typename T>
__host__ __device__ constexpr int record_used() {  // whole 16-byte pieces
  return (48 + (3 * NB - 1) * 2 * (int)sizeof(T) + 15) / 16 * 16;
}
__host__ __device__ constexpr int record_stride(int used) { return used > 64 && used < 128 ? 128 : used; }
size_t fused_record_bytes(int nb3, size_t cs) {
  return record_stride((int)((48 + (nb3 - 1) * cs + 15) / 16 * 16));
}
// Row of a q-point's phases e^{-i q.R_f}: one per +-d, n_f complex T in kFusedPhaseBytes.

// Everything the sweep reads beside the FC3 tables, one launch, a job a range
// of blocks (first[k] .. first[k + 1]):
//   0  mode records
//   1  phases e^{-i q1.R_f} of every mesh point, FP64 rounded to T
//   2  per box position (its lowest corner, any mesh point; boxes wrap) and
//      branch, four lanes each: the range of the physical frequencies (FP32, as
//      the sweep classifies them; lo > hi without any) and an upper bound of
//      |v| h / sqrt(12), the speed's share of the adaptive width (0 when fixed)
//   3  the list of every q; given a subset, the flags lw_live_q makes it from
struct TableJobs {
  unsigned first[5];
};
template <typename T>
__global__ __launch_bounds__(256) void lw_tables(
    TableJobs jobs, LwParams p, Boxes box, float hs, int rb, int phase_bytes, int subset,
    const double* __restrict__ evec, const double* __restrict__ omega, const double* __restrict__ occ,
    const double* __restrict__ vel, const float4* __restrict__ modef, const uint8_t* __restrict__ phys,
    const uint8_t* __restrict__ sel, const int32_t* __restrict__ fvec, int n_f,
    unsigned char* __restrict__ rec, unsigned char* __restrict__ phase_tab,
    float4* __restrict__ window, int32_t* __restrict__ list, int32_t* __restrict__ idx_of_q,
    int32_t* __restrict__ count) {
  using C = typename Cx<T>::type;
  const int nb3 = p.nb3, N0 = p.N[0], N1 = p.N[1], N2 = p.N[2];
  constexpr bool kTurned = sizeof(T) == 8;
  const unsigned blk = blockIdx.x;
  if (blk < jobs.first[1]) {
    const unsigned k = (blk - jobs.first[0]) * 256 + threadIdx.x;
    const unsigned m = k / nb3, j = k - m * nb3;
    if (m >= (unsigned)(p.nq * nb3)) return;
    unsigned char* r = rec + (size_t)m * rb;
    const unsigned q = m / nb3, s = m - q * nb3;
    const double2* e = reinterpret_cast<const double2*>(evec) + (size_t)q * nb3 * nb3 + s;
    double2 x = e[j * nb3], turn = make_double2(1.0, 0.0);
    const double2 x0 = e[0];
    const double a0 = hypot(x0.x, x0.y);
    if (kTurned && a0 > 1e-200) turn = make_double2(x0.x / a0, -x0.y / a0);
    if (j == 0) {
      double2* d = reinterpret_cast<double2*>(r);
      const double* v = vel + 3 * (size_t)m;
      d[0] = make_double2(omega[m], occ[m]);
      d[1] = make_double2(v[0], v[1]);
      double first = a0;
      if constexpr (!kTurned) {
        const C f = Cx<T>::make((T)x0.x, (T)x0.y);
        first = __builtin_bit_cast(double, f);
      }
      d[2] = make_double2(v[2], first);
    } else {
      if constexpr (kTurned) x = make_double2(x.x * turn.x - x.y * turn.y, x.x * turn.y + x.y * turn.x);
      reinterpret_cast<C*>(r + 48)[j - 1] = Cx<T>::make((T)x.x, (T)x.y);
    }
  } else if (blk < jobs.first[2]) {
    const unsigned k = (blk - jobs.first[1]) * 256 + threadIdx.x;
    if (n_f == 0 || k >= (unsigned)p.nq * (unsigned)n_f) return;
    const int q1 = k / n_f, d = k - q1 * n_f;
    const int b0 = q1 / (N1 * N2), b1 = (q1 / N2) % N1, b2 = q1 % N2;
    const int32_t* r = fvec + 3 * d;
    const int m0 = ((b0 * r[0]) % N0 + N0) % N0, m1 = ((b1 * r[1]) % N1 + N1) % N1,
              m2 = ((b2 * r[2]) % N2 + N2) % N2;
    const double f = (double)m0 / N0 + (double)m1 / N1 + (double)m2 / N2;
    double sn, cs;
    sincospi(-2.0 * f, &sn, &cs);
    reinterpret_cast<C*>(phase_tab + (size_t)q1 * phase_bytes)[d] = Cx<T>::make((T)cs, (T)sn);
  } else if (blk < jobs.first[3]) {
    const unsigned k = (blk - jobs.first[2]) * 256 + threadIdx.x;
    const int s_of = (k >> 2) / p.nq, q_of = (k >> 2) - s_of * p.nq, m = q_of * nb3 + s_of;
    float lo = __builtin_inff(), hi = -__builtin_inff(), v2 = 0.0f;
    const bool in = s_of < nb3;
    if (in) {
      const int q = q_of, s = s_of;
      const int a0 = q / (N1 * N2), a1 = (q / N2) % N1, a2 = q % N2;
      for (int ij = k & 3; ij < box.d[0] * box.d[1]; ij += 4) {
        const int i = ij / box.d[1], j = ij - i * box.d[1];
        const int b0 = a0 + i < N0 ? a0 + i : a0 + i - N0, b1 = a1 + j < N1 ? a1 + j : a1 + j - N1;
        const float4* row = modef + s * p.nq + (b0 * N1 + b1) * N2;
        for (int c = 0; c < box.d[2]; ++c) {
          const float4 f = row[a2 + c < N2 ? a2 + c : a2 + c - N2];
          if (f.w == f.w) {  // NaN: below the floor
            lo = fminf(lo, f.w);
            hi = fmaxf(hi, f.w);
            v2 = fmaxf(v2, f.x * f.x + f.y * f.y + f.z * f.z);
          }
        }
      }
    }
    for (int off = 1; off < 4; off <<= 1) {
      lo = fminf(lo, __shfl_xor(lo, off, 64));
      hi = fmaxf(hi, __shfl_xor(hi, off, 64));
      v2 = fmaxf(v2, __shfl_xor(v2, off, 64));
    }
    if (in && (k & 3) == 0) window[m] = make_float4(lo, hi, sqrtf(v2) * hs * 1.000001f, 0.0f);
  } else {
    const int q = (blk - jobs.first[3]) * 256 + threadIdx.x;
    if (q < p.nq && subset) {
      int f = 0;
      for (int s = 0; s < nb3; ++s) f |= phys[q * nb3 + s] & sel[q * nb3 + s];  // 0/1 bytes, no branch
      idx_of_q[q] = f;
    } else if (q < p.nq) {
      list[q] = q;
      idx_of_q[q] = q;
      if (q == 0) *count = p.nq;
    }
  }
}

constexpr int kWaitLds = 0xc07f;  // s_waitcnt lgkmcnt(0), the other counters left

// 16 CH bytes of each lane's row (tab + idx * stride) into LDS.  CH
// neighbouring lanes fetch a row's 16-byte pieces side by side, so that an
// instruction covers 64 / CH rows with whole cache lines: a lane fetching its
// own row piece by piece holds the return path for 64 cycles an instruction,
// and that path bounded the kernel (96 % busy on the diamond 24^3 mesh in
// FP64).  The pieces go to LDS directly, 64 consecutive ones an instruction:
// CH instructions, no registers.  Row l lies at st + 16 CH l, its pieces
// exchanged by pull_swap(l) where rows of a power of two of bytes would put
// every lane's on the same banks; pulled() gives a byte of the lane's own row.
// `st` is the wave's own; returns when the rows are there.  The pieces arrive
// by the memory pipe, which knows nothing of the LDS reads the wave still has
// under way (a wavefront fence orders the LDS instructions only): the first piece
// waits for those of the rows before, with its own row's index.
template <int CH>
__device__ __forceinline__ int pull_swap(int row) {
  return CH == 8 ? (row >> 1) & 7 : CH == 4 ? (row >> 2) & 3 : 0;
}
template <int CH>
__device__ __forceinline__ void pull_rows(const unsigned char* tab, int stride, int idx,
                                          unsigned char* st, int lane) {
  auto piece = [&](int k, int row, int byte) {  // row's index from the lane that holds it
    const int at = __builtin_amdgcn_ds_bpermute(row, idx);
    if (k == 0) __builtin_amdgcn_s_waitcnt(kWaitLds);
    const unsigned off = (unsigned)at * stride + byte;
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(tab + (size_t)off),
        (__attribute__((address_space(3))) void*)(st + 1024 * k), 16, 0, 0);
  };
  if constexpr (CH == 8 || CH == 4) {
    // 64 / CH rows on, pull_swap flips bit 2 (eight pieces) or nothing (four)
    int row = lane / CH * 4, byte = 16 * (lane % CH ^ pull_swap<CH>(lane / CH));
    asm volatile("" : "+v"(row), "+v"(byte));  // not kept in registers from batch to batch
#pragma unroll
    for (int k = 0; k < CH; ++k) piece(k, row + 4 * (64 / CH) * k, CH == 8 && k & 1 ? byte ^ 64 : byte);
  } else {
    int row = lane / CH * 4, part = lane % CH;
    asm volatile("" : "+v"(row), "+v"(part));
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      piece(k, row, 16 * part);
      part += 64 % CH;
      row += 4 * (64 / CH) + (part >= CH ? 4 : 0);
      part -= part >= CH ? CH : 0;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_wave_sync();
}
template <int CH>
__device__ __forceinline__ const unsigned char* pulled(const unsigned char* st, int lane, int byte) {
  const int row = lane * (16 * CH) + 16 * pull_swap<CH>(lane);
  return st + (CH == 8 || CH == 4 ? row ^ byte : row + byte);
}

// MODE (FusedMode): kModeGamma sums the linewidth terms into `part`;
// kModeCount makes only the cut decisions and writes the number of passing
// entries per wave and branch to tc.count; kModeRecord makes the same
// decisions, projects the passing entries and stores each one's
// temperature-independent factors at a fixed place of its mode's row: the row
// start, plus the counts of the earlier waves of its q, plus its rank among
// the wave's entries of that branch in queue order.
template <int NB, typename T, int MODE>
__global__ __launch_bounds__(kFusedThreads)
__attribute__((amdgpu_waves_per_eu(fused_waves_per_eu<NB, T>()))) void lw_fused(
    LwParams p, Boxes box, int n_rep, const int32_t* __restrict__ rep,
    const double* __restrict__ omega, const float4* __restrict__ modef, const float* __restrict__ freq,
    const uint8_t* __restrict__ phys, const uint8_t* __restrict__ sel,
    const double* __restrict__ evec, const unsigned char* __restrict__ rec,
    const unsigned char* __restrict__ phase_tab, const float4* __restrict__ window,
    const int32_t* __restrict__ t_ptr, const int32_t* __restrict__ t_i,
    const int32_t* __restrict__ t_l2, const double* __restrict__ t_coef,
    const int32_t* __restrict__ e_blk, const int32_t* __restrict__ e_bg,
    const int32_t* __restrict__ blk_f, const int32_t* __restrict__ pair_ptr,
    const int32_t* __restrict__ live_list, const int32_t* __restrict__ n_live_ptr, int n_chunk,
    double* __restrict__ part, TcOut tc) {
  constexpr int NB3 = 3 * NB;
  constexpr int BS = kFusedThreads;
  constexpr bool kRecord = MODE == kModeRecord;
  using C = typename Cx<T>::type;
  extern __shared__ double2 smem[];
  // a batch's records, then its rows of phases, are pulled through LDS, one
  // buffer a wave
  constexpr int RB = record_used<NB, T>(), kStride = record_stride(RB);
  constexpr int kPullBytes = MODE == kModeCount ? 48 : RB;  // >= 64 where phases are staged
  unsigned char* st = reinterpret_cast<unsigned char*>(smem) +
                      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (64 * kPullBytes);
  C* at = reinterpret_cast<C*>(reinterpret_cast<unsigned char*>(smem) +
                               kFusedWaves * 64 * kPullBytes);  // [n_blk][9][NB3]
  __shared__ uint32_t wq_q[kFusedWaves][kQueue];     // q1 | q2 << 16
  __shared__ uint16_t wq_code[kFusedWaves][kQueue];  // s | s' << 4 | s'' << 8 | both orderings << 12
  __shared__ uint32_t cq_q[kFusedWaves][kPairs];
  __shared__ uint16_t cq_code[kFusedWaves][kPairs];
  __shared__ long long rbase[kRecord ? kFusedWaves : 1][NB3];  // where the wave's entries of a branch start
  __shared__ int rlim[kRecord ? kFusedWaves : 1][NB3];         // and how many the count pass found
  __shared__ double2 phq[64];
  __shared__ double wq64[NB3];
  __shared__ float wq32[NB3];
  __shared__ double red[kFusedWaves][NB3];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N0 = p.N[0], N1 = p.N[1], N2 = p.N[2];
  // workgroup = one (live q, chunk) work item; the grid may hold more
  // workgroups than there are items
  const int n_work = *n_live_ptr * n_chunk;
  const int wk = blockIdx.x;
  if (wk >= n_work) return;
  const int kq = wk / n_chunk, chunk = wk - kq * n_chunk;
  const int q = live_list[kq];
  const int a0 = q / (N1 * N2), a1 = (q / N2) % N1, a2 = q % N2;
  const int t0 = (N0 - a0) % N0, t1 = (N1 - a1) % N1, t2 = (N2 - a2) % N2;

  // FP32 frequencies of the live branches, one per lane, NaN for the others
  // (they then fail every test), and the largest of all
  float w_lane = __builtin_nanf("");
  float wq_abs_max = 0.0f;
  unsigned live = 0;
#pragma unroll
  for (int s = 0; s < NB3; ++s) {
    const float w = (float)omega[q * NB3 + s];
    wq_abs_max = fmaxf(wq_abs_max, fabsf(w));
    const bool on = phys[q * NB3 + s] && sel[q * NB3 + s];
    live |= on ? (1u << s) : 0u;
    if (lane == s && on) w_lane = w;
  }
  if (tid < NB3) {
    wq64[tid] = omega[q * NB3 + tid];
    wq32[tid] = (float)omega[q * NB3 + tid];
  }
  const int sub = wk * kFusedWaves + wv;  // this wave's place among the counts
  if constexpr (kRecord) {
    if (lane < NB3) {
      long long b = tc.row_ptr[q * NB3 + lane];
      for (int c = kq * n_chunk * kFusedWaves; c < sub; ++c) b += tc.count[(size_t)c * NB3 + lane];
      rbase[wv][lane] = b;
      rlim[wv][lane] = tc.count[(size_t)sub * NB3 + lane];
    }
  }

  // 1. A~_q in LDS (the count pass projects nothing)
  if constexpr (MODE == kModeCount) __syncthreads();
  if constexpr (MODE != kModeCount) {
    for (int l = tid; l < n_rep; l += BS) {
      const int32_t* r = rep + 3 * l;
      int m0 = ((a0 * r[0]) % N0 + N0) % N0, m1 = ((a1 * r[1]) % N1 + N1) % N1,
          m2 = ((a2 * r[2]) % N2 + N2) % N2;
      double f = (double)m0 / N0 + (double)m1 / N1 + (double)m2 / N2;
      double sn, cs;
      sincospi(2.0 * f, &sn, &cs);
      phq[l] = make_double2(cs, sn);
    }
    const int n_at = p.n_blk * 9 * NB3;
    for (int k = tid; k < n_at; k += BS) at[k] = Cx<T>::make((T)0, (T)0);
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
      at[(e_blk[e] * 9 + e_bg[e]) * NB3 + s] = Cx<T>::make((T)re, (T)im);
    }
    __syncthreads();
  }

  constexpr int kPhaseCh = kFusedPhaseBytes / 16;
  double acc[NB3];
  int run[NB3];  // cache passes: entries of each branch so far (wave-uniform)
#pragma unroll
  for (int s = 0; s < NB3; ++s) {
    acc[s] = 0.0;
    run[s] = 0;
  }

  // 3. entries [0, n) of the wave's queue
  auto project = [&](int n) {
    {
      const int r = lane;
      const bool on = r < n;
      const uint32_t qq = on ? cq_q[wv][r] : 0u;
      const int code = on ? cq_code[wv][r] : 0;
      const int q1 = qq & 0xffff, q2 = qq >> 16;
      const int s = code & 15, s1 = (code >> 4) & 15, s2 = (code >> 8) & 15, dbl = code >> 12;
      const int m1 = q1 * NB3 + s1, m2 = q2 * NB3 + s2;
      // the partners' eigenvectors and (w, n, v)
      C x[NB3], y[NB3];
      double2 ra1, rb1, rc1, ra2, rb2, rc2;
      constexpr int CH = kPullBytes / 16;
      auto tail = [&](auto at_byte, double2& a, double2& b, double2& c) {
        a = *reinterpret_cast<const double2*>(at_byte(0));
        b = *reinterpret_cast<const double2*>(at_byte(16));
        c = *reinterpret_cast<const double2*>(at_byte(32));
      };
      auto vector = [&](auto at_byte, double first, C* e) {
        if constexpr (sizeof(T) == 8)
          e[0] = Cx<T>::make((T)first, (T)0);
        else
          e[0] = Cx<T>::make(__int_as_float(__double2loint(first)), __int_as_float(__double2hiint(first)));
        constexpr int kPer = 16 / sizeof(C);
#pragma unroll
        for (int j = 1; j < NB3; j += kPer) {
          typedef T Piece __attribute__((ext_vector_type(16 / sizeof(T))));
          const Piece v = *reinterpret_cast<const Piece*>(at_byte(48 + (j - 1) * (int)sizeof(C)));
          e[j] = Cx<T>::make(v[0], v[1]);
          if constexpr (kPer == 2) {
            if (j + 1 < NB3) e[j + 1] = Cx<T>::make(v[kPer], v[kPer + 1]);
          }
        }
      };
      int own_lane = lane;
      asm volatile("" : "+v"(own_lane));  // its addresses are not kept from batch to batch
      auto own = [&](int byte) { return pulled<CH>(st, own_lane, byte); };
      pull_rows<CH>(rec, kStride, m1, st, lane);
      tail(own, ra1, rb1, rc1);
      if constexpr (MODE != kModeCount) vector(own, rc1.y, x);
      lds_wave_sync();
      pull_rows<CH>(rec, kStride, m2, st, lane);
      tail(own, ra2, rb2, rc2);
      const double w1 = ra1.x, w2 = ra2.x, w = wq64[s];
      const double v1[3] = {rb1.x, rb1.y, rc1.x}, v2[3] = {rb2.x, rb2.y, rc2.x};
      // cache passes: the exact decision, and the entry's place in its row
      bool pass = on;
      int rank = 0;
      if constexpr (MODE != kModeGamma) {
        double s2p, s2m, Sp, Sm;
        widths2(p, v1, v2, s2p, s2m, Sp, Sm);
        pass = on && (exact_pass(p, w, w1, w2, Sp, Sm, true) || exact_pass(p, w, w1, w2, Sp, Sm, false) ||
                      (dbl && (exact_pass(p, w, w2, w1, Sp, Sm, true) ||
                               exact_pass(p, w, w2, w1, Sp, Sm, false))));
#pragma unroll
        for (int k = 0; k < NB3; ++k) {
          const unsigned long long m = __ballot(pass && s == k);
          if (s == k)
            rank = run[k] + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
          run[k] += __popcll(m);
        }
      }
      if constexpr (MODE == kModeCount) {
        lds_wave_sync();
        return;
      }
      // the weight before the second eigenvector and the phases arrive: what
      // it needs and what V needs are then not live together
      double wt = 0.0, am = 0.0;
      if (pass) {
        double sp, sm;
        widths_v(p, v1, v2, sp, sm);
        if constexpr (kRecord) {
          // a+ (n1 - n2) + 1/2 a- (n1 + n2 + 1) of this ordering plus, when
          // the entry stands for both, the mirrored one's a+r (n2 - n1) +
          // 1/2 a-r (n1 + n2 + 1): stored as c (n1 - n2) + d (n1 + n2 + 1)
          pair_factors(p, w, w1, w2, sp, sm, wt, am);
          if (dbl) {
            double apr, amr;
            pair_factors(p, w, w2, w1, sp, sm, apr, amr);
            wt -= apr;
            am += amr;
          }
        } else {
          wt = pair_weight_both(p, dbl, w, w1, w2, ra1.y, ra2.y, sp, sm);
        }
      }
      asm volatile("" : "+v"(own_lane) : "v"(wt));  // after the weight
      vector(own, rc2.y, y);
      lds_wave_sync();
      pull_rows<kPhaseCh>(phase_tab, 16 * kPhaseCh, q1, st, lane);
      if (pass) {
      auto phase = [&](int blk) {
        const int f = blk_f[blk];
        C v = *reinterpret_cast<const C*>(pulled<kPhaseCh>(st, own_lane, (f >> 1) * (int)sizeof(C)));
        if (f & 1) v.y = -v.y;
        return v;
      };
      T vr = 0, vi = 0;
      // V = sum_blk f_blk sum_beta x_beta (sum_gamma A~[blk][beta gamma] y_gamma):
      // complex multiply-adds as chains of fused multiply-adds into the
      // accumulators (four per product; the written form a.x b.x - a.y b.y
      // costs a multiply, a fused one and an add per component), and no
      // x (x) y table (nine complex values a block would have to keep or
      // recompute)
      // One block's term f_blk x_jb^T A~_blk y_kb into (vr, vi).
      auto block_term = [&](const C* ab, const C f, int jb, int kb) {
        T ur = 0, ui = 0;
#pragma unroll
        for (int be = 0; be < 3; ++be) {
          C a[3];
          T tr = 0, ti = 0;
#pragma unroll
          for (int ga = 0; ga < 3; ++ga) {
            a[ga] = ab[(be * 3 + ga) * NB3];
            const C v = y[3 * kb + ga];
            const bool real = sizeof(T) == 8 && 3 * kb + ga == 0;  // a turned eigenvector's first component
            tr = fma(a[ga].x, v.x, tr);
            if (!real) {
              tr = fma(-a[ga].y, v.y, tr);
              ti = fma(a[ga].x, v.y, ti);
            }
            ti = fma(a[ga].y, v.x, ti);
          }
          const C u = x[3 * jb + be];
          const bool real = sizeof(T) == 8 && 3 * jb + be == 0;
          ur = fma(u.x, tr, ur);
          ui = fma(u.x, ti, ui);
          if (!real) {
            ur = fma(-u.y, ti, ur);
            ui = fma(u.y, tr, ui);
          }
        }
        vr = fma(f.x, ur, vr);
        vr = fma(-f.y, ui, vr);
        vi = fma(f.x, ui, vi);
        vi = fma(f.y, ur, vi);
      };
#pragma unroll
      for (int jb = 0; jb < NB; ++jb) {
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
          const int b_lo = pair_ptr[jb * NB + kb], b_hi = pair_ptr[jb * NB + kb + 1];
          for (int blk = b_lo; blk < b_hi; ++blk)
            block_term(at + (size_t)blk * 9 * NB3 + s, phase(blk), jb, kb);
        }
      }
      const double vv = (double)vr * (double)vr + (double)vi * (double)vi;
      if constexpr (kRecord) {
        // both passes take the same decisions, so the rank is below the
        // count; a write outside this wave's share is refused
        if (rank < rlim[wv][s]) {
          const long long dst = rbase[wv][s] + rank;
          tc.pairs[dst] = make_uint2((unsigned)m1, (unsigned)m2);
          tc.factors[dst] = make_double2(vv * wt, 0.5 * (vv * am));
        } else {
          raise_flag(tc.flags, kFlagCache);
        }
      } else {
        const double c = wt * vv;
#pragma unroll
        for (int k = 0; k < NB3; ++k) acc[k] += (k == s) ? c : 0.0;
      }
      }
      lds_wave_sync();  // the buffer is free again
    }
  };

  // FP32 classification of the first n near pairs from the mode copies: a
  // candidate is any process with |x| < hi, the band's upper edge.  The
  // coalescence |x+| = |w + cp| and that of the mirrored ordering, |w - cp|
  // (= (w + w2) - w1), share the edge bp, and for w >= 0 the smaller of the two
  // is |w - |cp||, bitwise in FP32 (w + cp and w - cp round monotonically); so
  // one test covers both, with cpe = -|cp| on mirrored entries and cp
  // otherwise.  The decay |x-| is the same FP32 number for both.
  int n_cand = 0;  // wave-uniform
  auto classify = [&](int n, bool last) {
    for (int base = 0; base < n || (last && base == 0); base += 64) {
      const int r = base + lane;
      const bool on = r < n;
      const uint32_t qq = on ? wq_q[wv][r] : 0u;
      const int code = on ? wq_code[wv][r] : 0;
      const bool dbl = code >> 12;
      const float4 f1 = modef[((code >> 4) & 15) * p.nq + (qq & 0xffff)];
      const float4 f2 = modef[((code >> 8) & 15) * p.nq + (qq >> 16)];
      const float w = wq32[code & 15];
      float s2p, s2m, e_sig;
      widths2_f(p, f1, f2, s2p, s2m, e_sig);
      const float scl = wq_abs_max + fabsf(f1.w) + fabsf(f2.w);
      const float bp = make_band_f(s2p, scl, e_sig).hi, bm = make_band_f(s2m, scl, e_sig).hi;
      const float cp = f1.w - f2.w, cm = -f1.w - f2.w;
      const float cpe = dbl ? -fabsf(cp) : cp;
      const bool near = on && (fabsf(w + cpe) < bp || fabsf(w + cm) < bm);
      const unsigned long long m = __ballot(near);
      if (near) {
        const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)m, n_cand));
        cq_q[wv][slot] = qq;
        cq_code[wv][slot] = (uint16_t)code;
      }
      n_cand += __popcll(m);
      lds_wave_sync();
      while (n_cand >= 64 || (last && base + 64 >= n && n_cand > 0)) {
        project(min(n_cand, 64));
        // the rest, fewer than 64, moves to the front
        n_cand = max(n_cand - 64, 0);
        const uint32_t mq = cq_q[wv][64 + lane];
        const uint16_t mc = cq_code[wv][64 + lane];
        lds_wave_sync();
        cq_q[wv][lane] = mq;
        cq_code[wv][lane] = mc;
        lds_wave_sync();
      }
    }
  };

  // 2. sweep of the partner boxes: box index (i * waves + wave) * n_chunk +
  // chunk, so that the half of them the ordering q1 <_lex q2 empties is dealt
  // evenly
  const int d0 = box.d[0], d1 = box.d[1], d2 = box.d[2];
  const int k0 = lane / (d1 * d2), k1 = (lane / d2) % d1, k2 = lane % d2;  // this lane's point of a box
  const int n_box = box.n[0] * box.n[1] * box.n[2];
  const bool half = p.half != 0;
  const float hr = p.adaptive ? 2.008f : 0.0f;  // 2 sigma, with the slack of the FP32 bands (see below)
  const float r_min = 2.0f * (float)(p.adaptive ? p.sig_floor : p.sig_fixed) * 1.00001f;
  int fill = 0;  // wave-uniform
  for (int bi = wv * n_chunk + chunk; bi < n_box; bi += kFusedWaves * n_chunk) {
    const int p0 = bi / (box.n[1] * box.n[2]), p12 = bi - p0 * box.n[1] * box.n[2];
    const int p1 = p12 / box.n[2], p2 = p12 - p1 * box.n[2];
    const int o0 = p0 * d0, o1 = p1 * d1, o2 = p2 * d2;
    const int b0 = o0 + k0, b1 = o1 + k1, b2 = o2 + k2;
    bool valid = k0 < d0 && b0 < N0 && b1 < N1 && b2 < N2;
    const int q1 = valid ? (b0 * N1 + b1) * N2 + b2 : 0;
    const int q2 =
        valid ? (wrap_sub(t0, b0, N0) * N1 + wrap_sub(t1, b1, N1)) * N2 + wrap_sub(t2, b2, N2) : 0;
    if (half) valid = valid && q1 <= q2;
    const bool dbl = half && q1 < q2;
    if (!__ballot(valid)) continue;  // uniform
    // the box of q2: per axis c = t - b runs down from t - o, its lowest point
    // t - o - d + 1 (mod N)
    auto wrap = [](int x, int N) { return x < 0 ? (x + N < 0 ? x + 2 * N : x + N) : x; };
    const int c0 = wrap(t0 - o0 - d0 + 1, N0), c1 = wrap(t1 - o1 - d1 + 1, N1),
              c2 = wrap(t2 - o2 - d2 + 1, N2);
    const float4* win1 = window + (size_t)((o0 * N1 + o1) * N2 + o2) * NB3;
    const float4* win2 = window + (size_t)((c0 * N1 + c1) * N2 + c2) * NB3;
#pragma unroll 1
    for (int g = 0; g < NB3 * NB3; g += 64) {
      // which branches s of q can meet the cut with (s', s'') = this lane's:
      // |x| < 2 sigma for some frequencies of the ranges.  2 sigma <= 2 max(
      // floor, (|v1| + |v2|) h / sqrt(12)); the slack (0.4 % of the speeds' share,
      // 1e-6 of the frequencies) covers the bands' own margins and the rounding
      // of these tests, so no pair that passes its exact cut is dropped.
      unsigned bits = 0;
      float reach = 0.0f;
      const int cb = g + lane;
      if (cb < NB3 * NB3) {
        const float4 u = win1[cb / NB3], v = win2[cb % NB3];
        if (u.x <= u.y && v.x <= v.y) {
          reach = fmaxf(r_min, hr * (u.z + v.z)) + 1e-6f * (wq_abs_max + u.y + v.y) + 1e-8f;
          const float dlo = u.x - v.y, dhi = u.y - v.x;  // w1 - w2
          const float slo = u.x + v.x, shi = u.y + v.y;  // w1 + w2
#pragma unroll
          for (int s = 0; s < NB3; ++s) {
            const float w = __builtin_bit_cast(
                float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w_lane), s));
            const bool fwd = w + dlo < reach && w + dhi > -reach;
            const bool rev = half && w - dhi < reach && w - dlo > -reach;
            const bool dec = w - shi < reach && w - slo > -reach;
            bits |= (fwd || rev || dec) ? 1u << s : 0u;
          }
        }
      }
      unsigned long long todo = __ballot(bits != 0);
      if (!todo) continue;
      // the frequencies of the lane's points, w2 one (s', s'') ahead; the
      // same reach holds point by point, so a pair outside it fails its
      // classification too
      int l = __ffsll((long long)todo) - 1, row = -1;
      float w1 = 0.0f, w2n = freq[(g + l) % NB3 * p.nq + q2];
      while (todo) {
        const int cur = g + l;
        unsigned sb = (unsigned)__builtin_amdgcn_readlane((int)bits, l);
        const float rc = __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, reach), l));
        todo &= todo - 1;
        const float w2 = w2n;
        if (cur / NB3 != row) {
          row = cur / NB3;
          w1 = valid ? freq[row * p.nq + q1] : __builtin_nanf("");
        }
        if (todo) {
          l = __ffsll((long long)todo) - 1;
          w2n = freq[(g + l) % NB3 * p.nq + q2];
        }
        const float cp = w1 - w2, cm = -w1 - w2;  // NaN below the floor: fails every comparison
        const float cpe = dbl ? -fabsf(cp) : cp;
        const int code = row << 4 | (cur % NB3) << 8 | (dbl ? 1 << 12 : 0);
        while (sb) {  // uniform
          const int s = __ffs(sb) - 1;
          sb &= sb - 1;
          const float w =
              __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w_lane), s));
          const bool near = fabsf(w + cpe) < rc || fabsf(w + cm) < rc;
          const unsigned long long m = __ballot(near);
          if (!m) continue;
          if (near) {
            const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((unsigned)m, fill));
            wq_q[wv][slot] = (unsigned)q1 | (unsigned)q2 << 16;
            wq_code[wv][slot] = (uint16_t)(code | s);
          }
          fill += __popcll(m);
          if (fill >= kFlush) {
            lds_wave_sync();
            classify(kFlush, false);
            // the rest, fewer than 64, moves to the front
            const uint32_t mq = wq_q[wv][kFlush + lane];
            const uint16_t mc = wq_code[wv][kFlush + lane];
            lds_wave_sync();
            wq_q[wv][lane] = mq;
            wq_code[wv][lane] = mc;
            fill -= kFlush;
          }
        }
      }
    }
  }
  lds_wave_sync();
  classify(fill, true);

  if constexpr (MODE == kModeCount) {
#pragma unroll
    for (int s = 0; s < NB3; ++s)
      if (lane == s) tc.count[(size_t)sub * NB3 + s] = run[s];
    return;
  }
  if constexpr (kRecord) return;

  // 4. fixed order: a butterfly per wave, then the waves in turn
#pragma unroll
  for (int s = 0; s < NB3; ++s) {
    const double v = wave_sum_fixed(acc[s]);
    if (lane == 0) red[wv][s] = v;
  }
  __syncthreads();
  if (tid < NB3) {
    double sum = red[0][tid];
    for (int w = 1; w < kFusedWaves; ++w) sum += red[w][tid];
    part[(size_t)wk * NB3 + tid] = sum;
  }
}

// Row pointers of the temperature cache: the entry count of mode (q, s) is
// the sum over the waves of its q's work items (0 when q has no live mode),
// rows in mode order.  tc_rows counts and scans blocks of 1024 modes,
// tc_rows_sum scans the blocks' totals (at most 960 of them), tc_rows_add adds
// each block's start.  Up to kRowBlocks go one after the other in one workgroup,
// which needs neither (diamond, adaptive, FP64, the whole build: 4^3 129 us,
// 171 in three launches; 6^3, two blocks, 152 and 182; 10^3, six, 337 and 357;
// 11^3, eight, 454 and 465, in FP32 466 and 462).
constexpr int kRowBlocks = 8;

__global__ __launch_bounds__(1024) void tc_rows(int n_modes, int nb3, const int32_t* __restrict__ idx_of_q,
                                                int n_sub, const int32_t* __restrict__ count,
                                                long long* __restrict__ row_ptr,
                                                long long* __restrict__ block_sum) {
  __shared__ long long wave_tot[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n_turn = gridDim.x == 1 ? (n_modes + 1023) / 1024 : 1;
  long long total = 0;
  for (int t = 0; t < n_turn; ++t) {
    const int m = (blockIdx.x + t) * 1024 + tid;
    long long own = 0;
    if (m < n_modes) {
      const int q = m / nb3, s = m - q * nb3, k = idx_of_q[q];
      if (k >= 0)
        for (int c = 0; c < n_sub; ++c) own += count[((size_t)k * n_sub + c) * nb3 + s];
    }
    long long incl = own;
    for (int off = 1; off < 64; off <<= 1) {
      const long long v = __shfl_up(incl, off, 64);
      if (lane >= off) incl += v;
    }
    if (lane == 63) wave_tot[t & 1][wv] = incl;
    __syncthreads();
    long long before = total;
    for (int k = 0; k < 16; ++k) {
      before += k < wv ? wave_tot[t & 1][k] : 0;
      total += wave_tot[t & 1][k];
    }
    if (m < n_modes) row_ptr[m] = before + incl - own;
  }
  if (tid == 0) {
    block_sum[blockIdx.x] = total;
    if (gridDim.x == 1) row_ptr[n_modes] = total;
  }
}

__global__ __launch_bounds__(1024) void tc_rows_sum(int n_block, int n_modes, long long* __restrict__ block_sum,
                                                    long long* __restrict__ row_ptr) {
  __shared__ long long sums[1024];
  const int tid = threadIdx.x;
  const long long own = tid < n_block ? block_sum[tid] : 0;
  sums[tid] = own;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const long long v = tid >= off ? sums[tid - off] : 0;
    __syncthreads();
    sums[tid] += v;
    __syncthreads();
  }
  if (tid < n_block) block_sum[tid] = sums[tid] - own;
  if (tid == 1023) row_ptr[n_modes] = sums[1023];
}

__global__ void tc_rows_add(int n_modes, const long long* __restrict__ block_sum,
                            long long* __restrict__ row_ptr) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < n_modes) row_ptr[m] += block_sum[m / 1024];
}

size_t fused_lds_bytes(const kaldo_crystal* c, int prec) {
  const size_t cs = prec == KALDO_FP64 ? 16 : 8;
  return (size_t)c->bloch.n_blk * 9 * c->nb3 * cs;
}

// What the requests the kernel serves leave of the LDS beside the A~ tables;
// its own queues and sums take kFusedOwnLds at most.
static size_t fused_static_lds(bool record) { return 27968 + (record ? 8192 : 0); }
constexpr size_t kFusedOwnLds = 11264;

// The buffers of the batches' records (and phases, which take no more).
static size_t fused_staged(int nb3, size_t cs) {
  return (size_t)kFusedWaves * 64 * ((48 + (nb3 - 1) * cs + 15) / 16 * 16);
}

static bool fused_fits(const kaldo_crystal* c, int prec, bool record) {
  if (c->nb < 1 || c->nb > 5 || c->n_rep > 64) return false;
  return fused_lds_bytes(c, prec) + fused_static_lds(record) <= c->lds_max;
}

bool fused_supported(const kaldo_crystal* c, int prec) {
  if (const char* f = std::getenv("KALDO_FORCE_GENERIC"))
    if (f[0] == '1') return false;
  return fused_fits(c, prec, false);
}
bool fused_record_supported(const kaldo_crystal* c, int prec) { return fused_fits(c, prec, true); }

// Chunks per q from the number of live q-points the host can know of: at most
// min(N_q, n_subset) (the grid covers that many), estimated as n_subset / 3N_b
// (every branch of a q selected) when choosing the chunk count, for about
// kFusedItems work items, and no chunk of fewer than two boxes a wave.  (A fixed
// item count keeps the summation order, and so the bits of Gamma, the same on
// every device.)  With few boxes a chunk's set-up (about two of them: A~, the
// tables) counts, and so does the number of rounds of the workgroups the device
// holds at once, kResident of 256 CUs: 9^3 in FP64 took 109 us in two chunks,
// two rounds.
constexpr int kFewBoxes = 64;
static long resident(size_t cs) { return cs == 16 ? 768 : 1024; }
static int fused_upper(long nq, int64_t n_subset) {
  return (int)(n_subset > 0 ? std::min<long>(nq, n_subset) : nq);
}
static long fused_guess(const kaldo_crystal* c, long nq, int64_t n_subset) {
  return n_subset > 0 ? std::max<long>(1, n_subset / c->nb3) : nq;
}
static int fused_n_chunk(const kaldo_crystal* c, const int* N, const Boxes& box, int64_t n_subset, size_t cs) {
  const long guess = fused_guess(c, (long)N[0] * N[1] * N[2], n_subset);
  const long boxes = n_boxes(box);
  if (boxes <= kFewBoxes) {
    const long most = std::min<long>({(long)kFusedMaxChunks, boxes / kFusedWaves, kFusedItems / guess + 1});
    int best = 1;
    long cost = 0;
    for (int k = 1; k <= std::max<long>(1, most); ++k) {
      const long t = (guess * k + resident(cs) - 1) / resident(cs) *
                     (2 + (boxes + kFusedWaves * k - 1) / (kFusedWaves * k));
      if (k == 1 || t <= cost) best = k, cost = t;
    }
    return best;
  }
  const int most = (int)std::max<long>(1, std::min<long>(kFusedMaxChunks, boxes / (2 * kFusedWaves)));
  return std::min(fused_chunks((int)std::min<long>(guess, 1l << 30), kFusedItems), most);
}
// Most work items of any request on a mesh: upper x n_chunk is at most 16 N_q,
// and, n_chunk being at most items / guess + 1 with guess >= n_subset / (2 nb3),
// 2 nb3 items + N_q.
size_t fused_max_items(const kaldo_crystal* c, long nq) {
  return (size_t)std::min<long>(kFusedMaxChunks * nq, 2l * c->nb3 * kFusedItems + nq);
}

// Cells of one or two atoms with few phases (nearest-neighbour Phi3: diamond has
// four), whose sweep costs as much as their projections, where the batches'
// buffers fit beside the tables; the others' projections outweigh it and go
// in rounds (lw_rounds.hip has both sides).  In rounds too: meshes more than four
// times as long as thick, whose boxes have few neighbours in q and prune little
// (diamond 1x1x300, FP32, fixed 0.2 THz: 74 us by boxes, 54 in rounds; 30x30x1,
// adaptive, FP64 447 and 402), and in FP32 a few q of a small mesh, whose boxes
// make fewer than 256 workgroups: rounds' chunks are finer (8^3, 17 q, adaptive:
// 58 and 45).
bool fused_boxes_cell(const kaldo_crystal* c, int prec) {
  if (c->nb > 2 || c->bloch.n_f * 16 > (int)kFusedPhaseBytes) return false;
  const size_t cs = prec == KALDO_FP64 ? 16 : 8;
  return fused_lds_bytes(c, prec) + fused_staged(c->nb3, cs) + kFusedOwnLds <= c->lds_max;
}
bool fused_boxes(const kaldo_crystal* c, int prec, const int32_t* N, int64_t n_subset) {
  const size_t cs = prec == KALDO_FP64 ? 16 : 8;
  if (std::max({N[0], N[1], N[2]}) > 4l * std::min({N[0], N[1], N[2]}) || !fused_boxes_cell(c, prec)) return false;
  const long nq = (long)N[0] * N[1] * N[2];
  if (cs == 16 || n_subset <= 0 || nq > kRoundsPoints) return true;
  return fused_guess(c, nq, n_subset) * std::max(1l, nq / (64 * kFusedWaves)) >= 256;
}

// The fused launch of one mode: tables, live list, chunking and the kernel,
// then what the mode needs after it (the Gamma finish, or the cache's row
// pointers).  Count and record passes of one request see the same live list
// and chunk count, so they make the same cut decisions in the same order.
template <typename T, int MODE>
static int launch_fused_impl(const kaldo_crystal* c, const LwParams& p, const double* omega,
                             const double* occ, const double* vel, const float4* modef,
                             const uint8_t* phys, const uint8_t* sel, const double* evec,
                             const FusedWs& ws, int64_t n_subset, double scale, double* gamma, TcOut tc,
                             hipStream_t st) {
  using C = typename Cx<T>::type;
  const int nq = p.nq;
  const int n_modes = nq * c->nb3;
  int32_t* live_list = ws.qlist;
  int32_t* idx_of_q = ws.qlist + nq;
  int32_t* n_live = ws.qlist + 2 * nq;
  const Boxes box = choose_boxes(p.N);
  const float hs = p.adaptive ? (float)std::sqrt(p.h2 / 12.0) : 0.0f;
  const int rb = (int)fused_record_bytes(c->nb3, sizeof(C));
  auto blocks = [](long n) { return (unsigned)((n + 255) / 256); };
  TableJobs jobs{};
  jobs.first[1] = blocks((long)n_modes * c->nb3);
  jobs.first[2] = jobs.first[1] + (MODE == kModeCount ? 0u : blocks((long)nq * c->bloch.n_f));
  jobs.first[3] = jobs.first[2] + blocks(4l * n_modes);
  jobs.first[4] = jobs.first[3] + blocks(nq);
  KALDO_LAUNCH("lw_tables", lw_tables<T>, dim3(jobs.first[4]), dim3(256), 0, st, jobs, p, box, hs, rb,
               (int)kFusedPhaseBytes, n_subset > 0, evec, omega, occ, vel, modef, phys, sel, c->bloch.fvec, c->bloch.n_f, ws.rec, ws.phase_tab, ws.window,
               live_list, idx_of_q, n_live);
  if (n_subset > 0)
    KALDO_LAUNCH("lw_live_q", lw_live_q<true>, dim3(1), dim3(1024), 0, st, nq, c->nb3, phys, sel, live_list,
                 idx_of_q, n_live);
  const Fc3Bloch& b = c->bloch;
  const int n_chunk = fused_n_chunk(c, p.N, box, n_subset, sizeof(C));
  const unsigned grid = (unsigned)fused_upper(nq, n_subset) * n_chunk;
  // the count pass builds no A~ tables and stages the records' tails only
  const size_t at = MODE == kModeCount ? 0 : fused_lds_bytes(c, sizeof(T) == 8 ? KALDO_FP64 : KALDO_FP32);
  const size_t staged = MODE == kModeCount ? (size_t)kFusedWaves * 64 * 48 : fused_staged(c->nb3, sizeof(C));
  auto run = [&](auto kernel) {
    KALDO_LAUNCH("lw_fused", kernel, dim3(grid), dim3(kFusedThreads), at + staged, st, p, box, c->n_rep,
                 c->d_rep, omega, modef, ws.freq, phys, sel, evec, ws.rec, ws.phase_tab, ws.window,
                 b.t_ptr, b.t_i, b.t_l2, b.t_coef, b.e_blk, b.e_bg, b.blk_f, b.pair_ptr, live_list,
                 n_live, n_chunk, ws.part, tc);
  };
  if (c->nb == 1)
    run(lw_fused<1, T, MODE>);
  else if (c->nb == 2)
    run(lw_fused<2, T, MODE>);
  else {
    set_error("lw_fused: unsupported basis size");
    return KALDO_EUNSUPPORTED;
  }
  if (MODE == kModeGamma)
    KALDO_LAUNCH("lw_fused_finish", lw_fused_finish, dim3((n_modes + 255) / 256), dim3(256), 0, st,
                 n_modes, c->nb3, phys, sel, idx_of_q, n_chunk, ws.part, scale, gamma);
  if (MODE == kModeCount) {
    const int n_block = (n_modes + 1023) / 1024;
    KALDO_LAUNCH("tc_rows", tc_rows, dim3(n_block > kRowBlocks ? n_block : 1), dim3(1024), 0, st, n_modes, c->nb3, idx_of_q,
                 n_chunk * kFusedWaves, tc.count, tc.row_ptr, tc.block_sum);
    if (n_block > kRowBlocks) {
      KALDO_LAUNCH("tc_rows_sum", tc_rows_sum, dim3(1), dim3(1024), 0, st, n_block, n_modes, tc.block_sum,
                   tc.row_ptr);
      KALDO_LAUNCH("tc_rows_add", tc_rows_add, dim3((n_modes + 255) / 256), dim3(256), 0, st, n_modes,
                   tc.block_sum, tc.row_ptr);
    }
  }
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}

template <typename T>
int launch_fused(const kaldo_crystal* c, const LwParams& p, const double* omega, const double* occ,
                 const double* vel, const float4* modef, const uint8_t* phys, const uint8_t* sel,
                 const double* evec, const FusedWs& ws, int64_t n_subset, double scale, double* gamma,
                 hipStream_t st) {
  return launch_fused_impl<T, kModeGamma>(c, p, omega, occ, vel, modef, phys, sel, evec, ws, n_subset,
                                          scale, gamma, TcOut{}, st);
}

template <typename T>
int launch_fused_cache(const kaldo_crystal* c, const LwParams& p, int mode, const double* omega,
                       const double* occ, const double* vel, const float4* modef, const uint8_t* phys,
                       const uint8_t* sel, const double* evec, const FusedWs& ws, int64_t n_subset,
                       TcOut tc, hipStream_t st) {
  if (mode == kModeCount)
    return launch_fused_impl<T, kModeCount>(c, p, omega, occ, vel, modef, phys, sel, evec, ws, n_subset,
                                            0.0, nullptr, tc, st);
  return launch_fused_impl<T, kModeRecord>(c, p, omega, occ, vel, modef, phys, sel, evec, ws, n_subset,
                                           0.0, nullptr, tc, st);
}

#define KALDO_FUSED_FOR(T)                                                                          \
  template int launch_fused<T>(const kaldo_crystal*, const LwParams&, const double*, const double*, \
                               const double*, const float4*, const uint8_t*, const uint8_t*,        \
                               const double*, const FusedWs&, int64_t, double, double*,             \
                               hipStream_t);                                                        \
  template int launch_fused_cache<T>(const kaldo_crystal*, const LwParams&, int, const double*,     \
                                     const double*, const double*, const float4*, const uint8_t*,   \
                                     const uint8_t*, const double*, const FusedWs&, int64_t, TcOut, \
                                     hipStream_t);
KALDO_FUSED_FOR(float)
KALDO_FUSED_FOR(double)
#undef KALDO_FUSED_FOR

}  // namespace kaldo
