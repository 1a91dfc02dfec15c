// Gamma-point projection on the matrix cores.
//
// For each mode mu the vertex matrix is V_mu = E^T W_mu with W_mu = A_mu E
// (paper: Eq. phi3_proj with real eigenvectors).  When Phi3 is symmetric in
// its last two slots V_mu is symmetric, so only tiles (I, J) with I <= J of
// the 128 x 128 tiling are computed; an off-diagonal tile then stands for
// both orders of the partner pair, and its epilogue adds w(mu', mu'') +
// w(mu'', mu').  Without that symmetry every tile (I, J) is computed with the
// weight of its own order.  Tiles whose partner frequencies cannot meet the
// 2-sigma cut (in either order, for the symmetric form) are not launched, and
// inside a tile each wave multiplies only the 16 x 16 blocks that can (exact
// interval test on the frequency ranges of the strips' modes).
//
// Operands live in HBM transposed, k-contiguous: ET[m][k] = E[k][m] and
// WT[n][k] = W_mu[k][n], padded to a multiple of 128 with zeros.
//   FP32 form:  v_mfma_f32_16x16x4_f32 on FP32 operands.
//   BF16x3:     x = hi + lo with hi = bf16(x), lo = bf16(x - hi); each product
//               is hi*hi + hi*lo + lo*hi on v_mfma_f32_16x16x32_bf16 with
//               FP32 accumulation (lo*lo dropped).
// Workgroup: 512 threads = 8 waves, wave w owning rows 16 w .. 16 w + 15 of
// the tile as 8 MFMA 16 x 16 accumulators.  The K loop stages 128 x KT
// slices of both operands through LDS.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "lw_common.h"

namespace kaldo {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4;
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double d4;

constexpr int kMT = 128;   // output tile edge

__device__ __forceinline__ void split_bf16(float x, __bf16& hi, __bf16& lo) {
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}

// ET (FP64, FP32 or bf16 hi/lo) from E (FP64, [k][m]); zero padding beyond n.
// A non-finite entry of E raises kFlagNonFinite.
template <typename T>
__global__ void gm_prep_et(int n, int np, const double* __restrict__ E, T* __restrict__ et,
                           __bf16* __restrict__ eth, __bf16* __restrict__ etl,
                           int32_t* __restrict__ flags) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)np * np) return;
  const int m = idx / np, k = idx % np;
  const double x = (m < n && k < n) ? E[(size_t)k * n + m] : 0.0;
  if (!(x - x == 0.0)) raise_flag(flags, kFlagNonFinite);
  if (et) et[idx] = (T)x;
  if (eth) {
    // the high part rounds the FP32 value, not E's: the compiler otherwise
    // merges the two conversions into one from FP64
    float v = (float)x;
    asm("" : "+v"(v));
    __bf16 h, l;
    split_bf16(v, h, l);
    eth[idx] = h;
    etl[idx] = l;
  }
}

// E in FP32 with rows k-major (e32[k][m] = E[k][m], n x n): the SpMM stages
// its rows from this copy.
__global__ void gm_prep_e(int n, const double* __restrict__ E, float* __restrict__ e32) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < (long)n * n) e32[idx] = (float)E[idx];
}

// A_mu values in T for modes m0 .. m0 + nb - 1, in the ELL layout the SpMM
// reads with coalesced loads: the value of slot t of row b for mode j is
// avE[((t * batch / 4 + j / 4) * np + b) * 4 + j % 4] (zero for the padding
// slots and for rows b >= n).  A workgroup takes slot t, 16 rows and 256
// modes: the sums run with the modes across the threads (coalesced reads of
// E's rows), the tile is transposed through LDS, and each group of four modes
// is written as one run of 16 rows x 4 values.
constexpr int kAvRows = 16;
template <typename T>
__global__ __launch_bounds__(256) void gm_avals(int n, int np, int max_row, int m0, int nb, int batch,
                                                const int32_t* __restrict__ row_ptr,
                                                const int32_t* __restrict__ t_ptr,
                                                const int32_t* __restrict__ t_a,
                                                const double* __restrict__ t_coef,
                                                const double* __restrict__ E,
                                                T* __restrict__ avE) {
  __shared__ T tile[kAvRows][256 + 1];
  const int t = blockIdx.x, b0 = blockIdx.y * kAvRows, jh = blockIdx.z * 256;
  const int tid = threadIdx.x;
  const int j = jh + tid;  // this thread's mode in the batch
  for (int rb = 0; rb < kAvRows; ++rb) {
    const int b = b0 + rb;
    double s = 0.0;
    if (j < nb && b < n) {
      const int e = row_ptr[b] + t;
      if (e < row_ptr[b + 1])
        for (int u = t_ptr[e]; u < t_ptr[e + 1]; ++u) s += t_coef[u] * E[(size_t)t_a[u] * n + m0 + j];
    }
    tile[rb][tid] = (T)s;
  }
  __syncthreads();
  // 64 groups of four modes, each a run of kAvRows x 4 values
  for (int idx = tid; idx < 64 * kAvRows * 4; idx += 256) {
    const int jq = idx / (kAvRows * 4), w = idx % (kAvRows * 4), rb = w / 4, r = w % 4;
    if (jh + 4 * jq >= batch) break;  // a batch of fewer than 256 modes
    avE[(((size_t)t * (batch / 4) + jh / 4 + jq) * np + b0 + rb) * 4 + r] = tile[rb][4 * jq + r];
  }
}

// Frequency range [lo, hi] of the physical modes of each strip of 16 modes
// (lo > hi for a strip without any), one strip per 16 lanes.
constexpr int kStrip = 16;
__global__ __launch_bounds__(256) void gm_strip_ranges(int n, int ns, const double* __restrict__ omega,
                                                       const uint8_t* __restrict__ phys,
                                                       double2* __restrict__ srange) {
  const int m = blockIdx.x * 256 + threadIdx.x;
  const bool ok = m < n && phys[m];
  double lo = ok ? omega[m] : 1e300, hi = ok ? omega[m] : -1e300;
  for (int off = 1; off < kStrip; off <<= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  if (m % kStrip == 0 && m / kStrip < ns) srange[m / kStrip] = make_double2(lo, hi);
}

// Range of `count` consecutive strips.
__device__ __forceinline__ double2 gm_range(const double2* srange, int first, int count) {
  double2 r = srange[first];
  for (int k = 1; k < count; ++k) {
    r.x = fmin(r.x, srange[first + k].x);
    r.y = fmax(r.y, srange[first + k].y);
  }
  return r;
}

// Whether modes of the ranges a (first partner) and b (second) can hold a pair
// that meets the 2-sigma cut of mode frequency w, in the order (a, b) or, when
// both, in either (exact interval test).
__device__ __forceinline__ bool gm_can_meet(const LwParams& p, double w, double2 a, double2 b, bool both) {
  if (!(a.x <= a.y && b.x <= b.y)) return false;
  const double reach = 2.0 * p.sig_fixed * (1.0 + 1e-12) + 1e-9;
  auto can = [&](double2 u, double2 v) {
    const bool cp = (w + u.x - v.y) < reach && (w + u.y - v.x) > -reach;
    const bool cm = (w - u.y - v.y) < reach && (w - u.x - v.x) > -reach;
    return cp || cm;
  };
  return can(a, b) || (both && can(b, a));
}

struct GmTileInfo {
  int ti, tj;
};

// t-th tile: of the upper triangle (ti <= tj) for the symmetric form, of the
// full nt x nt tiling otherwise; row-major.
__host__ __device__ inline int gm_tile_count(int nt, bool sym) { return sym ? nt * (nt + 1) / 2 : nt * nt; }
__device__ __forceinline__ GmTileInfo gm_tile(int t, int nt, bool sym) {
  if (!sym) return {t / nt, t % nt};
  int ti = 0, rem = t;
  while (rem >= nt - ti) {
    rem -= nt - ti;
    ++ti;
  }
  return {ti, ti + rem};
}

// Live tiles of each mode: one wave per mode, tile t = 64 k + lane in bit
// `lane` of mask[mu][k] (n_word words a mode), and their number.  Then
// need[mu][J] = 1 when some strip pair the GEMM multiplies for mode mu reads
// the W columns of block J of kNeed columns (its rows lie in tiles I <= J / 2
// for the symmetric form, anywhere otherwise).  (One launch: with one each a
// step of a cell of one or two atoms took 46 us, with one 42.)
constexpr int kNeed = 64;
__global__ __launch_bounds__(256) void gm_live_mask(LwParams p, int nt, int n_tri, int n_word, int np, int n,
                                                    const double* __restrict__ omega,
                                                    const uint8_t* __restrict__ phys,
                                                    const uint8_t* __restrict__ sel,
                                                    const double2* __restrict__ srange,
                                                    unsigned long long* __restrict__ mask,
                                                    int32_t* __restrict__ count,
                                                    uint8_t* __restrict__ need) {
  const int mu = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (mu >= n) return;  // wave-uniform
  const bool sym = p.half != 0, on = sel[mu] && phys[mu];
  const double w = omega[mu];
  int c = 0;
  for (int k = 0; k < n_word; ++k) {
    const int t = 64 * k + lane;
    bool f = false;
    if (on && t < n_tri) {
      const GmTileInfo tt = gm_tile(t, nt, sym);
      f = gm_can_meet(p, w, gm_range(srange, tt.ti * (kMT / kStrip), kMT / kStrip),
                      gm_range(srange, tt.tj * (kMT / kStrip), kMT / kStrip), sym && tt.ti != tt.tj);
    }
    const unsigned long long m = __ballot(f);
    if (lane == 0) mask[(size_t)mu * n_word + k] = m;
    c += __popcll(m);
  }
  if (lane == 0) count[mu] = c;
  const int nj = np / kNeed;
  for (int J = lane; J < nj; J += 64) {
    bool any = false;
    if (on) {
      const double2 cols = gm_range(srange, J * (kNeed / kStrip), kNeed / kStrip);
      const int tj = J * kNeed / kMT, rows = (sym ? (tj + 1) * kMT : np) / kStrip;
      for (int I = 0; I < rows && !any; ++I)
        any = gm_can_meet(p, w, srange[I], cols, sym && I * kStrip / kMT != tj);
    }
    need[(size_t)mu * nj + J] = any ? 1 : 0;
  }
}

// Compacted list of the live (mode, tile) pairs of a batch, in (mode, tile)
// order: list[k] = jb * n_tri + t.  One workgroup per batch of `batch` <= 1024
// modes, a mode per thread after a scan of their counts; batch b's list starts
// at lists + b (batch n_tri + 1), its count is the region's last entry.  (One
// workgroup testing and compacting every pair took 85 us a step on the
// 512-atom glass.)
__global__ __launch_bounds__(1024) void gm_live_list(int n_tri, int n_word, int n, int batch,
                                                     const unsigned long long* __restrict__ mask,
                                                     const int32_t* __restrict__ count,
                                                     int32_t* __restrict__ lists) {
  __shared__ int wave_tot[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m0 = (int)blockIdx.x * batch, nb = min(batch, n - m0);
  int32_t* list = lists + (size_t)blockIdx.x * ((size_t)batch * n_tri + 1);
  const int own = tid < nb ? count[m0 + tid] : 0;
  int incl = own;
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off, 64);
    if (lane >= off) incl += v;
  }
  if (lane == 63) wave_tot[wv] = incl;
  __syncthreads();
  int at = incl - own;
  for (int k = 0; k < wv; ++k) at += wave_tot[k];
  if (tid < nb)
    for (int k = 0; k < n_word; ++k)
      for (unsigned long long m = mask[(size_t)(m0 + tid) * n_word + k]; m; m &= m - 1)
        list[at++] = tid * n_tri + 64 * k + (__ffsll((long long)m) - 1);
  if (tid == 1023) list[(size_t)batch * n_tri] = at;
}

__global__ void gm_zero(long n, double* __restrict__ x) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) x[k] = 0.0;
}

constexpr int kSpmmModes = 16;  // modes per workgroup
// Columns c' per workgroup and the LDS row stride of the staged E rows (16
// bytes of padding, so lanes reading the same columns of different rows fall
// in different banks): 272 bytes a row in either type.
template <typename T>
constexpr int spmm_cols() { return 256 / (int)sizeof(T); }
template <typename T>
constexpr int spmm_lds() { return 272 / (int)sizeof(T); }
// WT[j][c'][b] = sum_{k in row b} A_mu_j[b][col_k] E[col_k][c'], for a tile of
// kSpmmRows rows (one per lane), spmm_cols columns (a quarter per wave) and
// kSpmmModes modes.  The tile's E rows are staged in LDS; each lane walks its
// row's entries once per group of XW columns and updates XW x 16 accumulators
// per entry.  Writes are contiguous along b.  Products and sums in T; the
// split form stores hi and lo.
template <typename T>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3, sizeof(T) == 8 ? 2 : 3))) void gm_spmm(
    int n, int np, int nb, int batch, int n_rtiles, int max_row, const int32_t* __restrict__ col_ell,
    const int32_t* __restrict__ tile_u_ptr, const int32_t* __restrict__ tile_u,
    const T* __restrict__ avE, const T* __restrict__ ek, T* __restrict__ wt, __bf16* __restrict__ wth,
    __bf16* __restrict__ wtl, const uint8_t* __restrict__ need) {
  constexpr int COLS = spmm_cols<T>(), LDE = spmm_lds<T>();
  struct alignas(16) V4 {
    T v[4];
  };
  extern __shared__ float4 es4[];
  T* es = reinterpret_cast<T*>(es4);  // [n_u][LDE]
  const int rt = blockIdx.x, c0 = blockIdx.y * COLS, j0 = blockIdx.z * kSpmmModes;
  {
    // columns no strip the GEMM multiplies for these modes reads are not computed
    bool any = false;
    for (int j = 0; j < kSpmmModes && j0 + j < nb; ++j) any = any || need[(j0 + j) * (np / kNeed) + c0 / kNeed];
    if (!any) return;
  }
  const int b0 = rt * kSpmmRows;
  const bool has_rows = rt < n_rtiles;  // row tiles past the last row of A are zero
  const int u0 = has_rows ? tile_u_ptr[rt] : 0;
  const int n_u = has_rows ? tile_u_ptr[rt + 1] - u0 : 0;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int idx = tid; idx < n_u * COLS; idx += 256) {
    const int u = idx / COLS, x = idx % COLS;
    es[u * LDE + x] = (c0 + x < n) ? ek[(size_t)tile_u[u0 + u] * n + c0 + x] : (T)0;
  }
  __syncthreads();
  if (n_u == 0) {
    // no entries in these rows: W is zero there
    for (int idx = tid; idx < kSpmmModes * COLS * kSpmmRows; idx += 256) {
      const int j = idx / (COLS * kSpmmRows), x = (idx / kSpmmRows) % COLS, bb = idx % kSpmmRows;
      if (j0 + j >= nb) continue;
      const size_t g = ((size_t)(j0 + j) * np + c0 + x) * np + b0 + bb;
      if (wt) wt[g] = (T)0;
      if (wth) {
        wth[g] = (__bf16)0.0f;
        wtl[g] = (__bf16)0.0f;
      }
    }
    return;
  }
  const int b = b0 + lane;
  // every row takes max_row slots (padding slots hold zero values and read
  // staged row 0); the A values of slot t for the workgroup's 16 modes are
  // four groups of four that are contiguous across the wave's lanes
  const V4* av4 = reinterpret_cast<const V4*>(avE) + (size_t)(j0 / 4) * np + b;
  // each wave: its columns in passes of XW (XW x 16 accumulators), so every
  // nonzero's 16 mode values are loaded twice per column tile
  constexpr int XW = 32 / (int)sizeof(T);
  for (int xc = 0; xc < COLS / 4 / XW; ++xc) {
    const int x0 = wv * (COLS / 4) + XW * xc;
    T acc[XW][kSpmmModes];
#pragma unroll
    for (int x = 0; x < XW; ++x)
#pragma unroll
      for (int j = 0; j < kSpmmModes; ++j) acc[x][j] = 0;
    for (int t = 0; t < max_row; ++t) {
      const V4* ep = reinterpret_cast<const V4*>(&es[col_ell[(size_t)t * n + min(b, n - 1)] * LDE + x0]);
      V4 e[XW / 4];
#pragma unroll
      for (int x = 0; x < XW / 4; ++x) e[x] = ep[x];
      const V4* ap = av4 + (size_t)t * (batch / 4) * np;
      T a[kSpmmModes];
#pragma unroll
      for (int q = 0; q < kSpmmModes / 4; ++q) {
        const V4 v = ap[(size_t)q * np];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[4 * q + r] = v.v[r];
      }
#pragma unroll
      for (int j = 0; j < kSpmmModes; ++j)
#pragma unroll
        for (int x = 0; x < XW; ++x) acc[x][j] += a[j] * e[x / 4].v[x % 4];
    }
#pragma unroll
    for (int j = 0; j < kSpmmModes; ++j) {
      if (j0 + j >= nb) break;
#pragma unroll
      for (int x = 0; x < XW; ++x) {
        const size_t g = ((size_t)(j0 + j) * np + c0 + x0 + x) * np + b;
        const T v = acc[x][j];
        // W is read back only by the GEMM of this batch, long after it has
        // left the caches: streaming (non-temporal) stores
        if (wt) __builtin_nontemporal_store(v, &wt[g]);
        if (wth) {
          __bf16 h, l;
          split_bf16((float)v, h, l);
          __builtin_nontemporal_store(h, &wth[g]);
          __builtin_nontemporal_store(l, &wtl[g]);
        }
      }
    }
  }
}

// The vertex product of one live (mode, tile) pair, K in slices of KT, and the
// FP64 epilogue.  A workgroup's eight waves take 16 rows each and, of the 8
// strips of 16 columns, only those whose modes can meet the cut with its rows:
// the band of live pairs is narrower than a tile, and each wave crosses it
// alike; strips of rows or columns no wave multiplies are not fetched.  What
// bounds it is the operands' way in (W streams from HBM once per tile row:
// 5.5 GB a step on 512 atoms, 1.1 ms of 1.7 at the rate of a copy; the matrix
// units are busy a fifth of the time in FP32), hence two slices in flight.  Measured, us a step, whole tiles by four waves -> this: FP32 on 512
// atoms 3676 -> 1698, split on 384 atoms 835 -> 666; FP64 on 216 atoms 2444
// (generic VALU tiles of 64 x 64) -> 488.  A block's products keep their K
// order, so V is the same to the bit as with whole tiles.
enum GmForm { kGm32 = 0, kGmSplit = 1, kGm64 = 2 };
template <int FORM>
struct GmType {
  using T = float;
  using V4 = f4;
};
template <>
struct GmType<kGm64> {
  using T = double;
  using V4 = d4;
};
__device__ __forceinline__ f4 gm_mma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ d4 gm_mma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 gm_mma(bf16x8 a, bf16x8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr int kGemmThreads = 512;
// Waves per SIMD the registers are cut to: the FP32 form takes six, three
// workgroups a CU (512-atom glass 1.86 -> 1.70 ms a step against four; what
// spills is the epilogue's, outside the K loop), the others four (the split
// form 0.67 ms on 384 atoms, 0.87 with six; FP64's LDS holds two workgroups).
template <int FORM>
constexpr int gemm_waves() { return FORM == kGm32 ? 6 : 4; }
// The operands of one form: FP32 and FP64 as one array each, the split form
// as hi and lo (hi is at lo + the array's size).
template <int FORM>
__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(gemm_waves<FORM>()))) void gm_gemm(
    LwParams p, int n, int np, int m0, int n_tri, const typename GmType<FORM>::T* __restrict__ et,
    const __bf16* __restrict__ eth, const __bf16* __restrict__ etl,
    const typename GmType<FORM>::T* __restrict__ wt, const __bf16* __restrict__ wth,
    const __bf16* __restrict__ wtl, const double* __restrict__ omega, const double* __restrict__ occ,
    const uint8_t* __restrict__ phys, const double2* __restrict__ srange,
    const int32_t* __restrict__ live_list, const int32_t* __restrict__ live_count,
    double* __restrict__ partial) {
  using T = typename GmType<FORM>::T;
  using V4 = typename GmType<FORM>::V4;
  constexpr bool SPLIT = FORM == kGmSplit;
  constexpr int KT = SPLIT ? 32 : 16;
  // LDS rows padded by 16 bytes to stagger banks; FP32 and FP64 in two buffers
  constexpr int LDA = KT + (SPLIT ? 8 : 16 / (int)sizeof(T));
  constexpr int kBuf = kMT * LDA;
  __shared__ __attribute__((aligned(16))) T sA[SPLIT ? 4 : 2 * kBuf];
  __shared__ __attribute__((aligned(16))) T sB[SPLIT ? 4 : 2 * kBuf];
  __shared__ __attribute__((aligned(16))) __bf16 sAh[SPLIT ? kBuf : 8];
  __shared__ __attribute__((aligned(16))) __bf16 sAl[SPLIT ? kBuf : 8];
  __shared__ __attribute__((aligned(16))) __bf16 sBh[SPLIT ? kBuf : 8];
  __shared__ __attribute__((aligned(16))) __bf16 sBl[SPLIT ? kBuf : 8];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = np / kMT;
  // workgroup k takes the k-th live (mode, tile) pair; the rest of the grid
  // (sized for every pair) exits at once
  if ((int)blockIdx.x >= *live_count) return;
  const int pair = live_list[blockIdx.x];
  const int jb = pair / n_tri, t = pair % n_tri;
  const GmTileInfo tt = gm_tile(t, nt, p.half != 0);
  const int mu = m0 + jb;
  const int i0 = tt.ti * kMT, j0 = tt.tj * kMT;
  const double w = omega[mu];
  const bool offdiag = p.half != 0 && tt.ti != tt.tj;

  // column strips each wave's rows can meet, 8 bits a wave
  const unsigned long long live = __ballot(gm_can_meet(
      p, w, srange[i0 / kStrip + (lane >> 3)], srange[j0 / kStrip + (lane & 7)], offdiag));
  if (live == 0) return;  // the partial sums are zero already
  const unsigned mine = (unsigned)(live >> (8 * wv)) & 255u;
  // strips of rows and columns in some block multiplied: the others are not fetched
  auto row_on = [&](int r) { return (live >> (8 * (r / kStrip)) & 255ull) != 0; };
  auto col_on = [&](int r) { return (live & 0x0101010101010101ull << (r / kStrip)) != 0; };

  const size_t wbase = (size_t)jb * np * np;
  const int wm = kStrip * wv;  // wave rows inside the tile
  const int lr = lane & 15, lg = lane >> 4;
  V4 acc[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) acc[b] = V4{0, 0, 0, 0};

  // Staging registers are named scalars, not an array: the compiler moves a
  // private array indexed in a loop into LDS or scratch before unrolling, and
  // the prefetch then waits for its loads as soon as they are issued.
  if constexpr (!SPLIT) {
    // two LDS buffers: while a slice is multiplied the next is staged into the
    // idle one and the one after is on its way into registers; one barrier per
    // slice.
    // Each thread moves NP 16-byte pieces of both operands per slice.
    constexpr int PV = 16 / (int)sizeof(T);  // values per piece
    constexpr int PPR = KT / PV, RS = kGemmThreads / PPR;  // pieces per row, rows apart
    constexpr int NP = kMT / RS;
    static_assert(NP == 1 || NP == 2, "one or two pieces of each operand per thread");
    const int r0 = tid / PPR, cc = (tid % PPR) * PV;
    const T* ga = et + (size_t)(i0 + r0) * np + cc;
    const T* gb = wt + wbase + (size_t)(j0 + r0) * np + cc;
    const size_t rs = (size_t)RS * np;
    const int so = r0 * LDA + cc;
    const uint4 none = make_uint4(0, 0, 0, 0);
    // two slices in flight: set 0 holds the even ones, set 1 the odd ones
    uint4 pa00 = none, pa01 = none, pb00 = none, pb01 = none;
    uint4 pa10 = none, pa11 = none, pb10 = none, pb11 = none;
    const bool ra0 = row_on(r0), rb0 = col_on(r0);
    const bool ra1 = NP == 2 && row_on(r0 + RS), rb1 = NP == 2 && col_on(r0 + RS);
    auto fetch = [&](int k, uint4& a0, uint4& a1, uint4& b0, uint4& b1) {
      if (ra0) a0 = *reinterpret_cast<const uint4*>(ga + k);
      if (rb0) b0 = *reinterpret_cast<const uint4*>(gb + k);
      if (ra1) a1 = *reinterpret_cast<const uint4*>(ga + rs + k);
      if (rb1) b1 = *reinterpret_cast<const uint4*>(gb + rs + k);
    };
    auto stage = [&](int buf, const uint4& a0, const uint4& a1, const uint4& b0, const uint4& b1) {
      T* A = sA + buf * kBuf + so;
      T* B = sB + buf * kBuf + so;
      *reinterpret_cast<uint4*>(A) = a0;
      *reinterpret_cast<uint4*>(B) = b0;
      if constexpr (NP == 2) {
        *reinterpret_cast<uint4*>(A + RS * LDA) = a1;
        *reinterpret_cast<uint4*>(B + RS * LDA) = b1;
      }
    };
    fetch(0, pa00, pa01, pb00, pb01);
    fetch(KT, pa10, pa11, pb10, pb11);  // np >= 128: at least eight slices, an even number
    stage(0, pa00, pa01, pb00, pb01);
    __syncthreads();
    // K order inside the slice: lane group lg owns k in [4 lg, 4 lg + 4) and
    // MFMA step j pairs it with the group's j-th value (the same on both
    // operands), so a lane reads its k values with 16-byte LDS loads
    struct alignas(16) Q {
      T v[4];
    };
    auto multiply = [&](int buf) {
      if (!mine) return;
      const T* A = sA + buf * kBuf + (wm + lr) * LDA + 4 * lg;
      const T* B = sB + buf * kBuf + lr * LDA + 4 * lg;
      const Q a = *reinterpret_cast<const Q*>(A);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        if (!(mine >> b & 1u)) continue;  // wave-uniform
        const Q q = *reinterpret_cast<const Q*>(B + 16 * b * LDA);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[b] = gm_mma(a.v[j], q.v[j], acc[b]);
      }
    };
    for (int k0 = 0; k0 < np; k0 += 2 * KT) {
      const bool more = k0 + 2 * KT < np;
      if (more) fetch(k0 + 2 * KT, pa00, pa01, pb00, pb01);
      multiply(0);
      stage(1, pa10, pa11, pb10, pb11);
      __syncthreads();
      if (more) fetch(k0 + 3 * KT, pa10, pa11, pb10, pb11);
      multiply(1);
      if (more) stage(0, pa00, pa01, pb00, pb01);
      __syncthreads();
    }
  } else {
    // one LDS buffer, the next slice prefetched into registers while the
    // current one is multiplied: each thread moves one 16-byte piece (8 bf16)
    // of each of the four arrays per slice
    static_assert(kMT * (KT / 8) == kGemmThreads, "one piece per array and thread");
    const int r0 = tid / (KT / 8), cc = (tid % (KT / 8)) * 8;
    const size_t ra = (size_t)(i0 + r0) * np + cc, rb = wbase + (size_t)(j0 + r0) * np + cc;
    const int l0 = r0 * LDA + cc;
    const uint4 none = make_uint4(0, 0, 0, 0);
    uint4 xah = none, xal = none, xbh = none, xbl = none;
    const bool on_a = row_on(r0), on_b = col_on(r0);
    auto fetch = [&](int k) {
      if (on_a) {
        xah = *reinterpret_cast<const uint4*>(eth + ra + k);
        xal = *reinterpret_cast<const uint4*>(etl + ra + k);
      }
      if (on_b) {
        xbh = *reinterpret_cast<const uint4*>(wth + rb + k);
        xbl = *reinterpret_cast<const uint4*>(wtl + rb + k);
      }
    };
    auto stage = [&]() {
      *reinterpret_cast<uint4*>(&sAh[l0]) = xah;
      *reinterpret_cast<uint4*>(&sAl[l0]) = xal;
      *reinterpret_cast<uint4*>(&sBh[l0]) = xbh;
      *reinterpret_cast<uint4*>(&sBl[l0]) = xbl;
    };
    fetch(0);
    stage();
    __syncthreads();
    for (int k0 = 0; k0 < np; k0 += KT) {
      const bool more = k0 + KT < np;
      if (more) fetch(k0 + KT);
      if (mine) {
        const int oa = (wm + lr) * LDA + 8 * lg, ob = lr * LDA + 8 * lg;
        const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&sAh[oa]);
        const bf16x8 al = *reinterpret_cast<const bf16x8*>(&sAl[oa]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          if (!(mine >> b & 1u)) continue;  // wave-uniform
          const bf16x8 bh = *reinterpret_cast<const bf16x8*>(&sBh[ob + 16 * b * LDA]);
          const bf16x8 bl = *reinterpret_cast<const bf16x8*>(&sBl[ob + 16 * b * LDA]);
          acc[b] = gm_mma(al, bh, acc[b]);
          acc[b] = gm_mma(ah, bl, acc[b]);
          acc[b] = gm_mma(ah, bh, acc[b]);
        }
      }
      __syncthreads();  // every wave has read slice k0
      if (more) stage();
      __syncthreads();  // slice k0 + KT visible
    }
  }

  // Epilogue: accumulator item r of a lane is row row_of(r) of each 16 x 16
  // strip tile, column lr.  An off-diagonal tile of the symmetric form also
  // stands for its mirror.
  auto row_of = [&](int r) { return FORM == kGm64 ? 4 * r + lg : 4 * lg + r; };
  const double s2 = 2.0 * p.sig_fixed;
  double sum = 0.0;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (!(mine >> b & 1u)) continue;
    const int jn = j0 + 16 * b + lr;
    if (jn >= n || !phys[jn]) continue;
    const double w2 = omega[jn], n2 = occ[jn];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int im = i0 + wm + row_of(r);
      if (im >= n || !phys[im]) continue;
      const double w1 = omega[im];
      // quick reject: neither order of the pair is near the energy shell
      const double d1 = fabs(w + w1 - w2), d2 = fabs(w - w1 - w2);
      const double d3 = fabs(w + w2 - w1);
      const double lim = s2 * (1.0 + 1e-9) + 1e-9;
      if (d1 >= lim && d2 >= lim && (!offdiag || d3 >= lim)) continue;
      const double wt = pair_weight_both(p, offdiag, w, w1, w2, occ[im], n2, p.sig_fixed, p.sig_fixed);
      if (wt == 0.0) continue;
      const double v = (double)acc[b][r];
      sum += v * v * wt;
    }
  }
  // fixed order: a butterfly per wave, then the waves in turn
  __shared__ double red[kGemmThreads / 64];
  sum = wave_sum_fixed(sum);
  if (lane == 0) red[wv] = sum;
  __syncthreads();
  if (tid == 0) {
    double total = red[0];
    for (int k = 1; k < kGemmThreads / 64; ++k) total += red[k];
    partial[(size_t)mu * n_tri + t] = total;
  }
}

// One wave per mode, lanes over its tiles, a fixed butterfly.
__global__ __launch_bounds__(256) void gm_finish(int n, int n_tri, const double* __restrict__ partial,
                                                 const uint8_t* __restrict__ phys,
                                                 const uint8_t* __restrict__ sel,
                                                 double* __restrict__ gamma) {
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (m >= n || !sel[m]) return;  // wave-uniform
  double acc = 0.0;
  for (int t = lane; t < n_tri; t += 64) acc += partial[(size_t)m * n_tri + t];
  acc = wave_sum_fixed(acc);
  if (lane == 0) gamma[m] = phys[m] ? kPrefactor * acc : 0.0;
}

// The SpMM stages max_u rows of 272 bytes in LDS.
bool gm_supported(const kaldo_crystal* c) {
  return (size_t)c->gamma.max_u * spmm_lds<float>() * sizeof(float) <= 96 * 1024;
}

// Modes per launch: 512 (6.19 -> 5.88 ms a step of the 512-atom glass in FP32
// against 256; 768 measured the same); in FP64 256, which keeps W, the largest
// buffer, at the FP32 form's size, and 64 for cells of more than 4,096
// branches, whose W is as large as the generic kernels'.
template <int FORM>
static int gm_batch(int n) {
  return FORM != kGm64 ? 512 : n <= 4096 ? 256 : 64;
}
// Fewest modes per launch a smaller workspace is taken for: batches differ in
// time only.  FP64 goes down to the SpMM's sixteen, so that a workspace of the
// generic kernels' size, which is asked for at least, serves every cell it
// can (one of less than two tiles runs those kernels in it).  The other forms
// give up sixteen modes for the lists of live blocks.
template <int FORM>
static int gm_least_batch(int n) {
  return FORM != kGm64 ? gm_batch<FORM>(n) - kSpmmModes : kSpmmModes;
}

// Buffers of one form in the workspace.
template <int FORM>
struct GmWs {
  using T = typename GmType<FORM>::T;
  T *et, *ek, *av, *wt = nullptr;
  __bf16 *eth = nullptr, *etl = nullptr, *wth = nullptr, *wtl = nullptr;
  double* partial;
  double2* srange;
  uint8_t* need;
  int32_t *live_lists, *live_count;
  unsigned long long* live_mask;
  size_t total;
  GmWs(const kaldo_crystal* c, unsigned char* base, size_t batch) {
    const size_t n = c->nb3, np = (n + kMT - 1) / kMT * kMT;
    const size_t n_tri = gm_tile_count((int)(np / kMT), c->bloch.sym_jk != 0);
    size_t o = 0;
    auto take = [&](size_t bytes) {
      unsigned char* r = base + o;
      o += (bytes + 255) / 256 * 256;
      return r;
    };
    et = reinterpret_cast<T*>(take(np * np * sizeof(T)));
    ek = reinterpret_cast<T*>(take(FORM == kGm64 ? 0 : n * n * sizeof(T)));  // FP64: the caller's E
    if (FORM == kGmSplit) {
      eth = reinterpret_cast<__bf16*>(take(np * np * 2 * 2));  // hi and lo
      etl = eth + np * np;
    }
    av = reinterpret_cast<T*>(take((size_t)std::max(1, c->gamma.max_row) * np * batch * sizeof(T)));
    unsigned char* w = take(np * np * batch * sizeof(T));  // the split form's hi and lo: as much
    if (FORM == kGmSplit) {
      wth = reinterpret_cast<__bf16*>(w);
      wtl = wth + np * np * batch;
    } else {
      wt = reinterpret_cast<T*>(w);
    }
    partial = reinterpret_cast<double*>(take(n * n_tri * 8));
    srange = reinterpret_cast<double2*>(take(np / kStrip * 16));
    need = take(n * (np / kNeed));
    live_lists = reinterpret_cast<int32_t*>(take((n + batch - 1) / batch * (batch * n_tri + 1) * 4));
    live_mask = reinterpret_cast<unsigned long long*>(take(n * ((n_tri + 63) / 64) * 8));
    live_count = reinterpret_cast<int32_t*>(take(n * 4));
    total = o;
  }
};

template <int FORM>
static size_t gm_bytes(const kaldo_crystal* c, bool least) {
  return GmWs<FORM>(c, nullptr, least ? gm_least_batch<FORM>(c->nb3) : gm_batch<FORM>(c->nb3)).total;
}
size_t gm_workspace_bytes(const kaldo_crystal* c, int prec, bool least) {
  if (prec == KALDO_FP64) return gm_bytes<kGm64>(c, least);
  return prec == KALDO_BF16X3 ? gm_bytes<kGmSplit>(c, least) : gm_bytes<kGm32>(c, least);
}

template <int FORM>
static int run_gm_form(const char* gemm_name, const kaldo_crystal* c, const LwParams& p,
                       const double* omega, const double* evec, const double* occ,
                       const uint8_t* phys, const uint8_t* sel, unsigned char* ws, size_t bytes,
                       double* gamma, hipStream_t st) {
  using T = typename GmType<FORM>::T;
  // the largest batch the workspace holds (at least the least: the caller has checked)
  int batch = gm_batch<FORM>(c->nb3);
  while (batch > gm_least_batch<FORM>(c->nb3) && GmWs<FORM>(c, nullptr, batch).total > bytes) batch -= kSpmmModes;
  int32_t* flags = c->d_flags;
  const int n = c->nb3;
  const int np = (n + kMT - 1) / kMT * kMT;
  const int nt = np / kMT, n_tri = gm_tile_count(nt, p.half != 0);
  const GmWs<FORM> b(c, ws, batch);
  const long n_part = (long)n * n_tri;
  KALDO_LAUNCH("gm_zero", gm_zero, dim3((unsigned)((n_part + 255) / 256)), dim3(256), 0, st, n_part,
               b.partial);
  const long nn = (long)np * np;
  KALDO_LAUNCH("gm_strip_ranges", gm_strip_ranges, dim3((np + 255) / 256), dim3(256), 0, st, n,
               np / kStrip, omega, phys, b.srange);
  KALDO_LAUNCH("gm_prep_et", gm_prep_et<T>, dim3((nn + 255) / 256), dim3(256), 0, st, n, np, evec,
               FORM == kGmSplit ? nullptr : b.et, b.eth, b.etl, flags);
  const T* ek;
  if constexpr (FORM == kGm64) {
    ek = evec;
  } else {
    KALDO_LAUNCH("gm_prep_e", gm_prep_e, dim3((unsigned)(((long)n * n + 255) / 256)), dim3(256), 0, st,
                 n, evec, b.ek);
    ek = b.ek;
  }
  // the live (mode, tile) lists of every batch at once, one workgroup each
  const int n_batch = (n + batch - 1) / batch, n_word = (n_tri + 63) / 64;
  const size_t live_stride = (size_t)batch * n_tri + 1;
  KALDO_LAUNCH("gm_live_mask", gm_live_mask, dim3((unsigned)(n + 3) / 4), dim3(256), 0, st, p, nt, n_tri,
               n_word, np, n, omega, phys, sel, b.srange, b.live_mask, b.live_count, b.need);
  KALDO_LAUNCH("gm_live_list", gm_live_list, dim3((unsigned)n_batch), dim3(1024), 0, st, n_tri, n_word,
               n, batch, b.live_mask, b.live_count, b.live_lists);
  const size_t spmm_bytes = (size_t)c->gamma.max_u * spmm_lds<T>() * sizeof(T);
  for (int m0 = 0; m0 < n; m0 += batch) {
    const int nb = std::min(batch, n - m0);
    const int32_t* live_list = b.live_lists + (size_t)(m0 / batch) * live_stride;
    if (c->gamma.max_row > 0)
      KALDO_LAUNCH("gm_avals", gm_avals<T>, dim3((unsigned)c->gamma.max_row, (unsigned)(np / kAvRows),
                   (batch + 255) / 256), dim3(256), 0, st, n, np, c->gamma.max_row, m0, nb, batch,
                   c->gamma.row_ptr, c->gamma.t_ptr, c->gamma.t_a, c->gamma.t_coef, evec, b.av);
    KALDO_LAUNCH("gm_spmm", gm_spmm<T>, dim3(np / kSpmmRows, np / spmm_cols<T>(),
                 (nb + kSpmmModes - 1) / kSpmmModes), dim3(256), spmm_bytes, st, n, np, nb, batch,
                 c->gamma.n_rtiles, c->gamma.max_row, c->gamma.col_ell, c->gamma.tile_u_ptr,
                 c->gamma.tile_u, b.av, ek, b.wt, b.wth, b.wtl, b.need + (size_t)m0 * (np / kNeed));
    KALDO_LAUNCH(gemm_name, gm_gemm<FORM>, dim3(n_tri * nb), dim3(kGemmThreads), 0, st, p, n, np, m0, n_tri,
                 b.et, b.eth, b.etl, b.wt, b.wth, b.wtl, omega, occ, phys, b.srange, live_list,
                 live_list + (size_t)batch * n_tri, b.partial);
  }
  KALDO_LAUNCH("gm_finish", gm_finish, dim3((n + 3) / 4), dim3(256), 0, st, n, n_tri, b.partial, phys,
               sel, gamma);
  KALDO_HIP(hipGetLastError());
  return KALDO_OK;
}

int run_gm(const kaldo_crystal* c, const LwParams& p, const double* omega, const double* evec,
           const double* occ, const uint8_t* phys, const uint8_t* sel, unsigned char* ws,
           size_t bytes, int prec, double* gamma, hipStream_t st) {
  if (prec == KALDO_FP64)
    return run_gm_form<kGm64>("gm_gemm_fp64", c, p, omega, evec, occ, phys, sel, ws, bytes, gamma, st);
  if (prec == KALDO_BF16X3)
    return run_gm_form<kGmSplit>("gm_gemm_bf16x3", c, p, omega, evec, occ, phys, sel, ws, bytes, gamma, st);
  return run_gm_form<kGm32>("gm_gemm_fp32", c, p, omega, evec, occ, phys, sel, ws, bytes, gamma, st);
}

}  // namespace kaldo
