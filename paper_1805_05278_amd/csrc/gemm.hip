// MFMA GEMMs for gfx950: the six products of each EG recursion node (Alg. 2:
// M1 = V_L^T C, M2 = T_L^T M1, C -= V_L M2, M3 = V_L^T [0; V_R], M4 = M3 T_R,
// T12 = -T_L M4) and the compact-WY application of Q.
//
// One workgroup computes a BM x BN tile of C, its waves two down the rows and
// two or four across the columns, each a block of 16 x 16 MFMA tiles (the
// shapes stand at k_gemm).  Operands are staged through
// LDS in BK = 16 deep slices, k-major, with the next slice prefetched into
// registers while the current one is multiplied.  The MFMA computes C^T tiles
// (A' = op(B)^T, B' = op(A)^T) so that the lane-fast output index runs down a
// column of the column-major C and stores coalesce.
//
// Structure masks turn the stored unit lower trapezoidal V (R above its
// diagonal) and the upper triangular T into their mathematical values while
// they are loaded, so the factors never have to be copied out of A.
//
// Split-K (the paper's 1DMM with the K dimension distributed, Sec. 4 and
// Sec. 6.2) is used when the output has few tiles: each slice of K writes a
// partial product and a second kernel adds the partials in a fixed order, so
// results are bitwise reproducible.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "gemm.h"
#include "profiler.h"

namespace miqr {

struct GemmArgs {
  int64_t M, N, K, kchunk;
  double alpha, beta;
  const double* A;
  int64_t lda;
  const double* B;
  int64_t ldb;
  double* C;
  int64_t ldc;
  double* P;  // split-K partials (M x N each) or null
  int maskA, maskB;
  int add_identity;
};

// Tile of this workgroup.  Workgroups are dealt to the 8 XCDs in turn (id
// mod 8), and each XCD has its own L2; the linear id is remapped so that XCD
// k runs a contiguous range of the tile order.  The order walks groups of
// kGroup row tiles across all column tiles (column by column inside a group),
// split by split: the workgroups an XCD runs together share a few row panels
// of the left operand and column panels of the right one (or one split-K
// slice of V) in its L2, instead of every XCD fetching every panel.  Any
// bijection gives the same results: only the placement of the tiles changes.
struct TileId {
  int64_t x, y, z;
  __device__ TileId() {
    constexpr int64_t kXcd = 8, kGroup = 8;
    const int64_t gx = gridDim.x, gy = gridDim.y;
    const int64_t nb = gx * gy * gridDim.z;
    const int64_t id = blockIdx.x + gx * (blockIdx.y + gy * (int64_t)blockIdx.z);
    const int64_t q = nb / kXcd, r = nb % kXcd, k = id % kXcd, j = id / kXcd;
    const int64_t lid = k * q + min(k, r) + j;
    const int64_t per = gx * gy, t = lid % per;
    z = lid / per;
    const int64_t g = t / (kGroup * gy), x0 = g * kGroup, gs = min(gx - x0, kGroup);
    const int64_t u = t - g * kGroup * gy;
    x = x0 + u % gs;
    y = u / gs;
  }
};

template <int CMP>
struct MfmaTraits;

template <>
struct MfmaTraits<COMPUTE_F64> {
  typedef double T;
  typedef d4 Acc;
  static __device__ __forceinline__ Acc mma(T a, T b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return lk + 4 * r; }
};

template <>
struct MfmaTraits<COMPUTE_F32> {
  typedef float T;
  typedef f4 Acc;
  static __device__ __forceinline__ Acc mma(T a, T b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
};

// Per-thread global->register staging of one BK-deep slice of op(A) (BM x BK)
// or op(B)^T (BN x BK).  Element (i, k) of the slice is stored at
// (i, k) -> p[i + k ld] when the operand runs along i (not transposed A,
// transposed B) and at p[k + i ld] otherwise.  Each thread owns a fixed
// (i, k) pattern and a pointer advanced by a constant per slice, so the hot
// loop does no 64-bit multiplies.
template <int BX, int BK, bool ALONG_I, int NT = 256>
struct SliceLoader {
  static constexpr int L = BX * BK / NT;  // elements per thread
  const double* p;                         // this thread's first element
  int64_t step;                            // pointer advance per slice
  int64_t estride;                         // distance between a thread's elements
  int i, k;                                // position of the first element
  int di, dk;                              // position delta between elements
  __device__ void init(const double* base, int64_t ld, int64_t x0, int64_t kbeg, int t) {
    if (ALONG_I) {
      i = t % BX;
      k = t / BX;
      di = 0;
      dk = NT / BX;
      p = base + (x0 + i) + (kbeg + k) * ld;
      estride = (int64_t)dk * ld;
      step = (int64_t)BK * ld;
    } else {
      k = t % BK;
      i = t / BK;
      di = NT / BK;
      dk = 0;
      p = base + (kbeg + k) + (x0 + i) * ld;
      estride = (int64_t)di * ld;
      step = BK;
    }
  }
  // Issue the slice's loads.  Elements out of range read `safe` (a valid
  // address) instead; store() zeroes them and applies the structure mask.
  // No branch selects between loaded values here, so the loads stay in
  // flight across the MFMAs of the current slice.
  __device__ void load(double (&r)[L], bool plain, const double* safe, int64_t x0, int64_t X,
                       int64_t k0, int64_t kend) const {
#pragma unroll
    for (int s = 0; s < L; ++s) {
      const int64_t x = x0 + i + s * di, kk = k0 + k + s * dk;
      const bool ok = plain || (x < X && kk < kend);
      r[s] = *(ok ? p + s * estride : safe);
    }
  }
  // Store a loaded slice: out-of-range elements become 0, the structure
  // mask is applied on the stored (row, col) = along_i ? (x, kk) : (kk, x).
  template <typename T, int LD, bool TRANS>
  __device__ void store_masked(T (*S)[LD], const double (&r)[L], bool plain, int64_t x0, int64_t X,
                               int64_t k0, int64_t kend, int mask) const {
#pragma unroll
    for (int s = 0; s < L; ++s) {
      double v = r[s];
      if (!plain) {
        const int64_t x = x0 + i + s * di, kk = k0 + k + s * dk;
        const int64_t row = ALONG_I ? x : kk, col = ALONG_I ? kk : x;
        if (mask == MASK_UNIT_LOWER) v = (row < col) ? 0.0 : ((row == col) ? 1.0 : v);
        else if (mask == MASK_UPPER) v = (row > col) ? 0.0 : v;
        v = (x < X && kk < kend) ? v : 0.0;  // after the mask: no unit diagonal outside
      }
      if (TRANS) S[i + s * di][k + s * dk] = (T)v;
      else S[k + s * dk][i + s * di] = (T)v;
    }
  }
  // Loads and stores of a slice known to be plain (in range, mask-free).
  __device__ void load_plain(double (&r)[L]) const {
#pragma unroll
    for (int s = 0; s < L; ++s) r[s] = p[s * estride];
  }
  template <typename T, int LD, bool TRANS>
  __device__ void store_plain(T (*S)[LD], const double (&r)[L]) const {
#pragma unroll
    for (int s = 0; s < L; ++s) {
      if (TRANS) S[i + s * di][k + s * dk] = (T)r[s];
      else S[k + s * dk][i + s * di] = (T)r[s];
    }
  }
  __device__ void advance() { p += step; }
};

// Whether every element of a slice (rows x0 .. x0+BX-1 of op, k0 .. k0+BK-1)
// is in range and unaffected by the structure mask.
template <int BX, int BK, bool ALONG_I>
__host__ __device__ __forceinline__ bool slice_is_plain(int64_t x0, int64_t X, int64_t k0,
                                                        int64_t kend, int mask) {
  if (x0 + BX > X || k0 + BK > kend) return false;
  // stored row/col ranges
  const int64_t r0 = ALONG_I ? x0 : k0, r1 = ALONG_I ? x0 + BX - 1 : k0 + BK - 1;
  const int64_t c0 = ALONG_I ? k0 : x0, c1 = ALONG_I ? k0 + BK - 1 : x0 + BX - 1;
  if (mask == MASK_UNIT_LOWER) return r0 > c1;  // strictly below the diagonal
  if (mask == MASK_UPPER) return r1 <= c0;      // on or above the diagonal
  (void)r1; (void)c0;
  return true;
}

// The slabs s (k0 = kbeg + s BK) for which slice_is_plain holds form an
// interval: the masks cut a half-plane in (row, col), so the plain slabs of
// one operand are a prefix or a suffix of the full slabs.  Narrows [*lo, *hi)
// to that interval.
template <int BX, int BK, bool ALONG_I>
__host__ __device__ __forceinline__ void plain_slab_range(int64_t x0, int64_t X, int64_t kbeg,
                                                          int64_t kend, int mask, int* lo,
                                                          int* hi) {
  const int64_t nfull = (kend - kbeg) / BK;  // slabs wholly inside [kbeg, kend)
  int64_t l = *lo, h = min((int64_t)*hi, nfull);
  if (x0 + BX > X) h = 0;
  // first slab index with kbeg + s BK >= need, last with kbeg + s BK <= lim
  auto from = [&](int64_t need) {
    need -= kbeg;
    l = max(l, need <= 0 ? (int64_t)0 : (need + BK - 1) / BK);
  };
  auto upto = [&](int64_t lim) {
    lim -= kbeg;
    h = min(h, lim < 0 ? (int64_t)0 : lim / BK + 1);
  };
  if (mask == MASK_UNIT_LOWER) {
    if (ALONG_I) upto(x0 - BK);  // stored (x, kk): plain iff x0 > k0 + BK - 1
    else from(x0 + BX);          // stored (kk, x): plain iff k0 > x0 + BX - 1
  } else if (mask == MASK_UPPER) {
    if (ALONG_I) from(x0 + BX - 1);  // plain iff x0 + BX - 1 <= k0
    else upto(x0 - BK + 1);          // plain iff k0 + BK - 1 <= x0
  }
  if (l > h) l = h;
  *lo = (int)l;
  *hi = (int)h;
}

// Workgroup shapes: eight waves of 64 x 32 for 128 x 128 tiles, four of 32 x 32
// for 64 x 64.  Both leave four waves on a SIMD (at most 128 registers): with
// two, waves of one workgroup stop together at every slab's barrier and the
// MFMA pipe runs at about 60 % (measured with persistent workgroups that hid
// every load).  Long FP32 products keep four waves of 64 x 64 for their 128 x
// 128 tiles (few_waves below).
template <int BM>
constexpr int kThreads = BM == 128 ? 512 : 256;

template <int BM, int BN, bool TA, bool TB, int CMP, int NT>
__global__ __launch_bounds__(NT, (BM == 128 && NT == 256 ? 2 : 4)) void k_gemm(GemmArgs g) {
  constexpr int WC = NT / 128;  // waves across the columns (2 down the rows)
  typedef MfmaTraits<CMP> Tr;
  typedef typename Tr::T T;
  typedef typename Tr::Acc Acc;
  constexpr int BK = 16;
  constexpr int PAD = 1;
  constexpr int WM = BM / 2, WN = BN / WC, SA = WM / 16, SB = WN / 16;
  // op(A) runs along i in memory when A is not transposed; op(B)^T (N x K)
  // runs along j when B is transposed.
  constexpr bool A_ALONG = !TA, B_ALONG = TB;
  typedef SliceLoader<BM, BK, A_ALONG, NT> LA_t;
  typedef SliceLoader<BN, BK, B_ALONG, NT> LB_t;
  __shared__ T As[2][BK][BM + PAD];
  __shared__ T Bs[2][BK][BN + PAD];
  const int t = threadIdx.x, w = t >> 6, l = t & 63, li = l & 15, lk = l >> 4;
  const int wm = w & 1, wn = w >> 1;
  const TileId tid;
  const int64_t i0 = tid.x * BM, j0 = tid.y * BN;
  int64_t kbeg = tid.z * g.kchunk;
  int64_t kend = min(g.K, kbeg + g.kchunk);
  // Slabs that a structure mask zeroes for the whole tile are left out:
  // op(A)[x, k] is nonzero only for k <= x (from the tile's last row) or only
  // for k >= x (from its first), likewise op(B).
  if (g.maskA != MASK_NONE) {
    if ((g.maskA == MASK_UNIT_LOWER) == A_ALONG) kend = min(kend, i0 + BM);
    else kbeg = max(kbeg, i0 / BK * BK);
  }
  if (g.maskB != MASK_NONE) {
    if ((g.maskB == MASK_UNIT_LOWER) == B_ALONG) kend = min(kend, j0 + BN);
    else kbeg = max(kbeg, j0 / BK * BK);
  }
  const int nslab = kend > kbeg ? (int)((kend - kbeg + BK - 1) / BK) : 0;

  Acc acc[SA][SB];
#pragma unroll
  for (int a = 0; a < SA; ++a)
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[a][b][r] = 0;

  LA_t la;
  LB_t lb;
  la.init(g.A, g.lda, i0, kbeg, t);
  lb.init(g.B, g.ldb, j0, kbeg, t);
  double ra[LA_t::L], rb[LB_t::L];
  int64_t kf = kbeg;  // first k of the slice held in ra / rb
  bool pa = true, pb = true;
  auto fetch = [&](int64_t k0) {
    kf = k0;
    pa = slice_is_plain<BM, BK, A_ALONG>(i0, g.M, k0, kend, g.maskA);
    pb = slice_is_plain<BN, BK, B_ALONG>(j0, g.N, k0, kend, g.maskB);
    la.load(ra, pa, g.A, i0, g.M, k0, kend);
    lb.load(rb, pb, g.B, j0, g.N, k0, kend);
    la.advance();
    lb.advance();
  };

  // Slabs [s1, s2) are plain for both operands: they are loaded and staged
  // without per-element range and mask selects.  The others (a prefix and a
  // suffix: the slabs that meet a structure mask, the ragged last slab, and
  // every slab of a tile that crosses the matrix edge) take the checked
  // path.  Each loop below prefetches the slab after the current one with the
  // path that slab needs, so no loaded value is merged across paths.
  int s1 = 0, s2 = nslab;
  plain_slab_range<BM, BK, A_ALONG>(i0, g.M, kbeg, kend, g.maskA, &s1, &s2);
  plain_slab_range<BN, BK, B_ALONG>(j0, g.N, kbeg, kend, g.maskB, &s1, &s2);
  if (nslab > 0) {
    if (s1 == 0 && s2 > 0) {
      la.load_plain(ra);
      lb.load_plain(rb);
      la.advance();
      lb.advance();
      la.template store_plain<T, BM + PAD, false>(As[0], ra);
      lb.template store_plain<T, BN + PAD, false>(Bs[0], rb);
    } else {
      fetch(kbeg);
      la.template store_masked<T, BM + PAD, false>(As[0], ra, pa, i0, g.M, kf, kend, g.maskA);
      lb.template store_masked<T, BN + PAD, false>(Bs[0], rb, pb, j0, g.N, kf, kend, g.maskB);
    }
  }
  __syncthreads();
  auto compute = [&](int cur) {
#pragma unroll
    for (int ks = 0; ks < BK / 4; ++ks) {
      T af[SA], bf[SB];
#pragma unroll
      for (int a = 0; a < SA; ++a) af[a] = As[cur][4 * ks + lk][wm * WM + 16 * a + li];
#pragma unroll
      for (int b = 0; b < SB; ++b) bf[b] = Bs[cur][4 * ks + lk][wn * WN + 16 * b + li];
#pragma unroll
      for (int a = 0; a < SA; ++a)
#pragma unroll
        for (int b = 0; b < SB; ++b) acc[a][b] = Tr::mma(bf[b], af[a], acc[a][b]);
    }
  };
  int it = 0;
  // Next slab before s1: checked.
  for (; it + 1 < s1 && it < nslab; ++it) {
    const int cur = it & 1;
    fetch(kbeg + (int64_t)(it + 1) * BK);
    compute(cur);
    la.template store_masked<T, BM + PAD, false>(As[cur ^ 1], ra, pa, i0, g.M, kf, kend, g.maskA);
    lb.template store_masked<T, BN + PAD, false>(Bs[cur ^ 1], rb, pb, j0, g.N, kf, kend, g.maskB);
    __syncthreads();
  }
  // Next slab in [s1, s2): plain.
  for (; it + 1 < s2; ++it) {
    const int cur = it & 1;
    la.load_plain(ra);
    lb.load_plain(rb);
    la.advance();
    lb.advance();
    compute(cur);
    la.template store_plain<T, BM + PAD, false>(As[cur ^ 1], ra);
    lb.template store_plain<T, BN + PAD, false>(Bs[cur ^ 1], rb);
    __syncthreads();
  }
  // Next slab at or after s2 (or none): checked.
  for (; it < nslab; ++it) {
    const int cur = it & 1;
    const bool more = it + 1 < nslab;
    if (more) fetch(kbeg + (int64_t)(it + 1) * BK);
    compute(cur);
    if (more) {
      la.template store_masked<T, BM + PAD, false>(As[cur ^ 1], ra, pa, i0, g.M, kf, kend, g.maskA);
      lb.template store_masked<T, BN + PAD, false>(Bs[cur ^ 1], rb, pb, j0, g.N, kf, kend, g.maskB);
    }
    __syncthreads();
  }

  // Epilogue, one 16-row slice at a time.  The C values of slice a + 1 are
  // loaded before slice a is stored, so each slice's loads are in flight
  // while the previous slice is written (the read latency of C is otherwise
  // exposed once per slice).
  double cv[SB][4];
  auto load_c = [&](int a) {
    const int64_t i = i0 + wm * WM + 16 * a + li;
    const bool row_ok = i < g.M;
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + wn * WN + 16 * b + Tr::row(lk, r);
        cv[b][r] = (row_ok && j < g.N && !g.P && g.beta != 0.0)
                       ? g.C[i + j * g.ldc] : 0.0;
      }
  };
  load_c(0);
#pragma unroll
  for (int a = 0; a < SA; ++a) {
    const int64_t i = i0 + wm * WM + 16 * a + li;
    const bool row_ok = i < g.M;
    double out[SB][4];
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + wn * WN + 16 * b + Tr::row(lk, r);
        const double v = g.alpha * (double)acc[a][b][r];
        out[b][r] = g.P ? v : v + g.beta * cv[b][r] + ((g.add_identity && i == j) ? 1.0 : 0.0);
      }
    if (a + 1 < SA) load_c(a + 1);
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + wn * WN + 16 * b + Tr::row(lk, r);
        if (!row_ok || j >= g.N) continue;
        if (g.P) g.P[tid.z * g.M * g.N + i + j * g.M] = out[b][r];
        else g.C[i + j * g.ldc] = out[b][r];
      }
  }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// BF16 inputs (FP64 operands rounded when staged), FP32 accumulation on
// v_mfma_f32_16x16x32_bf16.  One MFMA k-step per 32-deep slice; tiles are
// stored i-major so that a lane's fragment (8 consecutive k) is one 16-byte
// LDS read.  Fragment layout: a = A[l % 16][8 (l / 16) + e],
// b = B[8 (l / 16) + e][l % 16], acc[r] = D[4 (l / 16) + r][l % 16].
template <int BM, int BN, bool TA, bool TB>
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmArgs g) {
  constexpr int BK = 32, KP = BK + 8;
  constexpr int WM = BM / 2, WN = BN / 2, SA = WM / 16, SB = WN / 16;
  constexpr bool A_ALONG = !TA, B_ALONG = TB;
  typedef SliceLoader<BM, BK, A_ALONG> LA_t;
  typedef SliceLoader<BN, BK, B_ALONG> LB_t;
  __shared__ __align__(16) __bf16 As[2][BM][KP];
  __shared__ __align__(16) __bf16 Bs[2][BN][KP];
  const int t = threadIdx.x, w = t >> 6, l = t & 63, li = l & 15, lk = l >> 4;
  const int wm = w & 1, wn = w >> 1;
  const TileId tid;
  const int64_t i0 = tid.x * BM, j0 = tid.y * BN;
  const int64_t kbeg = tid.z * g.kchunk;
  const int64_t kend = min(g.K, kbeg + g.kchunk);
  const int nslab = (int)((kend - kbeg + BK - 1) / BK);
  f4 acc[SA][SB];
#pragma unroll
  for (int a = 0; a < SA; ++a)
#pragma unroll
    for (int b = 0; b < SB; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
  LA_t la;
  LB_t lb;
  la.init(g.A, g.lda, i0, kbeg, t);
  lb.init(g.B, g.ldb, j0, kbeg, t);
  double ra[LA_t::L], rb[LB_t::L];
  int64_t kf = kbeg;  // first k of the slice held in ra / rb
  bool pa = true, pb = true;
  auto fetch = [&](int64_t k0) {
    kf = k0;
    pa = slice_is_plain<BM, BK, A_ALONG>(i0, g.M, k0, kend, g.maskA);
    pb = slice_is_plain<BN, BK, B_ALONG>(j0, g.N, k0, kend, g.maskB);
    la.load(ra, pa, g.A, i0, g.M, k0, kend);
    lb.load(rb, pb, g.B, j0, g.N, k0, kend);
    la.advance();
    lb.advance();
  };
  // Plain slabs [s1, s2) skip the per-element selects, as in k_gemm.
  int s1 = 0, s2 = nslab;
  plain_slab_range<BM, BK, A_ALONG>(i0, g.M, kbeg, kend, g.maskA, &s1, &s2);
  plain_slab_range<BN, BK, B_ALONG>(j0, g.N, kbeg, kend, g.maskB, &s1, &s2);
  if (nslab > 0) {
    if (s1 == 0 && s2 > 0) {
      la.load_plain(ra);
      lb.load_plain(rb);
      la.advance();
      lb.advance();
      la.template store_plain<__bf16, KP, true>(As[0], ra);
      lb.template store_plain<__bf16, KP, true>(Bs[0], rb);
    } else {
      fetch(kbeg);
      la.template store_masked<__bf16, KP, true>(As[0], ra, pa, i0, g.M, kf, kend, g.maskA);
      lb.template store_masked<__bf16, KP, true>(Bs[0], rb, pb, j0, g.N, kf, kend, g.maskB);
    }
  }
  __syncthreads();
  auto compute = [&](int cur) {
    bf16x8 af[SA], bf[SB];
#pragma unroll
    for (int a = 0; a < SA; ++a) af[a] = *(const bf16x8*)&As[cur][wm * WM + 16 * a + li][8 * lk];
#pragma unroll
    for (int b = 0; b < SB; ++b) bf[b] = *(const bf16x8*)&Bs[cur][wn * WN + 16 * b + li][8 * lk];
#pragma unroll
    for (int a = 0; a < SA; ++a)
#pragma unroll
      for (int b = 0; b < SB; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[b], af[a], acc[a][b], 0, 0, 0);
  };
  int it = 0;
  for (; it + 1 < s1 && it < nslab; ++it) {
    const int cur = it & 1;
    fetch(kbeg + (int64_t)(it + 1) * BK);
    compute(cur);
    la.template store_masked<__bf16, KP, true>(As[cur ^ 1], ra, pa, i0, g.M, kf, kend, g.maskA);
    lb.template store_masked<__bf16, KP, true>(Bs[cur ^ 1], rb, pb, j0, g.N, kf, kend, g.maskB);
    __syncthreads();
  }
  for (; it + 1 < s2; ++it) {
    const int cur = it & 1;
    la.load_plain(ra);
    lb.load_plain(rb);
    la.advance();
    lb.advance();
    compute(cur);
    la.template store_plain<__bf16, KP, true>(As[cur ^ 1], ra);
    lb.template store_plain<__bf16, KP, true>(Bs[cur ^ 1], rb);
    __syncthreads();
  }
  for (; it < nslab; ++it) {
    const int cur = it & 1;
    const bool more = it + 1 < nslab;
    if (more) fetch(kbeg + (int64_t)(it + 1) * BK);
    compute(cur);
    if (more) {
      la.template store_masked<__bf16, KP, true>(As[cur ^ 1], ra, pa, i0, g.M, kf, kend, g.maskA);
      lb.template store_masked<__bf16, KP, true>(Bs[cur ^ 1], rb, pb, j0, g.N, kf, kend, g.maskB);
    }
    __syncthreads();
  }
  // Epilogue as in k_gemm: slice a + 1 of C is loaded before slice a is stored.
  double cv[SB][4];
  auto load_c = [&](int a) {
    const int64_t i = i0 + wm * WM + 16 * a + li;
    const bool row_ok = i < g.M;
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + wn * WN + 16 * b + 4 * lk + r;
        cv[b][r] = (row_ok && j < g.N && !g.P && g.beta != 0.0)
                       ? g.C[i + j * g.ldc] : 0.0;
      }
  };
  load_c(0);
#pragma unroll
  for (int a = 0; a < SA; ++a) {
    const int64_t i = i0 + wm * WM + 16 * a + li;
    const bool row_ok = i < g.M;
    double out[SB][4];
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + wn * WN + 16 * b + 4 * lk + r;
        const double v = g.alpha * (double)acc[a][b][r];
        out[b][r] = g.P ? v : v + g.beta * cv[b][r] + ((g.add_identity && i == j) ? 1.0 : 0.0);
      }
    if (a + 1 < SA) load_c(a + 1);
#pragma unroll
    for (int b = 0; b < SB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + wn * WN + 16 * b + 4 * lk + r;
        if (!row_ok || j >= g.N) continue;
        if (g.P) g.P[tid.z * g.M * g.N + i + j * g.M] = out[b][r];
        else g.C[i + j * g.ldc] = out[b][r];
      }
  }
}

// C = sum_z P[z] (+ beta C).  A block covers 64 consecutive elements with 4
// groups of splits: group g sums partials g, g + 4, g + 8, ... in order, and
// the four group sums are added in a fixed order, so the result does not
// depend on scheduling.
__global__ __launch_bounds__(256) void k_splitk_reduce(const double* P, int nsplit, int64_t M,
                                                       int64_t N, double beta, double* C,
                                                       int64_t ldc, int add_identity) {
  __shared__ double part[4][64];
  const int64_t MN = M * N;
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  double s0 = 0.0, s1 = 0.0;
  if (e < MN) {
    int z = g;
    for (; z + 4 < nsplit; z += 8) {
      s0 += P[(int64_t)z * MN + e];
      s1 += P[(int64_t)(z + 4) * MN + e];
    }
    if (z < nsplit) s0 += P[(int64_t)z * MN + e];
  }
  part[g][lane] = s0 + s1;
  __syncthreads();
  if (g == 0 && e < MN) {
    const double s = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
    const int64_t i = e % M, j = e / M;
    double* cp = C + i + j * ldc;
    *cp = ((beta == 0.0) ? s : s + beta * *cp) + ((add_identity && i == j) ? 1.0 : 0.0);
  }
}

// Thin products (C of a few columns, e.g. right-hand sides): bound by one read
// of A, which the 64-column tiles above pay with eight times the MFMA work and a
// trip through LDS.

struct ThinArgs {
  int64_t M, N, K, kchunk;
  double alpha, beta;
  const double* A;
  int64_t lda;
  const double* B;
  int64_t ldb;
  double* C;
  int64_t ldc;
  double* Ws;
  int maskA;
};

// Stored entry (r, c) of an operand read as v under its structure.
__device__ __forceinline__ double masked(int mask, int64_t r, int64_t c, double v) {
  const bool keep = (mask == MASK_NONE) | ((mask == MASK_UNIT_LOWER) & (r > c)) |
                    ((mask == MASK_UPPER) & (r <= c));
  return keep ? v : ((mask == MASK_UNIT_LOWER) & (r == c)) ? 1.0 : 0.0;
}

// C (M x N) = alpha A^T B (+ beta C), A stored K x M, at most NC columns: lanes
// along the rows (half a contiguous kilobyte of a column per load; the MFMA
// operand layout's lanes touch sixteen columns, and that form took 165 us where
// this takes 105), 64 / NC columns of A per wave, their NC sums per lane in
// registers, the next rows' loads in flight while these are added up.  The 64
// sums of a wave are added across its lanes by recursive halving (63
// exchanges), which leaves sum l in lane l.  262144 x 256 (0.54 GB) by 4 and 8
// columns: 105 and 125 us, 193 and 200 us in 64 x 64 tiles.
template <int NC>
__global__ __launch_bounds__(256, 2) void k_thin_tn(ThinArgs a) {
  constexpr int CW = 64 / NC;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t m0 = ((int64_t)blockIdx.x * 4 + w) * CW;
  const int64_t k0 = (int64_t)blockIdx.y * a.kchunk, k1 = min(a.K, k0 + a.kchunk);
  if (m0 >= a.M) return;
  double acc[64];
#pragma unroll
  for (int e = 0; e < 64; ++e) acc[e] = 0.0;
  auto load = [&](int64_t r, double (&x)[CW], double (&y)[NC]) {
#pragma unroll
    for (int n = 0; n < NC; ++n) y[n] = a.B[r + min((int64_t)n, a.N - 1) * a.ldb];
#pragma unroll
    for (int c = 0; c < CW; ++c) x[c] = a.A[r + min(m0 + c, a.M - 1) * a.lda];
  };
  auto mul = [&](const double (&x)[CW], const double (&y)[NC]) {
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
      for (int n = 0; n < NC; ++n) acc[c * NC + n] = fma(x[c], y[n], acc[c * NC + n]);
  };
  // Rows under the operand's structure and the last rows of the chunk.
  auto edge = [&](int64_t r0) {
    const int64_t r = r0 + lane;
    double x[CW], y[NC];
    load(min(r, k1 - 1), x, y);
#pragma unroll
    for (int c = 0; c < CW; ++c) x[c] = r < k1 ? masked(a.maskA, r, m0 + c, x[c]) : 0.0;
#pragma unroll
    for (int n = 0; n < NC; ++n) y[n] = r < k1 ? y[n] : 0.0;
    mul(x, y);
  };
  int64_t r = k0;
  const int64_t plain = a.maskA == MASK_NONE ? 0 : (a.maskA == MASK_UNIT_LOWER ? m0 + CW : a.K);
  for (; r < k1 && r < plain; r += 64) edge(r);
  if (r + 64 <= k1) {
    double xa[CW], ya[NC], xb[CW], yb[NC];
    load(r + lane, xa, ya);
    for (; r + 192 <= k1; r += 128) {
      load(r + 64 + lane, xb, yb);
      mul(xa, ya);
      load(r + 128 + lane, xa, ya);
      mul(xb, yb);
    }
    mul(xa, ya);
    r += 64;
  }
  for (; r < k1; r += 64) edge(r);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const bool up = (lane & o) != 0;
#pragma unroll
    for (int e = 0; e < o; ++e) {
      const double lo = acc[e], hi = acc[e + o];
      acc[e] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, o);
    }
  }
  const int64_t m = m0 + lane / NC;
  const int n = lane % NC;
  if (m >= a.M || n >= a.N) return;
  const double v = a.alpha * acc[0];
  if (a.Ws) {
    a.Ws[(int64_t)blockIdx.y * a.M * a.N + m + n * a.M] = v;
  } else {
    double* cp = a.C + m + n * a.ldc;
    *cp = a.beta == 0.0 ? v : v + a.beta * *cp;
  }
}

// C (M x N) = alpha A B (+ beta C), A stored M x K: RPT rows per thread (one
// coalesced load of A per row and column of A), the NC sums of a row in
// registers, B's entries broadcast from LDS.  262144 x 256 by 4, 8 and 16
// columns: 98, 107 and 138 us, 193 to 212 us in 64 x 64 tiles.
template <int NC, int RPT>
__global__ __launch_bounds__(256) void k_thin_nn(ThinArgs a) {
  constexpr int KS = 2048 / NC, U = 8;  // a multiple of eight entries of bs per thread
  __shared__ __align__(16) double bs[KS][NC];
  const int nt = blockDim.x;
  const int64_t row0 = (int64_t)blockIdx.x * nt * RPT;
  const bool plain = a.maskA == MASK_NONE || (a.maskA == MASK_UNIT_LOWER && row0 >= a.K);
  int64_t row[RPT];
  const double* ap[RPT];
  double acc[RPT][NC];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    row[i] = row0 + i * nt + threadIdx.x;
    ap[i] = a.A + min(row[i], a.M - 1);
#pragma unroll
    for (int n = 0; n < NC; ++n) acc[i][n] = 0.0;
  }
  for (int64_t kb = 0; kb < a.K; kb += KS) {
    const int ks = (int)min((int64_t)KS, a.K - kb);
    __syncthreads();
    for (int e0 = threadIdx.x; e0 < KS * NC; e0 += 8 * nt) {
      double v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int e = e0 + i * nt, k = e % KS, n = e / KS;
        v[i] = a.B[k < ks && n < a.N ? kb + k + n * a.ldb : 0];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int e = e0 + i * nt, k = e % KS, n = e / KS;
        bs[k][n] = k < ks && n < a.N ? v[i] : 0.0;
      }
    }
    __syncthreads();
    auto load = [&](int k, double (&v)[RPT][U]) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < RPT; ++i) v[i][u] = ap[i][(kb + k + u) * a.lda];
    };
    auto mul = [&](int k, const double (&v)[RPT][U]) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int n = 0; n < NC; ++n) {
          const double b = bs[k + u][n];
#pragma unroll
          for (int i = 0; i < RPT; ++i) acc[i][n] = fma(v[i][u], b, acc[i][n]);
        }
    };
    // Columns under the operand's structure and the last ones (as above).
    auto edge = [&](int k) {
      double v[RPT][U];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < RPT; ++i) v[i][u] = ap[i][(kb + (k + u < ks ? k + u : 0)) * a.lda];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < RPT; ++i) asm volatile("" : "+v"(v[i][u]));
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < RPT; ++i)
          v[i][u] = k + u < ks ? masked(a.maskA, row[i], kb + k + u, v[i][u]) : 0.0;
      mul(k, v);
    };
    int k = 0;
    if (plain && ks >= U) {
      double x[RPT][U], y[RPT][U];
      load(0, x);
      for (; k + 3 * U <= ks; k += 2 * U) {
        load(k + U, y);
        mul(k, x);
        load(k + 2 * U, x);
        mul(k + U, y);
      }
      mul(k, x);
      k += U;
    }
    for (; k < ks; k += U) edge(k);
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    if (row[i] >= a.M) continue;
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      if (n >= a.N) continue;
      double* cp = a.C + row[i] + n * a.ldc;
      const double v = a.alpha * acc[i][n];
      *cp = a.beta == 0.0 ? v : v + a.beta * *cp;
    }
  }
}

template <int NC>
static void launch_thin_nn(const ThinArgs& a, hipStream_t s) {
  // Two rows per thread (half the LDS reads per byte of A) once that fills the
  // chip; one wave per workgroup where rows are few.
  auto blocks = [&](int64_t rows) { return dim3((unsigned)((a.M + rows - 1) / rows)); };
  if (a.M >= 131072)
    hipLaunchKernelGGL((k_thin_nn<NC, 2>), blocks(512), dim3(256), 0, s, a);
  else if (a.M >= 65536)
    hipLaunchKernelGGL((k_thin_nn<NC, 1>), blocks(256), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_thin_nn<NC, 1>), blocks(64), dim3(64), 0, s, a);
}

// The thin kernels take FP64 products with a plain B of at most 8 columns (A^T:
// with 16 the sums leave four columns of A per wave, 221 us against 203) or 16
// (138 us against 212), from a long dimension of 1024 on (below, both paths take
// a few microseconds).  A B is not split along K, so a depth over 128 wants rows
// that fill the chip, 64 for each of it (with Q^T c and R x = c around it, 3000 x
// 1000 by 16 columns 664 us, 442 in split GEMM tiles; 20000 x 1000 by 16 749 and
// 554 us; 262144 x 256 by 4 355 and about 450 us).
static bool thin(const GemmDesc& d) {
  if (d.compute != COMPUTE_F64 || d.tb != 'N' || d.maskB != MASK_NONE || d.add_identity)
    return false;
  if (d.ta == 'T') return d.N <= 8 && d.K >= 1024;
  return d.N <= 16 && d.M >= 1024 && d.K <= std::max<int64_t>(128, d.M / 64);
}

// Returns the number of chunks of K (more than one: partial sums in scratch).
static int64_t launch_thin(const GemmDesc& d, hipStream_t s, double* scratch, int64_t capacity) {
  ThinArgs a{d.M, d.N, d.K, d.K, d.alpha, d.beta, d.A, d.lda, d.B, d.ldb, d.C, d.ldc, nullptr,
             d.maskA};
  if (d.ta == 'N') {
    if (d.N <= 4) launch_thin_nn<4>(a, s);
    else if (d.N <= 8) launch_thin_nn<8>(a, s);
    else launch_thin_nn<16>(a, s);
    return 1;
  }
  // Chunks for two workgroups per CU, of at least 256 rows.
  const int64_t wc = d.N <= 4 ? 64 : 32, mg = (d.M + wc - 1) / wc;
  int64_t ns = std::max<int64_t>(1, std::min((512 + mg - 1) / mg, d.K / 256));
  ns = std::max<int64_t>(1, std::min(ns, scratch ? capacity / (d.M * d.N) : 0));
  a.kchunk = ((d.K + ns - 1) / ns + 63) / 64 * 64;
  ns = (d.K + a.kchunk - 1) / a.kchunk;
  if (ns > 1) a.Ws = scratch;
  const dim3 grid((unsigned)mg, (unsigned)ns);
  if (d.N <= 4) hipLaunchKernelGGL(k_thin_tn<4>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_thin_tn<8>, grid, dim3(256), 0, s, a);
  return ns;
}

// FP32 MFMA takes half the time of FP64, so a long product is bound by its loads,
// and eight loads of an operand in flight per thread beat four by more than the
// second pair of waves gives.  A^T B: 1024 x 3072 x 16384 1407 us against 1635, 512
// x 256 x 131072 399 against 495, 512 x 256 x 16384 68 against 69; A B: 16384 x
// 1024 x 2048 662 against 730, 131072 x 256 x 512 424 against 453.  Shorter ones
// (512 x 256 x 4096 transposed 38 against 32 us, 16384 x 1024 x 256 115 against
// 109) and tiles that cross the edge (1024 x 511 x 131072 1822 against 1676) want
// the waves.
static bool few_waves(const GemmDesc& d) {
  if (d.compute != COMPUTE_F32 || d.tb != 'N' || d.N % 128 != 0) return false;
  const double mnk = (double)d.M * (double)d.N * (double)d.K;
  return d.ta == 'T' ? d.M % 128 == 0 && mnk >= 2e9 : d.K >= 256 && mnk >= 1.6e10;
}

template <int BM, int BN, int CMP>
static void launch_t(const GemmDesc& d, const GemmArgs& g, dim3 grid, hipStream_t s) {
  constexpr int NT = kThreads<BM>;
  if (d.ta == 'N' && d.tb == 'N')
    hipLaunchKernelGGL((k_gemm<BM, BN, false, false, CMP, NT>), grid, dim3(NT), 0, s, g);
  else if (d.ta == 'T' && d.tb == 'N')
    hipLaunchKernelGGL((k_gemm<BM, BN, true, false, CMP, NT>), grid, dim3(NT), 0, s, g);
  else if (d.ta == 'N' && d.tb == 'T')
    hipLaunchKernelGGL((k_gemm<BM, BN, false, true, CMP, NT>), grid, dim3(NT), 0, s, g);
  else
    hipLaunchKernelGGL((k_gemm<BM, BN, true, true, CMP, NT>), grid, dim3(NT), 0, s, g);
}

static void launch_few(const GemmDesc& d, const GemmArgs& g, dim3 grid, hipStream_t s) {
  if (d.ta == 'T')
    hipLaunchKernelGGL((k_gemm<128, 128, true, false, COMPUTE_F32, 256>), grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((k_gemm<128, 128, false, false, COMPUTE_F32, 256>), grid, dim3(256), 0, s, g);
}

template <int BM, int BN>
static void launch_bf16(const GemmDesc& d, const GemmArgs& g, dim3 grid, hipStream_t s) {
  if (d.ta == 'N' && d.tb == 'N')
    hipLaunchKernelGGL((k_gemm_bf16<BM, BN, false, false>), grid, dim3(256), 0, s, g);
  else if (d.ta == 'T' && d.tb == 'N')
    hipLaunchKernelGGL((k_gemm_bf16<BM, BN, true, false>), grid, dim3(256), 0, s, g);
  else if (d.ta == 'N' && d.tb == 'T')
    hipLaunchKernelGGL((k_gemm_bf16<BM, BN, false, true>), grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((k_gemm_bf16<BM, BN, true, true>), grid, dim3(256), 0, s, g);
}

// Tile size and split of K.
static void choose(const GemmDesc& d, int64_t scratch, int64_t* BM, int64_t* nsplit,
                   int64_t* kchunk) {
  auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  // FP64: 128 x 128 tiles where they fill the chip, with splits of at least 256
  // two workgroups a CU (256 x 3072 x 2500: 103 us in 480 of them, 85 us in 64 x
  // 64 tiles; 1024 x 1024 x 2500 115 and 107); 64 x 64 otherwise, and for updates
  // of depth 128 and less, which move more bytes of C than an MFMA time's worth:
  // four small workgroups a CU keep more of them in flight (12288 x 3072 at depth
  // 128: 234 us against 257 us; at depth 256 388 against 378 us, at 512 (49152
  // rows) 2.51 against 2.64 ms; 2500 x 3072 at depth 1024 348 against 318 us).
  const int64_t t128 = cdiv(d.M, 128) * cdiv(d.N, 128);
  const bool wide = d.M >= 128 && d.N >= 128;
  *BM = 64;
  if (d.compute == COMPUTE_F64) {
    if (wide && (d.beta == 0.0 ? t128 * std::max<int64_t>(d.K / 256, 1) >= 512
                               : d.K > 128 && t128 >= 256))
      *BM = 128;
  } else if (wide && (t128 >= 128 || d.K >= 4096)) {
    *BM = 128;
  }
  const int64_t tiles = cdiv(d.M, *BM) * cdiv(d.N, *BM);
  // Split of K: the one with the least estimated time, in microseconds.  A slab
  // takes a workgroup's MFMA time for every workgroup on its CU, and not less
  // than a memory latency allows; the operands are read from memory once; split
  // partials are written, read back (with C) and cost a launch, and a block of the
  // reduction reads a quarter of them one after the other.  (128 x 128 x 16384:
  // 97 us in 32 slices of 512 one tile wide, 24 us in 64 to 128 slices of four
  // tiles; 128 x 3072 x 12288: 245 us in 576 workgroups, one full and one nearly
  // empty wave of them, 185 us in 504; 16384 x 64 updates of depth 64: 23 us split
  // in two, 12 us whole; 64 x 64 x 64: 9.4 us split in two, 10.1 whole; 64 x 64 x
  // 262144: 105 us in 1024 slices, 43 of it the reduction, 79 us in 512.)  Over
  // 1300 shapes the split chosen takes 2 % longer than the best one in FP64, 3 %
  // in FP32 and 4 % in BF16.  In these a slab waits for its loads, and a second
  // workgroup on the CU costs nothing (4096 x 511 x 512 in BF16: 65 us in two
  // slices, 50 us in four).
  const double slots = *BM == 64 ? 1024 : 512, mn = (double)d.M * (double)d.N;
  const int64_t cap = std::min(d.K / (d.K >= 1024 ? 64 : 32), (int64_t)((double)scratch / mn));
  const double two = d.compute == COMPUTE_F64 ? 3.4 : 2.6;
  const double reads = 8.0 * ((double)d.K * (double)(d.M + d.N) + (d.beta == 0.0 ? 1 : 2) * mn);
  auto cost = [&](int64_t ns) {
    const double wgs = (double)(tiles * ns), waves = std::ceil(wgs / slots);
    const double occ = std::min(slots / 256, std::ceil(wgs / 256));
    const double slab = *BM == 64 ? std::max(1.6, 0.43 * occ) : (occ > 1 ? two : 2.6);
    return std::max(waves * (2.0 + (double)d.K / (16.0 * ns) * slab), reads / 4.5e6) +
           (ns > 1 ? 2.0 + std::max(0.06 * ns, (ns + 1.5) * mn * 16 / 4e6) : 0);
  };
  *nsplit = 1;
  double best = cost(1);
  for (int64_t wgs : {64, 128, 256, 512, 1024, 1536, 2048}) {
    const int64_t ns = std::min(wgs / tiles, cap);
    if (ns < 2) continue;
    const double c = cost(ns);
    if (c < best) {
      best = c;
      *nsplit = ns;
    }
  }
  *kchunk = cdiv(cdiv(d.K, *nsplit), 32) * 32;
  *nsplit = cdiv(d.K, *kchunk);
}

hipError_t gemm(const GemmDesc& d, hipStream_t s, double* scratch, int64_t scratch_doubles,
                double* flops) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  if (d.K <= 0) {
    // C = beta C: reuse the reduction kernel with zero partials is wasteful;
    // a K = 0 product only happens for empty panels, which callers avoid.
    return hipSuccess;
  }
  int64_t BM = 64, nsplit = 1, kchunk = d.K;
  const bool is_thin = thin(d);
  if (!is_thin) choose(d, scratch ? scratch_doubles : 0, &BM, &nsplit, &kchunk);
  const bool big = BM == 128;
  const int64_t tm = (d.M + BM - 1) / BM, tn = (d.N + BM - 1) / BM;
  GemmArgs g{d.M, d.N, d.K, kchunk, d.alpha, d.beta, d.A, d.lda, d.B, d.ldb,
             d.C, d.ldc, nsplit > 1 ? scratch : nullptr, d.maskA, d.maskB, d.add_identity};
  dim3 grid((unsigned)tm, (unsigned)tn, (unsigned)nsplit);
  const double gbytes = 8.0 * ((double)d.M * d.K + (double)d.K * d.N +
                               (d.beta == 0.0 ? 1.0 : 2.0) * (double)d.M * d.N);
  {
    TimedLaunch tl(s, d.compute == COMPUTE_F32    ? "gemm_f32"
                      : d.compute == COMPUTE_BF16 ? "gemm_bf16"
                                                  : "gemm_f64",
                   gbytes, 2.0 * (double)d.M * d.N * d.K);
    if (is_thin) {
      nsplit = launch_thin(d, s, scratch, scratch_doubles);
    } else if (d.compute == COMPUTE_BF16) {
      if (big) launch_bf16<128, 128>(d, g, grid, s);
      else launch_bf16<64, 64>(d, g, grid, s);
    } else if (d.compute == COMPUTE_F32) {
      if (big && few_waves(d)) launch_few(d, g, grid, s);
      else if (big) launch_t<128, 128, COMPUTE_F32>(d, g, grid, s);
      else launch_t<64, 64, COMPUTE_F32>(d, g, grid, s);
    } else {
      if (big) launch_t<128, 128, COMPUTE_F64>(d, g, grid, s);
      else launch_t<64, 64, COMPUTE_F64>(d, g, grid, s);
    }
  }
  if (nsplit > 1) {
    const int64_t MN = d.M * d.N;
    TimedLaunch tr(s, "gemm_splitk_reduce", 8.0 * (double)MN * (nsplit + 2), (double)MN * nsplit);
    const int blocks = (int)((MN + 63) / 64);
    hipLaunchKernelGGL(k_splitk_reduce, dim3(blocks), dim3(256), 0, s, (const double*)scratch,
                       (int)nsplit, d.M, d.N, d.beta, d.C, d.ldc, d.add_identity);
  }
  if (flops) *flops += 2.0 * (double)d.M * (double)d.N * (double)d.K;
  return hipGetLastError();
}

}  // namespace miqr
