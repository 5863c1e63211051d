// TSQR panel factorisation for gfx950 (App. C of the paper: upsweep,
// downsweep, Householder reconstruction; base case of 1D-CAQR-EG, Sec. 6.1).
//
// Reduction structure.  The panel's rows are split evenly into leaf blocks of
// at most 128 or 256 rows (at least nbr rows each).  A workgroup reduces a
// *chain* of consecutive leaf blocks in sequence: the first block gets a
// local Householder QR of its own rows (App. C.1); every further block X_s is
// stacked under the running R and the stacked matrix is factored,
//     [R; X_s] = Q_s [R_new; 0],   Q_s = I - [I; Y_s] T_s [I; Y_s]^T,
// with the structure of the stacked triangle exploited: the reflector for
// column j touches only row j of R and the rows of X_s.  Above the leaves,
// a tree node takes the R factors of up to `arity` children and performs the
// same step once, with the R factors of children 1.. stacked into one X.  The
// paper's binomial tree is arity 2 with one leaf block per chain; wider nodes
// trade a larger local QR for fewer sequential levels (the paper's
// latency/bandwidth parameter).
//
// Downsweep (App. C.2).  Starting from B at the root, a node hands
// B - T B to its first child and -Y_s (T B) to the others; a leaf chain is
// walked backwards (M = T_s B, block s receives -Y_s M, B <- B - M) and its
// first block receives [B; 0] - V (Z B) with Z = T V_top^T stored by the
// factorisation.  Started from B = I this yields W, the leading columns of
// the Q-factor.
//
// Householder reconstruction (App. C.2).  The root workgroup follows the path
// to leaf block 0 only, forms X (top rows of W), runs the sign-modified LU
// X + S = L U, and returns T = U S L^{-T}, R = -S R_root, and U^{-1}.  The
// downsweep proper starts from [U^{-1}, -S D] so that one pass over the
// leaves yields V = W U^{-1} and, optionally, the thin Q = -W S D (the
// paper's remark that starting from U^{-1} saves the second broadcast).  The
// top rows of V are L, written from the reconstruction, with R above the
// diagonal.
#include <algorithm>

#include "common.h"
#include "lanes.h"
#include "profiler.h"
#include "tsqr.h"
#include "plan.h"

namespace miqr {

struct ChainQRArgs {
  double* X;       // leaf level: panel (in place); tree level: child R array
  int64_t ldx;
  int64_t xrows;   // leaf level: panel rows
  int nblocks, chain_len, nbr;
  double* Y;       // tree levels: Y per node (kYS doubles, leading dim kYL)
  double* T;       // leaf: per block; tree: per node
  double* R;       // per chain / node
};

// ------------------------------------------------------------ block QR
//
// One workgroup of four waves factors a block of up to 256 x 64: its own rows
// (a chain's first leaf block), or rows stacked under an upper triangular R
// (later leaf blocks, tree nodes).  It is the compact-WY recursion of
// Sec. 2.3 inside the block: 16-column sub-panels, each factored column by
// column and applied to the columns right of it with FP64 MFMA.
//
// Layout.  The block stays in registers: wave w holds RT row tiles of 16 rows
// and all four column tiles, in the MFMA accumulator layout (lane (g, cl)
// holds register r of rows m = g + 4 r of a tile in column cl).  Every column
// therefore lies across all four waves, one on each SIMD, and a column step
// is short everywhere at once: 4 RT products per lane for the dot products
// with the pivot column (broadcast inside the FMAs), a sum over the four
// lanes of a column, one exchange of 16 x 4 partial sums through LDS (the
// step's only barrier), the reflector in every wave alike, and 4 RT FMAs of
// update.  The pivot lane's own dot product is its squared norm, and the dot
// products with the columns left of the pivot are the Gram entries that T is
// built from, so a step has one sum and one exchange.  The next sub-panel is
// always in register slot 0 (slots rotate), so the sixteen unrolled steps
// exist once in the code.
//   V^T X contracts over rows in the order the registers hold them, so both
// operands come straight from registers; only V W' needs V with rows and
// columns exchanged, through a few LDS tiles private to the wave.
//   Products are summed from zero and added to the larger term last (the rows of
// X, B of the downsweep and of the reconstruction): sums that start from that
// term round at its size every time.  Against extended precision 200 x 64 had
// 1.09, 1.11 and 1.14 times the errors in R, V and T of the unblocked column
// loop so, 0.97, 0.94 and 0.99 times them as it is.
//   Bound: the chain of 64 dependent column steps (latency), not arithmetic
// (a 256 x 64 block is about 3 MFLOP, 10 us on one CU) or memory.  LDS is
// under 80 KB and registers under 256, so two workgroups share a CU, and one
// fits beside a GEMM workgroup of the look-ahead stream.
//   Measured (MI355X; before: a 512-thread body of one pivot half-wave per
// column, 140 KB of LDS, two lane reductions per column): tree node of five
// 64 x 64 children 72 -> 45 us, first 256 x 64 leaf blocks 107 -> 59 us at one
// per CU, leaf chains of 1048576 x 64 (512 chains of 8) 1081 -> 735 us.  A
// column step takes 845 cycles, 54 k of a tree node's 105 k.
//
// A register's row inside its tile is pi(g, r) = 8 (r / 2) + 2 g + r % 2: a
// lane's register pairs are adjacent rows, loaded and stored as 16 bytes, and
// the four lanes of a column cover 64 consecutive bytes.  MFMA never sees the
// order: it only contracts over it or maps it to itself.

constexpr int kTLD = 17;            // row stride of a 16 x 16 tile in LDS
constexpr int kTile = 16 * kTLD;    // doubles per tile

// Tile (p, c), p <= c, of an upper triangle of 16 x 16 tiles.
__device__ __forceinline__ int tri(int p, int c) { return c * (c + 1) / 2 + p; }

struct NodeLds {
  double r[10][kTile];               // running R, upper tiles, row-major
  double t[10][kTile];               // T, upper tiles, row-major
  double red[4][3][kTile];           // per wave: partial W of slots 1..3, then V tiles
  double wp[3][kTile];               // slot s: W' (right of the sub-panel) or G T_b (left of it)
  __align__(16) double part[2][16][4];  // a column step's partial dot products
  double prow[2][16];                // and its pivot row (first blocks)
};

// Column J of T_b: T[:, J] = -tau_J T[:, :J] G[:J, J] (Sec. 2.3), lane cl
// holding row cl in t and G[cl, J] in gd (wave 0).
template <int J>
__device__ __forceinline__ void t_column(int w, int cl, double (&t)[16], double gd, double tau) {
  if (w != 0) return;
  double s0 = 0.0, s1 = 0.0;
  if constexpr (J > 0) bcast_terms<0>(gd, t, s0, s1);
  if constexpr (J > 4) bcast_terms<4>(gd, t, s0, s1);
  if constexpr (J > 8) bcast_terms<8>(gd, t, s0, s1);
  if constexpr (J > 12) bcast_terms<12>(gd, t, s0, s1);
  t[J] = cl == J ? tau : -tau * (s0 + s1);
}

// Column J of a sub-panel (b) held in xs (this wave's rows of its 16
// columns).  first: the pivot row is row J of wave b's tile 0, which is
// published and cleared, so that the dot products see only the rows below
// it; stacked: the pivot row is row J of the diagonal tile of R.  t holds row
// cl of T_b (wave 0), gd and taup the last step's Gram column and tau: column
// J - 1 of T_b, T[:, j] = -tau_j T[:, :j] G[:j, j] (Sec. 2.3), is formed while
// the partial sums are exchanged.
template <int J, int NX>
__device__ __forceinline__ void node_step(bool first, int b, int w, int g, int cl,
                                          double (&xs)[NX], double (&t)[16], double& gd,
                                          double& taup, double& mysc, NodeLds& S) {
  constexpr int gj = (J >> 1) & 3, rj = ((J >> 3) << 1) | (J & 1), par = J & 1;
  double* rrowp = &S.r[tri(b, b)][J * kTLD];
  if (first && w == b) {
    if (g == gj) {
      S.prow[par][cl] = xs[rj];
      xs[rj] = cl >= J ? 0.0 : xs[rj];
    }
  }
  double d0 = 0.0, d1 = 0.0;
  dots_bcast<J>(xs, d0, d1);
  const double pd = rows_sum(d0 + d1);
  if (g == 0) S.part[par][cl][w] = pd;
  // R's row is read before the barrier: wave 1 rewrites it after.
  double rrow = rrowp[cl];
  if constexpr (J > 0) t_column<J - 1>(w, cl, t, gd, taup);
  lds_barrier();
  const double2 q0 = *(const double2*)&S.part[par][cl][0];
  const double2 q1 = *(const double2*)&S.part[par][cl][2];
  if (first) rrow = S.prow[par][cl];
  const double dot = (q0.x + q0.y) + (q1.x + q1.y);  // x_j . x_cl
  const double alpha = readlane(rrow, J), sig2 = readlane(dot, J);
  double bt, tr, z;
  reflector(alpha, sig2, bt, tr, z);
  const bool refl = sig2 != 0.0;
  const double beta = refl ? bt : alpha, sc = refl ? z : 0.0, tau = refl ? tr : 0.0;
  // v_J . x_cl (v_J has a one in the pivot row); for cl < J it is
  // v_cl . v_J once scaled.
  const double wv = rrow + sc * dot;
  const double tw = tau * wv;
  const double nf = cl > J ? -(tw * sc) : 0.0;
  update_bcast<J>(xs, nf);
  if (w == 1 && g == 0 && cl >= J) rrowp[cl] = cl == J ? beta : rrow - tw;
  gd = cl < J ? mysc * wv : 0.0;
  taup = tau;
  mysc = cl == J ? sc : mysc;
}

template <int J, int NX>
__device__ __forceinline__ void node_steps(bool first, int b, int w, int g, int cl,
                                           double (&xs)[NX], double (&t)[16], double& gd,
                                           double& taup, double& mysc, NodeLds& S) {
  if constexpr (J < 16) {
    node_step<J>(first, b, w, g, cl, xs, t, gd, taup, mysc, S);
    node_steps<J + 1>(first, b, w, g, cl, xs, t, gd, taup, mysc, S);
  } else {
    t_column<J - 1>(w, cl, t, gd, taup);
  }
}

// Householder QR of the block in x (x[c][t]: column tile c, row tile t of this
// wave).  On return x holds the basis (zero above and one on the diagonal of
// a first block), S.r the new R, S.t the block's T (both after a barrier).
// TRI (tree nodes): the stacked rows are upper triangular children, one per
// wave, so row tiles below the sub-panel's diagonal are zero and skipped.
// first: S.r zero on entry, tile 0 of wave w holds rows 16 w .. 16 w + 15.
template <int RT, bool TRI>
__device__ __forceinline__ void node_qr(bool first, d4 (&x)[4][RT], int nbr, int w, NodeLds& S) {
  const int nsub = (nbr + 15) >> 4;
  for (int b = 0; b < nsub; ++b) {
    const int pw = min(16, nbr - 16 * b), bb = tri(b, b);
    double mysc = 0.0;
    {
      const int l = lane_id(), g = l >> 4, cl = l & 15;
      double xs[4 * RT], t[16], gd = 0.0, taup = 0.0;
#pragma unroll
      for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) xs[4 * k + r] = x[0][k][r];
#pragma unroll
      for (int k = 0; k < 16; ++k) t[k] = 0.0;
      node_steps<0>(first, b, w, g, cl, xs, t, gd, taup, mysc, S);
      if (w == 0 && g == 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) S.t[bb][cl * kTLD + k] = t[k];
      }
#pragma unroll
      for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[0][k][r] = xs[4 * k + r] * mysc;
      if (first && w == b && cl < pw) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          x[0][0][r] = (8 * (r >> 1) + 2 * g + (r & 1) == cl) ? 1.0 : x[0][0][r];
      }
    }
    // Slot s holds column tile (b + s) mod 4: right of the sub-panel while
    // b + s < 4 (absent beyond nbr), left of it (basis already) otherwise.
    const int nright = nsub - b;  // slots 1 .. nright - 1 are right of it
    const int l = lane_id(), g = l >> 4, cl = l & 15;
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      if (s < nright || s >= 4 - b) {
        d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < RT; ++k) {
          if (!TRI || k <= b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc = mfma64(x[0][k][r], x[s][k][r], acc);
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) S.red[w][s - 1][(g + 4 * r) * kTLD + cl] = acc[r];
      }
    }
    lds_barrier();
    // Wave s adds slot s's partial products.  Right of the sub-panel:
    // W = V_b^T X (+ R's rows), W' = T_b^T W, R's rows lose W'.  Left of it:
    // V_b^T V_q = G^T, kept as G T_b for T's block column b.
    if (w > 0 && (w < nright || w >= 4 - b)) {
      const int c = (b + w) & 3;
      double v[4], tb[4];
      d4 o = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = (g + 4 * r) * kTLD + cl;
        v[r] = (S.red[0][w - 1][e] + S.red[1][w - 1][e]) + (S.red[2][w - 1][e] + S.red[3][w - 1][e]);
        tb[r] = S.t[bb][e];
      }
      if (w < nright) {
        double* rt = S.r[tri(b, c)];
        double rv[4];
        if (!first) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            rv[r] = rt[(g + 4 * r) * kTLD + cl];
            v[r] += rv[r];
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) o = mfma64(tb[r], v[r], o);
        if (!first) {
#pragma unroll
          for (int r = 0; r < 4; ++r) rt[(g + 4 * r) * kTLD + cl] = rv[r] - o[r];
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) o = mfma64(v[r], tb[r], o);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) S.wp[w - 1][(g + 4 * r) * kTLD + cl] = o[r];
    }
    lds_barrier();
    if (nright > 1) {
      // X -= V_b W' on the slots right of the sub-panel.
      double wn[3][4];
#pragma unroll
      for (int s = 1; s < 4; ++s)
        if (s < nright) {
#pragma unroll
          for (int p = 0; p < 4; ++p) wn[s - 1][p] = -S.wp[s - 1][(g + 4 * p) * kTLD + cl];
        }
#pragma unroll
      for (int k = 0; k < RT; ++k) {
        if (!TRI || k <= b) {
          double* vt = S.red[w][k % 3];
          double va[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) vt[(g + 4 * r) * kTLD + cl] = x[0][k][r];
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int p = 0; p < 4; ++p) va[p] = vt[cl * kTLD + g + 4 * p];
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int s = 1; s < 4; ++s)
            if (s < nright) {
              d4 vw = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
              for (int p = 0; p < 4; ++p) vw = mfma64(va[p], wn[s - 1][p], vw);
              x[s][k] += vw;
            }
        }
      }
      if (first && w == b) {
        // Rows 16 b .. of the tiles right of the sub-panel are rows of R.
#pragma unroll
        for (int s = 1; s < 4; ++s)
          if (s < nright) {
            double* rt = S.r[tri(b, b + s)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              rt[(8 * (r >> 1) + 2 * g + (r & 1)) * kTLD + cl] = x[s][0][r];
              x[s][0][r] = 0.0;
            }
          }
      }
    }
    // Block column b of T: T_pb = -sum_q T_pq (G_qb T_b), q = p .. b - 1, wave p.
    if (w < b) {
      d4 o = d4{0.0, 0.0, 0.0, 0.0};
      for (int q = w; q < b; ++q) {
        const double* tq = S.t[tri(w, q)];
        const double* hq = S.wp[q + 3 - b];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          o = mfma64(tq[cl * kTLD + g + 4 * r], hq[(g + 4 * r) * kTLD + cl], o);
      }
      double* tp = S.t[tri(w, b)];
#pragma unroll
      for (int r = 0; r < 4; ++r) tp[(g + 4 * r) * kTLD + cl] = -o[r];
    }
    // Rotate the slots: the next sub-panel to slot 0.
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      const d4 x0 = x[0][k];
      x[0][k] = x[1][k];
      x[1][k] = x[2][k];
      x[2][k] = x[3][k];
      x[3][k] = x0;
    }
  }
  for (int b = nsub; b < 4; ++b) {
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      const d4 x0 = x[0][k];
      x[0][k] = x[1][k];
      x[1][k] = x[2][k];
      x[2][k] = x[3][k];
      x[3][k] = x0;
    }
  }
}

// Two adjacent rows of a column; matrices need not be 16-byte aligned.
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// Rows row, row + 1 (row even) of a column with nrows rows, zero beyond them;
// nothing outside rows 0 .. nrows - 1 is read.
__device__ __forceinline__ void load_pair(const double* col, int row, int nrows, bool in,
                                          double& v0, double& v1) {
  if (nrows >= 2) {
    const d2u v = *(const d2u*)(col + min(row, nrows - 2));
    v0 = in ? (row + 1 < nrows ? v[0] : (row < nrows ? v[1] : 0.0)) : 0.0;
    v1 = (in && row + 1 < nrows) ? v[1] : 0.0;
  } else {
    const double v = col[0];
    v0 = (in && row == 0) ? v : 0.0;
    v1 = 0.0;
  }
}
__device__ __forceinline__ void store_pair(double* col, int row, int nrows, double v0, double v1) {
  if (row + 1 < nrows) {
    d2u v;
    v[0] = v0;
    v[1] = v1;
    *(d2u*)(col + row) = v;
  } else if (row < nrows) {
    col[row] = v0;
  }
}

// An nbr x nbr upper triangle from the tiles in LDS to a slot (column-major,
// leading dim kNB), zero elsewhere.  Eight LDS reads at a time (an entry below
// the diagonal reads the diagonal tile): one after the other with their stores the
// two triangles of a node took 6.5 thousand of its 105 thousand cycles (1024 x
// 64 with Q 156.2 -> 153.8 us, 4096 x 4096 20.52 -> 20.33 ms).
__device__ __forceinline__ void store_triangle(const double (*S)[kTile], double* G, int nbr) {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));  // the masks below are not held across a chain's blocks
  const int r = t & (kNB - 1), c0 = t / kNB;
  constexpr int kCols = 256 / kNB;  // columns stored at a time
#pragma unroll
  for (int h = 0; h < kTS / 256; h += 8) {
    double v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = c0 + kCols * (h + e), ct = kCols * (h + e) / 16;
      v[e] = S[tri(min(r >> 4, ct), ct)][(r & 15) * kTLD + (c & 15)];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = c0 + kCols * (h + e);
      G[t + 256 * (h + e)] = (r <= c && c < nbr) ? v[e] : 0.0;
    }
    __builtin_amdgcn_sched_barrier(0);  // eight values in registers at a time
  }
}
// And back: tiles of the upper triangle of a slot (its entries outside the
// triangle and beyond nbr are replaced by zero).
__device__ __forceinline__ void load_triangle(double (*S)[kTile], const double* G, int nbr) {
  double g[kTS / 256];
#pragma unroll
  for (int e = 0; e < kTS / 256; ++e) g[e] = G[threadIdx.x + 256 * e];
#pragma unroll
  for (int e = 0; e < kTS / 256; ++e) {
    const int i = threadIdx.x + 256 * e, r = i % kNB, c = i / kNB;
    if ((r >> 4) <= (c >> 4))
      S[tri(r >> 4, c >> 4)][(r & 15) * kTLD + (c & 15)] = (r <= c && c < nbr) ? g[e] : 0.0;
  }
}

// Leaf chains: the blocks of a chain in sequence, the first by itself, every
// later one stacked under the running R, which stays in LDS.  RT row tiles per
// wave: blocks of up to 64 RT rows.
template <int RT>
__global__ __launch_bounds__(256, 2) void k_tsqr_leaf(ChainQRArgs a) {
  __shared__ NodeLds S;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b0 = blockIdx.x * a.chain_len;
  const int b1 = min(b0 + a.chain_len, a.nblocks);
  const int nbr = a.nbr;
  d4 x[4][RT];
  for (int i = threadIdx.x; i < 10 * kTile; i += 256) (&S.r[0][0])[i] = 0.0;
  for (int b = b0; b < b1; ++b) {
    const bool first = b == b0;
    const int l = lane_id(), g = l >> 4, cl = l & 15;
    const int64_t rstart = ((int64_t)b * a.xrows) / a.nblocks;
    const int rows = (int)((((int64_t)b + 1) * a.xrows) / a.nblocks - rstart);
    double* src = a.X + rstart;
    // First row of this wave's row tile k: a first block keeps its top 64
    // rows (where the pivots are) one tile per wave.
    auto row0 = [&](int k) {
      return first ? (k == 0 ? 16 * w : 64 + 16 * (w * (RT - 1) + k - 1)) : 16 * (w * RT + k);
    };
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int col = 16 * c + cl;
      const double* cp = src + (int64_t)min(col, nbr - 1) * a.ldx;
#pragma unroll
      for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          double v0, v1;
          load_pair(cp, row0(k) + 8 * h + 2 * g, rows, col < nbr, v0, v1);
          x[c][k][2 * h] = v0;
          x[c][k][2 * h + 1] = v1;
        }
    }
    lds_barrier();  // R of the last block (or its zeros) is in LDS
    node_qr<RT, false>(first, x, nbr, w, S);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int col = 16 * c + cl;
      double* cp = src + (int64_t)col * a.ldx;
      if (col < nbr) {
#pragma unroll
        for (int k = 0; k < RT; ++k)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            store_pair(cp, row0(k) + 8 * h + 2 * g, rows, x[c][k][2 * h], x[c][k][2 * h + 1]);
      }
    }
    lds_barrier();  // T is complete
    double* Tb = a.T + (int64_t)b * kTS;
    if (!first) {
      store_triangle(S.t, Tb, nbr);
    } else {
      // Z = T V_top^T (upper triangular) in place of T.  Wave c forms block
      // column c, Z_pc = sum_q T_pq V_cq^T; V_cq is its own row tile 0.
      d4 z[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) z[p] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q <= w) {
          double* vt = S.red[w][0];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            vt[(8 * (r >> 1) + 2 * g + (r & 1)) * kTLD + cl] = x[q][0][r];
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double bv = vt[cl * kTLD + g + 4 * r];
#pragma unroll
            for (int p = 0; p <= q; ++p)
              z[p] = mfma64(S.t[tri(p, q)][cl * kTLD + g + 4 * r], bv, z[p]);
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * p + g + 4 * r, col = 16 * w + cl;
          Tb[row + col * kNB] = (row <= col && col < nbr) ? z[p][r] : 0.0;
        }
    }
  }
  lds_barrier();
  store_triangle(S.r, a.R + (int64_t)blockIdx.x * kTS, nbr);
}

// Tree nodes: the R factors of children 1 .. k - 1 stacked under child 0's.
// TRI: one child per wave (k <= 5), its triangle kept in place; else the
// children's rows packed one after the other (narrow panels with wide nodes).
template <bool TRI>
__global__ __launch_bounds__(256, 2) void k_tsqr_tree(ChainQRArgs a) {
  __shared__ NodeLds S;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = lane_id(), g = l >> 4, cl = l & 15;
  const int node = blockIdx.x;
  const int b0 = node * a.chain_len;
  const int k1 = min(a.chain_len, a.nblocks - b0) - 1;  // stacked children
  const int nbr = a.nbr;
  double* Tn = a.T + (int64_t)node * kTS;
  double* Rn = a.R + (int64_t)node * kTS;
  if (k1 == 0) {
    const double* R0 = a.X + (int64_t)b0 * kTS;
    for (int i = threadIdx.x; i < kTS; i += 256) {
      Tn[i] = 0.0;
      Rn[i] = R0[i];
    }
    return;
  }
  d4 x[4][4];
  const int rows = k1 * nbr;
  const double* child = a.X + (int64_t)(b0 + 1 + min(w, k1 - 1)) * kTS;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int col = 16 * c + cl;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (TRI) {
        if (k > c) {
          x[c][k] = d4{0.0, 0.0, 0.0, 0.0};
          continue;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int row = 16 * k + 8 * h + 2 * g;
          const d2u v = *(const d2u*)(child + row + col * kNB);
          const bool in = w < k1 && col < nbr;
          x[c][k][2 * h] = (in && row <= col) ? v[0] : 0.0;
          x[c][k][2 * h + 1] = (in && row + 1 <= col) ? v[1] : 0.0;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * (4 * w + k) + 8 * (r >> 1) + 2 * g + (r & 1);
          const int ch = min(row / nbr, k1 - 1), rr = min(row - ch * nbr, nbr - 1);
          const double v = a.X[(int64_t)(b0 + 1 + ch) * kTS + rr + min(col, nbr - 1) * kNB];
          x[c][k][r] = (row < rows && col < nbr) ? v : 0.0;
        }
      }
    }
  }
  load_triangle(S.r, a.X + (int64_t)b0 * kTS, nbr);
  lds_barrier();
  node_qr<4, TRI>(false, x, nbr, w, S);
  double* Yn = a.Y + (int64_t)node * kYS;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int col = 16 * c + cl;
    if (col >= nbr) continue;
#pragma unroll
    for (int k = 0; k < (TRI ? c + 1 : 4); ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int row = 16 * (TRI ? k : 4 * w + k) + 8 * h + 2 * g;
        if (TRI) {
          if (w < k1) store_pair(Yn + w * nbr + col * kYL, row, nbr, x[c][k][2 * h], x[c][k][2 * h + 1]);
        } else {
          store_pair(Yn + col * kYL, row, rows, x[c][k][2 * h], x[c][k][2 * h + 1]);
        }
      }
  }
  lds_barrier();
  store_triangle(S.t, Tn, nbr);
  store_triangle(S.r, Rn, nbr);
}

struct HRArgs {
  int L;  // number of tree levels above the leaves
  const double* T[kMaxLevels];
  int nblocks[kMaxLevels];
  int chain_len[kMaxLevels];
  const double* Rtop;    // R of the top node
  const double* A0;      // leaf block 0 (its basis, in place), leading dim lda
  int64_t lda;
  int nbr, nq, normalize;
  double* Tp;            // nbr x nbr kernel, leading dim ldt
  int64_t ldt;
  double* LR;            // kTS: strict lower L, upper R
  double* Broot;         // kBS: downsweep input of the top node
  double* sign;          // optional, nbr doubles
};

// Householder reconstruction (App. C.2) at the root, one workgroup of four
// waves.  It is a chain of small dependent steps (64 pivots and the products
// on the way to X), so it is built to need few barriers and to keep every
// operand in registers or one LDS read away: wave c holds column tile c of
// whatever is being formed, in MFMA accumulator layout, where an accumulator
// is the B operand of the next product as it stands.
//   1. X, the top rows of W: B <- B - T B along the path to leaf block 0 (B and
//      every T upper triangular: 20 tile products, shared evenly), then X =
//      [B; 0] - V (Z B), column tile by column tile.
//   2. Sign-modified LU of X, right-looking by 16 columns.  The wave that owns
//      the column tile eliminates its diagonal tile and the tiles below it
//      together, column by column in registers (the pivot's multipliers are
//      broadcast inside the FMAs), and L_bb^-1 alongside; the others then take
//      U_bj = L_bb^-1 X_bj and X_ij -= L_ib U_bj.  One barrier per 16 columns.
//   3. T = U S L^-T and U^-1 by tiles, by substitution; R = -S R_root.
// At most 256 registers, accumulation registers included: what one workgroup of
// the look-ahead's GEMM leaves when it ends.  With 340 the kernel waited for the
// end of whole update launches (up to 2.8 ms; 355 us on average beside the
// depth-512 updates of 65536 x 8192).
//   Measured (MI355X, 64 columns; before: one barrier per pivot, 127 in all,
// with the rows in registers of four threads each): 84 -> 27 us under 1024 rows,
// 126 -> 50 us under 1048576 (eleven path steps).  About half of it is the 64
// pivots (430 cycles each: readlane, reciprocal, up to 42 broadcast FMAs).
struct HrLds {
  double l[10][kTile];    // L, tile (i, b) at tri(b, i); strict lower and, below it, full tiles
  double u[10][kTile];    // U, tile (b, j) at tri(b, j)
  double li[4][kTile];    // L_bb^-1
  double ui[4][kTile];    // U_bb^-1
  double sv[kNB];         // S
  double dv[kNB];         // D
};

// D += A B for an A tile in LDS (row-major) and a B tile in registers.
__device__ __forceinline__ d4 hr_mul_tile(const double* A, const d4 B, int g, int cl, d4 D) {
#pragma unroll
  for (int r = 0; r < 4; ++r) D = mfma64(A[cl * kTLD + g + 4 * r], B[r], D);
  return D;
}
__device__ __forceinline__ void hr_put_tile(double* S, const d4 v, int g, int cl) {
#pragma unroll
  for (int r = 0; r < 4; ++r) S[(g + 4 * r) * kTLD + cl] = v[r];
}

// A product of two 64 x 64 upper triangles takes 20 products of 16 x 16 tiles;
// wave w forms the output tiles whose five are its share: (p, c) needs tiles
// (p, q) and (q, c) for q = p .. c.
struct TriShare {
  int p[5], q[5], c[5];
  bool last[5];  // the output tile is complete after this product
  __device__ explicit TriShare(int w) {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      int pp, qq, cc;
      if (w == 0) { pp = 0; qq = i < 4 ? i : 0; cc = i < 4 ? 3 : 0; }
      else if (w == 1) { pp = 0; qq = i < 3 ? i : i - 3; cc = i < 3 ? 2 : 1; }
      else if (w == 2) { pp = 1; qq = i < 3 ? 1 + i : i - 2; cc = i < 3 ? 3 : 2; }
      else { pp = i < 2 ? 2 : i - 1; qq = i < 2 ? 2 + i : i - 1; cc = i < 2 ? 3 : i - 1; }
      p[i] = pp;
      q[i] = qq;
      c[i] = cc;
      last[i] = qq == cc;
    }
  }
};

// Its five A operands from an upper triangle in a slot.
__device__ __forceinline__ void tri_load(const TriShare& sh, const double* T, int g, int cl,
                                         double (&m)[5][4]) {
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      m[i][r] = (T + 16 * sh.p[i] + 16 * sh.q[i] * kNB)[cl + (g + 4 * r) * kNB];
}
// O = A B, -A B or B - A B for the wave's output tiles: A in m, B's and O's
// tiles in LDS.
enum TriOut { TRI_POS, TRI_NEG, TRI_SUB };
template <TriOut OUT>
__device__ __forceinline__ void tri_mul(const TriShare& sh, const double (&m)[5][4],
                                        const double (*Bs)[kTile], double (*O)[kTile], int g,
                                        int cl) {
  d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const double* bs = Bs[tri(sh.q[i], sh.c[i])];
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = mfma64(m[i][r], bs[(g + 4 * r) * kTLD + cl], acc);
    if (sh.last[i]) {
      if constexpr (OUT == TRI_SUB) {
        const double* bt = Bs[tri(sh.p[i], sh.c[i])];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = bt[(g + 4 * r) * kTLD + cl] - acc[r];
      }
      hr_put_tile(O[tri(sh.p[i], sh.c[i])], OUT == TRI_NEG ? -acc : acc, g, cl);
      acc = d4{0.0, 0.0, 0.0, 0.0};
    }
  }
}
// B += M, the wave's tiles.
__device__ __forceinline__ void tri_add(const TriShare& sh, double (*B)[kTile],
                                        const double (*M)[kTile], int g, int cl) {
#pragma unroll
  for (int i = 0; i < 5; ++i)
    if (sh.last[i]) {
      double* bt = B[tri(sh.p[i], sh.c[i])];
      const double* mt = M[tri(sh.p[i], sh.c[i])];
#pragma unroll
      for (int r = 0; r < 4; ++r) bt[(g + 4 * r) * kTLD + cl] += mt[(g + 4 * r) * kTLD + cl];
    }
}

// Step J of the elimination of a 16-column tile whose diagonal tile sits in
// xc column by column: every lane holds all sixteen rows of column cl (the
// four lane groups alike), so row J is register J of each lane and needs no
// broadcast, and the multipliers are lane J's registers, broadcast inside the
// FMAs.  S_J = sgn(pivot) (+1 for >= 0) is added to the pivot; every lower row
// (xc below J; the rows of the tiles below in xb, when there are any) loses
// its multiple of row J; e
// carries the same operations on the identity (L_bb^-1).  The pivot's column
// keeps its unscaled entries; zs[J] = 1 / U_JJ scales them at the end.
template <int J>
__device__ __forceinline__ void hr_step(bool more, int cl, double (&xc)[16], double (&e)[16],
                                        double (&zs)[16], double (&xb)[12], double& sgn) {
  if constexpr (J < 16) {
    const double up = readlane(xc[J], J);
    const double s = up >= 0.0 ? 1.0 : -1.0, piv = up + s;
    // 1 / piv (|piv| >= 1): the hardware reciprocal and one third-order step.
    const double z0 = __builtin_amdgcn_rcp(piv);
    const double ez = fma(-piv, z0, 1.0);
    const double z = fma(z0, fma(ez, ez, ez), z0);
    const double f = cl > J ? -(xc[J] * z) : 0.0, fe = -(e[J] * z);
    bcast_fmacs<J, J + 1, 16>(xc, e, fe);
    bcast_fmacs_self<J, J + 1, 16>(xc, f);
    if (more) bcast_fmacs_self<J, 0, 12>(xb, f);
    xc[J] = cl == J ? piv : xc[J];
    sgn = cl == J ? s : sgn;
    zs[J] = z;
    hr_step<J + 1>(more, cl, xc, e, zs, xb, sgn);
  }
}

// U_bb^-1 by columns: lane cl solves U t = e_cl alone, rows 15 .. 0, U's
// entries broadcast from the lanes of their columns (u zero below the
// diagonal).
template <int J>
__device__ __forceinline__ void hr_uinv(const double (&u)[16], const double (&zs)[16],
                                        double (&t)[16]) {
  if constexpr (J >= 0) {
    t[J] *= zs[J];
    bcast_fmacs<J, 0, J>(u, t, -t[J]);
    hr_uinv<J - 1>(u, zs, t);
  }
}

__global__ __launch_bounds__(256, 2) void k_tsqr_hr(HRArgs a) {
  __shared__ HrLds S;
  const int t = threadIdx.x, c = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l = t & 63, g = l >> 4, cl = l & 15;
  const int nbr = a.nbr, nsub = (nbr + 15) >> 4;
  // The path: the T of every node from the root to leaf block 0, of the
  // stacked steps of leaf chain 0 (last to first), then Z of leaf block 0.
  const int b1c = min(a.chain_len[0], a.nblocks[0]);
  int nlev = 0;
  for (int lev = a.L; lev >= 1; --lev) nlev += (min(a.chain_len[lev], a.nblocks[lev]) >= 2);
  const int np = nlev + b1c;
  auto path = [&](int k) -> const double* {
    if (k < nlev) {
      int seen = 0;
      for (int lev = a.L; lev >= 1; --lev)
        if (min(a.chain_len[lev], a.nblocks[lev]) >= 2 && seen++ == k) return a.T[lev];
    }
    return a.T[0] + (int64_t)(k < np - 1 ? b1c - 1 - (k - nlev) : 0) * kTS;
  };
  d4 x[4];
  {
    // B in turn in the tiles that L and U take later.
    const TriShare sh(c);
    double ta[5][4];
    tri_load(sh, path(0), g, cl, ta);
#pragma unroll
    for (int p = 0; p < 4; ++p)
      if (p <= c) {  // B = I, column tile c
        d4 v = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (p == c && g + 4 * r == cl && 16 * c + cl < nbr) ? 1.0 : 0.0;
        hr_put_tile(S.l[tri(p, c)], v, g, cl);
      }
    // V_top of leaf block 0 (unit lower), tiles (p, q), q <= min(p, c).
    double v[10][4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = 0; q <= p; ++q)
        if (q <= c) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = 16 * p + cl, col = 16 * q + g + 4 * r;
            const double av = a.A0[min(row, nbr - 1) + (int64_t)min(col, nbr - 1) * a.lda];
            v[p * (p + 1) / 2 + q][r] =
                (row < nbr && col < nbr) ? (row > col ? av : (row == col ? 1.0 : 0.0)) : 0.0;
          }
        }
    double (*Bt)[kTile] = S.l, (*Mt)[kTile] = S.u;  // B, and the other buffer
    lds_barrier();
    for (int k = 0; k + 1 < np; ++k) {
      tri_mul<TRI_SUB>(sh, ta, Bt, Mt, g, cl);  // B - T B
      tri_load(sh, path(k + 1), g, cl, ta);
      lds_barrier();
      double (*const x)[kTile] = Bt;
      Bt = Mt;
      Mt = x;
    }
    tri_mul<TRI_NEG>(sh, ta, Bt, Mt, g, cl);  // -Z B
    lds_barrier();
    // Column tile c of X = [B; 0] - V (Z B).
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      x[p] = d4{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q <= c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double m = Mt[tri(q, c)][(g + 4 * r) * kTLD + cl];
#pragma unroll
          for (int p = q; p < 4; ++p) x[p] = mfma64(v[p * (p + 1) / 2 + q][r], m, x[p]);
        }
      }
#pragma unroll
    for (int p = 0; p < 4; ++p)
      if (p <= c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) x[p][r] += Bt[tri(p, c)][(g + 4 * r) * kTLD + cl];
      }
    lds_barrier();
  }
  // Sign-modified LU.  Slot k of x is row tile b + k (rotated every step).
  for (int b = 0; b < nsub; ++b) {
    const int nt = nsub - b;
    double xc[16], zs[16];
    if (c == b) {
      // The diagonal tile column by column (through its LDS tile), e = I.
      double e[16];
      double* lt = S.l[tri(b, b)];
      hr_put_tile(lt, x[0], g, cl);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        xc[i] = lt[i * kTLD + cl];
        e[i] = i == cl ? 1.0 : 0.0;
      }
      __builtin_amdgcn_wave_barrier();
      double sgn = 1.0, xb[12];
#pragma unroll
      for (int i = 0; i < 12; ++i) xb[i] = x[1 + i / 4][i % 4];
      hr_step<0>(nt > 1, cl, xc, e, zs, xb, sgn);
      double z = 1.0;  // this column's 1 / U_jj
#pragma unroll
      for (int i = 0; i < 16; ++i) z = i == cl ? zs[i] : z;
      if (g == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          S.li[b][i * kTLD + cl] = e[i];
          lt[i * kTLD + cl] = xc[i] * z;  // L below the diagonal
        }
        S.sv[16 * b + cl] = sgn;
      }
#pragma unroll
      for (int k = 1; k < 4; ++k)
        if (k < nt) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            S.l[tri(b, b + k)][(g + 4 * r) * kTLD + cl] = xb[4 * (k - 1) + r] * z;
        }
    }
    lds_barrier();
    if (c == b) {
      double m[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        m[i] = i == cl ? 1.0 : 0.0;
        xc[i] = i <= cl ? xc[i] : 0.0;
      }
      hr_uinv<15>(xc, zs, m);
      if (g == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          S.u[tri(b, b)][i * kTLD + cl] = xc[i];
          S.ui[b][i * kTLD + cl] = m[i];
        }
      }
    } else if (c > b && c < nsub) {
      const d4 u = hr_mul_tile(S.li[b], x[0], g, cl, d4{0.0, 0.0, 0.0, 0.0});
      hr_put_tile(S.u[tri(b, c)], u, g, cl);
#pragma unroll
      for (int k = 1; k < 4; ++k)
        if (k < nt) x[k] = hr_mul_tile(S.l[tri(b, b + k)], -u, g, cl, x[k]);
      x[0] = x[1];
      x[1] = x[2];
      x[2] = x[3];
    }
  }
  // R = -S R_root, optional D = sign(diag R).
  if (t < nbr) {
    const double r = -S.sv[t] * a.Rtop[t + t * kNB];
    const double d = (a.normalize && r < 0.0) ? -1.0 : 1.0;
    S.dv[t] = d;
    if (a.sign) a.sign[t] = d;
  }
  lds_barrier();
  double rtop[kTS / 256];  // the root's R, for the last step
#pragma unroll
  for (int i = 0; i < kTS / 256; ++i) rtop[i] = a.Rtop[t + 256 * i];
  if (c < nsub) {
    // Row tile c of T = U S L^-T, as column tile c of T^T, by substitution:
    //   (T^T)_kc = L_kk^-1 (S_k U_ck^T - sum_{c <= q < k} L_kq (T^T)_qc),  k = c ..
    // and column tile c of U^-1, into the downsweep's input:
    //   (U^-1)_ic = -U_ii^-1 sum_{i < q <= c} U_iq (U^-1)_qc,  i = c - 1 .. 0
    d4 y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c + k;
      if (i < nsub) {
        d4 acc;
        const double* ut = S.u[tri(c, i)];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = -S.sv[16 * i + g + 4 * r] * ut[cl * kTLD + g + 4 * r];
#pragma unroll
        for (int q = 0; q < k; ++q) acc = hr_mul_tile(S.l[tri(c + q, i)], y[q], g, cl, acc);
        y[k] = hr_mul_tile(S.li[i], -acc, g, cl, d4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * c + cl, cc = 16 * i + g + 4 * r;
          if (row < nbr && cc < nbr) a.Tp[row + cc * a.ldt] = (row <= cc) ? y[k][r] : 0.0;
        }
      }
    }
    for (int i = 0; i < c; ++i)  // tiles below T's diagonal
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * c + cl, cc = 16 * i + g + 4 * r;
        if (row < nbr && cc < nbr) a.Tp[row + cc * a.ldt] = 0.0;
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) y[0][r] = S.ui[c][(g + 4 * r) * kTLD + cl];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c - k;
      if (i >= 0) {
        if (k > 0) {
          d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int q = 0; q < k; ++q) acc = hr_mul_tile(S.u[tri(i, c - q)], y[q], g, cl, acc);
          y[k] = hr_mul_tile(S.ui[i], -acc, g, cl, d4{0.0, 0.0, 0.0, 0.0});
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + g + 4 * r, cc = 16 * c + cl;
          if (cc < nbr) a.Broot[row + cc * kNB] = (row <= cc) ? y[k][r] : 0.0;
        }
      }
    }
  }
  // The final L (strict lower) and R of the top rows.  Branch-free, so that the
  // LDS reads overlap.
  const double ds = -S.dv[t & 63] * S.sv[t & 63];
#pragma unroll
  for (int i = 0; i < kTS / 256; ++i) {
    const int r = t & 63, cc = (t >> 6) + 4 * i;
    const int tl = (r & 15) * kTLD + (cc & 15), rt = r >> 4, ct = cc >> 4;
    const double lv = S.l[tri(min(rt, ct), max(rt, ct))][tl];
    a.LR[t + 256 * i] = (r < nbr && cc < nbr) ? (r <= cc ? ds * rtop[i] : lv) : 0.0;
  }
  // With Q the downsweep also starts from -S D, columns nbr .. 2 nbr - 1 of
  // its input (it reads nothing below the diagonal, and no U^-1 beyond nbr).
  if (a.nq > nbr)
    for (int e = t; e < kNB * nbr; e += 256) {
      const int r = e % kNB, cc = e / kNB;
      a.Broot[r + (nbr + cc) * kNB] = (r == cc && r < nbr) ? ds : 0.0;
    }
}

struct DownArgs {
  int L;                 // tree levels above the leaves
  const double* T[kMaxLevels];   // [0]: per leaf block; [lev]: per node
  const double* Y[kMaxLevels];   // [lev]: per node
  int nblocks[kMaxLevels];
  int chain_len[kMaxLevels];
  const double* Broot;   // [U^-1 | -S D] of the root
  const double* LR;
  double* A;             // panel (basis in, V out)
  int64_t lda, xrows;
  double* Q;             // optional
  int64_t ldq;
  int nbr;
};

// Row `row` (per lane) of the basis as operands of a contraction over its
// columns: y[q][r] = Y[row][16 q + g + 4 r], zero beyond nbr (nothing outside
// the panel's columns is read).
__device__ __forceinline__ void down_load_row(const double* A, int64_t lda, int row, int nbr,
                                              int qn, int g, double (&y)[4][4]) {
  const double* Al = A + row + g * lda;
  if (nbr == kNB) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < qn) {
#pragma unroll
        for (int r = 0; r < 4; ++r) y[q][r] = Al[(16 * q + 4 * r) * lda];
      }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < qn) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool in = 16 * q + 4 * r + g < nbr;
          y[q][r] = 0.0;
          if (in) y[q][r] = Al[(16 * q + 4 * r) * lda];
        }
      }
  }
}

// Downsweep (App. C.2), tree and leaves in one launch: the workgroup of a leaf
// chain walks from the root to its chain by itself (M = T B, then B - M for a
// first child, -Y M for the others), then through its chain's blocks, last to
// first, writing -Y M (+ B on a first block's top rows).  B, T and the
// children's Y are upper triangular all the way down, so a level is two
// triangular products of 20 tile products, shared evenly by the four waves,
// with B and -M in LDS and the next matrix loaded meanwhile.
//   Without Q the walk starts from U^-1 and emits V = W U^-1.  With Q it starts
// from -S D, emits Q = -W S D, and V is Q (-S D U^-1), from Q's rows while they
// are in registers: one walk serves both.
//   Bound: under few rows the latency of the path (about 4.4 k cycles a level);
// under many the memory traffic of the panel (read the basis, write V and Q:
// 1.6 GB at 1048576 x 64 with Q, 514 us).  Measured (MI355X; before: a launch
// per tree level and one for the leaves): 1024 x 64 with Q 79 -> 23 us,
// 16384 x 64 118 -> 18 us, 1048576 x 64 with Q 936 -> 514 us.
template <bool WQ>
__global__ __launch_bounds__(256, 2) void k_tsqr_down(DownArgs a) {
  __shared__ double Bt[10][kTile];             // B
  __shared__ double Mt[10][kTile];             // -M
  __shared__ double Kt[WQ ? 10 : 1][kTile];    // -S D U^-1
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, g = l >> 4, cl = l & 15;
  const int chain = blockIdx.x, nbr = a.nbr, nsub = (nbr + 15) >> 4;
  const int part = blockIdx.y, parts = gridDim.y;
  const int b0 = chain * a.chain_len[0];
  const int b1 = min(b0 + a.chain_len[0], a.nblocks[0]);
  const TriShare sh(w);
  double ta[5][4], ya[5][4];
  // A child's basis (leading dim kYL).  Narrow panels read past the child's
  // rows and columns (inside the workspace: the level's R follows its Y) and
  // mask what they read.
  auto load_y = [&](const double* Y) {
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double v = (Y + 16 * sh.p[i] + 16 * sh.q[i] * kYL)[cl + (g + 4 * r) * kYL];
        ya[i][r] = (16 * sh.p[i] + cl < nbr && 16 * sh.q[i] + g + 4 * r < nbr) ? v : 0.0;
      }
  };
  // The path's nodes, lane k's at level k (integer divisions are slow: once,
  // side by side).
  int path = chain;
  for (int k = 1; k <= a.L; ++k) path = k <= l ? path / a.chain_len[k] : path;
  // Node of the path at a level, and which of its children the path takes.
  auto node_at = [&](int lev, int* pos) {
    const int node = __builtin_amdgcn_readlane(path, lev);
    *pos = __builtin_amdgcn_readlane(path, lev - 1) - node * a.chain_len[lev];
    return node;
  };
  auto load_level_t = [&](int lev) {  // level 0: the last block of the chain
    const int node = lev == 0 ? b1 - 1 : __builtin_amdgcn_readlane(path, lev);
    tri_load(sh, a.T[lev] + (int64_t)node * kTS, g, cl, ta);
  };
  auto load_level_y = [&](int lev) {
    int pos;
    const int node = node_at(lev, &pos);
    if (pos > 0) load_y(a.Y[lev] + (int64_t)node * kYS + (pos - 1) * nbr);
  };
  load_level_t(a.L);
  if (a.L > 0) load_level_y(a.L);
  // Start: U^-1, or -S D and K = -S D U^-1.
#pragma unroll
  for (int i = 0; i < kTS / 256; ++i) {
    const int r = threadIdx.x & 63, cc = (threadIdx.x >> 6) + 4 * i;
    double v = a.Broot[threadIdx.x + 256 * i];
    v = (r <= cc && cc < nbr) ? v : 0.0;
    const int e = (r & 15) * kTLD + (cc & 15), ti = tri(min(r, cc) >> 4, cc >> 4);
    if constexpr (WQ) {
      const double ds = a.Broot[r + (nbr + min(r, nbr - 1)) * kNB];
      if ((r >> 4) <= (cc >> 4)) {
        Kt[ti][e] = r < nbr ? ds * v : 0.0;
        Bt[ti][e] = (r == cc && r < nbr) ? ds : 0.0;
      }
    } else {
      if ((r >> 4) <= (cc >> 4)) Bt[ti][e] = v;
    }
  }
  lds_barrier();
  for (int lev = a.L; lev >= 1; --lev) {
    int pos;
    const int node = node_at(lev, &pos);
    const bool single = min(a.chain_len[lev], a.nblocks[lev] - node * a.chain_len[lev]) < 2;
    if (!single) tri_mul<TRI_NEG>(sh, ta, Bt, Mt, g, cl);
    load_level_t(lev - 1);
    lds_barrier();
    if (!single) {
      if (pos == 0) tri_add(sh, Bt, Mt, g, cl);
      else tri_mul<TRI_POS>(sh, ya, Mt, Bt, g, cl);
    }
    if (lev > 1) load_level_y(lev - 1);
    lds_barrier();
  }
  for (int b = b1 - 1; b >= b0; --b) {
    const bool first = b == b0;
    const int64_t rstart = ((int64_t)b * a.xrows) / a.nblocks[0];
    const int rows = (int)((((int64_t)b + 1) * a.xrows) / a.nblocks[0] - rstart);
    double* Ab = a.A + rstart;
    // Rows r0 .. r0 + 15 of the block are this wave's next; their basis is
    // loaded one step ahead.
    const int rstep = 64 * parts;
    int r0 = 16 * (w + 4 * part);
    double y[4][4];
    down_load_row(Ab, a.lda, min(r0 + cl, rows - 1), nbr, nsub, g, y);
    tri_mul<TRI_NEG>(sh, ta, Bt, Mt, g, cl);
    if (!first) tri_load(sh, a.T[0] + (int64_t)(b - 1) * kTS, g, cl, ta);
    lds_barrier();
    if (!first) tri_add(sh, Bt, Mt, g, cl);
    for (; r0 < rows; r0 += rstep) {
      const int row = min(r0 + cl, rows - 1);
      const bool in = r0 + cl < rows, top = first && r0 < 64;
      double yn[4][4];
      if (r0 + rstep < rows)
        down_load_row(Ab, a.lda, min(r0 + rstep + cl, rows - 1), nbr, nsub, g, yn);
      // D[col][row] = sum_k (-M)[k][col] Y[row][k] (+ B[row][col]).
      d4 acc[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        acc[c] = d4{0.0, 0.0, 0.0, 0.0};
        if (c >= nsub) continue;
#pragma unroll
        for (int q = 0; q <= c; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[c] = mfma64(Mt[tri(q, c)][(g + 4 * r) * kTLD + cl], y[q][r], acc[c]);
        if (top && r0 <= 16 * c) {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[c][r] += Bt[tri(r0 >> 4, c)][cl * kTLD + g + 4 * r];
        }
        if constexpr (WQ) {
          double* out = a.Q + rstart + row + (16 * c + g) * a.ldq;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (in && 16 * c + 4 * r + g < nbr) out[4 * r * a.ldq] = acc[c][r];
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c >= nsub) continue;
        d4 v = acc[c];
        if constexpr (WQ) {
          v = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int q = 0; q <= c; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              v = mfma64(Kt[tri(q, c)][(g + 4 * r) * kTLD + cl], acc[q][r], v);
        }
        double* out = Ab + row + (16 * c + g) * a.lda;
        const bool lr = b == 0 && r0 + cl < nbr;  // L and R instead
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (in && 16 * c + 4 * r + g < nbr)
            out[4 * r * a.lda] = lr ? a.LR[row + (16 * c + 4 * r + g) * kNB] : v[r];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[q][r] = yn[q][r];
    }
    lds_barrier();
  }
}

// ---------------------------------------------------------------- host side

TsqrPlan tsqr_plan(int64_t rows, int nbr, int leaf_rows, int chain, int arity, double* ws) {
  TsqrPlan p;
  p.rows = rows;
  p.nbr = nbr;
  const TsqrGeom g = tsqr_geometry(rows, nbr, leaf_rows, chain, arity);
  p.leaf_rows = g.leaf_rows;
  int64_t off = 0;
  auto take = [&](int64_t n) {
    double* ptr = ws ? ws + off : nullptr;
    off += (n + 31) & ~int64_t(31);
    return ptr;
  };
  TsqrLevel l0;
  l0.nblocks = (int)g.blocks;
  l0.chain_len = g.chain;
  l0.nchains = (int)g.chains;
  p.levels.push_back(l0);
  for (int l = 0; l < g.levels; ++l) {
    TsqrLevel lv;
    lv.nblocks = p.levels.back().nchains;
    lv.chain_len = g.arity;
    lv.nchains = (lv.nblocks + g.arity - 1) / g.arity;
    p.levels.push_back(lv);
  }
  for (size_t i = 0; i < p.levels.size(); ++i) {
    TsqrLevel& lv = p.levels[i];
    if (i == 0) {
      lv.T = take((int64_t)lv.nblocks * kTS);
    } else {
      lv.T = take((int64_t)lv.nchains * kTS);
      lv.Y = take((int64_t)lv.nchains * kYS);
    }
    lv.R = take((int64_t)lv.nchains * kTS);
    // Only the top level's B is used (64 KB a chain); the others keep their
    // place, which the shapes that qr_factor_noalloc accepts follow from.
    lv.B = take((int64_t)lv.nchains * kBS);
  }
  p.LR = take(kTS);
  p.workspace_doubles = off;
  return p;
}

hipError_t tsqr_factor(const TsqrPlan& p, hipStream_t s, double* P, int64_t ldp, double* Tp,
                       int64_t ldt, double* Q, int64_t ldq, int normalize, double* sign) {
  const int nbr = p.nbr;
  const int L = (int)p.levels.size() - 1;
  const double tri = 8.0 * nbr * (nbr + 1) / 2.0;  // bytes of one packed triangle
  const double pan = 8.0 * (double)p.rows * nbr;     // bytes of the panel
  // Upsweep.
  {
    const TsqrLevel& l0 = p.levels[0];
    ChainQRArgs a{P, ldp, p.rows, l0.nblocks, l0.chain_len, nbr, nullptr, l0.T, l0.R};
    // Read A, write V; write T per block and R per chain.  Flops: QR 2 m nb^2
    // plus the Gram products for T, m nb^2.
    TimedLaunch tl(s, "tsqr_chain_qr_leaf", 2.0 * pan + tri * (l0.nblocks + l0.nchains),
                   3.0 * (double)p.rows * nbr * nbr);
    if (p.leaf_rows == 256)
      hipLaunchKernelGGL((k_tsqr_leaf<4>), dim3(l0.nchains), dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((k_tsqr_leaf<2>), dim3(l0.nchains), dim3(256), 0, s, a);
  }
  for (int lev = 1; lev <= L; ++lev) {
    const TsqrLevel& lv = p.levels[lev];
    ChainQRArgs a{p.levels[lev - 1].R, kNB, 0, lv.nblocks, lv.chain_len, nbr, lv.Y, lv.T, lv.R};
    TimedLaunch tl(s, "tsqr_chain_qr_tree", tri * (2.0 * lv.nblocks + 3.0 * lv.nchains),
                   3.0 * (double)lv.nblocks * nbr * nbr * nbr);
    // One child per wave where a node has at most four stacked children;
    // wider nodes (narrow panels with an arity of the caller's) pack them.
    if (lv.chain_len <= 5)
      hipLaunchKernelGGL((k_tsqr_tree<true>), dim3(lv.nchains), dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((k_tsqr_tree<false>), dim3(lv.nchains), dim3(256), 0, s, a);
  }
  // Householder reconstruction at the root.
  const int nq = Q ? 2 * nbr : nbr;
  {
    HRArgs h{};
    h.L = L;
    for (int lev = 0; lev <= L; ++lev) {
      h.T[lev] = p.levels[lev].T;
      h.nblocks[lev] = p.levels[lev].nblocks;
      h.chain_len[lev] = p.levels[lev].chain_len;
    }
    h.Rtop = p.levels[L].R;
    h.A0 = P;
    h.lda = ldp;
    h.nbr = nbr;
    h.nq = nq;
    h.normalize = normalize;
    h.Tp = Tp;
    h.ldt = ldt;
    h.LR = p.LR;
    h.Broot = p.levels[L].B;
    h.sign = sign;
    TimedLaunch tl(s, "tsqr_hr_root", tri * 8.0, 6.0 * (double)nbr * nbr * nbr * (L + 2));
    hipLaunchKernelGGL(k_tsqr_hr, dim3(1), dim3(256), 0, s, h);
  }
  // Downsweep, tree and leaves.  Read the basis, write V (and Q); T per block
  // and per node.  Flops: 2 m nb nq for -Y M, nb^2 nq per block for M = T B.
  {
    DownArgs d{};
    d.L = L;
    int64_t nodes = 0;
    for (int lev = 0; lev <= L; ++lev) {
      d.T[lev] = p.levels[lev].T;
      d.Y[lev] = p.levels[lev].Y;
      d.nblocks[lev] = p.levels[lev].nblocks;
      d.chain_len[lev] = p.levels[lev].chain_len;
      if (lev > 0) nodes += p.levels[lev].nchains;
    }
    d.Broot = p.levels[L].B;
    d.LR = p.LR;
    d.A = P;
    d.lda = ldp;
    d.xrows = p.rows;
    d.Q = Q;
    d.ldq = ldq;
    d.nbr = nbr;
    const TsqrLevel& l0 = p.levels[0];
    TimedLaunch tl(s, "tsqr_down_leaf", pan * (Q ? 3.0 : 2.0) + tri * (l0.nblocks + 2.0 * nodes),
                   2.0 * (double)p.rows * nbr * nq + (double)l0.nblocks * nbr * nbr * nq);
    // Few chains: the rows of each chain's blocks go to up to four workgroups
    // (every one walks the path), so that the emission of a block's up to four
    // row tiles per wave is spread over idle CUs.
    const int parts = l0.nchains >= 256 ? 1 : std::min(p.leaf_rows / 64, 256 / l0.nchains);
    const dim3 grid(l0.nchains, parts);
    if (Q) hipLaunchKernelGGL(k_tsqr_down<true>, grid, dim3(256), 0, s, d);
    else hipLaunchKernelGGL(k_tsqr_down<false>, grid, dim3(256), 0, s, d);
  }
  return hipGetLastError();
}

}  // namespace miqr
