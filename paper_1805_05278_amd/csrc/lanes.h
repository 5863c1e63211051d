// Cross-lane helpers of the kernels that hold a 16-column panel in the MFMA
// accumulator layout (lane (q, cl) = (l / 16, l % 16) owns entries of column
// cl): broadcasts of a pivot column, sums over the four lanes of a column.
#pragma once
#include "common.h"

namespace miqr {

__device__ __forceinline__ unsigned lo32(double v) {
  return (unsigned)(unsigned long long)__double_as_longlong(v);
}
__device__ __forceinline__ unsigned hi32(double v) {
  return (unsigned)((unsigned long long)__double_as_longlong(v) >> 32);
}
__device__ __forceinline__ double join(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the four lanes cl, cl + 16, cl + 32, cl + 48: rows paired by
// v_permlane16_swap, then halves by v_permlane32_swap; each swap leaves one
// copy holding the lower partner in both places and the other the upper, so
// every lane forms the same sums in the same order.
__device__ __forceinline__ double rows_sum(double v) {
  {
    const auto l = __builtin_amdgcn_permlane16_swap(lo32(v), lo32(v), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi32(v), hi32(v), false, false);
    v = join(l[0], h[0]) + join(l[1], h[1]);
  }
  {
    const auto l = __builtin_amdgcn_permlane32_swap(lo32(v), lo32(v), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi32(v), hi32(v), false, false);
    v = join(l[0], h[0]) + join(l[1], h[1]);
  }
  return v;
}

__device__ __forceinline__ double readlane(double v, int lane) {
  return join((unsigned)__builtin_amdgcn_readlane((int)lo32(v), lane),
              (unsigned)__builtin_amdgcn_readlane((int)hi32(v), lane));
}

// The pivot broadcast fused into the FMAs: v_fmac_{f64,f32}_dpp with
// row_newbcast:J reads its first source from lane J of the lane's row.  One
// s_nop 1 at the head of each block gives the two wait states a DPP read
// needs after a VALU write of its source (the compiler does not look inside
// the asm); within a block no instruction DPP-reads a register written by
// the one before it.  Outputs of a block are early clobbers: they are written
// before its last inputs are read, and the compiler would give an output and an
// input of equal value (a zero sum and a zero entry) one register.  xs[4 t + r] is register r of row tile t.
//   d0 += sum_t (x_J[t][0] x[t][0] + x_J[t][2] x[t][2]), d1 likewise for
//   registers 1 and 3 (two chains for latency).
template <int J>
__device__ __forceinline__ void dots_bcast(const double (&xs)[16], double& d0, double& d1) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %2 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %3, %3 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %4, %4 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %5, %5 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %6, %6 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %7, %7 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %8, %8 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %9, %9 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %10, %10 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %11, %11 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %12, %12 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %13, %13 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %14, %14 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %15, %15 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %16, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %17, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(d0), "+&v"(d1)
      : "v"(xs[0]), "v"(xs[1]), "v"(xs[2]), "v"(xs[3]), "v"(xs[4]), "v"(xs[5]), "v"(xs[6]), "v"(xs[7]), "v"(xs[8]), "v"(xs[9]), "v"(xs[10]), "v"(xs[11]), "v"(xs[12]), "v"(xs[13]), "v"(xs[14]), "v"(xs[15]), "n"(J));
}
template <int J>
__device__ __forceinline__ void dots_bcast(const float (&xs)[16], float& d0, float& d1) {
  asm("s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %2, %2 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %3, %3 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %4, %4 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %5, %5 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %6, %6 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %7, %7 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %8, %8 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %9, %9 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %10, %10 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %11, %11 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %12, %12 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %13, %13 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %14, %14 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %15, %15 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %16, %16 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %17, %17 row_newbcast:%18 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(d0), "+&v"(d1)
      : "v"(xs[0]), "v"(xs[1]), "v"(xs[2]), "v"(xs[3]), "v"(xs[4]), "v"(xs[5]), "v"(xs[6]), "v"(xs[7]), "v"(xs[8]), "v"(xs[9]), "v"(xs[10]), "v"(xs[11]), "v"(xs[12]), "v"(xs[13]), "v"(xs[14]), "v"(xs[15]), "n"(J));
}
//   x[t][r] += x_J[t][r] nf (lane J's own entries are unchanged when its nf
//   is zero).
template <int J>
__device__ __forceinline__ void update_bcast(double (&xs)[16], double nf) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %1, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %2, %2, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %3, %3, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %4, %4, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %5, %5, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %6, %6, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %7, %7, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %8, %8, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %9, %9, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %10, %10, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %11, %11, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %12, %12, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %13, %13, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %14, %14, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %15, %15, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(xs[0]), "+&v"(xs[1]), "+&v"(xs[2]), "+&v"(xs[3]), "+&v"(xs[4]), "+&v"(xs[5]), "+&v"(xs[6]), "+&v"(xs[7]), "+&v"(xs[8]), "+&v"(xs[9]), "+&v"(xs[10]), "+&v"(xs[11]), "+&v"(xs[12]), "+&v"(xs[13]), "+&v"(xs[14]), "+&v"(xs[15])
      : "v"(nf), "n"(J));
}
template <int J>
__device__ __forceinline__ void update_bcast(float (&xs)[16], float nf) {
  asm("s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %0, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %1, %1, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %2, %2, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %3, %3, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %4, %4, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %5, %5, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %6, %6, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %7, %7, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %8, %8, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %9, %9, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %10, %10, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %11, %11, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %12, %12, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %13, %13, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %14, %14, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %15, %15, %16 row_newbcast:%17 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(xs[0]), "+&v"(xs[1]), "+&v"(xs[2]), "+&v"(xs[3]), "+&v"(xs[4]), "+&v"(xs[5]), "+&v"(xs[6]), "+&v"(xs[7]), "+&v"(xs[8]), "+&v"(xs[9]), "+&v"(xs[10]), "+&v"(xs[11]), "+&v"(xs[12]), "+&v"(xs[13]), "+&v"(xs[14]), "+&v"(xs[15])
      : "v"(nf), "n"(J));
}

// The same for half as many entries per lane.
template <int J>
__device__ __forceinline__ void dots_bcast(const double (&xs)[8], double& d0, double& d1) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %2 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %3, %3 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %4, %4 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %5, %5 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %6, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %7, %7 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %8, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %9, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(d0), "+&v"(d1)
      : "v"(xs[0]), "v"(xs[1]), "v"(xs[2]), "v"(xs[3]), "v"(xs[4]), "v"(xs[5]), "v"(xs[6]), "v"(xs[7]), "n"(J));
}
template <int J>
__device__ __forceinline__ void update_bcast(double (&xs)[8], double nf) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %1, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %2, %2, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %3, %3, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %4, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %5, %5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %6, %6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %7, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(xs[0]), "+&v"(xs[1]), "+&v"(xs[2]), "+&v"(xs[3]), "+&v"(xs[4]), "+&v"(xs[5]), "+&v"(xs[6]), "+&v"(xs[7])
      : "v"(nf), "n"(J));
}
//   s0 += sum over k = K, K + 2 of v_k t[k], s1 over k = K + 1, K + 3, where
//   v_k is lane k's v in each 16-lane row.
template <int K>
__device__ __forceinline__ void bcast_terms(double v, const double (&t)[16], double& s0,
                                            double& s1) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      : "+&v"(s0), "+&v"(s1)
      : "v"(v), "v"(t[K]), "v"(t[K + 1]), "v"(t[K + 2]), "v"(t[K + 3]), "n"(K), "n"(K + 1),
        "n"(K + 2), "n"(K + 3));
}

// y[i] += v_i f for i = I .. I + N - 1, v_i being lane i's v in each 16-lane row.
template <int I, int N>
__device__ __forceinline__ void bcast_axpy(double v, double f, double (&y)[16]) {
  if constexpr (N >= 4) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %1, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %3, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+&v"(y[I]), "+&v"(y[I + 1]), "+&v"(y[I + 2]), "+&v"(y[I + 3])
        : "v"(v), "v"(f), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
    bcast_axpy<I + 4, N - 4>(v, f, y);
  } else if constexpr (N >= 1) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+v"(y[I])
        : "v"(v), "v"(f), "n"(I));
    bcast_axpy<I + 1, N - 1>(v, f, y);
  }
}

// y[i] += x_J[i] f for i = I .. I + N - 1 (N <= 4), x_J being lane J's x in
// each 16-lane row.
template <int J, int N, int I, typename X, typename Y>
__device__ __forceinline__ void bcast_fmac(const X& x, Y& y, double f) {
  if constexpr (N >= 4) {
    double y0 = y[I], y1 = y[I + 1], y2 = y[I + 2], y3 = y[I + 3];
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %1, %5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %2, %6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %3, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+&v"(y0), "+&v"(y1), "+&v"(y2), "+&v"(y3)
        : "v"(x[I]), "v"(x[I + 1]), "v"(x[I + 2]), "v"(x[I + 3]), "v"(f), "n"(J));
    y[I] = y0, y[I + 1] = y1, y[I + 2] = y2, y[I + 3] = y3;
  } else if constexpr (N >= 1) {
    double y0 = y[I];
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+v"(y0)
        : "v"(x[I]), "v"(f), "n"(J));
    y[I] = y0;
    bcast_fmac<J, N - 1, I + 1>(x, y, f);
  }
}
// x[i] += x_J[i] f in place.
template <int J, int N, int I, typename X>
__device__ __forceinline__ void bcast_fmac_self(X& x, double f) {
  if constexpr (N >= 4) {
    double x0 = x[I], x1 = x[I + 1], x2 = x[I + 2], x3 = x[I + 3];
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %0, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %1, %1, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %2, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %3, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+&v"(x0), "+&v"(x1), "+&v"(x2), "+&v"(x3)
        : "v"(f), "n"(J));
    x[I] = x0, x[I + 1] = x1, x[I + 2] = x2, x[I + 3] = x3;
  } else if constexpr (N >= 1) {
    double x0 = x[I];
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        : "+v"(x0)
        : "v"(f), "n"(J));
    x[I] = x0;
    bcast_fmac_self<J, N - 1, I + 1>(x, f);
  }
}
// The same for i = I .. E - 1, four at a time.
template <int J, int I, int E, typename X, typename Y>
__device__ __forceinline__ void bcast_fmacs(const X& x, Y& y, double f) {
  if constexpr (I < E) {
    constexpr int N = (I & 3) ? 4 - (I & 3) : 4, M = N < E - I ? N : E - I;
    bcast_fmac<J, M, I>(x, y, f);
    bcast_fmacs<J, I + M, E>(x, y, f);
  }
}
template <int J, int I, int E, typename X>
__device__ __forceinline__ void bcast_fmacs_self(X& x, double f) {
  if constexpr (I < E) {
    constexpr int N = (I & 3) ? 4 - (I & 3) : 4, M = N < E - I ? N : E - I;
    bcast_fmac_self<J, M, I>(x, f);
    bcast_fmacs_self<J, I + M, E>(x, f);
  }
}

// Lane group QJ's value to all four groups (lanes cl, cl + 16, cl + 32,
// cl + 48): v_permlane16_swap leaves rows (0, 0, 2, 2) in one copy and
// (1, 1, 3, 3) in the other, v_permlane32_swap then halves (0, 1, 0, 1) and
// (2, 3, 2, 3).
template <int QJ>
__device__ __forceinline__ double group_bcast(double v) {
  unsigned lo = lo32(v), hi = hi32(v);
  {
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    lo = (QJ & 1) ? l[1] : l[0];
    hi = (QJ & 1) ? h[1] : h[0];
  }
  {
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    lo = (QJ & 2) ? l[1] : l[0];
    hi = (QJ & 2) ? h[1] : h[0];
  }
  return join(lo, hi);
}

// Workgroup barrier that orders LDS only: global loads in flight (a
// prefetch) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The lane index through an empty asm: addresses, masks and row numbers made
// from it are then computed where they are used.  Otherwise the compiler
// hoists them out of the sweep's loops as invariants and holds dozens of
// them in registers for the whole problem, spilling the tiles.
__device__ __forceinline__ int lane_id() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

}  // namespace miqr
