// 64 x 64 triangular building blocks in FP64: Cholesky factorisation of a block
// held in LDS, and substitution of rows held in registers against an upper
// triangle held in LDS.
#pragma once

#include <utility>

#include "common.h"

constexpr int kTri = 64;
constexpr int kTriS = kTri + 1;  // row stride of a block in LDS: columns read conflict-free

// 1 / sqrt(p) for p > 0: the hardware estimate and two Newton steps.
GAP_DEV double rsqrt_f64(double p) {
  double r = __builtin_amdgcn_rsq(p);
#pragma unroll
  for (int i = 0; i < 2; ++i) r = fma(r, 0.5 * fma(-p * r, r, 1.0), r);
  return r;
}

GAP_DEV double readlane_f64(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Lower Cholesky factor of the 64 x 64 block S (lower triangle read and
// overwritten), by a workgroup of 256 threads; S is complete on return.  Four
// steps of 16 columns: one wave factors the columns with a row per lane (the
// pivot's reciprocal root and the rows of L it needs come by readlane, so the
// chain per column has no LDS access, square root or division), then the four
// waves update the rest on the matrix cores.  Returns whether a pivot was not
// positive and finite (it is replaced by 1), the same value in every thread of
// wave 0 only.  The one-wave form it replaces, whose lanes formed each dot
// product from LDS, took 44 us a block; this one 19 us, launch and loads
// included, and 11 us on top of a Cholesky update that goes on to it.
GAP_DEV bool chol64_lds(double (*S)[kTriS]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, idx = lane & 15;
  bool bad = false;
  for (int s = 0; s < 4; ++s) {
    const int c0 = 16 * s;
    if (wave == 0) {
      double v[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = S[lane][c0 + c];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        double p = readlane_f64(v[c], c0 + c);
        const bool ok = p > 0.0 && isfinite(p);
        bad |= !ok;
        p = ok ? p : 1.0;
        const double r = rsqrt_f64(p);
        v[c] = lane == c0 + c ? p * r : v[c] * r;
#pragma unroll
        for (int q = c + 1; q < 16; ++q) v[q] -= v[c] * readlane_f64(v[c], c0 + q);
      }
#pragma unroll
      for (int c = 0; c < 16; ++c)
        if (lane >= c0 + c) S[lane][c0 + c] = v[c];
    }
    __syncthreads();
    // tiles (ti, tj), s < tj <= ti < 4, dealt to the waves
    int t = 0;
    for (int ti = s + 1; ti < 4; ++ti)
      for (int tj = s + 1; tj <= ti; ++tj, ++t) {
        if ((t & 3) != wave) continue;
        d4v acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = S[16 * ti + g + 4 * r][16 * tj + idx];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc = mfma_f64(-S[16 * ti + idx][c0 + 4 * g + q], S[16 * tj + idx][c0 + 4 * g + q], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) S[16 * ti + g + 4 * r][16 * tj + idx] = acc[r];
      }
    __syncthreads();
  }
  return bad;
}

// 1 / d: the hardware estimate and two Newton steps (0 and non-finite d give
// what the estimate gives).
GAP_DEV double rcp_f64(double d) {
  const double r0 = __builtin_amdgcn_rcp(d);
  double r = r0;
#pragma unroll
  for (int i = 0; i < 2; ++i) r = fma(r, fma(-d, r, 1.0), r);
  return isfinite(r) ? r : r0;
}

// The groups of sixteen entries (c, 16 k .. 16 k + 15) of U right of its
// diagonal, in the order row_solve64 needs them.
struct TriGroups {
  static constexpr int n = 156;
  int c[n], k[n];
  constexpr TriGroups() : c(), k() {
    int i = 0;
    for (int cc = 0; cc < kTri - 1; ++cc)
      for (int kk = (cc + 1) / 16; kk < kTri / 16; ++kk, ++i) c[i] = cc, k[i] = kk;
  }
};
constexpr TriGroups kTriGroups;
constexpr int kTriAhead = 3;  // groups read ahead

template <int I>
GAP_DEV void tri_read(d2v (&buf)[kTriAhead + 1][8], const d2v* u2) {
  if constexpr (I < TriGroups::n) {
    constexpr int c = kTriGroups.c[I], k = kTriGroups.k[I];
#pragma unroll
    for (int h = 0; h < 8; ++h)
      if (16 * k + 2 * h + 1 > c) buf[I % (kTriAhead + 1)][h] = u2[c * (kTri / 2) + 8 * k + h];
  }
}
template <int I>
GAP_DEV void tri_step(double (&x)[kTri], d2v (&buf)[kTriAhead + 1][8], const d2v* u2,
                      const double* rinv) {
  constexpr int c = kTriGroups.c[I], k = kTriGroups.k[I];
  if constexpr (k == (c + 1) / 16) x[c] *= rinv[c];
  tri_read<I + kTriAhead>(buf, u2);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 16; ++q)
    if (16 * k + q > c)
      x[16 * k + q] = fma(-x[c], buf[I % (kTriAhead + 1)][q / 2][q & 1], x[16 * k + q]);
}
template <int... I>
GAP_DEV void tri_steps(double (&x)[kTri], const d2v* u2, const double* rinv,
                       std::integer_sequence<int, I...>) {
  d2v buf[kTriAhead + 1][8];
  tri_read<0>(buf, u2);
  tri_read<1>(buf, u2);
  tri_read<2>(buf, u2);
  (tri_step<I>(x, buf, u2, rinv), ...);
}

// x <- x U^-1 for a lane's row x: U[c][q] (q >= c) at u[c * kTri + q] and the
// reciprocal diagonal at rinv[c], in LDS (u 16-byte aligned), the same for every
// lane.  Right-looking, so the updates of one column are independent of each
// other, with the entries of U read three groups of sixteen ahead of their use.
// (Left to the compiler's schedule the wave waits for a read at nearly every
// step; scalar loads of U from global memory cost a cache miss per eight
// entries, 57 us in all.)
GAP_DEV void row_solve64(double (&x)[kTri], const double* u, const double* rinv) {
  tri_steps(x, reinterpret_cast<const d2v*>(u), rinv,
            std::make_integer_sequence<int, TriGroups::n>{});
  x[kTri - 1] *= rinv[kTri - 1];
  // the values are made here: sunk to a guarded store after this, the updates
  // would leave all reads of U behind, and spill
#pragma unroll
  for (int c = 0; c < kTri; ++c) asm volatile("" : "+v"(x[c]));
}
