// 64 x 64 triangular building blocks in FP64: Cholesky factorisation of a block
// held in LDS, and the solution of rows held in registers against an upper
// triangle, on the matrix cores.
#pragma once

#include "common.h"

constexpr int kTri = 64;
constexpr int kTriS = kTri + 1;  // row stride of a block in LDS: columns read conflict-free

// 1 / sqrt(p) for p > 0 and 1 / d: the hardware estimate and one third-order
// step (its relative error e becomes of the order of e^3, below rounding).
GAP_DEV double rsqrt_f64(double p) {
  const double r = __builtin_amdgcn_rsq(p);
  const double e = fma(-p * r, r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}
GAP_DEV double rcp_f64(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, r, 1.0);
  return fma(r * e, 1.0 + e, r);
}

GAP_DEV double readlane_f64(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Lower Cholesky factor of the 64 x 64 block S (lower triangle read and
// overwritten; unit columns from 16 nb on), by a workgroup of 256 threads; S is
// complete on return.  nb steps of 16 columns: one wave factors the columns with a row per lane (the
// pivot's reciprocal root and the rows of L it needs come by readlane, so the
// chain per column has no LDS access, square root or division), then the four
// waves update the rest on the matrix cores.  Returns whether a pivot was not
// positive and finite (it is replaced by 1), the same value in every thread of
// wave 0 only.  The one-wave form it replaces, whose lanes formed each dot
// product from LDS, took 44 us a block; this one 19 us, launch and loads
// included, and 11 us on top of a Cholesky update that goes on to it.
GAP_DEV bool chol64_lds(double (*S)[kTriS], int nb = 4, int lane = threadIdx.x & 63) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, idx = lane & 15;
  bool bad = false;
  for (int s = 0; s < nb; ++s) {
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
    // tiles (ti, tj), s < tj <= ti < nb, dealt to the waves
    int t = 0;
    for (int ti = s + 1; ti < nb; ++ti)
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

// Inverses of the four 16 x 16 diagonal blocks of an upper triangle u(i, j), by
// one wave, a row per lane: inv[256 b + 16 i + c], zero below the diagonal.
template <class FU>
GAP_DEV void tri_inv16(FU u, double* inv, int lane = threadIdx.x & 63) {
  const int o = lane & 48, i = lane & 15;
  double y[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) y[c] = c == i ? 1.0 : 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    y[c] *= rcp_f64(u(o + c, o + c));
#pragma unroll
    for (int q = c + 1; q < 16; ++q) y[q] = fma(-y[c], u(o + c, o + q), y[q]);
  }
#pragma unroll
  for (int c = 0; c < 16; ++c) inv[16 * o + 16 * i + c] = y[c];
}

// Operands of x <- x U^-1 on the matrix cores for 16 rows x per wave: the 16 x 16
// blocks of U right of and on its diagonal (negated) and the inverses of the
// diagonal blocks.  As first operand (i = column of U, k = row): lane (g, idx)
// holds U[16 kb + g + 4 r][16 b + idx] for r = 0 .. 3.
struct TriOps {
  d4v off[6], dia[4], inv[4];  // off: (kb, b) = (0,1) (0,2) (1,2) (0,3) (1,3) (2,3)
};
template <class FU, class FI>
GAP_DEV void tri_ops(TriOps& t, FU u, FI inv, int lane = threadIdx.x & 63) {
  const int g = lane >> 4, idx = lane & 15;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = g + 4 * r;
      t.dia[b][r] = k <= idx ? -u(16 * b + k, 16 * b + idx) : 0.0;
      t.inv[b][r] = inv(256 * b + 16 * k + idx);
    }
#pragma unroll
    for (int kb = 0; kb < b; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        t.off[b * (b - 1) / 2 + kb][r] = -u(16 * kb + g + 4 * r, 16 * b + idx);
  }
}

// x <- x U^-1 for a wave's 16 rows: x[b][r] of lane (g, idx) is row idx, column
// 16 b + g + 4 r (the matrix core's result layout of the transpose, which is
// also what the next product takes as its second operand).  Each 16-column block
// is multiplied by the inverse of its diagonal block and corrected once with its
// residual, which leaves a backward error of rounding size, as a substitution
// does, while that block's condition is below 1e8 (it enters squared, times
// u^2): a Cholesky factor of a matrix that was found positive definite, and panels
// whose Gram passed its test.  For the rows of the unit matrix (an inverse) the error
// is a substitution's at any condition: 1.0 to 1.4 u |Y||U||Y| entry by entry, where a
// substitution has 0.8 to 2.9, for block conditions up to 2e14.  The substitution column by column took four times as long (33,000 cycles
// against 72 dependent matrix instructions for the 64 columns).
GAP_DEV void tri_solve16(const TriOps& t, d4v (&x)[4]) {
  auto mul = [](const d4v& a, const d4v& b, d4v c) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c = mfma_f64(a[r], b[r], c);
    return c;
  };
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    d4v a = x[b];
#pragma unroll
    for (int kb = 0; kb < b; ++kb) a = mul(t.off[b * (b - 1) / 2 + kb], x[kb], a);
    const d4v y = mul(t.inv[b], a, zero4());
    x[b] = mul(t.inv[b], mul(t.dia[b], y, a), y);
  }
}
