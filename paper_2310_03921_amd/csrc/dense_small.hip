// FP64 contractions of prediction and backward for calls with few atoms or
// few output tiles (a molecular-dynamics cell, a training batch of a small
// model), where the LDS-staged kernels of dense_f64.hip leave most of the chip
// idle: their blocks of 64 x 128 outputs give a 64-atom cell 2 to 16 blocks,
// each walking the whole contraction alone.
//
// Here a block owns 32 x 32 outputs and its four waves split the contraction:
// wave w takes the 16-deep chunks w, w + 4, ... of the block's range of k, as
// 2 x 2 matrix-core tiles whose operands come straight from L2 (no staging, no
// barrier in the loop), and the four partial tiles are added in LDS in wave
// order.  Where the outputs alone give too few blocks, the range of k is split
// over grid slices as well, whose partial outputs are summed in slice order.
// Bound by latency (a few dependent round trips to L2) at the small end and by
// L2 bandwidth (4 flop per byte) at the large end, where the staged kernels
// take over.  For 64 atoms, 2000 sparse points and 252 entries the P-stage went
// from 35 to 12 us and W X from 161 to 10 us; W^T D of 5021 atoms and 500
// points from 224 to 38 us.
#include <algorithm>

#include "launch.h"
#include "mma_f64.h"

namespace gapk {

namespace {

constexpr int kT = 32;        // edge of a block's output tile
constexpr int kTS = kT + 1;   // row stride of the tile in LDS

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

// An operand whose element k of row i lies at p[i * ld + k] / p[k * ld + i].
template <typename T>
struct RowOp {
  const T* p;
  int64_t ld, n;
  using Frag = FragRowK<T>;
  GAP_DEV Frag at(int64_t i, int64_t kmax) const { return {p + min(i, n - 1) * ld, kmax, true}; }
};
template <typename T>
struct ColOp {
  const T* p;
  int64_t ld, n;
  using Frag = FragColK<T>;
  GAP_DEV Frag at(int64_t i, int64_t kmax) const { return {p + min(i, n - 1), ld, kmax, true}; }
};
// Rows of W with column k scaled by cs[k].
struct FragScaled {
  FragRowK<double> w;
  const double* cs;
  struct Raw {
    Raw4<double> w, c;
  };
  GAP_DEV void frag(int64_t k0, int g, double out[4]) const {
    w.frag(k0, g, out);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t k = k0 + 4 * g + s;
      out[s] = k < w.kmax ? out[s] * cs[min(k, w.kmax - 1)] : 0.0;
    }
  }
  GAP_DEV void fast(int64_t k0, int g, Raw& r) const {
    w.fast(k0, g, r.w);
#pragma unroll
    for (int s = 0; s < 4; ++s) r.c.v[s] = cs[k0 + 4 * g + s];
  }
  GAP_DEV void cook(const Raw& r, double out[4]) const {
#pragma unroll
    for (int s = 0; s < 4; ++s) out[s] = r.w.v[s] * r.c.v[s];
  }
};
struct ScaledRowOp {
  const double* p;
  int64_t ld, n;
  const double* cs;
  using Frag = FragScaled;
  GAP_DEV Frag at(int64_t i, int64_t kmax) const {
    return {{p + min(i, n - 1) * ld, kmax, true}, cs};
  }
};

// v[q] = sum over k in [k_lo, k_hi) of A[row0 + t / 8][k] B[col0 + 4 (t % 8) + q][k]
// for thread t of the block's 256: the waves' products, added through LDS.
// Rows and columns past the operands' ends give values the caller drops.  k_lo
// is a multiple of 16; a last chunk cut by k_hi = K is read with guards.
template <class OA, class OB>
GAP_DEV void block_tile(const OA& A, const OB& B, int64_t row0, int64_t col0, int64_t k_lo,
                        int64_t k_hi, double (*red)[kT][kTS], double v[4]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, idx = lane & 15;
  typename OA::Frag fa[2];
  typename OB::Frag fb[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    fa[u] = A.at(row0 + 16 * u + idx, k_hi);
    fb[u] = B.at(col0 + 16 * u + idx, k_hi);
  }
  d4v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = zero4();
  auto products = [&](const double (&a)[2][4], const double (&b)[2][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(a[i][s], b[j][s], acc[i][j]);
  };
  // whole chunks, the next one in flight while the current one is multiplied
  const int64_t k_full = k_lo + ((k_hi - k_lo) & ~int64_t(15));
  const int64_t k_first = k_lo + 16 * wave;
  if (k_first < k_full) {
    const int64_t k_last = k_first + (k_full - 16 - k_first) / 64 * 64;
    typename OA::Frag::Raw ra[2][2];
    typename OB::Frag::Raw rb[2][2];
    auto fetch = [&](int64_t k, const int set) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        fa[u].fast(k, g, ra[set][u]);
        fb[u].fast(k, g, rb[set][u]);
      }
    };
    auto use = [&](const int set) {
      double a[2][4], b[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        fa[u].cook(ra[set][u], a[u]);
        fb[u].cook(rb[set][u], b[u]);
      }
      products(a, b);
    };
    fetch(k_first, 0);
    int64_t k = k_first;
    for (; k < k_last; k += 128) {
      fetch(k + 64, 1);
      use(0);
      fetch(min(k + 128, k_last), 0);  // (past the end: re-reads the last chunk, unused)
      use(1);
    }
    if (k == k_last) use(0);
  }
  if (k_full < k_hi && wave == (int)(((k_full - k_lo) >> 4) & 3)) {
    double a[2][4], b[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      fa[u].frag(k_full, g, a[u]);
      fb[u].frag(k_full, g, b[u]);
    }
    products(a, b);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][16 * i + g + 4 * r][16 * j + idx] = acc[i][j][r];
  __syncthreads();
  const int row = threadIdx.x >> 3, c4 = (threadIdx.x & 7) * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    v[q] = ((red[0][row][c4 + q] + red[1][row][c4 + q]) + red[2][row][c4 + q]) +
           red[3][row][c4 + q];
}

// out[z][i][j] = sum over slice z of k of A[i][k] B[j][k]; with `upper`, B[j][k]
// is zero for k > j and those k are left out.
template <class OA, class OB>
__global__ __launch_bounds__(256) void k_gemm_small(OA A, OB B, int64_t K, int64_t k_per,
                                                    int upper, double* __restrict__ out,
                                                    int64_t ldo, int64_t stride) {
  __shared__ double red[4][kT][kTS];
  const int64_t col0 = (int64_t)blockIdx.x * kT, row0 = (int64_t)blockIdx.y * kT;
  const int64_t k_lo = (int64_t)blockIdx.z * k_per;
  double v[4];
  const int64_t k_hi = min(upper ? min(K, col0 + kT) : K, k_lo + k_per);
  block_tile(A, B, row0, col0, k_lo, max(k_hi, k_lo), red, v);
  const int64_t row = row0 + (threadIdx.x >> 3), col = col0 + (threadIdx.x & 7) * 4;
  double* o = out + blockIdx.z * stride + row * ldo + col;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (row < A.n && col + q < B.n) o[q] = v[q];
}

// One level of the triangular inverse by doubling, for the pair of diagonal
// blocks blockIdx.z (the first s x s, the second possibly cut by n):
// STEP 0: tmp = R12 Y22 (Y22 upper: k <= column), and Y21 = 0;
// STEP 1: Y12 = -Y11 tmp (Y11 upper: k >= row).
template <int STEP>
__global__ __launch_bounds__(256) void k_trinv_level(const double* __restrict__ R, int64_t ldr,
                                                     double* __restrict__ Y, int64_t ldy,
                                                     int64_t n, int64_t s,
                                                     double* __restrict__ tmp) {
  __shared__ double red[4][kT][kTS];
  const int64_t b1 = 2 * s * (int64_t)blockIdx.z, b2 = b1 + s, s2 = min(s, n - b2);
  const int64_t col0 = (int64_t)blockIdx.x * kT, row0 = (int64_t)blockIdx.y * kT;
  if (col0 >= s2) return;
  double* tp = tmp + (int64_t)blockIdx.z * s * s;  // s x s2, row-major
  double v[4];
  if (STEP == 0)
    block_tile(ColOp<double>{R + b1 + b2 * ldr, ldr, s}, ColOp<double>{Y + b2 * ldy + b2, ldy, s2},
               row0, col0, 0, min(s2, col0 + kT), red, v);
  else
    block_tile(RowOp<double>{Y + b1 * ldy + b1, ldy, s}, ColOp<double>{tp, s2, s2}, row0, col0,
               row0, s, red, v);
  const int64_t i = row0 + (threadIdx.x >> 3), j = col0 + (threadIdx.x & 7) * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (i >= s || j + q >= s2) continue;
    if (STEP == 0) {
      tp[i * s2 + j + q] = v[q];
      Y[(b2 + j + q) * ldy + b1 + i] = 0.0;
    } else {
      Y[(b1 + i) * ldy + b2 + j + q] = -v[q];
    }
  }
}

// P-stage of k_pstage_q (same modes and outputs) on 32 x 32 tiles: e_part has a
// group per 32 sparse points, dc_part a row per 32 atoms.
template <typename TD, int MODE>
__global__ __launch_bounds__(256) void k_pstage_small(
    RowOp<TD> rows, RowOp<double> pts, int64_t D, int zeta, double delta,
    const double* __restrict__ cc, const double* __restrict__ g_e, double* __restrict__ W,
    int64_t ldw, double* __restrict__ e_part, double* __restrict__ dc_part,
    const double* __restrict__ Sx, int64_t ldsx) {
  __shared__ double red[4][kT][kTS];
  __shared__ double csum[4][kT];
  const int64_t n = rows.n, M = pts.n;
  const int64_t col0 = (int64_t)blockIdx.x * kT, row0 = (int64_t)blockIdx.y * kT;
  double p[4];
  block_tile(rows, pts, row0, col0, 0, D, red, p);
  const int64_t row = row0 + (threadIdx.x >> 3), col = col0 + (threadIdx.x & 7) * 4;
  const double d2 = delta * delta, d2z = d2 * zeta;
  const double ge = (MODE == 1 && row < n) ? g_e[row] : 0.0;
  double s[4] = {0.0, 0.0, 0.0, 0.0};  // the entry's share of the row or column sums
  if (row < n) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (col + q >= M) {
        if (MODE != 3 && W && col + q < ldw) W[row * ldw + col + q] = 0.0;  // row padding
        continue;
      }
      if (MODE == 3) {
        s[q] = -(Sx[row * ldsx + col + q] * p[q]);
        continue;
      }
      const double cm = cc[col + q], pz1 = ipow(p[q], zeta - 1), kval = d2 * pz1 * p[q];
      s[q] = MODE == 0 ? cm * kval : ge * kval;
      if (W) W[row * ldw + col + q] = MODE == 0 ? d2z * cm * pz1 : ge * d2z * cm * pz1;
    }
  }
  if (MODE == 0) {
    if (!e_part) return;
    double e = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) e += __shfl_xor(e, o);
    if ((threadIdx.x & 7) == 0 && row < n) e_part[blockIdx.x * n + row] = e;
    return;
  }
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) s[q] += __shfl_xor(s[q], o);
    if ((threadIdx.x & 63) < 8) csum[wave][(threadIdx.x & 7) * 4 + q] = s[q];
  }
  __syncthreads();
  if (threadIdx.x < kT && col0 + threadIdx.x < M)
    dc_part[blockIdx.y * M + col0 + threadIdx.x] =
        ((csum[0][threadIdx.x] + csum[1][threadIdx.x]) + csum[2][threadIdx.x]) +
        csum[3][threadIdx.x];
}

// Slices of the contraction: enough of them for about two blocks per compute
// unit, with at least 128 k (two chunks per wave) each.
int slices(int64_t tiles, int64_t K) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(512 / tiles, K / 128));
}
int64_t tiles(int64_t a, int64_t b) { return (int64_t)cdiv(a, kT) * cdiv(b, kT); }

template <class OA, class OB>
void launch_small(const OA& A, const OB& B, int64_t K, double* part, double* out, int64_t ldo,
                  hipStream_t st, int upper = 0) {
  const int64_t nz = slices(tiles(A.n, B.n), K);
  const int64_t k_per = ((K + nz - 1) / nz + 63) / 64 * 64;
  const unsigned z = cdiv(K, k_per);
  const dim3 grid(cdiv(B.n, kT), cdiv(A.n, kT), z);
  if (z == 1) {
    hipLaunchKernelGGL((k_gemm_small<OA, OB>), grid, dim3(256), 0, st, A, B, K, k_per, upper, out,
                       ldo, int64_t(0));
    return;
  }
  hipLaunchKernelGGL((k_gemm_small<OA, OB>), grid, dim3(256), 0, st, A, B, K, k_per, upper, part,
                     B.n, A.n * B.n);
  sum_parts_f64(part, z, A.n * B.n, out, A.n, ldo, B.n, st);
}

}  // namespace

size_t small_part_bytes(int64_t n_rows, int64_t n_cols, int64_t K) {
  const int64_t nz = slices(tiles(n_rows, n_cols), K);
  return nz > 1 ? sizeof(double) * nz * n_rows * n_cols : 0;
}

void small_pstage_f64(int mode, const void* rows, bool rows_f32, int64_t ldd, int64_t n,
                      const double* X, int64_t ldx, int64_t M, int64_t D, int zeta, double delta,
                      const double* c, const double* g_e, double* W, int64_t ldw, double* e_part,
                      double* dc_part, const double* Sx, int64_t ldsx, hipStream_t st) {
  const dim3 grid(cdiv(M, kT), cdiv(n, kT));
  const RowOp<double> pts{X, ldx, M};
  auto go = [&](auto kern, auto op) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, op, pts, D, zeta, delta, c, g_e, W, ldw,
                       e_part, dc_part, Sx, ldsx);
  };
  const RowOp<float> r32{static_cast<const float*>(rows), ldd, n};
  const RowOp<double> r64{static_cast<const double*>(rows), ldd, n};
  if (mode == 3)
    go(k_pstage_small<double, 3>, r64);
  else if (rows_f32)
    mode == 0 ? go(k_pstage_small<float, 0>, r32) : go(k_pstage_small<float, 1>, r32);
  else
    mode == 0 ? go(k_pstage_small<double, 0>, r64) : go(k_pstage_small<double, 1>, r64);
}

void small_wx_f64(const double* W, int64_t ldw, int64_t n, int64_t M, const double* cs,
                  const double* X, int64_t ldx, int64_t D, double* part, double* out, int64_t ldo,
                  hipStream_t st, bool upper) {
  const ColOp<double> x{X, ldx, D};
  if (cs)
    launch_small(ScaledRowOp{W, ldw, n, cs}, x, M, part, out, ldo, st, upper);
  else
    launch_small(RowOp<double>{W, ldw, n}, x, M, part, out, ldo, st, upper);
}

void small_trinv_level(const double* R, int64_t ldr, double* Y, int64_t ldy, int64_t n, int64_t s,
                       double* tmp, hipStream_t st) {
  const unsigned pairs = cdiv(n - s, 2 * s), t = cdiv(s, kT);
  hipLaunchKernelGGL(k_trinv_level<0>, dim3(t, t, pairs), dim3(256), 0, st, R, ldr, Y, ldy, n, s,
                     tmp);
  hipLaunchKernelGGL(k_trinv_level<1>, dim3(t, t, pairs), dim3(256), 0, st, R, ldr, Y, ldy, n, s,
                     tmp);
}

void small_wtd_f64(const double* W, int64_t ldw, int64_t n, int64_t M, const void* desc,
                   bool desc_f32, int64_t ldd, int64_t D, double* part, double* out, int64_t ldo,
                   hipStream_t st) {
  const ColOp<double> w{W, ldw, M};
  if (desc_f32)
    launch_small(w, ColOp<float>{static_cast<const float*>(desc), ldd, D}, n, part, out, ldo, st);
  else
    launch_small(w, ColOp<double>{static_cast<const double*>(desc), ldd, D}, n, part, out, ldo,
                 st);
}

}  // namespace gapk
