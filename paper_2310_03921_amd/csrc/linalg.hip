// FP64 linear algebra of the stable least-squares route (Sec. "Theory"):
//   A = [Sigma^-1/2 L-hat K_NM ; U_MM],  b = [Sigma^-1/2 y ; 0],
//   K_MM + jitter I = U^T U (Cholesky), A = QR (Householder), c = R^-1 Q^T b,
// plus the pieces of FP64 iterative refinement (semi-normal equations).
//
// Householder QR, right-looking and blocked (compact WY, Q = I - V T V^T):
//   panel: 64 columns at once, by Cholesky QR twice and the reconstruction of
//          the Householder vectors (all products on FP64 MFMA, three small
//          one-block steps); a cooperative kernel that adds shifted rounds takes
//          a panel whose columns are numerically dependent, and one that holds
//          the columns in registers a last block of up to sixteen.
//   trailing update: W = V^T C (split over row slabs on FP64 MFMA, then a
//          fixed-order reduction) and C -= V (T^T W) on FP64 MFMA, T from the
//          panel (from the Gram V^T V and tau where one of the other two
//          kernels took it).  b rides along as the last column.
#include <algorithm>

#include "launch.h"
#include "mma_f64.h"
#include "tri64.h"

namespace gapk {

namespace {

constexpr int kQrNB = 64;      // outer block width (compact-WY trailing update)
constexpr int kTrsvMaxBlocks = 256;  // multi-block triangular solve: n <= 64 * 256
constexpr int kPanelMaxGrid = 256;
// Workspace counter words: [0], [1] the states of an outer block's two panels (1:
// the panel is left to k_qr_panel_dep), [kPanelBar ..) that kernel's eight arrival counters.
constexpr int kPanelBar = 64;
constexpr int kPanelBarWords = 8 * 16;
constexpr int kCounterWords = 256;

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

// Values exchanged between blocks of one launch (which may run on different
// XCDs with separate L2 caches) are written and read with relaxed device-scope
// atomics, which bypass the non-coherent caches, and ordered with s_waitcnt.
// No device-scope fence is used: on this part such a fence writes back and
// invalidates a whole L2.
GAP_DEV double vload(const double* p) {
  const uint64_t bits = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_bit_cast(double, bits);
}
GAP_DEV void xstore(double* p, double v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, v),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A value the compiler takes as new, so that what is derived from it is formed where
// it is used and not kept in registers from one phase of a long kernel to the next.
GAP_DEV int64_t fresh(int64_t x) {
  asm volatile("" : "+s"(x));
  return x;
}
template <typename T>
GAP_DEV T* fresh(T* p) {
  asm volatile("" : "+s"(p));
  return p;
}
GAP_DEV int fresh(int x) {
  asm volatile("" : "+s"(x));
  return x;
}
GAP_DEV int fresh_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
GAP_DEV int fresh_lane() { return fresh_thread() & 63; }
// Wait until every memory operation this wave issued has completed.
GAP_DEV void wait_mem() { __builtin_amdgcn_s_waitcnt(0); }

// ----------------------------------------------------------- scale/stack ----
// rows r < n_rows: A[r][0:M] /= sigma_r, A[r][M] = y_r / sigma_r
__global__ void k_scale_rows(double* __restrict__ A, int64_t ld, int64_t n_rows, int64_t M,
                             const double* __restrict__ y, const double* __restrict__ sigma) {
  const int64_t col = blockIdx.y;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n_rows;
       r += (int64_t)gridDim.x * blockDim.x) {
    const double w = 1.0 / sigma[r];
    A[r + col * ld] = (col < M) ? A[r + col * ld] * w : y[r] * w;
  }
}

// rows n_rows + i (i < M): U = L^T (row i of U is column i of L), b = 0
__global__ void k_stack_u(double* __restrict__ A, int64_t ld, int64_t n_rows, int64_t M,
                          const double* __restrict__ L, int64_t ldl) {
  const int64_t col = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < M;
       i += (int64_t)gridDim.x * blockDim.x)
    A[(n_rows + i) + col * ld] = (col < M && col >= i) ? L[col + i * ldl] : 0.0;
}

// -------------------------------------------------------------- Cholesky ----
__global__ void k_chol_init(double* __restrict__ Lw, int64_t ldl, int64_t M, double jitter,
                            const double* __restrict__ Kmm, int64_t ldk) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < M;
       i += (int64_t)gridDim.x * blockDim.x)
    Lw[i + j * ldl] = Kmm[i + j * ldk] + (i == j ? jitter : 0.0);
}

// Lower triangle of the diagonal block at j0 (nbj <= 64 columns, completed with
// unit columns) from L into S, factored, and back; the inverses of its transposed
// factor's 16 x 16 diagonal blocks go to inv (1024 doubles).
GAP_DEV void chol_diag_block(double* __restrict__ Lw, int64_t ldl, int64_t j0, int nbj,
                             double (*S)[kTriS], double* __restrict__ inv, int* dev_err,
                             bool load) {
  if (load)
    for (int e = threadIdx.x; e < kTri * kTri; e += 256) {
      const int r = e & 63, c = e >> 6;
      if (r >= c) S[r][c] = r < nbj ? Lw[(j0 + r) + (j0 + c) * ldl] : (r == c ? 1.0 : 0.0);
    }
  __syncthreads();
  const bool bad = chol64_lds(S, (nbj + 15) / 16);
  if (bad && threadIdx.x == 0) atomicOr(dev_err, GAP_DEVERR_NOT_PD);
  if (threadIdx.x < 64) tri_inv16([&](int i, int j) { return S[j][i]; }, inv);
  for (int e = threadIdx.x; e < kTri * kTri; e += 256) {
    const int r = e & 63, c = e >> 6;
    if (r >= c && r < nbj) Lw[(j0 + r) + (j0 + c) * ldl] = S[r][c];
  }
}

__global__ __launch_bounds__(256) void k_chol_diag(double* __restrict__ Lw, int64_t ldl, int64_t j0,
                                                   int nbj, double* __restrict__ inv,
                                                   int* dev_err) {
  __shared__ double S[kTri][kTriS];
  chol_diag_block(Lw, ldl, j0, nbj, S, inv, dev_err, true);
}

// Rows below a full diagonal block: L[r, j0:j0+64] = A[r, j0:j0+64] L_dd^-T,
// sixteen rows per wave (34 us a block column when each entry waited for the dot
// product before it and divided).
__global__ __launch_bounds__(256) void k_chol_panel(double* __restrict__ Lw, int64_t ldl,
                                                    int64_t M, int64_t j0,
                                                    const double* __restrict__ inv) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int64_t r0 = j0 + kTri + (blockIdx.x * (int64_t)4 + wave) * 16;
  if (r0 >= M) return;
  double* A = Lw + j0 + j0 * ldl;
  double* row = Lw + min(r0 + idx, M - 1) + j0 * ldl;
  d4v x[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) x[b][r] = row[(16 * b + g + 4 * r) * ldl];
  TriOps t;
  tri_ops(t, [&](int i, int j) { return A[j + i * ldl]; },  // U[i][j] = L[j][i]
          [&](int e) { return inv[e]; });
  tri_solve16(t, x);
  // lanes past the last row hold that row too and store the same values
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) row[(16 * b + g + 4 * r) * ldl] = x[b][r];
}

// C[r][c] -= sum_k P[r][k] P[c][k] on the lower trailing block (r >= c), P the
// 64 columns at j0.  The first block goes on to factor its tile, the next
// diagonal block, while the others run.
__global__ __launch_bounds__(256) void k_chol_update(double* __restrict__ Lw, int64_t ldl,
                                                     int64_t M, int64_t j0,
                                                     double* __restrict__ inv, int* dev_err) {
  __shared__ double S[kTri][kTriS];
  const int64_t t0 = j0 + kTri;
  const int64_t cbase = t0 + (int64_t)blockIdx.x * 64;  // columns (MFMA rows)
  const int64_t rbase = t0 + (int64_t)blockIdx.y * 64;  // rows (MFMA columns)
  if (rbase + 63 < cbase) return;                        // tile strictly above the diagonal
  const bool next = blockIdx.x == 0 && blockIdx.y == 0;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int64_t c = cbase + wave * 16 + idx;
  FragColK<double> fa{Lw + (c < M ? c : 0) + j0 * ldl, ldl, kTri, c < M};
  FragColK<double> fb[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t r = rbase + u * 16 + idx;
    fb[u] = FragColK<double>{Lw + (r < M ? r : 0) + j0 * ldl, ldl, kTri, r < M};
  }
  d4v acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = zero4();
  wave_mma<4>(fa, fb, kTri, g, acc);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t r = rbase + u * 16 + idx;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t cc = cbase + wave * 16 + g + 4 * q;
      const bool in = r < M && cc < M && r >= cc;
      const double v = in ? Lw[r + cc * ldl] - acc[u][q] : (r == cc ? 1.0 : 0.0);
      if (next)
        S[r - rbase][cc - cbase] = v;
      else if (in)
        Lw[r + cc * ldl] = v;
    }
  }
  if (next)
    chol_diag_block(Lw, ldl, t0, (int)min((int64_t)kTri, M - t0), S, inv, dev_err, false);
}

// ------------------------------------------------------------------- QR ----
// Grid barrier on eight arrival counters, one per XCD slot of the block index
// (64 bytes apart), instead of one: the atomic adds of a few hundred blocks on a
// single address serialise at the memory-side atomic unit.  `round` counts the
// barriers completed including this one; counter x has seen round * n_x arrivals
// (n_x = blocks with index = x mod 8) when all blocks have arrived.  One wave
// polls all eight counters with one load per lane.  The counters are zeroed
// before the launch.
constexpr int kBarStride = 16;  // uints between arrival counters
GAP_DEV void grid_barrier_x8(unsigned int* arrive, unsigned int round, int* dev_err) {
  wait_mem();  // this wave's cross-block stores (device-scope atomics) have completed
  __syncthreads();
  if (threadIdx.x < 64) {
    const unsigned G = gridDim.x;
    if (threadIdx.x == 0)
      __hip_atomic_fetch_add(arrive + (blockIdx.x & 7) * kBarStride, 1u, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    const unsigned x = threadIdx.x & 7;
    const unsigned target = round * (G > x ? (G - x + 7) / 8 : 0u);
    uint64_t spins = 0;
    // Bounded wait: a barrier that does not complete within ~0.2 s sets the
    // error bit, and a set bit (checked every 64 polls) ends every later wait at
    // once, so a failed co-residency assumption costs one timeout, never a hang.
    for (;;) {
      const unsigned c =
          __hip_atomic_load(arrive + x * kBarStride, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
      if (__all(c >= target)) break;
      if ((spins & 63) == 63 &&
          (__hip_atomic_load(dev_err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
           GAP_DEVERR_SYNC))
        break;
      __builtin_amdgcn_s_sleep(1);
      if (++spins > (1ull << 22)) {
        if (threadIdx.x == 0) atomicOr(dev_err, GAP_DEVERR_SYNC);
        break;
      }
    }
  }
  __syncthreads();
}

// ------------------------------------------------------ 64-column panels ----
// P (rows j0 .. m - 1 of bw <= 64 columns) = Q R by Cholesky QR, twice, and the
// Householder vectors of that factorisation from Q (Ballard et al., Euro-Par /
// IPDPS 2014, "Reconstructing Householder vectors from Tall-Skinny QR"):
//   G1 = P^T P = R1^T R1, Q <- P R1^-1;  G2 = Q^T Q = R2^T R2, Q^ = Q R2^-1;
//   Q^ - [S; 0] = V U with V unit lower trapezoidal, U upper triangular and the
//   signs S_jj = -sign of the pivot's diagonal (LU without pivoting of the top
//   64 rows, |U_jj| >= 1), so that P = H [S R2 R1; 0], H = I - V T V^T,
//   T = -U S V1^-T (V1 the top block of V), tau_j = T_jj = -U_jj S_jj.
// The first pass leaves |Q^T Q - I| about cond(P)^2 u (columns scaled); while
// its entries are below 1/64 the second makes Q^ orthonormal to rounding, and the factors
// are as accurate as those of the column-by-column reduction (residual, Gram
// matrix and solutions agree with LAPACK's to rounding for condition numbers up
// to 1e12 over all columns).  A panel that fails the test (its columns dependent
// to about 1e-8, a zero column, an overflow) is left as it is and factored by
// k_qr_panel_dep.  One grid barrier and one reduction over blocks per column, as
// in the register-resident reduction this replaces, cost 6.8 us a column at
// 26,000 rows and 9.7 us at 353,000 (0.43 and 0.62 ms per 64 columns, and 0.13
// and 0.34 ms more for the updates between its 16-column steps); this takes
// 0.11 and 0.32 ms, at the small end the latency of its one-block steps
// (k_panel_vectors 45 us, k_panel_chol 16 us), at the large end the passes over
// the panel.
constexpr int kGramTiles = 10;                // lower 16 x 16 tiles of a 64 x 64 Gram
constexpr int kGram = kGramTiles * 256;       // their values
constexpr int kGramMaxBlocks = 256;
// What the panel kernels keep between launches (doubles).
constexpr int kInv16 = 4 * 256;               // inverses of a triangle's 16 x 16 diagonal blocks
constexpr int kPanU1 = 0;                     // R1, row-major upper, 64 x 64
constexpr int kPanInv1 = kPanU1 + 4096;
constexpr int kPanZ = kPanInv1 + kInv16;      // U R2, row-major upper
constexpr int kPanInvZ = kPanZ + 4096;
constexpr int kPanV1 = kPanInvZ + kInv16;     // V's top block transposed, row-major upper
constexpr int kPanInvV = kPanV1 + 4096;
constexpr int kPanUS = kPanInvV + kInv16;     // -U S, col-major
constexpr int kPanG = kPanUS + 4096;          // reduced Gram
constexpr int kPanDoubles = kPanG + kGram;

// Gram of up to 64 columns (col-major, rows 16-byte groups aligned) over the
// 16-row chunks c, c + nw, ...: a lane holds four consecutive rows of its column of
// each 16-column tile, which serve as both operands.
GAP_DEV void gram_chunks(const double* __restrict__ P, int64_t ld, int64_t rows, int bw, int64_t c,
                         int64_t nw, d4v (&acc)[kGramTiles],
                         int lane = threadIdx.x & 63) {
  const int g = lane >> 4, idx = lane & 15;
  const double* col[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) col[u] = P + (int64_t)min(16 * u + idx, bw - 1) * ld + 4 * g;
#pragma unroll
  for (int t = 0; t < kGramTiles; ++t) acc[t] = zero4();
  const int64_t nch = (rows + 15) / 16, full = rows / 16;
  auto products = [&](const d4v (&a)[4]) {
    int t = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j, ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t] = mfma_f64(a[i][q], a[j][q], acc[t]);
  };
  d4v cur[4], nxt[4];
  if (c < full) {
#pragma unroll
    for (int u = 0; u < 4; ++u) cur[u] = *reinterpret_cast<const d4v*>(col[u] + 16 * c);
    for (; c < full; c += nw) {
      const int64_t cn = c + nw < full ? c + nw : c;
#pragma unroll
      for (int u = 0; u < 4; ++u) nxt[u] = *reinterpret_cast<const d4v*>(col[u] + 16 * cn);
      __builtin_amdgcn_sched_barrier(0);
      products(cur);
#pragma unroll
      for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
    }
  }
  if (c < nch) {  // the last, partial chunk
    const int64_t left = rows - 16 * c - 4 * g;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) cur[u][q] = q < left ? col[u][16 * c + q] : 0.0;
    products(cur);
  }
}

// Sum of the block's four waves' Grams, in wave order, handed to put(e, value) by wave 0.
template <class FP>
GAP_DEV void gram_block_sum(const d4v (&acc)[kGramTiles], double* red, FP put,
                            int lane = threadIdx.x & 63) {
  const int wave = threadIdx.x >> 6;
  if (wave > 0) {
#pragma unroll
    for (int t = 0; t < kGramTiles; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[(wave - 1) * kGram + t * 256 + q * 64 + lane] = acc[t][q];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int t = 0; t < kGramTiles; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = t * 256 + q * 64 + lane;
        put(e, ((acc[t][q] + red[e]) + red[kGram + e]) + red[2 * kGram + e]);
      }
  }
}

__global__ __launch_bounds__(256) void k_panel_gram(const double* __restrict__ P, int64_t ld,
                                                    int64_t rows, int bw,
                                                    double* __restrict__ part) {
  __shared__ double red[3 * kGram];
  d4v acc[kGramTiles];
  gram_chunks(P, ld, rows, bw, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6),
              (int64_t)gridDim.x * 4, acc);
  gram_block_sum(acc, red,
                 [&](int e, double v) { part[(int64_t)blockIdx.x * kGram + e] = v; });
}

// The reduced Gram (value e of gram_block_sum's layout: load(e)) into the lower
// triangle of S, with unit columns from bw on.  Returns whether this thread saw an
// entry further than `far` from the unit matrix (or not a number).
template <class FL>
GAP_DEV bool gram_to_lds(FL load, int bw, double (*S)[kTriS], double far,
                         int tid = threadIdx.x) {
  bool off = false;
  double v[kGramTiles];
#pragma unroll
  for (int t = 0; t < kGramTiles; ++t) v[t] = load(256 * t + tid);
#pragma unroll
  for (int t = 0; t < kGramTiles; ++t) {
    const int q = (tid >> 6) & 3, lane = tid & 63;
    const int i = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3, j = t - i * (i + 1) / 2;
    const int r = 16 * i + (lane >> 4) + 4 * q, c = 16 * j + (lane & 15);
    const double unit = r == c ? 1.0 : 0.0;
    if (r >= c) {
      S[r][c] = r < bw ? v[t] : unit;
      off |= r < bw && !(fabs(v[t] - unit) < far);
    }
  }
  return off;
}

// R1 of the first Gram; sets the panel's state word (state[half], also set where
// the outer block's first panel is) and clears the barrier counters of
// k_qr_panel_dep.
__global__ __launch_bounds__(256) void k_panel_chol(int bw, int half, double* __restrict__ pan,
                                                    unsigned int* __restrict__ state,
                                                    unsigned int* __restrict__ arrive) {
  __shared__ double S[kTri][kTriS];
  (void)gram_to_lds([&](int e) { return pan[kPanG + e]; }, bw, S, INFINITY);
  __syncthreads();
  const bool bad = chol64_lds(S, (bw + 15) / 16);
  if (threadIdx.x == 0) state[half] = bad || (half && state[0]) ? 1u : 0u;
  if (threadIdx.x < kPanelBarWords) arrive[threadIdx.x] = 0u;
  for (int e = threadIdx.x; e < kTri * kTri; e += 256) {
    const int c = e >> 6, q = e & 63;  // U1[c][q] = L[q][c]
    pan[kPanU1 + e] = q >= c ? S[q][c] : 0.0;
  }
  if (threadIdx.x < 64) tri_inv16([&](int i, int j) { return S[j][i]; }, pan + kPanInv1);
}

// dst <- src U^-1 (both col-major, `bw` <= 64 columns), sixteen rows per wave at
// a time with U (row-major) and the inverses of its diagonal blocks held as
// operands in registers.  Blocks from na on take problem b.  Bound by the panel's
// traffic where it has many rows; a row per lane with U broadcast from LDS took
// 132 us at 349,000 rows (this one 94) and 18 us at 6,000 (12).
struct PanelSolve {
  const double* src;
  int64_t lds;
  double* dst;
  int64_t ldd, rows;
  int bw;
  const double *u, *inv;
};
// Tiles tile, tile + step, ... of sixteen rows; u(i, j) and inv(e): the triangle.
template <class FU, class FI>
GAP_DEV void solve_tiles(const PanelSolve& p, FU u, FI inv, int64_t tile, int64_t step,
                         int lane = threadIdx.x & 63) {
  const int g = lane >> 4, idx = lane & 15;
  const int64_t nt = (p.rows + 15) / 16;
  if (tile >= nt) return;
  // columns 16 b + g + 4 r of row 16 tile + idx (past the last row: that row again,
  // which stores the same values)
  auto load = [&](int64_t ti, d4v (&x)[4]) {
    const double* row = p.src + min(16 * ti + idx, p.rows - 1);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[b][r] = row[(int64_t)min(16 * b + g + 4 * r, p.bw - 1) * p.lds];
  };
  d4v cur[4], nxt[4];
  load(tile, cur);
  TriOps t;
  tri_ops(t, u, inv, lane);
  for (; tile < nt; tile += step) {
    load(min(tile + step, nt - 1), nxt);
    __builtin_amdgcn_sched_barrier(0);
    d4v x[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[b][r] = 16 * b + g + 4 * r < p.bw ? cur[b][r] : 0.0;
    tri_solve16(t, x);
    double* row = p.dst + min(16 * tile + idx, p.rows - 1);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = 16 * b + g + 4 * r;
        if (c < p.bw) row[c * p.ldd] = x[b][r];
        cur[b][r] = nxt[b][r];
      }
  }
}
constexpr int kSolveBlocks = 512;  // of four waves: two per SIMD
__global__ __launch_bounds__(256, 2) void k_panel_solve(PanelSolve pa, PanelSolve pb, int na,
                                                        const unsigned int* __restrict__ state) {
  if (*state) return;
  const bool second = (int)blockIdx.x >= na;
  const PanelSolve p = second ? pb : pa;
  solve_tiles(p, [&](int i, int j) { return p.u[i * kTri + j]; },
              [&](int e) { return p.inv[e]; },
              (int64_t)(second ? blockIdx.x - na : blockIdx.x) * 4 + (threadIdx.x >> 6),
              (int64_t)(second ? gridDim.x - na : na) * 4);
}

// LU without pivoting of B - diag(sg) for B (64 x 64, in LDS), sg_j = -sign of
// the pivot: U in and above the diagonal, unit L below.  256 threads, nb steps
// of 16 columns (zero columns of B from 16 nb on: U is 1 there): one wave factors them with a row per lane, then solves the
// rows to their right with a column per lane; the four waves update the rest.
GAP_DEV void lu64_signs(double (*B)[kTriS], double* sg, int nb, int lane) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, idx = lane & 15;
  if (wave == 1 && lane >= 16 * nb) {
    B[lane][lane] = 1.0;
    sg[lane] = -1.0;
  }
  for (int s = 0; s < nb; ++s) {
    const int c0 = 16 * s;
    if (wave == 0) {
      double v[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = B[lane][c0 + c];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const double p = readlane_f64(v[c], c0 + c);
        const double sign = p >= 0.0 ? -1.0 : 1.0;
        const double piv = p - sign;
        const double l = v[c] * rcp_f64(piv);
        v[c] = lane == c0 + c ? piv : (lane > c0 + c ? l : v[c]);
        const double lv = lane > c0 + c ? l : 0.0;
#pragma unroll
        for (int q = c + 1; q < 16; ++q) v[q] -= lv * readlane_f64(v[q], c0 + c);
        if (lane == 0) sg[c0 + c] = sign;
      }
      if (lane >= c0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) B[lane][c0 + c] = v[c];
      }
    }
    __syncthreads();
    if (wave == 0 && s + 1 < nb) {  // U12 = L11^-1 B12, a column per lane
      const int col = min(c0 + 16 + lane, kTri - 1);
      double y[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) y[i] = B[c0 + i][col];
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int k = i + 1; k < 16; ++k) y[k] -= B[c0 + k][c0 + i] * y[i];
      if (c0 + 16 + lane < kTri) {
#pragma unroll
        for (int i = 1; i < 16; ++i) B[c0 + i][col] = y[i];
      }
    }
    __syncthreads();
    int t = 0;
    for (int ti = s + 1; ti < 4; ++ti)
      for (int tj = s + 1; tj < nb; ++tj, ++t) {
        if ((t & 3) != wave) continue;
        d4v acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = B[16 * ti + g + 4 * r][16 * tj + idx];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc = mfma_f64(-B[16 * ti + idx][c0 + 4 * g + q], B[c0 + 4 * g + q][16 * tj + idx], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) B[16 * ti + g + 4 * r][16 * tj + idx] = acc[r];
      }
    __syncthreads();
  }
}

// Upper triangle of the product of two upper triangles given by element
// functions a(i, k) (i <= k) and b(k, j) (k <= j), handed to put(i, j, value)
// for every i <= j; 256 threads.
template <class FA, class FB, class FP>
GAP_DEV void upper_product64(FA a, FB b, FP put, int lane) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, idx = lane & 15;
  int t = 0;
  for (int ti = 0; ti < 4; ++ti)
    for (int tj = ti; tj < 4; ++tj, ++t) {
      if ((t & 3) != wave) continue;
      d4v acc = zero4();
      for (int tk = ti; tk <= tj; ++tk)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = 16 * ti + idx, k = 16 * tk + 4 * g + q, j = 16 * tj + idx;
          acc = mfma_f64(i <= k ? a(i, k) : 0.0, k <= j ? b(k, j) : 0.0, acc);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + g + 4 * r, j = 16 * tj + idx;
        if (i <= j) put(i, j, acc[r]);
      }
    }
}

// LDS of a panel's middle.
struct PanelLds {
  double S[kTri][kTriS], B[kTri][kTriS];
  __attribute__((aligned(16))) double u[kTri * kTri], u1[kTri * kTri];
  double inv[kInv16];
  double sg[kTri];
};

// The middle of the panel, by a workgroup: R2 from the second Gram (in S), the
// signs and L, U of Q^'s top rows (Q's in x: sixteen per wave, columns 16 b + g +
// 4 r of row idx), and from them R in A (if `out`) and Z = U R2 in S and put_z
// (V's other rows are q Z^-1).  put_u1 stores R1 in u1.  Leaves L and U in B and
// the signs in sg.
template <class FP, class FZ>
GAP_DEV void panel_middle(PanelLds& s, d4v (&x)[4], FP put_u1, FZ put_z, double* __restrict__ A,
                          int64_t ld, int64_t rows, int bw, bool out, int lane = threadIdx.x & 63) {
  const int wave = threadIdx.x >> 6, g = lane >> 4, idx = lane & 15;
  const int64_t qr = 16 * wave + idx;
  const int nb = (bw + 15) / 16;
  (void)chol64_lds(s.S, nb, lane);  // diagonally dominant: no bad pivot
  if (wave == 0) {
    tri_inv16([&](int i, int j) { return s.S[j][i]; }, s.inv, lane);
  } else {
    for (int e = 64 * (wave - 1) + lane; e < kTri * kTri; e += 192) {
      const int c = e >> 6, q = e & 63;
      s.u[e] = q >= c ? s.S[q][c] : 0.0;  // R2
    }
  }
  put_u1();
  __syncthreads();
  {  // Q^'s top rows
    TriOps t;
    tri_ops(t, [&](int i, int j) { return s.u[i * kTri + j]; }, [&](int e) { return s.inv[e]; },
            lane);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        x[b][r] = 16 * b + g + 4 * r < bw && qr < rows ? x[b][r] : 0.0;
    tri_solve16(t, x);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) s.B[qr][16 * b + g + 4 * r] = x[b][r];
  }
  __syncthreads();
  lu64_signs(s.B, s.sg, nb, lane);
  // R = S R2 R1 and Z = U R2 (S, the LDS array, is free for Z)
  if (out)
    upper_product64([&](int i, int k) { return s.u[i * kTri + k]; },
                    [&](int k, int j) { return s.u1[k * kTri + j]; },
                    [&](int i, int j, double v) {
                      if (j < bw) A[i + j * ld] = s.sg[i] * v;
                    },
                    lane);
  upper_product64([&](int i, int k) { return s.B[i][k]; },
                  [&](int k, int j) { return s.u[k * kTri + j]; },
                  [&](int i, int j, double v) {
                    put_z(i * kTri + j, v);
                    s.S[i][j] = v;
                  },
                  lane);
  __syncthreads();
}

// V's top rows (unit lower) into A, and tau, from the L and U that panel_middle left.
GAP_DEV void panel_top(const PanelLds& s, double* __restrict__ A, int64_t ld, int64_t rows, int bw,
                       double* __restrict__ tau) {
  if (threadIdx.x >= 192 && threadIdx.x - 192 < bw) {
    const int j = threadIdx.x - 192;
    tau[j] = -s.B[j][j] * s.sg[j];
  }
  for (int e = threadIdx.x; e < kTri * kTri; e += 256) {
    const int c = e >> 6, q = e & 63;
    if (q > c && q < rows && c < bw) A[q + c * ld] = s.B[q][c];
  }
}

// The one-block middle launch: the test that Q was near enough to orthonormal, then
// R, tau and V's top in A, and the operands of V's other rows and of T.  Bound by
// latency: 45 us, half of it the 64 columns of the Cholesky factor and the 64 of
// the LU.
__global__ __launch_bounds__(256) void k_panel_vectors(double* __restrict__ A, int64_t ld,
                                                       int64_t rows, int bw,
                                                       const double* __restrict__ Q, int64_t ldq,
                                                       double* __restrict__ pan,
                                                       double* __restrict__ tau,
                                                       unsigned int* __restrict__ state) {
  __shared__ PanelLds s;
  __shared__ int s_bad;
  if (*state) return;  // uniform: a whole-grid condition
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  if (threadIdx.x == 0) s_bad = 0;
  // Q's top rows, sixteen per wave, on their way while R2 is formed
  const int64_t qr = 16 * wave + idx;
  d4v x[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      x[b][r] = Q[(int64_t)min(16 * b + g + 4 * r, bw - 1) * ldq + min(qr, rows - 1)];
  d2v r1[8];  // this thread's share of R1
#pragma unroll
  for (int i = 0; i < 8; ++i)
    r1[i] = reinterpret_cast<const d2v*>(pan + kPanU1)[i * 256 + threadIdx.x];
  __syncthreads();  // s_bad
  if (gram_to_lds([&](int e) { return pan[kPanG + e]; }, bw, s.S, 1.0 / 64)) s_bad = 1;
  __syncthreads();
  if (s_bad) {
    if (threadIdx.x == 0) *state = 1u;
    return;
  }
  panel_middle(
      s, x,
      [&] {
#pragma unroll
        for (int i = 0; i < 8; ++i) reinterpret_cast<d2v*>(s.u1)[i * 256 + threadIdx.x] = r1[i];
      },
      [&](int e, double v) { pan[kPanZ + e] = v; }, A, ld, rows, bw, true);
  if (wave == 0) tri_inv16([&](int i, int j) { return s.S[i][j]; }, pan + kPanInvZ);
  if (wave == 1) tri_inv16([&](int i, int j) { return i == j ? 1.0 : s.B[j][i]; }, pan + kPanInvV);
  // (the waves at an inverse join when it is done) and T = (-U S) V1^-T: the rows of
  // -U S and V1^T for its solution
  panel_top(s, A, ld, rows, bw, tau);
  for (int e = threadIdx.x; e < kTri * kTri; e += 256) {
    const int c = e >> 6, q = e & 63;
    pan[kPanV1 + e] = q > c ? s.B[q][c] : (q == c ? 1.0 : 0.0);
    pan[kPanUS + e] = q <= c ? -s.B[q][c] * s.sg[c] : 0.0;
  }
}

// ---------------------------------------------- numerically dependent panels ----
// k_qr_panel_dep factors an outer block's columns from its first panel on whose
// state word is set (state[h]: panel h of 64 columns; the launch ends at once if
// neither is).  Nothing of the block was written after that panel, so its other
// panel is taken along.  A cooperative grid (it also runs as a single ordinary
// block) that does what the panel kernels do, with more rounds of Cholesky QR, shifted
// (Fukaya, Kannan, Nakatsukasa, Yamamoto, Yanagisawa, SIAM J. Sci. Comput. 2020):
//   G = X^T X, R = chol(G + kDepShift diag(G)), X <- X R^-1,
// from X = P until G is within 1/64 of the unit matrix.  The shift keeps the Cholesky
// factor defined whatever the columns (the Gram's own rounding is below it) and X's
// columns at most of length one, so a round lengthens what is left of a column
// outside the span of the others by up to 1 / sqrt(kDepShift) = 3e6 and adds
// a column-wise error of rounding size: two rounds for columns that depend up to
// 1e-9, or equal ones (whose rounding errors the rounds lengthen, as the
// column-by-column reduction does); at most three were seen.  Where that fails (a
// zero column, columns equal in a way that leaves no rounding error, an overflow)
// panel_columns goes through the rest of the block column by column.
// A 64-row group of the block belongs to one workgroup for the whole kernel, and
// a 16-row tile to one wave except in panel_columns, so no row passes from one
// workgroup to another; Grams, Q's top rows and V^T C go by device-scope atomics, and
// every workgroup forms the small factors for itself.
// A fit of 88,000 rows and 2,000 points with equal points in every 128: 330 ms when
// such blocks went column by column alone (a pass over up to 128 columns and a grid
// barrier per column), 29.2 now, 22.9 without equal points; 5,600 rows and 300
// points: 20.6, 2.1 and 1.4.  (48 and 5.1 with every panel by a reduction of sixteen
// columns in registers.)  Bound by the latency of its grid barriers and of the one-
// block steps each round repeats.
constexpr int kColT = 256;
constexpr double kDepShift = 0x1p-43;
constexpr int kDepRounds = 5;

struct DepArgs {
  double* A;  // the outer block at its diagonal, col-major
  int64_t ld, rows;
  int ow;     // its columns
  double* Q;  // [64][ldq]
  int64_t ldq;
  double* part;  // [grid][4096] partial sums
  double* pan;
  double *red, *piv;  // of panel_columns
  unsigned int* arrive;
  const unsigned int* state;
  double* tau;
  int* dev_err;
};

// Columns k0 .. ow - 1 one by one: per column one pass over the rows for each group
// of 64 columns, which applies the previous reflector and accumulates the norm and
// dot products of the next, then one grid barrier (`bar`: those completed).
GAP_DEV void panel_columns(const DepArgs& d, int k0, unsigned bar) {
  __shared__ double s_wred[kColT / 64][kTri];
  __shared__ double s_tw[2 * kTri], s_pv[2 * kTri], s_tot[2 * kTri];
  __shared__ double s_par[3];  // tau, beta, scale of the reflector just formed
  const int G = gridDim.x, wave = threadIdx.x >> 6, lane = fresh_lane(), ow = d.ow;
  const int64_t ld = fresh(d.ld);
  for (int k = k0; k <= ow; ++k) {
    double* rb = d.red + (size_t)(k & 1) * 2 * kTri * kPanelMaxGrid;
    double* pv = d.piv + (k & 1) * 2 * kTri;
    const int p = k > k0 ? k - 1 : k;  // first column this pass touches
    for (int o = p / kTri * kTri; o < ow; o += kTri) {
      double part[kTri];
#pragma unroll
      for (int j = 0; j < kTri; ++j) part[j] = 0.0;
      for (int64_t r = ((int64_t)blockIdx.x + (int64_t)G * wave) * 64 + lane; r < d.rows;
           r += (int64_t)G * kColT) {
        if (r < p) continue;
        double* row = d.A + r;
        double a[kTri];
#pragma unroll
        for (int j = 0; j < kTri; ++j) a[j] = (o + j >= p && o + j < ow) ? row[(o + j) * ld] : 0.0;
        if (k > k0) {  // reflector p = k - 1, whose v an earlier group has stored
          double v = r == p ? 1.0 : 0.0;
          if (p >= o) {
#pragma unroll
            for (int j = 0; j < kTri; ++j)
              if (o + j == p) {
                v = r == p ? 1.0 : a[j] * s_par[2];
                row[p * ld] = r == p ? s_par[1] : v;
              }
          } else if (r > p) {
            v = row[p * ld];
          }
#pragma unroll
          for (int j = 0; j < kTri; ++j)
            if (o + j >= k && o + j < ow) {
              a[j] -= s_tw[o + j] * v;
              row[(o + j) * ld] = a[j];
            }
        }
        if (k < ow && r == k) {
#pragma unroll
          for (int j = 0; j < kTri; ++j)
            if (o + j >= k && o + j < ow) xstore(pv + o + j, a[j]);
        } else if (k < ow && r > k && k < o + kTri) {
          const double ak = row[k * ld];  // (stored above, or by an earlier group)
#pragma unroll
          for (int j = 0; j < kTri; ++j) part[j] += ak * a[j];
        }
      }
      if (k == ow || o + kTri <= k) continue;  // uniform
#pragma unroll
      for (int j = 0; j < kTri; ++j) {
        const double t = wave_sum(part[j]);
        if (lane == 0) s_wred[wave][j] = t;
      }
      __syncthreads();
      if (threadIdx.x < kTri) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kColT / 64; ++w) t += s_wred[w][threadIdx.x];
        xstore(rb + (o + threadIdx.x) * kPanelMaxGrid + blockIdx.x, t);
      }
      __syncthreads();
    }
    if (k == ow) break;
    grid_barrier_x8(d.arrive, ++bar, d.dev_err);
    if (threadIdx.x >= k && threadIdx.x < ow) {
      double t = 0.0;
      for (int b = 0; b < G; ++b) t += vload(rb + threadIdx.x * kPanelMaxGrid + b);
      s_tot[threadIdx.x] = t;
      s_pv[threadIdx.x] = vload(pv + threadIdx.x);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const double alpha = s_pv[k], xnorm = sqrt(s_tot[k]);
      double tau = 0.0, beta = alpha, scale = 0.0;
      if (xnorm > 0.0) {
        beta = -copysign(hypot(alpha, xnorm), alpha);
        tau = (beta - alpha) / beta;
        scale = 1.0 / (alpha - beta);
      }
      s_par[0] = tau;
      s_par[1] = beta;
      s_par[2] = scale;
      if (blockIdx.x == 0) d.tau[k] = tau;
    }
    __syncthreads();
    if (threadIdx.x < ow) {
      const int j = threadIdx.x;
      s_tw[j] = j > k ? s_par[0] * (s_pv[j] + s_par[2] * s_tot[j]) : 0.0;
    }
    __syncthreads();
  }
}

// tot[e] = sum over the grid's blocks of part[block][e], e < n, in a fixed order: the
// blocks share the sums, sixteen lanes each.  Between two grid barriers.
GAP_DEV void grid_sum(const double* part, int n, double* tot) {
  const int G = gridDim.x, l = threadIdx.x & 15;
  for (int e = blockIdx.x + G * (threadIdx.x >> 4); e < n; e += G * (kColT / 16)) {
    double t = 0.0;
#pragma unroll 8
    for (int b = l; b < G; b += 16) t += vload(part + (int64_t)b * n + e);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) t += __shfl_xor(t, o);
    if (l == 0) xstore(tot + e, t);
  }
}

// C -= V T^T V^T C for the cw columns C after a full first panel: V in A (unit lower
// trapezoidal), T (row-major) in s.u, s.u1 free.  Tiles tile0, tile0 + nw, ... are
// this wave's.
GAP_DEV void dep_update(const DepArgs& d, PanelLds& s, int cw, int64_t tile0, int64_t nw,
                        unsigned& bar) {
  const int wave = threadIdx.x >> 6, lane = fresh_lane(), g = lane >> 4, idx = lane & 15;
  const int64_t nt = (d.rows + 15) / 16, ld = fresh(d.ld);
  double* C = d.A + kTri * ld;
  auto unit_lower = [](int64_t r, int c, double v) { return r == c ? 1.0 : (r > c ? v : 0.0); };
  // W = V^T C: lane (g, idx) holds rows 4 g .. + 3 of a tile's columns 16 u + idx
  d4v w[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) w[i][j] = zero4();
  for (int64_t t = tile0; t < nt; t += nw) {
    const int64_t r0 = 16 * t + 4 * g;
    d4v v[4], c[4];
    if (16 * t + 16 <= d.rows) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = *reinterpret_cast<const d4v*>(d.A + r0 + (16 * u + idx) * ld);
        c[u] = *reinterpret_cast<const d4v*>(C + r0 + min(16 * u + idx, cw - 1) * ld);
      }
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t r = min(r0 + q, d.rows - 1);
          v[u][q] = r0 + q < d.rows ? d.A[r + (16 * u + idx) * ld] : 0.0;
          c[u][q] = r0 + q < d.rows ? C[r + min(16 * u + idx, cw - 1) * ld] : 0.0;
        }
    }
    if (t < 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) v[u][q] = unit_lower(r0 + q, 16 * u + idx, v[u][q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) w[i][j] = mfma_f64(v[i][q], c[j][q], w[i][j]);
  }
  for (int k = 0; k < 4; ++k) {  // the waves in turn
    if (wave == k) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double* p = s.u1 + ((i * 4 + j) * 4 + r) * 64 + lane;
            *p = k ? *p + w[i][j][r] : w[i][j][r];
          }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < kTri * kTri; e += kColT)
    xstore(d.part + (int64_t)blockIdx.x * kTri * kTri + e, s.u1[e]);
  grid_barrier_x8(d.arrive, ++bar, d.dev_err);
  grid_sum(d.part, kTri * kTri, d.pan + kPanZ);
  grid_barrier_x8(d.arrive, ++bar, d.dev_err);
  {  // Wt = -T^T W in s.u1, row-major: columns 16 wave .. + 15
    d4v x[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        x[t][r] = vload(d.pan + kPanZ + ((t * 4 + wave) * 4 + r) * 64 + lane);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      d4v y = zero4();
#pragma unroll
      for (int t = 0; t <= u; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          y = mfma_f64(-s.u[(16 * t + g + 4 * r) * kTri + 16 * u + idx], x[t][r], y);
#pragma unroll
      for (int r = 0; r < 4; ++r) s.u1[(16 * u + g + 4 * r) * kTri + 16 * wave + idx] = y[r];
    }
  }
  __syncthreads();
  // C += V Wt: lane (g, idx) holds columns 16 b + g + 4 r of row idx (past the last
  // row: that row again, which stores the same values)
  for (int64_t t = tile0; t < nt; t += nw) {
    const int64_t row = min(16 * t + idx, d.rows - 1);
    d4v v[4], c[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = 16 * b + g + 4 * r;
        v[b][r] = unit_lower(row, k, d.A[row + k * ld]);
        c[b][r] = C[row + min(k, cw - 1) * ld];
      }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          c[b] = mfma_f64(s.u1[(16 * kb + g + 4 * r) * kTri + 16 * b + idx], v[kb][r], c[b]);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = 16 * b + g + 4 * r;
        if (k < cw) C[row + k * ld] = c[b][r];
      }
  }
  __syncthreads();
}

__global__ __launch_bounds__(kColT) void k_qr_panel_dep(DepArgs d) {
  const bool first = d.state[0] != 0u;
  if (!first && (d.ow <= kTri || d.state[1] == 0u)) return;
  __shared__ PanelLds s;
  __shared__ double inv_v[kInv16];
  __shared__ int s_flag;
  const int wave = threadIdx.x >> 6;
  const int64_t nw = (int64_t)gridDim.x * 4;
  // this wave's first tile of sixteen rows from tile `lo` on (its tiles: step nw)
  auto my_tile = [&](int lo) {
    int64_t t = (int64_t)blockIdx.x * 4 + wave;
    while (t < lo) t += nw;
    return t;
  };
  // `v` of any thread, in all threads of the block
  auto any_of = [&](bool v) {
    __syncthreads();
    if (threadIdx.x == 0) s_flag = 0;
    __syncthreads();
    if (v) s_flag = 1;
    __syncthreads();
    return s_flag != 0;
  };
  unsigned bar = 0;
  for (int h = first ? 0 : 1; h * kTri < d.ow; ++h) {
    const int bw = min(kTri, d.ow - h * kTri);
    double* P = d.A + (int64_t)h * kTri * d.ld;          // the panel's columns, block rows
    const bool owner = (int)blockIdx.x == h % (int)gridDim.x;  // of its top 64 rows
    double *tot = d.pan + kPanG, *top = d.pan + kPanV1;
    for (int round = 0;; ++round) {
      const double* X = round ? d.Q : P;
      const int64_t ldx = round ? d.ldq : d.ld;
      d4v acc[kGramTiles];
      gram_chunks(fresh(X), fresh(ldx), d.rows, bw, my_tile(4 * h), nw, acc,
                  fresh_lane());
      gram_block_sum(acc, &s.S[0][0], [&](int e, double v) {  // (S and B)
        xstore(d.part + (int64_t)blockIdx.x * kGram + e, v);
      }, fresh_lane());
      grid_barrier_x8(d.arrive, ++bar, d.dev_err);
      grid_sum(d.part, kGram, tot);
      grid_barrier_x8(d.arrive, ++bar, d.dev_err);
      const bool far = any_of(gram_to_lds([&](int e) { return vload(tot + e); }, bw, s.S, 1.0 / 64,
                                          fresh_thread()));
      if (round > 0 && !far) break;
      if (threadIdx.x < kTri) s.S[threadIdx.x][threadIdx.x] *= 1.0 + kDepShift;
      __syncthreads();
      const bool bad = chol64_lds(s.S, (bw + 15) / 16, fresh_lane());
      if (any_of(threadIdx.x == 0 && bad) || round == kDepRounds) {
        panel_columns(d, h * kTri, bar);
        return;
      }
      if (wave == 0) tri_inv16([&](int i, int j) { return s.S[j][i]; }, s.inv, fresh_lane());
      // the product of the rounds' factors
      if (round > 0) {
        upper_product64([&](int i, int k) { return s.S[k][i]; },
                        [&](int k, int j) { return s.u1[k * kTri + j]; },
                        [&](int i, int j, double v) { s.u[i * kTri + j] = v; }, fresh_lane());
        __syncthreads();
      }
      for (int e = fresh_thread(); e < kTri * kTri; e += kColT) {
        const int i = e >> 6, j = e & 63;
        s.u1[e] = i > j ? 0.0 : (round ? s.u[e] : s.S[j][i]);
      }
      __syncthreads();
      const PanelSolve q{fresh(X), fresh(ldx), fresh(d.Q), fresh(d.ldq), d.rows, fresh(bw), nullptr, nullptr};
      solve_tiles(q, [&](int i, int j) { return s.S[j][i]; }, [&](int e) { return s.inv[e]; },
                  my_tile(4 * h), nw, fresh_lane());
      if (owner) {  // Q's top rows, this wave's own
        const int lane = fresh_lane(), g = lane >> 4, idx = lane & 15;
        const int64_t row = h * kTri + 16 * wave + idx;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int c = 16 * b + g + 4 * r;
            xstore(top + (16 * wave + idx) * kTri + c,
                   d.Q[min(c, bw - 1) * d.ldq + min(row, d.rows - 1)]);
          }
      }
      __syncthreads();  // S is read no more
    }
    const int lane = fresh_lane(), g = lane >> 4, idx = lane & 15;
    d4v x[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        x[b][r] = vload(top + (16 * wave + idx) * kTri + 16 * b + g + 4 * r);
    double* Ad = P + h * kTri;  // at the panel's diagonal
    const int64_t rows_h = d.rows - h * kTri;
    panel_middle(s, x, [] {}, [](int, double) {}, Ad, d.ld, rows_h, bw, owner, lane);
    if (wave == 0) tri_inv16([&](int i, int j) { return s.S[i][j]; }, s.inv, lane);
    if (wave == 1)
      tri_inv16([&](int i, int j) { return i == j ? 1.0 : s.B[j][i]; }, inv_v, lane);
    if (owner) panel_top(s, Ad, d.ld, rows_h, bw, d.tau + h * kTri);
    __syncthreads();
    const PanelSolve v{fresh(d.Q), fresh(d.ldq), fresh(P), fresh(d.ld), d.rows, fresh(bw), nullptr, nullptr};
    solve_tiles(v, [&](int i, int j) { return s.S[i][j]; }, [&](int e) { return s.inv[e]; },
                my_tile(4 * (h + 1)), nw, fresh_lane());
    const int cw = d.ow - (h + 1) * kTri;
    if (cw <= 0) continue;
    {  // T = (-U S) V1^-T in u (the launch after this one forms it from V and tau)
      const int row = 16 * wave + idx;
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = 16 * b + g + 4 * r;
          x[b][r] = row <= c ? -s.B[row][c] * s.sg[c] : 0.0;
        }
      TriOps t;
      tri_ops(t, [&](int i, int j) { return i == j ? 1.0 : s.B[j][i]; },
              [&](int e) { return inv_v[e]; }, lane);
      tri_solve16(t, x);
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) s.u[row * kTri + 16 * b + g + 4 * r] = x[b][r];
    }
    __syncthreads();
    dep_update(d, s, cw, my_tile(0), nw, bar);
  }
}

// ------------------------------------------------------- narrow blocks ----
// Householder factorisation of an outer block of width <= kRRW with the whole
// panel held in registers across a cooperative grid: thread t of block b owns
// the panel rows (b * 512 + t) + q * (grid * 512), q < kRRQ.  Every column
// step applies the previous reflector to the thread's rows, forms per-block
// partial sums of the next column's norm and dot products, publishes them, and
// waits at a grid barrier; every block then reduces all partials in the same
// fixed order, so all blocks derive identical reflector parameters without a
// second barrier.  Partials alternate between two buffers so a block that is
// one step ahead never overwrites values a slower block is still reading.
// For a block this narrow the eight launches of a 64-column panel and its one-block
// steps of 64 columns cost more (four columns, 600 rows: 94 us of kernels against 25;
// 400,000 rows: 290 against 41; a least-squares call of 60 rows 242 against 170).
static_assert(kPanelMaxGrid <= 256, "the panel reduction reads at most 4 partials per lane");
constexpr int kRRW = 16;    // panel width
constexpr int kRRQ = 4;     // rows per thread
constexpr int kRRT = 512;   // threads per block
static_assert(kRRW == 16, "the panel's wave reduction is a 16-value butterfly");
__global__ __launch_bounds__(kRRT) void k_qr_panel_rr(double* __restrict__ A, int64_t ld,
                                                      int64_t m, int pw,
                                                      double* __restrict__ red,
                                                      double* __restrict__ piv,
                                                      unsigned int* __restrict__ arrive,
                                                      double* __restrict__ tau_all,
                                                      unsigned int* __restrict__ state,
                                                      int* __restrict__ dev_err) {
  __shared__ double s_wred[kRRT / 64][kRRW];
  __shared__ double s_tot[kRRW];
  __shared__ double s_tw[kRRW];
  __shared__ double s_par[3];  // tau, beta, scale of the reflector just formed
  __shared__ double s_pv[kRRW];  // the pivot row of the current column
  const int G = gridDim.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)G * kRRT;
  int64_t lrow[kRRQ];  // row, or -1
  double a[kRRQ][kRRW];
#pragma unroll
  for (int q = 0; q < kRRQ; ++q) {
    const int64_t lr = (int64_t)blockIdx.x * kRRT + threadIdx.x + q * stride;
    lrow[q] = (lr < m) ? lr : -1;
#pragma unroll
    for (int j = 0; j < kRRW; ++j)
      a[q][j] = (lrow[q] >= 0 && j < pw) ? A[lr + j * ld] : 0.0;
  }
  double beta_p = 0.0, scale_p = 0.0;
  for (int k = 0; k <= pw; ++k) {
    // 1. apply reflector k-1 to rows >= k-1.  Register arrays are indexed by
    //    absolute column only (selects against k), never by a k-relative
    //    index, which would force them out of registers.  tw[j] is zero for
    //    j <= k-1, and v is zero on rows above the reflector, so the update
    //    needs no condition.
    if (k > 0) {
      double tw[kRRW];
#pragma unroll
      for (int j = 0; j < kRRW; ++j) tw[j] = s_tw[j];
#pragma unroll
      for (int q = 0; q < kRRQ; ++q) {
        const bool at = lrow[q] == k - 1, below = lrow[q] > k - 1;
        double ak1 = 0.0;
#pragma unroll
        for (int j = 0; j < kRRW; ++j) ak1 = (j == k - 1) ? a[q][j] : ak1;
        const double v = at ? 1.0 : (below ? ak1 * scale_p : 0.0);
        const double nk1 = at ? beta_p : (below ? v : ak1);
#pragma unroll
        for (int j = 0; j < kRRW; ++j) {
          a[q][j] = (j == k - 1) ? nk1 : a[q][j];
          a[q][j] -= tw[j] * v;
        }
      }
    }
    if (k == pw) break;
    // 2. partial sums for column k over rows > k, by absolute column:
    //    part[k] = sum a_k^2, part[j] = sum a_k a_j (j > k); pivot row published
    double part[kRRW];
#pragma unroll
    for (int j = 0; j < kRRW; ++j) part[j] = 0.0;
#pragma unroll
    for (int q = 0; q < kRRQ; ++q) {
      double ak = 0.0;
#pragma unroll
      for (int j = 0; j < kRRW; ++j) ak = (j == k) ? a[q][j] : ak;
      ak = (lrow[q] > k) ? ak : 0.0;
      // columns j < k are summed too (no select per register) and never used
#pragma unroll
      for (int j = 0; j < kRRW; ++j) part[j] += ak * a[q][j];
      if (lrow[q] == k) {
        double* pv = piv + (k & 1) * kRRW;
#pragma unroll
        for (int j = 0; j < kRRW; ++j) xstore(pv + j, a[q][j]);
      }
    }
    // wave sums of the 16 partials by a halving butterfly (17 lane exchanges
    // instead of 16 separate 6-step reductions): lane l ends with the total of
    // column 8 b5 + 4 b4 + 2 b3 + b2 of its lane bits
    {
      double t8[8], t4[4], t2[2], t1;
      const bool u5 = lane & 32, u4 = lane & 16, u3 = lane & 8, u2 = lane & 4;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        t8[i] = (u5 ? part[i + 8] : part[i]) + __shfl_xor(u5 ? part[i] : part[i + 8], 32);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        t4[i] = (u4 ? t8[i + 4] : t8[i]) + __shfl_xor(u4 ? t8[i] : t8[i + 4], 16);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        t2[i] = (u3 ? t4[i + 2] : t4[i]) + __shfl_xor(u3 ? t4[i] : t4[i + 2], 8);
      t1 = (u2 ? t2[1] : t2[0]) + __shfl_xor(u2 ? t2[0] : t2[1], 4);
      t1 += __shfl_xor(t1, 2);
      t1 += __shfl_xor(t1, 1);
      const int jj = (u5 ? 8 : 0) + (u4 ? 4 : 0) + (u3 ? 2 : 0) + (u2 ? 1 : 0);
      if ((lane & 3) == 0 && jj >= k && jj < pw) s_wred[wave][jj - k] = t1;
    }
    const int ncnt = pw - k;
    __syncthreads();
    double* rb = red + (size_t)(k & 1) * kRRW * G;
    if (threadIdx.x < ncnt) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kRRT / 64; ++w) s += s_wred[w][threadIdx.x];
      xstore(rb + (int64_t)threadIdx.x * G + blockIdx.x, s);
    }
    grid_barrier_x8(arrive, (unsigned)(k + 1), dev_err);
    // the pivot row, read together with the partials below (one round trip)
    const double* pv = piv + (k & 1) * kRRW;
    if (threadIdx.x < kRRW) s_pv[threadIdx.x] = vload(pv + threadIdx.x);
    // 3. every block reduces all partials in the same order.  A wave reads the
    //    G <= 256 partials of its two columns (wave, wave + 8) with all eight
    //    loads in flight together (clamped addresses, out-of-range ones scaled
    //    by zero), so the reads cost one memory round trip, not one per load.
    if (wave < ncnt) {
      const int v0 = wave, v1 = min(wave + kRRT / 64, ncnt - 1);
      double x0[4], x1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int b = min(lane + 64 * i, G - 1);
        x0[i] = vload(rb + (int64_t)v0 * G + b);
        x1[i] = vload(rb + (int64_t)v1 * G + b);
      }
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double w = (lane + 64 * i < G) ? 1.0 : 0.0;
        s0 += w * x0[i];
        s1 += w * x1[i];
      }
      s0 = wave_sum(s0);
      s1 = wave_sum(s1);
      if (lane == 0) {
        s_tot[v0] = s0;
        if (wave + kRRT / 64 < ncnt) s_tot[wave + kRRT / 64] = s1;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const double alpha = s_pv[k];
      const double xnorm = sqrt(s_tot[0]);
      double tau = 0.0, beta = alpha, scale = 0.0;
      if (xnorm > 0.0) {
        beta = -copysign(hypot(alpha, xnorm), alpha);
        tau = (beta - alpha) / beta;
        scale = 1.0 / (alpha - beta);
      }
      s_par[0] = tau;
      s_par[1] = beta;
      s_par[2] = scale;
      if (blockIdx.x == 0) tau_all[k] = tau;
    }
    __syncthreads();
    if (threadIdx.x < kRRW) {
      const int j = threadIdx.x;
      s_tw[j] = (j > k && j < pw) ? s_par[0] * (s_pv[j] + s_par[2] * s_tot[j - k]) : 0.0;
    }
    beta_p = s_par[1];
    scale_p = s_par[2];
    __syncthreads();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *state = 1u;  // T is formed from V and tau
#pragma unroll
  for (int q = 0; q < kRRQ; ++q) {
    if (lrow[q] < 0) continue;
#pragma unroll
    for (int j = 0; j < kRRW; ++j)
      if (j < pw) A[lrow[q] + j * ld] = a[q][j];
  }
}

// sum_{q0 <= q < q1} a(q) b(q) with four independent partial sums, so that the
// LDS reads of four terms are in flight together (a single running sum waits
// for each read in turn)
template <class FA, class FB>
GAP_DEV double dot4(int q0, int q1, FA a, FB b) {
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  int q = q0;
  for (; q + 3 < q1; q += 4) {
    s0 += a(q) * b(q);
    s1 += a(q + 1) * b(q + 1);
    s2 += a(q + 2) * b(q + 2);
    s3 += a(q + 3) * b(q + 3);
  }
  for (; q < q1; ++q) s0 += a(q) * b(q);
  return (s0 + s1) + (s2 + s3);
}

// Trailing update, persistent over a 128-row block of C: the block stages
// V^T for its rows once in LDS (with the unit lower trapezoid applied), then
// walks the 64-wide column tiles of C.  W' = -(T^T W) tiles are double-buffered
// in LDS and the next C tile is prefetched into registers while the current
// one runs on the matrix cores; accumulators start as the C tile, so each C
// element is read and written once.  Eight waves: 2 (column halves) x 4 (row
// quarters), each a 32 x 32 block of (C column, C row) = (matrix-core row, col).
constexpr int kUR = 128;  // rows of C per block
constexpr int kUC = 64;   // columns per tile
template <int KW>
__global__ __launch_bounds__(512) void k_qr_upd(double* __restrict__ A, int64_t ld, int64_t m,
                                                int64_t j0, int pw, int64_t c_end, int64_t nct,
                                                const double* __restrict__ Wt,
                                                const unsigned int* __restrict__ skip) {
  if (*skip) return;  // the reflectors are not there yet
  // padded row strides: the four lane groups of a fragment read (rows kk .. kk+3)
  // fall on different banks
  __shared__ double sV[KW][kUR + 8];
  __shared__ double sW[2][KW][kUC + 8];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wc = wave & 1, wr = wave >> 1;
  const int64_t r0 = j0 + (int64_t)blockIdx.x * kUR;
  const int64_t cbeg = j0 + pw;
  const int ntile = (int)((c_end - cbeg + kUC - 1) / kUC);
  if (r0 - j0 >= KW && r0 + kUR <= m) {
    // below the unit triangle and inside the matrix: all loads issued at once
    // (rows kk >= pw read row pw - 1 and are zeroed after), not one guarded
    // load after another
    constexpr int kN = KW * kUR / 512;
    double tmp[kN];
#pragma unroll
    for (int t = 0; t < kN; ++t) {
      const int e = threadIdx.x + t * 512, kk = e / kUR, x = e % kUR;
      tmp[t] = A[(r0 + x) + (j0 + min(kk, pw - 1)) * ld];
    }
#pragma unroll
    for (int t = 0; t < kN; ++t) {
      const int e = threadIdx.x + t * 512, kk = e / kUR, x = e % kUR;
      sV[kk][x] = kk < pw ? tmp[t] : 0.0;
    }
  } else {
    for (int e = threadIdx.x; e < KW * kUR; e += 512) {
      const int kk = e / kUR, x = e % kUR;
      const int64_t r = r0 + x;
      double v = 0.0;
      if (kk < pw && r < m) {
        const int64_t rr = r - j0;
        v = (rr == kk) ? 1.0 : (rr > kk ? A[r + (j0 + kk) * ld] : 0.0);
      }
      sV[kk][x] = v;
    }
  }
  // W' tile in registers first (8 values per thread), written to LDS later
  double wreg[KW * kUC / 512];
  auto load_w = [&](int tile) {
#pragma unroll
    for (int t = 0; t < KW * kUC / 512; ++t) {
      // clamped, unconditional: rows kk >= pw meet zero rows of sV, columns
      // beyond c_end only feed outputs that are never stored
      const int e = threadIdx.x + t * 512;
      const int kk = min(e / kUC, pw - 1), x = e % kUC;
      const int64_t c = min(cbeg + (int64_t)min(tile, ntile - 1) * kUC + x, c_end - 1);
      wreg[t] = Wt[(int64_t)kk * nct + (c - j0)];
    }
  };
  auto store_w = [&](int buf) {
#pragma unroll
    for (int t = 0; t < KW * kUC / 512; ++t) {
      const int e = threadIdx.x + t * 512;
      sW[buf][e / kUC][e % kUC] = wreg[t];
    }
  };
  auto load_c = [&](int tile, d4v (&dst)[2][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int64_t rc = min(r0 + wr * 32 + j * 16 + idx, m - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t c = cbeg + (int64_t)tile * kUC + wc * 32 + i * 16 + g + 4 * q;
          dst[i][j][q] = A[rc + min(c, c_end - 1) * ld];
        }
      }
  };
  d4v acc[2][2], nxt[2][2];
  load_w(0);
  load_c(0, acc);
  store_w(0);
  __syncthreads();
  int buf = 0;
  for (int tile = 0; tile < ntile; ++tile) {
    const bool more = tile + 1 < ntile;
    if (more) {
      load_w(tile + 1);
      load_c(tile + 1, nxt);
    }
#pragma unroll
    for (int k0 = 0; k0 < KW; k0 += 4) {  // rows of sV at and beyond pw are zero
      const int kk = k0 + g;
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = sW[buf][kk][wc * 32 + i * 16 + idx];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = sV[kk][wr * 32 + j * 16 + idx];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(a[i], b[j], acc[i][j]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int64_t r = r0 + wr * 32 + j * 16 + idx;
        if (r >= m) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t c = cbeg + (int64_t)tile * kUC + wc * 32 + i * 16 + g + 4 * q;
          if (c < c_end) A[r + c * ld] = acc[i][j][q];
        }
      }
    if (more) store_w(buf ^ 1);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = nxt[i][j];
    buf ^= 1;
  }
}

// Buffer resources with a base in scalar registers: an access is that base
// plus a 32-bit per-lane offset plus a scalar offset, so a kernel that walks
// many columns of the column-major matrix keeps one offset register instead of
// a 64-bit address per column.  An access at or beyond the resource's size
// reads zero (a store is dropped).
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
GAP_DEV __amdgpu_buffer_rsrc_t uniform_rsrc(const double* p, uint32_t bytes) {
  const uint64_t x = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)hi << 32 | lo), 0, (int)bytes,
                                           0x00020000);
}
GAP_DEV double buf_ld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
GAP_DEV void buf_st(double x, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, voff, soff, 0);
}

// W = V^T C over row slabs, staged through LDS: a block owns one slab and a
// 128-wide column tile (relative to the panel start; columns < pw are the
// panel's own V columns, giving the Gram V^T V).  32-row chunks of V and C are
// double-buffered in LDS (register prefetch of the next chunk while the
// current one runs on the matrix cores).  Consecutive logical blocks on an XCD
// share the slab, so its V rows come from that XCD's L2.  Eight waves:
// 2 (V-column halves) x 4 (C-column quarters), 32 x 32 outputs each.
constexpr int kVC = 128;  // C columns per block
constexpr int kVK = 32;   // rows per chunk
__global__ __launch_bounds__(512) void k_qr_vtc2(const double* __restrict__ A, int64_t ld,
                                                 int64_t m, int64_t j0, int pw, int64_t nct,
                                                 int64_t slab, int64_t n_ct, int64_t total,
                                                 int64_t per_xcd, double* __restrict__ part) {
  // row strides padded (73 and 137 doubles) so that neither the row-wise stash
  // (consecutive threads -> consecutive rows) nor the fragment reads conflict
  __shared__ double sV[2][kVK][kQrNB + 9];
  __shared__ double sC[2][kVK][kVC + 9];
  const int64_t logical = xcd_logical_block(per_xcd);
  if (logical >= total) return;
  const int64_t s = logical / n_ct, ct = logical % n_ct;
  const int64_t r0 = j0 + s * slab, r1 = std::min(m, r0 + slab);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wv = wave & 1, wq = wave >> 1;
  const int64_t c0 = ct * kVC;  // first column (relative to j0) of the tile
  // per-thread slice of a chunk: V 4 elements, C 8 elements (rows fastest);
  // two register sets so chunk k+2 is in flight while chunk k+1 lands in LDS
  double rv[2][4], rc[2][8];
  auto fetch = [&](int64_t rk, int set) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = threadIdx.x + t * 512;
      const int x = e / kVK, kk = e % kVK;
      const int64_t r = rk + kk;
      double v = 0.0;
      if (x < pw && r < r1) {
        const int64_t rr = r - j0;
        v = (rr == x) ? 1.0 : (rr > x ? A[r + (j0 + x) * ld] : 0.0);
      }
      rv[set][t] = v;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = threadIdx.x + t * 512;
      const int x = e / kVK, kk = e % kVK;
      const int64_t r = rk + kk;
      const int64_t cp = c0 + x;
      double v = 0.0;
      if (cp < nct && r < r1) {
        if (cp < pw) {
          const int64_t rr = r - j0;
          v = (rr == cp) ? 1.0 : (rr > cp ? A[r + (j0 + cp) * ld] : 0.0);
        } else {
          v = A[r + (j0 + cp) * ld];
        }
      }
      rc[set][t] = v;
    }
  };
  auto stash = [&](int buf, int set) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = threadIdx.x + t * 512;
      sV[buf][e % kVK][e / kVK] = rv[set][t];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = threadIdx.x + t * 512;
      sC[buf][e % kVK][e / kVK] = rc[set][t];
    }
  };
  d4v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = zero4();
  auto compute = [&](int buf) {
#pragma unroll
    for (int k0 = 0; k0 < kVK; k0 += 4) {
      const int kk = k0 + g;
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = sV[buf][kk][wv * 32 + i * 16 + idx];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = sC[buf][kk][wq * 32 + j * 16 + idx];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(a[i], b[j], acc[i][j]);
    }
  };
  // chunk c covers rows r0 + c * kVK; chunk c lives in LDS buffer c & 1 and,
  // before that, in register set c & 1
  const int64_t nch = (r1 - r0 + kVK - 1) / kVK;
  fetch(r0, 0);
  if (nch > 1) fetch(r0 + kVK, 1);
  stash(0, 0);
  __syncthreads();
  for (int64_t c = 0; c < nch; c += 2) {
    // even chunk c in LDS buffer 0; chunk c+1 in register set 1
    if (c + 2 < nch) fetch(r0 + (c + 2) * kVK, 0);
    compute(0);
    if (c + 1 < nch) stash(1, 1);
    lds_barrier();
    if (c + 1 >= nch) break;
    if (c + 3 < nch) fetch(r0 + (c + 3) * kVK, 1);
    compute(1);
    if (c + 2 < nch) stash(0, 0);
    lds_barrier();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t cp = c0 + wq * 32 + j * 16 + idx;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ii = wv * 32 + i * 16 + g + 4 * q;
        if (ii < pw && cp < nct) part[(s * pw + ii) * nct + cp] = acc[i][j][q];
      }
    }
}

constexpr int kNarrowSlab = 512;  // rows per slab of a 64-wide update

// ---------------------------------------------- outer (128-wide) WY update ----
// The same two products as above for a reflector block up to kQrOB = 128 wide:
// one pass over the trailing columns per 128 reflectors halves the HBM traffic
// of the 64-wide update, and each C element then carries 256 flops per 16 bytes
// moved, enough to keep the FP64 matrix cores ahead of memory.
constexpr int kQrOB = 128;

// W = V^T C over row slabs with V up to 128 wide.  Eight waves: 2 (64-column
// halves of V) x 4 (32-column quarters of the 128-column C tile).
template <bool BUF>
__global__ __launch_bounds__(512) void k_qr_vtc3(const double* __restrict__ A, int64_t ld,
                                                 int64_t m, int64_t j0, int pw, int64_t nct,
                                                 int64_t slab, int64_t n_ct, int64_t total,
                                                 int64_t per_xcd, double* __restrict__ part) {
  __shared__ double sV[2][kVK][kQrOB + 9];
  __shared__ double sC[2][kVK][kVC + 9];
  const int64_t logical = xcd_logical_block(per_xcd);
  if (logical >= total) return;
  const int64_t s = logical / n_ct, ct = logical % n_ct;
  const int64_t r0 = j0 + s * slab, r1 = std::min(m, r0 + slab);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wv = wave & 1, wq = wave >> 1;
  const int64_t c0 = ct * kVC;
  // each thread stages one row (kk) of a chunk and the columns x0 + 16 t
  const int kk_t = threadIdx.x & (kVK - 1), x0 = threadIdx.x / kVK;
  double rv[8], rc[8], rv2[8], rc2[8];
  // Two fetch forms.  Interior chunks (every row inside the slab and below the
  // V triangle) load from clamped addresses with no condition at all: V
  // columns >= pw only feed W rows >= pw and C columns >= nct only feed W
  // columns >= nct, none of which are stored.  A guarded load compiles to a
  // branch that waits for the load on the spot, so guards are kept to the few
  // edge chunks (the V triangle at the top of the first slab, a partial last
  // chunk), which use the masked form.
  auto fetch_fast = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    const double* rowp = A + (rk + kk_t);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      rv[t] = rowp[(j0 + min(x0 + 16 * t, pw - 1)) * ld];
      rc[t] = rowp[(j0 + min(c0 + x0 + 16 * t, nct - 1)) * ld];
    }
  };
  auto fetch_masked = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    const int64_t r = rk + kk_t;
    const bool rin = r < r1;
    const int64_t rr = r - j0;
    const double* rowp = A + (rin ? r : 0);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int x = x0 + 16 * t;
      double v = 0.0;
      if (rin && x < pw) v = (rr == x) ? 1.0 : (rr > x ? rowp[(j0 + x) * ld] : 0.0);
      rv[t] = v;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int64_t cp = c0 + x0 + 16 * t;
      double v = 0.0;
      if (rin && cp < nct) {
        if (cp >= pw)
          v = rowp[(j0 + cp) * ld];
        else
          v = (rr == cp) ? 1.0 : (rr > cp ? rowp[(j0 + cp) * ld] : 0.0);
      }
      rc[t] = v;
    }
  };
  // The interior form through buffer resources based at the chunk's first row
  // of the first V column and of the tile's first C column: the thread's row
  // and column x0 are its offset, each t adds 16 columns as a scalar offset,
  // and columns past pw (V) or nct (C) lie outside the resources and read zero.
  const uint32_t xoff = (uint32_t)(((int64_t)x0 * ld + kk_t) * 8);
  const uint32_t vbytes = (uint32_t)((int64_t)pw * ld * 8);
  const uint32_t cbytes = (uint32_t)(std::min<int64_t>(nct - c0, kVC) * ld * 8);
  auto fetch_buf = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    const auto rsv = uniform_rsrc(A + j0 * ld + rk, vbytes);
    const auto rsc = uniform_rsrc(A + (j0 + c0) * ld + rk, cbytes);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      rv[t] = buf_ld(rsv, xoff, (uint32_t)(16 * t * ld * 8));
      rc[t] = buf_ld(rsc, xoff, (uint32_t)(16 * t * ld * 8));
    }
  };
  auto fetch = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    if (rk - j0 >= pw && rk + kVK <= r1) {
      if (BUF)
        fetch_buf(rk, rv, rc);
      else
        fetch_fast(rk, rv, rc);
    } else {
      fetch_masked(rk, rv, rc);
    }
  };
  auto stash = [&](int buf, const double (&rv)[8], const double (&rc)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      sV[buf][kk_t][x0 + 16 * t] = rv[t];
      sC[buf][kk_t][x0 + 16 * t] = rc[t];
    }
  };
  d4v acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = zero4();
  auto compute = [&](int buf, int k_lo, int k_hi) {
#pragma unroll
    for (int k0 = k_lo; k0 < k_hi; k0 += 4) {
      const int kk = k0 + g;
      double a[4], b[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sV[buf][kk][wv * 64 + i * 16 + idx];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = sC[buf][kk][wq * 32 + j * 16 + idx];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(a[i], b[j], acc[i][j]);
    }
  };
  // Chunks that meet the unit triangle of V (first slab) or end past the
  // matrix take the masked fetch one at a time; the interior ones run a
  // pipeline: chunk c is fetched into a register set two chunks ahead and
  // written to LDS buffer c & 1 in the middle of chunk c - 1's products (that
  // buffer was last read by chunk c - 2, before the previous barrier), so the
  // LDS writes overlap matrix-core work and the loads have a chunk and a half
  // to arrive.  The pipeline is straight-line code (fetches past the last
  // interior chunk re-read it, and its extra LDS write is never read), which
  // lets every wait for a fetch count the newer fetches still in flight.
  const int64_t nfull = (r1 - r0) / kVK;
  const int64_t c_lo = std::min<int64_t>(nfull, r0 - j0 >= pw ? 0 : (pw - (r0 - j0) + kVK - 1) / kVK);
  const int64_t c_hi = nfull;
  auto single = [&](int64_t c) {
    fetch_masked(r0 + c * kVK, rv, rc);
    lds_barrier();
    stash(0, rv, rc);
    lds_barrier();
    compute(0, 0, kVK);
  };
  for (int64_t c = 0; c < c_lo; ++c) single(c);
  if (c_hi > c_lo) {
    auto fetch_i = [&](int64_t c, double (&rv_)[8], double (&rc_)[8]) {
      const int64_t rk = r0 + std::min(c, c_hi - 1) * kVK;
      if (BUF)
        fetch_buf(rk, rv_, rc_);
      else
        fetch_fast(rk, rv_, rc_);
    };
    lds_barrier();
    fetch_i(c_lo, rv, rc);
    stash(0, rv, rc);
    fetch_i(c_lo + 1, rv2, rc2);
    lds_barrier();
    auto step = [&](int64_t c, double (&rnext)[8], double (&cnext)[8], double (&rfar)[8],
                    double (&cfar)[8]) {
      const int buf = (int)((c - c_lo) & 1);
      fetch_i(c + 2, rfar, cfar);
      compute(buf, 0, kVK / 2);
      stash(buf ^ 1, rnext, cnext);
      compute(buf, kVK / 2, kVK);
      lds_barrier();
    };
    int64_t c = c_lo;
    for (; c + 1 < c_hi; c += 2) {
      step(c, rv2, rc2, rv, rc);      // chunk c + 1 is in set 2, chunk c + 2 goes to set 1
      step(c + 1, rv, rc, rv2, rc2);  // chunk c + 2 is in set 1, chunk c + 3 goes to set 2
    }
    if (c < c_hi) step(c, rv2, rc2, rv, rc);
  }
  if (c_hi * kVK < r1 - r0) {
    lds_barrier();
    single(c_hi);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t cp = c0 + wq * 32 + j * 16 + idx;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ii = wv * 64 + i * 16 + g + 4 * q;
        if (ii < pw && cp < nct) part[(s * pw + ii) * nct + cp] = acc[i][j][q];
      }
    }
}

// The same product with four waves per block (each a 64 x 64 block of W) and
// 16-row chunks, so that the LDS of a block is 70 KB and two blocks share a
// compute unit: the two waves on a SIMD then belong to different blocks and
// are not held in step by one barrier, so one block's LDS writes and barrier
// overlap the other block's matrix-core products.
constexpr int kV5K = 16;
template <bool BUF>
__global__ __launch_bounds__(256, 2) void k_qr_vtc5(const double* __restrict__ A, int64_t ld,
                                                 int64_t m, int64_t j0, int pw, int64_t nct,
                                                 int64_t slab, int64_t n_ct, int64_t total,
                                                 int64_t per_xcd, double* __restrict__ part) {
  constexpr int kVK = kV5K;
  __shared__ double sV[2][kVK][kQrOB + 9];
  __shared__ double sC[2][kVK][kVC + 9];
  const int64_t logical = xcd_logical_block(per_xcd);
  if (logical >= total) return;
  const int64_t s = logical / n_ct, ct = logical % n_ct;
  const int64_t r0 = j0 + s * slab, r1 = std::min(m, r0 + slab);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wv = wave & 1, wq = wave >> 1;
  const int64_t c0 = ct * kVC;
  // each thread stages one row (kk) of a chunk and the columns x0 + 16 t
  const int kk_t = threadIdx.x & (kVK - 1), x0 = threadIdx.x / kVK;  // x0 < 16
  double rv[8], rc[8], rv2[8], rc2[8];
  // Two fetch forms.  Interior chunks (every row inside the slab and below the
  // V triangle) load from clamped addresses with no condition at all: V
  // columns >= pw only feed W rows >= pw and C columns >= nct only feed W
  // columns >= nct, none of which are stored.  A guarded load compiles to a
  // branch that waits for the load on the spot, so guards are kept to the few
  // edge chunks (the V triangle at the top of the first slab, a partial last
  // chunk), which use the masked form.
  auto fetch_fast = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    const double* rowp = A + (rk + kk_t);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      rv[t] = rowp[(j0 + min(x0 + 16 * t, pw - 1)) * ld];
      rc[t] = rowp[(j0 + min(c0 + x0 + 16 * t, nct - 1)) * ld];
    }
  };
  auto fetch_masked = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    const int64_t r = rk + kk_t;
    const bool rin = r < r1;
    const int64_t rr = r - j0;
    const double* rowp = A + (rin ? r : 0);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int x = x0 + 16 * t;
      double v = 0.0;
      if (rin && x < pw) v = (rr == x) ? 1.0 : (rr > x ? rowp[(j0 + x) * ld] : 0.0);
      rv[t] = v;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int64_t cp = c0 + x0 + 16 * t;
      double v = 0.0;
      if (rin && cp < nct) {
        if (cp >= pw)
          v = rowp[(j0 + cp) * ld];
        else
          v = (rr == cp) ? 1.0 : (rr > cp ? rowp[(j0 + cp) * ld] : 0.0);
      }
      rc[t] = v;
    }
  };
  // The interior form through buffer resources based at the chunk's first row
  // of the first V column and of the tile's first C column: the thread's row
  // and column x0 are its offset, each t adds 16 columns as a scalar offset,
  // and columns past pw (V) or nct (C) lie outside the resources and read zero.
  const uint32_t xoff = (uint32_t)(((int64_t)x0 * ld + kk_t) * 8);
  const uint32_t vbytes = (uint32_t)((int64_t)pw * ld * 8);
  const uint32_t cbytes = (uint32_t)(std::min<int64_t>(nct - c0, kVC) * ld * 8);
  auto fetch_buf = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    const auto rsv = uniform_rsrc(A + j0 * ld + rk, vbytes);
    const auto rsc = uniform_rsrc(A + (j0 + c0) * ld + rk, cbytes);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      rv[t] = buf_ld(rsv, xoff, (uint32_t)(16 * t * ld * 8));
      rc[t] = buf_ld(rsc, xoff, (uint32_t)(16 * t * ld * 8));
    }
  };
  auto fetch = [&](int64_t rk, double (&rv)[8], double (&rc)[8]) {
    if (rk - j0 >= pw && rk + kVK <= r1) {
      if (BUF)
        fetch_buf(rk, rv, rc);
      else
        fetch_fast(rk, rv, rc);
    } else {
      fetch_masked(rk, rv, rc);
    }
  };
  auto stash = [&](int buf, const double (&rv)[8], const double (&rc)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      sV[buf][kk_t][x0 + 16 * t] = rv[t];
      sC[buf][kk_t][x0 + 16 * t] = rc[t];
    }
  };
  d4v acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = zero4();
  auto compute = [&](int buf, int k_lo, int k_hi) {
#pragma unroll
    for (int k0 = k_lo; k0 < k_hi; k0 += 4) {
      const int kk = k0 + g;
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sV[buf][kk][wv * 64 + i * 16 + idx];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = sC[buf][kk][wq * 64 + j * 16 + idx];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma_f64(a[i], b[j], acc[i][j]);
    }
  };
  // Chunks that meet the unit triangle of V (first slab) or end past the
  // matrix take the masked fetch one at a time; the interior ones run a
  // pipeline: chunk c is fetched into a register set two chunks ahead and
  // written to LDS buffer c & 1 in the middle of chunk c - 1's products (that
  // buffer was last read by chunk c - 2, before the previous barrier), so the
  // LDS writes overlap matrix-core work and the loads have a chunk and a half
  // to arrive.  The pipeline is straight-line code (fetches past the last
  // interior chunk re-read it, and its extra LDS write is never read), which
  // lets every wait for a fetch count the newer fetches still in flight.
  const int64_t nfull = (r1 - r0) / kVK;
  const int64_t c_lo = std::min<int64_t>(nfull, r0 - j0 >= pw ? 0 : (pw - (r0 - j0) + kVK - 1) / kVK);
  const int64_t c_hi = nfull;
  auto single = [&](int64_t c) {
    fetch_masked(r0 + c * kVK, rv, rc);
    lds_barrier();
    stash(0, rv, rc);
    lds_barrier();
    compute(0, 0, kVK);
  };
  for (int64_t c = 0; c < c_lo; ++c) single(c);
  if (c_hi > c_lo) {
    auto fetch_i = [&](int64_t c, double (&rv_)[8], double (&rc_)[8]) {
      const int64_t rk = r0 + std::min(c, c_hi - 1) * kVK;
      if (BUF)
        fetch_buf(rk, rv_, rc_);
      else
        fetch_fast(rk, rv_, rc_);
    };
    lds_barrier();
    fetch_i(c_lo, rv, rc);
    stash(0, rv, rc);
    fetch_i(c_lo + 1, rv2, rc2);
    lds_barrier();
    auto step = [&](int64_t c, double (&rnext)[8], double (&cnext)[8], double (&rfar)[8],
                    double (&cfar)[8]) {
      const int buf = (int)((c - c_lo) & 1);
      fetch_i(c + 2, rfar, cfar);
      compute(buf, 0, kVK / 2);
      stash(buf ^ 1, rnext, cnext);
      compute(buf, kVK / 2, kVK);
      lds_barrier();
    };
    int64_t c = c_lo;
    for (; c + 1 < c_hi; c += 2) {
      step(c, rv2, rc2, rv, rc);      // chunk c + 1 is in set 2, chunk c + 2 goes to set 1
      step(c + 1, rv, rc, rv2, rc2);  // chunk c + 2 is in set 1, chunk c + 3 goes to set 2
    }
    if (c < c_hi) step(c, rv2, rc2, rv, rc);
  }
  if (c_hi * kVK < r1 - r0) {
    lds_barrier();
    single(c_hi);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t cp = c0 + wq * 64 + j * 16 + idx;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ii = wv * 64 + i * 16 + g + 4 * q;
        if (ii < pw && cp < nct) part[(s * pw + ii) * nct + cp] = acc[i][j][q];
      }
    }
}

// T of a 64-wide half whose panel was factored by k_qr_panel_dep or k_qr_panel_rr (its
// state word is set; other panels bring their T along), from the Gram G = V^T V held in W
// (row l at W + l * nct): T[0:i, i] = -tau_i T[0:i, 0:i] G[0:i, i], T[i][i] =
// tau_i.  Col-major, ld 64, one block per half; zero below the diagonal.
__global__ __launch_bounds__(256) void k_qr_larft(const double* __restrict__ W, int64_t nct,
                                                  int pw, const double* __restrict__ tau,
                                                  double* __restrict__ T,
                                                  const unsigned int* __restrict__ state) {
  __shared__ double sT[kQrNB][kQrNB + 1];
  __shared__ double sG[kQrNB][kQrNB + 1];
  if (state[blockIdx.x] == 0u) return;
  const int o = blockIdx.x * kQrNB;
  const int w = min(kQrNB, pw - o);
  __shared__ double sTau[kQrNB];  // staged once: a load per column would cost a round trip each
  if (threadIdx.x < kQrNB) sTau[threadIdx.x] = (int)threadIdx.x < w ? tau[o + threadIdx.x] : 0.0;
  for (int e = threadIdx.x; e < kQrNB * kQrNB; e += 256) {
    const int l = e / kQrNB, i = e % kQrNB;
    sG[l][i] = (l < w && i < w) ? W[(int64_t)(o + l) * nct + (o + i)] : 0.0;
    sT[l][i] = 0.0;
  }
  __syncthreads();
  const int l = threadIdx.x;
  for (int i = 0; i < w; ++i) {
    double z = 0.0;
    if (l < i) z = dot4(l, i, [&](int q) { return sT[l][q]; }, [&](int q) { return sG[q][i]; });
    __syncthreads();
    const double ti = sTau[i];
    if (l < i) sT[l][i] = -ti * z;
    if (l == i) sT[i][i] = ti;
    __syncthreads();
  }
  for (int e = threadIdx.x; e < kQrNB * kQrNB; e += 256)
    T[blockIdx.x * kQrNB * kQrNB + e] = sT[e % kQrNB][e / kQrNB];
}

// Wt = -T^T W over the trailing columns [pw, nct), T the factor of up to two
// 64-wide halves H = H1 H2: with T1, T2 (col-major, ld 64) and the coupling
// G12 = V1^T V2 that W holds in its own columns,
//   Wt1 = -T1^T W1,  Wt2 = -T2^T (W2 + G12^T Wt1),
// which is -T^T W for T = [T1, -T1 G12 T2; 0, T2] without forming it.  (The
// negated product, so that the update kernel adds V Wt to C.)  A block takes 64
// columns, a wave 16 of them; each product's result is the next one's operand in
// the registers it is in (lane group g holds rows g + 4 r, so step r contracts
// those rows).  The one-block products for T and the element-wise product this
// replaces took 140 us per 128 columns; this takes 10.
__global__ __launch_bounds__(256) void k_qr_wt(const double* __restrict__ W, int64_t nct, int pw,
                                               const double* __restrict__ T,
                                               double* __restrict__ Wt) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int64_t cp = pw + (int64_t)blockIdx.x * 64 + wave * 16 + idx;
  if (cp - idx >= nct) return;
  const double* wc = W + min(cp, nct - 1);
  // rows l = o + 16 t + g + 4 r of W's column, zero from pw on
  auto load_w = [&](int o, d4v (&x)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = o + 16 * t + g + 4 * r;
        const double v = wc[(int64_t)min(l, pw - 1) * nct];
        x[t][r] = l < pw ? v : 0.0;
      }
  };
  // y = -T^T x (T[l][kk] at T[kk * 64 + l], zero for l > kk)
  auto times_t = [&](const double* Th, const d4v (&x)[4], d4v (&y)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      y[u] = zero4();
#pragma unroll
      for (int t = 0; t <= u; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          y[u] = mfma_f64(-Th[(16 * u + idx) * kQrNB + 16 * t + g + 4 * r], x[t][r], y[u]);
    }
  };
  auto store = [&](int o, const d4v (&y)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int kk = o + 16 * u + g + 4 * r;
        if (kk < pw && cp < nct) Wt[(int64_t)kk * nct + cp] = y[u][r];
      }
  };
  d4v x[4], y[4];
  load_w(0, x);
  times_t(T, x, y);
  store(0, y);
  if (pw <= kQrNB) return;
  load_w(kQrNB, x);
#pragma unroll
  for (int u = 0; u < 4; ++u) {  // x += G12^T y
    const int k2 = kQrNB + 16 * u + idx;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double v = W[(int64_t)(16 * t + g + 4 * r) * nct + min(k2, pw - 1)];
        x[u] = mfma_f64(k2 < pw ? v : 0.0, y[t][r], x[u]);
      }
  }
  times_t(T + kQrNB * kQrNB, x, y);
  store(kQrNB, y);
}

// C -= V W' for a reflector block up to 128 wide, persistent over a 128-row
// block of C: V^T for the rows is staged once in LDS (unit lower trapezoid
// applied, zero rows beyond pw).  A W' = T^T W tile (128 x 64) is loaded into
// registers one tile ahead, together with the next C tile (16 + 16 values per
// thread), and moves through a two-deep LDS ring in 16-deep k chunks, so no
// global load is waited on inside a tile.  Accumulators start as the C tile.
// Eight waves: 2 (column halves) x 4 (row quarters), each a 32 x 32 block of
// (C column, C row) = (matrix-core row, column).
constexpr int kU3R = 128;
constexpr int kU3C = 64;
constexpr int kU3K = kQrOB / 16;  // k chunks per tile
__global__ __launch_bounds__(512) void k_qr_upd3(double* __restrict__ A, int64_t ld, int64_t m,
                                                 int64_t j0, int pw, int64_t c_end, int64_t nct,
                                                 const double* __restrict__ Wn) {
  __shared__ double sV[kQrOB][kU3R + 8];
  __shared__ double sW[2][16][kU3C + 4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wc = wave & 1, wr = wave >> 1;
  const int64_t r0 = j0 + (int64_t)blockIdx.x * kU3R;
  const int64_t cbeg = j0 + pw;
  const int ntile = (int)((c_end - cbeg + kU3C - 1) / kU3C);
  // All kU3K chunks are always run (rows of sV beyond pw are zero): only the
  // last outer block is narrower than kQrOB, and its trailing part is the
  // right-hand side alone.  A compile-time chunk count keeps the choice of the
  // next chunk's source free of selects that would wait on the prefetch.
  for (int e = threadIdx.x; e < kQrOB * kU3R; e += 512) {
    const int kk = e / kU3R, x = e % kU3R;
    const int64_t r = r0 + x;
    double v = 0.0;
    if (kk < pw && r < m) {
      const int64_t rr = r - j0;
      v = (rr == kk) ? 1.0 : (rr > kk ? A[r + (j0 + kk) * ld] : 0.0);
    }
    sV[kk][x] = v;
  }
  // -W' tile (Wn): thread t holds, for chunk kc, elements t and t + 512 of the
  // 16 x 64 chunk (row e / 64, column e % 64)
  auto load_w = [&](int tile, double (&dst)[kU3K][2]) {
#pragma unroll
    for (int kc = 0; kc < kU3K; ++kc)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // Unconditional load from a clamped (valid) address: a guarded load
        // becomes a branch whose join waits for every load in flight.  No mask
        // is needed: a clamped k row meets a zero row of sV, a clamped column
        // only feeds outputs that are never stored, and a tile beyond the last
        // is never used.
        const int e = threadIdx.x + h * 512;
        const int kk = min(kc * 16 + e / kU3C, pw - 1);  // rows >= pw meet zero rows of sV
        const int64_t c = min(cbeg + (int64_t)min(tile, ntile - 1) * kU3C + (e % kU3C), c_end - 1);
        dst[kc][h] = Wn[(int64_t)kk * nct + (c - j0)];
      }
  };
  auto store_w = [&](int buf, const double (&src)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = threadIdx.x + h * 512;
      sW[buf][e / kU3C][e % kU3C] = src[h];
    }
  };
  auto load_c = [&](int tile, d4v (&dst)[2][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // clamped, unconditional (rows or columns outside C are never stored)
        const int64_t rc = min(r0 + wr * 32 + j * 16 + idx, m - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t c =
              cbeg + (int64_t)min(tile, ntile - 1) * kU3C + wc * 32 + i * 16 + g + 4 * q;
          dst[i][j][q] = A[rc + min(c, c_end - 1) * ld];
        }
      }
  };
  d4v acc[2][2], nxt[2][2];
  double wcur[kU3K][2], wnxt[kU3K][2];
  load_c(0, acc);
  load_w(0, wcur);
  store_w(0, wcur[0]);
  __syncthreads();
  int buf = 0;
  for (int tile = 0; tile < ntile; ++tile) {
    load_c(tile + 1, nxt);
    load_w(tile + 1, wnxt);
#pragma unroll
    for (int kc = 0; kc < kU3K; ++kc) {
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const int kr = 4 * s4 + g;
        const int kk = kc * 16 + kr;
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = sW[buf][kr][wc * 32 + i * 16 + idx];
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = sV[kk][wr * 32 + j * 16 + idx];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(a[i], b[j], acc[i][j]);
      }
      // the next chunk: of this tile, or the first of the next tile
      if (kc + 1 < kU3K)
        store_w(buf ^ 1, wcur[kc + 1 < kU3K ? kc + 1 : 0]);
      else
        store_w(buf ^ 1, wnxt[0]);
      lds_barrier();
      buf ^= 1;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int64_t r = r0 + wr * 32 + j * 16 + idx;
        if (r >= m) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t c = cbeg + (int64_t)tile * kU3C + wc * 32 + i * 16 + g + 4 * q;
          if (c < c_end) A[r + c * ld] = acc[i][j][q];
        }
      }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = nxt[i][j];
#pragma unroll
    for (int kc = 0; kc < kU3K; ++kc) {
      wcur[kc][0] = wnxt[kc][0];
      wcur[kc][1] = wnxt[kc][1];
    }
  }
}

// C -= V W' for a full 128-wide reflector block, one barrier per 64-column
// tile.  Each of the eight waves owns 16 rows of the block's 128 and keeps
// their V (128 deep) in registers while it walks a row block; -W' (Wn) is the only
// shared operand and goes through LDS one whole 128 x 64 tile at a time,
// double-buffered.  A wave's block is 16 rows x 64 columns (four matrix-core tiles sharing the V
// operand).  Odd Wn rows are stored with their 16-column halves swapped so that
// the lane groups reading rows 4t + g and 4t + g + 1 meet different banks.
//
// The memory traffic of a tile is issued between its matrix-core products, not
// around them: the two waves of a SIMD run in step (one barrier per tile), so
// work issued before or after the products leaves the matrix pipe idle.  For
// that the next tile's Wn and C are fetched and the previous tile's result is
// stored in fixed steps of the products (two accumulators in turn), with buffer
// stores whose out-of-range offset drops the lanes that must not write, so no store
// sits in a branch.  Bound by both: 16 flop a byte at 53 TFLOP/s and 3.6 TB/s.
//
// Every global access is a wave-uniform base (scalar registers) plus a 32-bit
// per-lane byte offset, and no column is clamped: the last tile is shifted left
// to end at c_end (it needs c_end - cbeg >= 64) and stores only the columns the
// previous tile did not.  Per-access 64-bit addresses would take 64 registers.
//
// The tiles of all row blocks in turn are dealt to kU5Blocks blocks, one per
// compute unit, in even runs, so the last turn is as full as the others: with a
// block per 128 rows, 689 of them ran as three turns of 256 (88,200 rows, 1,873
// columns: 940 us, here 798; 56,000 rows in 410 blocks lost a fifth).  What
// a run loads for a row block leaves in one batch, as a compute unit has no second
// block to hide it behind.
constexpr int kU5Blocks = 256;
constexpr int kU5R = 128;  // rows per block (8 waves x 16)
constexpr int kU5C = 64;   // columns per tile
constexpr uint32_t kDropOffset = 0x80000000u;  // beyond any buffer this kernel makes
__global__ __launch_bounds__(512) void k_qr_upd5(double* __restrict__ A, int64_t ld, int64_t m,
                                                 int64_t j0, int64_t c_end, int64_t nct,
                                                 const double* __restrict__ Wn) {
  __shared__ double sW[2][kQrOB][kU5C];
  const int lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t cbeg = j0 + kQrOB;
  const int ntile = (int)((c_end - cbeg + kU5C - 1) / kU5C);
  const int64_t n_all = (m - j0 + kU5R - 1) / kU5R * ntile;
  const int64_t t_end = n_all * (blockIdx.x + 1) / gridDim.x;
#pragma clang loop unroll(disable)
  for (int64_t t_at = n_all * blockIdx.x / gridDim.x; t_at < t_end;) {
    const int tile_lo = (int)(t_at % ntile);
    const int tile_hi = (int)min((int64_t)ntile, tile_lo + (t_end - t_at));
    const int64_t r0 = j0 + t_at / ntile * kU5R;
    t_at += tile_hi - tile_lo;
    const int64_t rw = r0 + wave * 16 + idx;  // this lane's C row
    // C element (rw, c0 + 16 i + 4 q + g): base column pointer uniform, the row
    // and the lane group's column in the offset (rows past m read row m - 1)
    const uint32_t coff = (uint32_t)((min(rw, m - 1) - r0 + g * ld) * 8);
    double v[kQrOB / 4];  // V(rw, 4 t + g)
    // first column of a tile (the last one shifted to end at c_end)
    auto tile_col = [&](int tile) { return min(cbeg + (int64_t)tile * kU5C, c_end - kU5C); };
    // Wn tile: thread (wave, lane) stages rows wave + 8 h (h = 0..15), column lane
    const uint32_t woff = (uint32_t)lane * 8u;
    const uint32_t wbytes = (uint32_t)(kQrOB * nct * 8);
    auto load_w = [&](int tile, int h) {
      const auto rs = uniform_rsrc(
          Wn + (tile_col(min(tile, tile_hi - 1)) - j0) + (int64_t)wave * nct, wbytes);
      return buf_ld(rs, woff, (uint32_t)(8 * h * nct * 8));
    };
    auto store_w = [&](int buf, int h, double x) {
      const int k = wave + 8 * h;
      sW[buf][k][lane ^ ((k & 1) << 4)] = x;
    };
    // C (rows r0.., a tile's 64 columns) as four 16-column groups i: lane holds
    // (rw, c0 + 16 i + 4 q + g) in q; reads of rows past m read row m - 1
    const uint32_t cbytes = (uint32_t)(kU5C * ld * 8);  // a tile's extent from its base
    auto load_c = [&](int tile, int e) {
      const auto rs = uniform_rsrc(A + r0 + tile_col(min(tile, tile_hi - 1)) * ld, cbytes);
      return buf_ld(rs, coff, (uint32_t)(4 * e * ld * 8));
    };
    // Stores of a tile through a buffer resource based at its first column: a
    // lane that must not write (row past m, or a column the shifted last tile
    // shares with the previous one) gets an offset past the buffer's end, which
    // the hardware drops.  The tile before the first stores nothing.
    auto store_c = [&](int tile, int e, double x) {
      const int64_t c0 = tile_col(max(tile, tile_lo));
      const int shift = tile < tile_lo ? kU5C : (int)(cbeg + (int64_t)tile * kU5C - c0);
      const bool ok = rw < m && 4 * e + g >= shift;
      buf_st(x, uniform_rsrc(A + r0 + c0 * ld, cbytes), ok ? coff : kDropOffset,
             (uint32_t)(4 * e * ld * 8));
    };
    // a lane reads Wn row 4 t + g, columns 16 i + idx; odd rows are half-swapped
    const int sw = (g & 1) << 4;
    d4v nxt[4], acc0[4], acc1[4];
    double wst[8];
    // One tile: acc = nxt - V Wn, with the accesses of its neighbours spread over
    // the 32 steps of four products: the next tile's Wn (two halves of eight
    // registers) and C, then the stores of the previous tile's result.
    auto step = [&](int tile, int buf, d4v (&acc)[4], const d4v (&out)[4]) {
      const double* wb = &sW[buf][g][idx];
      double a[2][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[0][i] = wb[(i * 16) ^ sw];
#pragma unroll
      for (int t = 0; t < kQrOB / 4; ++t) {
        if (t + 1 < kQrOB / 4) {
#pragma unroll
          for (int i = 0; i < 4; ++i) a[(t + 1) & 1][i] = wb[(t + 1) * 4 * kU5C + ((i * 16) ^ sw)];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i] = mfma_f64(a[t & 1][i], v[t], t == 0 ? nxt[i] : acc[i]);
        if (t < 8) wst[t] = load_w(tile + 1, t);
        if (t >= 1 && t < 17) nxt[(t - 1) / 4][(t - 1) % 4] = load_c(tile + 1, t - 1);
        if (t >= 16 && t < 24) {
          store_w(buf ^ 1, t - 16, wst[t - 16]);
          wst[t - 16] = load_w(tile + 1, t - 8);
        }
        if (t >= 8 && t < 24) store_c(tile - 1, t - 8, out[(t - 8) / 4][(t - 8) % 4]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int h = 0; h < 8; ++h) store_w(buf ^ 1, 8 + h, wst[h]);
      lds_barrier();
    };
    {
      double w0[16];
#pragma unroll
      for (int h = 0; h < 16; ++h) w0[h] = load_w(tile_lo, h);
#pragma unroll
      for (int t = 0; t < kQrOB / 4; ++t)
        v[t] = buf_ld(uniform_rsrc(A + r0 + (j0 + 4 * t) * ld, (uint32_t)(4 * ld * 8)), coff, 0u);
#pragma unroll
      for (int e = 0; e < 16; ++e) nxt[e / 4][e % 4] = load_c(tile_lo, e);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < 16; ++h) store_w(0, h, w0[h]);
      const int64_t rr = rw - j0;
#pragma unroll
      for (int t = 0; t < kQrOB / 4; ++t) {
        const int k = 4 * t + g;
        v[t] = rw >= m || rr < k ? 0.0 : (rr == k ? 1.0 : v[t]);
      }
    }
    // nothing of the prologue may be left in flight at the loop head: a pending
    // load there would make the wait at the head of every tile wait for the
    // previous tile's accesses as well
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    int tile = tile_lo;
#pragma clang loop unroll(disable)
    for (; tile + 1 < tile_hi; tile += 2) {
      step(tile, 0, acc0, acc1);
      step(tile + 1, 1, acc1, acc0);
    }
    if (tile < tile_hi) {
      step(tile, 0, acc0, acc1);
#pragma unroll
      for (int e = 0; e < 16; ++e) store_c(tile, e, acc0[e / 4][e % 4]);
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) store_c(tile - 1, e, acc1[e / 4][e % 4]);
    }
  }
}

// ------------------------------------------------------- triangular solves ----
// One workgroup of 16 waves solves R x = z (TRANS = false, back substitution) or
// R^T x = z (TRANS = true, forward substitution), R upper triangular, col-major (ld).
// Blocks of 64 unknowns: the 64 x 64 diagonal block is staged in LDS and solved by
// wave 0 (one unknown per lane, the solved value broadcast by a lane shuffle); the
// off-diagonal part is a GEMV over all 16 waves.  x lives in LDS (n doubles).
// A zero or non-finite diagonal entry sets GAP_DEVERR_RANK (if dev_err).
template <bool TRANS>
GAP_DEV void trsv_blk_lds(const double* __restrict__ R, int64_t ld, int64_t n, double* xs,
                          double (&T)[64][65], int* dev_err) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t nb = (n + 63) / 64;
  for (int64_t b = 0; b < nb; ++b) {
    const int64_t blk = TRANS ? b : nb - 1 - b;
    const int64_t j0 = blk * 64;
    const int w = (int)min((int64_t)64, n - j0);
    __syncthreads();
    for (int e = tid; e < 64 * 64; e += 1024) {
      const int r = e & 63, c = e >> 6;
      T[r][c] = (r < w && c < w && r <= c) ? R[(j0 + r) + (j0 + c) * ld] : 0.0;
    }
    if (TRANS) {
      // x_j -= sum_{i < j0} R[i][j] x_i for the block's columns (left-looking)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cj = wave * 4 + q;
        if (cj < w) {
          const double* col = R + (j0 + cj) * ld;
          double s = 0.0;
          for (int64_t i = lane; i < j0; i += 64) s += col[i] * xs[i];
          s = wave_sum(s);
          if (lane == 0) xs[j0 + cj] -= s;
        }
      }
    }
    __syncthreads();
    if (wave == 0) {
      double t = lane < w ? xs[j0 + lane] : 0.0;
      bool bad = false;
      if (TRANS) {
        for (int c = 0; c < w; ++c) {
          const double d = T[c][c];
          bad |= (d == 0.0 || !isfinite(d));
          const double xc = __shfl(t, c) / d;
          if (lane == c) t = xc;
          else if (lane > c) t -= T[c][lane] * xc;
        }
      } else {
        for (int c = w - 1; c >= 0; --c) {
          const double d = T[c][c];
          bad |= (d == 0.0 || !isfinite(d));
          const double xc = __shfl(t, c) / d;
          if (lane == c) t = xc;
          else if (lane < c) t -= T[lane][c] * xc;
        }
      }
      if (lane < w) xs[j0 + lane] = t;
      if (bad && lane == 0 && dev_err) atomicOr(dev_err, GAP_DEVERR_RANK);
    }
    __syncthreads();
    if (!TRANS) {
      // x_i -= sum_{c in block} R[i][c] x_c for i < j0 (right-looking)
      for (int64_t i = tid; i < j0; i += 1024) {
        double s = 0.0;
#pragma unroll 8
        for (int c = 0; c < w; ++c) s += R[i + (j0 + c) * ld] * xs[j0 + c];
        xs[i] -= s;
      }
    }
  }
  __syncthreads();
}

template <bool TRANS>
__global__ __launch_bounds__(1024) void k_trsv_blk(const double* __restrict__ R, int64_t ld,
                                                   int64_t n, const double* z, double* x,
                                                   int* dev_err) {
  extern __shared__ double xs[];
  __shared__ double T[64][65];
  for (int64_t i = threadIdx.x; i < n; i += 1024) xs[i] = z[i];
  trsv_blk_lds<TRANS>(R, ld, n, xs, T, dev_err);
  for (int64_t i = threadIdx.x; i < n; i += 1024) x[i] = xs[i];
}

// Inverses of the 64 x 64 diagonal blocks of an upper-triangular matrix (col-
// major, ld) into the diagonal blocks of Y (row-major, ldy), zero below the
// diagonal: the rows of the unit matrix solved against the block, sixteen per
// wave.  One block per diagonal block.
__global__ __launch_bounds__(256) void k_trinv_diag(const double* __restrict__ R0, int64_t ld,
                                                    double* __restrict__ Y, int64_t n,
                                                    int64_t ldy, int* dev_err) {
  __shared__ double u[kTri][kTriS];
  __shared__ double inv[kInv16];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int64_t j0 = (int64_t)blockIdx.x * kTri;
  const double* R = R0 + j0 + j0 * ld;
  const int w = (int)min((int64_t)kTri, n - j0);
  for (int e = threadIdx.x; e < kTri * kTri; e += 256) {  // unit rows past the matrix
    const int r = e & 63, c = e >> 6;
    u[r][c] = (r <= c && c < w) ? R[r + c * ld] : (r == c ? 1.0 : 0.0);
  }
  __syncthreads();
  if (wave == 0) {
    const double d = u[lane][lane];
    if (d == 0.0 || !isfinite(d)) atomicOr(dev_err, GAP_DEVERR_RANK);
    tri_inv16([&](int i, int j) { return u[i][j]; }, inv);
  }
  __syncthreads();
  if (w <= 16) {  // that is all of it
    const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
    if (r < w && c < w) Y[(j0 + r) * ldy + j0 + c] = inv[threadIdx.x];
    return;
  }
  TriOps t;
  tri_ops(t, [&](int i, int j) { return u[i][j]; }, [&](int e) { return inv[e]; });
  const int row = 16 * wave + idx;
  d4v x[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) x[b][r] = row == 16 * b + g + 4 * r ? 1.0 : 0.0;
  tri_solve16(t, x);
  if (row >= w) return;
  double* y = Y + (j0 + row) * ldy + j0;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = 16 * b + g + 4 * r;
      if (c < w) y[c] = c < row ? 0.0 : x[b][r];
    }
}

// var[i] = base + sign * sum_j Z[i][j]^2 (row-major Z, one wave per row), the base
// var[i] (init 0), delta^2 (d_i . d_i)^zeta (1) or zero (2); init 3: as 1, and then
// var[i] is added.
template <typename TD>
__global__ __launch_bounds__(256) void k_var_rows(const double* __restrict__ Z, int64_t ldz,
                                                  int64_t n, int64_t m, double sign,
                                                  const TD* __restrict__ desc, int64_t ldd,
                                                  int64_t D, int zeta, double delta, int init,
                                                  double* __restrict__ var) {
  const int64_t i = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= n) return;
  double s = 0.0;
  for (int64_t j = lane; j < m; j += 64) {
    const double z = Z[i * ldz + j];
    s += z * z;
  }
  s = wave_sum(s);
  double kii = 0.0;
  if (init & 1) {
    double t = 0.0;
    for (int64_t k = lane; k < D; k += 64) {
      const double d = (double)desc[i * ldd + k];
      t += d * d;
    }
    t = wave_sum(t);
    double p = 1.0;
    for (int q = 0; q < zeta; ++q) p *= t;
    kii = delta * delta * p;
  }
  if (lane == 0) {
    const double v = (init ? kii : var[i]) + sign * s;
    var[i] = init == 3 ? v + var[i] : v;
  }
}

// Descriptors as FP64 rows [n][ldo] with zero row padding (columns D .. ldo - 1).
template <typename TD>
__global__ void k_desc_f64(const TD* __restrict__ desc, int64_t ldd, int64_t n, int64_t D,
                           double* __restrict__ out, int64_t ldo) {
  const int64_t i = blockIdx.y;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < ldo;
       k += (int64_t)gridDim.x * blockDim.x)
    out[i * ldo + k] = k < D ? (double)desc[i * ldd + k] : 0.0;
}

// CUR selection keys, padded to n_pad (a power of two) with -inf / index n_pad:
// key_i = l_i (u NULL) or log(u_i) / l_i (weighted sampling without replacement).
__global__ void k_cur_keys(const double* __restrict__ lev, const double* __restrict__ u,
                           int64_t n, int64_t n_pad, double* __restrict__ key,
                           int32_t* __restrict__ idx) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_pad;
       i += (int64_t)gridDim.x * blockDim.x) {
    double k = -HUGE_VAL;
    if (i < n) {
      const double l = lev[i];
      k = u ? (l > 0.0 ? log(u[i]) / l : -HUGE_VAL) : l;
      if (!(k == k)) k = -HUGE_VAL;  // NaN sorts last
    }
    key[i] = k;
    idx[i] = (int32_t)i;
  }
}

// One compare-exchange of a bitonic sort into decreasing key, ties by increasing
// index (a total order, so the result is unique): entries i < l = i ^ j of the
// run of length k that i belongs to.
GAP_DEV void bitonic_step(double* key, int32_t* idx, int64_t i, int64_t l, bool down) {
  const double ki = key[i], kl = key[l];
  const int32_t ii = idx[i], il = idx[l];
  const bool i_first = ki > kl || (ki == kl && ii < il);  // i precedes l in the final order
  if (down != i_first) {
    key[i] = kl;
    key[l] = ki;
    idx[i] = il;
    idx[l] = ii;
  }
}

__global__ void k_bitonic(double* __restrict__ key, int32_t* __restrict__ idx, int64_t n_pad,
                          int64_t j, int64_t k) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_pad;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = i ^ j;
    if (l > i) bitonic_step(key, idx, i, l, (i & k) == 0);
  }
}

// The stages j < kSortChunk of the runs k = k_lo, 2 k_lo, .. k_hi, a chunk of
// kSortChunk entries per block in LDS: one launch for the whole sort of up to
// 4096 entries and one per run length above (a launch per stage took 2.1 us each,
// 78 of them for 4096
// entries: 209 us for 2336 atoms, 56 in one block).
constexpr int kSortChunk = 4096;
__global__ __launch_bounds__(1024) void k_bitonic_lds(double* __restrict__ key,
                                                      int32_t* __restrict__ idx, int64_t n_pad,
                                                      int64_t k_lo, int64_t k_hi) {
  __shared__ double sk[kSortChunk];
  __shared__ int32_t si[kSortChunk];
  const int64_t base = (int64_t)blockIdx.x * kSortChunk;
  const int n = (int)min((int64_t)kSortChunk, n_pad - base);
  for (int e = threadIdx.x; e < n; e += 1024) {
    sk[e] = key[base + e];
    si[e] = idx[base + e];
  }
  for (int64_t k = k_lo; k <= k_hi; k <<= 1)
    for (int j = (int)min(k >> 1, (int64_t)(n >> 1)); j > 0; j >>= 1) {
      __syncthreads();
      for (int e = threadIdx.x; e < n / 2; e += 1024) {
        const int i = ((e & ~(j - 1)) << 1) | (e & (j - 1));
        bitonic_step(sk, si, i, i | j, ((base + i) & k) == 0);
      }
    }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += 1024) {
    key[base + e] = sk[e];
    idx[base + e] = si[e];
  }
}

// Multi-block form of the same solves: block t owns the 64 unknowns of column
// block b (b = t for the forward solve with R^T, b = nb - 1 - t for back
// substitution), so every block it depends on has a smaller index and was
// dispatched earlier; the launch is cooperative, so all blocks are resident.
// A block folds in each dependency block c as soon as c publishes its 64
// values (flag[c] == epoch): a 64 x 64 product, a quarter of R's tile per wave,
// whose entries are in registers before the wave starts to wait.  Then wave 0
// solves the diagonal block, a row (column) of it per lane in registers, and
// publishes the values with device-scope stores before the flag (cross-XCD
// exchange without an L2-flushing fence).  Waits are bounded and set
// GAP_DEVERR_SYNC on expiry, after which every wait returns at once.  Bound by
// the chain of blocks: 4.1 us a block, 13.6 us when the tile's loads and two
// barriers followed each wait and each of the 64 steps divided.
template <bool TRANS>
__global__ __launch_bounds__(256) void k_trsv_coop(const double* __restrict__ R, int64_t ld,
                                                   int64_t n, const double* z, double* x,
                                                   unsigned int* __restrict__ flag,
                                                   unsigned int epoch, int* dev_err) {
  __shared__ double T[64][65];
  __shared__ double part[4][64];
  const int nb = (int)((n + 63) / 64);
  const int b = TRANS ? (int)blockIdx.x : nb - 1 - (int)blockIdx.x;
  const int64_t j0 = (int64_t)b * 64;
  const int w = (int)min((int64_t)64, n - j0);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  for (int e = tid; e < 64 * 64; e += 256) {
    const int r = e & 63, c = e >> 6;
    T[r][c] = (r < w && c < w && r <= c) ? R[(j0 + r) + (j0 + c) * ld] : 0.0;
  }
  const int64_t me = min(j0 + lane, n - 1);
  const double zl = z[me];
  __syncthreads();
  // wave 0: this lane's row (TRANS: column) of the diagonal block
  double row[64], dg = 1.0;
  if (wave == 0) {
#pragma unroll
    for (int c = 0; c < 64; ++c) row[c] = TRANS ? T[c][lane] : T[lane][c];
    dg = lane < w ? T[lane][lane] : 1.0;
  }
  double acc = 0.0;
  const int ndep = TRANS ? b : nb - 1 - b;
  for (int d = 0; d < ndep; ++d) {
    const int c = TRANS ? d : nb - 1 - d;  // in the order the dependencies complete
    const int64_t c0 = (int64_t)c * 64 + wave * 16;
    // TRANS: unknown j0 + lane needs sum_i R[c0 + i][j0 + lane] y[c0 + i], else
    // sum_j R[j0 + lane][c0 + j] x[c0 + j]; indices past n are clamped (their
    // value is zero, or their lane is not stored)
    double t[16];
#pragma unroll
    for (int q = 0; q < 16; ++q)
      t[q] = TRANS ? R[c0 + q + me * ld] : R[me + min(c0 + q, n - 1) * ld];
    uint64_t spins = 0;
    while (__hip_atomic_load(flag + c, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != epoch) {
      if (dev_err && (__hip_atomic_load(dev_err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
                      GAP_DEVERR_SYNC))
        break;
      __builtin_amdgcn_s_sleep(1);
      if (++spins > (1ull << 22)) {
        if (dev_err && lane == 0) atomicOr(dev_err, GAP_DEVERR_SYNC);
        break;
      }
    }
    const int64_t xi = c0 + (lane & 15);
    const double xv = vload(x + min(xi, n - 1));
    const double xz = xi < n ? xv : 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc = fma(t[q], readlane_f64(xz, q), acc);
  }
  part[wave][lane] = acc;
  __syncthreads();
  if (wave == 0) {
    double t = lane < w ? zl - (((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane])
                        : 0.0;
    const bool bad = dg == 0.0 || !isfinite(dg);
    const double rinv = 1.0 / dg;
    // step c: the value of unknown c, then its share taken from the others (a
    // lane's own entry and those already solved are zero in its row)
#pragma unroll
    for (int s = 0; s < 64; ++s) {
      const int c = TRANS ? s : 63 - s;
      if (c < w) {
        const double xc = readlane_f64(t * rinv, c);
        const double u = fma(-row[c], xc, t);
        t = lane == c ? t : u;
      }
    }
    if (lane < w) xstore(x + j0 + lane, t * rinv);
    if (__any(bad) && lane == 0 && dev_err) atomicOr(dev_err, GAP_DEVERR_RANK);
    wait_mem();
    if (lane == 0) __hip_atomic_store(flag + b, epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__global__ __launch_bounds__(1024) void k_rdiag_minmax(const double* __restrict__ R, int64_t ld,
                                                       int64_t n, double* __restrict__ rd) {
  __shared__ double smin[16], smax[16];
  double lo = INFINITY, hi = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
    const double a = fabs(R[i + i * ld]);
    lo = fmin(lo, a);
    hi = fmax(hi, a);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
  if ((threadIdx.x & 63) == 0) {
    smin[threadIdx.x >> 6] = lo;
    smax[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
      lo = fmin(lo, smin[w]);
      hi = fmax(hi, smax[w]);
    }
    lo = fmin(lo, smin[0]);
    hi = fmax(hi, smax[0]);
    rd[0] = lo;
    rd[1] = hi;
  }
}

// ------------------------------------------------------------ refinement ----
// r_top[r] = (y_r - kc_r) / sigma_r;  r_bot[i] = -(U c)_i = -sum_{j >= i} L[j][i] c_j
__global__ void k_residual_top(const double* __restrict__ y, const double* __restrict__ sigma,
                               const double* __restrict__ kc, int64_t n, double* __restrict__ r) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    r[i] = (y[i] - kc[i]) / sigma[i];
}

__global__ __launch_bounds__(256) void k_residual_bot(const double* __restrict__ L, int64_t ldl,
                                                      int64_t M, const double* __restrict__ c,
                                                      double* __restrict__ rb) {
  const int64_t i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= M) return;
  double s = 0.0;
  for (int64_t j = i + lane; j < M; j += 64) s += L[j + i * ldl] * c[j];
  s = wave_sum(s);
  if (lane == 0) rb[i] = -s;
}

// g[m] += sum_{i <= m} U[i][m] r_bot[i] = sum_{i <= m} L[m][i] r_bot[i]
// 64 rows per block, 16 waves splitting i; partial sums combined in LDS in a fixed order.
__global__ __launch_bounds__(1024) void k_add_ut_r(const double* __restrict__ L, int64_t ldl,
                                                   int64_t M, const double* __restrict__ rb,
                                                   double* __restrict__ g) {
  __shared__ double part[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t mm = (int64_t)blockIdx.x * 64 + lane;
  double s = 0.0;
  if (mm < M)
    for (int64_t i = wave; i <= mm; i += 16) s += L[mm + i * ldl] * rb[i];
  part[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && mm < M) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += part[w][lane];
    g[mm] += t;
  }
}

__global__ void k_div(const double* __restrict__ a, const double* __restrict__ b, int64_t n,
                      double* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = a[i] / b[i];
}

__global__ void k_fill_f64(double* __restrict__ p, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_axpy(int64_t n, double a, const double* __restrict__ x, double* __restrict__ y) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] += a * x[i];
}

// out[0] += sum_i x_i^2 (one workgroup; fixed summation order)
__global__ __launch_bounds__(1024) void k_sumsq_add(const double* __restrict__ x, int64_t n,
                                                    double* __restrict__ out) {
  __shared__ double sp[16];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) s += x[i] * x[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sp[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sp[w];
    *out += t;
  }
}

__global__ __launch_bounds__(1024) void k_norm2(const double* __restrict__ x, int64_t n,
                                                double* __restrict__ out) {
  __shared__ double sp[16];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) s += x[i] * x[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sp[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sp[w];
    *out = sqrt(t);
  }
}

// Streamed-fit state after a fold: the top M + 1 rows of columns [0, M) keep
// R (upper triangle); what the QR left below the diagonal there (Householder
// vectors, and row M) is cleared.  With zero_corner (the initial state) row M
// of column M is cleared too.
__global__ void k_fold_tidy(double* __restrict__ T, int64_t ld, int64_t M, int zero_corner) {
  const int64_t col = blockIdx.y;
  const int64_t r0 = col < M ? col + 1 : (zero_corner ? M : M + 1);
  for (int64_t r = r0 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r <= M;
       r += (int64_t)gridDim.x * blockDim.x)
    T[r + col * ld] = 0.0;
}

__global__ void k_expand_cfg(const double* __restrict__ v, const int32_t* __restrict__ atom_cfg,
                             int64_t n, double* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t c = atom_cfg[i];
    out[i] = c >= 0 ? v[c] : 0.0;
  }
}

__global__ void k_fill_u32(unsigned int* __restrict__ p, int64_t n, unsigned int v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}


inline unsigned g256(int64_t n) { return std::max(1u, std::min(cdiv(n, 256), 65536u)); }

}  // namespace

void scale_rows(double* A, int64_t ld, int64_t n_rows, int64_t M, const double* y,
                const double* sigma, hipStream_t st) {
  if (n_rows <= 0) return;
  dim3 grid(std::min(cdiv(n_rows, 256), 4096u), (unsigned)(M + 1));
  hipLaunchKernelGGL(k_scale_rows, grid, dim3(256), 0, st, A, ld, n_rows, M, y, sigma);
}

void stack_u(double* A, int64_t ld, int64_t n_rows, int64_t M, const double* L, int64_t ldl,
             hipStream_t st) {
  dim3 grid(cdiv(M, 256), (unsigned)(M + 1));
  hipLaunchKernelGGL(k_stack_u, grid, dim3(256), 0, st, A, ld, n_rows, M, L, ldl);
}

void cholesky_lower(double* Lw, int64_t ldl, int64_t M, double jitter, const double* Kmm,
                    int64_t ldk, int* dev_err, hipStream_t st) {
  hipLaunchKernelGGL(k_chol_init, dim3(cdiv(M, 256), (unsigned)M), dim3(256), 0, st, Lw, ldl, M,
                     jitter, Kmm, ldk);
  double* inv = Lw + M * ldl;  // of the current diagonal block
  hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(256), 0, st, Lw, ldl, (int64_t)0,
                     (int)std::min<int64_t>(kTri, M), inv, dev_err);
  for (int64_t j0 = 0; j0 + kTri < M; j0 += kTri) {
    const unsigned nt = cdiv(M - j0 - kTri, kTri);
    hipLaunchKernelGGL(k_chol_panel, dim3(nt), dim3(256), 0, st, Lw, ldl, M, j0, inv);
    hipLaunchKernelGGL(k_chol_update, dim3(nt, nt), dim3(256), 0, st, Lw, ldl, M, j0, inv,
                       dev_err);
  }
}

int64_t chol_doubles(int64_t M) { return M * M + 1024; }

// Rows per slab of the 128-wide W = V^T C of rows [j0, m) and nct columns: as many
// slabs as give at most kVtcSlots blocks, two on each compute unit, so that all
// run at once and end together (blocks of one length: 688 of them take two full
// turns, and even 520 took 1.6 times as long as 504), and slabs of >= 256 rows,
// whose partials still cost less than reading V and C.  88,200 rows, 2,001 columns: 902 us
// in 688 blocks, 808 in 512.
constexpr int64_t kVtcSlots = 512;
static int64_t qr_slab_rows(int64_t m, int64_t j0, int64_t nct) {
  const int64_t rows = m - j0, n_ct = (nct + kVC - 1) / kVC;
  const int64_t n = std::max<int64_t>(kVtcSlots / n_ct, 1);
  return (std::max<int64_t>((rows + n - 1) / n, 256) + 31) / 32 * 32;
}

static int64_t qr_ldq(int64_t m) { return (m + 3) & ~int64_t(3); }

// Elements of the split-K partials buffer: the Gram partials of a panel, those of a
// dependent panel (64 x 64 per block), those of the 64-wide updates over short slabs
// (64 reflectors x 128 columns), or those of the 128-wide updates.  Both the workspace
// size and its binding use this one count.
static int64_t qr_part_elems(int64_t m, int64_t n) {
  int64_t e = std::max(((m + kNarrowSlab - 1) / kNarrowSlab + 1) * (int64_t)kQrNB * 2 * kQrNB,
                       (int64_t)std::max(kGramMaxBlocks * kGram, kPanelMaxGrid * kTri * kTri));
  for (int64_t j0 = 0; j0 < n; j0 += kQrOB) {
    const int64_t nct = n + 1 - j0, slab = qr_slab_rows(m, j0, nct);
    e = std::max(e, (m - j0 + slab - 1) / slab * kQrOB * nct);
  }
  return e;
}

size_t qr_workspace_bytes(int64_t m, int64_t n) {
  const int64_t ncols = n + 1;
  size_t d = 0;
  d += (size_t)qr_part_elems(m, n);            // part
  d += (size_t)kQrOB * ncols * 2;              // W, Wt
  d += (size_t)kQrOB * kQrOB;                  // T
  d += (size_t)kTri * qr_ldq(m);               // Q of a panel
  d += (size_t)kPanDoubles;                    // pan
  d += (size_t)4 * kTri * (kPanelMaxGrid + 1); // red and piv of panel_columns
  d += (size_t)n + 8;                          // tau
  return d * sizeof(double) + sizeof(unsigned int) * (kCounterWords + kTrsvMaxBlocks);  // counters, flags
}

void qr_bind_workspace(void* base, int64_t m, int64_t n, QrWork* w) {
  const int64_t ncols = n + 1;
  double* p = reinterpret_cast<double*>(base);
  auto take = [&](int64_t k) {
    double* q = p;
    p += k;
    return q;
  };
  w->Q = take(kTri * qr_ldq(m));  // (first: 32-byte aligned columns)
  w->pan = take(kPanDoubles);
  w->part_elems = qr_part_elems(m, n);
  w->part = take(w->part_elems);
  w->W = take(kQrOB * ncols);
  w->Wt = take(kQrOB * ncols);
  w->T = take(kQrOB * kQrOB);
  w->red = take(4 * kTri * (kPanelMaxGrid + 1));
  w->tau = take(n + 8);
  w->counter = reinterpret_cast<unsigned int*>(p);
  w->flags = w->counter + kCounterWords;
}

// Compact-WY update of columns [c0, c_end) with the pw reflectors stored in
// columns [j0, j0 + pw): W = V^T A[j0:m, j0:c_end), then A[j0:m, j0 + pw:c_end) -=
// V (T^T W) with the panel's T.
static void qr_wy_update(double* A, int64_t ld, int64_t m, int64_t j0, int pw, int64_t c_end,
                         QrWork* w, hipStream_t st) {
  const int64_t nct = c_end - j0;
  if (nct <= pw) return;
  {
    // Short slabs: a 64-wide update has one column tile, so the slabs alone
    // must give enough blocks to fill the device; the many partials are summed
    // by the multi-block row reduction.
    const int64_t nslab = (m - j0 + kNarrowSlab - 1) / kNarrowSlab;
    const int64_t n_ct = (nct + kVC - 1) / kVC;
    const int64_t total = nslab * n_ct, per_xcd = (total + 7) / 8;
    hipLaunchKernelGGL(k_qr_vtc2, dim3((unsigned)(8 * per_xcd)), dim3(512), 0, st, A, ld, m, j0,
                       pw, nct, (int64_t)kNarrowSlab, n_ct, total, per_xcd, w->part);
    reduce_rows_f64(w->part, nslab, (int64_t)pw * nct, w->W, st);
  }
  hipLaunchKernelGGL(k_qr_wt, dim3(cdiv(nct - pw, 64)), dim3(256), 0, st, w->W, nct, pw, w->T,
                     w->Wt);
  hipLaunchKernelGGL(k_qr_upd<kQrNB>, dim3(cdiv(m - j0, kUR)), dim3(512), 0, st, A, ld, m, j0, pw,
                     c_end, nct, w->Wt, w->counter);
}

// The same update for an outer block of up to kQrOB reflectors.
static void qr_wy_update_ob(double* A, int64_t ld, int64_t m, int64_t j0, int pw, int64_t c_end,
                            QrWork* w, hipStream_t st) {
  const int64_t nct = c_end - j0;
  if (nct <= pw) return;
  const int64_t slab = qr_slab_rows(m, j0, nct);
  const int64_t nslab = (m - j0 + slab - 1) / slab;
  const int64_t n_ct = (nct + kVC - 1) / kVC;
  const int64_t total = nslab * n_ct, per_xcd = (total + 7) / 8;
  // buffer offsets reach 128 columns of the matrix
  if ((int64_t)kVC * ld * 8 < ((int64_t)1 << 31))
    hipLaunchKernelGGL(k_qr_vtc5<true>, dim3((unsigned)(8 * per_xcd)), dim3(256), 0, st, A, ld,
                       m, j0, pw, nct, slab, n_ct, total, per_xcd, w->part);
  else
    hipLaunchKernelGGL(k_qr_vtc3<false>, dim3((unsigned)(8 * per_xcd)), dim3(512), 0, st, A, ld,
                       m, j0, pw, nct, slab, n_ct, total, per_xcd, w->part);
  reduce_rows_f64(w->part, nslab, (int64_t)pw * nct, w->W, st);
  hipLaunchKernelGGL(k_qr_larft, dim3(cdiv(pw, kQrNB)), dim3(256), 0, st, w->W, nct, pw,
                     w->tau + j0, w->T, w->counter);
  hipLaunchKernelGGL(k_qr_wt, dim3(cdiv(nct - pw, 64)), dim3(256), 0, st, w->W, nct, pw, w->T,
                     w->Wt);
  // the barrier-light kernel needs a full block, a full tile of trailing
  // columns and a 64-column tile of C within 31-bit offsets
  if (pw == kQrOB && nct - pw >= kU5C && ld < (int64_t)(1 << 22))
    hipLaunchKernelGGL(k_qr_upd5,
                       dim3((unsigned)std::min<int64_t>(
                           kU5Blocks, (int64_t)cdiv(m - j0, kU5R) * cdiv(nct - pw, kU5C))),
                       dim3(512), 0, st, A, ld, m, j0, c_end, nct, w->Wt);
  else
    hipLaunchKernelGGL(k_qr_upd3, dim3(cdiv(m - j0, kU3R)), dim3(512), 0, st, A, ld, m, j0, pw,
                       c_end, nct, w->Wt);
}

// Number of k_qr_panel_dep blocks that are co-resident on the current device (0 if unknown).
static int dep_capacity() {
  static const int cap = [] {
    int dev = 0, nb = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_qr_panel_dep, kColT, 0) == hipSuccess &&
        nb > 0)
      return std::min(nb * p.multiProcessorCount, kPanelMaxGrid);
    return 0;
  }();
  return cap;
}

// Householder factors of the bw <= 64 columns at j0, rows j0 .. m - 1, panel `half`
// of its outer block (or its state word set and nothing written).
static void qr_panel(double* A_, int64_t ld, int64_t m, int64_t j0, int bw, int half, QrWork* w,
                     hipStream_t st) {
  double* A = A_ + j0 + j0 * ld;
  const int64_t rows = m - j0, ldq = qr_ldq(m);
  unsigned int* state = w->counter + half;
  const unsigned gb = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>(kGramMaxBlocks, (rows + 127) / 128));
  auto gram = [&](const double* P, int64_t ldp) {
    hipLaunchKernelGGL(k_panel_gram, dim3(gb), dim3(256), 0, st, P, ldp, rows, bw, w->part);
    reduce_rows_f64(w->part, gb, kGram, w->pan + kPanG, st);
  };
  auto blocks = [](int64_t r) { return (unsigned)std::min<int64_t>((r + 63) / 64, kSolveBlocks); };
  const unsigned n1 = blocks(rows), n2 = rows > kTri ? blocks(rows - kTri) : 0;
  gram(A, ld);
  hipLaunchKernelGGL(k_panel_chol, dim3(1), dim3(256), 0, st, bw, half, w->pan, w->counter,
                     w->counter + kPanelBar);
  const PanelSolve q1{A, ld, w->Q, ldq, rows, bw, w->pan + kPanU1, w->pan + kPanInv1};
  hipLaunchKernelGGL(k_panel_solve, dim3(n1), dim3(256), 0, st, q1, q1, (int)n1, state);
  gram(w->Q, ldq);
  hipLaunchKernelGGL(k_panel_vectors, dim3(1), dim3(256), 0, st, A, ld, rows, bw, w->Q, ldq,
                     w->pan, w->tau + j0, state);
  // V's other rows, and T in one block more
  const PanelSolve v{w->Q + kTri, ldq, A + kTri, ld, rows - kTri, bw, w->pan + kPanZ,
                     w->pan + kPanInvZ};
  const PanelSolve t{w->pan + kPanUS, kTri, w->T + half * kTri * kTri, kTri, kTri, kTri,
                     w->pan + kPanV1, w->pan + kPanInvV};
  hipLaunchKernelGGL(k_panel_solve, dim3(n2 + 1), dim3(256), 0, st, v, t, (int)n2, state);
}

// The outer block at o0 from its first panel on that qr_panel left undone.  The
// launch costs about 25 us even where there is none (a cooperative launch goes
// through a queue of its own), so there is one per outer block.
static void qr_undone(double* A, int64_t ld, int64_t m, int64_t o0, int ow, QrWork* w,
                      hipStream_t st, int* dev_err) {
  const int64_t rows = m - o0;
  DepArgs d{A + o0 + o0 * ld, ld, rows, ow, w->Q, qr_ldq(m), w->part, w->pan,
            w->red, w->red + 4 * kTri * kPanelMaxGrid, w->counter + kPanelBar, w->counter,
            w->tau + o0, dev_err};
  const int64_t G = std::min<int64_t>(dep_capacity(), (rows + 127) / 128);
  void* args[] = {&d};
  if (G < 1 || hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&k_qr_panel_dep),
                                          dim3((unsigned)G), dim3(kColT), args, 0,
                                          st) != hipSuccess) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_qr_panel_dep, dim3(1), dim3(kColT), 0, st, d);
  }
}

// Blocks of k_qr_panel_rr for `rows` rows: as few as hold the panel (every column costs
// one grid barrier and a reduction over the blocks' partials), 0 if they cannot be
// co-resident.
static int64_t rr_blocks(int64_t rows) {
  static const int cap = [] {
    int dev = 0, nb = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_qr_panel_rr, kRRT, 0) == hipSuccess &&
        nb > 0)
      return std::min(nb * p.multiProcessorCount, kPanelMaxGrid);
    return 0;
  }();
  const int64_t G = (rows + kRRT * kRRQ - 1) / (kRRT * kRRQ);
  return G <= cap ? G : 0;
}

// An outer block of ow <= kRRW columns; false if the wide panels have to take it.
static bool qr_narrow(double* A, int64_t ld, int64_t m, int64_t o0, int ow, QrWork* w,
                      hipStream_t st, int* dev_err) {
  int64_t rows = m - o0;
  const int64_t G = ow <= kRRW ? rr_blocks(rows) : 0;
  if (G < 1) return false;
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, w->counter, (int64_t)kCounterWords, 0u);
  double *P = A + o0 + o0 * ld, *piv = w->red + 4 * kTri * kPanelMaxGrid, *tau = w->tau + o0;
  unsigned int* arrive = w->counter + kPanelBar;
  void* args[] = {&P, &ld, &rows, &ow, &w->red, &piv, &arrive, &tau, &w->counter, &dev_err};
  if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&k_qr_panel_rr),
                                 dim3((unsigned)G), dim3(kRRT), args, 0, st) == hipSuccess)
    return true;
  (void)hipGetLastError();
  return false;
}

void qr_factor(double* A, int64_t ld, int64_t m, int64_t ncols, int64_t n, QrWork* w,
               hipStream_t st, int* dev_err, Timer* tm) {
  Timer dummy;
  if (!tm) tm = &dummy;
  // Two levels: 64-wide panels inside 128-wide outer blocks (one 64-wide compact-
  // WY update of the outer block's second half), one 128-wide update of the
  // trailing matrix per outer block; a last outer block of up to sixteen columns is
  // one panel of its own kind.
  for (int64_t o0 = 0; o0 < n; o0 += kQrOB) {
    const int ow = (int)std::min<int64_t>(kQrOB, n - o0);
    tm->begin(TM_QR_PANEL);
    const bool narrow = qr_narrow(A, ld, m, o0, ow, w, st, dev_err);
    tm->end(TM_QR_PANEL);
    for (int64_t j0 = o0; !narrow && j0 < o0 + ow; j0 += kQrNB) {
      const int bw = (int)std::min<int64_t>(kQrNB, o0 + ow - j0);
      tm->begin(TM_QR_PANEL);
      qr_panel(A, ld, m, j0, bw, j0 > o0 ? 1 : 0, w, st);
      tm->end(TM_QR_PANEL);
      if (j0 + bw >= o0 + ow) continue;
      // rest of the outer block with this 64-wide block's reflectors
      tm->begin(TM_QR_UPDATE);
      qr_wy_update(A, ld, m, j0, bw, o0 + ow, w, st);
      tm->end(TM_QR_UPDATE);
    }
    if (!narrow) {
      tm->begin(TM_QR_PANEL);
      qr_undone(A, ld, m, o0, ow, w, st, dev_err);
      tm->end(TM_QR_PANEL);
    }
    if (o0 + ow >= ncols) continue;
    tm->begin(TM_QR_UPDATE);
    qr_wy_update_ob(A, ld, m, o0, ow, ncols, w, st);
    tm->end(TM_QR_UPDATE);
  }
}

// One triangular solve: the multi-block kernel when flags are given and it can
// be launched cooperatively, else the one-workgroup kernel.  x may alias z only
// for the one-workgroup form (it reads z into LDS first); the multi-block form
// reads z[j] only in the block that writes x[j], before it writes it.
static void trsv(bool trans, const double* A, int64_t ld, int64_t n, const double* z, double* x,
                 unsigned int* flags, int* dev_err, hipStream_t st) {
  const int nb = (int)((n + 63) / 64);
  if (flags && nb <= kTrsvMaxBlocks) {
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, flags, (int64_t)nb, 0u);
    unsigned int ep = 1;
    const double* A_ = A;
    int64_t ld_ = ld, n_ = n;
    const double* z_ = z;
    double* x_ = x;
    unsigned int* f_ = flags;
    int* e_ = dev_err;
    void* args[] = {&A_, &ld_, &n_, &z_, &x_, &f_, &ep, &e_};
    const void* kern = trans ? reinterpret_cast<const void*>(&k_trsv_coop<true>)
                             : reinterpret_cast<const void*>(&k_trsv_coop<false>);
    if (hipLaunchCooperativeKernel(kern, dim3((unsigned)nb), dim3(256), args, 0, st) ==
        hipSuccess)
      return;
    (void)hipGetLastError();
  }
  if (trans)
    hipLaunchKernelGGL(k_trsv_blk<true>, dim3(1), dim3(1024), (size_t)n * sizeof(double), st, A,
                       ld, n, z, x, dev_err);
  else
    hipLaunchKernelGGL(k_trsv_blk<false>, dim3(1), dim3(1024), (size_t)n * sizeof(double), st, A,
                       ld, n, z, x, dev_err);
}

void back_substitute(const double* A, int64_t ld, int64_t n, const double* z, double* x,
                     double* rd, int* dev_err, hipStream_t st, unsigned int* flags) {
  hipLaunchKernelGGL(k_rdiag_minmax, dim3(1), dim3(1024), 0, st, A, ld, n, rd);
  trsv(false, A, ld, n, z, x, flags, dev_err, st);
}

void seminormal_solve(const double* A, int64_t ld, int64_t n, double* x, hipStream_t st,
                      unsigned int* flags, double* tmp, int* dev_err) {
  // R^T y = x, then R x = y; the multi-block form needs y apart from x
  if (flags && tmp) {
    trsv(true, A, ld, n, x, tmp, flags, dev_err, st);
    trsv(false, A, ld, n, tmp, x, flags, dev_err, st);
  } else {
    trsv(true, A, ld, n, x, x, nullptr, nullptr, st);
    trsv(false, A, ld, n, x, x, nullptr, nullptr, st);
  }
}

void residual_top(const double* y, const double* sigma, const double* kc, int64_t n_rows,
                  double* r_top, hipStream_t st) {
  if (n_rows <= 0) return;
  hipLaunchKernelGGL(k_residual_top, dim3(g256(n_rows)), dim3(256), 0, st, y, sigma, kc, n_rows,
                     r_top);
}

void residual_bot(const double* L, int64_t ldl, int64_t M, const double* c, double* r_bot,
                  hipStream_t st) {
  hipLaunchKernelGGL(k_residual_bot, dim3(cdiv(M, 4)), dim3(256), 0, st, L, ldl, M, c, r_bot);
}

void add_ut_r(const double* L, int64_t ldl, int64_t M, const double* r_bot, double* g,
              hipStream_t st) {
  if (M <= 0) return;
  hipLaunchKernelGGL(k_add_ut_r, dim3(cdiv(M, 64)), dim3(1024), 0, st, L, ldl, M, r_bot, g);
}

void div_sigma(const double* r_top, const double* sigma, int64_t n, double* v, hipStream_t st) {
  hipLaunchKernelGGL(k_div, dim3(g256(n)), dim3(256), 0, st, r_top, sigma, n, v);
}

void fill_f64(double* p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_f64, dim3(g256(n)), dim3(256), 0, st, p, n, v);
}

void axpy_f64(int64_t n, double a, const double* x, double* y, hipStream_t st) {
  hipLaunchKernelGGL(k_axpy, dim3(g256(n)), dim3(256), 0, st, n, a, x, y);
}

void norm2_f64(const double* x, int64_t n, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_norm2, dim3(1), dim3(1024), 0, st, x, n, out);
}

void sumsq_add_f64(const double* x, int64_t n, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_sumsq_add, dim3(1), dim3(1024), 0, st, x, n, out);
}

// Y = R^-1 for an upper-triangular matrix of order n, by doubling: with the inverses
// of two neighbouring s x s diagonal blocks,
//   [R11 R12; 0 R22]^-1 = [Y11, -Y11 R12 Y22; 0, Y22],
// two products per level for all pairs of blocks at once (tmp: n * ldy doubles).
// A substitution per column and workgroup, the form this replaces, re-read the
// whole triangle for every column: 2.3 ms at n = 2000, now 0.17.
void trinv_upper(const double* R, int64_t ld, double* Y, int64_t n, int64_t ldy, double* tmp,
                 int* dev_err, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_trinv_diag, dim3(cdiv(n, kTri)), dim3(256), 0, st, R, ld, Y, n, ldy,
                     dev_err);
  for (int64_t s = kTri; s < n; s *= 2) small_trinv_level(R, ld, Y, ldy, n, s, tmp, st);
}

void var_rows(const double* Z, int64_t ldz, int64_t n, int64_t m, double sign, const void* desc,
              bool desc_f32, int64_t ldd, int64_t D, int zeta, double delta, int init,
              double* var, hipStream_t st) {
  if (n <= 0) return;
  dim3 grid(cdiv(n, 4));
  if (desc_f32)
    hipLaunchKernelGGL(k_var_rows<float>, grid, dim3(256), 0, st, Z, ldz, n, m, sign,
                       reinterpret_cast<const float*>(desc), ldd, D, zeta, delta, init, var);
  else
    hipLaunchKernelGGL(k_var_rows<double>, grid, dim3(256), 0, st, Z, ldz, n, m, sign,
                       reinterpret_cast<const double*>(desc), ldd, D, zeta, delta, init, var);
}

void desc_f64(const void* desc, bool desc_f32, int64_t ldd, int64_t n, int64_t D, double* out,
              int64_t ldo, hipStream_t st) {
  if (n <= 0) return;
  dim3 grid(cdiv(ldo, 256), (unsigned)n);
  if (desc_f32)
    hipLaunchKernelGGL(k_desc_f64<float>, grid, dim3(256), 0, st,
                       reinterpret_cast<const float*>(desc), ldd, n, D, out, ldo);
  else
    hipLaunchKernelGGL(k_desc_f64<double>, grid, dim3(256), 0, st,
                       reinterpret_cast<const double*>(desc), ldd, n, D, out, ldo);
}

int64_t cur_pad(int64_t n) {
  int64_t p = 1;
  while (p < n) p <<= 1;
  return p;
}

void cur_select_sort(const double* lev, const double* u, int64_t n, double* key, int32_t* idx,
                     hipStream_t st) {
  const int64_t n_pad = cur_pad(n);
  const unsigned grid = std::max(1u, std::min(cdiv(n_pad, 256), 65536u));
  hipLaunchKernelGGL(k_cur_keys, dim3(grid), dim3(256), 0, st, lev, u, n, n_pad, key, idx);
  const dim3 chunks(cdiv(n_pad, kSortChunk));
  hipLaunchKernelGGL(k_bitonic_lds, chunks, dim3(1024), 0, st, key, idx, n_pad, int64_t(2),
                     std::min<int64_t>(n_pad, kSortChunk));
  for (int64_t k = 2 * kSortChunk; k <= n_pad; k <<= 1) {
    for (int64_t j = k >> 1; j >= kSortChunk; j >>= 1)
      hipLaunchKernelGGL(k_bitonic, dim3(grid), dim3(256), 0, st, key, idx, n_pad, j, k);
    hipLaunchKernelGGL(k_bitonic_lds, chunks, dim3(1024), 0, st, key, idx, n_pad, k, k);
  }
}

void fold_tidy(double* T, int64_t ld, int64_t M, bool zero_corner, hipStream_t st) {
  // column M has rows > M only below the state, so it needs no clearing unless
  // the corner itself is reset
  dim3 grid(cdiv(M + 1, 256), (unsigned)(M + 1));
  hipLaunchKernelGGL(k_fold_tidy, grid, dim3(256), 0, st, T, ld, M, zero_corner ? 1 : 0);
}

void expand_cfg(const double* v, const int32_t* atom_cfg, int64_t n_atoms, double* out,
                hipStream_t st) {
  hipLaunchKernelGGL(k_expand_cfg, dim3(g256(n_atoms)), dim3(256), 0, st, v, atom_cfg, n_atoms,
                     out);
}

}  // namespace gapk
