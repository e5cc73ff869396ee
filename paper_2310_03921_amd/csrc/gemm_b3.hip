// Tiled BF16x3 GEMM for the predict and backward contractions (eq. epsilon and
// its derivatives): C[i][j] = sum_k A[i][k] B[j][k], both operands K-contiguous,
// every value split hi = bf16(fp32(x)), lo = bf16(fp32(x) - hi) while it is
// staged into LDS, products hi*hi + hi*lo + lo*hi on the BF16 matrix cores with
// FP32 accumulation (see mma_bf16.h).
//
// A block computes a 256 x 256 tile of C with eight waves (64 x 128 each: four
// A and eight B fragments, thirty-two accumulators), over 32-deep k blocks
// whose split A and B halves are double-buffered in LDS in matrix-core operand
// order (128 KB).  While a k block feeds the matrix cores the next one is converted
// and staged between its products, from registers loaded a k block earlier: a
// wave can issue three vector instructions in the time of one product, so the
// conversion costs the matrix cores nothing, where staging after the products left
// them idle (65536 x 4000 x 1000, FP32: W X 1532 -> 1314 us, 1.20 PFLOP/s of
// executed products; P-stages 1746 -> 1500 and 1723 -> 1471; W^T D 1580 -> 1442.
// The matrix cores are busy 64% of the time at 1.8 GHz.  Reading the next block's
// first fragments ahead of its barrier as well changed nothing).  A 256-wide tile
// moves 64 bytes of operands per 768 BF16 flop (12,288 per k block and thread
// pair), so at the matrix cores' rate the operand stream from L2 stays near
// 15 TB/s for the whole chip; a 128-wide tile would need twice that.
//
// Epilogues:
//   kPlain   C (FP64, row-major), or a split-K partial C + z * zstride;
//   kPEnergy P-stage of predict: P = D X^T, e_part[ct][i] = sum over the
//            columns of column tile ct of c_m k(p_im), W[i][m] = delta^2 zeta c_m p^(zeta-1)
//            (FP32, the forward W, whose product with X is the descriptor gradient);
//   kPBack   P-stage of the backward: dc_part[rt][m] = sum over the rows of row tile rt of
//            g_e[i] k(p_im), W[i][m] = g_e[i] delta^2 zeta c_m p^(zeta-1) (FP32).
// An operand may also be a column view (ColOp: element (r, k) at p[k ld + r]),
// which the backward's d_X = W^T D uses for both W and the descriptors, so that
// neither is transposed in memory.
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "mma_bf16.h"

namespace gapk {

namespace {

constexpr int kGT = 256;            // tile rows and columns
constexpr int kGThreads = 512;      // eight waves: 4 (64-row quarters) x 2 (128-column halves)
constexpr int kGStage = kGT * 32;   // elements of one operand per k block
constexpr int kGStageV = kGStage / 8 * 2;   // 16-byte LDS entries of one split block
constexpr int kGLds = 4 * kGStageV * 16;   // dynamic LDS bytes of a block (128 KB)
constexpr int kGRowStep = kGThreads / 4;   // rows between a thread's two staged rows
constexpr int kPlain = 0, kPEnergy = 1, kPBack = 2;

inline unsigned cdiv_u(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

// Staging of a 256 x 32 operand block, in two halves of 128 rows.  A half's
// loads are issued one k block before its values are converted and written to
// LDS, so neither the products nor the conversion wait for memory: a load
// fetches raw values from a clamped, valid address; k past the slice end is
// replaced by zeros, by selection, when the slice's last block is staged (CHECK).
// Rows past the operand's end repeat its last row: they feed only entries of C
// that are not kept.  Values are converted to FP32 and split into 16-byte hi / lo
// halves at [tile][hi | lo][lane] (lane = row % 16 + 16 group).
template <typename TOp>
struct Stage;

// Thread t of a row operand stages row 16 (t / 64) + t % 16 (+ 128 h) and k
// group (t / 16) % 4: the 64 lanes of a wave then write 64 consecutive
// 16-byte LDS entries, where four lanes of one row with consecutive k groups
// would meet in the same banks four at a time.
GAP_DEV int stage_row(int t) { return 16 * (t >> 6) + (t & 15); }
GAP_DEV int stage_grp(int t) { return (t >> 4) & 3; }

template <bool CHECK>
GAP_DEV void stage_split(const float v[8], int kleft, bf8v* __restrict__ d) {
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (!CHECK || e < kleft) ? v[e] : 0.f;
  bf8v hi, lo;
  split8(x, hi, lo);
  d[0] = hi;
  d[64] = lo;
}

// Rows (element (r, k) at p[r ld + k], ld a multiple of 4): thread t holds rows
// stage_row(t) + 128 h, entries k0 + 8 stage_grp(t) .. + 7, as two 4-wide loads whose
// start is clamped to the last 4-group that holds entries below K.  FP64 entries
// are rounded (settle) before the other half's are loaded: raw values of both
// halves at once would not fit the registers.
template <typename T>
struct Stage<const T*> {
  const T* row[2];
  T in[sizeof(T) == 8 ? 1 : 2][8];
  float v8[2][8];   // FP64: the rounded entries
  GAP_DEV void init(const T* __restrict__ p, int64_t ld, int64_t rows, int64_t r0) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      row[h] = p + min(r0 + stage_row(threadIdx.x) + kGRowStep * h, rows - 1) * ld;
  }
  GAP_DEV void load(int h, int64_t k0, int64_t K) {
    const int64_t k4 = (K - 1) & ~(int64_t)3;
    typedef T v4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t kk = min(k0 + 8 * stage_grp(threadIdx.x) + 4 * q, k4);
      const v4 x = *reinterpret_cast<const v4*>(row[h] + kk);
#pragma unroll
      for (int e = 0; e < 4; ++e) in[sizeof(T) == 8 ? 0 : h][4 * q + e] = x[e];
    }
  }
  GAP_DEV void settle(int h) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v8[h][e] = (float)in[0][e];
    }
  }
  template <bool CHECK>
  GAP_DEV void store(int h, int64_t k0, int64_t K, bf8v* __restrict__ dst) const {
    const int t = threadIdx.x, grp = stage_grp(t), r = stage_row(t) + kGRowStep * h;
    const float* v;
    if constexpr (sizeof(T) == 8) v = v8[h];
    else v = in[h];
    stage_split<CHECK>(v, (int)min(K - k0 - 8 * grp, (int64_t)8),
                       dst + (r >> 4) * 128 + (r & 15) + 16 * grp);
  }
};

// Pre-split operand rows: hi and lo halves [rows][ld], ld a multiple of 32,
// zero padded along k; 16-byte loads of both halves, no split.
struct SplitRows {
  const __bf16* hi;
  const __bf16* lo;
};
template <>
struct Stage<SplitRows> {
  const __bf16* rh[2];
  int64_t d;   // from hi to lo
  bf8v hi[2], lo[2];
  GAP_DEV void init(const SplitRows& s, int64_t ld, int64_t rows, int64_t r0) {
    d = s.lo - s.hi;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      rh[h] = s.hi + min(r0 + stage_row(threadIdx.x) + kGRowStep * h, rows - 1) * ld +
              8 * stage_grp(threadIdx.x);
  }
  GAP_DEV void load(int h, int64_t k0, int64_t) {
    hi[h] = *reinterpret_cast<const bf8v*>(rh[h] + k0);
    lo[h] = *reinterpret_cast<const bf8v*>(rh[h] + k0 + d);
  }
  GAP_DEV void settle(int) {}
  template <bool CHECK>
  GAP_DEV void store(int h, int64_t, int64_t, bf8v* __restrict__ dst) const {
    const int t = threadIdx.x, r = stage_row(t) + kGRowStep * h;
    bf8v* d = dst + (r >> 4) * 128 + (r & 15) + 16 * stage_grp(t);
    d[0] = hi[h];
    d[64] = lo[h];
  }
};

// Column view of a row-major matrix: element (r, k) at p[k * ld + r].  Thread t
// holds rows (t & 127) + 128 h and k group 8 (t >> 7) .. + 7, one load per k,
// so that for a given k a wave's lanes read 64 consecutive r (whole 256-byte
// runs for FP32); the block lands in the same LDS places as a row operand's.
// The k group is one per wave, so a load's address is a scalar base per k and the
// lane's column.
template <typename T>
struct ColOp {
  const T* p;
};
template <typename T>
struct Stage<ColOp<T>> {
  const T* base;   // column r0
  int64_t ld;
  uint32_t col[2];   // byte offset of the lane's column from r0
  T v[2][8];
  static GAP_DEV int grp() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 7); }
  GAP_DEV void init(const ColOp<T>& op, int64_t ld_, int64_t rows, int64_t r0) {
    base = op.p + r0;
    ld = ld_;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      col[h] = (uint32_t)sizeof(T) *
               (uint32_t)min((int64_t)(threadIdx.x & 127) + kGRowStep * h, rows - 1 - r0);
  }
  GAP_DEV void load(int h, int64_t k0, int64_t K) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const char* pk = reinterpret_cast<const char*>(base + min(k0 + 8 * grp() + e, K - 1) * ld);
      v[h][e] = *reinterpret_cast<const T*>(pk + col[h]);
    }
  }
  GAP_DEV void settle(int) {}
  template <bool CHECK>
  GAP_DEV void store(int h, int64_t k0, int64_t K, bf8v* __restrict__ dst) const {
    const int r = (threadIdx.x & 127) + kGRowStep * h;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (float)v[h][e];
    stage_split<CHECK>(x, (int)min(K - k0 - 8 * grp(), (int64_t)8),
                       dst + (r >> 4) * 128 + (r & 15) + 16 * grp());
  }
};

struct EpiArgs {
  int zeta;
  double delta;
  const double* c;      // [n_b] coefficients (P-stages)
  const double* g_e;    // [n_a] upstream gradient (backward P-stage)
  float* W;             // [n_a][ldw]
  int64_t ldw;
  double* e_part;       // [column tiles][n_a]
  double* dc_part;      // [row tiles][n_b]
  double* C;            // plain: [n_a][ldc] (+ z * zstride)
  int64_t ldc;
  int64_t zstride;
};

template <typename TA, typename TB, int EPI>
__global__ __launch_bounds__(kGThreads, 1) void k_gemm_b3(TA A, int64_t lda, int64_t n_a, TB B,
                                                          int64_t ldb, int64_t n_b, int64_t K,
                                                          int64_t k_per_z, EpiArgs ep) {
  // split operand blocks, double-buffered: [A | B][buf][8 tiles x (hi | lo) x 64 lanes]
  extern __shared__ bf8v smem[];
  auto sA = [&](int buf) { return smem + buf * kGStageV; };
  auto sB = [&](int buf) { return smem + (2 + buf) * kGStageV; };
  __shared__ double red[4][kGT];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int wr = wave & 3, wc = wave >> 2;   // 64-row quarter and 128-column half of the tile
  // tiles dealt by row tile: all column tiles of a row tile run on one XCD,
  // where they share the row tile's A rows in L2
  int64_t rt, ct;
  if (!xcd_group_tile((n_a + kGT - 1) / kGT, (n_b + kGT - 1) / kGT, rt, ct)) return;
  const int64_t i0 = rt * kGT, j0 = ct * kGT;
  const int64_t kz0 = (int64_t)blockIdx.y * k_per_z;
  const int64_t kz1 = min(K, kz0 + k_per_z);
  const int nkb = (int)((kz1 - kz0 + 31) / 32);

  f4v acc[4][8];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[a][b] = zero4f();

  Stage<TA> sa;
  Stage<TB> sb;
  sa.init(A, lda, n_a, i0);
  sb.init(B, ldb, n_b, j0);
  // The products of k block kb; between them (STORE) block kb + 1 is staged from
  // registers and (LOAD) block kb + 2 is loaded into the registers it leaves.
  auto block = [&](int kb, auto check, auto st, auto ld) {
    constexpr bool CHECK = decltype(check)::value, STORE = decltype(st)::value,
                   LOAD = decltype(ld)::value;
    const int buf = kb & 1;
    const int64_t k1 = kz0 + (int64_t)(kb + 1) * 32;
    const bf8v* xa = sA(buf) + lane + wr * 4 * 128;
    const bf8v* xb = sB(buf) + lane + wc * 8 * 128;
    bf8v ah[4], al[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      ah[a] = xa[a * 128];
      al[a] = xa[a * 128 + 64];
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bf8v bh = xb[b * 128], bl = xb[b * 128 + 64];
      const int h = b / 4;
      if (b % 4 == 0) {
        if constexpr (STORE) sa.template store<CHECK>(h, k1, kz1, sA(buf ^ 1));
        if (h ? LOAD : STORE) sa.settle(h ^ 1);
        if constexpr (LOAD) sa.load(h, k1 + 32, kz1);
      } else if (b % 2 == 0) {
        if constexpr (STORE) sb.template store<CHECK>(h, k1, kz1, sB(buf ^ 1));
        if constexpr (LOAD) sb.load(h, k1 + 32, kz1);
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[a][b] = mfma_bf16(ah[a], bh, acc[a][b]);
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[a][b] = mfma_bf16(ah[a], bl, acc[a][b]);
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[a][b] = mfma_bf16(al[a], bh, acc[a][b]);
    }
    __syncthreads();
  };
  const std::true_type yes;
  const std::false_type no;
  if (nkb > 0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      sa.load(h, kz0, kz1);
      sa.settle(h);
      sb.load(h, kz0, kz1);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      sa.template store<true>(h, kz0, kz1, sA(0));
      sb.template store<true>(h, kz0, kz1, sB(0));
    }
    if (nkb > 1) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        sa.load(h, kz0 + 32, kz1);
        if (h == 0) sa.settle(0);
        sb.load(h, kz0 + 32, kz1);
      }
    }
    __syncthreads();
    int kb = 0;
    for (; kb + 2 < nkb; ++kb) block(kb, no, yes, yes);
    if (kb + 1 < nkb) {
      block(kb, yes, yes, no);
      ++kb;
    }
    block(kb, no, no, no);
  }

  // C[4 g + r][idx] of fragment (a, b): row i0 + 64 wr + 16 a + 4 g + r,
  // column j0 + 128 wc + 16 b + idx
  if constexpr (EPI == kPlain) {
    double* C = ep.C + blockIdx.y * ep.zstride;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + 64 * wr + 16 * a + 4 * g + r;
        if (i >= n_a) continue;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const int64_t j = j0 + 128 * wc + 16 * b + idx;
          if (j < n_b) C[i * ep.ldc + j] = (double)acc[a][b][r];
        }
      }
  } else {
    // The element-wise arithmetic runs in FP32: p is an FP32 accumulation of the
    // split products and W is stored in FP32, so FP64 here would only cost
    // VALU time while the matrix cores idle; each lane's partial sums over
    // its own entries are FP32, and everything past them (lanes, halves,
    // tiles) is summed in FP64.
    const float d2 = (float)(ep.delta * ep.delta);
    const int zm1 = ep.zeta - 1;
    float cf[8], cw[8];   // c_m and delta^2 zeta c_m of this lane's columns
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int64_t j = j0 + 128 * wc + 16 * b + idx;
      const double cj = j < n_b ? ep.c[j] : 0.0;
      cf[b] = (float)cj;
      cw[b] = (float)(ep.delta * ep.delta * ep.zeta * cj);
    }
    // g_e of the wave's 64 rows, one per lane, loaded ahead of every W store
    // (the stores could alias g_e as far as the compiler knows, and a load
    // issued behind them would wait for all of them to complete); row
    // 16 a + 4 g + r of the quarter is read from its lane by a shuffle
    float ge_lane = 1.f;
    if (EPI == kPBack && i0 + 64 * wr + lane < n_a) ge_lane = (float)ep.g_e[i0 + 64 * wr + lane];
    double rowsum[4][4];   // kPEnergy: [a][r] partial row sums over this lane's columns
    float colsum[8];       // kPBack: [b] partial column sums over this lane's rows
#pragma unroll
    for (int b = 0; b < 8; ++b) colsum[b] = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      // p^(zeta-1) of the 32 entries of fragment row a: one walk over the
      // exponent's bits serves all of them
      float pw[8][4], x[8][4];
#pragma unroll
      for (int b = 0; b < 8; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pw[b][r] = 1.f;
          x[b][r] = acc[a][b][r];
        }
      for (int e = zm1; e > 0; e >>= 1) {
        if (e & 1) {
#pragma unroll
          for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) pw[b][r] *= x[b][r];
        }
        if (e > 1) {
#pragma unroll
          for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) x[b][r] *= x[b][r];
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + 64 * wr + 16 * a + 4 * g + r;
        const bool iv = i < n_a;
        float* wrow = ep.W + (iv ? i : 0) * ep.ldw + j0 + 128 * wc + idx;
        const float ge = EPI == kPBack ? __shfl(ge_lane, 16 * a + 4 * g + r) : 1.f;
        float rs = 0.f;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const float pz1 = pw[b][r];
          const float kv = d2 * pz1 * acc[a][b][r];
          if (iv && j0 + 128 * wc + 16 * b + idx < n_b) {
            if (EPI == kPEnergy) rs += cf[b] * kv;
            if (EPI == kPBack) colsum[b] += ge * kv;
            wrow[16 * b] = ge * cw[b] * pz1;
          }
        }
        rowsum[a][r] = rs;
      }
    }
    if constexpr (EPI == kPEnergy) {
      // row sums over the 16 columns of each fragment (lanes idx), then the
      // two column halves of the tile in a fixed order
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int o = 1; o < 16; o <<= 1) rowsum[a][r] += __shfl_xor(rowsum[a][r], o);
        }
      if (wc == 1 && idx == 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int r = 0; r < 4; ++r) red[wr][16 * a + 4 * g + r] = rowsum[a][r];
      }
      __syncthreads();
      if (wc == 0 && idx == 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int64_t i = i0 + 64 * wr + 16 * a + 4 * g + r;
            if (i < n_a)
              ep.e_part[ct * n_a + i] = rowsum[a][r] + red[wr][16 * a + 4 * g + r];
          }
      }
    } else {
      // column sums over the 16 rows of each fragment (lanes g, r), then the
      // four row quarters in a fixed order
      double cs[8];
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        cs[b] = colsum[b];
        cs[b] += __shfl_xor(cs[b], 16);
        cs[b] += __shfl_xor(cs[b], 32);
      }
      if (g == 0) {
#pragma unroll
        for (int b = 0; b < 8; ++b) red[wr][128 * wc + 16 * b + idx] = cs[b];
      }
      __syncthreads();
      if (wr == 0 && g == 0) {
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const int sl = 128 * wc + 16 * b + idx;
          const int64_t j = j0 + sl;
          if (j < n_b)
            ep.dc_part[rt * n_b + j] = ((red[0][sl] + red[1][sl]) + red[2][sl]) + red[3][sl];
        }
      }
    }
  }
}

// out[j] = sum over z of part[z][j] (fixed order)
__global__ void k_sum_parts(const double* __restrict__ part, int64_t nz, int64_t n,
                            int64_t stride, double* __restrict__ out, int64_t rows,
                            int64_t ldo, int64_t cols) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < rows * cols;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / cols, j = e - i * cols;
    double s = 0.0;
    for (int64_t z = 0; z < nz; ++z) s += part[z * stride + i * cols + j];
    out[i * ldo + j] = s;
  }
}

// Entries of k in each of nz slices, whole k blocks: so they may be fewer than nz.
inline int64_t k_per_slice(int64_t K, int nz) { return ((K + nz - 1) / nz + 31) / 32 * 32; }

template <typename TA, typename TB, int EPI>
void launch_gemm(TA A, int64_t lda, int64_t n_a, TB B, int64_t ldb, int64_t n_b, int64_t K,
                 int nz, const EpiArgs& ep, hipStream_t st) {
  const int64_t kpz = k_per_slice(K, nz);
  const dim3 grid(xcd_group_tile_blocks(cdiv_u(n_a, kGT), cdiv_u(n_b, kGT)),
                  (unsigned)cdiv_u(K, kpz));
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_b3<TA, TB, EPI>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kGLds);
    attr = true;
  }
  hipLaunchKernelGGL((k_gemm_b3<TA, TB, EPI>), grid, dim3(kGThreads), kGLds, st, A, lda, n_a, B,
                     ldb, n_b, K, kpz, ep);
}

}  // namespace

int64_t gemm_b3_col_blocks(int64_t n_b) { return (n_b + kGT - 1) / kGT; }
int64_t gemm_b3_row_blocks(int64_t n_a) { return (n_a + kGT - 1) / kGT; }

void pstage_b3t(int mode, const void* desc, bool desc_f32, int64_t ldd, int64_t n,
                const __bf16* Xh, const __bf16* Xl, int64_t M, int64_t D, int zeta,
                double delta, const double* c, const double* g_e, float* W, int64_t ldw,
                double* e_part, double* dc_part, hipStream_t st) {
  if (n <= 0 || M <= 0) return;
  EpiArgs ep{};
  ep.zeta = zeta;
  ep.delta = delta;
  ep.c = c;
  ep.g_e = g_e;
  ep.W = W;
  ep.ldw = ldw;
  ep.e_part = e_part;
  ep.dc_part = dc_part;
  // X is taken pre-split (rows [M][split_ld(D)], hi and lo halves)
  const SplitRows xs{Xh, Xl};
  const int64_t ldp = split_ld(D);
  if (mode == 0) {
    if (desc_f32)
      launch_gemm<const float*, SplitRows, kPEnergy>(static_cast<const float*>(desc), ldd, n, xs,
                                                     ldp, M, D, 1, ep, st);
    else
      launch_gemm<const double*, SplitRows, kPEnergy>(static_cast<const double*>(desc), ldd, n,
                                                      xs, ldp, M, D, 1, ep, st);
  } else {
    if (desc_f32)
      launch_gemm<const float*, SplitRows, kPBack>(static_cast<const float*>(desc), ldd, n, xs,
                                                   ldp, M, D, 1, ep, st);
    else
      launch_gemm<const double*, SplitRows, kPBack>(static_cast<const double*>(desc), ldd, n, xs,
                                                    ldp, M, D, 1, ep, st);
  }
}

void gemm_b3_wx(const float* W, int64_t ldw, int64_t n, int64_t M, const __bf16* Xth,
                const __bf16* Xtl, int64_t D, double* out, int64_t ldo, hipStream_t st) {
  if (n <= 0 || D <= 0) return;
  EpiArgs ep{};
  ep.C = out;
  ep.ldc = ldo;
  launch_gemm<const float*, SplitRows, kPlain>(W, ldw, n, SplitRows{Xth, Xtl}, split_ld(M), D, M,
                                               1, ep, st);
}

void sum_parts_f64(const double* part, int64_t nz, int64_t stride, double* out, int64_t rows,
                   int64_t ldo, int64_t cols, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return;
  const unsigned g = std::max(1u, std::min(cdiv_u(rows * cols, 256), 65536u));
  hipLaunchKernelGGL(k_sum_parts, dim3(g), dim3(256), 0, st, part, nz, rows * cols, stride, out,
                     rows, ldo, cols);
}

void gemm_b3_wtd(const float* W, int64_t ldw, int64_t M, int64_t n, const void* desc,
                 bool desc_f32, int64_t ldd, int64_t D, double* part, int nz, double* out,
                 int64_t ldo, hipStream_t st) {
  if (M <= 0 || D <= 0) return;
  EpiArgs ep{};
  ep.C = part;
  ep.ldc = D;
  ep.zstride = M * D;
  // out[m][d] = sum_i W[i][m] desc[i][d]: both operands are column views (k = i)
  const ColOp<float> w{W};
  if (n > 0 && desc_f32)
    launch_gemm<ColOp<float>, ColOp<float>, kPlain>(
        w, ldw, M, ColOp<float>{static_cast<const float*>(desc)}, ldd, D, n, nz, ep, st);
  else if (n > 0)
    launch_gemm<ColOp<float>, ColOp<double>, kPlain>(
        w, ldw, M, ColOp<double>{static_cast<const double*>(desc)}, ldd, D, n, nz, ep, st);
  const int64_t slices = n > 0 ? cdiv_u(n, k_per_slice(n, nz)) : 0;
  sum_parts_f64(part, slices, M * D, out, M, ldo, D, st);
}

}  // namespace gapk
