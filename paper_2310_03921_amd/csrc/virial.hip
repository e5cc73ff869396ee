// Virial observation rows of L-hat K_NM, FP64.
//
// A configuration's virial stress is a sum of partial derivatives of its local
// energies (Sec. "Theory": targets are totals of local energies or of their
// derivatives; Sec. "Theory" eq. GP_L: sigma_virial regularises such rows).
// For a homogeneous strain eps acting on the pair displacement vectors
// r_p -> (I + eps) r_p, the derivative of the local energy of atom i is
// sum over its pairs of r_p,alpha dE_i/dr_j(p),beta, so row (c, alpha, beta),
// column m is
//   K_V[(c, alpha, beta), m] = - sum_{p in c} r[p][alpha] S[src(p)][m] (J[p][beta] . x_m)
// with S = delta^2 zeta (d_i . x_m)^(zeta-1) of the pair's source atom.
//
// Work decomposition: a block owns one configuration and 64 sparse-point
// columns; its eight waves are four pair streams x two 32-column halves.  A
// stream takes the configuration's pairs 16 at a time (stream s the chunks s,
// s + 4, ...), contracts the three Jacobian rows of each pair with its columns'
// x_m on the FP64 matrix core (whole 16-deep steps load unconditionally, the
// next step's fragments ahead of the current step's matrix work; one guarded
// step covers a D that is not a multiple of 16), and accumulates the nine
// weighted sums in registers.  One cross-lane and cross-wave reduction in a
// fixed order ends the block, so results do not depend on scheduling.
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "mma_f64.h"

namespace gapk {

namespace {

constexpr int kVU = 2;  // 16-column tiles per wave; a wave pair covers the block's 64 columns
template <typename TJ>
__global__ __launch_bounds__(512) void k_virial_rows(
    const TJ* __restrict__ jac, int64_t ldj, int64_t D, const double* __restrict__ X,
    int64_t ldx, int64_t M, const double* __restrict__ S, int64_t ldS,
    const int64_t* __restrict__ cfg_ptr, const int64_t* __restrict__ pair_ptr,
    const int32_t* __restrict__ pair_src, const double* __restrict__ pair_r, int64_t n_atoms,
    int64_t n_pairs, double* __restrict__ K, int64_t ldk, int64_t n_ct, int64_t n_cfg) {
  __shared__ double red[4][9][64];
  int64_t c, ct;
  if (!xcd_group_tile(n_cfg, n_ct, c, ct)) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int stream = wave >> 1;  // pair chunks stream, stream + 4, ...
  const int64_t colbase = ct * 64 + (wave & 1) * 16 * kVU;
  const int64_t a0 = min(max(cfg_ptr[c], (int64_t)0), n_atoms);
  const int64_t a1 = min(max(cfg_ptr[c + 1], a0), n_atoms);
  const int64_t p_lo = min(max(pair_ptr[a0], (int64_t)0), n_pairs);
  const int64_t p_hi = min(max(pair_ptr[a1], p_lo), n_pairs);

  FragRowK<double> fb[kVU];
  const double* xr[kVU];
  int64_t colr[kVU];
#pragma unroll
  for (int u = 0; u < kVU; ++u) {
    colr[u] = colbase + u * 16 + idx;
    fb[u] = FragRowK<double>{X + (colr[u] < M ? colr[u] : 0) * ldx, D, colr[u] < M};
    xr[u] = X + min(colr[u], M - 1) * ldx + 4 * g;  // columns past M are never stored
  }
  double acc[9][kVU];
#pragma unroll
  for (int q = 0; q < 9; ++q)
#pragma unroll
    for (int u = 0; u < kVU; ++u) acc[q][u] = 0.0;
  const int64_t kfull = D & ~int64_t(15);  // whole 16-deep steps

  for (int64_t p0 = p_lo + 16 * stream; p0 < p_hi; p0 += 64) {
    // pairs past the configuration read its last pair's rows (never accumulated)
    const int64_t p = min(p0 + idx, p_hi - 1);
    const TJ* jr = jac + p * 3 * ldj + 4 * g;
    d4v G[3][kVU];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int u = 0; u < kVU; ++u) G[b][u] = zero4();
    // whole 16-deep steps with unconditional loads, the next step's fragments
    // loaded before this step's matrix work; then one guarded tail step
    double a[2][3][4], bx[2][kVU][4];
    auto load = [&](int64_t k0, int st) {
#pragma unroll
      for (int b = 0; b < 3; ++b) load4u(jr + b * ldj + k0, a[st][b]);
#pragma unroll
      for (int u = 0; u < kVU; ++u) load4u(xr[u] + k0, bx[st][u]);
    };
    auto step = [&](int st) {
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
          for (int u = 0; u < kVU; ++u) G[b][u] = mfma_f64(a[st][b][s4], bx[st][u][s4], G[b][u]);
    };
    int64_t k0 = 0;
    if (kfull > 0) load(0, 0);
    for (; k0 + 32 <= kfull; k0 += 32) {
      load(k0 + 16, 1);
      step(0);
      if (k0 + 32 < kfull) load(k0 + 32, 0);
      step(1);
    }
    if (k0 < kfull) {  // an odd number of whole steps: the last one is loaded in set 0
      step(0);
      k0 += 16;
    }
    if (k0 < D) {
      const TJ* jt = jac + p * 3 * ldj;
#pragma unroll
      for (int b = 0; b < 3; ++b) FragRowK<TJ>{jt + b * ldj, D, true}.frag(k0, g, a[0][b]);
#pragma unroll
      for (int u = 0; u < kVU; ++u) fb[u].frag(k0, g, bx[0][u]);
      step(0);
    }
    // C layout: lane holds pairs p0 + g + 4 r of each tile's column idx
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t pr = p0 + g + 4 * r;
      if (pr >= p_hi) continue;
      const int32_t src = pair_src[pr];
      if (src < 0 || src >= n_atoms) continue;
      const double rv[3] = {pair_r[3 * pr], pair_r[3 * pr + 1], pair_r[3 * pr + 2]};
#pragma unroll
      for (int u = 0; u < kVU; ++u) {
        const double sv = colr[u] < M ? S[(int64_t)src * ldS + colr[u]] : 0.0;
#pragma unroll
        for (int al = 0; al < 3; ++al)
#pragma unroll
          for (int b = 0; b < 3; ++b) acc[3 * al + b][u] += rv[al] * sv * G[b][u][r];
      }
    }
  }
  // sum the four lane groups (pair rows), then the four pair streams
#pragma unroll
  for (int q = 0; q < 9; ++q)
#pragma unroll
    for (int u = 0; u < kVU; ++u) {
      acc[q][u] += __shfl_xor(acc[q][u], 16);
      acc[q][u] += __shfl_xor(acc[q][u], 32);
    }
  if (g == 0) {
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
      for (int u = 0; u < kVU; ++u) red[stream][q][(wave & 1) * 16 * kVU + u * 16 + idx] = acc[q][u];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int64_t col = ct * 64 + threadIdx.x;
    if (col < M) {
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const double t = red[0][q][threadIdx.x] + red[1][q][threadIdx.x] +
                         red[2][q][threadIdx.x] + red[3][q][threadIdx.x];
        K[(9 * c + q) + col * ldk] = -t;
      }
    }
  }
}

// Unconditional 4-wide loads of a Jacobian row segment (32-byte aligned).
GAP_DEV void ldj4(const double* p, double out[4]) {
  const d4v v = *reinterpret_cast<const d4v*>(p);
  out[0] = v[0]; out[1] = v[1]; out[2] = v[2]; out[3] = v[3];
}
GAP_DEV void ldj4(const float* p, double out[4]) {
  const f4v v = *reinterpret_cast<const f4v*>(p);
  out[0] = v[0]; out[1] = v[1]; out[2] = v[2]; out[3] = v[3];
}

// The same rows for D <= 256 with the block's 64 columns of X resident in LDS for
// its lifetime, stored in the matrix core's operand order (as in the force-row
// kernel): twelve waves, wave w taking Jacobian component beta = w % 3 of pair
// stream w / 3, so three waves share a SIMD.  Every load in the pair loop reads
// a valid address (pairs past the configuration read its last pair, whose second
// share of the sums is left out by selection; k blocks past D the row's last four
// elements against zero rows of X, or for D % 4 != 0 (RAGGED), where the row's
// padding may hold anything, zeros in their place; columns past M are never
// stored); the next k block's (or the next chunk's first) Jacobian fragment is
// loaded before the current block's matrix work.
constexpr int kVNC = 4;  // 16-column tiles per block
constexpr int kVNG = 4;  // pair streams
constexpr int kVMaxKb = 16;  // D <= 256
template <typename TJ, bool RAGGED>
__global__ __launch_bounds__(192 * kVNG) void k_virial_rows_lds(
    const TJ* __restrict__ jac, int64_t ldj, int64_t D, const double* __restrict__ X,
    int64_t ldx, int64_t M, const double* __restrict__ S, int64_t ldS,
    const int64_t* __restrict__ cfg_ptr, const int64_t* __restrict__ pair_ptr,
    const int32_t* __restrict__ pair_src, const double* __restrict__ pair_r, int64_t n_atoms,
    int64_t n_pairs, double* __restrict__ K, int64_t ldk, int64_t n_ct, int64_t n_cfg, int nkb,
    int64_t slice) {
  extern __shared__ double xs[];  // [nkb][kVNC][2 halves][64 lanes][2]
  __shared__ double red[kVNG][9][16 * kVNC];
  int64_t c, ct;
  if (!xcd_group_tile(n_cfg, n_ct, c, ct)) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, idx = lane & 15;
  const int beta = wave % 3, stream = wave / 3;
  const int64_t colbase = ct * (16 * kVNC);
  for (int e = threadIdx.x; e < nkb * kVNC * 64; e += 192 * kVNG) {
    const int kb = e / (kVNC * 64), rem = e % (kVNC * 64);
    const int u = rem / 64, ln = rem % 64;
    const int64_t col = colbase + kVNC * (ln & 15) + u;  // lane idx of tile u: column kVNC idx + u
    double v[4];
    if (col < M)
      load4(X + col * ldx, (int64_t)kb * 16 + 4 * (ln >> 4), D, v);
    else
      zero_frag(v);
    const d2v lo = {v[0], v[1]}, hi = {v[2], v[3]};
    double* t = xs + (size_t)(e >> 6) * 256 + 2 * (e & 63);
    *reinterpret_cast<d2v*>(t) = lo;
    *reinterpret_cast<d2v*>(t + 128) = hi;
  }
  __syncthreads();

  const int64_t a0 = min(max(cfg_ptr[c], (int64_t)0), n_atoms);
  const int64_t a1 = min(max(cfg_ptr[c + 1], a0), n_atoms);
  const int64_t p_lo = min(max(pair_ptr[a0], (int64_t)0), n_pairs);
  const int64_t p_hi = min(max(pair_ptr[a1], p_lo), n_pairs);
  const int64_t kmax4 = RAGGED ? (D + 3) / 4 * 4 - 4 : D - 4;
  auto cut = [&](int kb, double a[4]) {  // the k block's entries past D
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = kb * 16 + 4 * g + q < D ? a[q] : 0.0;
  };
  const int64_t scol = min(colbase + kVNC * idx, ldS - kVNC);
  double acc[3][kVNC];
#pragma unroll
  for (int al = 0; al < 3; ++al)
#pragma unroll
    for (int u = 0; u < kVNC; ++u) acc[al][u] = 0.0;
  const d2v* xb = reinterpret_cast<const d2v*>(xs) + lane;
  auto xfrag = [&](int tile) -> d4v {
    const d2v lo = xb[tile * 128], hi = xb[tile * 128 + 64];
    const d4v f = {lo[0], lo[1], hi[0], hi[1]};
    return f;
  };
  // slice blockIdx.y of the configuration's chunks of pairs
  const int64_t step = 16 * kVNG * (int64_t)gridDim.y;
  const int64_t p_first = p_lo + 16 * (kVNG * (int64_t)blockIdx.y + stream);
  if (p_first < p_hi) {
    auto row_of = [&](int64_t p0) -> const TJ* {
      return jac + min(p0 + idx, p_hi - 1) * 3 * ldj + beta * ldj;
    };
    int64_t p0 = p_first;
    const TJ* jr = row_of(p0);
    double fa[4], fb[4];
    ldj4(jr + min((int64_t)4 * g, kmax4), fa);
    for (; p0 < p_hi; p0 += step) {
      const int64_t pn = p0 + step;
      const TJ* jn = row_of(pn < p_hi ? pn : p0);
      d4v G[kVNC];
#pragma unroll
      for (int u = 0; u < kVNC; ++u) G[u] = zero4();
      for (int kb = 0; kb < nkb; kb += 2) {  // nkb is even
        ldj4(jr + min((int64_t)(kb + 1) * 16 + 4 * g, kmax4), fb);
        if (RAGGED) cut(kb, fa);
        {
          d4v b[kVNC];
#pragma unroll
          for (int u = 0; u < kVNC; ++u) b[u] = xfrag(kb * kVNC + u);
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
            for (int u = 0; u < kVNC; ++u) G[u] = mfma_f64(fa[s4], b[u][s4], G[u]);
        }
        const bool more = kb + 2 < nkb;
        const TJ* jp = more ? jr + (int64_t)(kb + 2) * 16 : jn;
        ldj4(jp + min((int64_t)4 * g, kmax4 - (more ? (int64_t)(kb + 2) * 16 : 0)), fa);
        if (RAGGED) cut(kb + 1, fb);
        {
          d4v b[kVNC];
#pragma unroll
          for (int u = 0; u < kVNC; ++u) b[u] = xfrag((kb + 1) * kVNC + u);
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
            for (int u = 0; u < kVNC; ++u) G[u] = mfma_f64(fb[s4], b[u][s4], G[u]);
        }
      }
      // C layout: lane holds pairs p0 + g + 4 r of its four columns.  The gathers of all
      // four are issued before the first is used (the scheduler, left to itself, does them
      // one after the other to save registers that a block of twelve waves has anyway:
      // 30,000 atoms of 30 pairs, D 252, M 2000, 44.55 ms against 43.81).
      int32_t src[4];
      d4v sv[4];
      double rv[4][3];
      bool ok[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) src[r] = pair_src[min(p0 + g + 4 * r, p_hi - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t pr = p0 + g + 4 * r, pc = min(pr, p_hi - 1);
        ok[r] = pr < p_hi && src[r] >= 0 && src[r] < n_atoms;
        const int64_t sr = min(max((int64_t)src[r], (int64_t)0), n_atoms - 1);
        sv[r] = *reinterpret_cast<const d4v*>(S + sr * ldS + scol);
#pragma unroll
        for (int al = 0; al < 3; ++al) rv[r][al] = pair_r[3 * pc + al];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < kVNC; ++u) {
          const double w = ok[r] ? sv[r][u] * G[u][r] : 0.0;
#pragma unroll
          for (int al = 0; al < 3; ++al) acc[al][u] += rv[r][al] * w;
        }
      jr = jn;
    }
  }
  // sum the four lane groups (pair rows), then the four pair streams of each beta
#pragma unroll
  for (int al = 0; al < 3; ++al)
#pragma unroll
    for (int u = 0; u < kVNC; ++u) {
      acc[al][u] += __shfl_xor(acc[al][u], 16);
      acc[al][u] += __shfl_xor(acc[al][u], 32);
    }
  if (g == 0) {
#pragma unroll
    for (int al = 0; al < 3; ++al)
#pragma unroll
      for (int u = 0; u < kVNC; ++u) red[stream][3 * al + beta][kVNC * idx + u] = acc[al][u];
  }
  __syncthreads();
  if (threadIdx.x < 16 * kVNC) {
    const int64_t col = colbase + threadIdx.x;
    if (col < M) {
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        double t = red[0][q][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kVNG; ++w) t += red[w][q][threadIdx.x];
        K[blockIdx.y * slice + (9 * c + q) + col * ldk] = -t;
      }
    }
  }
}

}  // namespace

// Blocks that share a configuration's pairs: a block per configuration and 64
// points runs as long as the largest configuration, so where these are few they
// are cut into up to eight slices, summed in slice order (60 configurations of up
// to 70 atoms, M 301, D 150: 729 us in 300 blocks, 636 in 2 x 300, 571 in 3 x 300,
// 532 in 6 x 300, 568 in 13 x 300).  A slice takes at least one step of 64 pairs on
// average, and two where the blocks of one slice already take half the device: with less
// they only load the points once more each (12 configurations of 65 pairs, D 252, M 1000:
// 144 us in one slice, 196 in eight; of 518, M 301, 60 blocks: 177 in four, 166 in eight).
static int64_t virial_slices(int64_t n_cfg, int64_t n_pairs, int64_t M, int64_t D) {
  const int64_t blocks = std::max<int64_t>(n_cfg * ((M + 63) / 64), 1);
  if (D > 16 * kVMaxKb || blocks >= 1024) return 1;
  const int64_t slice = 16 * kVNG * (blocks < 128 ? 1 : 2) * std::max<int64_t>(n_cfg, 1);
  return std::max<int64_t>(1, std::min<int64_t>({8, 2048 / blocks, n_pairs / slice}));
}
size_t virial_part_bytes(int64_t n_cfg, int64_t n_pairs, int64_t M, int64_t D) {
  const int64_t ns = virial_slices(n_cfg, n_pairs, M, D);
  return ns > 1 ? sizeof(double) * ns * 9 * n_cfg * M : 0;
}

void virial_rows_f64(const void* jac, bool jac_f32, int64_t ldj, int64_t D, const double* X,
                     int64_t ldx, int64_t M, const double* S, int64_t ldS, const int64_t* cfg_ptr,
                     int64_t n_cfg, const int64_t* pair_ptr, const int32_t* pair_src,
                     const double* pair_r, int64_t n_atoms, int64_t n_pairs, double* K,
                     int64_t ldk, double* part, hipStream_t st) {
  if (n_cfg <= 0 || M <= 0) return;
  // the column tiles of a configuration stay on one XCD (its pairs' Jacobian
  // rows are then read from HBM once, into that XCD's L2); configurations are
  // dealt to the XCDs in turn
  const int64_t n_ct = (M + 63) / 64;
  dim3 grid(xcd_group_tile_blocks(n_cfg, n_ct));
  if (D <= 16 * kVMaxKb) {  // (S rows are padded to a multiple of four)
    const int nkb = 2 * (int)((D + 31) / 32);  // even, 16-deep blocks
    const size_t tile = (size_t)kVNC * 64 * 4 * sizeof(double);
    const int64_t ns = virial_slices(n_cfg, n_pairs, M, D);
    double* out = ns > 1 ? part : K;
    const int64_t ldo = ns > 1 ? 9 * n_cfg : ldk;
    grid.y = (unsigned)ns;
    auto go = [&](auto kern, auto j) {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(kVMaxKb * tile));
      hipLaunchKernelGGL(kern, grid, dim3(192 * kVNG), nkb * tile, st,
                         j, ldj, D, X, ldx, M, S, ldS, cfg_ptr, pair_ptr, pair_src, pair_r,
                         n_atoms, n_pairs, out, ldo, n_ct, n_cfg, nkb, 9 * n_cfg * M);
    };
    auto pick = [&](auto j) {
      using T = std::remove_const_t<std::remove_pointer_t<decltype(j)>>;
      D % 4 ? go(k_virial_rows_lds<T, true>, j) : go(k_virial_rows_lds<T, false>, j);
    };
    jac_f32 ? pick(static_cast<const float*>(jac)) : pick(static_cast<const double*>(jac));
    if (ns > 1) sum_parts_f64(part, ns, 9 * n_cfg * M, K, M, ldk, 9 * n_cfg, st);
    return;
  }
  if (jac_f32)
    hipLaunchKernelGGL(k_virial_rows<float>, grid, dim3(512), 0, st,
                       reinterpret_cast<const float*>(jac), ldj, D, X, ldx, M, S, ldS, cfg_ptr,
                       pair_ptr, pair_src, pair_r, n_atoms, n_pairs, K, ldk, n_ct, n_cfg);
  else
    hipLaunchKernelGGL(k_virial_rows<double>, grid, dim3(512), 0, st,
                       reinterpret_cast<const double*>(jac), ldj, D, X, ldx, M, S, ldS, cfg_ptr,
                       pair_ptr, pair_src, pair_r, n_atoms, n_pairs, K, ldk, n_ct, n_cfg);
}

}  // namespace gapk
