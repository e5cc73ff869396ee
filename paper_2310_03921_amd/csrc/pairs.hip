// Pair-list transposition for the L-hat accumulation of force observations.
//
// The descriptor derivatives come as a source-major pair list (atom i, slot k)
// pointing at atoms j(i,k).  A force observation on atom j sums over every pair
// pointing at j (Sec. "Theory", operator L-hat), so the force-row and force
// kernels walk a target-major view.  The view is built by a counting sort: the
// per-target counting atomics also give every pair a slot in its target's
// segment, an exclusive scan gives the segments, and a rank sort of each
// segment restores increasing pair order, so the result does not depend on the
// order in which the atomics arrived.
//
// Targets are also ordered by decreasing in-degree: the force-row kernel
// processes 16 targets per wavefront, one incoming pair of each per step, and
// grouping targets of similar degree keeps those steps nearly all useful.
// Within one degree the order is increasing atom index, so the 16 targets of
// a wavefront usually come from one or two neighbouring configurations and
// their incoming pairs' Jacobian rows lie close together in memory.
#include <cmath>

#include <algorithm>

#include "common.h"
#include "launch.h"

namespace gapk {

namespace {

constexpr int kDegBuckets = 1024;
constexpr int kScanPer = 4096;      // counts scanned by one block
constexpr int64_t kRankPerPair = 4;  // a segment is rank-sorted while n^2 <= this times the pairs
// The longest segment of n_pairs pairs that is rank-sorted (one wave holds 64 at no cost).
inline int rank_longest(int64_t n_pairs) {
  int64_t n = (int64_t)std::sqrt((double)(kRankPerPair * n_pairs));
  if (n * n > kRankPerPair * n_pairs) --n;
  return (int)std::max<int64_t>(n, 64);
}
constexpr int kSmallAtoms = 1024;   // limits of the one-block form
constexpr int kSmallPer = 12;       // pairs per thread
constexpr int kSmallPairs = 1024 * kSmallPer;

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// src[p] = i for the pairs p of atom i: sixteen lanes per atom.
GAP_DEV void write_pair_src(const int64_t* __restrict__ pair_ptr, int64_t i, int64_t n_pairs,
                            int32_t* __restrict__ src, int* dev_err) {
  int64_t lo = pair_ptr[i], hi = pair_ptr[i + 1];
  if (lo < 0 || hi > n_pairs || hi < lo) {
    atomicOr(dev_err, GAP_DEVERR_INDEX);
    lo = max((int64_t)0, min(lo, n_pairs));
    hi = max(lo, min(hi, n_pairs));
  }
  for (int64_t p = lo + (threadIdx.x & 15); p < hi; p += 16) src[p] = (int32_t)i;
}

// Inclusive scan of one value per thread over the 1024 threads of a block.
template <typename T>
GAP_DEV T block_scan_1024(T v, T* wave_tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  if (lane == 63) wave_tot[wave] = v;
  __syncthreads();
  T base = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) base += (w < wave) ? wave_tot[w] : 0;
  __syncthreads();
  return v + base;
}

// How many of lanes 0 .. n - 1's w (n <= 64; the lanes from n on hold INT32_MAX) are
// below this lane's v, PER lanes a step.  Four take fewer instructions, one a shorter chain
// of them: over many blocks four are faster (580,000 targets of 70 pairs: the transposition
// 2.31 ms, 3.36 with one), for the four waves a SIMD of the one-block form one is (217
// targets of 41 pairs: the kernel 26.9 us, 28.0 with four).
template <int PER>
GAP_DEV int wave_below(int32_t w, int32_t v, int n) {
  int r = 0;
  for (int q = 0; q < n; q += PER)
#pragma unroll
    for (int e = 0; e < PER; ++e) r += __builtin_amdgcn_readlane(w, q + e) < v ? 1 : 0;
  return r;
}

// Rank sort of one segment of n distinct values by one wave, in -> out (n uniform):
// up to 64 values, and any number.
template <int PER>
GAP_DEV void wave_sort_short(const int32_t* in, int n, int32_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int32_t v = lane < n ? in[lane] : INT32_MAX;
  const int r = wave_below<PER>(v, v, n);
  if (lane < n) out[r] = v;
}
GAP_DEV void wave_sort_segment(const int32_t* in, int n, int32_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  for (int a = 0; a < n; a += 64) {
    const int32_t v = a + lane < n ? in[a + lane] : 0;
    int r = 0;
    for (int b = 0; b < n; b += 64) {
      const int32_t w = b + lane < n ? in[b + lane] : INT32_MAX;  // never below a pair index
      r += wave_below<4>(w, v, min(64, n - b));
    }
    if (a + lane < n) out[r] = v;
  }
}

// The same from the list of pairs in order: those of target j, 256 pairs a step.
// A rank sort takes 0.3 ns per n^2 (a step of 64 lane reads for 64 x 64 values), this pass
// 2 to 9 ns a pair of the whole list, so a segment passes where n^2 is above four times the
// pairs.  (One target of 600 or 640 among 100,000 pairs: 0.13 ms by rank, 0.17 by a pass.
// A line at n = 2048 made 20,000 targets of 2,500 pairs each pass over all 50M: 804 ms, 18
// by rank; and one target of 2,000 among 100,000 pairs took 2.6 ms by rank at one lane a
// step, 0.24 by a pass.)
GAP_DEV void wave_scan_segment(const int32_t* __restrict__ pair_j, int64_t n_pairs, int32_t j,
                               int32_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  int32_t at = 0;
  for (int64_t p0 = 0; p0 < n_pairs; p0 += 256) {
    int32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = pair_j[min(p0 + 64 * q + lane, n_pairs - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool mine = v[q] == j && p0 + 64 * q + lane < n_pairs;
      const uint64_t m = __ballot(mine);
      if (mine) out[at + __popcll(m & ((1ull << lane) - 1))] = (int32_t)(p0 + 64 * q + lane);
      at += __popcll(m);
    }
  }
}

// The whole transposition in one block, for lists that fit its LDS and
// registers: a molecular-dynamics cell of 64 atoms and 1,900 pairs took nine
// launches and 189 us as separate kernels (most of it the serial sort of each
// segment by one thread), and one launch here (the whole energy-and-force call
// 389 -> 233 us).  Bound by latency: one round
// trip to memory for the pair list, then LDS.
__global__ __launch_bounds__(1024) void k_pairs_small(
    const int64_t* __restrict__ pair_ptr, const int32_t* __restrict__ pair_j, int n_atoms,
    int n_pairs, int rank_max, int64_t* __restrict__ tgt_ptr, int32_t* __restrict__ tgt_pair,
    int32_t* __restrict__ pair_src, int32_t* __restrict__ order, int* dev_err) {
  __shared__ int32_t cnt[kSmallAtoms], start[kSmallAtoms + 1], wave_tot[16];
  __shared__ int32_t list[kSmallPairs];
  __shared__ int longer;  // some segment holds more than 64 pairs
  const int t = threadIdx.x, wave = t >> 6;
  int32_t jv[kSmallPer];
#pragma unroll
  for (int q = 0; q < kSmallPer; ++q) jv[q] = pair_j[min(t + 1024 * q, max(n_pairs, 1) - 1)];
  cnt[t] = 0;
  if (t == 0) longer = 0;
#pragma unroll
  for (int q = 0; q < kSmallPer; ++q)
    if (t + 1024 * q < n_pairs) pair_src[t + 1024 * q] = -1;
  __syncthreads();
  bool bad = false;
  int32_t pos[kSmallPer];
#pragma unroll
  for (int q = 0; q < kSmallPer; ++q) {
    pos[q] = -1;
    if (t + 1024 * q < n_pairs) {
      if (jv[q] < 0 || jv[q] >= n_atoms)
        bad = true;
      else
        pos[q] = atomicAdd(&cnt[jv[q]], 1);
    }
  }
  if (bad) atomicOr(dev_err, GAP_DEVERR_INDEX);
  for (int i = t >> 4; i < n_atoms; i += 64)
    write_pair_src(pair_ptr, i, n_pairs, pair_src, dev_err);
  __syncthreads();
  const int32_t c = t < n_atoms ? cnt[t] : 0;
  if (c > 64) longer = 1;
  const int32_t incl = block_scan_1024(c, wave_tot);
  start[t] = incl - c;
  if (t == 1023) start[1024] = incl;
  if (t < n_atoms) tgt_ptr[t] = incl - c;
  if (t == 1023) tgt_ptr[n_atoms] = incl;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kSmallPer; ++q)
    if (pos[q] >= 0) list[start[jv[q]] + pos[q]] = t + 1024 * q;
  __syncthreads();
  int lo = start[wave], hi = start[wave + 1];  // (entries past n_atoms hold the total)
  for (int j = wave; j < n_atoms; j += 16) {
    const int jn = min(j + 16, kSmallAtoms - 1), lo_n = start[jn], hi_n = start[jn + 1];
    const int n = __builtin_amdgcn_readfirstlane(hi - lo);
    if (n <= 64) wave_sort_short<1>(list + lo, n, tgt_pair + lo);
    lo = lo_n;
    hi = hi_n;
  }
  if (__builtin_expect(longer, 0))  // (apart: their code would slow the loop above)
    for (int j = wave; j < n_atoms; j += 16) {
      const int at = start[j], n = __builtin_amdgcn_readfirstlane(start[j + 1] - at);
      if (n > rank_max)
        wave_scan_segment(pair_j, n_pairs, j, tgt_pair + at);
      else if (n > 64)
        wave_sort_segment(list + at, n, tgt_pair + at);
    }
  for (int p = start[1024] + t; p < n_pairs; p += 1024) tgt_pair[p] = 0;  // dropped pairs
  if (order != nullptr && t < n_atoms) {
    const int32_t d = min(c, kDegBuckets - 1);
    int r = 0;
    for (int i = 0; i < n_atoms; ++i) {
      const int32_t e = min(cnt[i], kDegBuckets - 1);
      r += (e > d || (e == d && i < t)) ? 1 : 0;
    }
    order[r] = t;
  }
}

__global__ void k_pairs_init(int32_t* __restrict__ cnt, int64_t n_cnt, int32_t* __restrict__ src,
                             int64_t n_pairs) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < max(n_cnt, n_pairs);
       i += (int64_t)gridDim.x * blockDim.x) {
    if (i < n_cnt) cnt[i] = 0;
    if (i < n_pairs) src[i] = -1;
  }
}

// Count the pairs of every target; the counting atomic's old value is the
// pair's slot in its target's segment.  The same launch writes the sources.
__global__ void k_count_targets(const int64_t* __restrict__ pair_ptr,
                                const int32_t* __restrict__ pair_j, int64_t n_pairs,
                                int64_t n_atoms, int32_t* __restrict__ cnt,
                                int32_t* __restrict__ slot, int32_t* __restrict__ src,
                                int* dev_err) {
  const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = t0; p < n_pairs; p += nt) {
    const int32_t j = pair_j[p];
    if (j < 0 || j >= n_atoms) {
      atomicOr(dev_err, GAP_DEVERR_INDEX);
      continue;
    }
    slot[p] = atomicAdd(&cnt[j], 1);
  }
  for (int64_t i = t0 >> 4; i < n_atoms; i += nt >> 4)
    write_pair_src(pair_ptr, i, n_pairs, src, dev_err);
}

// Exclusive scan of n int32 counts into n + 1 int64 offsets: block b scans
// counts [4096 b, 4096 (b + 1)) after summing all counts before them itself
// (coalesced 16-byte reads that hit L2), so no pass waits for another block.
// One block walking the whole list took 275 us for 116,000 counts.
__global__ __launch_bounds__(1024) void k_scan_counts(const int32_t* __restrict__ cnt, int64_t n,
                                                      int64_t* __restrict__ ptr) {
  __shared__ int64_t wave_tot[16];
  __shared__ int64_t base_s;
  const int t = threadIdx.x;
  const int64_t lo = (int64_t)blockIdx.x * kScanPer;
  const int4* c4 = reinterpret_cast<const int4*>(cnt);
  int64_t before = 0;
#pragma unroll 8
  for (int64_t e = t; e < lo / 4; e += 1024) {
    const int4 v = c4[e];
    before += (int64_t)v.x + v.y + v.z + v.w;
  }
  before = block_scan_1024(before, wave_tot);
  if (t == 1023) base_s = before;
  __syncthreads();
  int32_t v[4];
  int64_t s = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t i = lo + 4 * t + q;
    v[q] = i < n ? cnt[i] : 0;
    s += v[q];
  }
  const int64_t incl = block_scan_1024(s, wave_tot) + base_s;
  int64_t run = incl - s;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t i = lo + 4 * t + q;
    if (i < n) ptr[i] = run;
    run += v[q];
  }
  if (blockIdx.x == gridDim.x - 1 && t == 1023) ptr[n] = incl;
}

__global__ void k_place_pairs(const int32_t* __restrict__ pair_j, int64_t n_pairs, int64_t n_atoms,
                              const int64_t* __restrict__ tgt_ptr,
                              const int32_t* __restrict__ slot, int32_t* __restrict__ list) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n_pairs;
       p += (int64_t)gridDim.x * blockDim.x) {
    const int32_t j = pair_j[p];
    if (j < 0 || j >= n_atoms) continue;
    list[tgt_ptr[j] + slot[p]] = (int32_t)p;
  }
}

// Restore increasing pair order in every segment, list -> tgt_pair: one wave
// per target ranks its values in registers (a serial insertion sort by one
// thread per target took 1.27 ms for 116,000 targets of 30 pairs); segments longer
// than rank_max are rebuilt from the list, in a loop of their own.  Entries past
// the last segment (pairs dropped for an out-of-range target) hold pair 0, a
// valid index for readers that clamp a slot to the end of the list.
__global__ __launch_bounds__(256) void k_sort_segments(const int64_t* __restrict__ tgt_ptr,
                                                       int64_t n_atoms, int64_t n_pairs,
                                                       int rank_max,
                                                       const int32_t* __restrict__ pair_j,
                                                       const int32_t* __restrict__ list,
                                                       int32_t* __restrict__ tgt_pair) {
  const int64_t nw = (int64_t)gridDim.x * 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bool longer = false;
  for (int64_t j = (int64_t)blockIdx.x * 4 + wave; j < n_atoms; j += nw) {
    const int64_t lo = tgt_ptr[j];
    const int n = __builtin_amdgcn_readfirstlane((int)(tgt_ptr[j + 1] - lo));
    if (n <= 64)
      wave_sort_short<4>(list + lo, n, tgt_pair + lo);
    else if (n <= rank_max)
      wave_sort_segment(list + lo, n, tgt_pair + lo);
    else
      longer = true;
  }
  if (longer)
    for (int64_t j = (int64_t)blockIdx.x * 4 + wave; j < n_atoms; j += nw) {
      const int64_t lo = tgt_ptr[j];
      if (__builtin_amdgcn_readfirstlane((int)(tgt_ptr[j + 1] - lo)) > rank_max)
        wave_scan_segment(pair_j, n_pairs, (int32_t)j, tgt_pair + lo);
    }
  for (int64_t p = tgt_ptr[n_atoms] + blockIdx.x * (int64_t)256 + threadIdx.x; p < n_pairs;
       p += (int64_t)gridDim.x * 256)
    tgt_pair[p] = 0;
}

// Stable counting sort of the atoms by decreasing degree, 1024 atoms per
// block.  A wave finds each atom's place among its equals by comparing degrees
// lane by lane, a block adds up its waves, and a scan over blocks and degrees
// in between (k_degree_scan) gives every (block, degree) its start.  One
// workgroup walking all atoms took 5.7 ms for 116,000 atoms.
template <bool PLACE>
__global__ __launch_bounds__(1024) void k_degree_block(const int64_t* __restrict__ tgt_ptr,
                                                       int64_t n_atoms, int32_t* __restrict__ hist,
                                                       int32_t* __restrict__ order) {
  __shared__ uint16_t wh[16][kDegBuckets];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int64_t j = (int64_t)blockIdx.x * 1024 + t;
  const int d = j < n_atoms ? (int)min(tgt_ptr[j + 1] - tgt_ptr[j], (int64_t)kDegBuckets - 1) : -1;
  for (int e = t; e < 16 * kDegBuckets / 2; e += 1024) reinterpret_cast<uint32_t*>(wh)[e] = 0;
  __syncthreads();
  int lower = 0, same = 0;
#pragma unroll 8
  for (int q = 0; q < 64; ++q) {
    const bool eq = __builtin_amdgcn_readlane(d, q) == d;
    same += eq ? 1 : 0;
    lower += (eq && q < lane) ? 1 : 0;
  }
  if (d >= 0 && lower == 0) wh[wave][d] = (uint16_t)same;
  __syncthreads();
  int run = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int c = wh[w][t];
    wh[w][t] = (uint16_t)run;
    run += c;
  }
  int32_t* h = hist + (int64_t)blockIdx.x * kDegBuckets;
  if (!PLACE) {
    h[t] = run;
    return;
  }
  __syncthreads();
  if (d >= 0) order[h[d] + wh[wave][d] + lower] = (int32_t)j;
}

// hist[block][degree] -> start of that block's atoms of that degree in the
// order of decreasing degree, then increasing block.
__global__ __launch_bounds__(kDegBuckets) void k_degree_scan(int32_t* __restrict__ hist,
                                                             int64_t n_blk) {
  __shared__ int32_t wave_tot[16];
  const int b = kDegBuckets - 1 - (int)threadIdx.x;  // decreasing degree
  int32_t tot = 0;
#pragma unroll 8
  for (int64_t q = 0; q < n_blk; ++q) tot += hist[q * kDegBuckets + b];
  int32_t run = block_scan_1024(tot, wave_tot) - tot;
#pragma unroll 8
  for (int64_t q = 0; q < n_blk; ++q) {
    const int32_t c = hist[q * kDegBuckets + b];
    hist[q * kDegBuckets + b] = run;
    run += c;
  }
}

__global__ void k_atom_cfg(const int64_t* __restrict__ cfg_ptr, int64_t n_cfg, int64_t n_atoms,
                           int32_t* __restrict__ atom_cfg) {
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n_cfg;
       c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t lo = max((int64_t)0, cfg_ptr[c]), hi = min(n_atoms, cfg_ptr[c + 1]);
    for (int64_t i = lo; i < hi; ++i) atom_cfg[i] = (int32_t)c;
  }
}

inline unsigned grid_for(int64_t n, int block = 256) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return (unsigned)g;
}

}  // namespace

int64_t pair_scratch_ints(int64_t n_atoms, bool want_order) {
  const int64_t cnt = (n_atoms + 63) / 64 * 64;
  return cnt + (want_order ? (n_atoms + 1023) / 1024 * kDegBuckets : 0);
}

void pair_transpose(const int64_t* pair_ptr, const int32_t* pair_j, int64_t n_atoms,
                    int64_t n_pairs, int64_t* tgt_ptr, int32_t* tgt_pair, int32_t* pair_src,
                    int32_t* order, int32_t* scratch, int32_t* list, int* dev_err,
                    hipStream_t st) {
  const int rank_max = rank_longest(n_pairs);
  if (n_pairs > 0 && n_atoms > 0 && n_atoms <= kSmallAtoms && n_pairs <= kSmallPairs) {
    hipLaunchKernelGGL(k_pairs_small, dim3(1), dim3(1024), 0, st, pair_ptr, pair_j, (int)n_atoms,
                       (int)n_pairs, rank_max, tgt_ptr, tgt_pair, pair_src, order, dev_err);
    return;
  }
  int32_t* cnt = scratch;                               // n_atoms
  int32_t* hist = scratch + (n_atoms + 63) / 64 * 64;   // 1024 per 1024 atoms
  hipLaunchKernelGGL(k_pairs_init, dim3(grid_for(std::max(n_atoms, n_pairs))), dim3(256), 0, st,
                     cnt, n_atoms, pair_src, n_pairs);
  if (n_pairs > 0)
    hipLaunchKernelGGL(k_count_targets, dim3(grid_for(n_pairs)), dim3(256), 0, st, pair_ptr,
                       pair_j, n_pairs, n_atoms, cnt, tgt_pair, pair_src, dev_err);
  hipLaunchKernelGGL(k_scan_counts,
                     dim3((unsigned)std::max<int64_t>(1, (n_atoms + kScanPer - 1) / kScanPer)),
                     dim3(1024), 0, st, cnt, n_atoms, tgt_ptr);
  if (n_pairs > 0) {
    hipLaunchKernelGGL(k_place_pairs, dim3(grid_for(n_pairs)), dim3(256), 0, st, pair_j, n_pairs,
                       n_atoms, tgt_ptr, tgt_pair, list);
    hipLaunchKernelGGL(k_sort_segments, dim3(grid_for(n_atoms, 4)), dim3(256), 0, st, tgt_ptr,
                       n_atoms, n_pairs, rank_max, pair_j, list, tgt_pair);
  }
  if (order != nullptr && n_atoms > 0) {
    const unsigned nb = (unsigned)((n_atoms + 1023) / 1024);
    hipLaunchKernelGGL(k_degree_block<false>, dim3(nb), dim3(1024), 0, st, tgt_ptr, n_atoms, hist,
                       order);
    hipLaunchKernelGGL(k_degree_scan, dim3(1), dim3(kDegBuckets), 0, st, hist, (int64_t)nb);
    hipLaunchKernelGGL(k_degree_block<true>, dim3(nb), dim3(1024), 0, st, tgt_ptr, n_atoms, hist,
                       order);
  }
}

void atom_config(const int64_t* cfg_ptr, int64_t n_cfg, int64_t n_atoms, int32_t* atom_cfg,
                 hipStream_t st) {
  if (n_atoms > 0)
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n_atoms)), dim3(256), 0, st, atom_cfg, n_atoms,
                       -1);
  if (n_cfg <= 0) return;
  hipLaunchKernelGGL(k_atom_cfg, dim3(grid_for(n_cfg)), dim3(256), 0, st, cfg_ptr, n_cfg, n_atoms,
                     atom_cfg);
}

}  // namespace gapk
