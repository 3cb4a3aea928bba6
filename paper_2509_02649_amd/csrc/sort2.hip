// Two-pass bin sort of the point stream for the MFMA spreads.
//
// The matrix-core spreads take the points of one bin four at a time, so the type-1
// stage first orders the stream by bin.  A one-pass counting sort into the nbx^2
// bins sends consecutive points to unrelated addresses, and on HBM3E such
// scattered 8- and 64-byte writes run far below the streaming rate.  Here the order
// is reached in two counting passes over nbx buckets each (the bin row bx, then the
// bin column by inside a row).  A point's bin on an axis is set by the first cell of
// its kernel window, not by the cell it lies in, so that a bin's windows cover
// MB + w - 1 cells per axis.  A workgroup ranks a batch of points by bucket in LDS,
// stages the batch in bucket order, and writes each bucket's part as one contiguous
// run, so both passes write in runs and read in streams.
//
// 8..16 weight channels (records of 16 weight words, zero padded):
//   pass 1: X, Y (structure of arrays)          -> crd1 / wts1, grouped by bx
//   pass 2: one workgroup per (bx, slice) of it -> crd and, per point, its position
//           in crd1 / wts1, grouped by bin; the 64-byte weight blocks are not moved
//           again (the spread gathers them from wts1).
// 0..7 weight channels (records of 1, 2, 4 or 8 weight words):
//   pass 1 as above; pass 2 -> crd / wts, grouped by bin.
//
// With few bins (nbx^2 <= KONE) and 0..7 weight channels one counting pass over all bins does: a batch is staged as
// above, and its runs, 8 points and more, still fill most of a 64-byte line.
//
// The order of points inside a bin is not specified (LDS atomics rank them).
#include "fk_internal.h"
#include "fk_device.h"

#include <algorithm>

namespace fk {

namespace {

constexpr int BT = 1024;       // points per staged batch, one per thread
constexpr int KMAX = 256;      // largest bucket count (nf / MB for nf <= 1024)
constexpr int KONE = 1024;     // largest bin count of the one-pass sort (nf <= 256 with bins of 8 x 8 cells)

struct Stage {
  uint32_t cur[KMAX];             // next output position of every bucket
  uint32_t hist[KMAX];            // bucket counts of the current batch
  uint32_t lofs[KMAX];            // their exclusive prefix sums
  uint32_t total;
  uint16_t sbin[BT];              // bucket of every staged slot
  uint2 scrd[BT];
  uint4 swts[BT * 4];
};

// Rank of every point of the batch inside its bucket (LDS atomics), and the
// exclusive prefix sums of the batch's bucket counts (sm.lofs, sm.total).
template <class St>
__device__ __forceinline__ uint32_t rank_scan(St& sm, int nk, bool ok, int key) {
  const int tid = threadIdx.x;
  const uint32_t rank = ok ? atomicAdd(&sm.hist[key], 1u) : 0u;
  __syncthreads();
  if (tid < 64) {   // exclusive scan of the nk <= 256 counts in one wave
    const int per = (nk + 63) / 64;
    uint32_t s = 0;
    for (int i = 0; i < per; ++i) {
      const int b = tid * per + i;
      if (b < nk) s += sm.hist[b];
    }
    uint32_t x = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (tid >= o) x += y;
    }
    uint32_t run = x - s;
    for (int i = 0; i < per; ++i) {
      const int b = tid * per + i;
      if (b < nk) {
        sm.lofs[b] = run;
        run += sm.hist[b];
      }
    }
    if (tid == 63) sm.total = x;
  }
  __syncthreads();
  return rank;
}

// Write the staged coordinates as runs, one per bucket (after the staging barrier).
template <class St>
__device__ __forceinline__ void write_coords(St& sm, uint2* __restrict__ crd_out) {
  const int tid = threadIdx.x;
  if ((uint32_t)tid < sm.total) {
    const int b = sm.sbin[tid];
    crd_out[(size_t)sm.cur[b] + (tid - sm.lofs[b])] = sm.scrd[tid];
  }
}

// After the staged batch is written: advance the bucket cursors, clear the counts.
template <class St>
__device__ __forceinline__ void advance_cursors(St& sm, int nk) {
  __syncthreads();
  for (int b = threadIdx.x; b < nk; b += BT) {
    sm.cur[b] += sm.hist[b];
    sm.hist[b] = 0;
  }
  __syncthreads();
}

// Rank the batch by bucket, stage it in bucket order and write the runs.
// Every thread of the workgroup calls this once per batch with point t (key, U) and
// its weights v0..v3 (the four 16-byte quarters of its 64-byte block).
__device__ __forceinline__ void stage_batch(Stage& sm, int nk, bool ok, int key, uint2 U, uint4 v0, uint4 v1,
                                            uint4 v2, uint4 v3, uint2* __restrict__ crd_out,
                                            uint4* __restrict__ wts_out) {
  const int tid = threadIdx.x;
  const uint32_t rank = rank_scan(sm, nk, ok, key);
  if (ok) {
    const uint32_t s = sm.lofs[key] + rank;
    sm.sbin[s] = (uint16_t)key;
    sm.scrd[s] = U;
    sm.swts[s * 4 + 0] = v0;
    sm.swts[s * 4 + 1] = v1;
    sm.swts[s * 4 + 2] = v2;
    sm.swts[s * 4 + 3] = v3;
  }
  __syncthreads();
  const uint32_t total = sm.total;
  write_coords(sm, crd_out);
  for (uint32_t q = tid; q < total * 4; q += BT) {
    const uint32_t s = q >> 2;
    const int b = sm.sbin[s];
    wts_out[((size_t)sm.cur[b] + (s - sm.lofs[b])) * 4 + (q & 3)] = sm.swts[q];
  }
  advance_cursors(sm, nk);
}

// Pass 1 counts: bucket = bin row of every valid point, one row of nbx counts per
// workgroup (contiguous chunks of the input), and the totals rowtot (zeroed beforehand).  Each thread
// takes CU1 points per step, their loads issued together.
// ONE: the buckets are the nbx = ncol^2 bins.
constexpr int CU1 = 4;
template <typename TX, bool ONE = false>
__global__ __launch_bounds__(BT) void k_s2_count1(const TX* __restrict__ X, int64_t n, int64_t xstride,
                                                  double scale, uint32_t nf_fix, int fb, uint32_t wbias,
                                                  int tshift, int nbx, int ncol, int64_t chunk, uint32_t* __restrict__ cnt,
                                                  uint32_t* __restrict__ rowtot, int* flags) {
  __shared__ uint32_t hist[ONE ? KONE : KMAX];
  for (int i = threadIdx.x; i < nbx; i += blockDim.x) hist[i] = 0;
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = min(n, beg + chunk);
  for (int64_t j0 = beg + threadIdx.x; j0 < end; j0 += (int64_t)CU1 * BT) {
    double x1[CU1], x2[CU1];
#pragma unroll
    for (int u = 0; u < CU1; ++u) {
      const int64_t jc = min(j0 + (int64_t)u * BT, end - 1);
      x1[u] = (double)X[jc];
      x2[u] = (double)X[xstride + jc];
    }
#pragma unroll
    for (int u = 0; u < CU1; ++u) {
      if (j0 + (int64_t)u * BT >= end) break;
      uint32_t U1, U2;
      bool ok = to_fixed(x1[u], scale, nf_fix, &U1, flags);
      ok = to_fixed(x2[u], scale, nf_fix, &U2, flags) && ok;
      if (!ok) continue;
      int key = window_bin(U1, fb, wbias, (int)(nf_fix >> fb), tshift);
      if constexpr (ONE) key = key * ncol + window_bin(U2, fb, wbias, (int)(nf_fix >> fb), tshift);
      atomicAdd(&hist[key], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nbx; i += blockDim.x) {
    cnt[(int64_t)blockIdx.x * nbx + i] = hist[i];
    if (hist[i]) atomicAdd(&rowtot[i], hist[i]);
  }
}

// Exclusive prefix sums over the 1024 threads of a workgroup (sh: 16 words); the sum in total.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t y = sh[i];
    before += i < w ? y : 0u;
    all += y;
  }
  __syncthreads();   // sh may be reused
  *total = all;
  return before + x - v;
}

// Sum of a[0 .. count) by a workgroup, its loads coalesced and independent.
__device__ __forceinline__ uint32_t block_sum(const uint32_t* __restrict__ a, int64_t count, uint32_t* sh) {
  uint32_t s = 0, total;
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < count; i += 1024) s += a[i];
  (void)block_scan(s, sh, &total);
  return total;
}

// Offsets of pass 1 (in place of its counts cnt[k][b]): cnt[k][b] becomes the position at which
// workgroup k's points of bucket b start, in the order of the workgroups (the order of the input).
// rowtot: the buckets' totals.  Workgroup b takes bucket b: a thread per first-pass workgroup (at most
// kSortBlkMax = 1024), all columns side by side (one workgroup walking them took 17 us for 152 x 64
// counts and 57 for 512 x 256, this takes 4).
__global__ __launch_bounds__(1024) void k_s2_scan1(uint32_t* __restrict__ cnt, int nk, int nblk,
                                                   const uint32_t* __restrict__ rowtot,
                                                   uint64_t* __restrict__ start1) {
  __shared__ uint32_t sh[16];
  const int b = blockIdx.x, k = threadIdx.x;
  const uint32_t v = k < nblk ? cnt[(int64_t)k * nk + b] : 0u;
  const uint32_t base = block_sum(rowtot, b, sh);
  uint32_t total;
  const uint32_t p = base + block_scan(v, sh, &total);
  if (k < nblk) cnt[(int64_t)k * nk + b] = p;
  if (k == 0) {
    start1[b] = base;
    if (b == nk - 1) start1[nk] = (uint64_t)base + total;
  }
}

// The same for the one-pass sort (any nk): workgroup b takes the 16 buckets
// from 16 b, read together, and thread (g, i) the g-th part of bucket 16 b + i's column (a workgroup per bucket
// took 21 us for 512 x 1024 counts, of whose lines it used 4 bytes each; this takes 12 us).
__global__ __launch_bounds__(1024) void k_s2_scan_one(uint32_t* __restrict__ cnt, int nk, int nblk,
                                                      const uint32_t* __restrict__ tot, uint64_t* __restrict__ start) {
  __shared__ uint32_t sh[16], part[64][17];
  const int i = threadIdx.x & 15, g = threadIdx.x >> 4, b = blockIdx.x * 16 + i;
  const uint32_t first = block_sum(tot, blockIdx.x * 16, sh);
  const int k0 = (int)((int64_t)nblk * g / 64), k1 = (int)((int64_t)nblk * (g + 1) / 64);
  const bool on = b < nk;
  uint32_t sum = 0;
#pragma unroll 4
  for (int k = k0; k < k1; ++k) sum += on ? cnt[(int64_t)k * nk + b] : 0u;
  part[g][i] = sum;
  __syncthreads();
  uint32_t p = first;
  for (int j = 0; j < i; ++j) p += blockIdx.x * 16 + j < nk ? tot[blockIdx.x * 16 + j] : 0u;
  if (on && g == 0) {
    start[b] = p;
    if (b == nk - 1) start[nk] = (uint64_t)p + tot[b];
  }
  for (int j = 0; j < g; ++j) p += part[j][i];
#pragma unroll 4
  for (int k = k0; k < k1; ++k)
    if (on) {
      const uint32_t v = cnt[(int64_t)k * nk + b];
      cnt[(int64_t)k * nk + b] = p;
      p += v;
    }
}

// Workgroup `blk` of the second pass: its row and its part [q0, q1) of the row's points.  A row of len
// points has ceil(len / slice_pts) slices of equal size, so the work is even for any density; the grid
// holds one workgroup per row more than n / slice_pts.  False past the last slice.
__device__ __forceinline__ bool slice_of(const uint64_t* __restrict__ start1, int nrow, uint32_t slice_pts,
                                         uint32_t blk, int* row, uint64_t* q0, uint64_t* q1) {
  __shared__ uint32_t found[4];
  static_assert(KMAX % 64 == 0, "rows per lane");
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    constexpr int RP = KMAX / 64;   // rows per lane
    uint32_t ns[RP], sum = 0;
#pragma unroll
    for (int i = 0; i < RP; ++i) {
      const int r = lane * RP + i;
      const uint32_t len = r < nrow ? (uint32_t)(start1[r + 1] - start1[r]) : 0u;
      ns[i] = len / slice_pts + (len % slice_pts != 0);
      sum += ns[i];
    }
    uint32_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) found[3] = x;
    uint32_t first = x - sum;
#pragma unroll
    for (int i = 0; i < RP; ++i) {
      if (blk >= first && blk < first + ns[i]) {
        found[0] = lane * RP + i;
        found[1] = blk - first;
        found[2] = ns[i];
      }
      first += ns[i];
    }
  }
  __syncthreads();
  if (blk >= found[3]) return false;
  *row = (int)found[0];
  const uint64_t p0 = start1[*row], len = start1[*row + 1] - p0;
  *q0 = p0 + len * found[1] / found[2];
  *q1 = p0 + len * (found[1] + 1) / found[2];
  return true;
}

// Pass 1 scatter.  off holds, per workgroup and bucket, where its points of the bucket
// start.  The inputs of the next
// batch are loaded (unconditionally, index clamped to the chunk) while the current
// batch is ranked, staged and written.
template <typename TX>
__global__ __launch_bounds__(BT) void k_s2_scatter1(const TX* __restrict__ X, int64_t n,
                                                    int64_t xstride, const TX* __restrict__ Y, int nw,
                                                    double scale, uint32_t nf_fix, int fb, uint32_t wbias,
                                                    int tshift, int nbx, int64_t chunk,
                                                    const uint32_t* __restrict__ off,
                                                    uint2* __restrict__ crd1, uint4* __restrict__ wts1,
                                                    int* flags) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Stage& sm = *reinterpret_cast<Stage*>(smem_raw);
  const int tid = threadIdx.x;
  for (int b = tid; b < nbx; b += BT) {
    sm.cur[b] = off[(int64_t)blockIdx.x * nbx + b];
    sm.hist[b] = 0;
  }
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = min(n, beg + chunk);
  if (beg >= end) return;
  double nx1, nx2;
  float nw_[16];
  auto fetch = [&](int64_t j) {
    const int64_t jc = min(j, end - 1);
    nx1 = (double)X[jc];
    nx2 = (double)X[xstride + jc];
#pragma unroll
    for (int c = 0; c < 16; ++c) nw_[c] = (float)Y[(int64_t)min(c, nw - 1) * n + jc];
  };
  fetch(beg + tid);
  for (int64_t base = beg; base < end; base += BT) {
    const int64_t j = base + tid;
    const double x1 = nx1, x2 = nx2;
    float w[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) w[c] = nw_[c];
    fetch(base + BT + tid);
    bool ok = false;
    uint2 U = make_uint2(0u, 0u);
    if (j < end) {
      ok = to_fixed(x1, scale, nf_fix, &U.x, flags);
      ok = to_fixed(x2, scale, nf_fix, &U.y, flags) && ok;
    }
    uint32_t wb[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      float wc = (ok && c < nw) ? w[c] : 0.f;
      if (!(wc == wc) || isinf(wc)) {
        atomicOr(&flags[kFlagNaN], 1);
        wc = 0.f;
      }
      wb[c] = __float_as_uint(wc);
    }
    const int key = ok ? window_bin(U.x, fb, wbias, (int)(nf_fix >> fb), tshift) : 0;
    stage_batch(sm, nbx, ok, key, U, make_uint4(wb[0], wb[1], wb[2], wb[3]), make_uint4(wb[4], wb[5], wb[6], wb[7]),
                make_uint4(wb[8], wb[9], wb[10], wb[11]), make_uint4(wb[12], wb[13], wb[14], wb[15]), crd1, wts1);
  }
}

// Pass 2 counts: a workgroup counts the bin columns of its slice of a row, cnt2[workgroup][by]; CU1 loads
// in flight per thread.
__global__ __launch_bounds__(BT) void k_s2_count2(const uint2* __restrict__ crd1,
                                                  const uint64_t* __restrict__ start1, uint32_t slice_pts, int fb,
                                                  uint32_t wbias, int nf, int tshift, int nbx,
                                                  uint32_t* __restrict__ cnt2) {
  __shared__ uint32_t hist[KMAX];
  for (int i = threadIdx.x; i < nbx; i += BT) hist[i] = 0;
  int bx;
  uint64_t q0, q1;
  if (!slice_of(start1, nbx, slice_pts, blockIdx.x, &bx, &q0, &q1)) return;
  for (uint64_t p = q0 + threadIdx.x; p < q1; p += (uint64_t)CU1 * BT) {
    uint32_t y[CU1];
#pragma unroll
    for (int u = 0; u < CU1; ++u) y[u] = crd1[min(p + (uint64_t)u * BT, q1 - 1)].y;
#pragma unroll
    for (int u = 0; u < CU1; ++u)
      if (p + (uint64_t)u * BT < q1) atomicAdd(&hist[window_bin(y[u], fb, wbias, nf, tshift)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nbx; i += BT) cnt2[(int64_t)blockIdx.x * nbx + i] = hist[i];
}

// Offsets of pass 2 (in place of its counts), one workgroup per row: cnt2[slice][by] becomes the position
// at which the slice's points of bin (row, by) start, in the order of the slices, and start[row ncol + by]
// the bin's start (ncol buckets per row).  A row's slices are consecutive workgroups of the second pass; thread (g, by) takes
// the g-th part of them.
__global__ __launch_bounds__(1024) void k_s2_scan2(uint32_t* __restrict__ cnt2, const uint64_t* __restrict__ start1,
                                                   uint32_t slice_pts, int ncol, uint64_t* __restrict__ start) {
  __shared__ uint32_t sh[16];
  __shared__ uint32_t part[1024], tot[KMAX];
  const int row = blockIdx.x, t = threadIdx.x;
  auto slices = [&](int r) -> uint32_t {
    const uint32_t len = (uint32_t)(start1[r + 1] - start1[r]);
    return len / slice_pts + (len % slice_pts != 0);
  };
  uint32_t first;   // slices of the rows before
  (void)block_scan(t < row ? slices(t) : 0u, sh, &first);
  const uint32_t ns = slices(row);
  const int groups = 1024 / ncol, by = t % ncol, g = t / ncol;   // threads past groups ncol idle
  const bool on = g < groups;
  const uint32_t s0 = (uint32_t)((uint64_t)ns * g / groups), s1 = (uint32_t)((uint64_t)ns * (g + 1) / groups);
  uint32_t* c = cnt2 + (int64_t)first * ncol + by;
  uint32_t sum = 0;
  if (on) {
#pragma unroll 4
    for (uint32_t s = s0; s < s1; ++s) sum += c[(int64_t)s * ncol];
  }
  part[t] = sum;
  __syncthreads();
  uint32_t before = 0, all = 0;   // the bin's points in earlier groups, and in all
  if (on)
    for (int i = 0; i < groups; ++i) {
      const uint32_t v = part[i * ncol + by];
      before += i < g ? v : 0u;
      all += v;
    }
  if (t < ncol) tot[by] = all;
  uint32_t total;
  const uint32_t pre = block_scan(t < ncol ? all : 0u, sh, &total);
  const uint32_t base = (uint32_t)start1[row];
  if (t < ncol) {
    start[(int64_t)row * ncol + t] = base + pre;
    tot[t] = base + pre;
    if (t == 0 && row == (int)gridDim.x - 1) start[(int64_t)gridDim.x * ncol] = (uint64_t)base + total;
  }
  __syncthreads();
  if (on) {
    uint32_t run = tot[by] + before;
#pragma unroll 4
    for (uint32_t s = s0; s < s1; ++s) {
      const uint32_t v = c[(int64_t)s * ncol];
      c[(int64_t)s * ncol] = run;
      run += v;
    }
  }
}

// ---------------------------------------------------------------- narrow records
// The same two passes for 0..7 weight channels (the outer-product spread): records of
// WV = 0, 1, 2, 4 or 8 weight words per point (zero padded), staged word by word.  A
// record is small, so each thread takes NPT points per batch (BT NPT points between
// barriers, longer runs per bucket).
template <int WV>
constexpr int narrow_ppt() { return WV <= 2 ? 4 : (WV == 4 ? 2 : 1); }
constexpr int kPosPpt = 8;   // points per thread of the position pass (116 KB of LDS)
// Points per thread of the one-pass sort: twice as many for the length of its runs (FP64 points: registers).
template <typename TX, int WV>
constexpr int one_ppt() { return WV <= 1 && sizeof(TX) == 4 ? 8 : (WV <= 2 ? 4 : (WV == 4 ? 4 : 2)); }

template <int WV, int P = narrow_ppt<WV>(), int KM = KMAX>
struct StageN {
  static constexpr int NPT = P;
  uint32_t cur[KM];
  uint32_t hist[KM];
  uint32_t lofs[KM];
  uint32_t total;
  uint16_t sbin[BT * NPT];
  uint2 scrd[BT * NPT];
  uint32_t swts[BT * NPT * (WV > 0 ? WV : 1)];
};

// Exclusive prefix sums of the batch's bucket counts (after the rank atomics).
template <class St>
__device__ __forceinline__ void scan_counts(St& sm, int nk) {
  const int tid = threadIdx.x;
  __syncthreads();
  if (tid < 64) {
    const int per = (nk + 63) / 64;
    uint32_t s = 0;
    for (int i = 0; i < per; ++i) {
      const int b = tid * per + i;
      if (b < nk) s += sm.hist[b];
    }
    uint32_t x = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (tid >= o) x += y;
    }
    uint32_t run = x - s;
    for (int i = 0; i < per; ++i) {
      const int b = tid * per + i;
      if (b < nk) {
        sm.lofs[b] = run;
        run += sm.hist[b];
      }
    }
    if (tid == 63) sm.total = x;
  }
  __syncthreads();
}

template <int WV, int P, int KM>
__device__ __forceinline__ void write_batch_n(StageN<WV, P, KM>& sm, uint2* __restrict__ crd_out,
                                              uint32_t* __restrict__ wts_out) {
  const uint32_t total = sm.total;
  for (uint32_t q = threadIdx.x; q < total; q += BT) {
    const int b = sm.sbin[q];
    crd_out[(size_t)sm.cur[b] + (q - sm.lofs[b])] = sm.scrd[q];
  }
  if constexpr (WV > 0) {
    for (uint32_t q = threadIdx.x; q < total * WV; q += BT) {
      const uint32_t s = q / WV;
      const int b = sm.sbin[s];
      wts_out[((size_t)sm.cur[b] + (s - sm.lofs[b])) * WV + q % WV] = sm.swts[q];
    }
  }
}

// ONE: the buckets are the nbx = ncol^2 bins, and the records are in their final order.
template <typename TX, int WV, bool ONE>
__global__ __launch_bounds__(BT) void k_s2n_scatter1(const TX* __restrict__ X, int64_t n, int64_t xstride,
                                                     const TX* __restrict__ Y, int nw, double scale,
                                                     uint32_t nf_fix, int fb, uint32_t wbias, int tshift, int nbx, int ncol,
                                                     int64_t chunk, const uint32_t* __restrict__ off,
                                                     uint2* __restrict__ crd1, uint32_t* __restrict__ wts1,
                                                     int* flags) {
  constexpr int NPT = ONE ? one_ppt<TX, WV>() : narrow_ppt<WV>();
  using St = StageN<WV, NPT, ONE ? KONE : KMAX>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  St& sm = *reinterpret_cast<St*>(smem_raw);
  const int tid = threadIdx.x;
  for (int b = tid; b < nbx; b += BT) {
    sm.cur[b] = off[(int64_t)blockIdx.x * nbx + b];
    sm.hist[b] = 0;
  }
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = min(n, beg + chunk);
  if (beg >= end) return;
  const int nf = (int)(nf_fix >> fb);
  // next batch in flight: point base + u BT + tid of slot u (index clamped to the
  // chunk; no target row is read when nw = 0)
  TX nx1[NPT], nx2[NPT];
  float ny[NPT][WV > 0 ? WV : 1];
#define FK_FETCH1N(bb)                                                                     \
  _Pragma("unroll") for (int u = 0; u < NPT; ++u) {                                        \
    const int64_t jc = min((int64_t)(bb) + u * BT + tid, end - 1);                         \
    nx1[u] = X[jc];                                                                        \
    nx2[u] = X[xstride + jc];                                                              \
    _Pragma("unroll") for (int c = 0; c < WV; ++c)                                         \
      ny[u][c] = nw > 0 ? (float)Y[(int64_t)min(c, nw - 1) * n + jc] : 0.f;               \
  }
  FK_FETCH1N(beg);
  for (int64_t base = beg; base < end; base += (int64_t)BT * NPT) {
    TX x1[NPT], x2[NPT];
    float w[NPT][WV > 0 ? WV : 1];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      x1[u] = nx1[u];
      x2[u] = nx2[u];
#pragma unroll
      for (int c = 0; c < WV; ++c) w[u][c] = ny[u][c];
    }
    FK_FETCH1N(base + (int64_t)BT * NPT);
    bool ok[NPT];
    uint2 U[NPT];
    int key[NPT];
    uint32_t rank[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      ok[u] = false;
      U[u] = make_uint2(0u, 0u);
      if (base + u * BT + tid < end) {
        ok[u] = to_fixed((double)x1[u], scale, nf_fix, &U[u].x, flags);
        ok[u] = to_fixed((double)x2[u], scale, nf_fix, &U[u].y, flags) && ok[u];
      }
      key[u] = ok[u] ? window_bin(U[u].x, fb, wbias, nf, tshift) : 0;
      if constexpr (ONE) key[u] = ok[u] ? key[u] * ncol + window_bin(U[u].y, fb, wbias, nf, tshift) : 0;
      rank[u] = ok[u] ? atomicAdd(&sm.hist[key[u]], 1u) : 0u;
    }
    if constexpr (ONE) {
      __shared__ uint32_t sh[16];
      uint32_t total;
      __syncthreads();
      const uint32_t before = block_scan(tid < nbx ? sm.hist[tid] : 0u, sh, &total);
      if (tid < nbx) sm.lofs[tid] = before;
      if (tid == 0) sm.total = total;
      __syncthreads();
    } else {
      scan_counts(sm, nbx);
    }
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      if (!ok[u]) continue;
      const uint32_t s = sm.lofs[key[u]] + rank[u];
      sm.sbin[s] = (uint16_t)key[u];
      sm.scrd[s] = U[u];
#pragma unroll
      for (int c = 0; c < WV; ++c) {
        float wc = c < nw ? w[u][c] : 0.f;
        if (!(wc == wc) || isinf(wc)) {
          atomicOr(&flags[kFlagNaN], 1);
          wc = 0.f;
        }
        sm.swts[s * WV + c] = __float_as_uint(wc);
      }
    }
    __syncthreads();
    write_batch_n(sm, crd1, wts1);
    advance_cursors(sm, nbx);
  }
#undef FK_FETCH1N
}

// Pass 2 for narrow records.  Slot u of the batch holds points base + u BT + tid; the
// wave's 64 weight records of a slot are read as 64 WV contiguous words (word
// lane + 64 v of the wave's block), and each word is staged at the slot of its
// point, taken from the owning lane by a wave shuffle.  With kPosition (WV = 1) the
// record word is not read but is the point's position in the pass-1 output: the
// sorted stream then refers back to the weight blocks grouped by bin row.
template <int WV, bool kPosition, int NPT = narrow_ppt<WV>()>
__global__ __launch_bounds__(BT) void k_s2n_scatter2(const uint2* __restrict__ crd1,
                                                     const uint32_t* __restrict__ wts1,
                                                     const uint64_t* __restrict__ start1,
                                                     const uint32_t* __restrict__ off2,
                                                     uint32_t slice_pts, int fb,
                                                     uint32_t wbias, int nf, int tshift, int nbx,
                                                     uint2* __restrict__ crd, uint32_t* __restrict__ wts) {
  constexpr int WD = WV > 0 ? WV : 1;   // divisor for the word index (no words when WV = 0)
  extern __shared__ __align__(16) unsigned char smem_raw[];
  StageN<WV, NPT>& sm = *reinterpret_cast<StageN<WV, NPT>*>(smem_raw);
  const int tid = threadIdx.x;
  int bx;
  uint64_t q0, q1;
  if (!slice_of(start1, nbx, slice_pts, blockIdx.x, &bx, &q0, &q1)) return;
  for (int b = tid; b < nbx; b += BT) {
    sm.cur[b] = off2[(int64_t)blockIdx.x * nbx + b];
    sm.hist[b] = 0;
  }
  __syncthreads();
  const int lane = tid & 63;
  const uint64_t wb = (uint64_t)(tid & ~63);
  uint2 nU[NPT];
  uint32_t nv[NPT][WV > 0 ? WV : 1];
#define FK_FETCH2N(bb)                                                                      \
  _Pragma("unroll") for (int u = 0; u < NPT; ++u) {                                         \
    const uint64_t g0 = (uint64_t)(bb) + (uint64_t)u * BT;                                  \
    nU[u] = crd1[min(g0 + tid, q1 - 1)];                                                    \
    _Pragma("unroll") for (int v = 0; v < WV; ++v) {                                        \
      const uint32_t m = (uint32_t)lane + 64u * v;                                          \
      nv[u][v] = kPosition ? (uint32_t)(g0 + wb + m / WD)                                   \
                           : wts1[min(g0 + wb + m / WD, q1 - 1) * WV + m % WD];             \
    }                                                                                       \
  }
  FK_FETCH2N(q0);
  for (uint64_t base = q0; base < q1; base += (uint64_t)BT * NPT) {
    uint2 U[NPT];
    uint32_t v[NPT][WV > 0 ? WV : 1];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      U[u] = nU[u];
#pragma unroll
      for (int c = 0; c < WV; ++c) v[u][c] = nv[u][c];
    }
    FK_FETCH2N(base + (uint64_t)BT * NPT);
    bool ok[NPT];
    int key[NPT];
    uint32_t rank[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      ok[u] = base + (uint64_t)u * BT + tid < q1;
      key[u] = ok[u] ? window_bin(U[u].y, fb, wbias, nf, tshift) : 0;
      rank[u] = ok[u] ? atomicAdd(&sm.hist[key[u]], 1u) : 0u;
    }
    scan_counts(sm, nbx);
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const uint32_t s = ok[u] ? sm.lofs[key[u]] + rank[u] : 0xffffffffu;
      if (ok[u]) {
        sm.sbin[s] = (uint16_t)key[u];
        sm.scrd[s] = U[u];
      }
#pragma unroll
      for (int c = 0; c < WV; ++c) {
        const uint32_t m = (uint32_t)lane + 64u * c;
        const uint32_t su = __shfl(s, (int)(m / WD), 64);
        if (su != 0xffffffffu) sm.swts[su * WV + m % WD] = v[u][c];
      }
    }
    __syncthreads();
    write_batch_n(sm, crd, wts);
    advance_cursors(sm, nbx);
  }
#undef FK_FETCH2N
}

// ---------------------------------------------------------------- three dimensions
// The same two passes for the 3-D stage: bins of 8^3 window-start cells, numbered (bx nbx + by) nbx + bz (at
// most 2^15 of them); the first pass orders by the upper half of the bin number, the second by the lower
// half.  Records of R = 3 + nw words (fixed-point coordinates, weights), staged word by word.
struct Bin3 {
  uint32_t wbias;
  int fb, nf, nbx, lo;   // lo: bits of the second pass
  __device__ int operator()(const uint32_t* U) const {
    int b = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) b = b * nbx + window_bin(U[a], fb, wbias, nf, 3);
    return b;
  }
};

template <int R>
constexpr int ppt3() { return R <= 4 ? 4 : (R <= 8 ? 2 : 1); }

template <int R>
struct Stage3 {
  static constexpr int NPT = ppt3<R>();
  uint32_t cur[KMAX], hist[KMAX], lofs[KMAX];
  uint32_t total;
  uint8_t sbin[BT * NPT];
  uint32_t rec[BT * NPT * R];
};

template <typename TX>
__global__ __launch_bounds__(BT) void k_s3_count1(const TX* __restrict__ X, int64_t n, int64_t xstride, double scale,
                                                  uint32_t nf_fix, Bin3 bin, int nk, int64_t chunk,
                                                  uint32_t* __restrict__ cnt, uint32_t* __restrict__ rowtot, int* flags) {
  __shared__ uint32_t hist[KMAX];
  for (int i = threadIdx.x; i < nk; i += BT) hist[i] = 0;
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk, end = min(n, beg + chunk);
  for (int64_t j0 = beg + threadIdx.x; j0 < end; j0 += (int64_t)CU1 * BT) {
    double x[CU1][3];
#pragma unroll
    for (int u = 0; u < CU1; ++u) {
      const int64_t jc = min(j0 + (int64_t)u * BT, end - 1);
#pragma unroll
      for (int a = 0; a < 3; ++a) x[u][a] = (double)X[a * xstride + jc];
    }
#pragma unroll
    for (int u = 0; u < CU1; ++u) {
      if (j0 + (int64_t)u * BT >= end) break;
      uint32_t U[3];
      bool ok = true;
#pragma unroll
      for (int a = 0; a < 3; ++a) ok = to_fixed(x[u][a], scale, nf_fix, &U[a], flags) && ok;
      if (ok) atomicAdd(&hist[bin(U) >> bin.lo], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nk; i += BT) {
    cnt[(int64_t)blockIdx.x * nk + i] = hist[i];
    if (hist[i]) atomicAdd(&rowtot[i], hist[i]);
  }
}

template <int R>
__device__ __forceinline__ void write_batch3(Stage3<R>& sm, uint32_t* __restrict__ out) {
  const uint32_t words = sm.total * R;
  for (uint32_t q = threadIdx.x; q < words; q += BT) {
    const uint32_t s = q / R;
    const int b = sm.sbin[s];
    out[((size_t)sm.cur[b] + (s - sm.lofs[b])) * R + q % R] = sm.rec[q];
  }
}

template <typename TX, int R>
__global__ __launch_bounds__(BT) void k_s3_scatter1(const TX* __restrict__ X, int64_t n, int64_t xstride,
                                                    const TX* __restrict__ Y, double scale, uint32_t nf_fix, Bin3 bin,
                                                    int nk, int64_t chunk, const uint32_t* __restrict__ off,
                                                    uint32_t* __restrict__ rec1, int* flags) {
  constexpr int NPT = ppt3<R>(), NW = R - 3;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Stage3<R>& sm = *reinterpret_cast<Stage3<R>*>(smem_raw);
  const int tid = threadIdx.x;
  for (int b = tid; b < nk; b += BT) {
    sm.cur[b] = off[(int64_t)blockIdx.x * nk + b];
    sm.hist[b] = 0;
  }
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk, end = min(n, beg + chunk);
  for (int64_t base = beg; base < end; base += (int64_t)BT * NPT) {
    double x[NPT][3];
    float w[NPT][NW > 0 ? NW : 1];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const int64_t jc = min(base + u * BT + tid, end - 1);
#pragma unroll
      for (int a = 0; a < 3; ++a) x[u][a] = (double)X[a * xstride + jc];
#pragma unroll
      for (int c = 0; c < NW; ++c) w[u][c] = (float)Y[(int64_t)c * n + jc];
    }
    uint32_t U[NPT][3], rank[NPT];
    int key[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      bool ok = base + u * BT + tid < end;
      if (ok) {
#pragma unroll
        for (int a = 0; a < 3; ++a) ok = to_fixed(x[u][a], scale, nf_fix, &U[u][a], flags) && ok;
      }
      key[u] = ok ? bin(U[u]) >> bin.lo : -1;
      rank[u] = ok ? atomicAdd(&sm.hist[key[u]], 1u) : 0u;
    }
    scan_counts(sm, nk);
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      if (key[u] < 0) continue;
      const uint32_t s = sm.lofs[key[u]] + rank[u];
      sm.sbin[s] = (uint8_t)key[u];
      uint32_t* r = sm.rec + s * R;
#pragma unroll
      for (int a = 0; a < 3; ++a) r[a] = U[u][a];
#pragma unroll
      for (int c = 0; c < NW; ++c) {
        float wc = w[u][c];
        if (!(wc == wc) || isinf(wc)) {
          atomicOr(&flags[kFlagNaN], 1);
          wc = 0.f;
        }
        r[3 + c] = __float_as_uint(wc);
      }
    }
    __syncthreads();
    write_batch3(sm, rec1);
    advance_cursors(sm, nk);
  }
}

template <int R>
__global__ __launch_bounds__(BT) void k_s3_count2(const uint32_t* __restrict__ rec1, const uint64_t* __restrict__ start1,
                                                  int nrow, uint32_t slice_pts, Bin3 bin, uint32_t* __restrict__ cnt2) {
  __shared__ uint32_t hist[KMAX];
  const int nk = 1 << bin.lo;
  for (int i = threadIdx.x; i < nk; i += BT) hist[i] = 0;
  int row;
  uint64_t q0, q1;
  if (!slice_of(start1, nrow, slice_pts, blockIdx.x, &row, &q0, &q1)) return;
  for (uint64_t p = q0 + threadIdx.x; p < q1; p += (uint64_t)CU1 * BT) {
    uint32_t U[CU1][3];
#pragma unroll
    for (int u = 0; u < CU1; ++u) {
      const uint32_t* r = rec1 + min(p + (uint64_t)u * BT, q1 - 1) * R;
#pragma unroll
      for (int a = 0; a < 3; ++a) U[u][a] = r[a];
    }
#pragma unroll
    for (int u = 0; u < CU1; ++u)
      if (p + (uint64_t)u * BT < q1) atomicAdd(&hist[bin(U[u]) & (nk - 1)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nk; i += BT) cnt2[(int64_t)blockIdx.x * nk + i] = hist[i];
}

template <int R>
__global__ __launch_bounds__(BT) void k_s3_scatter2(const uint32_t* __restrict__ rec1,
                                                    const uint64_t* __restrict__ start1, int nrow,
                                                    const uint32_t* __restrict__ off2, uint32_t slice_pts, Bin3 bin,
                                                    uint32_t* __restrict__ rec) {
  constexpr int NPT = ppt3<R>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Stage3<R>& sm = *reinterpret_cast<Stage3<R>*>(smem_raw);
  const int tid = threadIdx.x, nk = 1 << bin.lo;
  int row;
  uint64_t q0, q1;
  if (!slice_of(start1, nrow, slice_pts, blockIdx.x, &row, &q0, &q1)) return;
  for (int b = tid; b < nk; b += BT) {
    sm.cur[b] = off2[(int64_t)blockIdx.x * nk + b];
    sm.hist[b] = 0;
  }
  __syncthreads();
  for (uint64_t base = q0; base < q1; base += (uint64_t)BT * NPT) {
    uint32_t v[NPT][R], rank[NPT];
    int key[NPT];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const uint32_t* r = rec1 + min(base + (uint64_t)u * BT + tid, q1 - 1) * R;
#pragma unroll
      for (int c = 0; c < R; ++c) v[u][c] = r[c];
    }
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const bool ok = base + (uint64_t)u * BT + tid < q1;
      key[u] = ok ? bin(v[u]) & (nk - 1) : -1;
      rank[u] = ok ? atomicAdd(&sm.hist[key[u]], 1u) : 0u;
    }
    scan_counts(sm, nk);
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      if (key[u] < 0) continue;
      const uint32_t s = sm.lofs[key[u]] + rank[u];
      sm.sbin[s] = (uint8_t)key[u];
#pragma unroll
      for (int c = 0; c < R; ++c) sm.rec[s * R + c] = v[u][c];
    }
    __syncthreads();
    write_batch3(sm, rec);
    advance_cursors(sm, nk);
  }
}

struct Sort2Geom {
  int nblk1;            // workgroups of the first pass
  int64_t chunk1;       // their points
  uint32_t slice_pts;   // points per workgroup of the second pass (at most)
  int nblk2;            // its workgroups: every row's last slice may be short
};

// First pass: blk workgroups of 65536 points or more; fewer points each, down to 2048, where those would not
// fill the 256 CUs (workgroups of 65536 left 1e7 points to 152 CUs and 30011 to one: 97 and 98 us for the
// scatter against 61 and 10).  Second pass: slices of slice_pts points, smaller ones, down to 8192, where n
// would not give 256 of them.
Sort2Geom sort2_geom(int64_t n, int nbx, int blk, int64_t slice_pts) {
  Sort2Geom g;
  const int64_t want = (n + 65535) / 65536;
  g.nblk1 = (int)std::min<int64_t>(blk, want >= 256 ? want : std::max<int64_t>(1, (n + 2047) / 2048));
  g.chunk1 = (n + g.nblk1 - 1) / g.nblk1;
  g.slice_pts = (uint32_t)std::max<int64_t>(8192, std::min<int64_t>(slice_pts, n / 256));
  g.nblk2 = (int)(nbx + n / g.slice_pts);
  return g;
}

struct SortArgs {
  hipStream_t st;
  int64_t n, xstride;
  int nw, nf, fb, tshift, nbx;
  uint32_t nf_fix, wbias;
  double scale;
  uint64_t* start;
  int* flags;
};

// Counts and offsets of the first pass.
template <typename TX>
void sort2_first(const SortArgs& a, const TX* X, const Sort2Geom& g, const Sort2Bufs& b) {
  hipLaunchKernelGGL(k_s2_count1<TX>, dim3(g.nblk1), dim3(BT), 0, a.st, X, a.n, a.xstride, a.scale, a.nf_fix, a.fb,
                     a.wbias, a.tshift, a.nbx, a.nbx, g.chunk1, b.cnt1, b.rowtot, a.flags);
  hipLaunchKernelGGL(k_s2_scan1, dim3(a.nbx), dim3(1024), 0, a.st, b.cnt1, a.nbx, g.nblk1, b.rowtot, b.start1);
}

// Counts, offsets and scatter of the second pass.
template <int WV, bool kPosition, int NPT>
void sort2_second(const SortArgs& a, const Sort2Geom& g, const Sort2Bufs& b, uint32_t* crd, uint32_t* wts) {
  const uint2* c1 = reinterpret_cast<const uint2*>(b.crd1);
  hipLaunchKernelGGL(k_s2_count2, dim3(g.nblk2), dim3(BT), 0, a.st, c1, b.start1, g.slice_pts, a.fb, a.wbias, a.nf,
                     a.tshift, a.nbx, b.cnt2);
  hipLaunchKernelGGL(k_s2_scan2, dim3(a.nbx), dim3(1024), 0, a.st, b.cnt2, b.start1, g.slice_pts, a.nbx, a.start);
  hipLaunchKernelGGL((k_s2n_scatter2<WV, kPosition, NPT>), dim3(g.nblk2), dim3(BT), sizeof(StageN<WV, NPT>), a.st, c1,
                     b.wts1, b.start1, b.cnt2, g.slice_pts, a.fb, a.wbias, a.nf, a.tshift, a.nbx,
                     reinterpret_cast<uint2*>(crd), wts);
}

template <int WV, typename TX>
void sort2_narrow(const SortArgs& a, const TX* X, const TX* Y, const Sort2Geom& g, const Sort2Bufs& b, uint32_t* crd,
                  uint32_t* wts) {
  if (sort2_one_pass(a.n, a.nbx, a.nw)) {
    const int nb = a.nbx * a.nbx;
    uint32_t* cnt = b.crd1;   // [nblk1][nb]; the first pass's records are not needed
    hipLaunchKernelGGL((k_s2_count1<TX, true>), dim3(g.nblk1), dim3(BT), 0, a.st, X, a.n, a.xstride, a.scale, a.nf_fix,
                       a.fb, a.wbias, a.tshift, nb, a.nbx, g.chunk1, cnt, b.rowtot, a.flags);
    hipLaunchKernelGGL(k_s2_scan_one, dim3((nb + 15) / 16), dim3(1024), 0, a.st, cnt, nb, g.nblk1, b.rowtot, a.start);
    hipLaunchKernelGGL((k_s2n_scatter1<TX, WV, true>), dim3(g.nblk1), dim3(BT),
                       sizeof(StageN<WV, one_ppt<TX, WV>(), KONE>), a.st, X, a.n, a.xstride, Y, a.nw, a.scale, a.nf_fix,
                       a.fb, a.wbias, a.tshift, nb, a.nbx, g.chunk1, cnt, reinterpret_cast<uint2*>(crd), wts, a.flags);
    return;
  }
  sort2_first(a, X, g, b);
  hipLaunchKernelGGL((k_s2n_scatter1<TX, WV, false>), dim3(g.nblk1), dim3(BT), sizeof(StageN<WV>), a.st, X, a.n,
                     a.xstride, Y, a.nw, a.scale, a.nf_fix, a.fb, a.wbias, a.tshift, a.nbx, a.nbx, g.chunk1, b.cnt1,
                     reinterpret_cast<uint2*>(b.crd1), b.wts1, a.flags);
  sort2_second<WV, false, narrow_ppt<WV>()>(a, g, b, crd, wts);
}

// Pass 2 of the 16-word records moves the coordinates and each point's position in the pass-1 output
// (into wts, one word per point); the weight blocks stay grouped by bin row in b.wts1.  Its records are
// 12 B, so a batch takes kPosPpt points per thread.
template <typename TX>
void sort2_wide(const SortArgs& a, const TX* X, const TX* Y, const Sort2Geom& g, const Sort2Bufs& b, uint32_t* crd,
                uint32_t* wts) {
  sort2_first(a, X, g, b);
  hipLaunchKernelGGL(k_s2_scatter1<TX>, dim3(g.nblk1), dim3(BT), sizeof(Stage), a.st, X, a.n, a.xstride, Y, a.nw,
                     a.scale, a.nf_fix, a.fb, a.wbias, a.tshift, a.nbx, g.chunk1, b.cnt1,
                     reinterpret_cast<uint2*>(b.crd1), reinterpret_cast<uint4*>(b.wts1), a.flags);
  sort2_second<1, true, kPosPpt>(a, g, b, crd, wts);
}

template <typename TX>
fk_status sort2_typed(const SortArgs& a, const TX* X, const TX* Y, const Sort2Geom& g, const Sort2Bufs& b,
                      uint32_t* crd, uint32_t* wts) {
  switch (sort2_words(a.nw)) {
    case 0: sort2_narrow<0>(a, X, Y, g, b, crd, wts); break;
    case 1: sort2_narrow<1>(a, X, Y, g, b, crd, wts); break;
    case 2: sort2_narrow<2>(a, X, Y, g, b, crd, wts); break;
    case 4: sort2_narrow<4>(a, X, Y, g, b, crd, wts); break;
    case 8: sort2_narrow<8>(a, X, Y, g, b, crd, wts); break;
    default: sort2_wide(a, X, Y, g, b, crd, wts); break;
  }
  return hipGetLastError() == hipSuccess ? FK_OK : FK_EHIP;
}

template <typename TX, int R>
void sort3_run(const SortArgs& a, const TX* X, const TX* Y, const Sort2Geom& g, const Sort2Bufs& b, const Bin3& bin,
               int nrow, uint32_t* rec) {
  const int ncol = 1 << bin.lo;
  hipLaunchKernelGGL(k_s3_count1<TX>, dim3(g.nblk1), dim3(BT), 0, a.st, X, a.n, a.xstride, a.scale, a.nf_fix, bin, nrow,
                     g.chunk1, b.cnt1, b.rowtot, a.flags);
  hipLaunchKernelGGL(k_s2_scan1, dim3(nrow), dim3(1024), 0, a.st, b.cnt1, nrow, g.nblk1, b.rowtot, b.start1);
  hipLaunchKernelGGL((k_s3_scatter1<TX, R>), dim3(g.nblk1), dim3(BT), sizeof(Stage3<R>), a.st, X, a.n, a.xstride, Y,
                     a.scale, a.nf_fix, bin, nrow, g.chunk1, b.cnt1, b.crd1, a.flags);
  hipLaunchKernelGGL(k_s3_count2<R>, dim3(g.nblk2), dim3(BT), 0, a.st, b.crd1, b.start1, nrow, g.slice_pts, bin, b.cnt2);
  hipLaunchKernelGGL(k_s2_scan2, dim3(nrow), dim3(1024), 0, a.st, b.cnt2, b.start1, g.slice_pts, ncol, a.start);
  hipLaunchKernelGGL(k_s3_scatter2<R>, dim3(g.nblk2), dim3(BT), sizeof(Stage3<R>), a.st, b.crd1, b.start1, nrow, b.cnt2,
                     g.slice_pts, bin, rec);
}

template <typename TX>
fk_status sort3_typed(const SortArgs& a, const TX* X, const TX* Y, const Sort2Geom& g, const Sort2Bufs& b,
                      const Bin3& bin, int nrow, uint32_t* rec) {
  switch (a.nw) {
    case 0: sort3_run<TX, 3>(a, X, Y, g, b, bin, nrow, rec); break;
    case 1: sort3_run<TX, 4>(a, X, Y, g, b, bin, nrow, rec); break;
    case 2: sort3_run<TX, 5>(a, X, Y, g, b, bin, nrow, rec); break;
    case 3: sort3_run<TX, 6>(a, X, Y, g, b, bin, nrow, rec); break;
    case 4: sort3_run<TX, 7>(a, X, Y, g, b, bin, nrow, rec); break;
    case 5: sort3_run<TX, 8>(a, X, Y, g, b, bin, nrow, rec); break;
    case 6: sort3_run<TX, 9>(a, X, Y, g, b, bin, nrow, rec); break;
    case 7: sort3_run<TX, 10>(a, X, Y, g, b, bin, nrow, rec); break;
    case 8: sort3_run<TX, 11>(a, X, Y, g, b, bin, nrow, rec); break;
    default: return FK_EINVAL;
  }
  return hipGetLastError() == hipSuccess ? FK_OK : FK_EHIP;
}

int sort3_bits(int nbx) {
  int b = 0;
  while ((1 << b) < nbx) ++b;
  return 3 * b;
}

}  // namespace

bool sort2_ok(int nbx) { return nbx >= 1 && nbx <= KMAX; }

int sort2_words(int nw) {
  if (nw >= 8) return 16;
  if (nw == 0) return 0;
  int wv = 1;
  while (wv < nw) wv <<= 1;
  return wv;
}

// One counting pass over all bins instead of two over rows and columns, wherever the bins are
// few enough for their cursors and a batch in LDS: 1024 bins, 2e7 points without targets 416 -> 168 us, 1e8 points
// with one target 1390 -> 1017 us, 30011 points with three 36 -> 23 us (and three launches less).
// The counts take the place of the first pass's records (2 n words, at least 1366 points for 1024 bins).
bool sort2_one_pass(int64_t n, int nbx, int nw) { return nw <= 7 && nbx * nbx <= KONE && n >= 4096; }

size_t sort2_totals(int64_t n, int nbx, int nw) { return (size_t)nbx * (sort2_one_pass(n, nbx, nw) ? nbx : 1); }

void sort2_carve(Carve& cv, int64_t n, int nbx, int wv, Sort2Bufs* b) {
  // the most first-pass workgroups and second-pass slices that any shape takes
  const Sort2Geom g = sort2_geom(n, nbx, kSortBlkMax, kSortSliceMin);
  b->cnt1 = cv.take<uint32_t>((size_t)g.nblk1 * nbx);
  b->start1 = cv.take<uint64_t>((size_t)nbx + 1);
  b->cnt2 = cv.take<uint32_t>((size_t)g.nblk2 * nbx);
  b->crd1 = cv.take<uint32_t>((size_t)n * 2);
  b->wts1 = cv.take<uint32_t>((size_t)n * wv);
}

fk_status sort2(hipStream_t st, const void* X, fk_dtype dt, int64_t n, int64_t xstride, const void* Y, int nw,
                int nf, int fb, int W, double scale, int tshift, int nbx, const T1Shape& shape, Sort2Bufs b,
                uint32_t* totals, uint32_t* crd, uint32_t* wts, uint64_t* start, int* flags) {
  if (!sort2_ok(nbx) || nw > 16 || (nf & (nf - 1)) != 0 || (nbx << tshift) != nf) return FK_EINVAL;
  if (n > (int64_t)0xffffffff) return FK_EINVAL;   // positions are 32-bit
  if (shape.sort_blk < 1 || shape.sort_blk > kSortBlkMax || shape.sort_slice < kSortSliceMin) return FK_EINVAL;
  const Sort2Geom g = sort2_geom(n, nbx, shape.sort_blk, shape.sort_slice);
  b.rowtot = totals;
  const uint32_t one = 1u << fb;
  const SortArgs a{st,  n,      xstride, nw,
                   nf,  fb,     tshift,  nbx,
                   (uint32_t)nf << fb, (one - 1u) + 8u * one - ((uint32_t)W << (fb - 1)), scale, start, flags};
  if (dt == FK_F64)
    return sort2_typed(a, static_cast<const double*>(X), static_cast<const double*>(Y), g, b, crd, wts);
  return sort2_typed(a, static_cast<const float*>(X), static_cast<const float*>(Y), g, b, crd, wts);
}

bool sort3_ok(int nf, int64_t n, int nw) {
  return nf >= 16 && (nf & (nf - 1)) == 0 && sort3_bits(nf / 8) <= 15 && n <= (int64_t)0xffffffff && nw <= 8;
}

void sort3_carve(Carve& cv, int64_t n, int nf, int nw, Sort2Bufs* b) {
  const int bits = sort3_bits(nf / 8), lo = bits / 2, nrow = 1 << (bits - lo);
  const Sort2Geom g = sort2_geom(n, nrow, kSortBlkMax, kSortSliceMin);
  b->rowtot = cv.take<uint32_t>((size_t)nrow);
  b->cnt1 = cv.take<uint32_t>((size_t)g.nblk1 * nrow);
  b->start1 = cv.take<uint64_t>((size_t)nrow + 1);
  b->cnt2 = cv.take<uint32_t>((size_t)g.nblk2 << lo);
  b->crd1 = cv.take<uint32_t>((size_t)n * (3 + nw));
}

fk_status sort3(hipStream_t st, const void* X, fk_dtype dt, int64_t n, int64_t xstride, const void* Y, int nw, int nf,
                int fb, int W, double scale, const Sort2Bufs& b, uint32_t* rec, uint64_t* start, int* flags) {
  if (!sort3_ok(nf, n, nw)) return FK_EINVAL;
  const int bits = sort3_bits(nf / 8), lo = bits / 2, nrow = 1 << (bits - lo);
  const Sort2Geom g = sort2_geom(n, nrow, 512, 65536);
  const uint32_t one = 1u << fb;
  const uint32_t wbias = (one - 1u) + 8u * one - ((uint32_t)W << (fb - 1));
  const Bin3 bin{wbias, fb, nf, nf / 8, lo};
  const SortArgs a{st, n, xstride, nw, nf, fb, 3, nf / 8, (uint32_t)nf << fb, wbias, scale, start, flags};
  FK_HIP(hipMemsetAsync(b.rowtot, 0, sizeof(uint32_t) * nrow, st));
  if (dt == FK_F64)
    return sort3_typed(a, static_cast<const double*>(X), static_cast<const double*>(Y), g, b, bin, nrow, rec);
  return sort3_typed(a, static_cast<const float*>(X), static_cast<const float*>(Y), g, b, bin, nrow, rec);
}

}  // namespace fk
