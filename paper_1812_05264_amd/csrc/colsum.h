// Fixed-order column reduction shared by the conjugate-gradient (overlap) and CGLS
// (rational) kernels.
#pragma once

#include <algorithm>

#include "device_util.h"

namespace rfo {

// Fixed-order column sums of part [nparts][sp] for a workgroup of 64 * kColWaves
// threads that owns the kColCols columns from blockIdx.x * kColCols: lane l of wave w
// adds, for column l % kColCols, the rows h, h + kColPh, ... of phase
// h = w * (64 / kColCols) + l / kColCols in increasing order, and the kColPh phase sums
// are then added in phase order, so the result is bitwise reproducible.  Many short
// chains rather than a few long ones: the partials come from other XCDs' caches, and
// the latency of each dependent round of loads sets the time.  Every thread of the
// workgroup must call it (it has a barrier); the sum of column c (returned in c) is
// returned to the threads with threadIdx.x < kColCols, zero to the others.
constexpr int kColWaves = 16, kColCols = 16, kColPh = kColWaves * (64 / kColCols);

__device__ __forceinline__ double colsum(const double *__restrict__ part, int nparts, int sp,
                                         double (*red)[kColCols], int &c) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int cl = lane % kColCols, ph = wave * (64 / kColCols) + lane / kColCols;
  c = blockIdx.x * kColCols + cl;
  double s = 0.0;
  if (c < sp) {
#pragma unroll 4
    for (int b = ph; b < nparts; b += kColPh) s += part[(int64_t)b * sp + c];
  }
  red[ph][cl] = s;
  __syncthreads();
  if (threadIdx.x >= kColCols) return 0.0;
  double t = red[0][cl];
  for (int h = 1; h < kColPh; ++h) t += red[h][cl];
  return t;
}

// ---------------------------------------------------------------------------
// Slabs: the vector updates of the solvers take a slab of C columns and a share of the rows per
// workgroup, and each first sums its columns' partials of the product before it.  All workgroups of a
// slab add them in the same order, so they agree on the scalars bitwise.
//
// C = 16: no launch of a reduction stands between the product and the update; on small matrices an
// iteration's time is its launches.  CGLS update and direction with and without, 128 columns, us: 117
// rows 11.0 + 7.5 and 4.2 + 5.3; 2,250 rows 11.2 + 9.3 and 5.0 + 6.4; 9,000 rows 18.5 + 20.8 and 14.9 + 20.4.
// C = 64: for vectors of 16 MiB and more (slab_wide) k_colreduce sums the partials to one row first, and
// the shares' rows interleave, so that all workgroups stream through the vectors together
// (64,000 rows, update and direction with their sums 65 and 122 us; 67 and 157 in slabs of 16).
// ---------------------------------------------------------------------------
constexpr int kSlabThreads = 1024, kSlabWaves = kSlabThreads / 64;

inline bool slab_wide(int64_t n, int sp) { return n * sp * (int64_t)sizeof(double) >= (int64_t)16 << 20; }

// Sum of v over the row lanes of the thread's column, to every thread, in a fixed order.
template <int C>
__device__ __forceinline__ double slab_total(double v, double (*red)[C]) {
#pragma unroll
  for (int o = C; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
  const int cl = threadIdx.x % C;
  if ((threadIdx.x & 63) < C) red[threadIdx.x >> 6][cl] = v;
  __syncthreads();
  double t = red[0][cl];
#pragma unroll
  for (int w = 1; w < kSlabWaves; ++w) t += red[w][cl];
  return t;
}

// Column sum of part [nparts][sp] for the thread's column c (C = 64: nparts is 1, no barrier).
template <int C>
__device__ __forceinline__ double slab_sum(const double *__restrict__ part, int nparts, int sp, int c,
                                           double (*red)[C]) {
  if (C == 64) return part[c];
  double s = 0.0;
#pragma unroll 8
  for (int b = threadIdx.x / C; b < nparts; b += kSlabThreads / C) s += part[(int64_t)b * sp + c];
  return slab_total<C>(s, red);
}

// row shares: a row per row lane, and no more workgroups than are resident (two per compute unit:
// a second round would wait for its sums a second time); in whole eights
template <int C>
inline int slab_shares(int64_t n, int sp) {
  const int64_t most = std::max<int64_t>(1, 512 / (sp / C));
  const int64_t shares = std::min<int64_t>(most, (n + kSlabThreads / C - 1) / (kSlabThreads / C));
  return (int)(shares >= 8 ? shares / 8 * 8 : shares);
}

// A workgroup's column (per thread) and rows.  C = 16: the slabs of a share go to one XCD, whose shares
// are neighbours, as in the products: whole rows, in the L2 that holds them.
template <int C>
struct Slab {
  int share, c;
  bool first;            // the workgroup that stores its slab's scalars
  int64_t lo, hi, step;  // the thread's rows
  __device__ Slab(int64_t n, int sp, int shares) {
    const int slabs = sp / C, b = blockIdx.x;
    int slab;
    if (shares % 8 == 0) {
      slab = (b >> 3) % slabs;
      share = (b & 7) * (shares >> 3) + (b >> 3) / slabs;
    } else {
      slab = b % slabs;
      share = b / slabs;
    }
    first = share == 0;
    c = slab * C + threadIdx.x % C;
    constexpr int R = kSlabThreads / C;
    if (C == 16) {
      lo = n * share / shares + threadIdx.x / C;
      hi = n * (share + 1) / shares;
      step = R;
    } else {
      lo = (int64_t)share * R + threadIdx.x / C;
      hi = n;
      step = (int64_t)shares * R;
    }
  }
};

// The elements of a kernel that leaves no partials (grid: Writer<C>::grid).  C = 16: a slab's rows; C =
// 64: 1024 neighbouring elements, one per thread.
template <int C>
struct Writer {
  int c;
  int64_t e, end, step;
  bool lead;   // the workgroup that stores its columns' scalars (C = 64: every one)
  bool first;  // its threads that do
  __device__ Writer(int64_t n, int sp) {
    if (C == 16) {
      const Slab<16> sl(n, sp, gridDim.x / (sp / 16));
      c = sl.c;
      e = sl.lo * sp + c;
      end = sl.hi * sp;
      step = sl.step * sp;
      lead = sl.first;
      first = lead && threadIdx.x < 16;
    } else {
      e = (int64_t)blockIdx.x * kSlabThreads + threadIdx.x;
      c = (int)(e % sp);
      end = n * sp;
      step = end;
      lead = true;
      first = e < sp;
    }
  }
  static unsigned grid(int64_t n, int64_t rows, int sp) {
    return C == 16 ? (unsigned)(sp / 16 * slab_shares<16>(n, sp)) : (unsigned)((rows * sp + kSlabThreads - 1) / kSlabThreads);
  }
};

}  // namespace rfo
