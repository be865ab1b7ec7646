// The whole recurrence of a small matrix of 1x1 blocks in one launch: one workgroup per probe column
// keeps y_k and y_{k-1} in LDS, runs every step, sums the column's moments and, for the density,
// accumulates P r.  (k_step.hip: a launch per step, for matrices that do not fit.)
//
// A step of such a matrix is shorter than its launch, and columns need nothing of each other, so a step
// here ends with a barrier of the workgroup.  Bound by the LDS gathers and the barrier where the matrix
// stays in registers, by the entries from the L2 (46 to 64 bytes a clock per compute unit) where it does
// not.  Calls of 200 terms with launches and so, us: moments, FP64, 64 probes, 512 rows 622 and 183, 4,096
// rows 723 and 261, 8,000 rows 969 and 715; 4,096 rows, 256 probes 1,154 and 346; density, dense probes, 300
// irregular rows 1,279 and 208, 5,003 rows 1,820 and 1,268.
//
// Rows are sorted by their length and taken 64 at a time, a lane per row (slices): entry pair q of a slice
// is one load of two values and one of two 16-bit columns per lane, coalesced.  Where a wave's slices fit
// its registers (RJ slices of at most WP pairs) the matrix is read once per call, otherwise (RJ = 0) each
// step streams it from the L2.  Row sums run in the order of the columns, as in k_step.hip.
#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

namespace {

constexpr int kRunBatch = 16;  // steps between reductions of the waves' moment sums

template <typename VT>
struct Pair {
  VecN<VT, 2> v;
  uint32_t c;
};

// Sum over the wave, to every lane, by register exchanges: a step waits for it.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint2 u = __builtin_bit_cast(uint2, v);
  return __builtin_bit_cast(double,
                            make_uint2((unsigned)__builtin_amdgcn_update_dpp(0, (int)u.x, CTRL, 0xf, 0xf, true),
                                       (unsigned)__builtin_amdgcn_update_dpp(0, (int)u.y, CTRL, 0xf, 0xf, true)));
}
__device__ __forceinline__ double run_sum(double v) {
  v += dpp<0xb1>(v);   // lane ^ 1
  v += dpp<0x4e>(v);   // lane ^ 2
  v += dpp<0x141>(v);  // the other quad of eight lanes
  v += dpp<0x140>(v);  // the other eight of sixteen
  const uint2 u = __builtin_bit_cast(uint2, v);
  const auto lo = __builtin_amdgcn_permlane16_swap(u.x, u.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(u.y, u.y, false, false);
  v = __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
  const uint2 w = __builtin_bit_cast(uint2, v);
  const auto lp = __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false);
  const auto hp = __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false);
  return __builtin_bit_cast(double, make_uint2(lp[0], hp[0])) + __builtin_bit_cast(double, make_uint2(lp[1], hp[1]));
}

}  // namespace

// MODE 0: moments r . y_k; 1: those and the density accumulator; 2: moments by doubling
template <typename VT, int MODE, int RJ, int WP>
__global__ __launch_bounds__(64 * kRunWaves) void k_run1(RunArgs a) {
  extern __shared__ double lds[];
  constexpr bool DBL = MODE == 2;
  const int n = a.n, c = blockIdx.x, sp = a.sp, tid = threadIdx.x, T = blockDim.x;
  const int wave = uniform(tid >> 6), lane = tid & 63, nw = T >> 6;
  VT *Y0 = reinterpret_cast<VT *>(lds), *Y1 = Y0 + n;
  __shared__ double red[2][kRunBatch][2][kRunWaves];
  __shared__ double first[2];  // moments 0 and 1
  VT *out_acc = MODE == 1 ? static_cast<VT *>(a.acc) : nullptr;
  if (c >= a.s) {  // padding column: no probe, weight zero
    for (int64_t k = tid; k < a.p; k += T) a.moments[k * sp + c] = 0.0;
    if (MODE == 1)
      for (int64_t i = tid; i < n; i += T) out_acc[i * sp + c] = (VT)0;
    return;
  }
  VT *accT = MODE == 1 ? static_cast<VT *>(a.work) + (int64_t)c * n : nullptr;
  double *rT = a.rwork ? a.rwork + (int64_t)c * n : nullptr;  // dense probes of direct moments
  const double alpha0 = MODE == 1 ? a.coef[0] : 0.0;
  uint32_t bits = 0;  // sign probes of the thread's rows

  Pair<VT> h[RJ > 0 ? RJ : 1][WP];
  int row[RJ > 0 ? RJ : 1];
  const VecN<VT, 2> *vals = static_cast<const VecN<VT, 2> *>(a.vals);
  auto load = [&](int64_t q) {
    Pair<VT> e;
    e.v = vals[q * 64 + lane];
    e.c = a.cols[q * 64 + lane];
    return e;
  };
  if constexpr (RJ > 0) {
#pragma unroll
    for (int j = 0; j < RJ; ++j) {
      const int sl = wave + j * nw;
      const int q0 = sl < a.n_slices ? sld(a.slice + sl) : 0, q1 = sl < a.n_slices ? sld(a.slice + sl + 1) : 0;
      row[j] = sl < a.n_slices ? a.perm[sl * 64 + lane] : -1;
#pragma unroll
      for (int q = 0; q < WP; ++q) {
        h[j][q].v.v[0] = h[j][q].v.v[1] = (VT)0;
        h[j][q].c = 0;
        if (q0 + q < q1) h[j][q] = load(q0 + q);
      }
    }
  }
  // f(row, slice number of the wave)
  auto rows = [&](auto &&f) {
    if constexpr (RJ > 0) {
#pragma unroll
      for (int j = 0; j < RJ; ++j) f(row[j], j);
    } else {
      for (int sl = wave, j = 0; sl < a.n_slices; sl += nw, ++j) f(a.perm[sl * 64 + lane], j);
    }
  };
  double m1 = 0.0, m2 = 0.0;
  rows([&](int I, int j) {
    if (I < 0) return;
    const double r = probe_value(a.sgn, a.rden, I, sp, c);
    if (r > 0.0) bits |= 1u << j;
    const VT v = (VT)r;
    Y0[I] = v;
    m1 = fma(r, (double)v, m1);
    if (rT) rT[I] = r;
    if (MODE == 1) accT[I] = (VT)(alpha0 * (double)v);
  });
  auto sums = [&](int set, int at) {
    m1 = run_sum(m1);
    if (DBL) m2 = run_sum(m2);
    if (lane == 0) {
      red[set][at][0][wave] = m1;
      if (DBL) red[set][at][1][wave] = m2;
    }
    m1 = m2 = 0.0;
  };
  auto total = [&](int set, int at, int which) {
    double t = red[set][at][which][0];
    for (int w = 1; w < nw; ++w) t += red[set][at][which][w];
    return t;
  };
  auto put = [&](int64_t k, double v) {
    if (k >= a.p) return;
    a.moments[k * sp + c] = v;
    if (k > 0 && !(fabs(v) <= first[0] * (1.0 + a.tol) + 1e-300)) atomicOr(a.flags, 4);
  };
  sums(0, 0);
  __syncthreads();
  if (tid == 0) {
    first[0] = total(0, 0, 0);
    put(0, first[0]);
  }
  __syncthreads();

  int64_t done = 0;  // density terms added
  for (int64_t k = 0; k < a.steps; ++k) {
    const VT *cur = k & 1 ? Y1 : Y0;
    VT *out = k & 1 ? Y0 : Y1;  // holds y_{k-1}
    int m = 0;
    VT al[3] = {(VT)0, (VT)0, (VT)0};
    if (MODE == 1) {
      const int pending = (int)(k + 1 - done);
      if (pending == 3 || k + 1 == a.steps) {
        m = pending;
        for (int i = 0; i < 3; ++i)
          if (i < m) al[i] = (VT)a.coef[done + 1 + i];
        done = k + 1;
      }
    }
    // what a row needs beside its neighbours, read ahead of them
    struct Own {
      VT old, x, acc;
      double r;
    };
    auto own = [&](int I, int j) {
      const int Ic = I < 0 ? 0 : I;
      Own o;
      o.old = out[Ic];
      if (DBL || m >= 2) o.x = cur[Ic];
      if (!DBL) o.r = rT ? rT[Ic] : (bits >> j) & 1u ? 1.0 : -1.0;
      if (MODE == 1 && m > 0) o.acc = accT[Ic];
      return o;
    };
    auto finish = [&](int I, const Own &o, VT s) {
      if (I < 0) return;
      const VT v = k == 0 ? s : fma((VT)-1, o.old, (VT)2 * s);
      out[I] = v;
      if (DBL) {
        m1 = fma((double)v, (double)v, m1);
        m2 = fma((double)v, (double)o.x, m2);
      } else {
        m1 = fma(o.r, (double)v, m1);
      }
      if (MODE == 1 && m > 0) {
        VT t = o.acc;
        if (m == 3) t = fma(al[0], o.old, t);
        if (m >= 2) t = fma(al[m - 2], o.x, t);
        accT[I] = fma(al[m - 1], v, t);
      }
    };
    auto add = [&](const Pair<VT> &e, VT s) {
      s = fma(e.v.v[0], cur[e.c & 0xffffu], s);
      return fma(e.v.v[1], cur[e.c >> 16], s);
    };
    if constexpr (RJ > 0) {
#pragma unroll
      for (int j = 0; j < RJ; ++j) {
        const Own o = own(row[j], j);
        VT s = (VT)0;
#pragma unroll
        for (int q = 0; q < WP; ++q) s = add(h[j][q], s);
        finish(row[j], o, s);
      }
    } else {
      for (int sl = wave, j = 0; sl < a.n_slices; sl += nw, ++j) {
        const int q0 = sld(a.slice + sl), q1 = sld(a.slice + sl + 1);
        const int I = a.perm[sl * 64 + lane];
        VT s = (VT)0;
        Own o;
        for (int q = q0; q < q1; q += WP) {
          Pair<VT> e[WP];
#pragma unroll
          for (int u = 0; u < WP; ++u)
            if (q + u < q1) e[u] = load(q + u);
          if (q == q0) o = own(I, j);
#pragma unroll
          for (int u = 0; u < WP; ++u)
            if (q + u < q1) s = add(e[u], s);
        }
        finish(I, o, s);
      }
    }
    const int set = (int)(k / kRunBatch) & 1, at = (int)(k % kRunBatch);
    sums(set, at);
    __syncthreads();
    // the sums of a batch are added while the waves go on: they write the other set for the next
    // kRunBatch steps
    if (k == 0 || at == kRunBatch - 1 || k + 1 == a.steps) {
      if (DBL && k == 0) {
        if (tid == 0) first[1] = total(0, 0, 1);
        __syncthreads();
      }
      if (tid <= at) {
        const int64_t j = k - at + tid + 1;  // the step's vector y_j
        const double t1 = total(set, tid, 0);
        if (DBL) {
          const double t2 = total(set, tid, 1);
          put(2 * j - 1, j == 1 ? t2 : 2.0 * t2 - first[1]);
          put(2 * j, 2.0 * t1 - first[0]);
        } else {
          put(j, t1);
        }
      }
    }
  }
  if (MODE == 1)
    rows([&](int I, int) {
      if (I >= 0) out_acc[(int64_t)I * sp + c] = accT[I];
    });
}

// matrix values in slice order: dst[e] = h[src[e]], zero where src[e] < 0
template <typename VT>
__global__ __launch_bounds__(kWG) void k_run_fill(const VT *__restrict__ h, const int32_t *__restrict__ src, int64_t n,
                                                  VT *__restrict__ dst) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = src[e] < 0 ? (VT)0 : h[src[e]];
}

hipError_t launch_run_fill(int precision, const void *h, const int32_t *src, int64_t n, void *dst, hipStream_t s) {
  const dim3 grid((unsigned)std::min<int64_t>(4096, (n + kWG - 1) / kWG));
  if (precision == 0)
    hipLaunchKernelGGL(k_run_fill<double>, grid, dim3(kWG), 0, s, static_cast<const double *>(h), src, n,
                       static_cast<double *>(dst));
  else
    hipLaunchKernelGGL(k_run_fill<float>, grid, dim3(kWG), 0, s, static_cast<const float *>(h), src, n,
                       static_cast<float *>(dst));
  return hipGetLastError();
}

namespace {

template <typename VT, int MODE>
const void *run_fn(int slices, int pairs) {
  const int rj = run_held(sizeof(VT), MODE, slices, pairs);
  constexpr bool kFull = sizeof(VT) == 8 && MODE != 2;  // 16 pairs beside their other values would spill
  if (rj > 0 && pairs <= 4) {
    if (rj == 1) return (const void *)k_run1<VT, MODE, 1, 4>;
    if (rj == 2) return (const void *)k_run1<VT, MODE, 2, 4>;
    if constexpr (!kFull) return (const void *)k_run1<VT, MODE, 4, 4>;
  } else if (rj > 0) {
    if (rj == 1) return (const void *)k_run1<VT, MODE, 1, 8>;
    if constexpr (!kFull) return (const void *)k_run1<VT, MODE, 2, 8>;
  }
  return (const void *)k_run1<VT, MODE, 0, 4>;
}

template <typename VT>
const void *run_fn_m(int mode, int slices, int pairs) {
  switch (mode) {
    case 0: return run_fn<VT, 0>(slices, pairs);
    case 1: return run_fn<VT, 1>(slices, pairs);
    default: return run_fn<VT, 2>(slices, pairs);
  }
}

}  // namespace

hipError_t launch_run(int precision, int mode, int max_pairs, const RunArgs &a, hipStream_t s) {
  const int64_t vt = precision == 0 ? 8 : 4;
  if (a.n < 1 || a.n > run_rows((int)vt) || a.sp < 1 || (mode == 1 && (!a.acc || !a.work))) return hipErrorInvalidValue;
  const int waves = std::min(kRunWaves, a.n_slices);
  const void *f = precision == 0 ? run_fn_m<double>(mode, a.n_slices, max_pairs)
                                 : run_fn_m<float>(mode, a.n_slices, max_pairs);
  const int bytes = (int)(2 * vt * a.n);
  // the same value on every call: other threads launch this kernel too
  const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(2 * vt * run_rows((int)vt)));
  if (e != hipSuccess) return e;
  void *args[] = {const_cast<RunArgs *>(&a)};
  return hipLaunchKernel(f, dim3((unsigned)a.sp), dim3(64 * waves), args, bytes, s);
}

}  // namespace rfo
