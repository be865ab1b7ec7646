// Masked outer products of 9x9 block vectors (density blocks and the segment gradient, see
// k_reduce.hip) with FP64 sums on the matrix cores.
//
// A block's sum over the probes is a 9 x K by K x 9 contraction, K = the probes:
//   G_IJ (+)= sum_t coef_t sum_c w_c (X_I[:, c] Y_J[:, c]^T (+ Y_I[:, c] X_J[:, c]^T)).
// v_mfma_f64_4x4x4 runs four independent 4x4x4 products per instruction; here they are four
// slices of K for the same 4 rows and 4 columns of the block, so one instruction takes 16 probes
// and a 4x4 tile of the block costs one register pair.  The nine rows are 4 + 4 + 1: rows and columns
// 0..7 make four tiles without padding, row 8 and column 8 are summed on the vector units beside
// them.  (v_mfma_f64_16x16x4 would compute 256 outputs for 81, at 46 TFLOP/s against 74.)
//
// The instruction wants the row of an operand in the low two bits of the lane.  Loading it so
// would take every four lanes of a load to four rows (at 16,000 atoms 3.55e9 cache accesses per launch
// against the 1.48e9 of a block per wave on the vector units, and slower: 582 ms against 556 for a gradient
// of 500 terms); the rows are therefore loaded with lanes along the probes and
// each four of them transposed within quads of lanes (two rounds of DPP exchanges).
//
// A workgroup takes up to kSddmm9Group blocks of one block row, so X_I and Y_I are loaded once for
// all of them and few block rows are in flight on an XCD; its waves split the (step t, probe set)
// items of the contraction between them and add their sums at the end in wave order: the result
// does not depend on timing.  The (step, probe) pairs are taken 64 to an item in one sequence, so
// a ragged probe count leaves no lanes idle.  FP32 vectors are converted on loading; every product and sum is FP64.
//
// Bound by the bytes of X_t and Y_t that miss the L2 at 16,000 atoms, by the instructions of the products
// and exchanges below about 4,000.  Gradient of 130 terms with the vector-unit kernel that took a block per
// wave, and with this one, ms: 16,000 atoms FP64 256 probes 147 and 143, 6,000 atoms 100 probes 31.5 and
// 25.4, 500 atoms 128 probes 5.5 and 3.5; 4,000 atoms FP32 288 probes (800 terms) 180 and 156.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

namespace {

constexpr int kMaxWaves9 = 8;

typedef const __attribute__((address_space(1))) char *GlobalBytes;

template <int I>
__device__ __forceinline__ unsigned quad_lane(unsigned v) {  // the value of lane I of the quad
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, I * 0x55, 0xf, 0xf, true);
}

// 32-bit words per lane of the nine rows of a block row, one probe a lane
template <typename VT>
struct Raw9 {
  unsigned v[9][sizeof(VT) / 4];
  __device__ __forceinline__ void set(int k, VT x) {
    if constexpr (sizeof(VT) == 8) {
      const uint2 u = __builtin_bit_cast(uint2, x);
      v[k][0] = u.x;
      v[k][1] = u.y;
    } else {
      v[k][0] = __builtin_bit_cast(unsigned, x);
    }
  }
};

// In a quad of lanes, row j of the lane p -> entry j of lane r: (row r, probe of lane j), for rows
// 0..3 and 4..7.
template <typename VT>
__device__ __forceinline__ void quad_transpose(Raw9<VT> &a, int lane) {
  const bool odd = lane & 1, high = lane & 2;
#pragma unroll
  for (int w = 0; w < (int)sizeof(VT) / 4; ++w)
#pragma unroll
    for (int b = 0; b < 8; b += 4) {
#pragma unroll
      for (int j = 0; j < 4; j += 2) quad_swap<1>(a.v[b + j][w], a.v[b + j + 1][w], odd);
#pragma unroll
      for (int j = 0; j < 2; ++j) quad_swap<2>(a.v[b + j][w], a.v[b + j + 2][w], high);
    }
}

// Operand of K chunk i (the probes of lane i of every quad): rows 0..3 (k = 0) and 4..7 (1) in the
// lanes' low bits, or row 8 (2)
template <typename VT>
__device__ __forceinline__ double operand(const Raw9<VT> &a, int k, int i) {
  unsigned v[2] = {0, 0};
#pragma unroll
  for (int w = 0; w < (int)sizeof(VT) / 4; ++w) {
    v[w] = a.v[k < 2 ? 4 * k + i : 8][w];
    if (k == 2) v[w] = i == 0 ? quad_lane<0>(v[w]) : i == 1 ? quad_lane<1>(v[w]) : i == 2 ? quad_lane<2>(v[w]) : quad_lane<3>(v[w]);
  }
  if constexpr (sizeof(VT) == 8) return __builtin_bit_cast(double, make_uint2(v[0], v[1]));
  else return (double)__builtin_bit_cast(float, v[0]);
}

}  // namespace

// PROBES: the right operand is the probes, 1 sign bits, 2 dense FP64
template <typename VT, bool SYM, int PROBES>
__global__ __launch_bounds__(64 * kMaxWaves9) __attribute__((amdgpu_waves_per_eu(2))) void k_sddmm9(SddmmArgs a) {
  constexpr int GB = kSddmm9Group;
  const int wave = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const int r = lane & 3;
  const int64_t gi = xcd_logical(blockIdx.x, gridDim.x);
  const int64_t q0 = sld(a.grp + gi), q1 = sld(a.grp + gi + 1);
  const int sp = a.sp;
  const int c_end = a.s_live > 0 ? min(a.s_live, sp) : sp;  // zero-weight columns past s_live add nothing
  // (step, probe) pairs in order, 64 to an item: a ragged probe count fills the lanes all the same.
  // (spread = 0, for step strides too far apart for a 32-bit offset: whole steps, padded.)
  const int pitch = a.spread ? c_end : ((c_end + 63) & ~63);
  const int64_t pairs = (int64_t)a.count * pitch;
  const int items = (int)((pairs + 63) >> 6);
  extern __shared__ double red[];  // [nw][GB][81]

  auto body = [&](auto nbc) {
    constexpr int NB = decltype(nbc)::value;
    int64_t nz[NB], J[NB];
#pragma unroll
    for (int g = 0; g < NB; ++g) {
      nz[g] = a.nzlist ? sld(a.nzlist + q0 + g) : q0 + g;
      J[g] = sld(a.col + nz[g]);
    }
    const int64_t I = sld(a.brow + nz[0]);
    double d[NB][2][2], e[NB][5];
#pragma unroll
    for (int g = 0; g < NB; ++g) {
#pragma unroll
      for (int k = 0; k < 4; ++k) d[g][k >> 1][k & 1] = 0.0;
#pragma unroll
      for (int k = 0; k < 5; ++k) e[g][k] = 0.0;
    }
    for (int it = wave; it < items; it += nw) {
      const int64_t first = (int64_t)it << 6;
      const int t0 = (int)(first / pitch);
      const int x = (int)(first - (int64_t)t0 * pitch) + lane, dt0 = x / pitch;
      // lanes past the last pair read the item's first step with weight zero: no branches
      const bool live = t0 + dt0 < a.count && x - dt0 * pitch < c_end;
      const int dt = live ? dt0 : 0, c = live ? x - dt0 * pitch : 0;
      const double w = live ? a.w[c] * (a.scale * ((a.j0 + t0 + dt == 0) ? a.first : a.rest)) : 0.0;
      const VT *X = static_cast<const VT *>(a.xbase) + (int64_t)t0 * a.xstride;
      const VT *Y = PROBES ? nullptr : static_cast<const VT *>(a.ybase) + (int64_t)t0 * a.ystride;
      const int64_t rowb = (int64_t)sp * (int)sizeof(VT);
      const uint32_t xoff = ((uint32_t)dt * (uint32_t)a.xstride + (uint32_t)c) * (uint32_t)sizeof(VT);
      const uint32_t yoff = ((uint32_t)dt * (uint32_t)a.ystride + (uint32_t)c) * (uint32_t)sizeof(VT);
      // one scalar base per row (opaque, or the compiler keeps the lanes' 64-bit addresses of every
      // block of the group over the loop)
      auto rows = [&](const VT *V, uint32_t off, int64_t B, Raw9<VT> &o) {
        GlobalBytes base = (GlobalBytes)reinterpret_cast<const char *>(V) + B * (9 * rowb);
        asm volatile("" : "+s"(base));
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          GlobalBytes row = base + k * rowb;
          asm volatile("" : "+s"(row));
          o.set(k, *reinterpret_cast<const __attribute__((address_space(1))) VT *>(row + off));
        }
      };
      // left operands with their weights, held for all blocks of the group
      double xa[3][4], ya[3][4];
      auto left = [&](const VT *V, uint32_t off, double(&o)[3][4]) {
        Raw9<VT> v;
        rows(V, off, I, v);
        Raw9<double> h;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          if constexpr (sizeof(VT) == 8) h.set(k, w * __builtin_bit_cast(double, make_uint2(v.v[k][0], v.v[k][1])));
          else h.set(k, w * (double)__builtin_bit_cast(float, v.v[k][0]));
        }
        quad_transpose(h, lane);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[k][i] = operand(h, k, i);
      };
      left(X, xoff, xa);
      if (SYM) left(Y, yoff, ya);
      auto outer = [&](int g, const double(&l)[3][4], const auto &v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double b0 = operand(v, 0, i), b1 = operand(v, 1, i), b8 = operand(v, 2, i);
          const double a0 = l[0][i], a1 = l[1][i], a8 = l[2][i];
          d[g][0][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a0, b0, d[g][0][0], 0, 0, 0);
          d[g][0][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a0, b1, d[g][0][1], 0, 0, 0);
          d[g][1][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a1, b0, d[g][1][0], 0, 0, 0);
          d[g][1][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a1, b1, d[g][1][1], 0, 0, 0);
          e[g][0] = fma(a0, b8, e[g][0]);  // rows 0..3 and 4..7 of column 8
          e[g][1] = fma(a1, b8, e[g][1]);
          e[g][2] = fma(a8, b0, e[g][2]);  // columns 0..3 and 4..7 of row 8
          e[g][3] = fma(a8, b1, e[g][3]);
          e[g][4] = fma(a8, b8, e[g][4]);
        }
      };
      if constexpr (PROBES != 0) {
#pragma unroll
        for (int g = 0; g < NB; ++g) {
          Raw9<double> v;
          if constexpr (PROBES == 1) {
            const int64_t rw = (int64_t)(sp >> 6) * 8;
            GlobalBytes base = (GlobalBytes)reinterpret_cast<const char *>(a.sgn) + J[g] * (9 * rw);
            asm volatile("" : "+s"(base));
#pragma unroll
            for (int k = 0; k < 9; ++k) {
              GlobalBytes row = base + k * rw;
              asm volatile("" : "+s"(row));
              const unsigned b = *reinterpret_cast<const __attribute__((address_space(1))) unsigned *>(row + (uint32_t)(c >> 5) * 4u);
              v.set(k, (b >> (c & 31)) & 1u ? 1.0 : -1.0);
            }
          } else {
            GlobalBytes base = (GlobalBytes)reinterpret_cast<const char *>(a.rden) + J[g] * (9 * 8 * (int64_t)sp);
            asm volatile("" : "+s"(base));
#pragma unroll
            for (int k = 0; k < 9; ++k) {
              GlobalBytes row = base + k * (8 * (int64_t)sp);
              asm volatile("" : "+s"(row));
              v.set(k, *reinterpret_cast<const __attribute__((address_space(1))) double *>(row + (uint32_t)c * 8u));
            }
          }
          quad_transpose(v, lane);
          outer(g, xa, v);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        Raw9<VT> yn, xn;  // the next block's rows, requested before this one's products
        rows(Y, yoff, J[0], yn);
        if (SYM) rows(X, xoff, J[0], xn);
#pragma unroll
        for (int g = 0; g < NB; ++g) {
          Raw9<VT> y = yn, x = xn;
          quad_transpose(y, lane);
          if (SYM) quad_transpose(x, lane);
          __builtin_amdgcn_sched_barrier(0);
          if (g + 1 < NB) {
            rows(Y, yoff, J[g + 1], yn);
            if (SYM) rows(X, xoff, J[g + 1], xn);
          }
          __builtin_amdgcn_sched_barrier(0);
          outer(g, xa, y);
          if (SYM) outer(g, ya, x);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // K slices: lanes 16 row + 4 slice + col of a tile, and lanes 4 slice + r of the edge sums
    double *mine = red + wave * (GB * 81);
#pragma unroll
    for (int g = 0; g < NB; ++g) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        double v = d[g][k >> 1][k & 1];
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 8, 64);
        if ((lane & 12) == 0) mine[g * 81 + (4 * (k >> 1) + (lane >> 4)) * 9 + 4 * (k & 1) + r] = v;
      }
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        double v = e[g][k];
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
        if (lane < (k < 4 ? 4 : 1)) mine[g * 81 + (k < 2 ? (4 * k + r) * 9 + 8 : k < 4 ? 72 + 4 * (k - 2) + r : 80)] = v;
      }
    }
    __syncthreads();
    for (int o = threadIdx.x; o < NB * 81; o += blockDim.x) {
      double v = red[o];
      for (int k = 1; k < nw; ++k) v += red[k * (GB * 81) + o];
      const int g = o / 81;
      double *p = a.G + (a.nzlist ? a.nzlist[q0 + g] : q0 + g) * 81 + (o - g * 81);
      *p = a.accumulate ? *p + v : v;
    }
  };
  switch ((int)(q1 - q0)) {
    case 1: body(std::integral_constant<int, 1>{}); break;
    case 2: body(std::integral_constant<int, 2>{}); break;
    case 3: body(std::integral_constant<int, 3>{}); break;
    case 4: body(std::integral_constant<int, 4>{}); break;
    case 5: body(std::integral_constant<int, 5>{}); break;
    default: body(std::integral_constant<int, GB>{}); break;
  }
}

template <typename VT>
static void launch_sddmm9_t(const SddmmArgs &a, dim3 grid, int waves, hipStream_t s) {
  const size_t lds = (size_t)waves * kSddmm9Group * 81 * sizeof(double);
  const dim3 wg(64 * waves);
  if (a.sym) hipLaunchKernelGGL((k_sddmm9<VT, true, 0>), grid, wg, lds, s, a);
  else if (a.ybase) hipLaunchKernelGGL((k_sddmm9<VT, false, 0>), grid, wg, lds, s, a);
  else if (a.sgn) hipLaunchKernelGGL((k_sddmm9<VT, false, 1>), grid, wg, lds, s, a);
  else hipLaunchKernelGGL((k_sddmm9<VT, false, 2>), grid, wg, lds, s, a);
}

hipError_t launch_sddmm9(int precision, const SddmmArgs &a, int cus, hipStream_t s) {
  if (a.n_grp == 0) return hipSuccess;
  if (a.bd != 9 || !a.grp || (a.sym && !a.ybase) || a.sp % 64 != 0) return hipErrorInvalidValue;
  // four waves per workgroup, eight where there is not a group for every compute unit (gradients with
  // four and eight, ms: 55 atoms 3.13 and 3.03, 300 atoms 2.91 and 2.97, 2,000 atoms 9.8 and 10.5)
  const int waves = a.n_grp < cus ? kMaxWaves9 : 4;
  // an item's 64 pairs reach over 63 / c_end + 1 steps
  const int live = a.s_live > 0 ? std::min(a.s_live, a.sp) : a.sp;
  const int64_t far = std::max(std::abs(a.xstride), std::abs(a.ystride));
  SddmmArgs b = a;
  b.spread = a.xstride >= 0 && a.ystride >= 0 &&
             (63 / live + 1) * far + live < (int64_t)(UINT32_MAX / sizeof(double));
  const dim3 grid((unsigned)a.n_grp);
  if (precision == 0) launch_sddmm9_t<double>(b, grid, waves, s);
  else launch_sddmm9_t<float>(b, grid, waves, s);
  return hipGetLastError();
}

}  // namespace rfo
