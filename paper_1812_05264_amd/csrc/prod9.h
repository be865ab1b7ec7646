// Block-row product of the 9x9 kernels on the matrix cores: Y_I = sum_J M_IJ X_J for one
// block row I and a tile of 16 * NT probe columns per wave, in FP64 (v_mfma_f64_4x4x4) or
// FP32 (v_mfma_f32_4x4x1), with PL planes of X sharing one matrix (2: complex vectors) and
// NM matrices on the same pattern sharing the gathers (2: H_hat and S).
//
// The nine rows of a block are 4 + 4 + 1: two row groups on the matrix cores, which so
// multiply no padding, and the ninth row on the vector units beside them.  Blocks are taken
// four at a time, their 36 columns (the rows of the X_J) as nine K steps of four: step 2u + h
// holds columns 4h .. 4h+3 of block u, step 8 column 8 of the four blocks, so that the row
// addresses of a step are one scalar base and one lane offset.  Lane l holds K slice k = l >> 4
// and probe column n = l & 15 of the tile:
//   FP64: A = M[4g + l%4][K row of slice k], B = X[K row][n]; the instruction's four 4x4 blocks
//         are four column groups of the same rows (A repeated), and it adds the four K slices,
//         so D of lane l is row 4g + (l >> 4), column n.
//   FP32: the instruction has K = 1 and sixteen 4x4 blocks; with CBSZ = 2 the four blocks of a
//         K slice (16 lanes) take one block's A (ABID), so lane l accumulates rows 4g .. 4g+3 of
//         column n over its own K slice, and the slices are added once per row (group_row);
//         one A register holds four K steps.
// The matrix entries of a chunk go through the wave's LDS slice: a lane needs 3 of them per
// K step and NT columns, where a product on the vector units broadcasts all 81 of a block to
// every lane.  A load instruction covers 16 * PW columns of four rows, so a tile may be
// narrow (few rows held in an XCD's L2, many waves for a small matrix) without narrower loads.
#pragma once

#include <type_traits>

#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

typedef float f4v __attribute__((ext_vector_type(4)));

template <typename VT>
struct Acc9;
template <>
struct Acc9<double> {
  double v;
};
template <>
struct Acc9<float> {
  f4v v;
};

constexpr int kB9 = 4;                   // blocks per chunk
constexpr int kB9Steps = 9;              // K steps of four K rows per chunk
constexpr int kB9Vals = kB9 * 81;        // matrix entries per chunk

// two 8-byte or four 4-byte matrix entries at the entries' own alignment
template <typename VT>
struct MatVec {
  static constexpr int N = 16 / sizeof(VT);
  struct __attribute__((packed, aligned(sizeof(VT)))) T {
    VT v[N];
  };
};

template <typename VT, int NT, int PL, int NM>
struct Prod9 {
  static constexpr int PW = NT * sizeof(VT) < 16 ? NT : (int)(16 / sizeof(VT));  // probes per access
  static constexpr int NP = NT / PW;                                             // accesses per row
  static constexpr int NC = NT * PL;
  static constexpr int NH = (kB9Vals + 64 * MatVec<VT>::N - 1) / (64 * MatVec<VT>::N);
  // LDS entries of one matrix' chunk (whole store rounds)
  static constexpr int LDSN = NH * 64 * MatVec<VT>::N;

  typedef const __attribute__((address_space(1))) char *GlobalBytes;

  // matrix entries of one chunk on their way
  struct Entries {
    typename MatVec<VT>::T v[NM][NH];
  };
  // gathered rows of one chunk
  struct Rows {
    VecN<VT, PW> x[kB9Steps][PL * NP];
  };

  Acc9<VT> g[NM][2][NC];
  VT r8[NM][NC];

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        r8[m][c] = (VT)0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if constexpr (sizeof(VT) == 8) g[m][q][c].v = 0.0;
          else g[m][q][c].v = f4v{0.f, 0.f, 0.f, 0.f};
        }
      }
  }

  // byte offset of this lane's first column in K slice 0 .. 3 of a row set
  static __device__ __forceinline__ uint32_t lane_bytes(int lane, int sp, int pt) {
    return (uint32_t)(((lane >> 4) * sp + pt * (16 * NT) + (lane & 15) * PW) * (int)sizeof(VT));
  }

  // block columns from chunk nz on (the array carries kStepPad entries past the last block)
  static __device__ __forceinline__ void columns(int32_t (&J)[kB9], const int32_t *col, int64_t nz) {
#pragma unroll
    for (int u = 0; u < kB9; ++u) J[u] = sld(col + nz + u);
  }

  // requests the matrix entries of chunk nz (the arrays carry kStepPad zero blocks past the last)
  static __device__ __forceinline__ void load_entries(Entries &h, const VT *const (&mat)[NM], int64_t nz,
                                                      int lane) {
    constexpr int MN = MatVec<VT>::N;
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int k = 0; k < NH; ++k)
        h.v[m][k] =
            *reinterpret_cast<const typename MatVec<VT>::T *>(mat[m] + nz * 81 + (k * 64 + lane) * MN);
  }

  // where the rows of a chunk are: one scalar address per plane and block, and a lane's address of
  // step 8
  struct Bases {
    GlobalBytes base[PL][kB9];
    GlobalBytes last[PL];
  };

  // the addresses of a chunk of rem blocks with columns J; rowb: bytes of a row, vb = lane_bytes.
  // The scalar ones are opaque, or the compiler adds the lane offset first and keeps 64-bit
  // addresses per lane
  static __device__ __forceinline__ void locate(Bases &bs, const int32_t (&J)[kB9], const VT *const (&x)[PL],
                                                int rem, int rowb, int lane, uint32_t vb) {
    const int ks = lane >> 4;
    int32_t Ju[kB9], Jl = J[0];  // Jl: block of this K slice in step 8
#pragma unroll
    for (int u = 0; u < kB9; ++u) Ju[u] = uniform(u < rem ? J[u] : J[0]);
#pragma unroll
    for (int u = 1; u < kB9; ++u) Jl = ks == u ? Ju[u] : Jl;
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
      const GlobalBytes x0 = (GlobalBytes)(reinterpret_cast<const char *>(x[pl]));
#pragma unroll
      for (int u = 0; u < kB9; ++u) {
        bs.base[pl][u] = x0 + (int64_t)Ju[u] * (int64_t)(9 * rowb);
        asm volatile("" : "+s"(bs.base[pl][u]));
      }
      // row 8 of block ks; vb holds ks rows too many for it
      bs.last[pl] = x0 + ((int64_t)Jl * 9 + 8 - ks) * (int64_t)rowb + vb;
    }
  }

  // requests the rows of K step T
  template <int T>
  static __device__ __forceinline__ void load_step(Rows &ch, const Bases &bs, int rowb, uint32_t vb) {
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
      GlobalBytes src;
      if constexpr (T == 8) src = bs.last[pl];
      else src = bs.base[pl][T / 2] + (T % 2 ? vb + 4u * (uint32_t)rowb : vb);
#pragma unroll
      for (int p = 0; p < NP; ++p) ch.x[T][pl * NP + p] = gather(src, p);
    }
  }

  // access p of a gathered row
  static __device__ __forceinline__ VecN<VT, PW> gather(GlobalBytes src, int p) {
    typedef VT V __attribute__((ext_vector_type(PW)));
    const V v = *reinterpret_cast<const __attribute__((address_space(1))) V *>(src + p * (16 * PW * (int)sizeof(VT)));
    VecN<VT, PW> r;
#pragma unroll
    for (int q = 0; q < PW; ++q) r.v[q] = v[q];
    return r;
  }

  template <typename F>
  static __device__ __forceinline__ void for_steps(F &&f) {
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{});
    f(std::integral_constant<int, 5>{});
    f(std::integral_constant<int, 6>{});
    f(std::integral_constant<int, 7>{});
    f(std::integral_constant<int, 8>{});
  }

  // the entries -> the wave's LDS slice hw[NM][LDSN], those past the row's last block as zeros
  static __device__ __forceinline__ void store_entries(const Entries &h, VT *hw, int rem, int lane) {
    constexpr int MN = MatVec<VT>::N;
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int k = 0; k < NH; ++k) {
        const int e = (k * 64 + lane) * MN;
        VecN<VT, MN> v;
#pragma unroll
        for (int q = 0; q < MN; ++q) v.v[q] = (rem >= kB9 || e + q < 81 * rem) ? h.v[m][k].v[q] : (VT)0;
        stv<VT, MN>(hw + m * LDSN + e, v);
      }
  }

  // adds the chunk's products; after(step) runs when the rows of a step are used up
  template <typename F>
  __device__ __forceinline__ void use(Rows &ch, const VT *hw, int lane, F &&after) {
    const int ks = lane >> 4, r = lane & 3;
    if constexpr (sizeof(VT) == 8) {
      // entry M[row][c] of block u sits at u * 81 + row * 9 + c.  The entries of step t + 1 are
      // read before the products of step t, and no further ahead (barriers for the compiler's
      // scheduler): all nine at once would take 54 registers
      double a0[2][NM], a1[2][NM], a8[2][NM];
      const VT *h0 = hw + 9 * r + ks, *h8 = hw + 9 * r + 81 * ks + 8;
      const VT *g0 = hw + 72 + ks, *g8 = hw + 80 + 81 * ks;
      auto entries = [&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int s = t & 1, o = t < 8 ? (t / 2) * 81 + (t % 2) * 4 : 0;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const VT *h = (t < 8 ? h0 : h8) + m * LDSN + o;
          a0[s][m] = h[0];
          a1[s][m] = h[36];
          a8[s][m] = ((t < 8 ? g0 : g8) + m * LDSN)[o];
        }
      };
      entries(std::integral_constant<int, 0>{});
      for_steps([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int s = t & 1;
        if constexpr (t + 1 < kB9Steps) entries(std::integral_constant<int, t + 1>{});
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const double b = ch.x[t][(c / NT) * NP + (c % NT) / PW].v[c % PW];
            g[m][0][c].v = __builtin_amdgcn_mfma_f64_4x4x4f64(a0[s][m], b, g[m][0][c].v, 0, 0, 0);
            g[m][1][c].v = __builtin_amdgcn_mfma_f64_4x4x4f64(a1[s][m], b, g[m][1][c].v, 0, 0, 0);
            r8[m][c] = fma(a8[s][m], b, r8[m][c]);
          }
        __builtin_amdgcn_sched_barrier(0);
        after(tc);
      });
    } else {
      // one A register per row group and four K steps: lane (K slice ks, step j = (lane >> 2) & 3,
      // row r) holds its entry of step 4T + j; T = 2 has step 8 alone
      float a0[NM][3], a1[NM][3], a8[NM][3];
      const int j = (lane >> 2) & 3;
      const int oj = (j >> 1) * 81 + (j & 1) * 4 + ks, o8 = 81 * ks + 8;
#pragma unroll
      for (int T = 0; T < 3; ++T) {
        const int o = T < 2 ? oj + T * 162 : o8;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const VT *h = hw + m * LDSN + o;
          a0[m][T] = h[9 * r];
          a1[m][T] = h[9 * r + 36];
          a8[m][T] = h[72];
        }
      }
      for_steps([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int T = t / 4, ab = t % 4;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          // row 8: the entry of this K step, from lane 4 * ab of every 16
          const float h8 = __builtin_bit_cast(
              float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a8[m][T]), 0x150 + 4 * ab, 0xf,
                                                 0xf, true));
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const float b = ch.x[t][(c / NT) * NP + (c % NT) / PW].v[c % PW];
            g[m][0][c].v = __builtin_amdgcn_mfma_f32_4x4x1f32(a0[m][T], b, g[m][0][c].v, 2, ab, 0);
            g[m][1][c].v = __builtin_amdgcn_mfma_f32_4x4x1f32(a1[m][T], b, g[m][1][c].v, 2, ab, 0);
            r8[m][c] = fmaf(h8, b, r8[m][c]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        after(tc);
      });
    }
  }

  // rows of group q for column c: row 4q + (lane >> 4) in every lane
  __device__ __forceinline__ VT group_row(int m, int q, int c) const {
    if constexpr (sizeof(VT) == 8) {
      return g[m][q][c].v;
    } else {
      // the four K slices (16-lane groups) of rows 0..3: after the two exchanges lane group i
      // holds the sum of row i
      const f4v d = g[m][q][c].v;
      const float s02 = swap_add<32>(d[0], d[2]), s13 = swap_add<32>(d[1], d[3]);
      return swap_add<16>(s02, s13);
    }
  }
  // row 8 of column c in every lane
  __device__ __forceinline__ VT row8(int m, int c) const {
    VT v = r8[m][c];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
  }

  // lanes whose group bit W is clear: a's sum over the pair of groups; the others: b's
  template <int W>
  static __device__ __forceinline__ float swap_add(float a, float b) {
    unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    if constexpr (W == 32) {
      const auto r = __builtin_amdgcn_permlane32_swap(ua, ub, false, false);
      ua = r[0];
      ub = r[1];
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
      ua = r[0];
      ub = r[1];
    }
    return __builtin_bit_cast(float, ua) + __builtin_bit_cast(float, ub);
  }

  // The whole block row [beg, end) by one wave, hw its LDS slice [NM][LDSN].  The rows of the
  // next chunk are requested step by step as the registers of this one's are used up, so that a
  // wave's gathers stay in flight during its products without a second set of registers.  A last
  // chunk of fewer than four blocks gathers its first block's rows again (lines already on their
  // way) and multiplies them by zeros: one path without branches.
  __device__ __forceinline__ void row(const VT *const (&mat)[NM], const int32_t *col, const VT *const (&x)[PL],
                                      int64_t beg, int64_t end, int rowb, int lane, uint32_t vb, VT *hw) {
    clear();
    if (beg >= end) return;
    int32_t J[kB9];
    Entries h;
    Rows ch;
    Bases bs;
    auto blocks = [&](int64_t nz) { return (int)min(end - nz, (int64_t)kB9); };
    auto put = [&](int64_t nz) {
      __builtin_amdgcn_wave_barrier();
      store_entries(h, hw, blocks(nz), lane);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    load_entries(h, mat, beg, lane);
    columns(J, col, beg);
    locate(bs, J, x, blocks(beg), rowb, lane, vb);
    for_steps([&](auto tc) { load_step<decltype(tc)::value>(ch, bs, rowb, vb); });
    int64_t nz = beg;
    columns(J, col, nz + kB9 < end ? nz + kB9 : nz);
    for (; nz + kB9 < end; nz += kB9) {
      put(nz);
      load_entries(h, mat, nz + kB9, lane);
      locate(bs, J, x, blocks(nz + kB9), rowb, lane, vb);
      columns(J, col, nz + 2 * kB9 < end ? nz + 2 * kB9 : nz);
      __builtin_amdgcn_sched_barrier(0);
      use(ch, hw, lane, [&](auto tc) { load_step<decltype(tc)::value>(ch, bs, rowb, vb); });
    }
    put(nz);
    use(ch, hw, lane, [](auto) {});
  }
};

}  // namespace rfo
