// Complex block product of the rational expansion for 9x9 blocks (see k_cgls.hip):
// out = (H_hat - z) x, or H_hat x - z (S x) with an overlap, on two real planes, with the column
// partials of |out_c|^2.  One wave takes one block row of 16 * NT probe columns in both planes, which
// share the matrix entries (prod9.h); TPW waves of a workgroup take neighbouring tiles of a block row.
//
// These matrices are small (a solve needs ten real vectors), so the bound is the chain of dependent
// loads of a block row and the waves in flight.  A wave with 64 or 128 columns on the vector units,
// one block's 81 entries broadcast from LDS at a time, left 250 block rows with 128 probes on 250
// waves: 32 us per product; here 1,000 waves of 32 columns.  Rational density of 24 poles, 250 atoms, 128
// probes: 423 -> 223 ms; 13 atoms, 16 poles: 171 -> 98.
#include "prod9.h"

namespace rfo {

template <int NT, bool HS>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(NT == 1 && !HS ? 4 : NT == 1 ? 3 : 2))) void k_cspmm9(
    CspArgs a) {
  constexpr int NM = HS ? 2 : 1;
  typedef Prod9<double, NT, 2, NM> Prod;
  constexpr int PW = Prod::PW, TW = 16 * NT;
  static_assert(Prod::NP == 1, "one access per row");
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int grp = lane >> 4, n = lane & 15;
  const int tpw = a.tpw, wt = wave & (tpw - 1), wr = wave / tpw;  // tile and row of the wave
  const int sp = a.sp;
  const bool nrm_on = a.part != nullptr;
  __shared__ double red[kWaves][4][TW];
  __shared__ __attribute__((aligned(16))) double hs[kWaves][NM * Prod::LDSN];
  double *hw = hs[wave];
  double *prow = nrm_on ? a.part + (int64_t)blockIdx.x * sp : nullptr;
  // a workgroup may skip tiles; those it meets are overwritten by flush
  if (nrm_on)
    for (int c = threadIdx.x; c < sp; c += kWG) prow[c] = 0.0;
  double nrm[PW];
#pragma unroll
  for (int e = 0; e < PW; ++e) nrm[e] = 0.0;
  auto flush = [&](int pg) {
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      red[wave][grp][n * PW + e] = nrm[e];
      nrm[e] = 0.0;
    }
    __syncthreads();
    // the first row's waves add the rows of their tile in order
    if (wr == 0 && lane < TW) {
      double s = 0.0;
      for (int w = wt; w < kWaves; w += tpw)
#pragma unroll
        for (int q = 0; q < 4; ++q) s += red[w][q][lane];
      prow[(int64_t)(pg * tpw + wt) * TW + lane] = s;
    }
    __syncthreads();
  };
  const double *mat[NM];
  mat[0] = a.hval;
  if constexpr (HS) mat[1] = a.sval;
  const double *const xs[2] = {a.x, a.x + a.plane};
  int cur = -1;
  for (Sched sc(a.n_pt / tpw, a.n_rg); sc.more(); sc.next()) {
    const int pg = sc.pt();
    const int64_t rg = sc.rg();
    if (pg != cur) {
      if (nrm_on && cur >= 0) flush(cur);
      cur = pg;
    }
    const int pt = pg * tpw + wt, c = pt * TW + n * PW;
    const int64_t r0 = rg * a.rows_per_wg;
    const int64_t r1 = min(a.nb, r0 + (int64_t)a.rows_per_wg);
    for (int64_t I = r0 + wr; I < r1; I += kWaves / tpw) {
      const int64_t beg = sld(a.row_ptr + I), end = sld(a.row_ptr + I + 1);
      Prod pr;
      pr.row(mat, a.col, xs, beg, end, sp * 8, lane, Prod::lane_bytes(lane, sp, pt), hw);
      // one scalar row: si = H_hat x of both planes, m = x or S x
      auto finish = [&](int64_t row, const double(&si)[2][PW], const double(&mi)[2][PW]) {
        const int64_t off = row * sp + c;
        VecN<double, PW> mr, mm, o_r, o_i;
        if constexpr (HS) {
#pragma unroll
          for (int e = 0; e < PW; ++e) {
            mr.v[e] = mi[0][e];
            mm.v[e] = mi[1][e];
          }
        } else {
          mr = ldv<double, PW>(xs[0] + off);
          mm = ldv<double, PW>(xs[1] + off);
        }
#pragma unroll
        for (int e = 0; e < PW; ++e) {
          // (h - z m) x with m x = (ar, ai):  re = h xr - zr ar + zi ai,  im = h xi - zr ai - zi ar
          const double vr = fma(a.zi, mm.v[e], fma(-a.zr, mr.v[e], si[0][e]));
          const double vi = fma(-a.zi, mr.v[e], fma(-a.zr, mm.v[e], si[1][e]));
          o_r.v[e] = vr;
          o_i.v[e] = vi;
          nrm[e] = fma(vi, vi, fma(vr, vr, nrm[e]));
        }
        stv<double, PW>(a.out + off, o_r);
        stv<double, PW>(a.out + a.plane + off, o_i);
      };
      double s8[2][PW], m8[2][PW];
#pragma unroll
      for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int e = 0; e < PW; ++e) {
          s8[pl][e] = pr.row8(0, pl * NT + e);
          m8[pl][e] = HS ? pr.row8(NM - 1, pl * NT + e) : 0.0;
        }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        double si[2][PW], mi[2][PW];
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
#pragma unroll
          for (int e = 0; e < PW; ++e) {
            si[pl][e] = pr.group_row(0, q, pl * NT + e);
            mi[pl][e] = HS ? pr.group_row(NM - 1, q, pl * NT + e) : 0.0;
          }
        finish(I * 9 + 4 * q + grp, si, mi);
      }
      if (grp == 0) finish(I * 9 + 8, s8, m8);
    }
  }
  if (nrm_on && cur >= 0) flush(cur);
}

namespace {

const void *select_cspmm9(int nt, bool hs) {
  if (nt == 1) return hs ? (const void *)k_cspmm9<1, true> : (const void *)k_cspmm9<1, false>;
  if (nt == 2) return hs ? (const void *)k_cspmm9<2, true> : (const void *)k_cspmm9<2, false>;
  return nullptr;
}

}  // namespace

int cspmm9_blocks_per_cu(int nt, bool hs) {
  const void *f = select_cspmm9(nt, hs);
  if (!f) return 0;
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kWG, 0) != hipSuccess) return 0;
  return nb;
}

hipError_t launch_cspmm9(int nt, const CspArgs &a, hipStream_t s) {
  const void *f = select_cspmm9(nt, a.sval != nullptr);
  if (!f || a.sp % 64 != 0 || a.n_pt * 16 * nt != a.sp || (a.tpw != 1 && a.tpw != 2) || a.grid % 8 != 0 ||
      a.grid <= 0)
    return hipErrorInvalidValue;
  CspArgs args = a;
  void *kargs[] = {&args};
  return hipLaunchKernel(f, dim3(a.grid), dim3(kWG), kargs, 0, s);
}

}  // namespace rfo
