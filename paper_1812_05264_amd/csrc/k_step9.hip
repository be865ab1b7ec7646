// Chebyshev step for 9x9 blocks in FP64 and FP32 (see k_step.hip for the recurrence, the fused
// moments and the schedule, prod9.h for the block-row product on the matrix cores).  One wave
// takes one block row of a tile of 16 * NT probe columns; TPW waves of a workgroup take
// neighbouring tiles of the same block row, the others the next rows.
//
// What bounds it: on small matrices the chain of dependent loads of one block row (few waves, so
// narrow tiles and the next chunk's gathers in flight during the products: 18.1 -> 6.9 us per step
// with 55 block rows and 64 probes, 25.8 -> 11.0 with 500 and 128, against one wave per block row of
// 64 or 128 columns on the vector units); on large ones the bytes from beyond the L2 (reads come
// at 28 TB/s from an XCD's L2, 7.2 TB/s from beyond it, whatever their shape), which the tile
// width sets together with the rows in flight: FP64, 256 probes, 16,000 block rows 486 -> 468 us,
// 6,000 171 -> 154, 4,000 with 128 probes 69 -> 55.
//
// Padding columns of a tile are read and computed like the others (dense probes: zeros).  Variants that skipped
// their loads held a predicate through the product loop and spilled up to 58 registers there: FP32, 100
// dense probes of 128 columns, 60 terms 1,641 us on 3,000 block rows against 990 without, FP64 1,658 and
// 1,343; nowhere faster (13 to 12,000 block rows, 1 to 288 probes, all modes: 0.57 to 1.01 of their time).
#include "moment_flush.h"
#include "prod9.h"

namespace rfo {

namespace {

// waves per SIMD the registers of a tile allow without spills in the product loop
template <typename VT, int NT>
constexpr int step9_waves() {
  return NT * sizeof(VT) <= 8 ? 4 : NT * sizeof(VT) <= 16 ? 3 : 2;
}

}  // namespace

template <typename VT, int NT, int MODE>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(step9_waves<VT, NT>()))) void k_step9(
    StepArgs a) {
  typedef Prod9<VT, NT, 1, 1> Prod;
  constexpr int PW = Prod::PW, NP = Prod::NP, TW = 16 * NT;
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int grp = lane >> 4, n = lane & 15;
  const int tpw = a.tpw, wt = wave & (tpw - 1), wr = wave / tpw;  // tile and row of the wave
  const int sp = a.sp;
  const int nw = sp >> 6;
  const VT *x = static_cast<const VT *>(a.x);
  const VT *prev = static_cast<const VT *>(a.prev);
  VT *out = static_cast<VT *>(a.out);
  VT *acc = static_cast<VT *>(a.acc);
  const bool has_prev = a.c2 != 0.0;
  const bool add_r = a.beta != nullptr;
  const bool mom_on = a.part != nullptr;
  // MODE 1: density accumulator terms; MODE 2: doubling moments <y,y>, <y,y_k>
  // instead of r.y; MODE 3: vector sources added to the output
  constexpr bool DBL = MODE == 2;
  constexpr bool SRC = MODE == 3;
  const bool need_r = add_r || (mom_on && !DBL);
  const double beta = add_r ? sld(a.beta) : 0.0;
  const int m = MODE == 1 ? a.acc_terms : 0;
  const int nsrc = SRC ? a.nsrc : 0;
  const VT *srcp[3];
  VT srw[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    srcp[t] = t < nsrc ? static_cast<const VT *>(a.src[t]) : nullptr;
    srw[t] = t < nsrc ? (VT)a.srcw[t] : (VT)0;
  }
  VT al[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) al[i] = i < m ? (VT)sld(a.alpha + i) : (VT)0;
  const VT c1 = (VT)a.c1, c2 = (VT)a.c2;
  __shared__ double red[kWaves][4][TW];
  __shared__ __attribute__((aligned(16))) VT hs[kWaves][Prod::LDSN];
  VT *hw = hs[wave];
  double *prow = mom_on ? a.part + (int64_t)blockIdx.x * sp : nullptr;
  double *prow2 = DBL && mom_on ? a.part2 + (int64_t)blockIdx.x * sp : nullptr;

  // moment sums of the lane's rows of the two row groups, and of row 8 (lane group p: access p)
  double mom[NT], mom2[NT], mom8[PW], mom82[PW];
#pragma unroll
  for (int t = 0; t < NT; ++t) mom[t] = mom2[t] = 0.0;
#pragma unroll
  for (int e = 0; e < PW; ++e) mom8[e] = mom82[e] = 0.0;
  int cur_pt = -1;
  // every column's partials start at zero (a workgroup may skip tiles, and the tiles past
  // the last real probe are not run); the tiles it meets are overwritten by flush
  if (mom_on && wave == 0)
    for (int c = lane; c < sp; c += 64) {
      prow[c] = 0.0;
      if (DBL) prow2[c] = 0.0;
    }
  auto flush1 = [&](double(&mm)[NT], double(&m8)[PW], double *dst, int pt) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      red[wave][grp][(t / PW) * (16 * PW) + n * PW + t % PW] = mm[t] + (grp == t / PW ? m8[t % PW] : 0.0);
      mm[t] = 0.0;
    }
#pragma unroll
    for (int e = 0; e < PW; ++e) m8[e] = 0.0;
    __syncthreads();
    // the first row's waves add the rows of their tile in order
    if (wr == 0 && pt * tpw + wt < a.n_pt)
      for (int c = lane; c < TW; c += 64) {
        double s = 0.0;
        for (int w = wt; w < kWaves; w += tpw)
#pragma unroll
          for (int q = 0; q < 4; ++q) s += red[w][q][c];
        dst[(int64_t)(pt * tpw + wt) * TW + c] = s;
      }
    __syncthreads();
  };
  auto flush = [&](int pt) {
    flush1(mom, mom8, prow, pt);
    if (DBL) flush1(mom2, mom82, prow2, pt);
  };

  const VT *const mat[1] = {static_cast<const VT *>(a.hval)};
  const VT *const xs[1] = {x};
  for (Sched sc((a.n_pt + tpw - 1) / tpw, a.n_rg, a.reverse != 0); sc.more(); sc.next()) {
    const int pg = sc.pt();  // group of tpw tiles
    const int64_t rg = sc.rg();
    if (pg != cur_pt) {
      if (mom_on && cur_pt >= 0) flush(cur_pt);
      cur_pt = pg;
    }
    const int pt = pg * tpw + wt;
    if (pt >= a.n_pt) continue;  // no such tile: the wave waits at the next flush
    // first column of each access of this lane
    int cc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) cc[p] = pt * TW + p * (16 * PW) + n * PW;
    const int64_t r0 = rg * a.rows_per_wg;
    const int64_t r1 = min(a.nb, r0 + (int64_t)a.rows_per_wg);
    // PW probes of one scalar row of the output: shift, sources, moments, store, accumulator
    auto finish = [&](int64_t row, int c, const VT(&si)[PW], double *mo, double *mo2) {
      const int64_t off = row * sp + c;
      VecN<VT, PW> pv, xv;
      if (has_prev) pv = ldv_nt<VT, PW>(prev + off);
      VecN<VT, PW> sv[3];
      if (SRC) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
          if (t < nsrc) sv[t] = ldv_nt<VT, PW>(srcp[t] + off);
      }
      if (m >= 2 || DBL) xv = ldv<VT, PW>(x + off);
      double r[PW];
      if (need_r) {
        if (a.sgn) {
          const uint64_t w = a.sgn[row * nw + (c >> 6)];
#pragma unroll
          for (int q = 0; q < PW; ++q) r[q] = ((w >> ((c + q) & 63)) & 1ull) ? 1.0 : -1.0;
        } else {
          const VecN<double, PW> rv = ldv<double, PW>(a.rden + off);
#pragma unroll
          for (int q = 0; q < PW; ++q) r[q] = rv.v[q];
        }
      }
      VecN<VT, PW> o;
#pragma unroll
      for (int q = 0; q < PW; ++q) {
        VT v = c1 * si[q];
        if (has_prev) v = fma(c2, pv.v[q], v);
        if (add_r) v = (VT)((double)v + beta * r[q]);
        if (SRC) {
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t < nsrc) v = fma(srw[t], sv[t].v[q], v);
        }
        o.v[q] = v;
        if (mom_on) {
          if (DBL) {
            mo[q] = fma((double)v, (double)v, mo[q]);
            mo2[q] = fma((double)v, (double)xv.v[q], mo2[q]);
          } else {
            mo[q] = fma(r[q], (double)v, mo[q]);
          }
        }
      }
      stv_nt<VT, PW>(out + off, o);
      if (m > 0) {
        VecN<VT, PW> av = ldv_nt<VT, PW>(acc + off);
        av = add_terms<VT, PW>(av, m, al, pv, xv, o);
        stv_nt<VT, PW>(acc + off, av);
      }
    };
    for (int64_t I = r0 + wr; I < r1; I += kWaves / tpw) {
      const int64_t beg = sld(a.row_ptr + I), end = sld(a.row_ptr + I + 1);
      Prod pr;
      pr.row(mat, a.col, xs, beg, end, sp * (int)sizeof(VT), lane, Prod::lane_bytes(lane, sp, pt), hw);
      VT s8[NT];
#pragma unroll
      for (int c = 0; c < NT; ++c) s8[c] = pr.row8(0, c);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          VT si[PW];
#pragma unroll
          for (int e = 0; e < PW; ++e) si[e] = pr.group_row(0, q, p * PW + e);
          finish(I * 9 + 4 * q + grp, cc[p], si, mom + p * PW, mom2 + p * PW);
        }
      // row 8: lane group p takes access p
      if (grp < NP) {
        VT si[PW];
        int c = cc[0];
#pragma unroll
        for (int e = 0; e < PW; ++e) si[e] = s8[e];
#pragma unroll
        for (int p = 1; p < NP; ++p)
          if (grp == p) {
            c = cc[p];
#pragma unroll
            for (int e = 0; e < PW; ++e) si[e] = s8[p * PW + e];
          }
        finish(I * 9 + 8, c, si, mom8, mom82);
      }
    }
  }
  if (mom_on && cur_pt >= 0) flush(cur_pt);
}

// ---------------------------------------------------------------------------
// FP32 on the vector units, 256 probe columns per wave (four per lane), for probe blocks that fill
// such tiles: there the products on the matrix cores (64 columns per wave) are no faster, since a
// block's nine rows read their operands four probes at a time either way, and read H four times.
// Per chunk of two blocks a wave loads the H_hat blocks with coalesced loads into its LDS slice
// and issues the neighbour-row gathers; the FMAs then read the entries back as LDS broadcasts.
// ---------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(kWG) void k_step9_wide(StepArgs a) {
  typedef float VT;
  constexpr int PPL = 4, U = 2, BD = 9, BB = 81;
  constexpr int CH = U * BB;                       // H_hat values per chunk
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int sp = a.sp;
  const int nw = sp >> 6;
  const VT *__restrict__ x = static_cast<const VT *>(a.x);
  const VT *prev = static_cast<const VT *>(a.prev);
  VT *out = static_cast<VT *>(a.out);
  VT *acc = static_cast<VT *>(a.acc);
  const VT *hval = static_cast<const VT *>(a.hval);
  const bool has_prev = a.c2 != 0.0;
  const bool add_r = a.beta != nullptr;
  const bool mom_on = a.part != nullptr;
  // MODE 1: density accumulator terms; MODE 2: doubling moments <y,y>, <y,y_k>
  // instead of r.y (the MODE 0 variants carry no code for either)
  constexpr bool DBL = MODE == 2;
  const bool need_r = add_r || (mom_on && !DBL);
  const double beta = add_r ? sld(a.beta) : 0.0;
  const int m = MODE == 1 ? a.acc_terms : 0;
  // MODE 3: vector sources added to the output (reverse recurrence with doubling)
  constexpr bool SRC = MODE == 3;
  const int nsrc = SRC ? a.nsrc : 0;
  const VT *srcp[3];
  VT srw[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    srcp[t] = t < nsrc ? static_cast<const VT *>(a.src[t]) : nullptr;
    srw[t] = t < nsrc ? (VT)a.srcw[t] : (VT)0;
  }
  VT al[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) al[i] = i < m ? (VT)sld(a.alpha + i) : (VT)0;
  const VT c1 = (VT)a.c1, c2 = (VT)a.c2;
  __shared__ double red[kWaves][64 * PPL];
  __shared__ VT hs[kWaves][CH];
  VT *hw = hs[wave];
  double *prow = mom_on ? a.part + (int64_t)blockIdx.x * sp : nullptr;

  double mom[PPL], mom2[PPL];
#pragma unroll
  for (int q = 0; q < PPL; ++q) mom[q] = mom2[q] = 0.0;
  int cur_pt = -1;
  double *prow2 = DBL && mom_on ? a.part2 + (int64_t)blockIdx.x * sp : nullptr;
  if (mom_on) zero_partials<PPL>(prow, a.n_pt, wave, lane);
  if (DBL && mom_on) zero_partials<PPL>(prow2, a.n_pt, wave, lane);

  for (Sched sc(a.n_pt, a.n_rg, a.reverse != 0); sc.more(); sc.next()) {
    const int pt = sc.pt();
    const int64_t rg = sc.rg();
    if (pt != cur_pt) {
      if (mom_on && cur_pt >= 0) {
        flush_tile<PPL>(mom, red, wave, lane, prow, cur_pt);
        if (DBL) flush_tile<PPL>(mom2, red, wave, lane, prow2, cur_pt);
      }
      cur_pt = pt;
    }
    const int c0 = pt * (64 * PPL) + lane * PPL;
    const int64_t r0 = rg * a.rows_per_wg;
    const int64_t r1 = min(a.nb, r0 + (int64_t)a.rows_per_wg);
    // one scalar row of the output: shift, sources, moments, store, accumulator
    auto finish_row = [&](int64_t I, int i, const VT(&si)[PPL]) {
        const int64_t row = I * BD + i;
        const int64_t off = row * sp + c0;
        VecN<VT, PPL> pv, xs;
        if (has_prev) pv = ldv_nt<VT, PPL>(prev + off);
        VecN<VT, PPL> sv[3];
        if (SRC) {
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t < nsrc) sv[t] = ldv_nt<VT, PPL>(srcp[t] + off);
        }
        if (m >= 2 || DBL) xs = ldv<VT, PPL>(x + off);
        double r[PPL];
        if (need_r) {
          if (a.sgn) {
            const uint64_t w = a.sgn[row * nw + (c0 >> 6)];
#pragma unroll
            for (int q = 0; q < PPL; ++q) r[q] = ((w >> ((c0 + q) & 63)) & 1ull) ? 1.0 : -1.0;
          } else {
            const VecN<double, PPL> rv = ldv<double, PPL>(a.rden + off);
#pragma unroll
            for (int q = 0; q < PPL; ++q) r[q] = rv.v[q];
          }
        }
        VecN<VT, PPL> o;
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
          VT v = c1 * si[q];
          if (has_prev) v = fma(c2, pv.v[q], v);
          if (add_r) v = (VT)((double)v + beta * r[q]);
          if (SRC) {
#pragma unroll
            for (int t = 0; t < 3; ++t)
              if (t < nsrc) v = fma(srw[t], sv[t].v[q], v);
          }
          o.v[q] = v;
          if (mom_on) {
            if (DBL) {
              mom[q] = fma((double)v, (double)v, mom[q]);
              mom2[q] = fma((double)v, (double)xs.v[q], mom2[q]);
            } else {
              mom[q] = fma(r[q], (double)v, mom[q]);
            }
          }
        }
        stv_nt<VT, PPL>(out + off, o);
        if (m > 0) {
          VecN<VT, PPL> av = ldv_nt<VT, PPL>(acc + off);
          av = add_terms<VT, PPL>(av, m, al, pv, xs, o);
          stv_nt<VT, PPL>(acc + off, av);
        }
    };
    for (int64_t I = r0 + wave; I < r1; I += kWaves) {
      const int64_t beg = sld(a.row_ptr + I), end = sld(a.row_ptr + I + 1);
      VT s[BD][PPL];
#pragma unroll
      for (int i = 0; i < BD; ++i)
#pragma unroll
        for (int q = 0; q < PPL; ++q) s[i][q] = (VT)0;
      constexpr int NH = (CH + 63) / 64;
      // H_hat chunk -> registers (coalesced) and the neighbour gathers
      auto load_chunk = [&](int64_t nz, VT(&hv)[NH], VecN<VT, PPL>(&xv)[U][BD]) {
        const VT *hsrc = hval + nz * BB;
#pragma unroll
        for (int k = 0; k < NH; ++k) {
          const int e = k * 64 + lane;
          if (e < CH) hv[k] = hsrc[e];
        }
        int64_t J[U];
#pragma unroll
        for (int u = 0; u < U; ++u) J[u] = sld(a.col + nz + u);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // a chunk slot past the row's end gathers nothing (its FMAs are skipped)
          if (u == 0 || nz + u < end) {
#pragma unroll
            for (int j = 0; j < BD; ++j)
              xv[u][j] = ldv<VT, PPL>(x + (J[u] * BD + j) * sp + c0);
          }
        }
      };
      // H_hat chunk -> LDS, then the FMAs with LDS broadcasts
      auto use_chunk = [&](int64_t nz, const VT(&hv)[NH], const VecN<VT, PPL>(&xv)[U][BD]) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < NH; ++k) {
          const int e = k * 64 + lane;
          if (e < CH) hw[e] = hv[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (nz + u < end) {
#pragma unroll
            for (int i = 0; i < BD; ++i)
#pragma unroll
              for (int j = 0; j < BD; ++j) {
                const VT h = (VT)hw[u * BB + i * BD + j];
#pragma unroll
                for (int q = 0; q < PPL; ++q) s[i][q] = fma(h, xv[u][j].v[q], s[i][q]);
              }
          }
        }
      };
      for (int64_t nz = beg; nz < end; nz += U) {
        VT hv[NH];
        VecN<VT, PPL> xv[U][BD];
        load_chunk(nz, hv, xv);
        use_chunk(nz, hv, xv);
      }
#pragma unroll
      for (int i = 0; i < BD; ++i) finish_row(I, i, s[i]);
    }
  }
  if (mom_on && cur_pt >= 0) {
    flush_tile<PPL>(mom, red, wave, lane, prow, cur_pt);
    if (DBL) flush_tile<PPL>(mom2, red, wave, lane, prow2, cur_pt);
  }
}

namespace {

template <typename VT, int NT>
const void *step9_fn(int mode) {
  switch (mode) {
    case 0: return (const void *)k_step9<VT, NT, 0>;
    case 1: return (const void *)k_step9<VT, NT, 1>;
    case 2: return (const void *)k_step9<VT, NT, 2>;
    case 3: return (const void *)k_step9<VT, NT, 3>;
    default: return nullptr;
  }
}

template <typename VT>
const void *step9_fn_t(int nt, int mode) {
  switch (nt) {
    case 1: return step9_fn<VT, 1>(mode);
    case 2: return step9_fn<VT, 2>(mode);
    case 4: return step9_fn<VT, 4>(mode);
    default: return nullptr;
  }
}

const void *step9_wide_fn(int mode) {
  switch (mode) {
    case 0: return (const void *)k_step9_wide<0>;
    case 1: return (const void *)k_step9_wide<1>;
    case 2: return (const void *)k_step9_wide<2>;
    case 3: return (const void *)k_step9_wide<3>;
    default: return nullptr;
  }
}

// nt = 16 FP32: k_step9_wide
const void *select_step9(int precision, int nt, int mode) {
  if (precision == 1 && nt == 16) return step9_wide_fn(mode);
  return precision == 0 ? step9_fn_t<double>(nt, mode) : step9_fn_t<float>(nt, mode);
}

}  // namespace

int step9_blocks_per_cu(int precision, int nt) {
  const void *f = select_step9(precision, nt, 0);
  if (!f) return 0;
  int nblk = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nblk, f, kWG, 0) != hipSuccess) return 0;
  return nblk;
}

hipError_t launch_step9(int precision, int nt, const StepArgs &a, hipStream_t s) {
  const void *f = select_step9(precision, nt, step_mode(a));
  if (!f || a.grid < 8 || (a.grid & 7) || a.n_pt * 16 * nt > a.sp || (a.tpw != 1 && a.tpw != 2))
    return hipErrorInvalidValue;
  void *args[] = {const_cast<StepArgs *>(&a)};
  return hipLaunchKernel(f, dim3((unsigned)a.grid), dim3(kWG), args, 0, s);
}

}  // namespace rfo
