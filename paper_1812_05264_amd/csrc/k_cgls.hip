// Rational expansion (paper: Rational approximation, Eq. rational_PQ with S = I):
// the shifted systems (H_hat - z) x = y for every probe column, solved by CGLS
// (conjugate gradients on the normal equations, the solver the paper applies to
// the indefinite complex-shifted matrices), and the per-pole accumulations.
//
// Complex block vectors are two real planes, re then im, each [n][sp] like the
// Chebyshev vectors, so the real H_hat multiplies both planes with the same
// gathers and block values.  Column sums (norms, inner products with the
// probes) are written as per-workgroup partials and reduced in a fixed order
// (launch_colreduce, or the vector kernel that uses them: colsum.h), so every scalar
// is bitwise reproducible.
#include "colsum.h"
#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

namespace {

template <int PPL>
__device__ __forceinline__ void flush_norm(double (&nrm)[PPL], double (*red)[64 * PPL], int wave,
                                           int lane, double *prow, int pt) {
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    red[wave][lane * PPL + q] = nrm[q];
    nrm[q] = 0.0;
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      double t = red[0][lane * PPL + q];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) t += red[w][lane * PPL + q];
      prow[pt * (64 * PPL) + lane * PPL + q] = t;
    }
  }
  __syncthreads();
}

}  // namespace

// out = (H_hat - z) x on complex planes, with the column partials of |out_c|^2;
// HS: out = H_hat x - z (S x) with the overlap S on the same pattern (H_hat then
// maps H with S).  Same persistent XCD-banded schedule as the Chebyshev step
// (Sched), for 1x1 blocks (9x9: k_cspmm9.hip): U neighbours per chunk, entries through the
// scalar cache.
template <int PPL, int U, bool HS>
__global__ __launch_bounds__(kWG) void k_cspmm(CspArgs a) {
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int sp = a.sp;
  const double *__restrict__ xr = a.x;
  const double *__restrict__ xi = a.x + a.plane;
  double *orr = a.out;
  double *oi = a.out + a.plane;
  const double zr = a.zr, zi = a.zi;
  const bool nrm_on = a.part != nullptr;
  __shared__ double red[kWaves][64 * PPL];
  double *prow = nrm_on ? a.part + (int64_t)blockIdx.x * sp : nullptr;
  if (nrm_on && wave == 0)
    for (int t = 0; t < a.n_pt; ++t)
#pragma unroll
      for (int q = 0; q < PPL; ++q) prow[t * (64 * PPL) + lane * PPL + q] = 0.0;
  double nrm[PPL];
#pragma unroll
  for (int q = 0; q < PPL; ++q) nrm[q] = 0.0;
  int cur_pt = -1;

  for (Sched sc(a.n_pt, a.n_rg); sc.more(); sc.next()) {
    const int pt = sc.pt();
    const int64_t rg = sc.rg();
    if (pt != cur_pt) {
      if (nrm_on && cur_pt >= 0) flush_norm<PPL>(nrm, red, wave, lane, prow, cur_pt);
      cur_pt = pt;
    }
    const int c0 = pt * (64 * PPL) + lane * PPL;
    const int64_t r0 = rg * a.rows_per_wg;
    const int64_t r1 = min(a.nb, r0 + (int64_t)a.rows_per_wg);
    for (int64_t I = r0 + wave; I < r1; I += kWaves) {
      const int64_t beg = sld(a.row_ptr + I), end = sld(a.row_ptr + I + 1);
      double sr[PPL], si[PPL];                      // H_hat x
      double tr[HS ? PPL : 1], ti[HS ? PPL : 1];    // S x
#pragma unroll
      for (int q = 0; q < PPL; ++q) sr[q] = si[q] = 0.0;
#pragma unroll
      for (int q = 0; q < (HS ? PPL : 1); ++q) tr[q] = ti[q] = 0.0;
      for (int64_t nz0 = beg; nz0 < end; nz0 += U) {
        int64_t J[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // slots past the row's end re-read the row itself with weight zero
          const int64_t Jc = sld(a.col + nz0 + u);
          J[u] = nz0 + u < end ? Jc : I;
        }
        VecN<double, PPL> vr[U], vi[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          vr[u] = ldv<double, PPL>(xr + J[u] * sp + c0);
          vi[u] = ldv<double, PPL>(xi + J[u] * sp + c0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const double h = nz0 + u < end ? sld(a.hval + nz0 + u) : 0.0;
#pragma unroll
          for (int q = 0; q < PPL; ++q) {
            sr[q] = fma(h, vr[u].v[q], sr[q]);
            si[q] = fma(h, vi[u].v[q], si[q]);
          }
          if constexpr (HS) {
            const double sv = nz0 + u < end ? sld(a.sval + nz0 + u) : 0.0;
#pragma unroll
            for (int q = 0; q < PPL; ++q) {
              tr[q] = fma(sv, vr[u].v[q], tr[q]);
              ti[q] = fma(sv, vi[u].v[q], ti[q]);
            }
          }
        }
      }
      const int64_t off = I * sp + c0;
      VecN<double, PPL> ar, ai;
      if constexpr (HS) {
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
          ar.v[q] = tr[q];
          ai.v[q] = ti[q];
        }
      } else {
        ar = ldv<double, PPL>(xr + off);
        ai = ldv<double, PPL>(xi + off);
      }
      VecN<double, PPL> o_r, o_i;
#pragma unroll
      for (int q = 0; q < PPL; ++q) {
        // (h - z m) x with m x = (ar, ai) = x (S = I) or S x:
        //   re = h xr - zr ar + zi ai,  im = h xi - zr ai - zi ar
        const double vr = fma(zi, ai.v[q], fma(-zr, ar.v[q], sr[q]));
        const double vi = fma(-zi, ar.v[q], fma(-zr, ai.v[q], si[q]));
        o_r.v[q] = vr;
        o_i.v[q] = vi;
        if (nrm_on) nrm[q] = fma(vi, vi, fma(vr, vr, nrm[q]));
      }
      stv<double, PPL>(orr + off, o_r);
      stv<double, PPL>(oi + off, o_i);
    }
  }
  if (nrm_on && cur_pt >= 0) flush_norm<PPL>(nrm, red, wave, lane, prow, cur_pt);
}

namespace {

template <bool HS>
const void *select_cspmm_t(int ppl, int u) {
  if (u == 8) return ppl == 2 ? (const void *)k_cspmm<2, 8, HS> : (const void *)k_cspmm<1, 8, HS>;
  return ppl == 2 ? (const void *)k_cspmm<2, 4, HS> : (const void *)k_cspmm<1, 4, HS>;
}

// u: neighbours per chunk (4 or 8); hs: with S
const void *select_cspmm(int ppl, int u, bool hs) {
  return hs ? select_cspmm_t<true>(ppl, u) : select_cspmm_t<false>(ppl, u);
}

// rows [lo, hi) of workgroup b when n rows are split over gridDim.x workgroups
__device__ __forceinline__ void row_range(int64_t n, int64_t &lo, int64_t &hi) {
  const int64_t G = gridDim.x, b = blockIdx.x;
  lo = n * b / G;
  hi = n * (b + 1) / G;
}

// Thread layout of the row-range kernels: with sp < kWG (and kWG a multiple of
// sp) the kWG / sp row lanes of a column take every (kWG / sp)-th row and their
// sums are combined in lane order (ColLanes::finish); otherwise one thread per
// column (a loop over columns when sp > kWG).
struct ColLanes {
  int nl, lr, c0, cstep;
  __device__ ColLanes(int sp) {
    nl = (sp < kWG && kWG % sp == 0) ? kWG / sp : 1;
    lr = nl > 1 ? (int)threadIdx.x / sp : 0;
    c0 = nl > 1 ? (int)threadIdx.x % sp : (int)threadIdx.x;
    cstep = nl > 1 ? sp : kWG;
  }
  // stores the column sum v of column c into out[c] (row lane 0 after combining)
  __device__ void finish(double v, int c, int sp, double *red, double *out) const {
    if (nl == 1) {
      out[c] = v;
      return;
    }
    red[threadIdx.x] = v;
    __syncthreads();
    if (lr == 0) {
      double t = red[c];
      for (int l = 1; l < nl; ++l) t += red[l * sp + c];
      out[c] = t;
    }
    __syncthreads();
  }
};

}  // namespace

int cspmm_blocks_per_cu(int ppl, int u, bool hs) {
  const void *f = select_cspmm(ppl, u, hs);
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kWG, 0) != hipSuccess) return 0;
  return nb;
}

hipError_t launch_cspmm(int ppl, int u, const CspArgs &a, hipStream_t s) {
  const void *f = select_cspmm(ppl, u, a.sval != nullptr);
  if (a.sp % (64 * ppl) != 0 || a.grid % 8 != 0 || a.grid <= 0) return hipErrorInvalidValue;
  CspArgs args = a;
  void *kargs[] = {&args};
  return hipLaunchKernel(f, dim3(a.grid), dim3(kWG), kargs, 0, s);
}

// dst_re = scale * y, dst_im = 0 (dst_im may be null)
__global__ __launch_bounds__(kWG) void k_cx_fill(const uint64_t *sgn, const double *rden,
                                                 int64_t n, int sp, double scale,
                                                 double *__restrict__ dre,
                                                 double *__restrict__ dim) {
  const int64_t total = n * sp;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = e / sp;
    const int c = (int)(e - row * sp);
    dre[e] = scale * probe_value(sgn, rden, row, sp, c);
    if (dim) dim[e] = 0.0;
  }
}

// r = y - q (q null: r = y); partials: part_rr = |r_c|^2, part_yy = y_c . y_c
__global__ __launch_bounds__(kWG) void k_cx_resid(const uint64_t *sgn, const double *rden,
                                                  const double *__restrict__ q, double *__restrict__ r,
                                                  int64_t n, int sp, int64_t plane,
                                                  double *__restrict__ part_rr,
                                                  double *__restrict__ part_yy) {
  int64_t lo, hi;
  row_range(n, lo, hi);
  const ColLanes cl(sp);
  __shared__ double red[kWG];
  for (int c = cl.c0; c < sp; c += cl.cstep) {
    double rr = 0.0, yy = 0.0;
    for (int64_t i = lo + cl.lr; i < hi; i += cl.nl) {
      const int64_t e = i * sp + c;
      const double y = probe_value(sgn, rden, i, sp, c);
      const double a = q ? y - q[e] : y;
      const double b = q ? -q[plane + e] : 0.0;
      r[e] = a;
      r[plane + e] = b;
      rr = fma(b, b, fma(a, a, rr));
      yy = fma(y, y, yy);
    }
    cl.finish(rr, c, sp, red, part_rr + (int64_t)blockIdx.x * sp);
    cl.finish(yy, c, sp, red, part_yy + (int64_t)blockIdx.x * sp);
  }
}

// One CGLS iteration's vector kernels on complex planes, real scalars sc = [yy | gam0 | qq | ssn | rr |
// alpha | beta | gam1] of sp each (gam of iteration it in gam{(it - 1) & 1}, so that no workgroup
// reads what another has replaced).
// k_cgls_update, after q = A p: qq = sums of pa [na][sp], alpha = gam / qq, r -= alpha q, part =
// [shares][sp] partials of |r|^2; *resmax = 0 for k_cgls_dir.
template <int C>
__global__ __launch_bounds__(kSlabThreads) void k_cgls_update(double *__restrict__ r,
                                                              const double *__restrict__ q,
                                                              const double *__restrict__ pa, int na,
                                                              double *__restrict__ sc, int odd, int64_t n, int sp,
                                                              int64_t plane, double *__restrict__ part, int shares,
                                                              double *__restrict__ resmax) {
  __shared__ double red[2][kSlabWaves][C];
  const Slab<C> sl(n, sp, shares);
  const int c = sl.c;
  const double qq = slab_sum<C>(pa, na, sp, c, red[0]);
  const double gam = sc[(odd ? 7 : 1) * sp + c];
  const double al = (gam > 0.0 && qq > 0.0) ? gam / qq : 0.0;
  if (sl.first && threadIdx.x < C) {
    sc[2 * sp + c] = qq;
    sc[5 * sp + c] = al;
    if (c == 0) *resmax = 0.0;
  }
  double rr = 0.0;
#pragma unroll 4
  for (int64_t i = sl.lo; i < sl.hi; i += sl.step) {
    const int64_t e = i * sp + c;
    const double a = fma(-al, q[e], r[e]);
    const double b = fma(-al, q[plane + e], r[plane + e]);
    r[e] = a;
    r[plane + e] = b;
    rr = fma(b, b, fma(a, a, rr));
  }
  rr = slab_total<C>(rr, red[1]);
  if (threadIdx.x < C) part[(int64_t)sl.share * sp + c] = rr;
}

// k_cgls_dir, after s = A^H r: ssn = sums of pa [na][sp], rr = sums of pb [nb][sp], beta = ssn / gam, the
// next gam = ssn; x += alpha p, p = s + beta p; *resmax = max_c rr / yy over columns with yy > 0 (an
// integer max on the bit patterns of non-negative doubles), +inf for a non-finite rr or ssn.
// The planes are taken as 2 n rows.
template <int C>
__global__ __launch_bounds__(kSlabThreads) void k_cgls_dir(const double *__restrict__ sv, double *__restrict__ p,
                                                           double *__restrict__ x, const double *__restrict__ pa,
                                                           int na, const double *__restrict__ pb, int nb,
                                                           double *__restrict__ sc, int odd, int64_t n2, int sp,
                                                           double *__restrict__ resmax) {
  __shared__ double red[2][kSlabWaves][C];
  const Writer<C> wr(n2, sp);
  const int c = wr.c;
  const double ssn = slab_sum<C>(pa, na, sp, c, red[0]);
  const double gam = sc[(odd ? 7 : 1) * sp + c], al = sc[5 * sp + c];
  const double be = gam > 0.0 ? ssn / gam : 0.0;
  if (wr.lead) {  // the whole workgroup: slab_sum has a barrier
    const double rr = slab_sum<C>(pb, nb, sp, c, red[1]);
    if (wr.first) {
      const double yy = sc[c];
      sc[3 * sp + c] = ssn;
      sc[4 * sp + c] = rr;
      sc[6 * sp + c] = be;
      sc[(odd ? 1 : 7) * sp + c] = ssn;
      double m = -1.0;
      if (yy > 0.0) m = rr / yy;
      if (!isfinite(rr) || !isfinite(ssn)) m = HUGE_VAL;
      if (m >= 0.0)
        atomicMax(reinterpret_cast<unsigned long long *>(resmax), (unsigned long long)__double_as_longlong(m));
    }
  }
#pragma unroll 4
  for (int64_t e = wr.e; e < wr.end; e += wr.step) {
    const double pv = p[e];
    x[e] = fma(al, pv, x[e]);
    p[e] = fma(be, pv, sv[e]);
  }
}

// partials of y_c . a_c and y_c . b_c; with acc: acc += wr a - wi b (= Re[(wr + i wi)(a + i b)])
__global__ __launch_bounds__(kWG) void k_cx_pdot(const uint64_t *sgn, const double *rden,
                                                 const double *__restrict__ yd,
                                                 const double *__restrict__ av,
                                                 const double *__restrict__ bv, int64_t n, int sp,
                                                 double *__restrict__ acc, double wr, double wi,
                                                 double *__restrict__ part_a,
                                                 double *__restrict__ part_b) {
  int64_t lo, hi;
  row_range(n, lo, hi);
  const ColLanes cl(sp);
  __shared__ double red[kWG];
  for (int c = cl.c0; c < sp; c += cl.cstep) {
    double sa = 0.0, sb = 0.0;
    for (int64_t i = lo + cl.lr; i < hi; i += cl.nl) {
      const int64_t e = i * sp + c;
      const double y = yd ? yd[e] : probe_value(sgn, rden, i, sp, c);
      const double a = av[e], b = bv[e];
      sa = fma(y, a, sa);
      sb = fma(y, b, sb);
      if (acc) acc[e] = fma(-wi, b, fma(wr, a, acc[e]));
    }
    cl.finish(sa, c, sp, red, part_a + (int64_t)blockIdx.x * sp);
    cl.finish(sb, c, sp, red, part_b + (int64_t)blockIdx.x * sp);
  }
}

// Start of a solve (one workgroup) on sc: gam0 = ssn, *resmax = max_c rr / yy over columns with yy > 0.
__global__ __launch_bounds__(kWG) void k_cgls_start(double *__restrict__ sc, int sp, double *__restrict__ resmax) {
  const double *yy = sc, *ssn = sc + 3 * sp, *rr = sc + 4 * sp;
  double *gam = sc + sp;
  double m = 0.0;
  for (int c = threadIdx.x; c < sp; c += blockDim.x) {
    gam[c] = ssn[c];
    if (yy[c] > 0.0) m = fmax(m, rr[c] / yy[c]);
    // a non-finite residual must reach the host check (fmax drops NaN)
    if (!isfinite(rr[c]) || !isfinite(ssn[c])) m = HUGE_VAL;
  }
  m = wave_max(m);
  __shared__ double red[kWaves];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = red[0];
    for (int w = 1; w < kWaves; ++w) t = fmax(t, red[w]);
    *resmax = t;
  }
}

// N, E, F of the rational estimate (one workgroup, fixed order):
//   per column c:  N_c = f0 m0 + 2 Re sum_k cn_k rho_kc
//                  E_c = f0 h + ew m0 + 2 Re sum_k ce_k rho_kc
//                  F_c = g1 h + g0 m0 + 2 Re sum_k cf_k rho_kc
// with m0 = r.r, h = (H r).(S^{-1} r) (S = I: r.H r), rho_kc = (S r_c) . x_kc and
// coef = [cn | ce | cf] complex per pole; out3 = sum_c w_c (N_c, E_c, F_c).
__global__ __launch_bounds__(kWG) void k_rational_traces(const double *__restrict__ rho,
                                                         const double *__restrict__ m01,
                                                         const double *__restrict__ w,
                                                         const double *__restrict__ coef,
                                                         int n_poles, int sp, RationalScalars k,
                                                         double *__restrict__ out3) {
  double acc[3] = {0.0, 0.0, 0.0};
  for (int c = threadIdx.x; c < sp; c += blockDim.x) {
    const double m0 = m01[c], rhr = m01[sp + c];
    double sn = 0.0, se = 0.0, sf = 0.0;
    for (int p = 0; p < n_poles; ++p) {
      const double pr = rho[(int64_t)p * 2 * sp + c], pi = rho[(int64_t)p * 2 * sp + sp + c];
      const double *cn = coef + 2 * p, *ce = coef + 2 * (n_poles + p), *cf = coef + 2 * (2 * n_poles + p);
      sn += cn[0] * pr - cn[1] * pi;
      se += ce[0] * pr - ce[1] * pi;
      sf += cf[0] * pr - cf[1] * pi;
    }
    const double wc = w[c];
    acc[0] = fma(wc, k.f0 * m0 + 2.0 * sn, acc[0]);
    acc[1] = fma(wc, k.f0 * rhr + k.ew * m0 + 2.0 * se, acc[1]);
    acc[2] = fma(wc, k.g1 * rhr + k.g0 * m0 + 2.0 * sf, acc[2]);
  }
  __shared__ double red[3][kWaves];
  for (int t = 0; t < 3; ++t) {
    const double v = wave_sum(acc[t]);
    if ((threadIdx.x & 63) == 0) red[t][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0.0;
    for (int wv = 0; wv < kWaves; ++wv) s += red[threadIdx.x][wv];
    out3[threadIdx.x] = s;
  }
}

namespace {
int ew_blocks(int64_t total) {
  int64_t b = (total + kWG - 1) / kWG;
  if (b > 65536) b = 65536;
  return (int)std::max<int64_t>(1, b);
}
}  // namespace

hipError_t launch_cx_fill(const uint64_t *sgn, const double *rden, int64_t n, int sp, double scale,
                          double *dre, double *dim, hipStream_t s) {
  hipLaunchKernelGGL(k_cx_fill, dim3(ew_blocks(n * sp)), dim3(kWG), 0, s, sgn, rden, n, sp, scale,
                     dre, dim);
  return hipGetLastError();
}

hipError_t launch_cx_resid(const uint64_t *sgn, const double *rden, const double *q, double *r,
                           int64_t n, int sp, double *part_rr, double *part_yy, hipStream_t s) {
  hipLaunchKernelGGL(k_cx_resid, dim3(cg_nparts(n)), dim3(kWG), 0, s, sgn, rden, q, r, n, sp,
                     n * sp, part_rr, part_yy);
  return hipGetLastError();
}

template <int C>
static void launch_cgls_update_t(double *r, const double *q, const double *pa, int na, double *sc, int64_t it,
                                 int64_t n, int sp, double *part, double *resmax, hipStream_t s) {
  const int shares = slab_shares<C>(n, sp);
  hipLaunchKernelGGL((k_cgls_update<C>), dim3(sp / C * shares), dim3(kSlabThreads), 0, s, r, q, pa, na, sc,
                     (int)((it - 1) & 1), n, sp, n * sp, part, shares, resmax);
}

hipError_t launch_cgls_update(double *r, const double *q, const double *pa, int na, double *sc, int64_t it,
                              int64_t n, int sp, double *part, double *resmax, hipStream_t s) {
  if (sp <= 0 || sp % 64 != 0 || n <= 0) return hipErrorInvalidValue;
  if (slab_wide(n, sp)) {
    const hipError_t e = launch_colreduce(pa, na, sp, sc + 2 * sp, s);  // |q|^2 itself
    if (e != hipSuccess) return e;
    launch_cgls_update_t<64>(r, q, sc + 2 * sp, 1, sc, it, n, sp, part, resmax, s);
  } else {
    launch_cgls_update_t<16>(r, q, pa, na, sc, it, n, sp, part, resmax, s);
  }
  return hipGetLastError();
}

template <int C>
static void launch_cgls_dir_t(const double *sv, double *p, double *x, const double *pa, int na, const double *pb,
                              int nb, double *sc, int64_t it, int64_t n, int sp, double *resmax, hipStream_t s) {
  hipLaunchKernelGGL((k_cgls_dir<C>), dim3(Writer<C>::grid(n, 2 * n, sp)), dim3(kSlabThreads), 0, s, sv, p, x, pa, na,
                     pb, nb, sc, (int)((it - 1) & 1), 2 * n, sp, resmax);
}

hipError_t launch_cgls_dir(const double *sv, double *p, double *x, const double *pa, int na, const double *pb,
                           double *sc, int64_t it, int64_t n, int sp, double *resmax, hipStream_t s) {
  if (sp <= 0 || sp % 64 != 0 || n <= 0) return hipErrorInvalidValue;
  if (!slab_wide(n, sp)) {
    launch_cgls_dir_t<16>(sv, p, x, pa, na, pb, slab_shares<16>(n, sp), sc, it, n, sp, resmax, s);
    return hipGetLastError();
  }
  // |s|^2 and |r|^2 themselves
  const hipError_t e =
      launch_colreduce(pa, na, sp, sc + 3 * sp, s, pb, slab_shares<64>(n, sp), sc + 4 * sp);
  if (e != hipSuccess) return e;
  launch_cgls_dir_t<64>(sv, p, x, sc + 3 * sp, 1, sc + 4 * sp, 1, sc, it, n, sp, resmax, s);
  return hipGetLastError();
}

hipError_t launch_cx_pdot(const uint64_t *sgn, const double *rden, const double *yd, const double *a,
                          const double *b, int64_t n, int sp, double *acc, double wr, double wi,
                          double *part_a, double *part_b, hipStream_t s) {
  hipLaunchKernelGGL(k_cx_pdot, dim3(cg_nparts(n)), dim3(kWG), 0, s, sgn, rden, yd, a, b, n, sp,
                     acc, wr, wi, part_a, part_b);
  return hipGetLastError();
}

// dst = alpha * src over n elements
__global__ __launch_bounds__(kWG) void k_cx_scale(const double *__restrict__ src,
                                                  double *__restrict__ dst, int64_t n,
                                                  double alpha) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = alpha * src[e];
}

hipError_t launch_cx_scale(const double *src, double *dst, int64_t n, double alpha, hipStream_t s) {
  hipLaunchKernelGGL(k_cx_scale, dim3(ew_blocks(n)), dim3(kWG), 0, s, src, dst, n, alpha);
  return hipGetLastError();
}

hipError_t launch_cgls_start(double *sc, int sp, double *resmax, hipStream_t s) {
  hipLaunchKernelGGL(k_cgls_start, dim3(1), dim3(kWG), 0, s, sc, sp, resmax);
  return hipGetLastError();
}

hipError_t launch_rational_traces(const double *rho, const double *m01, const double *w,
                                  const double *coef, int n_poles, int sp,
                                  const RationalScalars &k, double *out3, hipStream_t s) {
  hipLaunchKernelGGL(k_rational_traces, dim3(1), dim3(kWG), 0, s, rho, m01, w, coef, n_poles, sp,
                     k, out3);
  return hipGetLastError();
}

}  // namespace rfo
