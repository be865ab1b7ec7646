// Nonorthogonal basis (paper: Polynomial approximation with S, Eq. poly_PQ):
// the mapped Hamiltonian H_hat = [2H - (e_max + e_min) S]/(e_max - e_min) and
// the pieces of a conjugate-gradient solve S t = y for a block of probe columns
// (one independent CG per column; the matrix-vector product is the step kernel
// with S as its matrix).  Column reductions are two-pass and in a fixed order.
#include "colsum.h"
#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

__global__ __launch_bounds__(kWG) void k_map_overlap(const double *__restrict__ h,
                                                     const double *__restrict__ s,
                                                     const int64_t *__restrict__ tpos,
                                                     int64_t nnzb, int bd, double e_min,
                                                     double e_max, double *__restrict__ hhat,
                                                     int *flags) {
  const int bb = bd * bd;
  const int64_t total = nnzb * bb;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t nz = e / bb;
    const int rem = (int)(e - nz * bb);
    const int i = rem / bd, j = rem - (rem / bd) * bd;
    const double v = s[e];
    if (!isfinite(v)) atomicOr(flags, 1);
    const double vt = s[tpos[nz] * bb + j * bd + i];
    if (!(fabs(v - vt) <= 1e-10 * (fabs(v) + fabs(vt)))) atomicOr(flags, 2);
    hhat[e] = (2.0 * h[e] - (e_max + e_min) * v) / (e_max - e_min);
  }
}

hipError_t launch_map_overlap(const double *h, const double *s, const int64_t *tpos, int64_t nnzb,
                              int bd, double e_min, double e_max, double *hhat, int *flags,
                              hipStream_t st) {
  const int64_t total = nnzb * bd * bd;
  int64_t blocks = (total + kWG - 1) / kWG;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_map_overlap, dim3((unsigned)blocks), dim3(kWG), 0, st, h, s, tpos, nnzb, bd,
                     e_min, e_max, hhat, flags);
  return hipGetLastError();
}

namespace {

// rows [lo, hi) of workgroup b when n rows are split over gridDim.x workgroups
__device__ __forceinline__ void row_range(int64_t n, int64_t &lo, int64_t &hi) {
  const int64_t G = gridDim.x, b = blockIdx.x;
  lo = n * b / G;
  hi = n * (b + 1) / G;
}

}  // namespace

// out[c] = sum_b part[b][c] in the fixed order of colsum; blockIdx.y = 1: of part2 into out2.
__global__ __launch_bounds__(64 * kColWaves) void k_colreduce(const double *__restrict__ part,
                                                              int nparts,
                                                              const double *__restrict__ part2,
                                                              int nparts2, int sp,
                                                              double *__restrict__ out,
                                                              double *__restrict__ out2) {
  __shared__ double red[kColPh][kColCols];
  int c;
  const bool second = blockIdx.y == 1;
  const double t = colsum(second ? part2 : part, second ? nparts2 : nparts, sp, red, c);
  if (threadIdx.x < kColCols && c < sp) (second ? out2 : out)[c] = t;
}

// The row-range kernels below split a workgroup's threads into R = 256 / C row lanes of
// C columns (C = 64, 128 or 256, the widest that divides sp): rows lo + rl, lo + rl + R,
// ... for the C columns c0 + cl, column chunk by column chunk; the R row lanes of a
// column are then added in row-lane order, so the partials are bitwise reproducible.
__device__ __forceinline__ int cg_cols(int sp) {
  int C = 64;
  while (C < kWG && sp % (2 * C) == 0) C *= 2;
  return C;
}

// t = 0, r = y, p = y, part = column partials of y . y
__global__ __launch_bounds__(kWG) void k_cg_init(const double *__restrict__ y,
                                                 double *__restrict__ t, double *__restrict__ r,
                                                 double *__restrict__ p, int64_t n, int sp,
                                                 double *__restrict__ part) {
  int64_t lo, hi;
  row_range(n, lo, hi);
  const int C = cg_cols(sp), R = kWG / C;
  const int cl = threadIdx.x % C, rl = threadIdx.x / C;
  __shared__ double red[kWG];
  for (int c0 = 0; c0 < sp; c0 += C) {
    const int c = c0 + cl;
    double s = 0.0;
    for (int64_t i = lo + rl; i < hi; i += R) {
      const int64_t e = i * sp + c;
      const double v = y[e];
      t[e] = 0.0;
      r[e] = v;
      p[e] = v;
      s = fma(v, v, s);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (rl == 0) {
      double a = red[cl];
      for (int q = 1; q < R; ++q) a += red[q * C + cl];
      part[(int64_t)blockIdx.x * sp + c] = a;
    }
    __syncthreads();
  }
}

// One CG iteration after q = S p, on sc = [yy | rr0 | pq | rrn | alpha | beta | rr1] of sp each (rr of
// iteration it in rr{(it - 1) & 1}, so that no workgroup reads what another has replaced).  Columns
// with rr = 0 keep alpha = beta = 0.
// k_cg_update: pq = sums of spart [ns][sp] (p . q), alpha = rr / pq, t += alpha p, r -= alpha q, part =
// [shares][sp] partials of r . r; *resmax = 0 for k_cg_direction.
template <int C>
__global__ __launch_bounds__(kSlabThreads) void k_cg_update(double *__restrict__ t, double *__restrict__ r,
                                                            const double *__restrict__ p,
                                                            const double *__restrict__ q,
                                                            const double *__restrict__ spart, int ns,
                                                            double *__restrict__ sc, int odd, int64_t n, int sp,
                                                            double *__restrict__ part, int shares,
                                                            double *__restrict__ resmax) {
  __shared__ double red[2][kSlabWaves][C];
  const Slab<C> sl(n, sp, shares);
  const int c = sl.c;
  const double pq = slab_sum<C>(spart, ns, sp, c, red[0]);
  const double rr = sc[(odd ? 6 : 1) * sp + c];
  const double al = (rr > 0.0 && pq != 0.0) ? rr / pq : 0.0;
  if (sl.first && threadIdx.x < C) {
    sc[2 * sp + c] = pq;
    sc[4 * sp + c] = al;
    if (c == 0) *resmax = 0.0;
  }
  double s = 0.0;
#pragma unroll 4
  for (int64_t i = sl.lo; i < sl.hi; i += sl.step) {
    const int64_t e = i * sp + c;
    t[e] = fma(al, p[e], t[e]);
    const double rn = fma(-al, q[e], r[e]);
    r[e] = rn;
    s = fma(rn, rn, s);
  }
  s = slab_total<C>(s, red[1]);
  if (threadIdx.x < C) part[(int64_t)sl.share * sp + c] = s;
}

// k_cg_direction: rrn = sums of part [shares][sp], beta = rrn / rr, the next rr = rrn, p = r + beta p, and
// *resmax = max_c rrn / yy over columns with yy > 0, by an integer max on the bit patterns
// (non-negative doubles order as their bits, and a NaN ends above every finite value).
template <int C>
__global__ __launch_bounds__(kSlabThreads) void k_cg_direction(const double *__restrict__ r,
                                                               double *__restrict__ p,
                                                               const double *__restrict__ part, int np,
                                                               double *__restrict__ sc, int odd, int64_t n,
                                                               int sp, double *__restrict__ resmax) {
  __shared__ double red[kSlabWaves][C];
  const Writer<C> wr(n, sp);
  const int c = wr.c;
  const double rrn = slab_sum<C>(part, np, sp, c, red);
  const double rr = sc[(odd ? 6 : 1) * sp + c];
  const double be = rr > 0.0 ? rrn / rr : 0.0;
  if (wr.first) {
    sc[3 * sp + c] = rrn;
    sc[5 * sp + c] = be;
    sc[(odd ? 1 : 6) * sp + c] = rrn;
    const double yy = sc[c];
    if (yy > 0.0)
      atomicMax(reinterpret_cast<unsigned long long *>(resmax), (unsigned long long)__double_as_longlong(rrn / yy));
  }
#pragma unroll 4
  for (int64_t e = wr.e; e < wr.end; e += wr.step) p[e] = fma(be, p[e], r[e]);
}

// yy = rr0 = column sums of part [nparts][sp] (start of a solve), formed as in k_colreduce
__global__ __launch_bounds__(64 * kColWaves) void k_cg_start(const double *__restrict__ part, int nparts, int sp,
                                                             double *__restrict__ sc) {
  __shared__ double red[kColPh][kColCols];
  int c;
  const double v = colsum(part, nparts, sp, red, c);
  if (threadIdx.x >= kColCols || c >= sp) return;
  sc[c] = v;
  sc[sp + c] = v;
}

namespace {
// row ranges of the kernels outside the iterations: eight rows each (64 left 2,250 rows on 36
// workgroups: 18 us for 128 columns)
int cg_parts(int64_t n) { return (int)std::min<int64_t>(1024, (n + 7) / 8); }
}  // namespace

int cg_nparts(int64_t n) { return cg_parts(n); }

hipError_t launch_colreduce(const double *part, int nparts, int sp, double *out, hipStream_t s,
                            const double *part2, int nparts2, double *out2) {
  hipLaunchKernelGGL(k_colreduce, dim3((sp + kColCols - 1) / kColCols, part2 ? 2 : 1), dim3(64 * kColWaves), 0, s,
                     part, nparts, part2, nparts2, sp, out, out2);
  return hipGetLastError();
}

hipError_t launch_cg_init(const double *y, double *t, double *r, double *p, int64_t n, int sp,
                          double *part, double *sc, hipStream_t s) {
  if (sp <= 0 || sp % 64 != 0) return hipErrorInvalidValue;
  const int G = cg_parts(n);
  hipLaunchKernelGGL(k_cg_init, dim3(G), dim3(kWG), 0, s, y, t, r, p, n, sp, part);
  hipLaunchKernelGGL(k_cg_start, dim3((sp + kColCols - 1) / kColCols), dim3(64 * kColWaves), 0, s, part, G, sp,
                     sc);
  return hipGetLastError();
}

template <int C>
static hipError_t launch_cg_update_t(double *t, double *r, double *p, const double *q, const double *spart, int ns,
                                     int64_t it, int64_t n, int sp, double *part, double *sc, double *resmax,
                                     hipStream_t s) {
  const int shares = slab_shares<C>(n, sp), odd = (int)((it - 1) & 1);
  hipLaunchKernelGGL((k_cg_update<C>), dim3(sp / C * shares), dim3(kSlabThreads), 0, s, t, r, p, q, spart, ns, sc,
                     odd, n, sp, part, shares, resmax);
  const double *pr = part;
  int np = shares;
  if (C == 64) {
    pr = sc + 3 * sp;  // |r|^2 itself
    np = 1;
    const hipError_t e = launch_colreduce(part, shares, sp, sc + 3 * sp, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_cg_direction<C>), dim3(Writer<C>::grid(n, n, sp)), dim3(kSlabThreads), 0, s,
                     r, p, pr, np, sc, odd, n, sp, resmax);
  return hipGetLastError();
}

hipError_t launch_cg_update(double *t, double *r, double *p, const double *q, const double *spart, int ns,
                            int64_t it, int64_t n, int sp, double *part, double *sc, double *resmax,
                            hipStream_t s) {
  if (sp <= 0 || sp % 64 != 0 || n <= 0) return hipErrorInvalidValue;
  if (!slab_wide(n, sp)) return launch_cg_update_t<16>(t, r, p, q, spart, ns, it, n, sp, part, sc, resmax, s);
  const hipError_t e = launch_colreduce(spart, ns, sp, sc + 2 * sp, s);  // p . q itself
  if (e != hipSuccess) return e;
  return launch_cg_update_t<64>(t, r, p, q, sc + 2 * sp, 1, it, n, sp, part, sc, resmax, s);
}

// out = ca A + cb B + cc C + cr r (a null operand or a zero weight adds nothing; r is the
// probe block, sign bits or dense)
__global__ __launch_bounds__(kWG) void k_combine(double *__restrict__ out, double ca, const double *A,
                                                 double cb, const double *B, double cc, const double *C,
                                                 double cr, const uint64_t *__restrict__ sgn,
                                                 const double *__restrict__ rden, int64_t n, int sp) {
  const int64_t total = n * sp;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    double v = 0.0;
    if (A && ca != 0.0) v = fma(ca, A[e], v);
    if (B && cb != 0.0) v = fma(cb, B[e], v);
    if (C && cc != 0.0) v = fma(cc, C[e], v);
    if (cr != 0.0) {
      const int64_t row = e / sp;
      v = fma(cr, probe_value(sgn, rden, row, sp, (int)(e - row * sp)), v);
    }
    out[e] = v;
  }
}

hipError_t launch_combine(double *out, double ca, const double *A, double cb, const double *B, double cc,
                          const double *C, double cr, const uint64_t *sgn, const double *rden, int64_t n,
                          int sp, hipStream_t s) {
  int64_t blocks = (n * sp + kWG - 1) / kWG;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_combine, dim3((unsigned)blocks), dim3(kWG), 0, s, out, ca, A, cb, B, cc, C, cr, sgn,
                     rden, n, sp);
  return hipGetLastError();
}

}  // namespace rfo
