// Setup and reduction kernels of the randomized Fermi-operator path:
//   spectral map of H (Polynomial approximation: H_hat = (2H - (e_max+e_min)I)/(e_max-e_min)),
//   Gershgorin interval fallback, probe packing, Chebyshev coefficients of the
//   Fermi, energy-weighted and free-energy functions by Chebyshev-Gauss
//   quadrature, fixed-order moment reduction and the traces N, E, F
//   (Methods: free-energy function, electron count and band energy).
// Every reduction here runs in a fixed order: results are bitwise reproducible.
#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

// ---- spectral map -----------------------------------------------------------
__global__ __launch_bounds__(kWG) void k_map(const double *__restrict__ h,
                                             const int64_t *__restrict__ brow,
                                             const int32_t *__restrict__ col,
                                             const int64_t *__restrict__ tpos, int64_t nnzb,
                                             int bd, double e_min, double e_max,
                                             double *__restrict__ hhat64,
                                             float *__restrict__ hhat32, int *flags) {
  const int bb = bd * bd;
  const int64_t total = nnzb * bb;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t nz = e / bb;
    const int rem = (int)(e - nz * bb);
    const int i = rem / bd, j = rem - (rem / bd) * bd;
    const double v = h[e];
    if (!isfinite(v)) atomicOr(flags, 1);
    const double vt = h[tpos[nz] * bb + j * bd + i];
    if (!(fabs(v - vt) <= 1e-10 * (fabs(v) + fabs(vt)))) atomicOr(flags, 2);
    const bool diag = (brow[nz] == (int64_t)col[nz]) && (i == j);
    const double shifted = diag ? 2.0 * v - (e_max + e_min) : 2.0 * v;
    const double hh = shifted / (e_max - e_min);
    hhat64[e] = hh;
    if (hhat32) hhat32[e] = (float)hh;
  }
}

hipError_t launch_map(const double *h, const int64_t *brow, const int32_t *col,
                      const int64_t *tpos, int64_t nnzb, int bd, double e_min,
                      double e_max, double *hhat64, float *hhat32, int *flags,
                      hipStream_t s) {
  const int64_t total = nnzb * bd * bd;
  int64_t blocks = (total + kWG - 1) / kWG;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_map, dim3((unsigned)blocks), dim3(kWG), 0, s, h, brow, col, tpos,
                     nnzb, bd, e_min, e_max, hhat64, hhat32, flags);
  return hipGetLastError();
}

// ---- Gershgorin interval ----------------------------------------------------
__global__ __launch_bounds__(kWG) void k_gersh_rows(const double *__restrict__ h,
                                                    const int64_t *__restrict__ row_ptr,
                                                    const int32_t *__restrict__ col, int64_t nb,
                                                    int bd, double *__restrict__ scratch) {
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double lo = INFINITY, hi = -INFINITY;
  if (row < nb * bd) {
    const int64_t I = row / bd;
    const int i = (int)(row - I * bd);
    double center = 0.0, rad = 0.0;
    for (int64_t nz = row_ptr[I]; nz < row_ptr[I + 1]; ++nz) {
      for (int j = 0; j < bd; ++j) {
        const double v = h[(nz * bd + i) * bd + j];
        if ((int64_t)col[nz] == I && j == i) center = v;
        else rad += fabs(v);
      }
    }
    lo = center - rad;
    hi = center + rad;
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  __shared__ double slo[kWaves], shi[kWaves];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    slo[wave] = lo;
    shi[wave] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) {
      lo = fmin(lo, slo[w]);
      hi = fmax(hi, shi[w]);
    }
    scratch[2 * blockIdx.x] = fmin(lo, slo[0]);
    scratch[2 * blockIdx.x + 1] = fmax(hi, shi[0]);
  }
}

__global__ __launch_bounds__(kWG) void k_gersh_final(const double *__restrict__ scratch,
                                                     int nblk, double *out2) {
  double lo = INFINITY, hi = -INFINITY;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    lo = fmin(lo, scratch[2 * b]);
    hi = fmax(hi, scratch[2 * b + 1]);
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  __shared__ double slo[kWaves], shi[kWaves];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    slo[wave] = lo;
    shi[wave] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < kWaves; ++w) {
      lo = fmin(lo, slo[w]);
      hi = fmax(hi, shi[w]);
    }
    out2[0] = lo;
    out2[1] = hi;
  }
}

hipError_t launch_gershgorin(const double *h, const int64_t *row_ptr, const int32_t *col,
                             int64_t nb, int bd, double *scratch, double *out2,
                             hipStream_t s) {
  const int64_t rows = nb * bd;
  const int nblk = (int)((rows + kWG - 1) / kWG);
  hipLaunchKernelGGL(k_gersh_rows, dim3(nblk), dim3(kWG), 0, s, h, row_ptr, col, nb, bd,
                     scratch);
  hipLaunchKernelGGL(k_gersh_final, dim3(1), dim3(kWG), 0, s, scratch, nblk, out2);
  return hipGetLastError();
}

// ---- probes -------------------------------------------------------------------
// flags bit 0: some real entry is not +-1 (dense storage needed); bit 1: non-finite
__global__ __launch_bounds__(kWG) void k_probe_pack(const double *__restrict__ rden, int64_t n,
                                                    int s_real, int sp, uint64_t *__restrict__ sgn,
                                                    int *flags) {
  const int nw = sp >> 6;
  const int64_t total = n * nw;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = t / nw;
    const int w = (int)(t - row * nw);
    uint64_t bits = 0;
    for (int b = 0; b < 64; ++b) {
      const int c = w * 64 + b;
      const double v = rden[row * sp + c];
      if (c < s_real) {
        if (!isfinite(v)) atomicOr(flags, 2);
        if (v != 1.0 && v != -1.0) atomicOr(flags, 1);
      }
      if (v > 0.0) bits |= (1ull << b);
    }
    sgn[t] = bits;
  }
}

hipError_t launch_probe_pack(const double *rden, int64_t n, int s_real, int sp, uint64_t *sgn,
                             int *flags, hipStream_t st) {
  const int64_t total = n * (sp >> 6);
  int64_t blocks = (total + kWG - 1) / kWG;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_probe_pack, dim3((unsigned)blocks), dim3(kWG), 0, st, rden, n, s_real,
                     sp, sgn, flags);
  return hipGetLastError();
}

// ---- Chebyshev coefficients -----------------------------------------------------
// Node j of the nq-point Chebyshev-Gauss rule: x_j = cos(pi (j + 1/2)/nq), energy
// e_j = e_min (1 - x_j)/2 + e_max (1 + x_j)/2.  Samples of
//   f(e) = 2/(1 + exp((e - mu)/T)) = 1 - tanh((e - mu)/(2T)),  e f(e),
//   g(e) = -2T ln(1 + exp(-(e - mu)/T)) (stable softplus form),
// and the table cos(pi m/(2 nq)), m <= nq, a quarter turn: cos(pi k (j + 1/2)/nq) is the whole turn's
// entry (k (2j + 1)) mod 4 nq, so the argument reduction is exact for every k.
// Node nq - 1 - j has the cosine of node j times (-1)^k, so the sums run over half the nodes: the
// samples are kept as h_j + h_{nq-1-j} (even k, first nq/2 of nq) and h_j - h_{nq-1-j} (odd k).
//
// HALF = false, for the BF16 steps: all nodes in order, and the whole turn as the table (4 nq entries).
// The two ways round differently in the last bit, which means nothing to FP64 and FP32 vectors. The BF16
// gradient rounds z_j to eight bits in every step, and a last bit in its sources decides some of those
// roundings: it moved the forces by the path's whole error (1.1e-3 at 16,000 atoms, 1,000 terms). Their
// coefficients therefore keep one order of sums for good, at 1,084 us against 124 for 8,000 terms (0.03% of
// the 16,000-atom call that they belong to).
template <bool HALF>
__global__ __launch_bounds__(kWG) void k_coef_samples(double e_min, double e_max, double T,
                                                      double mu, int64_t nq,
                                                      double *__restrict__ samples,
                                                      double *__restrict__ costab) {
  const int64_t half = nq / 2, nodes = HALF ? half : nq, entries = HALF ? nq + 1 : 4 * nq;
  for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < entries;
       m += (int64_t)gridDim.x * blockDim.x) {
    costab[m] = cospi((double)m / (double)(2 * nq));
    if (m < nodes) {
      double h[2][3];
#pragma unroll
      for (int t = 0; t < (HALF ? 2 : 1); ++t) {
        const int64_t j = t ? nq - 1 - m : m;
        const double x = cos(M_PI * ((double)j + 0.5) / (double)nq);
        const double e = 0.5 * e_min * (1.0 - x) + 0.5 * e_max * (1.0 + x);
        const double f = 1.0 - tanh((e - mu) / (2.0 * T));
        const double z = -(e - mu) / T;
        const double softplus = fmax(z, 0.0) + log1p(exp(-fabs(z)));
        h[t][0] = f;
        h[t][1] = e * f;
        h[t][2] = -2.0 * T * softplus;
      }
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        samples[i * nq + m] = HALF ? h[0][i] + h[1][i] : h[0][i];
        if (HALF) samples[i * nq + half + m] = h[0][i] - h[1][i];
      }
    }
  }
}

// c_k = (2 - delta_k0)/nq sum_j h(e_j) cos(pi k (j + 1/2)/nq), a workgroup of NTHR threads per four k of
// one parity (the grid is even, so all its k have it).  The p * nq/2 scattered table reads are what
// costs, so the table is in LDS where it fits (NTAB entries; 0: read from memory): k (2j + 1) has k's
// parity, and so has every fold of it into the quarter turn, so every other entry will do.
// 1,024 terms: 21 us with one k per workgroup and the whole table in memory, 9.7 now; 4,000 terms: 290
// and 47.
template <int NTAB, int NTHR, bool HALF>
__global__ __launch_bounds__(NTHR) void k_coefs(const double *__restrict__ samples,
                                                const double *__restrict__ costab, int64_t nq,
                                                int64_t p, double *__restrict__ coef) {
  static_assert(HALF || NTAB == 0, "the table in LDS is a quarter turn");
  constexpr int K = 4, W = NTHR / 64;
  // one slot in 33 unused: the lanes of a wave are k entries apart
  __shared__ double tab[NTAB > 0 ? NTAB + NTAB / 32 : 1];
  auto slot = [](uint32_t i) { return i + (i >> 5); };
  __shared__ double red[3 * K][W];
  if (NTAB > 0) {
    const int odd = blockIdx.x & 1;
#pragma unroll 8
    for (int m = threadIdx.x; 2 * m + odd <= (int)nq; m += NTHR) tab[slot(m)] = costab[2 * m + odd];
    __syncthreads();
  }
  const uint32_t M = (uint32_t)(4 * nq), nodes = (uint32_t)(HALF ? nq / 2 : nq), quarter = (uint32_t)nq;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t groups = (p + 7) / 8 * 2;
  for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
    const int64_t k0 = (g >> 1) * 8 + (g & 1);
    uint32_t at[K], by[K];  // table position of the thread's node, and its advance per NTHR nodes
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const uint32_t k = (uint32_t)(k0 + 2 * u);  // < 2^20 + 8: the products fit 32 bits
      at[u] = k * (2 * threadIdx.x + 1) % M;
      by[u] = k * (2 * NTHR) % M;
    }
    const double *h = samples + (HALF && (g & 1) ? nodes : 0);
    double s[3][K];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int u = 0; u < K; ++u) s[i][u] = 0.0;
#pragma unroll 4
    for (uint32_t j = threadIdx.x; j < nodes; j += NTHR) {
      double hv[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) hv[i] = h[i * nq + j];
#pragma unroll
      for (int u = 0; u < K; ++u) {
        uint32_t m = at[u];
        const uint32_t next = m + by[u];
        at[u] = min(next, next - M);           // next - M wraps to the top where next < M
        bool neg = false;
        if (HALF) {
          m = min(m, M - m);                   // cos(-t) = cos t
          neg = m > quarter;                   // cos(pi - t) = -cos t
          m = min(m, 2 * quarter - m);
        }
        const double v = NTAB > 0 ? tab[slot(m >> 1)] : costab[m];
        const double cv = neg ? -v : v;
#pragma unroll
        for (int i = 0; i < 3; ++i) s[i][u] = fma(hv[i], cv, s[i][u]);
      }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const double v = wave_sum(s[i][u]);
        if (lane == 0) red[i * K + u][wave] = v;
      }
    __syncthreads();
    if (threadIdx.x < 3 * K) {
      const int i = threadIdx.x / K;
      const int64_t k = k0 + 2 * (threadIdx.x % K);
      double t = 0.0;
      for (int w = 0; w < W; ++w) t += red[threadIdx.x][w];
      if (k < p) coef[i * p + k] = (k == 0 ? 1.0 : 2.0) / (double)nq * t;
    }
    __syncthreads();
  }
}

hipError_t launch_coefficients(double e_min, double e_max, double T, double mu, int64_t p,
                               int64_t nq, bool half, double *samples, double *costab, double *coef,
                               hipStream_t s) {
  if (nq % 2 != 0 || nq < 2 || p > (1 << 20)) return hipErrorInvalidValue;
  const int64_t blocks = std::min<int64_t>(65536, ((half ? nq + 1 : 4 * nq) + kWG - 1) / kWG);
  const unsigned groups = (unsigned)((p + 7) / 8 * 2);
  if (!half) {
    hipLaunchKernelGGL(k_coef_samples<false>, dim3((unsigned)blocks), dim3(kWG), 0, s, e_min, e_max, T, mu, nq, samples,
                       costab);
    hipLaunchKernelGGL((k_coefs<0, 256, false>), dim3(groups), dim3(256), 0, s, samples, costab, nq, p, coef);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_coef_samples<true>, dim3((unsigned)blocks), dim3(kWG), 0, s, e_min, e_max, T, mu, nq, samples,
                     costab);
  if (nq <= 8192)  // 32 KB of LDS: several workgroups per compute unit
    hipLaunchKernelGGL((k_coefs<4097, 256, true>), dim3(groups), dim3(256), 0, s, samples, costab, nq, p, coef);
  else if (nq <= 32768)  // 128 KB: one, which keeps its table for all its k
    hipLaunchKernelGGL((k_coefs<16385, 1024, true>), dim3(std::min(groups, 256u)), dim3(1024), 0, s, samples, costab, nq, p,
                       coef);
  else
    hipLaunchKernelGGL((k_coefs<0, 1024, true>), dim3(groups), dim3(1024), 0, s, samples, costab, nq, p, coef);
  return hipGetLastError();
}

// ---- moments ---------------------------------------------------------------------
// flags bit 2: a moment exceeded its bound or is not finite.
// One workgroup of 16 waves per (moment index, 64-probe chunk): wave w sums the
// partial rows g = w, w + 16, ... into four interleaved accumulators (so that
// each lane keeps four loads in flight), adds them as (s0 + s1) + (s2 + s3), and
// wave 0 adds the 16 wave sums in order.  The order is fixed, so the moments are
// bitwise reproducible.
constexpr int kRedWaves = 16;

__global__ __launch_bounds__(64 * kRedWaves) void k_moment_reduce(const double *__restrict__ part, int ring,
                                                                  int64_t k0, int count, int n_rg, int sp,
                                                                  double *__restrict__ moments, int check,
                                                                  double tol, int *flags, int dbl) {
  const int chunks = sp >> 6;
  const int d = blockIdx.x / chunks;
  const int lane = threadIdx.x & 63;
  const int c = (blockIdx.x - d * chunks) * 64 + lane;
  const int wave = threadIdx.x >> 6;
  const int64_t k = k0 + d;
  const double *src = part + (int64_t)(k % ring) * n_rg * sp + c;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  int g = wave;
  for (; g + 3 * kRedWaves < n_rg; g += 4 * kRedWaves) {
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] += src[(int64_t)(g + u * kRedWaves) * sp];
  }
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (g + u * kRedWaves < n_rg) s[u] += src[(int64_t)(g + u * kRedWaves) * sp];
  __shared__ double red[kRedWaves][64];
  red[wave][lane] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (wave == 0) {
    double sum = red[0][lane];
    for (int w = 1; w < kRedWaves; ++w) sum += red[w][lane];
    // doubling: the partials hold <y_j, y_j> (k = 2j) or <y_j, y_{j-1}> (k = 2j-1);
    // T_2j = 2 T_j^2 - T_0 and T_2j-1 = 2 T_j T_j-1 - T_1 give the moment
    if (dbl && k >= 2) sum = 2.0 * sum - moments[(k & 1) * sp + c];
    moments[k * sp + c] = sum;
    if (check) {
      const double bound = moments[c] * (1.0 + tol) + 1e-300;
      if (!(fabs(sum) <= bound)) atomicOr(flags, 4);
    }
  }
}

hipError_t launch_moment_reduce(const double *part, int ring, int64_t k0, int count, int n_rg,
                                int sp, double *moments, int check, double tol, int *flags,
                                int dbl, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_moment_reduce, dim3((unsigned)(count * (sp >> 6))), dim3(64 * kRedWaves), 0, s, part,
                     ring, k0, count, n_rg, sp, moments, check, tol, flags, dbl);
  return hipGetLastError();
}

// ---- traces ----------------------------------------------------------------------
// out = [N, E, F] = sum_k c_k sum_c w_c mu[k][c] for the three coefficient sets: each wave takes every
// (kWaves G)-th k with its lanes along the probes, the G workgroups' sums part [3][G] are added in
// order by one more.  (One workgroup with a k per thread: 33 us for 1,024 moments of 64 probes,
// 3.3 + 1.6 now; 4,000 of 128 probes 260 and 6.6 + 5.6.)
__global__ __launch_bounds__(kWG) void k_traces(const double *__restrict__ moments,
                                                const double *__restrict__ w,
                                                const double *__restrict__ coef, int64_t p, int sp,
                                                double *__restrict__ part) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t step = (int64_t)gridDim.x * kWaves;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  for (int c = lane; c < sp; c += 64) {
    const double wc = w[c];
#pragma unroll 4
    for (int64_t k = (int64_t)blockIdx.x * kWaves + wave; k < p; k += step) {
      const double m = wc * moments[k * sp + c];
      s0 = fma(coef[k], m, s0);
      s1 = fma(coef[p + k], m, s1);
      s2 = fma(coef[2 * p + k], m, s2);
    }
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  __shared__ double red[3][kWaves];
  if (lane == 0) {
    red[0][wave] = s0;
    red[1][wave] = s1;
    red[2][wave] = s2;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int q = 0; q < kWaves; ++q) t += red[threadIdx.x][q];
    part[threadIdx.x * gridDim.x + blockIdx.x] = t;
  }
}

// one wave per sum
__global__ __launch_bounds__(192) void k_traces_sum(const double *__restrict__ part, int G,
                                                    double *__restrict__ out3) {
  const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double v = 0.0;
#pragma unroll 4
  for (int g = lane; g < G; g += 64) v += part[t * G + g];
  v = wave_sum(v);
  if (lane == 0) out3[t] = v;
}

hipError_t launch_traces(const double *moments, const double *w, const double *coef, int64_t p,
                         int sp, double *part, double *out3, hipStream_t s) {
  const int G = traces_parts(p);
  hipLaunchKernelGGL(k_traces, dim3(G), dim3(kWG), 0, s, moments, w, coef, p, sp, part);
  hipLaunchKernelGGL(k_traces_sum, dim3(1), dim3(192), 0, s, part, G, out3);
  return hipGetLastError();
}

// moments [p][sp] -> out [s][p] in tiles of 32 x 32 through LDS
__global__ __launch_bounds__(256) void k_moments_out(const double *__restrict__ mom, int64_t p, int sp, int64_t s,
                                                     double *__restrict__ out) {
  __shared__ double tile[32][33];
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const int64_t tiles = (s + 31) / 32, c0 = (int64_t)(blockIdx.x % tiles) * 32, k0 = (int64_t)(blockIdx.x / tiles) * 32;
  for (int r = y; r < 32; r += 8)
    if (k0 + r < p && c0 + x < s) tile[r][x] = mom[(k0 + r) * sp + c0 + x];
  __syncthreads();
  for (int r = y; r < 32; r += 8)
    if (c0 + r < s && k0 + x < p) out[(c0 + r) * p + k0 + x] = tile[x][r];
}

hipError_t launch_moments_out(const double *moments, int64_t p, int sp, int64_t s, double *out, hipStream_t st) {
  const int64_t blocks = (s + 31) / 32 * ((p + 31) / 32);
  if (blocks < 1 || blocks > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_moments_out, dim3((unsigned)blocks), dim3(256), 0, st, moments, p, sp, s, out);
  return hipGetLastError();
}

}  // namespace rfo
