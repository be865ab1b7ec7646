// Moment partials of a workgroup with lanes along probes (PPL per lane): the step kernels on the
// vector units and k_init.
#pragma once

#include "device_util.h"
#include "rfo_internal.h"

namespace rfo {

// Adds the four waves' partials of probe tile pt in a fixed order into the workgroup's row.
template <int PPL>
__device__ __forceinline__ void flush_tile(double (&mom)[PPL], double (*red)[64 * PPL], int wave,
                                           int lane, double *prow, int pt) {
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    red[wave][lane * PPL + q] = mom[q];
    mom[q] = 0.0;
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

// Zero this workgroup's partial row for every tile before the sweep: the tiles
// it never meets (with a stride above the units per tile it may skip some)
// must read as zero, and those it meets are overwritten by flush_tile.
template <int PPL>
__device__ __forceinline__ void zero_partials(double *prow, int n_pt, int wave, int lane) {
  if (wave != 0) return;
  for (int t = 0; t < n_pt; ++t)
#pragma unroll
    for (int q = 0; q < PPL; ++q) prow[t * (64 * PPL) + lane * PPL + q] = 0.0;
}

}  // namespace rfo
