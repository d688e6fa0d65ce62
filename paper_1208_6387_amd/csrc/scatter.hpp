// Scatter A^(s) of the column-major product results (signed Boolean assembly), FP64 or FP32 slabs.
#pragma once

#include "problem.hpp"

namespace rpf {

// Y[(mult DPN + c) ldy + j] = beta Y + sum over the multiplier's endpoints of sign (O y_loc)[c], y_loc summed
// over the K splits of its product.  A workgroup takes MB multipliers (consecutive lanes: consecutive
// boundary nodes of an interface, so a column's reads are contiguous) times CB = 256 / MB columns, and the rows
// of Y leave through LDS.  The loads of both endpoints and four splits at a time are in flight
// together: bound by their latency, so one thread per multiplier and column (a thread that walked
// the columns and splits of its multiplier took 45 us at 25,360 multipliers, 8 columns and 8 splits).
// CB is the least power of two that holds the columns, up to 8, so that no thread repeats a column.
template <int DPN, int CB, class Loc>
__global__ __launch_bounds__(256) void k_scatter_cols(int n_mult, const int* ep_q, const int* ep_bn,
                                                      const int8_t* ep_pat, const int8_t* ep_sign, const int* ep_occ,
                                                      const double* rot, Loc yl, int m, double* Y, int64_t ldy,
                                                      double beta) {
  constexpr int MB = 256 / CB, U = 4;
  __shared__ double out[MB * DPN][CB + 1];
  const int tid = threadIdx.x, lm = tid & (MB - 1), lj = tid / MB;
  const int mult = blockIdx.x * MB + lm, j = blockIdx.y * CB + lj;
  const int mc = min(mult, n_mult - 1), jc = min(j, m - 1);
  double acc[DPN];
#pragma unroll
  for (int c = 0; c < DPN; ++c) acc[c] = 0.0;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int q = ep_q[2 * mc + e];
    const int p = q < 0 ? 0 : ep_pat[2 * mc + e];
    const int64_t ld = yl.ld[p], slab = yl.slab[p];
    const int nsp = q < 0 ? 0 : yl.nsplit[p], bn = q < 0 ? 0 : ep_bn[2 * mc + e];
    const bool rm = yl.by_rows(p);
    // element c of this endpoint: base[c sc]
    const auto* base = rm ? yl.base[p] + (int64_t)bn * DPN * ld + (int64_t)max(q, 0) * m + jc
                          : yl.base[p] + ((int64_t)max(q, 0) * m + jc) * ld + (int64_t)bn * DPN;
    const int64_t sc = rm ? ld : 1;
    double v[DPN];
#pragma unroll
    for (int c = 0; c < DPN; ++c) v[c] = 0.0;
    for (int z0 = 0; z0 < nsp; z0 += U) {
      double x[U][DPN];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < DPN; ++c) x[u][c] = (double)base[min(z0 + u, nsp - 1) * slab + c * sc];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < DPN; ++c)
          if (z0 + u < nsp) v[c] = z0 + u == 0 ? x[u][c] : v[c] + x[u][c];
    }
    if (q >= 0) {
      const double sg = (double)ep_sign[2 * mc + e];
      if (DPN == 3 && rot) {
        const double* O = rot + 9 * (int64_t)ep_occ[2 * mc + e];
#pragma unroll
        for (int c = 0; c < DPN; ++c)
          acc[c] += sg * (O[3 * c] * v[0] + O[3 * c + 1] * v[1 % DPN] + O[3 * c + 2] * v[2 % DPN]);
      } else {
#pragma unroll
        for (int c = 0; c < DPN; ++c) acc[c] += sg * v[c];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < DPN; ++c) out[lm * DPN + c][lj] = acc[c];
  __syncthreads();
  const int wj = tid & (CB - 1), gj = blockIdx.y * CB + wj;
#pragma unroll
  for (int u = 0; u < DPN; ++u) {
    const int lr = tid / CB + u * MB;  // 256 / CB = MB rows a pass
    const int64_t row = (int64_t)blockIdx.x * MB * DPN + lr;
    if (row < (int64_t)n_mult * DPN && gj < m) {
      double* y = Y + row * ldy + gj;
      *y = beta == 0.0 ? out[lr][wj] : out[lr][wj] + beta * *y;
    }
  }
}

template <class Loc>
void launch_scatter_cols(rpf_problem pb, const Loc& yl, int m, double* Y, int64_t ldy, double beta, hipStream_t s) {
  const double* rot = pb->has_rot ? pb->d_rot.p : nullptr;
#define RPF_SC(D, CB)                                                                                             \
  hipLaunchKernelGGL((k_scatter_cols<D, CB, Loc>), dim3((unsigned)cdiv(pb->n_mult, 256 / CB), (unsigned)cdiv(m, CB)), \
                     dim3(256), 0, s, pb->n_mult, pb->d_ep_q.p, pb->d_ep_bn.p, pb->d_ep_pat.p, pb->d_ep_sign.p,    \
                     pb->d_ep_occ.p, rot, yl, m, Y, ldy, beta)
#define RPF_SD(D)               \
  do {                          \
    if (m > 4) RPF_SC(D, 8);    \
    else if (m > 2) RPF_SC(D, 4); \
    else if (m > 1) RPF_SC(D, 2); \
    else RPF_SC(D, 1);          \
  } while (0)
  switch (pb->dpn) {
    case 1: RPF_SD(1); break;
    case 2: RPF_SD(2); break;
    default: RPF_SD(3);
  }
#undef RPF_SD
#undef RPF_SC
  RPF_LAUNCH_CHECK();
}

}  // namespace rpf
