// Dense FP64 building blocks for gfx950: MFMA GEMM (with split-K), blocked
// band-aware Cholesky, triangular solves through inverted diagonal blocks,
// small symmetric eigen-decompositions and block orthonormalisation.
//
// The Cholesky factors of a pattern's interior stiffness, of S + Z Z^T and of
// the coarse matrix G^T G (section 2 of the paper) all run through potrf; the
// flexibility product S+ W (section 3.2) and every trailing update run through
// the same MFMA GEMM.
#include "common.hpp"
#include "problem.hpp"

#include <algorithm>
#include <cmath>

namespace rpf {

// ============================================================================ GEMM
// Column-major C = alpha op(A) op(B) + beta C with v_mfma_f64_16x16x4_f64.
// The MFMA is issued with the B fragment as its first operand, so the 16x16
// accumulator holds a transposed C block: lane l, item r is C[l % 16][l / 16 + 4 r]
// (the f64 accumulator layout strides its 4 items by 4 rows), and lanes 0..15
// of one item store 16 consecutive doubles of a column of C (coalesced).
// Operand tiles are staged through LDS (k-major); the next K tile is loaded
// into registers while the current one is consumed.
// One output tile (tx, ty) of K split z, called with the same tile by every thread of the
// workgroup (consecutive tiles of the grouped kernel reuse the LDS: the barrier that opens each k
// stage orders a tile's stores after the previous tile's reads).  SHORT: each k stage is added up by itself and
// then to the tile, so that the rounding grows with the stage's length and not with K's.
template <int BM, int BN, int WGM, int WGN, bool TA, bool TB, int BK = 16, bool SHORT = false>
__device__ __forceinline__ void dgemm_tile(int64_t M, int64_t N, int64_t K, double alpha, const double* A,
                                           int64_t lda, const double* B, int64_t ldb, double beta, double* C,
                                           int64_t ldc, int lower, int64_t kchunk, double* part, int tx, int ty,
                                           int z) {
  constexpr int PAD = 2;
  constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 16, TN = WTN / 16;
  constexpr int EA = BM * BK / 256, EB = BN * BK / 256;
  static_assert(WGM * WGN == 4 && TM >= 1 && TN >= 1 && EA >= 1 && EB >= 1, "bad tile");
  __shared__ double sA[BK][BM + PAD];
  __shared__ double sB[BK][BN + PAD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int64_t m0 = (int64_t)tx * BM, n0 = (int64_t)ty * BN;
  if (lower && n0 >= m0 + BM) return;  // tile strictly above the diagonal
  const int64_t kbeg = (int64_t)z * kchunk;
  const int64_t kend = K < kbeg + kchunk ? K : kbeg + kchunk;

  v4d acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  v4d sum[SHORT ? TM : 1][SHORT ? TN : 1];
  if constexpr (SHORT) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) sum[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  }

  double ra[EA], rb[EB];
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int idx = tid + e * 256;
      const int mm = TA ? idx / BK : idx % BM;
      const int kk = TA ? idx % BK : idx / BM;
      const int64_t gm = m0 + mm, gk = k0 + kk;
      ra[e] = (gm < M && gk < kend) ? (TA ? A[gm * lda + gk] : A[gk * lda + gm]) : 0.0;
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int idx = tid + e * 256;
      const int nn = TB ? idx % BN : idx / BK;
      const int kk = TB ? idx / BN : idx % BK;
      const int64_t gn = n0 + nn, gk = k0 + kk;
      rb[e] = (gn < N && gk < kend) ? (TB ? B[gk * ldb + gn] : B[gn * ldb + gk]) : 0.0;
    }
  };
  auto sstore = [&]() {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int idx = tid + e * 256;
      const int mm = TA ? idx / BK : idx % BM;
      const int kk = TA ? idx % BK : idx / BM;
      sA[kk][mm] = ra[e];
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int idx = tid + e * 256;
      const int nn = TB ? idx % BN : idx / BK;
      const int kk = TB ? idx / BN : idx % BK;
      sB[kk][nn] = rb[e];
    }
  };

  if (kbeg < kend) gload(kbeg);
  for (int64_t k0 = kbeg; k0 < kend; k0 += BK) {
    __syncthreads();
    sstore();
    __syncthreads();
    if (k0 + BK < kend) gload(k0 + BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = sA[kk + (lane >> 4)][wm * WTM + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = sB[kk + (lane >> 4)][wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(bf[j], af[i], acc[i][j], 0, 0, 0);
    }
    if constexpr (SHORT) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = k0 + BK < kend ? v4d{0.0, 0.0, 0.0, 0.0} : sum[i][j];
        }
    }
  }

#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm * WTM + i * 16 + (lane & 15);
        const int64_t n = n0 + wn * WTN + j * 16 + (lane >> 4) + 4 * r;
        if (m < M && n < N && (!lower || m >= n)) {
          const double v = alpha * acc[i][j][r];
          if (part) {
            part[((int64_t)z * N + n) * M + m] = v;
          } else {
            double* c = C + n * ldc + m;
            *c = (beta == 0.0) ? v : v + beta * *c;
          }
        }
      }
}

template <int BM, int BN, int WGM, int WGN, bool TA, bool TB, int BK = 16>
__global__ __launch_bounds__(256) void k_dgemm(int64_t M, int64_t N, int64_t K, double alpha,
                                               const double* A, int64_t lda, const double* B,
                                               int64_t ldb, double beta, double* C, int64_t ldc,
                                               int lower, int64_t kchunk, double* part) {
  int tx, ty;
  xcd_tile(gridDim.x, gridDim.y, tx, ty);
  dgemm_tile<BM, BN, WGM, WGN, TA, TB, BK>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, lower, kchunk, part, tx, ty,
                                       blockIdx.z);
}

// Every pattern's FP64 flexibility product in one persistent launch (see k_gemm_bf16_group):
// C_p = A_p B_p into split-K slabs part_p (M x N each, column-major).
template <int BM, int BN>
__global__ __launch_bounds__(256) void k_dgemm_group(const DGroup g) {
  for (int t = blockIdx.x; t < g.start[g.n]; t += gridDim.x) {
    int p = 0;
    while (t >= g.start[p + 1]) ++p;
    const int l = t - g.start[p];
    const int per_z = g.tm[p] * g.tn[p];
    const int z = l / per_z, r = l - z * per_z;
    dgemm_tile<BM, BN, 2, 2, false, false>(g.M[p], g.N[p], g.K[p], 1.0, g.A[p], g.lda[p], g.B[p], g.ldb[p], 0.0,
                                           nullptr, 0, 0, g.kchunk[p], g.part[p], r % g.tm[p], r / g.tm[p], z);
  }
}

// FP64 C = alpha A B (+ beta C), column-major; A: M x K with lda, B: K x N with ldb, its k-contiguous
// columns padded with zeros to a multiple of 32; M and lda even (16-byte loads of A).  The
// flexibility product's large-problem kernel: 128 x 128 tiles, eight waves of 64 x 32 (two per
// SIMD, so one wave's LDS waits overlap the other's MFMAs), 32-k stages loaded straight into two
// LDS buffers, the next stage issued right after the barrier that opens the current one (a whole
// stage of MFMA work covers the load latency).  Same per-accumulator summation order as k_dgemm,
// so the same bits.  A stage: A as 32 k-rows of 128 doubles (+16 pad: the two k-rows a
// half-wave reads sit on opposite bank halves); B as 128 n-rows of 32 doubles with 16-byte chunk
// kc stored at kc ^ (n % 16) (conflict-free fragment reads).  Rows past M or N are clamped to the
// last row (their results are never stored); k-rows of A past K are clamped too and meet the
// zero padding of B.
template <bool BETA>
__global__ __launch_bounds__(512) void k_dgemm_big(int M, int N, int K, double alpha, const double* __restrict__ A,
                                                   int64_t lda, const double* __restrict__ B, int64_t ldb, double beta,
                                                   double* __restrict__ C, int64_t ldc, int lower, int kchunk,
                                                   int64_t slab) {
  // K split z: its columns of A and rows of B, into a slab of its own (kchunk a multiple of the stage)
  {
    const int k0 = (int)blockIdx.z * kchunk;
    K = min(K - k0, kchunk);
    A += (int64_t)k0 * lda;
    B += k0;
    C += (int64_t)blockIdx.z * slab;
  }
  constexpr int BK = 32, RA = 128 + 16, SA = BK * RA, SB = 128 * BK;
  __shared__ __attribute__((aligned(1024))) double lA0[SA];
  __shared__ __attribute__((aligned(1024))) double lA1[SA];
  __shared__ __attribute__((aligned(1024))) double lB0[SB];
  __shared__ __attribute__((aligned(1024))) double lB1[SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;  // wave tile 64 (m) x 32 (n)
  int tx, ty;
  xcd_tile(gridDim.x, gridDim.y, tx, ty);
  const int m0 = tx * 128, n0 = ty * 128;
  // lower: only tiles that reach the lower triangle (n <= m somewhere) are computed
  if (lower && n0 > m0 + 127) return;
  const int nst = (K + BK - 1) / BK;
  // loads of a stage: wave w takes A k-rows 4w .. 4w + 3 (lane l: doubles m0 + 2l, 2l + 1) and
  // B blocks 4w .. 4w + 3 of four n-rows (lane l: n-row l / 16, chunk (l % 16) ^ (n % 16))
  const int am = min(m0 + 2 * lane, M - 2);
  const double* asrc = A + am;
  const double* bsrc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int nl = 4 * (4 * wave + e) + (lane >> 4);
    const int n = min(n0 + nl, N - 1);
    const int kc = (lane & 15) ^ (nl & 15);
    bsrc[e] = B + (int64_t)n * ldb + 2 * kc;
  }
  auto issue = [&](double* la, double* lb, int k0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int kr = 4 * wave + e;
      const int k = min(k0 + kr, K - 1);  // k past K: finite A values times zero B padding
      __builtin_amdgcn_global_load_lds((const void*)(asrc + (int64_t)k * lda), (void*)(la + kr * RA), 16, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      __builtin_amdgcn_global_load_lds((const void*)(bsrc[e] + k0), (void*)(lb + (4 * wave + e) * 128), 16, 0, 0);
  };
  v4d acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  const int fl = lane & 15, fk = lane >> 4;
  auto stage = [&](const double* la, const double* lb, double* na, double* nb, int s) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (s + 1 < nst) issue(na, nb, (s + 1) * BK);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int k = kk + fk;
      double af[4], bf[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) af[i] = la[k * RA + wm * 64 + i * 16 + fl];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = wn * 32 + j * 16 + fl;
        bf[j] = lb[n * BK + (((k >> 1) ^ (n & 15)) << 1) + (k & 1)];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(bf[j], af[i], acc[i][j], 0, 0, 0);
    }
  };
  if (nst > 0) issue(lA0, lB0, 0);
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    stage(lA0, lB0, lA1, lB1, s);
    stage(lA1, lB1, lA0, lB0, s + 1);
  }
  if (s < nst) stage(lA0, lB0, lA1, lB1, s);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm * 64 + i * 16 + fl;
        const int n = n0 + wn * 32 + j * 16 + fk + 4 * r;
        if (m < M && n < N) {
          double* c = C + (int64_t)n * ldc + m;
          const double v = alpha * acc[i][j][r];
          *c = BETA ? v + beta * *c : v;
        }
      }
}


static bool flex_shape(int64_t M, int64_t N, int64_t K, const double* A, int64_t lda, const double* B, int64_t ldb) {
  return M >= 2 && N >= 1 && K >= 1 && !(M & 1) && !(lda & 1) && ldb % 32 == 0 && K <= ldb && M <= INT32_MAX &&
         N <= INT32_MAX && K <= INT32_MAX && !((uintptr_t)A & 15) && !((uintptr_t)B & 15);
}

bool dgemm_flex(hipStream_t s, int64_t M, int64_t N, int64_t K, double alpha, const double* A, int64_t lda,
                const double* B, int64_t ldb, double beta, double* C, int64_t ldc, bool lower) {
  if (!flex_shape(M, N, K, A, lda, B, ldb)) return false;
  const dim3 grid((unsigned)cdiv(M, 128), (unsigned)cdiv(N, 128));
  const int kc = (int)(cdiv(K, 32) * 32);
  if (beta == 0.0)
    RPF_TIMED_LAUNCH((k_dgemm_big<false>), grid, dim3(512), 0, s, (int)M, (int)N, (int)K, alpha, A, lda, B, ldb, beta,
                     C, ldc, lower ? 1 : 0, kc, (int64_t)0);
  else
    RPF_TIMED_LAUNCH((k_dgemm_big<true>), grid, dim3(512), 0, s, (int)M, (int)N, (int)K, alpha, A, lda, B, ldb, beta,
                     C, ldc, lower ? 1 : 0, kc, (int64_t)0);
  RPF_LAUNCH_CHECK();
  return true;
}

bool dgemm_flex_partials(hipStream_t s, int64_t M, int64_t N, int64_t K, const double* A, int64_t lda, const double* B,
                         int64_t ldb, double* part, int64_t kchunk) {
  if (!flex_shape(M, N, K, A, lda, B, ldb) || kchunk < 32 || kchunk % 32) return false;
  RPF_TIMED_LAUNCH((k_dgemm_big<false>), dim3((unsigned)cdiv(M, 128), (unsigned)cdiv(N, 128), (unsigned)cdiv(K, kchunk)),
                   dim3(512), 0, s, (int)M, (int)N, (int)K, 1.0, A, lda, B, ldb, 0.0, part, M, 0, (int)kchunk, M * N);
  RPF_LAUNCH_CHECK();
  return true;
}

// Sum of the split-K partials: one wavefront per output, lanes stride over the
// splits (fixed order, so the result is deterministic).
// Few slabs, many outputs: one thread per output, slabs summed in order (coalesced over outputs).
__global__ __launch_bounds__(256) void k_splitk_reduce_thread(int64_t M, int64_t N, int splits, const double* part,
                                                              double beta, double* C, int64_t ldc) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t MN = M * N;
  if (idx >= MN) return;
  double s = 0.0;
  for (int z = 0; z < splits; ++z) s += part[(int64_t)z * MN + idx];
  const int64_t m = idx % M, n = idx / M;
  double* c = C + n * ldc + m;
  *c = (beta == 0.0) ? s : s + beta * *c;
}

// Sum of the split partial slabs: a workgroup covers 16 consecutive outputs (lane & 15, so each
// slab row read is 128 contiguous bytes) and its 16 thread rows take every 16th slab, eight loads
// in flight at clamped (always valid) slabs; the 16 row sums are then added in LDS in a fixed
// order.  C = sum (+ beta C), M x N column-major with leading dimension ldc.
__global__ __launch_bounds__(256) void k_splitk_reduce(int64_t M, int64_t N, int splits, const double* part,
                                                       double beta, double* C, int64_t ldc) {
  __shared__ double red[16][17];
  const int tx = threadIdx.x & 15, tz = threadIdx.x >> 4;
  const int64_t MN = M * N;
  const int64_t idx = (int64_t)blockIdx.x * 16 + tx;
  const int64_t ic = min(idx, MN - 1);
  double sum = 0.0;
  constexpr int U = 8;
  for (int z0 = tz; z0 < splits; z0 += 16 * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = part[(int64_t)min(z0 + 16 * u, splits - 1) * MN + ic];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (z0 + 16 * u < splits) sum += v[u];
  }
  red[tz][tx] = sum;
  __syncthreads();
  if (tz == 0 && idx < MN) {
    double t = 0.0;
#pragma unroll
    for (int z = 0; z < 16; ++z) t += red[z][tx];
    const int64_t m = idx % M, n = idx / M;
    double* c = C + n * ldc + m;
    *c = (beta == 0.0) ? t : t + beta * *c;
  }
}

namespace {
enum Cfg { BIG, M16, N16, SMALL };

Cfg pick_cfg(int64_t M, int64_t N) {
  if (M <= 16) return M16;
  if (N <= 16) return N16;
  if (M <= 64 && N <= 64) return SMALL;
  // 256 CUs: fall back to 64x64 tiles when 128x128 tiles cannot give two per CU
  if (cdiv(M, 128) * cdiv(N, 128) < 512) return SMALL;
  return BIG;
}

void tile_of(Cfg c, int& bm, int& bn) {
  switch (c) {
    case BIG: bm = 128; bn = 128; break;
    case M16: bm = 16; bn = 256; break;
    case N16: bm = 256; bn = 16; break;
    default: bm = 64; bn = 64; break;
  }
}

template <bool TA, bool TB>
void launch_cfg(Cfg c, dim3 grid, hipStream_t s, int64_t M, int64_t N, int64_t K, double alpha,
                const double* A, int64_t lda, const double* B, int64_t ldb, double beta, double* C,
                int64_t ldc, int lower, int64_t kchunk, double* part) {
  switch (c) {
    case BIG:
      RPF_TIMED_LAUNCH((k_dgemm<128, 128, 2, 2, TA, TB>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B,
                         ldb, beta, C, ldc, lower, kchunk, part);
      break;
    case M16:
      RPF_TIMED_LAUNCH((k_dgemm<16, 256, 1, 4, TA, TB>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B,
                         ldb, beta, C, ldc, lower, kchunk, part);
      break;
    case N16:
      RPF_TIMED_LAUNCH((k_dgemm<256, 16, 4, 1, TA, TB>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B,
                         ldb, beta, C, ldc, lower, kchunk, part);
      break;
    default:
      RPF_TIMED_LAUNCH((k_dgemm<64, 64, 2, 2, TA, TB>), grid, dim3(256), 0, s, M, N, K, alpha, A, lda, B,
                         ldb, beta, C, ldc, lower, kchunk, part);
      break;
  }
}

void launch_gemm(hipStream_t s, bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha,
                 const double* A, int64_t lda, const double* B, int64_t ldb, double beta, double* C,
                 int64_t ldc, bool lower, int splits, double* part) {
  const Cfg c = pick_cfg(M, N);
  int bm, bn;
  tile_of(c, bm, bn);
  int64_t kchunk = K;
  if (splits > 1) kchunk = cdiv(cdiv(K, splits), 16) * 16;
  const int64_t gz = splits > 1 ? cdiv(K, kchunk) : 1;
  RPF_CHECK(cdiv(N, bn) <= 65535 && gz <= 65535, RPF_EINVAL, "dgemm: grid too large");
  dim3 grid((unsigned)cdiv(M, bm), (unsigned)cdiv(N, bn), (unsigned)gz);
  const int low = lower ? 1 : 0;
  if (!ta && !tb) launch_cfg<false, false>(c, grid, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, low, kchunk, part);
  else if (!ta && tb) launch_cfg<false, true>(c, grid, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, low, kchunk, part);
  else if (ta && !tb) launch_cfg<true, false>(c, grid, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, low, kchunk, part);
  else launch_cfg<true, true>(c, grid, s, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, low, kchunk, part);
  RPF_LAUNCH_CHECK();
}
}  // namespace

void dgemm(hipStream_t s, bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha, const double* A,
           int64_t lda, const double* B, int64_t ldb, double beta, double* C, int64_t ldc, bool lower) {
  if (M <= 0 || N <= 0) return;
  if (K <= 0 && beta == 1.0) return;  // nothing to add; K = 0 otherwise scales C by beta
  launch_gemm(s, ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, lower, 1, nullptr);
}

// resident workgroups of a kernel on the whole device (occupancy times compute units), cached
template <typename Kern>
static int resident_blocks(Kern k, int threads) {
  int per_cu = 0, dev = 0;
  RPF_HIP(hipGetDevice(&dev));
  RPF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, threads, 0));
  hipDeviceProp_t prop;
  RPF_HIP(hipGetDeviceProperties(&prop, dev));
  return std::max(1, per_cu) * std::max(1, prop.multiProcessorCount);
}

void dgemm_group(hipStream_t s, int tile, const DGroup& g) {
  const int total = g.start[g.n];
  if (total == 0) return;
  if (tile == 128) {
    static const int cap = resident_blocks(k_dgemm_group<128, 128>, 256);
    RPF_TIMED_LAUNCH((k_dgemm_group<128, 128>), dim3((unsigned)std::min(total, cap)), dim3(256), 0, s, g);
  } else {
    RPF_CHECK(tile == 64, RPF_EINVAL, "dgemm_group: tile must be 64 or 128");
    static const int cap = resident_blocks(k_dgemm_group<64, 64>, 256);
    RPF_TIMED_LAUNCH((k_dgemm_group<64, 64>), dim3((unsigned)std::min(total, cap)), dim3(256), 0, s, g);
  }
  RPF_LAUNCH_CHECK();
}

int gemm_tiles(int64_t M, int64_t N) {
  const Cfg c = pick_cfg(M, N);
  int bm, bn;
  tile_of(c, bm, bn);
  return (int)(cdiv(M, bm) * cdiv(N, bn));
}

void dgemm_partials(hipStream_t s, int64_t M, int64_t N, int64_t K, const double* A, int64_t lda, const double* B,
                    int64_t ldb, double* part, int splits) {
  if (M <= 0 || N <= 0) return;
  launch_gemm(s, false, false, M, N, K, 1.0, A, lda, B, ldb, 0.0, nullptr, 0, false, splits, part);
}

int gemm_splitk_count(int64_t M, int64_t N, int64_t K) {
  const Cfg c = pick_cfg(M, N);
  int bm, bn;
  tile_of(c, bm, bn);
  const int64_t tiles = cdiv(M, bm) * cdiv(N, bn);
  int64_t sp = cdiv(1024, tiles);
  sp = std::min<int64_t>(sp, std::max<int64_t>(1, K / 256));
  sp = std::max<int64_t>(1, std::min<int64_t>(sp, 1024));
  return (int)sp;
}

void dgemm_splitk(hipStream_t s, bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha,
                  const double* A, int64_t lda, const double* B, int64_t ldb, double beta, double* C,
                  int64_t ldc, double* ws, int splits) {
  if (M <= 0 || N <= 0) return;
  if (splits <= 1 || K <= 0) {
    dgemm(s, ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, false);
    return;
  }
  const int64_t kchunk = cdiv(cdiv(K, splits), 16) * 16;
  const int gz = (int)cdiv(K, kchunk);
  launch_gemm(s, ta, tb, M, N, K, alpha, A, lda, B, ldb, 0.0, nullptr, 0, false, splits, ws);
  if (gz <= 32)
    hipLaunchKernelGGL(k_splitk_reduce_thread, dim3((unsigned)cdiv(M * N, 256)), dim3(256), 0, s, M, N, gz, ws, beta,
                       C, ldc);
  else
    hipLaunchKernelGGL(k_splitk_reduce, dim3((unsigned)cdiv(M * N, 16)), dim3(256), 0, s, M, N, gz, ws, beta, C,
                       ldc);
  RPF_LAUNCH_CHECK();
}

// ============================================================================ tall-skinny Gram
// Partial C (a x b) = X^T Y over a chunk of rows, X and Y row-major (N x a, N x b).
// Workgroup (tile, chunk): tile = (ti, tj) 16 x 16 block of C; each wave takes 4
// rows per v_mfma_f64_16x16x4_f64 (the k dimension of the MFMA runs over rows),
// the 4 waves are summed in LDS and the partial goes to part[chunk][j][i].
__global__ __launch_bounds__(256) void k_gram_partial(int64_t N, int a, int b, const double* X, int64_t ldx,
                                                      const double* Y, int64_t ldy, int64_t chunk, double* part) {
  __shared__ double red[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ta = (a + 15) / 16;
  const int i0 = (blockIdx.x % ta) * 16, j0 = (blockIdx.x / ta) * 16;
  const int64_t r_beg = (int64_t)blockIdx.y * chunk;
  const int64_t r_end = min(N, r_beg + chunk);
  const int i = i0 + (lane & 15), j = j0 + (lane & 15);
  const bool iok = i < a, jok = j < b;
  v4d acc = {0.0, 0.0, 0.0, 0.0};
  // four row groups in flight per wave (loads issued before the MFMAs consume them)
  for (int64_t r0 = r_beg + 4 * wave; r0 < r_end; r0 += 64) {
    double xa[4], yb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t row = r0 + 16 * u + (lane >> 4);
      const bool rok = row < r_end;
      xa[u] = (rok && iok) ? X[row * ldx + i] : 0.0;
      yb[u] = (rok && jok) ? Y[row * ldy + j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u], yb[u], acc, 0, 0, 0);
  }
  // accumulator item r of lane l is C[i0 + l/16 + 4r][j0 + l%16]
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][((lane >> 4) + 4 * r) * 16 + (lane & 15)] = acc[r];
  __syncthreads();
  const int t = threadIdx.x;
  const int ci = i0 + t / 16, cj = j0 + t % 16;
  if (ci < a && cj < b)
    part[((int64_t)blockIdx.y * b + cj) * a + ci] = red[0][t] + red[1][t] + red[2][t] + red[3][t];
}

// Pair form: C = X^T [Y1 | Y2] for a <= 16 and b1, b2 <= 16, each workgroup computing both
// 16 x 16 tiles from one read of X (the two Grams of a block step share their left operand).
// part[chunk] holds a x (b1 + b2), column-major.
__global__ __launch_bounds__(256) void k_gram_pair(int64_t N, int a, const double* X, int64_t ldx, int b1,
                                                   const double* Y1, int64_t ldy1, int b2, const double* Y2,
                                                   int64_t ldy2, int64_t chunk, double* part) {
  __shared__ double red[4][2][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r_beg = (int64_t)blockIdx.x * chunk;
  const int64_t r_end = min(N, r_beg + chunk);
  const int i = lane & 15, j = lane & 15;
  const bool iok = i < a, j1 = j < b1, j2 = j < b2;
  v4d acc1 = {0.0, 0.0, 0.0, 0.0}, acc2 = {0.0, 0.0, 0.0, 0.0};
  if (b1 > 0 && b2 > 0 && r_end > r_beg) {
    // loads at clamped (always valid) rows and columns, masked afterwards, and the next group's
    // loads issued before this group's MFMAs: no load behind a branch, two groups in flight
    const int ic = min(i, a - 1), jc1 = min(j, b1 - 1), jc2 = min(j, b2 - 1);
    double xa[4], y1[4], y2[4], nx[4], n1[4], n2[4];
    auto load = [&](int64_t r0, double* x, double* p1, double* p2) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t row = min(r0 + 16 * u + (lane >> 4), r_end - 1);
        x[u] = X[row * ldx + ic];
        p1[u] = Y1[row * ldy1 + jc1];
        p2[u] = Y2[row * ldy2 + jc2];
      }
    };
    auto mma = [&](int64_t r0, const double* x, const double* p1, const double* p2) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool rok = r0 + 16 * u + (lane >> 4) < r_end;
        const double xv = (rok && iok) ? x[u] : 0.0;
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, (rok && j1) ? p1[u] : 0.0, acc1, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, (rok && j2) ? p2[u] : 0.0, acc2, 0, 0, 0);
      }
    };
    // two register sets in turn (no copies): the loads of one group are in flight while the
    // MFMAs of the other run; a prefetch past the last group reads the clamped last row
    int64_t r0 = r_beg + 4 * wave;
    load(r0, xa, y1, y2);
    for (; r0 < r_end; r0 += 128) {
      load(r0 + 64, nx, n1, n2);
      mma(r0, xa, y1, y2);
      if (r0 + 64 >= r_end) break;
      load(r0 + 128, xa, y1, y2);
      mma(r0 + 64, nx, n1, n2);
    }
  } else {
    for (int64_t r0 = r_beg + 4 * wave; r0 < r_end; r0 += 64) {
      double xa[4], y1[4], y2[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t row = r0 + 16 * u + (lane >> 4);
        const bool rok = row < r_end;
        xa[u] = (rok && iok) ? X[row * ldx + i] : 0.0;
        y1[u] = (rok && j1) ? Y1[row * ldy1 + j] : 0.0;
        y2[u] = (rok && j2) ? Y2[row * ldy2 + j] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u], y1[u], acc1, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[u], y2[u], acc2, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[wave][0][((lane >> 4) + 4 * r) * 16 + (lane & 15)] = acc1[r];
    red[wave][1][((lane >> 4) + 4 * r) * 16 + (lane & 15)] = acc2[r];
  }
  __syncthreads();
  const int t = threadIdx.x;
  const int ci = t / 16, cj = t % 16;
  const int bt = b1 + b2;
  double* pc = part + (int64_t)blockIdx.x * a * bt;
  if (ci < a && cj < b1) pc[(int64_t)cj * a + ci] = red[0][0][t] + red[1][0][t] + red[2][0][t] + red[3][0][t];
  if (ci < a && cj < b2) pc[(int64_t)(b1 + cj) * a + ci] = red[0][1][t] + red[1][1][t] + red[2][1][t] + red[3][1][t];
}

// Wide form (X with many columns, e.g. all stored search directions).  The a columns are split
// into ga groups of at most 32 column tiles, spread evenly; a workgroup covers one group against
// one 16-column tile of Y over a chunk of rows.  Its four waves are WT tile slices (TW tiles each)
// times 4/WT row slices: few tiles are split over rows instead of leaving waves idle, and each Y
// fragment feeds TW MFMAs.  The row slices' sums are added in LDS before the partial is written.
// With more than 4 tiles (a > 64), TW is 5 to 8.
struct WideShape {
  int ga, wt, tw;
};
static WideShape wide_shape(int a) {
  const int ta = (a + 15) / 16;
  const int ga = (ta + 31) / 32;
  const int tg = (ta + ga - 1) / ga;
  const int wt = tg <= 8 ? 1 : (tg <= 16 ? 2 : 4);
  return {ga, wt, (tg + wt - 1) / wt};
}

template <int TW>
__global__ __launch_bounds__(256) void k_gram_wide(int64_t N, int a, int b, const double* X, int64_t ldx,
                                                   const double* Y, int64_t ldy, int64_t chunk, int ga, int wt,
                                                   double* part) {
  __shared__ double red[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr_n = 4 / wt, wslice = wave % wt, wrow = wave / wt;
  const int grp = blockIdx.x % ga, tj = blockIdx.x / ga;
  const int ta = (a + 15) / 16, tg = (ta + ga - 1) / ga;
  const int tbase = grp * tg + wslice * TW;
  const int tend = min(ta, (grp + 1) * tg);
  const int j = tj * 16 + (lane & 15);
  const bool jok = j < b;
  const int64_t r_beg = (int64_t)blockIdx.y * chunk;
  const int64_t r_end = min(N, r_beg + chunk);
  v4d acc[TW];
#pragma unroll
  for (int t = 0; t < TW; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
  if (r_end > r_beg) {
    // loads at clamped (always valid) rows and columns, masked before the MFMAs, and the next
    // group of 8 rows loaded while this group's MFMAs run (two register sets in turn)
    const int jc = min(j, b - 1);
    int ic[TW];
    bool iok[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      const int i = (tbase + t) * 16 + (lane & 15);
      ic[t] = min(i, a - 1);
      iok[t] = tbase + t < tend && i < a;
    }
    double yb[2], xa[2][TW], ny[2], nx[2][TW];
    auto load = [&](int64_t r0, double* y, double (*x)[TW]) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int64_t row = min(r0 + 4 * u + (lane >> 4), r_end - 1);
        y[u] = Y[row * ldy + jc];
#pragma unroll
        for (int t = 0; t < TW; ++t) x[u][t] = X[row * ldx + ic[t]];
      }
    };
    auto mma = [&](int64_t r0, const double* y, const double (*x)[TW]) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bool rok = r0 + 4 * u + (lane >> 4) < r_end;
        const double yv = (rok && jok) ? y[u] : 0.0;
#pragma unroll
        for (int t = 0; t < TW; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((rok && iok[t]) ? x[u][t] : 0.0, yv, acc[t], 0, 0, 0);
      }
    };
    // this wave's row slice: groups of 8 rows r_beg + 8 (wrow + wr_n q), q = 0, 1, ...
    const int64_t step = 8 * (int64_t)wr_n;
    int64_t r0 = r_beg + 8 * wrow;
    if (r0 < r_end) {
      load(r0, yb, xa);
      for (; r0 < r_end; r0 += 2 * step) {
        load(r0 + step, ny, nx);
        mma(r0, yb, xa);
        if (r0 + step >= r_end) break;
        load(r0 + 2 * step, yb, xa);
        mma(r0 + step, ny, nx);
      }
    }
  }
  double* pc = part + (int64_t)blockIdx.y * a * b;
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    if (wr_n > 1) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][64 * r + lane] = acc[t][r];
      __syncthreads();
      if (wrow == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double v = red[wave][64 * r + lane];
          for (int q = 1; q < wr_n; ++q) v += red[wave + wt * q][64 * r + lane];
          acc[t][r] = v;
        }
      }
    }
    if (wrow == 0 && tbase + t < tend) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ci = (tbase + t) * 16 + (lane >> 4) + 4 * r, cj = tj * 16 + (lane & 15);
        if (ci < a && cj < b) pc[(int64_t)cj * a + ci] = acc[t][r];
      }
    }
  }
}

static bool gram_is_wide(int a) { return a > 64; }

int gram_chunks(int64_t N, int a, int b) {
  // about one to two workgroups per CU in total for the narrow form and about four for the wide
  // one, at least 256 rows per chunk
  const int64_t tiles = gram_is_wide(a) ? (int64_t)wide_shape(a).ga * cdiv(b, 16) : cdiv(a, 16) * cdiv(b, 16);
  int64_t g = cdiv(gram_is_wide(a) ? 1024 : 256, tiles);
  g = std::min<int64_t>(g, std::max<int64_t>(1, cdiv(N, 256)));
  return (int)std::max<int64_t>(1, std::min<int64_t>(g, 2048));
}

void gram(hipStream_t s, int64_t N, int a, int b, const double* X, int64_t ldx, const double* Y, int64_t ldy,
          double* C, double* ws) {
  if (a <= 0 || b <= 0) return;
  const int g = gram_chunks(N, a, b);
  const int64_t chunk = cdiv(N, g);
  const int gz = (int)cdiv(N, chunk);
  RPF_CHECK(gz <= 65535, RPF_EINVAL, "gram: too many chunks");
  double* part = gz == 1 ? C : ws;  // a single chunk's partial sums are the result
  if (gram_is_wide(a)) {
    const WideShape w = wide_shape(a);
    const dim3 grid((unsigned)(w.ga * cdiv(b, 16)), (unsigned)gz);
    switch (w.tw) {
#define RPF_WIDE(TW)                                                                                         \
  case TW:                                                                                                   \
    hipLaunchKernelGGL(k_gram_wide<TW>, grid, dim3(256), 0, s, N, a, b, X, ldx, Y, ldy, chunk, w.ga, w.wt, part); \
    break;
      RPF_WIDE(5) RPF_WIDE(6) RPF_WIDE(7) RPF_WIDE(8)
#undef RPF_WIDE
      default:
        RPF_CHECK(false, RPF_EINVAL, "gram: unexpected wide shape");
    }
  } else {
    const int64_t tiles = cdiv(a, 16) * cdiv(b, 16);
    hipLaunchKernelGGL(k_gram_partial, dim3((unsigned)tiles, (unsigned)gz), dim3(256), 0, s, N, a, b, X, ldx, Y,
                       ldy, chunk, part);
  }
  RPF_LAUNCH_CHECK();
  if (gz == 1) return;
  hipLaunchKernelGGL(k_splitk_reduce, dim3((unsigned)cdiv((int64_t)a * b, 16)), dim3(256), 0, s, (int64_t)a,
                     (int64_t)b, gz, ws, 0.0, C, (int64_t)a);
  RPF_LAUNCH_CHECK();
}

// rows per chunk of gram_pair: four workgroups per CU, since one wave per SIMD does not keep enough
// loads in flight for this memory-bound pass (the partial sums are still reduced in a fixed order)
static int64_t gram_pair_rows(int64_t N) {
  return cdiv(N, std::min<int64_t>(1024, std::max<int64_t>(1, cdiv(N, 256))));
}
int gram_pair_chunks(int64_t N) { return (int)cdiv(N, gram_pair_rows(N)); }

void gram_pair(hipStream_t s, int64_t N, int a, const double* X, int64_t ldx, int b1, const double* Y1,
               int64_t ldy1, int b2, const double* Y2, int64_t ldy2, double* C, double* ws) {
  if (a <= 0 || b1 + b2 <= 0) return;
  if (a > 16 || b1 > 16 || b2 > 16) {
    gram(s, N, a, b1, X, ldx, Y1, ldy1, C, ws);
    gram(s, N, a, b2, X, ldx, Y2, ldy2, C + (int64_t)a * b1, ws);
    return;
  }
  const int64_t chunk = gram_pair_rows(N);
  const int gz = gram_pair_chunks(N);
  // a single chunk's partial sums are the result
  hipLaunchKernelGGL(k_gram_pair, dim3((unsigned)gz), dim3(256), 0, s, N, a, X, ldx, b1, Y1, ldy1, b2, Y2, ldy2,
                     chunk, gz == 1 ? C : ws);
  RPF_LAUNCH_CHECK();
  if (gz == 1) return;
  hipLaunchKernelGGL(k_splitk_reduce, dim3((unsigned)cdiv((int64_t)a * (b1 + b2), 16)), dim3(256), 0, s, (int64_t)a,
                     (int64_t)(b1 + b2), gz, ws, 0.0, C, (int64_t)a);
  RPF_LAUNCH_CHECK();
}

// ============================================================================ row-block products
// Y[l*ldy + j] = beta Y + alpha sum_i X[l*ldx + i] M[i + a*j] for N rows and a
// small a x b matrix M (column-major).  A workgroup owns 64 rows; slices of 32
// columns of X are staged through LDS with coalesced loads (consecutive lanes
// read consecutive columns of a row), M slices likewise; lane (r, q) then forms
// outputs 4q..4q+3 of row r.  Used for the block updates of the interface
// solver (rows = interface dofs, row-major blocks).
__global__ __launch_bounds__(256) void k_rows_gemm(int64_t N, int a, int b, double alpha, const double* X,
                                                   int64_t ldx, const double* Mm, int64_t mrow, double beta, double* Y,
                                                   int64_t ldy) {
  __shared__ double sx[64][33];
  __shared__ double sm[32][16];
  const int tid = threadIdx.x;
  const int r = tid & 63, q = tid >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  const int64_t row = row0 + r;
  for (int j0 = 0; j0 < b; j0 += 16) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    // each 32-column chunk of X (and of M) is loaded into registers at clamped (always valid)
    // positions one chunk ahead, while the current chunk is multiplied from LDS: no load waits
    // behind a branch, and one chunk's loads are in flight during the other's FMAs
    double xr[8], mv[2];
    auto load = [&](int i0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int idx = tid + 256 * e;
        const int ii = idx & 31, rr = idx >> 5;
        const int64_t gr = min(row0 + rr, N - 1);
        xr[e] = X[gr * ldx + min(i0 + ii, a - 1)];
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int idx = tid + 256 * e;
        const int ic = min(i0 + (idx & 31), a - 1), jc = min(j0 + (idx >> 5), b - 1);
        mv[e] = mrow > 0 ? Mm[(int64_t)ic * mrow + jc] : Mm[(int64_t)ic + (int64_t)a * jc];
      }
    };
    load(0);
    for (int i0 = 0; i0 < a; i0 += 32) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int idx = tid + 256 * e;
        const int ii = idx & 31, rr = idx >> 5;
        sx[rr][ii] = (row0 + rr < N && i0 + ii < a) ? xr[e] : 0.0;
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int idx = tid + 256 * e;
        const int ii = idx & 31, jj = idx >> 5;
        sm[ii][jj] = (i0 + ii < a && j0 + jj < b) ? mv[e] : 0.0;
      }
      __syncthreads();
      load(i0 + 32);
#pragma unroll 8
      for (int ii = 0; ii < 32; ++ii) {
        const double xv = sx[r][ii];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] += xv * sm[ii][4 * q + u];
      }
    }
    if (row < N) {
      // the old values of the four outputs are read together (clamped to a valid column)
      double yo[4] = {0.0, 0.0, 0.0, 0.0};
      if (beta != 0.0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) yo[u] = Y[row * ldy + min(j0 + 4 * q + u, b - 1)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + 4 * q + u;
        if (j < b) Y[row * ldy + j] = (beta == 0.0) ? alpha * acc[u] : beta * yo[u] + alpha * acc[u];
      }
    }
  }
}

// Same product for many rows, a long inner dimension and at most 16 columns of M (e.g. the
// orthogonalisation against all stored blocks), on FP64 MFMA 16x16x4 with X rows as the M
// dimension.  A workgroup owns 64 rows and walks X in 32-column chunks.  A chunk is loaded with
// whole 128-byte lines per row (16 lanes of 16 bytes per row, four rows per load instruction; the
// MFMA operand layout, 4 lanes per row, would split every line over two instructions, which
// measured a fifth slower) into registers one chunk ahead, at clamped (always valid) positions, and
// stored masked into one of two LDS buffers with the matching 32 rows of M; wave w then multiplies
// rows 16 w .. 16 w + 15 from LDS, two accumulators in turn.  VEC: 16-byte loads (a and ldx even,
// X aligned).
template <bool VEC>
__global__ __launch_bounds__(256) void k_rows_mfma(int64_t N, int a, int b, double alpha, const double* X,
                                                   int64_t ldx, const double* Mm, int64_t mrow, double beta, double* Y,
                                                   int64_t ldy) {
  __shared__ double sx[2][64][34];
  __shared__ double sm[2][32][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = lane & 15, q = lane >> 4;
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  // chunk staging: piece p = tid + 256 i is row p >> 4, columns k0 + 2 (p & 15) + {0, 1}; M entry
  // e = tid + 256 i is row k0 + (e >> 4), column e & 15
  double2 xr[4];
  double mr[2];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = tid + 256 * i, r = p >> 4, sg = p & 15;
      const double* xrow = X + min(row0 + r, N - 1) * ldx;
      if (VEC) {
        xr[i] = *reinterpret_cast<const double2*>(xrow + min(k0 + 2 * sg, a - 2));
      } else {
        xr[i].x = xrow[min(k0 + 2 * sg, a - 1)];
        xr[i].y = xrow[min(k0 + 2 * sg + 1, a - 1)];
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = tid + 256 * i, kk = e >> 4, j = e & 15;
      const int kc = min(k0 + kk, a - 1), jc = min(j, b - 1);
      mr[i] = mrow > 0 ? Mm[(int64_t)kc * mrow + jc] : Mm[(int64_t)kc + (int64_t)a * jc];
    }
  };
  auto sstore = [&](int buf, int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = tid + 256 * i, r = p >> 4, sg = p & 15;
      const int c = k0 + 2 * sg;
      double2 v;
      v.x = c < a ? xr[i].x : 0.0;
      v.y = c + 1 < a ? xr[i].y : 0.0;
      *reinterpret_cast<double2*>(&sx[buf][r][2 * sg]) = v;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = tid + 256 * i, kk = e >> 4, j = e & 15;
      sm[buf][kk][j] = k0 + kk < a ? mr[i] : 0.0;
    }
  };
  v4d acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};  // even and odd k-steps
  gload(0);
  sstore(0, 0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < a; k0 += 32) {
    // the next chunk's loads are in flight while this chunk is multiplied; they go into the other
    // buffer, whose last readers all passed the barrier that ended the previous chunk
    gload(k0 + 32);
#pragma unroll
    for (int st = 0; st < 8; st += 2) {
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(sx[buf][16 * wave + m][4 * st + q], sm[buf][4 * st + q][m], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(sx[buf][16 * wave + m][4 * st + 4 + q], sm[buf][4 * st + 4 + q][m], acc1,
                                                  0, 0, 0);
    }
    sstore(buf ^ 1, k0 + 32);
    __syncthreads();
    buf ^= 1;
  }
  // lane holds rows 16 w + q + 4 r, column m; the old values are read together first
  const bool jok = m < b;
  const int jc = min(m, b - 1);
  double yo[4];
  if (beta != 0.0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) yo[r] = Y[min(row0 + 16 * wave + q + 4 * r, N - 1) * ldy + jc];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t row = row0 + 16 * wave + q + 4 * r;
    const double v = acc0[r] + acc1[r];
    if (jok && row < N) Y[row * ldy + m] = (beta == 0.0) ? alpha * v : beta * yo[r] + alpha * v;
  }
}

// Same product for few rows and a long inner dimension (e.g. the coarse solve with the explicit
// inverse of G^T G): one wavefront per row, lanes stride the inner index (coalesced reads of the
// row of X), 16 output columns per pass reduced across the wavefront with shuffles.
__global__ __launch_bounds__(256) void k_rows_gemm_wave(int64_t N, int a, int b, double alpha, const double* X,
                                                        int64_t ldx, const double* Mm, int64_t mrow, double beta,
                                                        double* Y, int64_t ldy) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= N) return;
  const double* x = X + row * ldx;
  for (int j0 = 0; j0 < b; j0 += 16) {
    const int nj = min(16, b - j0);
    double acc[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) acc[u] = 0.0;
    // the 16 M entries of a step are loaded at clamped (always valid) columns and masked, so they
    // are one batch in flight instead of one load behind each column test
    for (int i = lane; i < a; i += 64) {
      const double xv = x[i];
      double mv[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int uc = min(u, nj - 1);
        mv[u] = mrow > 0 ? Mm[(int64_t)i * mrow + j0 + uc] : Mm[(int64_t)i + (int64_t)a * (j0 + uc)];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (u < nj) acc[u] += xv * mv[u];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u)
      for (int off = 32; off > 0; off >>= 1) acc[u] += __shfl_xor(acc[u], off, 64);
    if (lane < nj) {
      double v = 0.0;
#pragma unroll
      for (int u = 0; u < 16; ++u) v = (lane == u) ? acc[u] : v;
      double* y = Y + row * ldy + j0 + lane;
      *y = (beta == 0.0) ? alpha * v : beta * *y + alpha * v;
    }
  }
}

// Thin products (a <= 64 inner, b <= 16 outputs per row): one thread per row.  M is
// staged once per workgroup in LDS (read back as broadcasts); each thread streams its
// row of X with 16-byte loads and writes its row of Y the same way, so the kernel runs
// at the memory rate.  blockIdx.y selects one of up to two (X, Y) pairs sharing M.
struct RowsPair {
  const double* X;
  double* Y;
  int64_t ldx, ldy;
  double alpha, beta;
  const double* Z;  // source of the beta term (NULL: Y itself), row stride ldz
  int64_t ldz;
};
struct RowsPairs {
  RowsPair p[2];
  double* colsq;  // optional: per-workgroup column sums of squares of pair 1's output (k_rows_tile)
  double* sq;     // optional, one workgroup of rows: those sums at their place, stride ldsq, and *raised after
  int64_t ldsq;   // the b x b entries
  const double* raised;
};

__global__ __launch_bounds__(256) void k_rows_small(int64_t N, int a, int b, const double* Mm, int64_t mrow,
                                                    RowsPairs pr, int vec) {
  __shared__ double sm[64 * 16];
  {
    // staged from clamped (always valid) positions and masked, so the four loads are in flight together
    double mv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = threadIdx.x + 256 * q;
      const int ic = min(e >> 4, a - 1), jc = min(e & 15, b - 1);
      mv[q] = mrow > 0 ? Mm[(int64_t)ic * mrow + jc] : Mm[ic + (int64_t)a * jc];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = threadIdx.x + 256 * q;
      sm[e] = ((e >> 4) < a && (e & 15) < b) ? mv[q] : 0.0;
    }
  }
  __syncthreads();
  const RowsPair& P = pr.p[blockIdx.y];
  const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (row >= N) return;
  double acc[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.0;
  const double* x = P.X + row * P.ldx;
  for (int i0 = 0; i0 < a; i0 += 8) {
    double xv[8];
    if (vec && i0 + 8 <= a) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double2 t = *reinterpret_cast<const double2*>(x + i0 + 2 * u);
        xv[2 * u] = t.x;
        xv[2 * u + 1] = t.y;
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = x[min(i0 + u, a - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = (i0 + u < a) ? xv[u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double* mr = sm + (i0 + u) * 16;
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] += xv[u] * mr[j];
    }
  }
  double* y = P.Y + row * P.ldy;
  const double* z = P.Z ? P.Z + row * P.ldz : y;
  if (vec && (b & 1) == 0) {
    double2 zt[8];
    if (P.beta != 0.0) {
#pragma unroll
      for (int j = 0; j < 16; j += 2) zt[j / 2] = *reinterpret_cast<const double2*>(z + min(j, b - 2));
    }
#pragma unroll
    for (int j = 0; j < 16; j += 2) {
      if (j < b) {
        double2 o;
        if (P.beta == 0.0) {
          o.x = P.alpha * acc[j];
          o.y = P.alpha * acc[j + 1];
        } else {
          o.x = P.beta * zt[j / 2].x + P.alpha * acc[j];
          o.y = P.beta * zt[j / 2].y + P.alpha * acc[j + 1];
        }
        *reinterpret_cast<double2*>(y + j) = o;
      }
    }
  } else {
    double zv[16];
    if (P.beta != 0.0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) zv[j] = z[min(j, b - 1)];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (j < b) y[j] = (P.beta == 0.0) ? P.alpha * acc[j] : P.beta * zv[j] + P.alpha * acc[j];
  }
}

// Narrow products (a, b <= 16): 256 rows per workgroup.  The rows of X are copied into LDS with
// lane-consecutive loads (a row is a contiguous run of a doubles), each thread then forms its row
// of the product from LDS, and the result leaves through LDS with lane-consecutive stores, so
// global traffic is coalesced in both directions.  blockIdx.y selects one of the (X, Y) pairs.
__global__ __launch_bounds__(256) void k_rows_tile(int64_t N, int a, int b, const double* Mm, int64_t mrow,
                                                   RowsPairs pr) {
  __shared__ double sm[16][16];
  __shared__ double xs[256][17];
  const int tid = threadIdx.x, er = tid >> 4, ec = tid & 15;  // element (er + 16 u, ec) of the tile in pass u
  const RowsPair& P = pr.p[blockIdx.y];
  const int64_t r0 = (int64_t)blockIdx.x * 256;
  const int rows = (int)min<int64_t>(256, N - r0);
  // every load of the tile at clamped (always valid) addresses, in flight together, masked afterwards:
  // one memory latency (18 us at 76,080 x 8 with loads behind width tests)
  double t[16], zv[16];
  const int mi = min(er, a - 1), mj = min(ec, b - 1);
  const double mv = mrow > 0 ? Mm[(int64_t)mi * mrow + mj] : Mm[mi + (int64_t)a * mj];
  const double* src = P.Z ? P.Z : P.Y;
  const int64_t lds = P.Z ? P.ldz : P.ldy;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int64_t row = r0 + min(er + 16 * u, rows - 1);
    t[u] = P.X[row * P.ldx + min(ec, a - 1)];
    if (P.beta != 0.0) zv[u] = src[row * lds + mj];
  }
  sm[er][ec] = (er < a && ec < b) ? mv : 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) xs[er + 16 * u][ec] = ec < a ? t[u] : 0.0;
  __syncthreads();
  double acc[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const double xv = xs[tid][i];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] += xv * sm[i][j];
  }
  __syncthreads();  // xs is reused for the output rows
#pragma unroll
  for (int j = 0; j < 16; ++j) xs[tid][j] = acc[j];
  __syncthreads();
  // with colsq, a thread sums the squares of its column of the tile and the column sums are formed in a
  // fixed order (deterministic)
  const bool want_sq = pr.colsq != nullptr && blockIdx.y == 1;
  double myq = 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int rr = er + 16 * u;
    if (rr >= rows || ec >= b) continue;
    const double v = P.alpha * xs[rr][ec];
    const double out = (P.beta == 0.0) ? v : P.beta * zv[u] + v;
    P.Y[(r0 + rr) * P.ldy + ec] = out;
    myq += out * out;
  }
  if (want_sq) {
    __syncthreads();
    double* red = &xs[0][0];
    red[tid] = myq;
    __syncthreads();
    if (tid < b) {
      double q = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) q += red[tid + 16 * k];
      if (pr.sq) {
        pr.sq[tid * pr.ldsq] = q;
        if (tid == 0) pr.sq[b * b] = *pr.raised;
      } else {
        pr.colsq[(int64_t)blockIdx.x * b + tid] = q;
      }
    }
  }
}

// Residual update of a block step with both of its by-products from the same pass:
// Y = beta Y + alpha X M (X: N x a rows, M: a x b column-major, a, b <= 16), the per-workgroup
// column sums of squares of the new Y (sqpart[wg * b + c], fixed order, deterministic), and
// the per-workgroup Gram partial X^T Y_new (gpart[(wg * b + j) * a + i]) - the next step's
// X^T R, which would otherwise take another pass over both blocks.  The rows of X and of the new
// Y stay in LDS; the Gram partial is formed with v_mfma_f64_16x16x4_f64 (each wave four rows per
// MFMA over its 64 rows) and the four waves are summed in LDS.
__global__ __launch_bounds__(256) void k_rows_update_gram(int64_t N, int a, int b, const double* Mm,
                                                          const double* X, int64_t ldx, double alpha, double beta,
                                                          double* Y, int64_t ldy, double* part) {
  __shared__ double sm[16][16];
  __shared__ double xs[256][17];
  __shared__ double ys[256][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int er = tid >> 4, ec = tid & 15;  // element (er + 16 u, ec) of the tile in pass u
  const int64_t r0 = (int64_t)blockIdx.x * 256;
  const int rows = (int)min<int64_t>(256, N - r0);
  // every load of the tile at clamped (always valid) addresses, in flight together, masked afterwards
  double zv[16];
  {
    double t[16];
    const double mv = Mm[min(er, a - 1) + (int64_t)a * min(ec, b - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int64_t row = r0 + min(er + 16 * u, rows - 1);
      t[u] = X[row * ldx + min(ec, a - 1)];
      if (beta != 0.0) zv[u] = Y[row * ldy + min(ec, b - 1)];
    }
    sm[er][ec] = (er < a && ec < b) ? mv : 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) xs[er + 16 * u][ec] = (er + 16 * u < rows && ec < a) ? t[u] : 0.0;
  }
  __syncthreads();
  {
    double acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const double xv = xs[tid][i];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] += xv * sm[i][j];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) ys[tid][j] = acc[j];
  }
  __syncthreads();
  double myq = 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int rr = er + 16 * u;
    const double v = alpha * ys[rr][ec];
    const bool in = rr < rows && ec < b;  // the rest counts as zero in the Gram
    const double out = in ? ((beta == 0.0) ? v : beta * zv[u] + v) : 0.0;
    if (in) Y[(r0 + rr) * ldy + ec] = out;
    ys[rr][ec] = out;
    myq += out * out;
  }
  __syncthreads();
  // Gram partial over this tile's rows: wave w takes rows 64 w .. 64 w + 63
  v4d g = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int row = wave * 64 + 4 * q + (lane >> 4);
    g = __builtin_amdgcn_mfma_f64_16x16x4f64(xs[row][lane & 15], ys[row][lane & 15], g, 0, 0, 0);
  }
  __syncthreads();  // xs becomes the reduction buffer
  double* red = &xs[0][0];
  // accumulator item r of lane l is (i = l / 16 + 4 r, j = l % 16)
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave * 256 + ((lane >> 4) + 4 * r) * 16 + (lane & 15)] = g[r];
  red[1024 + tid] = myq;
  __syncthreads();
  // record: the Gram (a x b, column-major), then the squared norms of the b columns
  double* rec = part + (int64_t)blockIdx.x * (a * b + b);
  if (er < a && ec < b) rec[ec * a + er] = red[tid] + red[256 + tid] + red[512 + tid] + red[768 + tid];
  if (tid < b) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) t += red[1024 + tid + 16 * k];
    rec[a * b + tid] = t;
  }
}

// Two row-block products from one read of X (N x a, a <= 16), for the block step that starts from
// the residual: Z = R - X M1 (b columns) and Lam += X M2 (c columns), M1, M2 column-major with
// a rows (b, c <= 16).  X is the previous step's direction block: the orthogonalisation of the new
// block and the deferred solution update of the previous one share its pass.  Rows of X enter LDS
// with lane-consecutive loads, each thread forms its row of both products, and the results leave
// through LDS with lane-consecutive stores (the loads of R and Lam for a tile all in flight).
__global__ __launch_bounds__(256) void k_rows_orth_lam(int64_t N, int a, int b, int c, const double* M1,
                                                       const double* M2, const double* X, int64_t ldx,
                                                       const double* R, int64_t ldr, double* Z, int64_t ldz,
                                                       double* Lam, int64_t ldl) {
  __shared__ double sm1[16][16];
  __shared__ double sm2[16][16];
  __shared__ double xs[256][17];
  __shared__ double ys[256][17];
  const int tid = threadIdx.x, er = tid >> 4, ec = tid & 15;
  const int64_t r0 = (int64_t)blockIdx.x * 256;
  const int rows = (int)min<int64_t>(256, N - r0);
  // the loads of X, R and Lam, at clamped (always valid) places, are all issued before anything waits:
  // one memory latency per workgroup (10 us at 76,080 x 8, where loads behind width tests took 16)
  double t[16], rv[16], lv[16];
  const double v1 = M1[min(er, a - 1) + (int64_t)a * min(ec, b - 1)];
  const double v2 = M2[min(er, a - 1) + (int64_t)a * min(ec, c - 1)];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int64_t row = r0 + min(er + 16 * u, rows - 1);
    t[u] = X[row * ldx + min(ec, a - 1)];
    rv[u] = R[row * ldr + min(ec, b - 1)];
    lv[u] = Lam[row * ldl + min(ec, c - 1)];
  }
  sm1[er][ec] = (er < a && ec < b) ? v1 : 0.0;
  sm2[er][ec] = (er < a && ec < c) ? v2 : 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) xs[er + 16 * u][ec] = ec < a ? t[u] : 0.0;
  __syncthreads();
  double acc1[16], acc2[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc1[j] = acc2[j] = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const double xv = xs[tid][i];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      acc1[j] += xv * sm1[i][j];
      acc2[j] += xv * sm2[i][j];
    }
  }
  __syncthreads();  // xs is reused for the first product
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    xs[tid][j] = acc1[j];
    ys[tid][j] = acc2[j];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int rr = er + 16 * u;
    if (rr >= rows) continue;
    if (ec < b) Z[(r0 + rr) * ldz + ec] = rv[u] - xs[rr][ec];
    if (ec < c) Lam[(r0 + rr) * ldl + ec] = lv[u] + ys[rr][ec];
  }
}

namespace {
bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

void launch_rows_small(hipStream_t s, int64_t N, int a, int b, const double* Mm, int64_t mrow, const RowsPairs& pr,
                       int npairs) {
  if (a <= 16 && b <= 16) {
    hipLaunchKernelGGL(k_rows_tile, dim3((unsigned)cdiv(N, 256), (unsigned)npairs), dim3(256), 0, s, N, a, b, Mm,
                       mrow, pr);
    RPF_LAUNCH_CHECK();
    return;
  }
  int vec = 1;
  for (int k = 0; k < npairs; ++k) {
    const RowsPair& q = pr.p[k];
    vec &= aligned16(q.X) && aligned16(q.Y) && (q.ldx % 2 == 0) && (q.ldy % 2 == 0) &&
           (!q.Z || (aligned16(q.Z) && q.ldz % 2 == 0));
  }
  hipLaunchKernelGGL(k_rows_small, dim3((unsigned)cdiv(N, 256), (unsigned)npairs), dim3(256), 0, s, N, a, b, Mm,
                     mrow, pr, vec);
  RPF_LAUNCH_CHECK();
}
}  // namespace

void rows_gemm_from(hipStream_t s, int64_t N, int a, int b, double alpha, const double* X, int64_t ldx,
                    const double* M, double beta, const double* Z, int64_t ldz, double* Y, int64_t ldy) {
  if (N <= 0 || b <= 0) return;
  RPF_CHECK(a <= 64 && b <= 16, RPF_EINVAL, "rows_gemm_from: block too wide");
  RowsPairs pr{};
  pr.p[0] = {X, Y, ldx, ldy, alpha, beta, Z, ldz};
  pr.p[1] = pr.p[0];
  launch_rows_small(s, N, a, b, M, 0, pr, 1);
}

// out[c * ldo] = sum_z part[z * b + c]: one workgroup per column c, a fixed partition of z over the
// threads and a fixed tree (deterministic).
__global__ __launch_bounds__(256) void k_colsum(int nz, int b, const double* part, const double* raised, double* out,
                                                int64_t ldo) {
  __shared__ double red[256];
  const int c = blockIdx.x, tid = threadIdx.x;
  double v = 0.0;
  for (int z = tid; z < nz; z += 256) v += part[(int64_t)z * b + c];
  red[tid] = v;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  if (tid == 0) out[(int64_t)c * ldo] = red[0];
  if (tid == 0 && c == 0) out[(int64_t)b * b] = *raised;
}

bool rows_gemm2_sq(hipStream_t s, int64_t N, int a, int b, const double* M, double alpha1, const double* X1,
                   int64_t ldx1, double beta1, double* Y1, int64_t ldy1, double alpha2, const double* X2,
                   int64_t ldx2, double beta2, double* Y2, int64_t ldy2, double* part, const double* raised, double* sq,
                   int64_t ldsq) {
  if (N <= 0 || b <= 0 || a > 16 || b > 16) return false;
  RowsPairs pr{};
  pr.p[0] = {X1, Y1, ldx1, ldy1, alpha1, beta1, nullptr, 0};
  pr.p[1] = {X2, Y2, ldx2, ldy2, alpha2, beta2, nullptr, 0};
  pr.colsq = part;
  const unsigned nwg = (unsigned)cdiv(N, 256);
  if (nwg == 1) {
    pr.sq = sq;
    pr.ldsq = ldsq;
    pr.raised = raised;
  }
  hipLaunchKernelGGL(k_rows_tile, dim3(nwg, 2), dim3(256), 0, s, N, a, b, M, (int64_t)0, pr);
  RPF_LAUNCH_CHECK();
  if (nwg == 1) return true;
  // sq[c * ldsq] = sum over workgroups of part[wg * b + c]
  hipLaunchKernelGGL(k_colsum, dim3((unsigned)b), dim3(256), 0, s, (int)nwg, b, part, raised, sq, ldsq);
  RPF_LAUNCH_CHECK();
  return true;
}

// Sums groups of `per` of the nrec records of len doubles (record r at part[r len]): workgroup g the
// records g per .. g per + per - 1, thread t element t, eight loads in flight, in a fixed order.
__global__ __launch_bounds__(320) void k_recsum(int nrec, int len, int per, const double* part, double* out) {
  const int t = threadIdx.x;
  if (t >= len) return;
  const int r0 = blockIdx.x * per, r1 = min(nrec, r0 + per);
  double v[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = 0.0;
  for (int r = r0; r < r1; r += 8) {
    double x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = part[(int64_t)min(r + u, r1 - 1) * len + t];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (r + u < r1) v[u] += x[u];
  }
  out[(int64_t)blockIdx.x * len + t] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// The records of rows_update_gram (n of them left) to what the next block step starts from, in one
// workgroup: C = P^T R (m x m) and the squared norms (to sq, stride ldsq, unless NULL, with *raised after
// the m x m entries), then B = T^T C
// (its diagonal only with diag) and M = T B.
__global__ __launch_bounds__(1024) void k_recsum_coef(int n, int m, const double* rec, const double* T, int diag,
                                                      const double* raised, double* sq, int64_t ldsq, double* B,
                                                      double* M) {
  __shared__ double c[16 * 17], st[256], sb[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int len = m * m + m;
  if (tid < m * m) st[tid] = T[tid];
  // wave w sums the elements w, w + 16, ..: lane l the records l, l + 64, then across the lanes
  for (int e0 = wave; e0 < len; e0 += 64) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = min(e0 + 16 * u, len - 1);
      v[u] = 0.0;
      for (int r = lane; r < n; r += 64) v[u] += rec[(int64_t)r * len + e];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v[u] += __shfl_xor(v[u], off, 64);
      if (lane == 0 && e0 + 16 * u < len) c[e0 + 16 * u] = v[u];
    }
  }
  __syncthreads();
  if (sq && tid < m) sq[tid * ldsq] = c[m * m + tid];
  if (sq && tid == 0) sq[(int64_t)m * m] = *raised;
  const int r = tid % m, col = tid / m;
  double v = 0.0;
  if (tid < m * m && (!diag || r == col))
    for (int k = 0; k < m; ++k) v += st[k + r * m] * c[k + col * m];
  if (tid < m * m) {
    sb[tid] = v;
    B[tid] = v;
  }
  __syncthreads();
  if (tid < m * m) {
    v = 0.0;
    for (int k = 0; k < m; ++k) v += st[r + k * m] * sb[k + col * m];
    M[tid] = v;
  }
}

bool rows_orth_lam(hipStream_t s, int64_t N, int a, int b, int c, const double* X, int64_t ldx, const double* M1,
                   const double* R, int64_t ldr, double* Z, int64_t ldz, const double* M2, double* Lam, int64_t ldl) {
  if (N <= 0 || a <= 0 || a > 16 || b <= 0 || b > 16 || c <= 0 || c > 16) return false;
  hipLaunchKernelGGL(k_rows_orth_lam, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, s, N, a, b, c, M1, M2, X, ldx, R,
                     ldr, Z, ldz, Lam, ldl);
  RPF_LAUNCH_CHECK();
  return true;
}

constexpr int UPD_GROUPS = 64;  // records left for the last, single workgroup
size_t update_gram_workspace(int64_t N, int a, int b) { return (size_t)(cdiv(N, 256) + UPD_GROUPS) * (a * b + b); }

bool rows_update_gram(hipStream_t s, int64_t N, int a, int b, const double* M, const double* X, int64_t ldx,
                      double alpha, double beta, double* Y, int64_t ldy, double* sq, int64_t ldsq, double* part,
                      const double* T, bool diag, const double* raised, double* Bo, double* Mo) {
  if (N <= 0 || a <= 0 || a > 16 || b != a) return false;
  const int nwg = (int)cdiv(N, 256), len = a * b + b;
  hipLaunchKernelGGL(k_rows_update_gram, dim3((unsigned)nwg), dim3(256), 0, s, N, a, b, M, X, ldx, alpha, beta, Y,
                     ldy, part);
  RPF_LAUNCH_CHECK();
  const double* rec = part;
  int n = nwg;
  if (nwg > UPD_GROUPS) {
    const int per = (int)cdiv(nwg, UPD_GROUPS);
    n = (int)cdiv(nwg, per);
    double* tmp = part + (int64_t)nwg * len;
    hipLaunchKernelGGL(k_recsum, dim3((unsigned)n), dim3(320), 0, s, nwg, len, per, part, tmp);
    rec = tmp;
  }
  hipLaunchKernelGGL(k_recsum_coef, dim3(1), dim3(1024), 0, s, n, a, rec, T, diag ? 1 : 0, raised, sq, ldsq,
                     Bo, Mo);
  RPF_LAUNCH_CHECK();
  return true;
}

void rows_gemm2(hipStream_t s, int64_t N, int a, int b, const double* M, int64_t mrow, double alpha1,
                const double* X1, int64_t ldx1, double beta1, double* Y1, int64_t ldy1, double alpha2,
                const double* X2, int64_t ldx2, double beta2, double* Y2, int64_t ldy2) {
  if (N <= 0 || b <= 0) return;
  if (a <= 64 && b <= 16) {
    RowsPairs pr{};
    pr.p[0] = {X1, Y1, ldx1, ldy1, alpha1, beta1, nullptr, 0};
    pr.p[1] = {X2, Y2, ldx2, ldy2, alpha2, beta2, nullptr, 0};
    launch_rows_small(s, N, a, b, M, mrow, pr, 2);
  } else {
    rows_gemm(s, N, a, b, alpha1, X1, ldx1, M, beta1, Y1, ldy1, mrow);
    rows_gemm(s, N, a, b, alpha2, X2, ldx2, M, beta2, Y2, ldy2, mrow);
  }
}

void rows_gemm(hipStream_t s, int64_t N, int a, int b, double alpha, const double* X, int64_t ldx, const double* Mm,
               double beta, double* Y, int64_t ldy, int64_t mrow) {
  if (N <= 0 || b <= 0) return;
  if (a <= 64 && b <= 16 && N >= 4096) {
    RowsPairs pr{};
    pr.p[0] = {X, Y, ldx, ldy, alpha, beta, nullptr, 0};
    pr.p[1] = pr.p[0];
    launch_rows_small(s, N, a, b, Mm, mrow, pr, 1);
    return;
  }
  if (a >= 128 && cdiv(N, 64) < 512) {
    // few row blocks: a wavefront per row keeps the whole chip busy on the inner dimension
    hipLaunchKernelGGL(k_rows_gemm_wave, dim3((unsigned)cdiv(N, 4)), dim3(256), 0, s, N, a, b, alpha, X, ldx, Mm, mrow,
                       beta, Y, ldy);
  } else if (b <= 16 && a >= 2) {
    const bool vec = (a % 2) == 0 && (ldx % 2) == 0 && (reinterpret_cast<uintptr_t>(X) % 16) == 0;
    if (vec)
      hipLaunchKernelGGL(k_rows_mfma<true>, dim3((unsigned)cdiv(N, 64)), dim3(256), 0, s, N, a, b, alpha, X, ldx, Mm,
                         mrow, beta, Y, ldy);
    else
      hipLaunchKernelGGL(k_rows_mfma<false>, dim3((unsigned)cdiv(N, 64)), dim3(256), 0, s, N, a, b, alpha, X, ldx,
                         Mm, mrow, beta, Y, ldy);
  } else {
    hipLaunchKernelGGL(k_rows_gemm, dim3((unsigned)cdiv(N, 64)), dim3(256), 0, s, N, a, b, alpha, X, ldx, Mm, mrow,
                       beta, Y, ldy);
  }
  RPF_LAUNCH_CHECK();
}

// ============================================================================ Cholesky
// Value of v in lane J of this lane's row of sixteen: one cross-lane move, no scalar registers and no LDS.
template <int J>
__device__ __forceinline__ double row_lane(double v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x150 + J, 0xf, 0xf, true);
}

// 1 / d, d well inside the range of the format, to the rounding of the division: a third-order step on the
// hardware estimate and a last correction.  It stands on the serial chain of the factorisation.
__device__ __forceinline__ double pivot_recip(double d) {
  const double r = __builtin_amdgcn_rcp(d), e = __builtin_fma(-d, r, 1.0);
  const double q = __builtin_fma(__builtin_fma(e, e, e), r, r);
  return __builtin_fma(__builtin_fma(-d, q, 1.0), q, q);
}

// Steps J .. 15 of the elimination of a symmetric 16 x 16 tile and of the identity beside it: lane c of
// every row of sixteen holds column c of each (a, x), and both take the same row operations
// row_i -= (a_iJ / d_J) row_J; r = 1 / d_J.  At the end a_j (j <= c) is d_j l_cj and x is the inverse of
// the unit factor.  Row J + 1 goes first, so that the next reciprocal runs under the rest of the step.
template <int J = 0>
__device__ __forceinline__ void eliminate(double (&a)[16], double (&x)[16], double r) {
  if constexpr (J < 15) {
    const double ta = -a[J] * r, tx = -x[J] * r;
    double next = 0.0;
#pragma unroll
    for (int i = J + 1; i < 16; ++i) {
      const double f = row_lane<J>(a[i]);
      a[i] = __builtin_fma(f, ta, a[i]);
      x[i] = __builtin_fma(f, tx, x[i]);
      if (i == J + 1) next = pivot_recip(row_lane<J + 1>(a[J + 1]));
    }
    // keeps x beside a: left alone, the compiler runs a through all steps first and spills the factors
#pragma unroll
    for (int i = J + 1; i < 16; ++i) asm volatile("" : "+v"(a[i]), "+v"(x[i]));
    eliminate<J + 1>(a, x, next);
  }
}
template <int J = 0>
__device__ __forceinline__ void scale_rows(double (&a)[16], double (&x)[16], double rs) {
  if constexpr (J < 16) {
    const double f = row_lane<J>(rs);
    a[J] *= f;
    x[J] *= f;
    scale_rows<J + 1>(a, x, rs);
  }
}

// One NB x NB (128 x 128) diagonal block: its Cholesky factor L and W = L^{-1}, one workgroup of sixteen
// waves, in 16-wide steps over one LDS array.  M[c][r] holds A(r, c) and then L(r, c) for r >= c (columns
// contiguous, as in memory), and M[r][c] holds W(r, c) for r > c in the half that L leaves free; the
// row stride of 144 doubles puts the two k-rows that a half-wave reads on opposite bank halves.  Step k:
//   (1) wave 0 factors the 16 x 16 tile k and inverts it (eliminate);
//   (2) L_ik = A_ik W_kk^T for the tiles below, and W_k,j = W_kk Acc_k,j for the tiles left of it;
//   (3) A_ij -= L_ik L_jk^T and Acc_ij -= L_ik W_kj, tile by tile on FP64 MFMA.  Wave 0 takes the next
//       diagonal tile and goes straight on with its step (1) while the other waves do the rest.
// A block takes 34.5 us by the device's clock: 3.2 us for the entry loads, 0.5 for the last store, and 3.9 a step:
// 2.4 the serial tile (1), 0.35 its update before it, 0.6 the products (2), 0.5 waiting for the other waves
// (1.1 in the second step, none in the last).  Rows and columns from jb on are those of the identity.  dinv: W by rows, dinv[r NB + c], zeros above the diagonal.
__global__ __launch_bounds__(1024) void k_potrf_diag(double* Ag, int64_t lda, int jb, double* dinv, int* status,
                                                    int blk) {
  static_assert(NB == 128, "k_potrf_diag assumes 128 x 128 blocks");
  constexpr int QB = 16, LD = NB + 16, NT = NB / QB;
  __shared__ double M[NB * LD];
  __shared__ double Wd[QB * QB];  // W_kk of the current step, Wd[q][c] = W_kk(c, q)
  __shared__ double wdiag[NB];
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int fl = lane & 15, fk = lane >> 4;
  if (tid == 0) bad = 0;
  {
    // all 16 loads of a thread at clamped (always valid) addresses, issued together and masked
    // afterwards: a load behind a branch would cost one round trip to memory each
    double v[NB * NB / 1024];
    const int r = tid & (NB - 1), c0 = tid >> 7;
#pragma unroll
    for (int u = 0; u < NB * NB / 1024; ++u) {
      const int c = min(c0 + 8 * u, jb - 1);  // rows above the diagonal read the diagonal's line again
      v[u] = Ag[(int64_t)c * lda + min(max(r, c), jb - 1)];
    }
#pragma unroll
    for (int u = 0; u < NB * NB / 1024; ++u) {
      const int c = c0 + 8 * u;
      if (r >= c) M[c * LD + r] = (r < jb && c < jb) ? v[u] : ((r == c) ? 1.0 : 0.0);
    }
  }
  const int nk = (jb + QB - 1) / QB;
  // rows of the identity past the tiles of jb, which no step reaches
  for (int e = QB * nk * NB + tid; e < NB * NB; e += 1024) {
    const int r = e >> 7, c = e & (NB - 1);
    dinv[e] = r == c ? 1.0 : 0.0;
  }
  __syncthreads();
  // step (1) of tile k, by wave 0
  auto factor_tile = [&](int k) {
    const int o = QB * k;
    double a[QB], x[QB];
#pragma unroll
    for (int i = 0; i < QB; ++i) {
      a[i] = M[(i >= fl) ? (o + fl) * LD + o + i : (o + i) * LD + o + fl];
      x[i] = i == fl ? 1.0 : 0.0;
    }
    auto own = [&] {  // entry c of lane c
      double d = 0.0;
#pragma unroll
      for (int j = 0; j < QB; ++j) d = j == fl ? a[j] : d;
      return d;
    };
    // a diagonal far from one is brought there by powers of two (exactly): A = P A' P, L = P L'
    double d = M[(o + fl) * LD + o + fl];
    const bool far = __any(!(d > 1e-200 && d < 1e200));
    int e = 0;
    if (far) {
      (void)frexp(d, &e);
      e >>= 1;
#pragma unroll
      for (int i = 0; i < QB; ++i) a[i] = ldexp(a[i], -e - __shfl(e, (lane & 48) + i, 64));
    }
    eliminate(a, x, pivot_recip(row_lane<0>(a[0])));
    d = own();
    if (__any(!(d > 0.0)) && lane == 0) bad = 1;
    double dl = sqrt(d), dw = 1.0 / dl;
    scale_rows(a, x, dw);
    if (far) {
      dl = ldexp(dl, e);
      dw = ldexp(dw, -e);
#pragma unroll
      for (int j = 0; j < QB; ++j) {
        a[j] = ldexp(a[j], e);
        x[j] = ldexp(x[j], -e);
      }
    }
    if (fk == 0) {
#pragma unroll
      for (int j = 0; j < QB; ++j) {
        // L(c, j) for c >= j, W(j, c) for j > c
        M[(o + j) * LD + o + fl] = (j < fl) ? a[j] : (j == fl ? dl : x[j]);
        Wd[fl * QB + j] = j > fl ? x[j] : (j == fl ? dw : 0.0);
      }
      wdiag[o + fl] = dw;
    }
  };
  // tile product D[row][col] = sum_q P[q][row] Q[q][col], both operands 16-row slabs of LDS
  auto tile_mma = [&](const double* P, int ldp, const double* Q, int ldq, v4d acc) {
#pragma unroll
    for (int q = 0; q < QB; q += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(q + fk) * ldp + fl], Q[(q + fk) * ldq + fl], acc, 0, 0, 0);
    return acc;
  };
  // C[row][col] -= (that product)
  auto tile_sub = [&](double* C, const double* P, const double* Q) {
    const v4d acc = tile_mma(P, LD, Q, LD, v4d{0.0, 0.0, 0.0, 0.0});
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double* c = C + (fk + 4 * r) * LD + fl;
      *c -= acc[r];
    }
  };
  // the finished columns of L and rows of W of step k, by nt threads
  auto store_tile = [&](int k, int t, int nt) {
    const int o = QB * k;
    for (int e = t; e < QB * NB; e += nt) {
      const int i = o + (e >> 7), j = e & (NB - 1);
      const double v = M[i * LD + j];
      if (j >= i && j < jb && i < jb) Ag[(int64_t)i * lda + j] = v;                // L(j, i)
      dinv[i * NB + j] = j < i ? v : (j == i ? wdiag[i] : 0.0);                    // W(i, j)
    }
  };
  for (int k = 0; k < nk; ++k) {
    const int o = QB * k, p = o - QB;
    // (3) of step k - 1, and (1)
    if (wave == 0) {
      if (k > 0) tile_sub(M + o * LD + o, M + p * LD + o, M + p * LD + o);
      factor_tile(k);
    } else if (k > 0) {
      store_tile(k - 1, tid - 64, 1024 - 64);
      const int nr = nk - k;                  // tile rows below step k - 1
      const int ntri = nr * (nr + 1) / 2;     // trailing tiles; the first is wave 0's
      const int total = ntri + nr * k;
      for (int u = wave; u < total; u += 15) {
        if (u < ntri) {
          int i = 0, b = u;
          while (b > i) b -= ++i;             // u -> (i, b), b <= i
          const int oi = o + QB * i, oj = o + QB * b;
          // as D[j][i], so that the tile's i runs along M's rows
          tile_sub(M + oj * LD + oi, M + p * LD + oj, M + p * LD + oi);
        } else {
          const int v = u - ntri;
          const int oi = o + QB * (v / k), kk = v % k;
          double* C = M + oi * LD + QB * kk;
          if (kk < k - 1) {
            tile_sub(C, M + p * LD + oi, M + p * LD + QB * kk);
          } else {
            // the first product into this tile, with W_pp itself: its strict lower part and diagonal
            v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < QB; q += 4) {
              const int qq = q + fk;
              const double m = M[(p + qq) * LD + p + fl], g = wdiag[p + fl];
              acc = __builtin_amdgcn_mfma_f64_16x16x4f64(M[(p + qq) * LD + oi + fl],
                                                         qq > fl ? m : (qq == fl ? g : 0.0), acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) C[(fk + 4 * r) * LD + fl] = -acc[r];
          }
        }
      }
    }
    __syncthreads();
    // (2) tiles below (as W_kk A_ik^T: M holds A transposed) and to the left, the same product of M
    for (int u = wave; u < nk - 1; u += 16) {
      double* C = M + o * LD + QB * (u >= k ? u + 1 : u);
      const v4d acc = tile_mma(Wd, QB, C, LD, v4d{0.0, 0.0, 0.0, 0.0});
#pragma unroll
      for (int r = 0; r < 4; ++r) C[(fk + 4 * r) * LD + fl] = acc[r];
    }
    __syncthreads();
  }
  if (nk > 0) store_tile(nk - 1, tid, 1024);
  if (tid == 0 && bad) atomicCAS(status, 0, blk + 1);
}

LaunchEvents& launch_events() {
  static thread_local LaunchEvents ev;
  return ev;
}

Envelope Envelope::dense(int64_t n) {
  Envelope e;
  const int64_t nb = cdiv(n, NB);
  e.rend.assign(nb, n);
  e.cstart.assign(nb, 0);
  return e;
}

// L21 = A21 W^T in place for an NB-wide column block (jb columns) on two ranges of rows (C0: below the
// diagonal block; C1: the boundary rows), W = L11^{-1} by rows (dinv).  One workgroup per 32 rows reads
// all of its columns before it writes any.  Wave w takes the column tiles w and 7 - w, nine 16 x 16
// blocks of the triangle in all, whose W operands are loaded before the rows are waited for: one load
// latency and 72 MFMAs a wave, 5 us where the four k-stages of the general product took 11.
__global__ __launch_bounds__(256) void k_panel(double* C0, int64_t ld0, int64_t len0, double* C1, int64_t ld1,
                                               int64_t len1, int jb, const double* dinv) {
  static_assert(NB == 128, "k_panel assumes 128-wide blocks");
  constexpr int LD = 40;  // the two k-rows of a half-wave (two apart) on opposite bank halves
  __shared__ double As[NB * LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fl = lane & 15, fk = lane >> 4;
  const int64_t t0 = (len0 + 31) / 32;
  const bool second = (int64_t)blockIdx.x >= t0;
  const int64_t off = 32 * (second ? (int64_t)blockIdx.x - t0 : (int64_t)blockIdx.x);
  double* C = (second ? C1 : C0) + off;
  const int64_t lda = second ? ld1 : ld0;
  const int nr = (int)min<int64_t>(32, (second ? len1 : len0) - off);
  double2 wv[18];
  const int n1 = 2 * (w + 1);  // 8-k groups of tile w, then 18 - n1 of tile 7 - w
#pragma unroll
  for (int g = 0; g < 18; ++g) {
    const int j = g < n1 ? w : 7 - w, q0 = 8 * (g < n1 ? g : g - n1);
    wv[g] = *(const double2*)(dinv + (16 * j + fl) * NB + q0 + 2 * fk);
  }
  {
    double v[16];
    const int r = min(tid & 31, nr - 1);
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = C[(int64_t)min((tid >> 5) + 8 * u, jb - 1) * lda + r];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int q = (tid >> 5) + 8 * u;
      As[q * LD + (tid & 31)] = q < jb ? v[u] : 0.0;
    }
  }
  __syncthreads();
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) acc[i][rt] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int g = 0; g < 18; ++g) {
    const int q = 8 * (g < n1 ? g : g - n1) + 2 * fk;
    double x[2], y[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      x[rt] = As[q * LD + 16 * rt + fl];
      y[rt] = As[(q + 1) * LD + 16 * rt + fl];
    }
    const int i = g < n1 ? 0 : 1;
    if (i == 0) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        acc[0][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[g].x, x[rt], acc[0][rt], 0, 0, 0);
        acc[0][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[g].y, y[rt], acc[0][rt], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        acc[1][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[g].x, x[rt], acc[1][rt], 0, 0, 0);
        acc[1][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[g].y, y[rt], acc[1][rt], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = 16 * (i == 0 ? w : 7 - w) + fk + 4 * r, row = 16 * rt + fl;
        if (c < jb && row < nr) C[(int64_t)c * lda + row] = acc[i][rt][r];
      }
}

// C -= X Y^T for two ranges of rows in one launch, Y the first N rows of X0: rows X0 (len0) only where they
// reach the lower triangle, rows X1 (len1, the boundary rows) in full; K columns.  64 x 64
// tiles with 64-k stages: a rank-NB update is two stages, so two load latencies.
template <bool SHORT>
__global__ __launch_bounds__(256) void k_rank_update(int64_t len0, const double* X0, double* C0, int64_t ld0,
                                                     int64_t len1, const double* X1, double* C1, int64_t ld1,
                                                     int64_t N, int64_t K) {
  const int t0 = (int)((len0 + 63) / 64);
  const bool second = (int)blockIdx.x >= t0;
  const int64_t ld = second ? ld1 : ld0;
  dgemm_tile<64, 64, 2, 2, false, true, 64, SHORT>(second ? len1 : len0, N, K, -1.0, second ? X1 : X0, ld, X0, ld0, 1.0,
                                                   second ? C1 : C0, ld, second ? 0 : 1, K, nullptr,
                                                   second ? (int)blockIdx.x - t0 : (int)blockIdx.x, blockIdx.y, 0);
}

// columns [r0, cend) of the rows [r0, rend) of the factor and of the first len1 boundary rows, minus the
// K columns from j0.  A factor without boundary rows (dense: of S + Z Z^T, S + sigma I, a coarse matrix) adds up 64
// products at a time, as 64-wide blocks would: in one run of 256, S+ of a 7^3 brick was 6.6 eps off and
// that of a 7 x 11 x 5 one 12.9, now 4.9 and 9.1 (64-wide blocks: 5.3 and 11.7).  Beside the boundary rows, whose
// S is as accurate either way, the second set of accumulators cost 4 % of a 20^3 brick's setup.
static void rank_update(hipStream_t s, double* A, int64_t lda, const BoundaryRows& bnd, int64_t len1, int64_t j0,
                        int64_t K, int64_t r0, int64_t rend, int64_t cend) {
  const int64_t N = cend - r0;
  if (N <= 0 || K <= 0) return;
  RPF_CHECK(cdiv(N, 64) <= 65535, RPF_EINVAL, "potrf: grid too large");
  const dim3 grid((unsigned)(cdiv(rend - r0, 64) + cdiv(len1, 64)), (unsigned)cdiv(N, 64));
  if (bnd.n == 0)
    hipLaunchKernelGGL(k_rank_update<true>, grid, dim3(256), 0, s, rend - r0, A + j0 * lda + r0, A + r0 * lda + r0, lda,
                       (int64_t)0, (const double*)nullptr, (double*)nullptr, (int64_t)0, N, K);
  else
    hipLaunchKernelGGL(k_rank_update<false>, grid, dim3(256), 0, s, rend - r0, A + j0 * lda + r0, A + r0 * lda + r0,
                       lda, len1, bnd.p + j0 * bnd.ld, bnd.p + r0 * bnd.ld, bnd.ld, N, K);
  RPF_LAUNCH_CHECK();
}

// Two levels: NB-wide steps (diagonal block, panel) inside panels of PANEL = 2 NB columns.  A step
// updates only the columns of its own panel (rank NB); everything to the right of a panel gets
// one rank-PANEL update once the panel is done, so the trailing matrix and the boundary rows are
// read and written once per panel instead of once per step.  A step is bound by the latency of its three
// dependent launches, so the rows below and the boundary rows share each of them.  The result is the
// same factor (the updates of one column commute).
bool gemm_nt_flex(hipStream_t s, int64_t M, int64_t N, int64_t K, double alpha, const double* X, int64_t ldx,
                  const double* Y, int64_t ldy, double beta, double* C, int64_t ldc, bool lower, DevBuf<double>& wa,
                  DevBuf<double>& wb);

void potrf(hipStream_t s, double* A, int64_t lda, int64_t n_fac, const Envelope& env, double* dinv, int* status,
           const BoundaryRows& bnd) {
  constexpr int64_t PANEL = 2 * NB;
  // rows from which a trailing update goes to the large-problem kernel (which needs copies of its
  // operands): below, its 128 x 128 tiles leave CUs idle
  constexpr int64_t LARGE = 4096;
  const int64_t nblk = cdiv(n_fac, NB);
  RPF_CHECK((int64_t)env.rend.size() >= nblk && (bnd.n == 0 || (int64_t)bnd.active.size() >= nblk), RPF_EINVAL,
            "potrf: envelope too short");
  DevBuf<double> wa, wb;  // operand copies of the large rank-PANEL updates
  for (int64_t P0 = 0; P0 < n_fac; P0 += PANEL) {
    const int64_t P1 = std::min<int64_t>(P0 + PANEL, n_fac);
    int64_t pend = P1;  // rows (and columns) reached by the panel's envelope
    int64_t act = 0;    // boundary rows reached by the panel
    for (int64_t j0 = P0; j0 < P1; j0 += NB) {
      const int64_t t = j0 / NB;
      const int jb = (int)std::min<int64_t>(NB, n_fac - j0);
      double* dt = dinv + t * NB * NB;
      hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(1024), 0, s, A + j0 * lda + j0, lda, jb, dt, status, (int)t);
      RPF_LAUNCH_CHECK();
      const int64_t r0 = j0 + jb;
      const int64_t rend = std::max<int64_t>(r0, std::min<int64_t>(env.rend[t], n_fac));
      pend = std::max(pend, rend);
      act = bnd.n ? bnd.active[t] : 0;
      const int64_t tiles = cdiv(rend - r0, 32) + cdiv(act, 32);
      if (tiles > 0) {
        hipLaunchKernelGGL(k_panel, dim3((unsigned)tiles), dim3(256), 0, s, A + j0 * lda + r0, lda, rend - r0,
                           bnd.p + j0 * bnd.ld, bnd.ld, act, jb, dt);
        RPF_LAUNCH_CHECK();
      }
      // the remaining columns of this panel (rows within the envelope, boundary rows)
      rank_update(s, A, lda, bnd, act, j0, jb, r0, rend, std::min(rend, P1));
    }
    // rank-PANEL update of everything right of the panel (the boundary-boundary block is deferred);
    // rows of a step's columns past its own envelope end are zero, so one product over the
    // panel's whole envelope is exact
    if (pend > P1) {
      const int64_t K = P1 - P0, N = pend - P1;
      double* pc = A + P0 * lda + P1;
      const bool done0 = N >= LARGE && gemm_nt_flex(s, N, N, K, -1.0, pc, lda, pc, lda, 1.0, A + P1 * lda + P1, lda, true,
                                                    wa, wb);
      const bool done1 = act >= LARGE && gemm_nt_flex(s, act, N, K, -1.0, bnd.p + P0 * bnd.ld, bnd.ld, pc, lda, 1.0,
                                                      bnd.p + P1 * bnd.ld, bnd.ld, false, wa, wb);
      if (!done0)
        rank_update(s, A, lda, bnd, done1 ? 0 : act, P0, K, P1, pend, pend);
      else if (!done1 && act > 0)
        dgemm(s, false, true, act, N, K, -1.0, bnd.p + P0 * bnd.ld, bnd.ld, pc, lda, 1.0, bnd.p + P1 * bnd.ld, bnd.ld);
    }
  }
  RPF_HIP(hipStreamSynchronize(s));  // the operand copies are freed on return
}

// Bt[j ldb + k] = X[j + k ldx] for j < rows, k < cols, and 0 for cols <= k < ldb: the transpose of a
// column-major rows x cols block with zero-padded rows, through 64 x 64 LDS tiles (coalesced on
// both sides).  Grid: (cdiv(ldb, 64), cdiv(rows, 64)).
__global__ __launch_bounds__(256) void k_transpose_pad(int64_t rows, int64_t cols, const double* X, int64_t ldx,
                                                       double* Bt, int64_t ldb) {
  __shared__ double t[64][65];
  const int64_t k0 = (int64_t)blockIdx.x * 64, j0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int r = ty; r < 64; r += 4) {
    const int64_t k = k0 + r, j = j0 + tx;
    t[r][tx] = (k < cols && j < rows) ? X[j + k * ldx] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 64; r += 4) {
    const int64_t j = j0 + r, k = k0 + tx;
    if (j < rows && k < ldb) Bt[j * ldb + k] = t[tx][r];
  }
}

// C = alpha X Y^T + beta C (X: M x K, Y: N x K, column-major) on the large-problem kernel when the
// shape is large enough: X is used in place when its layout allows it (else copied with an even
// leading dimension), Y^T is copied with k-contiguous rows padded to 32.  wa, wb: grow-only
// workspaces kept by the caller across calls.  Returns false (nothing launched) for small shapes.
bool gemm_nt_flex(hipStream_t s, int64_t M, int64_t N, int64_t K, double alpha, const double* X, int64_t ldx,
                  const double* Y, int64_t ldy, double beta, double* C, int64_t ldc, bool lower, DevBuf<double>& wa,
                  DevBuf<double>& wb) {
  if (M < 1024 || (M & 1) || N < 128 || K < 64 || M > INT32_MAX || N > INT32_MAX) return false;
  const double* Ause = X;
  int64_t lda = ldx;
  if ((ldx & 1) || ((uintptr_t)X & 15)) {
    wa.ensure((size_t)M * K);
    copy_matrix(s, X, ldx, wa.p, M, M, K);
    Ause = wa.p;
    lda = M;
  }
  const int64_t ldb = cdiv(K, 32) * 32;
  wb.ensure((size_t)N * ldb);
  hipLaunchKernelGGL(k_transpose_pad, dim3((unsigned)cdiv(ldb, 64), (unsigned)cdiv(N, 64)), dim3(256), 0, s, N, K, Y,
                     ldy, wb.p, ldb);
  RPF_LAUNCH_CHECK();
  return dgemm_flex(s, M, N, K, alpha, Ause, lda, wb.p, ldb, beta, C, ldc, lower);
}

// The boundary rows are sorted by the first interior column that they reach, so the columns of a group
// meet a prefix of them: the product is taken group by group on that prefix.  On the 20^3 brick that is
// a third of the flops of one product over all rows and columns (1,069 GFLOP).
void schur_update(hipStream_t s, double* S, int64_t lds, int64_t n_fac, const BoundaryRows& bnd) {
  constexpr int64_t GROUP = 8 * NB;  // S is read and written once per group
  DevBuf<double> wa, wb;
  for (int64_t c0 = 0; c0 < n_fac; c0 += GROUP) {
    const int64_t K = std::min<int64_t>(GROUP, n_fac - c0);
    // an even count for the large-problem kernel (rows past the prefix are zero in these columns)
    const int64_t act = std::min(bnd.n, bnd.active[(c0 + K - 1) / NB] + (bnd.active[(c0 + K - 1) / NB] & 1));
    if (act == 0) continue;
    const double* X = bnd.p + c0 * bnd.ld;
    // lower tiles only: S is symmetric and only its lower triangle is read afterwards
    if (!gemm_nt_flex(s, act, act, K, -1.0, X, bnd.ld, X, bnd.ld, 1.0, S, lds, true, wa, wb))
      dgemm(s, false, true, act, act, K, -1.0, X, bnd.ld, X, bnd.ld, 1.0, S, lds, true);
  }
  RPF_HIP(hipStreamSynchronize(s));  // the copies are freed on return
}

// Panel triangular solve for many right-hand sides: one workgroup owns PW = 16 H columns of B and
// walks all diagonal blocks in order (persistent), left-looking: for block t it forms
// B_t - L_t,band X_band on FP64 MFMA, stages the result in LDS and multiplies it by the inverted
// diagonal block, overwriting B_t with X_t.  Forward (L X = B) uses the rows of block t from column
// lo[t]; backward (L^T X = B) the rows j0 + 64 .. hi[t] of column block t.  The band is split over
// the four waves (wave w takes every fourth group of 16 k, all 64 rows of the block and the H
// 16-column parts: 4 H independent accumulators, each L fragment used H times from registers),
// the loads of a wave's next group are in flight while the MFMAs of the current one run, and the
// four partial products are summed in LDS.  The band operands come from L2 (every workgroup reads
// the same band of L; its own panel of X was written by itself one block earlier); the band's L2
// traffic is one read per PW right-hand sides.  UP (backward only): the band of L^T is read from the
// mirrored upper triangle, L^T[row][k] = A[row + k ldl], sixteen consecutive rows per load like the
// forward solve, instead of sixteen columns of L 8 bytes each.
template <bool FWD, int H, bool UP = false>
__global__ __launch_bounds__(256) void k_trsm_panel(const double* L, int64_t ldl, int64_t n, const double* dinv,
                                                    const int64_t* lo, const int64_t* hi, double* B, int64_t ldb,
                                                    int64_t nrhs) {
  constexpr int PW = 16 * H, SB = 64;  // rows of a step: half of a diagonal block
  __shared__ double S[SB][PW + 1];
  __shared__ double red[4][SB][PW + 1];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t col0 = (int64_t)blockIdx.x * PW + li;  // this lane's column in part 0 (part h: + 16 h)
  bool cok[H];
#pragma unroll
  for (int h = 0; h < H; ++h) cok[h] = col0 + 16 * h < nrhs;
  const int64_t nblk = (n + SB - 1) / SB;
  for (int64_t step = 0; step < nblk; ++step) {
    const int64_t t = FWD ? step : nblk - 1 - step;
    const int64_t j0 = t * SB;
    const int jb = (int)min<int64_t>(SB, n - j0);
    v4d acc[4][H];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < H; ++h) acc[q][h] = v4d{0.0, 0.0, 0.0, 0.0};
    int64_t kb, ke;
    if (FWD) {
      kb = max<int64_t>(0, lo[t / 2]);
      ke = j0;
    } else {
      kb = j0 + jb;
      ke = min<int64_t>(hi[t / 2], n);
    }
    // group g covers k in [kb + 16 g, kb + 16 g + 16); wave w takes g = w, w + 4, ...
    auto load = [&](int64_t k0, double* a, double* b) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t k = k0 + 4 * u + lk;
        const bool kok = k < ke;
#pragma unroll
        for (int h = 0; h < H; ++h) b[H * u + h] = (kok && cok[h]) ? B[k + (col0 + 16 * h) * ldb] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t row = j0 + 16 * q + li;
          a[4 * q + u] = (kok && row < j0 + jb) ? ((FWD || UP) ? L[row + k * ldl] : L[k + row * ldl]) : 0.0;
        }
      }
    };
    double a[16], b[4 * H], na[16], nb[4 * H];
    int64_t k0 = kb + 16 * w;
    if (k0 < ke) load(k0, a, b);
    for (; k0 < ke; k0 += 64) {
      const bool more = k0 + 64 < ke;
      if (more) load(k0 + 64, na, nb);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int h = 0; h < H; ++h)
            acc[q][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[4 * q + u], b[H * u + h], acc[q][h], 0, 0, 0);
      if (more) {
#pragma unroll
        for (int u = 0; u < 16; ++u) a[u] = na[u];
#pragma unroll
        for (int u = 0; u < 4 * H; ++u) b[u] = nb[u];
      }
    }
    // accumulator item r of tile (q, h), lane l: row 16 q + l/16 + 4 r, column 16 h + l % 16
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[w][16 * q + lk + 4 * r][16 * h + li] = acc[q][h][r];
    __syncthreads();
    for (int e = tid; e < SB * PW; e += 256) {
      const int ri = e / PW, cj = e % PW;
      const int64_t gc = (int64_t)blockIdx.x * PW + cj;
      const double bv = (ri < jb && gc < nrhs) ? B[j0 + ri + gc * ldb] : 0.0;
      S[ri][cj] = bv - (red[0][ri][cj] + red[1][ri][cj] + red[2][ri][cj] + red[3][ri][cj]);
    }
    __syncthreads();
    // X_t = inv(L_tt) S (forward) or inv(L_tt)^T S (backward): the inverse stands by rows; wave w
    // forms rows 16 w .. 16 w + 15 of every column part
    v4d x[H];
#pragma unroll
    for (int h = 0; h < H; ++h) x[h] = v4d{0.0, 0.0, 0.0, 0.0};
    const double* D = dinv + (t / 2) * NB * NB + (t & 1) * (SB * NB + SB);
#pragma unroll 4
    for (int kk = 0; kk < SB; kk += 4) {
      const int k = kk + lk, i = 16 * w + li;
      const double av = FWD ? D[k + i * NB] : D[i + k * NB];
#pragma unroll
      for (int h = 0; h < H; ++h) x[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, S[k][16 * h + li], x[h], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ri = 16 * w + lk + 4 * r;
      if (ri < jb) {
#pragma unroll
        for (int h = 0; h < H; ++h)
          if (cok[h]) B[j0 + ri + (col0 + 16 * h) * ldb] = x[h][r];
      }
    }
    __syncthreads();  // X_t is read by the band products of the following blocks
  }
}

// ============================================================================ block inverses
// X = the inverses of the diagonal blocks of bw rows (a multiple of NB) of a lower factor L, each bw x bw
// column-major in a slab of its own, from the inverted NB x NB blocks: the pairs of inverted blocks of
// h rows are joined level by level (h = NB, 2 NB, ..), X21 = -X22 (L21 X11), so the work is a few
// launches of large products instead of a serial walk over the rows.  What the products skip
// is known to be zero: L21 X11 starts at the column's own row, X22 T ends at the row's own column.
__device__ inline int64_t block_rows(int64_t n, int64_t j, int64_t h) { return min(h, max<int64_t>(n - j, 0)); }

// X11 of every NB block: the transpose of dinv (by rows), zeros above the diagonal; 64 x 64 through LDS
__global__ __launch_bounds__(256) void k_place_dinv(int64_t n, int64_t bw, const double* dinv, double* X) {
  __shared__ double t[64][65];
  const int64_t d = blockIdx.y, j = d * NB;
  const int r0 = (blockIdx.x & 1) * 64, c0 = (blockIdx.x >> 1) * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int r = ty; r < 64; r += 4) t[r][tx] = dinv[d * NB * NB + (r0 + r) * NB + c0 + tx];
  __syncthreads();
  const int64_t lj = j % bw;
  double* x = X + (j / bw) * bw * bw + lj * bw + lj;
  for (int c = ty; c < 64; c += 4)
    if (j + r0 + tx < n && j + c0 + c < n) x[(c0 + c) * bw + r0 + tx] = t[tx][c];
}

// One level.  Grid: (row tiles, column tiles, pairs); T: h x h per pair.
template <int TILE, int BK, bool SECOND>
__global__ __launch_bounds__(256) void k_join_blocks(int64_t n, int64_t bw, int64_t h, const double* L, int64_t ldl,
                                                     double* X, double* T) {
  const int64_t j = 2 * h * (int64_t)blockIdx.z;  // bw is a multiple of 2 h, or holds the whole factor
  const int64_t M = block_rows(n, j + h, h);
  const int64_t i0 = (int64_t)blockIdx.x * TILE, j0 = (int64_t)blockIdx.y * TILE;
  if (i0 >= M) return;
  const int64_t lj = j % bw;
  double* X11 = X + (j / bw) * bw * bw + lj * bw + lj;
  double* Tp = T + (int64_t)blockIdx.z * h * h;
  if (!SECOND)
    dgemm_tile<TILE, TILE, 2, 2, false, false, BK, BK == 64>(M, h, h - j0, 1.0, L + (j + j0) * ldl + j + h, ldl, X11 + j0, bw, 0.0,
                                                   Tp, h, 0, h, nullptr, blockIdx.x, blockIdx.y, 0);
  else
    dgemm_tile<TILE, TILE, 2, 2, false, false, BK, BK == 64>(M, h, min<int64_t>(i0 + TILE, M), -1.0, X11 + h * bw + h, bw, Tp, h,
                                                   0.0, X11 + h, bw, 0, h, nullptr, blockIdx.x, blockIdx.y, 0);
}

static int64_t join_scratch(int64_t n, int64_t bw) {
  int64_t most = 1;
  for (int64_t h = NB; h < bw; h *= 2) most = std::max(most, cdiv(n, 2 * h) * h * h);
  return most;
}

static void invert_blocks(hipStream_t s, const double* L, int64_t ldl, int64_t n, const double* dinv, double* X,
                          int64_t bw, double* T) {
  hipLaunchKernelGGL(k_place_dinv, dim3(4, (unsigned)cdiv(n, NB)), dim3(256), 0, s, n, bw, dinv, X);
  for (int64_t h = NB; h < bw; h *= 2) {
    const int64_t pairs = cdiv(n, 2 * h);
    if (n <= h) break;
    // 64 x 64 tiles until they alone fill the chip several times over
    if (pairs * (h / 64) * (h / 64) < 4096) {
      const dim3 g((unsigned)(h / 64), (unsigned)(h / 64), (unsigned)pairs);
      hipLaunchKernelGGL((k_join_blocks<64, 64, false>), g, dim3(256), 0, s, n, bw, h, L, ldl, X, T);
      hipLaunchKernelGGL((k_join_blocks<64, 64, true>), g, dim3(256), 0, s, n, bw, h, L, ldl, X, T);
    } else {
      const dim3 g((unsigned)(h / 128), (unsigned)(h / 128), (unsigned)pairs);
      hipLaunchKernelGGL((k_join_blocks<128, 16, false>), g, dim3(256), 0, s, n, bw, h, L, ldl, X, T);
      hipLaunchKernelGGL((k_join_blocks<128, 16, true>), g, dim3(256), 0, s, n, bw, h, L, ldl, X, T);
    }
    RPF_LAUNCH_CHECK();
  }
}

// Lower tiles of Y = X^T X, X lower triangular (ld bw): tile row i0 takes the rows of X from i0 on.
template <int TILE, int BK>
__global__ __launch_bounds__(256) void k_xtx(int64_t n, const double* X, int64_t bw, double* Y, int64_t ldy) {
  const int64_t i0 = (int64_t)blockIdx.x * TILE;
  dgemm_tile<TILE, TILE, 2, 2, true, false, BK, BK == 64>(n, n, n - i0, 1.0, X + i0, bw, X + i0, bw, 0.0, Y, ldy, 1, n, nullptr,
                                                blockIdx.x, blockIdx.y, 0);
}

// The 64 x 64 tiles here and in k_join_blocks add up 64 products at a time: with one run of sums S+ of a 9 x 8 x 8
// brick was 7.5 eps off, where solves by 64-row blocks had given 6.9; now 5.8 (7^3: 6.1, 5.3, 4.9).  The 128 x 128
// ones do without (S+ at 17^3: 20 eps, 22 by blocks).
//
// Y = (L L^T)^{-1} from a dense lower Cholesky factor L (n x n, ld ldl) and its inverted diagonal
// blocks: X = L^{-1} by joining blocks, then Y = X^T X, its lower triangle only (the upper one is left
// to the caller, see mirror_lower and add_outer).  Two thirds n^3 flops in about 2 log2(n / NB) + 2
// launches.
void potri_lower(hipStream_t s, const double* L, int64_t ldl, int64_t n, const double* dinv, double* Y,
                 int64_t ldy) {
  if (n <= 0) return;
  const int64_t bw = cdiv(n, NB) * NB;
  DevBuf<double> X((size_t)bw * bw), T(join_scratch(n, bw));
  invert_blocks(s, L, ldl, n, dinv, X.p, bw, T.p);
  if (n < 4096)
    hipLaunchKernelGGL((k_xtx<64, 64>), dim3((unsigned)cdiv(n, 64), (unsigned)cdiv(n, 64)), dim3(256), 0, s, n, X.p, bw,
                       Y, ldy);
  else
    hipLaunchKernelGGL((k_xtx<128, 16>), dim3((unsigned)cdiv(n, 128), (unsigned)cdiv(n, 128)), dim3(256), 0, s, n, X.p,
                       bw, Y, ldy);
  RPF_LAUNCH_CHECK();
  RPF_HIP(hipStreamSynchronize(s));  // the workspaces are freed on return
}

// B (n x n, ldb) = A (lower triangle of n x n, lda) + alpha Z Z^T + sigma I, Z n x k (ld n, k <= KDET - 1):
// its lower triangle, and with `full` the mirrored upper one too, in one pass over 64 x 64 tiles.
__global__ __launch_bounds__(256) void k_add_outer(int64_t n, const double* A, int64_t lda, int k, const double* Z,
                                                   double alpha, double sigma, double* B, int64_t ldb, int full) {
  __shared__ double t[64][65];
  __shared__ double zr[8][64], zc[8][64];
  const int64_t r0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
  if (c0 > r0) return;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int q = ty; q < k; q += 4) {
    zr[q][tx] = r0 + tx < n ? Z[q * n + r0 + tx] : 0.0;
    zc[q][tx] = c0 + tx < n ? alpha * Z[q * n + c0 + tx] : 0.0;
  }
  __syncthreads();
  const int64_t r = r0 + tx;
  double v[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) v[u] = A[min(c0 + ty + 4 * u, n - 1) * lda + min(r, n - 1)];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int lc = ty + 4 * u;
    const int64_t c = c0 + lc;
    double x = v[u];
    for (int q = 0; q < k; ++q) x += zr[q][tx] * zc[q][lc];
    if (r == c) x += sigma;
    t[lc][tx] = x;
    if (r < n && c < n && r >= c) B[c * ldb + r] = x;
  }
  if (!full) return;
  __syncthreads();
  for (int lr = ty; lr < 64; lr += 4) {  // row r0 + lr of the lower tile is a column of the upper one
    const int64_t cc = r0 + lr, rr = c0 + tx;
    if (cc < n && rr < cc) B[cc * ldb + rr] = t[tx][lr];
  }
}

void add_outer(hipStream_t s, int64_t n, const double* A, int64_t lda, int k, const double* Z, double alpha,
               double sigma, double* B, int64_t ldb, bool full) {
  if (n <= 0) return;
  RPF_CHECK(k <= 8, RPF_EINVAL, "add_outer: more than 8 columns");
  hipLaunchKernelGGL(k_add_outer, dim3((unsigned)cdiv(n, 64), (unsigned)cdiv(n, 64)), dim3(256), 0, s, n, A, lda, k, Z,
                     alpha, sigma, B, ldb, full ? 1 : 0);
  RPF_LAUNCH_CHECK();
}

// ============================================================================ triangular solves
// up_b = (lo_b)^T for the bw x bw blocks of the inverses, 64 x 64 tiles through LDS
__global__ __launch_bounds__(256) void k_transpose_blocks(int64_t bw, const double* lo, double* up) {
  __shared__ double t[64][65];
  const double* x = lo + (int64_t)blockIdx.z * bw * bw;
  double* y = up + (int64_t)blockIdx.z * bw * bw;
  const int64_t r0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int c = ty; c < 64; c += 4) t[c][tx] = x[(c0 + c) * bw + r0 + tx];
  __syncthreads();
  for (int r = ty; r < 64; r += 4) y[(r0 + r) * bw + c0 + tx] = t[tx][r];
}

void build_tri_inv(hipStream_t s, const double* L, int64_t ldl, int64_t n, const double* dinv, TriInv& inv) {
  if (n <= 0) return;
  const int64_t nb = cdiv(n, TRI_BW), len = nb * TRI_BW * TRI_BW;
  inv.lo.ensure((size_t)len);
  inv.up.ensure((size_t)len);
  // the joined blocks below the diagonal fit in the slab of the transposes until those are made
  static_assert(TRI_BW == 4 * NB, "scratch of the last level: half a slab a pair");
  fill(s, inv.lo.p, len, 0.0);
  invert_blocks(s, L, ldl, n, dinv, inv.lo.p, TRI_BW, inv.up.p);
  hipLaunchKernelGGL(k_transpose_blocks, dim3(TRI_BW / 64, TRI_BW / 64, (unsigned)nb), dim3(256), 0, s, TRI_BW,
                     inv.lo.p, inv.up.p);
  RPF_LAUNCH_CHECK();
}

// C (M x c) = beta C + alpha op(A) X with few columns (16 per workgroup): a workgroup takes
// 16 R rows, its W waves a part of K each, 32 k at a time with the next 32 on their way, and the
// W partial results are added in LDS.  TA: op(A) = A^T, A stored K x M.  X(k, j) is X[k xk + j xj], C(m, j)
// is C[m cm + j cj].  A walk over a 512-row block
// is four load latencies a wave (5 us at 6,700 rows and 8 columns), where the general product has 32
// dependent k-stages of 16 (14 to 17 us at K = 128 alone).
template <bool TA, int R, int W>
__global__ __launch_bounds__(64 * W) void k_skinny(int64_t M, int64_t c, int64_t K, double alpha, const double* A,
                                                int64_t lda, const double* X, int64_t xk, int64_t xj, double beta,
                                                double* C, int64_t cm, int64_t cj) {
  constexpr int U = 8;  // MFMA steps of a batch
  __shared__ double red[W][16 * R][17];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int fl = lane & 15, fk = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.x * 16 * R, c0 = (int64_t)blockIdx.y * 16;
  const int64_t kc = (K + 8 * W - 1) / (8 * W) * 8;  // a wave's part
  const int64_t kb = min(w * kc, K), ke = min(kb + kc, K);
  const double* Xc = X + min(c0 + fl, c - 1) * xj;
  const double* Ar[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int64_t m = min(m0 + 16 * i + fl, M - 1);
    Ar[i] = TA ? A + m * lda : A + m;
  }
  v4d acc[R];
#pragma unroll
  for (int i = 0; i < R; ++i) acc[i] = v4d{0.0, 0.0, 0.0, 0.0};
  double a[R][U], x[U], na[R][U], nx[U];
  auto load = [&](int64_t k0, double (&pa)[R][U], double (&px)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + 4 * u + fk, kk = min(k, K - 1);
#pragma unroll
      for (int i = 0; i < R; ++i) pa[i][u] = TA ? Ar[i][kk] : Ar[i][kk * lda];
      px[u] = Xc[kk * xk];
    }
  };
  if (kb < ke) load(kb, a, x);
  for (int64_t k0 = kb; k0 < ke; k0 += 4 * U) {
    const bool more = k0 + 4 * U < ke;
    if (more) load(k0 + 4 * U, na, nx);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = k0 + 4 * u + fk < ke;
#pragma unroll
      for (int i = 0; i < R; ++i)
        acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? x[u] : 0.0, in ? a[i][u] : 0.0, acc[i], 0, 0, 0);
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u] = nx[u];
#pragma unroll
        for (int i = 0; i < R; ++i) a[i][u] = na[i][u];
      }
    }
  }
  // item r of lane l: column l / 16 + 4 r, row l % 16
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[w][16 * i + fl][fk + 4 * r] = acc[i][r];
  __syncthreads();
  for (int e = tid; e < 256 * R; e += 64 * W) {
    const int row = e & (16 * R - 1), col = e / (16 * R);
    if (m0 + row < M && c0 + col < c) {
      double v = red[0][row][col];
#pragma unroll
      for (int q = 1; q < W; ++q) v += red[q][row][col];
      v *= alpha;
      double* o = C + (c0 + col) * cj + (m0 + row) * cm;
      *o = beta == 0.0 ? v : v + beta * *o;
    }
  }
}

// Two row tiles a workgroup where that still gives every CU one, else one.
static void launch_skinny(hipStream_t s, bool ta, int64_t M, int64_t c, int64_t K, double alpha, const double* A,
                          int64_t lda, const double* X, int64_t xk, int64_t xj, double beta, double* C, int64_t cm,
                          int64_t cj) {
  const bool two = cdiv(M, 32) * cdiv(c, 16) >= 256;
  // waves that share a row block's K: more of them while the chip has room and each still gets 16 k (an application
  // with 888 rows and 81 columns, 336 workgroups: 25.2 us with 4 waves, 28.7 with 16; the coarse solve of 384 unknowns,
  // 24 workgroups: the projection 22.8 us with 4, 21.5 with 16)
  const int w = (int64_t)cdiv(M, two ? 32 : 16) * cdiv(c, 16) > 256 || K < 256 ? 4 : 16;
  const dim3 g((unsigned)cdiv(M, two ? 32 : 16), (unsigned)cdiv(c, 16));
#define RPF_SK(TA, R, W) \
  RPF_TIMED_LAUNCH((k_skinny<TA, R, W>), g, dim3(64 * W), 0, s, M, c, K, alpha, A, lda, X, xk, xj, beta, C, cm, cj)
  if (ta) {
    if (two) RPF_SK(true, 2, 4);
    else if (w == 4) RPF_SK(true, 1, 4);
    else RPF_SK(true, 1, 16);
  } else {
    if (two) RPF_SK(false, 2, 4);
    else if (w == 4) RPF_SK(false, 1, 4);
    else RPF_SK(false, 1, 16);
  }
#undef RPF_SK
  RPF_LAUNCH_CHECK();
}

// up to this many columns k_skinny is the faster one (64 x 64 tiles re-read less of A above): an application with 888
// rows takes 26.7 us at 96 columns, and 34.3 on the tiles at 104; with 486 rows 23.6 and 54.3
constexpr int64_t SKINNY = 96;
void few_columns(hipStream_t s, bool ta, int64_t M, int64_t c, int64_t K, double alpha, const double* A, int64_t lda,
                 const double* X, int64_t ldx, double beta, double* C, int64_t ldc) {
  if (M <= 0 || c <= 0 || K <= 0) return;
  if (c > SKINNY) dgemm(s, ta, false, M, c, K, alpha, A, lda, X, ldx, beta, C, ldc);
  else launch_skinny(s, ta, M, c, K, alpha, A, lda, X, 1, ldx, beta, C, 1, ldc);
}

void few_columns_rows(hipStream_t s, int64_t M, int64_t c, int64_t K, const double* A, int64_t lda, const double* X,
                      int64_t ldx, double* C, int64_t ldc) {
  if (M > 0 && c > 0 && K > 0) launch_skinny(s, false, M, c, K, 1.0, A, lda, X, ldx, 1, 0.0, C, ldc, 1);
}

// the lower triangle of an n x n block, zeros above
__global__ void k_copy_lower(int64_t n, const double* A, int64_t lda, double* B, int64_t ldb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * n) {
    const int64_t r = i % n, c = i / n;
    B[c * ldb + r] = r >= c ? A[c * lda + r] : 0.0;
  }
}

// The serial chain of a solve is its diagonal blocks: they are taken TRI_BW = 512 rows at a time through
// explicit inverses, two launches each (X_T = inv(L_TT) B_T, then the rows below in the envelope).
// The forward solution goes to a second buffer and the backward one returns to B, so nothing is
// copied; more columns than the buffer's bound are taken in turn.  Many columns of a banded factor instead take
// one persistent pass each way.
// refine: each block's solution is corrected once by its residual, X += inv(L_TT) (B_T - L_TT X), which leaves a
// residual of the substitution's size for any condition of the block; without it the residual grows with that
// (random matrices of 700 rows, condition 1e11: 1.3 eps |A| |X| against 0.34; interior stiffnesses: no larger than
// with 64-row inverses, 0.27 and 0.28).
void potrs(hipStream_t s, const double* L, int64_t ldl, int64_t n, const double* dinv, const TriInv& inv,
           const Envelope& env, double* B, int64_t ldb, int64_t nrhs, bool upper, bool refine) {
  if (n <= 0 || nrhs <= 0) return;
  const int64_t nblk = cdiv(n, NB);
  bool dense = true;
  for (int64_t t = 0; t < nblk && dense; ++t) dense = env.cstart[t] <= 0 && env.rend[t] >= n;
  if (!dense && nrhs >= 2048) {
    std::vector<int64_t> bounds(2 * nblk);
    for (int64_t t = 0; t < nblk; ++t) {
      bounds[t] = env.cstart[t];
      bounds[nblk + t] = env.rend[t];
    }
    DevBuf<int64_t> db;
    db.upload(bounds.data(), bounds.size(), s);
    // 16 columns per workgroup, two workgroups per CU, where the band of L (or of the mirrored L^T)
    // is read sixteen rows at a time: 12.7 ms each way at 8192 columns of the 20^3 pattern (32
    // columns, one workgroup per CU: 14 ms forward, 14.3 ms backward).  Without the mirror the
    // backward reads columns of L, and 32 columns per workgroup halve that less efficient band
    // traffic (15.5 ms; 21 ms at 16).
    hipLaunchKernelGGL((k_trsm_panel<true, 1>), dim3((unsigned)cdiv(nrhs, 16)), dim3(256), 0, s, L, ldl, n, dinv, db.p,
                       db.p + nblk, B, ldb, nrhs);
    if (upper)
      hipLaunchKernelGGL((k_trsm_panel<false, 1, true>), dim3((unsigned)cdiv(nrhs, 16)), dim3(256), 0, s, L, ldl, n,
                         dinv, db.p, db.p + nblk, B, ldb, nrhs);
    else
      hipLaunchKernelGGL((k_trsm_panel<false, 2>), dim3((unsigned)cdiv(nrhs, 32)), dim3(256), 0, s, L, ldl, n, dinv,
                         db.p, db.p + nblk, B, ldb, nrhs);
    RPF_LAUNCH_CHECK();
    RPF_HIP(hipStreamSynchronize(s));  // the bounds buffer is freed on return
    return;
  }
  // at most 512 MB of second buffer, at least 512 columns at a time, at most a grid's; one NB block needs its own inverse only (and
  // no correction up to 64 rows, which were one block of the 64-row inverses)
  const int64_t most = std::min<int64_t>((int64_t)1 << 22, std::max<int64_t>(512, ((int64_t)1 << 26) / n));
  const int64_t nT = cdiv(n, TRI_BW), per = TRI_BW / NB;
  DevBuf<double> F((size_t)n * std::min(nrhs, most)), Lt, Rt;
  refine = refine && n > 64;
  if (refine) {
    Lt.alloc((size_t)TRI_BW * TRI_BW);
    Rt.alloc((size_t)TRI_BW * std::min(nrhs, most));
  }
  for (int64_t c0 = 0; c0 < nrhs; c0 += most, B += most * ldb) {
    const int64_t nc = std::min(most, nrhs - c0);
    // X = op(L_TT)^{-1} Y for the jb rows of block t
    auto block = [&](bool back, int64_t t, int64_t jb, const double* Y, int64_t ldy, double* X, int64_t ldx) {
      // op(L_TT)^{-1} as it is stored: dinv holds it by rows
      const bool one = n <= NB, ta = one && !back;
      const double* inv_t = one ? dinv : (back ? inv.up.p : inv.lo.p) + t * TRI_BW * TRI_BW;
      const int64_t ldi = one ? NB : TRI_BW;
      few_columns(s, ta, jb, nc, jb, 1.0, inv_t, ldi, Y, ldy, 0.0, X, ldx);
      if (!refine) return;
      const int64_t j0 = t * TRI_BW;
      hipLaunchKernelGGL(k_copy_lower, dim3((unsigned)cdiv(jb * jb, 256)), dim3(256), 0, s, jb, L + j0 * ldl + j0, ldl, Lt.p,
                         TRI_BW);
      RPF_LAUNCH_CHECK();
      copy_matrix(s, Y, ldy, Rt.p, TRI_BW, jb, nc);
      few_columns(s, back, jb, nc, jb, -1.0, Lt.p, TRI_BW, X, ldx, 1.0, Rt.p, TRI_BW);
      few_columns(s, ta, jb, nc, jb, 1.0, inv_t, ldi, Rt.p, TRI_BW, 1.0, X, ldx);
    };
    for (int64_t t = 0; t < nT; ++t) {
      const int64_t j0 = t * TRI_BW, jb = std::min(TRI_BW, n - j0), r0 = j0 + jb;
      const int64_t rend = std::min(env.rend[std::min((t + 1) * per, nblk) - 1], n);
      block(false, t, jb, B + j0, ldb, F.p + j0, n);
      few_columns(s, false, rend - r0, nc, jb, -1.0, L + j0 * ldl + r0, ldl, F.p + j0, n, 1.0, B + r0, ldb);
    }
    for (int64_t t = nT - 1; t >= 0; --t) {
      const int64_t j0 = t * TRI_BW, jb = std::min(TRI_BW, n - j0);
      int64_t cs = j0;
      for (int64_t q = t * per; q < std::min((t + 1) * per, nblk); ++q) cs = std::min(cs, std::max<int64_t>(0, env.cstart[q]));
      block(true, t, jb, F.p + j0, n, B + j0, ldb);
      few_columns(s, !upper, j0 - cs, nc, jb, -1.0, upper ? L + j0 * ldl + cs : L + cs * ldl + j0, ldl, B + j0, ldb, 1.0,
                  F.p + cs, n);
    }
  }
  RPF_HIP(hipStreamSynchronize(s));  // the second buffer is freed on return
}

// ============================================================================ elementwise helpers
__global__ void k_fill(double* p, int64_t count, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

__global__ void k_copy_matrix(const double* src, int64_t lds, double* dst, int64_t ldd, int64_t rows, int64_t cols) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < rows * cols) {
    const int64_t r = i % rows, c = i / rows;
    dst[c * ldd + r] = src[c * lds + r];
  }
}

__global__ void k_mirror_lower(double* A, int64_t lda, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * n) {
    const int64_t r = i % n, c = i / n;
    if (r < c) A[c * lda + r] = A[r * lda + c];
  }
}

void fill(hipStream_t s, double* p, int64_t count, double v) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)cdiv(count, 256)), dim3(256), 0, s, p, count, v);
  RPF_LAUNCH_CHECK();
}

void copy_matrix(hipStream_t s, const double* src, int64_t lds, double* dst, int64_t ldd, int64_t rows,
                 int64_t cols) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(k_copy_matrix, dim3((unsigned)cdiv(rows * cols, 256)), dim3(256), 0, s, src, lds, dst, ldd,
                     rows, cols);
  RPF_LAUNCH_CHECK();
}

// One 64 x 64 tile of column block t (blockIdx.y), rows r0 = t 64 + 64 blockIdx.x up to rend[t]: read
// down the columns, written along the rows (both coalesced, through LDS); only entries below the
// diagonal are copied, so the lower triangle is untouched.
__global__ __launch_bounds__(256) void k_mirror_env(double* A, int64_t lda, int64_t n, const int64_t* rend) {
  __shared__ double t[64][65];
  const int64_t j0 = (int64_t)blockIdx.y * 64;
  const int64_t r0 = j0 + (int64_t)blockIdx.x * 64;
  const int64_t re = min(rend[blockIdx.y], n);
  if (r0 >= re) return;
  const int jb = (int)min<int64_t>(64, n - j0);
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int c = ty; c < jb; c += 4) {
    const int64_t r = r0 + tx;
    t[c][tx] = r < re ? A[r + (j0 + c) * lda] : 0.0;
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t r = r0 + i;
    const int c = tx;
    if (r < re && c < jb && r > j0 + c) A[(j0 + c) + r * lda] = t[c][i];
  }
}

void mirror_envelope(hipStream_t s, double* A, int64_t lda, int64_t n, const Envelope& env) {
  if (n <= 0) return;
  const int64_t nblk = cdiv(n, 64);  // the kernel's 64-column tiles, each with the rows of its NB block
  RPF_CHECK((int64_t)env.rend.size() >= cdiv(n, NB), RPF_EINVAL, "mirror_envelope: envelope too short");
  std::vector<int64_t> re(nblk);
  int64_t tiles = 1;
  for (int64_t t = 0; t < nblk; ++t) {
    re[t] = env.rend[t * 64 / NB];
    tiles = std::max<int64_t>(tiles, cdiv(std::min(re[t], n) - t * 64, 64));
  }
  DevBuf<int64_t> d;
  d.upload(re.data(), re.size(), s);
  hipLaunchKernelGGL(k_mirror_env, dim3((unsigned)tiles, (unsigned)nblk), dim3(256), 0, s, A, lda, n, d.p);
  RPF_LAUNCH_CHECK();
  RPF_HIP(hipStreamSynchronize(s));  // the bounds buffer is freed on return
}

void mirror_lower(hipStream_t s, double* A, int64_t lda, int64_t n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_mirror_lower, dim3((unsigned)cdiv(n * n, 256)), dim3(256), 0, s, A, lda, n);
  RPF_LAUNCH_CHECK();
}

// ============================================================================ small eigenproblems
// Parallel cyclic Jacobi (Brent-Luk ordering: m/2 disjoint rotations per step,
// m-1 steps per sweep), one workgroup per matrix, m <= 64.
constexpr int EIG_MAX = 64;

struct JacobiShared {
  int pp[EIG_MAX / 2], qq[EIG_MAX / 2], order[EIG_MAX], nrot;
  double cc[EIG_MAX / 2], ss[EIG_MAX / 2], floor_abs;
};
// Eigenpairs of the symmetric m x m matrix a (row stride ld, LDS), by every thread of the workgroup:
// the eigenvalues are left on its diagonal, the vectors in the columns of v (the identity on entry),
// their ascending order in sh.order.
__device__ void jacobi_eigen(double* a, double* v, int ld, int m, JacobiShared& sh) {
  const int tid = threadIdx.x, nth = blockDim.x;
  const int me = m + (m & 1);  // even count for the round-robin schedule
  const int npair = me / 2;
  __syncthreads();
  // threshold Jacobi: a pair is rotated only while |a_pq| > 1e-13 sqrt(|a_pp a_qq|) (relative
  // accuracy of the eigenvalues to about 1e-13, ample for eta^{-1/2}) and |a_pq| > 1e-15
  // max_i |a_ii| (eigenvalues below 1e-12 of the largest are dropped by the caller, and
  // below this floor a rotation only moves rounding noise); the sweeps stop once a whole
  // sweep rotates nothing
  for (int sweep = 0; sweep < 30 && m >= 2; ++sweep) {
    if (tid == 0) {
      sh.nrot = 0;
      double d = 0.0;
      for (int i = 0; i < m; ++i) d = fmax(d, fabs(a[(i) * ld + (i)]));
      sh.floor_abs = fmax(1e-15 * d, 1e-300);
    }
    __syncthreads();
    for (int step = 0; step < me - 1; ++step) {
      // circle method: indices 0..me-2 rotate, me-1 is fixed
      if (tid < npair) {
        int i, j;
        if (tid == 0) {
          i = step;
          j = me - 1;
        } else {
          i = (step + tid) % (me - 1);
          j = (step - tid + (me - 1)) % (me - 1);
        }
        const int p = i < j ? i : j, q = i < j ? j : i;
        double c = 1.0, sn = 0.0;
        if (q < m) {
          const double apq = a[(p) * ld + (q)];
          if (fabs(apq) > 1e-13 * sqrt(fabs(a[(p) * ld + (p)] * a[(q) * ld + (q)])) && fabs(apq) > sh.floor_abs) {
            atomicAdd(&sh.nrot, 1);
            const double theta = (a[(q) * ld + (q)] - a[(p) * ld + (p)]) / (2.0 * apq);
            const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(1.0 + theta * theta));
            c = 1.0 / sqrt(1.0 + t * t);
            sn = t * c;
          }
        }
        sh.pp[tid] = p;
        sh.qq[tid] = q;
        sh.cc[tid] = c;
        sh.ss[tid] = sn;
      }
      __syncthreads();
      // columns: A <- A J, V <- V J
      for (int idx = tid; idx < npair * m; idx += nth) {
        const int k = idx / m, r = idx % m;
        const int p = sh.pp[k], q = sh.qq[k];
        if (q >= m) continue;
        const double c = sh.cc[k], sn = sh.ss[k];
        const double x = a[(r) * ld + (p)], y = a[(r) * ld + (q)];
        a[(r) * ld + (p)] = c * x - sn * y;
        a[(r) * ld + (q)] = sn * x + c * y;
        const double vx = v[(r) * ld + (p)], vy = v[(r) * ld + (q)];
        v[(r) * ld + (p)] = c * vx - sn * vy;
        v[(r) * ld + (q)] = sn * vx + c * vy;
      }
      __syncthreads();
      // rows: A <- J^T A
      for (int idx = tid; idx < npair * m; idx += nth) {
        const int k = idx / m, col = idx % m;
        const int p = sh.pp[k], q = sh.qq[k];
        if (q >= m) continue;
        const double c = sh.cc[k], sn = sh.ss[k];
        const double x = a[(p) * ld + (col)], y = a[(q) * ld + (col)];
        a[(p) * ld + (col)] = c * x - sn * y;
        a[(q) * ld + (col)] = sn * x + c * y;
      }
      __syncthreads();
    }
    if (sh.nrot == 0) break;  // uniform: read after the last barrier of the sweep
    __syncthreads();
  }
  __syncthreads();
  if (tid == 0) {
    for (int i = 0; i < m; ++i) sh.order[i] = i;
    for (int i = 0; i < m; ++i) {
      int best = i;
      for (int j = i + 1; j < m; ++j)
        if (a[(sh.order[j]) * ld + (sh.order[j])] < a[(sh.order[best]) * ld + (sh.order[best])]) best = j;
      const int t = sh.order[i];
      sh.order[i] = sh.order[best];
      sh.order[best] = t;
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(256) void k_syev_jacobi(const double* Ain, int m, double* Vout, double* wout) {
  __shared__ double a[EIG_MAX * (EIG_MAX + 1)];
  __shared__ double v[EIG_MAX * (EIG_MAX + 1)];
  __shared__ JacobiShared sh;
  const int ld = EIG_MAX + 1;
  const double* A = Ain + (int64_t)blockIdx.x * m * m;
  double* V = Vout + (int64_t)blockIdx.x * m * m;
  double* w = wout + (int64_t)blockIdx.x * m;
  for (int i = threadIdx.x; i < m * m; i += blockDim.x) {
    const int r = i % m, c = i / m;
    a[r * ld + c] = 0.5 * (A[c * m + r] + A[r * m + c]);
    v[r * ld + c] = (r == c) ? 1.0 : 0.0;
  }
  jacobi_eigen(a, v, ld, m, sh);
  for (int i = threadIdx.x; i < m * m; i += blockDim.x) {
    const int r = i % m, c = i / m;
    V[c * m + r] = v[r * ld + sh.order[c]];
  }
  for (int i = threadIdx.x; i < m; i += blockDim.x) w[i] = a[sh.order[i] * (ld + 1)];
}

void syev_small(hipStream_t s, const double* A, int m, double* V, double* w, int batch) {
  RPF_CHECK(m >= 1 && m <= EIG_MAX, RPF_EINVAL, "syev_small: m out of range");
  // one wavefront is enough (and its barriers are cheapest) while m/2 * m <= 128 work items
  const int threads = (m <= 16) ? 64 : 256;
  hipLaunchKernelGGL(k_syev_jacobi, dim3(batch), dim3(threads), 0, s, A, m, V, w);
  RPF_LAUNCH_CHECK();
}

// LDS written by one lane of a wavefront, read by others of it
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The small matrices of a block step, in one workgroup.  Normalisation of the new block (section 3.3): T
// with T^T eta T = I on the kept directions.
// The energy of column c before the orthogonalisation is |B_c|^2 + eta_cc (B = P_stored^T Z,
// ka x m, ld ka; F-orthonormal stored blocks).  Diagonal form (classical CG per load case):
// T = diag(eta_cc^{-1/2}) keeping eta_cc > tau * energy_c.  Block form: the eigen rule keeps w_i >
// tau * max(w_max, max_c energy_c); when a Cholesky factor eta = L L^T exists with
// 1 / |L^{-1}|_F^2 (a lower bound of w_min) above tau * max(trace eta, max_c energy_c) (an upper
// bound of that reference), no eigenpair would be dropped and T = L^{-T} spans the same
// directions, so it is used; otherwise T = V diag(w^{-1/2}) over the kept eigenpairs.  When nothing is
// kept, 1 goes to raised.  Then alpha = T (T^T zr) (m x nr; the diagonal of T^T zr only in the
// diagonal form), to one or two places.  MM >= m is the unrolled register length; the first wave forms
// T, the four of them the eigenpairs and the products (as separate launches, these took 4.5 us each).
template <int MM>
__global__ __launch_bounds__(256) void k_block_coef(int m, int nr, const double* eta, const double* zr, int diag_only,
                                                    int ka, const double* B, double tau, double* T, int* drops,
                                                    double* raised, double* alpha, double* alpha2) {
  __shared__ double epre[64];
  __shared__ double Ls[MM][MM + 1];  // the factor; the Jacobi iteration's matrix
  __shared__ double Vs[MM][MM + 1];  // its vectors; T^T zr
  __shared__ double es[MM * MM];     // eta; T
  __shared__ double zs[MM * MM];
  __shared__ double rdiag[MM];
  __shared__ JacobiShared sh;
  __shared__ double emax_s, trace_s;
  __shared__ int bad_s, ok_s, kept_s;
  const int tid = threadIdx.x, t = tid & 63, wave = tid >> 6;
  for (int e = tid; e < m * nr; e += 256) zs[e] = zr[e];
  if (wave == 0) {
  // eta staged in LDS, and B read, by loads at clamped (always valid) addresses whose values are
  // masked afterwards: no load sits behind a branch, so each group is issued together and waited
  // for once instead of one global-memory round trip at a time
  {
    constexpr int EU = (MM * MM + 63) / 64;
    double ev[EU];
    const int mm = m * m;
#pragma unroll
    for (int u = 0; u < EU; ++u) ev[u] = eta[min(t + 64 * u, mm - 1)];
#pragma unroll
    for (int u = 0; u < EU; ++u)
      if (t + 64 * u < MM * MM) es[t + 64 * u] = (t + 64 * u < mm) ? ev[u] : 0.0;
  }
  wave_sync();
  {
    // squared column norms of B: every column's loads of a 64-row chunk are issued together
    double part[MM];
#pragma unroll
    for (int c = 0; c < MM; ++c) part[c] = 0.0;
    for (int i0 = 0; i0 < ka; i0 += 64) {
      const int i = i0 + t;
      const int ic = min(i, ka - 1);
      double bv[MM];
#pragma unroll
      for (int c = 0; c < MM; ++c) bv[c] = B[(int64_t)min(c, m - 1) * ka + ic];
#pragma unroll
      for (int c = 0; c < MM; ++c) {
        const double b = (c < m && i < ka) ? bv[c] : 0.0;
        part[c] += b * b;
      }
    }
    // lane t holds eta_tt; every reduction below is a butterfly across the wave (no serial loops
    // of dependent loads on one lane)
    const double dg = t < m ? es[t * m + t] : 0.0;
    // all MM butterflies in straight-line code (columns past m are zeros), so they interleave
    double mine = 0.0;
#pragma unroll
    for (int c = 0; c < MM; ++c) {
      double acc = part[c];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
      acc += __shfl(dg, c, 64);
      if (t == c) mine = acc;
    }
    if (t < m) epre[t] = mine;
    double me = mine, tr = fmax(dg, 0.0);
    for (int off = 32; off > 0; off >>= 1) {
      me = fmax(me, __shfl_xor(me, off, 64));
      tr += __shfl_xor(tr, off, 64);
    }
    if (t == 0) {
      emax_s = me;
      trace_s = tr;
      bad_s = 0;
    }
  }
  wave_sync();
  if (diag_only) {
    bool keep = false;
    if (t < m) {
      const double wi = es[t * m + t];
      keep = wi > 0.0 && wi > tau * epre[t];
      if (!keep) atomicAdd(drops, 1);
    }
    const bool any = __any(keep);
    const double tc = keep ? 1.0 / sqrt(es[t * m + t]) : 0.0;
    wave_sync();
    for (int i = t; i < m * m; i += 64) {
      es[i] = 0.0;
      T[i] = 0.0;
    }
    wave_sync();
    if (t < m) {
      es[t * m + t] = tc;
      T[t * m + t] = tc;
    }
    if (t == 0) {
      if (!any) raised[0] = 1.0;
      ok_s = 1;
    }
  } else {
  // Cholesky, lane t owns row t
  double a[MM];
#pragma unroll
  for (int c = 0; c < MM; ++c) a[c] = (t < m && c < m && c <= t) ? 0.5 * (es[c * m + t] + es[t * m + c]) : 0.0;
  // (fully unrolled with compile-time indices into a[]: a loop left with a runtime bound would index
  // the register array dynamically; the column of L is read from LDS in one independent batch)
#pragma unroll
  for (int j = 0; j < MM; ++j) {
    if (j < m) {
      if (t == j) {
        double d = a[j];
        if (!(d > 0.0)) {
          bad_s = 1;
          d = 1.0;
        }
        a[j] = sqrt(d);
        rdiag[j] = 1.0 / a[j];
      }
      wave_sync();
      if (t > j && t < m) {
        a[j] *= rdiag[j];
        Ls[t][j] = a[j];
      }
      wave_sync();
      double lc[MM];
#pragma unroll
      for (int c = j + 1; c < MM; ++c) lc[c] = Ls[c][j];
      if (t > j && t < m) {
        const double ltj = a[j];
#pragma unroll
        for (int c = j + 1; c < MM; ++c)
          if (c <= t) a[c] -= ltj * lc[c];
      }
    }
  }
  wave_sync();
  // column t of L^{-1}, right-looking
  double x[MM];
#pragma unroll
  for (int r = 0; r < MM; ++r) x[r] = (r == t) ? 1.0 : 0.0;
#pragma unroll
  for (int k = 0; k < MM; ++k) {
    if (k < m) {
      x[k] *= rdiag[k];
      const double xk = x[k];
#pragma unroll
      for (int r = k + 1; r < MM; ++r)
        if (r < m) x[r] -= Ls[r][k] * xk;
    }
  }
  double fro = 0.0;
#pragma unroll
  for (int r = 0; r < MM; ++r) fro += (t < m && r < m) ? x[r] * x[r] : 0.0;
  for (int off = 32; off > 0; off >>= 1) fro += __shfl_xor(fro, off, 64);
  const double ref_up = fmax(trace_s, emax_s);
  const bool ok = bad_s == 0 && fro > 0.0 && (1.0 / fro) > tau * ref_up;
  if (ok && t < m) {
    // T = L^{-T}: T[c + m r] = (L^{-1})[r][c] = x[r] of lane c
#pragma unroll
    for (int r = 0; r < MM; ++r)
      if (r < m) {
        T[t + (int64_t)m * r] = x[r];
        es[t + m * r] = x[r];
      }
  }
  if (t == 0) ok_s = ok ? 1 : 0;
  }
  }
  __syncthreads();
  if (!ok_s) {
    // the factor did not settle it: eigenpairs of eta
    for (int i = tid; i < m * m; i += 256) {
      const int r = i % m, c = i / m;
      Ls[r][c] = 0.5 * (eta[c * m + r] + eta[r * m + c]);
      Vs[r][c] = (r == c) ? 1.0 : 0.0;
    }
    if (tid == 0) kept_s = 0;
    jacobi_eigen(&Ls[0][0], &Vs[0][0], MM + 1, m, sh);
    const double ref = fmax(Ls[sh.order[m - 1]][sh.order[m - 1]], emax_s);
    if (tid < m) {
      const double wi = Ls[sh.order[tid]][sh.order[tid]];
      const bool keep = wi > 0.0 && wi > tau * ref;
      rdiag[tid] = keep ? 1.0 / sqrt(wi) : 0.0;
      if (keep) atomicAdd(&kept_s, 1);
      else atomicAdd(drops, 1);
    }
    __syncthreads();
    if (tid == 0 && kept_s == 0) raised[0] = 1.0;
    for (int i = tid; i < m * m; i += 256) {
      const int r = i % m, c = i / m;
      const double v = Vs[r][sh.order[c]] * rdiag[c];
      T[c * m + r] = v;
      es[c * m + r] = v;
    }
    __syncthreads();
  }
  double* gs = &Vs[0][0];
  for (int e = tid; e < m * nr; e += 256) {
    const int r = e % m, col = e / m;
    double v = 0.0;
    if (!diag_only || r == col)
      for (int k = 0; k < m; ++k) v += es[k + r * m] * zs[k + col * m];
    gs[e] = v;
  }
  __syncthreads();
  for (int e = tid; e < m * nr; e += 256) {
    const int r = e % m, col = e / m;
    double v = 0.0;
    for (int k = 0; k < m; ++k) v += es[r + k * m] * gs[k + col * m];
    alpha[e] = v;
    if (alpha2) alpha2[e] = v;
  }
}

void block_coef(hipStream_t s, int m, int nr, const double* eta, const double* zr, bool diag_only, int ka,
                const double* B, double tau, double* T, int* drops, double* raised, double* alpha, double* alpha2) {
  RPF_CHECK(m >= 1 && m <= EIG_MAX && nr <= m, RPF_EINVAL, "block_coef: block width");
#define RPF_BC(MM)                                                                                                   \
  hipLaunchKernelGGL(k_block_coef<MM>, dim3(1), dim3(256), 0, s, m, nr, eta, zr, diag_only ? 1 : 0, ka, B, tau, T, drops, \
                     raised, alpha, alpha2)
  if (m <= 8) RPF_BC(8);
  else if (m <= 16) RPF_BC(16);
  else if (m <= 32) RPF_BC(32);
  else RPF_BC(64);
#undef RPF_BC
  RPF_LAUNCH_CHECK();
}

// ============================================================================ orthonormalisation
__device__ inline double block_sum(double v, double* red) {
  const int tid = threadIdx.x;
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double t = 0.0;
  if (tid == 0) {
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
    red[16] = t;
  }
  __syncthreads();
  t = red[16];
  __syncthreads();
  return t;
}

__global__ __launch_bounds__(1024) void k_mgs2(double* Y, int64_t n, int64_t ld, int k) {
  __shared__ double red[17];
  const int tid = threadIdx.x;
  for (int j = 0; j < k; ++j) {
    double* yj = Y + (int64_t)j * ld;
    for (int pass = 0; pass < 2; ++pass) {
      for (int i = 0; i < j; ++i) {
        const double* yi = Y + (int64_t)i * ld;
        double d = 0.0;
        for (int64_t r = tid; r < n; r += blockDim.x) d += yi[r] * yj[r];
        d = block_sum(d, red);
        for (int64_t r = tid; r < n; r += blockDim.x) yj[r] -= d * yi[r];
        __syncthreads();
      }
    }
    double nn = 0.0;
    for (int64_t r = tid; r < n; r += blockDim.x) nn += yj[r] * yj[r];
    nn = block_sum(nn, red);
    const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
    for (int64_t r = tid; r < n; r += blockDim.x) yj[r] *= inv;
    __syncthreads();
  }
}

__device__ inline double read_lane(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l), hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

// Sums over the workgroup of v[0..7] (NW waves), to every thread.  Halving exchanges leave each lane with
// one of the eight sums over its wave, so 13 cross-lane moves and one barrier serve all of them; the
// caller alternates between the two buffers.
template <int NW>
__device__ inline void block_sum8(const double (&v)[8], double (*red)[8], double (&out)[8]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double a[4], b[2], c;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool hi = lane & 32;
    a[i] = (hi ? v[i + 4] : v[i]) + __shfl_xor(hi ? v[i] : v[i + 4], 32, 64);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool hi = lane & 16;
    b[i] = (hi ? a[i + 2] : a[i]) + __shfl_xor(hi ? a[i] : a[i + 2], 16, 64);
  }
  {
    const bool hi = lane & 8;
    c = (hi ? b[1] : b[0]) + __shfl_xor(hi ? b[0] : b[1], 8, 64);
  }
#pragma unroll
  for (int off = 4; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((lane & 7) == 0) red[wave][lane >> 3] = c;
  __syncthreads();
  constexpr int G = NW < 8 ? NW : 8;
  double t = red[lane & (G - 1)][lane >> 3];
  if (NW > 8) t += red[8 + (lane & 7)][lane >> 3];
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
#pragma unroll
  for (int i = 0; i < 8; ++i) out[i] = read_lane(t, 8 * i);
}

// Up to 8 columns of at most T R rows in registers: classical Gram-Schmidt with every projection taken
// twice (as orthogonal as the modified form taken twice).  A column's norm is summed with the next one's first
// projection, so k columns are 2k - 1 reductions.  It is bound by them, and a reduction by the waves that share
// the LDS unit for its moves: 34 rows take 12 us in 4 waves (30 in 16 waves with a reduction for each norm),
// 888 rows 18 in 4 waves of 4 rows a lane, 2,598 rows 31 in 8 waves of 8 (32 in 16 waves of 4).
// The general kernel above re-reads the columns for each of its 64 reductions (160 us at 2,598 rows, 74 us at 64).
template <int T, int R>
__global__ __launch_bounds__(T) void k_gs2(double* Y, int64_t n, int64_t ld, int k) {
  __shared__ double red[2][T / 64][8];
  const int tid = threadIdx.x;
  double v[8][R];
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = tid + T * r;
      const double x = Y[(int64_t)min(j, k - 1) * ld + min(row, n - 1)];
      v[j][r] = (j < k && row < n) ? x : 0.0;
    }
  int buf = 0;
  double d[8], p[8];
  // column j to unit length, given its squared norm
  auto scale = [&](int j, double nn) {
    const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[j][r] *= inv;
      const int64_t row = tid + T * r;
      if (row < n) Y[(int64_t)j * ld + row] = v[j][r];
    }
    return inv;
  };
#pragma unroll
  for (int j = 1; j < 8; ++j) {
    if (j < k) {
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          p[i] = 0.0;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (i < j) p[i] += v[i][r] * v[j][r];
            else if (i == 7 && pass == 0) p[i] += v[j - 1][r] * v[j - 1][r];
          }
        }
        block_sum8<T / 64>(p, red[buf], d);
        buf ^= 1;
        if (pass == 0) d[j - 1] *= scale(j - 1, d[7]);
#pragma unroll
        for (int i = 0; i < j; ++i)
#pragma unroll
          for (int r = 0; r < R; ++r) v[j][r] -= d[i] * v[i][r];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j == k - 1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) p[0] += v[j][r] * v[j][r];
      block_sum8<T / 64>(p, red[buf], d);
      scale(j, d[0]);
    }
}

void orthonormalize(hipStream_t s, double* Y, int64_t n, int64_t ld, int k) {
  if (k <= 0 || n <= 0) return;
#define RPF_GS(T, R) hipLaunchKernelGGL((k_gs2<T, R>), dim3(1), dim3(T), 0, s, Y, n, ld, k)
  if (k <= 8 && n <= 512) RPF_GS(256, 2);
  else if (k <= 8 && n <= 1024) RPF_GS(256, 4);
  else if (k <= 8 && n <= 2048) RPF_GS(512, 4);
  else if (k <= 8 && n <= 4096) RPF_GS(512, 8);
  else hipLaunchKernelGGL(k_mgs2, dim3(1), dim3(1024), 0, s, Y, n, ld, k);
#undef RPF_GS
  RPF_LAUNCH_CHECK();
}

}  // namespace rpf
