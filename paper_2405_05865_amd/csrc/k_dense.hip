// Small dense FP64 work on s x s matrices: the Gram products C~^T C~ and A^^T A^
// (Algorithms 1 and 3), symmetric combinations, and the explicit
// SPD inverses M2^{-1}, M3a^{-1}, M3b^{-1} the algorithms precompute.
//
// The inverse is computed by block Gauss-Jordan sweeps without pivoting. For SPD M
// every pivot block is a Schur complement of M, hence SPD, so no pivoting is needed;
// each pivot block is factored by Cholesky (a non-positive pivot flags the matrix as
// not positive definite) and the Schur complements are formed in Cholesky form.
#include "msp_internal.h"

#include <hip/hip_bf16.h>

namespace {

constexpr int TILE = 64;

typedef double v4d __attribute__((ext_vector_type(4)));

// Gram partial: G_part[z] = X[rows of split z]^T X[rows of split z], lower 64 x 64 tiles,
// mirrored. Bound by the FP64 matrix cores (2 s^2 flops per row of X, half of them by the
// symmetry): a wavefront keeps a whole tile as 4 x 4 accumulators of 16x16x4 MFMA, so a step
// of four rows is eight 8-byte loads per lane (whole 128-byte lines per 16 lanes, from cache
// after the first tile) for sixteen MFMAs, and nothing is staged in LDS. The four wavefronts
// of a block take every fourth step of the split and their tiles are added in LDS in wavefront
// order. The Gram products of 32768 x 512 and 2048 x 512 together: 888 us with 4 x 4 register
// tiles on the vector units, 260 us with this (the matrix cores' own time is about 135 us).
template <class T>
__global__ void __launch_bounds__(256, 2) k_gram(const T* __restrict__ X, int64_t rows, int64_t s, int64_t ldx,
                                              int64_t rows_per_split, double* __restrict__ Gp) {
  __shared__ double sum[TILE][TILE + 1];
  // map blockIdx.x to a lower tile (ti >= tj)
  int t = blockIdx.x, ti = 0;
  while (t > ti) { t -= ti + 1; ++ti; }
  const int tj = t;
  const int64_t i0 = (int64_t)ti * TILE, j0 = (int64_t)tj * TILE;
  const int64_t rb = (int64_t)blockIdx.y * rows_per_split;
  const int64_t re = min(rows, rb + rows_per_split);
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64, c = lane & 15, g = lane >> 4;
  const T *pa[4], *pb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {  // columns beyond s repeat the last one and are not stored
    pa[q] = X + min(i0 + 16 * q + c, s - 1);
    pb[q] = X + min(j0 + 16 * q + c, s - 1);
  }
  v4d acc[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[p][q] = v4d{0, 0, 0, 0};
  auto load = [&](int64_t r, double(&a)[4], double(&b)[4]) {
    const bool ok = r + g < re;
    const int64_t o = min(r + g, rows - 1) * ldx;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = ok ? (double)pa[q][o] : 0.0;
      b[q] = ok ? (double)pb[q][o] : 0.0;
    }
  };
  double a[4], b[4];
  int64_t r = rb + 4 * w;
  if (r < re) load(r, a, b);
  for (; r < re; r += 16) {
    double na[4] = {}, nb[4] = {};
    if (r + 16 < re) load(r + 16, na, nb);  // the next step's loads are in flight meanwhile
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p], b[q], acc[p][q], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = na[q];
      b[q] = nb[q];
    }
  }
  // element e of lane (c, g) is tile row 4 e + g, column c
  for (int ww = 0; ww < 4; ++ww) {
    if (w == ww) {
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            double& d = sum[16 * p + 4 * e + g][16 * q + c];
            d = ww == 0 ? acc[p][q][e] : d + acc[p][q][e];
          }
    }
    __syncthreads();
  }
  double* G = Gp + (int64_t)blockIdx.y * s * s;
  for (int e = threadIdx.x; e < TILE * TILE; e += 256) {
    const int p = e / TILE, q = e % TILE;
    if (i0 + p < s && j0 + q < s) G[(i0 + p) * s + j0 + q] = sum[p][q];
    if (ti != tj && i0 + q < s && j0 + p < s) G[(j0 + p) * s + i0 + q] = sum[q][p];
  }
}

__global__ void k_sum_splits(const double* __restrict__ Gp, int splits, int64_t len, double* __restrict__ G) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= len) return;
  double acc = 0.0;
  for (int z = 0; z < splits; ++z) acc += Gp[(int64_t)z * len + i];
  G[i] = acc;
}

// out = sym(a P + b Q) + c I, one thread per unordered pair (safe in place)
__global__ void k_combine_sym(int64_t s, double a, const double* P, double b, const double* Q, double c,
                              double* out) {
  const int64_t i = blockIdx.y * (int64_t)blockDim.y + threadIdx.y;
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= s || j >= s || j > i) return;
  double v = 0.5 * a * (P[i * s + j] + P[j * s + i]);
  if (Q) v += 0.5 * b * (Q[i * s + j] + Q[j * s + i]);
  if (i == j) v += c;
  out[i * s + j] = v;
  out[j * s + i] = v;
}

__global__ void k_trace(int64_t s, const double* __restrict__ M, double* out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < s; i += 256) acc += M[i * s + i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

__global__ void k_add_diag_scaled(int64_t s, double* M, const double* tr, double rel) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < s) M[i * s + i] += rel * (*tr) / (double)s;
}

// One block Gauss-Jordan sweep over pivots K = [k0, k0 + nbk). Tile of 64 x 64 per block.
// The pivot block is factored X_KK = L L^T (Cholesky; a pivot <= 0 flags the matrix as not
// positive definite) and every product with X_KK^{-1} is taken through Li = L^{-1}:
//   X_KK <- Li^T Li,  X_KJ <- Li^T (Li X_KJ),  X_IK <- -(X_IK Li^T) Li,
//   X_IJ <- X_IJ - (X_IK Li^T)(Li X_KJ).
// The trailing update is then the Cholesky form of the Schur complement, whose error
// does not grow with the conditioning of X_KK (an explicit inverse of the pivot block
// there would lose the small trailing pivots of ill-conditioned SPD matrices).
//
// A step is bound by the serial chain through its pivot block, which every block repeats (a
// launch of its own would cost as much). One wavefront runs it without barriers: lane i holds
// row i in registers, the pivot and the multiplier of the next column (the critical chain) travel
// by lane reads, the other multipliers through LDS as broadcasts; the reciprocal square root of
// the pivot serves all divisions by it. The other wavefronts load the tile's rows and columns
// meanwhile. As a block-wide Cholesky with three barriers per column, and
// products reading both operands of every multiply-add from LDS, a step took 63 us at s = 512
// and s = 1024; this takes 19 and 22 us.
__device__ __forceinline__ double lane_read(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

template <int NB>
__global__ void __launch_bounds__(256) k_bgj_step(const double* __restrict__ in, double* __restrict__ out, int s,
                                                  int k0, int32_t* status) {
  static_assert(NB == 32, "one pivot row per lane of a half wavefront");
  __shared__ __align__(16) double LiT[NB][NB + 2];    // LiT[c][a] = Li[a][c]
  __shared__ __align__(16) double Lc[2][NB];          // the column of L being eliminated
  __shared__ double Lk[TILE][NB + 1];                 // X[I, K], then X[I, K] Li^T
  __shared__ __align__(16) double Uk[NB][TILE + 2];   // X[K, J], then Li X[K, J]
  const int nbk = min(NB, s - k0);
  const int I = blockIdx.y * TILE, J = blockIdx.x * TILE;
  const int t = threadIdx.x, w = t / 64, lane = t % 64;
  if (w == 0) {
    const int i = lane % NB;  // the upper half repeats the lower
    const double* row = in + (int64_t)(k0 + min(i, nbk - 1)) * s + k0;
    double a[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
      a[j] = row[min(j, nbk - 1)];  // loads without branches; the padding follows
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (i >= nbk || j >= nbk) a[j] = i == j ? 1.0 : 0.0;
    // column i of L^{-1} by forward substitution beside the factor (x[j] = 0 above the
    // diagonal): one multiplier read serves both
    bool bad = false;
    double x[NB];
#pragma unroll
    for (int r = 0; r < NB; ++r) x[r] = r == i ? 1.0 : 0.0;
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      const double d = lane_read(a[p], p);
      bad |= !(d > 0.0);
      const double inv = rsqrt(d > 0.0 ? d : 1.0);
      a[p] *= inv;  // lane p: d / sqrt(d)
      x[p] *= inv;
      Lc[p & 1][i] = a[p];
      if (p + 1 < NB) {
        const double l = lane_read(a[p], p + 1);
        a[p + 1] = fma(-a[p], l, a[p + 1]);
        x[p + 1] = fma(-x[p], l, x[p + 1]);
      }
#pragma unroll
      for (int j = p + 2; j < NB; ++j) {
        const double l = Lc[p & 1][j];
        a[j] = fma(-a[p], l, a[j]);
        x[j] = fma(-x[p], l, x[j]);
      }
    }
    // stored here, by both halves and before any branch: the compiler moves the whole
    // substitution behind a branch that its results are not needed in front of
#pragma unroll
    for (int r = 0; r < NB; ++r) LiT[i][r] = x[r];
    if (bad && lane == 0 && blockIdx.x == 0 && blockIdx.y == 0) *status = 1;
  } else {
    for (int e = t - 64; e < TILE * NB; e += 192) {
      const int a = e / NB, b = e % NB;
      const int i = I + a;
      Lk[a][b] = (i < s && b < nbk) ? in[(int64_t)i * s + k0 + b] : 0.0;
    }
    for (int e = t - 64; e < NB * TILE; e += 192) {
      const int a = e / TILE, b = e % TILE;
      const int j = J + b;
      Uk[a][b] = (j < s && a < nbk) ? in[(int64_t)(k0 + a) * s + j] : 0.0;
    }
  }
  // the tile's own elements, four rows by four columns per thread, in flight over the factor
  const int r0 = t / 16 * 4, q0 = t % 16 * 4;
  double acc[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = I + r0 + p, j = J + q0 + q;
      acc[p][q] = (i < s && j < s) ? in[(int64_t)i * s + j] : 0.0;
    }
  __syncthreads();
  // Uk <- Li Uk and Lk <- Lk Li^T: wavefront w takes the eight rows (columns) 8 w .. of Li,
  // a lane one column of Uk and one row of Lk
  {
    double tu[8], tl[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) tu[q] = tl[q] = 0.0;
    const int a0 = 8 * w;
    for (int c = 0; c < a0 + 8; ++c) {  // Li is lower triangular
      const double u = Uk[c][lane], l = Lk[lane][c];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double m = LiT[c][a0 + q];
        tu[q] = fma(m, u, tu[q]);
        tl[q] = fma(l, m, tl[q]);
      }
    }
    __syncthreads();
    // rows (columns) of the tile that belong to K take Li itself: the update below is then one
    // product for every element, base - Lk Uk off K and + Lk Uk (-, off the pivot rows) on it
    const int ik = I + lane - k0, jk = J + lane - k0;
    const bool irow = ik >= 0 && ik < nbk, jcol = jk >= 0 && jk < nbk;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      Uk[a0 + q][lane] = jcol ? LiT[jk][a0 + q] : tu[q];
      Lk[lane][a0 + q] = irow ? LiT[ik][a0 + q] : tl[q];
    }
    __syncthreads();
  }
  double prod[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) prod[p][q] = 0.0;
#pragma unroll 4
  for (int c = 0; c < NB; ++c) {
    double a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = Lk[r0 + q][c];
      b[q] = Uk[c][q0 + q];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) prod[p][q] = fma(a[p], b[q], prod[p][q]);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = I + r0 + p, j = J + q0 + q;
      if (i >= s || j >= s) continue;
      const bool ik = i >= k0 && i < k0 + nbk, jk = j >= k0 && j < k0 + nbk;
      out[(int64_t)i * s + j] = ik ? prod[p][q] : (jk ? -prod[p][q] : acc[p][q] - prod[p][q]);
    }
}

__global__ void k_copy(int64_t len, const double* __restrict__ a, double* __restrict__ b) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < len) b[i] = a[i];
}

// symmetrise the final inverse (rounding leaves it nearly symmetric)
__global__ void k_sym_avg(int64_t s, double* M) {
  const int64_t i = blockIdx.y * (int64_t)blockDim.y + threadIdx.y;
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= s || j >= s || j >= i) return;
  const double v = 0.5 * (M[i * s + j] + M[j * s + i]);
  M[i * s + j] = v;
  M[j * s + i] = v;
}

// part[b] = the sum of A[i, i] over block b's share of the rows, in FP64 (every element is a
// line and often a page of its own: many blocks)
constexpr int kDiagBlocks = 64;
template <class T>
__global__ void __launch_bounds__(256) k_diag_sum(const T* __restrict__ A, int64_t n, int64_t lda,
                                                  double* __restrict__ part) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += 256 * kDiagBlocks) acc += (double)A[i * lda + i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// row sums of the Frobenius product <Winv, C^T C>_F: block i, part[i]
__global__ void __launch_bounds__(256) k_frob_rows(const double* __restrict__ Winv, const double* __restrict__ CtC,
                                                   int64_t s, double* __restrict__ part) {
  __shared__ double red[256];
  const int64_t o = (int64_t)blockIdx.x * s;
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < s; i += 256) acc = fma(Winv[o + i], CtC[o + i], acc);
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// the estimate (2/l) max(tr A - <Winv, C^T C>_F, 0) from the s row sums and the diagonal's
// partials after them, in one block in a fixed order; scal[0] = tr A, scal[1] = <Winv, C^T C>_F,
// scal[2] = the estimate
__global__ void __launch_bounds__(1024) k_lambda0_est(const double* __restrict__ part, int64_t len, double l,
                                                      double* scal) {
  __shared__ double red[1024];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < len; i += 1024) acc += part[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double tr = 0.0;
    for (int b = 0; b < kDiagBlocks; ++b) tr += part[len + b];
    scal[0] = tr;
    scal[1] = red[0];
    const double deficit = tr - red[0];
    // below 1e-6 tr A: the mu bias and rounding of an exact recovery (rank A <= s), taken as 0
    scal[2] = deficit > 1e-6 * tr ? (2.0 / l) * deficit : 0.0;
  }
}

}  // namespace

size_t lambda0_part_doubles(int64_t s) { return (size_t)s + kDiagBlocks; }

hipError_t launch_lambda0_est(hipStream_t st, const double* Winv, const double* CtC, int64_t s, const void* A,
                              msp_dtype t, int64_t n, int64_t lda, double l, double* scal, double* part) {
  hipLaunchKernelGGL(k_frob_rows, dim3((unsigned)s), dim3(256), 0, st, Winv, CtC, s, part);
  double* dp = part + s;
  if (t == MSP_F64)
    hipLaunchKernelGGL(k_diag_sum<double>, dim3(kDiagBlocks), dim3(256), 0, st, (const double*)A, n, lda, dp);
  else if (t == MSP_F32)
    hipLaunchKernelGGL(k_diag_sum<float>, dim3(kDiagBlocks), dim3(256), 0, st, (const float*)A, n, lda, dp);
  else
    hipLaunchKernelGGL(k_diag_sum<__hip_bfloat16>, dim3(kDiagBlocks), dim3(256), 0, st, (const __hip_bfloat16*)A, n, lda,
                       dp);
  hipLaunchKernelGGL(k_lambda0_est, dim3(1), dim3(1024), 0, st, part, s, l, scal);
  return hipGetLastError();
}

template <class T>
hipError_t gram_t(hipStream_t st, const T* X, int64_t rows, int64_t s, int64_t ldx, double* G, double* part,
                  int splits) {
  const int nt = (int)((s + TILE - 1) / TILE);
  const int tiles = nt * (nt + 1) / 2;
  const int64_t rps = ((rows + splits - 1) / splits + 15) / 16 * 16;
  double* dst = (splits == 1) ? G : part;
  hipLaunchKernelGGL(k_gram<T>, dim3(tiles, splits), dim3(256), 0, st, X, rows, s, ldx, rps, dst);
  if (splits > 1) {
    const int64_t len = s * s;
    hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, st, part, splits, len, G);
  }
  return hipGetLastError();
}

hipError_t launch_gram(hipStream_t st, const double* X, int64_t rows, int64_t s, int64_t ldx, double* G,
                       double* part, int splits) {
  return gram_t<double>(st, X, rows, s, ldx, G, part, splits);
}

hipError_t launch_gram_f32(hipStream_t st, const float* X, int64_t rows, int64_t s, int64_t ldx, double* G,
                           double* part, int splits) {
  return gram_t<float>(st, X, rows, s, ldx, G, part, splits);
}

int gram_splits(int64_t rows, int64_t s) {
  const int nt = (int)((s + TILE - 1) / TILE);
  const int tiles = nt * (nt + 1) / 2;
  int splits = 512 / tiles;  // two blocks per compute unit are resident: no second round
  const int64_t max_by_rows = (rows + 255) / 256;
  if (splits > max_by_rows) splits = (int)max_by_rows;
  if (splits < 1) splits = 1;
  if (splits > 16) splits = 16;
  return splits;
}

hipError_t launch_combine_sym(hipStream_t st, int64_t s, double a, const double* P, double b, const double* Q,
                              double c, double* out) {
  dim3 blk(16, 16), grd((unsigned)((s + 15) / 16), (unsigned)((s + 15) / 16));
  hipLaunchKernelGGL(k_combine_sym, grd, blk, 0, st, s, a, P, b, Q, c, out);
  return hipGetLastError();
}

hipError_t launch_symmetrize(hipStream_t st, int64_t s, double* Wm) {
  return launch_combine_sym(st, s, 1.0, Wm, 0.0, nullptr, 0.0, Wm);
}

hipError_t launch_trace(hipStream_t st, int64_t s, const double* M, double* out) {
  hipLaunchKernelGGL(k_trace, dim3(1), dim3(256), 0, st, s, M, out);
  return hipGetLastError();
}

hipError_t spd_inverse(hipStream_t st, int64_t s, double* M, double* tmp, double shift_rel, double* scal,
                       int32_t* status) {
  constexpr int NB = 32;
  hipLaunchKernelGGL(k_trace, dim3(1), dim3(256), 0, st, s, M, scal);
  hipLaunchKernelGGL(k_add_diag_scaled, dim3((unsigned)((s + 255) / 256)), dim3(256), 0, st, s, M, scal, shift_rel);
  const int nt = (int)((s + TILE - 1) / TILE);
  double* a = M;
  double* b = tmp;
  for (int k0 = 0; k0 < s; k0 += NB) {
    hipLaunchKernelGGL(k_bgj_step<NB>, dim3(nt, nt), dim3(256), 0, st, a, b, (int)s, k0, status);
    double* t = a;
    a = b;
    b = t;
  }
  if (a != M) {
    const int64_t len = s * s;
    hipLaunchKernelGGL(k_copy, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, st, len, a, M);
  }
  dim3 blk(16, 16), grd((unsigned)((s + 15) / 16), (unsigned)((s + 15) / 16));
  hipLaunchKernelGGL(k_sym_avg, grd, blk, 0, st, s, M);
  return hipGetLastError();
}
