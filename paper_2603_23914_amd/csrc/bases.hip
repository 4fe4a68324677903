// The compression step on the GPU (paper Sec. 3.1: low-rank SVD of the head-merged cache; Alg. 1,
// compress step; the appendix's implementation details name randomized SVD).
//
// ap_compute_bases: decompression matrix D [r, HD] of X [n, HD], rows = approximate leading right
// singular vectors in decreasing order of singular value, by the published randomized range-finder
// scheme run on the ROW space with l = r + oversampling vectors, the start block given by the caller:
//
//     P <- Omega [l, HD]
//     power_iters + 1 times:   Yt = P X^T   [l, n]      matrix cores (compact_gemm.hip), 16-bit out
//                              M  = Yt X    [l, HD]     matrix cores, fp32 out (X^T from transpose16)
//                              P  = rows of M made orthonormal: S = M M^T in fp64 (gram_f64),
//                                   S = L L^T (chol_update / chol_panel, panels of 32 columns),
//                                   P = L^-1 M (tri_inverse, gemm_nn; fp64 accumulation)
//     Rayleigh-Ritz:           Zt = P X^T [l, n] fp32,  S = Zt Zt^T [l, l]  (= P X^T X P^T)
//                              S = J Lambda J^T by one-sided Jacobi on the rows of S (jacobi_pair)
//                              D = (J^T P)[:r] in decreasing order of Lambda,  sigma = sqrt(Lambda)
//
// The matrices that lose information when rounded (M, whose singular values span the square of the
// cache's spectrum, and the small Gram matrices) stay in fp32 / fp64; what goes back into the matrix
// cores as a 16-bit operand is either the cache itself (exact) or a block with orthonormal rows.
//
// ap_decompress: Alg. 1 "retrieve cache" as a matrix, Xtilde[t] = C[t, :rank_t] D[:rank_t]: what the
// periodic re-compression decomposes again (next to the uncompressed tail).
#include "ap_common.hpp"
#include "lane_ops.hpp"
#include "mfma_ops.hpp"

namespace ap {
namespace {

__device__ __forceinline__ double wave_sum_d(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

constexpr int kJacobiSweeps = 12;      // at most; a matrix without a rotation in a sweep is done
constexpr int kSweepSlots = 16;        // rotation counters per matrix, one per sweep
constexpr float kJacobiTol = 1e-5f;    // |a.b| <= tol |a||b|: far below what 16-bit storage of the result keeps

// ---- out[c][r] = in[r][c] for 16-bit elements; columns rows .. ld_out-1 of out are zero-filled.
//      grid (ceil(ld_out / 64), ceil(cols / 64), batch), 256 threads.
__global__ void __launch_bounds__(256)
transpose16(const uint16_t* __restrict__ in, int64_t in_bstride, int ld_in, uint16_t* __restrict__ out,
            int64_t out_bstride, int ld_out, int rows, int cols) {
  __shared__ uint16_t tile[64][66];
  const int tid = threadIdx.x, r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  in += (size_t)blockIdx.z * in_bstride;
  out += (size_t)blockIdx.z * out_bstride;
  for (int e = tid; e < 64 * 64; e += 256) {
    const int rr = e >> 6, cc = e & 63;
    const int r = r0 + rr, c = c0 + cc;
    tile[rr][cc] = (r < rows && c < cols) ? in[(size_t)r * ld_in + c] : (uint16_t)0;
  }
  __syncthreads();
  for (int e = tid; e < 64 * 64; e += 256) {
    const int cc = e >> 6, rr = e & 63;
    const int r = r0 + rr, c = c0 + cc;
    if (c < cols && r < ld_out) out[(size_t)c * ld_out + r] = tile[rr][cc];
  }
}

// ---- zero the columns n .. ld-1 of a 16-bit [rows][ld] matrix.  grid (rows, batch), 64 threads.
__global__ void fill_pad16(uint16_t* __restrict__ a, int64_t bstride, int ld, int n) {
  uint16_t* row = a + (size_t)blockIdx.y * bstride + (size_t)blockIdx.x * ld;
  for (int c = n + threadIdx.x; c < ld; c += 64) row[c] = 0;
}

// ---- C̃[t, j] = j < rank[t] ? C[t, j] : 0 (16-bit).  grid (ceil(T / 4), batch), 256 threads.
__global__ void __launch_bounds__(256)
mask_coeffs(const uint16_t* __restrict__ C, int64_t c_bstride, const int32_t* __restrict__ rank, int64_t r_bstride,
            uint16_t* __restrict__ out, int64_t o_bstride, int T, int r) {
  const int b = blockIdx.y;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const int rk = rank[(size_t)b * r_bstride + t];
  const uint16_t* src = C + (size_t)b * c_bstride + (size_t)t * r;
  uint16_t* dst = out + (size_t)b * o_bstride + (size_t)t * r;
  for (int j = threadIdx.x & 63; j < r; j += 64) dst[j] = j < rk ? src[j] : (uint16_t)0;
}

// fp64 matrix-core product: A operand lane (i = lane & 15, k = lane >> 4), B operand lane
// (j = lane & 15, k = lane >> 4), result element e of lane (j, g): row g + 4 e, column j.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
typedef double f64x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f64x4_t mfma_f64(double a, double b, f64x4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---- S = A A^T in fp64 for A [l][lda] fp32 (m columns used, m % 8 == 0), the lower triangle of
//      tiles, mirrored on the way out.  Bound by the fp64 matrix pipe: a wave owns 32 x 32 results
//      (2 x 2 products) and takes its operands straight from global memory, 16 bytes of a row per
//      lane = four k of the product (the order of k is free as long as both operands agree), the
//      next sixteen columns requested while the current ones are multiplied; no LDS, no barrier.
//      SPLIT_K = false: a workgroup's four waves form a 64 x 64 tile.  SPLIT_K = true: they share
//      ONE 32 x 32 tile, a quarter of the columns each, and meet in LDS: for few or small matrices,
//      which would leave most of the chip idle.  Measured at 16 matrices of 544 x 4096: 1.29 ms with
//      fp64 FMAs from LDS tiles, see launch_gram for both forms of this one.
//      grid (tiles of the lower triangle, batch), 256 threads.
template <bool SPLIT_K>
__global__ void __launch_bounds__(256)
gram_f64(const float* __restrict__ A, int64_t a_bstride, int lda, double* __restrict__ S, int64_t s_bstride,
         int l, int m) {
  __shared__ double red[SPLIT_K ? 3 * 1024 : 1];
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // tile (ti, tj), tj <= ti, of the lower triangle
  int ti = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
  while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
  while (ti * (ti + 1) / 2 > (int)blockIdx.x) --ti;
  const int tj = (int)blockIdx.x - ti * (ti + 1) / 2;
  const int i0 = SPLIT_K ? ti * 32 : ti * 64 + (w >> 1) * 32;
  const int j0 = SPLIT_K ? tj * 32 : tj * 64 + (w & 1) * 32;
  if (!SPLIT_K && (i0 >= l || j0 >= l)) return;          // (no barrier in this form)
  A += (size_t)blockIdx.y * a_bstride;
  S += (size_t)blockIdx.y * s_bstride;
  const float* rows[4];                                  // rows past the end repeat the last one
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int ri = i0 + 16 * u + n, rj = j0 + 16 * u + n;
    rows[u] = A + (size_t)(ri < l ? ri : l - 1) * lda;
    rows[2 + u] = A + (size_t)(rj < l ? rj : l - 1) * lda;
  }
  const int chunks = (m + 15) >> 4;                      // sixteen columns each; the last may be half
  const int c_lo = SPLIT_K ? (int)((int64_t)w * chunks / 4) : 0;
  const int c_hi = SPLIT_K ? (int)((int64_t)(w + 1) * chunks / 4) : chunks;
  f32x4_t nx[4];
  auto load = [&](int c) {
    const int col = c * 16 + 4 * g;
    const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u) nx[u] = col < m ? *(const f32x4_t*)(rows[u] + col) : z;
  };
  f64x4_t acc[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) acc[u][v] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  if (c_lo < c_hi) load(c_lo);
  for (int c = c_lo; c < c_hi; ++c) {
    f32x4_t cur[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) cur[u] = nx[u];
    load(c + 1 < c_hi ? c + 1 : c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double a0 = cur[0][e], a1 = cur[1][e], b0 = cur[2][e], b1 = cur[3][e];
      acc[0][0] = mfma_f64(a0, b0, acc[0][0]);
      acc[0][1] = mfma_f64(a0, b1, acc[0][1]);
      acc[1][0] = mfma_f64(a1, b0, acc[1][0]);
      acc[1][1] = mfma_f64(a1, b1, acc[1][1]);
    }
  }
  if (SPLIT_K) {                                         // the four partial tiles, added in wave order
    if (w > 0) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
          for (int e = 0; e < 4; ++e) red[((w - 1) * 16 + (u * 2 + v) * 4 + e) * 64 + lane] = acc[u][v][e];
    }
    __syncthreads();
    if (w > 0) return;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[u][v][e] += red[(k * 16 + (u * 2 + v) * 4 + e) * 64 + lane];
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + 16 * u + g + 4 * e, j = j0 + 16 * v + n;
        if (i < l && j < l) {
          S[(size_t)i * l + j] = acc[u][v][e];
          S[(size_t)j * l + i] = acc[u][v][e];
        }
      }
}

void launch_gram(const float* A, int64_t a_bstride, int lda, double* S, int64_t s_bstride, int l, int m, int batch,
                 hipStream_t st) {
  // 64 x 64 tiles once they give every CU two workgroups; below that the quarter-size tiles with
  // the column axis split over the four waves.
  const int t64 = (l + 63) / 64, t32 = (l + 31) / 32;
  if ((int64_t)t64 * (t64 + 1) / 2 * batch >= 512)
    hipLaunchKernelGGL(gram_f64<false>, dim3(t64 * (t64 + 1) / 2, batch), dim3(256), 0, st, A, a_bstride, lda, S, s_bstride, l, m);
  else
    hipLaunchKernelGGL(gram_f64<true>, dim3(t32 * (t32 + 1) / 2, batch), dim3(256), 0, st, A, a_bstride, lda, S, s_bstride, l, m);
}

// ---- Cholesky S = L L^T in place (the lower triangle of S becomes L), fp64, in panels of 32
//      columns.  Per panel two launches:
//   chol_update   rows c0 .. l-1 of the panel minus the contribution of the columns left of it:
//                 S[i][c] -= sum_{j < c0} L[i][j] L[c][j]; a workgroup per 32 x 32 tile
//   chol_panel    one workgroup per matrix: the 32 x 32 diagonal block is factored in LDS, then
//                 every row below solves its 32 unknowns against it (a thread per row)
//      A pivot below 1e-13 of the largest diagonal entry (dmax) marks a direction that the rows
//      do not span: its column of L and its diagonal entry are zero, its row of L^-1 is zero,
//      so the corresponding row of P = L^-1 M is zero and drops out later.
__global__ void __launch_bounds__(256)
diag_max(const double* __restrict__ S, int64_t s_bstride, int l, double* __restrict__ dmax) {
  const double* Sb = S + (size_t)blockIdx.x * s_bstride;
  __shared__ double red[4];
  double m = 0.0;
  for (int i = threadIdx.x; i < l; i += 256) m = fmax(m, Sb[(size_t)i * l + i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) dmax[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// grid (ceil((l - c0) / 32), batch), 256 threads = 16 x 16, 2 x 2 results each
__global__ void __launch_bounds__(256)
chol_update(double* __restrict__ S, int64_t s_bstride, int l, int c0) {
  __shared__ double As[32][33], Bs[32][33];
  double* L = S + (size_t)blockIdx.y * s_bstride;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int i0 = c0 + blockIdx.x * 32;
  double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  for (int k0 = 0; k0 < c0; k0 += 32) {              // c0 is a multiple of 32
    for (int e = tid; e < 1024; e += 256) {
      const int rr = e >> 5, kk = e & 31;
      As[rr][kk] = i0 + rr < l ? L[(size_t)(i0 + rr) * l + k0 + kk] : 0.0;
      Bs[rr][kk] = c0 + rr < l ? L[(size_t)(c0 + rr) * l + k0 + kk] : 0.0;
    }
    __syncthreads();
#pragma unroll 8
    for (int kk = 0; kk < 32; ++kk) {
      const double a0 = As[2 * ty][kk], a1 = As[2 * ty + 1][kk];
      const double b0 = Bs[2 * tx][kk], b1 = Bs[2 * tx + 1][kk];
      acc[0][0] = fma(a0, b0, acc[0][0]);
      acc[0][1] = fma(a0, b1, acc[0][1]);
      acc[1][0] = fma(a1, b0, acc[1][0]);
      acc[1][1] = fma(a1, b1, acc[1][1]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int i = i0 + 2 * ty + u, c = c0 + 2 * tx + v;
      if (i < l && c < l) L[(size_t)i * l + c] -= acc[u][v];
    }
}

// grid (batch), 256 threads
__global__ void __launch_bounds__(256)
chol_panel(double* __restrict__ S, int64_t s_bstride, int l, int c0, const double* __restrict__ dmax) {
  __shared__ double Dg[32][33];
  double* L = S + (size_t)blockIdx.x * s_bstride;
  const int tid = threadIdx.x;
  const int nb = l - c0 < 32 ? l - c0 : 32;
  const double tol = dmax[blockIdx.x] * 1e-13;
  for (int e = tid; e < 1024; e += 256) {
    const int rr = e >> 5, cc = e & 31;
    Dg[rr][cc] = (rr < nb && cc < nb && cc <= rr) ? L[(size_t)(c0 + rr) * l + c0 + cc] : 0.0;
  }
  __syncthreads();
  // unblocked Cholesky of the diagonal block (right-looking, 32 short steps)
  for (int k = 0; k < nb; ++k) {
    const double piv = Dg[k][k];
    const bool dead = !(piv > tol);
    const double d = dead ? 0.0 : sqrt(piv), inv = dead ? 0.0 : 1.0 / d;
    __syncthreads();
    if (tid == 0) Dg[k][k] = d;
    if (tid > k && tid < nb) Dg[tid][k] *= inv;
    __syncthreads();
    for (int e = tid; e < 1024; e += 256) {
      const int i = e >> 5, j = e & 31;
      if (i > k && j > k && j <= i && i < nb) Dg[i][j] -= Dg[i][k] * Dg[j][k];
    }
    __syncthreads();
  }
  for (int e = tid; e < 1024; e += 256) {
    const int rr = e >> 5, cc = e & 31;
    if (rr < nb && cc < nb) L[(size_t)(c0 + rr) * l + c0 + cc] = cc <= rr ? Dg[rr][cc] : 0.0;
  }
  // rows below the block: x Dg^T = t, forward substitution, a thread per row
  for (int i = c0 + 32 + tid; i < l; i += 256) {
    double* row = L + (size_t)i * l + c0;
    double x[32];
#pragma unroll
    for (int c = 0; c < 32; ++c) x[c] = row[c];
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      double v = x[c];
#pragma unroll
      for (int j = 0; j < 32; ++j)
        if (j < c) v = fma(-x[j], Dg[c][j], v);
      const double d = Dg[c][c];
      x[c] = d == 0.0 ? 0.0 : v / d;
    }
#pragma unroll
    for (int c = 0; c < 32; ++c) row[c] = x[c];
  }
}

// X = L^-1 (lower triangular, fp64) by forward substitution, a wave per column j: the column's
// entries found so far sit in LDS, row i's dot product with them is spread over the lanes.  Rows
// of a dead pivot stay zero.  grid (ceil(l / 4), batch), 256 threads; dynamic LDS 4 * l doubles.
__global__ void __launch_bounds__(256)
tri_inverse(const double* __restrict__ S, int64_t s_bstride, double* __restrict__ X, int64_t x_bstride, int l) {
  extern __shared__ double xcol[];                      // [4][l]
  const double* L = S + (size_t)blockIdx.y * s_bstride;
  double* Li = X + (size_t)blockIdx.y * x_bstride;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = blockIdx.x * 4 + w;
  if (j >= l) return;
  double* x = xcol + (size_t)w * l;
  for (int i = lane; i < j; i += 64) Li[(size_t)i * l + j] = 0.0;     // above the diagonal
  for (int i = j; i < l; ++i) {
    const double* rowi = L + (size_t)i * l;
    double s = 0.0;
    for (int k = j + lane; k < i; k += 64) s = fma(rowi[k], x[k], s);
    s = wave_sum_d(s);
    const double dii = rowi[i];
    const double v = dii == 0.0 ? 0.0 : ((i == j ? 1.0 : 0.0) - s) / dii;
    if (lane == 0) {
      x[i] = v;
      Li[(size_t)i * l + j] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// ---- C = A B with A [M][K] fp64, B [K][N] fp32, fp64 accumulation; C as fp32 and / or in 16-bit
//      storage.  lower: A is lower triangular (a wave stops at its last row's diagonal).
//      Bound by the fp64 matrix pipe.  A wave owns 32 rows x 64 columns (2 x 4 products) and takes
//      its operands straight from global memory: a lane's 16 bytes of an A row are two k, its 16
//      bytes of a B row are one k of FOUR column tiles (tile c holds columns 4 j + c, so a lane's
//      results are four consecutive columns and leave as one 16-byte store).  Eight k per stage, the
//      next stage requested while the current one is multiplied.  The four waves of a workgroup
//      (2 x 2) share their operand rows in L1; XCD-aware numbering keeps a matrix's A (2.4 MB at
//      l = 544) in one XCD's L2.
//      grid (ceil(M / 64) * N / 128 (+ padding) * batch), 256 threads; N % 64 == 0, K even.
template <class Tag>
__global__ void __launch_bounds__(256)
gemm_nn(const double* __restrict__ A, int64_t a_bstride, int lda, const float* __restrict__ Bm, int64_t b_bstride,
        int ldb, float* __restrict__ C32, int64_t c32_bstride, uint16_t* __restrict__ C16, int64_t c16_bstride,
        int ldc, int M, int N, int K, int lower, int batch) {
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int MT = (M + 63) >> 6, NT = (N + 127) >> 7, per = MT * NT;
  int b, t;
  const int id = (int)blockIdx.x;
  if (batch % 8 == 0) {                                  // matrix b on XCD b % 8
    const int k = id >> 3;
    b = (k / per) * 8 + (id & 7);
    t = k % per;
  } else {
    b = id / per;
    t = id - b * per;
  }
  // longest row blocks first (lower: the work grows with the row)
  const int mt = MT - 1 - t / NT, nt = t % NT;
  const int m0 = mt * 64 + (w >> 1) * 32, n0 = nt * 128 + (w & 1) * 64;
  if (m0 >= M || n0 >= N) return;
  A += (size_t)b * a_bstride;
  Bm += (size_t)b * b_bstride;
  const double* arow[2];                                 // rows past the end repeat the last one
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = m0 + 16 * u + n;
    arow[u] = A + (size_t)(i < M ? i : M - 1) * lda;
  }
  const float* bcol = Bm + n0 + 4 * n;
  f64x4_t acc[2][4];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[u][v] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  const int kend = lower ? (m0 + 32 < K ? m0 + 32 : K) : K;
  f64x2_t na[2];
  f32x4_t nb[2];
  auto load = [&](int k0) {                              // k of element e: k0 + 2 g + e
    const int k = k0 + 2 * g;
    const bool in = k < kend;                            // kend is even: both elements or none
    const int kc = in ? k : 0;
    const f64x2_t z = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const f64x2_t v = *(const f64x2_t*)(arow[u] + kc);
      na[u] = in ? v : z;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) nb[e] = *(const f32x4_t*)(bcol + (size_t)(kc + e) * ldb);
  };
  load(0);
  for (int k0 = 0; k0 < kend; k0 += 8) {
    f64x2_t ca[2];
    f32x4_t cb[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) { ca[e] = na[e]; cb[e] = nb[e]; }
    load(k0 + 8 < kend ? k0 + 8 : k0);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double bv = cb[e][v];
        acc[0][v] = mfma_f64(ca[0][e], bv, acc[0][v]);
        acc[1][v] = mfma_f64(ca[1][e], bv, acc[1][v]);
      }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = m0 + 16 * u + g + 4 * e, j = n0 + 4 * n;
      if (i >= M) continue;
      const f32x4_t f = {(float)acc[u][0][e], (float)acc[u][1][e], (float)acc[u][2][e], (float)acc[u][3][e]};
      if (C32) *(f32x4_t*)(C32 + (size_t)b * c32_bstride + (size_t)i * ldc + j) = f;
      if (C16) {
        const u32x2_t h = {pack2(f[0], f[1], Tag{}), pack2(f[2], f[3], Tag{})};
        *(u32x2_t*)(C16 + (size_t)b * c16_bstride + (size_t)i * ldc + j) = h;
      }
    }
}

// ---- W [l][lp] fp32 <- S [l][l] fp64, columns l .. lp-1 zero; the sweeps' rotation counters to zero.
//      grid (ceil(l * lp / 256), batch), 256 threads.
__global__ void __launch_bounds__(256)
jacobi_init(const double* __restrict__ S, int64_t s_bstride, float* __restrict__ W, int64_t w_bstride, int l, int lp,
            int* __restrict__ rotations) {
  const int e = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (e < l * lp) {
    const int i = e / lp, c = e - i * lp;
    W[(size_t)b * w_bstride + e] = c < l ? (float)S[(size_t)b * s_bstride + (size_t)i * l + c] : 0.f;
  }
  if (e < kSweepSlots) rotations[b * kSweepSlots + e] = 0;
}

// ---- One-sided Jacobi on the rows of W [l][lp] (fp32), block version.  The rows are cut into blocks
//      of 16; one launch takes disjoint pairs of blocks (round-robin over the blocks), a workgroup per
//      pair.  For a symmetric positive semi-definite W = S the rows converge to lambda_i j_i^T, the
//      eigenvectors scaled by their eigenvalues.
//      A workgroup never holds its 32 rows: it forms their Gram matrix G on the fp32 matrix
//      instructions, runs one cyclic sweep of two-sided rotations on G (31 steps of 16 disjoint pairs,
//      the same rotations that the rows themselves would see) while the product Q of the rotations is
//      built next to it, and multiplies the rows by Q on the matrix instructions.  The chain of 31
//      steps is what bounds it, so a step is kept short: G and Q are 32 x 32 in LDS, double-buffered,
//      one barrier a step.  The pairs of a step are always positions (k, 16 + k); what a step writes
//      goes to the position of the next step's partner (the circle method: position 0 stays, the
//      others move on by one, and after 31 steps everything is back), so all addresses are constants.
//      Waves 0-3 own 2 x 2 of G per thread and each work out all 16 rotations themselves; waves 4-7
//      follow one step behind with Q.
//      Blocks of 16: 17 pairs of a 544-row matrix, which fills the chip from 16 matrices on; the
//      number of steps per sweep hardly depends on the block (1023 against 1071 with blocks of 32),
//      nor does the number of sweeps (8 in both, the last of which only looks).
//      G is scaled by a power of two to a largest diagonal entry in [1, 2): no overflow in the angles.
//      Measured at 16 matrices of 544 rows: 24 us a launch, 7.0 ms in all; with the rows themselves in
//      LDS (blocks of 32, three dot products and a rotation of 544 columns per pair) 190 us a launch
//      and 21.9 ms.
//      rotations[b][sweep] counts the pairs of blocks that had work; a matrix whose previous sweep
//      had none is done.
//      grid (pairs * batch), 512 threads.
__global__ void __launch_bounds__(512)
jacobi_pair(float* __restrict__ W, int64_t w_bstride, int l, int lp, int nblk, int step, int sweep, float tol,
            int* __restrict__ rotations, int batch) {
  constexpr int PITCH = 48;                             // 16 mod 32: two neighbouring rows fill the banks
  __shared__ float part[8][3 * 256];
  __shared__ float gm[2][32 * PITCH], qm[2][32 * PITCH];
  __shared__ f32x2_t csn[2][16];                        // cosine and sine of a step's pairs
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int npair = nblk >> 1, id = (int)blockIdx.x;
  int b, k;
  if (batch % 8 == 0) {                                 // matrix b stays on XCD b % 8, in its L2
    b = (id >> 3) / npair * 8 + (id & 7);
    k = (id >> 3) % npair;
  } else {
    b = id / npair;
    k = id - b * npair;
  }
  if (sweep > 0 && rotations[b * kSweepSlots + sweep - 1] == 0) return;
  // round-robin over nblk blocks (nblk even; a block index >= the real count is an empty block)
  const int nm1 = nblk - 1;
  int ba, bb;
  if (k == 0) { ba = nm1; bb = step; }
  else { ba = (step + k) % nm1; bb = (step + nm1 - k) % nm1; }
  if (ba * 16 >= l && bb * 16 >= l) return;
  float* Wb = W + (size_t)b * w_bstride;

  // G = rows rows^T: lane n holds row n of either block, four columns of each sixteen
  const int ra = ba * 16 + n, rb = bb * 16 + n;
  const float* pa = Wb + (size_t)(ra < l ? ra : 0) * lp + 4 * g;
  const float* pb = Wb + (size_t)(rb < l ? rb : 0) * lp + 4 * g;
  f32x4_t g00 = {0.f, 0.f, 0.f, 0.f}, g01 = g00, g11 = g00;
  const f32x4_t z4 = g00;
  for (int c0 = w; c0 < lp >> 4; c0 += 40) {            // five sixteens of columns on their way at once
    f32x4_t va[5], vb[5];
#pragma unroll
    for (int t = 0; t < 5; ++t)
      if (c0 + 8 * t < lp >> 4) {
        va[t] = *(const f32x4_t*)(pa + (c0 + 8 * t) * 16);
        vb[t] = *(const f32x4_t*)(pb + (c0 + 8 * t) * 16);
      }
#pragma unroll
    for (int t = 0; t < 5; ++t)
      if (c0 + 8 * t < lp >> 4) {
        const f32x4_t x = ra < l ? va[t] : z4, y = rb < l ? vb[t] : z4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          g00 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], x[e], g00, 0, 0, 0);
          g01 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], g01, 0, 0, 0);
          g11 = __builtin_amdgcn_mfma_f32_16x16x4f32(y[e], y[e], g11, 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int at = (4 * g + e) * 16 + n;
    part[w][at] = g00[e];
    part[w][256 + at] = g01[e];
    part[w][512 + at] = g11[e];
  }
  __syncthreads();
  float own[2];                                         // elements tid and tid + 512 of G
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = (tid >> 5) + 16 * u, j = tid & 31;
    const int at = u == 0 ? (j < 16 ? i * 16 + j : 256 + i * 16 + j - 16)
                          : (j < 16 ? 256 + j * 16 + i - 16 : 512 + (i - 16) * 16 + j - 16);
    float s = part[0][at];
#pragma unroll
    for (int q = 1; q < 8; ++q) s += part[q][at];
    own[u] = s;
    gm[0][i * PITCH + j] = s;
  }
  __syncthreads();
  const float dg = gm[0][(lane & 31) * (PITCH + 1)];    // the diagonal, in every wave
  float dmx = dg;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) dmx = fmaxf(dmx, __shfl_xor(dmx, o));
  int work = 0;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = (tid >> 5) + 16 * u, j = tid & 31;
    const float di = __shfl(dg, i), dj = __shfl(dg, j);
    if (i != j && fabsf(own[u]) > tol * (sqrtf(di) * sqrtf(dj))) work = 1;
  }
  if (!__syncthreads_or(work)) return;                  // every pair is orthogonal already
  if (tid == 0) atomicAdd(&rotations[b * kSweepSlots + sweep], 1);
  const int sh = 1 - __builtin_amdgcn_frexp_expf(dmx);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = (tid >> 5) + 16 * u, j = tid & 31;
    gm[0][i * PITCH + j] = ldexpf(own[u], sh);
    qm[0][i * PITCH + j] = i == j ? 1.f : 0.f;
  }
  // the rows again, now a row of a block per (kk, g) and two columns per lane, on their way meanwhile
  const int units = lp >> 5;
  f32x2_t pre[3][8];
  auto row_of = [&](int i) { return i < 16 ? ba * 16 + i : bb * 16 + i - 16; };
  auto load_unit = [&](int u, f32x2_t (&v)[8]) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int row = row_of(4 * kk + g);
      v[kk] = *(const f32x2_t*)(Wb + (size_t)(row < l ? row : 0) * lp + u * 32 + 2 * n);
    }
  };
#pragma unroll
  for (int t = 0; t < 3; ++t)
    if (w + 8 * t < units) load_unit(w + 8 * t, pre[t]);
  __syncthreads();

  const int I = 4 * (w & 3) + g;
  auto moved = [](int p) { return p == 0 ? 0 : p == 15 ? 31 : p == 16 ? 1 : p < 15 ? p + 1 : p - 1; };
  const int r0 = moved(I) * PITCH, r1 = moved(16 + I) * PITCH, c0 = moved(n), c1 = moved(16 + n);
#pragma unroll 2
  for (int s = 0; s < 32; ++s) {
    if (w < 4) {
      if (s < 31) {
        const float* cur = gm[s & 1];
        float* nxt = gm[(s & 1) ^ 1];
        const float al = cur[n * (PITCH + 1)], be = cur[(16 + n) * (PITCH + 1)], ga = cur[n * PITCH + 16 + n];
        const float a00 = cur[I * PITCH + n], a01 = cur[I * PITCH + 16 + n];
        const float a10 = cur[(16 + I) * PITCH + n], a11 = cur[(16 + I) * PITCH + 16 + n];
        // the rotation that makes the pair n orthogonal (any residue is far below the tolerance)
        const float zeta = (be - al) * __builtin_amdgcn_rcpf(ga + ga);
        float t = __builtin_amdgcn_rcpf(fabsf(zeta) + __builtin_amdgcn_sqrtf(fmaf(zeta, zeta, 1.f)));
        t = fabsf(ga) > 1e-30f ? copysignf(t, zeta) : 0.f;
        const float h = fmaf(t, t, 1.f);
        float cs = __builtin_amdgcn_rsqf(h);
        cs = fmaf(cs * 0.5f, fmaf(-h * cs, cs, 1.f), cs);   // one Newton step: cos^2 + sin^2 = 1 to rounding
        const float sn = cs * t;
        const float ci = __shfl(cs, I), si = __shfl(sn, I);
        if (w == 0 && g == 0) csn[s & 1][n] = f32x2_t{cs, sn};
        const float b00 = fmaf(ci, a00, -si * a10), b01 = fmaf(ci, a01, -si * a11);
        const float b10 = fmaf(si, a00, ci * a10), b11 = fmaf(si, a01, ci * a11);
        nxt[r0 + c0] = fmaf(cs, b00, -sn * b01);
        nxt[r0 + c1] = fmaf(sn, b00, cs * b01);
        nxt[r1 + c0] = fmaf(cs, b10, -sn * b11);
        nxt[r1 + c1] = fmaf(sn, b10, cs * b11);
      }
    } else if (s > 0) {
      const float* cur = qm[(s & 1) ^ 1];
      float* nxt = qm[s & 1];
      const f32x2_t r = csn[(s & 1) ^ 1][I];
      const float a00 = cur[I * PITCH + n], a01 = cur[I * PITCH + 16 + n];
      const float a10 = cur[(16 + I) * PITCH + n], a11 = cur[(16 + I) * PITCH + 16 + n];
      nxt[r0 + n] = fmaf(r[0], a00, -r[1] * a10);
      nxt[r0 + 16 + n] = fmaf(r[0], a01, -r[1] * a11);
      nxt[r1 + n] = fmaf(r[1], a00, r[0] * a10);
      nxt[r1 + 16 + n] = fmaf(r[1], a01, r[0] * a11);
    }
    __syncthreads();
  }

  // rows <- Q rows
  const float* Q = qm[1];
  float qa[2][8];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qa[t][kk] = Q[(16 * t + n) * PITCH + 4 * kk + g];
  auto apply_unit = [&](int u, const f32x2_t (&v)[8]) {
    f32x4_t acc[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) { acc[t][0] = z4; acc[t][1] = z4; }
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const f32x2_t x = row_of(4 * kk + g) < l ? v[kk] : f32x2_t{0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t][kk], x[c], acc[t][c], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = row_of(16 * t + 4 * g + e);
        if (row < l) *(f32x2_t*)(Wb + (size_t)row * lp + u * 32 + 2 * n) = f32x2_t{acc[t][0][e], acc[t][1][e]};
      }
  };
#pragma unroll
  for (int t = 0; t < 3; ++t)
    if (w + 8 * t < units) apply_unit(w + 8 * t, pre[t]);
  for (int u = w + 24; u < units; u += 8) {
    f32x2_t v[8];
    load_unit(u, v);
    apply_unit(u, v);
  }
}

// ---- eigenvalues = row norms.  grid (ceil(l / 4), batch), 256 threads: a wave per row.
__global__ void __launch_bounds__(256)
eig_norms(const float* __restrict__ W, int64_t w_bstride, int l, int lp, double* __restrict__ lam) {
  const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6), b = blockIdx.y;
  if (i >= l) return;
  const float* row = W + (size_t)b * w_bstride + (size_t)i * lp;
  double s = 0.0;
  for (int c = lane; c < l; c += 64) { const double v = row[c]; s = fma(v, v, s); }
  s = wave_sum_d(s);
  if (lane == 0) lam[(size_t)b * l + i] = sqrt(s);
}

// ---- rows in decreasing order of their norm (ties by row index); the r leading rows, normalised,
//      become R [r][l] (fp64) and sigma[i] = sqrt(lambda_i).  grid (ceil(l / 4), batch), 256 threads:
//      a wave per row, which counts the rows before its own (one workgroup per matrix, which also
//      took the norms, needed 197 us at 16 x 544 rows).
__global__ void __launch_bounds__(256)
eig_select(const float* __restrict__ W, int64_t w_bstride, const double* __restrict__ lam, int l, int lp, int r,
           double* __restrict__ R, int64_t r_bstride, float* __restrict__ sigma, int64_t sig_bstride) {
  const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6), b = blockIdx.y;
  if (i >= l) return;
  const double* lb = lam + (size_t)b * l;
  const double li = lb[i];
  int p = 0;
  for (int j = lane; j < l; j += 64) p += (lb[j] > li || (lb[j] == li && j < i)) ? 1 : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) p += __shfl_xor(p, o);
  if (p >= r) return;
  if (lane == 0 && sigma) sigma[(size_t)b * sig_bstride + p] = (float)sqrt(li);
  const double inv = li > 0.0 ? 1.0 / li : 0.0;
  const float* row = W + (size_t)b * w_bstride + (size_t)i * lp;
  for (int c = lane; c < l; c += 64) R[(size_t)b * r_bstride + (size_t)p * l + c] = (double)row[c] * inv;
}

struct BasesLayout {
  size_t xt, yt, m32, p16, p32, zt, s64, linv, w32, rsel, state, dmax, lam, total;
  int n_pad, lp;
};
BasesLayout bases_layout(int B, int n, int HD, int l, int r) {
  BasesLayout w;
  w.n_pad = (n + 63) / 64 * 64;
  w.lp = (l + 31) / 32 * 32;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t at = off; off += round_up(bytes, 256); return at; };
  w.xt = take((size_t)B * HD * w.n_pad * 2);
  w.yt = take((size_t)B * l * w.n_pad * 2);
  w.m32 = take((size_t)B * l * HD * 4);
  w.p16 = take((size_t)B * l * HD * 2);
  w.p32 = take((size_t)B * l * HD * 4);
  w.zt = take((size_t)B * l * w.n_pad * 4);
  w.s64 = take((size_t)B * l * l * 8);
  w.linv = take((size_t)B * l * l * 8);
  w.w32 = take((size_t)B * l * w.lp * 4);
  w.rsel = take((size_t)B * r * l * 8);
  w.state = take((size_t)B * kSweepSlots * 4);
  w.dmax = take((size_t)B * 8);
  w.lam = take((size_t)B * l * 8);
  w.total = off;
  return w;
}

template <class Tag>
void launch_gemm_nn(const double* A, int64_t a_bs, int lda, const float* Bm, int64_t b_bs, int ldb, float* C32,
                    int64_t c32_bs, uint16_t* C16, int64_t c16_bs, int ldc, int M, int N, int K, int lower, int batch,
                    hipStream_t st) {
  const int per = ((M + 63) / 64) * ((N + 127) / 128);
  hipLaunchKernelGGL((gemm_nn<Tag>), dim3((unsigned)(per * batch)), dim3(256), 0, st, A, a_bs, lda, Bm,
                     b_bs, ldb, C32, c32_bs, C16, c16_bs, ldc, M, N, K, lower, batch);
}

template <class Tag>
ap_status run_bases(const BasesArgs& a) {
  const int B = a.B, n = a.n, HD = a.HD, r = a.r, l = a.r + a.oversample;
  const BasesLayout w = bases_layout(B, n, HD, l, r);
  char* ws = (char*)a.workspace;
  uint16_t* Xt = (uint16_t*)(ws + w.xt);
  uint16_t* Yt = (uint16_t*)(ws + w.yt);
  float* M32 = (float*)(ws + w.m32);
  uint16_t* P16 = (uint16_t*)(ws + w.p16);
  float* P32 = (float*)(ws + w.p32);
  float* Zt = (float*)(ws + w.zt);
  double* S = (double*)(ws + w.s64);
  double* Linv = (double*)(ws + w.linv);
  float* W = (float*)(ws + w.w32);
  double* Rsel = (double*)(ws + w.rsel);
  int* rotations = (int*)(ws + w.state);
  double* dmax = (double*)(ws + w.dmax);
  double* lam = (double*)(ws + w.lam);
  hipStream_t st = a.stream;
  const int np = w.n_pad;
  const ap_dtype dt = a.dt;

  hipLaunchKernelGGL(transpose16, dim3(np / 64, (HD + 63) / 64, B), dim3(256), 0, st, (const uint16_t*)a.X,
                     (int64_t)n * HD, HD, Xt, (int64_t)HD * np, np, n, HD);
  if (np > n) hipLaunchKernelGGL(fill_pad16, dim3(l, B), dim3(64), 0, st, Yt, (int64_t)l * np, np, n);
  const void* Pcur = a.Omega;
  int64_t p_bs = a.omega_batch_stride;
  ap_status s;
  for (int it = 0; it <= a.power_iters; ++it) {
    // Yt = P X^T  [l, n]
    NtGemmArgs g1{Pcur, p_bs, HD, a.X, (int64_t)n * HD, HD, Yt, (int64_t)l * np, np, nullptr, 0, B, l, n, HD, dt, 0, st};
    if ((s = launch_gemm_nt(g1)) != AP_OK) return s;
    // M = Yt X  [l, HD]  (X^T supplies rows that are contiguous along the token axis)
    NtGemmArgs g2{Yt, (int64_t)l * np, np, Xt, (int64_t)HD * np, np, M32, (int64_t)l * HD, HD, nullptr, 0, B, l, HD, np, dt, 2, st};
    if ((s = launch_gemm_nt(g2)) != AP_OK) return s;
    // rows of M made orthonormal
    launch_gram(M32, (int64_t)l * HD, HD, S, (int64_t)l * l, l, HD, B, st);
    hipLaunchKernelGGL(diag_max, dim3(B), dim3(256), 0, st, S, (int64_t)l * l, l, dmax);
    for (int c0 = 0; c0 < l; c0 += 32) {
      if (c0 > 0)
        hipLaunchKernelGGL(chol_update, dim3((l - c0 + 31) / 32, B), dim3(256), 0, st, S, (int64_t)l * l, l, c0);
      hipLaunchKernelGGL(chol_panel, dim3(B), dim3(256), 0, st, S, (int64_t)l * l, l, c0, dmax);
    }
    hipLaunchKernelGGL(tri_inverse, dim3((l + 3) / 4, B), dim3(256), (size_t)4 * l * 8, st, S, (int64_t)l * l, Linv, (int64_t)l * l, l);
    launch_gemm_nn<Tag>(Linv, (int64_t)l * l, l, M32, (int64_t)l * HD, HD, P32, (int64_t)l * HD, P16, (int64_t)l * HD,
                        HD, l, HD, l, 1, B, st);
    Pcur = P16;
    p_bs = (int64_t)l * HD;
  }
  // Rayleigh-Ritz in the span of P
  NtGemmArgs g4{P16, (int64_t)l * HD, HD, a.X, (int64_t)n * HD, HD, Zt, (int64_t)l * np, np, nullptr, 0, B, l, n, HD, dt, 2, st};
  if ((s = launch_gemm_nt(g4)) != AP_OK) return s;
  launch_gram(Zt, (int64_t)l * np, np, S, (int64_t)l * l, l, n, B, st);
  const int lp = w.lp;
  const int64_t w_bs = (int64_t)l * lp;
  hipLaunchKernelGGL(jacobi_init, dim3((l * lp + 255) / 256, B), dim3(256), 0, st, S, (int64_t)l * l, W, w_bs, l, lp, rotations);
  int nblk = (l + 15) / 16;
  nblk += nblk & 1;                                      // an even number of blocks (the last may be empty)
  for (int sweep = 0; sweep < kJacobiSweeps; ++sweep)
    for (int step = 0; step < nblk - 1; ++step)
      hipLaunchKernelGGL(jacobi_pair, dim3(nblk / 2 * B), dim3(512), 0, st, W, w_bs, l, lp, nblk, step, sweep, kJacobiTol,
                         rotations, B);
  hipLaunchKernelGGL(eig_norms, dim3((l + 3) / 4, B), dim3(256), 0, st, W, w_bs, l, lp, lam);
  hipLaunchKernelGGL(eig_select, dim3((l + 3) / 4, B), dim3(256), 0, st, W, w_bs, lam, l, lp, r, Rsel, (int64_t)r * l, a.sigma,
                     (int64_t)r);
  // D = R P  [r, HD]
  launch_gemm_nn<Tag>(Rsel, (int64_t)r * l, l, P32, (int64_t)l * HD, HD, nullptr, 0, (uint16_t*)a.Bm, (int64_t)r * HD,
                      HD, r, HD, l, 0, B, st);
  return check_launch("ap_compute_bases");
}

}  // namespace

size_t bases_workspace(int B, int n, int HD, int r, int oversample) {
  return bases_layout(B, n, HD, r + oversample, r).total;
}

ap_status launch_compute_bases(const BasesArgs& a) {
  return a.dt == AP_F16 ? run_bases<F16Tag>(a) : run_bases<BF16Tag>(a);
}

size_t decompress_workspace(int B, int T, int HD, int r, bool ranks) {
  return round_up((size_t)B * HD * r * 2, 256) + (ranks ? round_up((size_t)B * T * r * 2, 256) : 0);
}

// Xtilde[b, t, :] = C[b, t, :rank] D[b][:rank]  (16-bit in and out, fp32 accumulation)
ap_status launch_decompress(const void* C, const void* Bm, int64_t bstride, const int32_t* rank, void* X, int B, int T,
                            int T_cap, int HD, int r, ap_dtype dt, void* workspace, hipStream_t st) {
  uint16_t* Dt = (uint16_t*)workspace;                                     // [B or 1][HD][r]
  const int nb = bstride ? B : 1;
  hipLaunchKernelGGL(transpose16, dim3((r + 63) / 64, (HD + 63) / 64, nb), dim3(256), 0, st, (const uint16_t*)Bm,
                     bstride, HD, Dt, (int64_t)HD * r, r, r, HD);
  const void* A = C;
  int64_t a_bs = (int64_t)T_cap * r;
  if (rank) {
    uint16_t* Cm = (uint16_t*)((char*)workspace + round_up((size_t)B * HD * r * 2, 256));
    hipLaunchKernelGGL(mask_coeffs, dim3((T + 3) / 4, B), dim3(256), 0, st, (const uint16_t*)C, (int64_t)T_cap * r, rank,
                       (int64_t)T, Cm, (int64_t)T * r, T, r);
    A = Cm;
    a_bs = (int64_t)T * r;
  }
  NtGemmArgs g{A, a_bs, r, Dt, bstride ? (int64_t)HD * r : 0, r, X, (int64_t)T * HD, HD, nullptr, 0, B, T, HD, r, dt, 0, st};
  ap_status s = launch_gemm_nt(g);
  return s != AP_OK ? s : check_launch("ap_decompress");
}

}  // namespace ap
