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
//                                   S = L L^T (chol_panel, panels of 32 columns),
//                                   P = L^-1 M (tri_inverse, gemm_nn; fp64 accumulation)
//     Rayleigh-Ritz:           Zt = P X^T [l, n] fp32,  S = Zt Zt^T [l, l]  (= P X^T X P^T)
//                              S = L L^T,  L = J Sigma V^T by one-sided Jacobi on the columns of L (jacobi_pair)
//                              D = (J^T P)[:r] in decreasing order of Sigma, the singular values
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

// Matrix b of a flat grid of `per` workgroups per matrix and the workgroup's number t within it;
// matrix b on XCD b % 8 where that comes out even, so that what one launch leaves in an L2 is found
// there by the next.
__device__ __forceinline__ void matrix_of(int id, int per, int batch, int& b, int& t) {
  if (batch % 8 == 0) {
    b = (id >> 3) / per * 8 + (id & 7);
    t = (id >> 3) % per;
  } else {
    b = id / per;
    t = id - b * per;
  }
}

constexpr int kFirstCheck = 4;         // sweeps before this one do not ask whether the matrix is done (jacobi_check)
constexpr int kFullEvery = 4, kFullFrom = 8;   // steps and sweeps that turn the pairs within the blocks too
constexpr int kJacobiSweeps = 10;      // at most
constexpr int kSweepSlots = 16;        // per matrix: pairs of blocks that had work, one count per sweep, then whether a
                                       // sweep has work, one flag per sweep from kFirstCheck on
constexpr float kJacobiTol = 1e-5f;    // |a.b| <= tol |a||b|: far below what 16-bit storage of the result keeps

// ---- out[c][r] = in[r][c] for 16-bit elements; columns rows .. ld_out-1 of out are zero-filled.
//      Bound by memory: 16 bytes per lane in and out, 2-byte pieces only in LDS (195 us against 437 with
//      2-byte loads and stores at 16 x 4224 x 4096).  ld_in, cols, ld_out multiples of 8, out with
//      16-byte aligned rows.  WIDE: in too; without it only `in` itself is aligned and the batches may
//      lie any number of elements apart.
//      grid (ceil(ld_out / 64), ceil(cols / 64), batch), 256 threads.
template <bool WIDE>
__global__ void __launch_bounds__(256)
transpose16(const uint16_t* __restrict__ in, int64_t in_bstride, int ld_in, uint16_t* __restrict__ out,
            int64_t out_bstride, int ld_out, int rows, int cols) {
  constexpr int P = 72;                                  // elements per LDS row: 16-byte aligned
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * P];        // [column][row]
  const int tid = threadIdx.x, r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  in += (size_t)blockIdx.z * in_bstride;
  out += (size_t)blockIdx.z * out_bstride;
  u32x4_t v[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {                          // lanes 0-7 one row, ...: 128-byte pieces
    const int rr = (tid >> 3) + 32 * u, c = c0 + (tid & 7) * 8;
    const u32x4_t z = {0, 0, 0, 0};
    const uint16_t* src = in + (size_t)(r0 + rr) * ld_in + c;
    v[u] = z;
    if (r0 + rr < rows && c < cols) {
      if constexpr (WIDE) {
        v[u] = *(const u32x4_t*)src;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][e] = (uint32_t)src[2 * e] | (uint32_t)src[2 * e + 1] << 16;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int rr = (tid >> 3) + 32 * u, cc = (tid & 7) * 8;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile[(cc + 2 * e) * P + rr] = (uint16_t)v[u][e];
      tile[(cc + 2 * e + 1) * P + rr] = (uint16_t)(v[u][e] >> 16);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int cc = (tid >> 3) + 32 * u, r = r0 + (tid & 7) * 8;
    if (c0 + cc < cols && r < ld_out)
      *(u32x4_t*)(out + (size_t)(c0 + cc) * ld_out + r) = *(const u32x4_t*)(tile + cc * P + (tid & 7) * 8);
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
//      tiles, mirrored on the way out.  Bound by the fp64 matrix pipe.  The order of k is free as long as
//      both operands agree: a lane's 16 bytes of a row are four k of the product.
//      gram_f64 (64 x 64 tiles, a wave 32 x 32): 32 columns a stage go through LDS, the next stage's in
//      registers meanwhile.  Straight from memory, as gram_split takes them, a load's neighbouring lanes
//      are in different rows, which costs the CU 60 cycles an instruction against 16, as much as the
//      products take.  XCD-aware numbering keeps a matrix in one XCD's L2.  Waves whose 32 x 32 lies past the
//      end or above the diagonal do not multiply.  16 matrices of 544 x 4096: 512 us (612 straight from
//      memory, 1290 with fp64 FMAs), 20.5 GFLOP at 40 TFLOP/s; the pipe itself gives 47.5 (products of
//      registers, two waves per SIMD).
//      grid (tiles of the lower triangle * batch), 256 threads.
constexpr int kGramPitch = 36;                           // floats per LDS row: 16 rows start in 16 quads of banks
__global__ void __launch_bounds__(256)
gram_f64(const float* __restrict__ A, int64_t a_bstride, int lda, double* __restrict__ S, int64_t s_bstride,
         int l, int m, int batch) {
  __shared__ __attribute__((aligned(16))) float stage[2][128 * kGramPitch];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t64 = (l + 63) >> 6;
  int b, t;
  matrix_of((int)blockIdx.x, t64 * (t64 + 1) / 2, batch, b, t);
  // tile (ti, tj), tj <= ti, of the lower triangle
  int ti = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
  while (ti * (ti + 1) / 2 > t) --ti;
  const int tj = t - ti * (ti + 1) / 2;
  A += (size_t)b * a_bstride;
  S += (size_t)b * s_bstride;
  const int row = tid >> 3, piece = (tid & 7) * 4;       // a stage: 64 rows of either side, 128 bytes each
  const float* src[4];                                   // rows past the end repeat the last one
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = (u < 2 ? ti : tj) * 64 + (u & 1) * 32 + row;
    src[u] = A + (size_t)(i < l ? i : l - 1) * lda;
  }
  f32x4_t nx[4];
  auto load = [&](int c) {
    const int col = c * 32 + piece;
    const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const f32x4_t v = *(const f32x4_t*)(src[u] + (col < m ? col : 0));
      nx[u] = col < m ? v : z;
    }
  };
  f64x4_t acc[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) acc[u][v] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  const int stages = (m + 31) >> 5;
  const int ra = ((w >> 1) * 32 + n) * kGramPitch + 4 * g, rb = (64 + (w & 1) * 32 + n) * kGramPitch + 4 * g;
  const int i0 = ti * 64 + (w >> 1) * 32, j0 = tj * 64 + (w & 1) * 32;
  const bool mine = i0 < l && j0 <= i0;                  // else past the end, or the mirror image of another wave's
  load(0);
  for (int c = 0; c < stages; ++c) {
    float* buf = stage[c & 1];
#pragma unroll
    for (int u = 0; u < 4; ++u) *(f32x4_t*)(buf + (u * 32 + row) * kGramPitch + piece) = nx[u];
    if (c + 1 < stages) load(c + 1);
    lds_barrier();
    if (!mine) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4_t a0v = *(const f32x4_t*)(buf + ra + 16 * h), a1v = *(const f32x4_t*)(buf + ra + 16 * kGramPitch + 16 * h);
      const f32x4_t b0v = *(const f32x4_t*)(buf + rb + 16 * h), b1v = *(const f32x4_t*)(buf + rb + 16 * kGramPitch + 16 * h);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double a0 = a0v[e], a1 = a1v[e], b0 = b0v[e], b1 = b1v[e];
        acc[0][0] = mfma_f64(a0, b0, acc[0][0]);
        acc[0][1] = mfma_f64(a0, b1, acc[0][1]);
        acc[1][0] = mfma_f64(a1, b0, acc[1][0]);
        acc[1][1] = mfma_f64(a1, b1, acc[1][1]);
      }
    }
  }
  if (!mine) return;
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

// ---- the same for few or small matrices, which would leave most of the chip idle: the four waves share ONE
//      32 x 32 tile, a quarter of the columns each, operands straight from memory, and meet in LDS.
//      grid (tiles of the lower triangle, batch), 256 threads.
__global__ void __launch_bounds__(256)
gram_split(const float* __restrict__ A, int64_t a_bstride, int lda, double* __restrict__ S, int64_t s_bstride,
         int l, int m) {
  __shared__ double red[3 * 1024];
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // tile (ti, tj), tj <= ti, of the lower triangle
  int ti = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
  while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
  while (ti * (ti + 1) / 2 > (int)blockIdx.x) --ti;
  const int tj = (int)blockIdx.x - ti * (ti + 1) / 2;
  const int i0 = ti * 32, j0 = tj * 32;
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
  const int c_lo = (int)((int64_t)w * chunks / 4), c_hi = (int)((int64_t)(w + 1) * chunks / 4);
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
  // the four partial tiles, added in wave order
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
    hipLaunchKernelGGL(gram_f64, dim3(t64 * (t64 + 1) / 2 * batch), dim3(256), 0, st, A, a_bstride, lda, S, s_bstride, l, m, batch);
  else
    hipLaunchKernelGGL(gram_split, dim3(t32 * (t32 + 1) / 2, batch), dim3(256), 0, st, A, a_bstride, lda, S, s_bstride, l, m);
}

// ---- the largest diagonal entry of S and the sum of all: out[b], out[batch + b].  grid (batch), 256 threads.
__global__ void __launch_bounds__(256)
diag_stats(const double* __restrict__ S, int64_t s_bstride, int l, double* __restrict__ out) {
  const double* Sb = S + (size_t)blockIdx.x * s_bstride;
  __shared__ double red[8];
  double m = 0.0, sum = 0.0;
  for (int i = threadIdx.x; i < l; i += 256) {
    const double v = Sb[(size_t)i * l + i];
    m = fmax(m, v);
    sum += v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  sum = wave_sum_d(sum);
  if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = m; red[4 + (threadIdx.x >> 6)] = sum; }
  __syncthreads();
  if (threadIdx.x == 0) {
    out[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    out[gridDim.x + blockIdx.x] = (red[4] + red[5]) + (red[6] + red[7]);
  }
}

// ---- Cholesky S = L L^T, fp64, in panels of 32 columns, one launch per panel; off the diagonal the
//      lower triangle of S becomes L block by block, the diagonal blocks' INVERSES go to X (nothing
//      needs the diagonal blocks themselves: later panels and the inverse use what is below them).
//      A workgroup owns the 32 x 32 tile of its rows in this panel and works out the panel's diagonal
//      block next to it, every workgroup for itself: the products with the columns on the left for
//      both on the fp64 matrix instructions (a quarter of those columns per wave, added in LDS), the
//      factor of the diagonal block by one wave with two lanes per row (32 dependent steps, the
//      longest part of the chain), its inverse from two 16 x 16 halves, and the tile times that
//      inverse transposed.  What bounds it is this chain, not the arithmetic: 13-22 us a panel at 16
//      matrices of 544, 0.3 ms for all seventeen (an update launch and a one-workgroup factor launch
//      per panel with fp64 FMAs from LDS: 92 us a panel, 1.5 ms).
//      A pivot below 1e-13 of the largest diagonal entry (dmax) marks a direction that the rows
//      do not span: its column of L and its diagonal entry are zero, its row of L^-1 is zero,
//      so the corresponding row of P = L^-1 M is zero and drops out later.
//      FACTOR: X takes the diagonal blocks themselves, lower triangles.
//      grid (tiles from the diagonal down * batch), 256 threads.  l even.
template <bool FACTOR>
__global__ void __launch_bounds__(256)
chol_panel(double* __restrict__ S, double* __restrict__ X, int l, int c0, const double* __restrict__ dmax, int batch) {
  constexpr int P = 33, PC = 34;
  __shared__ double red[4][7 * 256];
  __shared__ double Dt[32 * P], At[32 * P], Di[32 * P], Lc[32 * PC], invd[32];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, t;
  matrix_of((int)blockIdx.x, (l - c0 + 31) >> 5, batch, b, t);
  double* L = S + (size_t)b * l * l;
  const int i0 = c0 + 32 * t;
  if (c0 > 0) {
    const double* rows[4];                               // the panel's rows, the tile's rows; past the end: the last
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int rc = c0 + 16 * u + n, ri = i0 + 16 * u + n;
      rows[u] = L + (size_t)(rc < l ? rc : l - 1) * l + 2 * g;
      rows[2 + u] = L + (size_t)(ri < l ? ri : l - 1) * l + 2 * g;
    }
    f64x4_t d00 = {0.0, 0.0, 0.0, 0.0}, d10 = d00, d11 = d00, a00 = d00, a01 = d00, a10 = d00, a11 = d00;
    const int k_lo = (c0 >> 2) * w, k_hi = k_lo + (c0 >> 2);   // a multiple of 8 columns each
    f64x2_t nx[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) nx[u] = *(const f64x2_t*)(rows[u] + k_lo);
    for (int k = k_lo; k < k_hi; k += 8) {
      f64x2_t cur[4];
      const int kn = k + 8 < k_hi ? k + 8 : k;
#pragma unroll
      for (int u = 0; u < 4; ++u) { cur[u] = nx[u]; nx[u] = *(const f64x2_t*)(rows[u] + kn); }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        d00 = mfma_f64(cur[0][e], cur[0][e], d00);
        d10 = mfma_f64(cur[1][e], cur[0][e], d10);
        d11 = mfma_f64(cur[1][e], cur[1][e], d11);
        if (t > 0) {
          a00 = mfma_f64(cur[2][e], cur[0][e], a00);
          a01 = mfma_f64(cur[2][e], cur[1][e], a01);
          a10 = mfma_f64(cur[3][e], cur[0][e], a10);
          a11 = mfma_f64(cur[3][e], cur[1][e], a11);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int at = (g + 4 * e) * 16 + n;
      red[w][at] = d00[e];
      red[w][256 + at] = d10[e];
      red[w][512 + at] = d11[e];
      red[w][768 + at] = a00[e];
      red[w][1024 + at] = a01[e];
      red[w][1280 + at] = a10[e];
      red[w][1536 + at] = a11[e];
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 7; ++q) {                          // S minus those products, tile by tile (tid = row, column)
    const int tr = q < 3 ? (q > 0) : (q > 4), tc = q < 3 ? (q > 1) : (q + 1) & 1;
    const int i = 16 * tr + (tid >> 4), c = 16 * tc + (tid & 15), row = (q < 3 ? c0 : i0) + i;
    double v = row < l && c0 + c < l ? L[(size_t)row * l + c0 + c] : 0.0;
    if (c0 > 0 && row < l && c0 + c < l)
      v -= (red[0][q * 256 + tid] + red[1][q * 256 + tid]) + (red[2][q * 256 + tid] + red[3][q * 256 + tid]);
    (q < 3 ? Dt : At)[i * P + c] = v;
  }
  __syncthreads();
  if (w == 0) {
    // the factor: lane (i, h) holds columns 16 h .. 16 h + 15 of row i; what a step does to columns
    // and rows that are finished, or to the unused upper triangle, is never read
    const int i = lane & 31, h = lane >> 5;
    const double tol = dmax[b] * 1e-13;
    double a[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) a[c] = h == 1 && i < 16 ? 0.0 : Dt[i * P + 16 * h + c];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int from = k + 32 * (k >> 4);                // the lane with the pivot
      const int2 pw = __builtin_bit_cast(int2, a[k & 15]);
      const double piv = __builtin_bit_cast(
          double, make_int2(__builtin_amdgcn_readlane(pw.x, from), __builtin_amdgcn_readlane(pw.y, from)));
      const bool live = piv > tol;
      const double ps = live ? piv : 1.0;
      double y = __builtin_amdgcn_rsq(ps);               // and two Newton steps: 1 / sqrt to rounding
      y = fma(y * 0.5, fma(-ps * y, y, 1.0), y);
      y = fma(y * 0.5, fma(-ps * y, y, 1.0), y);
      const double inv = live ? y : 0.0;
      if (h == (k >> 4)) Lc[k * PC + i] = a[k & 15] * inv;
      if (lane == 0) invd[k] = inv;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const double lik = Lc[k * PC + i];
#pragma unroll
      for (int c = 0; c < 16; ++c)
        if (16 + c > k) a[c] = fma(-lik, Lc[k * PC + 16 * h + c], a[c]);
    }
    // inverses of the two 16 x 16 halves of the diagonal: lane (column n, half g & 1), by columns
    const int hb = 16 * (g & 1);
    double x[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) x[c] = c == n ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      x[k] *= invd[hb + k];
#pragma unroll
      for (int c = k + 1; c < 16; ++c) x[c] = fma(-Lc[(hb + k) * PC + hb + c], x[k], x[c]);
    }
    if (g < 2) {
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        Di[(hb + c) * P + hb + n] = c < n ? 0.0 : x[c];
        if (g == 0) Di[c * P + 16 + n] = 0.0;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // below them: -(lower half)^-1 (L's lower left block) (upper half)^-1
    f64x4_t y = {0.0, 0.0, 0.0, 0.0}, z = y;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) y = mfma_f64(Lc[(4 * kk + g) * PC + 16 + n], Di[(4 * kk + g) * P + n], y);
    // element e of lane (n, g) of a product is row g + 4 e: as an operand that is k = g of group e
#pragma unroll
    for (int e = 0; e < 4; ++e) z = mfma_f64(Di[(16 + n) * P + 16 + 4 * e + g], y[e], z);
#pragma unroll
    for (int e = 0; e < 4; ++e) Di[(16 + g + 4 * e) * P + n] = -z[e];
  }
  __syncthreads();
  if (t == 0) {
    double* Xd = X + (size_t)b * l * l + (size_t)c0 * l + c0;
    for (int e = tid; e < 1024; e += 256) {
      const int i = e >> 5, c = e & 31;
      if (c0 + i < l && c0 + c < l) Xd[(size_t)i * l + c] = !FACTOR ? Di[i * P + c] : i >= c ? Lc[c * PC + i] : 0.0;
    }
    return;
  }
  // the tile times the inverse transposed, 16 x 16 per wave
  const int tr = 16 * (w >> 1), tc = 16 * (w & 1);
  f64x4_t y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) y = mfma_f64(At[(tr + n) * P + 4 * kk + g], Di[(tc + n) * P + 4 * kk + g], y);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = i0 + tr + g + 4 * e;
    if (row < l) L[(size_t)row * l + c0 + tc + n] = y[e];   // a tile below the diagonal has all its columns
  }
}

// ---- X = L^-1 in the blocks below the diagonal, from L's blocks there and the inverses of its diagonal
//      blocks (already in X): X_ij = -X_ii sum_{j <= k < i} L_ik X_kj.  A workgroup owns a column of
//      32 x 32 blocks and goes down it; the sum on the fp64 matrix instructions, its k shared out to
//      the four waves and added in LDS.  Blocks above the diagonal are not written: gemm_nn does not
//      read them.  The longest column first.  131 us at 16 matrices of 544 (a wave per column of
//      single rows, a reduction over the wave per element: 969 us).
//      grid ((blocks - 1) * batch), 256 threads.  l even.
__global__ void __launch_bounds__(256)
tri_inverse(const double* __restrict__ S, double* __restrict__ X, int l, int batch) {
  constexpr int P = 33;
  __shared__ double red[4][4 * 256], Ts[32 * P];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = (l + 31) >> 5;
  int b, j;
  matrix_of((int)blockIdx.x, nb - 1, batch, b, j);
  const double* L = S + (size_t)b * l * l;
  double* Xb = X + (size_t)b * l * l;
  const int jc = 32 * j;
  for (int i = j + 1; i < nb; ++i) {
    const double* rows[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ri = 32 * i + 16 * u + n;
      rows[u] = L + (size_t)(ri < l ? ri : l - 1) * l + 2 * g;
    }
    const double* cols = Xb + (size_t)(2 * g) * l + jc + n;
    f64x4_t acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) acc[u][v] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    const int per = 8 * (i - j), k_lo = jc + w * per, k_hi = k_lo + per;
    f64x2_t na[2], nx[2];                                // two k of either row tile, of either column tile
    auto load = [&](int k) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        na[u] = *(const f64x2_t*)(rows[u] + k);
        nx[u] = f64x2_t{cols[(size_t)k * l + 16 * u], cols[(size_t)(k + 1) * l + 16 * u]};
      }
    };
    load(k_lo);
    for (int k = k_lo; k < k_hi; k += 8) {
      f64x2_t ca[2], cx[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) { ca[u] = na[u]; cx[u] = nx[u]; }
      load(k + 8 < k_hi ? k + 8 : k);
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 2; ++v) acc[u][v] = mfma_f64(ca[u][e], cx[v][e], acc[u][v]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[w][(u * 2 + v) * 256 + (g + 4 * e) * 16 + n] = acc[u][v][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int at = q * 256 + tid;
      Ts[(16 * (q >> 1) + (tid >> 4)) * P + 16 * (q & 1) + (tid & 15)] = (red[0][at] + red[1][at]) + (red[2][at] + red[3][at]);
    }
    __syncthreads();
    // times -X_ii, 16 x 16 per wave; columns of X_ii past l meet rows of the sum that count for nothing
    const int tr = 16 * (w >> 1), tc = 16 * (w & 1), ri = 32 * i + tr + n;
    f64x4_t y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int k = 4 * kk + g;
      const double a = ri < l && 32 * i + k < l ? Xb[(size_t)ri * l + 32 * i + k] : 0.0;
      y = mfma_f64(a, Ts[k * P + tc + n], y);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 32 * i + tr + g + 4 * e;
      if (row < l) Xb[(size_t)row * l + jc + tc + n] = -y[e];
    }
    __syncthreads();                                     // the next rows' sum reads this block
  }
}

// S [l][l] -> L below the diagonal blocks of S; X: L^-1 (lower triangle of blocks) or, FACTOR, L's diagonal blocks.
template <bool FACTOR>
void launch_cholesky(double* S, double* X, int l, double* dstat, int batch, hipStream_t st) {
  hipLaunchKernelGGL(diag_stats, dim3(batch), dim3(256), 0, st, S, (int64_t)l * l, l, dstat);
  for (int c0 = 0; c0 < l; c0 += 32)
    hipLaunchKernelGGL(chol_panel<FACTOR>, dim3((l - c0 + 31) / 32 * batch), dim3(256), 0, st, S, X, l, c0, dstat, batch);
  if (!FACTOR && l > 32)
    hipLaunchKernelGGL(tri_inverse, dim3(((l + 31) / 32 - 1) * batch), dim3(256), 0, st, S, X, l, batch);
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
  matrix_of((int)blockIdx.x, per, batch, b, t);
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

// ---- W [l][lp] fp32 <- L^T, L [l][l] fp64 lower triangular: blocks of 32 below the diagonal in S, on it in X;
//      columns l .. lp-1 zero; the sweeps' counters and flags to zero.
//      grid (lp / 32, lp / 32, batch), 256 threads.
__global__ void __launch_bounds__(256)
jacobi_init(const double* __restrict__ S, const double* __restrict__ X, float* __restrict__ W, int64_t w_bstride, int l,
            int lp, int* __restrict__ state) {
  __shared__ float tile[32 * 33];
  const int b = blockIdx.z, c0 = blockIdx.x * 32, j0 = blockIdx.y * 32, x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const double* L = (c0 == j0 ? X : S) + (size_t)b * l * l;
#pragma unroll
  for (int k = 0; k < 32; k += 8) {
    const int c = c0 + y + k, j = j0 + x;                // row c of L
    tile[(y + k) * 33 + x] = c0 >= j0 && c < l && j < l ? (float)L[(size_t)c * l + j] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 32; k += 8)
    if (j0 + y + k < l) W[(size_t)b * w_bstride + (size_t)(j0 + y + k) * lp + c0 + x] = tile[x * 33 + y + k];
  if (c0 == 0 && j0 == 0 && threadIdx.x < 2 * kSweepSlots) state[b * 2 * kSweepSlots + threadIdx.x] = 0;
}

// The pairs of blocks that a launch takes from the round-robin over nblk blocks: those of one step, `skip` left
// out (none if skip >= nblk / 2), or (gather) pair `skip` of `count` steps from `step` on.
struct PairSet { int step, skip, gather, count; };

// ---- One-sided Jacobi on the rows of W [l][lp] (fp32), block version.  The rows are cut into blocks
//      of 16; one launch takes disjoint pairs of blocks (round-robin over the blocks), a workgroup per
//      pair.  For W = L^T, S = L L^T, the rows converge to sigma_i j_i^T, S's eigenvectors scaled by the square
//      roots of its eigenvalues.  (From W = S they converge to lambda_i j_i^T in more sweeps: 7 against 6 for
//      singular values j^-0.7 after two power iterations, 12 against 7 for j^-1.5, more than 15 against 9 where nothing was
//      iterated, simulated on the host.)
//      A workgroup never holds its 32 rows: it forms their Gram matrix G on the fp32 matrix
//      instructions, turns pairs of rows in two-sided rotations of G (steps of 16 disjoint pairs, the same
//      rotations that the rows themselves would see) while the product Q of the rotations is
//      built next to it, and multiplies the rows by Q on the matrix instructions.  The chain of
//      steps is what bounds it, so a step is kept short: G and Q are 32 x 32 in LDS, double-buffered,
//      one barrier a step, which leaves the rows' loads in flight alone.  The pairs of a step are always
//      positions (k, 16 + k); what a step writes goes to the position of the next step's partner, so all
//      addresses are constants.  `turns` = 16: every row of one block meets every row of the other (the
//      second block's positions move on by one).  31: every pair of the 32 rows (the circle method: position
//      0 stays, the others move on by one).  A row meets its own block's rows in 1 launch of 4 only: that
//      took as many sweeps as in every launch, over two spectra of 512 directions and a few random
//      matrices simulated on the host; in 1 launch of 33 a sweep more.
//      Waves 0-3 own 2 x 2 of G per thread and each work out all 16 rotations themselves; waves 4-7
//      follow one step behind with Q.
//      Blocks of 16: 17 pairs of a 544-row matrix, which fills the chip from 16 matrices on; the
//      number of steps per sweep hardly depends on the block (1023 against 1071 with blocks of 32),
//      nor does the number of sweeps (8 in both, the last of which only looks).
//      G is scaled by a power of two to a largest diagonal entry in [1, 2): no overflow in the angles.
//      A pair (x, y) is turned as x - sn (y + ta x), y + sn (x - ta y), ta the tangent of half the angle: the
//      cosine of a small angle rounds to 1 in fp32, and thousands of such rotations made the rows longer
//      (sigma of 544 equal directions 4.9e-5 too large with cosine and sine, see the test of it).
//      Measured at 16 matrices of 544 rows: 20 us a launch of 16 turns, 25 of 31, 4.9 ms in all (from W = S, a
//      last sweep that only looks and twelve sweeps' launches 5.4), of a launch's
//      15.5 us inside the kernel 4.4 the rows and G (out of memory: the L2s do not hold them over a launch),
//      1.6 its sum and the check, 5.5 the steps, 4.1 the rows' product.  31 turns in every launch, all pairs of
//      a step in one launch and the rows asked for after the check: 24 us and 7.0 ms; with the rows
//      themselves in LDS (blocks of 32, three dot products and a rotation of 544 columns per pair) 190 us a
//      launch and 21.9 ms.
//      state[b][sweep] counts the pairs of blocks that had work; from kFirstCheck on a sweep goes over the
//      matrices that jacobi_check has flagged for it.
//      grid (ps.count * batch), 512 threads.
__global__ void __launch_bounds__(512)
jacobi_pair(float* __restrict__ W, int64_t w_bstride, int l, int lp, int nblk, PairSet ps, int sweep, int turns,
            float tol, int* __restrict__ state, int batch) {
  constexpr int PITCH = 48;                             // 16 mod 32: two neighbouring rows fill the banks
  __shared__ float part[8][3 * 256];
  __shared__ float gm[2][32 * PITCH], qm[2][32 * PITCH];
  __shared__ f32x2_t rot[2][16];                        // sine and tangent of half the angle of a step's pairs
  __shared__ uint64_t busy[8];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, k;                                             // W stays in one XCD's L2
  matrix_of((int)blockIdx.x, ps.count, batch, b, k);
  if (sweep >= kFirstCheck && state[(2 * b + 1) * kSweepSlots + sweep] == 0) return;
  // round-robin over nblk blocks (nblk even; a block index >= the real count is an empty block)
  const int nm1 = nblk - 1;
  int ba, bb, step = ps.step;
  if (ps.gather) { step += k; k = ps.skip; }
  else if (k >= ps.skip) ++k;
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
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int at = (4 * g + e) * 16 + n;
    part[w][at] = g00[e];
    part[w][256 + at] = g01[e];
    part[w][512 + at] = g11[e];
  }
  lds_barrier();
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
  lds_barrier();
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
  const uint64_t vote = __ballot(work);
  if (lane == 0) busy[w] = vote;
  lds_barrier();
  uint64_t any = busy[0];
#pragma unroll
  for (int q = 1; q < 8; ++q) any |= busy[q];
  if (any == 0) return;                                 // every pair is orthogonal already
  if (tid == 0) atomicAdd(&state[2 * b * kSweepSlots + sweep], 1);
  const int sh = 1 - __builtin_amdgcn_frexp_expf(dmx);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int i = (tid >> 5) + 16 * u, j = tid & 31;
    gm[0][i * PITCH + j] = ldexpf(own[u], sh);
    qm[0][i * PITCH + j] = i == j ? 1.f : 0.f;
  }
  lds_barrier();

  const int I = 4 * (w & 3) + g;
  const bool within = turns == 31;
  auto moved = [&](int p) {
    if (!within) return p < 16 ? p : 16 + ((p + 1) & 15);
    return p == 0 ? 0 : p == 15 ? 31 : p == 16 ? 1 : p < 15 ? p + 1 : p - 1;
  };
  const int r0 = moved(I) * PITCH, r1 = moved(16 + I) * PITCH, c0 = moved(n), c1 = moved(16 + n);
  for (int s = 0; s <= turns; ++s) {                    // (by twos, with constant buffers: the same time)
    if (w < 4) {
      if (s < turns) {
        const float* cur = gm[s & 1];
        float* nxt = gm[(s & 1) ^ 1];
        const float al = cur[n * (PITCH + 1)], be = cur[(16 + n) * (PITCH + 1)], ga = cur[n * PITCH + 16 + n];
        const float a00 = cur[I * PITCH + n], a01 = cur[I * PITCH + 16 + n];
        const float a10 = cur[(16 + I) * PITCH + n], a11 = cur[(16 + I) * PITCH + 16 + n];
        // the rotation that makes the pair n orthogonal (any residue is far below the tolerance): the tangent
        // of its angle, 2 ga / (|d| + sqrt(d^2 + 4 ga^2)) with d's sign, whose denominator is at least |2 ga|
        // also where the squares vanish
        const float d = be - al, g2 = ga + ga;
        const float den = fmaxf(fabsf(d) + __builtin_amdgcn_sqrtf(fmaf(d, d, g2 * g2)), fabsf(g2));
        float t = (d < 0.f ? -g2 : g2) * __builtin_amdgcn_rcpf(den);
        t = fabsf(ga) > 1e-30f ? t : 0.f;
        const float cs = __builtin_amdgcn_rsqf(fmaf(t, t, 1.f)), sn = cs * t;
        const float ta = sn * __builtin_amdgcn_rcpf(1.f + cs);   // tan of half the angle: cos = 1 - sn ta
        const float si = __shfl(sn, I), ti = __shfl(ta, I);
        if (w == 0 && g == 0) rot[s & 1][n] = f32x2_t{sn, ta};
        const float b00 = fmaf(-si, fmaf(ti, a00, a10), a00), b01 = fmaf(-si, fmaf(ti, a01, a11), a01);
        const float b10 = fmaf(si, fmaf(-ti, a10, a00), a10), b11 = fmaf(si, fmaf(-ti, a11, a01), a11);
        nxt[r0 + c0] = fmaf(-sn, fmaf(ta, b00, b01), b00);
        nxt[r0 + c1] = fmaf(sn, fmaf(-ta, b01, b00), b01);
        nxt[r1 + c0] = fmaf(-sn, fmaf(ta, b10, b11), b10);
        nxt[r1 + c1] = fmaf(sn, fmaf(-ta, b11, b10), b11);
      }
    } else if (s > 0) {
      const float* cur = qm[(s & 1) ^ 1];
      float* nxt = qm[s & 1];
      const f32x2_t r = rot[(s & 1) ^ 1][I];
      const float a00 = cur[I * PITCH + n], a01 = cur[I * PITCH + 16 + n];
      const float a10 = cur[(16 + I) * PITCH + n], a11 = cur[(16 + I) * PITCH + 16 + n];
      nxt[r0 + n] = fmaf(-r[0], fmaf(r[1], a00, a10), a00);
      nxt[r0 + 16 + n] = fmaf(-r[0], fmaf(r[1], a01, a11), a01);
      nxt[r1 + n] = fmaf(r[0], fmaf(-r[1], a10, a00), a10);
      nxt[r1 + 16 + n] = fmaf(r[0], fmaf(-r[1], a11, a01), a11);
    }
    lds_barrier();
  }

  // rows <- Q rows
  const float* Q = qm[turns & 1];
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

// ---- whether a matrix has work for sweep `sweep`: any two rows of W further from orthogonal than tol.  A sweep that
//      only looks costs 34 launches of 10 us at 16 matrices of 544, this one launch.  A matrix whose last sweep had
//      work in most of its `pairs` is flagged without a look.
//      64 x 64 tiles of W W^T as in gram_f64, in fp32 products; the rows' norms from what goes through LDS.
//      grid (tiles of the lower triangle * batch), 256 threads.
__global__ void __launch_bounds__(256)
jacobi_check(const float* __restrict__ W, int64_t w_bstride, int l, int lp, int sweep, int pairs, float tol,
             int* __restrict__ state, int batch) {
  __shared__ __attribute__((aligned(16))) float stage[2][128 * kGramPitch];
  __shared__ float norm[128];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t64 = (l + 63) >> 6;
  int b, t;
  matrix_of((int)blockIdx.x, t64 * (t64 + 1) / 2, batch, b, t);
  int* flag = state + (2 * b + 1) * kSweepSlots + sweep;
  if (sweep > kFirstCheck && flag[-1] == 0) return;
  if (2 * state[2 * b * kSweepSlots + sweep - 1] > pairs) {
    if (t == 0 && tid == 0) *flag = 1;
    return;
  }
  int ti = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
  while (ti * (ti + 1) / 2 > t) --ti;
  const int tj = t - ti * (ti + 1) / 2;
  W += (size_t)b * w_bstride;
  const int row = tid >> 3, piece = (tid & 7) * 4;       // a stage: 64 rows of either side, 32 columns each
  const float* src[4];
  float sq[4];
  f32x4_t nx[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = (u < 2 ? ti : tj) * 64 + (u & 1) * 32 + row;
    src[u] = W + (size_t)(i < l ? i : l - 1) * lp + piece;   // rows past the end repeat the last one
    nx[u] = *(const f32x4_t*)src[u];
    sq[u] = 0.f;
  }
  f32x4_t acc[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) acc[u][v] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int stages = lp >> 5;
  const int ra = ((w >> 1) * 32 + n) * kGramPitch + 4 * g, rb = (64 + (w & 1) * 32 + n) * kGramPitch + 4 * g;
  for (int c = 0; c < stages; ++c) {
    float* buf = stage[c & 1];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      *(f32x4_t*)(buf + (u * 32 + row) * kGramPitch + piece) = nx[u];
#pragma unroll
      for (int e = 0; e < 4; ++e) sq[u] = fmaf(nx[u][e], nx[u][e], sq[u]);
      nx[u] = *(const f32x4_t*)(src[u] + (c + 1 < stages ? c + 1 : c) * 32);
    }
    lds_barrier();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4_t a0 = *(const f32x4_t*)(buf + ra + 16 * h), a1 = *(const f32x4_t*)(buf + ra + 16 * kGramPitch + 16 * h);
      const f32x4_t b0 = *(const f32x4_t*)(buf + rb + 16 * h), b1 = *(const f32x4_t*)(buf + rb + 16 * kGramPitch + 16 * h);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[e], b0[e], acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[e], b1[e], acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[e], b0[e], acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[e], b1[e], acc[1][1], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float s = group_sum<8>(sq[u]);
    if ((tid & 7) == 0) norm[u * 32 + row] = sqrtf(s);
  }
  lds_barrier();
  int work = 0;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {                      // element e of lane (n, g): row 4 g + e, column n
        const int i = (w >> 1) * 32 + 16 * u + 4 * g + e, j = (w & 1) * 32 + 16 * v + n;
        if (ti * 64 + i < l && tj * 64 + j < ti * 64 + i && fabsf(acc[u][v][e]) > tol * (norm[i] * norm[64 + j])) work = 1;
      }
  if (__ballot(work) != 0 && lane == 0) *flag = 1;
}

// ---- singular values = row norms.  grid (ceil(l / 4), batch), 256 threads: a wave per row.
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
//      become R [r][l] (fp64) and sigma.  Thousands of rotations in fp32 change the rows' lengths by some 1e-6, all
//      of them alike; what they may not change is the sum of squares, S's trace, which sigma is scaled to.
//      grid (ceil(l / 4), batch), 256 threads: a wave per row, which counts the rows before its own (one workgroup per
//      matrix, which also took the norms, needed 197 us at 16 x 544 rows).
__global__ void __launch_bounds__(256)
eig_select(const float* __restrict__ W, int64_t w_bstride, const double* __restrict__ lam, const double* __restrict__ trace,
           int l, int lp, int r, double* __restrict__ R, int64_t r_bstride, float* __restrict__ sigma, int64_t sig_bstride) {
  const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6), b = blockIdx.y;
  if (i >= l) return;
  const double* lb = lam + (size_t)b * l;
  const double li = lb[i];
  int p = 0;
  double sum = 0.0;
  for (int j = lane; j < l; j += 64) {
    p += (lb[j] > li || (lb[j] == li && j < i)) ? 1 : 0;
    sum = fma(lb[j], lb[j], sum);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) p += __shfl_xor(p, o);
  sum = wave_sum_d(sum);
  if (p >= r) return;
  if (lane == 0 && sigma) sigma[(size_t)b * sig_bstride + p] = (float)(sum > 0.0 ? li * sqrt(trace[b] / sum) : li);
  const double inv = li > 0.0 ? 1.0 / li : 0.0;
  const float* row = W + (size_t)b * w_bstride + (size_t)i * lp;
  for (int c = lane; c < l; c += 64) R[(size_t)b * r_bstride + (size_t)p * l + c] = (double)row[c] * inv;
}

struct BasesLayout {
  size_t xt, yt, m32, p16, p32, zt, s64, linv, w32, rsel, state, dstat, lam, total;
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
  w.state = take((size_t)B * 2 * kSweepSlots * 4);
  w.dstat = take((size_t)B * 2 * 8);
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
  int* state = (int*)(ws + w.state);
  double* dstat = (double*)(ws + w.dstat);
  double* lam = (double*)(ws + w.lam);
  hipStream_t st = a.stream;
  const int np = w.n_pad;
  const ap_dtype dt = a.dt;

  hipLaunchKernelGGL((transpose16<true>), dim3(np / 64, (HD + 63) / 64, B), dim3(256), 0, st, (const uint16_t*)a.X,
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
    launch_cholesky<false>(S, Linv, l, dstat, B, st);
    // (the fp32 copy is what D is made from in the end: the last iteration's only)
    launch_gemm_nn<Tag>(Linv, (int64_t)l * l, l, M32, (int64_t)l * HD, HD, it == a.power_iters ? P32 : nullptr,
                        (int64_t)l * HD, P16, (int64_t)l * HD, HD, l, HD, l, 1, B, st);
    Pcur = P16;
    p_bs = (int64_t)l * HD;
  }
  // Rayleigh-Ritz in the span of P
  NtGemmArgs g4{P16, (int64_t)l * HD, HD, a.X, (int64_t)n * HD, HD, Zt, (int64_t)l * np, np, nullptr, 0, B, l, n, HD, dt, 2, st};
  if ((s = launch_gemm_nt(g4)) != AP_OK) return s;
  launch_gram(Zt, (int64_t)l * np, np, S, (int64_t)l * l, l, n, B, st);
  const int lp = w.lp;
  const int64_t w_bs = (int64_t)l * lp;
  launch_cholesky<true>(S, Linv, l, dstat, B, st);       // (Linv: the diagonal blocks)
  hipLaunchKernelGGL(jacobi_init, dim3(lp / 32, lp / 32, B), dim3(256), 0, st, S, Linv, W, w_bs, l, lp, state);
  int nblk = (l + 15) / 16;
  nblk += nblk & 1;                                      // an even number of blocks (the last may be empty)
  const int P = nblk / 2, nm1 = nblk - 1;
  // Two workgroups on one CU hold each other up (15.5 us alone, 16.5 and 22 together: the steps fill half the
  // CU's issue slots, and the rows come in later), so a launch that puts a second one on a few CUs only lasts
  // as long as one that does on all.  Where a pair less per matrix keeps to one per CU, each step leaves out
  // pair `skip`; with skip a quarter of the steps, up to half the steps' pairs touch each block once and are
  // made up for in one launch.  From eight pairs on: below, the additional launches outweigh it.  (For a given batch
  // one band of 32 directions: 513 to 544 of 16 matrices, 225 to 256 of 35.)
  const int skip = nm1 / 4, run = min(2 * skip, nm1 - 2 * skip);
  const bool spare = P >= 8 && P * B > 256 && (P - 1) * B <= 256;
  auto turn = [&](int sweep, PairSet ps, int turns) {
    hipLaunchKernelGGL(jacobi_pair, dim3(ps.count * B), dim3(512), 0, st, W, w_bs, l, lp, nblk, ps, sweep, turns, kJacobiTol,
                       state, B);
  };
  const int t64 = (l + 63) / 64;
  for (int sweep = 0; sweep < kJacobiSweeps; ++sweep) {
    if (sweep >= kFirstCheck)
      hipLaunchKernelGGL(jacobi_check, dim3(t64 * (t64 + 1) / 2 * B), dim3(256), 0, st, W, w_bs, l, lp, sweep, P * nm1, kJacobiTol,
                         state, B);
    for (int step = 0; step < nm1; ++step) {
      const bool out = spare && step < 2 * run;
      turn(sweep, PairSet{step, out ? skip : P, 0, out ? P - 1 : P}, step % kFullEvery == 0 || sweep >= kFullFrom ? 31 : 16);
      if (out && (step + 1) % run == 0) turn(sweep, PairSet{step + 1 - run, skip, 1, run}, 16);
    }
  }
  hipLaunchKernelGGL(eig_norms, dim3((l + 3) / 4, B), dim3(256), 0, st, W, w_bs, l, lp, lam);
  hipLaunchKernelGGL(eig_select, dim3((l + 3) / 4, B), dim3(256), 0, st, W, w_bs, lam, dstat + B, l, lp, r, Rsel, (int64_t)r * l, a.sigma,
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
  // any distance between the bases is taken; one that is no multiple of 8 elements leaves their rows
  // without the 16-byte alignment that wide loads need
  auto kern = bstride % 8 == 0 ? transpose16<true> : transpose16<false>;
  hipLaunchKernelGGL(kern, dim3((r + 63) / 64, (HD + 63) / 64, nb), dim3(256), 0, st, (const uint16_t*)Bm,
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
