// Per-step products on ONE basis for all sequences (basis_batch_stride = 0): every basis row then
// serves all of them, so the appends, the fold and the expansion are matrix products and run on the
// matrix cores; with a basis per sequence they are matrix-vector products (basis_gemv.hip).
//
//   shared_project   c[b, j]  = Bm[j, :] . x[b, :]                 the appended rows (keys and values)
//                    q'[h, j] = scale Bm[j, slice of h] . q[b, h]  the folded queries, hi + lo halves
//                    in one launch
//   shared_expand    out[b, h, :] = (sum_s w_s U_s[b, h, :] / sum_s w_s l_s) . Bv[:, slice of h]
//
// Products of two 16-bit values are exact in the matrix cores' fp32 sums.  The expansion multiplies the merged fp32
// sums with the basis: fp16 in fp32 products (v_mfma_f32_16x16x4_f32); bfloat16 with the sums cut into three
// bfloat16 values, whose products are exact, so the result is that of fp32 products.
#include "ap_common.hpp"
#include "lane_ops.hpp"
#include "mfma_ops.hpp"

namespace ap {
namespace {

// Workgroups go round the XCDs: unit numbers in one run per XCD, so that neighbouring units (the same
// basis rows, the same head's slice) meet in one L2.  Numbers >= units are spare.
__device__ __forceinline__ int run_per_xcd(int id, int units) { return (id & 7) * ((units + 7) >> 3) + (id >> 3); }

struct ProjectParams {
  const uint16_t* Bm[2];    // [r][HD]: keys' basis, values' basis
  const uint16_t* x[2];     // [B][HD] token rows to project
  uint16_t* C[2];           // [B][T_cap][r], row `row0` written
  const uint16_t* q;        // [B][H][d]
  uint16_t* Qp;             // [B][2][Hp][r]
  int B, H, G, Hp, HD, r, row0, T_cap;
  int dot_units, fold_units, dot_blocks;
  float scale;
};

// 512 threads.  Two kinds of workgroups, the longer first:
//   dot    16 basis rows x 16 NB sequences, 256 elements of the hidden axis a stage: a wave takes 32 of
//          them, four stages are in flight in registers, two in LDS; the waves' sums are added in order
//   fold   one key/value head, 128 basis rows x 64 (sequence, query head) columns, a wave 64 x 16
// Operands go through LDS: loaded straight into the products' operand registers, neighbouring lanes hold
// different rows and every lane is an address of its own (60 cycles a load against 16; 31 us for 64
// sequences, 40 heads, rank 640, and 17 through LDS; matrix-vector products per sequence: 76).
template <class Tag, int KS, int NB>
__global__ void __launch_bounds__(512) shared_project(const ProjectParams p) {
  constexpr int d = KS * 32;
  extern __shared__ __attribute__((aligned(16))) uint16_t smem_sp[];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int HD = p.HD, r = p.r;
  const u32x4_t z = {0, 0, 0, 0};
  if ((int)blockIdx.x < p.dot_blocks) {
    const int u = run_per_xcd(blockIdx.x, p.dot_units);
    if (u >= p.dot_units) return;
    const int nbt = (p.B + 16 * NB - 1) / (16 * NB);
    const int jj = u / nbt, bt = u - jj * nbt, job = jj & 1, j0 = (jj >> 1) * 16, b0 = bt * 16 * NB;
    constexpr int kRing = 4, kRows = 16 + 16 * NB, kPitch = 256 + 8;
    const int row = tid >> 5, ch = (tid & 31) * 8;            // this thread's piece of 16 rows at a time
    const uint16_t* src[1 + NB];
    src[0] = p.Bm[job] + (size_t)(j0 + row) * HD;
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int b = b0 + 16 * t + row;                        // past the batch: a repeat, dropped
      src[1 + t] = p.x[job] + (size_t)(b < p.B ? b : p.B - 1) * HD;
    }
    u32x4_t ring[kRing][1 + NB];
    auto load_stage = [&](u32x4_t (&v)[1 + NB], int st) {
      const int k = st * 256 + ch < HD ? st * 256 + ch : 0;
#pragma unroll
      for (int i = 0; i < 1 + NB; ++i) v[i] = *(const u32x4_t*)(src[i] + k);
    };
    f32x4_t acc[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int nst = (HD + 255) >> 8;
#pragma unroll
    for (int i = 0; i < kRing; ++i) load_stage(ring[i], i);
    for (int s0 = 0; s0 < nst; s0 += kRing) {                 // stages past the hidden axis are zeros
#pragma unroll
      for (int i = 0; i < kRing; ++i) {
        uint16_t* buf = smem_sp + (i & 1) * kRows * kPitch;
        const bool in = (s0 + i) * 256 + ch < HD;
#pragma unroll
        for (int t = 0; t < 1 + NB; ++t) *(u32x4_t*)(buf + (16 * t + row) * kPitch + ch) = in ? ring[i][t] : z;
        load_stage(ring[i], s0 + i + kRing);
        lds_barrier();
        const u32x4_t av = *(const u32x4_t*)(buf + n * kPitch + w * 32 + g * 8);
#pragma unroll
        for (int t = 0; t < NB; ++t)
          acc[t] = Mfma<Tag>::run(av, *(const u32x4_t*)(buf + (16 + 16 * t + n) * kPitch + w * 32 + g * 8), acc[t]);
      }
    }
    lds_barrier();
    f32x4_t (*part)[NB][64] = (f32x4_t(*)[NB][64])smem_sp;
#pragma unroll
    for (int t = 0; t < NB; ++t) part[w][t][lane] = acc[t];
    lds_barrier();
    if (w < NB) {
      f32x4_t s = part[0][w][lane];
#pragma unroll
      for (int k = 1; k < 8; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += part[k][w][lane][e];
      const int b = b0 + 16 * w + n;
      if (b < p.B) {
        u32x2_t v = {pack2(s[0], s[1], Tag{}), pack2(s[2], s[3], Tag{})};
        *(u32x2_t*)(p.C[job] + ((size_t)b * p.T_cap + p.row0) * r + j0 + 4 * g) = v;
      }
    }
    return;
  }
  // ---- fold
  const int id = blockIdx.x - p.dot_blocks;
  const int u = run_per_xcd(id, p.fold_units);
  if (u >= p.fold_units) return;
  const int njb = (r + 127) >> 7, N = p.B * p.G, nct = (N + 63) >> 6;
  const int jb = u % njb, cu = u / njb, ct = cu % nct, kvh = cu / nct;
  constexpr int kPitch = d + 8, kLanes = d / 8, kPass = 512 / kLanes, kN = (192 + kPass - 1) / kPass;
  const int ch = tid % kLanes * 8, prow = tid / kLanes;
  {
    const uint16_t* bcol = p.Bm[0] + (size_t)kvh * d + ch;
    u32x4_t v[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const int row = i * kPass + prow;                       // 128 basis rows, then 64 columns of queries
      const uint16_t* src;
      if (i * kPass < 128) {
        const int j = jb * 128 + row;
        src = bcol + (size_t)(j < r ? j : r - 1) * HD;
      } else {
        const int c = ct * 64 + row - 128, cc = c < N ? c : N - 1, b = cc / p.G;
        src = p.q + ((size_t)b * p.H + kvh * p.G + (cc - b * p.G)) * d + ch;
      }
      v[i] = *(const u32x4_t*)src;
    }
    __builtin_amdgcn_sched_barrier(0);                        // all requests before the first use
#pragma unroll
    for (int i = 0; i < kN; ++i)
      if (i * kPass + prow < 192) *(u32x4_t*)(smem_sp + (i * kPass + prow) * kPitch + ch) = v[i];
  }
  lds_barrier();
  const int j0 = jb * 128 + (w >> 2) * 64, c = ct * 64 + (w & 3) * 16 + n;
  if (j0 < r) {
    // operand row m of product t is basis row 32 (t / 2) + 8 (m / 4) + 4 (t % 2) + m % 4: a lane then ends with
    // eight consecutive rank positions per pair of products, and a store of 16 bytes a lane fills 64 bytes a column
    const uint16_t* arow = smem_sp + ((w >> 2) * 64 + (n >> 2) * 8 + (n & 3)) * kPitch + g * 8;
    const uint16_t* qrow = smem_sp + (128 + (w & 3) * 16 + n) * kPitch + g * 8;
    u32x4_t qv[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) qv[k] = *(const u32x4_t*)(qrow + k * 32);
    uint32_t hi[4][2], lo[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KS; ++k)
        acc = Mfma<Tag>::run(*(const u32x4_t*)(arow + ((t >> 1) * 32 + (t & 1) * 4) * kPitch + k * 32), qv[k], acc);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float x = acc[2 * e] * p.scale, y = acc[2 * e + 1] * p.scale;
        hi[t][e] = cvt_pack(x, y, Tag{});
        lo[t][e] = cvt_pack(x - lo_to_f32(hi[t][e], Tag{}), y - hi_to_f32(hi[t][e], Tag{}), Tag{});
      }
    }
    if (c < N) {
      const int b = c / p.G, h = kvh * p.G + c - b * p.G;
      uint16_t* o = p.Qp + (((size_t)b * 2) * p.Hp + h) * r + j0 + 8 * g;
      uint16_t* ol = o + (size_t)p.Hp * r;
#pragma unroll
      for (int t = 0; t < 4; t += 2) {
        *(u32x4_t*)(o + 16 * t) = u32x4_t{hi[t][0], hi[t][1], hi[t + 1][0], hi[t + 1][1]};
        *(u32x4_t*)(ol + 16 * t) = u32x4_t{lo[t][0], lo[t][1], lo[t + 1][0], lo[t + 1][1]};
      }
    }
  }
  if (p.Hp > p.H) {                                           // padded heads stay 0: a share for every workgroup
    const int per = (p.Hp - p.H) * r / 8, total = p.B * 2 * per, share = (total + p.fold_units - 1) / p.fold_units;
    const int end = (int64_t)(u + 1) * share < total ? (u + 1) * share : total;
    for (int64_t i = (int64_t)u * share + tid; i < end; i += 512) {
      const int bp = (int)i / per;
      *(u32x4_t*)(p.Qp + ((size_t)bp * p.Hp + p.H) * r + (size_t)((int)i - bp * per) * 8) = z;
    }
  }
}

struct SharedExpandParams {
  const float* part_ml;     // [B][S][H][2]
  const float* part_U;      // [B][S][H][r]
  const uint16_t* Bv;       // [r][HD]
  void* out;                // [B][H][d]
  float* lse;               // [B][H] or null
  int B, H, G, HD, r, S, units;
};

// Two fp32 values as sums of three bfloat16 values each, eight bits at a time from the top: exact from 2^-100 on, and
// never above the value itself (rounded, a sum between the largest bfloat16 and the largest fp32 would be infinite).
// What is not finite stays in the first part.
__device__ __forceinline__ void split3(float x, float y, uint32_t (&v)[3]) {
  auto top = [](float f) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, f) & 0xffff0000u); };
  auto pack = [](float lo, float hi) {
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x07060302);
  };
  const float rx = __builtin_isfinite(x) ? x - top(x) : 0.f, ry = __builtin_isfinite(y) ? y - top(y) : 0.f;
  v[0] = pack(x, y);
  v[1] = pack(rx, ry);
  v[2] = pack(rx - top(rx), ry - top(ry));
}

// A workgroup (512 threads) merges and expands 16 (sequence, query head) columns of one key/value head.
// The merge (32 lanes a column) leaves U*, times L or what is left of it, in LDS; the waves then take every eighth group of 32
// basis rows.  A lane loads VEC = d / 16 consecutive elements of eight rows: product i holds the hidden columns VEC a + i, so a
// lane ends with VEC consecutive columns per accumulator row.
//   bfloat16  U* as three 16-bit parts, eight rows of an element the operand of one product (byte permutes); the
//             parts' products are exact and summed in fp32, smallest first.  With an infinite basis element the parts
//             could cancel, and parts of a sum below 2^-100 lose bits: a wave that ends with something that is not
//             finite, or a workgroup with such sums, does the fp32 products
//   fp16      fp32 products (v_mfma_f32_16x16x4_f32), four rows each: fp16 has too few exponents for parts of a
//             sum that is small beside its column's largest
// 64 x 640, 40 heads, four splits: bfloat16 12.9 us (26.3 with a workgroup per head and sequence), most of it loads on
// their way; fp16 16.1 us (12.1 with three fp16 parts, which were 7e-4 off where 2^-30 of the largest was all).
template <class Tag, bool OUT_F32, int VEC>
__global__ void __launch_bounds__(512) shared_expand(const SharedExpandParams p) {
  constexpr int d = VEC * 16, DW = VEC / 2;                   // DW dwords of a row per lane
  constexpr int kChunks = 5, kU = 4;                          // 4 x 32 columns a chunk, r <= 640; splits at a time
  constexpr bool kParts = __is_same(Tag, BF16Tag);
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int u = run_per_xcd(blockIdx.x, p.units);
  if (u >= p.units) return;
  const int S = p.S, H = p.H, r = p.r, G = p.G, N = p.B * G, nct = (N + 15) >> 4;
  const int kvh = u / nct, ct = u - kvh * nct, sp = S + 1;
  const int pitch = r + 8, pitch32 = r + 4;
  uint16_t* parts = (uint16_t*)smem;                          // bfloat16: U* as [3][16][pitch]
  float* ustar = smem;                                        // fp16: as [16][pitch32]
  float* wgt = smem + (kParts ? 3 * 16 * pitch / 2 : 16 * pitch32);   // [16][sp] weights
  int* flags = (int*)(wgt + 16 * sp);                         // bfloat16: per wave, sums too small for parts
  float* sums = smem;                                         // [4][16][d + 4], once U* is used up
  // ---- this thread's column; the first splits' sums
  const int c = tid >> 5, ci = tid & 31;
  const int cc = ct * 16 + c < N ? ct * 16 + c : N - 1;       // past the columns: a repeat, dropped
  const int b = cc / G, h = kvh * G + cc - b * G;
  const uint32_t split_bytes = (uint32_t)H * r * 4;
  const auto bsum = make_buffer(p.part_U + ((size_t)b * S * H + h) * r, (uint32_t)(S - 1) * split_bytes + r * 4);
  const float* ml = p.part_ml + ((size_t)b * S * H + h) * 2;
  const f32x2_t ml0 = *(const f32x2_t*)(ml + (size_t)(ci < S ? ci : S - 1) * H * 2);
  const f32x2_t ml1 = *(const f32x2_t*)(ml + (size_t)(ci + 32 < S ? ci + 32 : S - 1) * H * 2);
  u32x4_t uv[kChunks][kU];
  auto load_sums = [&](int s0) {                              // zeros past the rank
#pragma unroll
    for (int s = 0; s < kU; ++s) {
      const uint32_t so = (uint32_t)(s0 + s < S ? s0 + s : S - 1) * split_bytes;
#pragma unroll
      for (int k = 0; k < kChunks; ++k) uv[k][s] = buffer_load16(bsum, 128 * k + 4 * ci < r ? so + 512 * k + 16 * ci : 0x80000000u);
    }
  };
  load_sums(0);
  // ---- basis rows, requested next: group i of this wave is rows 32 (w + 8 i) + 8 g + t
  constexpr int kAhead = VEC > 8 ? 1 : 2;
  const int groups = r >> 5;
  uint32_t bv[kAhead][8][DW];
  const uint16_t* bcol = p.Bv + (size_t)kvh * d + n * VEC;
  auto load_group = [&](uint32_t (&dst)[8][DW], int gi) {
    const int gc = gi < groups ? gi : groups - 1;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint16_t* src = bcol + (size_t)(gc * 32 + 8 * g + t) * p.HD;
      if constexpr (DW == 1) dst[t][0] = *(const uint32_t*)src;
      else if constexpr (DW == 2) { const u32x2_t v = *(const u32x2_t*)src; dst[t][0] = v[0]; dst[t][1] = v[1]; }
      else {
#pragma unroll
        for (int k = 0; k < DW / 4; ++k) {
          const u32x4_t v = *(const u32x4_t*)(src + 8 * k);
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[t][4 * k + e] = v[e];
        }
      }
    }
  };
#pragma unroll
  for (int k = 0; k < kAhead; ++k) load_group(bv[k], w + 8 * k);
  // ---- weights 2^(m_s - m*) and their weighted sum of l (S <= 64: two splits a lane)
  float m = fmaxf(ml0[0], ml1[0]);                            // past the splits: repeats of the last
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  const float w0 = ci < S ? fast_exp2(ml0[0] - m) : 0.f, w1 = ci + 32 < S ? fast_exp2(ml1[0] - m) : 0.f;
  float L = ci < S ? w0 * ml0[1] : 0.f;
  L = ci + 32 < S ? fmaf(w1, ml1[1], L) : L;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) L += __shfl_xor(L, o);
  if (ci < S) wgt[c * sp + ci] = w0;
  if (ci + 32 < S) wgt[c * sp + ci + 32] = w1;
  if (p.lse && ci == 0 && ct * 16 + c < N) p.lse[(size_t)b * H + h] = (m + log2f(L)) * kLn2;
  __builtin_amdgcn_wave_barrier();                            // a column's weights stay within its half wave
  // ---- sum_s w_s U_s; the division by L is left to the results, which are fewer.  bfloat16, where the sums may be near
  // the end of fp32: but for a power of two that brings L to [0.5, 1), so that nothing is larger than with U* itself
  const int le = kParts ? __builtin_amdgcn_frexp_expf(L) : 0;
  f32x4_t ua[kChunks];
#pragma unroll
  for (int k = 0; k < kChunks; ++k) ua[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < S; s0 += kU) {
    if (s0) load_sums(s0);
#pragma unroll
    for (int s = 0; s < kU; ++s) {
      if (s0 + s < S) {
        const float ws = wgt[c * sp + s0 + s];
#pragma unroll
        for (int k = 0; k < kChunks; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) ua[k][e] = fmaf(ws, __builtin_bit_cast(f32x4_t, uv[k][s])[e], ua[k][e]);
      }
    }
  }
  uint32_t least = ~0u;                                       // twice the bits of the smallest |U*| but 0, less 1
#pragma unroll
  for (int k = 0; k < kChunks; ++k) {
    if (128 * k + 4 * ci < r) {
      if constexpr (kParts) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ua[k][e] = ldexpf(ua[k][e], -le);
        uint32_t v[2][3];
#pragma unroll
        for (int e = 0; e < 2; ++e) split3(ua[k][2 * e], ua[k][2 * e + 1], v[e]);
#pragma unroll
        for (int q = 0; q < 3; ++q) *(u32x2_t*)(parts + (q * 16 + c) * pitch + 128 * k + 4 * ci) = u32x2_t{v[0][q], v[1][q]};
#pragma unroll
        for (int e = 0; e < 4; ++e) least = min(least, (__builtin_bit_cast(uint32_t, ua[k][e]) << 1) - 1u);
      } else {
        *(f32x4_t*)(ustar + c * pitch32 + 128 * k + 4 * ci) = ua[k];
      }
    }
  }
  int whole = 0;                                              // bfloat16: U* is in LDS as fp32 after all
  if constexpr (kParts) {
    const bool any = __any(least < (__builtin_bit_cast(uint32_t, 0x1p-100f) << 1) - 1u);
    if (lane == 0) flags[w] = any;
    lds_barrier();
#pragma unroll
    for (int k = 0; k < 8; ++k) whole |= flags[k];
    if (whole) {
#pragma unroll
      for (int k = 0; k < kChunks; ++k)
        if (128 * k + 4 * ci < r) *(f32x4_t*)(ustar + c * pitch32 + 128 * k + 4 * ci) = ua[k];
    }
  }
  if (!kParts || whole) lds_barrier();
  // ---- expansion
  f32x4_t acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto use_group_f32 = [&](const uint32_t (&src)[8][DW], int gi) {
    float uf[8];                                              // of rows 8 g + t
    if (kParts && !whole) {
#pragma unroll
      for (int t = 0; t < 8; ++t) uf[t] = 0.f;
#pragma unroll
      for (int q = 2; q >= 0; --q) {
        const u32x4_t v = *(const u32x4_t*)(parts + (q * 16 + n) * pitch + gi * 32 + 8 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uf[2 * e] += lo_to_f32(v[e], Tag{});
          uf[2 * e + 1] += hi_to_f32(v[e], Tag{});
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < 8; t += 4) {
        const f32x4_t v = *(const f32x4_t*)(ustar + n * pitch32 + gi * 32 + 8 * g + t);
#pragma unroll
        for (int e = 0; e < 4; ++e) uf[t + e] = v[e];
      }
    }
    constexpr int kC = VEC < 16 ? 2 : 1;                      // sums of a few rows each, added up in pairs: fewer roundings
    f32x4_t part[kC][VEC];                                    // on the way
#pragma unroll
    for (int t = 0; t < 8; ++t)                               // rows 8 g' + t, g' = 0 .. 3
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        const float x = i & 1 ? hi_to_f32(src[t][i >> 1], Tag{}) : lo_to_f32(src[t][i >> 1], Tag{});
        const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
        part[t % kC][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, uf[t], t < kC ? zero : part[t % kC][i], 0, 0, 0);
      }
#pragma unroll
    for (int k = kC / 2; k > 0; k >>= 1)
#pragma unroll
      for (int j = 0; j < k; ++j)
#pragma unroll
        for (int i = 0; i < VEC; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) part[j][i][e] += part[j + k][i][e];
#pragma unroll
    for (int i = 0; i < VEC; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][e] += part[0][i][e];
  };
  auto use_group = [&](const uint32_t (&src)[8][DW], int gi) {
    if constexpr (kParts) {
      constexpr int kWide = VEC < 4 ? VEC : 4;                // products in flight side by side
      u32x4_t uq[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) uq[q] = *(const u32x4_t*)(parts + (q * 16 + n) * pitch + gi * 32 + 8 * g);
#pragma unroll
      for (int i0 = 0; i0 < VEC; i0 += kWide) {
        u32x4_t a[kWide];
#pragma unroll
        for (int i = 0; i < kWide; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            a[i][e] = __builtin_amdgcn_perm(src[2 * e + 1][(i0 + i) >> 1], src[2 * e][(i0 + i) >> 1], (i & 1) ? 0x07060302 : 0x05040100);
#pragma unroll
        for (int q = 2; q >= 0; --q)
#pragma unroll
          for (int i = 0; i < kWide; ++i) acc[i0 + i] = Mfma<Tag>::run(a[i], uq[q], acc[i0 + i]);
      }
    } else {
      use_group_f32(src, gi);
    }
  };
  for (int gi = whole ? groups : w; gi < groups; gi += 8 * kAhead) {
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (gi + 8 * k < groups) use_group(bv[k], gi + 8 * k);
      if (gi + 8 * (k + kAhead) < groups) load_group(bv[k], gi + 8 * (k + kAhead));
    }
  }
  if constexpr (kParts) {
    float nothing = 0.f;                                      // NaN once something is not finite
#pragma unroll
    for (int i = 0; i < VEC; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) nothing = fmaf(acc[i][e], 0.f, nothing);
    if (whole || __any(nothing != 0.f)) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      for (int gi = w; gi < groups; gi += 8) {
        load_group(bv[0], gi);
        use_group_f32(bv[0], gi);
      }
    }
  }
  // ---- the waves' sums in a fixed order: 4..7 onto 0..3, then those four
  constexpr int dp = d + 4;
  float* mine = sums + (w & 3) * 16 * dp + n * dp;
  lds_barrier();
  if (w >= 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < VEC; ++i) mine[(4 * g + e) * VEC + i] = acc[i][e];
  }
  lds_barrier();
  if (w < 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < VEC; ++i) mine[(4 * g + e) * VEC + i] += acc[i][e];
  }
  lds_barrier();
  if (ct * 16 + c >= N) return;
  for (int e4 = ci; e4 < d / 4; e4 += 32) {
    f32x4_t s = *(const f32x4_t*)(sums + c * dp + 4 * e4);
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      const f32x4_t t = *(const f32x4_t*)(sums + (k * 16 + c) * dp + 4 * e4);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += t[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] /= ldexpf(L, -le);
    const size_t o = ((size_t)b * H + h) * d + 4 * e4;
    if (OUT_F32) *(f32x4_t*)((float*)p.out + o) = s;
    else *(u32x2_t*)((uint16_t*)p.out + o) = u32x2_t{pack2(s[0], s[1], Tag{}), pack2(s[2], s[3], Tag{})};
  }
}

template <class Tag, int NB, int KS>
void launch_project(const ProjectParams& p, int blocks, hipStream_t stream) {
  const size_t dot = (size_t)2 * (16 + 16 * NB) * 264 * 2, fold = (size_t)192 * (KS * 32 + 8) * 2;
  const size_t lds = p.dot_units && dot > fold ? dot : fold;
  hipLaunchKernelGGL((shared_project<Tag, KS, NB>), dim3(blocks), dim3(512), lds, stream, p);
}
template <class Tag, int NB>
void launch_project(const ProjectParams& p, int d, int blocks, hipStream_t stream) {
  switch (d) {
    case 32: launch_project<Tag, NB, 1>(p, blocks, stream); break;
    case 64: launch_project<Tag, NB, 2>(p, blocks, stream); break;
    case 128: launch_project<Tag, NB, 4>(p, blocks, stream); break;
    default: launch_project<Tag, NB, 8>(p, blocks, stream); break;
  }
}
template <class Tag, bool OUT_F32>
void launch_expand(const SharedExpandParams& p, int d, hipStream_t stream) {
  const dim3 grid((p.units + 7) / 8 * 8);
  const size_t u = __is_same(Tag, BF16Tag) ? (size_t)3 * 16 * (p.r + 8) / 2 : (size_t)16 * (p.r + 4);
  const size_t merge = (u + 16 * (p.S + 1) + 8) * 4, sums = (size_t)4 * 16 * (d + 4) * 4;
  const size_t lds = merge > sums ? merge : sums;
  switch (d) {
    case 32: hipLaunchKernelGGL((shared_expand<Tag, OUT_F32, 2>), grid, dim3(512), lds, stream, p); break;
    case 64: hipLaunchKernelGGL((shared_expand<Tag, OUT_F32, 4>), grid, dim3(512), lds, stream, p); break;
    case 128: hipLaunchKernelGGL((shared_expand<Tag, OUT_F32, 8>), grid, dim3(512), lds, stream, p); break;
    default:                                                  // (fp16 does not come here: shared_expand_applies)
      if constexpr (__is_same(Tag, BF16Tag))
        hipLaunchKernelGGL((shared_expand<Tag, OUT_F32, 16>), grid, dim3(512), lds, stream, p);
      break;
  }
}

}  // namespace

// Where the matrix products take over from the passes per sequence, whose time is B r HD bytes out of the L2s.
// The fold alone: everywhere but with short rows and little of it (us a call there / here: 8 x 256 rows of 5120
// 18.2 / 17.2, 64 x 640 of 4096 59.9 / 44.5, 2 x 256 of 2048 11.1 / 11.3).  With the appended rows, whose products
// walk the hidden axis in few workgroups: from about 1.25 HD rows on, and not at small ranks (64 sequences,
// rank 64, 40 heads of 128 20.5 / 24.2; 16 x 256 of 4096 20.1 / 18.8; 12 x 256 of 8192 25.2 / 27.2;
// 64 x 640 of 5120 124 / 70).
bool shared_project_applies(int B, int H, int H_kv, int d, int r, bool appends) {
  const int64_t HD = (int64_t)H_kv * d, rows = (int64_t)B * r;
  if (B < 2) return false;
  if (!appends) return HD >= 2560 || H > H_kv || rows >= 16384;
  return r >= 192 && rows >= 5120 && 4 * rows >= 5 * HD;
}
// The expansion's merge is longer than that of a workgroup per head (all columns' sums pass through B H / 16
// workgroups, four splits at a time): few splits and much to expand.  Us a call there / here: 64 x 256, 64 heads
// 34.4 / 28.7, 64 x 640, 64 heads of 64 60.5 / 53.5, but 48 x 256, 40 heads 27.2 / 28.0.  The fp32 products of fp16
// are worth it with one round of splits and heads up to 128: 64 x 256, 64 heads 32.9 / 30.1, 64 x 448, 32 heads
// 33.0 / 31.8, but with six and eight splits 40 x 640, 32 heads 32.1 / 35.7 and 32 x 640, 40 heads 35.6 / 38.9, with
// heads of 256 48 x 320, 32 heads 28.1 / 33.9.
bool shared_expand_applies(ap_dtype dt, int B, int H, int d, int r, int S) {
  if (dt == AP_F16 && (S > 4 || d > 128)) return false;
  return S <= 8 && (int64_t)B * r * H * d * 2 >= (192ll << 20);
}

// Fold of q (and, with k_new and v_new, both appended rows) on shared bases, r % 64 == 0.
ap_status launch_shared_project(ap_dtype dt, const void* Bk, const void* Bv, const void* k_new, const void* v_new,
                                const void* q, void* Ck, void* Cv, void* Qp, int B, int H, int H_kv, int Hp, int d,
                                int r, int row, int T_cap, float scale, hipStream_t stream) {
  ProjectParams p{{(const uint16_t*)Bk, (const uint16_t*)Bv}, {(const uint16_t*)k_new, (const uint16_t*)v_new},
                  {(uint16_t*)Ck, (uint16_t*)Cv}, (const uint16_t*)q, (uint16_t*)Qp, B, H, H / H_kv, Hp, H_kv * d, r,
                  row, T_cap, 0, 0, 0, scale};
  const int nb = B > 16 ? 2 : 1;
  p.dot_units = k_new ? r / 16 * 2 * ((B + 16 * nb - 1) / (16 * nb)) : 0;
  p.fold_units = H_kv * ((r + 127) / 128) * ((B * p.G + 63) / 64);
  p.dot_blocks = (p.dot_units + 7) / 8 * 8;
  const int blocks = p.dot_blocks + (p.fold_units + 7) / 8 * 8;
  if (dt == AP_F16) nb == 2 ? launch_project<F16Tag, 2>(p, d, blocks, stream) : launch_project<F16Tag, 1>(p, d, blocks, stream);
  else nb == 2 ? launch_project<BF16Tag, 2>(p, d, blocks, stream) : launch_project<BF16Tag, 1>(p, d, blocks, stream);
  return AP_OK;
}

ap_status launch_shared_expand(ap_dtype dt, bool out_f32, const float* part_ml, const float* part_U, const void* Bv,
                               void* out, float* lse, int B, int H, int H_kv, int d, int r, int nsplit, hipStream_t stream) {
  const int G = H / H_kv;
  const SharedExpandParams p{part_ml, part_U, (const uint16_t*)Bv, out, lse, B, H, G, H_kv * d, r, nsplit,
                             H_kv * ((B * G + 15) / 16)};
  if (dt == AP_F16) out_f32 ? launch_expand<F16Tag, true>(p, d, stream) : launch_expand<F16Tag, false>(p, d, stream);
  else out_f32 ? launch_expand<BF16Tag, true>(p, d, stream) : launch_expand<BF16Tag, false>(p, d, stream);
  return AP_OK;
}

}  // namespace ap
