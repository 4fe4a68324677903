// attn_heads: the whole of a short context's attention for one head in one workgroup, from the folded query to
// the output (paper Alg. 1: scores, softmax, weighted sum, expansion), for 16-bit coefficients at uniform rank.
//
// A short pass is bound by its chain of dependent launches (3 to 4 us each, however little they do) and, inside
// one, by the chain of memory round trips.  Here nothing has to be merged, so one launch takes the place of two
// (attention over token splits, merge and expansion), and of three where the query is folded here as well
// (calls that append nothing: FOLD); everything a workgroup reads is asked for at its start.  The price is that
// every head of a sequence reads all of its coefficient rows, out of L2: attn_heads_applies says up to where.
// One query per head has no use for the matrix cores: 32 heads x 321 tokens x 64 columns are 0.7 M products.
//
//   (FOLD) q'[j] = scale Bk[j, head] . q      d / 8 lanes per basis row; 16-bit high and low parts, as the
//                                             other paths have them
//   scores s[t] = C_k[t] . q'                 eight lanes per token row, a row's 16-byte chunks l, l + 8, ..
//   sums   U[j] = sum_t 2^(s[t] - m) C_v[t,j] the same lanes per row, added over the rows' lanes, then the waves
//   out    = (U / l) . Bv[:, head]            a wave per block of basis rows, two columns per lane
#include "ap_common.hpp"
#include "lane_ops.hpp"
#include <hip/hip_ext.h>
#include <type_traits>

namespace ap {
namespace {

constexpr int kThreads = 1024, kWaves = kThreads / 64, kRows = kThreads / 8;   // token rows per round

struct HeadsParams {
  const uint16_t* q;      // FOLD: [B][H][d]
  const uint16_t* Bk;     // FOLD: [B or 1][r][HD]
  const uint16_t* Qp;     // else: folded queries, high and low parts
  FoldedLayout folded;
  const uint16_t* Ck;     // [B][T_cap][r]
  const uint16_t* Cv;
  const uint16_t* Bv;     // [B or 1][r][HD]
  int64_t bstride;
  void* out;              // [B][H][d]
  float* lse;             // [B][H] or null
  float* scores;          // [B][T_cap][H] scaled logits in natural-log units, or null
  int B, H, G, Hp, HD, T, T_cap, out_f32;
  float scale;
};

// NC = r / 64 chunks of a row per lane, D the head's width.  grid (B H), 1024 threads; dynamic LDS: scores, T rounded up to kRows.
template <class Tag, int NC, int D, bool FOLD>
__global__ void __launch_bounds__(kThreads) attn_heads(const HeadsParams p) {
  constexpr int r = NC * 64;
  constexpr int RB = NC == 1 ? 4 : NC == 2 ? 2 : 1;      // rounds on their way at once
  constexpr int CPD = D / 8, FROWS = kThreads / CPD;     // lanes per basis row of the fold, rows a round
  constexpr int NF = (r + FROWS - 1) / FROWS;
  constexpr int HALF = D / 2, STEPS = NC * D / 32;       // the expansion: 64 lanes x 2 columns a step
  extern __shared__ __attribute__((aligned(16))) float s_lds[];
  __shared__ float red[kWaves * (r > D ? r : D)];        // sums per wave: [wave][r], then [wave][D]
  __shared__ __attribute__((aligned(16))) uint16_t qp[2][r];
  __shared__ float ustar[r], mred[kWaves], lred[kWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = p.H, T = p.T, HD = p.HD;
  // a sequence's heads read the same rows: on one XCD where whole eights of sequences allow it
  const int id = __builtin_amdgcn_readfirstlane((int)blockIdx.x);
  int b, h;
  if (p.B % 8 == 0) { b = (id >> 3) / H * 8 + (id & 7); h = (id >> 3) % H; }
  else { b = id / H; h = id - b * H; }
  const size_t slice = (size_t)b * p.bstride + (size_t)(h / p.G) * D;

  // ---- requests, in the order in which they are needed
  const int fr = tid / CPD, fc = tid % CPD;
  u32x4_t qv, bk[NF];
  if constexpr (FOLD) {
    qv = *(const u32x4_t*)(p.q + ((size_t)b * H + h) * D + fc * 8);
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int j = fr + k * FROWS;
      bk[k] = *(const u32x4_t*)(p.Bk + slice + (size_t)(j < r ? j : r - 1) * HD + fc * 8);
    }
  }
  const int l8 = tid & 7, rr = tid >> 3;
  u32x4_t qh[NC], ql[NC];
  if constexpr (!FOLD) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const uint16_t* src = p.Qp + ((size_t)b * 2) * p.Hp * r + p.folded.at(h, (l8 + 8 * c) * 8, r);
      qh[c] = *(const u32x4_t*)src;
      ql[c] = *(const u32x4_t*)(src + (size_t)p.Hp * r);
    }
  }
  const size_t seq = (size_t)b * p.T_cap * r;
  const auto kbuf = make_buffer(p.Ck + seq, (uint32_t)T * (r * 2));   // rows past the last one are zeros
  const auto vbuf = make_buffer(p.Cv + seq, (uint32_t)T * (r * 2));
  auto load_rows = [&](const buffer_t& buf, u32x4_t (&dst)[RB][NC], int t0) {
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        dst[u][c] = buffer_load16(buf, (uint32_t)(t0 + u * kRows + rr) * (r * 2) + (l8 + 8 * c) * 16);
  };
  u32x4_t kr[RB][NC], vr[RB][NC];
  load_rows(kbuf, kr, 0);
  load_rows(vbuf, vr, 0);
  // the expansion's rows: wave w rows w r / 16 .. of its head's slice, two columns per lane
  const uint16_t* Bv = p.Bv + slice + (size_t)w * (r / kWaves) * HD;
  uint32_t bv[STEPS];
#pragma unroll
  for (int k = 0; k < STEPS; ++k) {
    const int at = k * 64 + lane;                        // pair of columns in the wave's block of rows
    bv[k] = *(const uint32_t*)(Bv + (size_t)(at / HALF) * HD + at % HALF * 2);
  }

  if constexpr (FOLD) {
    // ---- the folded query
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int j = fr + k * FROWS;
      const float x = group_sum<CPD>(dot8<Tag>(bk[k], qv, 0.f)) * p.scale;
      const uint16_t hi = f32_to_bits(x, Tag{});
      if (fc == 0 && j < r) {
        qp[0][j] = hi;
        qp[1][j] = f32_to_bits(x - bits_to_f32(hi, Tag{}), Tag{});
      }
    }
    lds_barrier();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      qh[c] = *(const u32x4_t*)&qp[0][(l8 + 8 * c) * 8];
      ql[c] = *(const u32x4_t*)&qp[1][(l8 + 8 * c) * 8];
    }
  }

  // ---- scores and their maximum
  float m = -INFINITY;
  for (int t0 = 0; t0 < T; t0 += RB * kRows) {
    if (t0 > 0) load_rows(kbuf, kr, t0);
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int t = t0 + u * kRows + rr;
      float a = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) a = dot8<Tag>(kr[u][c], ql[c], a);
#pragma unroll
      for (int c = 0; c < NC; ++c) a = dot8<Tag>(kr[u][c], qh[c], a);
      a = group_sum<8>(a);
      a = t < T ? a : -INFINITY;
      m = fmaxf(m, a);
      if (l8 == 0 && t0 + u * kRows < T) s_lds[t] = a;
    }
  }
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
  if (lane == 0) mred[w] = m;
  lds_barrier();
  m = mred[0];
#pragma unroll
  for (int k = 1; k < kWaves; ++k) m = fmaxf(m, mred[k]);

  if (p.scores)
    for (int t = tid; t < T; t += kThreads) p.scores[((size_t)b * p.T_cap + t) * H + h] = s_lds[t] * kLn2;
  // ---- weights and the weighted sum of the value rows
  float acc[NC][8], l = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[c][e] = 0.f;
  for (int t0 = 0; t0 < T; t0 += RB * kRows) {
    if (t0 > 0) load_rows(vbuf, vr, t0);
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int t = t0 + u * kRows + rr;
      const float x = s_lds[t < T ? t : T - 1];
      const float pw = t < T ? fast_exp2(x - m) : 0.f;
      l += pw;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[c][2 * e] = fmaf(pw, lo_to_f32(vr[u][c][e], Tag{}), acc[c][2 * e]);
          acc[c][2 * e + 1] = fmaf(pw, hi_to_f32(vr[u][c][e], Tag{}), acc[c][2 * e + 1]);
        }
    }
  }
  // over the wave's eight rows: each exchange halves the columns that a lane still carries
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float v4[4], v2[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float keep = lane & 32 ? acc[c][4 + e] : acc[c][e], give = lane & 32 ? acc[c][e] : acc[c][4 + e];
      v4[e] = keep + __shfl_xor(give, 32);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float keep = lane & 16 ? v4[2 + e] : v4[e], give = lane & 16 ? v4[e] : v4[2 + e];
      v2[e] = keep + __shfl_xor(give, 16);
    }
    const float keep = lane & 8 ? v2[1] : v2[0], give = lane & 8 ? v2[0] : v2[1];
    const int col = (l8 + 8 * c) * 8 + (lane >> 5 & 1) * 4 + (lane >> 4 & 1) * 2 + (lane >> 3 & 1);
    red[w * r + col] = keep + __shfl_xor(give, 8);
  }
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) l += __shfl_xor(l, o);
  if (lane == 0) lred[w] = l;
  lds_barrier();
  float L = lred[0];
#pragma unroll
  for (int k = 1; k < kWaves; ++k) L += lred[k];
  if (tid < r) {
    float a = red[tid];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) a += red[k * r + tid];
    ustar[tid] = a / L;
  }
  if (p.lse && tid == 0) p.lse[(size_t)b * H + h] = (m + log2f(L)) * kLn2;
  lds_barrier();

  // ---- expansion
  float o0 = 0.f, o1 = 0.f;
#pragma unroll
  for (int k = 0; k < STEPS; ++k) {
    const float u = ustar[w * (r / kWaves) + (k * 64 + lane) / HALF];
    o0 = fmaf(u, lo_to_f32(bv[k], Tag{}), o0);
    o1 = fmaf(u, hi_to_f32(bv[k], Tag{}), o1);
  }
#pragma unroll
  for (int x = HALF; x < 64; x <<= 1) { o0 += __shfl_xor(o0, x); o1 += __shfl_xor(o1, x); }
  if (lane < HALF) { red[w * D + 2 * lane] = o0; red[w * D + 2 * lane + 1] = o1; }
  lds_barrier();
  if (tid < D) {
    float a = red[tid];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) a += red[k * D + tid];
    const size_t at = ((size_t)b * H + h) * D + tid;
    if (p.out_f32) ((float*)p.out)[at] = a;
    else ((uint16_t*)p.out)[at] = f32_to_bits(a, Tag{});
  }
}

}  // namespace

// Where a head per workgroup is the shorter way: its rows come out of L2 at some 120 GB/s per CU, T r 4 bytes for
// every 256 workgroups, against the launches that it saves, two without an append, else one.  Us a pass over token
// splits / here, 32 heads of 128 in bf16: one sequence of 321 tokens, rank 64 step 14.8 / 10.0, attention alone 14.2 / 5.5; 8 of
// 700, rank 128 16.5 / 15.5, 16.1 / 10.3; 8 of 321, rank 256 19.5 / 18.6, 17.1 / 12.3; of 800 21.2 / 23.4 (left there),
// 18.5 / 16.5; 16 of 300, rank 128 17.9 / 21.0 (left there), 16.9 / 14.7.
bool attn_heads_applies(int B, int H, int d, int T, int r, bool appends) {
  if (r % 64 != 0 || r > 256 || (d != 64 && d != 128)) return false;
  const int64_t rounds = ((int64_t)B * H + 255) / 256, work = (int64_t)T * r * rounds;
  if (rounds > 2 || (rounds == 2 && r > 64 && appends)) return false;
  int64_t most = appends ? (r <= 128 ? 88 << 10 : 96 << 10) : r == 64 ? 256 << 10 : r == 128 ? 208 << 10 : 192 << 10;
  if (rounds == 2 && r > 64) most = most * 3 / 4;
  // a head tile of their own costs the other kernels less: 15 of 1930, 16 heads of 64, rank 64 12.1 / 16.3 a step
  if (H <= 16) most /= 2 * rounds;
  return work <= most;
}

ap_status launch_attn_heads(const DecodeArgs& a, const uint16_t* Qp, FoldedLayout folded, float scale) {
  const int Hp = (a.H + 15) / 16 * 16;
  const HeadsParams p{(const uint16_t*)a.q, (const uint16_t*)a.Bk, Qp, folded, (const uint16_t*)a.Ck, (const uint16_t*)a.Cv,
                      (const uint16_t*)a.Bv, a.basis_batch_stride, a.out, a.lse, a.scores, a.B, a.H, a.H / a.H_kv, Hp,
                      a.H_kv * a.d, a.T, a.T_cap, a.dt_out == AP_F32, scale};
  const size_t lds = (size_t)(a.T + kRows - 1) / kRows * kRows * 4;
  hipEvent_t ev0, ev1;
  const bool timed = prof_events(&ev0, &ev1);          // the coefficient-streaming kernel of this call
  auto go = [&](auto tag, auto nc, auto d, auto fold) {
    auto kern = attn_heads<decltype(tag), decltype(nc)::value, decltype(d)::value, decltype(fold)::value>;
    if (timed) hipExtLaunchKernelGGL(kern, dim3(a.B * a.H), dim3(kThreads), (uint32_t)lds, a.stream, ev0, ev1, 0u, p);
    else hipLaunchKernelGGL(kern, dim3(a.B * a.H), dim3(kThreads), lds, a.stream, p);
  };
  auto by_fold = [&](auto tag, auto nc, auto d) {
    if (Qp) go(tag, nc, d, std::false_type{}); else go(tag, nc, d, std::true_type{});
  };
  auto by_width = [&](auto tag, auto nc) {
    if (a.d == 64) by_fold(tag, nc, std::integral_constant<int, 64>{});
    else by_fold(tag, nc, std::integral_constant<int, 128>{});
  };
  auto by_rank = [&](auto tag) {
    switch (a.r / 64) {
      case 1: by_width(tag, std::integral_constant<int, 1>{}); break;
      case 2: by_width(tag, std::integral_constant<int, 2>{}); break;
      case 3: by_width(tag, std::integral_constant<int, 3>{}); break;
      default: by_width(tag, std::integral_constant<int, 4>{}); break;
    }
  };
  if (a.dt == AP_F16) by_rank(F16Tag{}); else by_rank(BF16Tag{});
  return check_launch(a.k_new ? "ap_decode_step" : "ap_decode_attn");
}

}  // namespace ap
