// Per-step passes over the decompression matrices (bases) in 16-bit storage: bandwidth-bound
// matrix-vector products that read every basis byte exactly once, whole rows at a time.
//
//   basis_rows<DOT, FOLD>   one pass over Bm [r, HD] of every sequence, each wave streaming
//                           whole rows (HD contiguous elements, 128-bit loads, several rows
//                           in flight) and producing, per row j,
//       DOT :  c[j]     = Bm[j, :] . x                 the appended token's coefficient
//                                                      (paper Sec. 3.1 projection, one row)
//       FOLD:  q'[h, j] = scale * Bm[j, head h] . q_h  the query folded through the key basis
//                                                      (Alg. 1 scores by associativity)
//                           With both, the append of a key row and the fold of the query
//                           share one pass over B_k.
//   merge_expand            combine the token splits of attn_partial and expand through B_v:
//                           out[h, :] = (sum_s w_s U_s[h, :] / sum_s w_s l_s) . Bv[:, head h]
//                           (Alg. 1 output by associativity).  A workgroup owns one head, or a
//                           slice of its columns, and keeps eight rows in flight per thread.
// Products of two 16-bit values are exact in fp32; sums are fp32 (v_dot2c_f32_*).
#include "ap_common.hpp"
#include "lane_ops.hpp"
#include "mfma_ops.hpp"
#include <algorithm>

namespace ap {
namespace {

struct RowsParams {
  const uint16_t* Bm;     // [B][r][HD] (bstride elements between sequences, 0 = shared)
  int64_t bstride;
  const uint16_t* x;      // DOT:  [B][HD] the token row to project
  const uint16_t* q;      // FOLD: [B][H][d] (= [B][HD])
  uint16_t* C;            // DOT:  [B][T_cap][r], row `row0` written
  uint16_t* Qp;           // FOLD: folded queries (FoldedLayout, tiled), hi / lo parts
  int H, Hp, d, HD, r, row0, T_cap;
  int rpw;                // consecutive rows per wave (a workgroup owns 4 * rpw rows)
  float scale;
  FastDiv by_heads;       // FOLD: Hp
  // PAIR: a second DOT job of the same shape in the same launch (blockIdx.z = 1), e.g. the
  // value row of a step appended next to the key row
  const uint16_t* Bm2;
  const uint16_t* x2;
  uint16_t* C2;
};

template <class Tag>
__device__ __forceinline__ void split_hi_lo(float x, uint16_t& hi, uint16_t& lo) {
  hi = f32_to_bits(x, Tag{});
  lo = f32_to_bits(x - bits_to_f32(hi, Tag{}), Tag{});
}

// grid (ceil(r / (4 rpw)), B), 256 threads.  KPC = 512-element passes that cover the hidden
// axis; a wave walks its rows through a ring of NBUF row buffers in registers, so NBUF - 1
// rows (HD * 2 bytes each) are in flight while one is reduced.
// LPH = d / 8 lanes share a head (FOLD; 1 when the kernel does not fold).
// PAIR: grid.z = 2; the workgroups of z = 1 run the second job (DOT only) on Bm2, x2, C2.
// G: query heads that read the same slice of a row (grouped queries; each has its own dot products).
template <class Tag, int KPC, int NBUF, bool DOT, bool FOLD, int LPH, bool PAIR = false, int G = 1>
__global__ void __launch_bounds__(256) basis_rows(const RowsParams p) {
  extern __shared__ __attribute__((aligned(16))) float qtile[];   // FOLD: [Hp][4 rpw + 1]
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rpw = p.rpw, rows_wg = 4 * rpw, pitch = rows_wg + 1;
  const int b = blockIdx.y, j0 = blockIdx.x * rows_wg;
  const int HD = p.HD, r = p.r;
  const bool second = PAIR && blockIdx.z == 1;
  const bool fold = FOLD && !second;
  const uint16_t* Bb = (second ? p.Bm2 : p.Bm) + (size_t)b * p.bstride;
  const uint16_t* xv = second ? p.x2 : p.x;
  uint16_t* Cb = second ? p.C2 : p.C;
  u32x4_t buf[NBUF][KPC];
  // passes beyond the hidden axis re-read the lane's first chunk (their vector slices are
  // zero), so the loads carry no branches and issue back to back
  int eoff[KPC];
#pragma unroll
  for (int pp = 0; pp < KPC; ++pp)
    eoff[pp] = (pp * 512 + lane * 8) < HD ? pp * 512 + lane * 8 : (lane * 8 < HD ? lane * 8 : 0);
  auto load_row = [&](u32x4_t (&dst)[KPC], int i) {         // row i of this wave
    int j = j0 + w * rpw + i;
    j = j < r ? j : r - 1;                                  // rows past the end: harmless repeats
    const uint16_t* row = Bb + (size_t)j * HD;
#pragma unroll
    for (int pp = 0; pp < KPC; ++pp) {
      // wide rows (read once per launch) are streamed with the non-temporal hint, which pays only
      // with a shallow ring: at HD = 5120 one row in flight per wave and the hint 77 us, two rows
      // in flight 80 us without and 87 us with it
      if constexpr (KPC == 10) dst[pp] = __builtin_nontemporal_load((const u32x4_t*)(row + eoff[pp]));
      else dst[pp] = *(const u32x4_t*)(row + eoff[pp]);
    }
  };
  // this lane's slices of the vectors: elements 512 pp + 8 lane .. +7 of the hidden axis.
  constexpr int dshift = FOLD ? 31 - __builtin_clz((unsigned)(LPH * 8)) : 0;   // log2(d)
  // They are requested BEFORE the first rows, so that a row's arrival implies theirs and no
  // wait on them ever drains the row ring.
  u32x4_t xs[DOT ? KPC : 1], qs[FOLD ? KPC : 1][G];
#pragma unroll
  for (int pp = 0; pp < KPC; ++pp) {
    const int e0 = pp * 512 + lane * 8;
    const u32x4_t z = {0, 0, 0, 0};
    if (DOT) xs[pp] = e0 < HD ? *(const u32x4_t*)(xv + (size_t)b * HD + e0) : z;
    if constexpr (FOLD && G == 1) {
      qs[pp][0] = e0 < HD && fold ? *(const u32x4_t*)(p.q + (size_t)b * HD + e0) : z;
    } else if constexpr (FOLD) {
#pragma unroll
      for (int k = 0; k < G; ++k)
        qs[pp][k] = e0 < HD && fold ? *(const u32x4_t*)(p.q + (size_t)b * G * HD + ((e0 >> dshift) * G + k) * (LPH * 8) + (e0 & (LPH * 8 - 1))) : z;
    }
  }
  const int last = rpw - 1;
#pragma unroll
  for (int u = 0; u + 1 < NBUF; ++u) load_row(buf[u], u < last ? u : last);
  if (fold) {
    for (int i = tid; i < p.Hp * pitch; i += 256) qtile[i] = 0.f;   // padded heads stay 0
    __syncthreads();
  }
  auto reduce_row = [&](const u32x4_t (&row)[KPC], int i) {
    const int jl = w * rpw + i;
    const bool live = i < rpw && j0 + jl < r;
    if (DOT) {
      float acc = 0.f;
#pragma unroll
      for (int pp = 0; pp < KPC; ++pp) acc = dot8<Tag>(row[pp], xs[pp], acc);
      acc = wave_sum(acc);
      if (lane == 0 && live)
        Cb[((size_t)b * p.T_cap + p.row0) * r + j0 + jl] = f32_to_bits(acc, Tag{});
    }
    if (fold) {
#pragma unroll
      for (int pp = 0; pp < KPC; ++pp) {
        const int e0 = pp * 512 + lane * 8;
#pragma unroll
        for (int k = 0; k < G; ++k) {
          float part = dot8<Tag>(row[pp], qs[pp][k], 0.f);
          part = group_sum<LPH>(part);
          if ((lane & (LPH - 1)) == 0 && e0 < HD && live)
            qtile[((e0 >> dshift) * G + k) * pitch + jl] = part * p.scale;
        }
      }
    }
  };
  // The ring advances without branches: every slot of the unrolled body requests a row and
  // reduces one (past the wave's last row the request repeats that row, a cache hit, and the
  // reduction's result is dropped), so the compiler's wait counts stay exact.
  const int rpw_pad = (rpw + NBUF - 1) / NBUF * NBUF;
  for (int i = 0; i < rpw_pad; i += NBUF) {
#pragma unroll
    for (int u = 0; u < NBUF; ++u) {
      const int nx = i + u + NBUF - 1;
      load_row(buf[(u + NBUF - 1) % NBUF], nx < last ? nx : last);
      reduce_row(buf[u], i + u);
    }
  }
  if (fold) {
    __syncthreads();
    // four rank positions of a head per thread (r and rows_wg are multiples of four), neighbouring heads next to
    // each other (a head's row of 2-byte stores per part instead: 21 sequences, 32 / 8 heads, rank 256 8.5 us against
    // 7.8, 32 of 40 heads, rank 192 15.2 against 14.4)
    uint16_t* Qb = p.Qp + (size_t)b * 2 * p.Hp * r;
    constexpr FoldedLayout tiles{true};
    for (int i = tid; i < p.Hp * rpw; i += 256) {
      const int jq = p.by_heads(i), h = i - jq * p.Hp, jl = 4 * jq;
      if (j0 + jl < r) {
        uint16_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) split_hi_lo<Tag>(qtile[h * pitch + jl + e], hi[e], lo[e]);
        uint16_t* dst = Qb + tiles.at(h, j0 + jl, r);
        *(u32x2_t*)dst = u32x2_t{hi[0] | (uint32_t)hi[1] << 16, hi[2] | (uint32_t)hi[3] << 16};
        *(u32x2_t*)(dst + (size_t)p.Hp * r) = u32x2_t{lo[0] | (uint32_t)lo[1] << 16, lo[2] | (uint32_t)lo[3] << 16};
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// fold_heads: the fold for grouped queries, q'[h, j] = scale * Bk[j, slice of key/value head
// h / G] . q_h.  A workgroup owns one key/value head and 64 basis rows; groups of LPH = d / 8
// lanes take one row each (four rows in flight per group) and dot it with the queries of all
// G heads that share the slice, so every basis byte is loaded once.
//   grid (H_kv * ceil(G / 8), ceil(r / 64), B), 256 threads; the workgroups of key/value
//   head 0 also write the padding heads H .. Hp-1 as zeros.
// ------------------------------------------------------------------------------------------
template <class Tag, int LPH>
__global__ void __launch_bounds__(256)
fold_heads(const uint16_t* __restrict__ Bk, int64_t bstride, const uint16_t* __restrict__ q,
           uint16_t* __restrict__ Qp, int H, int G, int Hp, int r, float scale) {
  constexpr int d = LPH * 8;
  constexpr int NG = 256 / LPH;                 // rows per pass of the workgroup
  const int nsub = (G + 7) >> 3;                // query heads are taken eight at a time
  const int kvh = blockIdx.x / nsub, sub = blockIdx.x - kvh * nsub;
  const int b = blockIdx.z, tid = threadIdx.x;
  const int jb = blockIdx.y * 64;
  int jend = jb + 64;
  jend = jend < r ? jend : r;
  if (blockIdx.x == 0) {
    for (int i = tid; i < (Hp - H) * (jend - jb); i += 256) {
      const int h = H + i / (jend - jb), j = jb + i % (jend - jb);
      Qp[(((size_t)b * 2 + 0) * Hp + h) * r + j] = 0;
      Qp[(((size_t)b * 2 + 1) * Hp + h) * r + j] = 0;
    }
  }
  const int g = tid / LPH, li = tid % LPH;
  const size_t HD = (size_t)(H / G) * d;
  const int h0 = kvh * G + sub * 8;             // first query head of this workgroup
  int nq = G - sub * 8;
  nq = nq < 8 ? nq : 8;
  u32x4_t qv[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int hk = k < nq ? h0 + k : h0;        // unused slots repeat the first head
    qv[k] = *(const u32x4_t*)(q + ((size_t)b * H + hk) * d + li * 8);
  }
  const uint16_t* col = Bk + (size_t)b * bstride + (size_t)kvh * d + li * 8;
  for (int j0 = jb; j0 < jend; j0 += NG * 4) {
    u32x4_t rowv[4];
    int j[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      j[u] = j0 + u * NG + g;
      const int jc = j[u] < jend ? j[u] : jend - 1;          // in-bounds repeat, result dropped
      rowv[u] = *(const u32x4_t*)(col + (size_t)jc * HD);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (k < nq) {                                         // wave-uniform
          const float v = group_sum<LPH>(dot8<Tag>(rowv[u], qv[k], 0.f)) * scale;
          if (li == 0 && j[u] < jend) {
            uint16_t hi, lo;
            split_hi_lo<Tag>(v, hi, lo);
            Qp[(((size_t)b * 2 + 0) * Hp + h0 + k) * r + j[u]] = hi;
            Qp[(((size_t)b * 2 + 1) * Hp + h0 + k) * r + j[u]] = lo;
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// merge_expand: a workgroup merges the token splits of ONE head over a slice of js columns and
// expands that slice through its rows of B_v.  What bounds it is the chain of memory round trips,
// so everything that does not depend on anything is requested at the start: the splits' (m, l)
// pairs, the first splits' sums, the first eight rows of B_v per thread; the merge runs while the
// rows arrive.  The loads go through buffers that end with the slice, so that no lane has a branch
// and the waits stay exact.  Workgroups are numbered in runs per XCD: neighbouring heads, which
// share the rows' pages, with a basis per sequence; the same head of all sequences with a shared
// basis, which then stays in that XCD's L2.  plain: in launch order, so that all XCDs walk the rows of
// the same few sequences, where the bases do not fit the L2s anyway.
// Against two heads per workgroup, whose rows were requested after the merge, and a launch of its
// own that merged more than sixteen splits (us a pass): eight sequences of 32 heads, rank 512, 32
// splits 46.3 -> 39.3; sixteen of them with 16 splits 74.7 -> 70.8; one sequence, 256 splits 47.6 ->
// 39.7; 64 sequences on one shared basis, rank 640 223 -> 218.
// FEW: at most kFewSplits.  Every thread then takes all (m, l) pairs and one column at a time, so that
// the merge needs no exchange and half the registers (62 against 112: eight waves per SIMD, not four),
// which is what many heads with little work each want; without it 48 x 40 heads of rank 64 lost a tenth
// against two heads per workgroup.  Us a pass there / without FEW / with it: 64 sequences of 40 heads,
// rank 128 on a shared basis 25.4 / 27.3 / 25.0, 48 of 64 heads, rank 320 51.2 / 53.8 / 47.6, 24 of 32
// heads of 64, rank 64 13.4 / 14.1 / 12.8.
// SLICED: several slices per head; their sums go to pout [B][nslice][H d], which reduce_out adds up.
//   grid (H * nslice, B), one dimension being too short for all of them; NT threads, without FEW NT >= S
//   and NT >= js / 4; dynamic LDS: (without FEW) weights [S], ustar [js], sums max(4 NT, NT / 64 d)
// ------------------------------------------------------------------------------------------
struct MergeExpandParams {
  const float* part_ml;     // [B][S][H][2]
  const float* part_U;      // [B][S][H][r]
  const uint16_t* Bv;       // [B or 1][r][(H / G) d]
  int64_t bstride;
  void* out;                // [B][H][d]
  float* lse;               // [B][H] or null
  float* pout;              // SLICED: [B][nslice][H d]
  int B, H, HD, r, S, nslice, js, plain;
  FastDiv by_first, by_slice, by_group;   // B with a shared basis, else H; nslice; G
};
constexpr int kFewSplits = 8;

template <class Tag, bool OUT_F32, bool SLICED, bool FEW, int NT, int LPR>
__global__ void __launch_bounds__(NT) merge_expand(const MergeExpandParams p) {
  constexpr int d = LPR * 8, ROWS = NT / LPR, NW = NT / 64;   // a row segment per LPR lanes
  constexpr int kRows = 8, kU = 8;                            // loads in flight per thread of either kind
  extern __shared__ __attribute__((aligned(16))) float smem_me[];
  __shared__ float redw[2 * NW];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int S = p.S, H = p.H, r = p.r, js = p.js;
  float* wgt = smem_me;                                       // [S rounded up to 4]
  float* ustar = FEW ? smem_me : wgt + ((S + 3) & ~3);        // [js]
  float* sums = ustar + js;
  // ---- which head, sequence, slice
  const uint32_t total = gridDim.x * gridDim.y;               // < 2^32: B and H are at most 65535
  uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
  if ((total & 7) == 0 && !p.plain) id = (id & 7) * (total >> 3) + (id >> 3);
  int b, h, sl;
  if (p.bstride == 0) {
    const uint32_t t = p.by_first(id);
    b = (int)(id - t * (uint32_t)p.B);
    h = (int)p.by_slice(t);
    sl = (int)t - h * p.nslice;
  } else {
    const uint32_t t = p.by_first(id);
    h = (int)(id - t * (uint32_t)H);
    b = (int)p.by_slice(t);
    sl = (int)t - b * p.nslice;
  }
  const int kvh = (int)p.by_group((uint32_t)h);
  const int j0 = sl * js;
  // ---- requests: B_v rows, then (m, l), then the first sums
  const int rg = tid / LPR, cc = tid % LPR;
  const size_t HD = (size_t)p.HD;
  const uint16_t* Bb = p.Bv + (size_t)b * p.bstride + (size_t)j0 * HD + (size_t)kvh * d;
  u32x4_t wv[kRows];
  const uint32_t row_bytes = (uint32_t)HD * 2;
  const auto brow = make_buffer(Bb, (uint32_t)(js - 1) * row_bytes + d * 2);
  auto load_rows = [&](int j) {                               // rows j + k ROWS; zeros past the slice
#pragma unroll
    for (int k = 0; k < kRows; ++k) wv[k] = buffer_load16(brow, (uint32_t)(j + k * ROWS) * row_bytes + cc * 16);
  };
  const size_t pb = (size_t)b * S * H + h;                    // + s H
  const uint32_t split_bytes = (uint32_t)H * r * 4;           // H <= 64 here, or S <= 8: far below 4 GiB
  const auto bsum = make_buffer(p.part_U + pb * r + j0, (uint32_t)(S - 1) * split_bytes + js * 4);
  if constexpr (FEW) {
    float wv[kFewSplits], lv[kFewSplits], uv[kFewSplits];
#pragma unroll
    for (int k = 0; k < kFewSplits; ++k) {
      const f32x2_t ml = *(const f32x2_t*)(p.part_ml + (pb + (size_t)(k < S ? k : 0) * H) * 2);
      wv[k] = ml[0];
      lv[k] = ml[1];
    }
    auto load_sums = [&](int c) {                             // zeros past the last split
#pragma unroll
      for (int k = 0; k < kFewSplits; ++k) uv[k] = buffer_load4(bsum, (uint32_t)k * split_bytes + 4 * c);
    };
    load_sums(tid < js ? tid : 0);
    load_rows(rg);
    // ---- weights 2^(m_s - m*) and their weighted sum of l
    float m = wv[0], L = 0.f;
#pragma unroll
    for (int k = 1; k < kFewSplits; ++k) m = k < S ? fmaxf(m, wv[k]) : m;
#pragma unroll
    for (int k = 0; k < kFewSplits; ++k) {
      wv[k] = k < S ? fast_exp2(wv[k] - m) : 0.f;
      L = k < S ? fmaf(wv[k], lv[k], L) : L;
    }
    if (p.lse && tid == 0 && sl == 0) p.lse[(size_t)b * H + h] = (m + log2f(L)) * kLn2;
    // ---- ustar[j] = sum_s w_s U_s[j] / L
    for (int c = tid; c < js; c += NT) {
      if (c != tid) load_sums(c);
      float a = 0.f;
#pragma unroll
      for (int k = 0; k < kFewSplits; ++k) a = fmaf(wv[k], uv[k], a);
      ustar[c] = a / L;
    }
    lds_barrier();
  } else {
    const int nc4 = js >> 2, ngrp = NT / nc4;                   // four columns per thread, splits dealt to groups
    const int grp = tid / nc4, c4 = tid - grp * nc4;
    u32x4_t uv[kU];
    auto load_sums = [&](int s0) {                              // splits s0 + grp + k ngrp; zeros past the last
#pragma unroll
      for (int k = 0; k < kU; ++k) uv[k] = buffer_load16(bsum, (uint32_t)(s0 + grp + k * ngrp) * split_bytes + 16 * c4);
    };
    const size_t ml0 = (pb + (size_t)(tid < S ? tid : 0) * H) * 2;
    const f32x2_t ml = *(const f32x2_t*)(p.part_ml + ml0);
    load_sums(0);
    load_rows(rg);
    // ---- weights 2^(m_s - m*) and their weighted sum of l
    const float mv = tid < S ? ml[0] : -INFINITY;
    float m = mv;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (lane == 0) redw[w] = m;
    lds_barrier();
    m = redw[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) m = fmaxf(m, redw[k]);
    float L = 0.f;
    if (tid < S) {
      const float ws = fast_exp2(mv - m);
      wgt[tid] = ws;
      L = ws * ml[1];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) L += __shfl_xor(L, o);
    if (lane == 0) redw[NW + w] = L;
    lds_barrier();
    L = redw[NW];
#pragma unroll
    for (int k = 1; k < NW; ++k) L += redw[NW + k];
    if (p.lse && tid == 0 && sl == 0) p.lse[(size_t)b * H + h] = (m + log2f(L)) * kLn2;
    // ---- ustar[j] = sum_s w_s U_s[j] / L: a group's splits in order, then the groups in order
    f32x4_t acc4 = {0.f, 0.f, 0.f, 0.f};
    auto add_sums = [&](int s0) {
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        const int s = s0 + grp + k * ngrp;
        const float ws = s < S ? wgt[s] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc4[e] = fmaf(ws, __builtin_bit_cast(f32x4_t, uv[k])[e], acc4[e]);
      }
    };
    add_sums(0);
    for (int s0 = kU * ngrp; s0 < S; s0 += kU * ngrp) {
      load_sums(s0);
      add_sums(s0);
    }
    if (grp < ngrp) *(f32x4_t*)(sums + grp * js + 4 * c4) = acc4;
    lds_barrier();
    for (int j = tid; j < js; j += NT) {
      float a = sums[j];
      for (int k = 1; k < ngrp; ++k) a += sums[k * js + j];
      ustar[j] = a / L;
    }
    lds_barrier();
  }
  // ---- expansion: thread (rg, cc) owns 8 columns and rows rg, rg + ROWS, ..
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto use_rows = [&](int j) {
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int jj = j + k * ROWS;
      const float u = jj < js ? ustar[jj] : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] = fmaf(u, lo_to_f32(wv[k][e], Tag{}), acc[2 * e]);
        acc[2 * e + 1] = fmaf(u, hi_to_f32(wv[k][e], Tag{}), acc[2 * e + 1]);
      }
    }
  };
  use_rows(rg);
  for (int j = rg + kRows * ROWS; j < js; j += kRows * ROWS) {
    load_rows(j);
    use_rows(j);
  }
  // the lanes of a wave that share columns, then the waves
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o);
  if (lane < LPR) {
    *(f32x4_t*)(sums + w * d + cc * 8) = f32x4_t{acc[0], acc[1], acc[2], acc[3]};
    *(f32x4_t*)(sums + w * d + cc * 8 + 4) = f32x4_t{acc[4], acc[5], acc[6], acc[7]};
  }
  lds_barrier();
  for (int i = tid; i < d; i += NT) {
    float sum = sums[i];
#pragma unroll
    for (int k = 1; k < NW; ++k) sum += sums[k * d + i];
    if (SLICED) p.pout[((size_t)b * p.nslice + sl) * H * d + (size_t)h * d + i] = sum;
    else if (OUT_F32) ((float*)p.out)[((size_t)b * H + h) * d + i] = sum;
    else ((uint16_t*)p.out)[((size_t)b * H + h) * d + i] = f32_to_bits(sum, Tag{});
  }
}


// ------------------------------------------------------------------------------------------
// expand_append: the expansion through B_v and the append of the new token's value row in ONE
// pass over B_v (a fused decode step).  attn_partial has scored all T tokens but summed the
// value coefficients of the T-1 older ones only, exporting the newest token's softmax weight;
// that token's weighted coefficient sum is its own coefficient row c_v[j] = B_v[j, :] . v_new,
// which a whole-row pass produces row by row.  So for basis row j
//     U*[h, j]  = A[h, j] + beta[h] * c_v[j]
//     out[h, :] += U*[h, j] * B_v[j, head h]
// with A the merged, normalised partial sums of the older tokens and beta[h] the new token's
// softmax weight.  A workgroup owns a block of rows; its per-column sums go to a partial buffer
// that reduce_out adds up in a fixed order (deterministic).
//   grid (ceil(r / rpw), B), 128 threads; dynamic LDS: A [H][rpw + 1], statistics.
// ------------------------------------------------------------------------------------------
struct ExpandParams {
  const uint16_t* Bv;
  int64_t bstride;
  const uint16_t* v_new;    // [B][HD]
  uint16_t* Cv;             // [B][T_cap][r]: row T-1 is written
  const float* part_ml;     // [B][S][H][2] (reference exponent, sum) over all T tokens
  const float* part_U;      // [B][S][H][r] over tokens 0 .. T-2
  const float* pnew;        // [B][H] weight of token T-1 relative to the reference of the split that holds it
  const int* pnew_split;    // [B] that split, or null: the last one
  const int32_t* rank_v;    // [B][T] per-token value ranks, or null: the new token counts at rank r
  float* pout;              // [B][nob][HD] per-row-block column sums
  float* lse;               // [B][H] or null
  int H, d, HD, r, T, T_cap, nsplit, rpw, nob;
};

template <class Tag, int KPC, int NBUF>
__global__ void __launch_bounds__(128) expand_append(const ExpandParams p) {
  // Two waves share the workgroup's rows, each owning KPC / 2 of the 512-element passes over
  // the hidden axis (so the column sums fit in registers); the two halves of a row's dot
  // product meet in LDS once per row.
  constexpr int KH = KPC / 2;
  extern __shared__ __attribute__((aligned(16))) float lds_ea[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int half = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rpw = p.rpw, pitch = rpw + 1;
  const int b = blockIdx.y, j0 = blockIdx.x * rpw;
  const int H = p.H, HD = p.HD, r = p.r, S = p.nsplit;
  float* Atile = lds_ea;                       // [H][pitch]
  float* mstar = Atile + H * pitch;            // [H]
  float* invL = mstar + H;                     // [H]
  float* beta = invL + H;                      // [H]
  float* dotx = beta + H;                      // [2][2] half dot products, double-buffered
  float* wsp = dotx + 4;                       // [S][H] split weights (when they fit)
  const bool wsp_fits = S * H <= 4096;
  const uint16_t* Bb = p.Bv + (size_t)b * p.bstride;

  // ---- row ring: requests go out first (see basis_rows)
  u32x4_t buf[NBUF][KH];
  int eoff[KH];
  bool inside[KH];
#pragma unroll
  for (int pp = 0; pp < KH; ++pp) {
    const int e0 = (half * KH + pp) * 512 + lane * 8;
    inside[pp] = e0 < HD;
    eoff[pp] = inside[pp] ? e0 : (lane * 8 < HD ? lane * 8 : 0);
  }
  auto load_row = [&](u32x4_t (&dst)[KH], int i) {
    int j = j0 + i;
    j = j < r ? j : r - 1;
    const uint16_t* row = Bb + (size_t)j * HD;
#pragma unroll
    // (a basis row is read once per launch: non-temporal, measured 92.2 -> 88.3 us; the same hint
    // costs basis_rows 7 us and is not used there)
    for (int pp = 0; pp < KH; ++pp) dst[pp] = __builtin_nontemporal_load((const u32x4_t*)(row + eoff[pp]));
  };
  u32x4_t vs[KH];
#pragma unroll
  for (int pp = 0; pp < KH; ++pp) {
    const u32x4_t z = {0, 0, 0, 0};
    vs[pp] = inside[pp] ? *(const u32x4_t*)(p.v_new + (size_t)b * HD + eoff[pp]) : z;
  }
  const int last = rpw - 1;
#pragma unroll
  for (int u = 0; u + 1 < NBUF; ++u) load_row(buf[u], u < last ? u : last);

  // ---- merged softmax statistics: one thread per head
  if (tid < H) {
    const int h = tid;
    const size_t pb = (size_t)b * S * H + h;
    // the splits' (reference exponent, sum) pairs, eight loads in flight at a time
    float m = -INFINITY;
    for (int s0 = 0; s0 < S; s0 += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = s0 + u < S ? p.part_ml[(pb + (size_t)(s0 + u) * H) * 2] : -INFINITY;
#pragma unroll
      for (int u = 0; u < 8; ++u) m = fmaxf(m, v[u]);
    }
    float L = 0.f, wlast = 0.f;
    const int snew = p.pnew_split ? p.pnew_split[b] : S - 1;
    for (int s0 = 0; s0 < S; s0 += 8) {
      float v[8], lv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool on = s0 + u < S;
        v[u] = on ? p.part_ml[(pb + (size_t)(s0 + u) * H) * 2] : -INFINITY;
        lv[u] = on ? p.part_ml[(pb + (size_t)(s0 + u) * H) * 2 + 1] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (s0 + u < S) {
          const float ws = fast_exp2(v[u] - m);
          L += lv[u] * ws;
          if (wsp_fits) wsp[(s0 + u) * H + h] = ws;
          if (s0 + u == snew) wlast = ws;
        }
      }
    }
    mstar[h] = m;
    invL[h] = 1.0f / L;
    beta[h] = wlast * p.pnew[(size_t)b * H + h] / L;
    if (p.lse && blockIdx.x == 0) p.lse[(size_t)b * H + h] = (m + log2f(L)) * kLn2;
  }
  __syncthreads();
  // ---- A[h][jl] = sum_s 2^(m_s - m*) U_s[h, j0 + jl] / L
  if (wsp_fits) {
    // four (head, row) pairs and four splits at a time: sixteen loads in flight per thread, so
    // the whole tile takes a few round trips to memory (the row ring stands still meanwhile)
    const int n = H * rpw;
    for (int i0 = tid; i0 < n; i0 += 4 * 128) {
      int hh[4], jj[4];
      bool ok[4];
      size_t base[4];
      float acc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 128 * u;
        const int h = i < n ? i / rpw : 0, jl = i < n ? i - h * rpw : 0;
        hh[u] = h;
        jj[u] = jl;
        ok[u] = i < n && j0 + jl < r;
        base[u] = ((size_t)b * S * H + h) * r + (ok[u] ? j0 + jl : 0);
        acc[u] = 0.f;
      }
      for (int s0 = 0; s0 < S; s0 += 4) {
        float uv[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k)
            uv[u][k] = s0 + k < S ? p.part_U[base[u] + (size_t)(s0 + k) * H * r] : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (s0 + k < S) acc[u] = fmaf(wsp[(s0 + k) * H + hh[u]], uv[u][k], acc[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + 128 * u < n) Atile[hh[u] * pitch + jj[u]] = ok[u] ? acc[u] * invL[hh[u]] : 0.f;
    }
  } else {
    for (int i = tid; i < H * rpw; i += 128) {
      const int h = i / rpw, jl = i - h * rpw;
      float acc = 0.f;
      if (j0 + jl < r) {
        const size_t pb = (size_t)b * S * H + h;
        const float m = mstar[h];
        for (int s = 0; s < S; ++s)
          acc = fmaf(fast_exp2(p.part_ml[(pb + (size_t)s * H) * 2] - m),
                     p.part_U[(pb + (size_t)s * H) * r + j0 + jl], acc);
        acc *= invL[h];
      }
      Atile[h * pitch + jl] = acc;
    }
  }
  __syncthreads();

  // the new token's own value rank limits the rows in which its coefficient counts
  int rvn = r;
  if (p.rank_v) {
    rvn = p.rank_v[(size_t)b * p.T + p.T - 1];
    rvn = rvn < 0 ? 0 : (rvn < r ? rvn : r);
  }
  const int dshift = 31 - __builtin_clz((unsigned)p.d);
  float bt[KH];
  int arow[KH];                                // A row (head) of this lane's chunk in every pass
#pragma unroll
  for (int pp = 0; pp < KH; ++pp) {
    const int h = inside[pp] ? eoff[pp] >> dshift : 0;
    bt[pp] = inside[pp] ? beta[h] : 0.f;
    arow[pp] = h * pitch;
  }
  float o[KH][8];
#pragma unroll
  for (int pp = 0; pp < KH; ++pp)
#pragma unroll
    for (int e = 0; e < 8; ++e) o[pp][e] = 0.f;

  auto use_row = [&](const u32x4_t (&row)[KH], int i) {
    const bool live = i < rpw && j0 + i < r;
    float acc = 0.f;
#pragma unroll
    for (int pp = 0; pp < KH; ++pp) acc = dot8<Tag>(row[pp], vs[pp], acc);
    acc = wave_sum(acc);
    float* slot = dotx + (i & 1) * 2;
    if (lane == 0) slot[half] = acc;
    // both waves run the same number of rows.  Only LDS traffic has to be ordered here: a full
    // __syncthreads() would also wait for the row loads in flight and drain the ring.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const float c = slot[0] + slot[1];
    const uint16_t cbits = f32_to_bits(c, Tag{});
    if (lane == 0 && half == 0 && live) p.Cv[((size_t)b * p.T_cap + p.T - 1) * r + j0 + i] = cbits;
    const float cr = live && j0 + i < rvn ? bits_to_f32(cbits, Tag{}) : 0.f;   // the stored (rounded) coefficient
    const int jc = live ? i : 0;
#pragma unroll
    for (int pp = 0; pp < KH; ++pp) {
      const float wgt = live ? fmaf(bt[pp], cr, Atile[arow[pp] + jc]) : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[pp][2 * e] = fmaf(wgt, lo_to_f32(row[pp][e], Tag{}), o[pp][2 * e]);
        o[pp][2 * e + 1] = fmaf(wgt, hi_to_f32(row[pp][e], Tag{}), o[pp][2 * e + 1]);
      }
    }
  };
  const int rpw_pad = (rpw + NBUF - 1) / NBUF * NBUF;
  for (int i = 0; i < rpw_pad; i += NBUF) {
#pragma unroll
    for (int u = 0; u < NBUF; ++u) {
      const int nx = i + u + NBUF - 1;
      if (NBUF > 1) load_row(buf[(u + NBUF - 1) % NBUF], nx < last ? nx : last);
      else load_row(buf[0], i < last ? i : last);
      use_row(buf[u], i + u);
    }
  }
  // ---- the two waves own disjoint columns: straight to the partial buffer
  float* dst = p.pout + ((size_t)b * p.nob + blockIdx.x) * HD;
#pragma unroll
  for (int pp = 0; pp < KH; ++pp) {
    if (inside[pp]) {
      const f32x4_t v0 = {o[pp][0], o[pp][1], o[pp][2], o[pp][3]};
      const f32x4_t v1 = {o[pp][4], o[pp][5], o[pp][6], o[pp][7]};
      *(f32x4_t*)(dst + eoff[pp]) = v0;
      *(f32x4_t*)(dst + eoff[pp] + 4) = v1;
    }
  }
}

// out[b, c] = sum over row blocks of pout[b][blk][c], in block order.  grid (ceil(HD/1024), B).
template <class Tag, bool OUT_F32>
__global__ void __launch_bounds__(256)
reduce_out(const float* __restrict__ pout, void* __restrict__ out, int HD, int nob) {
  const int b = blockIdx.y, c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= HD) return;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  int k = 0;
  for (; k + 8 <= nob; k += 8) {                         // eight loads in flight, summed in block order
    f32x4_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = *(const f32x4_t*)(pout + ((size_t)b * nob + k + u) * HD + c);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; k < nob; ++k) acc += *(const f32x4_t*)(pout + ((size_t)b * nob + k) * HD + c);
  if (OUT_F32) {
    *(f32x4_t*)((float*)out + (size_t)b * HD + c) = acc;
  } else {
    u32x2_t v = {pack2(acc[0], acc[1], Tag{}), pack2(acc[2], acc[3], Tag{})};
    *(u32x2_t*)((uint16_t*)out + (size_t)b * HD + c) = v;
  }
}


// ------------------------------------------------------------------------------------------
// merge_splits: many token splits (small batches) are merged once, in parallel, before the
// expansion: U'[h, j] = sum_s 2^(m_s - m*) U_s[h, j], l' = sum_s 2^(m_s - m*) l_s, m' = m*, written
// as a single split, and the deferred token's weight is rescaled to the merged reference.
//   grid (ceil(r / 64), H, B), 256 threads = 4 groups of splits x 64 columns.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
merge_splits(const float* __restrict__ part_ml, const float* __restrict__ part_U,
             float* __restrict__ out_ml, float* __restrict__ out_U, float* __restrict__ pnew,
             const int* __restrict__ pnew_split, int H, int r, int S) {
  extern __shared__ __attribute__((aligned(16))) float lds_ms[];   // [S] weights, then [4][64]
  __shared__ float red[8];
  const int tid = threadIdx.x, lane = tid & 63, grp = tid >> 6;
  const int h = blockIdx.y, b = blockIdx.z;
  const size_t pb = (size_t)b * S * H + h;                 // + s*H
  float* wgt = lds_ms;
  float* acc4 = lds_ms + S;
  // m* = max_s m_s
  float m = -INFINITY;
  for (int s = tid; s < S; s += 256) m = fmaxf(m, part_ml[(pb + (size_t)s * H) * 2]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if (lane == 0) red[grp] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float L = 0.f;
  for (int s = tid; s < S; s += 256) {
    const float ws = fast_exp2(part_ml[(pb + (size_t)s * H) * 2] - m);
    wgt[s] = ws;
    L += ws * part_ml[(pb + (size_t)s * H) * 2 + 1];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) L += __shfl_xor(L, o);
  if (lane == 0) red[4 + grp] = L;
  __syncthreads();
  L = (red[4] + red[5]) + (red[6] + red[7]);
  const int j = blockIdx.x * 64 + lane;
  float acc = 0.f;
  if (j < r) {
    int s = grp;
    for (; s + 28 < S; s += 32) {                          // eight loads in flight
      float u[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) u[k] = part_U[(pb + (size_t)(s + 4 * k) * H) * r + j];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc = fmaf(wgt[s + 4 * k], u[k], acc);
    }
    for (; s < S; s += 4) acc = fmaf(wgt[s], part_U[(pb + (size_t)s * H) * r + j], acc);
  }
  acc4[grp * 64 + lane] = acc;
  __syncthreads();
  if (grp == 0 && j < r)
    out_U[((size_t)b * H + h) * r + j] = (acc4[lane] + acc4[64 + lane]) + (acc4[128 + lane] + acc4[192 + lane]);
  if (blockIdx.x == 0 && tid == 0) {
    out_ml[((size_t)b * H + h) * 2] = m;
    out_ml[((size_t)b * H + h) * 2 + 1] = L;
    if (pnew) pnew[(size_t)b * H + h] *= wgt[pnew_split ? pnew_split[b] : S - 1];   // its split's weight
  }
}

}  // namespace
int basis_rows_per_wave(int B, int r, int HD, int jobs, int G, bool shared);
namespace {

template <class Tag, bool DOT, bool FOLD, bool PAIR>
ap_status launch_rows(RowsParams p, int B, hipStream_t stream) {
  const int rpw = basis_rows_per_wave(B, p.r, p.HD, PAIR ? 2 : 1, 1, p.bstride == 0);
  p.rpw = rpw;
  const int rows_wg = 4 * rpw;
  const dim3 grid((p.r + rows_wg - 1) / rows_wg, B, PAIR ? 2 : 1);
  const size_t lds = FOLD ? (size_t)p.Hp * (rows_wg + 1) * 4 : 0;
  const int kpc = (p.HD + 511) / 512;
#define AP_ROWS(K, NB)                                                                        \
  if (kpc <= K) {                                                                             \
    if (!FOLD) hipLaunchKernelGGL((basis_rows<Tag, K, NB, DOT, FOLD, 1, PAIR>), grid, dim3(256), lds, stream, p);            \
    else if (p.d == 128) hipLaunchKernelGGL((basis_rows<Tag, K, NB, DOT, FOLD, FOLD ? 16 : 1, PAIR>), grid, dim3(256), lds, stream, p); \
    else if (p.d == 64) hipLaunchKernelGGL((basis_rows<Tag, K, NB, DOT, FOLD, FOLD ? 8 : 1, PAIR>), grid, dim3(256), lds, stream, p);   \
    else if (p.d == 256) hipLaunchKernelGGL((basis_rows<Tag, K, NB, DOT, FOLD, FOLD ? 32 : 1, PAIR>), grid, dim3(256), lds, stream, p); \
    else hipLaunchKernelGGL((basis_rows<Tag, K, NB, DOT, FOLD, FOLD ? 4 : 1, PAIR>), grid, dim3(256), lds, stream, p);                  \
    return AP_OK;                                                                             \
  }
  AP_ROWS(2, 3) AP_ROWS(4, 3) AP_ROWS(8, 3) AP_ROWS(10, 2)
  AP_ROWS(16, (DOT && FOLD) ? 1 : 2)
#undef AP_ROWS
  set_error("basis pass: H*d=%d exceeds 8192", p.HD);
  return AP_ERR_UNSUPPORTED;
}

// Grouped queries: the key row's append, the fold of all G query heads per slice, and the value row's
// append in one launch.
template <class Tag, int KPC, int LPH, int G>
ap_status launch_rows_grouped(RowsParams p, int B, hipStream_t stream) {
  const int rpw = basis_rows_per_wave(B, p.r, p.HD, 2, G, p.bstride == 0);
  p.rpw = rpw;
  const dim3 grid((p.r + 4 * rpw - 1) / (4 * rpw), B, 2);
  const size_t lds = (size_t)p.Hp * (4 * rpw + 1) * 4;
  hipLaunchKernelGGL((basis_rows<Tag, KPC, 3, true, true, LPH, true, G>), grid, dim3(256), lds, stream, p);
  return AP_OK;
}
template <class Tag, int KPC, int LPH>
ap_status launch_rows_grouped(const RowsParams& p, int G, int B, hipStream_t stream) {
  if (G == 2) return launch_rows_grouped<Tag, KPC, LPH, 2>(p, B, stream);
  if (G == 4 || KPC > 2) return launch_rows_grouped<Tag, KPC, LPH, 4>(p, B, stream);
  return launch_rows_grouped<Tag, KPC, LPH, (KPC > 2 ? 4 : 8)>(p, B, stream);
}
template <class Tag>
ap_status launch_rows_grouped(const RowsParams& p, int G, int B, hipStream_t stream) {
  if (p.HD <= 1024)
    return p.d == 128 ? launch_rows_grouped<Tag, 2, 16>(p, G, B, stream) : launch_rows_grouped<Tag, 2, 8>(p, G, B, stream);
  return p.d == 128 ? launch_rows_grouped<Tag, 4, 16>(p, G, B, stream) : launch_rows_grouped<Tag, 4, 8>(p, G, B, stream);
}

}  // namespace

// A step of a grouped-query model whose basis rows are short (HD columns, H heads in groups of G): the
// launch above.  One launch instead of two (the appends; fold_heads) and B_k once instead of twice:
// 34.7 -> 31.9 us a pass at 21 sequences, 32 / 8 heads, rank 256, 3001 tokens.
bool rows_grouped_applies(int G, int d, int HD) {
  return (G == 2 || G == 4 || G == 8) && (d == 64 || d == 128) && HD <= (G == 8 ? 1024 : 2048);
}
ap_status launch_rows_grouped(ap_dtype dt, const void* Bk, const void* Bv, int64_t bstride, const void* k_new,
                              const void* v_new, const void* q, void* Ck, void* Cv, void* Qp, int B, int H, int H_kv,
                              int Hp, int d, int r, int row, int T_cap, float scale, hipStream_t stream) {
  const RowsParams p{(const uint16_t*)Bk, bstride, (const uint16_t*)k_new, (const uint16_t*)q, (uint16_t*)Ck,
                     (uint16_t*)Qp, H, Hp, d, H_kv * d, r, row, T_cap, 4, scale, FastDiv(Hp, (int64_t)Hp * r), (const uint16_t*)Bv,
                     (const uint16_t*)v_new, (uint16_t*)Cv};
  return dt == AP_F16 ? launch_rows_grouped<F16Tag>(p, H / H_kv, B, stream) : launch_rows_grouped<BF16Tag>(p, H / H_kv, B, stream);
}

bool basis_rows_applies(int HD, int B) { return HD % 8 == 0 && HD <= 8192 && B <= 65535; }

// Append (x != null) and / or fold (q != null) in one pass over Bm.  With Bm2, x2, C2 (and x)
// given, a second append of the same shape (C2's row row0 = Bm2 . x2) runs in the same launch.
ap_status launch_basis_rows(ap_dtype dt, const void* Bm, int64_t bstride, const void* x,
                            const void* q, void* C, void* Qp, int B, int H, int Hp, int d, int HD,
                            int r, int row0, int T_cap, float scale, hipStream_t stream,
                            const void* Bm2, const void* x2, void* C2) {
  RowsParams p{(const uint16_t*)Bm, bstride, (const uint16_t*)x, (const uint16_t*)q,
               (uint16_t*)C, (uint16_t*)Qp, H, Hp, d, HD, r, row0, T_cap, 4, scale, FastDiv(Hp, (int64_t)Hp * r),
               (const uint16_t*)Bm2, (const uint16_t*)x2, (uint16_t*)C2};
  const bool dot = x != nullptr, fold = q != nullptr, pair = Bm2 != nullptr;
  if (pair && !(dot && x2 && C2)) {
    set_error("basis pass: a second append needs a first one and all of Bm2, x2, C2");
    return AP_ERR_INVALID_ARG;
  }
  if (dt == AP_F16) {
    if (pair) return fold ? launch_rows<F16Tag, true, true, true>(p, B, stream) : launch_rows<F16Tag, true, false, true>(p, B, stream);
    if (dot && fold) return launch_rows<F16Tag, true, true, false>(p, B, stream);
    if (dot) return launch_rows<F16Tag, true, false, false>(p, B, stream);
    return launch_rows<F16Tag, false, true, false>(p, B, stream);
  }
  if (pair) return fold ? launch_rows<BF16Tag, true, true, true>(p, B, stream) : launch_rows<BF16Tag, true, false, true>(p, B, stream);
  if (dot && fold) return launch_rows<BF16Tag, true, true, false>(p, B, stream);
  if (dot) return launch_rows<BF16Tag, true, false, false>(p, B, stream);
  return launch_rows<BF16Tag, false, true, false>(p, B, stream);
}

ap_status launch_fold_heads(ap_dtype dt, const void* Bk, int64_t bstride, const void* q, void* Qp, int B,
                            int H, int H_kv, int Hp, int d, int r, float scale, hipStream_t stream) {
  const int G = H / H_kv;
  const dim3 grid(H_kv * ((G + 7) / 8), (r + 63) / 64, B);
#define AP_FH(TAG, L)                                                                                   \
  hipLaunchKernelGGL((fold_heads<TAG, L>), grid, dim3(256), 0, stream, (const uint16_t*)Bk, bstride,    \
                     (const uint16_t*)q, (uint16_t*)Qp, H, G, Hp, r, scale)
  if (dt == AP_F16) {
    switch (d) { case 32: AP_FH(F16Tag, 4); break; case 64: AP_FH(F16Tag, 8); break;
                 case 128: AP_FH(F16Tag, 16); break; default: AP_FH(F16Tag, 32); break; }
  } else {
    switch (d) { case 32: AP_FH(BF16Tag, 4); break; case 64: AP_FH(BF16Tag, 8); break;
                 case 128: AP_FH(BF16Tag, 16); break; default: AP_FH(BF16Tag, 32); break; }
  }
#undef AP_FH
  return AP_OK;
}

// Rows of a basis per wave.  jobs: 2 where the launch also appends the value row; G: query heads per slice;
// shared: one basis for all sequences, whose rows come out of the L2s.
// Many rows: about five workgroups per CU, two of them resident at a time: the start and the end of a
// workgroup (vector slices in, folded tile out) then overlap other workgroups' streaming.
// Few: what counts is how evenly the workgroups fall on the 256 CUs, against a wave's vector slices, which
// are as long as a row (two where it also appends).  Alone in its launch a job wants every CU used once:
// two rows up to 256 workgroups, four up to 256 of those, and beyond that two again, as three rounds of
// two rows are fewer than two of four.  Two jobs go through one CU at a time: the same with 512.
// Us a pass at 4 / 2 rows, HD = 4096: one job 2048 rows 17.9 / 17.2, 2560 19.0 / 19.6, 4160 28.8 / 27.3; two
// jobs 2048 rows 23.9 / 22.9, 3072 26.8 / 27.7, 4608 36.9 / 34.6.  Rows of at most 2048 elements are too
// short for more than two to pay (HD = 2048, two jobs: 15.8 / 15.1 at 2048 rows, 20.4 / 19.6 at 4160).
// HD 4097 - 5120, two jobs: its ring of two rows leaves room for one workgroup, 256 again, and then four
// (2048 rows 28.8 / 29.3, 4608 40.6 / 41.6); above that no ring, more waves help longer (HD = 6144: 2496
// rows 27.4 / 26.4, 3072 36.4 / 36.9, 4608 48.6 / 46.1).  One basis for all: 2560 rows of 4096 21.7 / 21.2
// (two jobs) and 16.8 / 16.5, 5120 26.6 / 29.7, 2048 of 5120 24.1 / 23.5, 3072 25.3 / 27.4 and 17.7 / 18.3.
// More than 5120 rows: HD = 4096 8192 rows 49.1 / 50.3, shared 10240 31.7 / 34.9; only short ones gain
// (12288 rows of 512 17.7 / 17.1, 6144 of 1024 17.2 / 16.8, two jobs), and odd numbers of rows, whose folded
// pieces are not aligned, do not pay elsewhere (15360 rows of 5120 at 4 / 3: 55.5 / 92.0).
// Several heads per slice are work that grows with the rows: 32 heads on 8 of 64 6144 rows 19.1 / 18.1, 64
// on 16 of 128 6144 rows 34.9 / 33.2, shared 7296 30.7 / 31.4, 10240 rows 47.4 / 49.2.
// One row: 64 rows in all 17.2 / 16.8 at 4 / 2 and 16.4, 256 rows of 8192 22.5 / 19.6 and 18.5.
int basis_rows_per_wave(int B, int r, int HD, int jobs, int G, bool shared) {
  const int64_t rows = (int64_t)B * r, bytes = rows * HD * 2;
  const int rpw = (int)((rows + 5119) / 5120);
  if (rpw > 4) return rpw > 32 ? 32 : rpw;
  if (rows <= 256) return 1;
  if (G > 1) return bytes >= (28ll << 20) ? 4 : (rpw < 2 ? 2 : rpw);
  if (rows > 5120) return jobs == 2 && bytes < (16ll << 20) ? rpw : 4;
  if (HD <= 2048) return 2;
  const bool short_ring = HD > 4096 && HD <= 5120;
  if (jobs == 1 && shared && !short_ring) return 2;
  const int64_t wg2 = (int64_t)((r + 7) / 8) * B * jobs, wg4 = (int64_t)((r + 15) / 16) * B * jobs;
  if (jobs == 1) return wg2 <= 256 || wg4 > 256 ? 2 : 4;
  if (short_ring) return wg2 <= (shared ? 512 : 256) ? 2 : 4;
  return wg2 <= (shared || HD > 5120 ? 640 : 512) || (wg4 > 512 && !shared) ? 2 : 4;
}
// expand_append: about four two-wave workgroups per CU in one round, but never more than 16 row
// blocks per sequence at large batches (each block writes an HD-wide partial output that
// reduce_out reads back; measured at 64 sequences of rank 640 with the non-temporal row loads:
// 16 blocks 292 us per step, 10 blocks 292, 8 blocks 295, 32 blocks 310, 5 blocks 328); small
// batches, whose partial outputs are small anyway, take up to 64 blocks so that the launch still
// fills the chip.
int expand_rows_per_pair(int B, int r) {
  int rpw = (int)(((int64_t)B * r + 1023) / 1024);
  const int nob_max = B >= 32 ? 16 : B >= 16 ? 32 : 64;
  const int floor_rows = (r + nob_max - 1) / nob_max;
  if (rpw < floor_rows) rpw = floor_rows;
  return rpw < 4 ? 4 : (rpw > 128 ? 128 : rpw);
}

ap_status launch_merge_splits(const float* part_ml, const float* part_U, float* out_ml, float* out_U,
                              float* pnew, const int* pnew_split, int B, int H, int r, int S,
                              hipStream_t stream) {
  const size_t lds = ((size_t)S + 256) * 4;
  hipLaunchKernelGGL(merge_splits, dim3((r + 63) / 64, H, B), dim3(256), lds, stream, part_ml, part_U,
                     out_ml, out_U, pnew, pnew_split, H, r, S);
  return AP_OK;
}
int expand_row_blocks(int B, int r) { return (r + expand_rows_per_pair(B, r) - 1) / expand_rows_per_pair(B, r); }

ap_status launch_expand_append(ap_dtype dt, bool out_f32, const void* Bv, int64_t bstride,
                               const void* v_new, void* Cv, const float* part_ml,
                               const float* part_U, const float* pnew, const int* pnew_split,
                               const int32_t* rank_v, float* pout, void* out,
                               float* lse, int B, int H, int d, int r, int T, int T_cap, int nsplit,
                               hipStream_t stream) {
  ExpandParams p{(const uint16_t*)Bv, bstride, (const uint16_t*)v_new, (uint16_t*)Cv, part_ml, part_U,
                 pnew, pnew_split, rank_v, pout, lse, H, d, H * d, r, T, T_cap, nsplit, expand_rows_per_pair(B, r),
                 expand_row_blocks(B, r)};
  const dim3 grid(p.nob, B);
  const size_t lds = ((size_t)H * (p.rpw + 1) + 3 * (size_t)H + 4 + (nsplit * H <= 4096 ? (size_t)nsplit * H : 0)) * 4;
  const int kpc = (p.HD + 511) / 512;
#define AP_EA(TAG, K, NB)                                                                        \
  if (kpc <= K) {                                                                                \
    hipLaunchKernelGGL((expand_append<TAG, K, NB>), grid, dim3(128), lds, stream, p);            \
    break;                                                                                       \
  }
  do {
    if (dt == AP_F16) { AP_EA(F16Tag, 2, 3) AP_EA(F16Tag, 4, 3) AP_EA(F16Tag, 8, 3) AP_EA(F16Tag, 10, 2) AP_EA(F16Tag, 16, 2) }
    else { AP_EA(BF16Tag, 2, 3) AP_EA(BF16Tag, 4, 3) AP_EA(BF16Tag, 8, 3) AP_EA(BF16Tag, 10, 2) AP_EA(BF16Tag, 16, 2) }
    set_error("expand: H*d=%d exceeds 8192", p.HD);
    return AP_ERR_UNSUPPORTED;
  } while (0);
#undef AP_EA
  const dim3 g2((p.HD + 1023) / 1024, B);
  if (dt == AP_F16) {
    if (out_f32) hipLaunchKernelGGL((reduce_out<F16Tag, true>), g2, dim3(256), 0, stream, pout, out, p.HD, p.nob);
    else hipLaunchKernelGGL((reduce_out<F16Tag, false>), g2, dim3(256), 0, stream, pout, out, p.HD, p.nob);
  } else {
    if (out_f32) hipLaunchKernelGGL((reduce_out<BF16Tag, true>), g2, dim3(256), 0, stream, pout, out, p.HD, p.nob);
    else hipLaunchKernelGGL((reduce_out<BF16Tag, false>), g2, dim3(256), 0, stream, pout, out, p.HD, p.nob);
  }
  return AP_OK;
}

namespace {
template <class Tag, bool OUT_F32, bool SLICED, bool FEW, int NT>
void launch_me(const MergeExpandParams& p, int d, hipStream_t stream) {
  const dim3 grid(p.H * p.nslice, p.B);
  const int most = FEW ? NT / 64 * d : (4 * NT > NT / 64 * d ? 4 * NT : NT / 64 * d);
  const size_t lds = ((size_t)(FEW ? 0 : (p.S + 3) & ~3) + p.js + most) * 4;
  switch (d) {
    case 32: hipLaunchKernelGGL((merge_expand<Tag, OUT_F32, SLICED, FEW, NT, 4>), grid, dim3(NT), lds, stream, p); break;
    case 64: hipLaunchKernelGGL((merge_expand<Tag, OUT_F32, SLICED, FEW, NT, 8>), grid, dim3(NT), lds, stream, p); break;
    case 128: hipLaunchKernelGGL((merge_expand<Tag, OUT_F32, SLICED, FEW, NT, 16>), grid, dim3(NT), lds, stream, p); break;
    default: hipLaunchKernelGGL((merge_expand<Tag, OUT_F32, SLICED, FEW, NT, 32>), grid, dim3(NT), lds, stream, p); break;
  }
}
template <class Tag, bool OUT_F32, bool FEW>
void launch_me_nt(const MergeExpandParams& p, int d, int nt, hipStream_t stream) {
  if (nt == 64) launch_me<Tag, OUT_F32, false, FEW, 64>(p, d, stream);
  else if (nt == 128) launch_me<Tag, OUT_F32, false, FEW, 128>(p, d, stream);
  else launch_me<Tag, OUT_F32, false, FEW, 256>(p, d, stream);
}
template <class Tag, bool OUT_F32>
void launch_me_form(const MergeExpandParams& p, int d, int nt, hipStream_t stream) {
  if (p.nslice > 1) {
    launch_me<Tag, OUT_F32, true, false, 256>(p, d, stream);
    const int HD = p.H * d;
    hipLaunchKernelGGL((reduce_out<Tag, OUT_F32>), dim3((HD + 1023) / 1024, p.B), dim3(256), 0, stream, p.pout, p.out, HD, p.nslice);
  } else if (p.S <= kFewSplits) {
    launch_me_nt<Tag, OUT_F32, true>(p, d, nt, stream);
  } else {
    launch_me_nt<Tag, OUT_F32, false>(p, d, nt, stream);
  }
}
// Threads per workgroup.  passes: of 256 threads over a slice's rows.  Fewer threads where that leaves one
// few rows, the sooner the more workgroups there are to fill the chip; 32 lanes' rows (d = 32) are too
// short for the middle form.  Us a pass at 256 / 128 / 64 threads:
//   few splits: 1 pass, 3072 heads 21.8 / 18.6 / 17.0; 2, 384 11.1 / 10.7 / 10.4; 4, 384 11.2 / 10.6 / 10.8;
//   4, 4096 28.4 / 24.6 / 23.3; 8, 64 10.1 / 10.3 / 11.3; 8, 2560 26.1 / 25.0 / 24.7; 20, 1920 40.1 / 38.8 / 40.6;
//   d = 32, 8 passes, 4096 heads 92.0 / 102.2 / 98.8
//   more: rank 192 82.1 / 80.9 (1280 heads), rank 64 17.3 / 16.8 (32 heads) and 96.3 / 93.5 / 92.4 (2048), 640
//   heads, 12 splits 16.7 / 16.1 / 15.0; 47 splits, 32 heads, 8 passes 12.8 / 13.4 / 14.5
int merge_expand_threads(int64_t heads, int d, int js, int S) {
  const int passes = js * (d / 8) / 256;
  if (S <= kFewSplits) {
    if (passes <= 2 || (passes <= 4 && heads >= 2048)) return 64;
    if (d == 32) return 256;
    return passes <= 4 || (passes <= 24 && heads >= 768) ? 128 : 256;
  }
  const int fit = S > js / 4 ? S : js / 4;                // a thread per split and per four columns at least
  if (S <= 32 && fit <= 64 && (passes <= 2 || (passes <= 4 && heads >= 512))) return 64;
  return fit <= 128 && (passes <= 4 || (passes <= 12 && S <= 32)) ? 128 : 256;
}
}  // namespace

// pout: room for expand_row_blocks(B, r) slices of [B][H d] sums, or null (one slice per head then).
ap_status launch_merge_expand(ap_dtype dt, bool out_f32, const float* part_ml, const float* part_U,
                              const void* Bv, int64_t bstride, void* out, float* lse, float* pout, int B, int H,
                              int H_kv, int d, int r, int nsplit, hipStream_t stream) {
  AP_REQUIRE(nsplit >= 1 && nsplit <= kMergeExpandSplits && r % 4 == 0 && r <= 1024, AP_ERR_UNSUPPORTED,
             "merge_expand: %d splits of rank %d (at most %d, and r %% 4 == 0, r <= 1024)", nsplit, r, kMergeExpandSplits);
  // Slices of a head (and a launch more, which adds them up): once the sums of its splits are more
  // than one workgroup pulls in while the launch would run.  Per pass with one slice / the slices
  // chosen here: 256 splits of rank 512 28.7 / 24.6 us, 125 of 640 36.9 / 34.1; but 256 of 256
  // 16.9 / 18.3, 85 of 448 31.5 / 33.3.
  int nslice = 1;
  if (pout && r % 64 == 0 && (int64_t)nsplit * r * 4 > 288 * 1024)
    for (int k = 2; k <= 8; ++k)
      if (r / 64 % k == 0 && k <= expand_row_blocks(B, r)) nslice = k;
  const int js = r / nslice, nt = merge_expand_threads((int64_t)B * H, d, js, nsplit);
  // Bases that do not fit the XCDs' L2s (32 MB) in launch order: 64 sequences of 64 heads of 128, rank 64
  // 42.4 us with two heads per workgroup, 44.5 in runs per XCD, 42.0 in launch order; 16 of them, rank 512,
  // 16 splits 84.4, 87.0, 80.8.  Not with heads of 32, whose 64-byte pieces would share their lines across
  // XCDs (64 x 64 heads, rank 320 63.4 / 71.8), nor of 256 (no difference), nor with
  // grouped queries, whose heads share a slice that every XCD would then fetch (40 x 32/8 heads, rank 448
  // 43.6 / 52.5).
  const int plain = bstride && H == H_kv && (d == 64 || d == 128) && (int64_t)B * r * H_kv * d * 2 >= (32ll << 20);
  MergeExpandParams p{part_ml, part_U, (const uint16_t*)Bv, bstride, out, lse, pout, B, H, H_kv * d, r, nsplit, nslice, js, plain,
                      FastDiv(bstride ? H : B, (int64_t)B * H * nslice), FastDiv(nslice, (int64_t)std::max(B, H) * nslice), FastDiv(H / H_kv, H)};
  if (dt == AP_F16) {
    if (out_f32) launch_me_form<F16Tag, true>(p, d, nt, stream);
    else launch_me_form<F16Tag, false>(p, d, nt, stream);
  } else {
    if (out_f32) launch_me_form<BF16Tag, true>(p, d, nt, stream);
    else launch_me_form<BF16Tag, false>(p, d, nt, stream);
  }
  return AP_OK;
}

}  // namespace ap
