// float32-arithmetic path of the routed attention (float32 inputs of any
// width, and d = 32): forward and backward on v_mfma_f32_32x32x2_f32, whose
// products and sums are float32.
//
// A wave holds 32 queries (key side of the backward: 32 keys) and walks
// 32-row tiles of the other side from LDS.  With lane = 32 g + c, the
// instruction takes A (32 x 2: lane holds row c, slot g), B (2 x 32: column c,
// slot g) and C (32 x 32: column c, rows 8j + 4g + i in accumulator 4j + i):
//   scores      S^T = K Q^T: slot g of step s is element g D/2 + s, so a lane
//               reads its half of a tile row in 16-byte pieces and holds its
//               half of the query row in registers;
//   weighted    O^T += V^T P^T: step e takes rows 8j + i (g = 0) and 8j + 4 + i
//   sums        (g = 1), i.e. accumulator e of the scores is the B operand as
//               it is, and a lane reads one value of column c per step.
// The four waves of a workgroup share one 32-row block and take every fourth
// tile each (QW = 1), or share a 64-row block in two pairs that take every
// second tile (QW = 2: see f32_qw), or hold a 32-row block each (QW = 4: see
// f32_short); the waves' partial results are merged in order through LDS.
//
// Masked (query, key) pairs get weight zero; where a tile that has such pairs
// also holds a non-finite value (zero times it would be NaN), its weighted
// sums are formed row by row instead (f32_sum_checked), so a token never sees
// a later one's values.
//
// What bounds it: with short segments (B 2, T 1000, H 16, K 4, d 64: 250 rows)
// the chain of a block (offsets, tokens, rows, two or three rounds of staging,
// products and barrier, merge): forward 27 us, query side 46, key side 39.
// One lane per row with operands broadcast from LDS, in 64- or 256-row blocks,
// took 255, 418 and 506 us.  With long ones (T 8192, H 16, K 8) the products:
// 55 TFLOP/s of the 154 that a large float32 product reaches; the staging and
// the softmax are not hidden behind them.  Loading the next tiles' rows into
// registers during the products did not help (same at 250 rows, 5-15 % slower
// at 1000 and more: fewer registers for the operand reads).
#include <cfloat>
#include <cmath>

#include "common.h"
#include "internal.h"
#include "launch.h"
#include "tile.h"

namespace namoh {

constexpr int kFThreads = 256;
constexpr int kFSegLds = 1024;   // segment offsets staged in LDS up to this many

template <int D, int QW> struct FShape {
  static constexpr int HD = D / 2;             // a lane's half row
  static constexpr int DT = D / 32;            // 32-column accumulators per row
  static constexpr int LD = D + 4;             // LDS row stride: 16 rows' 16-byte reads cover all banks
  static constexpr int KS = 4 / QW;            // waves that split the tiles of one block
  static constexpr int ROWS = 32 * KS;         // rows staged at once, a tile per part
  static constexpr int BM = 32 * QW;           // block rows of a workgroup
  // keys and values (queries and output gradients) of a staging; later the
  // parts' rows of one gradient or two (KS BM = 128 rows each)
  // (QW = 4, forward only: one part)
  static constexpr int BUF = (QW == 4 ? 1 : 2) * 128 * LD;
  static constexpr int MINB = D == 128 ? 1 : QW == 4 ? 3 : 2;
};

struct FBlock { int s, a, n, r0; };   // segment, first packed row, length, first row of the block

// Blocks of BM rows are numbered seg0 / BM + s (disjoint and increasing over
// the segments, below Nr / BM + BH + 1).  False for a number between segments
// and for offsets that are not a packing.  s_off: scratch in LDS that is free
// again when the function returns.
template <int BM>
NAMOH_DEV bool f32_block(const int32_t* __restrict__ seg_offsets, int BH, int T, int Nr, int* s_off,
                         FBlock& o) {
  const int gt = block_x(), lane = thread_x() % kWave;
  const bool in_lds = BH <= kFSegLds;
  if (in_lds)
    for (int i = thread_x(); i <= BH; i += kFThreads) s_off[i] = seg_offsets[i];
  __syncthreads();
  if (in_lds) {
    int cnt = 0;
    for (int s0 = 0; s0 < BH; s0 += kWave) {
      const int si = s0 + lane;
      cnt += __popcll(__ballot(si < BH && s_off[min(si, BH)] / BM + si <= gt));
    }
    o.s = max(cnt - 1, 0);
    o.a = s_off[o.s];
    o.n = s_off[o.s + 1] - o.a;
  } else {
    int lo = 0, hi = BH;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (seg_offsets[mid] / BM + mid <= gt) lo = mid; else hi = mid;
    }
    o.s = lo;
    o.a = seg_offsets[lo];
    o.n = seg_offsets[lo + 1] - o.a;
  }
  o.s = __builtin_amdgcn_readfirstlane(o.s);
  o.a = __builtin_amdgcn_readfirstlane(o.a);
  o.n = __builtin_amdgcn_readfirstlane(o.n);
  o.r0 = (gt - (o.a / BM + o.s)) * BM;
  __syncthreads();
  return o.r0 >= 0 && o.r0 < o.n && o.a >= 0 && o.n <= T && o.a + o.n <= Nr;
}

NAMOH_DEV f32x16 f32_zero16() {
  f32x16 z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}

NAMOH_DEV bool f32_bad4(const float4 x) {   // any of the four not finite
  return !(fabsf(x.x) <= FLT_MAX) || !(fabsf(x.y) <= FLT_MAX) || !(fabsf(x.z) <= FLT_MAX) ||
         !(fabsf(x.w) <= FLT_MAX);
}

// tile (32 rows, row stride LD) x the lane's half row b
template <int D>
NAMOH_DEV f32x16 f32_scores(const float* tile, const float (&b)[D / 2], int c, int g) {
  const float* row = tile + c * (D + 4) + g * (D / 2);
  f32x16 S = f32_zero16();
#pragma unroll
  for (int s = 0; s < D / 2; s += 4) {
    const float4 a = *reinterpret_cast<const float4*>(row + s);
    S = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b[s], S, 0, 0, 0);
    S = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b[s + 1], S, 0, 0, 0);
    S = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b[s + 2], S, 0, 0, 0);
    S = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b[s + 3], S, 0, 0, 0);
  }
  return S;
}

// acc[dt][4j + i] (column c, element 32 dt + 8j + 4g + i) += sum over the
// tile's rows of row[element] * P(row, c)
template <int D>
NAMOH_DEV void f32_sum(f32x16 (&acc)[D / 32], const float* tile, const f32x16& P, int c, int g) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float* p = tile + (8 * (e >> 2) + 4 * g + (e & 3)) * (D + 4) + c;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[32 * dt], P[e], acc[dt], 0, 0, 0);
  }
}

// The same one row at a time, kept only in the columns that see the row
// (ok(row)): what a masked row holds does not reach the others.
template <int D, typename OK>
NAMOH_DEV void f32_sum_checked(f32x16 (&acc)[D / 32], const float* tile, const f32x16& P, int c, int g,
                               OK ok) {
#pragma unroll 1
  for (int row = 0; row < 32; ++row) {
    const bool mine = ((row >> 2) & 1) == g;    // this half of the wave holds the row's weights
    const float w = mine ? P[4 * (row >> 3) + (row & 3)] : 0.f;
    const bool keep = ok(row);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      const float x = mine ? tile[row * (D + 4) + 32 * dt + c] : 0.f;
      const f32x16 t = __builtin_amdgcn_mfma_f32_32x32x2f32(x, w, acc[dt], 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[dt][e] = keep ? t[e] : acc[dt][e];
    }
  }
}

template <int D>
NAMOH_DEV void f32_clear(f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) acc[dt] = f32_zero16();
}

// Row c of the wave's block from its accumulators (element 32 dt + 8j + 4g + i
// in acc[dt][4j + i]) to dst (16-byte stores).
template <int D>
NAMOH_DEV void f32_store_row(float* dst, const f32x16 (&acc)[D / 32], float f, int g) {
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<float4*>(dst + 32 * dt + 8 * j + 4 * g) =
          make_float4(acc[dt][4 * j] * f, acc[dt][4 * j + 1] * f, acc[dt][4 * j + 2] * f,
                      acc[dt][4 * j + 3] * f);
}

// Half a row (elements g D/2 .. ) times f into registers.
template <int D>
NAMOH_DEV void f32_half_row(float (&x)[D / 2], const float* row, float f, int g) {
#pragma unroll
  for (int s = 0; s < D / 2; s += 4) {
    const float4 v = *reinterpret_cast<const float4*>(row + g * (D / 2) + s);
    x[s] = v.x * f;
    x[s + 1] = v.y * f;
    x[s + 2] = v.z * f;
    x[s + 3] = v.w * f;
  }
}

// Staging of rows [r0, r0 + ROWS) of two packed [*, D] arrays (rows past n as
// zeros): load() into registers, store() from there into LDS; store() is true
// if one of the thread's values is not finite.
template <int D, int ROWS>
struct F32Stage {
  static constexpr int C4 = D / 4, PER = ROWS * C4 / kFThreads;
  float *t0, *t1;
  const float *x0, *x1;
  size_t a;
  int n, tid, r0;
  float4 v0[PER], v1[PER];
  NAMOH_DEV void load(int r) {
    r0 = r;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int u = tid + m * kFThreads, rr = u / C4, c4 = u - rr * C4;
      const size_t o = (a + min(r0 + rr, n - 1)) * D + 4 * c4;
      v0[m] = *reinterpret_cast<const float4*>(x0 + o);
      v1[m] = *reinterpret_cast<const float4*>(x1 + o);
    }
  }
  NAMOH_DEV bool store() {
    bool bad = false;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int u = tid + m * kFThreads, rr = u / C4, c4 = u - rr * C4;
      if (r0 + rr >= n) v0[m] = v1[m] = make_float4(0.f, 0.f, 0.f, 0.f);
      bad = bad || f32_bad4(v0[m]) || f32_bad4(v1[m]);
      *reinterpret_cast<float4*>(t0 + rr * (D + 4) + 4 * c4) = v0[m];
      *reinterpret_cast<float4*>(t1 + rr * (D + 4) + 4 * c4) = v1[m];
    }
    return bad;
  }
};

// Causal attention of the wave's query (row r of the segment, half row qf in
// log2 units) over the key tiles up to its own one: unnormalised output acc,
// running maximum m, and l, the sum over the lane's own keys (the two lanes of
// a query hold the two halves).  m starts at the lowest finite value: a tile
// whose scores are all -inf (a part's first one, say) weighs nothing and is not
// -inf - -inf = NaN.
template <int D, int QW, typename Stage>
NAMOH_DEV void f32_attend(f32x16 (&acc)[D / 32], float& m, float& l, const float (&qf)[D / 2], int r,
                          int qt, int part, bool active, int ntile, float* sk, float* sv, int c,
                          int g, Stage& stage) {
  using S = FShape<D, QW>;
  f32_clear<D>(acc);
  m = -FLT_MAX;
  l = 0.f;
  for (int t0 = 0; t0 < ntile; t0 += S::KS) {
    stage.load(32 * t0);
    __syncthreads();
    const bool bad = __syncthreads_or(stage.store());
    const int tile = t0 + part;
    if (active && tile <= qt) {
      f32x16 P = f32_scores<D>(sk + 32 * part * S::LD, qf, c, g);
      const int k0 = 32 * tile + 4 * g;
      if (tile == qt) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (k0 + 8 * (e >> 2) + (e & 3) > r) P[e] = -INFINITY;
      }
      float mx = P[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, P[e]);
      const float mn = fmaxf(m, pair_max32(mx));
      if (__any(mn > m)) {
        const float corr = exp2f(m - mn);
        l *= corr;
#pragma unroll
        for (int dt = 0; dt < S::DT; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[dt][e] *= corr;
        m = mn;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        P[e] = exp2f(P[e] - m);
        l += P[e];
      }
      const float* vt = sv + 32 * part * S::LD;
      if (__builtin_expect(bad && tile == qt, 0))
        f32_sum_checked<D>(acc, vt, P, c, g, [&](int row) { return 32 * tile + row <= r; });
      else
        f32_sum<D>(acc, vt, P, c, g);
    }
  }
}

// Partial results of the waves that split a block's tiles: rows
// [part][block row][D + 4] in LDS; their sum in part order.
template <int D, int QW>
NAMOH_DEV float4 f32_sum_parts(const float* buf, int row, int c4) {
  using S = FShape<D, QW>;
  float4 o = *reinterpret_cast<const float4*>(buf + row * S::LD + 4 * c4);
#pragma unroll
  for (int p = 1; p < S::KS; ++p) {
    const float4 x = *reinterpret_cast<const float4*>(buf + (S::BM * p + row) * S::LD + 4 * c4);
    o = make_float4(o.x + x.x, o.y + x.y, o.z + x.z, o.w + x.w);
  }
  return o;
}

// ---------------------------------------------------------------------------
// Forward: keys and values gathered by perm_token; keys (and queries) rotated
// by the cos/sin table as they are staged.
template <bool BF16>
NAMOH_DEV float4 f32_load4(const void* base, size_t i) {
  if constexpr (BF16) {
    const uint2 w = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(base) + i);
    return make_float4(lo_bf16(w.x), hi_bf16(w.x), lo_bf16(w.y), hi_bf16(w.y));
  } else {
    return *reinterpret_cast<const float4*>(static_cast<const float*>(base) + i);
  }
}

// (x1, x2) = elements j0 .. j0 + 3 and their partners; u, w = (cos, sin) x 4
NAMOH_DEV void f32_rope4(float4& x1, float4& x2, const float4 u, const float4 w) {
  const float4 a = x1, b = x2;
  x1 = make_float4(a.x * u.x - b.x * u.y, a.y * u.z - b.y * u.w, a.z * w.x - b.z * w.y, a.w * w.z - b.w * w.w);
  x2 = make_float4(b.x * u.x + a.x * u.y, b.y * u.z + a.y * u.w, b.z * w.x + a.z * w.y, b.w * w.z + a.w * w.w);
}

// Staging of rows [r0, r0 + ROWS) of a segment's keys (rotated) and values,
// gathered by token; the tokens of the tiles after the next are read ahead.
template <int D, bool BF16, int ROWS>
struct F32Gather {
  static constexpr int G = D / 8, PER = ROWS * G / kFThreads;
  float *sk, *sv;
  const void *k, *v;
  const float2* table;
  const int32_t* perm;   // of the segment
  size_t head;
  int n, T, rope_mode, tid, r0;
  int tok[PER];
  float4 k1[PER], k2[PER], v1[PER], v2[PER], cu[PER], cw[PER];
  NAMOH_DEV void tokens(int r) {
#pragma unroll
    for (int m = 0; m < PER; ++m)
      tok[m] = static_cast<int>(min(static_cast<unsigned>(perm[min(r + (tid + m * kFThreads) / G, n - 1)]),
                                    static_cast<unsigned>(T - 1)));
  }
  NAMOH_DEV void load(int r) {
    r0 = r;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int u = tid + m * kFThreads, rr = u / G, j0 = 4 * (u - rr * G);
      const size_t o = (head + tok[m]) * D + j0;
      k1[m] = f32_load4<BF16>(k, o);
      k2[m] = f32_load4<BF16>(k, o + D / 2);
      v1[m] = f32_load4<BF16>(v, o);
      v2[m] = f32_load4<BF16>(v, o + D / 2);
      // (without rotation the table is not written; its rows are then unused)
      const float4* cs = reinterpret_cast<const float4*>(
          table + static_cast<size_t>(rope_mode == 0 ? min(r0 + rr, n - 1) : tok[m]) * (D / 2) + j0);
      cu[m] = cs[0];
      cw[m] = cs[1];
    }
    tokens(r + ROWS);
  }
  NAMOH_DEV bool store() {
    bool bad = false;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int u = tid + m * kFThreads, rr = u / G, j0 = 4 * (u - rr * G);
      if (rope_mode != 2) f32_rope4(k1[m], k2[m], cu[m], cw[m]);
      if (r0 + rr >= n) k1[m] = k2[m] = v1[m] = v2[m] = make_float4(0.f, 0.f, 0.f, 0.f);
      bad = bad || f32_bad4(v1[m]) || f32_bad4(v2[m]);
      float* ko = sk + rr * (D + 4) + j0;
      float* vo = sv + rr * (D + 4) + j0;
      *reinterpret_cast<float4*>(ko) = k1[m];
      *reinterpret_cast<float4*>(ko + D / 2) = k2[m];
      *reinterpret_cast<float4*>(vo) = v1[m];
      *reinterpret_cast<float4*>(vo + D / 2) = v2[m];
    }
    return bad;
  }
};

template <int D, bool BF16, int QW>
__global__ __launch_bounds__(kFThreads, (FShape<D, QW>::MINB)) void k_f32_attn(
    const void* __restrict__ q, const void* __restrict__ k, const void* __restrict__ v,
    const float2* __restrict__ table, const int32_t* __restrict__ seg_offsets,
    const int32_t* __restrict__ perm_token, int BH, int T, int Nr, int rope_mode, float scale_log2,
    float* __restrict__ hout) {
  using S = FShape<D, QW>;
  constexpr int HD = S::HD, LD = S::LD;
  __shared__ __attribute__((aligned(16))) float buf[S::BUF];
  __shared__ float2 s_ml[S::KS * S::BM];
  float* sk = buf;
  float* sv = buf + S::ROWS * LD;
  FBlock w;
  if (!f32_block<S::BM>(seg_offsets, BH, T, Nr, reinterpret_cast<int*>(buf), w)) return;
  const int tid = thread_x(), lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c = lane & 31, g = lane >> 5;
  const int qw = wave % QW, part = wave / QW;
  const int qt = w.r0 / 32 + qw, r = 32 * qt + c;
  const bool active = 32 * qt < w.n;
  const size_t head = static_cast<size_t>(w.s) * T;
  F32Gather<D, BF16, S::ROWS> stage{sk, sv, k, v, table, perm_token + w.a, head, w.n, T, rope_mode, tid};
  const int rr = min(r, w.n - 1);
  const int t = static_cast<int>(min(static_cast<unsigned>(perm_token[w.a + rr]), static_cast<unsigned>(T - 1)));
  stage.tokens(0);
  float qf[HD];
  {
    const float2* cs = table + static_cast<size_t>(rope_mode == 0 ? rr : t) * HD;
#pragma unroll
    for (int s = 0; s < HD; s += 4) {
      float4 x1 = f32_load4<BF16>(q, (head + t) * D + s), x2 = f32_load4<BF16>(q, (head + t) * D + HD + s);
      if (rope_mode != 2)
        f32_rope4(x1, x2, reinterpret_cast<const float4*>(cs + s)[0],
                  reinterpret_cast<const float4*>(cs + s)[1]);
      const float4 x = g ? x2 : x1;
      qf[s] = x.x * scale_log2;
      qf[s + 1] = x.y * scale_log2;
      qf[s + 2] = x.z * scale_log2;
      qf[s + 3] = x.w * scale_log2;
    }
  }
  f32x16 acc[S::DT];
  float m, l;
  const int ntile = min((w.n + 31) / 32, w.r0 / 32 + QW);
  f32_attend<D, QW>(acc, m, l, qf, r, qt, part, active, ntile, sk, sv, c, g, stage);
  l = pair_sum32(l);
  float* hrow = hout + static_cast<size_t>(w.a) * D;
  {
    __syncthreads();
    f32_store_row<D>(buf + (S::BM * part + 32 * qw + c) * LD, acc, 1.f, g);
    if (g == 0) s_ml[S::BM * part + 32 * qw + c] = make_float2(m, l);
    __syncthreads();
#pragma unroll
    for (int u = tid; u < S::BM * (D / 4); u += kFThreads) {
      const int qi = u / (D / 4), c4 = u - qi * (D / 4);
      if (w.r0 + qi >= w.n) continue;
      float M = s_ml[qi].x, L = 0.f;
#pragma unroll
      for (int p = 1; p < S::KS; ++p) M = fmaxf(M, s_ml[S::BM * p + qi].x);
      float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int p = 0; p < S::KS; ++p) {
        const float2 ml = s_ml[S::BM * p + qi];
        const float f = exp2f(ml.x - M);
        const float4 x = *reinterpret_cast<const float4*>(buf + (S::BM * p + qi) * LD + 4 * c4);
        L = fmaf(f, ml.y, L);
        o.x = fmaf(f, x.x, o.x);
        o.y = fmaf(f, x.y, o.y);
        o.z = fmaf(f, x.z, o.z);
        o.w = fmaf(f, x.w, o.w);
      }
      const float inv = 1.f / L;
      *reinterpret_cast<float4*>(hrow + static_cast<size_t>(w.r0 + qi) * D + 4 * c4) =
          make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
    }
  }
}

// ---------------------------------------------------------------------------
// Backward, on packed float32 rows (k_bwd_gather).  Query side: one pass for
// the log-sum-exp (log2 units) and O, from which D = <dO, O> and the gate
// gradient, and one for dQ~ = scale sum_j P_ij (dO_i . v_j - D_i) k~_j.
template <int D, int QW>
__global__ __launch_bounds__(kFThreads, (FShape<D, QW>::MINB)) void k_f32_bwd_q(
    const float* __restrict__ Qr, const float* __restrict__ Kr, const float* __restrict__ Vp,
    const float* __restrict__ dOp, const float* __restrict__ dout,
    const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ perm_token, int BH, int H,
    int T, int Nr, float scale, float* __restrict__ lse, float* __restrict__ Dr,
    float* __restrict__ dgp, float* __restrict__ dQr) {
  using S = FShape<D, QW>;
  constexpr int HD = S::HD, LD = S::LD;
  __shared__ __attribute__((aligned(16))) float buf[S::BUF];
  __shared__ float2 s_ml[S::KS * S::BM], s_stat[S::BM];
  float* sk = buf;
  float* sv = buf + S::ROWS * LD;
  FBlock w;
  if (!f32_block<S::BM>(seg_offsets, BH, T, Nr, reinterpret_cast<int*>(buf), w)) return;
  const int tid = thread_x(), lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c = lane & 31, g = lane >> 5;
  const int qw = wave % QW, part = wave / QW;
  const int qt = w.r0 / 32 + qw, r = 32 * qt + c;
  const bool active = 32 * qt < w.n;
  const size_t row = static_cast<size_t>(w.a) + min(r, w.n - 1);
  const int b = w.s / H;
  auto dout_row = [&](size_t packed) {
    const int t = min(static_cast<unsigned>(perm_token[packed]), static_cast<unsigned>(T - 1));
    return dout + (static_cast<size_t>(b) * T + t) * D;
  };
  F32Stage<D, S::ROWS> stage{sk, sv, Kr, Vp, static_cast<size_t>(w.a), w.n, tid};
  float qf[HD];
  f32_half_row<D>(qf, Qr + row * D, scale * 1.4426950408889634f, g);
  f32x16 acc[S::DT];
  float m, l;
  const int ntile = min((w.n + 31) / 32, w.r0 / 32 + QW);
  f32_attend<D, QW>(acc, m, l, qf, r, qt, part, active, ntile, sk, sv, c, g, stage);
  l = pair_sum32(l);
  float lse2, dsum;
  {
    __syncthreads();
    f32_store_row<D>(buf + (S::BM * part + 32 * qw + c) * LD, acc, 1.f, g);
    if (g == 0) s_ml[S::BM * part + 32 * qw + c] = make_float2(m, l);
    __syncthreads();
    // eight threads per query
#pragma unroll
    for (int u = tid; u < 8 * S::BM; u += kFThreads) {
      const int qi = u / 8, e0 = (u & 7) * (D / 8);
      const size_t qrow = static_cast<size_t>(w.a) + min(w.r0 + qi, w.n - 1);
      const float* dorow = dOp + qrow * D + e0;
      const float* dtrow = dout_row(qrow) + e0;
      float M = s_ml[qi].x, Ls = 0.f, f[S::KS];
#pragma unroll
      for (int p = 1; p < S::KS; ++p) M = fmaxf(M, s_ml[S::BM * p + qi].x);
#pragma unroll
      for (int p = 0; p < S::KS; ++p) {
        f[p] = exp2f(s_ml[S::BM * p + qi].x - M);
        Ls = fmaf(f[p], s_ml[S::BM * p + qi].y, Ls);
      }
      const float inv = 1.f / Ls;
      float gs = 0.f, ds = 0.f;
#pragma unroll
      for (int e = 0; e < D / 8; e += 4) {
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int p = 0; p < S::KS; ++p) {
          const float4 x = *reinterpret_cast<const float4*>(buf + (S::BM * p + qi) * LD + e0 + e);
          o.x = fmaf(f[p], x.x, o.x);
          o.y = fmaf(f[p], x.y, o.y);
          o.z = fmaf(f[p], x.z, o.z);
          o.w = fmaf(f[p], x.w, o.w);
        }
        const float4 x = *reinterpret_cast<const float4*>(dorow + e);
        const float4 y = *reinterpret_cast<const float4*>(dtrow + e);
        ds = fmaf(x.w, o.w, fmaf(x.z, o.z, fmaf(x.y, o.y, fmaf(x.x, o.x, ds))));
        gs = fmaf(y.w, o.w, fmaf(y.z, o.z, fmaf(y.y, o.y, fmaf(y.x, o.x, gs))));
      }
      ds = group_sum<8>(ds) * inv;
      gs = group_sum<8>(gs) * inv;
      if ((u & 7) == 0) {
        const float q2 = M + log2f(Ls);
        s_stat[qi] = make_float2(q2, ds);
        if (w.r0 + qi < w.n) {
          lse[qrow] = q2;
          Dr[qrow] = ds;
          dgp[qrow] = gs;
        }
      }
    }
    __syncthreads();
    lse2 = s_stat[32 * qw + c].x;
    dsum = s_stat[32 * qw + c].y;
  }
  // ---- second pass ----------------------------------------------------------
  float dof[HD];
  f32_half_row<D>(dof, dOp + row * D, 1.f, g);
  f32_clear<D>(acc);
  for (int t0 = 0; t0 < ntile; t0 += S::KS) {
    stage.load(32 * t0);
    __syncthreads();
    const bool bad = __syncthreads_or(stage.store());
    const int tile = t0 + part;
    if (active && tile <= qt) {
      const float* ktile = sk + 32 * part * LD;
      f32x16 P = f32_scores<D>(ktile, qf, c, g);
      const f32x16 dP = f32_scores<D>(sv + 32 * part * LD, dof, c, g);
      const int k0 = 32 * tile + 4 * g;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        P[e] = exp2f(P[e] - lse2) * (dP[e] - dsum) * scale;
        if (tile == qt && k0 + 8 * (e >> 2) + (e & 3) > r) P[e] = 0.f;
      }
      if (__builtin_expect(bad && tile == qt, 0))
        f32_sum_checked<D>(acc, ktile, P, c, g, [&](int kr) { return 32 * tile + kr <= r; });
      else
        f32_sum<D>(acc, ktile, P, c, g);
    }
  }
  {
    __syncthreads();
    f32_store_row<D>(buf + (S::BM * part + 32 * qw + c) * LD, acc, 1.f, g);
    __syncthreads();
#pragma unroll
    for (int u = tid; u < S::BM * (D / 4); u += kFThreads) {
      const int qi = u / (D / 4), c4 = u - qi * (D / 4);
      const float4 o = f32_sum_parts<D, QW>(buf, qi, c4);
      if (w.r0 + qi < w.n)
        *reinterpret_cast<float4*>(dQr + (static_cast<size_t>(w.a) + w.r0 + qi) * D + 4 * c4) = o;
    }
  }
}

// ---------------------------------------------------------------------------
// Key side: the wave's 32 keys against the query tiles from their own one on,
// dV_j = sum_{i >= j} P_ij dO_i and dK~_j = scale sum_{i >= j} P_ij (dO_i . v_j
// - D_i) q~_i in one pass.
template <int D, int QW>
__global__ __launch_bounds__(kFThreads, (FShape<D, QW>::MINB)) void k_f32_bwd_kv(
    const float* __restrict__ Qr, const float* __restrict__ Kr, const float* __restrict__ Vp,
    const float* __restrict__ dOp, const float* __restrict__ lse, const float* __restrict__ Dr,
    const int32_t* __restrict__ seg_offsets, int BH, int T, int Nr, float scale,
    float* __restrict__ dKr, float* __restrict__ dVp) {
  using S = FShape<D, QW>;
  constexpr int HD = S::HD, LD = S::LD;
  __shared__ __attribute__((aligned(16))) float buf[S::BUF];
  __shared__ __attribute__((aligned(16))) float s_lse[S::ROWS], s_D[S::ROWS];
  float* sq = buf;
  float* sdo = buf + S::ROWS * LD;
  FBlock w;
  if (!f32_block<S::BM>(seg_offsets, BH, T, Nr, reinterpret_cast<int*>(buf), w)) return;
  const int tid = thread_x(), lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c = lane & 31, g = lane >> 5;
  const int kw = wave % QW, part = wave / QW;
  const int kt0 = w.r0 / 32 + kw, j = 32 * kt0 + c;
  const size_t row = static_cast<size_t>(w.a) + min(j, w.n - 1);
  F32Stage<D, S::ROWS> stage{sq, sdo, Qr, dOp, static_cast<size_t>(w.a), w.n, tid};
  float kf[HD], vf[HD];
  f32_half_row<D>(kf, Kr + row * D, scale * 1.4426950408889634f, g);
  f32_half_row<D>(vf, Vp + row * D, 1.f, g);
  f32x16 aK[S::DT], aV[S::DT];
  f32_clear<D>(aK);
  f32_clear<D>(aV);
  const int ntile = (w.n + 31) / 32;
  for (int t0 = w.r0 / 32; t0 < ntile; t0 += S::KS) {
    stage.load(32 * t0);
    const size_t srow = static_cast<size_t>(w.a) + min(32 * t0 + tid % S::ROWS, w.n - 1);
    const float nl = lse[srow], nd = Dr[srow];
    __syncthreads();
    if (tid < S::ROWS) {
      s_lse[tid] = nl;
      s_D[tid] = nd;
    }
    const bool bad = __syncthreads_or(stage.store());
    const int lt = part, tile = t0 + part;
    if (tile >= kt0 && tile < ntile) {
      const float* qtile = sq + 32 * lt * LD;
      const float* dtile = sdo + 32 * lt * LD;
      f32x16 P = f32_scores<D>(qtile, kf, c, g);
      f32x16 dS = f32_scores<D>(dtile, vf, c, g);
      const bool edge = tile == kt0 || tile == ntile - 1;
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const float4 ls = *reinterpret_cast<const float4*>(s_lse + 32 * lt + 8 * e4 + 4 * g);
        const float4 dd = *reinterpret_cast<const float4*>(s_D + 32 * lt + 8 * e4 + 4 * g);
        const float la[4] = {ls.x, ls.y, ls.z, ls.w}, da[4] = {dd.x, dd.y, dd.z, dd.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = 4 * e4 + i, qr = 32 * tile + 8 * e4 + 4 * g + i;
          const float p = exp2f(P[e] - la[i]);
          const bool off = edge && (qr < j || qr >= w.n);
          P[e] = off ? 0.f : p;
          dS[e] = off ? 0.f : p * (dS[e] - da[i]) * scale;
        }
      }
      if (__builtin_expect(bad && tile == kt0, 0)) {
        // (rows past n are staged as zeros)
        auto ok = [&](int qr) { return 32 * tile + qr >= j; };
        f32_sum_checked<D>(aV, dtile, P, c, g, ok);
        f32_sum_checked<D>(aK, qtile, dS, c, g, ok);
      } else {
        f32_sum<D>(aV, dtile, P, c, g);
        f32_sum<D>(aK, qtile, dS, c, g);
      }
    }
  }
  {
    __syncthreads();
    f32_store_row<D>(buf + (S::BM * part + 32 * kw + c) * LD, aK, 1.f, g);
    f32_store_row<D>(buf + (128 + S::BM * part + 32 * kw + c) * LD, aV, 1.f, g);
    __syncthreads();
#pragma unroll
    for (int u = tid; u < 2 * S::BM * (D / 4); u += kFThreads) {
      const int which = u / (S::BM * (D / 4)), x = u - which * S::BM * (D / 4);
      const int ki = x / (D / 4), c4 = x - ki * (D / 4);
      const float4 o = f32_sum_parts<D, QW>(buf + which * 128 * LD, ki, c4);
      if (w.r0 + ki < w.n)
        *reinterpret_cast<float4*>((which ? dVp : dKr) + (static_cast<size_t>(w.a) + w.r0 + ki) * D + 4 * c4) = o;
    }
  }
}

// ---------------------------------------------------------------------------
// One 32-row block per workgroup gives the most workgroups and the shortest
// serial chains; at d = 128 (one workgroup per compute unit by registers)
// 64-row blocks halve the staging per product: B 2, T 2048, H 32, K 8 forward
// 212 -> 151 us, backward 879 -> 675 us.  At d <= 64 they gain 3 to 14 % with
// many balanced rows and lose as much with few or skewed ones (B 1, T 2048,
// H 8, K 4, skewed: 93 -> 137, 323 -> 478 us); 128-row blocks lose more.
constexpr int f32_qw(int D) { return D == 128 ? 2 : 1; }

// Many short segments (d = 64, forward): a workgroup per 128 rows whose waves
// take a query block each of one tile after the other, instead of one query
// block with the tiles split over the waves: with a few rows a segment three
// of four staged tiles were empty.  Forward in us, split tiles -> query blocks,
// 64 heads, 4 selected (zipf: skewed routing): 40 sequences of 79 tokens 64 -> 45,
// 200 of 60 (2 selected) 240 -> 157, 16 of 200 46 -> 31, zipf, 32 heads 40 -> 38; 16
// of 300 48 -> 34, but zipf 55 -> 72, 16 of 600, zipf 99 -> 118: long segments want
// the split.  16 heads x 16 sequences, 1 selected, 100 tokens, zipf 21 -> 22.5.
static bool f32_short(int d, int BH, int T) { return d == 64 && BH >= 512 && T <= 256; }

template <int BM>
static dim3 f32_grid(int Nr, int BH) { return dim3(static_cast<unsigned>(Nr / BM + BH + 1)); }

template <int D, bool BF16, int QW = f32_qw(D)>
static void run_f32_attn(const void* q, const void* k, const void* v, const float2* table,
                         const int32_t* seg_offsets, const int32_t* perm_token, int BH, int T,
                         int Nr, int rope_mode, float scale_log2, float* hout, hipStream_t st) {
  launch_k("attn", k_f32_attn<D, BF16, QW>, f32_grid<32 * QW>(Nr, BH), dim3(kFThreads), st, q, k, v,
           table, seg_offsets, perm_token, BH, T, Nr, rope_mode, scale_log2, hout);
}

hipError_t launch_f32_attn(const void* q, const void* k, const void* v, int dtype, int d,
                           const float2* table, const int32_t* seg_offsets,
                           const int32_t* perm_token, int BH, int T, int Nr, int rope_mode,
                           float scale, float* hout, hipStream_t st) {
  const float sl2 = scale * 1.4426950408889634f;
#define NAMOH_F32(DD, BF) \
  run_f32_attn<DD, BF>(q, k, v, table, seg_offsets, perm_token, BH, T, Nr, rope_mode, sl2, hout, st)
  if (dtype == 1) {
    if (d != 32) return hipErrorInvalidValue;   // (the wider bf16 heads run on bf16 products)
    NAMOH_F32(32, true);
  } else if (d == 32) {
    NAMOH_F32(32, false);
  } else if (f32_short(d, BH, T)) {
    run_f32_attn<64, false, 4>(q, k, v, table, seg_offsets, perm_token, BH, T, Nr, rope_mode, sl2, hout, st);
  } else if (d == 64) {
    NAMOH_F32(64, false);
  } else {
    NAMOH_F32(128, false);
  }
#undef NAMOH_F32
  return hipGetLastError();
}

template <int D, int QW>
static hipError_t run_f32_bwd(const F32BwdRows& w, const float* dout, const int32_t* seg_offsets,
                              const int32_t* perm_token, int BH, int H, int T, int Nr, float scale,
                              hipStream_t st) {
  const dim3 grid = f32_grid<32 * QW>(Nr, BH);
  launch_k("bwd_dq", k_f32_bwd_q<D, QW>, grid, dim3(kFThreads), st, w.Qr, w.Kr, w.Vp, w.dOp, dout,
           seg_offsets, perm_token, BH, H, T, Nr, scale, w.lse, w.Dr, w.dgp, w.dQr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_k("bwd_dkdv", k_f32_bwd_kv<D, QW>, grid, dim3(kFThreads), st, w.Qr, w.Kr, w.Vp, w.dOp,
           w.lse, w.Dr, seg_offsets, BH, T, Nr, scale, w.dKr, w.dVp);
  return hipGetLastError();
}

hipError_t launch_f32_bwd(const F32BwdRows& w, const float* dout, int d, const int32_t* seg_offsets,
                          const int32_t* perm_token, int BH, int H, int T, int Nr, float scale,
                          hipStream_t st) {
#define NAMOH_F32B(DD)                                                                            \
  return run_f32_bwd<DD, f32_qw(DD)>(w, dout, seg_offsets, perm_token, BH, H, T, Nr, scale, st)
  if (d == 32) NAMOH_F32B(32);
  if (d == 64) NAMOH_F32B(64);
  NAMOH_F32B(128);
#undef NAMOH_F32B
}

}  // namespace namoh
