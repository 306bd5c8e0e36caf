// One decoding step: route the new token, append it to its selected heads'
// caches, attend over each selected head's history, gate and combine.
//
// Sec. 3.1: routing uses only the current token, so incremental decoding is
// the same causal computation as prefill; the new token's rank in head h is
// that head's current length n (Eq. namoh-head-rope) and it attends to itself.
// Sec. 3.2: only the active heads' queries run, and only their caches are read
// or written.  Eq. namoh-kv-cost: the step reads sum over the selected heads
// of (n + 1) cached rows, which makes it HBM-bound.
//
//   k_decode_attn          split over chunks (up to 512 rows) of every selected head's
//                          history.  Every workgroup routes its sequence's
//                          token itself; the one whose chunk the new token
//                          ends rotates its key (angles in double) and writes
//                          the cache row.  16-byte coalesced loads of K and V
//                          rows (a row spans d*esize/16 lanes), several rows
//                          in flight per lane, online softmax in exp2 domain,
//                          one (max, sum, acc[d]) partial per chunk.
//   k_decode_route         the routing, the append and the queries' rotation as
//                          a launch before it, where many sequences have short
//                          histories.
//   k_decode_combine       merges the chunk partials of each head by
//                          log-sum-exp, sums the gated head outputs and
//                          advances the cache lengths.
//   k_prefill_cache        the prefill -> decode hand-off: every packed
//                          prompt row (segment b*H + h, rank r, token t)
//                          writes its rotated key and its value to row r of
//                          head h's caches; cache_len = the segment lengths.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "launch.h"

namespace namoh {

constexpr int kDecChunk = 512;   // cached rows per attention workgroup, at most
constexpr int kDecUnroll = 8;    // rows per lane in flight

// Rows per chunk of a history of L rows with nchunk chunks to spend (512 rows
// each hold the cache's capacity).  With few workgroups in the launch (`fine`)
// a short history is spread over all of them, in multiples of 64 KB of keys
// and values in bf16 (128 rows at d = 128, a 32-row block per wave of the
// matrix-core kernel): 8 sequences, 4 of 16 groups of 4 heads, 512 rows each,
// d 128: 16.3 -> 9.7 us.  Smaller chunks only add prologues and partials: 4
// sequences, 8 heads of 900 rows, d 64, in 256 rows 9.9 us, in 128 rows 10.8;
// and so do they with the chip full anyway (64 sequences x 8 heads).
constexpr int dec_min_rows(int d) { return 16384 / d; }
template <int D>
NAMOH_DEV int dec_chunk_rows(int L, int nchunk, int fine) {
  constexpr int R = dec_min_rows(D);
  if (!fine) return kDecChunk;
  return min(kDecChunk, ((L + nchunk - 1) / nchunk + R - 1) / R * R);
}
constexpr long kDecFineGroups = 1024;   // workgroups of a launch: four per compute unit

template <bool BF16>
NAMOH_DEV float ld_elem(const void* p, size_t i) {
  if constexpr (BF16) return bf16_to_f32(static_cast<const uint16_t*>(p)[i]);
  else return static_cast<const float*>(p)[i];
}

template <bool BF16>
NAMOH_DEV void st_elem(void* p, size_t i, float x) {
  if constexpr (BF16) static_cast<uint16_t*>(p)[i] = f32_to_bf16(x);
  else static_cast<float*>(p)[i] = x;
}

// What a step's attention workgroups need besides the partials.  Routed heads:
// logits .. topk_idx; shared heads (SHARED): window, every head selected.
struct DecStep {
  const float *logits, *bias;
  const void *q, *k, *v;
  void *k_cache, *v_cache;
  const int32_t *cache_len, *seq_pos;
  int H, K;                // heads, selected heads (shared: Hs, Hs)
  long cap;
  double log_base;
  int rope_mode, gate_mode, window;
  float qscale;
  int32_t* topk_idx;
  float* gates;
  int32_t* dev_status;
  int nchunk, fine;        // chunks per head; dec_chunk_rows
  float *part_acc, *part_ml;
};
// And what k_decode_route leaves for them (a kernel without it has the smaller
// arguments: the 16 bytes cost 0.4 us of host time a call).
struct DecAhead : DecStep {
  int32_t* ahead;          // history (or -1) of every selected head
  float* qrot;             // its rotated, scaled queries [G, D]
};
template <bool AHEAD>
using DecArgs = std::conditional_t<AHEAD, DecAhead, DecStep>;

// The head a workgroup (selected head bk, chunk) works on: its history before
// the new token (rows of it that are read), the first one's ring row, and the
// new token's row and rotation position.
struct DecHead {
  size_t bh;      // b * H + head
  int hist, ring0, chunk;  // chunk: rows per chunk
  long slot, pos;
};

// Every wave finds its workgroup's head by itself (lane = head: one round of
// loads, then the rank of every head under (logit desc, index asc) by H
// comparisons), so no launch of its own is needed for the routing.  A step of
// one sequence with short histories is a chain of latencies: routing and
// append, attention and combine as three kernels took 5.8 + 5.6 + 3.0 us and
// two more gaps, now 7.6 + 2.1 us (32 heads, 8 selected, 300 rows, d 64); with
// 64 sequences 10.3 + 185.3 + 7.4, now 189 + 6.6 us.  The
// workgroups of chunk 0 write topk_idx, gates and the status.  False: nothing
// to do (no such head, a full cache, a chunk past the history).
template <int D, bool SHARED>
NAMOH_DEV bool dec_head(const DecStep& a, int bk, int chunk, DecHead& o) {
  const int lane = thread_x() % 64;
  const int b = bk / a.K, kk = bk - (bk / a.K) * a.K;
  int n;
  if constexpr (SHARED) {
    n = a.cache_len[b];
    const bool over = n < 0 || (a.window == 0 && n >= a.cap);
    if (over) {
      if (chunk == 0 && thread_x() == 0 && a.dev_status) a.dev_status[0] = 1;
      return false;
    }
    const int hist = a.window > 0 ? min(n, a.window - 1) : n;
    o.chunk = dec_chunk_rows<D>(hist + 1, a.nchunk, a.fine);
    // most workgroups of a cache far larger than its histories end here, before
    // the divisions
    if (chunk * o.chunk > hist) return false;
    o.bh = bk;
    o.hist = hist;
    const uint32_t cap = static_cast<uint32_t>(a.cap);
    o.ring0 = static_cast<int>(static_cast<uint32_t>(n - hist) % cap);
    o.slot = static_cast<uint32_t>(n) % cap;
    o.pos = n;
    return true;
  } else {
    const bool real = lane < a.H;
    const size_t bl = static_cast<size_t>(b) * a.H + min(lane, a.H - 1);
    const float l = real ? a.logits[bl] : 0.f;
    const int len = a.cache_len[bl];
    // selection key: the logit, or with loss-free balancing biases the score
    // float(a + b) with the affinity a = softmax of the logits in double
    // (App. "Auxiliary-Loss-Free Balancing", Eq. namoh-biased-routing)
    float key = l, aff = 0.f;
    if (a.bias != nullptr) {
      float mx = real ? l : -INFINITY;
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s));
      const double ex = real ? exp(static_cast<double>(l) - static_cast<double>(mx)) : 0.0;
      double z = ex;
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) z += __shfl_xor(z, s);
      const double af = ex / z;
      aff = static_cast<float>(af);
      key = real ? static_cast<float>(af + static_cast<double>(a.bias[min(lane, a.H - 1)])) : 0.f;
    }
    // ranks below `need` (the workgroup that writes the selection: all K): the
    // maximum of what is left, lowest index first, `need` times over, or H
    // comparisons where those are fewer instructions (or a key is NaN).  With
    // many workgroups the VALU is the limit, with few this chain (32 heads, 8
    // selected, d 64, comparisons -> maxima: 945 sequences of 24 rows 61 -> 56 us a
    // step, one of 300 rows 10.6 -> 9.7)
    const int need = kk == 0 && chunk == 0 ? a.K : kk + 1;
    int rank = a.H;
    if (5 * need <= 2 * a.H && __ballot(real && key != key) == 0) {
      const uint32_t u = __float_as_uint(key + 0.f);   // (-0 and 0 are equal)
      int left = real ? static_cast<int>(u ^ (static_cast<int>(u) < 0 ? 0x7FFFFFFFu : 0u)) : INT32_MIN;
      for (int r = 0; r < need; ++r) {
        const uint64_t at = __ballot(left == wave_max_i(left));
        if (lane == __ffsll(static_cast<long long>(at)) - 1) {
          rank = r;
          left = INT32_MIN;
        }
      }
    } else {
      rank = 0;
      for (int j = 0; j < a.H; ++j) {
        const float kj = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(key), j));
        rank += (kj > key) || (kj == key && j < lane);
      }
    }
    const bool sel = real && rank < a.K;
    if (kk == 0 && chunk == 0) {
      const uint64_t first = __ballot(real && rank == 0);
      const float lmax = __shfl(l, first == 0 ? 0 : __ffsll(static_cast<long long>(first)) - 1);
      const float e_sel = sel ? expf(l - lmax) : 0.f;
      float e_den = a.gate_mode == 1 ? (real ? expf(l - lmax) : 0.f) : e_sel;
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) e_den += __shfl_xor(e_den, s);
      if (sel && thread_x() < 64) {
        a.topk_idx[static_cast<size_t>(b) * a.K + rank] = lane;
        a.gates[static_cast<size_t>(b) * a.K + rank] = a.bias != nullptr ? aff : e_sel / e_den;
      }
    }
    const uint64_t mk = __ballot(sel && rank == kk);
    if (mk == 0) {  // only reachable with NaN logits (outside the contract)
      if (chunk == 0 && thread_x() == 0) {
        a.topk_idx[bk] = -1;
        if (a.dev_status) a.dev_status[0] = 2;
      }
      return false;
    }
    const int h = __ffsll(static_cast<long long>(mk)) - 1;
    n = __builtin_amdgcn_readlane(len, h);
    if (n < 0 || n >= a.cap) {
      if (chunk == 0 && thread_x() == 0 && a.dev_status) a.dev_status[0] = 1;
      return false;
    }
    o.bh = static_cast<size_t>(b) * a.H + h;
    o.hist = n;
    o.ring0 = 0;
    o.slot = n;
    o.pos = a.rope_mode == 0 ? n : (a.rope_mode == 1 ? a.seq_pos[b] : 0);
  }
  o.chunk = dec_chunk_rows<D>(o.hist + 1, a.nchunk, a.fine);
  return chunk * o.chunk <= o.hist;
}

// (cos, sin) of the new token's angles into s_cs, and in the workgroup whose
// chunk ends with it (`owner`) its rotated key and its value: into the caches
// and into s_new (key, then value).  Thread j < D / 2 takes pair j.
template <int D, bool BF16>
NAMOH_DEV void dec_new_token(const DecStep& a, const DecHead& o, bool owner, float2* s_cs, void* s_new) {
  const int j = thread_x();
  if (j >= D / 2) return;
  const size_t src = o.bh * D;
  float k1 = 0.f, k2 = 0.f, v1 = 0.f, v2 = 0.f;
  if (owner) {
    k1 = ld_elem<BF16>(a.k, src + j);
    k2 = ld_elem<BF16>(a.k, src + j + D / 2);
    v1 = ld_elem<BF16>(a.v, src + j);
    v2 = ld_elem<BF16>(a.v, src + j + D / 2);
  }
  float2 w = make_float2(1.f, 0.f);
  if (a.rope_mode != 2)
    w = rope_cos_sin(static_cast<double>(o.pos) * exp(-(2.0 * j / D) * a.log_base));
  s_cs[j] = w;
  if (owner) {
    const float r1 = k1 * w.x - k2 * w.y, r2 = k2 * w.x + k1 * w.y;
    const size_t dst = (o.bh * a.cap + o.slot) * D;
    st_elem<BF16>(a.k_cache, dst + j, r1);
    st_elem<BF16>(a.k_cache, dst + j + D / 2, r2);
    st_elem<BF16>(a.v_cache, dst + j, v1);
    st_elem<BF16>(a.v_cache, dst + j + D / 2, v2);
    st_elem<BF16>(s_new, j, r1);
    st_elem<BF16>(s_new, j + D / 2, r2);
    st_elem<BF16>(s_new, D + j, v1);
    st_elem<BF16>(s_new, D + j + D / 2, v2);
  }
}

template <bool BF16>
NAMOH_DEV void dec_unpack(const u32x4 x, float* f) {
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (BF16) {
      f[2 * e] = lo_bf16(w[e]);
      f[2 * e + 1] = hi_bf16(w[e]);
    } else {
      f[e] = __uint_as_float(w[e]);
    }
  }
}

// The routing, the append and the queries' rotation as a launch of their own
// (one wave per selected head, G query heads each), for launches of many short
// chunks: see dec_route_ahead.
template <int D, bool BF16>
__global__ __launch_bounds__(64) void k_decode_route(const DecAhead a, int G) {
  __shared__ float2 s_cs[D / 2];
  __shared__ u32x4 s_new[2 * D * (BF16 ? 2 : 4) / 16];
  const int bk = block_x(), j = thread_x();
  DecHead hd;
  const bool ok = dec_head<D, false>(a, bk, 0, hd);
  if (j == 0) a.ahead[bk] = ok ? hd.hist : -1;
  if (!ok) return;
  dec_new_token<D, BF16>(a, hd, true, s_cs, s_new);
  if (j >= D / 2) return;
  const float2 w = s_cs[j];   // (written by this thread)
  for (int u = 0; u < G; ++u) {
    const size_t src = (hd.bh * G + u) * D + j, dst = (static_cast<size_t>(bk) * G + u) * D + j;
    const float q1 = ld_elem<BF16>(a.q, src), q2 = ld_elem<BF16>(a.q, src + D / 2);
    a.qrot[dst] = (q1 * w.x - q2 * w.y) * a.qscale;
    a.qrot[dst + D / 2] = (q2 * w.x + q1 * w.y) * a.qscale;
  }
}

// dec_head after k_decode_route: the new token's row is one of the history's.
template <int D>
NAMOH_DEV bool dec_head_ahead(const DecAhead& a, int bk, int chunk, DecHead& o) {
  const int n = __builtin_amdgcn_readfirstlane(a.ahead[bk]);
  const int h = __builtin_amdgcn_readfirstlane(a.topk_idx[bk]);
  if (n < 0) return false;
  o.bh = static_cast<size_t>(bk / a.K) * a.H + h;
  o.hist = n + 1;
  o.ring0 = 0;
  o.chunk = dec_chunk_rows<D>(n + 1, a.nchunk, a.fine);
  return chunk * o.chunk <= n;
}

// GQ queries per history row (the query heads of a key/value group; 1
// without groups): each row is read once and scored against all of them, with
// one online softmax per query; the partial of query u of selected head bk is
// (bk * GQ + u) * nchunk + chunk.
// SHARED (shared heads): the caches may be rings of cap rows; history row r is
// physical row (ring0 + r) mod cap.
// The new token's row is not read from the cache (the workgroup whose chunk it
// ends writes it): it is scored from LDS after the history.  The first rows of
// the history are loaded before the new token's angles are formed.
// AHEAD: k_decode_route ran before.
template <int D, bool BF16, int GQ = 1, bool SHARED = false, bool AHEAD = false>
__global__ __launch_bounds__(256) void k_decode_attn(const DecArgs<AHEAD> a) {
  constexpr int EPG = BF16 ? 8 : 4;   // elements per 16-byte granule
  constexpr int G = D / EPG;          // lanes per row
  constexpr int RPW = 64 / G;         // rows per wave per step
  constexpr int RPB = 4 * RPW;        // rows per workgroup per step
  // rows per lane in flight, fewer with more queries per row (registers)
  constexpr int U = GQ <= 2 ? kDecUnroll : (GQ == 4 ? kDecUnroll / 2 : kDecUnroll / 4);
  __shared__ float s_ml[GQ][RPB][2];
  __shared__ float s_acc[GQ][RPB][D];
  __shared__ float2 s_cs[D / 2];
  __shared__ u32x4 s_new[2 * G];

  const int bk = block_x() / a.nchunk;
  const int chunk = block_x() - bk * a.nchunk;
  DecHead hd;
  if constexpr (AHEAD) {
    if (!dec_head_ahead<D>(a, bk, chunk, hd)) return;
  } else {
    if (!dec_head<D, SHARED>(a, bk, chunk, hd)) return;
  }
  const int r0 = chunk * hd.chunk;
  const int r1 = min(hd.hist, r0 + hd.chunk);   // cached rows [r0, r1)
  const bool owner = !AHEAD && hd.hist < r0 + hd.chunk;   // the new row ends this chunk
  const size_t rowbase = hd.bh * a.cap;
  const int tid = thread_x();
  const int lane = tid % 64, wave = tid / 64;
  const int sub = lane % G;
  const int grp = wave * RPW + lane / G;
  const u32x4* kc = static_cast<const u32x4*>(a.k_cache);
  const u32x4* vc = static_cast<const u32x4*>(a.v_cache);
  u32x4 kx[U], vx[U];
  auto load_rows = [&](int rb) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = rb + u * RPB + grp;
      kx[u] = vx[u] = u32x4{0u, 0u, 0u, 0u};
      if (r < r1) {
        long pr = r;
        if constexpr (SHARED) {
          pr += hd.ring0;
          if (pr >= a.cap) pr -= a.cap;
        }
        const size_t gi = (rowbase + pr) * G + sub;
        kx[u] = kc[gi];
        vx[u] = vc[gi];
      }
    }
  };
  float qv[GQ][EPG];
  if constexpr (AHEAD) {
#pragma unroll
    for (int u = 0; u < GQ; ++u)
#pragma unroll
      for (int e = 0; e < EPG; ++e)
        qv[u][e] = a.qrot[(static_cast<size_t>(bk) * GQ + u) * D + sub * EPG + e];
    load_rows(r0);
  } else {
    // the lane's granule of each query and its rotation partner's
    u32x4 qx[GQ], qy[GQ];
    const int mate = sub < G / 2 ? sub + G / 2 : sub - G / 2;
#pragma unroll
    for (int u = 0; u < GQ; ++u) {
      const u32x4* qrow = static_cast<const u32x4*>(a.q) + (hd.bh * GQ + u) * G;
      qx[u] = qrow[sub];
      qy[u] = qrow[mate];
    }
    load_rows(r0);
    dec_new_token<D, BF16>(a, hd, owner, s_cs, s_new);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GQ; ++u) {
      float x[EPG], y[EPG];
      dec_unpack<BF16>(qx[u], x);
      dec_unpack<BF16>(qy[u], y);
#pragma unroll
      for (int e = 0; e < EPG; ++e) {
        const float2 w = s_cs[(sub % (G / 2)) * EPG + e];
        qv[u][e] = (sub < G / 2 ? x[e] * w.x - y[e] * w.y : x[e] * w.x + y[e] * w.y) * a.qscale;
      }
    }
  }
  float m[GQ], lsum[GQ], acc[GQ][EPG];
#pragma unroll
  for (int u = 0; u < GQ; ++u) {
    m[u] = -1e30f;
    lsum[u] = 0.f;
#pragma unroll
    for (int e = 0; e < EPG; ++e) acc[u][e] = 0.f;
  }

  // the first UU rows in kx, vx (row u of the lane counts if r + u step < end)
  auto take_rows = [&](auto uu, int r, int step, int end) {
    constexpr int UU = decltype(uu)::value;
    float sc[GQ][UU];
#pragma unroll
    for (int u = 0; u < UU; ++u) {
      float f[EPG];
      dec_unpack<BF16>(kx[u], f);
#pragma unroll
      for (int qq = 0; qq < GQ; ++qq) {
        float dsum = 0.f;
#pragma unroll
        for (int e = 0; e < EPG; ++e) dsum = fmaf(qv[qq][e], f[e], dsum);
        dsum = group_sum<G>(dsum);
        sc[qq][u] = r + u * step < end ? dsum : -INFINITY;
      }
    }
    float p[GQ][UU];
#pragma unroll
    for (int qq = 0; qq < GQ; ++qq) {
      float mx = sc[qq][0];
#pragma unroll
      for (int u = 1; u < UU; ++u) mx = fmaxf(mx, sc[qq][u]);
      const float mnew = fmaxf(m[qq], mx);
      const float corr = __builtin_amdgcn_exp2f(m[qq] - mnew);
      lsum[qq] *= corr;
#pragma unroll
      for (int e = 0; e < EPG; ++e) acc[qq][e] *= corr;
#pragma unroll
      for (int u = 0; u < UU; ++u) {
        p[qq][u] = __builtin_amdgcn_exp2f(sc[qq][u] - mnew);
        lsum[qq] += p[qq][u];
      }
      m[qq] = mnew;
    }
#pragma unroll
    for (int u = 0; u < UU; ++u) {
      float f[EPG];
      dec_unpack<BF16>(vx[u], f);
#pragma unroll
      for (int qq = 0; qq < GQ; ++qq)
#pragma unroll
        for (int e = 0; e < EPG; ++e) acc[qq][e] = fmaf(p[qq][u], f[e], acc[qq][e]);
    }
  };
  for (int rb = r0; rb < r1; rb += RPB * U) {
    if (rb > r0) load_rows(rb);
    // as few of the row slots as hold the rows that are left (the others would
    // change nothing): 945 sequences x 8 heads of 24 rows, d 64, 56 -> 47 us
    const int left = r1 - rb;
    if (left > RPB * U / 2) take_rows(std::integral_constant<int, U>{}, rb + grp, RPB, r1);
    else if (left > RPB * U / 4) take_rows(std::integral_constant<int, U / 2>{}, rb + grp, RPB, r1);
    else take_rows(std::integral_constant<int, U / 4 ? U / 4 : 1>{}, rb + grp, RPB, r1);
  }
  if (owner && wave == 0) {
    // the new token's row, in the first row group only: the others' weight for
    // it is zero, and zero times an infinite value would be NaN
    kx[0] = vx[0] = u32x4{0u, 0u, 0u, 0u};
    if (grp == 0) {
      kx[0] = s_new[sub];
      vx[0] = s_new[G + sub];
    }
    take_rows(std::integral_constant<int, 1>{}, grp, 1, 1);
  }
#pragma unroll
  for (int qq = 0; qq < GQ; ++qq) {
    if (sub == 0) {
      s_ml[qq][grp][0] = m[qq];
      s_ml[qq][grp][1] = lsum[qq];
    }
#pragma unroll
    for (int e = 0; e < EPG; ++e) s_acc[qq][grp][sub * EPG + e] = acc[qq][e];
  }
  __syncthreads();
  for (int t2 = tid; t2 < GQ * D; t2 += 256) {
    const int qq = t2 / D, dd = t2 - (t2 / D) * D;
    float M = -1e30f;
    for (int gi = 0; gi < RPB; ++gi) M = fmaxf(M, s_ml[qq][gi][0]);
    float Ls = 0.f, A = 0.f;
    for (int gi = 0; gi < RPB; ++gi) {
      const float w = __builtin_amdgcn_exp2f(s_ml[qq][gi][0] - M);
      Ls = fmaf(s_ml[qq][gi][1], w, Ls);
      A = fmaf(s_acc[qq][gi][dd], w, A);
    }
    const size_t pi = (static_cast<size_t>(bk) * GQ + qq) * a.nchunk + chunk;
    a.part_acc[pi * D + dd] = A;
    if (dd == 0) {
      a.part_ml[2 * pi] = M;
      a.part_ml[2 * pi + 1] = Ls;
    }
  }
}

// Grouped decode on the matrix cores (GQ = 4 or 8 query heads share each
// cached row).  A wave takes 128 rows of the chunk in blocks of 32 and uses
// v_mfma_f32_16x16x32_bf16 (lane l: A row / B column / C column l % 16,
// reduction slots 8 (l / 16) .. + 7; C rows 4 (l / 16) + i in accumulator
// i):
//   the block's key and value rows are loaded whole (each lane a 16-byte
//     granule of D / 16 consecutive rows: coalesced 16-byte loads) and
//     rearranged through wave-private LDS: key rows row-major with padded
//     rows (s_k), and each lane's run of rows of one column written as one
//     run of a V^T row (s_vt); the next block's loads are issued before the
//     current block is processed;
//   S[q][r] = Q K^T for two 16-row tiles: A = the GQ rotated queries (rows
//     >= GQ zero), B = the key rows read back from s_k;
//   online softmax per query in exp2 units: the 16 lanes of one reduction
//     group hold a query's 16 scores of a tile;
//   O[q][d] += P V over the 32 rows: A = P and B = V^T read from the
//     wave-private LDS tiles (P as [query][row], V^T as [d][row], both
//     16-byte reads).
// LDS: about 81 KB per workgroup at D = 128, so the two workgroups per
// compute unit that the launch bounds ask for fill its 160 KB.
// The reduction group kg = l / 16 of every layout holds queries 4 kg .. 4 kg
// + 3, so a lane's rescale factors apply to its own output accumulators.
// Partials as in k_decode_attn: (bk * GQ + q) * nchunk + chunk.
template <int D, int GQ, bool AHEAD>
__global__ __launch_bounds__(256, 2) void k_decode_attn_mfma(const DecArgs<AHEAD> a) {
  static_assert(GQ == 4 || GQ == 8, "queries per cached row");
  static_assert(D == 64 || D == 128, "head width");
  constexpr int KS = D / 32;           // reduction steps of the score product
  constexpr int NT = D / 16;           // 16-column output tiles
  constexpr int VP = 40;               // padded row length (elements) of the LDS tiles
  // the V^T tiles are dead after the loop; the per-wave output rows reuse them
  static_assert(4 * GQ * D * 4 <= 4 * D * VP * 2, "output rows fit the V^T tiles");
  constexpr int KP = D + 8;             // padded key row (elements) of the LDS key tile
  constexpr int GR = D / 8;             // 16-byte granules per cached row
  constexpr int RPL = GR / 2;           // rows per lane per 32-row block (coalesced loads)
  __shared__ __attribute__((aligned(16))) uint16_t s_vt[4][D * VP];
  __shared__ __attribute__((aligned(16))) uint16_t s_k[4][32 * KP];
  __shared__ __attribute__((aligned(16))) uint16_t s_p[4][16 * VP];
  __shared__ float s_ml[4][GQ][2];
  // the new token's factors share the probabilities' tiles (read before the
  // loop writes those): with 512 bytes more only one workgroup would fit
  float2* const s_cs = reinterpret_cast<float2*>(&s_p[0][0]);
  static_assert(sizeof(s_p) >= D / 2 * sizeof(float2), "factors fit");
  __shared__ u32x4 s_new[2 * GR];
  float (*s_o)[GQ][D] = reinterpret_cast<float (*)[GQ][D]>(&s_vt[0][0]);

  const int bk = block_x() / a.nchunk;
  const int chunk = block_x() - bk * a.nchunk;
  DecHead hd;
  if constexpr (AHEAD) {
    if (!dec_head_ahead<D>(a, bk, chunk, hd)) return;
  } else {
    if (!dec_head<D, false>(a, bk, chunk, hd)) return;
  }
  const int r0 = chunk * hd.chunk;
  const int n = AHEAD ? hd.hist - 1 : hd.hist;   // the new token's row
  const int r1 = min(n + 1, r0 + hd.chunk);
  const bool owner = n < r0 + hd.chunk;
  const size_t rowbase = hd.bh * a.cap;
  const int tid = thread_x();
  const int lane = tid % 64, wave = tid / 64;
  const int j16 = lane & 15, kg = lane >> 4;
  // (after k_decode_route: many workgroups, and the waves share short chunks)
  const int rpw = AHEAD ? ((r1 - r0 + 3) / 4 + 31) / 32 * 32 : hd.chunk / 4;
  const int w0 = r0 + wave * rpw;
  const int w1 = min(r1, w0 + rpw);

  // the lane's queries' granules (A operand rows >= GQ are zero: they read
  // query GQ - 1 and are cleared after the loads; a load under a branch would
  // be waited for at the join, one round trip per load)
  u32x4 qx[KS];
  float4 qf[KS][2];
  if constexpr (AHEAD) {
    const float4* qrow = reinterpret_cast<const float4*>(
        a.qrot + (static_cast<size_t>(bk) * GQ + min(j16, GQ - 1)) * D + 8 * kg);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qf[s][0] = qrow[8 * s];
      qf[s][1] = qrow[8 * s + 1];
    }
  } else {
    const u32x4* qrow = static_cast<const u32x4*>(a.q) + (hd.bh * GQ + min(j16, GQ - 1)) * GR + kg;
#pragma unroll
    for (int s = 0; s < KS; ++s) qx[s] = qrow[4 * s];
  }
  float m[4], l[4];
  f32x4 O[NT];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    m[i] = -1e30f;
    l[i] = 0.f;
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) O[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  const u32x4* kc = static_cast<const u32x4*>(a.k_cache);
  const u32x4* vc = static_cast<const u32x4*>(a.v_cache);
  uint16_t* vt = s_vt[wave];
  uint16_t* pt = s_p[wave];
  // Coalesced loads: lane (granule lane % GR, row group lane / GR) reads rows
  // RPL * group + i, i < RPL, of the block, so each load instruction covers
  // whole rows.  Rows past the wave's end read its last row (finite values;
  // masked).  The next block is loaded while the current one is processed
  // (its loads are issued unconditionally, clamped like the tail).
  const int lg = lane % GR, lq = lane / GR;
  u32x4 kx[RPL], vx[RPL], kn[RPL], vn[RPL];
  auto load_block = [&](int rb, u32x4 (&kd)[RPL], u32x4 (&vd)[RPL]) {
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const size_t row = rowbase + min(rb + RPL * lq + i, w1 - 1);
      kd[i] = kc[row * GR + lg];
      vd[i] = vc[row * GR + lg];
    }
  };
  if (w0 < w1) load_block(w0, kx, vx);
  bf16x8 qa[KS];
  const bool keep = j16 < GQ;
  if constexpr (AHEAD) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const float x[8] = {qf[s][0].x, qf[s][0].y, qf[s][0].z, qf[s][0].w,
                          qf[s][1].x, qf[s][1].y, qf[s][1].z, qf[s][1].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) qa[s][e] = static_cast<__bf16>(keep ? x[e] : 0.f);
    }
  } else {
    dec_new_token<D, true>(a, hd, owner, s_cs, s_new);
    __syncthreads();
    // rotated, scaled queries: pair (j, j + D / 2) is granules s and s + KS / 2
#pragma unroll
    for (int s = 0; s < KS / 2; ++s) {
      float x[8], y[8];
      dec_unpack<true>(qx[s], x);
      dec_unpack<true>(qx[s + KS / 2], y);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float2 w = s_cs[32 * s + 8 * kg + e];
        qa[s][e] = static_cast<__bf16>(keep ? (x[e] * w.x - y[e] * w.y) * a.qscale : 0.f);
        qa[s + KS / 2][e] = static_cast<__bf16>(keep ? (y[e] * w.x + x[e] * w.y) * a.qscale : 0.f);
      }
    }
    __syncthreads();
  }
  for (int rb = w0; rb < w1; rb += 32) {
    load_block(min(rb + 32, w1 - 1), kn, vn);
    if (!AHEAD && rb + 32 > n) {   // the new token's row (and rows clamped to it) from LDS
      const u32x4 nk = s_new[lg], nv = s_new[GR + lg];
#pragma unroll
      for (int i = 0; i < RPL; ++i)
        if (min(rb + RPL * lq + i, w1 - 1) == n) {
          kx[i] = nk;
          vx[i] = nv;
        }
    }
    // key rows into the wave's LDS tile (row-major, padded rows), values
    // transposed into V^T: lane's RPL consecutive rows of one granule become,
    // per column, one RPL-element run of a V^T row
    uint16_t* kt = s_k[wave];
#pragma unroll
    for (int i = 0; i < RPL; ++i)
      *reinterpret_cast<u32x4*>(&kt[(RPL * lq + i) * KP + 8 * lg]) = kx[i];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      uint32_t run[RPL / 2];
#pragma unroll
      for (int m = 0; m < RPL / 2; ++m) {
        const uint32_t a = vx[2 * m][e / 2], c2 = vx[2 * m + 1][e / 2];
        run[m] = (e & 1) ? ((a >> 16) | (c2 & 0xFFFF0000u)) : ((a & 0xFFFFu) | (c2 << 16));
      }
      uint16_t* dst = &s_vt[wave][(8 * lg + e) * VP + RPL * lq];
      if constexpr (RPL == 8)
        *reinterpret_cast<u32x4*>(dst) = u32x4{run[0], run[1], run[2], run[3]};
      else
        *reinterpret_cast<uint2*>(dst) = make_uint2(run[0], run[1]);
    }
    f32x4 S[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      S[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 kb =
            *reinterpret_cast<const bf16x8*>(&kt[(16 * tt + j16) * KP + 32 * s + 8 * kg]);
        S[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[s], kb, S[tt], 0, 0, 0);
      }
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
      if (rb + 16 * tt + j16 >= w1) S[tt] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float mx = fmaxf(S[0][i], S[1][i]);
      mx = group_max<16>(mx);
      const float mnew = fmaxf(m[i], mx);
      const float corr = __builtin_amdgcn_exp2f(m[i] - mnew);
      m[i] = mnew;
      const float p0 = __builtin_amdgcn_exp2f(S[0][i] - mnew);
      const float p1 = __builtin_amdgcn_exp2f(S[1][i] - mnew);
      float ps = p0 + p1;
      ps = group_sum<16>(ps);
      l[i] = l[i] * corr + ps;
#pragma unroll
      for (int t = 0; t < NT; ++t) O[t][i] *= corr;
      pt[(4 * kg + i) * VP + j16] = f32_to_bf16(p0);
      pt[(4 * kg + i) * VP + 16 + j16] = f32_to_bf16(p1);
    }
    // the tiles are wave-private: LDS operations of one wave complete in order
    const bf16x8 pa = *reinterpret_cast<const bf16x8*>(&pt[j16 * VP + 8 * kg]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bf16x8 vb = *reinterpret_cast<const bf16x8*>(&vt[(16 * t + j16) * VP + 8 * kg]);
      O[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, vb, O[t], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      kx[i] = kn[i];
      vx[i] = vn[i];
    }
  }

  // ---- merge the four waves' partials of every query -----------------------
  __syncthreads();   // every wave is done with its V^T tile (reused for s_o)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int q = 4 * kg + i;
    if (q < GQ) {
      if (j16 == 0) {
        s_ml[wave][q][0] = m[i];
        s_ml[wave][q][1] = l[i];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) s_o[wave][q][16 * t + j16] = O[t][i];
    }
  }
  __syncthreads();
  for (int t2 = tid; t2 < GQ * D; t2 += 256) {
    const int q = t2 / D, dd = t2 - (t2 / D) * D;
    float M = -1e30f;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, s_ml[w][q][0]);
    float Ls = 0.f, A = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float sc = __builtin_amdgcn_exp2f(s_ml[w][q][0] - M);
      Ls = fmaf(s_ml[w][q][1], sc, Ls);
      A = fmaf(s_o[w][q][dd], sc, A);
    }
    const size_t pi = (static_cast<size_t>(bk) * GQ + q) * a.nchunk + chunk;
    a.part_acc[pi * D + dd] = A;
    if (dd == 0) {
      a.part_ml[2 * pi] = M;
      a.part_ml[2 * pi + 1] = Ls;
    }
  }
}

// One workgroup per sequence; wave w merges the chunk partials of the heads w,
// w + NWV, ... (lane c holds chunk c's max and sum; the accumulators are read
// column-wise, d = lane + 64 i), then the gated head outputs are summed in
// head order.  With key/value groups (G query heads per selected head) the G
// heads of a slot share its gate and are summed in head order.  Shared heads
// (SHARED): every head, gate 1, one length per sequence.  The cache lengths
// are advanced here, after every wave (and the attention) has read them.
template <int D, bool OUT_BF16, int NWV, bool SHARED>
__global__ __launch_bounds__(64 * NWV) void k_decode_combine(
    const float* __restrict__ gates, const int32_t* __restrict__ topk_idx, int32_t* cache_len,
    const float* __restrict__ part_acc, const float* __restrict__ part_ml, int H, int K, long cap,
    int window, int nchunk, int fine, void* __restrict__ out, int G, int accumulate) {
  constexpr int DPL = (D + 63) / 64;  // output columns per lane
  __shared__ float s_o[NWV][D];
  const int b = block_x();
  const int tid = thread_x(), lane = tid % 64, wave = tid / 64;
  int32_t* len = SHARED ? cache_len + b : cache_len + static_cast<size_t>(b) * H;
  const int len_l = SHARED ? len[0] : len[min(lane, H - 1)];   // lane = head
  float o[DPL];
#pragma unroll
  for (int i = 0; i < DPL; ++i) o[i] = 0.f;
  for (int vk = wave; vk < K * G; vk += NWV) {
    const int kk = vk / G;
    const size_t bk = static_cast<size_t>(b) * K + kk;
    const size_t bq = bk * G + (vk - kk * G);   // the head's partials
    // the first 64 chunks' (max, sum) and the first chunk's row are loaded
    // before the history's length is known (past it they are not used)
    const float2* ml = reinterpret_cast<const float2*>(part_ml) + bq * nchunk;
    const float* pa = part_acc + bq * nchunk * D;
    const float2 ml0 = ml[min(lane, nchunk - 1)];
    float a0[DPL];
#pragma unroll
    for (int i = 0; i < DPL; ++i) a0[i] = pa[min(lane + 64 * i, D - 1)];
    float gate = 1.f;
    int L;
    if constexpr (SHARED) {
      const int p = len_l;
      L = p < 0 || (window == 0 && p >= cap) ? 0 : (window > 0 ? min(p + 1, window) : p + 1);
    } else {
      gate = gates[bk];
      const int h = __builtin_amdgcn_readfirstlane(topk_idx[bk]);
      const int n = h >= 0 && h < H ? __builtin_amdgcn_readlane(len_l, h) : -1;
      L = n >= 0 && n < cap ? n + 1 : 0;
    }
    if (L == 0) continue;
    const int rows = dec_chunk_rows<D>(L, nchunk, fine);
    const int nc = (L + rows - 1) / rows;
    float M = lane < nc ? ml0.x : -1e30f;
    for (int c = lane + 64; c < nc; c += 64) M = fmaxf(M, ml[c].x);
    M = group_max<64>(M);
    float Ls = lane < nc ? ml0.y * __builtin_amdgcn_exp2f(ml0.x - M) : 0.f;
    for (int c = lane + 64; c < nc; c += 64) Ls += ml[c].y * __builtin_amdgcn_exp2f(ml[c].x - M);
    Ls = group_sum<64>(Ls);
    const float scale = gate / Ls;
    float w = __builtin_amdgcn_exp2f(__shfl(ml0.x, 0) - M);
    float a[DPL];
#pragma unroll
    for (int i = 0; i < DPL; ++i) a[i] = a0[i] * w;
#pragma unroll 8
    for (int c = 1; c < nc; ++c) {
      w = __builtin_amdgcn_exp2f(ml[c].x - M);
#pragma unroll
      for (int i = 0; i < DPL; ++i)
        a[i] = fmaf(pa[static_cast<size_t>(c) * D + min(lane + 64 * i, D - 1)], w, a[i]);
    }
#pragma unroll
    for (int i = 0; i < DPL; ++i) o[i] = fmaf(a[i], scale, o[i]);
  }
#pragma unroll
  for (int i = 0; i < DPL; ++i) {
    const int d = lane + 64 * i;
    if (d < D) s_o[wave][d] = o[i];
  }
  __syncthreads();   // every wave has read the lengths
  if constexpr (SHARED) {
    if (tid == 0 && len_l >= 0 && (window > 0 || len_l < cap)) len[0] = len_l + 1;
  } else if (tid < K) {
    const int h = topk_idx[static_cast<size_t>(b) * K + tid];
    if (h >= 0 && h < H) {
      const int n = len[h];
      if (n >= 0 && n < cap) len[h] = n + 1;
    }
  }
  if (tid < D) {
    const size_t oi = static_cast<size_t>(b) * D + tid;
    float r = 0.f;
    if (accumulate) {   // added to what out holds (shared heads after the routed step)
      if constexpr (OUT_BF16) r = bf16_to_f32(static_cast<const uint16_t*>(out)[oi]);
      else r = static_cast<const float*>(out)[oi];
    }
#pragma unroll
    for (int w = 0; w < NWV; ++w) r += s_o[w][tid];
    if constexpr (OUT_BF16) static_cast<uint16_t*>(out)[oi] = f32_to_bf16(r);
    else static_cast<float*>(out)[oi] = r;
  }
}

template <int D, bool SHARED>
static void launch_dec_combine(const DecStep& a, int32_t* cache_len, int B, int G, void* out,
                               int out_dtype, int accumulate, hipStream_t st) {
  auto run = [&](auto kernel, int nwv) {
    kernel<<<B, 64 * nwv, 0, st>>>(a.gates, a.topk_idx, cache_len, a.part_acc, a.part_ml, a.H, a.K,
                                   a.cap, a.window, a.nchunk, a.fine, out, G, accumulate);
  };
  // a wave per head while there are up to 8; 16 waves for more
  if (a.K * G <= 8) {
    if (out_dtype == 1) run(k_decode_combine<D, true, 8, SHARED>, 8);
    else run(k_decode_combine<D, false, 8, SHARED>, 8);
  } else {
    if (out_dtype == 1) run(k_decode_combine<D, true, 16, SHARED>, 16);
    else run(k_decode_combine<D, false, 16, SHARED>, 16);
  }
}

// Chunks per head (partials to hold and workgroups to launch) with `heads`
// active heads in the call: 512-row chunks hold the capacity, and where they
// leave compute units idle there is one per dec_min_rows rows as long as the
// launch stays within one workgroup per compute unit.  Steps of attention and
// combine, 512-row chunks -> these: 2 shared heads over a window of 512, d 128, 8
// sequences 11.1 -> 8.2 us, 64 sequences 12.7 -> 10.1; one sequence, 8 heads of
// 4000 rows, d 128, 13.5 -> 11.8; of 300 rows, d 64, 9.8 -> 9.0.  Up to 512
// workgroups: the same, but 14.6 for 13.1 where the capacity (2051) is far above
// the histories (520) and the rest of the launch finds no rows.
constexpr long kDecSpreadGroups = 256;
static int dec_nchunk(size_t heads, int cap, int d) {
  const long nc = (static_cast<long>(cap) + kDecChunk - 1) / kDecChunk;
  const long fit = kDecSpreadGroups / std::max<long>(static_cast<long>(heads), 1);
  return static_cast<int>(std::max(nc, std::min((static_cast<long>(cap) + dec_min_rows(d) - 1) / dec_min_rows(d), fit)));
}

// Partials to make room for (per query head): no fewer than heads *
// dec_nchunk(heads, cap, d), and never fewer for more heads or a larger cap,
// so a workspace sized for a program's largest batch serves its smaller ones,
// whose heads are cut into more chunks (the chunks alone: 17 sequences of 8
// heads, d 128, cap 512, have 136 partials, 16 have 256).
static size_t dec_partials(size_t heads, int cap, int d) {
  const size_t whole = heads * ((static_cast<size_t>(cap) + kDecChunk - 1) / kDecChunk);
  const size_t fine = whole * (kDecChunk / dec_min_rows(d));
  return std::max(whole, std::min(fine, static_cast<size_t>(kDecSpreadGroups)));
}

// Routing ahead (k_decode_route): where a launch has many workgroups of few
// rows each, finding the head, forming the angles and rotating the queries in
// every one of them costs more than a launch (the VALU is the limit; on the
// matrix cores two or three workgroups per compute unit, each a chain of
// latencies).  A step in us, routed in every workgroup -> ahead:
//   g 1, d 64   945 sequences x 8 heads of 24 rows 46 -> 32, 512 x 8 of 100 34 -> 30,
//               256 x 8 of 30 16.8 -> 15.8; but 128 x 8 of 100 12.5 -> 14.2, 1024 x 4
//               of 1000 193 -> 198;
//   g 1, d 128  600 x 16 of 20 55 -> 32; but 512 x 8 of 400 161 -> 165;
//   g 1, d 32   1009 x 4 of 355 78 -> 57, 400 x 8 of 1000 91 -> 85;
//   g 4, d 64   489 x 8 of 162 100 -> 66; d 128, 723 x 4 of 80 67 -> 48, 306 x 1 of
//               1277 56 -> 52; but g 8, d 64, 665 x 1 of 1546 59 -> 65.
// The lengths are on the device, so the rule goes by the capacity; the
// workspace has room for it at any capacity (sizes never decrease in it).
static bool dec_ahead_room(size_t heads, int cap, int d, int G) {
  return heads * dec_nchunk(heads, cap, d) > (G >= 4 || d == 32 ? 1024 : 2000);
}
static bool dec_route_ahead(size_t heads, int cap, int d, int G) {
  if (!dec_ahead_room(heads, cap, d, G)) return false;
  if (G >= 4) return cap <= 1792;
  return d == 32 ? cap <= 2048 : static_cast<long>(cap) * d <= 25600;
}

struct DecWs {
  int32_t* ahead;
  float* qrot;
  float* part_acc;
  float* part_ml;
  size_t bytes;
};

static DecWs carve_dec(void* ws, int B, int K, int d, int cap, int G = 1) {
  const size_t BK = static_cast<size_t>(B) * K;
  const size_t np = dec_partials(BK, cap, d);
  Carver cv(ws);
  DecWs w{};
  if (dec_ahead_room(BK, cap, d, G)) {
    w.ahead = cv.take<int32_t>(BK);
    w.qrot = cv.take<float>(BK * G * d);
  }
  w.part_acc = cv.take<float>(np * G * d);
  w.part_ml = cv.take<float>(np * G * 2);
  w.bytes = cv.off;
  return w;
}

size_t decode_workspace_bytes(int B, int /*H*/, int K, int d, int cap, int G) {
  return carve_dec(nullptr, B, K, d, cap, G).bytes;
}

// ---------------------------------------------------------------------------
// Scratch of the decode step that allocates nothing (namoh_decode_step_noalloc):
// the step's workspace (the per-chunk partials) in a file-scope device array.
// Every GPU the library runs on holds its own copy for the life of the process;
// every call on one GPU uses that GPU's copy, so calls that overlap on one GPU
// race.  Nothing in it needs to start at zero: each chunk writes the partial the
// combine reads.
constexpr size_t kDecodeScratchBytes = static_cast<size_t>(32) << 20;
static __device__ __attribute__((aligned(256))) unsigned char scratch[kDecodeScratchBytes];

size_t decode_scratch_bytes() { return kDecodeScratchBytes; }

// Device address of the array on the current device.  In host code the
// array's name only stands in for the symbol; its device address comes from
// hipGetSymbolAddress, taken once per device (with that device current) and
// kept.
hipError_t decode_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  *ptr = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Prefill -> decode hand-off (Sec. 3.2, efficient execution: a decoding step
// reads and extends only its active heads' caches, so those must hold the
// prompt's rotated keys and values of each head in rank order, Eq.
// namoh-head-rope).  A workgroup takes 4096 / D consecutive packed rows: the
// segment of each row by binary search over seg_offsets (staged in LDS), then one 8-pair
// group (elements j..j+7 and j+d/2..j+d/2+7) per thread, 16-byte loads and
// stores, angles formed and reduced in double as in the decode append.  Rows
// whose offsets are not a packing of [0, Nr) with ranks below cap and tokens
// below T are skipped.
constexpr int kCacheThreads = 256;
constexpr int kCacheSegLds = 2048;   // segment offsets staged in LDS up to this many segments
template <int D>
constexpr int cache_rows() { return kCacheThreads * 16 / D; }

template <bool BF16>
NAMOH_DEV void ld8(const void* p, size_t i, float* x) {
  if constexpr (BF16) {
    const uint4 u = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(p) + i);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[2 * e] = lo_bf16(w[e]);
      x[2 * e + 1] = hi_bf16(w[e]);
    }
  } else {
    const float4 a = *reinterpret_cast<const float4*>(static_cast<const float*>(p) + i);
    const float4 c = *reinterpret_cast<const float4*>(static_cast<const float*>(p) + i + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = c.x; x[5] = c.y; x[6] = c.z; x[7] = c.w;
  }
}

template <bool BF16>
NAMOH_DEV void st8(void* p, size_t i, const float* x) {
  if constexpr (BF16) {
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p) + i) =
        make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                   pack_bf16x2(x[6], x[7]));
  } else {
    *reinterpret_cast<float4*>(static_cast<float*>(p) + i) = make_float4(x[0], x[1], x[2], x[3]);
    *reinterpret_cast<float4*>(static_cast<float*>(p) + i + 4) = make_float4(x[4], x[5], x[6], x[7]);
  }
}

template <int D, bool BF16>
__global__ __launch_bounds__(kCacheThreads) void k_prefill_cache(
    const void* __restrict__ k, const void* __restrict__ v,
    const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ perm_token, int BH,
    int H, int T, int Nr, long cap, double log_base, int rope_mode, int nblocks,
    void* __restrict__ k_cache, void* __restrict__ v_cache, int32_t* __restrict__ cache_len) {
  constexpr int RW = cache_rows<D>();
  constexpr int G = D / 16;   // 8-pair groups per row
  static_assert(RW * G == kCacheThreads, "one group per thread");
  __shared__ double s_theta[D / 2];
  __shared__ int s_seg[RW], s_rank[RW], s_tok[RW];
  __shared__ int s_off[kCacheSegLds + 1];
  const int tid = thread_x();
  const int row0 = block_x() * RW;
  for (int s = block_x() * kCacheThreads + tid; s < BH; s += nblocks * kCacheThreads)
    cache_len[s] = seg_offsets[s + 1] - seg_offsets[s];
  if (tid < D / 2) s_theta[tid] = exp(-(2.0 * tid / D) * log_base);
  const bool in_lds = BH <= kCacheSegLds;
  if (in_lds)
    for (int i = tid; i <= BH; i += kCacheThreads) s_off[i] = seg_offsets[i];
  __syncthreads();
  const int32_t* off = in_lds ? s_off : seg_offsets;
  if (tid < RW) {
    const int pr = row0 + tid;
    int seg = -1, rank = -1, tok = -1;
    if (pr < Nr) {
      tok = perm_token[pr];
      int lo = 0, hi = BH;   // the last segment starting at or before pr
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= pr) lo = mid; else hi = mid;
      }
      seg = lo;
      rank = pr - off[lo];
      if (rank < 0 || rank >= cap || pr >= off[lo + 1] || tok < 0 || tok >= T) seg = -1;
    }
    s_seg[tid] = seg;
    s_rank[tid] = rank;
    s_tok[tid] = tok;
  }
  __syncthreads();
  const int row = tid / G, j0 = (tid - row * G) * 8;
  const int seg = s_seg[row];
  if (seg < 0) return;
  const int r = s_rank[row], t = s_tok[row];
  const size_t src = (static_cast<size_t>(seg) * T + t) * D;
  const size_t dst = (static_cast<size_t>(seg) * cap + r) * D;
  float k1[8], k2[8], v1[8], v2[8];
  ld8<BF16>(k, src + j0, k1);
  ld8<BF16>(k, src + j0 + D / 2, k2);
  ld8<BF16>(v, src + j0, v1);
  ld8<BF16>(v, src + j0 + D / 2, v2);
  if (rope_mode != 2) {
    const double pos = rope_mode == 0 ? r : t;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float2 w = rope_cos_sin(pos * s_theta[j0 + e]);
      const float a = k1[e], c = k2[e];
      k1[e] = a * w.x - c * w.y;
      k2[e] = c * w.x + a * w.y;
    }
  }
  st8<BF16>(k_cache, dst + j0, k1);
  st8<BF16>(k_cache, dst + j0 + D / 2, k2);
  st8<BF16>(v_cache, dst + j0, v1);
  st8<BF16>(v_cache, dst + j0 + D / 2, v2);
}

template <int D, bool BF16>
static hipError_t run_prefill_cache(const void* k, const void* v, int B, int T, int H, int K,
                                    float rope_base, int rope_mode, const int32_t* seg_offsets,
                                    const int32_t* perm_token, void* k_cache, void* v_cache,
                                    int32_t* cache_len, int cap, hipStream_t st) {
  const int BH = B * H;
  const long Nr = static_cast<long>(B) * T * K;
  const double log_base = rope_mode == 2 ? 0.0 : std::log(static_cast<double>(rope_base));
  constexpr int RW = cache_rows<D>();
  const long blocks = std::max((Nr + RW - 1) / RW,
                               static_cast<long>((BH + kCacheThreads - 1) / kCacheThreads));
  k_prefill_cache<D, BF16><<<static_cast<unsigned>(blocks), kCacheThreads, 0, st>>>(
      k, v, seg_offsets, perm_token, BH, H, T, static_cast<int>(Nr), cap, log_base, rope_mode,
      static_cast<int>(blocks), k_cache, v_cache, cache_len);
  return hipGetLastError();
}

hipError_t launch_prefill_cache(const void* k, const void* v, int dtype, int B, int T, int H,
                                int K, int d, float rope_base, int rope_mode,
                                const int32_t* seg_offsets, const int32_t* perm_token,
                                void* k_cache, void* v_cache, int32_t* cache_len, int cap,
                                hipStream_t st) {
#define NAMOH_PC(DD, BF)                                                                       \
  return run_prefill_cache<DD, BF>(k, v, B, T, H, K, rope_base, rope_mode, seg_offsets,       \
                                   perm_token, k_cache, v_cache, cache_len, cap, st)
  if (dtype == 1) {
    if (d == 32) NAMOH_PC(32, true);
    if (d == 64) NAMOH_PC(64, true);
    NAMOH_PC(128, true);
  }
  if (d == 32) NAMOH_PC(32, false);
  if (d == 64) NAMOH_PC(64, false);
  NAMOH_PC(128, false);
#undef NAMOH_PC
}

template <int D, bool BF16, int GQ = 1>
static hipError_t run_decode(const float* logits, const float* bias, const void* q, const void* k,
                             const void* v, void* k_cache, void* v_cache,
                             int32_t* cache_len, const int32_t* seq_pos, int B,
                             int H, int K, int cap, float rope_base,
                             int rope_mode, int gate_mode, float scale,
                             int32_t* topk_idx, float* gates, void* out,
                             int out_dtype, int32_t* dev_status, void* ws,
                             hipStream_t st) {
  const DecWs w = carve_dec(ws, B, K, D, cap, GQ);
  const int nc = dec_nchunk(static_cast<size_t>(B) * K, cap, D);
  const double log_base = rope_mode == 2 ? 0.0 : std::log(static_cast<double>(rope_base));
  const DecStep a{logits, bias, q, k, v, k_cache, v_cache, cache_len, seq_pos, H, K, cap, log_base,
                  rope_mode, gate_mode, 0, scale * 1.4426950408889634f, topk_idx, gates, dev_status,
                  nc, static_cast<long>(B) * K * nc <= kDecFineGroups, w.part_acc, w.part_ml};
  const dim3 grid(static_cast<unsigned>(static_cast<size_t>(B) * K * nc));
  auto attn = [&](auto ahead, const auto& args) {
    constexpr bool AHEAD = decltype(ahead)::value;
    if constexpr (BF16 && (GQ == 4 || GQ == 8))
      launch_k("decode_attn", k_decode_attn_mfma<D, GQ, AHEAD>, grid, dim3(256), st, args);
    else
      launch_k("decode_attn", k_decode_attn<D, BF16, GQ, false, AHEAD>, grid, dim3(256), st, args);
  };
  if (dec_route_ahead(static_cast<size_t>(B) * K, cap, D, GQ)) {
    const DecAhead aa{a, w.ahead, w.qrot};
    launch_k("decode_route", k_decode_route<D, BF16>, dim3(static_cast<unsigned>(B * K)), dim3(64), st, aa, GQ);
    attn(std::true_type{}, aa);
  } else {
    attn(std::false_type{}, a);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_dec_combine<D, false>(a, cache_len, B, GQ, out, out_dtype, 0, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Shared heads in the decode step (Sec. 4.4, shared heads for local context):
// the new token of sequence b, at global position p = cache_len[b], enters
// every one of the Hs always-active heads.  Its key (rotated at p, or not at
// all) and value go to row p mod cap of the head's caches, and its query
// attends over the keys at positions max(0, p + 1 - window) .. p (window 0:
// 0 .. p), itself included; the head outputs are summed without a gate.
// With a window the caches are rings that keep the most recent cap >= window
// tokens; without one row p must exist (p < cap), else the step skips the
// sequence and reports it.
//
// The kernels are the routed step's (k_decode_attn and k_decode_combine with
// SHARED): every head of the sequence, its new row at the ring slot, gates 1,
// added to out.
// Prefill -> decode hand-off of the shared heads: token t of the prompt
// (rotated at t, or not at all) goes to row t mod cap of every shared head's
// caches, for the last min(T, cap) tokens (with a window the earlier ones are
// never read again); cache_len[b] = T.  One thread per (row, rotation pair).
template <int D, bool BF16>
__global__ __launch_bounds__(256) void k_shared_prefill_cache(
    const void* __restrict__ k, const void* __restrict__ v, int T, int Hs, long cap,
    long first, double log_base, int rope_mode, void* __restrict__ k_cache,
    void* __restrict__ v_cache, int32_t* __restrict__ cache_len, long nrows) {
  const long idx = static_cast<long>(block_x()) * 256 + thread_x();
  const long row = idx / (D / 2);
  const int j = static_cast<int>(idx - row * (D / 2));
  if (row >= nrows) return;
  const long keep = T - first;              // tokens first .. T - 1
  const long bs = row / keep;               // b * Hs + s
  const long t = first + (row - bs * keep);
  if (j == 0 && t == T - 1 && bs % Hs == 0) cache_len[bs / Hs] = T;
  float cs = 1.f, sn = 0.f;
  if (rope_mode != 2) {
    const float2 w = rope_cos_sin(static_cast<double>(t) * exp(-(2.0 * j / D) * log_base));
    cs = w.x;
    sn = w.y;
  }
  const size_t src = (static_cast<size_t>(bs) * T + t) * D;
  const size_t dst = (static_cast<size_t>(bs) * cap + t % cap) * D;
  const float k1 = ld_elem<BF16>(k, src + j), k2 = ld_elem<BF16>(k, src + j + D / 2);
  st_elem<BF16>(k_cache, dst + j, k1 * cs - k2 * sn);
  st_elem<BF16>(k_cache, dst + j + D / 2, k2 * cs + k1 * sn);
  st_elem<BF16>(v_cache, dst + j, ld_elem<BF16>(v, src + j));
  st_elem<BF16>(v_cache, dst + j + D / 2, ld_elem<BF16>(v, src + j + D / 2));
}

struct SharedDecWs {
  float* part_acc;
  float* part_ml;
  size_t bytes;
};

static SharedDecWs carve_shared_dec(void* ws, int B, int Hs, int d, int cap) {
  const size_t BS = static_cast<size_t>(B) * Hs;
  const size_t np = dec_partials(BS, cap, d);
  Carver cv(ws);
  SharedDecWs w;
  w.part_acc = cv.take<float>(np * d);
  w.part_ml = cv.take<float>(np * 2);
  w.bytes = cv.off;
  return w;
}

size_t shared_decode_workspace_bytes(int B, int Hs, int d, int cap) {
  return carve_shared_dec(nullptr, B, Hs, d, cap).bytes;
}

template <int D, bool BF16>
static hipError_t run_shared_decode(const void* q, const void* k, const void* v, void* k_cache,
                                    void* v_cache, int32_t* cache_len, int B, int Hs, int cap,
                                    int window, float rope_base, int rope_mode, float scale,
                                    void* out, int out_dtype, int accumulate,
                                    int32_t* dev_status, void* ws, hipStream_t st) {
  const SharedDecWs w = carve_shared_dec(ws, B, Hs, D, cap);
  const int nc = dec_nchunk(static_cast<size_t>(B) * Hs, cap, D);
  const double log_base = rope_mode == 2 ? 0.0 : std::log(static_cast<double>(rope_base));
  const DecStep a{nullptr, nullptr, q, k, v, k_cache, v_cache, cache_len, nullptr, Hs, Hs, cap,
                  log_base, rope_mode, 0, window, scale * 1.4426950408889634f, nullptr, nullptr,
                  dev_status, nc, static_cast<long>(B) * Hs * nc <= kDecFineGroups, w.part_acc,
                  w.part_ml};
  const dim3 grid(static_cast<unsigned>(static_cast<size_t>(B) * Hs * nc));
  launch_k("decode_attn", k_decode_attn<D, BF16, 1, true>, grid, dim3(256), st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_dec_combine<D, true>(a, cache_len, B, 1, out, out_dtype, accumulate, st);
  return hipGetLastError();
}

hipError_t launch_shared_decode(const void* q, const void* k, const void* v, int dtype,
                                void* k_cache, void* v_cache, int32_t* cache_len, int B, int Hs,
                                int d, int cap, int window, float rope_base, int rope_mode,
                                float scale, void* out, int out_dtype, int accumulate,
                                int32_t* dev_status, void* ws, hipStream_t st) {
#define NAMOH_SDEC(DD, BF)                                                                    \
  return run_shared_decode<DD, BF>(q, k, v, k_cache, v_cache, cache_len, B, Hs, cap, window, \
                                   rope_base, rope_mode, scale, out, out_dtype, accumulate,  \
                                   dev_status, ws, st)
  if (dtype == 1) {
    if (d == 32) NAMOH_SDEC(32, true);
    if (d == 64) NAMOH_SDEC(64, true);
    NAMOH_SDEC(128, true);
  }
  if (d == 32) NAMOH_SDEC(32, false);
  if (d == 64) NAMOH_SDEC(64, false);
  NAMOH_SDEC(128, false);
#undef NAMOH_SDEC
}

hipError_t launch_shared_prefill_cache(const void* k, const void* v, int dtype, int B, int T,
                                       int Hs, int d, int cap, float rope_base, int rope_mode,
                                       void* k_cache, void* v_cache, int32_t* cache_len,
                                       hipStream_t st) {
  const long first = T > cap ? static_cast<long>(T) - cap : 0;
  const long nrows = static_cast<long>(B) * Hs * (T - first);
  const long threads = nrows * (d / 2);
  const unsigned grid = static_cast<unsigned>((threads + 255) / 256);
  const double log_base = rope_mode == 2 ? 0.0 : std::log(static_cast<double>(rope_base));
#define NAMOH_SPC(DD, BF)                                                                       \
  k_shared_prefill_cache<DD, BF><<<grid, 256, 0, st>>>(k, v, T, Hs, cap, first, log_base,       \
                                                        rope_mode, k_cache, v_cache, cache_len, \
                                                        nrows)
  if (dtype == 1) {
    if (d == 32) NAMOH_SPC(32, true);
    else if (d == 64) NAMOH_SPC(64, true);
    else NAMOH_SPC(128, true);
  } else {
    if (d == 32) NAMOH_SPC(32, false);
    else if (d == 64) NAMOH_SPC(64, false);
    else NAMOH_SPC(128, false);
  }
#undef NAMOH_SPC
  return hipGetLastError();
}

hipError_t launch_decode(const float* logits, const float* bias, const void* q, const void* k,
                         const void* v, int dtype, void* k_cache,
                         void* v_cache, int32_t* cache_len,
                         const int32_t* seq_pos, int B, int H, int K, int d,
                         int cap, float rope_base, int rope_mode,
                         int gate_mode, float scale, int32_t* topk_idx,
                         float* gates, void* out, int out_dtype,
                         int32_t* dev_status, void* ws, hipStream_t st) {
#define NAMOH_DEC(DD, BF)                                                               \
  return run_decode<DD, BF>(logits, bias, q, k, v, k_cache, v_cache, cache_len, seq_pos, B, H, \
                            K, cap, rope_base, rope_mode, gate_mode, scale, topk_idx,    \
                            gates, out, out_dtype, dev_status, ws, st)
  if (dtype == 1) {
    if (d == 32) NAMOH_DEC(32, true);
    if (d == 64) NAMOH_DEC(64, true);
    NAMOH_DEC(128, true);
  }
  if (d == 32) NAMOH_DEC(32, false);
  if (d == 64) NAMOH_DEC(64, false);
  NAMOH_DEC(128, false);
#undef NAMOH_DEC
}

hipError_t launch_decode_grouped(const float* logits, const void* q, const void* k, const void* v,
                                 void* k_cache, void* v_cache, int32_t* cache_len,
                                 const int32_t* seq_pos, int B, int H, int K, int G, int d, int cap,
                                 float rope_base, int rope_mode, int gate_mode, float scale,
                                 int32_t* topk_idx, float* gates, void* out, int out_dtype,
                                 int32_t* dev_status, void* ws, hipStream_t st) {
#define NAMOH_DECG(DD, GG)                                                                    \
  return run_decode<DD, true, GG>(logits, nullptr, q, k, v, k_cache, v_cache, cache_len, seq_pos, \
                                  B, H, K, cap, rope_base, rope_mode, gate_mode, scale, topk_idx, \
                                  gates, out, out_dtype, dev_status, ws, st)
  if (d == 64) {
    if (G == 1) NAMOH_DECG(64, 1);
    if (G == 2) NAMOH_DECG(64, 2);
    if (G == 4) NAMOH_DECG(64, 4);
    if (G == 8) NAMOH_DECG(64, 8);
  } else if (d == 128) {
    if (G == 1) NAMOH_DECG(128, 1);
    if (G == 2) NAMOH_DECG(128, 2);
    if (G == 4) NAMOH_DECG(128, 4);
    if (G == 8) NAMOH_DECG(128, 8);
  }
#undef NAMOH_DECG
  return hipErrorInvalidValue;
}

}  // namespace namoh
