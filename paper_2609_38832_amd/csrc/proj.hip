// Routed per-head projections (Sec. 3.1, Eq. namoh-qkv, and the output
// aggregation of Eq. namoh-attention with W_O^(i) kept).
//
// Tokens are dispatched to their heads before projection: for every
// (batch b, head i) segment the packed rows r < n_{b,i} are the tokens of the
// ordered index set I_i, and only those pairs are projected.
//
//   k_proj_tile<QKV>  [q|k|v]_{t,i} = x_t W_QKV[i]^T for the segment's rows:
//                     a grouped GEMM (M = sum over b of n_{b,i}, N = 3d,
//                     K = d_model) whose data rows are gathered by token;
//                     the 8-column runs of each result row go straight to
//                     the dense q, k, v rows of the pair (other rows are
//                     never written).
//   k_out_map +       dense output projection (out_dense): the tokens'
//   k_proj_tile<OUT>  gated head rows against the stacked W_O over all heads.
//   k_proj_gemm +     per-pair output projection (otherwise): Y_r = h_r
//   k_combine         W_O[i]^T for every packed head-output row r (bf16 rows
//                     in packed order), then o_t = sum_k g_{t,k}
//                     Y[slot_pos(t,k)] in k order.
//
// The products are formed transposed, C^T = W X^T, on
// v_mfma_f32_32x32x16_bf16 (weights as the A operand, data rows as the B
// operand; operand order in tile.h), so each lane holds 16 output columns of
// one data row, as four runs of 4 consecutive columns.  K is walked in
// chunks of 64 staged through LDS (rows of 128 bytes with the 64-bank
// granule swizzle).  fp32 accumulation; operands bf16.
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "tile.h"

namespace namoh {

constexpr int kProjRows = 128;       // data rows per workgroup (4 waves x 32)
constexpr int kProjKC = 64;          // reduction chunk
constexpr int kProjThreads = 256;
constexpr int kProjSegLds = 1024;    // segment offsets staged in LDS up to this many

enum ProjMode { kProjQKV = 0, kProjOut = 1 };

// Packed 128-row tiles of segment s are numbered from seg0 / 128 + s (the
// same argument as seg_tile0 for 64-row tiles: disjoint, increasing, below
// Nr / 128 + BH + 1).
NAMOH_DEV int seg_ptile0(int seg0, int s) { return seg0 / kProjRows + s; }

template <int NT>
struct ProjLds {
  uint16_t w[NT * kProjKC];          // weight rows (output columns) x 64 k
  uint16_t x[kProjRows * kProjKC];   // data rows x 64 k
  int off[kProjSegLds + 1];
};

// Round 8 floats to bf16 (RNE) as one 16-byte granule.
NAMOH_DEV u32x4 f32x8_to_bf16(const float4 a, const float4 b) {
  return u32x4{pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y),
               pack_bf16x2(b.z, b.w)};
}

// Chunk k0 of the thread's data granules (rows xrow[e], 16-byte granule
// (tid + 256 e) % 8; padding rows ~0 give zeros) and weight granules (row
// (tid + 256 e) / 8 of wbase) into registers.
template <int XG, int WG, bool SRC_F32>
NAMOH_DEV void proj_load(u32x4 (&xr)[XG], u32x4 (&wr)[WG], const void* __restrict__ src,
                         const size_t (&xrow)[XG], const uint16_t* __restrict__ wbase, int kdim,
                         int k0, int tid) {
#pragma unroll
  for (int e = 0; e < XG; ++e) {
    const int gr = (tid + e * kProjThreads) % 8;
    xr[e] = u32x4{0u, 0u, 0u, 0u};
    if (xrow[e] != ~static_cast<size_t>(0)) {
      if constexpr (SRC_F32) {
        const float4* p =
            reinterpret_cast<const float4*>(static_cast<const float*>(src) + xrow[e] + k0 + 8 * gr);
        xr[e] = f32x8_to_bf16(p[0], p[1]);
      } else {
        xr[e] = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(src) + xrow[e] + k0 +
                                                8 * gr);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < WG; ++e) {
    const int u = tid + e * kProjThreads;
    wr[e] = *reinterpret_cast<const u32x4*>(wbase + static_cast<size_t>(u / 8) * kdim + k0 +
                                            8 * (u % 8));
  }
}

// Per-pair output projection: one workgroup computes 128 packed rows x NT
// columns of one segment with four waves of 32 rows; the next chunk is loaded
// into registers while the current one is multiplied from LDS.  src = packed
// head outputs [Nr, d] (f32 if SRC_F32, else bf16; rounded to bf16 as they
// are staged), w = W_O [H, d_model, d] bf16, kdim = d, N = d_model; output Y
// [Nr, d_model] bf16 (dst).
template <int NT, bool SRC_F32>
__global__ __launch_bounds__(kProjThreads, 2) void k_proj_gemm(
    const void* __restrict__ src, const uint16_t* __restrict__ w,
    const int32_t* __restrict__ seg_offsets, int BH, int H, int T, int Nr, int kdim, int N,
    uint16_t* __restrict__ dst) {
  static_assert(NT % 32 == 0 && (NT * kProjKC / 8) % kProjThreads == 0, "column tile");
  constexpr int CT = NT / 32;                                  // 32-column MFMA tiles
  constexpr int XG = kProjRows * kProjKC / 8 / kProjThreads;   // data granules per thread
  constexpr int WG = NT * kProjKC / 8 / kProjThreads;          // weight granules per thread
  __shared__ __attribute__((aligned(16))) ProjLds<NT> L;
  const int tid = thread_x();
  const int lane = tid % kWave, wave = tid / kWave;
  const int c = lane & 31, g = lane >> 5;
  const int gt = block_x();
  const int n0 = static_cast<int>(__builtin_amdgcn_workgroup_id_y()) * NT;

  // ---- segment of row tile gt (as in the packing kernel) ------------------
  const bool in_lds = BH <= kProjSegLds;
  if (in_lds)
    for (int i = tid; i <= BH; i += kProjThreads) L.off[i] = seg_offsets[i];
  __syncthreads();
  const int32_t* off = in_lds ? L.off : seg_offsets;
  int s;
  if (in_lds) {
    int cnt = 0;
    for (int s0 = 0; s0 < BH; s0 += kWave) {
      const int si = s0 + lane;
      cnt += __popcll(__ballot(si < BH && seg_ptile0(off[si], si) <= gt));
    }
    s = cnt - 1;
  } else {
    int lo = 0, hi = BH;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (seg_ptile0(off[mid], mid) <= gt) lo = mid; else hi = mid;
    }
    s = lo;
  }
  const int seg0 = off[s];
  const int n = off[s + 1] - seg0;
  const int r0 = (gt - seg_ptile0(seg0, s)) * kProjRows;
  // a tile in a gap between segments, or offsets that are not a packing
  if (r0 < 0 || r0 >= n || seg0 < 0 || n > T || seg0 + n > Nr) return;
  const int hh = s - (s / H) * H;

  // ---- the thread's data rows and weight rows -----------------------------
  // data granule u = tid + 256 e: row u / 8, 16-byte granule u % 8 of the
  // chunk; weight granule likewise over NT rows
  size_t xrow[XG];   // element offset of the row's start in src (or ~0: padding)
#pragma unroll
  for (int e = 0; e < XG; ++e) {
    const int r = r0 + (tid + e * kProjThreads) / 8;
    xrow[e] = ~static_cast<size_t>(0);
    if (r < n) xrow[e] = static_cast<size_t>(seg0 + r) * kdim;
  }
  const uint16_t* wbase = w + (static_cast<size_t>(hh) * N + n0) * kdim;

  u32x4 xr[XG], wr[WG];
  f32x16 C[CT];
#pragma unroll
  for (int t2 = 0; t2 < CT; ++t2)
#pragma unroll
    for (int e = 0; e < 16; ++e) C[t2][e] = 0.f;

  proj_load<XG, WG, SRC_F32>(xr, wr, src, xrow, wbase, kdim, 0, tid);
  const int drow = 32 * wave + c;   // this lane's data row in the tile (B operand column)
  for (int k0 = 0; k0 < kdim; k0 += kProjKC) {
    __syncthreads();            // the previous chunk's operand reads are done
#pragma unroll
    for (int e = 0; e < XG; ++e) {
      const int u = tid + e * kProjThreads, row = u / 8;
      *reinterpret_cast<u32x4*>(&L.x[row * kProjKC + swz<8>(row, u % 8) * 8]) = xr[e];
    }
#pragma unroll
    for (int e = 0; e < WG; ++e) {
      const int u = tid + e * kProjThreads, row = u / 8;
      *reinterpret_cast<u32x4*>(&L.w[row * kProjKC + swz<8>(row, u % 8) * 8]) = wr[e];
    }
    __syncthreads();
    if (k0 + kProjKC < kdim) proj_load<XG, WG, SRC_F32>(xr, wr, src, xrow, wbase, kdim, k0 + kProjKC, tid);
#pragma unroll
    for (int ks = 0; ks < kProjKC / 16; ++ks) {
      const bf16x8 bx =
          *reinterpret_cast<const bf16x8*>(&L.x[drow * kProjKC + swz<8>(drow, 2 * ks + g) * 8]);
#pragma unroll
      for (int t2 = 0; t2 < CT; ++t2) {
        const int wrow = 32 * t2 + c;
        const bf16x8 aw =
            *reinterpret_cast<const bf16x8*>(&L.w[wrow * kProjKC + swz<8>(wrow, 2 * ks + g) * 8]);
        C[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aw, bx, C[t2], 0, 0, 0);
      }
    }
  }

  // ---- epilogue: lane (c, g) holds data row drow, output columns
  // n0 + 32 t2 + 8 j + 4 g + i (i < 4) in accumulator 4 j + i ---------------
  const int r = r0 + drow;
  if (r >= n) return;
  {
    const size_t orow = static_cast<size_t>(seg0 + r) * N;
#pragma unroll
    for (int t2 = 0; t2 < CT; ++t2)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = n0 + 32 * t2 + 8 * j + 4 * g;
        *reinterpret_cast<uint2*>(dst + orow + col) =
            make_uint2(pack_bf16x2(C[t2][4 * j], C[t2][4 * j + 1]),
                       pack_bf16x2(C[t2][4 * j + 2], C[t2][4 * j + 3]));
      }
  }
}

// ---------------------------------------------------------------------------
// Output projection as one dense product over all heads of a token tile:
// o_t = sum_i [i selected for t] (g_{t,i} h_{t,i}) W_O[i]^T is the product of
// the gated head rows, laid out as a [B*T, H*d] operand whose blocks of
// unselected heads are zero, with the stacked weights [H*d, d_model].  That is
// H/K times the multiply-adds of the per-pair form, but no per-pair rows go
// through HBM: each token's gated rows are gathered straight into the operand
// tile, and the sum over the token's heads is the MFMA accumulation (head
// order, fp32).  Chosen when H*d is small against K (see out_dense).
//
// k_out_map (32 tokens per workgroup): map[t * H + i] = packed row of head i
// for token t, or Nr when i is not selected (the head of a packed row is that
// of its segment: largest j with seg_offsets[j] <= row, head j % H); the
// gated rows G[r] = g h_r rounded to bf16 for every routed pair (r =
// slot_pos[t, k], g = gates[t, k]); and G[Nr] = 0, the row every unselected
// head reads.
constexpr int kMapTokens = 32;

template <bool SRC_F32>
__global__ __launch_bounds__(256) void k_out_map(
    const void* __restrict__ head_out, const float* __restrict__ gates,
    const int32_t* __restrict__ slot_pos, const int32_t* __restrict__ seg_offsets, long BT, int H,
    int K, int BH, int Nr, int d, int32_t* __restrict__ map, uint16_t* __restrict__ grows) {
  __shared__ int s_off[kProjSegLds + 1];
  __shared__ int s_tbl[kMapTokens * 64];
  __shared__ int s_row[kMapTokens * 64];
  __shared__ float s_gate[kMapTokens * 64];
  const int tid = thread_x();
  const long t0 = static_cast<long>(block_x()) * kMapTokens;
  const int nt = static_cast<int>(min(static_cast<long>(kMapTokens), BT - t0));
  const bool in_lds = BH <= kProjSegLds;
  if (in_lds)
    for (int i = tid; i <= BH; i += 256) s_off[i] = seg_offsets[i];
  for (int i = tid; i < nt * H; i += 256) s_tbl[i] = Nr;
  if (block_x() == 0)
    for (int i = tid; i < d / 8; i += 256)
      *reinterpret_cast<u32x4*>(grows + static_cast<size_t>(Nr) * d + 8 * i) = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  const int32_t* off = in_lds ? s_off : seg_offsets;
  for (int i = tid; i < nt * K; i += 256) {
    const size_t gi = static_cast<size_t>(t0) * K + i;
    const int r = slot_pos[gi];
    const bool ok = r >= 0 && r < Nr;
    s_row[i] = ok ? r : -1;
    s_gate[i] = gates[gi];
    if (!ok) continue;
    int lo = 0, hi = BH;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (off[mid] <= r) lo = mid; else hi = mid;
    }
    s_tbl[(i / K) * H + lo % H] = r;
  }
  __syncthreads();
  for (int i = tid; i < nt * H; i += 256) map[static_cast<size_t>(t0) * H + i] = s_tbl[i];
  const int g8 = d / 8;
  for (int u = tid; u < nt * K * g8; u += 256) {
    const int i = u / g8, q = u - (u / g8) * g8;
    const int r = s_row[i];
    if (r < 0) continue;
    const float g = s_gate[i];
    const size_t o = static_cast<size_t>(r) * d + 8 * q;
    float f[8];
    if constexpr (SRC_F32) {
      const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(head_out) + o);
      const float4 a = p[0], b = p[1];
      f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    } else {
      const u32x4 h = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(head_out) + o);
      const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f[2 * e] = lo_bf16(hw[e]);
        f[2 * e + 1] = hi_bf16(hw[e]);
      }
    }
    *reinterpret_cast<u32x4*>(grows + o) =
        u32x4{pack_bf16x2(g * f[0], g * f[1]), pack_bf16x2(g * f[2], g * f[3]),
              pack_bf16x2(g * f[4], g * f[5]), pack_bf16x2(g * f[6], g * f[7])};
  }
}

// ---------------------------------------------------------------------------
// Tiled GEMM of both projections: a workgroup computes TM data rows x TN
// output columns with WM x WN waves (8 waves of 64 rows x TN / 2 columns, two
// per SIMD; short launches: see kSmallTM).  The reduction runs in chunks of 64
// through LDS stages (two; small tiles: rounds of three) that are filled straight from
// memory (no staging registers, no LDS stores), one whole 128-byte line per
// row: chunks of 32 (half lines, four stages) asked
// the L2 for every line twice and ran at 8 TB/s of L2 traffic, Q/K/V 151 us
// against 140 us at d_model 2048.  Every unselected head's row lies outside
// the OUT buffer, so three quarters of its data loads (K = H / 4) cost no
// memory traffic.  What bounds it now: with all data rows in the L2 Q/K/V
// still takes 117 of 121 us, without any load 105 us, of which about 10 us a
// tile are its prologue (offsets, tokens, first chunk: three dependent
// round trips) and epilogue, as one workgroup holds a compute unit's LDS.
// Measured, staged through registers before (one wave of 128 x TN / 2 per
// SIMD) and now: B T = 16384, H 32, K 8, d 64, d_model 2048: Q/K/V 160 ->
// 121 us (0.85 PFLOP/s), output 157 -> 114 us (1.2 PFLOP/s executed); B T =
// 6002, d 128, d_model 4096: Q/K/V 192 -> 172 us.  Waves of 128 x TN / 2 (one
// per SIMD) 139 / 151 us, two workgroups of 128 rows per compute unit 135 us.
//   kProjQKV: the data rows are 256-row pieces of a head's routed tokens, the
//     sequences of the batch one after another (only each head's last tile is
//     padded, not each segment's); gathered x rows; columns of W_QKV[h].
//   kProjOut: the data rows are consecutive tokens; the reduction runs over
//     H * d (chunk c belongs to head c / (d / 64)); the rows are the tokens'
//     gated head rows G found through the head map (the zero row for
//     unselected heads).
constexpr int kXcds = 8;        // XCDs of the device; workgroup i runs on XCD i % 8
constexpr int kXcdCus = 32;     // compute units of an XCD
constexpr int kTileKC = 64;     // reduction chunk: 128-byte LDS rows, one memory line each
constexpr int kTileMaxB = 256;  // sequences whose row counts are staged (more: per-segment tiles)

template <int TM>
NAMOH_DEV int seg_btile0(int seg0, int s) { return seg0 / TM + s; }

// Largest head count whose map tile fits beside the stages of a TN-wide tile.
constexpr int tile_map_heads(int TN) { return TN == 256 ? 32 : 64; }

template <int TM, int TN, int HM, int ST>
struct TileLds {
  // stage: TM data rows, then TN weight rows, of 64 elements each, their
  // 16-byte granules swizzled (swz<8>)
  uint16_t ring[ST][(TM + TN) * kTileKC];
  int32_t map[TM * HM];                 // OUT: head map [h][row]
};
template <int TM, int TN, int ST>
struct TileLds<TM, TN, 0, ST> {
  uint16_t ring[ST][(TM + TN) * kTileKC];
};

// 16 bytes per lane straight into LDS (lane l at lds + 16 l).  Inline
// assembly: see lds_dma16.
NAMOH_DEV void lds_dma16_global(const uint16_t* p, uint32_t lds) {
  asm volatile("global_load_lds_dwordx4 %1, off" ::"{m0}"(lds), "v"(p) : "memory");
}

// Tiles run one per compute unit, so a last round that fills at most half of
// the units would leave the others idle for a whole tile: its tiles are split
// into two halves of TM / 2 rows, two workgroups each.  Workgroup i of a group
// with n tiles on `units` compute units: its tile (>= n: none) and half (-1:
// the whole tile).
struct TailTile { int tile, half; };
NAMOH_DEV TailTile tail_tile(int i, int n, int units) {
  const int rem = n % units, full = n - rem;
  if (rem == 0 || 2 * rem > units || i < full) return {i, -1};
  const int u = i - full;
  return {u < 2 * rem ? full + u % rem : n, u / rem};
}
// The rows of that half (r0, nrow: the whole tile's); false if it has none.
template <int TM, typename R>
NAMOH_DEV bool take_half(int half, R& r0, int& nrow) {
  if (half < 0) return true;
  r0 += half * (TM / 2);
  nrow = min(TM / 2, nrow - half * (TM / 2));
  return nrow > 0;
}

template <int MODE, int TM, int TN, int WM, int WN, int OCC, bool OUT_BF16, int ST = 2>
__global__ __launch_bounds__(WM * WN * kWave, OCC) void k_proj_tile(
    const uint16_t* __restrict__ src, const uint16_t* __restrict__ w,
    const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ perm_token,
    const int32_t* __restrict__ map, int B, int H, int T, long BT, int Nr, int kdim, int N, int d,
    int n_col_tiles, int by_head, void* __restrict__ dst0, void* __restrict__ dst1,
    void* __restrict__ dst2) {
  constexpr int NW = WM * WN, NT = NW * kWave;     // TM / WM rows x TN / WN columns per wave
  constexpr int CT = TN / WN / 32;                 // 32-column tiles per wave
  constexpr int WI = TN / 8 / NW;                  // 1 KB weight loads per wave and chunk
  constexpr int STAGE = (TM + TN) * kTileKC * 2;   // bytes
  constexpr int HM = MODE == kProjOut ? tile_map_heads(TN) : 0;
  static_assert(TM == WM * 64 && NW % 2 == 0 && TM / 2 % (8 * NW) == 0 && WI * NW * 8 == TN && CT * WN * 32 == TN,
                "tile shape");
  __shared__ __attribute__((aligned(16))) TileLds<TM, TN, HM, ST> L;
  static_assert(sizeof(TileLds<TM, TN, HM, ST>) <= 160 * 1024, "LDS");
  const int tid = thread_x();
  const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c = lane & 31, g = lane >> 5;
  const int wr = wave / WN, wc = wave % WN;
  const int bid = block_x();

  // ---- the tile's data rows -------------------------------------------------
  int hh = 0, n0, nrow;
  long t0 = 0;
  if constexpr (MODE == kProjQKV) {
    // staged in the ring before it is used
    int* rowbt = reinterpret_cast<int*>(&L.ring[0][0]);  // b * T + t of the tile's rows
    int* cum = rowbt + TM;
    int* off = cum + 2 * kTileMaxB;                      // segment offsets
    static_assert((TM + 2 * kTileMaxB + kTileMaxB * 64 + 1) * 4 <= sizeof(L.ring) &&
                  NW * kWave <= 2 * kTileMaxB, "staging");
    if (by_head != 0) {
      // tiles of all heads in head order; workgroup bid runs on XCD bid % 8
      // (dispatch is round-robin over the XCDs), and each XCD takes one
      // contiguous eighth of the tiles, so its L2 holds the weights of few
      // heads at a time and all XCDs have the same number of tiles.  Lane h of
      // wave v sums head h's rows over the sequences b = v, v + NW, ...
      for (int i = tid; i <= B * H; i += NT) off[i] = seg_offsets[i];
      __syncthreads();
      int sum = 0;
      for (int b = wave; b < B; b += NW) {
        const int s = b * H + min(lane, H - 1);
        sum += min(max(off[s + 1] - off[s], 0), T);
      }
      cum[wave * kWave + lane] = sum;
      __syncthreads();
      int rows = 0;
#pragma unroll
      for (int v = 0; v < NW; ++v) rows += cum[v * kWave + lane];
      __syncthreads();
      const int nt = lane < H ? (rows + TM - 1) / TM * n_col_tiles : 0;
      const int incl = wave_inclusive_scan(nt);
      const int ntiles = __builtin_amdgcn_readlane(incl, kWave - 1);
      const int per = (ntiles + kXcds - 1) / kXcds;
      const TailTile tt = tail_tile(bid / kXcds, per, kXcdCus);
      const int tile = (bid % kXcds) * per + tt.tile;
      if (tt.tile >= per || tile >= ntiles) return;
      hh = __popcll(__ballot(incl <= tile));
      const int total = __shfl(rows, hh);
      const int i = tile - __shfl(incl - nt, hh);   // tile of the head: rows first, then columns
      const int j = i / n_col_tiles;
      n0 = (i - j * n_col_tiles) * TN;
      // rows before sequence b of this head (wave 0)
      if (wave == 0) {
        int base = 0;
        for (int b0 = 0; b0 < B; b0 += kWave) {
          const int b = b0 + lane, s = min(b, B - 1) * H + hh;
          const int n = b < B ? min(max(off[s + 1] - off[s], 0), T) : 0;
          const int incl = wave_inclusive_scan(n);
          if (b < B) cum[b] = base + incl - n;
          base += __builtin_amdgcn_readfirstlane(__shfl(incl, kWave - 1));
        }
      }
      __syncthreads();
      int r0 = j * TM;
      nrow = min(TM, total - r0);
      if (!take_half<TM>(tt.half, r0, nrow)) return;
      for (int r = tid; r < TM; r += NT) {
        // padding rows repeat the last row (their results are never stored)
        const int rr = r0 + min(r, nrow - 1);
        int lo = 0, hi = B;
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (cum[mid] <= rr) lo = mid; else hi = mid;
        }
        const unsigned p = static_cast<unsigned>(off[lo * H + hh] + rr - cum[lo]);
        const unsigned t = perm_token[min(p, static_cast<unsigned>(Nr - 1))];
        rowbt[r] = lo * T + static_cast<int>(min(t, static_cast<unsigned>(T - 1)));
      }
      __syncthreads();
    } else {
      // many sequences: tiles of each segment, numbered seg0 / TM + s
      const int rt0 = bid / n_col_tiles;
      n0 = (bid - rt0 * n_col_tiles) * TN;
      int lo = 0, hi = B * H;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg_btile0<TM>(seg_offsets[mid], mid) <= rt0) lo = mid; else hi = mid;
      }
      const int seg0 = seg_offsets[lo], n = seg_offsets[lo + 1] - seg0;
      const int r0 = (rt0 - seg_btile0<TM>(seg0, lo)) * TM;
      if (r0 < 0 || r0 >= n || seg0 < 0 || n > T || seg0 + n > Nr) return;
      hh = lo % H;
      nrow = min(TM, n - r0);
      for (int r = tid; r < TM; r += NT) {
        const unsigned t = perm_token[seg0 + r0 + min(r, nrow - 1)];
        rowbt[r] = (lo / H) * T + static_cast<int>(min(t, static_cast<unsigned>(T - 1)));
      }
      __syncthreads();
    }
  } else {
    const int ntiles = static_cast<int>((BT + TM - 1) / TM) * n_col_tiles;
    const TailTile tt = tail_tile(bid, ntiles, kXcds * kXcdCus);
    if (tt.tile >= ntiles) return;
    const int rt0 = tt.tile / n_col_tiles;
    n0 = (tt.tile - rt0 * n_col_tiles) * TN;
    t0 = static_cast<long>(rt0) * TM;
    nrow = static_cast<int>(min(static_cast<long>(TM), BT - t0));
    if (!take_half<TM>(tt.half, t0, nrow)) return;
    // the tile's head map, head-major (rows past the end repeat the last row;
    // their results are never stored)
    for (int i = tid; i < TM * H; i += NT) {
      const int row = i % TM, h = i / TM;
      const int32_t m = map[(static_cast<size_t>(t0) + min(row, nrow - 1)) * H + h];
      L.map[i] = static_cast<unsigned>(m) <= static_cast<unsigned>(Nr) ? m : Nr;
    }
    __syncthreads();
  }
  hh = __builtin_amdgcn_readfirstlane(hh);
  n0 = __builtin_amdgcn_readfirstlane(n0);
  const int cph = d / kTileKC;                         // chunks per head (OUT)
  const int nchunk = MODE == kProjQKV ? kdim / kTileKC : H * cph;

  // The tile with RT 32-row blocks per wave: 2, or 1 for tiles of at most
  // TM / 2 rows (split tails, a head's last rows).
  auto body = [&](auto rtc) {
  constexpr int RT = decltype(rtc)::value;
  constexpr int XI = RT * WM * 4 / NW;                 // 1 KB data loads per wave and chunk
  // ---- loads ------------------------------------------------------------------
  // load i of a wave fills LDS rows 8 (i NW + wave) .. + 7 of the tile; the
  // lane that fills position p of row r fetches granule swz<8>(r, p), the same
  // for all i
  const int xr = 8 * wave + lane / 8;                  // row of load 0 (load i: + 8 NW i)
  const int lg = swz<8>(xr, lane & 7);
  const uint32_t ring0 = lds_address(&L.ring[0][0]) + wave * 1024;
  size_t xo[XI];                                       // QKV: byte offset of the rows' granules
  int xm[XI];                                          // OUT: the rows' packed rows, next head
  int ebt[RT];                                         // QKV: the lane's result rows
  if constexpr (MODE == kProjQKV) {
    const int* rowbt = reinterpret_cast<const int*>(&L.ring[0][0]);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) ebt[rt] = rowbt[(32 * RT) * wr + 32 * rt + c];
#pragma unroll
    for (int i = 0; i < XI; ++i)
      xo[i] = (static_cast<size_t>(rowbt[xr + 8 * NW * i]) * kdim + 8 * lg) * 2;
    __syncthreads();   // the staged rows are read; the ring may be written
  }
  const int wstride = MODE == kProjQKV ? kdim : d;     // elements of a weight row
  const uint32_t wvoff = static_cast<uint32_t>((xr * wstride + 8 * lg) * 2);
  const uint32_t wstep = static_cast<uint32_t>(8 * NW * wstride * 2);
  // Each workgroup starts the reduction at another chunk (up to 15 on): the
  // weight rows lie d_model elements apart, so workgroups in step would ask
  // for lines of the same few L2 channels at once (d_model 2048: 131 -> 121
  // us, 4096: 179 -> 172 us; offsets over the whole reduction lose the L2 hits
  // that workgroups near one another share, 199 us).
  const int rot = MODE == kProjQKV ? ((bid / kXcds) & 15) % nchunk : 0;
  int ldc = rot, ldh = 0;     // next chunk to load; OUT: of head ldh
  const uint16_t* wb = w + (static_cast<size_t>(hh) * N + n0) * wstride;
  auto read_map = [&]() {
    if constexpr (MODE == kProjOut) {
#pragma unroll
      for (int i = 0; i < XI; ++i) xm[i] = L.map[ldh * TM + xr + 8 * NW * i];
    }
  };
  read_map();
  const bool far = MODE == kProjOut && (static_cast<size_t>(Nr) + 1) * d * 2 >= (1ull << 32);
  // load i of the data rows / weight rows of chunk ldc into a stage; next()
  auto load_x = [&](int stage, int i) {
    const uint32_t dst = ring0 + stage * STAGE + i * NW * 1024;
    const int koff = __builtin_amdgcn_readfirstlane(ldc * kTileKC * 2);
    if constexpr (MODE == kProjQKV) {
      lds_dma16_global(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(src) + koff + xo[i]), dst);
    } else if (far) {
      lds_dma16_global(src + static_cast<size_t>(xm[i]) * d + koff / 2 + 8 * lg, dst);
    } else {
      // rows of unselected heads (Nr) lie past the buffer's end and read as zero
      lds_dma16(buffer_rsrc(src, static_cast<uint32_t>(Nr) * d * 2), dst,
                static_cast<uint32_t>(xm[i]) * static_cast<uint32_t>(d * 2) + 16 * lg, koff);
    }
  };
  auto load_w = [&](int stage, int i) {
    const int koff = __builtin_amdgcn_readfirstlane(ldc * kTileKC * 2);
    lds_dma16(buffer_rsrc(MODE == kProjQKV ? wb : wb + static_cast<size_t>(ldh) * N * d, 0xFFFFFFFFu),
              ring0 + stage * STAGE + TM * kTileKC * 2 + i * NW * 1024, wvoff + i * wstep, koff);
  };
  auto next = [&]() {
    ++ldc;
    if constexpr (MODE == kProjQKV) {
      if (ldc == nchunk) ldc = 0;
    } else if (ldc == cph) {
      ldc = 0;
      if (++ldh == H) ldh = 0;
      read_map();
    }
  };

  f32x16 C[CT][RT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int e = 0; e < 16; ++e) C[ct][rt][e] = 0.f;

  const int fx = (32 * RT) * wr + c, fw = TM + (TN / WN) * wc + c;
  bf16x8 bx[2][RT], aw[2][CT];
  auto read_frags = [&](int stage, int ks, int set) {
    const uint16_t* st = &L.ring[stage][0];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      bx[set][rt] = *reinterpret_cast<const bf16x8*>(st + (fx + 32 * rt) * kTileKC + swz<8>(c, 2 * ks + g) * 8);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      aw[set][ct] = *reinterpret_cast<const bf16x8*>(st + (fw + 32 * ct) * kTileKC + swz<8>(c, 2 * ks + g) * 8);
  };
  // the products of one step, `behind(k)` issued behind the k-th
  auto mfmas = [&](int set, auto behind) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        C[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aw[set][ct], bx[set][rt], C[ct][rt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        behind(ct * RT + rt);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto nothing = [](int) {};
  // publishes the stage whose loads are in flight: every wave's loads have
  // landed, and every wave's reads of the other stage have returned
  auto publish = [&]() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  if constexpr (ST > 2) {
    // Few tiles: what bounds them is the latency of the loads, so a round
    // loads ST chunks at once.  When all of them have landed (a full wait:
    // loads into LDS are only ever published that way, see tile_dma), every
    // wave takes its fragments of the whole round into registers; the second
    // barrier frees the stages, and the next round's loads run behind this
    // one's products.  Past the last chunk loads wrap around to valid rows
    // that no product uses.
    auto load_round = [&]() {
#pragma unroll
      for (int s = 0; s < ST; ++s) {
#pragma unroll
        for (int i = 0; i < XI; ++i) load_x(s, i);
#pragma unroll
        for (int i = 0; i < WI; ++i) load_w(s, i);
        next();
      }
    };
    load_round();
    for (int ch = 0; ch < nchunk; ch += ST) {
      publish();
      bf16x8 rx[ST][4][RT], rw[ST][4][CT];
#pragma unroll
      for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const uint16_t* st = &L.ring[s][0];
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            rx[s][ks][rt] = *reinterpret_cast<const bf16x8*>(st + (fx + 32 * rt) * kTileKC + swz<8>(c, 2 * ks + g) * 8);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            rw[s][ks][ct] = *reinterpret_cast<const bf16x8*>(st + (fw + 32 * ct) * kTileKC + swz<8>(c, 2 * ks + g) * 8);
        }
      publish();   // (no load is in flight: every wave's reads have returned)
      if (ch + ST < nchunk) load_round();
#pragma unroll
      for (int s = 0; s < ST; ++s) {
        if (ch + s >= nchunk) break;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              C[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rw[s][ks][ct], rx[s][ks][rt], C[ct][rt], 0, 0, 0);
      }
    }
  } else {
    // One chunk: four 16-wide steps, the fragments of the next one read during
    // each.  The barrier stands before the last step: it publishes the next
    // chunk, whose first fragments that step reads, and frees this chunk's
    // stage for the chunk after the next.  That one's loads go one behind each
    // product, the data rows (longer latency) in this step and the weight rows
    // in the first step of the next chunk: issued together they fill the load
    // queue and the waves stand before it instead of feeding the matrix units.
    static_assert(XI <= CT * RT && WI <= CT * RT, "a load behind each product");
  #pragma unroll
    for (int i = 0; i < XI; ++i) load_x(0, i);
  #pragma unroll
    for (int i = 0; i < WI; ++i) load_w(0, i);
    next();
    publish();
    read_frags(0, 0, 0);
    if (nchunk > 1)
  #pragma unroll
      for (int i = 0; i < XI; ++i) load_x(1, i);
    auto chunk = [&](int stage, bool more1, bool more2) {
      __builtin_amdgcn_sched_barrier(0);
      read_frags(stage, 1, 1);
      mfmas(0, [&](int k) { if (k < WI && more1) load_w(stage ^ 1, k); });
      next();
      read_frags(stage, 2, 0);
      mfmas(1, nothing);
      read_frags(stage, 3, 1);
      mfmas(0, nothing);
      publish();
      read_frags(stage ^ 1, 0, 0);
      mfmas(1, [&](int k) { if (k < XI && more2) load_x(stage, k); });
    };
    int ch = 0;
    for (; ch + 1 < nchunk; ch += 2) {
      chunk(0, true, ch + 2 < nchunk);
      chunk(1, ch + 2 < nchunk, ch + 3 < nchunk);
    }
    if (ch < nchunk) chunk(0, false, false);
  }

  // ---- epilogue: lane (c, g) holds data row 64 wr + 32 rt + c, output
  // columns n0 + TN/2 wc + 32 ct + 8 j + 4 g + i in accumulator 4 j + i; the
  // two halves of a wave swap runs so that a lane stores 8 consecutive
  // columns (j even: lanes g = 0, j odd: g = 1) -------------------------------
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int r = (32 * RT) * wr + 32 * rt + c;
    const bool ok = r < nrow;
    size_t orow;
    float chk = 0.f;
    if constexpr (MODE == kProjQKV) {
      const int bt = ebt[rt], b = bt / T;
      orow = ((static_cast<size_t>(b) * H + hh) * T + (bt - b * T)) * d;
    } else {
      orow = static_cast<size_t>(t0 + r) * N;
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const f32x16& A = C[ct][rt];
      const int col0 = n0 + (TN / WN) * wc + 32 * ct;
      if constexpr (MODE == kProjOut) {
#pragma unroll
        for (int e = 0; e < 16; ++e) chk = fmaf(A[e], 0.f, chk);   // NaN if one is not finite
      }
      if constexpr (MODE == kProjOut && !OUT_BF16) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (ok)
            *reinterpret_cast<float4*>(static_cast<float*>(dst0) + orow + col0 + 8 * j + 4 * g) =
                make_float4(A[4 * j], A[4 * j + 1], A[4 * j + 2], A[4 * j + 3]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
          uint32_t e0 = pack_bf16x2(A[4 * j], A[4 * j + 1]), e1 = pack_bf16x2(A[4 * j + 2], A[4 * j + 3]);
          uint32_t o0 = pack_bf16x2(A[4 * j + 4], A[4 * j + 5]), o1 = pack_bf16x2(A[4 * j + 6], A[4 * j + 7]);
          const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
          const u32x4 v = u32x4{s0[0], s1[0], s0[1], s1[1]};
          const int col = col0 + 8 * (j + g);
          if (!ok) continue;
          if constexpr (MODE == kProjQKV) {
            const int which = col / d, cc = col - which * d;   // an 8-column run inside q, k or v
            uint16_t* dst = static_cast<uint16_t*>(which == 0 ? dst0 : (which == 1 ? dst1 : dst2));
            *reinterpret_cast<u32x4*>(dst + orow + cc) = v;
          } else {
            *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(dst0) + orow + col) = v;
          }
        }
      }
    }
    if constexpr (MODE == kProjOut) {
      // A non-finite weight of a head that the token did not select met a zero
      // of its row: where a result is not finite it is formed again over the
      // selected heads alone (lane (c, g): its row, half of the wave's columns).
      if (__builtin_expect(__any(!(chk == 0.f)), 0)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the wave's stores are done
        constexpr int PER = OUT_BF16 ? 2 : 1;              // results per word
        const int col0 = n0 + (TN / WN) * wc + 16 * CT * g;
        const uint32_t* row = reinterpret_cast<const uint32_t*>(dst0) + (orow + col0) / PER;
        for (int x = 0; ok && x < 16 * CT; ++x) {
          uint32_t v = __hip_atomic_load(row + x / PER, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if constexpr (OUT_BF16) v = (x & 1) ? v & 0xFFFF0000u : v << 16;
          if ((v & 0x7F800000u) != 0x7F800000u) continue;
          float sum = 0.f;
          for (int h = 0; h < H; ++h) {
            const int m = L.map[h * TM + r];
            if (m == Nr) continue;
            const u32x4* a = reinterpret_cast<const u32x4*>(src + static_cast<size_t>(m) * d);
            const u32x4* b = reinterpret_cast<const u32x4*>(w + (static_cast<size_t>(h) * N + col0 + x) * d);
            for (int i = 0; i < d / 8; ++i) {
              const u32x4 av = a[i], bv = b[i];
#pragma unroll
              for (int e = 0; e < 4; ++e)
                sum = fmaf(hi_bf16(av[e]), hi_bf16(bv[e]), fmaf(lo_bf16(av[e]), lo_bf16(bv[e]), sum));
            }
          }
          if constexpr (OUT_BF16) static_cast<uint16_t*>(dst0)[orow + col0 + x] = f32_to_bf16(sum);
          else static_cast<float*>(dst0)[orow + col0 + x] = sum;
        }
      }
    }
  }
  };
  if (nrow <= TM / 2)
    body(std::integral_constant<int, 1>{});
  else
    body(std::integral_constant<int, 2>{});
}

// Workspace rule of the output projection: head map and gated rows, or the
// per-pair rows.
static bool out_ws_dense(int H, int K, int d) { return static_cast<long>(H) * d <= 384L * K && H <= 64; }
static size_t out_dense_bytes(int B, int T, int H, int K, int d) {
  return align_up(static_cast<size_t>(B) * T * H * sizeof(int32_t)) +
         align_up((static_cast<size_t>(B) * T * K + 1) * d * 2);
}
static size_t out_pair_bytes(int B, int T, int K, int d_model) {
  return align_up(static_cast<size_t>(B) * T * K * d_model * 2);
}
// The form.  The dense one executes H / K times the multiply-adds at matrix
// rate (1.1-1.2 PFLOP/s of them with full rounds of 256 x 256 tiles), the
// per-pair one writes and re-reads B T K rows of d_model.  Measured (us,
// dense against per-pair, d_model 2048): 8192 tokens H d = 512 K 63 / 92
// (d 64, H 32), 115 / 232 (d 128, H 32); 1024 K 59 / 58 (d 64) but 105 / 118
// (d 128: rows of 256 bytes, twice the products per row); 2048 K 99 / 70.
// With few tiles the dense form's serial reduction of H d stands alone on few
// compute units: 3000 tokens, d_model 512 (24 tiles) 33 / 19, d_model 2048
// (96 tiles) 39 / 42; at 1024 K, d 128: 96 tiles 65 / 51, 256 tiles as above.
// Where the workspace rule says per-pair, the dense form's map and rows fit
// into the per-pair rows' space except at the smallest d_model.
static bool out_dense(int B, int T, int H, int K, int d, int d_model) {
  if (out_ws_dense(H, K, d)) return true;
  const size_t tiles = (static_cast<size_t>(B) * T + 255) / 256 * (d_model / 256);
  const long lim = d == 128 && tiles >= 256 ? 1024 : 512;
  return static_cast<long>(H) * d <= lim * K && H <= 64 && tiles >= 96 &&
         out_dense_bytes(B, T, H, K, d) <= out_pair_bytes(B, T, K, d_model);
}

template <int TM, int TN, int WM, int WN, int OCC, int ST = 2>
static void launch_out_tile(const uint16_t* grows, const uint16_t* w_o, const int32_t* map, long BT,
                            int Nr, int H, int d, int d_model, void* out, bool out_bf16,
                            hipStream_t st) {
  const int nct = d_model / TN;
  const unsigned tiles = static_cast<unsigned>(((BT + TM - 1) / TM) * nct);
  constexpr unsigned units = kXcds * kXcdCus;
  const unsigned rem = tiles % units;
  const unsigned grid = tiles + (2 * rem <= units ? rem : 0);   // second halves of a split tail
  if (out_bf16)
    k_proj_tile<kProjOut, TM, TN, WM, WN, OCC, true, ST><<<grid, WM * WN * kWave, 0, st>>>(
        grows, w_o, nullptr, nullptr, map, 0, H, 0, BT, Nr, d, d_model, d, nct, 0, out, nullptr, nullptr);
  else
    k_proj_tile<kProjOut, TM, TN, WM, WN, OCC, false, ST><<<grid, WM * WN * kWave, 0, st>>>(
        grows, w_o, nullptr, nullptr, map, 0, H, 0, BT, Nr, d, d_model, d, nct, 0, out, nullptr, nullptr);
}

// ---------------------------------------------------------------------------
static unsigned proj_row_tiles(int B, int T, int H, int K) {
  const size_t Nr = static_cast<size_t>(B) * T * K;
  return static_cast<unsigned>(Nr / kProjRows + static_cast<size_t>(B) * H + 1);
}

template <int TM, int TN, int WM, int WN, int OCC, int ST = 2>
static void launch_qkv_tile(const uint16_t* x, const uint16_t* w, int B, int T, int H, int K, int d,
                            int d_model, const int32_t* seg_offsets, const int32_t* perm_token,
                            void* q, void* k, void* v, hipStream_t st) {
  const int N = 3 * d, nct = N / TN;
  // at most Nr / TM full tiles and one partial tile per head, dealt to the
  // XCDs in equal shares; or numbered by segment
  const size_t BT = static_cast<size_t>(B) * T;
  const bool by_head = B <= kTileMaxB;
  const size_t tiles = BT * K / TM + (by_head ? H : static_cast<size_t>(B) * H + 1);
  // (by head: and the second halves of a split tail)
  const size_t grid = by_head ? ((tiles * nct + kXcds - 1) / kXcds + kXcdCus / 2) * kXcds : tiles * nct;
  k_proj_tile<kProjQKV, TM, TN, WM, WN, OCC, false, ST><<<static_cast<unsigned>(grid), WM * WN * kWave, 0, st>>>(
      x, w, seg_offsets, perm_token, nullptr, B, H, T, static_cast<long>(BT), B * T * K, d_model, N,
      d, nct, by_head ? 1 : 0, q, k, v);
}

// Tiles of 128 x 64 with rounds of three chunks where a launch is short of
// 256-row tiles.  There a chunk costs the latency of its loads (0.8 us for
// Q/K/V, 1.0 us for the output, 32 of them in a row at d_model 2048), not its
// products: smaller tiles put more compute units on it, and a round pays the
// latency once for three chunks.  The lines lie where the small tiles stop
// fitting into one round of workgroups: two per compute unit for Q/K/V, one for
// the output (which holds the head map as well).  256-row tiles -> these, H 32,
// K 8, d 64, d_model 2048: Q/K/V 300 tokens 26 -> 14 us, 1000 29 -> 20, 2000
// (471 tiles) 30 -> 29, but 3000 (660) 32 -> 38; output 300 tokens 33 -> 19 us,
// 1000 (256 tiles) 35 -> 26.5, but 1200 (320) 35 -> 39.  d 128, d_model 4096:
// Q/K/V 300 tokens 48 -> 31, 700 52 -> 43, 1500 56 -> 72.
constexpr int kSmallTM = 128, kSmallTN = 64, kSmallStages = 3;
constexpr size_t kTileUnits = kXcds * kXcdCus;
static bool qkv_small(int B, int T, int H, int K, int d) {
  const size_t rows = static_cast<size_t>(B) * T * K / kSmallTM + H;
  return B <= kTileMaxB && rows * (3 * d / kSmallTN) <= 2 * kTileUnits;
}
static bool out_small(long BT, int d_model) {
  return static_cast<size_t>((BT + kSmallTM - 1) / kSmallTM) * (d_model / kSmallTN) <= kTileUnits;
}

hipError_t launch_qkv_proj(const void* x, const void* w_qkv, int B, int T, int H, int K, int d,
                           int d_model, const int32_t* seg_offsets, const int32_t* perm_token,
                           void* q, void* k, void* v, hipStream_t st) {
  if ((3 * d) % 192 != 0 || d_model % kProjKC != 0) return hipErrorInvalidValue;
  prof_mark("qkv_proj", true, st);
  const auto launch = qkv_small(B, T, H, K, d) ? launch_qkv_tile<kSmallTM, kSmallTN, 2, 2, 2, kSmallStages>
                                               : launch_qkv_tile<256, 192, 4, 2, 2>;
  launch(static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w_qkv), B, T, H, K, d, d_model,
         seg_offsets, perm_token, q, k, v, st);
  prof_mark("qkv_proj", false, st);
  return hipGetLastError();
}

size_t out_proj_workspace_bytes(int B, int T, int H, int K, int d, int d_model) {
  return out_ws_dense(H, K, d) ? out_dense_bytes(B, T, H, K, d) : out_pair_bytes(B, T, K, d_model);
}

hipError_t launch_out_proj(const void* head_out, int head_out_dtype, const void* w_o,
                           const float* gates, const int32_t* slot_pos,
                           const int32_t* seg_offsets, int B, int T, int H, int K, int d,
                           int d_model, void* out, int out_dtype, void* ws, hipStream_t st) {
  if (d % kProjKC != 0 || d_model % 128 != 0) return hipErrorInvalidValue;
  if (out_dense(B, T, H, K, d, d_model)) {
    const long BT = static_cast<long>(B) * T;
    int32_t* map = static_cast<int32_t*>(ws);
    uint16_t* grows = reinterpret_cast<uint16_t*>(static_cast<char*>(ws) +
                                                  align_up(static_cast<size_t>(BT) * H * sizeof(int32_t)));
    const unsigned mgrid = static_cast<unsigned>((BT + kMapTokens - 1) / kMapTokens);
    prof_mark("out_proj", true, st);
    if (head_out_dtype == 0)
      k_out_map<true><<<mgrid, 256, 0, st>>>(head_out, gates, slot_pos, seg_offsets, BT, H, K, B * H,
                                             B * T * K, d, map, grows);
    else
      k_out_map<false><<<mgrid, 256, 0, st>>>(head_out, gates, slot_pos, seg_offsets, BT, H, K, B * H,
                                              B * T * K, d, map, grows);
    const uint16_t* w = static_cast<const uint16_t*>(w_o);
    if (out_small(BT, d_model))
      launch_out_tile<kSmallTM, kSmallTN, 2, 2, 1, kSmallStages>(grows, w, map, BT, B * T * K, H, d, d_model,
                                                                 out, out_dtype == 1, st);
    else if (d_model % 256 == 0 && H <= tile_map_heads(256))
      launch_out_tile<256, 256, 4, 2, 2>(grows, w, map, BT, B * T * K, H, d, d_model, out, out_dtype == 1, st);
    else
      launch_out_tile<256, 128, 4, 2, 2>(grows, w, map, BT, B * T * K, H, d, d_model, out, out_dtype == 1, st);
    prof_mark("out_proj", false, st);
    return hipGetLastError();
  }
  uint16_t* Y = static_cast<uint16_t*>(ws);
  const dim3 grid(proj_row_tiles(B, T, H, K), static_cast<unsigned>(d_model / 128));
  prof_mark("out_proj", true, st);
  if (head_out_dtype == 0)
    k_proj_gemm<128, true><<<grid, kProjThreads, 0, st>>>(
        head_out, static_cast<const uint16_t*>(w_o), seg_offsets, B * H, H, T, B * T * K, d, d_model,
        Y);
  else
    k_proj_gemm<128, false><<<grid, kProjThreads, 0, st>>>(
        head_out, static_cast<const uint16_t*>(w_o), seg_offsets, B * H, H, T, B * T * K, d, d_model,
        Y);
  prof_mark("out_proj", false, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  prof_mark("out_combine", true, st);
  e = launch_combine_rows(Y, gates, slot_pos, static_cast<long>(B) * T, K, d_model, B * T * K,
                          out, out_dtype, st);
  prof_mark("out_combine", false, st);
  return e;
}

}  // namespace namoh
