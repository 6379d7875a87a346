// Chunk attention backward with the cached context detached (Sec. 3.3), bf16 MFMA with
// fp32 accumulation.  Two kernels (one for launches with few rows, below), no atomics, deterministic:
//   dq    : one workgroup per query tile, walks ALL visible keys (ring + chunk):
//             Delta[q] = <dO_q, O_q> (taken while the query's dO row is loaded, and
//             written out for the second kernel),
//             S^T = K Q~^T - LSE (Q~ arrives pre-multiplied by log2(e)/sqrt(D) and the accumulators
//             start from -LSE*log2(e): the product is the exponent of 2), P^T = exp2(S^T), dP^T = V dO^T,
//             dS^T = P^T o (dP^T - Delta), dQ~^T += K^T dS^T
//   dkv   : one workgroup per tile of CHUNK keys, walks all query tiles:
//             S = Q~ K~^T, P, dV^T += dO^T P, dP = dO V^T, dS, dK~^T += Q~^T dS
//           Cached keys / values get no gradient, so no workgroup exists for them.
// As in the forward every product is arranged so that the accumulator of one product is
// directly the B operand of the next, and the LDS tile of the other operand is read
// either by rows (contraction over D) or through the transposing read (contraction over
// the tile's rows).
#include "kernels.hpp"
#include "mfma_common.hpp"
#include "ring_state.hpp"

namespace astro {
namespace {

// Waves per dQ workgroup.  Eight (one workgroup per CU, half the tile traffic from L2) was
// measured slower, 4.87 vs 4.73 ms: a barrier over eight waves and a wider ragged last query tile.
constexpr int kDqWaves = 4;
constexpr int KT = kBwdKeyTile;  // rows per LDS tile

struct BwdParams {
  const __bf16* q_rot;
  const __bf16* kc_rot;
  const __bf16* v_chunk;
  const __bf16* k_cache;
  const __bf16* v_cache;
  const __bf16* out;
  const __bf16* dout;
  const float* lse;
  float* delta;   // [B][H][Nq]  -<dO, O>
  float* lse2;    // [B][H][Nq]  -LSE * log2(e), written next to delta by the dQ kernel
  float* dq;      // [B, Nq, H, D]  w.r.t. the un-rotated queries
  float* dk;      // [B, Nq, H, D]  w.r.t. the un-rotated chunk keys
  float* dv;      // [B, Nq, H, D]
  RotaryTables rot;
  int H, Nq, BH, tiles;  // BH = candidates * heads; tiles = workgroups per pair of the kernel being launched
  int group;             // candidates per cache stream
  int block_rows;        // causal block inside the chunk in token rows, 0 = none
  bool by_xcd;           // order of the workgroups, see order_by_xcd()
  bool terms_ready;      // few rows: delta and lse2 are there already
  int64_t cache_rows;
  float scale;
  FewDivisors div;  // few rows
  StreamInts hist_rows;
};

// ---- dQ -----------------------------------------------------------------------
// 16x16x32 MFMAs: a wave's 32 queries are two sub-blocks of 16 (qs); lane (i = lane % 16,
// g = lane / 16) holds, for queries 16*qs + i, the accumulator rows 4g .. 4g+3 of every 16-row tile.
template <int D>
struct DqWave {
  static constexpr int KS = D / 32;  // k-steps of a contraction over D
  static constexpr int DT = D / 16;  // 16-row tiles of dQ~^T
  bf16x8 qreg[2][KS], doreg[2][KS];  // B operands: Q~ and dO rows of this lane's two queries
  f32x4 neg_lse2[2];   // -LSE*log2(e) of the two queries, four copies: the accumulators of S start from it
  // -Delta of the two queries, four copies each: the accumulators of dP^T start from them, so
  // the product comes out as dP^T - Delta
  f32x4 neg_delta[2];
  f32x4 dq[DT][2];
  OperandAddr16<D> addr;
  int g;

  __device__ __forceinline__ void init(int lane) {
    g = lane >> 4;
    addr.init(lane);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) dq[dt][qs] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- the pieces of one 32-key block kb of a tile -------------------------------------
  // S^T - LSE*log2(e) = K Q~^T - LSE*log2(e): 16 MFMAs, each pair behind the read of its K fragment
  __device__ __forceinline__ void s_product(const char* ks, int kb, f32x4 (&s)[2][2]) const {
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        const bf16x8 a = read_rows16<D>(ks, addr.row[st], 32 * kb + 16 * kh);
#pragma unroll
        for (int qs = 0; qs < 2; ++qs) s[kh][qs] = mfma16(a, qreg[qs][st], st == 0 ? neg_lse2[qs] : s[kh][qs]);
      }
  }
  // keys of the block that do not count for a query: score replaced so that P and dS are exactly 0
  __device__ __forceinline__ void mask(int kb, const int (&live)[2], f32x4 (&s)[2][2]) const {
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int qs = 0; qs < 2; ++qs)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[kh][qs][r] = 32 * kb + 16 * kh + 4 * g + r >= live[qs] ? kNegBig : s[kh][qs][r];
  }
  // P^T = exp2(S^T - LSE*log2(e)), in place: 16 exponentials
  __device__ __forceinline__ void probabilities(f32x4 (&s)[2][2]) const {
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[kh][qs][r] = fast_exp2(s[kh][qs][r]);
  }
  // dP^T - Delta = V dO^T - Delta: 16 MFMAs
  __device__ __forceinline__ void dp_product(const char* vs, int kb, f32x4 (&dp)[2][2]) const {
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        const bf16x8 a = read_rows16<D>(vs, addr.row[st], 32 * kb + 16 * kh);
#pragma unroll
        for (int qs = 0; qs < 2; ++qs) dp[kh][qs] = mfma16(a, doreg[qs][st], st == 0 ? neg_delta[qs] : dp[kh][qs]);
      }
  }
  // dS^T = P^T o (dP^T - Delta) as the B operand of the next product (k-slots 8g .. 8g+3 <- keys
  // 4g .., k-slots 8g+4 .. <- keys 16 + 4g ..): 24 vector-ALU instructions
  __device__ __forceinline__ void ds_operand(const f32x4 (&pr)[2][2], const f32x4 (&dp)[2][2], bf16x8 (&dsb)[2]) const {
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int r = 0; r < 4; ++r) dsb[qs][4 * kh + r] = (__bf16)(pr[kh][qs][r] * dp[kh][qs][r]);
  }
  // dQ~^T[d][q] += K^T[d][key] dS^T[key][q]: 16 MFMAs
  __device__ __forceinline__ void dq_product(const char* ks, int kb, const bf16x8 (&dsb)[2]) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8 a = read_cols16<D>(ks, addr.tr[dt], 32 * kb);
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) dq[dt][qs] = mfma16(a, dsb[qs], dq[dt][qs]);
    }
  }

  // One 64-key tile of which the first live[qs] keys count for this lane's query qs (live_min,
  // wave-uniform: the fewest over the wave).  The others lie past the end of their segment
  // (zero rows in LDS) or in a causal block the query does not see; their score is replaced
  // so that P and dS are exactly 0 (left alone, P = exp(0 - LSE) could overflow for a query
  // whose logits are all very negative, and inf * 0 would poison dQ~ = dS K~).
  // Each product reads its operand fragments just ahead of its MFMAs.  Requesting the next
  // product's fragments one MFMA behind the current one (no product then starts by waiting for
  // LDS) was measured slower with the 32x32x16 kernel, 5.05 vs 4.93 ms: it needs all 256
  // registers and the kernel is not bound by LDS latency.
  // Vector-ALU instructions issue while an MFMA executes, also within one wave: the
  // exponentials (which need S only) sit between the MFMAs of the dP product, 4.56 -> 4.41 ms.
  // Going further lost: the dS operand of one query sub-block under the dQ MFMAs of the other
  // (K^T fragments held for both: all 256 registers, 4.64 ms); the scores of the next key block
  // carried along so that the dS operand sits under their MFMAs (spills in the tile loop, 7.4 ms);
  // the first two operand fragments of the dP and dQ products requested one phase early (4.54 vs 4.48 ms).
  __device__ __forceinline__ void tile(const char* ks, const char* vs, const int (&live)[2], int live_min) {
#pragma unroll
    for (int kb = 0; kb < KT / 32; ++kb) block(ks, vs, kb, live, live_min);
  }
  __device__ __forceinline__ void block(const char* ks, const char* vs, int kb, const int (&live)[2], int live_min) {
    f32x4 s[2][2], dp[2][2];  // [16-key half][query sub-block]
    bf16x8 dsb[2];
    s_product(ks, kb, s);
    if (live_min < 32 * (kb + 1)) mask(kb, live, s);
    // keep the phases apart: hoisting every LDS read of a key block to its top costs
    // more registers than two resident waves per SIMD have
    __builtin_amdgcn_sched_barrier(0);
    probabilities(s);
    dp_product(vs, kb, dp);
#pragma unroll
    for (int i = 0; i < 4 * KS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);  // one exponential
    }
    __builtin_amdgcn_sched_barrier(0);
    ds_operand(s, dp, dsb);
    __builtin_amdgcn_sched_barrier(0);
    dq_product(ks, kb, dsb);
  }

  // Q~ and dO rows of the lane's two queries from a block of 32 in LDS
  __device__ __forceinline__ void take_queries(const char* qtile, const char* dotile) {
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        qreg[qs][st] = read_rows16<D>(qtile, addr.row[st], 16 * qs);
        doreg[qs][st] = read_rows16<D>(dotile, addr.row[st], 16 * qs);
      }
  }

  // Q~ and dO rows of the lane's two queries, their row terms -LSE*log2(e) and -Delta; bh = stream-head
  // pair of the chunk tensors, write_terms: this wave leaves the row terms for later launches
  __device__ __forceinline__ void load_queries(const BwdParams& p, int b, int h, int q0, bool write_terms) {
    const int64_t bh = (int64_t)b * p.H + h;
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      const int q = q0 + 16 * qs;
      const bool live = q < p.Nq;
      const __bf16* qrow = p.q_rot + (bh * p.Nq + (live ? q : 0)) * D;
      const int64_t token_row = (((int64_t)b * p.Nq + (live ? q : 0)) * p.H + h) * D;
      const __bf16* drow = p.dout + token_row;
      const __bf16* orow = p.out + token_row;
      // Delta = <dO_q, O_q>: this lane holds the quarter 32*st + 8g .. +7 of the row, the lanes
      // i + 16, i + 32, i + 48 the others
      float dsum = 0.f;
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0}, y = x, o = x;
        if (live) {
          x = *reinterpret_cast<const bf16x8*>(qrow + st * 32 + g * 8);
          y = *reinterpret_cast<const bf16x8*>(drow + st * 32 + g * 8);
          o = *reinterpret_cast<const bf16x8*>(orow + st * 32 + g * 8);
        }
        qreg[qs][st] = x;
        doreg[qs][st] = y;
#pragma unroll
        for (int j = 0; j < 8; ++j) dsum = fmaf((float)y[j], (float)o[j], dsum);
      }
      dsum += __shfl_xor(dsum, 16);
      dsum += __shfl_xor(dsum, 32);
      // a dead query row gets P = exp2(0 - big) = 0 everywhere
      const float nl = live ? -p.lse[bh * p.Nq + q] * kLog2e : -1.0e30f;
      neg_lse2[qs] = f32x4{nl, nl, nl, nl};
      neg_delta[qs] = f32x4{-dsum, -dsum, -dsum, -dsum};
      // the row terms of the query, for the dK/dV kernel (negative there too)
      if (write_terms && live && g == 0) {
        p.delta[bh * p.Nq + q] = -dsum;
        p.lse2[bh * p.Nq + q] = nl;
      }
    }
  }
};

// Key split of launches that fill the CUs' places at most once and only in part (12 heads of one stream
// are 444 workgroups on 512 places: 68 CUs hold one workgroup and idle half of the launch; 3 heads are
// 111).  With `ways` = 2 the last 1 / (k + 1) of every item's key tiles go to helper workgroups, one per k
// items, so that all do the same number of tiles; with `ways` = 3 every item is cut in three and has two
// helpers.  Main and helpers leave fp32 partial sums that a small launch adds up and turns back.
// ways = 1: no split.
struct DqSplit {
  int ways, k;
  // [B, Nq, H, D]: the helpers' sums (the dK and dV outputs: the kernel that fills them runs later)
  float *part1, *part2;
  __host__ __device__ int helpers(int items) const { return ways == 3 ? 2 * items : (items + k - 1) / k; }
  // first tile of part `which` of an item of `ntiles` tiles (a helper of k items spends about two tiles on each besides)
  __device__ int first_tile(int which, int ntiles) const {
    if (ways == 3) return which * ntiles / 3;
    const int cut = (k * ntiles + 2 * (k - 1) + k) / (k + 1);
    return which == 0 ? 0 : (which == 1 && cut < ntiles ? cut : ntiles);
  }
};

// One item (kSplit: part `which` of it, 0 = the main workgroup's)
template <int D, int kWaves, bool kSplit>
__device__ __forceinline__ void dq_item(const BwdParams& p, const DqSplit& split, const WorkItem& item, int which, char* lds) {
  using Wave = DqWave<D>;
  constexpr int TILE_BYTES = KT * D * 2;
  const PairIndex pair = split_pair(item.bh, p.H, p.group);
  const int b = pair.b, h = pair.h;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g = lane >> 4;
  const int hist = p.hist_rows.v[pair.cache_b];
  const int q0 = (item.tile * kWaves + wave) * 32 + i16;  // this lane's queries: q0 and q0 + 16
  const int64_t bh = (int64_t)b * p.H + h;
  // chunk rows each of this lane's queries sees, the fewest any lane of the wave sees (its
  // first query) and the most any wave of the workgroup sees (its last query)
  const int q_last = p.Nq - 1;
  int vis[2];
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) vis[qs] = visible_chunk_rows(q0 + 16 * qs < q_last ? q0 + 16 * qs : q_last, p.Nq, p.block_rows);
  const int q_wave = (item.tile * kWaves + __builtin_amdgcn_readfirstlane(wave)) * 32;
  const int vis_wave = visible_chunk_rows(q_wave < q_last ? q_wave : q_last, p.Nq, p.block_rows);
  const int q_wg = (item.tile + 1) * kWaves * 32 - 1;
  const int vis_wg = visible_chunk_rows(q_wg < q_last ? q_wg : q_last, p.Nq, p.block_rows);
  const int hist_tiles = (hist + KT - 1) / KT;
  const int ntiles = hist_tiles + (vis_wg + KT - 1) / KT;
  const int t_begin = kSplit ? split.first_tile(which, ntiles) : 0;
  const int t_end = kSplit ? split.first_tile(which + 1, ntiles) : ntiles;

  Wave w;
  w.init(lane);
  w.load_queries(p, b, h, q0, which == 0);

  const RowSegment k_hist = make_segment(p.k_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const RowSegment v_hist = make_segment(p.v_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const RowSegment k_chunk = make_segment(p.kc_rot + bh * p.Nq * D, D, p.Nq, D);
  const RowSegment v_chunk = make_segment(p.v_chunk + ((int64_t)b * p.Nq * p.H + h) * D, (int64_t)p.H * D, p.Nq, D);
  TileStreamer<D, KT, kWaves> ts;
  ts.init();
  const uint32_t off_dense = ts.lane_offset(k_hist);
  const uint32_t off_vchunk = ts.lane_offset(v_chunk);
  auto issue = [&](int t) {
    char* kbuf = lds + ((t - t_begin) & 1) * 2 * TILE_BYTES;
    if (t < hist_tiles) {
      ts.issue(k_hist, off_dense, t * KT, kbuf);
      ts.issue(v_hist, off_dense, t * KT, kbuf + TILE_BYTES);
    } else {
      ts.issue(k_chunk, off_dense, (t - hist_tiles) * KT, kbuf);
      ts.issue(v_chunk, off_vchunk, (t - hist_tiles) * KT, kbuf + TILE_BYTES);
    }
  };
  if (t_begin < t_end) issue(t_begin);
  wait_vmem();
  __syncthreads();

  // two tiles per trip so that each LDS buffer is a compile-time offset of the operand reads
  auto step = [&](int t, auto buf_c) __attribute__((always_inline)) {
    if (t + 1 < t_end) issue(t + 1);
    const char* kbuf = lds + decltype(buf_c)::value * 2 * TILE_BYTES;
    int live[2];
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) live[qs] = t < hist_tiles ? hist - t * KT : vis[qs] - (t - hist_tiles) * KT;
    w.tile(kbuf, kbuf + TILE_BYTES, live, t < hist_tiles ? hist - t * KT : vis_wave - (t - hist_tiles) * KT);
    wait_vmem();
    __syncthreads();
  };
  for (int t = t_begin; t < t_end; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    if (t + 1 < t_end) step(t + 1, std::integral_constant<int, 1>{});
  }

  // dQ~ -> dQ: the rotation is turned back here (each lane holds both halves of its pairs), so the
  // gradient goes out once, token-major, instead of through a rotated fp32 copy and another pass
  const bool rope = !kSplit && p.rot.n_t + p.rot.n_h + p.rot.n_w != 0;
  // (Here a look-up stays with its store: all of them ahead of the first, as in dkv_wave(), gained nothing at 30 - 128 pairs and cost 0.7 % of a step
  // of four clips, 12 heads, 4680 rows, where 8608 us became 8665; the other workgroup of the CU
  // covers them.)
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) {
    const int q = q0 + 16 * qs;
    if (q < p.Nq) {
      float* row = (which == 0 ? p.dq : (which == 1 ? split.part1 : split.part2)) + (((int64_t)b * p.Nq + q) * p.H + h) * D;
      TokenTables tt{};
      if (rope) tt = token_tables(p.rot, b, q);
#pragma unroll
      for (int dt = 0; dt < Wave::DT; ++dt) {
        f32x4 x = w.dq[dt][qs];
        if constexpr (!kSplit) {
          x = x * p.scale;
          if (rope) x = unrotate_quad(p.rot, tt, 4 * dt + g, x);
        }
        *reinterpret_cast<f32x4*>(row + 16 * dt + 4 * g) = x;
      }
    }
  }
}

template <int D, int OCC, int kWaves, bool kSplit>
__global__ void __launch_bounds__(kWaves * 64, OCC) attn_bwd_dq_kernel(BwdParams p, DqSplit split) {
  __shared__ __attribute__((aligned(1024))) char lds[4 * KT * D * 2];  // K0 V0 K1 V1
  if constexpr (!kSplit) {
    const WorkItem item = work_item(p.tiles, p.BH, p.by_xcd);
    if (item.valid) dq_item<D, kWaves, false>(p, split, item, 0, lds);
  } else {
    // one loop for all, so that the code of an item is there once: a main workgroup and a helper of a cut in
    // three have one item, the others k consecutive ones (an XCD's helpers stay with one or two pairs)
    const int items = p.tiles * p.BH;
    const int block = (int)blockIdx.x;
    auto order = [&](int i, int n) { return p.by_xcd ? xcd_order(i, n) : i; };
    int which = 0, first, count = 1;
    if (block < items) {
      first = order(block, items);
    } else if (split.ways == 3) {
      which = block < 2 * items ? 1 : 2;
      first = order(block - which * items, items);
    } else {
      which = 1;
      first = order(block - items, split.helpers(items)) * split.k;
      count = items - first < split.k ? items - first : split.k;
    }
    for (int i = first; i < first + count; ++i) dq_item<D, kWaves, true>(p, split, WorkItem{i % p.tiles, i / p.tiles, true}, which, lds);
  }
}

// dQ = R(phi)^T (main + helper sums) / sqrt(D) of a split launch: bytes only (ways + 1 times dQ), four quads
// of D per thread in flight.  Look-ups ahead of the first store and divisions of 32 bits, us: two ways, 12 pairs of 128 20.0 ->
// 15.4, 16 of 64 15.1 -> 10.9; three, 3 pairs of 128 8.7 -> 6.4, 14 23.8 -> 22.8, 4 of 64 7.2 -> 5.4 (81 registers instead of 62).
template <int D, int kWays>
__global__ void __launch_bounds__(256) dq_merge_kernel(BwdParams p, DqSplit split, int64_t n_quads) {
  constexpr int kUnroll = 4, QPR = D / 4;
  const bool rope = p.rot.n_t + p.rot.n_h + p.rot.n_w != 0;
  const int64_t i0 = (int64_t)blockIdx.x * (256 * kUnroll) + threadIdx.x;
  f32x4 x[kWays][kUnroll];
  QuadAngles angles[kUnroll];  // requested with the sums, before the first store
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int64_t i = i0 + u * 256;
    if (i < n_quads) {
      x[0][u] = *reinterpret_cast<const f32x4*>(p.dq + i * 4);
      x[1][u] = *reinterpret_cast<const f32x4*>(split.part1 + i * 4);
      if constexpr (kWays == 3) x[2][u] = *reinterpret_cast<const f32x4*>(split.part2 + i * 4);
      if (rope) {
        // (rows of 256 bytes and more: their number fits 32 bits)
        const uint32_t bq = (uint32_t)(i / QPR) / (uint32_t)p.H, b = bq / (uint32_t)p.Nq;
        angles[u] = quad_angles(p.rot, token_tables(p.rot, (int)b, (int)(bq - b * (uint32_t)p.Nq)), (int)(i % QPR));
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int64_t i = i0 + u * 256;
    if (i >= n_quads) continue;
    f32x4 v = x[0][u];
#pragma unroll
    for (int w = 1; w < kWays; ++w) v += x[w][u];
    v = v * p.scale;
    if (rope) v = unrotate_quad(angles[u], v);
    *reinterpret_cast<f32x4*>(p.dq + i * 4) = v;
  }
}

// ---- dK, dV of the chunk's keys ---------------------------------------------------
// One workgroup = 8 waves = 128 keys in 4 blocks of 32 (every lane owns one key), each block
// seen by two waves.  The "value" wave computes S = Q~ K~^T, P and dV^T += dO^T P, and hands P
// (bf16, in the lane-private order of its accumulator registers) to its partner through LDS; the
// "key" wave picks it up one period later and computes dP = dO V^T, dS = P o (dP - Delta) and
// dK~^T += Q~^T dS.  Both gradients in one wave need more registers than two waves per SIMD
// have, and two independent workgroups per key tile each compute S and the exponentials (five
// products instead of four; that is how it was before: 1.22 ms at the 12-head, 21-frame,
// batch-4 shape).  A query tile is used in two consecutive periods, so tiles, row terms and P
// live in rings of three LDS slots, and a period is unrolled three times so that every slot is
// a compile-time offset.
constexpr int kPairWaves = 8;
constexpr int kPairThreads = kPairWaves * 64;
constexpr int QT = 64;  // query rows per LDS tile

template <int D>
struct DkvLds {
  static constexpr int TILE_BYTES = QT * D * 2;
  static constexpr int SLOT_TILES = 2 * TILE_BYTES;              // Q~ tile, dO tile
  static constexpr int SLOT_PROBS = 4 * (QT / 32) * 2 * 1024;    // key block x query block x half: 64 lanes x 16 B
  static constexpr int SLOT_TERMS = 2 * QT * 4;                  // LSE*log2e [QT], Delta [QT]
  static constexpr int kProbs = 3 * SLOT_TILES;
  static constexpr int kTerms = kProbs + 3 * SLOT_PROBS;
  static constexpr int kTotal = kTerms + 3 * SLOT_TERMS;
  static_assert(kTotal <= 160 * 1024, "one workgroup per CU must fit the LDS");
};

// Scheduling pattern for a product of kSteps operand fragments (kReads LDS reads and two MFMAs
// each) placed next to independent vector-ALU work: fragment reads run one step ahead of their
// MFMAs, and each pair of MFMAs is followed by a share of the vector-ALU instructions.
template <int kSteps, int kReads>
__device__ __forceinline__ void interleave() {
  __builtin_amdgcn_sched_group_barrier(0x100, 2 * kReads, 0);  // the first two fragments
#pragma unroll
  for (int i = 0; i < kSteps; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // two MFMAs
    __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);  // vector-ALU work of the other block
    if (i + 2 < kSteps) __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);  // the fragment after next
  }
}

// 16x16x32 MFMAs: a wave's 32 keys are two sub-blocks of 16 (ks); lane (i = lane % 16,
// g = lane / 16) holds, for keys 16*ks + i, the accumulator rows 4g .. 4g+3 of every 16-row tile.
// Tile rows below first[ks] (per lane; first_max, wave-uniform, = the largest over the wave) are
// queries of an earlier causal block than the lane's key ks: they do not see it, P = 0.
template <int D>
struct ValueWave {
  static constexpr int KS = D / 32;  // k-steps of a contraction over D
  static constexpr int DT = D / 16;  // 16-row tiles of dV^T
  bf16x8 kreg[2][KS];  // B operand: K~ rows of this lane's two keys
  f32x4 dv[DT][2];
  OperandAddr16<D> addr;
  int g;

  __device__ __forceinline__ void init(int lane) {
    g = lane >> 4;
    addr.init(lane);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) dv[dt][ks] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- the three phases of one block of 32 queries qb of a tile --------------------------
  // S[q][key] - LSE[q]*log2(e), the exponent of 2 (Q~ is pre-multiplied, the accumulators start from
  // the rows' terms): rows = 32 queries in two halves of 16 (qh), column = the lane's key ks
  __device__ __forceinline__ void s_product(const char* qs, int qb, const f32x4 (&l4)[2], f32x4 (&s)[2][2]) const {
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        const bf16x8 a = read_rows16<D>(qs, addr.row[st], 32 * qb + 16 * qh);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) s[qh][ks] = mfma16(a, kreg[ks][st], st == 0 ? l4[qh] : s[qh][ks]);
      }
  }
  // queries of an earlier causal block than the lane's key do not see it: P = 0
  __device__ __forceinline__ void mask(int qb, const int (&first)[2], f32x4 (&s)[2][2]) const {
#pragma unroll
    for (int qh = 0; qh < 2; ++qh)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[qh][ks][r] = 32 * qb + 16 * qh + 4 * g + r < first[ks] ? kNegBig : s[qh][ks][r];
  }
  // P as the B operand of the next product (k-slots 8g .. 8g+3 <- queries 4g .., 8g+4 .. <- queries
  // 16 + 4g ..), also handed to the key wave through LDS
  __device__ __forceinline__ void probabilities(const f32x4 (&s)[2][2], int qb, char* probs, bf16x8 (&pb)[2]) const {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh)
#pragma unroll
        for (int r = 0; r < 4; ++r) pb[ks][4 * qh + r] = (__bf16)fast_exp2(s[qh][ks][r]);
    *reinterpret_cast<bf16x8*>(probs + (2 * qb) * 1024) = pb[0];
    *reinterpret_cast<bf16x8*>(probs + (2 * qb + 1) * 1024) = pb[1];
  }
  // dV^T[d][key] += dO^T[d][q] P[q][key]
  __device__ __forceinline__ void dv_product(const char* dos, int qb, const bf16x8 (&pb)[2]) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8 a = read_cols16<D>(dos, addr.tr[dt], 32 * qb);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) dv[dt][ks] = mfma16(a, pb[ks], dv[dt][ks]);
    }
  }

  // One tile of 64 queries = two blocks.  A wave's own MFMAs and vector-ALU work overlap only when
  // independent instructions of both kinds are next to each other, so the blocks are software
  // pipelined: the exponentials of block 0 sit between the MFMAs of S(1), those of block 1 between
  // the MFMAs of dV(0).  (Phase by phase, as it was before, a period took about twice the time of
  // its MFMAs.)
  // qs / dos = Q~ and dO tiles, lse_t = -LSE*log2(e) of the tile's rows, probs = this wave's part of a P slot
  __device__ __forceinline__ void tile(const char* qs, const char* dos, const float* lse_t, char* probs,
                                       const int (&first)[2], int first_max) {
    static_assert(QT == 64, "two blocks per tile");
    f32x4 s0[2][2], s1[2][2], l0[2], l1[2];
    bf16x8 p0[2], p1[2];
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) {
      l0[qh] = *reinterpret_cast<const f32x4*>(lse_t + 16 * qh + 4 * g);
      l1[qh] = *reinterpret_cast<const f32x4*>(lse_t + 32 + 16 * qh + 4 * g);
    }
    s_product(qs, 0, l0, s0);
    if (first_max > 0) mask(0, first, s0);
    __builtin_amdgcn_sched_barrier(0);
    s_product(qs, 1, l1, s1);
    probabilities(s0, 0, probs, p0);
    interleave<2 * KS, 1>();
    __builtin_amdgcn_sched_barrier(0);
    if (first_max > 32) mask(1, first, s1);
    __builtin_amdgcn_sched_barrier(0);
    dv_product(dos, 0, p0);
    probabilities(s1, 1, probs, p1);
    interleave<DT, 2>();
    __builtin_amdgcn_sched_barrier(0);
    dv_product(dos, 1, p1);
  }
};

template <int D>
struct KeyWave {
  static constexpr int KS = D / 32;
  static constexpr int DT = D / 16;
  bf16x8 vreg[2][KS];  // B operand: V rows of this lane's two keys
  f32x4 dk[DT][2];
  OperandAddr16<D> addr;
  int g;

  __device__ __forceinline__ void init(int lane) {
    g = lane >> 4;
    addr.init(lane);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) dk[dt][ks] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // dP[q][key] - Delta[q] = <dO_q, V_key> - Delta[q]: the accumulators start from the rows' terms
  __device__ __forceinline__ void dp_product(const char* dos, int qb, const f32x4 (&d4)[2], f32x4 (&dp)[2][2]) const {
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        const bf16x8 a = read_rows16<D>(dos, addr.row[st], 32 * qb + 16 * qh);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) dp[qh][ks] = mfma16(a, vreg[ks][st], st == 0 ? d4[qh] : dp[qh][ks]);
      }
  }
  // dS = P o (dP - Delta) as the B operand of the last product
  __device__ __forceinline__ void ds_operand(const bf16x8 (&pb)[2], const f32x4 (&dp)[2][2], bf16x8 (&dsb)[2]) const {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh)
#pragma unroll
        for (int r = 0; r < 4; ++r) dsb[ks][4 * qh + r] = (__bf16)((float)pb[ks][4 * qh + r] * dp[qh][ks][r]);
  }
  // dK~^T[d][key] += Q~^T[d][q] dS[q][key]
  __device__ __forceinline__ void dk_product(const char* qs, int qb, const bf16x8 (&dsb)[2]) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8 a = read_cols16<D>(qs, addr.tr[dt], 32 * qb);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) dk[dt][ks] = mfma16(a, dsb[ks], dk[dt][ks]);
    }
  }

  // One tile of 64 queries, software pipelined like the value wave's: dS of block 0 is formed
  // between the MFMAs of dP(1), dS of block 1 between those of dK(0).
  // qs / dos = Q~ and dO tiles, delta_t = -Delta of the tile's rows, probs = the partner's P of this tile
  __device__ __forceinline__ void tile(const char* qs, const char* dos, const float* delta_t, const char* probs) {
    static_assert(QT == 64, "two blocks per tile");
    f32x4 dp0[2][2], dp1[2][2], d0[2], d1[2];
    bf16x8 p0[2], p1[2], ds0[2], ds1[2];
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) {
      d0[qh] = *reinterpret_cast<const f32x4*>(delta_t + 16 * qh + 4 * g);
      d1[qh] = *reinterpret_cast<const f32x4*>(delta_t + 32 + 16 * qh + 4 * g);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      p0[ks] = *reinterpret_cast<const bf16x8*>(probs + ks * 1024);
      p1[ks] = *reinterpret_cast<const bf16x8*>(probs + (2 + ks) * 1024);
    }
    dp_product(dos, 0, d0, dp0);
    __builtin_amdgcn_sched_barrier(0);
    dp_product(dos, 1, d1, dp1);
    ds_operand(p0, dp0, ds0);
    interleave<2 * KS, 1>();
    __builtin_amdgcn_sched_barrier(0);
    dk_product(qs, 0, ds0);
    ds_operand(p1, dp1, ds1);
    interleave<DT, 2>();
    __builtin_amdgcn_sched_barrier(0);
    dk_product(qs, 1, ds1);
  }
};

// The dK/dV kernel over the resident ring rows instead of the chunk's keys (non-detached backward, group
// 1): where the gradients go and what is needed to turn dK~ back at the frame each slot holds.
struct RingGrads {
  float* dk;  // [B, C*T, H, D]  w.r.t. the keys as they were appended (un-rotated); null = not stored
  float* dv;  // [B, C*T, H, D]; null = not stored
  const double* inv_freq_t;
  int C, S;
  StreamInts start, next_n, sink_shift;  // see launch_attn_bwd_hist_bf16
};
struct ChunkGrads {};  // the chunk's keys: everything is in BwdParams
// Both in one launch (bwd_joins): a pair's keys are its resident ring rows and then the chunk's, cut into blocks of 128 without
// regard to where the chunk begins, and every query sees all of them: under causal blocks a block of both would take its chunk rows
// past queries that do not see them, where a gradient that is not finite leaves 0 * inf in theirs.  Two launches each end with a
// partly filled round of workgroups (12 pairs, 28080 + 4680 rows: 2640 and 444 on 256 CUs, eleven rounds and two, against 3072,
// twelve: the whole pass 3513 -> 3419 us; D = 64, 16 pairs, 12480 + 3120 rows 877 -> 830).
struct AllGrads : RingGrads {};
template <typename Grads>
constexpr bool kHasRing = !std::is_same_v<Grads, ChunkGrads>;
// Row of a key of the launch: of the ring, or (with in_chunk) of the chunk
struct KeyRow {
  int row;
  bool in_chunk;
};
template <typename Grads>
__device__ __forceinline__ int keys_of(int hist, int Nq) {
  return std::is_same_v<Grads, AllGrads> ? hist + Nq : kHasRing<Grads> ? hist : Nq;
}
template <typename Grads>
__device__ __forceinline__ KeyRow key_row(int j, int hist) {
  if constexpr (std::is_same_v<Grads, AllGrads>)
    return j < hist ? KeyRow{j, false} : KeyRow{j - hist, true};
  else
    return KeyRow{j, !kHasRing<Grads>};
}

// (cos, sin) of the temporal pairs at the frames of ring slots first .. first + n - 1 of stream b, for `threads` threads
__device__ __forceinline__ void fill_slot_table(float2* tab, const BwdParams& p, const RingGrads& r, int b, int first, int n,
                                                int thread, int threads) {
  for (int e = thread; e < n * p.rot.n_t; e += threads) {
    const int slot = first + e / p.rot.n_t, j = e % p.rot.n_t;
    const int frame = r.start.v[b] + (int)frame_number_in_slot(slot, r.next_n.v[b], r.C, r.S) + (slot < r.S ? r.sink_shift.v[b] : 0);
    double sn, cs;
    sincos((double)frame * r.inv_freq_t[j], &sn, &cs);
    tab[e] = make_float2((float)cs, (float)sn);
  }
}

// Everything one wave does, in its role (kKey: a key wave, else a value wave).  Both roles
// stream the tiles and meet at the same barriers, one per period.
template <int D, bool kKey, typename Grads>
__device__ __forceinline__ void dkv_wave(const BwdParams& p, const Grads& grads, const WorkItem& item, int wave, char* lds) {
  constexpr bool kRing = kHasRing<Grads>;
  using L = DkvLds<D>;
  using Wave = std::conditional_t<kKey, KeyWave<D>, ValueWave<D>>;
  const int b = item.bh / p.H, h = item.bh % p.H;
  const int lane = threadIdx.x & 63;
  const int kw = wave & 3;  // key block of the workgroup's four
  const int i16 = lane & 15, g = lane >> 4;
  const int64_t bh = (int64_t)b * p.H + h;
  // this lane's two keys jc and jc + 16: chunk rows, or (non-detached backward) resident ring rows of the stream
  const int hist = kRing ? p.hist_rows.v[b] : 0, n_keys = keys_of<Grads>(hist, p.Nq);
  const int jc = (item.tile * 4 + kw) * 32 + i16;
  const int ntiles = (p.Nq + QT - 1) / QT;
  // first query row that sees each of this lane's keys (ring rows and what goes out with them are seen by every query),
  // the largest over the wave (its last key) and the smallest over the workgroup (its first key)
  const int block_rows = kRing ? 0 : p.block_rows;
  const int j_last = n_keys - 1;
  int first_q[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) first_q[ks] = first_query_row_seeing(jc + 16 * ks < j_last ? jc + 16 * ks : j_last, block_rows);
  const int j_wave = (item.tile * 4 + kw) * 32 + 31;
  const int first_q_wave = first_query_row_seeing(j_wave < j_last ? j_wave : j_last, block_rows);
  const int t_begin = first_query_row_seeing(item.tile * 128, block_rows) / QT;

  Wave w;
  w.init(lane);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    // B operand of the role's first product: V row (key wave) or K~ row (value wave) of the lane's key ks
    const bool live = jc + 16 * ks < n_keys;
    const KeyRow j0 = key_row<Grads>(live ? jc + 16 * ks : 0, hist);
    const __bf16* row;
    if constexpr (kKey)
      row = j0.in_chunk ? p.v_chunk + (((int64_t)b * p.Nq + j0.row) * p.H + h) * D : p.v_cache + (bh * p.cache_rows + j0.row) * D;
    else
      row = j0.in_chunk ? p.kc_rot + (bh * p.Nq + j0.row) * D : p.k_cache + (bh * p.cache_rows + j0.row) * D;
#pragma unroll
    for (int st = 0; st < D / 32; ++st) {
      bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0};
      if (live) x = *reinterpret_cast<const bf16x8*>(row + st * 32 + g * 8);
      if constexpr (kKey)
        w.vreg[ks][st] = x;
      else
        w.kreg[ks][st] = x;
    }
  }

  const RowSegment q_rows = make_segment(p.q_rot + bh * p.Nq * D, D, p.Nq, D);
  const RowSegment do_rows = make_segment(p.dout + ((int64_t)b * p.Nq * p.H + h) * D, (int64_t)p.H * D, p.Nq, D);
  TileStreamer<D, QT, kPairWaves> ts;
  ts.init();
  const uint32_t off_q = ts.lane_offset(q_rows), off_do = ts.lane_offset(do_rows);
  // Row terms of a tile's queries: wave 0 fetches LSE*log2e and wave 1 Delta with a direct-to-LDS
  // load of 4 bytes per lane, so no register, branch or wait of the tile loop depends on them.
  // Rows past Nq read as zeros; they cannot contribute: their Q~ and dO rows are zero in LDS as
  // well, so dP, Delta and with them dS and the dV terms are 0.
  const __amdgpu_buffer_rsrc_t term_rows = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((wave == 0 ? p.lse2 : p.delta) + bh * p.Nq), 0, p.Nq * 4, 0x00020000);
  const int term_lane = lane * 4;
  auto issue = [&](int t, int slot) __attribute__((always_inline)) {
    typedef __attribute__((address_space(3))) void* lds_ptr;
    char* qbuf = lds + slot * L::SLOT_TILES;
    ts.issue(q_rows, off_q, t * QT, qbuf);
    ts.issue(do_rows, off_do, t * QT, qbuf + L::TILE_BYTES);
    if (!kKey && wave < 2)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(term_rows, (lds_ptr)(lds + L::kTerms + slot * L::SLOT_TERMS + wave * QT * 4),
                                               4, t * QT * 4 + term_lane, 0, 0, 0);
  };
  issue(t_begin, 0);
  wait_vmem();
  __syncthreads();

  // Period n: the value waves work on tile n (slot S), the key waves on tile n - 1 (slot S - 1),
  // tile n + 1 streams into slot S + 1; the last period has only the key waves' tile left.
  const int probs_lane = kw * (QT / 32) * 2 * 1024 + lane * 16;
  // Ring rows: the epilogue needs (cos, sin) of the temporal pairs at the frames of this workgroup's
  // keys.  The value waves have no tile in the last period: they compute the table there, into that
  // period's own slot, which no tile was loaded for.  (By the key waves in their idle first period, into
  // LDS of its own, the loop came out slower: 3661 against 3531 us for the whole pass of one clip.)  Where it
  // does not fit the slot (frames of a token and many temporal pairs) all waves do it afterwards in the
  // idle tile ring.
  int slot_first = 0, slot_count = 0;
  bool in_slot = true;
  if constexpr (kRing) {
    const int j_first = item.tile * 128, j_end = j_first + 128 < hist ? j_first + 128 : hist;
    slot_first = j_first / p.rot.T;
    slot_count = j_first < j_end ? (j_end - 1) / p.rot.T - slot_first + 1 : 0;
    static_assert(129 * (D / 2) * 8 <= 3 * L::SLOT_TILES, "the largest table fits the tile ring");
    in_slot = slot_count * p.rot.n_t * (int)sizeof(float2) <= L::SLOT_TILES;
  }
  auto period = [&](int n, auto slot_c) __attribute__((always_inline)) {
    constexpr int S = decltype(slot_c)::value, PREV = (S + 2) % 3, NEXT = (S + 1) % 3;
    if (n + 1 < ntiles) issue(n + 1, NEXT);
    if constexpr (kKey) {
      if (n > t_begin)
        w.tile(lds + PREV * L::SLOT_TILES, lds + PREV * L::SLOT_TILES + L::TILE_BYTES,
               reinterpret_cast<const float*>(lds + L::kTerms + PREV * L::SLOT_TERMS) + QT,
               lds + L::kProbs + PREV * L::SLOT_PROBS + probs_lane);
    } else {
      if constexpr (kRing) {
        if (n == ntiles && in_slot)
          fill_slot_table(reinterpret_cast<float2*>(lds + S * L::SLOT_TILES), p, grads, b, slot_first, slot_count, threadIdx.x, 256);
      }
      if (n < ntiles) {
        const int first[2] = {first_q[0] - n * QT, first_q[1] - n * QT};
        w.tile(lds + S * L::SLOT_TILES, lds + S * L::SLOT_TILES + L::TILE_BYTES,
               reinterpret_cast<const float*>(lds + L::kTerms + S * L::SLOT_TERMS),
               lds + L::kProbs + S * L::SLOT_PROBS + probs_lane, first, first_q_wave - n * QT);
      }
    }
    wait_vmem();
    __syncthreads();
  };
  for (int n = t_begin;;) {
    period(n, std::integral_constant<int, 0>{});
    if (++n > ntiles) break;
    period(n, std::integral_constant<int, 1>{});
    if (++n > ntiles) break;
    period(n, std::integral_constant<int, 2>{});
    if (++n > ntiles) break;
  }

  const float2* slot_tab = nullptr;
  if constexpr (kRing) {
    slot_tab = reinterpret_cast<const float2*>(lds + (in_slot ? (ntiles - t_begin) % 3 * L::SLOT_TILES : 0));
    if (!in_slot) {
      fill_slot_table(reinterpret_cast<float2*>(lds), p, grads, b, slot_first, slot_count, threadIdx.x, kPairThreads);
      __syncthreads();
    }
    if (!(kKey ? grads.dk : grads.dv)) return;
  }

  // dV as it is; dK~ is turned back to dK here.  All look-ups are requested before the first store: the compiler cannot tell
  // the gradients from the tables, so one behind a store waits for it.  Launch with each look-up at its store / so, us: chunk, D = 128
  // 48 pairs x 4680 rows 952 / 948, 12 pairs 254 / 251.5, D = 64 16 pairs 160 / 158, 48 pairs x 1200 52.5 / 50.5; ring of 18 frames, 12
  // pairs of 128 1432 / 1418, 16 of 64 with 12 frames 778 / 766.  The price is 74 (ring 102) scalar registers kept in vector registers.
  const bool rope = kKey && p.rot.n_t + p.rot.n_h + p.rot.n_w != 0;
  QuadAngles angles[2][D / 16];
  if (rope) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int j = jc + 16 * ks < j_last ? jc + 16 * ks : j_last;
      TokenTables tt;
      const KeyRow key = key_row<Grads>(j, hist);
      if (!key.in_chunk) {
        const int slot = key.row / p.rot.T, rem = key.row - slot * p.rot.T, y = rem / p.rot.gw, x = rem - y * p.rot.gw;
        tt = TokenTables{slot_tab + (slot - slot_first) * p.rot.n_t, p.rot.tab_h + y * p.rot.n_h, p.rot.tab_w + x * p.rot.n_w};
      } else {
        tt = token_tables(p.rot, b, key.row);
      }
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) angles[ks][dt] = quad_angles(p.rot, tt, 4 * dt + g);
    }
  }
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int j = jc + 16 * ks;
    if (j >= n_keys) continue;
    const KeyRow key = key_row<Grads>(j, hist);
    float* row = nullptr;
    if constexpr (kRing) row = (kKey ? grads.dk : grads.dv) + (((int64_t)b * p.cache_rows + key.row) * p.H + h) * D;
    if (key.in_chunk) row = (kKey ? p.dk : p.dv) + (((int64_t)b * p.Nq + key.row) * p.H + h) * D;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) {
      f32x4 x;
      if constexpr (kKey) {
        x = w.dk[dt][ks] * kLn2;  // dK~ = dS^T Q~ / sqrt(D), and the staged Q~ carries log2(e)/sqrt(D)
        if (rope) x = unrotate_quad(angles[ks][dt], x);
      } else {
        x = w.dv[dt][ks];
      }
      *reinterpret_cast<f32x4*>(row + 16 * dt + 4 * g) = x;
    }
  }
}

template <int D, typename Grads>
__global__ void __launch_bounds__(kPairThreads, 1) attn_bwd_dkv_kernel(BwdParams p, Grads grads) {
  constexpr bool kRing = kHasRing<Grads>;
  __shared__ __attribute__((aligned(1024))) char lds[DkvLds<D>::kTotal];
  // one pair's operands through one L2: 183 instead of 202 us at D = 64 (16 heads, 592 workgroups, causal, which take the
  // kernel below now); at D = 128, where a pair's operands alone are half an L2, no gain (1.01 against 1.00 ms at batch 4)
  const WorkItem item = work_item(p.tiles, p.BH, D == 64 && (!kRing || p.by_xcd));
  if (!item.valid) return;
  const int n_keys = keys_of<Grads>(kRing ? p.hist_rows.v[item.bh / p.H] : 0, p.Nq);
  if (item.tile * 128 >= n_keys) return;  // whole workgroup, before any barrier
  // waves 0..3 accumulate dV, waves 4..7 dK; the branch is per wave, and both sides execute
  // the same sequence of barriers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= 4)
    dkv_wave<D, true>(p, grads, item, wave, lds);
  else
    dkv_wave<D, false>(p, grads, item, wave, lds);
}

// ---- the same at D = 64 --------------------------------------------------------------------------------
// Both gradients of 32 keys fit one wave's registers (64 accumulators), so there are no roles: a workgroup is four waves, each with
// its own block of 32 of the 128 keys, P does not go through LDS, dS is formed from it in 32 bits, and three workgroups share a CU (34 KB of LDS,
// 168 registers) instead of one (100 KB).  Bound by waiting: 0.41 of a wave's time, matrix cores busy 0.35 (16 heads, 4680 rows in causal blocks,
// 158 us; roles 182, 0.30): the fragments of dV and dK are read one at a time, right in front of their MFMAs, and the loads of the next tile are
// waited for in front of the first transposing read.  Which launches take it: dkv_halves().
template <int D>
struct KeyBlockWave {
  static constexpr int KS = D / 32, DT = D / 16;
  bf16x8 kreg[2][KS], vreg[2][KS];  // B operands: K~ and V rows of this lane's two keys
  f32x4 dk[DT][2], dv[DT][2];
  OperandAddr16<D> addr;
  int g;

  __device__ __forceinline__ void init(int lane) {
    g = lane >> 4;
    addr.init(lane);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) dk[dt][ks] = dv[dt][ks] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // rows of a tile from row0 on times the lane's keys, the accumulators starting from the rows' terms
  __device__ __forceinline__ void product(const char* tile, int row0, const float* terms, const bf16x8 (&keys)[2][KS], f32x4 (&s)[2][2]) const {
    f32x4 t4[2];
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) t4[qh] = *reinterpret_cast<const f32x4*>(terms + row0 + 16 * qh + 4 * g);
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        const bf16x8 a = read_rows16<D>(tile, addr.row[st], row0 + 16 * qh);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) s[qh][ks] = mfma16(a, keys[ks][st], st == 0 ? t4[qh] : s[qh][ks]);
      }
  }
  __device__ __forceinline__ void accumulate(const char* tile, int row0, const bf16x8 (&x)[2], f32x4 (&acc)[DT][2]) const {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8 a = read_cols16<D>(tile, addr.tr[dt], row0);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) acc[dt][ks] = mfma16(a, x[ks], acc[dt][ks]);
    }
  }
  // 32 queries of a tile: lse_t / delta_t = -LSE*log2(e) and -Delta of its rows; rows below first[ks] do not see the lane's key
  // ks (first_max, wave-uniform: largest over the wave)
  __device__ __forceinline__ void block(const char* qs, const char* dos, const float* lse_t, const float* delta_t, int row0,
                                        const int (&first)[2], int first_max) {
    f32x4 s[2][2], dp[2][2];
    bf16x8 pb[2], dsb[2];
    product(qs, row0, lse_t, kreg, s);
    if (first_max > row0) {
#pragma unroll
      for (int qh = 0; qh < 2; ++qh)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[qh][ks][r] = row0 + 16 * qh + 4 * g + r < first[ks] ? kNegBig : s[qh][ks][r];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qh = 0; qh < 2; ++qh)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[qh][ks][r] = fast_exp2(s[qh][ks][r]);
    product(dos, row0, delta_t, vreg, dp);
#pragma unroll
    for (int i = 0; i < 4 * KS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // two exponentials
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pb[ks][4 * qh + r] = (__bf16)s[qh][ks][r];
          dsb[ks][4 * qh + r] = (__bf16)(s[qh][ks][r] * dp[qh][ks][r]);
        }
    __builtin_amdgcn_sched_barrier(0);
    accumulate(dos, row0, pb, dv);
    accumulate(qs, row0, dsb, dk);
  }
};

// kHalves = 2: twice the waves, each takes one of a tile's two blocks of queries, and the two waves of a key block add up
// through LDS at the end.
template <int D, int kHalves, typename Grads>
__global__ void __launch_bounds__(kHalves * 256, kHalves == 1 ? 3 : 2) attn_bwd_dkv_block_kernel(BwdParams p, Grads grads) {
  constexpr bool kRing = kHasRing<Grads>;
  constexpr int TILE_BYTES = QT * D * 2, SLOT_BYTES = 2 * TILE_BYTES, SLOT_TERMS = 2 * QT * 4;
  constexpr int kWaves = 4 * kHalves, kSumBytes = 2 * (D / 16) * 1024;  // one gradient of 32 keys
  // Two tiles, then their row terms.  (A third slot gains nothing here: the compiler cannot tell which LDS the loads of a step write
  // and waits for them in front of its first transposing read, so a tile has half a block's time to land either way.)
  constexpr int kTerms = 2 * SLOT_BYTES, kTileBytes = kTerms + 2 * SLOT_TERMS;
  __shared__ __attribute__((aligned(1024))) char lds[kHalves == 1 || kTileBytes > 8 * kSumBytes ? kTileBytes : 8 * kSumBytes];
  const WorkItem item = work_item(p.tiles, p.BH, !kRing || p.by_xcd);
  if (!item.valid) return;
  const int b = item.bh / p.H, h = item.bh % p.H;
  // this lane's two keys jc and jc + 16: chunk rows, or (non-detached backward) resident ring rows of the stream
  const int hist = kRing ? p.hist_rows.v[b] : 0, n_keys = keys_of<Grads>(hist, p.Nq);
  if (item.tile * 128 >= n_keys) return;  // whole workgroup, before any barrier
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kw = wave & 3, half = wave >> 2;
  const int i16 = lane & 15, g = lane >> 4;
  const int64_t bh = (int64_t)b * p.H + h;
  const int j_wave = (item.tile * 4 + kw) * 32, jc = j_wave + i16, j_last = n_keys - 1;
  const int ntiles = (p.Nq + QT - 1) / QT;
  // as in dkv_wave()
  const int block_rows = kRing ? 0 : p.block_rows;
  int first_q[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) first_q[ks] = first_query_row_seeing(jc + 16 * ks < j_last ? jc + 16 * ks : j_last, block_rows);
  const int first_q_wave = first_query_row_seeing(j_wave + 31 < j_last ? j_wave + 31 : j_last, block_rows);
  const int t_begin = first_query_row_seeing(item.tile * 128, block_rows) / QT;

  const RowSegment q_rows = make_segment(p.q_rot + bh * p.Nq * D, D, p.Nq, D);
  const RowSegment do_rows = make_segment(p.dout + ((int64_t)b * p.Nq * p.H + h) * D, (int64_t)p.H * D, p.Nq, D);
  TileStreamer<D, QT, kWaves> ts;
  ts.init();
  const uint32_t off_q = ts.lane_offset(q_rows), off_do = ts.lane_offset(do_rows);
  // Row terms as in dkv_wave(): rows past Nq read as zeros, and their Q~ and dO rows are zero in LDS as well
  const __amdgpu_buffer_rsrc_t term_rows =
      __builtin_amdgcn_make_buffer_rsrc((void*)((wave == 0 ? p.lse2 : p.delta) + bh * p.Nq), 0, p.Nq * 4, 0x00020000);
  auto issue = [&](int t, int slot) __attribute__((always_inline)) {
    typedef __attribute__((address_space(3))) void* lds_ptr;
    char* qbuf = lds + slot * SLOT_BYTES;
    ts.issue(q_rows, off_q, t * QT, qbuf);
    ts.issue(do_rows, off_do, t * QT, qbuf + TILE_BYTES);
    if (wave < 2)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(term_rows, (lds_ptr)(lds + kTerms + slot * SLOT_TERMS + wave * QT * 4), 4,
                                               t * QT * 4 + lane * 4, 0, 0, 0);
  };
  issue(t_begin, 0);

  KeyBlockWave<D> w;
  w.init(lane);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const bool live = jc + 16 * ks < n_keys;
    const KeyRow j0 = key_row<Grads>(live ? jc + 16 * ks : 0, hist);
    const __bf16* krow = j0.in_chunk ? p.kc_rot + (bh * p.Nq + j0.row) * D : p.k_cache + (bh * p.cache_rows + j0.row) * D;
    const __bf16* vrow = j0.in_chunk ? p.v_chunk + (((int64_t)b * p.Nq + j0.row) * p.H + h) * D : p.v_cache + (bh * p.cache_rows + j0.row) * D;
#pragma unroll
    for (int st = 0; st < D / 32; ++st) {
      bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0}, y = x;
      if (live) {
        x = *reinterpret_cast<const bf16x8*>(krow + st * 32 + g * 8);
        y = *reinterpret_cast<const bf16x8*>(vrow + st * 32 + g * 8);
      }
      w.kreg[ks][st] = x;
      w.vreg[ks][st] = y;
    }
  }
  wait_vmem();
  __syncthreads();
  auto step = [&](int t, auto slot_c) __attribute__((always_inline)) {
    constexpr int S = decltype(slot_c)::value;
    if (t + 1 < ntiles) issue(t + 1, S ^ 1);
    const char* qs = lds + S * SLOT_BYTES;
    const float* terms = reinterpret_cast<const float*>(lds + kTerms + S * SLOT_TERMS);
    const int first[2] = {first_q[0] - t * QT, first_q[1] - t * QT};
    if constexpr (kHalves == 2) {
      w.block(qs, qs + TILE_BYTES, terms, terms + QT, 32 * half, first, first_q_wave - t * QT);
    } else {
#pragma unroll
      for (int qb = 0; qb < QT / 32; ++qb) w.block(qs, qs + TILE_BYTES, terms, terms + QT, 32 * qb, first, first_q_wave - t * QT);
    }
    wait_vmem();
    __syncthreads();
  };
  for (int t = t_begin; t < ntiles; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    if (t + 1 < ntiles) step(t + 1, std::integral_constant<int, 1>{});
  }

  // the first half's waves finish dV, the second's dK, each with what the other has of it
  const bool has_dv = kHalves == 1 || half == 0, has_dk = kHalves == 1 || half == 1;
  if constexpr (kHalves == 2) {
    f32x4* const mine = reinterpret_cast<f32x4*>(lds + wave * kSumBytes);
    const f32x4* const others = reinterpret_cast<const f32x4*>(lds + (wave ^ 4) * kSumBytes);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) mine[(2 * dt + ks) * 64 + lane] = has_dv ? w.dk[dt][ks] : w.dv[dt][ks];
    __syncthreads();
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const f32x4 x = others[(2 * dt + ks) * 64 + lane];
        w.dv[dt][ks] += x;  // (only one of the two is stored)
        w.dk[dt][ks] += x;
      }
    __syncthreads();
  }

  // ring rows: (cos, sin) of the temporal pairs at the frames of this workgroup's keys, in the idle slots
  const bool rope = p.rot.n_t + p.rot.n_h + p.rot.n_w != 0;
  const float2* slot_tab = nullptr;
  int slot_first = 0;
  if constexpr (kRing) {
    const int j_first = item.tile * 128, j_end = j_first + 128 < hist ? j_first + 128 : hist;
    static_assert(129 * (D / 2) * 8 <= sizeof lds, "the largest table fits");
    slot_first = j_first / p.rot.T;
    slot_tab = reinterpret_cast<const float2*>(lds);
    fill_slot_table(reinterpret_cast<float2*>(lds), p, grads, b, slot_first, j_first < j_end ? (j_end - 1) / p.rot.T - slot_first + 1 : 0, threadIdx.x, kWaves * 64);
    __syncthreads();
  }
  // all look-ups before the first store, as in dkv_wave()
  QuadAngles angles[2][D / 16];
  if (rope && has_dk) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int j = jc + 16 * ks < j_last ? jc + 16 * ks : j_last;
      TokenTables tt;
      const KeyRow key = key_row<Grads>(j, hist);
      if (!key.in_chunk) {
        const int slot = key.row / p.rot.T, rem = key.row - slot * p.rot.T, y = rem / p.rot.gw, x = rem - y * p.rot.gw;
        tt = TokenTables{slot_tab + (slot - slot_first) * p.rot.n_t, p.rot.tab_h + y * p.rot.n_h, p.rot.tab_w + x * p.rot.n_w};
      } else {
        tt = token_tables(p.rot, b, key.row);
      }
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) angles[ks][dt] = quad_angles(p.rot, tt, 4 * dt + g);
    }
  }
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int j = jc + 16 * ks;
    if (j >= n_keys) continue;
    const KeyRow key = key_row<Grads>(j, hist);
    float *dk_to = p.dk, *dv_to = p.dv;
    if constexpr (kRing)
      if (!key.in_chunk) dk_to = grads.dk, dv_to = grads.dv;
    const int64_t at = (((int64_t)b * (key.in_chunk ? p.Nq : p.cache_rows) + key.row) * p.H + h) * D + 4 * g;
    if (has_dv && (!kRing || dv_to)) {
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) *reinterpret_cast<f32x4*>(dv_to + at + 16 * dt) = w.dv[dt][ks];
    }
    if (has_dk && (!kRing || dk_to)) {
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        f32x4 x = w.dk[dt][ks] * kLn2;  // dK~ = dS^T Q~ / sqrt(D), and the staged Q~ carries log2(e)/sqrt(D)
        if (rope) x = unrotate_quad(angles[ks][dt], x);
        *reinterpret_cast<f32x4*>(dk_to + at + 16 * dt) = x;
      }
    }
  }
}

// the dK / dV launch of p.tiles blocks of 128 keys per pair, by the kernel that dkv_halves() says
template <int D, typename Grads>
void launch_dkv(const BwdParams& p, const Grads& grads, int halves, hipStream_t stream) {
  const int workgroups = work_grid_size(p.tiles, p.BH);
  if constexpr (D == 64) {
    if (halves == 1)
      attn_bwd_dkv_block_kernel<D, 1><<<dim3(workgroups), 256, 0, stream>>>(p, grads);
    else if (halves == 2)
      attn_bwd_dkv_block_kernel<D, 2><<<dim3(workgroups), 512, 0, stream>>>(p, grads);
  }
  if constexpr (D == 128 || !std::is_same_v<Grads, AllGrads>)
    if (halves == 0) attn_bwd_dkv_kernel<D><<<dim3(workgroups), kPairThreads, 0, stream>>>(p, grads);
}

// ---- launches with few rows ------------------------------------------------------------------------
// With 128 queries (or keys) per workgroup a chunk of a few hundred tokens and a few heads is a
// handful of workgroups that walk all rows of the other side one tile after another.  Here a
// workgroup owns ONE block of 32 queries (dQ) or 32 chunk keys (dK and dV), its waves share the
// other side (FewRows), and both kinds of workgroup go out in ONE launch: the key side takes Delta
// from dO and O itself instead of waiting for the query side.  All sums over the waves are fp32 in a
// fixed order.  What bounds it: the tiles a CU pulls per 32 queries, as in the forward's kernel of
// this kind; for short walks the chain launch, operand loads, tile, combine (6 us at D = 64).  With one wave per SIMD a
// chain costs its latency, so before the walk operands are shared through LDS and requested together, and behind it the
// rotary look-ups are in flight before the waves meet (each wave loading all of its operands, shuffles for the row
// sums and a look-up per block where it was used took 60 % of a short call).  Backward before / now, us: D = 64 64 rows, 2
// heads, 320 keys 7.1 / 5.9; 260 rows, 16 pairs, 1040 keys 14.1 / 11.8; 400 rows, 48 pairs, 2000 keys 41.3 / 37.3;
// D = 128 64 rows, 2 heads, 320 keys 11.2 / 8.5; 234 rows, 16 pairs, 702 keys 17.1 / 13.9; 330 rows, 16 pairs, 1540 keys 28.4 /
// 22.8;672 rows, 3 pairs, 1120 keys 30.1 / 24.1 with four waves.  Two tiles per wave in flight (double the LDS)
// were slower: 41.7 at the 330 rows, where two workgroups no longer share a CU, and 17.1 at the 234, where each has one anyway.
// One wave of the key side: S = Q~ K~^T, P and dV^T += dO^T P, or (kDk) also dP = dO V^T, dS and
// dK~^T += Q~^T dS.  One wave of 256 registers does not hold both accumulators at D = 128, so half of
// the waves take dV and half dK; S is computed by both.  Layout as in the pair of waves above.
template <int D, bool kDk>
struct FewKeysWave {
  static constexpr int KS = D / 32, DT = D / 16;
  bf16x8 kreg[2][KS], vreg[2][KS];
  f32x4 acc[DT][2];
  OperandAddr16<D> addr;
  int g;

  __device__ __forceinline__ void init(int lane) {
    g = lane >> 4;
    addr.init(lane);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) acc[dt][ks] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // lse_t / delta_t = -LSE*log2(e) and -Delta of the tile's rows; rows below first[ks] do not see the
  // lane's key ks (first_max: largest over the wave)
  __device__ __forceinline__ void tile(const char* qs, const char* dos, const float* lse_t, const float* delta_t,
                                       const int (&first)[2], int first_max) {
    f32x4 s[2][2];
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        const bf16x8 a = read_rows16<D>(qs, addr.row[st], 16 * qh);
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_t + 16 * qh + 4 * g);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) s[qh][ks] = mfma16(a, kreg[ks][st], st == 0 ? l4 : s[qh][ks]);
      }
    if (first_max > 0) {
#pragma unroll
      for (int qh = 0; qh < 2; ++qh)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[qh][ks][r] = 16 * qh + 4 * g + r < first[ks] ? kNegBig : s[qh][ks][r];
    }
    bf16x8 x[2];  // P or dS as the B operand of the last product
    if constexpr (kDk) {
      f32x4 dp[2][2];
#pragma unroll
      for (int st = 0; st < KS; ++st)
#pragma unroll
        for (int qh = 0; qh < 2; ++qh) {
          const bf16x8 a = read_rows16<D>(dos, addr.row[st], 16 * qh);
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(delta_t + 16 * qh + 4 * g);
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) dp[qh][ks] = mfma16(a, vreg[ks][st], st == 0 ? d4 : dp[qh][ks]);
        }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int qh = 0; qh < 2; ++qh)
#pragma unroll
          for (int r = 0; r < 4; ++r) x[ks][4 * qh + r] = (__bf16)(fast_exp2(s[qh][ks][r]) * dp[qh][ks][r]);
    } else {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int qh = 0; qh < 2; ++qh)
#pragma unroll
          for (int r = 0; r < 4; ++r) x[ks][4 * qh + r] = (__bf16)fast_exp2(s[qh][ks][r]);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8 a = read_cols16<D>(kDk ? qs : dos, addr.tr[dt], 0);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) acc[dt][ks] = mfma16(a, x[ks], acc[dt][ks]);
    }
  }
};

// The (cos, sin) with which a wave turns its `kShare` 16 x 16 blocks of a summed gradient back, all requested before
// the waves meet for the sum (each looked up where it was used they cost about 1000 cycles a block).
template <int D, int kShare>
struct FewAngles {
  QuadAngles q[kShare];
  bool rope;
  // blocks unit0 .. unit0 + kShare - 1: rows row0 + 16 * (unit % 2), columns 16 * (unit / 2) + 4 * g ..
  __device__ __forceinline__ void load(const RotaryTables& r, int b, int unit0, int row0, int row_last, int g) {
    rope = r.n_t + r.n_h + r.n_w != 0;
    if (!rope) return;
    // block u lies in the rows of block u & 1 (unit0 is even where a wave has more than one block)
    constexpr int kRows = kShare > 1 ? 2 : 1;
    TokenTables t[kRows];
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const int row = row0 + 16 * ((unit0 + i) & 1);
      t[i] = token_tables_small(r, b, row < row_last ? row : row_last);
    }
#pragma unroll
    for (int u = 0; u < kShare; ++u) q[u] = quad_angles(r, t[u % kRows], 4 * ((unit0 + u) >> 1) + g);
  }
  __device__ __forceinline__ f32x4 turn_back(int u, f32x4 x) const { return rope ? unrotate_quad(q[u], x) : x; }
};

template <int D, int kWaves>
__device__ __forceinline__ void few_dq(const BwdParams& p, const WorkItem& item, int hist_of_lane, char* lds, float (*terms)[kFewMaxRows]) {
  using F = FewRows<D, kWaves>;
  using Wave = DqWave<D>;
  const PairIndex pair = few_split_pair(item.bh, p.H, p.group, p.div);
  const int b = pair.b, h = pair.h;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  const int hist = __builtin_amdgcn_readlane(hist_of_lane, pair.cache_b);
  const int64_t bh = (int64_t)b * p.H + h;
  const int q_first = item.tile * 32, q0 = q_first + i16, q_last = p.Nq - 1;
  const int vis_first = visible_chunk_rows(q_first, p.Nq, p.block_rows);
  const int vis_last = visible_chunk_rows(q_first + 31 < q_last ? q_first + 31 : q_last, p.Nq, p.block_rows);
  int vis[2];
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) vis[qs] = visible_chunk_rows(q0 + 16 * qs < q_last ? q0 + 16 * qs : q_last, p.Nq, p.block_rows);
  const int hist_tiles = (hist + 31) / 32, ntiles = hist_tiles + (vis_last + 31) / 32;
  const int t_begin = F::begin(wave, kWaves, 0, ntiles), t_end = F::begin(wave + 1, kWaves, 0, ntiles);

  const u32x4 k_hist = segment_words(p.k_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const u32x4 v_hist = segment_words(p.v_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const u32x4 k_chunk = segment_words(p.kc_rot + bh * p.Nq * D, D, p.Nq, D);
  const u32x4 v_chunk = segment_words(p.v_chunk + ((int64_t)b * p.Nq * p.H + h) * D, (int64_t)p.H * D, p.Nq, D);
  char* ktile = lds + wave * F::kWaveBytes;
  char* vtile = ktile + F::kTileBytes;
  PrivateStream<D> ps;
  ps.init(lane);
  auto issue_k = [&](int t) __attribute__((always_inline)) {
    const bool in_hist = t < hist_tiles;
    ps.issue(in_hist ? k_hist : k_chunk, D * 2, (in_hist ? t : t - hist_tiles) * 32, ktile);
  };
  auto issue_v = [&](int t) __attribute__((always_inline)) {
    const bool in_hist = t < hist_tiles;
    ps.issue(in_hist ? v_hist : v_chunk, in_hist ? D * 2 : p.H * D * 2, (in_hist ? t : t - hist_tiles) * 32, vtile);
  };
  if (t_begin < t_end) {
    issue_k(t_begin);
    issue_v(t_begin);
  }
  Wave w;
  w.init(lane);
  // Q~ and dO of the block, once for all waves (each had loaded all of both, and O for Delta, in 64-byte pieces: 4400 - 8000
  // cycles until the first product), where the key side has its row terms.  Delta = <dO, O>: 8 components to a lane.
  char* const qtile = reinterpret_cast<char*>(terms);
  char* const dotile = qtile + F::kTileBytes;
  static_assert(sizeof(float[2][kFewMaxRows]) >= 2 * F::kTileBytes, "both tiles fit");
  {
    constexpr int CPR = D / 8, kRows = kWaves * 64 / CPR, kTrips = kRows < 32 ? 32 / kRows : 1;
    const int64_t tok = ((int64_t)b * p.Nq * p.H + h) * D;
    const int r = threadIdx.x / CPR, c = threadIdx.x % CPR;
    bf16x8 x[kTrips], y[kTrips];
    float l[kTrips];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int row = u * kRows + r, q = q_first + row < p.Nq ? q_first + row : q_last;
      x[u] = *reinterpret_cast<const bf16x8*>(p.dout + tok + (int64_t)q * p.H * D + c * 8);
      y[u] = *reinterpret_cast<const bf16x8*>(p.out + tok + (int64_t)q * p.H * D + c * 8);
      l[u] = p.lse[bh * p.Nq + q];
    }
    const u32x4 q_rows = segment_words(p.q_rot + bh * p.Nq * D, D, p.Nq, D);
    const u32x4 do_rows = segment_words(p.dout + tok, (int64_t)p.H * D, p.Nq, D);
    for (int u = wave; u < PrivateStream<D>::kInsts; u += kWaves) {
      ps.issue_part(q_rows, D * 2, q_first, u, qtile);
      ps.issue_part(do_rows, p.H * D * 2, q_first, u, dotile);
    }
    float d[kTrips];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      d[u] = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) d[u] = fmaf((float)x[u][j], (float)y[u][j], d[u]);
      d[u] = sum_neighbours<CPR>(d[u]);
    }
    wait_vmem();
    __syncthreads();
    w.take_queries(qtile, dotile);
    __syncthreads();
    // the row terms go where Q~ was: with room of their own two workgroups would no longer fit a CU's LDS at D = 128
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int row = u * kRows + r, q = q_first + row;
      if (c != 0 || row >= 32) continue;
      const bool live = q < p.Nq;
      // a dead query row gets P = exp2(0 - big) = 0 everywhere
      const float nl = live ? -l[u] * kLog2e : -1.0e30f, nd = live ? -d[u] : 0.f;
      terms[0][row] = nl;
      terms[0][32 + row] = nd;
      if (live && !p.terms_ready) {  // for later launches
        p.lse2[bh * p.Nq + q] = nl;
        p.delta[bh * p.Nq + q] = nd;
      }
    }
    __syncthreads();
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      const float nl = terms[0][16 * qs + i16], nd = terms[0][32 + 16 * qs + i16];
      w.neg_lse2[qs] = f32x4{nl, nl, nl, nl};
      w.neg_delta[qs] = f32x4{nd, nd, nd, nd};
    }
  }
  for (int t = t_begin; t < t_end; ++t) {
    const int row0 = (t < hist_tiles ? t : t - hist_tiles) * 32;
    const int live[2] = {(t < hist_tiles ? hist : vis[0]) - row0, (t < hist_tiles ? hist : vis[1]) - row0};
    wait_vmem_except<PrivateStream<D>::kInsts>();  // the K tile; the V tile behind it may be in flight
    wave_lds_sync();
    f32x4 s[2][2], dp[2][2];
    bf16x8 dsb[2];
    w.s_product(ktile, 0, s);
    if ((t < hist_tiles ? hist : vis_first) - row0 < 32) w.mask(0, live, s);
    __builtin_amdgcn_sched_barrier(0);
    wait_vmem();
    wave_lds_sync();
    w.probabilities(s);
    w.dp_product(vtile, 0, dp);
    w.ds_operand(s, dp, dsb);
    w.dq_product(ktile, 0, dsb);
    wait_lds();
    wave_lds_sync();
    // (V refilled right behind dP, so that S has to wait for both, was slower: 35.5 against 33.5 us at
    // 70 workgroups x 133 tiles, D = 128)
    if (t + 1 < t_end) {
      issue_k(t + 1);
      issue_v(t + 1);
    }
  }
  constexpr int kShare = F::kUnits / kWaves;
  FewAngles<D, kShare> angles;
  angles.load(p.rot, b, wave * kShare, q0, q_last, g);
  wave_lds_sync();
#pragma unroll
  for (int dt = 0; dt < Wave::DT; ++dt)
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) *reinterpret_cast<f32x4*>(ktile + ((dt * 2 + qs) * 64 + lane) * 16) = w.dq[dt][qs];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kShare; ++u) {
    const int unit = wave * kShare + u, dt = unit >> 1, q = q0 + 16 * (unit & 1);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) x += *reinterpret_cast<const f32x4*>(lds + wv * F::kWaveBytes + (unit * 64 + lane) * 16);
    x = angles.turn_back(u, x * p.scale);
    if (q < p.Nq) *reinterpret_cast<f32x4*>(p.dq + (((int64_t)b * p.Nq + q) * p.H + h) * D + 16 * dt + 4 * g) = x;
  }
}

// Row terms of all queries of one pair: terms[0][q] = -LSE*log2(e), terms[1][q] = -Delta = -<dO, O>.
// Rows past the end (up to the tile) are 0: their Q~ and dO rows are zero in LDS, so they add nothing.
template <int D, int kWaves>
__device__ __forceinline__ void few_row_terms(const BwdParams& p, int b, int h, float (*terms)[kFewMaxRows]) {
  constexpr int CPR = D / 8, kRows = kWaves * 64 / CPR, kUnroll = 4;
  const int64_t bh = (int64_t)b * p.H + h;
  const int n = (p.Nq + 31) & ~31;
  const int r = threadIdx.x / CPR, c = threadIdx.x % CPR;
  const int64_t first = ((int64_t)b * p.Nq * p.H + h) * D + c * 8;
  for (int q0 = 0; q0 < n; q0 += kRows * kUnroll) {
    bf16x8 x[kUnroll], y[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int q = q0 + u * kRows + r;
      const int64_t at = first + (int64_t)(q < p.Nq ? q : 0) * p.H * D;
      x[u] = *reinterpret_cast<const bf16x8*>(p.dout + at);
      y[u] = *reinterpret_cast<const bf16x8*>(p.out + at);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int q = q0 + u * kRows + r;
      float d = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) d = fmaf((float)x[u][j], (float)y[u][j], d);
      d = sum_neighbours<CPR>(d);
      if (c == 0 && q < n) terms[1][q] = q < p.Nq ? -d : 0.f;
    }
  }
  for (int q = threadIdx.x; q < n; q += kWaves * 64) terms[0][q] = q < p.Nq ? -p.lse[bh * p.Nq + q] * kLog2e : 0.f;
}

// What a wave of the key side loads before it has the row terms: the workgroup's keys (and their values, which only the dK
// waves use) and its first tiles.  part = its share of the query tiles among kWaves / 2.
template <int D, int kWaves>
struct FewKeysOperands {
  using F = FewRows<D, kWaves>;
  int j_first, t_begin, t_end;
  u32x4 q_rows, do_rows;
  PrivateStream<D> ps;
  bf16x8 k[2][D / 32], v[2][D / 32];

  __device__ __forceinline__ void issue(const BwdParams& p, int t, char* qtile) const {
    ps.issue(q_rows, D * 2, t * 32, qtile);
    ps.issue(do_rows, p.H * D * 2, t * 32, qtile + F::kTileBytes);
  }
  __device__ __forceinline__ void init(const BwdParams& p, int b, int h, int tile, int part, char* qtile) {
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int64_t bh = (int64_t)b * p.H + h, tok = ((int64_t)b * p.Nq * p.H + h) * D;
    j_first = tile * 32;
    const int t_first = first_query_row_seeing(j_first, p.block_rows) / 32, ntiles = (p.Nq + 31) / 32;
    t_begin = F::begin(part, kWaves / 2, t_first, ntiles), t_end = F::begin(part + 1, kWaves / 2, t_first, ntiles);
    q_rows = segment_words(p.q_rot + bh * p.Nq * D, D, p.Nq, D);
    do_rows = segment_words(p.dout + tok, (int64_t)p.H * D, p.Nq, D);
    ps.init(lane);
    if (t_begin < t_end) issue(p, t_begin, qtile);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int j = j_first + i16 + 16 * ks < p.Nq ? j_first + i16 + 16 * ks : 0;  // a key past the end is computed like key 0 and never stored
      const __bf16* krow = p.kc_rot + (bh * p.Nq + j) * D;
      const __bf16* vrow = p.v_chunk + tok + (int64_t)j * p.H * D;
#pragma unroll
      for (int st = 0; st < D / 32; ++st) {
        k[ks][st] = *reinterpret_cast<const bf16x8*>(krow + st * 32 + g * 8);
        v[ks][st] = *reinterpret_cast<const bf16x8*>(vrow + st * 32 + g * 8);
      }
    }
  }
};

// The row terms of all pairs in a launch of its own.  Bound by its bytes (out, dout once) and a launch, 2 us; a row to 8 or
// 16 lanes, in the order in which the tensors lie in memory.
template <int D>
__global__ void __launch_bounds__(256) few_row_terms_kernel(BwdParams p, uint32_t n_rows) {
  constexpr int CPR = D / 8, kRows = 256 / CPR, kUnroll = 2;
  const int c = threadIdx.x % CPR;
  bf16x8 x[kUnroll], y[kUnroll];
  float l[kUnroll];
  int64_t at[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t i = (blockIdx.x * kUnroll + u) * kRows + threadIdx.x / CPR, row = i < n_rows ? i : n_rows - 1;  // (b * Nq + q) * H + h
    const uint32_t bq = row / (uint32_t)p.H, b = bq / (uint32_t)p.Nq;
    at[u] = ((int64_t)b * p.H + (row - bq * p.H)) * p.Nq + (bq - b * p.Nq);
    x[u] = *reinterpret_cast<const bf16x8*>(p.dout + (int64_t)row * D + c * 8);
    y[u] = *reinterpret_cast<const bf16x8*>(p.out + (int64_t)row * D + c * 8);
    l[u] = p.lse[at[u]];
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    float d = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) d = fmaf((float)x[u][j], (float)y[u][j], d);
    d = sum_neighbours<CPR>(d);
    if (c == 0 && (blockIdx.x * kUnroll + u) * kRows + threadIdx.x / CPR < n_rows) {
      p.delta[at[u]] = -d;
      p.lse2[at[u]] = -l[u] * kLog2e;
    }
  }
}

// one wave's share of the key side
template <int D, int kWaves, bool kDk>
__device__ __forceinline__ void few_dkv_wave(const BwdParams& p, const FewKeysOperands<D, kWaves>& op, char* qtile, const float (*terms)[kFewMaxRows]) {
  using Wave = FewKeysWave<D, kDk>;
  const int lane = threadIdx.x & 63;
  const int j_first = op.j_first, j0 = j_first + (lane & 15), j_last = p.Nq - 1;
  int first_q[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) first_q[ks] = first_query_row_seeing(j0 + 16 * ks < j_last ? j0 + 16 * ks : j_last, p.block_rows);
  const int first_q_max = first_query_row_seeing(j_first + 31 < j_last ? j_first + 31 : j_last, p.block_rows);
  char* const dotile = qtile + FewRows<D, kWaves>::kTileBytes;
  Wave w;
  w.init(lane);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int st = 0; st < D / 32; ++st) {
      w.kreg[ks][st] = op.k[ks][st];
      if constexpr (kDk) w.vreg[ks][st] = op.v[ks][st];
    }
  for (int t = op.t_begin; t < op.t_end; ++t) {
    const int first[2] = {first_q[0] - t * 32, first_q[1] - t * 32};
    wait_vmem();
    wave_lds_sync();
    w.tile(qtile, dotile, terms[0] + t * 32, terms[1] + t * 32, first, first_q_max - t * 32);
    wait_lds();
    wave_lds_sync();
    if (t + 1 < op.t_end) op.issue(p, t + 1, qtile);
  }
  wave_lds_sync();
#pragma unroll
  for (int dt = 0; dt < Wave::DT; ++dt)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) *reinterpret_cast<f32x4*>(qtile + ((dt * 2 + ks) * 64 + lane) * 16) = w.acc[dt][ks];
}

template <int D, int kWaves>
__device__ __forceinline__ void few_dkv(const BwdParams& p, const WorkItem& item, char* lds, float (*terms)[kFewMaxRows]) {
  using F = FewRows<D, kWaves>;
  const int b = quotient(item.bh, p.div.heads), h = item.bh - b * p.H;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  constexpr int kHalf = kWaves / 2;
  char* const qtile = lds + wave * F::kWaveBytes;
  FewKeysOperands<D, kWaves> op;
  op.init(p, b, h, item.tile, wave % kHalf, qtile);
  if (p.terms_ready) {
    const int64_t at = ((int64_t)b * p.H + h) * p.Nq;
    for (int q = threadIdx.x; q < ((p.Nq + 31) & ~31); q += kWaves * 64) {
      terms[0][q] = q < p.Nq ? p.lse2[at + q] : 0.f;
      terms[1][q] = q < p.Nq ? p.delta[at + q] : 0.f;
    }
  } else {
    few_row_terms<D, kWaves>(p, b, h, terms);
  }
  __syncthreads();
  const bool is_dv = wave < kHalf;
  constexpr int kShare = F::kUnits / kHalf;
  const int unit0 = (wave % kHalf) * kShare, j0 = item.tile * 32 + i16;
  FewAngles<D, kShare> angles;
  angles.rope = false;
  if (is_dv) {
    few_dkv_wave<D, kWaves, false>(p, op, qtile, terms);
  } else {
    few_dkv_wave<D, kWaves, true>(p, op, qtile, terms);
    angles.load(p.rot, b, unit0, j0, p.Nq - 1, g);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kShare; ++u) {
    const int unit = unit0 + u, dt = unit >> 1, j = j0 + 16 * (unit & 1);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < kHalf; ++wv)
      x += *reinterpret_cast<const f32x4*>(lds + (wv + (is_dv ? 0 : kHalf)) * F::kWaveBytes + (unit * 64 + lane) * 16);
    if (!is_dv) x = angles.turn_back(u, x * kLn2);  // dK~ = dS^T Q~ / sqrt(D), and the staged Q~ carries log2(e)/sqrt(D)
    if (j < p.Nq) *reinterpret_cast<f32x4*>((is_dv ? p.dv : p.dk) + (((int64_t)b * p.Nq + j) * p.H + h) * D + 16 * dt + 4 * g) = x;
  }
}

// grid: first the workgroups of the query side (the longer walk), then those of the key side;
// p.tiles = blocks of 32 rows per pair, the same number on both sides
template <int D, int kWaves>
__global__ void __launch_bounds__(kWaves * 64, 2) attn_bwd_few_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[kWaves * FewRows<D, kWaves>::kWaveBytes];
  __shared__ __attribute__((aligned(16))) float terms[2][kFewMaxRows];
  static_assert(ASTRO_MAX_BATCH == 64, "one stream per lane");
  const int hist_of_lane = p.hist_rows.v[threadIdx.x & 63];
  // the arguments in one round of scalar loads, as in the forward's kernel of this kind
  asm volatile("" ::"s"(p.tiles), "s"(p.BH), "s"((int)p.by_xcd), "s"(p.H), "s"(p.group), "s"(p.Nq), "s"(p.block_rows), "s"(p.div.tiles),
               "s"(p.div.group), "s"(p.div.heads), "s"(p.k_cache), "s"(p.v_cache), "s"(p.kc_rot), "s"(p.v_chunk), "s"(p.cache_rows),
               "s"(p.q_rot), "s"(p.dout), "s"(p.out), "s"(p.lse), "s"((int)p.terms_ready));
  const int n_side = p.tiles * p.BH;
  const bool key_side = (int)blockIdx.x >= n_side;
  const WorkItem item = few_work_item(p.tiles, p.BH, p.by_xcd, p.div, (int)blockIdx.x - (key_side ? n_side : 0));
  if (!item.valid) return;
  if (key_side)
    few_dkv<D, kWaves>(p, item, lds, terms);
  else
    few_dq<D, kWaves>(p, item, hist_of_lane, lds, terms);
}

template <int D>
BwdParams make_params(const DevGeom& g, const AttnOperands& op, const void* out, const float* lse, const void* dout,
                      float* dq, float* dk, float* dv, void* scratch) {
  BwdParams p;
  p.q_rot = (const __bf16*)op.q_rot;
  p.kc_rot = (const __bf16*)op.kc_rot;
  p.v_chunk = (const __bf16*)op.v_chunk;
  p.k_cache = (const __bf16*)op.k_cache;
  p.v_cache = (const __bf16*)op.v_cache;
  p.out = (const __bf16*)out;
  p.dout = (const __bf16*)dout;
  p.lse = lse;
  p.delta = (float*)scratch;
  p.lse2 = p.delta + (size_t)g.B * g.H * op.Nq;
  p.dq = dq;
  p.dk = dk;
  p.dv = dv;
  p.rot = RotaryTables{op.tab_t, g.tab_h, g.tab_w, g.n_t, g.n_h, g.n_w, g.gw, g.T, op.Nq / g.T};
  p.H = g.H;
  p.BH = g.B * g.H;
  p.tiles = 0;
  p.Nq = op.Nq;
  p.cache_rows = (int64_t)g.C * g.T;
  p.scale = 1.0f / sqrtf((float)D);
  p.hist_rows = op.hist_rows;
  p.group = op.group;
  p.block_rows = op.block_rows;
  p.by_xcd = true;
  p.terms_ready = false;
  p.div = FewDivisors{};
  return p;
}

template <int D>
constexpr int kDqPlaces = dq_places_per_cu(D);

template <int D>
hipError_t launch(const DevGeom& g, const AttnOperands& op, const void* out, const float* lse, const void* dout,
                  float* dq, float* dk, float* dv, void* scratch, bool keys_later, hipStream_t stream) {
  BwdParams p = make_params<D>(g, op, out, lse, dout, dq, dk, dv, scratch);
  const CallShape shape = call_shape(g, op);
  if (const int waves = bwd_few_waves(shape)) {
    p.terms_ready = bwd_terms_first(shape);
    if (p.terms_ready) {
      ProfileScope prof("attn_bwd_few_row_terms", stream);
      const uint32_t n_rows = (uint32_t)p.BH * op.Nq, per_block = 2 * 256 / (D / 8);
      few_row_terms_kernel<D><<<dim3((n_rows + per_block - 1) / per_block), 256, 0, stream>>>(p, n_rows);
    }
    ProfileScope prof("attn_bwd_few_bf16", stream);
    p.tiles = (op.Nq + 31) / 32;
    p.div = few_divisors(p.tiles, p.group, p.H);
    const dim3 grid(2 * work_grid_size(p.tiles, p.BH));
    if (waves == 8)
      attn_bwd_few_kernel<D, 8><<<grid, 8 * 64, 0, stream>>>(p);
    else
      attn_bwd_few_kernel<D, 4><<<grid, 4 * 64, 0, stream>>>(p);
    return hipGetLastError();
  }
  p.tiles = (op.Nq + kDqWaves * 32 - 1) / (kDqWaves * 32);
  const int items = work_grid_size(p.tiles, p.BH);
  const DqWays ways = dq_ways(shape);
  p.by_xcd = order_by_xcd(shape, items);
  const DqSplit split{ways.ways, ways.k, dk, dv};
  {
    ProfileScope prof("attn_bwd_dq_bf16", stream);
    if (split.ways == 1)
      attn_bwd_dq_kernel<D, kDqPlaces<D>, kDqWaves, false><<<dim3(items), kDqWaves * 64, 0, stream>>>(p, split);
    else
      attn_bwd_dq_kernel<D, kDqPlaces<D>, kDqWaves, true><<<dim3(items + split.helpers(items)), kDqWaves * 64, 0, stream>>>(p, split);
  }
  if (split.ways != 1) {
    ProfileScope prof("attn_bwd_dq_merge", stream);
    const int64_t n_quads = (int64_t)p.BH * op.Nq * D / 4;
    const dim3 grid((unsigned)((n_quads + 1023) / 1024));
    if (split.ways == 2)
      dq_merge_kernel<D, 2><<<grid, 256, 0, stream>>>(p, split, n_quads);
    else
      dq_merge_kernel<D, 3><<<grid, 256, 0, stream>>>(p, split, n_quads);
  }
  const int ktile = 128;
  if (!keys_later) {
    ProfileScope prof("attn_bwd_dkv_bf16", stream);
    p.tiles = (op.Nq + ktile - 1) / ktile;
    launch_dkv<D>(p, ChunkGrads{}, dkv_halves(shape, chunk_blocks(shape)), stream);
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_hist(const DevGeom& g, const AttnOperands& op, const float* lse, const void* dout, float* dk, float* dv,
                       const RingGrads& grads, const void* scratch, hipStream_t stream) {
  BwdParams p = make_params<D>(g, op, nullptr, lse, dout, nullptr, dk, dv, const_cast<void*>(scratch));
  int max_hist = 0;
  for (int b = 0; b < g.B; ++b) max_hist = op.hist_rows.v[b] > max_hist ? op.hist_rows.v[b] : max_hist;
  if (max_hist == 0) return hipSuccess;
  const int ktile = 128;
  p.tiles = (max_hist + (dk ? op.Nq : 0) + ktile - 1) / ktile;
  const CallShape shape = call_shape(g, op);
  p.by_xcd = order_by_xcd(shape, work_grid_size(p.tiles, p.BH));
  const int halves = dkv_halves(shape, dk ? chunk_blocks(shape) : shape.ring_blocks);  // (of both: see bwd_joins())
  auto run = [&](const auto& to) {
    ProfileScope prof(dk ? "attn_bwd_dkv_joint_bf16" : "attn_bwd_dkv_hist_bf16", stream);
    launch_dkv<D>(p, to, halves, stream);
  };
  if (dk) {
    run(AllGrads{grads});
  } else if (op.in_order) {  // dV and dK share bytes, dK's stay: one after the other
    RingGrads one = grads;
    one.dk = nullptr;
    run(one);
    one.dk = grads.dk;
    one.dv = nullptr;
    run(one);
  } else {
    run(grads);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bwd_hist_bf16(const DevGeom& g, const AttnOperands& op, const float* lse, const void* dout,
                                     float* dk, float* dv, float* dk_hist, float* dv_hist, const StreamInts& start,
                                     const StreamInts& next_n, const StreamInts& sink_shift, const void* scratch, hipStream_t stream) {
  if (op.group != 1) return hipErrorInvalidValue;
  const RingGrads grads{dk_hist, dv_hist, g.inv_freq_t, g.C, g.S, start, next_n, sink_shift};
  if (g.D == 128) return launch_hist<128>(g, op, lse, dout, dk, dv, grads, scratch, stream);
  return launch_hist<64>(g, op, lse, dout, dk, dv, grads, scratch, stream);
}

bool bf16_bwd_joins(const DevGeom& g, const AttnOperands& op) { return bwd_joins(call_shape(g, op)); }

// Delta and LSE*log2e per (stream, head, query)
size_t bf16_bwd_workspace_bytes(const DevGeom& g, int Nq) { return 2 * (size_t)g.B * g.H * Nq * sizeof(float); }

hipError_t launch_attn_bwd_bf16(const DevGeom& g, const AttnOperands& op, const void* out, const float* lse,
                                const void* dout, float* dq, float* dk, float* dv, void* scratch, bool keys_later,
                                hipStream_t stream) {
  if (g.D == 128) return launch<128>(g, op, out, lse, dout, dq, dk, dv, scratch, keys_later, stream);
  return launch<64>(g, op, out, lse, dout, dq, dk, dv, scratch, keys_later, stream);
}

}  // namespace astro
