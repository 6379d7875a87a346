// Chunk attention forward over the rolling cache, bf16 MFMA with fp32 accumulation.
//
// One workgroup = 4 wavefronts = 4 * 32 consecutive queries of one (stream, head).
// The visible keys (resident ring rows, then the chunk's own rows) are walked in tiles of
// 32; K and V tiles are streamed into a ring of LDS stages by direct-to-LDS loads issued
// two tiles ahead, one barrier per tile.  Everything is computed transposed so that
// every lane owns ONE query:
//   S^T[key][q] = K * Q~^T      (A = K tile from LDS, B = Q~ held in registers; Q~ arrives
//                                pre-multiplied by log2(e)/sqrt(D), so S^T is the exponent of 2)
//   O^T[d][q]  += V^T * P^T     (A = V tile through the transposing LDS read,
//                                B = P^T taken straight from the S^T accumulators)
// so the row maximum / sum of the softmax are in-lane reductions plus one exchange with
// the partner lane l^32, and the rescale factor is a per-lane scalar.
//
// Order inside a tile: the K operand reads are issued first, then the global->LDS loads
// of the tile two ahead (their issue stalls while the memory pipeline is busy, which now
// overlaps the LDS latency of the K reads), then the QK MFMAs, softmax, V reads and PV
// MFMAs.  Runs of full tiles inside one key segment take a branch-free copy of the tile
// code (no tail handling, no segment or end-of-loop tests); only the few tiles around the
// segment boundaries take the general one.
//
// Softmax reference: probabilities are taken relative to a per-query reference M that is
// only raised when a tile's probabilities relative to it sum to more than kSumLimit; fp32
// accumulators and the bf16 exponent range make any smaller excess exact enough, and
// both the row maximum and the 64 accumulator multiplies of a rescale leave the common path.
// A query's first reference is snapped to 0 when its first tile's maximum is moderate, and a wave
// whose references are all 0 takes exp2 of the score itself: no subtraction per score either.
// The softmax's vector-ALU work of a tile has no independent MFMAs of the same wave to sit between
// (taking the probabilities of the first 16 keys between the MFMAs of the other 16 was measured
// slower as the scheduler ordered it, 3.34 vs 3.22 ms, and equal with the exact order pinned in
// assembly, 3.03-3.08 vs 3.01-3.03 ms); the overlap comes from
// three workgroups (three waves per SIMD) being resident per CU.
#include "kernels.hpp"
#include "mfma_common.hpp"

namespace astro {
namespace {

constexpr int KT = kFwdKeyTile;
constexpr float kSumLimit = 0x1p44f;  // a lane's 16 probabilities may sum to this before the reference moves
// a first tile whose rows sum to less than this relative to 0 takes its reference from its maximum instead
constexpr float kFirstSumLimit = 0x1p-32f;

struct FwdParams {
  const __bf16* q_rot;
  const __bf16* kc_rot;
  const __bf16* v_chunk;
  const __bf16* k_cache;
  const __bf16* v_cache;
  __bf16* out;
  float* lse;
  // key-range split: workgroup (pair, split, tile) walks the split's share of the key tiles and
  // writes its own normalised output and log-sum-exp to part `split`; a merge launch combines them
  int splits;
  __bf16* out_part;  // [splits][B, Nq, H, D]
  float* lse_part;   // [splits][B][H][Nq]
  int H, Nq, BH, q_tiles, group;  // BH = candidates * heads; group = candidates per cache stream
  int block_rows;                 // causal block inside the chunk in token rows, 0 = none
  bool by_xcd;                    // order of the workgroups, see order_by_xcd()
  bool in_turn;                   // few rows: the waves take the key tiles in turn, not a contiguous share each
  int64_t cache_rows;  // C*T
  FewDivisors div;     // few rows
  StreamInts hist_rows;
};

// 16x16x32 MFMAs: a wave's 32 queries are two sub-blocks of 16 (qs); lane (i = lane % 16,
// g = lane / 16) holds, for queries 16*qs + i, the accumulator rows 4g .. 4g+3 of every 16-row
// tile, so a query's row statistics are spread over the four lanes i, i+16, i+32, i+48; they
// are only combined at the end of the kernel and on the rare path that moves the reference.
template <int D>
struct FwdWave {
  static constexpr int KS = D / 32;   // k-steps of the QK product
  static constexpr int KF = 2 * KS;   // K operand fragments of a 32-key tile: step x 16-key half
  static constexpr int DT = D / 16;   // 16-row tiles of O^T

  bf16x8 qreg[2][KS];
  f32x4 o[DT][2];
  float mc[2], l_run[2];  // softmax reference in log2 units (the units of the scores), per-lane partial row sum
  // every reference of the wave is exactly 0 (wave-uniform): the exponent is the score itself
  bool zero_ref;
  OperandAddr16<D> addr;
  int g;

  __device__ __forceinline__ void init(int lane) {
    g = lane >> 4;
    zero_ref = false;
    addr.init(lane);
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      mc[qs] = kNegBig;
      l_run[qs] = 0.f;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) o[dt][qs] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  __device__ __forceinline__ void init_zero_ref() {
    mc[0] = mc[1] = 0.f;
    zero_ref = true;
  }

  // over the four lanes that share a query
  static __device__ __forceinline__ float row_sum(float x) { return sum_quarters(x); }

  // p = exp2(s - mc) (kZeroRef: mc is 0 for the whole wave, no subtraction) rounded to bf16, packed as the B operands of the PV
  // product (k-slots 8g .. 8g+3 <- keys 4g .., 8g+4 .. <- keys 16 + 4g ..); sum = this lane's
  // part of the row sums, taken over the rounded values.
  template <bool kZeroRef>
  __device__ __forceinline__ void probabilities(const f32x4 (&s)[2][2], bf16x8 (&pb)[2], float (&sum)[2]) const {
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      sum[qs] = 0.f;
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const f32x2 e = kZeroRef ? f32x2{fast_exp2(s[kh][qs][r]), fast_exp2(s[kh][qs][r + 1])}
                                   : f32x2{fast_exp2(s[kh][qs][r] - mc[qs]), fast_exp2(s[kh][qs][r + 1] - mc[qs])};
          const bf16x2 pk = __builtin_convertvector(e, bf16x2);
          sum[qs] = add_pair(pk, sum[qs]);
          pb[qs][4 * kh + r] = pk[0];
          pb[qs][4 * kh + r + 1] = pk[1];
        }
    }
  }

  // A operands of the first half of the QK product's k-steps: 32 keys x D/2.  The other half is
  // read behind the MFMAs of the first (registers for all of them at once are not there).
  static constexpr int KH = KF / 2;
  __device__ __forceinline__ void read_k(const char* ks, bf16x8 (&kf)[KH]) const {
#pragma unroll
    for (int j = 0; j < KH; ++j) kf[j] = read_rows16<D>(ks, addr.row[j >> 1], 16 * (j & 1));
  }

  // S^T tile of 32 keys x this wave's 32 queries from K operands in registers.  With kTail
  // and any_dead (wave-uniform), only the first live[qs] rows of the tile count for this lane's
  // query qs: the others lie past their segment (K and V rows zero in LDS) or in a causal block
  // the query does not see, and get a score that makes their probability exactly 0.
  template <bool kTail>
  __device__ __forceinline__ void scores(const bf16x8 (&kf)[KH], const char* ks, const int (&live)[2], bool any_dead,
                                         f32x4 (&s)[2][2]) const {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    bf16x8 hi[KH];
#pragma unroll
    for (int j = 0; j < KH; ++j) {  // fragment j: k-step j / 2, key half j % 2
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) s[j & 1][qs] = mfma16(kf[j], qreg[qs][j >> 1], j < 2 ? zero : s[j & 1][qs]);
      hi[j] = read_rows16<D>(ks, addr.row[(KH + j) >> 1], 16 * (j & 1));
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // two MFMAs
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // then one LDS read
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < KH; ++j)
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) s[j & 1][qs] = mfma16(hi[j], qreg[qs][(KH + j) >> 1], s[j & 1][qs]);
    if (kTail && any_dead) mask(live, s);
  }

  __device__ __forceinline__ void mask(const int (&live)[2], f32x4 (&s)[2][2]) const {
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int qs = 0; qs < 2; ++qs)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[kh][qs][r] = 16 * kh + 4 * g + r >= live[qs] ? kNegBig : s[kh][qs][r];
  }

  // The same scores for the rare path that moves the reference: every operand fragment is read
  // right before its MFMAs, so the path adds no registers to what the common one needs.
  template <bool kTail>
  __device__ __forceinline__ void scores_again(const char* ks, const int (&live)[2], bool any_dead, f32x4 (&s)[2][2]) const {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KF; ++j) {
      const bf16x8 a = read_rows16<D>(ks, addr.row[j >> 1], 16 * (j & 1));
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) s[j & 1][qs] = mfma16(a, qreg[qs][j >> 1], j < 2 ? zero : s[j & 1][qs]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kTail && any_dead) mask(live, s);
  }

  // One 32-key tile: kf = its K operands (read from ks), vs = its V rows in LDS; live (per
  // lane and query) and any_dead (wave-uniform) are only looked at when kTail.
  // first (wave-uniform): the wave's first tile, tried with the reference 0 that init_zero_ref() has set;
  // if a row's probabilities come out too small for it, the reference is taken from the tile's maximum.
  // before_pv() runs when the K tile is done with and before the V tile is read.
  template <bool kTail, typename Hook>
  __device__ __forceinline__ void tile(const bf16x8 (&kf)[KH], const char* ks, const char* vs, const int (&live)[2],
                                       bool any_dead, bool first, Hook before_pv) {
    // Probabilities relative to the current reference.  No maximum is taken on the common
    // path: a tile whose logits outgrow the reference shows up as a huge (or infinite) row
    // sum; only then the scores are computed again (the first copy is gone: the exponentials
    // are taken in place), the reference is raised and the probabilities are redone.
    bf16x8 pb[2];
    float sum[2];
    {
      f32x4 s[2][2];
      scores<kTail>(kf, ks, live, any_dead, s);
      if (__builtin_expect(zero_ref, 1))
        probabilities<true>(s, pb, sum);
      else
        probabilities<false>(s, pb, sum);
    }
    bool rescale = __any(!(sum[0] <= kSumLimit) || !(sum[1] <= kSumLimit));
    if (first) {
      rescale = rescale || __any(!(row_sum(sum[0]) >= kFirstSumLimit) || !(row_sum(sum[1]) >= kFirstSumLimit));
      if (rescale) mc[0] = mc[1] = kNegBig;  // nothing is accumulated yet
    }
    if (__builtin_expect(rescale, 0)) {
      f32x4 s[2][2];
      scores_again<kTail>(ks, live, any_dead, s);
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) {
        float mx = fmaxf(fmaxf(s[0][qs][0], s[0][qs][1]), fmaxf(s[0][qs][2], s[0][qs][3]));
        mx = fmaxf(mx, fmaxf(fmaxf(s[1][qs][0], s[1][qs][1]), fmaxf(s[1][qs][2], s[1][qs][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16));  // over the four lanes that share the query
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // never below -1e28: a query that has seen nothing but masked keys so far (scores of
        // -1e30) keeps probabilities of exactly 0 instead of exp2(rounding error of 1e29)
        float mc_new = fmaxf(fmaxf(mc[qs], mx), -1.0e28f);
        // A query's FIRST reference (nothing accumulated yet) is snapped to 0 when its tile maximum
        // is moderate, as it is for any ordinary logits: while every reference of the wave is 0 the
        // common path needs no subtraction in front of the exponential.  fp32 sums and the bf16
        // exponent range hold 2^44 above and 2^-90 below such a reference.
        if (mc[qs] < -1.0e27f && mc_new > -32.f && mc_new < 32.f) mc_new = 0.f;
        const float alpha = fast_exp2(mc[qs] - mc_new);
        l_run[qs] *= alpha;
        // whole-tuple products: the compiler then updates the accumulators where they are
        // (element by element it copies all of them, which the tile loop has no registers for)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt][qs] = o[dt][qs] * alpha;
        mc[qs] = mc_new;
      }
      zero_ref = __all(mc[0] == 0.f && mc[1] == 0.f);
      probabilities<false>(s, pb, sum);
    }
    l_run[0] += sum[0];
    l_run[1] += sum[1];
    // O^T += V^T P^T.  Half of the V operand fragments are requested up front; those of the
    // second half are read one by one behind the MFMAs of the first, into the registers
    // these have just released.
    before_pv();
    constexpr int HALF = DT / 2;
    bf16x8 v0[HALF], v1[HALF];
#pragma unroll
    for (int dt = 0; dt < HALF; ++dt) v0[dt] = read_cols16<D>(vs, addr.tr[dt], 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < HALF; ++dt) {
      o[dt][0] = mfma16(v0[dt], pb[0], o[dt][0]);
      o[dt][1] = mfma16(v0[dt], pb[1], o[dt][1]);
      v1[dt] = read_cols16<D>(vs, addr.tr[HALF + dt], 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // two MFMAs
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // then two LDS reads
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < HALF; ++dt) {
      o[HALF + dt][0] = mfma16(v1[dt], pb[0], o[HALF + dt][0]);
      o[HALF + dt][1] = mfma16(v1[dt], pb[1], o[HALF + dt][1]);
    }
  }
};

// kCausal: the chunk has causal blocks (block_rows > 0), so the chunk rows a query sees differ
// from lane to lane; without it that count is the uniform Nq and costs no vector register.
template <int D, int kStages, int kWaves, int OCC, bool kCausal>
__global__ void __launch_bounds__(kWaves * 64, OCC) attn_fwd_bf16_kernel(FwdParams p) {
  using Wave = FwdWave<D>;
  constexpr int kAhead = kStages - 1;  // tiles in flight ahead of the one being processed
  constexpr int TILE_BYTES = KT * D * 2;
  constexpr int STAGE_BYTES = 2 * TILE_BYTES;  // K tile, V tile
  __shared__ __attribute__((aligned(1024))) char lds[kStages * STAGE_BYTES];
  // per-lane count of visible chunk rows: kept in LDS, not in a register the tile loop has no room for
  __shared__ int vis_lds[kCausal ? 2 * kWaves * 64 : 1];

  const WorkItem item = work_item(p.q_tiles, p.BH * p.splits, p.by_xcd);
  if (!item.valid) return;
  const int split = item.bh % p.splits;
  const PairIndex pair = split_pair(item.bh / p.splits, p.H, p.group);
  const int b = pair.b, h = pair.h;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g = lane >> 4;
  const int hist = p.hist_rows.v[pair.cache_b];
  const int q0 = (item.tile * kWaves + wave) * 32 + i16;  // this lane's queries: q0 and q0 + 16
  // chunk rows each of this lane's queries sees, the fewest any lane of the wave sees (its first
  // query) and the most any wave of the workgroup sees (its last query)
  const int q_last = p.Nq - 1;
  const int block_rows = kCausal ? p.block_rows : 0;
  const int q_wave = (item.tile * kWaves + __builtin_amdgcn_readfirstlane(wave)) * 32;
  const int q_wg = (item.tile + 1) * kWaves * 32 - 1;
  const int vis_wave = visible_chunk_rows(q_wave < q_last ? q_wave : q_last, p.Nq, block_rows);
  const int vis_wg = visible_chunk_rows(q_wg < q_last ? q_wg : q_last, p.Nq, block_rows);
  if constexpr (kCausal) {
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
      vis_lds[qs * kWaves * 64 + threadIdx.x] = visible_chunk_rows(q0 + 16 * qs < q_last ? q0 + 16 * qs : q_last, p.Nq, block_rows);
  }
  // key tiles: first the resident ring rows, then the chunk rows the workgroup sees, each with its own tail
  const int hist_tiles = (hist + KT - 1) / KT;
  const int ntiles = hist_tiles + (vis_wg + KT - 1) / KT;
  // this workgroup's share [t_begin, t_end) of them (all of them without a split)
  const int t_begin = (int)((int64_t)split * ntiles / p.splits);
  const int t_end = (int)((int64_t)(split + 1) * ntiles / p.splits);
  const int64_t bh = (int64_t)b * p.H + h;

  Wave w;
  w.init(lane);
  // Q~ as the B operand: lane (i, g) holds Q~[q][32*st + 8g .. +7] of its two queries
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) {
    const int q = q0 + 16 * qs;
    const __bf16* qrow = p.q_rot + (bh * p.Nq + (q < p.Nq ? q : 0)) * D;
#pragma unroll
    for (int st = 0; st < Wave::KS; ++st) {
      bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0};
      if (q < p.Nq) x = *reinterpret_cast<const bf16x8*>(qrow + st * 32 + g * 8);
      w.qreg[qs][st] = x;
    }
  }

  const RowSegment k_hist = make_segment(p.k_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const RowSegment v_hist = make_segment(p.v_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const RowSegment k_chunk = make_segment(p.kc_rot + bh * p.Nq * D, D, p.Nq, D);
  const RowSegment v_chunk = make_segment(p.v_chunk + ((int64_t)b * p.Nq * p.H + h) * D, (int64_t)p.H * D, p.Nq, D);
  using Streamer = TileStreamer<D, KT, kWaves>;
  Streamer ts;
  ts.init();
  const uint32_t off_dense = ts.lane_offset(k_hist);    // stride D: ring K, ring V, rotated chunk K
  const uint32_t off_vchunk = ts.lane_offset(v_chunk);  // stride H*D
  auto issue_hist = [&](int t, char* stage) __attribute__((always_inline)) {
    ts.issue(k_hist, off_dense, t * KT, stage);
    ts.issue(v_hist, off_dense, t * KT, stage + TILE_BYTES);
  };
  auto issue = [&](int t, char* stage) __attribute__((always_inline)) {
    const bool in_hist = t < hist_tiles;
    const int row0 = (in_hist ? t : t - hist_tiles) * KT;
    const RowSegment ks = in_hist ? k_hist : k_chunk;
    const RowSegment vs = in_hist ? v_hist : v_chunk;
    ts.issue(ks, off_dense, row0, stage);
    ts.issue(vs, in_hist ? off_dense : off_vchunk, row0, stage + TILE_BYTES);
  };
  // rows of tile t that count for this lane's query qs, and whether any lane of the wave has fewer than all
  auto live_in = [&](int t, int qs) __attribute__((always_inline)) {
    if (t < hist_tiles) return hist - t * KT;
    if constexpr (kCausal)
      return vis_lds[qs * kWaves * 64 + threadIdx.x] - (t - hist_tiles) * KT;  // own entry: no barrier needed
    else
      return vis_wave - (t - hist_tiles) * KT;
  };
  auto any_dead_in = [&](int t) __attribute__((always_inline)) {
    return (t < hist_tiles ? hist - t * KT : vis_wave - (t - hist_tiles) * KT) < KT;
  };
  // Invariant at the top of tile t: tiles t .. t+kAhead-1 have landed and are visible to
  // every wave except the last of them, whose loads may still be in flight; the stage of
  // tile t+kAhead (= that of tile t-1) is free.
  constexpr int kLoadsPerTile = 2 * Streamer::kInsts;  // per wave
#pragma unroll
  for (int t = 0; t < kAhead; ++t)
    if (t_begin + t < t_end) issue(t_begin + t, lds + t * STAGE_BYTES);
  if (t_end - t_begin >= kAhead && kAhead > 1)
    wait_vmem_except<kLoadsPerTile>();
  else
    wait_vmem();
  __syncthreads();

  // kGeneric: any tile.  kHist: tile t is a full tile of ring rows and tile t+kAhead is one
  // too (possibly ragged), so nothing has to be tested: the bulk of a long window.
  constexpr int kGeneric = 0, kHist = 1;
  auto step = [&](int t, auto stage_c, auto mode_c) __attribute__((always_inline)) {
    constexpr int ST = decltype(stage_c)::value;
    constexpr int MODE = decltype(mode_c)::value;
    char* stage = lds + ST * STAGE_BYTES;
    char* refill = lds + ((ST + kAhead) % kStages) * STAGE_BYTES;
    bf16x8 kf[Wave::KH];
    w.read_k(stage, kf);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MODE == kHist)
      issue_hist(t + kAhead, refill);
    else if (t + kAhead < t_end)
      issue(t + kAhead, refill);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MODE == kGeneric) {
      const int live[2] = {live_in(t, 0), live_in(t, 1)};
      w.template tile<true>(kf, stage, stage + TILE_BYTES, live, any_dead_in(t), false, [] {});
    } else {
      const int live[2] = {KT, KT};
      w.template tile<false>(kf, stage, stage + TILE_BYTES, live, false, false, [] {});
    }
    // keep the next tile's K reads behind this tile's last MFMA: started earlier they
    // would need registers that are not there
    __builtin_amdgcn_sched_barrier(0);
    // tile t+1 .. t+kAhead-1 must have landed before the next tile starts; the newest may stay in flight
    if (kAhead > 1 && (MODE != kGeneric || t + kAhead < t_end))
      wait_vmem_except<kLoadsPerTile>();
    else
      wait_vmem();
    __syncthreads();
  };
  // kStages tiles per trip so that every LDS stage is a compile-time offset
  auto group = [&](int t, auto mode_c) __attribute__((always_inline)) {
    constexpr bool kAll = decltype(mode_c)::value != kGeneric;  // all kStages tiles exist
    step(t, std::integral_constant<int, 0>{}, mode_c);
    if (kStages > 1 && (kAll || t + 1 < t_end)) step(t + 1, std::integral_constant<int, 1 % kStages>{}, mode_c);
    if (kStages > 2 && (kAll || t + 2 < t_end)) step(t + 2, std::integral_constant<int, 2 % kStages>{}, mode_c);
    if (kStages > 3 && (kAll || t + 3 < t_end)) step(t + 3, std::integral_constant<int, 3 % kStages>{}, mode_c);
    static_assert(kStages <= 4, "unroll more steps");
  };
  int t = t_begin;
  const int fast_end = hist_tiles < t_end ? hist_tiles : t_end;
  for (; t + kStages - 1 + kAhead < fast_end; t += kStages) group(t, std::integral_constant<int, kHist>{});
  for (; t < t_end; t += kStages) group(t, std::integral_constant<int, kGeneric>{});

  // ---- epilogue: normalise, write O [B, Nq, H, D] bf16 and LSE [B, H, Nq] (of this split's keys)
  __bf16* out = p.out;
  float* lse = p.lse;
  if (p.splits > 1) {
    out = p.out_part + (int64_t)split * ((int64_t)p.BH * p.Nq * D);
    lse = p.lse_part + (int64_t)split * ((int64_t)p.BH * p.Nq);
  }
  // A key range in which a query sees nothing (no tiles at all: a split of a workgroup that sees
  // few keys under the causal mask; or only keys of later causal blocks: row sum 0) reports zero
  // output and a log-sum-exp of -1e30, which is weight 0 in the merge.  Every query sees its own
  // block, so some range of it is real.
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) {
    // the query's row sum: over the four lanes that share it
    const float l_tot = Wave::row_sum(w.l_run[qs]);
    const bool nothing = !(l_tot > 0.f);
    const float inv = nothing ? 0.f : 1.f / l_tot;
    const int q = q0 + 16 * qs;
    if (q < p.Nq) {
      __bf16* orow = out + (((int64_t)b * p.Nq + q) * p.H + h) * D;
#pragma unroll
      for (int dt = 0; dt < Wave::DT; ++dt) {
        bf16x4 x;
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = (__bf16)(w.o[dt][qs][c] * inv);
        *reinterpret_cast<bf16x4*>(orow + 16 * dt + 4 * g) = x;
      }
      if (g == 0) lse[bh * p.Nq + q] = nothing ? kNegBig : w.mc[qs] * kLn2 + __logf(l_tot);
    }
  }
}

// ---- launches with few queries -------------------------------------------------------------------
// With 128 queries per workgroup a call of a few hundred queries and a few heads is a handful of
// workgroups that walk all keys one tile after another while most of the chip idles.  Here a
// workgroup owns ONE block of 32 queries and its waves share the KEYS: wave w walks its own part of
// the key tiles, contiguous or every kWaves-th, through its own LDS buffers (no barrier in the loop), and the
// waves' unnormalised results are combined through LDS at the end.  Against the key split over
// workgroups that needs no second launch, and partial results stay fp32.  What bounds it: a CU pulls
// 16 KB of tiles (D = 128) per 32 keys for 32 queries, about 0.18 us at the 40 B per clock and CU these
// loads reach; calls of a few tiles are the chain launch, operand loads, tile, combine (5 us).
// The first tile's reference is tried at 0 (init_zero_ref): a wave walks few tiles, so recomputing the
// first one's scores for its maximum, as the general kernel does, would be a large part of the work.
//
// RawChunk: the workgroups rotate queries and chunk keys themselves, so no pre-pass has to end before the
// scores can begin: a call of a few tiles is that chain (one 64-token frame, 2 heads of 64, 4 resident frames: 10.1 -> 6.9 us).
// With one wave per SIMD every vector instruction costs its latency, about 8 cycles, so their number is what
// counts: the waves share the rotation of the queries through LDS, and a wave turns a chunk key tile in its
// buffer with positions found once per row and the lane's four rotary pairs fixed (a lane's own queries and positions
// per look-up: 45 % more instructions, 1.5 - 3 us more).  At D = 64 it keeps to the 128 registers of four workgroups per CU
// with one or two of them in scratch.
struct StagedChunk {};  // the operands are in q_rot and kc_rot
struct RawChunk {
  const __bf16 *q, *k;  // [B, Nq, H, D] as the caller passed them
  __bf16 *q_rot, *kc_rot;
  float2* tab_t;  // what the pre-pass would leave here goes there too, for a later call; null = it is not wanted
  const double* inv_freq_t;
  const float2 *tab_h, *tab_w;
  int gh, gw, T, n_t, n_h, n_w, n_frames;
  float q_scale;
  StreamInts first_frame;  // by candidate
};
// The same with the chunk's keys turned by all waves together before the walk (fwd_turns_together): a wave that turns a tile
// on its way spends 1770 cycles on it and 1000 waiting for its keys behind the tile before, of 11200 in a short call.  The
// eight waves turn theirs next to the queries, which are waited for and turned either way (2150 cycles of 9900 with both), and
// a chunk tile's values are requested a tile earlier.
struct RawChunkTogether : RawChunk {};

// The (cos, sin) a workgroup's chunk tokens need, in LDS: [n_frames][n_t], [gh][n_h], [gw][n_w], at most kEntries.
template <int kEntries>
struct ChunkTables {
  const float2* tab;
  int T, gw, n_t, nb, n_h, n_w, off_h, off_w;
  float inv_T, inv_gw;
  static constexpr int kBits = 10;
  static_assert(kEntries < 1 << kBits, "three entry numbers to a word");

  // fills `to` (the caller's barrier makes it visible)
  template <int kThreads>
  __device__ __forceinline__ void init(const RawChunk& r, float2* to, int b) {
    tab = to;
    T = r.T, gw = r.gw, n_t = r.n_t, nb = r.n_t + r.n_h, n_h = r.n_h, n_w = r.n_w;
    off_h = r.n_frames * r.n_t, off_w = off_h + r.gh * r.n_h;
    inv_T = 1.f / r.T, inv_gw = 1.f / r.gw;
    const int n_rows = r.gh * r.n_h, n_all = n_rows + r.gw * r.n_w;
    // the row and column tables are requested before the sines of the frames are computed
    constexpr int kUnroll = (kEntries + kThreads - 1) / kThreads;
    float2 x[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int e = u * kThreads + (int)threadIdx.x;
      if (e < n_all) x[u] = e < n_rows ? r.tab_h[e] : r.tab_w[e - n_rows];
    }
    for (int e = threadIdx.x; e < off_h; e += kThreads) {
      const int fi = e / n_t;
      double sn, cs;
      sincos((double)(r.first_frame.v[b] + fi) * r.inv_freq_t[e - fi * n_t], &sn, &cs);
      to[e] = make_float2((float)cs, (float)sn);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int e = u * kThreads + (int)threadIdx.x;
      if (e < n_all) to[off_h + e] = x[u];
    }
  }
  // First entries of the frame, row and column of chunk token `tok`, kBits each.  A quotient's distance from the next
  // integer is at least half a divisor's inverse, the product's error 2^-23 of it: exact below 2^22 tokens.
  __device__ __forceinline__ uint32_t position(int tok) const {
    const int f = (int)(((float)tok + 0.5f) * inv_T), rem = tok - f * T;
    const int y = (int)(((float)rem + 0.5f) * inv_gw), x = rem - y * gw;
    return (uint32_t)(f * n_t) | (uint32_t)(off_h + y * n_h) << kBits | (uint32_t)(off_w + x * n_w) << 2 * kBits;
  }
  // Which part of a position pairs 4c .. 4c + 3 take and how far behind it they are.
  struct Quad {
    uint32_t shift[4], at[4];
  };
  __device__ __forceinline__ Quad pairs(int c) const {
    Quad q;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 4 * c + v;
      q.shift[v] = j < n_t ? 0 : (j < nb ? kBits : 2 * kBits);
      q.at[v] = j - (j < n_t ? 0 : (j < nb ? n_t : nb));
    }
    return q;
  }
  __device__ __forceinline__ void cos_sin(const Quad& q, uint32_t position, float2 (&cs)[4]) const {
#pragma unroll
    for (int v = 0; v < 4; ++v) cs[v] = tab[__builtin_amdgcn_ubfe(position, q.shift[v], kBits) + q.at[v]];
  }
};

template <int D, int kWaves, bool kCausal, typename Chunk>
__global__ void __launch_bounds__(kWaves * 64, D == 128 ? 2 : 4) attn_fwd_few_kernel(FwdParams p, Chunk chunk) {
  constexpr bool kRaw = std::is_base_of_v<RawChunk, Chunk>;
  constexpr bool kTogether = std::is_same_v<Chunk, RawChunkTogether>;
  using F = FewRows<D, kWaves>;
  using Wave = FwdWave<D>;
  __shared__ __attribute__((aligned(1024))) char lds[kWaves * F::kWaveBytes];
  __shared__ __attribute__((aligned(1024))) char ctiles[kTogether ? fwd_together_tiles(D) * F::kTileBytes : 16];
  __shared__ float2 stats[kWaves][32];  // softmax reference and row sum of each wave's keys
  constexpr int kEntries = kTogether ? fwd_together_entries(D) : fwd_table_entries(D);
  __shared__ float2 tab[kRaw ? kEntries : 1];
  __shared__ __attribute__((aligned(1024))) char qtile[kRaw ? F::kTileBytes : 16];

  const int hist_of_lane = p.hist_rows.v[threadIdx.x & 63];
  // What the first loads' addresses come from, in one round of scalar loads: read where they are used, one after another, the
  // arguments were four rounds to memory, and with three integer divisions 2300 of a short call's 12000 cycles (64 rows, 2
  // heads of 64, 256 resident 6.26 -> 5.74 us, forward and backward 12.98 -> 12.21; 72 rows, 6 pairs of 128 9.8 -> 9.2).
  asm volatile("" ::"s"(p.q_tiles), "s"(p.BH), "s"((int)p.by_xcd), "s"(p.H), "s"(p.group), "s"(p.Nq), "s"(p.div.tiles), "s"(p.div.group),
               "s"(p.div.heads), "s"(p.k_cache), "s"(p.v_cache), "s"(p.v_chunk), "s"(p.cache_rows));
  if constexpr (kRaw)
    asm volatile("" ::"s"(chunk.q), "s"(chunk.k), "s"(chunk.inv_freq_t), "s"(chunk.tab_h), "s"(chunk.tab_w), "s"(chunk.gh), "s"(chunk.gw),
                 "s"(chunk.T), "s"(chunk.n_t), "s"(chunk.n_h), "s"(chunk.n_w), "s"(chunk.n_frames));
  else
    asm volatile("" ::"s"(p.q_rot), "s"(p.kc_rot), "s"((int)p.in_turn));
  if constexpr (kCausal) asm volatile("" ::"s"(p.block_rows));
  const WorkItem item = few_work_item(p.q_tiles, p.BH, p.by_xcd, p.div, (int)blockIdx.x);
  if (!item.valid) return;
  const PairIndex pair = few_split_pair(item.bh, p.H, p.group, p.div);
  const int b = pair.b, h = pair.h;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  // Every lane loads one stream's count and the wanted one is picked: indexed, the load would wait for the pair to be
  // computed from other arguments (512 rows, 16 heads, empty ring 17.7 against 18.0 us, three 99-row frames at D = 64 10.3 and 10.6).
  static_assert(ASTRO_MAX_BATCH == 64, "one stream per lane");
  const int hist = __builtin_amdgcn_readlane(hist_of_lane, pair.cache_b);
  const int64_t bh = (int64_t)b * p.H + h;
  const int q_first = item.tile * 32, q_last = p.Nq - 1;
  const int q0 = q_first + i16;  // this lane's queries: q0 and q0 + 16
  const int block_rows = kCausal ? p.block_rows : 0;
  const int vis_first = visible_chunk_rows(q_first, p.Nq, block_rows);
  const int vis_last = visible_chunk_rows(q_first + 31 < q_last ? q_first + 31 : q_last, p.Nq, block_rows);
  int vis[2];
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) vis[qs] = visible_chunk_rows(q0 + 16 * qs < q_last ? q0 + 16 * qs : q_last, p.Nq, block_rows);
  const int hist_tiles = (hist + KT - 1) / KT;
  const int ntiles = hist_tiles + (vis_last + KT - 1) / KT;

  const u32x4 k_hist = segment_words(p.k_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const u32x4 v_hist = segment_words(p.v_cache + (int64_t)pair.cache_bh * p.cache_rows * D, D, hist, D);
  const int64_t chunk_at = ((int64_t)b * p.Nq * p.H + h) * D;  // token-major tensors
  const int token_stride = p.H * D;
  const u32x4 v_chunk = segment_words(p.v_chunk + chunk_at, token_stride, p.Nq, D);
  u32x4 k_chunk;
  uint32_t k_stride = D * 2;
  if constexpr (kRaw) {
    k_chunk = segment_words(chunk.k + chunk_at, token_stride, p.Nq, D);
    k_stride = token_stride * 2;
  } else {
    k_chunk = segment_words(p.kc_rot + bh * p.Nq * D, D, p.Nq, D);
  }
  char* ktile = lds + wave * F::kWaveBytes;
  char* vtile = ktile + F::kTileBytes;
  PrivateStream<D> ps;
  ps.init(lane);
  auto issue_k = [&](int t) __attribute__((always_inline)) {
    const bool in_hist = t < hist_tiles;
    ps.issue(in_hist ? k_hist : k_chunk, in_hist ? D * 2 : k_stride, (in_hist ? t : t - hist_tiles) * KT, ktile);
  };
  auto issue_v = [&](int t) __attribute__((always_inline)) {
    const bool in_hist = t < hist_tiles;
    ps.issue(in_hist ? v_hist : v_chunk, in_hist ? D * 2 : token_stride * 2, (in_hist ? t : t - hist_tiles) * KT, vtile);
  };
  // in turn where the chunk may have to be rotated, so that its tiles fall to all waves (and the sums are the same if it is
  // not); else a share each, 0.8 % faster on long walks
  const bool in_turn = kRaw || p.in_turn;
  const int t_begin = in_turn ? wave : F::begin(wave, kWaves, 0, ntiles), t_end = in_turn ? ntiles : F::begin(wave + 1, kWaves, 0, ntiles);
  const int t_step = in_turn ? kWaves : 1;
  if (t_begin < t_end) {
    if (!kTogether || t_begin < hist_tiles) issue_k(t_begin);
    issue_v(t_begin);
  }

  Wave w;
  w.init(lane);
  w.init_zero_ref();
  ChunkTables<kEntries> tables;
  if constexpr (kTogether) {
    // A 16-byte unit of the chunk's keys per thread and trip, and of the block's queries where the rows are the same, turned
    // into LDS for all waves.
    constexpr int CPR = D / 8, kRows = kWaves * 64 / CPR, kTrips = fwd_together_tiles(D) * KT / kRows;
    static_assert(kRows % 32 == 0 && kTrips * kRows == fwd_together_tiles(D) * KT, "the rows of a trip are whole tiles, and the trips all of them");
    const int c = threadIdx.x % CPR, r0 = threadIdx.x / CPR, n_rows = (ntiles - hist_tiles) * KT;
    bf16x8 xk[kTrips], xq[kTrips];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int row = u * kRows + r0;
      xk[u] = xq[u] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
      if (row < n_rows && row < p.Nq) {
        const int64_t at = chunk_at + row * token_stride + c * 8;
        xk[u] = *reinterpret_cast<const bf16x8*>(chunk.k + at);
        if ((uint32_t)(row - q_first) < 32u) xq[u] = *reinterpret_cast<const bf16x8*>(chunk.q + at);
      }
    }
    tables.template init<kWaves * 64>(chunk, tab, b);
    const auto pairs = tables.pairs(c);
    uint32_t position[kTrips];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) position[u] = tables.position(u * kRows + r0 < p.Nq ? u * kRows + r0 : q_last);
    __syncthreads();
    if (chunk.tab_t && item.tile == 0 && h == 0)
      for (int e = threadIdx.x; e < tables.off_h; e += kWaves * 64) chunk.tab_t[(int64_t)b * tables.off_h + e] = tab[e];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int row = u * kRows + r0;
      if (row >= n_rows) continue;
      float2 cs[4];
      tables.cos_sin(pairs, position[u], cs);
      const bf16x8 k = rotate8(xk[u], cs, 1.f);
      *reinterpret_cast<bf16x8*>(ctiles + lds_chunk_offset16<D>(row, c)) = k;
      if ((uint32_t)(row - q_first) < 32u) {
        const bf16x8 q = rotate8(xq[u], cs, chunk.q_scale);
        *reinterpret_cast<bf16x8*>(qtile + lds_chunk_offset16<D>(row - q_first, c)) = q;
        if (chunk.tab_t && row < p.Nq) {
          *reinterpret_cast<bf16x8*>(chunk.q_rot + (bh * p.Nq + row) * D + c * 8) = q;
          *reinterpret_cast<bf16x8*>(chunk.kc_rot + (bh * p.Nq + row) * D + c * 8) = k;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
#pragma unroll
      for (int st = 0; st < Wave::KS; ++st) w.qreg[qs][st] = read_rows16<D>(qtile, w.addr.row[st], 16 * qs);
  } else if constexpr (kRaw) {
    // a 16-byte unit of the block's queries per thread and trip, rotated into LDS for all waves
    constexpr int CPR = D / 8, kThreads = kWaves * 64, kTrips = (32 * CPR + kThreads - 1) / kThreads;
    const int c = threadIdx.x % CPR;
    bf16x8 x[kTrips];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int row = (u * kThreads + (int)threadIdx.x) / CPR, q = q_first + row;
      x[u] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
      if (row < 32 && q < p.Nq) x[u] = *reinterpret_cast<const bf16x8*>(chunk.q + chunk_at + (int64_t)q * token_stride + c * 8);
    }
    tables.template init<kThreads>(chunk, tab, b);
    __syncthreads();
    const auto pairs = tables.pairs(c);
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int row = (u * kThreads + (int)threadIdx.x) / CPR, q = q_first + row;
      if (row >= 32) continue;
      float2 cs[4];
      tables.cos_sin(pairs, tables.position(q < p.Nq ? q : q_last), cs);
      x[u] = rotate8(x[u], cs, chunk.q_scale);
      *reinterpret_cast<bf16x8*>(qtile + lds_chunk_offset16<D>(row, c)) = x[u];
      if (chunk.tab_t && q < p.Nq) *reinterpret_cast<bf16x8*>(chunk.q_rot + (bh * p.Nq + q) * D + c * 8) = x[u];
    }
    if (chunk.tab_t && item.tile == 0 && h == 0)
      for (int e = threadIdx.x; e < tables.off_h; e += kThreads) chunk.tab_t[(int64_t)b * tables.off_h + e] = tab[e];
    __syncthreads();
#pragma unroll
    for (int qs = 0; qs < 2; ++qs)
#pragma unroll
      for (int st = 0; st < Wave::KS; ++st) w.qreg[qs][st] = read_rows16<D>(qtile, w.addr.row[st], 16 * qs);
  } else {
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      const int q = q0 + 16 * qs;
      const __bf16* qrow = p.q_rot + (bh * p.Nq + (q < p.Nq ? q : 0)) * D;
#pragma unroll
      for (int st = 0; st < Wave::KS; ++st) {
        bf16x8 x = {0, 0, 0, 0, 0, 0, 0, 0};
        if (q < p.Nq) x = *reinterpret_cast<const bf16x8*>(qrow + st * 32 + g * 8);
        w.qreg[qs][st] = x;
      }
    }
  }
  // rotates the wave's tile `t` of chunk keys where it is; the workgroup that owns these rows as queries leaves them for a later call
  auto rotate_keys = [&](int t) __attribute__((always_inline)) {
    if constexpr (kRaw) {
      constexpr int CPR = D / 8, kRows = 64 / CPR, kUnits = KT / kRows;
      const int c = lane % CPR, r0 = lane / CPR, row0 = (t - hist_tiles) * KT;
      const auto pairs = tables.pairs(c);
      const int tok = row0 + (lane & 31);  // each lane finds one row's position
      const uint32_t position = tables.position(tok < p.Nq ? tok : q_last);
      // all of the tile first: the compiler cannot tell a unit's place from another's and would wait for each in turn
      bf16x8 k[kUnits];
#pragma unroll
      for (int u = 0; u < kUnits; ++u) k[u] = *reinterpret_cast<const bf16x8*>(ktile + lds_chunk_offset16<D>(u * kRows + r0, c));
#pragma unroll
      for (int u0 = 0; u0 < kUnits; u0 += 4) {  // the look-ups of four units in flight
        float2 cs[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) tables.cos_sin(pairs, __shfl(position, (u0 + u) * kRows + r0), cs[u]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u0 + u] = rotate8(k[u0 + u], cs[u], 1.f);
      }
#pragma unroll
      for (int u = 0; u < kUnits; ++u) *reinterpret_cast<bf16x8*>(ktile + lds_chunk_offset16<D>(u * kRows + r0, c)) = k[u];
      if (chunk.tab_t && t - hist_tiles == item.tile) {
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
          const int j = row0 + u * kRows + r0;
          if (j < p.Nq) *reinterpret_cast<bf16x8*>(chunk.kc_rot + (bh * p.Nq + j) * D + c * 8) = k[u];
        }
      }
      wave_lds_sync();
    }
  };
  if constexpr (kTogether) {
    // Ring tiles as below, then the wave's one chunk tile: its keys are there, and its values have been requested into
    // the buffer that the last ring tile's keys had left.
    static_assert(fwd_together_tiles(D) <= kWaves, "a wave has one of them at most");
    int t = t_begin;
    for (; t < hist_tiles; t += t_step) {
      wait_vmem_except<PrivateStream<D>::kInsts>();  // the K tile; the V tile behind it may be in flight
      wave_lds_sync();
      bf16x8 kf[Wave::KH];
      w.read_k(ktile, kf);
      const int live[2] = {hist - t * KT, hist - t * KT};
      w.template tile<true>(kf, ktile, vtile, live, hist - t * KT < KT, t == t_begin, [&] {
        wait_lds();
        wave_lds_sync();
        if (t + t_step < hist_tiles)
          issue_k(t + t_step);
        else if (t + t_step < t_end)
          ps.issue(v_chunk, token_stride * 2, (t + t_step - hist_tiles) * KT, ktile);
        if (t + t_step < t_end)
          wait_vmem_except<PrivateStream<D>::kInsts>();
        else
          wait_vmem();
        wave_lds_sync();
      });
      wait_lds();
      wave_lds_sync();
      if (t + t_step < hist_tiles) issue_v(t + t_step);
    }
    if (t < t_end) {
      const int row0 = (t - hist_tiles) * KT;
      const char* kt = ctiles + row0 * D * 2;
      bf16x8 kf[Wave::KH];
      w.read_k(kt, kf);
      const int live[2] = {vis[0] - row0, vis[1] - row0};
      w.template tile<true>(kf, kt, t == t_begin ? vtile : ktile, live, vis_first - row0 < KT, t == t_begin, [&] {
        wait_vmem();
        wave_lds_sync();
      });
    }
  } else {
    for (int t = t_begin; t < t_end; t += t_step) {
      wait_vmem_except<PrivateStream<D>::kInsts>();  // the K tile; the V tile behind it may be in flight
      wave_lds_sync();
      if (t >= hist_tiles) rotate_keys(t);
      bf16x8 kf[Wave::KH];
      w.read_k(ktile, kf);
      const int row0 = (t < hist_tiles ? t : t - hist_tiles) * KT;
      const int live[2] = {(t < hist_tiles ? hist : vis[0]) - row0, (t < hist_tiles ? hist : vis[1]) - row0};
      // each buffer is refilled as soon as its tile is done with
      w.template tile<true>(kf, ktile, vtile, live, (t < hist_tiles ? hist : vis_first) - row0 < KT, t == t_begin, [&] {
        wait_lds();
        wave_lds_sync();
        if (t + t_step < t_end) {
          issue_k(t + t_step);
          wait_vmem_except<PrivateStream<D>::kInsts>();
        } else {
          wait_vmem();
        }
        wave_lds_sync();
      });
      wait_lds();
      wave_lds_sync();
      if (t + t_step < t_end) issue_v(t + t_step);
    }
  }

  // every wave leaves its unnormalised result and its statistics (own buffer, own tiles are done) ...
  wave_lds_sync();
#pragma unroll
  for (int qs = 0; qs < 2; ++qs) {
    const float l = Wave::row_sum(w.l_run[qs]);
    // a wave without tiles, or whose keys this query does not see (row sum 0), has weight 0
    if (g == 0) stats[wave][16 * qs + i16] = make_float2(l > 0.f ? w.mc[qs] : kNegBig, l);
#pragma unroll
    for (int dt = 0; dt < Wave::DT; ++dt) *reinterpret_cast<f32x4*>(ktile + ((dt * 2 + qs) * 64 + lane) * 16) = w.o[dt][qs];
  }
  __syncthreads();
  // ... and takes a share of the blocks of the sum, weighted to the largest reference
  constexpr int kShare = F::kUnits / kWaves;
#pragma unroll
  for (int u = 0; u < kShare; ++u) {
    const int unit = wave * kShare + u, dt = unit >> 1, qs = unit & 1;
    const int q = q0 + 16 * qs;
    float m = kNegBig, l = 0.f;
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) m = fmaxf(m, stats[wv][16 * qs + i16].x);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) {
      const float2 st = stats[wv][16 * qs + i16];
      const float wt = fast_exp2(st.x - m);
      l = fmaf(wt, st.y, l);
      x += *reinterpret_cast<const f32x4*>(lds + wv * F::kWaveBytes + (unit * 64 + lane) * 16) * wt;
    }
    if (q < p.Nq) {
      const bool nothing = !(l > 0.f);  // as in the general kernel: logits that are not finite
      const float inv = nothing ? 0.f : 1.f / l;
      bf16x4 y;
#pragma unroll
      for (int c = 0; c < 4; ++c) y[c] = (__bf16)(x[c] * inv);
      *reinterpret_cast<bf16x4*>(p.out + (((int64_t)b * p.Nq + q) * p.H + h) * D + 16 * dt + 4 * g) = y;
      if (dt == 0 && g == 0) p.lse[bh * p.Nq + q] = nothing ? kNegBig : m * kLn2 + __logf(l);
    }
  }
}

// Combine the per-split results: softmax over the union of the splits' keys is the average of the
// splits' outputs weighted by exp(lse_s - lse).  Bound by the parts' bytes (they were written just
// before: 57 MB at 4 splits of 4680 x 12 rows of 128).  Sixteen bytes per lane, so a wave takes 64 / CPR rows of
// (stream, query, head), and all parts of a row are in flight before the first is used (one wave per
// row and 4 bytes per lane, a part at a time: 29 us there).
template <int D>
__global__ void __launch_bounds__(256) fwd_merge_kernel(FwdParams p, int64_t n_rows) {
  constexpr int CPR = D / 8;
  const int64_t row = (int64_t)blockIdx.x * (256 / CPR) + threadIdx.x / CPR;  // (b*Nq + q)*H + h
  if (row >= n_rows) return;
  const int c = threadIdx.x % CPR;
  // (rows of 128 bytes and more: their number fits 32 bits)
  const uint32_t bq = (uint32_t)row / (uint32_t)p.H, b = bq / (uint32_t)p.Nq;
  const int h = (int)((uint32_t)row - bq * p.H), q = (int)(bq - b * p.Nq);
  const int64_t lse_at = ((int64_t)b * p.H + h) * p.Nq + q;
  const int64_t out_stride = (int64_t)p.BH * p.Nq * D, lse_stride = (int64_t)p.BH * p.Nq;
  bf16x8 o[kMaxFwdSplits];
  float l[kMaxFwdSplits];
  float m = kNegBig;
#pragma unroll
  for (int s = 0; s < kMaxFwdSplits; ++s)
    if (s < p.splits) {
      o[s] = *reinterpret_cast<const bf16x8*>(p.out_part + s * out_stride + row * D + c * 8);
      l[s] = p.lse_part[s * lse_stride + lse_at];
      m = fmaxf(m, l[s]);
    }
  float tot = 0.f, a[8] = {};
#pragma unroll
  for (int s = 0; s < kMaxFwdSplits; ++s)
    if (s < p.splits) {
      const float w = __expf(l[s] - m);
      tot += w;
#pragma unroll
      for (int j = 0; j < 8; ++j) a[j] = fmaf(w, (float)o[s][j], a[j]);
    }
  const float inv = 1.f / tot;
  bf16x8 x;
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = (__bf16)(a[j] * inv);
  *reinterpret_cast<bf16x8*>(p.out + row * D + c * 8) = x;
  if (c == 0) p.lse[lse_at] = m + __logf(tot);
}

FwdParams make_params(const DevGeom& g, const AttnOperands& op, void* out, float* lse) {
  FwdParams p;
  p.q_rot = (const __bf16*)op.q_rot;
  p.kc_rot = (const __bf16*)op.kc_rot;
  p.v_chunk = (const __bf16*)op.v_chunk;
  p.k_cache = (const __bf16*)op.k_cache;
  p.v_cache = (const __bf16*)op.v_cache;
  p.out = (__bf16*)out;
  p.lse = lse;
  p.H = g.H;
  p.Nq = op.Nq;
  p.cache_rows = (int64_t)g.C * g.T;
  p.hist_rows = op.hist_rows;
  p.group = op.group;
  p.block_rows = op.block_rows;
  p.BH = g.B * g.H;
  p.q_tiles = 0;
  p.by_xcd = true;
  p.in_turn = false;
  p.div = FewDivisors{};
  p.splits = 1;
  p.out_part = nullptr;
  p.lse_part = nullptr;
  return p;
}

// (cos, sin) that a chunk's rotation takes
int64_t fwd_entries(const DevGeom& g, const AttnOperands& op) {
  return (int64_t)(op.Nq / g.T) * g.n_t + (int64_t)g.gh * g.n_h + (int64_t)g.gw * g.n_w;
}

template <int D, int kWaves, bool kCausal>
hipError_t launch_few(const DevGeom& g, const AttnOperands& op, void* out, float* lse, hipStream_t stream) {
  FwdParams p = make_params(g, op, out, lse);
  p.q_tiles = (op.Nq + 31) / 32;
  p.div = few_divisors(p.q_tiles, p.group, p.H);
  const dim3 grid(work_grid_size(p.q_tiles, p.BH)), block(kWaves * 64);
  if (const ChunkSource* from = op.raw) {
    const RawChunk c{(const __bf16*)from->q, (const __bf16*)from->k, (__bf16*)op.q_rot, (__bf16*)op.kc_rot,
               from->leave ? (float2*)op.tab_t : nullptr, g.inv_freq_t, g.tab_h, g.tab_w, g.gh, g.gw, g.T, g.n_t, g.n_h, g.n_w,
               op.Nq / g.T, from->q_scale, from->first_frame};
    ProfileScope prof("attn_fwd_few_rotating_bf16", stream);
    if constexpr (kWaves == 8) {
      if (fwd_turns_together(call_shape(g, op), fwd_entries(g, op))) {
        attn_fwd_few_kernel<D, kWaves, kCausal, RawChunkTogether><<<grid, block, 0, stream>>>(p, RawChunkTogether{c});
        return hipGetLastError();
      }
    }
    attn_fwd_few_kernel<D, kWaves, kCausal, RawChunk><<<grid, block, 0, stream>>>(p, c);
  } else {
    p.in_turn = bf16_fwd_rotates(g, op);
    ProfileScope prof("attn_fwd_few_bf16", stream);
    attn_fwd_few_kernel<D, kWaves, kCausal, StagedChunk><<<grid, block, 0, stream>>>(p, StagedChunk{});
  }
  return hipGetLastError();
}

template <int D, int kStages, int kWaves, int OCC, bool kCausal>
hipError_t launch(const DevGeom& g, const AttnOperands& op, void* out, float* lse, void* parts, hipStream_t stream) {
  FwdParams p = make_params(g, op, out, lse);
  const int qtile = kWaves * 32;
  p.q_tiles = (op.Nq + qtile - 1) / qtile;
  // a launch that would leave the chip under two rounds of workgroups is split over the keys
  const CallShape shape = call_shape(g, op);
  p.splits = parts ? fwd_splits(shape) : 1;
  p.by_xcd = order_by_xcd(shape, p.q_tiles * p.BH * p.splits);
  p.out_part = (__bf16*)parts;
  p.lse_part = (float*)((char*)parts + (size_t)p.splits * p.BH * op.Nq * D * 2);
  dim3 grid(work_grid_size(p.q_tiles, p.BH * p.splits));
  {
    ProfileScope prof("attn_fwd_bf16", stream);
    attn_fwd_bf16_kernel<D, kStages, kWaves, OCC, kCausal><<<grid, dim3(kWaves * 64), 0, stream>>>(p);
  }
  if (p.splits > 1) {
    const int64_t n_rows = (int64_t)p.BH * op.Nq;
    ProfileScope prof("attn_fwd_merge", stream);
    constexpr int kRows = 256 / (D / 8);
    fwd_merge_kernel<D><<<dim3((unsigned)((n_rows + kRows - 1) / kRows)), 256, 0, stream>>>(p, n_rows);
  }
  return hipGetLastError();
}

}  // namespace

bool bf16_fwd_rotates(const DevGeom& g, const AttnOperands& op) {
  return g.n_t + g.n_h + g.n_w != 0 && fwd_rotates(call_shape(g, op), fwd_entries(g, op));
}

size_t bf16_fwd_split_bytes(const DevGeom& g, int Nq) {
  if (!fwd_may_split(g.n_cus, g.B * g.H, Nq)) return 0;
  return (size_t)kMaxFwdSplits * g.B * g.H * Nq * ((size_t)g.D * 2 + sizeof(float));
}

hipError_t launch_attn_fwd_bf16(const DevGeom& g, const AttnOperands& op, void* out, float* lse, void* parts,
                                hipStream_t stream) {
  const bool causal = op.block_rows > 0;
  const int waves = fwd_few_waves(call_shape(g, op));
  if (waves != 0 && g.D == 128) {
    if (waves == 8) return causal ? launch_few<128, 8, true>(g, op, out, lse, stream) : launch_few<128, 8, false>(g, op, out, lse, stream);
    return causal ? launch_few<128, 4, true>(g, op, out, lse, stream) : launch_few<128, 4, false>(g, op, out, lse, stream);
  }
  if (waves != 0) {
    if (waves == 8) return causal ? launch_few<64, 8, true>(g, op, out, lse, stream) : launch_few<64, 8, false>(g, op, out, lse, stream);
    return causal ? launch_few<64, 4, true>(g, op, out, lse, stream) : launch_few<64, 4, false>(g, op, out, lse, stream);
  }
  if (g.D == 128)
    return causal ? launch<128, 3, 4, 3, true>(g, op, out, lse, parts, stream) : launch<128, 3, 4, 3, false>(g, op, out, lse, parts, stream);
  return causal ? launch<64, 3, 4, 3, true>(g, op, out, lse, parts, stream) : launch<64, 3, 4, 3, false>(g, op, out, lse, parts, stream);
}

}  // namespace astro
