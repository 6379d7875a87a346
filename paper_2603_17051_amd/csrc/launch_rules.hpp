// Which kernel an attention call of the bf16 path takes and into how many key ranges it is cut: plain functions of
// sizes, without HIP.
#pragma once
#include <cstddef>
#include <cstdint>
#include <initializer_list>

namespace astro {

inline int blocks_of(int rows, int block) { return (rows + block - 1) / block; }

// What the rules look at of one call.
struct CallShape {
  int D, n_cus;
  int pairs;               // candidates * heads
  int Nq, block_rows;      // chunk rows; causal block in rows, 0 = none
  int max_hist;            // resident rows of the stream with the most
  double mean_hist;
  double xcd_load;  // key rows in the heaviest contiguous eighth of the workgroups over the mean eighth's
  bool in_order;    // see AttnOperands::in_order
  int ring_blocks, joint_blocks;  // blocks of 128 keys over all pairs: of resident rows, of resident and then chunk rows
};

// xcd_load of streams with these many key rows each
inline double heaviest_eighth(const int32_t* hist, int streams, int Nq) {
  double sum = 0., heaviest = 0.;
  for (int b = 0; b < streams; ++b) sum += (double)hist[b] + Nq;
  for (int x = 0; x < 8; ++x) {  // in units of 1 / 8 stream: eighth x is [x * streams, (x + 1) * streams), stream b is [8 b, 8 b + 8)
    double load = 0.;
    for (int b = x * streams / 8; b < streams && 8 * b < (x + 1) * streams; ++b) {
      const int from = 8 * b > x * streams ? 8 * b : x * streams;
      const int to = 8 * b + 8 < (x + 1) * streams ? 8 * b + 8 : (x + 1) * streams;
      load += (to - from) * ((double)hist[b] + Nq);
    }
    heaviest = load > heaviest ? load : heaviest;
  }
  return sum > 0. ? heaviest / sum : 1.;
}

inline CallShape make_call_shape(int D, int n_cus, int pairs, int Nq, int block_rows, bool in_order, const int32_t* hist, int streams) {
  CallShape c{D, n_cus, pairs, Nq, block_rows, hist[0], 0., 1., in_order, 0, 0};
  int64_t sum = 0;
  bool even = true;
  for (int b = 0; b < streams; ++b) {
    c.max_hist = hist[b] > c.max_hist ? hist[b] : c.max_hist;
    even = even && hist[b] == hist[0];
    sum += hist[b];
    c.ring_blocks += pairs / streams * blocks_of(hist[b], 128);
    c.joint_blocks += pairs / streams * blocks_of(hist[b] + Nq, 128);
  }
  c.mean_hist = (double)sum / streams;
  if (!even) c.xcd_load = heaviest_eighth(hist, streams, Nq);
  return c;
}


// keys a query sees, over all streams and, under causal blocks, over the chunk
inline double mean_keys(const CallShape& c) {
  if (c.block_rows <= 0 || c.block_rows >= c.Nq) return c.mean_hist + c.Nq;
  double seen = 0.;
  for (int first = 0; first < c.Nq; first += c.block_rows) {
    const int end = first + c.block_rows < c.Nq ? first + c.block_rows : c.Nq;
    seen += (double)(end - first) * end;
  }
  return c.mean_hist + seen / c.Nq;
}

// Whether the general kernels' launch of `workgroups` gives each XCD a contiguous eighth of them.  With streams of
// different lengths the XCDs that got the short ones idle: two streams of 0 and 10 production frames, 3
// heads, forward 371 us against 295 in the plain order.  Over 800 launches of 2 - 8 streams of random lengths the
// contiguous order costs nothing up to 1.2 times the mean load in the heaviest eighth (the median of contiguous over
// plain is 0.98 to 1.00, then 1.02 at 1.2 - 1.3, 1.06 at 1.3 - 1.5, 1.10 and more above); where
// every workgroup has a CU to itself the order does not change what an XCD does.  (The kernels for few
// rows keep the contiguous order: their workgroups are short and pull more through the L2s.)
inline bool order_by_xcd(const CallShape& c, int workgroups) { return c.xcd_load < 1.15 || workgroups <= c.n_cus; }

// n / d for 0 <= n and 0 < d below 2^15, from the divisor's inverse that the host passes: (n + 1/2) / d lies at least 1 / 2d
// from an integer, and the inverse, rounded down, takes less than (2n + 1) / 2^32 off.  A launch of few rows has three
// such divisions in front of its first load, 40 dependent instructions each by the compiler's way.
constexpr uint32_t inverse_of(int d) { return 0x80000000u / (uint32_t)d; }
constexpr int quotient(int n, uint32_t inverse) { return (int)((uint64_t)(2u * (uint32_t)n + 1u) * inverse >> 32); }
struct FewDivisors {
  uint32_t tiles, group, heads;
};
inline FewDivisors few_divisors(int tiles, int group, int heads) { return {inverse_of(tiles), inverse_of(group), inverse_of(heads)}; }

// ==== forward ======================================================================================
constexpr int kMaxFwdSplits = 8;  // most key ranges of a launch
constexpr int kFwdKeyTile = 32;   // keys per LDS tile

// ---- key-range split of launches that cannot fill the chip -----------------------------------
// With fewer than six workgroups per CU, two rounds at D = 128 (one stream of 12 heads and 37 query tiles is
// 444 workgroups on 768 places), each (pair, query tile) may be cut into `splits` key ranges, at most kMaxFwdSplits and never less than
// kMinTilesPerSplit key tiles each.
constexpr int kMinTilesPerSplit = 4, kFwdWorkgroupsPerCu = 3;

// whether a launch of this size may be cut at all (the workspace then holds kMaxFwdSplits partial results)
inline bool fwd_may_split(int n_cus, int pairs, int Nq) { return blocks_of(Nq, 128) * pairs < 2 * kFwdWorkgroupsPerCu * n_cus; }

inline int fwd_splits(const CallShape& c) {
  if (!fwd_may_split(c.n_cus, c.pairs, c.Nq)) return 1;
  const int items = blocks_of(c.Nq, 128) * c.pairs, places = kFwdWorkgroupsPerCu * c.n_cus;
  // Key tiles of the mean workgroup.  Ranges of a stream with few frames, or of the first causal blocks, may come
  // out empty or unseen for some queries: both report weight 0 to the merge.  (By the workgroup with the fewest
  // tiles, four streams of 0, 7, 9 and 10 frames, 72 workgroups, were not cut at all because of the first: 236 us,
  // 62 in seven ranges.)
  const double tiles = mean_keys(c) / kFwdKeyTile;
  // Enough parts for two rounds ...
  int s = (2 * places + items - 1) / items;
  if (s > kMaxFwdSplits) s = kMaxFwdSplits;
  if (s > tiles / kMinTilesPerSplit) s = (int)(tiles / kMinTilesPerSplit);
  if (s <= 1) return 1;
  if (c.in_order) return s;  // the merge launch writes the outputs
  // ... unless another count is clearly better by this estimate, in us: items * n / places rounds of 1 / n of the walk
  // each, where a last round with j workgroups on a CU takes tail[j] of a full one; a part and item for writing and
  // merging it, and the merge launch; a share of what the longest stream's walk is over the mean.  Fitted to every
  // count at 2517 shapes of 1 to 1535 workgroups (median error 3 %); what it then picks is 0.6 % (D = 128) and 1.1 % (D = 64)
  // slower than the best count in the mean.  It replaces an estimate with three workgroups per CU and a merge twice as
  // dear, which left D = 64 launches uncut that gain by it: 240 workgroups x 165 tiles 110 us uncut, 64 in four; 480 x 341
  // 239 uncut, 194 in five.
  const bool d128 = c.D == 128;
  const int per_cu = d128 ? 3 : 4;  // workgroups a CU holds: 166 registers, or 108
  const double per_tile = d128 ? 0.95 : 0.63, launch = d128 ? 3.4 : 3.5, per_part = d128 ? 0.013 : 0.006;
  static constexpr double kTail[2][4] = {{0.53, 0.74, 1., 1.}, {0.51, 0.66, 0.88, 1.}};
  auto cost = [&](int n) {
    const int64_t wgs = (int64_t)items * n, round = (int64_t)per_cu * c.n_cus, rest = wgs % round;
    const double rounds = (double)(wgs / round) + (rest ? kTail[d128 ? 0 : 1][(rest + c.n_cus - 1) / c.n_cus - 1] : 0.);
    const double over = 0.4 * (c.max_hist - c.mean_hist) / kFwdKeyTile;
    return per_tile * (rounds * tiles + over) / n + (n > 1 ? launch + per_part * wgs : 0.);
  };
  int best = 1;
  for (int n = 2; n <= kMaxFwdSplits && n <= tiles / kMinTilesPerSplit; ++n)
    if (cost(n) < cost(best)) best = n;
  return cost(best) < 0.93 * cost(s) ? best : s;
}

// ---- which launches take one block of 32 queries per workgroup -------------------------------------
// Such a workgroup pulls every key tile for 32 queries only, four times the tile traffic per query of
// the general kernel, and needs no merge launch.  Its time follows the workgroups on the fullest CU times the
// tiles, so the product below is bounded, and lower where the last round of CUs is nearly empty.  Measured (us;
// few / general):
//   D = 128: 4 workgroups x 10 tiles 7.1 / 10.7, 144 x 33 12.2 / 23.8, 132 x 109 24.5 / 31.2, 140 x 133
//            28.1 / 33.7, 320 x 140 42 / 48, 624 x 29 24 / 48; lost: 70 x 133 26.7 / 24.5, 156 x 232 45.1 /
//            43.8, 270 x 164 58 / 44, 288 x 136 55 / 39, 576 x 6 25 / 22, 640 x 8 28 / 26, 392 x 634 167 / 161
//   D = 64:  4 x 10 5.1 / 9.6, 144 x 33 8.2 / 19.9, 140 x 133 16.3 / 26.6, 156 x 232 25.6 / 34.0, 960 x 112 55 / 58, 1440 x 60
//            49 / 58; lost: 294 x 342 72 / 51, 279 x 495 88 / 65, 288 x 456 89 / 58, 294 x 634 117 / 80
// Many short walks are many prologues and combines: from the third workgroup per CU on it took, by tiles, 1.01 - 1.19
// of the general kernel's time at D = 128 below 24 tiles and 0.97 - 1.07 above, 1.05 - 1.6 from the fifth on
// (1728 x 8 51 / 44); at D = 64 0.82 - 1.0 up to the fifth, 0.97 - 1.05 from 12 tiles on up to the eighth, 1.0 - 1.27
// beyond (8320 x 26 144 / 125).
// Below half a round the general kernel's key split reaches CUs that this one leaves idle, hence the
// lower bound there.  The walk is the longest stream's; where streams differ, the general kernel, which cuts
// it, takes over at half the bounds and beyond three (D = 128) or five workgroups per CU (longest and mean walk: 1056 x
// 180, 89 88 / 56; 432 x 216, 148 46 / 38; 1536 x 28, 19 61 / 48; the other way 480 x 54, 42 30 / 39; 7 % in the mean of 85 such
// launches).  Returns the waves per workgroup, 0 = the general kernel: eight where every CU has one workgroup at
// most and the walk has 16 tiles (D = 64: 8) or more, else four.  Four waves are one per SIMD, whose tile then costs its
// latency: of 1000 shapes eight take, by tiles, D = 64 0.95 of the time at 5 - 16, 0.9 at 17 - 32, 0.83 at 64 and 0.7 above
// 100 (144 x 34 9.6 against 11.9 us, 192 x 135 17.7 / 24.7), D = 128 0.9 from 8 tiles on and 0.85 above 64 (128 x 23 12.1 / 14.1, 132 x
// 82 22.1 / 28.0).  At D = 128 the line could lie at 8 tiles by that (medians 0.90 at 8 - 11 tiles, 39 shapes, 0.91 at 12 - 15, 44); it
// is not there yet.  Where two workgroups of four
// share a CU nothing is gained (312 x 153, D = 64 32.0 / 32.8) or lost (D = 128 1.2).  Sixteen waves: 10.2 at the 144 x 34.
inline int fwd_few_waves(const CallShape& c) {
  if (c.in_order) return 0;
  const int64_t wgs = (int64_t)blocks_of(c.Nq, 32) * c.pairs;
  const int64_t tiles = blocks_of(c.max_hist, kFwdKeyTile) + blocks_of(c.Nq, kFwdKeyTile);
  const int64_t walk = wgs > c.n_cus ? tiles * wgs / c.n_cus : tiles;
  const int64_t per_cu = (wgs + c.n_cus - 1) / c.n_cus;  // on the fullest CU
  const double fill = (double)wgs / (per_cu * c.n_cus);
  const bool half_full = 2 * wgs >= c.n_cus, uneven = c.xcd_load >= 1.15;
  int64_t limit;
  if (c.D == 128) {
    if (per_cu > 4 || (per_cu > 2 && tiles < 24)) return 0;
    limit = !half_full ? 112 : per_cu == 2 && fill < 0.63 ? 100 : 200;
  } else {
    if (per_cu > 8 || (per_cu > 5 && tiles < 12)) return 0;
    limit = !half_full ? 300 : per_cu > 2 ? 900 : per_cu == 2 && fill < 0.7 ? 250 : 400;
  }
  if (uneven) limit = per_cu > (c.D == 128 ? 3 : 5) ? 0 : limit / 2;
  if (walk > limit) return 0;
  return wgs <= c.n_cus && tiles >= (c.D == 128 ? 16 : 8) ? 8 : 4;
}

// Whether such a launch rotates queries and chunk keys itself instead of waiting for a pre-pass; `entries` =
// (cos, sin) its chunk needs, which have to fit the LDS next to the tiles of the two (D = 64: four) workgroups of
// four waves a CU holds.  It saves the pre-pass, 4 us of the chain, and every workgroup rotates all chunk keys it
// sees, about 1 us per tile of a wave.  Measured (us; rotating / pre-pass and attention), by chunk tiles per wave:
//   four waves, D = 64: 0.5 7.5 / 11.4, 1 8.4 / 10.8, 2 10.5 / 12.0, 2.75 13.2 / 14.3, 3 11.7 / 12.6; lost: 3.25 11.9 / 11.7, 6.5 14.1 / 12.0
//   four waves, D = 128: 0.5 8.5 / 10.6, 1 12.6 / 13.5, 1.25 11.8 / 11.9, 1.5 11.7 / 12.3, 2 10.8 / 11.4; lost: 2.25 16.2 / 14.7, 4.25 18.6 / 15.3
//   eight waves, ratio over 800 shapes, D = 64: 0.5 0.80, 1 0.82, 1.5 0.88, 2 0.92, 2.5 0.96, 3 1.01; D = 128: 0.82, 0.86, 0.94, 0.97, lost:
//   2.5 1.02, 3 1.06
// most chunk tiles of such a launch
constexpr int fwd_rotated_tiles(int D, int waves) { return D == 128 ? 2 * waves : waves == 8 ? 20 : 3 * waves; }
constexpr int fwd_table_entries(int D) { return D == 128 ? 896 : 384; }
inline bool fwd_rotates(const CallShape& c, int64_t entries) {
  const int waves = fwd_few_waves(c);
  return entries <= fwd_table_entries(c.D) && blocks_of(c.Nq, kFwdKeyTile) <= fwd_rotated_tiles(c.D, waves);
}

// Whether the eight waves of such a launch turn the chunk's keys together into LDS before the walk instead of each its own
// tiles on the way.  All wait for all of it, so the chunk has to be short: up to a tile a wave at D = 64, and what fits the LDS
// next to the tiles at D = 128.  Measured (us, each its own / together): D = 64, chunk + ring tiles, 2 + 8 5.8 / 5.3, 4 + 13 6.6 / 6.3, 4 + 72
// 10.8 / 10.3, 4 + 23 7.9 / 7.4, 7 + 100 14.1 / 12.7; D = 128, 2 + 16 9.2 / 8.4, 2 + 24 10.2 / 9.3.  With room for sixteen tiles, two to a wave,
// 9 + 25 gained 0.2 and 16 + 48 0.3, but the short ones lost 0.3 to the longer code.
constexpr int fwd_together_tiles(int D) { return D == 128 ? 2 : 8; }
constexpr int fwd_together_entries(int D) { return D == 128 ? 512 : 384; }
inline bool fwd_turns_together(const CallShape& c, int64_t entries) {
  return fwd_few_waves(c) == 8 && blocks_of(c.Nq, kFwdKeyTile) <= fwd_together_tiles(c.D) && entries <= fwd_together_entries(c.D);
}

// ==== backward =====================================================================================
constexpr int kBwdKeyTile = 64;    // keys per LDS tile of the general dQ kernel
constexpr int kFewMaxRows = 2048;  // most chunk rows of the kernel for few rows (it holds their row terms in LDS)

// Which launches take blocks of 32 rows: those whose blocks of 128 rows would leave most CUs with one
// workgroup or none.  Measured (us of the backward; few / general, split where it splits; blocks of 128 x key tiles of 64):
//   D = 128: 2 blocks 11 / 25, 48 25 / 55, 80 x 45 63 / 98, 96 x 56 73 / 80, 104 x 317 261 / 278; lost: 120 x 128 156 / 145,
//            144 x 15 71 / 66, 144 x 21 96 / 78, 160 x 20 93 / 76, 156 x 463 563 / 406, 192 x 14 70 / 60
//   D = 64:  2 blocks 7 / 16, 48 14 / 33, 104 137 / 165, 120 x 128 82 / 90, 192 x 14 32 / 38; lost: 156 x 463 267 / 236, 216 x 32
//            83 / 67, 240 x 35 77 / 67, 256 x 35 90 / 70, 256 x 9 46 / 43, 224 x 49 74 / 67
// Over 3800 shapes it takes 0.6 - 1.0 of the general kernels' time (medians by number of tiles) just below these lines
// and 1.0 - 1.3 just above them.  Walks of 40 tiles and more, which the general dQ kernel splits, have the line
// lower, short ones higher (129 - 144 blocks below 15 tiles at D = 128 0.67 - 0.88, 225 - 240 below 10 at D = 64 0.9 - 1.0).
// Returns the waves per workgroup, 0 = the general kernels: eight where the workgroups of both sides have a CU
// each and the walk is more than 24 tiles, four otherwise.  Of 1400 shapes eight take, by tiles, 1.05 - 1.15 of the time of four below 16,
// 1.0 at 17 - 24, 0.95 at 25 - 32, 0.9 to 48, 0.85 to 64, 0.75 above 100 (24 x 114, D = 128 24.6 / 31.0 us); with more workgroups
// 1.2 - 1.5 (176 x 49 28.8 / 22.8), 1.0 - 1.15 from 64 tiles on (132 x 82 31.3 / 29.1) up to 160 workgroups, where 0.8 - 1.0 remains above 192 tiles.
inline int bwd_few_waves(const CallShape& c) {
  if (c.in_order) return 0;
  const int64_t blocks = (int64_t)blocks_of(c.Nq, 128) * c.pairs;
  const int tiles = (c.max_hist + c.Nq) / kBwdKeyTile;
  const int sixteenths = c.D == 128 ? (tiles >= 40 ? 7 : tiles >= 15 ? 8 : 9)  // of the CUs
                                    : (tiles >= 40 ? 8 : tiles >= 10 ? 12 : tiles >= 3 ? 15 : 16);
  if (c.Nq > kFewMaxRows || 16 * blocks > sixteenths * (int64_t)c.n_cus) return 0;
  const int64_t wgs = (int64_t)blocks_of(c.Nq, 32) * c.pairs;
  const int tiles32 = (c.max_hist + c.Nq) / 32;
  return 2 * wgs <= c.n_cus ? (tiles32 > 24 ? 8 : 4) : 8 * wgs <= 5 * (int64_t)c.n_cus && tiles32 > 192 ? 8 : 4;
}

// Whether the row terms of such a launch (-LSE log2(e) and -Delta of every query) come from a launch of their own.  Otherwise
// every workgroup of the key side computes those of its whole pair, dO and O once more for each block of 32 keys; that is
// cheaper than a launch (2 us) for short chunks, and hidden behind the query side where the ring is much longer
// than the chunk.  Backward with the launch over without, by chunk rows, at 400 shapes: D = 128, ring below 3 chunks 256 - 383 0.95 -
// 1.00, 384 - 511 0.92 - 1.00, 512 - 699 0.90 - 0.95, 700 - 999 0.86 - 0.97, above 0.83 - 1.00 (one 1.05), ring above 1.0 - 1.1; D = 64, ring below
// 2 chunks 384 - 511 0.98 - 1.08, 512 - 699 0.93 - 1.03, above 0.82 - 0.98, ring above up to 1.1.  672 rows, 3 pairs, 448 ring rows 21.1 -> 19.0 us.
inline bool bwd_terms_first(const CallShape& c) {
  return c.D == 128 ? c.Nq >= 384 && c.max_hist < 3 * (int64_t)c.Nq : c.Nq >= 512 && c.max_hist < 2 * (int64_t)c.Nq;
}

// Which kernel a dK / dV launch over so many blocks of 128 keys takes (blocks with keys: workgroups past the end of a shorter stream
// return at once): 0 = a pair of waves per block of 32 keys (roles), 1 or 2 = that many waves with both gradients each.  At D = 64
// one wave holds both; three such workgroups share a CU where a workgroup of roles has it alone, so launches of more than one to a
// CU gain.  Up to there two waves per block share the queries, and it is the length of the walk that decides: the roles' epilogue is
// shorter, and with ring rows their table of frames is computed beside the last tile.  Measured (us of the launch, D = 64; tiles of 64
// queries, roles / two waves / one wave, the same at 17 and at 255 workgroups within a tenth):
//   chunk: 7 tiles 17.1 / 17.9 / 20.1, 10 20.9 / 21.0 / 24.8, 12 23.2 / 22.6 / 27.4, 14 24.5 / 24.3 / 29.9, 16 26.5 / 25.8 / 32.7, 20 30.2 / 28.7 / 37.8, 25 35.7 /
//          33.7 / 45.4, 28 37.4 / 34.8 / 48.1, 34 39.6 / 36.7 / 53.9
//   ring:  8 tiles 16.8 / 17.6, 12 20.5 / 20.7, 16 24.1 / 23.8, 20 27.6 / 26.8 / 33.4, 24 31.2 / 29.7, 28 34.7 / 32.9, 32 38.3 / 36.0
//   more than one to a CU: 7 tiles, 288 workgroups 27.9 / 29.6 / 24.1, 34 tiles, 272 78.1 / 72.6 / 65.4, 340 79.2 / 72.5 / 66.8
inline int dkv_halves(const CallShape& c, int blocks) {
  if (c.D == 128) return 0;
  if (blocks > c.n_cus) return 1;
  return blocks_of(c.Nq, 64) >= 14 ? 2 : 0;
}
inline int chunk_blocks(const CallShape& c) { return blocks_of(c.Nq, 128) * c.pairs; }

// Whether the ring's key blocks and the chunk's go out in one launch (non-detached backward).  It takes the kernel that the chunk's
// launch takes by itself, so dK and dV of the chunk are the detached backward's bit for bit.  Under causal blocks it would take keys
// past queries that do not see them.  One wave per block: a launch less with a partly filled end of its own, always a gain.  Otherwise
// a CU works on one block at a time, and the launch has to save a round of them; where it saves none, a short walk still gains
// from the launch that is not there, and a long one loses to the instance for both, which is 1 % slower.  Measured (us of forward and
// backward, one launch / two, or their ratio; rounds of the launch / of chunk + ring):
//   D = 128: 12 / 2 + 11 3419 / 3513, 24 / 4 + 21 6950 / 7087, 48 / 7 + 42 13549 / 13964, 7 / 2 + 6 619 / 655, 2 / 1 + 2 554 / 671; as many rounds, by rounds times
//           tiles of 64 queries: to 12 0.94 - 0.97, to 32 0.96 - 1.01, to 66 0.985 - 1.00, 116 - 148 1.01
//   D = 64, one wave: 296 chunk and 392 ring blocks 472 / 530, 592 and 2352 1766 / 1811
//   D = 64, two waves: 2 / 1 + 2 333 / 384, 342 / 394, 3 / 1 + 3 510 / 545, 165 / 176, 5 / 1 + 5 860 / 878, 6 / 1 + 6 982 / 992; as many, to 62 0.96 - 1.003, 105 - 222 1.02 -
//           1.06 (2 / 1 + 1 at 148 0.99)
//   D = 64, roles: 5 / 1 + 5 123 / 116, 7 / 1 + 7 167 / 151 (in two launches the ring's takes one wave)
inline bool bwd_joins(const CallShape& c) {
  if (c.in_order || c.block_rows != 0 || c.max_hist == 0 || bwd_few_waves(c) != 0) return false;
  const int chunk = chunk_blocks(c), halves = dkv_halves(c, chunk);
  if (halves == 1) return true;
  if (c.D == 64 && halves == 0) return false;
  const int rounds = blocks_of(c.joint_blocks, c.n_cus), apart = blocks_of(chunk, c.n_cus) + blocks_of(c.ring_blocks, c.n_cus);
  return rounds < apart || rounds * blocks_of(c.Nq, 64) <= 64;
}

// dQ workgroups a CU holds: 244 registers (split 256), or 165 (split 168, 8 more in scratch)
constexpr int dq_places_per_cu(int D) { return D == 128 ? 2 : 3; }

// How a dQ launch is split over the keys: `ways` parts (1 = not, 2 = a helper per k items, 3 = two helpers per item;
// items = workgroups without a split).  By an estimate in us: rounds of places times the tiles of a part, where a
// last round with j workgroups on a CU takes tail[j] of a full one; with a split, the merge launch and a part of it per
// item.  Fitted to every way at 2235 shapes of 2 to 1500 items (median error 3 %); what it picks is 0.3 % (D =
// 128) and 0.6 % (D = 64) slower than the best way in the mean.  Measured (us of the backward; split / not, D = 128 unless
// said otherwise):
//   111 items x 512 tiles in three 478 / 807, 156 x 463 in three 406 (in two 518) / 674, 185 x 317 in two 460 / 552, 300 x
//   488 894 / 1109, 444 x 512 a helper per seven 1306 / 1345, 518 x 366 in three 1369 / 1627, 740 x 366 in two 1695 /
//   1758, D = 64 592 x 366 792 / 856; not split: 480 x 45 a helper per fifteen 241 / 195, 480 x 80 325 / 284, 384 x 40 187 / 181,
//   D = 64 480 x 40 106 / 93, 640 x 45 157 / 149, 720 x 45 198 / 166, 432 x 86 174 / 163
// A helper of several items whose walks differ finishes with the longest, so streams of different lengths have a helper each
// (444 items, 1560 to 17160 rows, D = 64: a helper per eight 562, each 508).
struct DqWays {
  int ways = 1, k = 1;
};
inline DqWays dq_ways(const CallShape& c) {
  const int items = blocks_of(c.Nq, 128) * c.pairs, places = dq_places_per_cu(c.D) * c.n_cus;
  if (c.in_order || 2 * items > 3 * places) return {};
  const bool d128 = c.D == 128;
  const double tiles = mean_keys(c) / kBwdKeyTile;
  const double per_tile = d128 ? 2.17 : 1.71, launch = d128 ? 5.9 : 6.4, per_item = d128 ? 0.042 : 0.022;
  static constexpr double kTail[2][3] = {{0.69, 1., 1.}, {0.52, 0.71, 1.}};
  auto cost = [&](const DqWays& w) {
    const int wgs = w.ways == 1 ? items : w.ways == 3 ? 3 * items : items + blocks_of(items, w.k), rest = wgs % places;
    const double rounds = wgs / places + (rest ? kTail[d128 ? 0 : 1][blocks_of(rest, c.n_cus) - 1] : 0.);
    // a helper spends about two tiles more on each item after its first
    const double part = w.ways == 1 ? tiles : w.ways == 3 ? tiles / 3 : (w.k * tiles + 2 * (w.k - 1)) / (w.k + 1);
    return per_tile * rounds * part + (w.ways == 1 ? 0. : launch + per_item * items * (w.ways == 3 ? 1.5 : 1.));
  };
  DqWays best;
  double least = 0.98 * cost(best);  // (a split that gains less is not worth its partial sums)
  auto consider = [&](const DqWays& w) {
    if (cost(w) < least) {
      least = cost(w);
      best = w;
    }
  };
  consider({3, 1});
  consider({2, 1});
  if (c.xcd_load < 1.15) {
    int fits = 1;  // fewest items per helper with which all fit the places at once
    while (fits < 16 && items + blocks_of(items, fits) > places) ++fits;
    for (const int k : {2, 4, 8, fits})
      if (items + blocks_of(items, k) <= places) consider({2, k});
  }
  return best;
}

}  // namespace astro
