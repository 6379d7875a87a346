// Reads calls, one per line (D pairs Nq block_rows in_order streams and the resident rows of each stream; 256
// CUs), and prints what the launch rules of paper_2603_17051_amd/csrc/launch_rules.hpp answer: few-rows
// waves and key ranges of the forward, few-rows waves, ways and k of the backward, contiguous eighths or not,
// the most (cos, sin) of a forward that rotates for itself (0 = it does not) and of one whose waves turn the keys together, whether a backward of few rows has its row
// terms computed first, which kernel dK and dV take over the chunk's keys and over the ring's, whether those go out in one launch.
#include <cstdio>

#include "../../paper_2603_17051_amd/csrc/launch_rules.hpp"

int main() {
  int D, pairs, Nq, block_rows, in_order, streams;
  while (std::scanf("%d %d %d %d %d %d", &D, &pairs, &Nq, &block_rows, &in_order, &streams) == 6) {
    int32_t hist[64];
    for (int b = 0; b < streams; ++b)
      if (b >= 64 || std::scanf("%d", &hist[b]) != 1) return 1;
    const astro::CallShape c = astro::make_call_shape(D, 256, pairs, Nq, block_rows, in_order != 0, hist, streams);
    const astro::DqWays w = astro::dq_ways(c);
    int entries = 1024;
    while (entries > 0 && !astro::fwd_rotates(c, entries)) --entries;
    int together = entries;
    while (together > 0 && !astro::fwd_turns_together(c, together)) --together;
    std::printf("%d %d %d %d %d %d %d %d %d %d %d %d\n", astro::fwd_few_waves(c), astro::fwd_splits(c), astro::bwd_few_waves(c), w.ways, w.k,
                astro::order_by_xcd(c, astro::blocks_of(Nq, 128) * pairs), entries, together, astro::bwd_terms_first(c),
                astro::dkv_halves(c, astro::chunk_blocks(c)), astro::dkv_halves(c, c.ring_blocks), astro::bwd_joins(c));
  }
  return 0;
}
