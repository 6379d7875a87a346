// Reads calls, one per line (D pairs Nq block_rows min_hist max_hist in_order, on 256 CUs), and prints what the
// launch rules of paper_2603_17051_amd/csrc/launch_rules.hpp answer: few-rows waves and key ranges of the
// forward, few-rows waves, ways and k of the backward.
#include <cstdio>

#include "../../paper_2603_17051_amd/csrc/launch_rules.hpp"

int main() {
  astro::CallShape c{};
  int in_order;
  while (std::scanf("%d %d %d %d %d %d %d", &c.D, &c.pairs, &c.Nq, &c.block_rows, &c.min_hist, &c.max_hist, &in_order) == 7) {
    c.n_cus = 256;
    c.in_order = in_order != 0;
    const astro::DqWays w = astro::dq_ways(c);
    std::printf("%d %d %d %d %d\n", astro::fwd_few_waves(c), astro::fwd_splits(c), astro::bwd_few_waves(c), w.ways, w.k);
  }
  return 0;
}
