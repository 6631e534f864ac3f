// Test driver for the host rules that shape launches (CPU only).  Reads configurations from stdin, one per line:
//     T H W n_text batch heads head_dim block topk_ratio cum_prob threads
// and prints for each: batch * heads, the pairs heads_per_launch() gives a launch with `threads` threads per query block,
// and the workgroups of a launch of all pairs and of one of that many.
#include <cstdio>

#include "jenga_internal.h"

int main() {
  jenga_plan p = {};
  jenga_config& c = p.cfg;
  int threads;
  while (std::scanf("%d %d %d %d %d %d %d %d %lf %lf %d", &c.T, &c.H, &c.W, &c.n_text, &c.batch, &c.heads, &c.head_dim,
                    &c.block, &c.topk_ratio, &c.cum_prob, &threads) == 11) {
    int why = 0;
    if (!jenga::config_ok(c, &why) || jenga::build_host_tables(&p) != JENGA_OK) {
      std::printf("refused\n");
      continue;
    }
    const int all = c.batch * c.heads, some = jenga::heads_per_launch(&p, threads);
    std::printf("%d %d %d %d\n", all, some, jenga::plan_work(&p, all).n_wg, jenga::plan_work(&p, some).n_wg);
  }
  return 0;
}
