// Test driver for the host rules that shape launches (CPU only).  Reads configurations from stdin, one per line:
//     T H W n_text batch heads head_dim block topk_ratio cum_prob threads
// and prints for each: batch * heads, the pairs heads_per_launch() gives a launch with `threads` threads per query block,
// and the workgroups of a launch of all pairs and of one of that many.  With the argument "switch" the lines are
//     channels T_in H_in W_in T_out H_out W_out aligned
// and the output is what stage_switch_tiles() says: tiled, output rows per workgroup, floats of LDS.  With the argument
// "work" the lines are configurations without the last column, and the output is how often the query block that is dealt
// out least and most often is, the share, and how many text blocks are on an XCD without a vision block of their head.
// With the argument "deal" the lines are the same configurations; a launch's positions are gone through as the kernel does and
// the output is: parts of a text list, lists cut at the end, the parts dealt out least and most often, slots used and slots there are.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <set>
#include <utility>
#include <vector>

#include "jenga_internal.h"

static int stage_switch() {
  int c, i[3], o[3], aligned;
  while (std::scanf("%d %d %d %d %d %d %d %d", &c, i, i + 1, i + 2, o, o + 1, o + 2, &aligned) == 8) {
    const jenga::StageTiles s = jenga::stage_switch_tiles(c, i[0], i[1], i[2], o[0], o[1], o[2], aligned != 0);
    std::printf("%d %u %lld\n", (int)s.tiled, s.rows_per_wg, s.floats);
  }
  return 0;
}

static int work() {
  jenga_plan p = {};
  jenga_config& c = p.cfg;
  while (std::scanf("%d %d %d %d %d %d %d %d %lf %lf", &c.T, &c.H, &c.W, &c.n_text, &c.batch, &c.heads, &c.head_dim,
                    &c.block, &c.topk_ratio, &c.cum_prob) == 10) {
    if (jenga::build_host_tables(&p) != JENGA_OK) return 1;
    const jenga::WorkMap w = jenga::plan_work(&p, c.batch * c.heads);
    std::vector<int> times((size_t)w.n_bh * w.M, 0);
    std::set<std::pair<int, int>> vision;
    int bh, i, apart = 0;
    for (int n = w.n_wg - 1; n >= 0; --n) {   // vision blocks first
      if (!jenga::map_work(n, w, &bh, &i)) continue;
      ++times[(size_t)bh * w.M + i];
      if (i < w.M_v) vision.insert({n & 7, bh});
      else if (!vision.count({n & 7, bh})) ++apart;
    }
    std::printf("%d %d %d %d\n", *std::min_element(times.begin(), times.end()),
                *std::max_element(times.begin(), times.end()), w.share, apart);
  }
  return 0;
}

static int deal() {
  jenga_plan p = {};
  jenga_config& c = p.cfg;
  while (std::scanf("%d %d %d %d %d %d %d %d %lf %lf", &c.T, &c.H, &c.W, &c.n_text, &c.batch, &c.heads, &c.head_dim,
                    &c.block, &c.topk_ratio, &c.cum_prob) == 10) {
    if (jenga::build_host_tables(&p) != JENGA_OK) return 1;
    const jenga::WorkMap w = jenga::plan_work(&p, c.batch * c.heads);
    const jenga::Deal d = jenga::plan_deal(&p, w, false);
    std::vector<int> done((size_t)w.n_bh * w.M, 0), parts_of((size_t)w.n_bh * w.M, 0);
    std::set<int> slots, rows;
    int n, part, parts, slot, bh, i, least = 1 << 30, most = 0;
    for (int r = 0; r < d.positions(); ++r)
      for (int x = 0; x < 8; ++x) {
        if (!jenga::deal_position(r, x, d, w, &n, &part, &parts, &slot) || !jenga::map_work(n, w, &bh, &i)) continue;
        const size_t row = (size_t)bh * w.M + i;
        if (part < 0 || part >= parts || (slot >= 0) != (parts > 1)) return 2;
        done[row] += 1;
        parts_of[row] = parts;
        if (slot >= 0 && (slot >= d.slots() || !slots.insert(slot).second)) return 3;
        // where merge_kernel finds the row: text rows first, then the others
        if (slot >= 0) {
          const int text = d.text_rows(), y = i >= w.M_v ? n : text + n - w.text_wgs - 8 * d.whole;
          const int first = y < text ? y * d.text_parts : text * d.text_parts + (y - text) * d.parts;
          if (y < 0 || y >= text + d.tail_rows() || first + part != slot) return 4;
        }
      }
    for (size_t row = 0; row < done.size(); ++row) {
      least = std::min(least, done[row] - parts_of[row]);
      most = std::max(most, done[row] - parts_of[row]);
      if (done[row] == 0) return 5;
    }
    std::printf("%d %d %d %d %d %d\n", d.text_parts, d.parts > 1 ? d.tail : 0, least, most, (int)slots.size(), d.slots());
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && std::strcmp(argv[1], "deal") == 0) return deal();
  if (argc > 1 && std::strcmp(argv[1], "work") == 0) return work();
  if (argc > 1 && std::strcmp(argv[1], "switch") == 0) return stage_switch();
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
