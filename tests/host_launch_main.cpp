// Test driver for the host rules that shape launches (CPU only).  Reads configurations from stdin, one per line:
//     T H W n_text batch heads head_dim block topk_ratio cum_prob threads
// and prints for each: batch * heads, the pairs heads_per_launch() gives a launch with `threads` threads per query block,
// and the workgroups of a launch of all pairs and of one of that many.  With the argument "switch" the lines are
//     channels T_in H_in W_in T_out H_out W_out aligned
// and the output is what stage_switch_tiles() says: tiled, output rows per workgroup, floats of LDS.  With the argument
// "work" the lines are configurations without the last column, and the output is how often the query block that is dealt
// out least and most often is, the share, and how many text blocks are on an XCD without a vision block of their head.
// With the argument "deal" and optionally the flags of all plans the lines are the same configurations; a launch's positions are
// gone through as the kernel does, then the rows of its merge: every row has to be written once, from slots that hold its parts.
// The output is: parts of a text list, lists cut at the end, the parts dealt out least and most often, slots used and slots there
// are, positions of an XCD that its counter does not deal out, bytes of the workspace beside packed K and V.  With the argument "keys"
// the output is whether attention takes steps of 32 keys in a call that cuts lists and in one that does not.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
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

// Positions of a launch as the kernel goes through them, then the rows of its merge.
static int deal(unsigned flags) {
  jenga_plan p = {};
  jenga_config& c = p.cfg;
  c.flags = flags;
  while (std::scanf("%d %d %d %d %d %d %d %d %lf %lf", &c.T, &c.H, &c.W, &c.n_text, &c.batch, &c.heads, &c.head_dim,
                    &c.block, &c.topk_ratio, &c.cum_prob) == 10) {
    int why = 0;
    if (!jenga::config_ok(c, &why) || jenga::build_host_tables(&p) != JENGA_OK) return 1;
    const jenga::WorkMap w = jenga::plan_work(&p, c.batch * c.heads);
    const jenga::Deal cut = jenga::plan_deal(&p, w, false);
    if (cut.whole < 0 || cut.tail < 0) return 2;
    const size_t all = (size_t)w.n_bh * w.M;
    int least = 1 << 30, most = 0, used = 0;
    for (const jenga::Deal& d : {cut.vision_whole(), cut}) {   // the same workgroups, without and with the counters
      used = 0;
      std::vector<int> done(all, 0), parts_of(all, 0), written(all, 0);
      std::vector<long long> slot_row(d.slots(), -1);   // row whose part is in a slot
      std::vector<int> slot_part(d.slots(), -1);
      int n, part, parts, slot, bh, i;
      for (int r = 0; r < cut.positions() + (cut.positions() + 3) / 4; ++r)
        for (int x = 0; x < 8; ++x) {
          if (!jenga::deal_position(r, x, d, w, &n, &part, &parts, &slot) || !jenga::map_work(n, w, &bh, &i)) continue;
          const size_t row = (size_t)bh * w.M + i;
          if (part < 0 || part >= parts || (slot >= 0) != (parts > 1)) return 3;
          done[row] += 1;
          parts_of[row] = parts;
          if (slot < 0) {
            written[row] += 1;
            continue;
          }
          if (slot >= d.slots() || slot_row[slot] >= 0) return 4;
          slot_row[slot] = (long long)row;
          slot_part[slot] = part;
          ++used;
        }
      for (int y = 0; y < cut.text_rows() + cut.tail_rows(); ++y) {
        if (!jenga::merge_row(y, d, w, &n, &parts, &slot) || !jenga::map_work(n, w, &bh, &i)) continue;
        const size_t row = (size_t)bh * w.M + i;
        written[row] += 1;
        for (int s = 0; s < parts; ++s)
          if (slot + s >= d.slots() || slot_row[slot + s] != (long long)row || slot_part[slot + s] != s) return 5;
      }
      for (size_t row = 0; row < all; ++row) {
        least = std::min(least, done[row] - parts_of[row]);
        most = std::max(most, done[row] - parts_of[row]);
        if (done[row] == 0 || written[row] != 1) return 6;
      }
    }
    std::printf("%d %d %d %d %d %d %d %llu\n", cut.text_parts, cut.parts > 1 ? cut.tail : 0, least, most, used, cut.slots(), p.attn_first,
                (unsigned long long)(p.info.attn_workspace_bytes - p.packed_bytes));
  }
  return 0;
}

static int keys() {
  jenga_plan p = {};
  jenga_config& c = p.cfg;
  c.flags = 7;
  while (std::scanf("%d %d %d %d %d %d %d %d %lf %lf", &c.T, &c.H, &c.W, &c.n_text, &c.batch, &c.heads, &c.head_dim,
                    &c.block, &c.topk_ratio, &c.cum_prob) == 10) {
    int why = 0;
    if (!jenga::config_ok(c, &why) || jenga::build_host_tables(&p) != JENGA_OK) return 1;
    std::printf("%d %d\n", (int)jenga::attn_keys32(&p, true), (int)jenga::attn_keys32(&p, false));
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && std::strcmp(argv[1], "keys") == 0) return keys();
  if (argc > 1 && std::strcmp(argv[1], "deal") == 0) return deal(argc > 2 ? (unsigned)std::atoi(argv[2]) : 0u);
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
