// The host-only half of the C ABI (see include/jenga.h): configuration checks, plan tables without a
// device, table export, status strings.  No HIP in this file, so that it can be built and run under
// the host sanitizers together with jenga_plan.cpp.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include "jenga_internal.h"

namespace jenga {

bool config_ok(const jenga_config& c, int* why) {
  *why = JENGA_EINVAL;
  if (c.T < 1 || c.H < 1 || c.W < 1 || c.n_text < 0 || c.batch < 1 || c.heads < 1) return false;
  if (!(c.topk_ratio > 0.0 && c.topk_ratio <= 1.0)) return false;
  if (!(c.cum_prob >= 0.0 && c.cum_prob < 1.0)) return false;
  if (!std::isfinite(c.text_bias)) return false;   // NaN and +-inf: exp2(-inf + inf) would poison a row
  if (c.flags & ~15u) return false;
  *why = JENGA_EUNSUPPORTED;
  if (c.head_dim != 64 && c.head_dim != 128) return false;
  if (c.block != 32 && c.block != 64 && c.block != 128) return false;
  // at most 2^24 vision tokens; multiply step by step so that no product can overflow
  const long long lim = 1ll << 24;
  if (c.T > lim || c.H > lim || c.W > lim || (long long)c.T * c.H > lim) return false;
  const long long nv = (long long)c.T * c.H * c.W;
  if (nv > lim || c.n_text > (1 << 20)) return false;
  const long long M = (nv + c.block - 1) / c.block + (c.n_text + c.block - 1) / c.block;
  if (M > 2048) return false;   // select keeps a row of M block probabilities in one wavefront
  if ((long long)c.batch * c.heads > 65535) return false;
  return true;
}

// The largest group of output rows whose input rows fit the LDS tile.
StageTiles stage_switch_tiles(long long channels, int T_in, int H_in, int W_in, int T_out, int H_out, int W_out, bool on_16) {
  constexpr long long TILE_FLOATS = 12288;   // 48 KB of LDS for the staged clean-latent estimate
  auto window_len_max = [](long long n_in, long long n_out) { return (n_in + n_out - 1) / n_out + 1; };
  const unsigned quads_per_row = ((unsigned)W_out + 3u) / 4u;
  const long long nt_max = window_len_max(T_in, T_out);
  StageTiles s;
  s.rows_per_wg = quads_per_row >= 256u ? 1u : 256u / quads_per_row;
  if (s.rows_per_wg > (unsigned)H_out) s.rows_per_wg = (unsigned)H_out;
  auto tile_floats = [&](unsigned rows) {
    // input rows touched by `rows` consecutive output rows: at most floor((rows-1)*H_in/H_out) + window + 1
    const long long nh = ((long long)(rows - 1) * H_in) / H_out + window_len_max(H_in, H_out) + 1;
    const long long plane = (nh < H_in ? nh : H_in) * W_in;
    // rows off the 16-byte grid are read from the boundary below them
    return nt_max * (W_in % 4 == 0 ? plane : (plane + 6) & ~3ll);
  };
  while (s.rows_per_wg > 1 && tile_floats(s.rows_per_wg) > TILE_FLOATS) --s.rows_per_wg;
  s.floats = tile_floats(s.rows_per_wg);
  // Rows off the 16-byte grid: with the chip full a workgroup costs 1 to 1.8 ns however little it has to read and write,
  // and small planes are done sooner directly, above all where every window is a single cell.  Direct -> tiled, by the
  // larger of a quarter of the cells it reads and of those it writes:
  //   windows of one cell: 26214 x 8 x 2 x 5 -> 2 x 5 (2)     13 -> 214 us      1134 x 8 x 11 x 21 -> 11 x 21 (57)  10.7 -> 16.0 us
  //                        748 x 8 x 14 x 25 -> 14 x 25 (87)  10.8 -> 12.2 us   497 x 8 x 17 x 31 -> 17 x 31 (131)  10.4 -> 10.8 us
  //   others:              2880 x 8 x 7 x 13 -> 10 x 18 (45)  24.4 -> 27.6 us   8 x 33 x 3 -> 66 x 5 (82)            7 % slower
  //                        1134 x 8 x 11 x 21 -> 15 x 29 (109)  26 -> 16 us     227 x 8 x 18 x 33 -> 25 x 46 (252)  18.2 -> 9.8 us
  //                        16 x 33 x 45 x 79 -> 67 x 117 (614)  30 -> 13.6 us
  // No shape tried (W 1 to 1001, up, down and equal) was slower tiled from 192 and 96 on.
  const long long rows_in = std::min<long long>(H_in, ((long long)s.rows_per_wg * H_in + H_out - 1) / H_out);
  const long long read = std::max(1, T_in / T_out) * rows_in * W_in / 4, written = (long long)s.rows_per_wg * W_out / 4;
  const bool one_cell = T_out % T_in == 0 && H_out % H_in == 0 && W_out % W_in == 0;
  const bool worth_it = W_in % 4 == 0 || std::max(read, written) >= (one_cell ? 192 : 96);
  // a workgroup of 256 threads for every (channel, t) plane: below 2^32 threads in x, which a grid has to stay under
  s.tiled = on_16 && worth_it && s.floats <= TILE_FLOATS && channels * T_out < 1ll << 24;
  return s;
}

}  // namespace jenga

extern "C" {

int jenga_plan_info(const jenga_plan* p, jenga_plan_info_t* info) {
  if (!p || !info) return JENGA_EINVAL;
  *info = p->info;
  return JENGA_OK;
}

int jenga_plan_export(const jenga_plan* p, int32_t* perm, int32_t* inv_perm, uint8_t* adja) {
  if (!p) return JENGA_EINVAL;
  const size_t nv = (size_t)p->info.N_v;
  if (perm) std::memcpy(perm, p->perm.data(), nv * sizeof(int32_t));
  if (inv_perm) std::memcpy(inv_perm, p->inv_perm.data(), nv * sizeof(int32_t));
  if (adja) {
    const int mv = p->info.M_v;
    const bool on = (p->cfg.flags & JENGA_FLAG_ADJACENCY) != 0;
    for (int i = 0; i < mv; ++i)
      for (int j = 0; j < mv; ++j)
        adja[(size_t)i * mv + j] =
            on ? (uint8_t)((p->fixed_bits[(size_t)i * p->nt64 + (j >> 6)] >> (j & 63)) & 1ull) : 0;
  }
  return JENGA_OK;
}

int jenga_plan_tables(const jenga_config* cfg, jenga_plan_info_t* info, int32_t* perm, int32_t* inv_perm,
                      uint8_t* adja) {
  if (!cfg || !info) return JENGA_EINVAL;
  int why;
  if (!jenga::config_ok(*cfg, &why)) return why;
  jenga_plan* p = new (std::nothrow) jenga_plan();
  if (!p) return JENGA_ENOMEM;
  p->cfg = *cfg;
  p->d_src_of_pos = nullptr;
  p->d_blk_valid = nullptr;
  p->d_fixed_bits = nullptr;
  int rc = JENGA_OK;
  try {
    rc = jenga::build_host_tables(p);
  } catch (const std::bad_alloc&) {
    rc = JENGA_ENOMEM;
  }
  if (rc == JENGA_OK) {
    *info = p->info;
    rc = jenga_plan_export(p, perm, inv_perm, adja);
  }
  delete p;
  return rc;
}

const char* jenga_strerror(int status) {
  switch (status) {
    case JENGA_OK: return "ok";
    case JENGA_EINVAL: return "invalid argument";
    case JENGA_EUNSUPPORTED: return "configuration not supported by this build";
    case JENGA_EWORKSPACE: return "workspace too small";
    case JENGA_EHIP: return "HIP runtime or kernel launch failure";
    case JENGA_ENOMEM: return "out of memory";
    default: return "unknown status";
  }
}

}  // extern "C"
