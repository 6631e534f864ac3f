// Internal declarations shared by the host plan code and the HIP translation units.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>
#include "jenga.h"

#ifdef __HIPCC__
#define JENGA_HOST_DEVICE __host__ __device__
#else   // the host-only sources and their tests
#define JENGA_HOST_DEVICE
#endif

struct jenga_plan {
  jenga_config cfg;
  jenga_plan_info_t info;
  int device;
  int nt64;  // 64-bit words per row of the fixed-mask table: ceil(M / 64)
  // attention: a list longer than attn_chunk entries is cut into up to attn_parts parts (1: lists stay whole);
  // attn_chunk = 0: every list into attn_parts ranges of key blocks
  int attn_parts, attn_chunk;
  int attn_heads;  // (batch, head) pairs per launch where lists are cut
  float attn_long; // > 0: attn_tail lists are cut if the call's vision lists have that many blocks on average
  int attn_first;  // > 0: then the positions of an XCD behind that many are dealt out by counters too
  int attn_text_parts;  // parts that the lists of text query blocks are cut into
  int attn_len;    // expected blocks of a vision list: K_top and the fixed ones
  int attn_tail;   // lists that are cut, all into attn_parts, at the end of each XCD's
  bool attn_over_kv; // their results lie where packed K would, or packed V: not needed when K and V are read in place
  // bytes of the attention workspace that hold packed K, packed V and launch parameters; parts lie behind them
  uint64_t packed_bytes;
  // host tables
  std::vector<int32_t> perm, inv_perm;
  std::vector<int32_t> src_of_pos;  // [N_pad] index into the thw-side sequence, -1 for a pad
  std::vector<int32_t> blk_valid;   // [M] valid tokens per block
  std::vector<uint64_t> fixed_bits; // [M_v][nt64] adjacency and condition bits per query block
  // device copies
  int32_t* d_src_of_pos;
  int32_t* d_blk_valid;
  uint64_t* d_fixed_bits;
};

namespace jenga {

// Validates a configuration; on failure *why is the jenga_status to return.
bool config_ok(const jenga_config& c, int* why);

// Curve order of a T x H x W grid: fills cells with the thw index of each curve position.
void curve_order(int T, int H, int W, bool use_curve, std::vector<int32_t>& perm);

// Host tables of a plan (no device work).  Returns a jenga_status.
int build_host_tables(jenga_plan* plan);

// Workgroups of the attention kernel for blocks of 64 and 128 tokens that are resident on a CU, by registers and LDS (which is given
// out in pieces of 1280 bytes); 64 tokens at D = 128: in steps of 32 keys, four in steps of 64.
constexpr int attn_h_per_cu(int block, int head_dim) {
  return block == 64 ? (head_dim == 128 ? 6 : 8) : (head_dim == 128 ? 3 : 4);
}

// Work mapping shared by the attention kernels.  The text query blocks of every (batch, head) are
// dense rows, several times longer than a vision row: they are dealt out first, ahead of all vision
// blocks, so that none of them starts late and runs on alone at the end.  The vision blocks follow.
// Workgroups are dealt round-robin to the 8 XCDs; `share` of them (8, 4, 2 or 1) work on the same head
// at a time and split its query blocks into contiguous runs of `chunk`, whose selections overlap; the
// heads are divided evenly among the 8 / share groups.  plan_work() says how `share` is chosen.
struct WorkMap {
  int n_bh, M, M_v;
  int share, chunk;   // XCDs per head, query blocks of a head per XCD
  int log_share;
  int units;          // n_bh * chunk: query blocks (with fillers) per member of a group, over all groups
  int text_wgs, n_wg; // workgroups of the text blocks, all workgroups
};

// The query block of workgroup n (see WorkMap).  Returns false for the filler workgroups at the end of a run.
JENGA_HOST_DEVICE inline bool map_work(int n, const WorkMap& w, int* bh, int* i) {
  const int M_c = w.M - w.M_v;
  if (n < w.text_wgs) {
    int t = n;
    if (w.share < 8) {   // XCD x: eighth x of the text blocks, as of the units below, so that both are of the same heads
      const int n_text = w.n_bh * M_c, x = n & 7;
      t = (n_text * x >> 3) + (n >> 3);
      if (t >= n_text * (x + 1) >> 3) return false;
    }
    *bh = t / M_c;
    *i = w.M_v + t % M_c;
    return true;
  }
  n -= w.text_wgs;
  const int xcd = n & 7, group = xcd >> w.log_share, member = xcd & (w.share - 1), log_groups = 3 - w.log_share;
  const int first = (int)(((long long)w.units * group) >> log_groups);
  const int end = (int)(((long long)w.units * (group + 1)) >> log_groups);
  const int u = first + (n >> 3);
  if (u >= end) return false;
  *bh = u / w.chunk;
  *i = member * w.chunk + u % w.chunk;
  return *i < w.M_v;
}

// Work of a launch in positions, the same number for each XCD: text query blocks in `text_parts` parts each, `whole` vision
// blocks, `tail` vision blocks in `parts` parts each.
struct Deal {
  int text, text_parts, whole, tail, parts;
  JENGA_HOST_DEVICE int positions() const { return text * text_parts + whole + tail * parts; }
  // the same launch where the counters are not used: workgroups beyond the positions have nothing to do
  JENGA_HOST_DEVICE Deal vision_whole() const { return {text, text_parts, whole + tail, 0, 1}; }
  JENGA_HOST_DEVICE int text_rows() const { return text_parts > 1 ? 8 * text : 0; }   // that are cut
  JENGA_HOST_DEVICE int tail_rows() const { return parts > 1 ? 8 * tail : 0; }
  JENGA_HOST_DEVICE int slots() const { return text_rows() * text_parts + tail_rows() * parts; }
};

// What position r of XCD x is: part `part` of `parts` of workgroup *n of map_work(); its partial result goes to slot *slot, -1 if
// the list is whole.  Returns false where there is nothing to do.
JENGA_HOST_DEVICE inline bool deal_position(int r, int x, const Deal& d, const WorkMap& w, int* n, int* part, int* parts,
                                            int* slot) {
  const int text = d.text * d.text_parts;
  int row0 = 0, slot0 = 0, rows = w.text_wgs;
  *parts = d.text_parts;
  if (r >= text) rows = w.n_wg;
  if (r >= text + d.whole) {
    r -= text + d.whole;
    row0 = w.text_wgs + 8 * d.whole;
    slot0 = d.text_rows() * d.text_parts;
    *parts = d.parts;
  } else if (r >= text) {
    r -= text;
    row0 = w.text_wgs;
    *parts = 1;
  }
  const int row = r / *parts * 8 + x;
  *part = r % *parts;
  *slot = *parts > 1 ? slot0 + row * *parts + *part : -1;
  *n = row0 + row;
  return *n < rows;
}

// Row y of those that are cut, text rows first: workgroup *n of map_work(), whose *parts results start at slot *slot.
// Returns false where there is none.
JENGA_HOST_DEVICE inline bool merge_row(int y, const Deal& d, const WorkMap& w, int* n, int* parts, int* slot) {
  const int text = d.text_rows();
  const bool is_text = y < text;
  *parts = is_text ? d.text_parts : d.parts;
  *slot = is_text ? y * *parts : text * d.text_parts + (y - text) * *parts;
  *n = is_text ? y : w.text_wgs + 8 * d.whole + y - text;
  return *n < (is_text ? w.text_wgs : w.n_wg);
}

// The mapping for `n_bh` (batch, head) pairs of the plan.
WorkMap plan_work(const jenga_plan* p, int n_bh);

// The positions of a launch for all of them; whole: nothing is cut.
Deal plan_deal(const jenga_plan* p, const WorkMap& work, bool whole);

// Whether a call takes steps of 32 keys (blocks of 64 tokens, D = 128); may_cut: the call cuts the lists that the plan says.
bool attn_keys32(const jenga_plan* p, bool may_cut);

// (batch, head) pairs of the plan that one launch with `threads` threads per query block can take.
int heads_per_launch(const jenga_plan* p, int threads);

// How jenga_stage_switch does a shape: tiled (input rows staged in LDS) or directly from global memory.
struct StageTiles {
  bool tiled;
  unsigned rows_per_wg;   // output rows of a workgroup
  long long floats;       // LDS tile
};
// on_16: inputs 16-byte aligned
StageTiles stage_switch_tiles(long long channels, int T_in, int H_in, int W_in, int T_out, int H_out, int W_out, bool on_16);

// Kernel launchers (defined in the .hip files).  All return a jenga_status.
// 1 to 3 tensors of the plan's shape
int launch_permute(const jenga_plan* p, const void* const* src, void* const* dst, int tensors, bool forward,
                   void* stream);
int launch_permute_rows(const jenga_plan* p, const void* src, void* dst, int row_bytes, void* stream);
// pooled: the block means are in the workspace already (launch_permute_pool)
int launch_select(const jenga_plan* p, const void* q, const void* k, int32_t* sel_count,
                  int32_t* sel_index, uint8_t* mask, void* ws, bool pooled, void* stream);
// Q, K and V into curve order, and the block means of Q and K into the selection's workspace.
int launch_permute_pool(const jenga_plan* p, const void* const src[3], void* const dst[3], void* select_ws, void* stream);
// Looks up the address of the static selection scratch on `device` (the current device) once.
int select_scratch_init(int device);
int launch_pack(const jenga_plan* p, const void* k, const void* v, void* ws, void* stream);
// Whether launch_attention can read K and V as they are instead of packed.
bool reads_kv_in_place(const jenga_plan* p);
// K (which = 0) or V as it is into its half of a packed workspace, for a call that reads in place but cannot read this one
// there; returns the copy in *copied.
int launch_keep(const jenga_plan* p, const void* src, void* ws, int which, const void** copied, void* stream);
// k, v: to be read in place (one of them may be a copy in the workspace), or NULL (packed in the workspace).  may_split: the
// call has the workspace to itself and may write behind the packed tiles, or where they would be.  thw: where the rows go on the
// thw side, or NULL.
int launch_attention(const jenga_plan* p, const void* q, const void* k, const void* v, void* packed_ws, bool may_split,
                     const int32_t* sel_count, const int32_t* sel_index, void* out, float* lse, void* thw, void* stream);

}  // namespace jenga
