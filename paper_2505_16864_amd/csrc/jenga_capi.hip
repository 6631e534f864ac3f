// The device half of the C ABI (see include/jenga.h): plan life cycle on the device, argument validation of
// the hot calls, dispatch to the launchers.  The host-only entry points live in jenga_host.cpp.
#include <hip/hip_runtime.h>

#include <cstring>
#include <new>

#include "jenga_internal.h"

namespace {

// The plan's tables live on the device that was current at creation; a hot call made with another
// device current would launch there with pointers that device cannot read.
bool on_plan_device(const jenga_plan* p) {
  int dev = -1;
  return hipGetDevice(&dev) == hipSuccess && dev == p->device;
}

bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

// The work of jenga_block_sparse_attn; out_thw: the rows in the thw-side order too, or NULL.
int attention(const jenga_plan* p, const void* q, const void* k, const void* v, const int32_t* sel_count,
              const int32_t* sel_index, void* out_curve, float* lse_or_null, void* workspace, void* out_thw, void* stream) {
  // Where K and V are read in place, one that an output lies over, or that is off the 16-byte grid, which the copies into LDS
  // want (ordinary loads take any address), is copied first; if both are, they are packed.
  const size_t rows = (size_t)p->cfg.batch * p->cfg.heads * p->info.N_pad, bytes = rows * p->cfg.head_dim * 2;
  auto moved = [&](const void* x) {
    return ((uintptr_t)x & 15u) != 0 || overlap(x, bytes, out_curve, bytes) ||
           (lse_or_null && overlap(x, bytes, lse_or_null, rows * 4));
  };
  const bool k_moved = moved(k), v_moved = moved(v);
  int rc = JENGA_OK;
  if (!jenga::reads_kv_in_place(p) || (k_moved && v_moved)) {
    rc = jenga::launch_pack(p, k, v, workspace, stream);
    k = v = nullptr;
  } else if (k_moved) {
    rc = jenga::launch_keep(p, k, workspace, 0, &k, stream);
  } else if (v_moved) {
    rc = jenga::launch_keep(p, v, workspace, 1, &v, stream);
  }
  if (rc != JENGA_OK) return rc;
  return jenga::launch_attention(p, q, k, v, workspace, true, sel_count, sel_index, out_curve, lse_or_null, out_thw, stream);
}

template <typename T>
int to_device(const std::vector<T>& h, T** d) {
  *d = nullptr;
  const size_t bytes = (h.size() ? h.size() : 1) * sizeof(T);
  if (hipMalloc((void**)d, bytes) != hipSuccess) return JENGA_ENOMEM;
  if (!h.empty() && hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess)
    return JENGA_EHIP;
  return JENGA_OK;
}

}  // namespace

extern "C" {

int jenga_plan_create(const jenga_config* cfg, jenga_plan** out) {
  if (!cfg || !out) return JENGA_EINVAL;
  *out = nullptr;
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
  if (rc == JENGA_OK && hipGetDevice(&p->device) != hipSuccess) rc = JENGA_EHIP;
  if (rc == JENGA_OK) rc = jenga::select_scratch_init(p->device);
  if (rc == JENGA_OK) rc = to_device(p->src_of_pos, &p->d_src_of_pos);
  if (rc == JENGA_OK) rc = to_device(p->blk_valid, &p->d_blk_valid);
  if (rc == JENGA_OK) rc = to_device(p->fixed_bits, &p->d_fixed_bits);
  if (rc != JENGA_OK) {
    jenga_plan_destroy(p);
    return rc;
  }
  *out = p;
  return JENGA_OK;
}

int jenga_plan_destroy(jenga_plan* p) {
  if (!p) return JENGA_OK;
  int rc = JENGA_OK;
  if (p->d_src_of_pos && hipFree(p->d_src_of_pos) != hipSuccess) rc = JENGA_EHIP;
  if (p->d_blk_valid && hipFree(p->d_blk_valid) != hipSuccess) rc = JENGA_EHIP;
  if (p->d_fixed_bits && hipFree(p->d_fixed_bits) != hipSuccess) rc = JENGA_EHIP;
  delete p;
  return rc;
}

int jenga_curve_permute(const jenga_plan* p, const void* src_thw, void* dst_curve, void* stream) {
  if (!p || !src_thw || !dst_curve) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  return jenga::launch_permute(p, &src_thw, &dst_curve, 1, true, stream);
}

int jenga_curve_permute_qkv(const jenga_plan* p, const void* q_thw, const void* k_thw, const void* v_thw, void* q_curve,
                            void* k_curve, void* v_curve, void* stream) {
  if (!p || !q_thw || !k_thw || !v_thw || !q_curve || !k_curve || !v_curve) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  const void* src[3] = {q_thw, k_thw, v_thw};
  void* dst[3] = {q_curve, k_curve, v_curve};
  // One launch moves the three at the same time.  A result that lies over another tensor (K's over Q, which has moved
  // by then) needs them one after the other.
  const size_t rows = (size_t)p->cfg.batch * p->cfg.heads, row = (size_t)p->cfg.head_dim * 2;
  const size_t src_bytes = rows * (p->info.N_v + p->cfg.n_text) * row, dst_bytes = rows * p->info.N_pad * row;
  bool one_launch = true;
  for (int t = 0; t < 3; ++t)
    for (int u = 0; u < 3; ++u)
      if (t != u && (overlap(dst[t], dst_bytes, src[u], src_bytes) || overlap(dst[t], dst_bytes, dst[u], dst_bytes)))
        one_launch = false;
  if (one_launch) return jenga::launch_permute(p, src, dst, 3, true, stream);
  for (int t = 0; t < 3; ++t) {
    const int rc = jenga::launch_permute(p, src + t, dst + t, 1, true, stream);
    if (rc != JENGA_OK) return rc;
  }
  return JENGA_OK;
}

int jenga_curve_permute_rows(const jenga_plan* p, const void* src_rows, void* dst_rows, int32_t row_bytes,
                             void* stream) {
  if (!p || !src_rows || !dst_rows) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  if (row_bytes < 16 || row_bytes > 4096 || (row_bytes & (row_bytes - 1)) != 0) return JENGA_EUNSUPPORTED;
  return jenga::launch_permute_rows(p, src_rows, dst_rows, row_bytes, stream);
}

int jenga_unpermute(const jenga_plan* p, const void* src_curve, void* dst_thw, void* stream) {
  if (!p || !src_curve || !dst_thw) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  return jenga::launch_permute(p, &src_curve, &dst_thw, 1, false, stream);
}

int jenga_select_blocks(const jenga_plan* p, const void* q_curve, const void* k_curve, int32_t* sel_count,
                        int32_t* sel_index, uint8_t* mask_or_null, void* workspace, size_t workspace_bytes,
                        void* stream) {
  if (!p || !q_curve || !k_curve || !sel_count || !sel_index || !workspace) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  if (((uintptr_t)workspace & 255u) != 0) return JENGA_EINVAL;
  if (workspace_bytes < p->info.select_workspace_bytes) return JENGA_EWORKSPACE;
  return jenga::launch_select(p, q_curve, k_curve, sel_count, sel_index, mask_or_null, workspace, false, stream);
}

int jenga_block_sparse_attn(const jenga_plan* p, const void* q, const void* k, const void* v,
                            const int32_t* sel_count, const int32_t* sel_index, void* out_curve,
                            float* lse_or_null, void* workspace, size_t workspace_bytes, void* stream) {
  if (!p || !q || !k || !v || !sel_count || !sel_index || !out_curve || !workspace) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  if (((uintptr_t)workspace & 255u) != 0) return JENGA_EINVAL;
  if (workspace_bytes < p->info.attn_workspace_bytes) return JENGA_EWORKSPACE;
  return attention(p, q, k, v, sel_count, sel_index, out_curve, lse_or_null, workspace, nullptr, stream);
}

int jenga_forward(const jenga_plan* p, const void* q_thw, const void* k_thw, const void* v_thw, void* q_curve,
                  void* k_curve, void* v_curve, int32_t* sel_count, int32_t* sel_index, uint8_t* mask_or_null,
                  void* select_workspace, size_t select_workspace_bytes, void* out_curve, float* lse_or_null,
                  void* attn_workspace, size_t attn_workspace_bytes, void* out_thw, void* stream) {
  if (!p || !q_thw || !k_thw || !v_thw || !q_curve || !k_curve || !v_curve || !sel_count || !sel_index ||
      !select_workspace || !out_curve || !attn_workspace || !out_thw)
    return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  if ((((uintptr_t)select_workspace | (uintptr_t)attn_workspace) & 255u) != 0) return JENGA_EINVAL;
  if (select_workspace_bytes < p->info.select_workspace_bytes || attn_workspace_bytes < p->info.attn_workspace_bytes)
    return JENGA_EWORKSPACE;
  const size_t bh = (size_t)p->cfg.batch * p->cfg.heads, row = (size_t)p->cfg.head_dim * 2, M = (size_t)p->info.M;
  const size_t thw_bytes = bh * (p->info.N_v + p->cfg.n_text) * row, curve_bytes = bh * p->info.N_pad * row;
  // The fused launches write what the calls for the single steps would write a launch later: a tensor that lies over one that is
  // still being read there goes through those calls.
  const void* src[3] = {q_thw, k_thw, v_thw};
  void* dst[3] = {q_curve, k_curve, v_curve};
  bool fused_in = 3ll * p->cfg.batch <= 65535, fused_out = true;
  for (int t = 0; t < 3; ++t) {
    for (int u = 0; u < 3; ++u)
      if (overlap(dst[t], curve_bytes, src[u], thw_bytes) || (t != u && overlap(dst[t], curve_bytes, dst[u], curve_bytes)))
        fused_in = false;
    if (overlap(select_workspace, p->info.select_workspace_bytes, src[t], thw_bytes) ||
        overlap(select_workspace, p->info.select_workspace_bytes, dst[t], curve_bytes))
      fused_in = false;
    if (overlap(out_thw, thw_bytes, dst[t], curve_bytes)) fused_out = false;
  }
  if (overlap(out_thw, thw_bytes, out_curve, curve_bytes) ||
      overlap(out_thw, thw_bytes, attn_workspace, p->info.attn_workspace_bytes) ||
      overlap(out_thw, thw_bytes, sel_count, bh * M * 4) || overlap(out_thw, thw_bytes, sel_index, bh * M * M * 4) ||
      (lse_or_null && overlap(out_thw, thw_bytes, lse_or_null, bh * p->info.N_pad * 4)))
    fused_out = false;
  int rc = fused_in ? jenga::launch_permute_pool(p, src, dst, select_workspace, stream)
                    : jenga_curve_permute_qkv(p, q_thw, k_thw, v_thw, q_curve, k_curve, v_curve, stream);
  if (rc == JENGA_OK)
    rc = jenga::launch_select(p, q_curve, k_curve, sel_count, sel_index, mask_or_null, select_workspace, fused_in, stream);
  if (rc == JENGA_OK)
    rc = attention(p, q_curve, k_curve, v_curve, sel_count, sel_index, out_curve, lse_or_null, attn_workspace,
                   fused_out ? out_thw : nullptr, stream);
  if (rc == JENGA_OK && !fused_out) rc = jenga_unpermute(p, out_curve, out_thw, stream);
  return rc;
}

int jenga_pack_kv(const jenga_plan* p, const void* k, const void* v, void* workspace, size_t workspace_bytes,
                  void* stream) {
  if (!p || !k || !v || !workspace) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  if (((uintptr_t)workspace & 255u) != 0) return JENGA_EINVAL;
  if (workspace_bytes < p->packed_bytes) return JENGA_EWORKSPACE;
  return jenga::launch_pack(p, k, v, workspace, stream);
}

int jenga_block_sparse_attn_packed(const jenga_plan* p, const void* q, void* packed_kv_workspace,
                                   size_t workspace_bytes, const int32_t* sel_count, const int32_t* sel_index,
                                   void* out_curve, float* lse_or_null, void* stream) {
  if (!p || !q || !packed_kv_workspace || !sel_count || !sel_index || !out_curve) return JENGA_EINVAL;
  if (!on_plan_device(p)) return JENGA_EINVAL;
  if (((uintptr_t)packed_kv_workspace & 255u) != 0) return JENGA_EINVAL;
  if (workspace_bytes < p->packed_bytes) return JENGA_EWORKSPACE;
  return jenga::launch_attention(p, q, nullptr, nullptr, packed_kv_workspace, false, sel_count, sel_index, out_curve,
                                 lse_or_null, nullptr, stream);
}

}  // extern "C"
