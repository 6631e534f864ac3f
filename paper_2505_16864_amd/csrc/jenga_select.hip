// Block selection (Sec. 3.1 Eq. 3; appendix Alg. 3 and Eq. 5) in two kernels:
//   pool_kernel    BlockPool: per-block mean of Q (vision blocks) and K (all blocks)   HBM-bound
//   select_kernel  S = Q^ K^T / sqrt(d_k) on the float64 matrix cores into LDS, then one wavefront per query block:
//                  softmax, N_k, top-N_k, union, compaction
//
// All arithmetic is float64: the outcome is a set of integers, and in float64 the sums of bf16
// inputs are exact and the remaining rounding (1e-16 relative) is far below the spacing of the
// block probabilities, so the sets do not depend on the order of summation.
//
// A row of R stays in registers (NT values per lane) and is never sorted.  Positive doubles order like their bit
// patterns, so the N-th largest value is found by building its bit pattern from the top bit down, counting with wave
// ballots; the cumulative-probability rule uses the same descent on the sum of the values at or above the candidate.
// A descent starts below the bits that all values share, compares high words as long as the low ones are undecided,
// and goes on with one value per lane as soon as 64 are left in question.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "jenga_internal.h"

// Workspace of jenga_select_blocks_static: one copy per GPU, held from module load to process end.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)JENGA_SELECT_STATIC_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {

__device__ inline double bf16_bits_to_double(uint32_t bits16) {
  return (double)__uint_as_float(bits16 << 16);
}

// Where channel d of block j lies in its pooled row: pieces of 64 bytes, their order rotated by an exclusive or with the
// block index.  select_kernel reads the same piece of 16 consecutive blocks at a time; without the rotation those lie
// a row (1 KB at D = 128) apart and fall on a quarter of the L2's channels (the products of 929 x 931 blocks x 24 heads:
// 175 us without it, 105 us with).
template <int D>
__device__ inline int pooled_pos(int j, int d) {
  return ((((d >> 3) ^ j) & (D / 8 - 1)) << 3) | (d & 7);
}

// grid (M, batch*heads, 2): z = 0 pools Q (vision blocks only), z = 1 pools K (all blocks).
// q, k: curve side [bh][n_pad][D]; qh: [bh][M_v][D]; kh: [bh][M][D].  A thread issues up to four row
// loads before it adds them, so that enough bytes are in flight to stream from HBM.
template <int D>
__global__ __launch_bounds__(256) void pool_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                   double* __restrict__ qh, double* __restrict__ kh,
                                                   const int32_t* __restrict__ blk_valid, int n_pad, int m, int M_v,
                                                   int M) {
  constexpr int CH = D / 8;      // 16-byte chunks per row
  constexpr int G = 256 / CH;    // rows in flight per pass
  __shared__ double red[G][D];
  const int j = blockIdx.x, bh = blockIdx.y;
  const bool is_q = blockIdx.z == 0;
  if (is_q && j >= M_v) return;
  const uint16_t* x = is_q ? q : k;
  double* out = is_q ? qh : kh;
  const int n_blk = is_q ? M_v : M;
  const int c = threadIdx.x % CH, g = threadIdx.x / CH;
  const int nv = blk_valid[j];
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  const uint4* base = (const uint4*)(x + ((size_t)bh * n_pad + (size_t)j * m) * D);
  for (int r0 = g; r0 < nv; r0 += 4 * G) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + u * G;
      v[u] = r < nv ? base[(size_t)r * CH + c] : make_uint4(0, 0, 0, 0);   // +0.0 for the rows past the end
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += bf16_bits_to_double(w[e] & 0xFFFFu);
        acc[2 * e + 1] += bf16_bits_to_double(w[e] >> 16);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[g][c * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    double s = 0.0;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) s += red[gg][threadIdx.x];
    out[((size_t)bh * n_blk + j) * D + pooled_pos<D>(j, threadIdx.x)] = s / (double)nv;
  }
}

// Q, K and V of jenga_forward into curve order, and the means of Q and K from the same rows: the pooling's pass over both, and
// its launch.  A workgroup moves one block of one (batch, head); grid (heads, M, 3 * batch), so that neighbours read neighbouring heads
// of the same tokens.  Sums in pool_kernel's order, so the means are the same bits.
// Whole jenga_forward (this, and rows written to the thw side by the attention kernels), four calls -> one: 9 blocks of 32 x 2 heads,
// D = 64, 22.6 -> 14.3 us (five launches -> three, of which each is 2.5 us however little it does), 17 of 128 x 8, D = 128, 55.6 ->
// 51.4 us (inputs that no cache holds 61.6 -> 57.2), 931 x 24 48.34 -> 48.09 ms: 0.53 ms of pooling and un-permute go, and the
// attention's second store takes half of that back.
struct Moves {
  const uint4* src[3];
  uint4* dst[3];
  double* mean[2];
};
template <int M_TOK, int D>
__global__ __launch_bounds__(256) void permute_pool_kernel(Moves moves, const int32_t* __restrict__ src_of_pos,
                                                           const int32_t* __restrict__ blk_valid, int n_src, int M_v,
                                                           int batch) {
  constexpr int CH = D / 8, G = 256 / CH, ROWS = M_TOK / G;   // pieces of a row, rows at a time, rows of a thread
  __shared__ double red[G][D];
  const int h = blockIdx.x, j = blockIdx.y, heads = gridDim.x, M = gridDim.y;
  const int tensor = blockIdx.z / batch, b = blockIdx.z - tensor * batch;
  const int c = threadIdx.x % CH, g = threadIdx.x / CH;
  const uint4* src = moves.src[tensor] + ((size_t)b * n_src * heads + h) * CH + c;
  uint4* dst = moves.dst[tensor] + (((size_t)b * heads + h) * M + j) * (M_TOK * CH) + threadIdx.x;
  int s[ROWS];
#pragma unroll
  for (int u = 0; u < ROWS; ++u) s[u] = src_of_pos[j * M_TOK + u * G + g];
  uint4 v[ROWS];
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    v[u] = make_uint4(0, 0, 0, 0);
    if (s[u] >= 0) v[u] = src[(size_t)s[u] * heads * CH];
  }
#pragma unroll
  for (int u = 0; u < ROWS; ++u) dst[u * 256] = v[u];
  if (tensor == 2 || (tensor == 0 && j >= M_v)) return;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += bf16_bits_to_double(w[e] & 0xFFFFu);
      acc[2 * e + 1] += bf16_bits_to_double(w[e] >> 16);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[g][c * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    double sum = 0.0;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) sum += red[gg][threadIdx.x];
    const size_t row = ((size_t)b * heads + h) * (tensor == 0 ? M_v : M) + j;
    moves.mean[tensor][row * D + pooled_pos<D>(j, threadIdx.x)] = sum / (double)blk_valid[j];
  }
}

// Wave-wide reductions in the vector ALU (DPP): six dependent steps of a few cycles each, where the same through
// __shfl_xor is twelve LDS round trips.  The result is uniform.
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_move(double old, double x) {
  const uint64_t o = (uint64_t)__double_as_longlong(old), v = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_update_dpp((uint32_t)o, (uint32_t)v, CTRL, ROW_MASK, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp((uint32_t)(o >> 32), (uint32_t)(v >> 32), CTRL, ROW_MASK, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ inline uint64_t readlane64(uint64_t x, int lane) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(x >> 32), lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((uint32_t)x, lane);
}
__device__ inline double lane63(double x) {
  return __longlong_as_double((long long)readlane64((uint64_t)__double_as_longlong(x), 63));
}
// row_shr 1, 2, 4, 8 sum each row of 16 lanes into its last lane; row_bcast 15 and 31 add the rows up
__device__ inline double wave_sum(double v) {
  v += dpp_move<0x111, 0xF>(0.0, v);
  v += dpp_move<0x112, 0xF>(0.0, v);
  v += dpp_move<0x114, 0xF>(0.0, v);
  v += dpp_move<0x118, 0xF>(0.0, v);
  v += dpp_move<0x142, 0xA>(0.0, v);
  v += dpp_move<0x143, 0xC>(0.0, v);
  return lane63(v);
}
__device__ inline double wave_max(double v) {
  v = fmax(v, dpp_move<0x111, 0xF>(v, v));
  v = fmax(v, dpp_move<0x112, 0xF>(v, v));
  v = fmax(v, dpp_move<0x114, 0xF>(v, v));
  v = fmax(v, dpp_move<0x118, 0xF>(v, v));
  v = fmax(v, dpp_move<0x142, 0xA>(v, v));
  v = fmax(v, dpp_move<0x143, 0xC>(v, v));
  return lane63(v);
}
__device__ inline uint32_t wave_min_u32(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x112, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x118, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x142, 0xA, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(v, v, 0x143, 0xC, 0xF, false));
  return __builtin_amdgcn_readlane(v, 63);
}

// Descent over the bit patterns of a row of R (one wavefront, NT values per lane), highest bit first.  The answer lies
// in [lo, end); bits above `b` are decided.  n_lo and n_end count the values at or above lo and end.
struct Interval {
  uint64_t lo, end;
  int b, n_lo, n_end;
};

// Compacts the at most 64 values inside the interval to one per lane, 0 in the lanes left over.
template <int NT>
__device__ __forceinline__ uint64_t values_inside(const double (&r)[NT], const Interval& v, int M, int lane, double* row) {
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  int base = 0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const uint64_t key = (uint64_t)__double_as_longlong(r[t]);
    const bool in = t * 64 + lane < M && key >= v.lo && key < v.end;
    const uint64_t m = __ballot(in);
    if (in) row[base + (int)__popcll(m & lt_mask)] = r[t];
    base += (int)__popcll(m);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the other lanes' values, same wavefront
  const uint64_t key = lane < base ? (uint64_t)__double_as_longlong(row[lane]) : 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return key;
}

// One row of the selection by one wavefront: softmax of the scores r (value t of lane l: block 64 t + l, -inf past M), N_k, the
// top N_k (`row`: LDS for 64 of the values), the union with `fixed_lane` (lane t holds word t of the row's fixed mask),
// compaction.  See the head of this file.
template <int NT>
__device__ __forceinline__ void select_row(double (&r)[NT], double* row, uint64_t fixed_lane, int32_t* idx_out,
                                           uint8_t* mask_out, int* count, int M, int K_top, double p) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  double mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < NT; ++t) mx = fmax(mx, r[t]);
  mx = wave_max(mx);
  double z = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int j = t * 64 + lane;
    r[t] = j < M ? exp(r[t] - mx) : 0.0;
    z += r[t];
  }
  z = wave_sum(z);
  if (z != z) {   // an undefined or infinite score: no order to select by, every block is kept
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int j = t * 64 + lane;
      if (j < M) {
        idx_out[j] = j;
        if (mask_out) mask_out[j] = 1;
      }
    }
    if (lane == 0) *count = M;
    return;
  }
  if constexpr (NT == 1) {
    // One value per lane: its rank and C_n by comparing it with every other, no chain of dependent reductions.
    // (The kernel on 17 blocks x 8 heads: 9.8 -> 9.0 us.  It grows with M: on 48 blocks x 16 heads the two are about
    // equal, and above 64 the descents are taken.)
    const double mine = r[0] = r[0] / z;
    int rank = 0;
    double sum_before = 0.0;
#pragma unroll 4
    for (int j = 0; j < M; ++j) {
      const double rj = __longlong_as_double((long long)readlane64((uint64_t)__double_as_longlong(mine), j));
      const bool before = rj > mine || (rj == mine && j < lane);
      rank += before ? 1 : 0;
      sum_before += before ? rj : 0.0;
    }
    const bool valid = lane < M;
    const int n_star = (int)__popcll(__ballot(valid && sum_before + mine <= p)) + 1;
    const uint64_t fixed = readlane64(fixed_lane, 0);
    const bool sel = valid && (rank < max(n_star, K_top) || ((fixed >> lane) & 1ull));
    const uint64_t sel_mask = __ballot(sel);
    if (sel) idx_out[__popcll(sel_mask & lt_mask)] = lane;
    if (mask_out && valid) mask_out[lane] = sel ? 1 : 0;
    if (lane == 0) *count = (int)__popcll(sel_mask);
    return;
  }
  uint32_t hi_min = 0xFFFFFFFFu;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    r[t] = r[t] / z;   // >= 0: bit order is value order
    if (t * 64 + lane < M) hi_min = min(hi_min, (uint32_t)__double2hiint(r[t]));
  }
  hi_min = wave_min_u32(hi_min);
  // The largest value is exp(0) / z.  The leading bits that it shares with the smallest are those of every value.
  const uint32_t hi_max = __builtin_amdgcn_readfirstlane((uint32_t)__double2hiint(1.0 / z));
  Interval all;
  all.b = 31 + (hi_min == hi_max ? 0 : 32 - __builtin_clz(hi_min ^ hi_max));
  all.lo = ((uint64_t)hi_max << 32) & ~((2ull << all.b) - 1ull);
  all.end = all.lo + (2ull << all.b);
  all.n_lo = M;
  all.n_end = 0;
  auto count_from = [&](uint64_t cand, int b) {   // values at or above cand, whose bits below b are zero
    int n = 0;
    if (b >= 32) {
#pragma unroll
      for (int t = 0; t < NT; ++t) n += (int)__popcll(__ballot((uint32_t)__double2hiint(r[t]) >= (uint32_t)(cand >> 32)));
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) n += (int)__popcll(__ballot((uint64_t)__double_as_longlong(r[t]) >= cand));
    }
    return n;
  };

  // value of the K_top-th largest: the largest pattern with at least K_top values at or above it.  Stops as soon as
  // exactly K_top values lie there: that set is the answer whatever the remaining bits are.
  Interval v = all;
  while (v.b >= 0 && v.n_lo != K_top && v.n_lo - v.n_end > 64) {
    const uint64_t cand = v.lo | (1ull << v.b);
    const int n = count_from(cand, v.b);
    if (n >= K_top) {
      v.lo = cand;
      v.n_lo = n;
    } else {
      v.end = cand;
      v.n_end = n;
    }
    --v.b;
  }
  if (v.b >= 0 && v.n_lo != K_top) {   // at most 64 candidates are left
    const uint64_t mine = values_inside<NT>(r, v, M, lane, row);
    const int above = v.n_end;
    for (; v.b >= 0 && v.n_lo != K_top; --v.b) {
      const uint64_t cand = v.lo | (1ull << v.b);
      const int n = above + (int)__popcll(__ballot(mine >= cand));
      if (n >= K_top) {
        v.lo = cand;
        v.n_lo = n;
      }
    }
  }
  const uint64_t tau_k = v.lo;
  const bool exact = v.n_lo == K_top;   // the K_top values are those at or above tau_k
  int cnt_gt = 0;
  double sum_gt = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bool gt = (uint64_t)__double_as_longlong(r[t]) > tau_k;
    cnt_gt += (int)__popcll(__ballot(gt));
    sum_gt += gt ? r[t] : 0.0;
  }
  sum_gt = wave_sum(sum_gt);
  const double topk_mass = sum_gt + (double)(K_top - cnt_gt) * __longlong_as_double((long long)tau_k);

  uint64_t tau = tau_k;
  int n_keep = K_top;
  if (!(topk_mass > p)) {
    // Cumulative-probability rule: the largest pattern whose upper set still sums to more than p.  It is one of the
    // row's values below the K_top already summed; once the interval holds a single value, that is the answer.
    v = all;
    v.end = exact ? tau_k : tau_k + 1;
    v.n_end = exact ? K_top : cnt_gt;
    double f_end = exact ? topk_mass : sum_gt;   // sum of the values at or above end
    while (v.b >= 0 && v.n_lo - v.n_end > 64) {
      const uint64_t cand = v.lo | (1ull << v.b);
      if (cand < v.end) {
        int n = 0;
        double f = 0.0;
        if (v.b >= 32) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const bool ge = (uint32_t)__double2hiint(r[t]) >= (uint32_t)(cand >> 32);
            n += (int)__popcll(__ballot(ge));
            f += ge ? r[t] : 0.0;
          }
        } else {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const bool ge = (uint64_t)__double_as_longlong(r[t]) >= cand;
            n += (int)__popcll(__ballot(ge));
            f += ge ? r[t] : 0.0;
          }
        }
        f = wave_sum(f);
        if (f > p) {
          v.lo = cand;
          v.n_lo = n;
        } else {
          v.end = cand;
          v.n_end = n;
          f_end = f;
        }
      }
      --v.b;
    }
    if (v.b >= 0 && v.n_lo > v.n_end) {
      const uint64_t mine = values_inside<NT>(r, v, M, lane, row);
      const int above = v.n_end;
      for (; v.b >= 0 && v.n_lo - v.n_end != 1; --v.b) {
        const uint64_t cand = v.lo | (1ull << v.b);
        if (cand >= v.end) continue;
        const bool ge = mine >= cand;
        const int n = above + (int)__popcll(__ballot(ge));
        const double f = f_end + wave_sum(ge ? __longlong_as_double((long long)mine) : 0.0);
        if (f > p) {
          v.lo = cand;
          v.n_lo = n;
        } else {
          v.end = cand;
          v.n_end = n;
        }
      }
      if (v.n_lo - v.n_end == 1) {
        const uint64_t who = __ballot(mine >= v.lo && mine < v.end && mine != 0);
        if (who != 0) v.lo = readlane64(mine, __builtin_ctzll(who));   // 0: the one value left is 0.0, and so is lo
      }
    }
    const uint64_t tau_p = v.lo;
    int g_cnt = 0, e_cnt = 0;
    double g_sum = 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bool valid = t * 64 + lane < M;
      const uint64_t key = (uint64_t)__double_as_longlong(r[t]);
      const bool gt = key > tau_p;
      g_cnt += (int)__popcll(__ballot(gt));
      e_cnt += (int)__popcll(__ballot(valid && key == tau_p));
      g_sum += gt ? r[t] : 0.0;
    }
    g_sum = wave_sum(g_sum);
    const double tv = __longlong_as_double((long long)tau_p);
    int tn = 1;
    while (tn < e_cnt && !(g_sum + (double)tn * tv > p)) ++tn;
    const int n_star = g_cnt + tn;
    if (n_star > K_top) {
      n_keep = n_star;
      tau = tau_p;
      cnt_gt = g_cnt;
    }
  }
  n_keep = min(n_keep, M);
  const int need = n_keep - cnt_gt;   // taken from the values equal to tau, lowest index first

  int taken = 0, out_pos = 0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int j = t * 64 + lane;
    const bool valid = j < M;
    const uint64_t key = (uint64_t)__double_as_longlong(r[t]);
    const bool eq = valid && key == tau;
    const uint64_t eq_mask = __ballot(eq);
    const uint64_t fixed = readlane64(fixed_lane, t);
    bool sel = (valid && key > tau) || (eq && taken + (int)__popcll(eq_mask & lt_mask) < need);
    taken += (int)__popcll(eq_mask);
    sel = (sel || ((fixed >> lane) & 1ull)) && valid;
    const uint64_t sel_mask = __ballot(sel);
    if (sel) idx_out[out_pos + (int)__popcll(sel_mask & lt_mask)] = j;
    out_pos += (int)__popcll(sel_mask);
    if (mask_out && valid) mask_out[j] = sel ? 1 : 0;
  }
  if (lane == 0) *count = out_pos;
}

// Scores and selection of ROWS query blocks of one (batch, head) against all M <= 64 * NT key blocks.  First the
// wavefronts share the columns: S = Q^ K^T / sqrt(D) in 16 x 16 tiles of v_mfma_f64_16x16x4_f64, K^ straight from
// global memory (16 rows x 64 bytes a load, K^ of a head stays in the L2 of the XCD that works on it), Q^ from LDS, which
// every wavefront needs whole: read from memory by each it was as much for the L1 as all of K^.  Results
// to LDS.  Then every wavefront selects for one row.  S never leaves the CU.
//
// A row goes to the registers of its wavefront a range of columns at a time, so that LDS need not hold all of S and two
// workgroups fit a CU: one multiplies while the other selects.  That takes 64 registers, hence half a row of K^ in flight at
// a time, and up to 448 blocks (one range) and from there to 768 (ranges of 256 columns) they are enough.  Up to 1024 the values alone
// are 32 of them: one range, one workgroup a CU.  Above, 16 rows have no room at all; 8 rows in two ranges do, in 128 registers.
// 8 rows for 1024 too: 88 us (16 rows 102) on 800 blocks x 12 heads, D = 64, but 57 (47) on 1000 x 3 and 282 (278) on 931 x 24,
// D = 128, for which K^ is read twice as often.
// The 8-row kernel multiplies four rows of Q^ at a time by the same 16 columns (v_mfma_f64_4x4x4_4b_f64, Q^'s rows in each of
// the four blocks), so that no row is computed twice as in 16 x 16 tiles (2048 x 2: 114 -> 106 us); K^ of the next tile asked
// for ahead of this one's products changed nothing.
// Row stride = 16 mod 32 doubles, so the four rows a tile is written to at a time fall on different banks.
//
// NT is as many values per lane as M needs, up to 512 blocks; rounded up to a power of two, 262 blocks cost a third more for the
// rows.
//
// Time of the kernel, median of ten to twenty launches, now and before (Q^ from memory, unless it says so):
//   17 blocks x 8 heads, D = 128      8.0 us (8.7; a launch alone takes 2.5)
//   48 x 16, D = 64                  11.1 us (11.9)
//   222 x 12, D = 128                20.3 us (24)
//   262 x 24, D = 128                26.1 us (39.6: one workgroup per CU, two rounds of them)
//   600 x 24, D = 128               111 us (135: all of S in LDS, one workgroup a CU); 760 x 12 96 (112), 500 x 24 90 (91)
//   2048 x 2, D = 64                 95 us (115); before, with the products above, one workgroup a CU and two rounds of them: 103
//   1500 x 8, D = 128               295 us (330 likewise)
//   931 x 24, D = 128                220 to 290 us (240 to 270): products 28 k, the last wavefront's 20 k longer, rows 21 k
// Registers that do not fit go to scratch: 1 at 10 values a lane, 11 at 12 (2 at D = 64), 24 at 32, where a wavefront's row alone
// takes 64 of its 128.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Columns of S that are in LDS at a time
template <int NT, int ROWS>
constexpr int select_cols() { return ROWS == 8 ? 32 * NT : NT < 8 || NT == 16 ? 64 * NT : 256; }

template <int D, int NT, int ROWS>
__global__ __launch_bounds__(64 * ROWS, NT == 16 ? 1 : ROWS == 8 ? 4 : 8) void select_kernel(
    const double* __restrict__ qh, const double* __restrict__ kh, const uint64_t* __restrict__ fixed_bits,
    int32_t* __restrict__ sel_count, int32_t* __restrict__ sel_index, uint8_t* __restrict__ mask, int M_v, int M, int n_tiles,
    int n_units, int K_top, double p, int nt64) {
  constexpr int COLS = select_cols<NT, ROWS>(), PASSES = (64 * NT + COLS - 1) / COLS;
  __shared__ double S[ROWS][COLS + 16];
  __shared__ __align__(1024) f64x2 A[ROWS * D / 2];   // the pooled query rows, as they lie in memory
  // workgroup n runs on XCD n % 8: each XCD gets a contiguous run of (head, row tile) units
  const int per_xcd = (n_units + 7) / 8;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || unit >= n_units) return;
  const int bh = unit / n_tiles, i0 = unit % n_tiles * ROWS;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = i0 + wave;
  uint64_t fixed_lane = 0;   // asked for here, needed at the end
  if (i < M_v && lane < nt64) fixed_lane = fixed_bits[(size_t)i * nt64 + lane];

  double r[NT];
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    if (i0 < M_v) {
      // wavefront w brings row w (in the first pass), then takes every ROWS-th tile of columns
      constexpr int CHUNK = D / 16 < 8 ? D / 16 : 8;   // steps whose loads are in flight at a time
      const int g = lane >> 4, c = lane & 15;
      if (pass == 0 && (D == 128 || lane < 32))
        A[wave * (D / 2) + lane] = ((const f64x2*)(qh + ((size_t)bh * M_v + min(i, M_v - 1)) * D))[lane];
      __syncthreads();
      // lane l: row l % 16 of both operands, channels 8 s + 2 (l / 16) and the next in step s; pooled_pos() in bytes is an
      // exclusive or of the row's place with 64 s
      auto place = [&](int row, int j) { return (uint32_t)(row * D * 8 + (j & (D / 8 - 1)) * 64 + g * 16); };
      constexpr bool QUADS = ROWS == 8;   // tiles of 4 x 16: rows l % 4 of Q^, and those four further
      const int ra = QUADS ? c & 3 : c;
      const uint32_t at_a = place(ra, min(i0 + ra, M_v - 1)), at_a4 = place(ra + 4, min(i0 + ra + 4, M_v - 1));
      const char* k_head = (const char*)(kh + (size_t)bh * M * D);
      const double inv = 1.0 / sqrt((double)D);
      for (int j0 = pass * COLS + 16 * wave; j0 < min(M, (pass + 1) * COLS); j0 += 16 * ROWS) {
        const int jb = min(j0 + c, M - 1);
        const uint32_t at_b = place(jb, jb);
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        double quad[2][2] = {{0.0, 0.0}, {0.0, 0.0}};   // [four rows][even and odd channels]
#pragma unroll
        for (int s0 = 0; s0 < D / 8; s0 += CHUNK) {
          f64x2 b[CHUNK];
          uint32_t a0 = at_a, a4 = at_a4;
          asm volatile("" : "+v"(a0), "+v"(a4));   // the places are formed here and not kept over the loop
#pragma unroll
          for (int s = 0; s < CHUNK; ++s) b[s] = *(const f64x2*)(k_head + (at_b ^ (uint32_t)(64 * (s0 + s))));
#pragma unroll
          for (int s = 0; s < CHUNK; ++s) {
            const f64x2 a = *(const f64x2*)((const char*)A + (a0 ^ (uint32_t)(64 * (s0 + s))));
            if constexpr (QUADS) {
              const f64x2 a_up = *(const f64x2*)((const char*)A + (a4 ^ (uint32_t)(64 * (s0 + s))));
              quad[0][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a.x, b[s].x, quad[0][0], 0, 0, 0);
              quad[1][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a_up.x, b[s].x, quad[1][0], 0, 0, 0);
              quad[0][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a.y, b[s].y, quad[0][1], 0, 0, 0);
              quad[1][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a_up.y, b[s].y, quad[1][1], 0, 0, 0);
            } else {
              acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b[s].x, acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b[s].y, acc, 0, 0, 0);
            }
          }
        }
        // register e, or four rows e, of lane l: row 4 e + l / 16, column l % 16; columns past M are never read
#pragma unroll
        for (int e = 0; e < ROWS / 4; ++e)
          S[4 * e + g][j0 - pass * COLS + c] = (QUADS ? quad[e & 1][0] + quad[e & 1][1] : acc[e]) * inv;
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < COLS / 64 && pass * (COLS / 64) + t < NT; ++t) {
      const int j = pass * COLS + t * 64 + lane;
      r[pass * (COLS / 64) + t] = j < M ? S[wave][t * 64 + lane] : -INFINITY;
    }
    if (pass + 1 < PASSES) __syncthreads();
  }

  if (i >= M) return;
  const size_t out_row = (size_t)bh * M + i;
  int32_t* idx_out = sel_index + out_row * M;
  uint8_t* mask_out = mask ? mask + out_row * M : nullptr;
  if (i >= M_v) {   // text query block: sees every block (Alg. 2)
    for (int j = lane; j < M; j += 64) {
      idx_out[j] = j;
      if (mask_out) mask_out[j] = 1;
    }
    if (lane == 0) sel_count[out_row] = M;
    return;
  }
  select_row<NT>(r, S[wave], fixed_lane, idx_out, mask_out, sel_count + out_row, M, K_top, p);
}

// Where the pooled rows of Q and K lie in the workspace.
template <int D>
void pooled_rows(const jenga_plan* p, void* ws, double** qh, double** kh) {
  const size_t q_bytes = (size_t)p->cfg.batch * p->cfg.heads * p->info.M_v * D * 8;
  *qh = (double*)ws;
  *kh = (double*)((char*)ws + ((q_bytes + 255) & ~(size_t)255));
}

template <int D>
int run_select(const jenga_plan* p, const void* q, const void* k, int32_t* sel_count, int32_t* sel_index,
               uint8_t* mask, void* ws, bool pooled, hipStream_t st) {
  const jenga_config& c = p->cfg;
  const jenga_plan_info_t& f = p->info;
  const int bh = c.batch * c.heads;
  double *qh, *kh;
  pooled_rows<D>(p, ws, &qh, &kh);
  if (f.M_v > 0 && !pooled)
    pool_kernel<D><<<dim3(f.M, bh, 2), 256, 0, st>>>((const uint16_t*)q, (const uint16_t*)k, qh, kh, p->d_blk_valid,
                                                    f.N_pad, c.block, f.M_v, f.M);
#define JENGA_SELECT(NTV, ROWS)                                                                                      \
  do {                                                                                                               \
    const int tiles = (f.M + ROWS - 1) / ROWS, units = tiles * bh;                                                   \
    select_kernel<D, NTV, ROWS><<<dim3((units + 7) / 8 * 8), 64 * ROWS, 0, st>>>(                                    \
        qh, kh, p->d_fixed_bits, sel_count, sel_index, mask, f.M_v, f.M, tiles, units, f.K_top, c.cum_prob, p->nt64); \
  } while (0)
  switch (p->nt64) {
    case 1: JENGA_SELECT(1, 16); break;
    case 2: JENGA_SELECT(2, 16); break;
    case 3: JENGA_SELECT(3, 16); break;
    case 4: JENGA_SELECT(4, 16); break;
    case 5: JENGA_SELECT(5, 16); break;
    case 6: JENGA_SELECT(6, 16); break;
    case 7: JENGA_SELECT(7, 16); break;
    case 8: JENGA_SELECT(8, 16); break;
    case 9: case 10: JENGA_SELECT(10, 16); break;
    case 11: case 12: JENGA_SELECT(12, 16); break;
    default:
      if (p->nt64 <= 16) JENGA_SELECT(16, 16);
      else JENGA_SELECT(32, 8);
  }
#undef JENGA_SELECT
  return hipGetLastError() == hipSuccess ? JENGA_OK : JENGA_EHIP;
}

// ---- scratch of the allocation-free entry point ------------------------------------------------
// One array per GPU, resident from module load until the process ends.  The name below is only a
// host-side handle: device code and HIP calls get the address hipGetSymbolAddress returns for the
// device that is current, looked up once per device and kept here.
constexpr int MAX_DEVICES = 64;
void* scratch_of_device[MAX_DEVICES] = {};
std::mutex scratch_lock;

// Address of `scratch` on `device`, which must be the current device; nullptr on failure.
void* scratch_address(int device) {
  if (device < 0 || device >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> guard(scratch_lock);
  if (scratch_of_device[device] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    scratch_of_device[device] = ptr;
  }
  return scratch_of_device[device];
}

}  // namespace

namespace jenga {

int select_scratch_init(int device) { return scratch_address(device) != nullptr ? JENGA_OK : JENGA_EHIP; }

int launch_select(const jenga_plan* p, const void* q, const void* k, int32_t* sel_count, int32_t* sel_index,
                  uint8_t* mask, void* ws, bool pooled, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (p->cfg.head_dim == 128) return run_select<128>(p, q, k, sel_count, sel_index, mask, ws, pooled, st);
  return run_select<64>(p, q, k, sel_count, sel_index, mask, ws, pooled, st);
}

template <int D>
static int run_permute_pool(const jenga_plan* p, const void* const src[3], void* const dst[3], void* ws, hipStream_t st) {
  const jenga_config& c = p->cfg;
  const jenga_plan_info_t& f = p->info;
  double *qh, *kh;
  pooled_rows<D>(p, ws, &qh, &kh);
  Moves moves = {{(const uint4*)src[0], (const uint4*)src[1], (const uint4*)src[2]},
                 {(uint4*)dst[0], (uint4*)dst[1], (uint4*)dst[2]},
                 {qh, kh}};
  const dim3 grid(c.heads, f.M, 3 * c.batch);
  if (c.block == 128)
    permute_pool_kernel<128, D><<<grid, 256, 0, st>>>(moves, p->d_src_of_pos, p->d_blk_valid, f.N_v + c.n_text, f.M_v, c.batch);
  else if (c.block == 64)
    permute_pool_kernel<64, D><<<grid, 256, 0, st>>>(moves, p->d_src_of_pos, p->d_blk_valid, f.N_v + c.n_text, f.M_v, c.batch);
  else
    permute_pool_kernel<32, D><<<grid, 256, 0, st>>>(moves, p->d_src_of_pos, p->d_blk_valid, f.N_v + c.n_text, f.M_v, c.batch);
  return hipGetLastError() == hipSuccess ? JENGA_OK : JENGA_EHIP;
}

int launch_permute_pool(const jenga_plan* p, const void* const src[3], void* const dst[3], void* select_ws, void* stream) {
  if (p->cfg.head_dim == 128) return run_permute_pool<128>(p, src, dst, select_ws, (hipStream_t)stream);
  return run_permute_pool<64>(p, src, dst, select_ws, (hipStream_t)stream);
}

}  // namespace jenga

extern "C" int jenga_select_blocks_static(const jenga_plan* p, const void* q_curve, const void* k_curve,
                                          int32_t* sel_count, int32_t* sel_index, uint8_t* mask_or_null,
                                          void* stream) {
  if (!p || !q_curve || !k_curve || !sel_count || !sel_index) return JENGA_EINVAL;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != p->device) return JENGA_EINVAL;
  if (p->info.select_workspace_bytes > STATIC_SCRATCH_BYTES) return JENGA_EWORKSPACE;
  void* ws = scratch_address(dev);   // looked up when the plan was created; never allocates
  if (ws == nullptr) return JENGA_EHIP;
  // every byte of the scratch that select_kernel reads is written first by pool_kernel of this same call, so nothing
  // has to be cleared between calls
  return jenga::launch_select(p, q_curve, k_curve, sel_count, sel_index, mask_or_null, ws, false, stream);
}
