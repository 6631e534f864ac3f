// Block-sparse flash attention for gfx950 (appendix Alg. 4; Alg. 2 for the text rows; Eq. 1 inside
// the visited blocks).
//
// One workgroup owns one query block of BLK rows of one (batch, head) and walks the ascending list of its
// selected key blocks; a wavefront has 32 query rows.  Blocks of 64 and 128 tokens: BLK/32 wavefronts share the
// key tiles through LDS (attn_h_kernel); blocks of 32: nothing to share, the list is split over the wavefronts
// of the workgroup (attn_kernel).  Per key tile:
//     S^T = K Q^T         v_mfma_f32_32x32x16_bf16, K fragments from LDS or global memory, Q fragments in
//                         registers
//     online softmax      float32, base-2 exponent, statistics per query row; the reference the exponent is
//                         taken against moves only when a row sum leaves its range, row sums are float32 sums
//                         of P
//     O^T += V^T P^T      v_mfma_f32_32x32x16_bf16, V^T fragments likewise, P^T straight from the S^T
//                         accumulators
// Working on the transposed products keeps one query row in one lane (column) of every
// accumulator, so the row maximum and row sum are lane-local (one cross-half exchange), and the
// accumulator layout of S^T is already the B-operand layout PV needs: P never goes through LDS.
//
// A call that is given K and V themselves reads them as they are in the in-order kernels for blocks of 64 and 128 tokens
// (K_ROWS).  For the others both are first re-tiled once per call (pack_kernel) into "fragment order": for every
// block a 16-byte piece per (fragment, lane) in exactly the order the LDS reads want them, so that a tile
// moves global -> LDS as a straight copy and every LDS read is a conflict-free 1 KB wave read.  A packed
// workspace always holds that order, whatever the walk: plans of one grid may share it.
// The packed V tile is transposed, with its key index permuted to match the accumulator layout:
//     accumulator register r of kv-tile mt, lane l  <->  key 32*mt + 8*(r/4) + 4*(l/32) + r%4,
//     query (l%32).
#include <hip/hip_runtime.h>

#include <cmath>

#include <type_traits>
#include <utility>

#include "jenga_internal.h"

namespace {

using jenga::map_work;
using jenga::WorkMap;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two floats -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Launch parameters, behind the packed tiles: the pace of the paced walk, the eight counters of a queue (see take_item) and
// behind them whether it is used.
constexpr int PARAM_QUEUE = 8, QUEUE_USED = 8;

// jenga_forward: rows go to the thw side from the kernel that has them in registers, beside the curve side.  These are instances of
// their own: as a branch in one kernel for all, small calls that have no such rows took 1 to 4 % longer (attention, 9 blocks of 64 x
// 3 heads, D = 64, 12.0 -> 12.6 us, 20 of 32 x 3, D = 128, 9.7 -> 10.1).
// thw: [batch][n_src][heads][D]; first: (batch, head) pair that the launch's first one is.
struct NoThwRows {};
struct ThwRows {
  uint16_t* thw;
  const int32_t* src_of_pos;
  int n_src, heads, first;
  // channel 0 of row `pos` of the launch's pair bh; nullptr: a pad
  template <int D>
  __device__ __forceinline__ uint16_t* row(int bh, int pos) const {
    const int s = src_of_pos[pos], b = (first + bh) / heads, h = first + bh - b * heads;
    return s < 0 ? nullptr : thw + (((size_t)b * n_src + s) * heads + h) * D;
  }
  // The kernel's first argument, read again where it is called: kept over attn_h's loop it would cost scalar registers there
  // (up to 9 more, spilled ones in four of the kernels).
  __device__ __forceinline__ static ThwRows argument() {
    ThwRows t = {};
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    t = *(const __attribute__((address_space(4))) ThwRows*)at;
#endif
    return t;
  }
};

// grid (M, batch*heads, 2).  z = 0: K tile -> fragment order; z = 1: V tile -> transposed fragment order, pad rows zeroed.
// A workgroup each, so that the two chains of loads and stores run side by side: 931 blocks x 24 heads (2.9 GB) 531 ->
// 511 us = 5.7 TB/s, 262 x 24 156 -> 145 us; HBM-bound from there on.
template <int BLK, int D>
__global__ __launch_bounds__(256) void pack_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                   uint4* __restrict__ kp, uint4* __restrict__ vp,
                                                   const int32_t* __restrict__ blk_valid, int M, int n_pad) {
  constexpr int KS = D / 16, PS = BLK / 16, CH = D / 8;
  constexpr int TILE_CHUNKS = BLK * D / 8;
  constexpr int LDV = D + 8;   // padded row length (elements) of the staged V tile
  __shared__ uint16_t vl[BLK * LDV];
  const int j = blockIdx.x, bh = blockIdx.y;
  const int nv = blk_valid[j];
  const size_t row0 = (size_t)bh * n_pad + (size_t)j * BLK;
  const uint4* ksrc = (const uint4*)(k + row0 * D);
  const uint4* vsrc = (const uint4*)(v + row0 * D);
  uint4* kdst = kp + ((size_t)bh * M + j) * TILE_CHUNKS;
  uint4* vdst = vp + ((size_t)bh * M + j) * TILE_CHUNKS;

  if (blockIdx.z == 0) {
#pragma unroll
    for (int o = threadIdx.x; o < TILE_CHUNKS; o += 256) {
      const int lane = o & 63, f = o >> 6;
      const int ks = f % KS, mt = f / KS;
      const int row = 32 * mt + (lane & 31);
      kdst[o] = ksrc[row * CH + 2 * ks + (lane >> 5)];
    }
    return;
  }
  for (int o = threadIdx.x; o < TILE_CHUNKS; o += 256) {
    const int row = o / CH, cc = o % CH;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (row < nv) val = vsrc[o];
    *(uint4*)&vl[row * LDV + cc * 8] = val;
  }
  __syncthreads();
  for (int o = threadIdx.x; o < TILE_CHUNKS; o += 256) {
    const int lane = o & 63, f = o >> 6;
    const int ps = f % PS, dt = f / PS;
    const int hl = lane >> 5, d = 32 * dt + (lane & 31);
    uint32_t w[4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      const int e = 2 * e2;
      const int kv0 = 16 * ps + 8 * (e / 4) + 4 * hl + (e % 4);
      w[e2] = (uint32_t)vl[kv0 * LDV + d] | ((uint32_t)vl[(kv0 + 1) * LDV + d] << 16);
    }
    vdst[o] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// One DMA instruction, global -> LDS without passing through registers: every lane hands over its
// own 16-byte global address (wave-uniform 64-bit base in SGPRs + 32-bit per-lane byte offset); the
// data of the wave lands contiguously (1 KB) behind the wave-uniform LDS byte address in M0.
// Written as asm so that the compiler does not track these copies: it would otherwise order every
// later LDS read of the same array behind them with a full vmcnt(0) wait.  Completion is tracked by
// vmcnt and waited for explicitly (wait_vmem) before the barrier that publishes a tile.
// The LDS byte address is lds_addr, a number that the caller keeps in an SGPR, plus `lds_off`.
__device__ __forceinline__ void dma_1kb_to_lds_at(const void* uniform_base, uint32_t lane_byte_off, uint32_t lds_addr,
                                                  int lds_off) {
  const uint64_t b = (uint64_t)uniform_base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  const uint64_t base = ((uint64_t)hi << 32) | lo;
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr), "v"(lane_byte_off), "s"(base), "i"(lds_off)
               : "memory", "m0", "scc");
}

__device__ inline void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0) only

// compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// One 1 KB MFMA fragment (16 bytes per lane) from LDS, issued here and now: the compiler's own
// scheduling reads one fragment, waits, multiplies, and so leaves the LDS latency open before
// every MFMA.  Reads issued through lds_frag are complete only after lds_wait on their registers.
// Between the two asm statements the destination registers are in flight: the code is correct only
// as long as the compiler does not copy or reuse them there.  lds_wait ties them ("+v") so that the
// allocator has no reason to, and tests/test_kernel_listing.py checks the generated listing of every
// build for exactly this (no instruction between a read and its wait touches the read's registers).
// Folding read, MFMAs and wait of a group into one asm statement removes the assumption but was
// measured 4 % slower here: with S live the register budget of three wavefronts per SIMD only leaves
// room for groups of two, and the compiler can no longer lay the softmax arithmetic under the MFMAs.
template <int BYTE_OFF>
__device__ __forceinline__ void lds_frag(u32x4& dst, uint32_t lane_addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(lane_addr), "n"(BYTE_OFF) : "memory");
}
// x ^ y, formed where it stands: hoisted out of a loop it would take a register there.
__device__ __forceinline__ uint32_t xor_here(uint32_t x, int y) {
  uint32_t r;
  asm volatile("v_xor_b32 %0, %1, %2" : "=v"(r) : "i"(y), "v"(x));
  return r;
}

// 64 bits per lane, transposed: the 16 lanes of a group name 4 rows of 16 bf16 each, a row by 4 lanes of 8 bytes; lane i gets
// column i, row 0 first.
template <int BYTE_OFF>
__device__ __forceinline__ void lds_columns(u32x2& dst, uint32_t lane_addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(lane_addr), "n"(BYTE_OFF) : "memory");
}
__device__ __forceinline__ void lds_wait(u32x2 (&g)[4][2]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(g[0][0]), "+v"(g[0][1]), "+v"(g[1][0]), "+v"(g[1][1]), "+v"(g[2][0]), "+v"(g[2][1]), "+v"(g[3][0]),
                 "+v"(g[3][1])
               :
               : "memory");
}
__device__ __forceinline__ void lds_wait(u32x4 (&g)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]), "+v"(g[3]) : : "memory");
}

// max over the two lanes l and l ^ 32 (the two halves of a query row's keys), in the vector ALU
__device__ inline float max_with_other_half(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
#else
  return x;   // host pass only; never executed
#endif
}

// Alg. 4 keeps a running maximum m of every row and rescales l and O whenever it grows.  Here the row
// maximum is not on the common path: the maximum over the 32 logits of a lane (16 v_max3, a cross-half
// exchange, a compare) is a chain that has to finish after the last MFMA of S and before the first exponential can issue, in
// every step of every wavefront.  Without it a step forms its probabilities against the reference as
// it stands and only looks at the sum: while a lane's 32 probabilities add up to at most P_SUM_MAX they
// are all representable, and so are the float32 sums and products built from them (bf16 and float32
// share the exponent range; 2^30 times the row length times |V| stays far below 2^127).  A sum above
// the bound, infinite or undefined sends the step down the exact path: logits again (the K half is
// still in LDS), row maximum, rescale, probabilities <= 1.  The first step of a row starts there.
// The reference never exceeds the largest logit seen, so the largest term is never lost to underflow.
constexpr float P_SUM_MAX = 1073741824.0f;   // 2^30

// ---------------------------------------------------------------------------------------------
// attn_h_kernel: blocks of 128 tokens, walked in half blocks of 64 keys, and blocks of 64 tokens.
//
// A wavefront does its softmax between its two runs of MFMAs, so it is the other wavefronts of the
// SIMD that keep the MFMA pipe fed meanwhile: occupancy matters.  A step over 64 keys needs half
// the S and P registers and half the LDS of a step over 128, which lets three workgroups (twelve
// wavefronts) live on a CU instead of two.
//
// Blocks of 64 tokens run the same loop with two wavefronts, one step per block.  At D = 128 that takes 32 KB of LDS, which is given
// out in pieces of 1280 bytes: four workgroups on a CU, two wavefronts per SIMD, where registers allow three.  Steps of 32 keys
// (attn_keys32_kernel) take half and put six there; their barriers cost a lone workgroup 1.3 times the time a block (1.2 us ->
// 1.6), and with all places taken a workgroup needs 3.6 us a block instead of 2.5, so that a text row ends later.  attn_keys32() in
// jenga_plan.cpp says which calls take them.
// At D = 64 the softmax, not the matrix core, is the longer part of a step (32 exponentials of 16 cycles and 80 other vector
// instructions of 4 against 512 cycles of MFMA; 1100 cycles are measured), and four wavefronts per SIMD (128 registers) fit.
//
// PACED (JENGA_FLAG_PACED_WALK): the selected blocks are not visited in list order.  A position G sweeps
// over the key blocks once per lap, derived from the constant-frequency clock that every CU reads
// (s_memrealtime), and a workgroup always takes the first block of its list that it has not visited yet
// at or after G (wrapping around).  Softmax attention does not depend on the order of the keys, so the
// result is the same up to rounding; what changes is when a tile is asked for: all workgroups of an XCD
// now ask for neighbouring tiles at neighbouring times, and the 4 MB L2, which catches a seventh of the
// tile reads of the in-order walk, catches more than half of them (measured on the 720p workload).
// The price: the order, and with it the last bits of the output, can differ from run to run.
// ---------------------------------------------------------------------------------------------
template <int FIRST, int N>
struct Tiles {   // of 32 keys
  static constexpr int first = FIRST, n = N;
};
template <int BLK, int D>
constexpr int attn_h_min_waves() { return D == 128 ? 3 : 4; }   // wavefronts per SIMD that the registers have to allow

// SPLIT: lists are cut into parts, a workgroup each; the parts' O, reference and sum go to the workspace and merge_kernel puts
// them together.  Grids that leave the chip idle: every list into Split::of(cnt) parts of equal length.  Others: what
// the launch's Deal says.
struct Split {
  int parts, chunk;   // most parts of a list, list entries from which on there is one more part (0: always all parts)
  int stride;         // workgroups per part
  jenga::Deal deal;   // if deal.parts > 0
  int first;          // with a queue: positions of an XCD that it does not deal out (all, where the plan has no counters)
  float* o;           // [slot][BLK/32][D/32][4][64][4]: O in accumulator order
  float* stat;        // [slot][2][BLK]: reference, sum; slot = (batch*head*M + block) * parts + part, or by deal_position()
  __device__ int of(int cnt) const { return chunk == 0 ? parts : max(1, min(parts, (cnt + chunk - 1) / chunk)); }
};

// Work for one workgroup of a launch that is dealt out by counters, one per XCD (workgroup n runs on XCD n % 8): XCDs that
// have the same work to do need up to a tenth more or less time for it than others.  The value 8 r + x stands for position r
// of XCD x (deal_position).  An XCD whose own are all taken goes on with those of the one that has most left.  -1: all are taken.
// A launch has a quarter more workgroups than there are positions, so that a fast XCD finds some to run; the others end
// here, in a few us.  (One workgroup that loops over positions keeps the kernel's arguments in scalar registers over
// the loop: 20 to 70 spilled ones.)  The workgroups of the first generation do not ask, all at once, but take the position of their
// own number: 34 shapes of 1 to 4 generations, 0.15 to 2.8 ms, 2 % less on average, 10 % where a workgroup lasts 100 us.
__device__ inline int take_item(uint32_t* queue, int n_end) {
  int x = blockIdx.x & 7;
  for (;;) {
    const int n = 8 * (int)__hip_atomic_fetch_add(queue + x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + x;
    if (n < n_end) return n;
    int least = n_end;
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      const int next = 8 * (int)__hip_atomic_load(queue + y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + y;
      if (next < least) {
        least = next;
        x = y;
      }
    }
    if (least == n_end) return -1;
  }
}

// KEYS: of a step.  THW: the kernel's first argument is a ThwRows.
template <int BLK, int D, int KEYS, bool PACED, bool SPLIT, bool K_ROWS, bool THW>
__device__ __forceinline__ void attn_h(
    const uint16_t* __restrict__ q, const u32x4* __restrict__ kp, const u32x4* __restrict__ vp,
    const int32_t* __restrict__ sel_count, const int32_t* __restrict__ sel_index,
    uint16_t* __restrict__ out, float* __restrict__ lse, const WorkMap& work, int n_pad, int pad_v, int pad_c,
    float scale_log2e, float bias_log2e, const uint32_t* __restrict__ pace_params, const Split& split, uint32_t* queue) {
  constexpr int KS = D / 16, DT = D / 32, PS = BLK / 16, MH = KEYS / 32, PH = KEYS / 16;
  constexpr int NW = BLK / 32, NTHR = 64 * NW, HALVES = BLK / KEYS;   // wavefronts, threads, steps per key block
  // Sets of keys that a step forms and adds up probabilities in, against a reference that may move between them.  Blocks of 64
  // tokens at D = 128: sets of 32 keys in either kind of step, so that results are the same bits whichever a call takes.
  constexpr int SETS = BLK == 64 && D == 128 && KEYS == 64 ? 2 : 1;
  constexpr int TILE_CHUNKS = BLK * D / 8, HALF_CHUNKS = KEYS * D / 8, CPT = HALF_CHUNKS / NTHR;
  static_assert(HALVES >= 1 && (!PACED || HALVES == 2), "the paced walk needs two steps a block");
  // The keys of the step: fragments from packed tiles, or (K_ROWS) rows of D channels as they lie in K and V, with the
  // 16-byte pieces of a row rotated by an exclusive or on the way.  K: with k_swizzle(row), so that the 16 rows that are
  // read at a time fall on different banks.  V is read by columns, ds_read_b64_tr_b16, which hands a lane 4 keys of its
  // channel: two of them are a fragment, in the key order of the accumulators.  There v_swizzle(row) spreads the 4 rows x
  // 64 bytes that half a wavefront reads over the banks.  A copy brings whole rows: with 4 rows x 64 bytes for every 16 lanes
  // of it, which would have left both reads without address arithmetic, 222 blocks of 64 x 12 took 609 instead of 493 us.
  // The addresses are formed where they are needed (xor_here; ten instructions a step): hoisted, they cost spills.
  // No packing, against V packed (before, with K packed too): layer of 222 blocks of 64 x 12 heads 521 -> 486 us, 17
  // blocks x 8 59.5 -> 56.2, 48 x 16 at D = 64 133.1 -> 130.2, 262 x 24 4.48 -> 4.45 ms (the columns take twice as many LDS
  // instructions as fragments).  The paced walk keeps packed tiles where it is paced, and so does whoever has packed them already.
  static_assert(!(PACED && K_ROWS) || SPLIT, "only cut lists, which are visited in ascending order");
  __shared__ __align__(256) u32x4 Ks[HALF_CHUNKS];
  __shared__ __align__(256) u32x4 Vs[HALF_CHUNKS];   // fragments (dt, p2) of the same keys, or rows
  __shared__ uint32_t rem_bits[PACED ? 64 : 1];   // PACED: bitmap of the blocks still to visit, 32 per word
  __shared__ int pace_slot[2];                    // PACED: G for the next pick, published by thread 0

  int n = blockIdx.x, part = 0, n_parts = 1, slot = -1;   // slot: of the partial result, -1: the whole list
  const bool dealt = SPLIT && split.deal.parts > 0;
  if constexpr (SPLIT) {
    if (dealt) {
      jenga::Deal deal = split.deal;
      if (queue != nullptr && __builtin_amdgcn_readfirstlane((int)queue[QUEUE_USED]) == 0) {
        deal = deal.vision_whole();
      } else if (queue != nullptr && n >= 8 * split.first) {
        volatile int* taken = (volatile int*)Ks;   // no tile is in there yet
        if (threadIdx.x == 0) *taken = take_item(queue, 8 * deal.positions());
        __syncthreads();
        n = __builtin_amdgcn_readfirstlane(*taken);
        __syncthreads();
        if (n < 0) return;
      }
      if (!jenga::deal_position(n >> 3, n & 7, deal, work, &n, &part, &n_parts, &slot)) return;
    } else {
      part = n / split.stride;
      n -= part * split.stride;
    }
  }
  int bh, i;
  if (!map_work(n, work, &bh, &i)) return;
  const int M = work.M, M_v = work.M_v;
  if (SPLIT && !dealt) {
    n_parts = split.of(min(max(sel_count[(size_t)bh * M + i], 0), M));
    if (part >= n_parts) return;
    if (n_parts > 1) slot = (bh * M + i) * split.parts + part;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hl = lane >> 5, ql = lane & 31;
  const int qrow = i * BLK + 32 * wave + ql;

  bf16x8 qf[KS];
  {
    const u32x4* qp = (const u32x4*)(q + ((size_t)bh * n_pad + qrow) * D);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, qp[2 * ks + hl]);
  }

  int cnt = sel_count[(size_t)bh * M + i];
  cnt = min(max(cnt, 0), M);
  const int32_t* idx = sel_index + ((size_t)bh * M + i) * M;
  if constexpr (SPLIT && !PACED) {   // positions [cnt * part / n_parts, cnt * (part + 1) / n_parts) of the list
    const int lo = cnt * part / n_parts;
    cnt = cnt * (part + 1) / n_parts - lo;
    idx += lo;
  }
  uint32_t rem = 0, pace_k = 0;
  if constexpr (PACED) {
    // the list as a bitmap (a block listed twice is visited once); lane w of every wavefront holds word w
    if (pace_params != nullptr) pace_k = pace_params[0];   // 0: ascending order
    if (tid < 64) rem_bits[tid] = 0;
    __syncthreads();
    for (int t = tid; t < cnt; t += NTHR) {
      const int jj = min(max(idx[t], 0), M - 1);
      atomicOr(&rem_bits[jj >> 5], 1u << (jj & 31));
    }
    __syncthreads();
    rem = rem_bits[lane];
    int pc = __popc(rem);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) pc += __shfl_xor(pc, o, 64);
    cnt = __builtin_amdgcn_readfirstlane(pc);
    if (SPLIT && n_parts > 1) {   // the same positions of the bitmap
      const int lo = cnt * part / n_parts, hi = cnt * (part + 1) / n_parts;
      const int own = __popc(rem);
      int before = own;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(before, o, 64);
        before += lane >= o ? x : 0;
      }
      before -= own;   // set bits in the words of the lanes below
      uint32_t kept = 0;
      for (int r = before; rem != 0; ++r) {
        const uint32_t bit = rem & (0u - rem);
        kept |= r >= lo && r < hi ? bit : 0u;
        rem ^= bit;
      }
      rem = kept;
      cnt = hi - lo;
    }
  }
  // G: the low 32 bits of the clock times 2^32 / lap wrap once per lap; the high half of that times M is the block
  auto pace_now = [&]() { return (int)__umulhi((uint32_t)__builtin_amdgcn_s_memrealtime() * pace_k, (uint32_t)M); };
  // The first remaining block at or after G, else the first one after the wrap.  Every wavefront runs this on its
  // own copy of the bitmap with the same G, so the four agree without exchanging the result.  Needs rem != 0.
  // G is wave-uniform, so most of this is scalar arithmetic.
  auto pick = [&](int G_any_lane) {
    const int G = __builtin_amdgcn_readfirstlane(G_any_lane);
    const int w0 = G >> 5;
    const uint32_t low = (1u << (G & 31)) - 1u;
    uint32_t mw = lane == w0 ? rem & ~low : rem;
    uint64_t bal = __builtin_amdgcn_ballot_w64(mw != 0) & (~0ull << w0);
    if (bal == 0) {   // nothing left at or after G: every remaining block lies before it
      mw = rem;
      bal = __builtin_amdgcn_ballot_w64(rem != 0);
    }
    const int src = __builtin_ctzll(bal);
    const int bit = __builtin_ctz(__builtin_amdgcn_readlane(mw, src));
    rem &= lane == src ? ~(1u << bit) : ~0u;
    return src * 32 + bit;
  };
  const int steps = HALVES * cnt;
  const u32x4* kbase = kp + (size_t)bh * M * TILE_CHUNKS;
  const u32x4* vbase = vp + (size_t)bh * M * TILE_CHUNKS;

  // K half h of block j is one contiguous run of the packed tile; V half h is PH fragments out of
  // every PS of each channel tile: wave w copies fragments f = c*NW + w, f = dt*PH + p2
  const uint32_t ks_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)Ks + (uint32_t)wave * 1024u);
  const uint32_t vs_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)Vs + (uint32_t)wave * 1024u);
  constexpr int CH = D / 8, ROWS_PER_COPY = NTHR / CH;
  auto k_swizzle = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
  auto v_swizzle = [](int row) { return D == 128 ? (row & 3) * 4 : (row & 2) * 2; };
  const uint32_t k_off = (uint32_t)(K_ROWS ? tid / CH * CH + (tid % CH ^ k_swizzle(tid / CH)) : tid) * 16u;
  const uint32_t v_off = (uint32_t)(K_ROWS ? tid / CH * CH + (tid % CH ^ v_swizzle(tid / CH)) : lane) * 16u;
  auto k_half_to_lds = [&](int j, int h) {
    const char* kt = (const char*)(kbase + (size_t)j * TILE_CHUNKS + h * HALF_CHUNKS);
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      dma_1kb_to_lds_at(kt + (size_t)c * (NTHR * 16),
                        K_ROWS ? k_off ^ (uint32_t)k_swizzle(c * ROWS_PER_COPY) * 16u : k_off,
                        ks_wave, c * (NTHR * 16));
  };
  auto v_half_to_lds = [&](int j, int h) {
    const u32x4* vt = vbase + (size_t)j * TILE_CHUNKS + (K_ROWS ? h * HALF_CHUNKS : PH * h * 64);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int f = c * NW + wave, dt = f / PH, p2 = f % PH;
      dma_1kb_to_lds_at(vt + (size_t)(K_ROWS ? c * NTHR : (dt * PS + p2) * 64), v_off, vs_wave, c * (NTHR * 16));
    }
  };

  float m_run = -INFINITY, l_run = 0.f;
  bool unset = true;   // no row has a reference yet (uniform: every row sees the same keys)
  f32x16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) O[dt][r] = 0.f;
  const uint32_t ks_lane =
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)Ks +
      (K_ROWS ? ql * (2 * D) + (hl ^ k_swizzle(ql)) * 16 : lane * 16);
  // (m2, ks) = (e & 1, 2 g + e / 2) of two tiles, (first, 4 g + e) of one; K_ROWS: piece 2 ks + hl of row 32 m2 + ql
  auto k_frags = [&](u32x4 (&dst)[4], auto G, auto TILES) {
    typedef decltype(TILES) T;
    constexpr int g = decltype(G)::value, PER = 4 / T::n;   // values of ks in a group
    uint32_t at[PER];
    static_for<PER>([&](auto U) {
      constexpr int ks = PER * g + decltype(U)::value;
      at[decltype(U)::value] = K_ROWS && ks > 0 ? xor_here(ks_lane, ks * 32) : ks_lane;
    });
    static_for<4>([&](auto E) {
      constexpr int e = decltype(E)::value, m2 = T::first + e % T::n, ks = PER * g + e / T::n;
      lds_frag<K_ROWS ? m2 * 64 * D : (m2 * KS + ks) * 1024>(dst[e], at[e / T::n]);
    });
  };
  // K_ROWS: columns 32 dt + 16 (lane / 16 % 2) + lane % 16 of four rows
  const int v_row = 4 * hl + ((lane >> 2) & 3);
  const uint32_t vs_lane =
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)Vs +
      (K_ROWS ? v_row * (2 * D) + v_swizzle(v_row) * 16 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8 : lane * 16);

  // The block index of the next step is fetched a step ahead, and the valid-token count of a
  // block follows from its index, so no step waits on a scalar load it has just issued.
  int j_next = 0;
  if constexpr (PACED) {
    if (tid == 0) pace_slot[0] = pace_now();
    __syncthreads();
    if (cnt > 0) j_next = pick(pace_slot[0]);
  } else {
    if (cnt > 0) j_next = min(max(idx[0], 0), M - 1);
  }
  if (cnt > 0) k_half_to_lds(j_next, 0);

  auto step = [&](int st, int h) __attribute__((always_inline)) {
    const int j = j_next;
    wait_vmem();       // this wave's part of the K half has landed
    __syncthreads();   // K half of this step is in LDS; every wave is past the previous PV
    v_half_to_lds(j, h);

    // S^T = K Q^T for tiles of this step's keys, with the pad keys of a ragged block set to -inf.  Fragments come in groups of
    // four (k_frags); group g + 1 is in flight while the MFMAs of group g run, and the accumulators of two tiles alternate.
    f32x16 S[MH];
    const int nv = BLK - (j == M_v - 1 ? pad_v : (j == M - 1 ? pad_c : 0));
    auto logits = [&](auto TILES) {
      typedef decltype(TILES) T;
#pragma unroll
      for (int m2 = T::first; m2 < T::first + T::n; ++m2)
#pragma unroll
        for (int r = 0; r < 16; ++r) S[m2][r] = 0.f;
      {
        constexpr int NG = KS * T::n / 4;
        u32x4 A[2][4];
        k_frags(A[0], std::integral_constant<int, 0>{}, TILES);
        static_for<NG>([&](auto G) {
          constexpr int g = decltype(G)::value;
          lds_wait(A[g & 1]);
          if constexpr (g + 1 < NG)
            k_frags(A[(g + 1) & 1], std::integral_constant<int, g + 1>{}, TILES);
          static_for<4>([&](auto E) {
            constexpr int e = decltype(E)::value, m2 = T::first + e % T::n, ks = 4 / T::n * g + e / T::n;
            S[m2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, A[g & 1][e]), qf[ks], S[m2],
                                                            0, 0, 0);
          });
        });
      }

      if (nv < BLK) {   // sequence-length mask: pad keys of a ragged block
        asm volatile("");   // a real, rarely taken branch
        int valid = nv - KEYS * h - 4 * hl;
#pragma unroll
        for (int m2 = T::first; m2 < T::first + T::n; ++m2)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (r % 4 == 0) asm volatile("" : "+v"(valid));   // four comparisons at a time: 32 masks would be 64 scalar registers
            if (32 * m2 + 8 * (r / 4) + (r % 4) >= valid) S[m2][r] = -INFINITY;
          }
      }
    };

    // ---- online softmax on S^T (lane = query row, registers = keys) ----
    const float bias = (i < M_v && j >= M_v) ? bias_log2e : 0.f;
    bf16x8 pb[PH];
    // P = 2^(S * scale + off) of set G as bf16 fragments for the second product; returns this lane's sum of them
    auto probabilities = [&](float off, auto G) {
      constexpr int P_SET = PH / SETS, p_first = decltype(G)::value * P_SET;
      float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
      for (int p2 = p_first; p2 < p_first + P_SET; ++p2) {
        uint32_t w[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(S[p2 >> 1][8 * (p2 & 1) + 2 * e2], scale_log2e, off));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(S[p2 >> 1][8 * (p2 & 1) + 2 * e2 + 1], scale_log2e, off));
          w[e2] = pack_bf16x2(p0, p1);
          rs0 += p0;
          rs1 += p1;
        }
        u32x4 pw = {w[0], w[1], w[2], w[3]};
        pb[p2] = __builtin_bit_cast(bf16x8, pw);
      }
      return rs0 + rs1;
    };
    // the block of the next step, looked up under the arithmetic of this one
    auto advance = [&]() {
      if constexpr (PACED) {
        // G is sampled during the first half step of a block (the clock read has time to return under the
        // softmax) and turned into the next block by every wavefront during the second half step
        if (h == 0) {
          if (tid == 0) pace_slot[((st >> 1) + 1) & 1] = pace_now();
        } else if (st + 1 < steps) {
          j_next = pick(pace_slot[((st >> 1) + 1) & 1]);                 // used after the next barrier
        }
      } else {
        j_next = min(max(idx[min(st + 1, steps - 1) / HALVES], 0), M - 1);   // used after the next barrier
      }
    };
    // Common path: probabilities against the reference as it stands, no row maximum (see P_SUM_MAX).  Exact
    // path: the logits again, the reference moved to the row maximum (the rescaling step of Alg. 4), and
    // probabilities <= 1 in place of the first attempt.  Each branch forms and consumes its own S, so S never
    // occupies registers beside a finished P.
    typedef std::integral_constant<int, 0> Set0;
    typedef std::integral_constant<int, SETS - 1> Set1;
    typedef Tiles<0, MH> All;
    float rs[SETS], alpha_mid;   // set where they are used: a value from before the products would take a register there
    bool in_range = false, mid = false;   // mid: O is to be rescaled by alpha_mid between the sets
    const bool first = unset;
    if (!first) {
      logits(All{});
      advance();
      rs[0] = probabilities(bias - m_run, Set0{});
      if constexpr (SETS == 2) rs[1] = probabilities(bias - m_run, Set1{});
      in_range = __ballot(!((SETS == 2 ? rs[0] + rs[SETS - 1] : rs[0]) <= P_SUM_MAX)) == 0;
    }
    if (!in_range) {
      asm volatile("");   // a real branch: the first step of a row, then almost never
      // the reference moved to the maximum of a set; returns the factor for what has been added up so far
      auto move_reference = [&](auto TILES) {
        typedef decltype(TILES) T;
        float mx = -INFINITY;
#pragma unroll
        for (int m2 = T::first; m2 < T::first + T::n; ++m2)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[m2][r]);
        mx = max_with_other_half(mx);
        const float m_new = fmaxf(m_run, fmaf(mx, scale_log2e, bias));
        const float alpha = m_new == m_run ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
        m_run = m_new;
        unset = __ballot(m_run == -INFINITY) != 0;
        return alpha;
      };
      auto finite = [&]() { return m_run == -INFINITY ? 0.f : bias - m_run; };   // every key so far was padding: keep it finite
      auto rescale = [&](float alpha) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) O[dt][r] *= alpha;
      };
      if constexpr (SETS == 1) {
        logits(All{});
        if (first) advance();
        rescale(move_reference(All{}));
        rs[0] = probabilities(finite(), Set0{});
      } else {   // one set after the other, and only if it is the one that is out of range
        logits(Tiles<0, 1>{});
        if (first) advance();
        if (first || __ballot(!(rs[0] <= P_SUM_MAX)) != 0) rescale(move_reference(Tiles<0, 1>{}));
        l_run += probabilities(finite(), Set0{});
        rs[0] = 0.f;
        logits(Tiles<1, 1>{});
        rs[1] = probabilities(finite(), Set1{});
        mid = unset || __ballot(!(rs[1] <= P_SUM_MAX)) != 0;
        if (mid) {
          alpha_mid = move_reference(Tiles<1, 1>{});
          rs[1] = probabilities(finite(), Set1{});
        }
      }
    }
    l_run += rs[0];
    if constexpr (SETS == 2) l_run += rs[1];

    wait_vmem();       // this wave's part of the V half has landed
    if (K_ROWS && nv < BLK) {   // pad rows hold anything, and their probabilities are zero
      asm volatile("" : : : "memory");   // a real, rarely taken branch; nothing is written before the copies have landed
      int at = threadIdx.x;
      asm volatile("" : "+v"(at));
#pragma unroll 1
      for (; at < HALF_CHUNKS; at += NTHR)
        if (KEYS * h + at / CH >= nv) Vs[at] = u32x4{0, 0, 0, 0};
    }
    __syncthreads();   // V half is in LDS; every wave is done reading the K half
    if (st + 1 < steps) k_half_to_lds(j_next, HALVES == 2 ? (st + 1) & 1 : 0);

    // O^T += V^T P^T, fragments (dt, p2) in groups of four, pipelined as above
    {
      constexpr int NG = DT * PH / 4;
      typedef typename std::conditional<K_ROWS, u32x2[2], u32x4>::type Frag;
      Frag A[2][4];
      uint32_t vs_dt[DT];   // K_ROWS: formed here and now, not kept over the loop
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vs_dt[dt] = K_ROWS && dt > 0 ? xor_here(vs_lane, dt * 64) : vs_lane;
      auto v_frag = [&](Frag& dst, auto DTV, auto P2V) {
        constexpr int dt = decltype(DTV)::value, p2 = decltype(P2V)::value;
        if constexpr (K_ROWS) {   // keys 16 p2 + 4 hl + 0..3 and the same plus 8
          lds_columns<p2 * 32 * D>(dst[0], vs_dt[dt]);
          lds_columns<p2 * 32 * D + 16 * D>(dst[1], vs_dt[dt]);
        } else {
          lds_frag<(dt * PH + p2) * 1024>(dst, vs_lane);
        }
      };
      // of group g: a set after the other, of each two channel tiles at a time
      constexpr int NG_SET = NG / SETS, RUN = PH / SETS / 2;
      constexpr auto dt_of = [](int g, int e) { return 2 * (g % NG_SET / RUN) + (e & 1); };
      constexpr auto p2_of = [](int g, int e) { return g / NG_SET * (PH / SETS) + 2 * (g % RUN) + e / 2; };
      static_for<4>([&](auto E) {
        constexpr int e = decltype(E)::value;
        v_frag(A[0][e], std::integral_constant<int, e & 1>{}, std::integral_constant<int, e / 2>{});
      });
      static_for<NG>([&](auto G) {
        constexpr int g = decltype(G)::value;
        lds_wait(A[g & 1]);
        if constexpr (SETS == 2 && g == NG / 2) {   // the first set has been added up
          if (mid) {
            asm volatile("");   // a real, rarely taken branch
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
              for (int r = 0; r < 16; ++r) O[dt][r] *= alpha_mid;
          }
        }
        if constexpr (g + 1 < NG)
          static_for<4>([&](auto E) {
            constexpr int e = decltype(E)::value, g1 = g + 1;
            v_frag(A[g1 & 1][e], std::integral_constant<int, dt_of(g1, e)>{}, std::integral_constant<int, p2_of(g1, e)>{});
          });
        static_for<4>([&](auto E) {
          constexpr int e = decltype(E)::value, dt = dt_of(g, e), p2 = p2_of(g, e);
          u32x4 a;
          if constexpr (K_ROWS)
            a = __builtin_shufflevector(A[g & 1][e][0], A[g & 1][e][1], 0, 1, 2, 3);
          else
            a = A[g & 1][e];
          O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pb[p2], O[dt], 0, 0, 0);
        });
      });
    }
  };
  if constexpr (KEYS == 32) {   // a block an iteration
    for (int st = 0; st < steps; st += 2) {
      step(st, 0);
      step(st + 1, 1);
    }
  } else {
    for (int st = 0; st < steps; ++st) step(st, HALVES == 2 ? st & 1 : 0);
  }

  // ---- normalise and store: lane holds row qrow, channels 32*dt + 8*g + 4*hl + {0..3} ----
  // The indices are derived again from the thread index (through an opaque copy, so that they are not the values
  // computed before the loop): kept live across the loop they would cost registers there.
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int hl_e = (tid_e >> 5) & 1, ql_e = tid_e & 31;
  const int row_e = 32 * wave + ql_e;
  const size_t qrow_e = (size_t)bh * n_pad + (size_t)i * BLK + row_e;
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if constexpr (SPLIT) {
    if (slot >= 0) {
      float4* o = (float4*)split.o + ((size_t)slot * NW + wave) * (DT * 4 * 64) + (tid_e & 63);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          o[(dt * 4 + g) * 64] = make_float4(O[dt][4 * g], O[dt][4 * g + 1], O[dt][4 * g + 2], O[dt][4 * g + 3]);
      if (hl_e == 0) {
        split.stat[(size_t)slot * 2 * BLK + row_e] = m_run;
        split.stat[((size_t)slot * 2 + 1) * BLK + row_e] = l_tot;
      }
      return;
    }
  }
  const int rows_valid = BLK - (i == M_v - 1 ? pad_v : (i == M - 1 ? pad_c : 0));   // = blk_valid[i], without the load
  const bool row_ok = row_e < rows_valid && l_tot > 0.f;
  const float inv = row_ok ? 1.0f / l_tot : 0.f;
  // natural-log sum of exp(logit) over the visited keys: the running maximum is in base-2 units
  if (lse != nullptr && hl_e == 0)
    lse[qrow_e] = row_ok ? (m_run + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f : -INFINITY;
  uint16_t* orow = out + qrow_e * D;
  uint2 w[DT][4];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      w[dt][g].x = row_ok ? pack_bf16x2(O[dt][4 * g] * inv, O[dt][4 * g + 1] * inv) : 0u;
      w[dt][g].y = row_ok ? pack_bf16x2(O[dt][4 * g + 2] * inv, O[dt][4 * g + 3] * inv) : 0u;
      *(uint2*)(orow + 32 * dt + 8 * g + 4 * hl_e) = w[dt][g];
    }
  if constexpr (THW) {
    uint16_t* trow = ThwRows::argument().row<D>(bh, i * BLK + row_e);
    if (trow == nullptr) return;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) *(uint2*)(trow + 32 * dt + 8 * g + 4 * hl_e) = w[dt][g];
  }
}

#define JENGA_ATTN_H_PARAMETERS                                                                                       \
  const uint16_t *__restrict__ q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp,                         \
      const int32_t *__restrict__ sel_count, const int32_t *__restrict__ sel_index, uint16_t *__restrict__ out,       \
      float *__restrict__ lse, WorkMap work, int n_pad, int pad_v, int pad_c, float scale_log2e, float bias_log2e,    \
      const uint32_t *__restrict__ pace_params, Split split, uint32_t *queue
#define JENGA_ATTN_H_ARGUMENTS \
  q, kp, vp, sel_count, sel_index, out, lse, work, n_pad, pad_v, pad_c, scale_log2e, bias_log2e, pace_params, split, queue

template <int BLK, int D, bool PACED, bool SPLIT, bool K_ROWS>
__global__ __launch_bounds__(2 * BLK, (attn_h_min_waves<BLK, D>())) void attn_h_kernel(JENGA_ATTN_H_PARAMETERS) {
  attn_h<BLK, D, 64, PACED, SPLIT, K_ROWS, false>(JENGA_ATTN_H_ARGUMENTS);
}
template <int BLK, int D, bool PACED, bool SPLIT, bool K_ROWS>
__global__ __launch_bounds__(2 * BLK, (attn_h_min_waves<BLK, D>())) void attn_h_thw_kernel(ThwRows, JENGA_ATTN_H_PARAMETERS) {
  attn_h<BLK, D, 64, PACED, SPLIT, K_ROWS, true>(JENGA_ATTN_H_ARGUMENTS);
}

// Blocks of 64 tokens at D = 128 in steps of 32 keys.  The same bits as in steps of 64.
template <bool SPLIT, bool K_ROWS>
__global__ __launch_bounds__(128, (attn_h_min_waves<64, 128>())) void attn_keys32_kernel(JENGA_ATTN_H_PARAMETERS) {
  attn_h<64, 128, 32, false, SPLIT, K_ROWS, false>(JENGA_ATTN_H_ARGUMENTS);
}
template <bool SPLIT, bool K_ROWS>
__global__ __launch_bounds__(128, (attn_h_min_waves<64, 128>())) void attn_keys32_thw_kernel(ThwRows, JENGA_ATTN_H_PARAMETERS) {
  attn_h<64, 128, 32, false, SPLIT, K_ROWS, true>(JENGA_ATTN_H_ARGUMENTS);
}

// merge_kernel: grid (BLK / 32, M, batch * heads) or, with a Deal, (BLK / 32, rows that are cut), one wavefront per channel tile
// of 32 query rows.  Puts the parts of the lists that attn_h_kernel<.., SPLIT> cut together, in the order of the parts; the other
// rows are done already.
template <int BLK, int D, typename Thw>
__global__ __launch_bounds__(2 * D) void merge_kernel(const int32_t* __restrict__ sel_count, uint16_t* __restrict__ out,
                                                      float* __restrict__ lse, WorkMap work, int n_pad, int pad_v,
                                                      int pad_c, Split split, const uint32_t* __restrict__ queue,
                                                      Thw thw_rows) {
  constexpr int DT = D / 32, NW = BLK / 32;
  const int M = work.M, M_v = work.M_v, wave = blockIdx.x;
  int i = blockIdx.y, bh = blockIdx.z, n_parts;
  size_t slot = (size_t)bh * M + i;
  if (split.deal.parts > 0) {
    int n, first;
    const jenga::Deal deal = queue != nullptr && queue[QUEUE_USED] == 0 ? split.deal.vision_whole() : split.deal;
    if (!jenga::merge_row(blockIdx.y, deal, work, &n, &n_parts, &first) || !map_work(n, work, &bh, &i)) return;
    slot = first;
  } else {
    n_parts = split.of(min(max(sel_count[slot], 0), M));
    if (n_parts == 1) return;
    slot *= split.parts;
  }
  const int lane = threadIdx.x & 63, dt = threadIdx.x >> 6, hl = lane >> 5, row = 32 * wave + (lane & 31);
  const float4* o = (const float4*)split.o + (slot * NW + wave) * (DT * 4 * 64) + dt * 4 * 64 + lane;
  const float* stat = split.stat + slot * 2 * BLK + row;

  float m = -INFINITY, l = 0.f, sum[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) sum[r] = 0.f;
  for (int s = 0; s < n_parts; ++s) m = fmaxf(m, stat[s * 2 * BLK]);
  const float ref = m == -INFINITY ? 0.f : m;
  for (int s0 = 0; s0 < n_parts; s0 += 4) {   // the loads of four parts in flight at a time
    float4 v[4][4];
    float w[4], ls[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int s = min(s0 + u, n_parts - 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) v[u][g] = o[(size_t)s * NW * (DT * 4 * 64) + g * 64];
      w[u] = stat[s * 2 * BLK];
      ls[u] = stat[(s * 2 + 1) * BLK];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u >= n_parts) break;
      const float weight = __builtin_amdgcn_exp2f(w[u] - ref);
      l += weight * ls[u];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        sum[4 * g] += weight * v[u][g].x;
        sum[4 * g + 1] += weight * v[u][g].y;
        sum[4 * g + 2] += weight * v[u][g].z;
        sum[4 * g + 3] += weight * v[u][g].w;
      }
    }
  }
  const int rows_valid = BLK - (i == M_v - 1 ? pad_v : (i == M - 1 ? pad_c : 0));
  const bool row_ok = row < rows_valid && l > 0.f;
  const float inv = row_ok ? 1.0f / l : 0.f;
  const size_t qrow = (size_t)bh * n_pad + (size_t)i * BLK + row;
  if (lse != nullptr && threadIdx.x < 32)
    lse[qrow] = row_ok ? (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
  uint16_t* orow = out + qrow * D + 32 * dt + 4 * hl;
  uint2 packed[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    packed[g].x = row_ok ? pack_bf16x2(sum[4 * g] * inv, sum[4 * g + 1] * inv) : 0u;
    packed[g].y = row_ok ? pack_bf16x2(sum[4 * g + 2] * inv, sum[4 * g + 3] * inv) : 0u;
    *(uint2*)(orow + 8 * g) = packed[g];
  }
  if constexpr (std::is_same<Thw, ThwRows>::value) {
    uint16_t* trow = thw_rows.template row<D>(bh, i * BLK + row);
    if (trow == nullptr) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) *(uint2*)(trow + 32 * dt + 4 * hl + 8 * g) = packed[g];
  }
}

// ---------------------------------------------------------------------------------------------
// attn_kernel: blocks of 32 tokens.
//
// A query block is one MFMA tile of rows, so no two wavefronts want the same key tile and staging it in LDS would
// only add a copy, a barrier and its latency.  Every wavefront works alone: packed fragments go straight from
// global memory to registers (coalesced 1 KB loads), K of the next block in flight under the softmax and the
// second product, V under the logits and the softmax.  The NS wavefronts of a workgroup share one query block and
// take every NS-th entry of its list, which keeps the chip busy on small grids and keeps the dense text rows
// (every block of the sequence) from running on alone; their partial results meet in LDS at the end, in a fixed
// order.  No barrier inside the loop.
//
// Measured on 2048 blocks x 2 heads, D = 64, k = 0.05 (lists of 291 of 2048 blocks on average): 0.75 ms, against 1.77 ms
// for one wavefront per query block that staged its tiles in LDS.  What bounds it there is the path behind the L2: 32
// rows read 8 KB of K and V for 0.26 MFLOP, 10.6 GB in all, from a head (16 MB) that an XCD's 4 MB do not hold; 5.5 GB
// miss, at 7.4 TB/s.  In three passes over ranges of key blocks (RANGE) 1.35 GB miss and it takes 0.52 to 0.56 ms and
// 0.02 for the merge; 0.42 ms were left in a timing variant whose loads all hit the L1.  Eight wavefronts per list at
// D = 64 (two workgroups fill a CU), four at D = 128 (the registers leave room for eight).
// ---------------------------------------------------------------------------------------------
//
// RANGE: K and V of a head do not fit an XCD's L2.  A pass over all query blocks takes the entries of one of
// `split.parts` ranges of key blocks, which then stays in the L2, and the next pass the next range; O, reference and sum
// of the passes go to the workspace and merge_kernel puts them together.
//
// ROWS (D = 64): K and V as they lie, for grids so small that packing them, a launch, is what counts (reads_kv_in_place).  K
// fragments are then 32 rows x 32 bytes instead of 1 KB in one piece; V goes through LDS, 32 rows per wavefront, and is
// read by columns as in attn_h_kernel, the next rows only after that.  The same bits either way.
template <int D, int NS, bool RANGE, bool ROWS, typename Thw>
__device__ __forceinline__ void attn_32(
    const uint16_t* __restrict__ q, const u32x4* __restrict__ kp, const u32x4* __restrict__ vp,
    const int32_t* __restrict__ sel_count, const int32_t* __restrict__ sel_index, uint16_t* __restrict__ out,
    float* __restrict__ lse, const WorkMap& work, int n_pad, int pad_v, int pad_c, float scale_log2e, float bias_log2e,
    const Split& split, const Thw& thw_rows) {
  constexpr bool THW = std::is_same<Thw, ThwRows>::value;
  constexpr int BLK = 32, KS = D / 16, DT = D / 32, PS = BLK / 16, TILE_CHUNKS = BLK * D / 8, CH = D / 8;
  // one channel tile of every wavefront's O, accumulator order; ROWS: before that, 32 rows of V for every wavefront
  static_assert(!ROWS || D == 64, "32 rows of V take the room of a channel tile");
  __shared__ __align__(1024) float part[NS][16][64];
  __shared__ float stat[NS][2][32];    // reference and sum of every row

  __shared__ uint16_t in_range[RANGE ? 2048 : 1];   // the list's entries in this pass's range, in list order
  __shared__ int wave_entries[RANGE ? NS : 1];

  int bh, i;
  const int range = RANGE ? blockIdx.x / split.stride : 0;
  if (!map_work(RANGE ? blockIdx.x - range * split.stride : blockIdx.x, work, &bh, &i)) return;
  const int M = work.M, M_v = work.M_v;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hl = lane >> 5, ql = lane & 31;
  const size_t qrow = (size_t)bh * n_pad + (size_t)i * BLK + ql;

  bf16x8 qf[KS];
  {
    const u32x4* qp = (const u32x4*)(q + qrow * D);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, qp[2 * ks + hl]);
  }

  int cnt = sel_count[(size_t)bh * M + i];
  cnt = min(max(cnt, 0), M);
  const int32_t* idx = sel_index + ((size_t)bh * M + i) * M;
  if constexpr (RANGE) {
    const int lo = M * range / split.parts, hi = M * (range + 1) / split.parts;
    int kept = 0;
    for (int t0 = 0; t0 < cnt; t0 += 64 * NS) {
      const int t = t0 + threadIdx.x;
      const int jj = t < cnt ? min(max(idx[t], 0), M - 1) : -1;
      const bool in = jj >= lo && jj < hi;
      const uint64_t in_wave = __ballot(in);
      if (lane == 0) wave_entries[wave] = (int)__popcll(in_wave);
      __syncthreads();
      int pos = kept + (int)__popcll(in_wave & ((1ull << lane) - 1ull));
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        pos += s < wave ? wave_entries[s] : 0;
        kept += wave_entries[s];
      }
      if (in) in_range[pos] = (uint16_t)jj;
      __syncthreads();
    }
    cnt = __builtin_amdgcn_readfirstlane(kept);
  }
  const u32x4* kbase = kp + (size_t)bh * M * TILE_CHUNKS + (ROWS ? ql * CH + hl : lane);
  const u32x4* vbase = vp + (size_t)bh * M * TILE_CHUNKS + (ROWS ? 0 : lane);
  u32x4 kf[KS], vf[ROWS ? 1 : DT * PS];
  auto load_k = [&](int j) {
#pragma unroll
    for (int f = 0; f < KS; ++f) kf[f] = kbase[(size_t)j * TILE_CHUNKS + f * (ROWS ? 2 : 64)];
  };
  // ROWS: the 16-byte pieces of a row of V rotated as in attn_h_kernel
  auto v_swizzle = [](int row) { return (row & 2) * 2; };
  const uint32_t v_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)part + (uint32_t)wave * (TILE_CHUNKS * 16));
  const uint32_t v_off = (uint32_t)(lane / CH * CH + (lane % CH ^ v_swizzle(lane / CH))) * 16u;
  const int v_row = 4 * hl + ((lane >> 2) & 3);
  const uint32_t v_lane = v_wave + v_row * (2 * D) + v_swizzle(v_row) * 16 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  auto load_v = [&](int j) {
    if constexpr (ROWS) {
#pragma unroll
      for (int c = 0; c < TILE_CHUNKS / 64; ++c)
        dma_1kb_to_lds_at(vbase + (size_t)j * TILE_CHUNKS + c * 64, v_off, v_wave, c * 1024);
    } else {
#pragma unroll
      for (int f = 0; f < DT * PS; ++f) vf[f] = vbase[(size_t)j * TILE_CHUNKS + f * 64];
    }
  };
  auto listed = [&](int t) {
    return RANGE ? __builtin_amdgcn_readfirstlane((int)in_range[t]) : min(max(idx[t], 0), M - 1);
  };

  float m_run = -INFINITY, l_run = 0.f;
  bool unset = true;   // no row has a reference yet (uniform: every row sees the same keys)
  f32x16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) O[dt][r] = 0.f;

  int j = 0, j_next = 0;   // a list entry is fetched a block ahead of the loads that need it
  if (wave < cnt) {
    j = listed(wave);
    load_k(j);
    load_v(j);
    j_next = listed(min(wave + NS, cnt - 1));
  }
  for (int t = wave; t < cnt; t += NS) {
    const bool more = t + NS < cnt;
    const int j_after = listed(min(t + 2 * NS, cnt - 1));
    f32x16 S;
#pragma unroll
    for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[ks]), qf[ks], S, 0, 0, 0);
    if (more) load_k(j_next);

    const int nv = BLK - (j == M_v - 1 ? pad_v : (j == M - 1 ? pad_c : 0));
    if (nv < BLK) {   // sequence-length mask: pad keys of a ragged block
      asm volatile("");   // a real, rarely taken branch
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r / 4) + 4 * hl + (r % 4) >= nv) S[r] = -INFINITY;
    }
    const float bias = (i < M_v && j >= M_v) ? bias_log2e : 0.f;
    bf16x8 pb[PS];
    auto probabilities = [&](float off) {
      float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
      for (int ps = 0; ps < PS; ++ps) {
        uint32_t w[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(S[8 * ps + 2 * e2], scale_log2e, off));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(S[8 * ps + 2 * e2 + 1], scale_log2e, off));
          w[e2] = pack_bf16x2(p0, p1);
          rs0 += p0;
          rs1 += p1;
        }
        u32x4 pw = {w[0], w[1], w[2], w[3]};
        pb[ps] = __builtin_bit_cast(bf16x8, pw);
      }
      return rs0 + rs1;
    };
    // as in attn_h_kernel: no row maximum while the sums stay in range (P_SUM_MAX); S is still there for the
    // exact path
    float rs = 0.f;
    bool in_range = false;
    if (!unset) {
      rs = probabilities(bias - m_run);
      in_range = __ballot(!(rs <= P_SUM_MAX)) == 0;
    }
    if (!in_range) {
      asm volatile("");   // a real branch: the first block of a row, then almost never
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[r]);
      mx = max_with_other_half(mx);
      const float m_new = fmaxf(m_run, fmaf(mx, scale_log2e, bias));
      const float alpha = m_new == m_run ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
      m_run = m_new;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[dt][r] *= alpha;
      rs = probabilities(m_run == -INFINITY ? 0.f : bias - m_run);   // every key so far was padding: keep it finite
      unset = __ballot(m_run == -INFINITY) != 0;
    }
    l_run += rs;

    if constexpr (ROWS) {
      wait_vmem();   // this wavefront's rows of V have landed
      if (nv < BLK) {   // pad rows hold anything, and their probabilities are zero
        asm volatile("" : : : "memory");
        u32x4* rows = (u32x4*)part + wave * TILE_CHUNKS;
        for (int at = lane; at < TILE_CHUNKS; at += 64)
          if (at / CH >= nv) rows[at] = u32x4{0, 0, 0, 0};
        asm volatile("" : : : "memory");
      }
      static_for<DT / 2>([&](auto G) {   // two channel tiles at a time
        constexpr int g = decltype(G)::value;
        u32x2 A[4][2];
        static_for<4>([&](auto E) {
          constexpr int e = decltype(E)::value, dt = 2 * g + (e & 1), ps = e / 2;
          lds_columns<ps * 32 * D>(A[e][0], v_lane ^ dt * 64);
          lds_columns<ps * 32 * D + 16 * D>(A[e][1], v_lane ^ dt * 64);
        });
        lds_wait(A);
        static_for<4>([&](auto E) {
          constexpr int e = decltype(E)::value, dt = 2 * g + (e & 1), ps = e / 2;
          const u32x4 a = __builtin_shufflevector(A[e][0], A[e][1], 0, 1, 2, 3);
          O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pb[ps], O[dt], 0, 0, 0);
        });
      });
    } else {
#pragma unroll
      for (int ps = 0; ps < PS; ++ps)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[dt * PS + ps]), pb[ps], O[dt],
                                                          0, 0, 0);
    }
    if (more) load_v(j_next);
    j = j_next;
    j_next = j_after;
  }

  // ---- merge the NS partial rows, normalise, store ----
  const float l_wave = l_run + __shfl_xor(l_run, 32, 64);
  if (hl == 0) {
    stat[wave][0][ql] = m_run;
    stat[wave][1][ql] = l_wave;
  }
  __syncthreads();
  float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s) m_all = fmaxf(m_all, stat[s][0][ql]);
  const float ref = m_all == -INFINITY ? 0.f : m_all;
#pragma unroll
  for (int s = 0; s < NS; ++s) l_all += stat[s][1][ql] * __builtin_amdgcn_exp2f(stat[s][0][ql] - ref);
  const int rows_valid = BLK - (i == M_v - 1 ? pad_v : (i == M - 1 ? pad_c : 0));
  const bool row_ok = ql < rows_valid && l_all > 0.f;
  const size_t slot = ((size_t)bh * M + i) * split.parts + range;
  if (RANGE && threadIdx.x < 32) {
    split.stat[(slot * 2) * BLK + ql] = m_all;
    split.stat[(slot * 2 + 1) * BLK + ql] = l_all;
  }
  if (!RANGE && lse != nullptr && threadIdx.x < 32)
    lse[qrow] = row_ok ? (m_all + __builtin_amdgcn_logf(l_all)) * 0.6931471805599453f : -INFINITY;
  // weight of this wavefront's part
  const float mine = RANGE ? __builtin_amdgcn_exp2f(m_run - ref) : row_ok ? __builtin_amdgcn_exp2f(m_run - ref) / l_all : 0.f;
  constexpr int RP = 16 / NS;   // accumulator registers of a channel tile that one wavefront adds up
  uint16_t* trow = nullptr;
  if constexpr (THW) trow = thw_rows.template row<D>(bh, i * BLK + ql);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    if (dt > 0) __syncthreads();   // the previous tile has been read
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][r][lane] = O[dt][r] * mine;
    __syncthreads();
    float sum[RP];
#pragma unroll
    for (int u = 0; u < RP; ++u) {
      sum[u] = 0.f;
#pragma unroll
      for (int s = 0; s < NS; ++s) sum[u] += part[s][wave * RP + u][lane];
    }
    // register r of a channel tile holds channel 8 * (r / 4) + 4 * hl + r % 4
    const int r0 = wave * RP;
    if constexpr (RANGE) {
      float* o = split.o + (((slot * DT + dt) * 4 + r0 / 4) * 64 + lane) * 4 + r0 % 4;
#pragma unroll
      for (int u = 0; u < RP; u += 2) *(float2*)(o + u) = make_float2(sum[u], sum[u + 1]);
      continue;
    }
    const int channel = 32 * dt + 8 * (r0 / 4) + 4 * hl + r0 % 4;
    uint16_t* o = out + qrow * D + channel;
    uint32_t w[RP / 2];
#pragma unroll
    for (int u = 0; u < RP; u += 2) {
      w[u / 2] = row_ok ? pack_bf16x2(sum[u], sum[u + 1]) : 0u;
      *(uint32_t*)(o + u) = w[u / 2];
    }
    if (THW && trow != nullptr) {
#pragma unroll
      for (int u = 0; u < RP; u += 2) *(uint32_t*)(trow + channel + u) = w[u / 2];
    }
  }
}

#define JENGA_ATTN_32_PARAMETERS                                                                                      \
  const uint16_t *__restrict__ q, const u32x4 *__restrict__ kp, const u32x4 *__restrict__ vp,                         \
      const int32_t *__restrict__ sel_count, const int32_t *__restrict__ sel_index, uint16_t *__restrict__ out,       \
      float *__restrict__ lse, WorkMap work, int n_pad, int pad_v, int pad_c, float scale_log2e, float bias_log2e
#define JENGA_ATTN_32_ARGUMENTS \
  q, kp, vp, sel_count, sel_index, out, lse, work, n_pad, pad_v, pad_c, scale_log2e, bias_log2e

template <int D, int NS, bool RANGE>
__global__ __launch_bounds__(64 * NS, (D == 128 ? 2 : 4)) void attn_kernel(JENGA_ATTN_32_PARAMETERS, Split split) {
  attn_32<D, NS, RANGE, false>(JENGA_ATTN_32_ARGUMENTS, split, NoThwRows{});
}
template <int D, int NS>
__global__ __launch_bounds__(64 * NS, (D == 128 ? 2 : 4)) void attn_32_thw_kernel(JENGA_ATTN_32_PARAMETERS, ThwRows thw_rows) {
  attn_32<D, NS, false, false>(JENGA_ATTN_32_ARGUMENTS, Split{}, thw_rows);
}

// K and V in place.
template <int D, int NS, typename Thw>
__global__ __launch_bounds__(64 * NS, 4) void attn_rows_kernel(JENGA_ATTN_32_PARAMETERS, Thw thw_rows) {
  attn_32<D, NS, false, true>(JENGA_ATTN_32_ARGUMENTS, Split{}, thw_rows);
}

// What a launch has to know of the lists' lengths.  One workgroup.
// Lap of the paced walk, common to all workgroups of a launch: a fixed fraction of the time a workgroup needs for
// a list of mean length (a tuning constant: between 0.45 and 0.9 the measured time is flat, at 1.0 and above the
// workgroups run ahead of the sweep and the gain goes).  Writes 2^32 / lap (in ticks of
// the 100 MHz clock) to params[0].
// A queue, if there is one: its counters, and whether it is used, which takes vision lists of `long_list` blocks on average.  The
// plan goes by the length it expects (split_lists), but lists are the caller's: on lists of 2 to 30 blocks counters and cuts cost
// up to 360 us a call.  492 blocks of 64 x 12 heads, D = 64, p = 0.9, lists of 2 / 8 / 30 / 60: with them 218 / 257 / 407 / 617 us,
// lists dealt out in order and whole 45 / 84 / 229 / 435; 736 x 12 likewise at p = 0.5, selected lists of 153 blocks, 3 % faster without.
#ifndef JENGA_PACE_FACTOR
#define JENGA_PACE_FACTOR 0.6f
#endif
__global__ __launch_bounds__(1024) void list_lengths_kernel(const int32_t* __restrict__ sel_count, int n_rows, int M, int M_v,
                                                            float ticks_per_block, uint32_t* __restrict__ params,
                                                            uint32_t* queue, int queue_first, float long_list) {
  __shared__ float part[2][16];
  if (queue != nullptr && threadIdx.x < 8) queue[threadIdx.x] = queue_first;
  float s = 0.f, vision = 0.f;
  for (int t0 = threadIdx.x; t0 < n_rows; t0 += 4096) {   // four loads in flight per thread
    int c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = t0 + u * 1024 < n_rows ? sel_count[t0 + u * 1024] : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float len = (float)min(max(c[u], 0), M);
      s += len;
      if ((t0 + u * 1024) % M < M_v) vision += len;
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    vision += __shfl_xor(vision, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = s;
    part[1][threadIdx.x >> 6] = vision;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float total = 0.f, total_vision = 0.f;
    for (int w = 0; w < 16; ++w) {
      total += part[0][w];
      total_vision += part[1][w];
    }
    const float mean = total / (float)max(n_rows, 1);
    const float lap = fminf(fmaxf(JENGA_PACE_FACTOR * mean * ticks_per_block, 1024.f), 1e9f);
    params[0] = (uint32_t)(4294967296.0 / (double)lap);
    if (queue != nullptr) queue[QUEUE_USED] = total_vision >= long_list * (float)(n_rows / M * M_v);
  }
}

__global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  for (size_t t = (size_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (size_t)gridDim.x * 256) dst[t] = src[t];
}

// Counters of a launch that deals its query blocks out as workgroups become free, and whether the call's lists are long (QUEUE_USED);
// nullptr where the plan does not ask.
uint32_t* attn_queue(const jenga_plan* p, void* ws) {
  return p->attn_long > 0.f ? (uint32_t*)((char*)ws + p->packed_bytes - 256) + PARAM_QUEUE : nullptr;
}

template <int BLK, int D>
int run_pack(const jenga_plan* p, const void* k, const void* v, void* ws, hipStream_t st) {
  const jenga_config& c = p->cfg;
  const jenga_plan_info_t& f = p->info;
  const int bh = c.batch * c.heads;
  const size_t half = (((size_t)bh * f.N_pad * D * 2) + 255) & ~(size_t)255;
  uint4* kp = (uint4*)ws;
  uint4* vp = (uint4*)((char*)ws + half);
  pack_kernel<BLK, D><<<dim3(f.M, bh, 2), 256, 0, st>>>((const uint16_t*)k, (const uint16_t*)v, kp, vp, p->d_blk_valid,
                                                       f.M, f.N_pad);
  return hipGetLastError() == hipSuccess ? JENGA_OK : JENGA_EHIP;
}

template <int BLK, int D, typename Thw>
int run_attention(const jenga_plan* p, const void* q, const void* k, const void* v, void* ws, bool may_split,
                  const int32_t* sel_count, const int32_t* sel_index, void* out, float* lse, Thw thw_rows, hipStream_t st) {
  constexpr bool THW = std::is_same<Thw, ThwRows>::value;
  const jenga_config& c = p->cfg;
  const jenga_plan_info_t& f = p->info;
  const int bh = c.batch * c.heads;
  const size_t half = (((size_t)bh * f.N_pad * D * 2) + 255) & ~(size_t)255;
  const bool k_rows = k != nullptr;
  const u32x4* kp = k_rows ? (const u32x4*)k : (const u32x4*)ws;
  const u32x4* vp = k_rows ? (const u32x4*)v : (const u32x4*)((const char*)ws + half);
  uint32_t* params = (uint32_t*)((char*)ws + 2 * half);
  const float log2e = 1.4426950408889634f;
  const float scale = log2e / sqrtf((float)D), bias = c.text_bias * log2e;
  const uint16_t* qb = (const uint16_t*)q;
  uint16_t* ob = (uint16_t*)out;
  if constexpr (BLK == 32) {   // in-order walk only
    constexpr int NS = D == 128 ? 4 : 8;
    const bool ranges = may_split && p->attn_parts > 1;
    Split split = {};
    if (ranges) {   // the launches share the area of the partial results
      split.parts = p->attn_parts;
      split.o = (float*)((char*)ws + p->packed_bytes);
      split.stat = split.o + (size_t)p->attn_heads * f.M * split.parts * BLK * D;
    }
    const int most = ranges ? p->attn_heads : jenga::heads_per_launch(p, 64 * NS);
    for (int first = 0; first < bh; first += most) {
      const int n = bh - first < most ? bh - first : most;
      const size_t row0 = (size_t)first * f.N_pad, list0 = (size_t)first * f.M;
      const WorkMap work = jenga::plan_work(p, n);
      const uint16_t* q0 = qb + row0 * D;
      const u32x4 *kp0 = kp + row0 * (D / 8), *vp0 = vp + row0 * (D / 8);
      const int32_t *count0 = sel_count + list0, *index0 = sel_index + list0 * f.M;
      uint16_t* ob0 = ob + row0 * D;
      float* lse0 = lse != nullptr ? lse + row0 : nullptr;
      if constexpr (THW) thw_rows.first = first;
      if (ranges) {
        split.stride = (work.n_wg + 7) & ~7;
        attn_kernel<D, NS, true><<<dim3(split.parts * split.stride), 64 * NS, 0, st>>>(
            q0, kp0, vp0, count0, index0, ob0, lse0, work, f.N_pad, f.pad_v, f.pad_c, scale, bias, split);
        merge_kernel<BLK, D><<<dim3(1, f.M, n), 2 * D, 0, st>>>(count0, ob0, lse0, work, f.N_pad, f.pad_v, f.pad_c,
                                                                split, nullptr, thw_rows);
        continue;
      }
      if constexpr (D == 64) {
        if (k_rows) {
          attn_rows_kernel<D, NS><<<dim3(work.n_wg), 64 * NS, 0, st>>>(q0, kp0, vp0, count0, index0, ob0, lse0, work, f.N_pad,
                                                                       f.pad_v, f.pad_c, scale, bias, thw_rows);
          continue;
        }
      }
      if constexpr (THW)
        attn_32_thw_kernel<D, NS><<<dim3(work.n_wg), 64 * NS, 0, st>>>(q0, kp0, vp0, count0, index0, ob0, lse0, work, f.N_pad,
                                                                       f.pad_v, f.pad_c, scale, bias, thw_rows);
      else
        attn_kernel<D, NS, false><<<dim3(work.n_wg), 64 * NS, 0, st>>>(q0, kp0, vp0, count0, index0, ob0, lse0, work, f.N_pad,
                                                                       f.pad_v, f.pad_c, scale, bias, split);
    }
  } else {
    const bool paced = BLK == 128 && (c.flags & JENGA_FLAG_PACED_WALK);
    const WorkMap work = jenga::plan_work(p, bh);
    const bool keys32 = jenga::attn_keys32(p, may_split);
    Split split = {};
    uint32_t *queue = may_split ? attn_queue(p, ws) : nullptr, *pace = nullptr;
#define JENGA_ATTN_H_VALUES \
  qb, kp, vp, sel_count, sel_index, ob, lse, work, f.N_pad, f.pad_v, f.pad_c, scale, bias, pace, split, queue
#define JENGA_ATTN(PACED, SPLIT, K_ROWS, WGS)                                                                    \
  do {                                                                                                           \
    if constexpr (BLK == 64 && D == 128) {                                                                       \
      if (keys32) {                                                                                              \
        if constexpr (THW)                                                                                       \
          attn_keys32_thw_kernel<SPLIT, K_ROWS><<<dim3(WGS), 2 * BLK, 0, st>>>(thw_rows, JENGA_ATTN_H_VALUES);   \
        else                                                                                                     \
          attn_keys32_kernel<SPLIT, K_ROWS><<<dim3(WGS), 2 * BLK, 0, st>>>(JENGA_ATTN_H_VALUES);                 \
        break;                                                                                                   \
      }                                                                                                          \
    }                                                                                                            \
    if constexpr (THW)                                                                                           \
      attn_h_thw_kernel<BLK, D, PACED, SPLIT, K_ROWS><<<dim3(WGS), 2 * BLK, 0, st>>>(thw_rows, JENGA_ATTN_H_VALUES); \
    else                                                                                                         \
      attn_h_kernel<BLK, D, PACED, SPLIT, K_ROWS><<<dim3(WGS), 2 * BLK, 0, st>>>(JENGA_ATTN_H_VALUES);            \
  } while (0)
    if (paced && !(may_split && p->attn_long == 0.f && p->attn_parts > 1)) pace = params;   // parts of short grids: ascending order
    if (pace != nullptr || queue != nullptr) {
      // a workgroup spends about 6.3 us (D = 128; 3.6 us at D = 64) on a block of 128 keys when three share a CU
      list_lengths_kernel<<<1, 1024, 0, st>>>(sel_count, bh * f.M, f.M, f.M_v, D == 128 ? 630.f : 360.f, params, queue,
                                              p->attn_first, p->attn_long);
    }
    const bool dealt = p->attn_long > 0.f || p->attn_text_parts > 1;
    if (may_split && (dealt || p->attn_parts > 1)) {
      int wgs, slots;
      dim3 merge;
      split.o = (float*)((char*)ws + p->packed_bytes);
      if (dealt) {
        if (p->attn_over_kv) split.o = (float*)(k == (const void*)ws ? (char*)ws + half : (char*)ws);
        // where both K and V are packed there all the same, lists stay whole
        split.deal = jenga::plan_deal(p, work, p->attn_over_kv && !k_rows);
        wgs = 8 * split.deal.positions();
        split.first = p->attn_first > 0 ? p->attn_first : split.deal.positions();
        if (p->attn_first > 0) wgs += (wgs + 3) / 4;
        slots = split.deal.slots();
        merge = dim3(BLK / 32, split.deal.text_rows() + split.deal.tail_rows(), 1);
      } else {
        split.parts = p->attn_parts;
        split.chunk = p->attn_chunk;
        split.stride = (work.n_wg + 7) & ~7;   // a multiple of the XCDs, which a query block's parts then share
        wgs = split.parts * split.stride;
        slots = bh * f.M * split.parts;
        merge = dim3(BLK / 32, f.M, bh);
      }
      split.stat = split.o + (size_t)slots * BLK * D;
      if constexpr (BLK == 128) {
        if (paced && k_rows) JENGA_ATTN(true, true, true, wgs);
        else if (paced) JENGA_ATTN(true, true, false, wgs);
      }
      if (k_rows && !paced) JENGA_ATTN(false, true, true, wgs);
      else if (!paced) JENGA_ATTN(false, true, false, wgs);
      if (slots > 0)
        merge_kernel<BLK, D><<<merge, 2 * D, 0, st>>>(sel_count, ob, lse, work, f.N_pad, f.pad_v, f.pad_c, split, queue,
                                                     thw_rows);
      return hipGetLastError() == hipSuccess ? JENGA_OK : JENGA_EHIP;
    }
    if constexpr (BLK == 128) {
      if (paced) JENGA_ATTN(true, false, false, work.n_wg);
    }
    if (k_rows) JENGA_ATTN(false, false, true, work.n_wg);
    else if (!paced) JENGA_ATTN(false, false, false, work.n_wg);
#undef JENGA_ATTN
#undef JENGA_ATTN_H_VALUES
  }
  return hipGetLastError() == hipSuccess ? JENGA_OK : JENGA_EHIP;
}

}  // namespace

namespace jenga {

#define JENGA_FOR_SHAPES(X) X(128, 128) X(64, 128) X(32, 128) X(128, 64) X(64, 64) X(32, 64)

int launch_pack(const jenga_plan* p, const void* k, const void* v, void* ws, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int blk = p->cfg.block, d = p->cfg.head_dim;
#define X(B, DD) \
  if (blk == B && d == DD) return run_pack<B, DD>(p, k, v, ws, st);
  JENGA_FOR_SHAPES(X)
#undef X
  return JENGA_EUNSUPPORTED;
}

int launch_keep(const jenga_plan* p, const void* src, void* ws, int which, const void** copied, void* stream) {
  const size_t bytes = (size_t)p->cfg.batch * p->cfg.heads * p->info.N_pad * p->cfg.head_dim * 2;
  char* dst = (char*)ws + which * ((bytes + 255) & ~(size_t)255);
  copy_kernel<<<2048, 256, 0, (hipStream_t)stream>>>((const uint4*)src, (uint4*)dst, bytes / 16);
  *copied = dst;
  return hipGetLastError() == hipSuccess ? JENGA_OK : JENGA_EHIP;
}

int launch_attention(const jenga_plan* p, const void* q, const void* k, const void* v, void* ws, bool may_split,
                     const int32_t* sel_count, const int32_t* sel_index, void* out, float* lse, void* thw, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int blk = p->cfg.block, d = p->cfg.head_dim;
  const ThwRows rows = {(uint16_t*)thw, p->d_src_of_pos, p->info.N_v + p->cfg.n_text, p->cfg.heads, 0};
#define X(B, DD)                                                                                                      \
  if (blk == B && d == DD)                                                                                            \
    return thw != nullptr                                                                                             \
               ? run_attention<B, DD>(p, q, k, v, ws, may_split, sel_count, sel_index, out, lse, rows, st)            \
               : run_attention<B, DD>(p, q, k, v, ws, may_split, sel_count, sel_index, out, lse, NoThwRows{}, st);
  JENGA_FOR_SHAPES(X)
#undef X
  return JENGA_EUNSUPPORTED;
}

}  // namespace jenga
