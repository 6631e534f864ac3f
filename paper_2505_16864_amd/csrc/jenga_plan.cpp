// Host-side plan: curve permutation, padded layout, adjacency bits.
//
// Sec. 3.1 of the paper: the re-ordering G (Eq. 2) and the masks B_cond and B_adja depend only
// on the resolution, so they are computed once per grid on the host (Alg. 1, "compute block
// reordering and adjacency masks") and kept on the device inside the plan.
//
// The curve restates the published generalized-Hilbert recursion that Sec. 3.1 cites for Eq. 2 (the
// paper only names it); the slab fallback and the choice of the outermost travel axis (longest
// side, ties w, h, t) are this library's.  Equality with the cited project's exact ordering is not
// claimed.  A box with corner p and signed edge vectors A (travel axis), B, C is visited from p
// to the neighbouring corner along A:
//   - two sides of length 1: a straight line;
//   - one side of length 1: the planar rule in the other two axes;
//   - A long (2a > 3b and 2a > 3c): two halves across A;
//   - one side axis clearly longer than the other (3b > 4c or 3c > 4b): three pieces in the
//     plane of A and that axis (out over the first half of A, across, back);
//   - otherwise five pieces along the 8-cell Hilbert path with face-sharing cells merged.
// Cuts are at floor(n/2), raised by one when odd and n > 2.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "jenga_internal.h"

namespace jenga {
namespace {

struct V3 {
  int x[3];
};
inline V3 operator+(V3 a, V3 b) { return {{a.x[0] + b.x[0], a.x[1] + b.x[1], a.x[2] + b.x[2]}}; }
inline V3 operator-(V3 a) { return {{-a.x[0], -a.x[1], -a.x[2]}}; }
inline V3 operator-(V3 a, V3 b) { return a + (-b); }
inline V3 operator*(V3 a, int s) { return {{a.x[0] * s, a.x[1] * s, a.x[2] * s}}; }
inline int length(V3 a) { return std::abs(a.x[0]) + std::abs(a.x[1]) + std::abs(a.x[2]); }
inline int sgn(int v) { return (v > 0) - (v < 0); }
inline V3 unit(V3 a) { return {{sgn(a.x[0]), sgn(a.x[1]), sgn(a.x[2])}}; }
inline int half_cut(int n) {
  int h = n / 2;
  if ((h & 1) && n > 2) ++h;
  return h;
}

struct Walker {
  int H, W;
  int32_t* out;
  size_t n;

  void emit(V3 p) { out[n++] = (int32_t)((p.x[0] * H + p.x[1]) * W + p.x[2]); }

  void line(V3 p, V3 step, int count) {
    for (int i = 0; i < count; ++i) emit(p + step * i);
  }

  // slab: travel axis A (a > 1), side axis B (b > 1), flat axis F (length 1)
  void planar(V3 p, V3 A, V3 B, V3 F) {
    const int a = length(A), b = length(B);
    const V3 dA = unit(A), dB = unit(B);
    const int a2 = half_cut(a), b2 = half_cut(b);
    const V3 A2 = dA * a2, B2 = dB * b2, Ar = dA * (a - a2), Br = dB * (b - b2);
    if (2 * a > 3 * b) {
      box(p, A2, B, F);
      box(p + A2, Ar, B, F);
      return;
    }
    box(p, B2, A2, F);
    box(p + B2, A, Br, F);
    box(p + (A - dA) + (B2 - dB), -B2, -Ar, F);
  }

  void box(V3 p, V3 A, V3 B, V3 C) {
    const int a = length(A), b = length(B), c = length(C);
    const V3 dA = unit(A), dB = unit(B), dC = unit(C);
    if (b == 1 && c == 1) return line(p, dA, a);
    if (a == 1 && c == 1) return line(p, dB, b);
    if (a == 1 && b == 1) return line(p, dC, c);
    if (a == 1) return (b >= c) ? box(p, B, C, A) : box(p, C, B, A);
    if (b == 1) return planar(p, A, C, B);
    if (c == 1) return planar(p, A, B, C);

    const int a2 = half_cut(a), b2 = half_cut(b), c2 = half_cut(c);
    const V3 A2 = dA * a2, B2 = dB * b2, C2 = dC * c2;
    const V3 Ar = dA * (a - a2), Br = dB * (b - b2), Cr = dC * (c - c2);
    const V3 endA = A - dA, endB2 = B2 - dB, endC = C - dC, endC2 = C2 - dC;

    if (2 * a > 3 * b && 2 * a > 3 * c) {
      box(p, A2, B, C);
      box(p + A2, Ar, B, C);
    } else if (3 * b > 4 * c) {
      box(p, B2, C, A2);
      box(p + B2, A, Br, C);
      box(p + endA + endB2, -B2, C, -Ar);
    } else if (3 * c > 4 * b) {
      box(p, C2, A2, B);
      box(p + C2, A, B, Cr);
      box(p + endA + endC2, -C2, -Ar, B);
    } else {
      box(p, B2, C2, A2);
      box(p + B2, C, A2, Br);
      box(p + endB2 + endC, A, -B2, -Cr);
      box(p + endA + B2 + endC, -C, -Ar, Br);
      box(p + endA + endB2, -B2, C2, -Ar);
    }
  }
};

}  // namespace

void curve_order(int T, int H, int W, bool use_curve, std::vector<int32_t>& perm) {
  const size_t n = (size_t)T * H * W;
  perm.resize(n);
  if (!use_curve) {
    for (size_t i = 0; i < n; ++i) perm[i] = (int32_t)i;
    return;
  }
  // outermost travel axis: the longest side; ties prefer w, then h, then t
  struct Side {
    int len, axis, pref;
  } s[3] = {{W, 2, 0}, {H, 1, 1}, {T, 0, 2}};
  std::sort(s, s + 3, [](const Side& l, const Side& r) {
    return l.len != r.len ? l.len > r.len : l.pref < r.pref;
  });
  V3 v[3];
  for (int i = 0; i < 3; ++i) {
    v[i] = {{0, 0, 0}};
    v[i].x[s[i].axis] = s[i].len;
  }
  Walker w{H, W, perm.data(), 0};
  w.box({{0, 0, 0}}, v[0], v[1], v[2]);
}

// Fewer XCDs on a head mean more of the workgroups that share an L2 read the same keys at about the same time: with
// share = 8 and M_v = 234 an XCD's 128 resident workgroups belong to four heads, with share = 1 to one.  So the
// largest share is taken that still gives an XCD enough query blocks of one head to fill it, but the heads that
// are then in flight at once have to stay in the 256 MB last-level cache (720p: a head is 61 MB, and share = 1 costs
// 8 %).  Attention time, launches back to back, at share 8 / 4 / 2 / 1, the rule's choice marked:
//   47 blocks x 16 heads, D = 64            138 / 137 / 132 / 111* us (each XCD also gets its own text rows)
//   220 blocks of 64 x 12 heads, D = 128    511 / 476 / 469 / 472* us
//   260 blocks x 24 heads, D = 128          4.40 / 4.35 / 4.33* / 4.33 ms
//   2032 blocks of 32 x 2 heads, D = 64     0.75* / 0.88 / 0.90 / 0.88 ms
//   929 blocks x 24 heads, D = 128          20.8* / 20.5 / 20.8 / 22.4 ms (k = 0.1)
//
// With few XCDs per head a head with long lists keeps its XCDs busy longer than the others.  Lists have about the same
// length as long as K_top decides it; where the cumulative-probability rule does (p well above k) heads differ, and
// a grid of several generations of workgroups stays at share = 8 (248 blocks x 12 heads, p = 0.9: share = 2 is up to
// 2.3 % slower).
WorkMap plan_work(const jenga_plan* p, int n_bh) {
  const jenga_config& c = p->cfg;
  const int M = p->info.M, M_v = p->info.M_v;
  // workgroups resident on the 32 CUs of an XCD: by registers and LDS 2, 3 to 4 or 6 to 8 per CU
  const int slots_per_xcd = 32 * (c.block == 32 ? 2 : attn_h_per_cu(c.block, c.head_dim));
  const size_t head_kv_bytes = (size_t)p->info.N_pad * c.head_dim * 4;
  WorkMap w;
  const bool even = c.cum_prob <= 2.0 * c.topk_ratio || (long long)n_bh * M <= 8ll * slots_per_xcd;
  w.n_bh = n_bh;
  w.M = M;
  w.M_v = M_v;
  int share = 8;
  while (even && share > 1 && M_v / share < slots_per_xcd &&
         (size_t)(16 / share) * head_kv_bytes <= (size_t)192 << 20)
    share /= 2;
  w.share = share;
  w.log_share = share == 8 ? 3 : share == 4 ? 2 : share == 2 ? 1 : 0;
  w.chunk = (M_v + share - 1) / share;
  w.units = n_bh * w.chunk;
  const int n_text = n_bh * (M - M_v);
  w.text_wgs = share == 8 ? n_text : 8 * ((n_text + 7) / 8);
  const int groups = 8 / share;
  w.n_wg = w.text_wgs + 8 * ((w.units + groups - 1) / groups);
  return w;
}

// A grid has fewer than 2^32 threads in x.
int heads_per_launch(const jenga_plan* p, int threads) {
  int heads = p->cfg.batch * p->cfg.heads;
  while ((long long)plan_work(p, heads).n_wg * threads >= 1ll << 32) heads = (heads + 1) / 2;
  return heads;
}

// Whether the attention kernel cuts the lists of this plan, and where.
//
// With fewer query blocks than resident workgroups the longest lists (the text rows see every block) decide the time:
// a step takes 1.2 us with one workgroup on a CU and 2.3 us with three.  Cut, a list costs about 6 us a part (index
// and Q loads, first tiles, the part's way through memory) and the launch that puts the parts together.  So a part
// gets the length that makes about 0.6 workgroups per place on the chip, six steps of 64 keys at least while there is
// a CU for every query block and 24 from there on; at three quarters of the places lists stay whole.  Attention with
// packing, lists whole -> cut:
//   D = 128, blocks of 128:  18 query blocks 31 -> 23 us, 136 52 -> 44, 368 137 -> 116, 552 171 -> 158; 736 183 -> 191
//   D = 64, blocks of 128:   192 96 -> 54, 384 101 -> 82; 768 131 -> 139
//   D = 128, blocks of 64:   168 35 -> 32, 608 120 -> 97; 1824 202 -> 210
// Lists of about a dozen steps lose what they gain (408 query blocks of 11.6 entries: 75 us whole, 80 us in parts of 8),
// and so do lists that are cut into halves of that length: from 3/8 of the places on nothing is cut where the longest
// list, all blocks, is up to one and a half parts.  Attention with packing, cut -> whole, p = 0.9: 408 query blocks, 17 a head
// 15 % less at D = 64, 12 % at D = 128; 560, 14 a head, D = 64 60.7 -> 55.4 us; 720 of 64 tokens, 30 a head, D = 128 14 % less.
// With fewer query blocks cutting is still the better one (264 of 64 tokens, 33 a head, D = 128: 25 % less).
//
// Blocks of 32 tokens share their list among the wavefronts of a workgroup already; they are read 32 rows at a time, and
// what bounds them is K and V of a head that is larger than an XCD's 4 MB L2.  There the parts are ranges of key blocks,
// one pass each, and every list has them all.  Time in 1 / 2 / 3 / 4 parts, the rule's choice marked:
//   16.8 MB a head (2048 blocks, D = 64, lists of 291)   777 / 598 / 587* / 602 us
//   11.1 MB (678 blocks, D = 128, lists of 138)          319 / 285* / 299 / 309 us
//   6.5 MB (398 blocks, D = 128, lists of 137)           650 / 611* / 633 / 680 us
//   5.0 MB (303 blocks, D = 128, lists of 77)            206* / 221 / 238 / 261 us
//
// The ranges' results take 2 to 3 times as much as K and V of a head.  So that the workspace does not grow with
// batch * heads, a launch takes as many heads as RANGE_AREA_BYTES holds results of (one at least, which is 98 MiB at most), and
// the next launch the next heads in the same area, which then stays in the last-level cache.  Attention with packing,
// all heads in one launch / area of 64 / 128* / 256 / 512 MiB:
//   2048 blocks x 24 heads, D = 128 (2.4 GB)     18.24 / 17.90 / 17.90* / 18.08 / 18.18 ms
//   2048 x 40, D = 64 (2.1 GB)                   12.68 / 12.57 / 12.24* / 12.26 / 12.44 ms
//   708 x 40, D = 128 (0.9 GB)                   3.87 / 3.74 / 3.62* / 3.71 / 3.83 ms
//   408 x 24, D = 128 (0.3 GB)                   1.30 / 1.28 / 1.26* / 1.27 / 1.31 ms
//   1503 x 16, D = 128 (1.2 GB)                  4.97 / 5.00 / 5.01* / 4.84 / 4.87 ms
//
// With more query blocks than resident workgroups, all of about the same length, it is not lists that are too long: at 720p
// XCDs that were dealt the same work took 44 to 49.5 ms for it.  There the query blocks behind the first generation of
// workgroups are dealt out by counters (take_item in jenga_attn.hip), so that XCDs end together: 929 blocks x 24 heads
// 49.3 -> 46.7 ms (k = 0.3, paced) and 21.0 -> 20.1 ms (k = 0.1); 20 shapes of 1.1 to 4.6 generations of 128-token blocks,
// layers of 0.3 to 1.3 ms, 0 to 4 % less, none more.  Workgroups that last less than about 200 us (their blocks at the time a
// block takes on a full chip) lose to the counter and to the cuts.  Layer, as dealt out by map_work -> by counters, on lists of
// 52 us (29 blocks of 64 x 80 heads, D = 128) 204 -> 252 us, 106 us (297 of 64 x 40, D = 64) 1127 -> 1300, 120 us (36 x 48, D = 64)
// 326 -> 358, 150 to 180 us (four shapes) 2 to 4 % more; 200 to 220 us the same, from 260 us on 1 to 14 % less.  At D = 64 the line
// lies higher: four shapes of 205 to 252 us 0.4 to 2.5 % more, 273 us 1 % and from 400 us on 0.3 to 14 % less.  Even lists of
// 64-token blocks last longer than that only where heads are large, and lose 1 to 6 % there too.
// The plan goes by an expected length: K_top and the fixed blocks, or p^2 of all blocks where the cumulative rule decides, an estimate
// for low-frequency activations (their lists hold 0.76 to 0.81 of all blocks at p = 0.9, 0.26 at 0.45, 0.21 to 0.37 at 0.5).  Whether
// lists are dealt out by counters and cut at the end the lists of the call then decide (list_lengths_kernel).
// The first generation is the resident workgroups; of 64 tokens at D = 128 the four a CU of steps of 64 keys, also where steps of 32 leave
// room for six (then the others ask the counter: with all six 0.5 to 0.8 % less on 222 x 24 and x 40, p = 0.9).
// What remains is the last generation, which runs out over the time of one workgroup.  There half a generation of lists is
// cut, into two: 1 to 3 % less from two generations on, but below two, where this reaches into the first one, up to
// 5 % more (1416 query blocks at D = 128 601 -> 633 us).  Lists of uneven length (p well above k) into three, whatever the
// grid: 128 tokens 1 to 13 % less (248 blocks x 12 heads 4.50 -> 4.21 ms), 64 tokens 1 to 10 % less, none more.  With more text
// than vision blocks all vision lists may be cut: 10 grids with 2 to 86 % as many vision as text blocks took 13 % less to 2 % more.
//
// From three quarters of the places on, the lists of the text rows are what can be too long: all blocks, where a vision
// row sees `usual`.  In one generation the fullest CU decides: ceil(rows / 256) workgroups, one of them a text row.
// Cutting text rows adds workgroups, so they get the number of parts with the least load, and none where a CU gets one more
// for it (768 query blocks, 16 of them text: 115 -> 123 us).  With more query blocks a text row is cut where it alone lasts as
// long as the launch.  Attention, whole -> cut: 732 query blocks, 61 a head, D = 128 201 -> 180 us; 972, 81 a head, D = 64
// 183 -> 158; 1104, 138 a head, D = 128 507 -> 498; blocks of 64 at D = 64: 1944, 162 a head 180 -> 137, 8196, 683 a
// head at k = 0.1 1401 -> 1270; 38 shapes 3 % less on average, none above 1 % more.  A text row has to last 400 us for it, beyond
// one generation: with 920 query blocks of 128, 23 a head (145 us), a layer took 241 whole and 250 us cut, 888, 37 a head 211 and 215.
//
// Even lists of blocks of 64 tokens at D = 128 that take steps of 32 keys (attn_keys32): a text row lasts as long as the launch sooner,
// and with one to two generations a cut of 64 lists per XCD at the end evens out how many workgroups the CUs are left with, without
// counters.  It pays where no text row is left whole.  Attention, whole -> text rows cut -> lists at the end too, k = 0.25: 222 blocks x 12 heads
// 486 -> 439 -> 426 us, x 8 416 -> 332 -> 297, 121 x 16 252 -> 222 -> 208, x 13 247 -> 200 -> 175, x 20 271 -> 261 -> 258.  No text: 120 x 14
// 203 -> 186, x 20 245 -> 253.  Lists of 24 blocks: 62 x 32 136 -> 152.  From 2.3 generations on nothing changes (222 x 16, x 24).
// Text rows of less than 110 blocks: 92 x 24 204 -> 206; 62 x 32 137 -> 141.
// The parts of text rows are what a call with short lists of its own waits for: alone on a CU a block takes 1.3 times as long in
// these steps (1.6 us), so there are a third more parts than above, and two where text rows would stay whole, as far as one generation takes
// them and they are no more than an eightieth of the rows (268 x 8, 64 text rows in 4 parts instead of 3, 456 -> 470 us).
// Lists of 1 to 4 blocks, steps of 64 keys / of 32 without this / with it: 222 x 8 103 / 108 / 92 us, 120 x 9 49 / 61 / 52, 300 x 5
// 105 / 136 / 114, 222 x 24 318 / 470 / 258, 492 x 24 778 / 1194 / 659; 160 x 9, whose generation is full, 64 / 81 / 81.  Selected lists are the same to 1 % (120 x 9 102.7 -> 102.9, 222 x 24 716 -> 717, 300 x 16 846 -> 838, 110 x 15
// 122.7 -> 125.1); whole text rows of less than 150 blocks lose 2 % (62 x 60, 92 x 40) and stay whole.
constexpr uint64_t RANGE_AREA_BYTES = 128ull << 20;

Deal plan_deal(const jenga_plan* p, const WorkMap& work, bool whole) {
  Deal d;
  d.text = (work.text_wgs + 7) / 8;
  d.text_parts = whole ? 1 : p->attn_text_parts;
  d.tail = whole ? 0 : p->attn_tail;
  d.parts = d.tail > 0 ? p->attn_parts : 1;
  d.whole = (work.n_wg - work.text_wgs + 7) / 8 - d.tail;
  return d;
}

// Blocks of 64 tokens at D = 128, steps of 32 keys or of 64: six workgroups a CU or four, each slower (attn_h in jenga_attn.hip).  Up to
// 1024 workgroups all are resident in either kind, and those of 64 keys end first; up to 1536 only those of 32 do without a second
// generation; up to 2048 those of 64 have two full ones; from there on the matrix cores are busier with six.  A text row that stays
// whole ends after the others where it has more than 1.5 times the blocks that a place works off in the launch (in one generation 2.2
// times the blocks of a list), and then it counts how fast one workgroup is.  Attention, 64 -> 32 keys a step, k = 0.25:
//   up to 1024:  41 blocks x 8 heads 38.1 -> 41.5 us, 84 x 10 72 -> 78, 300 x 3 248 -> 285, no text 40 x 24 34.0 -> 35.4, 100 x 10 67 -> 70
//   up to 1536:  lists cut into parts 120 x 6 106 -> 103, 305 x 2 218 -> 200, 369 x 2 326 -> 298, 71 x 3 42.3 -> 39.6; no text
//                62 x 20 68 -> 59, 120 x 12 137 -> 115; text rows cut 30 x 40 50.5 -> 44.8, 120 x 9 119 -> 104, 160 x 9 184 -> 153
//   up to 2048:  no text 62 x 28 84 -> 88, 92 x 18 113 -> 118, 40 x 40 60 -> 63; 90 x 20, k = 0.7, 283 -> 297
//   above:       no text 62 x 40 115 -> 108, 120 x 20 196 -> 182, 222 x 16 478 -> 463; 62 x 60 178 -> 171, 222 x 24 776 -> 735, 492 x 24
//                4.41 -> 4.05 ms, text rows cut 222 x 12 402 -> 387
//   text rows whole (packed entry, short text rows, uneven lists): 120 x 12 packed 171 -> 221, 222 x 12 packed 392 -> 464, 62 x 32 106 ->
//                130, 92 x 24 151 -> 187, 222 x 40 at k = 0.05 440 -> 583, 138 x 10 at p = 0.9 209 -> 264
// Lists that p decides about are taken at the K_top that they have at least, from p = 0.7 on at the p^2 of all blocks that they are expected
// to have (98 x 12, p = 0.9, packed, 298 -> 261, 59 x 40 326 -> 303; lists of 0.28 of the blocks all the same 138 x 10 209 -> 264).  Their
// heads are spread over all XCDs (plan_work), and with more than one generation six workgroups a CU then read more of a head's tiles
// past the L2 than four do, except where a list holds most blocks of a head of up to 8 MB.  64 -> 32 keys: p = 0.3, k = 0.1, 220 x 40
// 1319 -> 1456 us, 94 x 40 328 -> 366; p = 0.5 440 x 24 4.28 -> 4.58 ms; p = 0.7 444 x 24 6.78 -> 7.15, 220 x 24 1.96 -> 1.93; p = 0.9 96 x 40
// 921 -> 874 us, 222 x 24 2.61 -> 2.44 ms, 304 x 24 4.76 -> 4.67, 319 x 12 2.36 -> 2.60, 444 x 24 9.75 -> 10.05; one generation: p = 0.3
// 94 x 16 154 -> 135 us, p = 0.5 220 x 6 413 -> 374.
bool attn_keys32(const jenga_plan* p, bool may_cut) {
  const jenga_config& c = p->cfg;
  const jenga_plan_info_t& f = p->info;
  if (c.block != 64 || c.head_dim != 128) return false;
  const long long bh = (long long)c.batch * c.heads, rows = bh * f.M;
  const bool short_grid = p->attn_long == 0.f && p->attn_text_parts == 1 && p->attn_parts > 1;   // all lists are cut
  const bool text_cut = may_cut && (short_grid || p->attn_text_parts > 1), uneven = c.cum_prob > 2.0 * c.topk_ratio;
  const double usual = std::max((double)p->attn_len, c.cum_prob * c.cum_prob * f.M);
  long long wgs = rows, resident = 1024;
  if (may_cut && short_grid) {
    auto parts = [&](double len) { return std::max(1ll, std::min<long long>(p->attn_parts, (long long)std::ceil(len / p->attn_chunk))); };
    wgs = bh * (f.M_v * parts(usual) + f.M_c * parts(f.M));
    if (parts(usual) > 1) resident = 900;   // expected workgroups; those of the longer lists come on top
  } else if (text_cut) {
    wgs += bh * f.M_c * (p->attn_text_parts - 1);
  }
  if (wgs <= resident) return false;
  const bool dense = c.cum_prob >= 0.7;
  if (f.M_c > 0 && !text_cut) {
    const double list = dense ? usual : p->attn_len;
    if (f.M > (wgs <= 1536 ? 2.2 : 1.5 * rows / 1536) * list) return false;
  }
  if (may_cut && !uneven && p->attn_tail > 0) return true;
  if (wgs > 1536 && uneven && (!dense || 4ll * f.N_pad * c.head_dim > 8 << 20)) return false;
  return wgs <= 1536 || wgs > 2048;
}

static void split_lists(jenga_plan* plan) {
  const jenga_config& c = plan->cfg;
  const jenga_plan_info_t& f = plan->info;
  plan->attn_parts = 1;
  plan->attn_first = plan->attn_tail = 0;
  plan->attn_long = 0.f;
  plan->attn_text_parts = 1;
  plan->attn_chunk = f.M;
  plan->attn_heads = c.batch * c.heads;
  const long long rows = (long long)c.batch * c.heads * f.M;
  // expected list length: K_top and the blocks that are always on
  long long fixed = 0;
  for (uint64_t w : plan->fixed_bits) fixed += __builtin_popcountll(w);
  const long long len = std::min<long long>(f.M, f.K_top + (fixed + f.M_v - 1) / f.M_v);
  plan->attn_len = (int)len;
  if (c.block == 32) {
    const long long bytes = 4ll * f.N_pad * c.head_dim;   // K and V of a head
    const int parts = bytes >= 12 << 20 ? 3 : bytes >= 6 << 20 ? 2 : 1;
    if (rows >= 512 && len >= 32 * parts) {
      plan->attn_parts = parts;
      plan->attn_chunk = 0;
      const uint64_t head_bytes = (uint64_t)f.M * parts * 32 * (c.head_dim + 2) * 4;
      const int most = (int)std::max<uint64_t>(1, std::min<uint64_t>(RANGE_AREA_BYTES / head_bytes, 65535));
      const int launches = (plan->attn_heads + most - 1) / most;
      plan->attn_heads = (plan->attn_heads + launches - 1) / launches;
    }
    return;
  }
  const bool b64_d128 = c.block == 64 && c.head_dim == 128, uneven = c.cum_prob > 2.0 * c.topk_ratio, fine_even = b64_d128 && !uneven;
  // What the lists of short grids and uneven ones are cut by.  Five a CU of 64 tokens at D = 128, which take steps of 64 keys there and have
  // four: the rules were measured with it.
  const long long cut_places = 256ll * (b64_d128 ? 5 : attn_h_per_cu(c.block, c.head_dim));
  const long long places = fine_even ? 256ll * attn_h_per_cu(c.block, c.head_dim) : cut_places;
  if (4 * rows >= 3 * cut_places) {
    const WorkMap work = plan_work(plan, c.batch * c.heads);
    const double usual = std::max((double)len, c.cum_prob * c.cum_prob * f.M), gens = (double)rows / places;
    const double block_us = c.block == 128 ? (c.head_dim == 128 ? 6.3 : 3.6) : (c.head_dim == 128 ? 2.6 : 1.8);
    const long long text_rows = (long long)c.batch * c.heads * f.M_c;
    const double long_list = (c.head_dim == 128 ? 200.0 : 320.0) / block_us;
    if (rows > places && (c.block == 128 || uneven) && usual >= long_list) {
      plan->attn_long = (float)long_list;
      plan->attn_first = 32 * (b64_d128 ? 4 : attn_h_per_cu(c.block, c.head_dim));
      if (uneven || rows >= 2 * places) {
        // beyond the first generation, and vision lists: text rows, dealt out first, may be most of the grid
        const int positions = (work.n_wg + 7) / 8, vision = (work.n_wg - work.text_wgs + 7) / 8;
        plan->attn_tail = std::min({positions - plan->attn_first, plan->attn_first / 2, vision});
        plan->attn_parts = uneven ? 3 : 2;
      }
    } else if (fine_even && rows > places && gens < (text_rows > 0 ? 2.25 : 1.3) && usual >= 28) {
      plan->attn_tail = std::min(64, (work.n_wg - work.text_wgs + 7) / 8);
      plan->attn_parts = 2;
    }
    // Text rows may be most of the grid too: as many parts as there is room for beside the lists cut at the end, in the area
    // or where packed K would lie.
    const bool in_place = c.block == 64 || !(c.flags & JENGA_FLAG_PACED_WALK);
    const uint64_t room = std::max<uint64_t>(RANGE_AREA_BYTES, in_place ? (plan->packed_bytes - 256) / 2 : 0);
    const uint64_t part_bytes = (uint64_t)c.block * (c.head_dim + 2) * 4;
    const uint64_t text_slots = room / part_bytes - 8ull * plan->attn_tail * plan->attn_parts;
    const int most = work.text_wgs > 0 && work.text_wgs <= 32768   // rows of a merge
                         ? (int)std::min<uint64_t>(8, text_slots / ((work.text_wgs + 7) / 8 * 8)) : 1;
    if (gens <= 1.0) {
      double least = f.M + ((rows + 255) / 256 - 1) * usual - 384 / c.block;
      for (int parts = 2; parts <= most; ++parts) {
        const double load = std::max((double)f.M / parts, usual) + ((rows + text_rows * (parts - 1) + 255) / 256 - 1) * usual;
        if (load < least) {
          least = load;
          plan->attn_text_parts = parts;
        }
      }
    } else if ((fine_even ? f.M >= 110 : f.M * block_us >= 400.0) && f.M > (gens < 1.5 ? 1.15 : fine_even ? 1.55 : 1.8) * gens * usual) {
      plan->attn_text_parts = std::max(1, std::min(most, (int)std::ceil(f.M / (gens * usual))));
    }
    if (plan->attn_first == 0 && text_rows > 0 && plan->attn_text_parts == 1) {
      plan->attn_tail = 0;
      plan->attn_parts = 1;
    }
    if (f.M >= 110 && text_rows > 0 && (fine_even || attn_keys32(plan, true))) {
      const int parts = plan->attn_text_parts, more = parts > 1 ? parts + (parts + 1) / 3 : f.M >= 150 ? 2 : 1;
      plan->attn_text_parts = std::max(parts, std::min(most, more));
      while (plan->attn_text_parts > parts && (80 * text_rows * (plan->attn_text_parts - parts) > rows ||
                                               (gens <= 1.0 && 8ll * plan_deal(plan, work, false).positions() > places)))
        --plan->attn_text_parts;
      if (!attn_keys32(plan, true)) plan->attn_text_parts = parts;
    }
    if (plan->attn_tail > 0 && plan->attn_first == 0) plan->attn_long = 28.f;
    return;
  }
  const long long shortest = (rows <= 256 ? 6 : 24) * 64 / c.block;
  const long long chunk = std::max(shortest, (5 * rows * len + 3 * cut_places - 1) / (3 * cut_places));
  if (8 * rows >= 3 * cut_places && 2 * f.M <= 3 * chunk) return;
  plan->attn_parts = (int)std::min(std::min(8ll, 2 * cut_places / rows), (f.M + chunk - 1) / chunk);
  plan->attn_chunk = (int)chunk;
}

// Blocks of 32 tokens: packing is a launch of 2.5 us, and reading in place costs more a block.  At head dim 64 attention takes,
// packed / in place: 9 blocks x 2 heads 8.4 / 6.5 us, 14 x 2 8.9 / 7.5, 23 x 3 8.6 / 8.1, 23 x 8 9.0 / 8.7, 44 x 8 15.7 /
// 18.8; at 128 it is never shorter (14 x 2 9.1 / 9.4).
// A plan with the paced walk reads in place where the grid is so short that its lists are cut and visited in ascending order: layer,
// packed / in place, 8 blocks x 12 heads 42.4 / 37.8 us, 40 x 3 78 / 73, 110 x 2 150 / 143.  Paced, the address arithmetic costs
// as much as the packing.
bool reads_kv_in_place(const jenga_plan* p) {
  if (p->cfg.block == 32) return p->cfg.head_dim == 64 && p->info.M <= 24 && p->cfg.batch * p->cfg.heads * p->info.M <= 256;
  const bool short_grid = p->attn_long == 0.f && p->attn_text_parts == 1 && p->attn_parts > 1;
  return p->cfg.block == 64 || !(p->cfg.flags & JENGA_FLAG_PACED_WALK) || short_grid;
}

int build_host_tables(jenga_plan* plan) {
  const jenga_config& c = plan->cfg;
  jenga_plan_info_t& f = plan->info;
  const int m = c.block;
  const long long nv = (long long)c.T * c.H * c.W;
  f.N_v = (int32_t)nv;
  f.M_v = (int32_t)((nv + m - 1) / m);
  f.M_c = (c.n_text + m - 1) / m;
  f.M = f.M_v + f.M_c;
  f.N_pad = f.M * m;
  f.pad_v = f.M_v * m - f.N_v;
  f.pad_c = f.M_c * m - c.n_text;
  // Alg. 3 uses k*M_v as a slice bound without saying how it is rounded: floor, guarded against
  // products such as 0.3*260 that land a hair below an integer, and never less than one block.
  f.K_top = f.M_v > 0 ? std::max(1, (int)std::floor(c.topk_ratio * f.M_v + 1e-6)) : 0;
  plan->nt64 = (f.M + 63) / 64;

  curve_order(c.T, c.H, c.W, (c.flags & JENGA_FLAG_CURVE) != 0, plan->perm);
  plan->inv_perm.assign(f.N_v, 0);
  for (int i = 0; i < f.N_v; ++i) plan->inv_perm[plan->perm[i]] = i;

  plan->src_of_pos.assign(f.N_pad, -1);
  for (int i = 0; i < f.N_v; ++i) plan->src_of_pos[i] = plan->perm[i];
  for (int i = 0; i < c.n_text; ++i) plan->src_of_pos[(size_t)f.M_v * m + i] = f.N_v + i;

  plan->blk_valid.assign(f.M, m);
  if (f.M_v > 0) plan->blk_valid[f.M_v - 1] = m - f.pad_v;
  if (f.M_c > 0) plan->blk_valid[f.M - 1] = m - f.pad_c;

  // fixed bits of query block i: text key blocks (condition mask) and blocks holding a token
  // within Chebyshev distance 1 of one of i's tokens (adjacency mask, 26-neighbourhood + self)
  plan->fixed_bits.assign((size_t)f.M_v * plan->nt64, 0);
  auto set_bit = [&](int i, int j) { plan->fixed_bits[(size_t)i * plan->nt64 + (j >> 6)] |= 1ull << (j & 63); };
  if (c.flags & JENGA_FLAG_CONDITION)
    for (int i = 0; i < f.M_v; ++i)
      for (int j = f.M_v; j < f.M; ++j) set_bit(i, j);
  if (c.flags & JENGA_FLAG_ADJACENCY) {
    for (int t = 0; t < c.T; ++t)
      for (int h = 0; h < c.H; ++h)
        for (int w = 0; w < c.W; ++w) {
          const int bi = plan->inv_perm[((size_t)t * c.H + h) * c.W + w] / m;
          for (int dt = -1; dt <= 1; ++dt) {
            const int t2 = t + dt;
            if (t2 < 0 || t2 >= c.T) continue;
            for (int dh = -1; dh <= 1; ++dh) {
              const int h2 = h + dh;
              if (h2 < 0 || h2 >= c.H) continue;
              for (int dw = -1; dw <= 1; ++dw) {
                const int w2 = w + dw;
                if (w2 < 0 || w2 >= c.W) continue;
                set_bit(bi, plan->inv_perm[((size_t)t2 * c.H + h2) * c.W + w2] / m);
              }
            }
          }
        }
  }

  // workspaces
  const uint64_t bh = (uint64_t)c.batch * c.heads;
  auto align256 = [](uint64_t x) { return (x + 255) & ~255ull; };
  // select: pooled Q [bh][M_v][d] f64, pooled K [bh][M][d] f64; the third term was room for scores [bh][M_v][M] f64, which
  // stay in LDS now: it is kept so that what jenga_select_blocks_static takes and refuses stays as documented
  f.select_workspace_bytes = align256(bh * f.M_v * c.head_dim * 8) + align256(bh * f.M * c.head_dim * 8) +
                             align256(bh * (uint64_t)f.M_v * f.M * 8);
  // attention: K and V re-tiled, bf16, one tile per (batch, head, block)
  plan->packed_bytes = 2 * align256(bh * (uint64_t)f.N_pad * c.head_dim * 2) + 256;   // packed K, packed V, launch parameters
  f.attn_workspace_bytes = plan->packed_bytes;
  split_lists(plan);
  // and, where lists are cut, O and two statistics per row and part, float32
  const bool dealt = plan->attn_long > 0.f || plan->attn_text_parts > 1;
  const uint64_t slots = dealt                  ? plan_deal(plan, plan_work(plan, (int)bh), false).slots()
                         : plan->attn_parts > 1 ? (uint64_t)plan->attn_heads * f.M * plan->attn_parts
                                                : 0;
  const uint64_t parts = align256(slots * m * (c.head_dim + 2) * 4);
  plan->attn_over_kv = dealt && reads_kv_in_place(plan) && parts <= (plan->packed_bytes - 256) / 2;
  if (!plan->attn_over_kv) f.attn_workspace_bytes += parts;
  return JENGA_OK;
}

}  // namespace jenga
