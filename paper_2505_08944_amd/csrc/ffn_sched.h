// Work division of an FFN launch (bf16 / fp8 weights): shared by the re-batch,
// which chooses how the last round of tiles is cut, and the FFN kernels, which
// deal the work items.
//
// Tiles are numbered family by family (256, 128, 64 rows).  The first
// `whole` of them -- full rounds of the grid -- are one work item each.  The
// others, a partial round, would leave CUs idle: they are cut, either all into
// column halves or not, and then along K into nsp[family] pieces (at least
// kMinSplitSteps steps each), whose f32 partial sums meet in the workspace.
// Halves need no sums, but read the rows twice.  Items are dealt round by round; odd rounds in
// reverse, so that a workgroup that got one of a round's larger items gets
// one of the next round's smaller ones.
#pragma once

#include "aep_internal.h"

namespace aep {

// A wave-uniform value, in a scalar register whatever unit computed it.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

struct Sched {
  int b1, b2, total;  // first tile of families 1 and 2, and the number of tiles
  int whole, items;
  int full;           // full rounds of items
  bool mixed;         // 256-row tiles beside a sixth as many smaller ones or more
  int halves;         // 2: tail tiles are cut into column halves, 1: not
  int nsp;            // pieces per tail tile or half: family f in bits 4f .. 4f + 3
  __device__ __forceinline__ int first(int f) const { return f == 0 ? 0 : f == 1 ? b1 : f == 2 ? b2 : total; }
  // first tail tile of family f and how many there are
  __device__ __forceinline__ int tail0(int f) const { return max(first(f), whole); }
  __device__ __forceinline__ int tail(int f) const { return max(0, first(f + 1) - tail0(f)); }
  __device__ __forceinline__ int pieces(int f) const { return (nsp >> (4 * f)) & 15; }
  __device__ __forceinline__ int tail_items(int f) const { return tail(f) * halves * pieces(f); }
};

__device__ __forceinline__ void sched_tiles(Sched& s, int t0, int t1, int t2, int nwg) {
  s.b1 = t0;
  s.b2 = t0 + t1;
  s.total = s.b2 + t2;
  s.whole = s.total - uni(s.total % nwg);
  s.items = s.total;
  s.halves = 1;
  s.nsp = 0x111;
}

// -------------------------------------------------------- dealing the items
__device__ __forceinline__ int item_family(const Sched& s, int item) {
  if (item < s.whole) return item < s.b1 ? 0 : (item < s.b2 ? 1 : 2);
  const int j = item - s.whole;
  const int m0 = s.tail_items(0), m1 = s.tail_items(1);
  return j < m0 ? 0 : (j < m0 + m1 ? 1 : 2);
}
// Items of one kind have one tile shape: family and, in bit 2, column halves.
__device__ __forceinline__ int item_kind(const Sched& s, int item) {
  return item_family(s, item) | (item >= s.whole && s.halves == 2 ? 4 : 0);
}

// Work item of workgroup slot lin (XCD-blocked: lin / (nwg / 8) is its XCD)
// in round r, -1 for none.
__device__ __forceinline__ int round_item(const Sched& s, int r, int nwg, int xcd, int xj) {
  const int base = r * nwg;
  const int cnt = s.items - base;
  if (cnt <= 0) return -1;
  const int lin = xcd * (nwg >> 3) + xj;
  const int rl = (r & 1) ? nwg - 1 - lin : lin;
  if (cnt >= nwg) return base + rl;
  // a partial round: over all XCDs, unless the round before it was a mix of
  // families; then the workgroups that had its smaller items come first
  if (r > 0 && item_family(s, base - nwg) != item_family(s, base - 1)) return rl < cnt ? base + rl : -1;
  const int q = (cnt + 7) >> 3;
  const int idx = xcd * q + xj;
  return xj < q && idx < cnt ? base + idx : -1;
}

// The r-th item of workgroup slot (xcd, xj); -1 past its last one.  In a
// mixed launch odd XCDs take their rounds from the last to the first: the
// 256-row tiles, which come first, are bound by the matrix cores and the
// smaller ones by HBM, so the two kinds run side by side instead of one after
// the other (1999 tokens of the fine-grained layer: -4%; all but pure launches
// of large tiles, which share weight bands between the XCDs: +2%).
__device__ __forceinline__ int nth_item(const Sched& s, int r, int nwg, int xcd, int xj) {
  if (!(xcd & 1) || !s.mixed) return round_item(s, r, nwg, xcd, xj);
  const int nr = s.full + (round_item(s, s.full, nwg, xcd, xj) >= 0 ? 1 : 0);
  return r < nr ? round_item(s, nr - 1 - r, nwg, xcd, xj) : -1;
}

// -------------------------------------------------- cutting the last round
// A cut is a number below kCuts: pieces - 1 of family f in bits 3f .. 3f + 2,
// column halves in bit 9.
constexpr int kCutBits = 3;
constexpr int kCuts = 2 << (3 * kCutBits);
static_assert(kMaxSplit == 1 << kCutBits, "pieces of a tile in kCutBits bits");
__device__ __forceinline__ int cut_pieces(int cut, int f) { return 1 + ((cut >> (kCutBits * f)) & (kMaxSplit - 1)); }
__device__ __forceinline__ int cut_halves(int cut) { return 1 + (cut >> (3 * kCutBits)); }

// Time of one K step of a tile or half, and of adding the sums of n pieces, in
// units of 0.01 us.  A step takes longer the more CUs stream weights beside it:
// from the first value, with few of them, to the second, with all.  With the
// weights in HBM, d = 4096, f = 2048, gate/up, a tile per CU: 16 experts of
// 256, 128 and 64 rows 117, 110 and 105 us with bf16 weights, whose streaming
// bounds all heights alike, and 113, 78 and 63 with fp8, whose half as many
// bytes leave a 256-row step to its MFMAs and the widening; 8 experts in halves
// 73, 58 and 55 (fp8 74, 53 and 43), in two pieces of whole tiles 86, 66 and 63
// (76, 51, 44).  Adding 2 to 8 pieces took 17 to 45 us in 256-row tiles and 10
// to 28 in 64-row ones.  The cuts that these constants choose for 844 launches
// of 1 to 32 experts, each timed under all cuts worth trying, were 0.9% slower
// than the best on average.
__device__ __forceinline__ float step_time(bool fp8, int f, int halves, float busy) {
  const int lo = fp8 ? (halves == 1 ? (f == 0 ? 165 : f == 1 ? 70 : 60) : (f == 0 ? 85 : f == 1 ? 65 : 45))
                     : (halves == 1 ? (f == 0 ? 75 : f == 1 ? 70 : 60) : (f == 0 ? 60 : f == 1 ? 45 : 35));
  const int hi = fp8 ? (halves == 1 ? (f == 0 ? 165 : f == 1 ? 100 : 90) : (f == 0 ? 100 : f == 1 ? 65 : 50))
                     : (halves == 1 ? (f == 0 ? 175 : f == 1 ? 150 : 145) : (f == 0 ? 105 : f == 1 ? 80 : 75));
  return (float)lo + (float)(hi - lo) * busy;
}
__device__ __forceinline__ float sums_time(int f, int halves, int n) {
  const int t = f == 0 ? 515 + 325 * n : f == 1 ? 420 + 270 * n : 335 + 195 * n;
  return n == 1 ? 0.f : (halves == 1 ? 1.f : 0.8f) * (float)t;
}
// f32 values of one piece's sums
__device__ __forceinline__ int part_floats(int f, int halves) { return ((kBM * kBN) >> f) / halves; }

// What a cut makes of the last rounds, from the round before the tail on (its
// items may differ in size): where the kinds of items end, and their times.
struct CutRounds {
  int base0, last, items;  // first and last round's first item, items in all
  int w0, w1, end[3];      // last item + 1: whole tiles of families 0 and 1, pieces of each family
  float w[3], c[3], cl[3];  // a whole tile; a piece, in a full round and in the last
  float inv_nwg;
};

// False: the cut is not possible.
__device__ __forceinline__ bool cut_rounds(CutRounds& q, const Sched& s, bool fp8, int nwg, int KT, int64_t split_bytes,
                                           int cut) {
  const int halves = cut_halves(cut);
  int64_t floats = 0;
  q.items = s.whole;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const int n = cut_pieces(cut, f), tl = s.tail(f) * halves;
    if (n > 1 && (tl == 0 || KT < n * kMinSplitSteps)) return false;
    floats += (int64_t)tl * ((n - 1) * part_floats(f, halves));
    q.items += tl * n;
    q.end[f] = q.items;
  }
  if (floats * 4 > split_bytes || q.items - s.whole > 4 * nwg) return false;
  q.inv_nwg = __builtin_amdgcn_rcpf((float)nwg);
  q.base0 = max(0, s.whole - nwg);
  q.last = (int)(((float)q.items - 0.5f) * q.inv_nwg) * nwg;
  q.w0 = min(s.b1, s.whole);
  q.w1 = min(s.b2, s.whole);
  const float busy = (float)(q.items - q.last) * q.inv_nwg;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const int n = cut_pieces(cut, f);
    const float steps = (float)KT * __builtin_amdgcn_rcpf((float)n), sums = sums_time(f, halves, n);
    q.w[f] = step_time(fp8, f, 1, 1.f) * (float)KT;
    q.c[f] = step_time(fp8, f, halves, 1.f) * steps + sums;
    q.cl[f] = step_time(fp8, f, halves, busy) * steps + sums;
  }
  return true;
}

// A workgroup's sum over these rounds, in the order in which items are dealt,
// changes only where one of its rounds passes from one kind of item to the
// next; the workgroups that follow such a passage, and the first, stand for
// all.  This is the sum of the i-th of them (of kCutSlots); the largest is the
// time of the cut.
constexpr int kCutSlots = 8;
__device__ __forceinline__ float cut_load(const CutRounds& q, const Sched& s, int nwg, int i) {
  const int e = i == 1 ? q.w0 : i == 2 ? q.w1 : i == 3 ? s.whole : i == 4 ? q.end[0] : i == 5 ? q.end[1]
              : i == 6 ? q.end[2] : q.base0;
  const int d = max(0, e - q.base0), r = (int)(((float)d + 0.5f) * q.inv_nwg), p = d - r * nwg;
  int at = p == 0 ? 0 : (r & 1) ? nwg - p : p;
  float sum = 0.f;
  for (int base = q.base0; base < q.items; base += nwg) {
    const int it = base + at;
    at = nwg - 1 - at;  // the next round is reversed
    const bool last = base == q.last;
    const float t0 = last ? q.cl[0] : q.c[0], t1 = last ? q.cl[1] : q.c[1], t2 = last ? q.cl[2] : q.c[2];
    const float tw = it < q.w0 ? q.w[0] : it < q.w1 ? q.w[1] : q.w[2];
    const float tp = it < q.end[0] ? t0 : it < q.end[1] ? t1 : it < q.end[2] ? t2 : 0.f;
    sum += it < s.whole ? tw : tp;
  }
  return sum;
}

// (time, cut) in one word: the smallest word is the cut to take, the fewest
// pieces where times are equal.  ~0: no cut.
constexpr uint32_t kNoCut = 0xffffffffu;
__device__ __forceinline__ uint32_t cut_word(float time, int cut) {
  return (uint32_t)min(time, (float)((1 << (31 - 3 * kCutBits)) - 2)) * kCuts + (uint32_t)cut;
}
// Something to gain: a tail, and no small share of many rounds.  (And a counter
// for each half of up to nwg - 1 tiles.)
__device__ __forceinline__ bool cut_pays(const Sched& s, int nwg) {
  return s.whole != s.total && s.whole < 8 * nwg && 2 * nwg <= kSplitCounters;
}

// Takes the cut of a word (kNoCut: none) and settles the rounds.
__device__ __forceinline__ void sched_cut(Sched& s, uint32_t word, int nwg) {
  const int cut = word == kNoCut ? 0 : (int)(word % kCuts);
  s.halves = cut_halves(cut);
  s.nsp = cut_pieces(cut, 0) | cut_pieces(cut, 1) << 4 | cut_pieces(cut, 2) << 8;
  s.items = s.whole + s.tail_items(0) + s.tail_items(1) + s.tail_items(2);
  s.full = uni(s.items / nwg);
  s.mixed = s.b1 > 0 && 6 * (s.total - s.b1) >= s.b1;
}

}  // namespace aep
