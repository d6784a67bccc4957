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
__device__ __forceinline__ int step_time(bool fp8, int f, int halves, int busy, int nwg) {
  const int lo = fp8 ? (halves == 1 ? (f == 0 ? 165 : f == 1 ? 70 : 60) : (f == 0 ? 85 : f == 1 ? 65 : 45))
                     : (halves == 1 ? (f == 0 ? 75 : f == 1 ? 70 : 60) : (f == 0 ? 60 : f == 1 ? 45 : 35));
  const int hi = fp8 ? (halves == 1 ? (f == 0 ? 165 : f == 1 ? 100 : 90) : (f == 0 ? 100 : f == 1 ? 65 : 50))
                     : (halves == 1 ? (f == 0 ? 175 : f == 1 ? 150 : 145) : (f == 0 ? 105 : f == 1 ? 80 : 75));
  return lo + (hi - lo) * busy / nwg;
}
__device__ __forceinline__ int piece_time(bool fp8, int f, int halves, int KT, int n, int busy, int nwg) {
  const int sums = f == 0 ? 515 + 325 * n : f == 1 ? 420 + 270 * n : 335 + 195 * n;
  return step_time(fp8, f, halves, busy, nwg) * KT / n + (n == 1 ? 0 : halves == 1 ? sums : sums * 4 / 5);
}
// f32 values of one piece's sums
__device__ __forceinline__ int part_floats(int f, int halves) { return ((kBM * kBN) >> f) / halves; }

// The time of the last rounds under a cut: the largest sum of one workgroup's
// items, from the round before the tail on (its items may differ in size), in
// the order in which they are dealt.  A workgroup's sum changes only where one
// of its rounds passes from one kind of item to the next, so the slots that
// follow such a passage, and slot 0, stand for all.
__device__ __forceinline__ int cut_time(const Sched& s, bool fp8, int nwg, int KT, int halves, const int (&n)[3]) {
  int end[3], items = s.whole;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    items += s.tail(f) * halves * n[f];
    end[f] = items;
  }
  const int base0 = max(0, s.whole - nwg), last = (items - 1) / nwg * nwg;
  int w[3], c[3], cl[3];  // a whole tile; an item of the tail, in a full round and in the last
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    w[f] = piece_time(fp8, f, 1, KT, 1, nwg, nwg);
    c[f] = piece_time(fp8, f, halves, KT, n[f], nwg, nwg);
    cl[f] = piece_time(fp8, f, halves, KT, n[f], items - last, nwg);
  }
  const int w0 = min(s.b1, s.whole), w1 = min(s.b2, s.whole);
  auto load = [&](int lin) {
    int sum = 0, at = lin;
    for (int base = base0; base < items; base += nwg) {
      const int it = base + at;
      at = nwg - 1 - at;  // the next round is reversed
      if (it < s.whole)
        sum += it < w0 ? w[0] : it < w1 ? w[1] : w[2];
      else if (it < end[0])
        sum += base == last ? cl[0] : c[0];
      else if (it < end[1])
        sum += base == last ? cl[1] : c[1];
      else if (it < end[2])
        sum += base == last ? cl[2] : c[2];
    }
    return sum;
  };
  int worst = load(0);
  const int edge[6] = {w0, w1, s.whole, end[0], end[1], end[2]};
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const int e = edge[i];
    if (e <= base0 || (i > 0 && e == edge[i - 1])) continue;
    const int r = (e - base0) / nwg, at = e - base0 - r * nwg;
    if (at > 0) worst = max(worst, load(r & 1 ? nwg - at : at));
  }
  return worst;
}

// (time, cut) in one word: the smallest word is the cut to take, the fewest
// pieces where times are equal.  ~0: not possible.
constexpr uint32_t kNoCut = 0xffffffffu;
__device__ __forceinline__ uint32_t cut_word(const Sched& s, bool fp8, int nwg, int KT, int64_t split_bytes,
                                             int cut) {
  const int n[3] = {cut_pieces(cut, 0), cut_pieces(cut, 1), cut_pieces(cut, 2)}, halves = cut_halves(cut);
  int64_t floats = 0;
  int items = 0;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const int tl = s.tail(f) * halves;
    if (n[f] > 1 && (tl == 0 || KT < n[f] * kMinSplitSteps)) return kNoCut;
    floats += (int64_t)tl * ((n[f] - 1) * part_floats(f, halves));
    items += tl * n[f];
  }
  if (floats * 4 > split_bytes || items > 4 * nwg) return kNoCut;
  return (uint32_t)min(cut_time(s, fp8, nwg, KT, halves, n), (1 << (31 - 3 * kCutBits)) - 2) * kCuts + (uint32_t)cut;
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
