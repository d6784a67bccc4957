// The device code of k_ffn.hip compiled for the host, with the hardware
// replaced by a recorder: what the tests read off it is the order of its LDS
// accesses and the work division that it picks.  Included after the mock
// below: ffn_device.inc, the part of k_ffn.hip before its host launchers, in
// which every LDS operand read has become lds_read, the direct-to-LDS load
// lds_load and the piece hand-over's flag words LdsFlag (ffn_host.py).
#include <limits.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define address_space(n)
#define __bf16 unsigned short
#define __HIP_MEMORY_SCOPE_AGENT 0

using std::max;
using std::min;
typedef int hipError_t;
typedef void* hipStream_t;
struct uint2 { unsigned x, y; };
struct uint4 { unsigned x, y, z, w; };
struct float4 { float x, y, z, w; };
static inline uint2 make_uint2(unsigned x, unsigned y) { return {x, y}; }
static inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
static inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
static inline float __uint_as_float(unsigned u) { return __builtin_bit_cast(float, u); }
static inline unsigned __float_as_uint(float f) { return __builtin_bit_cast(unsigned, f); }
#define __expf expf
template <typename T>
static T __shfl_xor(T v, int) { return v; }
struct Idx { unsigned x; };
static Idx threadIdx, blockIdx, gridDim;

// ------------------------------------------------------------- the recorder
// One thread at a time runs the whole program.  Barriers are the workgroup's,
// so the number of barriers passed (epoch) orders accesses of different
// waves; within a wave the number of waits and barriers (seq) does.  An operand read is
// known to be complete at the next wait for lgkmcnt 0 (or compiler-made
// barrier, which waits for what the compiler sees), a direct load has landed
// when a wait for vmcnt covers it; vmcnt counts the stores of the epilogue too.
struct Access {
  int wave, word, issue, done, issue_seq, done_seq;  // word: 0 .. 3 of the 16 bytes, -1: all
};
static unsigned char* lds_mem;
static std::vector<std::vector<Access>> reads, writes;  // per 16 bytes of LDS
static int epoch, seq;
static std::vector<std::pair<int, int>> rd_pend, fl_pend;  // chunk, index: incomplete reads, flag writes
static std::vector<std::pair<int, int>> vm;                // outstanding vector memory operations (-1: a store)
static int cnt_word;  // what the piece counter's word reads as

static void begin(std::vector<std::vector<Access>>& all, const void* at, int word,
                  std::vector<std::pair<int, int>>& pend) {
  const int chunk = (int)(((const unsigned char*)at - lds_mem) >> 4);
  all[chunk].push_back({(int)threadIdx.x >> 6, word, epoch, INT_MAX, seq, INT_MAX});
  pend.push_back({chunk, (int)all[chunk].size() - 1});
}
static void finish(std::vector<std::vector<Access>>& all, std::pair<int, int> a) {
  all[a.first][a.second].done = epoch;
  all[a.first][a.second].done_seq = seq;
}
static void reads_done() {
  for (auto a : rd_pend) finish(reads, a);
  rd_pend.clear();
}
static void mock_waitcnt(unsigned imm) {
  const size_t vmcnt = (imm & 15) | ((imm >> 14) & 3) << 4;
  while (vm.size() > vmcnt) {
    if (vm[0].first >= 0) finish(writes, vm[0]);
    vm.erase(vm.begin());
  }
  if (((imm >> 8) & 15) == 0) reads_done();
  ++seq;
}
static void mock_barrier() {
  ++epoch;
  ++seq;
}
static void __syncthreads() {
  reads_done();
  for (auto a : fl_pend) finish(writes, a);
  fl_pend.clear();
  mock_barrier();
}
template <typename T>
static T lds_read(const unsigned char* p) {
  begin(reads, p, -1, rd_pend);
  return T{};
}
static void lds_load(uint32_t lds_addr) { begin(writes, lds_mem + lds_addr + 16 * (threadIdx.x & 63), -1, vm); }
struct LdsFlag {
  int* p;
  explicit LdsFlag(unsigned char* m) : p((int*)m) {}
  struct Ref {
    int* p;
    int word;
    operator int() const {
      begin(reads, p, word, rd_pend);
      return *p;
    }
    void operator=(int v) {
      begin(writes, p, word, fl_pend);
      *p = v;
    }
  };
  Ref operator[](int i) const { return Ref{p + i, i}; }
};

#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_s_waitcnt(v) mock_waitcnt(v)
#define __builtin_amdgcn_s_barrier() mock_barrier()
#define __builtin_amdgcn_sched_barrier(v) ((void)0)
#define __builtin_amdgcn_s_sleep(v) ((void)0)
#define __builtin_amdgcn_s_memtime() 0ull
#define __builtin_amdgcn_s_memrealtime() 0ull
#define __builtin_amdgcn_rcpf(x) (1.f / (x))
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, s, h) (bf16x2_t{})
#define __builtin_amdgcn_make_buffer_rsrc(b, s, n, f) 0
#define __builtin_amdgcn_raw_buffer_store_b128(...) vm.push_back({-1, 0})
#define __builtin_amdgcn_raw_buffer_load_b128(...) (u32x4_t{})
#define __hip_atomic_fetch_add(p, v, o, s) (cnt_word & 15)
#define __hip_atomic_load(p, o, s) (cnt_word)
#define __hip_atomic_store(p, v, o, s) ((void)0)
typedef int __amdgpu_buffer_rsrc_t;
struct Swapped {
  unsigned v[2];
  unsigned operator[](int i) const { return v[i]; }
};
#define __builtin_amdgcn_permlane16_swap(a, b, x, y) (Swapped{{(a), (b)}})

#include "ffn_device.inc"

using namespace aep;

// Two accesses of the same bytes, one or both of them loads, must be apart: one
// complete before the other is issued, and a barrier between the two where
// they are of different waves.  (Loads of one wave land in order.)
static bool ordered(const Access& r, const Access& w) {
  if (r.word >= 0 && w.word >= 0 && r.word != w.word) return true;
  if (r.wave == w.wave) return r.done_seq < w.issue_seq || w.done_seq < r.issue_seq;
  return r.done < w.issue || w.done < r.issue;
}

// The tiles of families 0, 1, 2 in rounds of 8 workgroups: whole[f] rounds of
// whole tiles, then (tail) 4 tiles of every family, in column halves (bit 1 of
// tail), and each of these in two pieces (bit 0).  arrival: this workgroup's
// place among a tile's pieces.  Returns the number of
// unordered pairs, the first of them in `msg`; -1 where waves pass different
// numbers of barriers.
template <bool GATED, bool FP8>
static long order_violations(int KT, const int* whole, int tail, int arrival, int xcd, bool mixed, long* n_reads,
                             char* msg, int msg_n) {
  static std::vector<unsigned char> mem(kFfnLds);
  lds_mem = mem.data();
  reads.assign(kFfnLds / 16, {});
  writes.assign(kFfnLds / 16, {});
  cnt_word = arrival ? 1 | 1 << 4 | 0 << 8 : 0;

  const int nwg = 8;
  Sched sc;
  int tiles[3], all = 0, nwhole = 0;
  for (int f = 0; f < 3; ++f) nwhole += 8 * whole[f];
  // (the tail must be the last tiles, so it is of one family where whole
  // rounds of a later family exist)
  for (int f = 0; f < 3; ++f) tiles[f] = 8 * whole[f];
  if (tail)
    for (int f = 0; f < 3; ++f)
      if (f == 2 || (whole[1] + whole[2] == 0) || (f == 1 && whole[2] == 0)) tiles[f] += 4;
  for (int f = 0; f < 3; ++f) all += tiles[f];
  sched_tiles(sc, tiles[0], tiles[1], tiles[2], nwg);
  sc.whole = nwhole;  // (a tail of more than a round stays one)
  sched_cut(sc, (tail & 1 ? 1 << 6 | 1 << 3 | 1 : 0) | (tail & 2 ? 1 << 9 : 0), nwg);
  sc.mixed = mixed;

  // one group per 4 tiles: 4 columns of tiles, one row tile
  const int cols = 4;
  std::vector<GroupDesc> groups(all / cols);
  std::vector<WeightDesc> wtab(groups.size());
  std::vector<int32_t> tg(all);
  std::vector<uint16_t> scales(2 * cols * kBN);
  for (int t = 0; t < all; ++t) tg[t] = t / cols;
  for (int g = 0; g < (int)groups.size(); ++g) {
    const int t0 = g * cols, f = t0 < sc.b1 ? 0 : t0 < sc.b2 ? 1 : 2;
    groups[g] = GroupDesc{};
    groups[g].n = kBM >> f;
    groups[g].t0[f] = groups[g].t0[3 + f] = t0 - sc.first(f);
    groups[g].nrt[f] = 1;
    wtab[g] = WeightDesc{};
    wtab[g].s_gu = wtab[g].s_down = scales.data();
  }
  int32_t cnt[64] = {};
  float slots[4];
  FfnParams p{};
  p.groups = groups.data();
  p.wtab = wtab.data();
  p.tile_group = tg.data();
  p.split_slots = slots;
  p.split_cnt = cnt;
  p.K = KT * kBK;
  p.n_out = cols * (GATED ? kBN / 2 : kBN);

  int barriers = -1;
  bool uneven = false;
  for (int tid = 0; tid < 512; ++tid) {
    threadIdx.x = (unsigned)tid;
    epoch = seq = 0;
    vm.clear();
    rd_pend.clear();
    fl_pend.clear();
    int r = 0;
    int item = nth_item(sc, r, nwg, xcd, 0);
    while (item >= 0) {
      const int kind = item_kind(sc, item);
      if (kind == 0)
        run_family<GATED, FP8, 0, 2>(p, sc, lds_mem, 0, nwg, xcd, 0, r, item);
      else if (kind == 1)
        run_family<GATED, FP8, 1, 2>(p, sc, lds_mem, 0, nwg, xcd, 0, r, item);
      else if (kind == 2)
        run_family<GATED, FP8, 2, 2>(p, sc, lds_mem, 0, nwg, xcd, 0, r, item);
      else if (kind == 4)
        run_family<GATED, FP8, 0, 1>(p, sc, lds_mem, 0, nwg, xcd, 0, r, item);
      else if (kind == 5)
        run_family<GATED, FP8, 1, 1>(p, sc, lds_mem, 0, nwg, xcd, 0, r, item);
      else
        run_family<GATED, FP8, 2, 1>(p, sc, lds_mem, 0, nwg, xcd, 0, r, item);
    }
    if (barriers >= 0 && epoch != barriers) uneven = true;
    barriers = epoch;
  }
  if (uneven) return -1;
  long bad = 0;
  *n_reads = 0;
  for (size_t c = 0; c < reads.size(); ++c) {
    *n_reads += (long)reads[c].size();
    for (const Access& a : reads[c])
      for (const Access& w : writes[c])
        if (!ordered(a, w) && bad++ == 0)
          snprintf(msg, msg_n, "LDS byte %zu: read by wave %d in slot %d .. %d, loaded by wave %d in slot %d .. %d",
                   c * 16, a.wave, a.issue, a.done, w.wave, w.issue, w.done);
    for (const Access& a : writes[c])
      for (const Access& w : writes[c])
        if (a.wave < w.wave && !ordered(a, w) && bad++ == 0)
          snprintf(msg, msg_n, "LDS byte %zu: loaded by wave %d in slot %d .. %d and by wave %d in slot %d .. %d",
                   c * 16, a.wave, a.issue, a.done, w.wave, w.issue, w.done);
  }
  return bad;
}

// The cut of a launch of these tiles (pieces per family in bits 4f .., column
// halves in bit 12), chosen as the device does.
extern "C" int ffn_cut(int fp8, int t0, int t1, int t2, int nwg, int KT, long split_bytes) {
  Sched s;
  sched_tiles(s, t0, t1, t2, nwg);
  uint32_t word = kNoCut;
  CutRounds q;
  if (cut_pays(s, nwg))
    for (int cut = 0; cut < kCuts; ++cut)
      if (cut_rounds(q, s, fp8, nwg, KT, split_bytes, cut)) {
        float time = 0.f;
        for (int i = 0; i < kCutSlots; ++i) time = max(time, cut_load(q, s, nwg, i));
        word = min(word, cut_word(time, cut));
      }
  sched_cut(s, word, nwg);
  return s.nsp | (s.halves - 1) << 12;
}

// The largest cost of a workgroup in the last rounds under a cut (pieces per
// family in bits 4f .., halves in bit 12): every workgroup, item by item.  -1: a cut that is
// not possible.
extern "C" double ffn_cut_cost(int fp8, int t0, int t1, int t2, int nwg, int KT, long split_bytes, int nsp) {
  Sched s;
  sched_tiles(s, t0, t1, t2, nwg);
  const int halves = 1 + (nsp >> 12);
  long floats = 0, pieces = 0;
  for (int f = 0; f < 3; ++f) {
    const int n = (nsp >> (4 * f)) & 15;
    if (n > 1 && (s.tail(f) == 0 || KT / n < kMinSplitSteps)) return -1;
    floats += (long)s.tail(f) * (n - 1) * (kBM >> f) * kBN;
    pieces += (long)s.tail(f) * halves * n;
  }
  if (4 * floats > split_bytes || pieces > 4 * nwg) return -1;
  s.nsp = nsp & 0xfff;
  s.halves = halves;
  for (int f = 0; f < 3; ++f) s.items += s.tail(f) * (s.pieces(f) * halves - 1);
  const int base0 = max(0, s.whole - nwg);
  std::vector<double> sum(nwg, 0.);
  for (int item = base0; item < s.items; ++item) {
    const int f = item_family(s, item), r = (item - base0) / nwg, at = (item - base0) % nwg;
    const int busy = min(nwg, s.items - item / nwg * nwg), n = s.pieces(f);
    sum[r & 1 ? nwg - 1 - at : at] +=
        item < s.whole ? (double)step_time(fp8, f, 1, 1.f) * KT
                       : (double)step_time(fp8, f, halves, (float)busy / (float)nwg) * KT / n + sums_time(f, halves, n);
  }
  return *std::max_element(sum.begin(), sum.end());
}

extern "C" long ffn_order_violations(int gated, int fp8, int KT, const int* whole, int tail, int arrival, int xcd,
                                     int mixed, long* n_reads, char* msg, int msg_n) {
  auto go = [&](auto fn) { return fn(KT, whole, tail, arrival, xcd, mixed != 0, n_reads, msg, msg_n); };
  if (gated) return fp8 ? go(order_violations<true, true>) : go(order_violations<true, false>);
  return fp8 ? go(order_violations<false, true>) : go(order_violations<false, false>);
}
