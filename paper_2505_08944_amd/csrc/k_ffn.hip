// Ragged grouped SwiGLU expert FFN (the contraction hot spot of a drained
// layer).  Two persistent launches per batch:
//
//   gate/up:  h[r, c] = silu(x_r . W_gate[c]) * (x_r . W_up[c])   (K = d)
//   down:     y[r, c] = h_r . W_down[c]                            (K = f)
//
// bf16 / fp8-weight path: 512-thread workgroups, one per CU, K step 64, tiles
// of 256 columns (gate/up: 128 features of W_gate and the same 128 of W_up)
// and 256, 128 or 64 rows.  The plan kernel covers a group's rows with full
// 256-row tiles and one remainder tile of the smallest height that holds the
// rest, so an expert's weights are read ceil(rows / 256) times.  It lays the
// tiles of all groups end to end, family by family; this kernel deals them to
// the workgroups, those of the last, partial round in column halves, K pieces
// or both (ffn_sched.h).
//
// Ping-pong.  The eight waves form two groups of four; a SIMD runs one wave
// of each.  A workgroup barrier ends every slot, and in a slot one group
// issues the MFMAs of its next phase while the other reads that phase's
// operands from LDS and issues the direct-to-LDS loads of a later K step; the
// next slot swaps the roles.  The matrix cores therefore always have a wave
// with its operands in registers, and the memory slot's latencies hide behind
// the other group's MFMAs.  One expert of 8192 rows (d = 4096, f = 14336, whole
// rounds of tiles, launches back to back): 2600 / 2500 cycles per K step in
// gate/up / down, prologues and epilogues included, against the 2048 its MFMAs
// take, at 1.8 GHz; a card that held 1.5 - 1.65 GHz took 2220 / 2144 cycles,
// the same 1.4 us, so neither the clock nor the cycles bound it alone.  One wave
// per SIMD (four waves of 128 x 128, the operand reads and refills spread
// between the MFMAs) took about 3000 cycles there.  The shader clock under this
// load is what the power limit leaves, so the MFMA shape matters: 32x32x16
// (twice the accumulator traffic per operation) ran at 1.3 - 1.4 GHz on the
// card where 16x16x32 ran at 1.5 - 1.6.
//
// f32 path (f32 activations and weights): 64 x 64 tiles of 32 x 32 f32 MFMA
// blocks, operands straight from global memory.
#include <limits.h>

#include <algorithm>

#include "aep_device.h"
#include "ffn_sched.h"

namespace aep {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2v_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

struct FfnParams {
  const GroupDesc* groups;
  const WeightDesc* wtab;
  const int32_t* tile_totals;
  const uint32_t* cut;        // how the last round is cut (written with the re-batch)
  const int32_t* tile_group;  // group of each tile of this launch (written by the plan)
  float* split_slots;         // split-K partial sums
  int32_t* split_cnt;         // pieces finished per tile (zero between launches)
  const void* a;  // x_perm (gate/up) or h (down)
  void* out;      // h (gate/up) or y (down)
  int K;      // reduction length: d (gate/up) or f (down)
  int n_out;  // output columns: f (gate/up) or d (down)
  unsigned long long* clk;  // clock probe (nullptr: off)
  int clk_n;
};


typedef __attribute__((address_space(3))) void* lds_vptr;

// A raw buffer resource over [base, base + bytes): stride 0, 32-bit data
// format, every access bounds-checked against bytes (an access past the end
// reads zeros without touching memory and writes nothing).  Its words are
// kept apart, as scalars, and only put together where a load uses them.
typedef int i32x4_t __attribute__((ext_vector_type(4)));
struct Rsrc {
  int lo, hi, bytes;
  __device__ __forceinline__ i32x4_t words() const { return i32x4_t{lo, hi, bytes, 0x00020000 /* data format 32 */}; }
};
__device__ __forceinline__ Rsrc make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  return Rsrc{__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
              __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu)),
              __builtin_amdgcn_readfirstlane((int)bytes)};
}

// Tables of earlier launches (plan, weights), read through the scalar cache:
// a vector load would be waited for together with every direct-to-LDS load in
// flight, which drains the operand ring at each tile (vmcnt counts both).
template <typename T>
using const_ptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ const_ptr<T> as_const(const T* p) {
  return (const_ptr<T>)(uintptr_t)p;
}

// One direct buffer -> LDS load: lane l reads the 16 bytes at byte offset
// voff + soff of the resource and writes them to lds_addr + 16 * l (M0 holds
// lds_addr).  Issued through inline asm so that the compiler does not see an
// LDS write it cannot disambiguate (it would otherwise wait for every
// outstanding load before each LDS read); the kernel orders these loads
// itself with wait_vmcnt + barriers.  Nor does the compiler see to the wait
// states that such a load needs: one after the write of M0 (here), five after
// a vector instruction writes one of its scalar registers.  Waiting for these
// here as well (s_nop 3) cost 2 - 3% of large launches; test_ffn_waits_host.py
// follows every path into every load of the built code instead.
__device__ __forceinline__ void dload16(i32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds_addr) {
  // (one wait state between the write of M0 and its use)
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc),
               "s"(soff), "s"(__builtin_amdgcn_readfirstlane(lds_addr))
               : "memory", "m0");
}

// s_waitcnt with only vmcnt (or only lgkmcnt) constrained (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
}
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xf | (3 << 14) | (0x7 << 4)); }

// Workgroup barrier that orders nothing but the instruction stream: the
// waits before it are explicit.
__device__ __forceinline__ void slot_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Tile order inside one group's nrow x ncol grid of 256-row tiles: panels of
// PANEL column tiles, row tiles one after another inside a panel, the
// columns of a row tile adjacent.  An XCD gets runs of 32 consecutive tiles,
// so it works on a compact block of tiles (4 x 8 for gate/up, 8 x 4 for
// down): per K step its L2 sees a few row bands of A and column bands of B.
// Panels of 4 measured 1-4% faster in the down launch (few column tiles,
// long K), panels of 8 in gate/up.
template <int PANEL>
__device__ __forceinline__ void panel_decode(int local, int nrow, int ncol, int& rt, int& ct) {
  const int per = PANEL * nrow;
  const int pi = local / per;
  const int within = local - pi * per;
  const int w = min(PANEL, ncol - pi * PANEL);  // the last panel may be narrower
  rt = within / w;
  ct = pi * PANEL + (within - rt * w);
}

// One work item: `rows` rows of a group from row y_row0 (h and y) / x_row0
// (x_perm) on, column tile nti, K steps [k0, k0 + kn).
struct Item {
  int g, nti, rows, y_row0, kn;  // what the epilogue needs
  int x_row0, k0, rot;           // what the load stream needs as well
};
// Where a tail tile's item stands among its pieces.
struct Piece {
  int n, piece, cnt;  // pieces, this one, their counter
  int64_t slot;       // float offset of their partial sums
  int tile, half;     // half: column half of the tile (0 if it is not cut)
};

__device__ __forceinline__ Piece decode_piece(const Sched& s, int item, int f) {
  Piece q{1, 0, 0, 0, item, 0};
  if (item < s.whole) return q;
  int j = item - s.whole;
  int64_t slot = 0;
#pragma unroll
  for (int e = 0; e < 2; ++e)
    if (f > e) {
      j -= s.tail_items(e);
      q.cnt += s.tail(e) * s.halves;
      slot += (int64_t)s.tail(e) * s.halves * (s.pieces(e) - 1) * part_floats(e, s.halves);
    }
  q.n = s.pieces(f);
  const int ti = q.n == 1 ? j : uni(j / q.n);
  q.piece = j - ti * q.n;
  q.tile = s.tail0(f) + (s.halves == 2 ? ti >> 1 : ti);
  q.half = s.halves == 2 ? ti & 1 : 0;
  q.cnt += ti;
  q.slot = slot + (int64_t)ti * (q.n - 1) * part_floats(f, s.halves);
  return q;
}

template <bool GATED, int FAM, int NB>
__device__ __forceinline__ Item decode_item(const FfnParams& p, const Sched& s, int item, int ncol, int KT) {
  constexpr int f = FAM;
  const Piece q = decode_piece(s, item, f);
  Item it;
  it.k0 = q.n == 1 ? 0 : uni(q.piece * KT / q.n);
  it.kn = q.n == 1 ? KT : uni((q.piece + 1) * KT / q.n) - it.k0;
  it.g = uni(as_const(p.tile_group)[q.tile]);
  const const_ptr<GroupDesc> gd = as_const(p.groups) + it.g;
  const int local = q.tile - s.first(f) - gd->t0[(GATED ? 0 : 3) + f];
  int m0;
  if (f == 0) {
    int rt;
    panel_decode<GATED ? 8 : 4>(local, gd->nrt[0], ncol, rt, it.nti);
    m0 = rt * kBM;
  } else {
    it.nti = local;
    m0 = gd->row1;
  }
  if (f == 0 && NB == 2) {
    it.rot = 0;
  } else {
    // Smaller tiles stream weights: tiles that run together start their K
    // walk at different steps, so they do not read the same DRAM channels
    // in lockstep (a load-only probe: 0.68 -> 0.79 of peak bandwidth).
    // 256-row tiles share bands with their neighbours in an XCD's L2, which
    // a rotation would pull apart.
    it.rot = uni((int)((7u * (unsigned)(q.tile + q.half)) % (unsigned)it.kn));
  }
  if (NB == 1) it.nti = 2 * it.nti + q.half;
  it.rows = uni(gd->n - m0);
  it.x_row0 = uni(gd->x_row0 + m0);
  it.y_row0 = uni(gd->y_row0 + m0);
  it.nti = uni(it.nti);
  return it;
}

// ------------------------------------------------------------- tile families
// A K step's LDS stage holds the A rows (128 bytes each) in units of up to
// 128 rows (256 where there is one B unit), then NB B units of 128 rows (128
// bytes each, 64 for fp8): two in a whole tile, one in a column half.  B unit
// b, rows 32w .. 32w + 31 belong to wave column w: gate/up: 16 gate features
// and the same 16 up features (tile features 16 NB w + 16 b ...), so a lane
// holds both accumulators of an output; down: 32 output columns.
// 16-byte chunk c of row r sits at position c ^ (r % 8) (fp8 B rows: c ^
// ((r / 4) % 4)), which spreads the rows one read covers over the banks; the
// loader lanes fetch the chunk that belongs at their fixed LDS position.
template <bool FP8, int FAM, int NB>
struct Fam {
  static constexpr int kRows = kBM >> FAM;
  static constexpr bool kFour = FAM == 0 && NB == 2;     // four phases per K step, else one
  static constexpr int kUnits = kFour ? 2 : 1;           // A units per stage
  static constexpr int kUnitRows = kRows / kUnits;       // 128, 128, 64; of halves 256, 128, 64
  static constexpr int RF = kUnitRows / 32;              // 16-row fragments per wave and unit
  static constexpr int kA = kUnitRows * 128;             // bytes of an A unit
  static constexpr int kB = 128 * (FP8 ? 64 : 128);      // bytes of a B unit
  static constexpr int kStage = kUnits * kA + NB * kB;
  // ring depth: what fits 160 KB
  static constexpr int kStages = NB == 2 ? (FAM == 0 ? (FP8 ? 3 : 2) : FAM == 1 ? (FP8 ? 5 : 3) : (FP8 ? 6 : 4))
                                         : (FAM == 0 ? (FP8 ? 4 : 3) : FAM == 1 ? (FP8 ? 6 : 5) : (FP8 ? 8 : 6));
  static constexpr int kCols = kBN / 2 * NB;             // B rows: output columns, or gate and up features
  static constexpr int kLA = kUnitRows / 64;             // loads per wave: an A unit
  static constexpr int kLB = FP8 ? 1 : 2;                // ... and a B unit
  static_assert(kStages * kStage <= kFfnLds, "the ring fits the LDS");
};

// The load stream: which item's which K step the next stage is filled from.
// It runs kStages steps ahead of the MFMAs, across items.
struct Stream {
  Rsrc a, b;
  int k, k0, kend, left;
  __device__ __forceinline__ void next() {
    --left;
    k = k + 1 == kend ? k0 : k + 1;
  }
};

template <bool GATED, bool FP8, int FAM, int NB>
__device__ __forceinline__ void stream_set(Stream& st, const FfnParams& p, const Item& it, int wave) {
  const int K = p.K;
  const const_ptr<WeightDesc> wd = as_const(p.wtab) + it.g;
  const uint16_t* a = reinterpret_cast<const uint16_t*>(p.a) + (int64_t)(GATED ? it.x_row0 : it.y_row0) * K;
  // rows past the group's end and columns past the matrix are out of the
  // resources' range: they read as zeros, cost no traffic, and their outputs
  // are not stored
  st.a = make_rsrc(a, (uint32_t)min(it.rows, Fam<FP8, FAM, NB>::kRows) * (uint32_t)K * 2u);
  const unsigned char* w =
      reinterpret_cast<const unsigned char*>(GATED ? ((wave & 1) ? wd->up : wd->gate) : wd->down);
  // (the second half of the last tile may lie past the matrix)
  const int c0 = min(it.nti * (Fam<FP8, FAM, NB>::kCols / (GATED ? 2 : 1)), p.n_out);
  constexpr uint32_t esz = FP8 ? 1u : 2u;
  st.b = make_rsrc(w + (int64_t)c0 * K * esz, (uint32_t)(p.n_out - c0) * (uint32_t)K * esz);
  st.k0 = it.k0;
  st.kend = it.k0 + it.kn;
  st.k = it.k0 + it.rot;
  st.left = it.kn;
}
__device__ __forceinline__ void stream_null(Stream& st) {
  // every lane is out of range (the scalar offset stays 0): no traffic
  st.a.bytes = 0;
  st.b.bytes = 0;
  st.k = st.k0 = 0;
  st.kend = 1;
  st.left = INT_MAX;
}

// Runs the chain of items of family FAM and NB B units that starts at round r
// of this workgroup (whose item is `item`); leaves r and item at the first one
// of another kind (item < 0: none left).
template <bool GATED, bool FP8, int FAM, int NB>
__device__ __forceinline__ void run_family(const FfnParams& p, const Sched& sc, unsigned char* smem,
                                           uint32_t lds_base, int nwg, int xcd, int xj, int& r, int& item) {
  using F = Fam<FP8, FAM, NB>;
  constexpr bool kFour = F::kFour;
  constexpr int kOut = F::kCols / (GATED ? 2 : 1);  // output columns of an item
  constexpr int RF = F::RF, NU = F::kUnits, NST = F::kStages;
  int tid = threadIdx.x;
  // per-lane offsets are recomputed here instead of being kept live across
  // the other families' loops
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1, grp = wave >> 2;
  const int rr = lane & 15, hh = lane >> 4;
  const int K = p.K, KT = K / kBK, n_out = p.n_out;
  const int ncol = (n_out + (GATED ? kBN / 2 : kBN) - 1) / (GATED ? kBN / 2 : kBN);

  // loader offsets: the same for every tile (the resources move)
  uint32_t aoff[NU][F::kLA], boff[NB][F::kLB];
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int i = 0; i < F::kLA; ++i) {
      const int row = (wave * F::kLA + i) * 8 + (lane >> 3);
      aoff[u][i] = (uint32_t)(u * 128 + row) * (uint32_t)K * 2u + (uint32_t)(((lane & 7) ^ (lane >> 3)) << 4);
    }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < F::kLB; ++i) {
      const int lr = wave * 16 + (FP8 ? (lane >> 2) : i * 8 + (lane >> 3));
      const int c = FP8 ? ((lane & 3) ^ ((lr >> 2) & 3)) : ((lane & 7) ^ (lr & 7));
      const int col = GATED ? (wave >> 1) * (16 * NB) + b * 16 + (lr & 15) : b * 128 + lr;
      boff[b][i] = (uint32_t)col * (uint32_t)K * (FP8 ? 1u : 2u) + (uint32_t)(c << 4);
    }
  const uint32_t la = lds_base + wave * (F::kLA * 1024), lb = lds_base + NU * F::kA + wave * (F::kLB * 1024);

  Stream st;
  auto load_a = [&](int u, int stage) {
#pragma unroll
    for (int i = 0; i < F::kLA; ++i)
      dload16(st.a.words(), aoff[u][i], (uint32_t)st.k * 128u, la + stage * F::kStage + u * F::kA + i * 1024);
  };
  auto load_b = [&](int b, int stage) {
#pragma unroll
    for (int i = 0; i < F::kLB; ++i)
      dload16(st.b.words(), boff[b][i], (uint32_t)st.k * (FP8 ? 64u : 128u), lb + stage * F::kStage + b * F::kB + i * 1024);
  };

  // operands of one phase, and the accumulators [A unit][B unit][row
  // fragment][column fragment]: rows of the MFMA result are columns of the
  // output, so a lane holds four consecutive output columns of one row.
  // rn: a B unit as read; it becomes rb[b] in widen(b) -- for fp8 weights by
  // the exact conversion of its bytes, and with four phases for B unit 0 because
  // the last phase of a step still multiplies by rb[0] while the next step's
  // unit is read.
  bf16x8_t ra[RF][2], rb[NB][2][2];
  uint4 rn[FP8 && !kFour ? NB : 1][2][FP8 ? 1 : 2];
  f32x4_t acc[NU][NB][RF][2];
  const int wrow = wm * (F::kUnitRows / 2) + rr;
  auto read_a = [&](int u, int stage) {
    const unsigned char* q = smem + stage * F::kStage + u * F::kA + wrow * 128;
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        // fp8: a lane's 16 weight bytes are 16 consecutive k, so its two
        // activation chunks are consecutive too
        const int c = FP8 ? 2 * hh + k : 4 * k + hh;
        ra[i][k] = *reinterpret_cast<const bf16x8_t*>(q + i * 2048 + ((c ^ (rr & 7)) << 4));
      }
  };
  // b = 2: unit 0, kept aside
  auto read_b = [&](int b, int stage) {
    const unsigned char* q = smem + stage * F::kStage + NU * F::kA + (b & 1) * F::kB;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int lr = wn * 32 + j * 16 + rr;
      if constexpr (FP8) {
        rn[kFour ? 0 : b][j][0] = *reinterpret_cast<const uint4*>(q + lr * 64 + ((hh ^ ((rr >> 2) & 3)) << 4));
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const uint4 v = *reinterpret_cast<const uint4*>(q + lr * 128 + (((4 * k + hh) ^ (rr & 7)) << 4));
          if (b == 2)
            rn[0][j][k] = v;
          else
            rb[b][j][k] = __builtin_bit_cast(bf16x8_t, v);
        }
      }
    }
  };
  auto widen = [&](int b) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (FP8) {
        const uint4 v = rn[kFour ? 0 : b][j][0];
        const uint2 w0 = e4m3x4_to_bf16x4(v.x), w1 = e4m3x4_to_bf16x4(v.y);
        const uint2 w2 = e4m3x4_to_bf16x4(v.z), w3 = e4m3x4_to_bf16x4(v.w);
        rb[b][j][0] = __builtin_bit_cast(bf16x8_t, make_uint4(w0.x, w0.y, w1.x, w1.y));
        rb[b][j][1] = __builtin_bit_cast(bf16x8_t, make_uint4(w2.x, w2.y, w3.x, w3.y));
      } else if (kFour && b == 0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) rb[0][j][k] = __builtin_bit_cast(bf16x8_t, rn[0][j][k]);
      }
    }
  };
  auto mma = [&](int u, int b) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[u][b][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rb[b][j][k], ra[i][k], acc[u][b][i][j], 0, 0, 0);
  };

  Item cur = decode_item<GATED, FAM, NB>(p, sc, item, ncol, KT), nxt = cur;
  bool split = cur.kn < KT;  // a piece of a tile
  bool has_next = false;     // the stream has moved on to nxt, item nitem
  int nitem = -1;
  stream_set<GATED, FP8, FAM, NB>(st, p, cur, wave);

  __syncthreads();
  int stage = 0;  // stage of the K step being computed
  // Loads in flight after the wait of a phase.  Four phases per step: those of
  // the last 4 * NST - 2 phases; else NST - 2 steps.
  constexpr int kFlight = kFour ? (2 * NST - 1) * (F::kLA + F::kLB) : (NST - 2) * (F::kLA + NB * F::kLB);
  static_assert(kFlight < 64, "vmcnt range");
  constexpr int kAhead = kFour ? NST : NST - 1;  // steps the stream is ahead
  for (int s = 0; s < kAhead; ++s) {
    if (st.left == 0) stream_null(st);
    load_b(0, s);
    load_a(0, s);
    if constexpr (NB == 2) load_b(1, s);
    if constexpr (NU == 2) load_a(1, s);
    st.next();
  }
  wait_vmcnt<kFlight>();
  slot_barrier();
  if constexpr (kFour) {
    read_b(2, 0);
    // the first phase refills this unit, each wave for another one's reads too
    wait_lgkm0();
    slot_barrier();
  }
  if (grp == 1) slot_barrier();

  int t = cur.kn;  // K steps of cur still to compute
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[u][b][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  for (;;) {
    if (st.left == 0) {
      // The stream follows the chain into the next item of the kind if this
      // one is whole and long enough that the stream is at most one item
      // ahead.
      const int ni = !has_next && !split && KT > 2 * NST ? nth_item(sc, r + 1, nwg, xcd, xj) : -1;
      if (ni >= 0 && item_kind(sc, ni) == (FAM | (NB == 1 ? 4 : 0))) {
        nxt = decode_item<GATED, FAM, NB>(p, sc, ni, ncol, KT);
        nitem = ni;
        has_next = true;
        stream_set<GATED, FP8, FAM, NB>(st, p, nxt, wave);
      } else {
        stream_null(st);
      }
    }
    // steps until the stream or the item ends
    int seg = min(t, st.left);
    t -= seg;
    do {
      const int ns = stage + 1 == NST ? 0 : stage + 1;
      if constexpr (kFour) {
        // Four phases per K step, one per (A unit, B unit) pair, in an order
        // in which each needs one new operand unit: A0, B1, A1, then B0 of
        // the next step.  A phase's loads refill the unit that was read one
        // phase earlier, kAhead steps ahead.
#define FFN_PHASE(READS, LOADS, WIDEN, MMA) \
  do {                                      \
    READS;                                  \
    LOADS;                                  \
    wait_vmcnt<kFlight>();                  \
    wait_lgkm0();                           \
    WIDEN;                                  \
    slot_barrier();                         \
    MMA;                                    \
    slot_barrier();                         \
  } while (0)
        FFN_PHASE(read_a(0, stage), load_b(0, stage), widen(0), mma(0, 0));
        FFN_PHASE(read_b(1, stage), load_a(0, stage), widen(1), mma(0, 1));
        FFN_PHASE(read_a(1, stage), load_b(1, stage), (void)0, mma(1, 1));
        FFN_PHASE(read_b(2, ns), load_a(1, stage); st.next(), (void)0, mma(1, 0));
#undef FFN_PHASE
      } else {
        // One phase per K step; the stage read in the last phase is refilled.
        const int fs = stage == 0 ? NST - 1 : stage - 1;
        read_a(0, stage);
#pragma unroll
        for (int b = 0; b < NB; ++b) read_b(b, stage);
        load_a(0, fs);
#pragma unroll
        for (int b = 0; b < NB; ++b) load_b(b, fs);
        st.next();
        wait_vmcnt<kFlight>();
        wait_lgkm0();
#pragma unroll
        for (int b = 0; b < NB; ++b) widen(b);
        slot_barrier();
#pragma unroll
        for (int b = 0; b < NB; ++b) mma(0, b);
        slot_barrier();
      }
      stage = ns;
    } while (--seg);
    if (t > 0) continue;

    constexpr int kPart = F::kRows * F::kCols;  // floats
    constexpr int kFrags = NU * NB * RF * 2;
    // split tiles: what the finisher adds to its own sums
    Piece pc{1, 0, 0, 0, 0, 0};
    unsigned tags = 0;
    if (split) {
      pc = decode_piece(sc, item, FAM);
      // Split tile.  The pieces arrive on the tile's counter word: bits 0-3
      // count arrivals, bits 4-7 finished parts, bits 8 + 3a the piece that
      // part a holds.  All but the last arrival store their f32 sums as a
      // part; the last one waits for the parts (their workgroups have
      // finished their K steps and only store, so the wait ends) and adds
      // everything in piece order, so results do not depend on the order of
      // arrival.  Parts and counter are written and read at agent scope (at
      // the level that is coherent across the XCDs' L2 caches); a part's
      // stores have completed (vmcnt 0, barrier) before it is counted, and
      // the finisher's loads are issued after it has seen the count.
      if (grp == 0) slot_barrier();  // the groups are in step again
      wait_vmcnt<0>();
      slot_barrier();  // the ring is free
      volatile __attribute__((address_space(3))) int* flag =
          (volatile __attribute__((address_space(3))) int*)smem;
      int32_t* cnt = p.split_cnt + pc.cnt;
      if (tid == 0)
        flag[0] = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 15;
      __syncthreads();
      const int arrival = __builtin_amdgcn_readfirstlane(flag[0]);
      if (arrival < pc.n - 1) {
        __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(p.split_slots + pc.slot + (int64_t)arrival * kPart, 0, kPart * 4, 0x00020000);
        const int vo = (wave * kFrags * 64 + lane) * 16;
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < RF; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[u][b][i][j]), rs, vo,
                                                       (((u * NB + b) * RF + i) * 2 + j) * 1024, 16 /* sc1 */);
        wait_vmcnt<0>();
        __syncthreads();  // every wave's part has completed
        if (tid == 0)
          __hip_atomic_fetch_add(cnt, 16 + (pc.piece << (8 + 3 * arrival)), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
        r += 1;
        item = nth_item(sc, r, nwg, xcd, xj);
        return;
      }
      if (tid == 0) {
        int w;
        while ((((w = __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 4) & 15) < pc.n - 1)
          __builtin_amdgcn_s_sleep(1);
        flag[1] = w;
        __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
      }
      __syncthreads();
      tags = (unsigned)uni(flag[1]) >> 8;
    }
    // own sums (piece pc.piece) and the parts of the others, in piece order
    auto add_parts = [&](f32x4_t (&sum)[RF][2], int u, int b) {
#pragma unroll
      for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) sum[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      for (int q = 0; q < pc.n; ++q) {
        if (q == pc.piece) {
#pragma unroll
          for (int i = 0; i < RF; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) sum[i][j] += acc[u][b][i][j];
          continue;
        }
        int a = 0;  // the part that holds piece q
        for (int z = 0; z < pc.n - 1; ++z)
          if ((int)((tags >> (3 * z)) & 7u) == q) a = z;
        __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            p.split_slots + pc.slot + (int64_t)a * kPart, 0, kPart * 4, 0x00020000);
        const int vo = (wave * kFrags * 64 + lane) * 16;
        u32x4_t v[RF][2];
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            v[i][j] = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, (((u * NB + b) * RF + i) * 2 + j) * 1024,
                                                            16 /* sc1 */);
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) sum[i][j] += __builtin_bit_cast(f32x4_t, v[i][j]);
      }
    };

    // Epilogue, from the registers: a lane holds output columns 4hh .. 4hh + 3
    // of a 16-column fragment for one row; a swap of odd and even 16-lane
    // rows between two packed fragments gives it 8 consecutive columns, one
    // 16-byte store.  No LDS, no barrier: the waves go straight on to the
    // next item, whose first stages the stream has already requested.  Rows
    // past the group's end are out of the resource's range.
    {
      const int rows = min(cur.rows, F::kRows);
      __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
          reinterpret_cast<uint16_t*>(p.out) + (int64_t)cur.y_row0 * n_out, 0,
          (int)((uint32_t)rows * (uint32_t)n_out * 2u), 0x00020000);
      auto store8 = [&](const uint2 x, const uint2 y, int row, int col) {
        const auto s0 = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
        const u32x4_t v = {(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
        const uint32_t off = ((uint32_t)row * (uint32_t)n_out + (uint32_t)col) * 2u;
        __builtin_amdgcn_raw_buffer_store_b128(v, ro, row < rows && col < n_out ? off : 0xfffffff0u, 0, 0);
      };
      auto pack = [](float a, float b) {
        bf16x2v_t v;
        v[0] = (__bf16)a;
        v[1] = (__bf16)b;
        return __builtin_bit_cast(uint32_t, v);
      };
      const const_ptr<WeightDesc> wd = as_const(p.wtab) + cur.g;
      // four bf16 scales from column c on: vector loads, as lanes differ; the
      // wait for them drains the ring once per tile
      auto scales = [&](const uint16_t* s, int c) {
        uint2 v;  // the caller's scales are 2-byte aligned
        __builtin_memcpy(&v, s + min(c, n_out - 4), 8);
        return f32x4_t{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xffff0000u)};
      };
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        f32x4_t sg, su;
        if constexpr (FP8) {
          if constexpr (GATED) {
            const int c = cur.nti * kOut + wn * (16 * NB) + b * 16 + hh * 4;
            sg = scales(wd->s_gu, c);
            // the up scales start at element n_out, a multiple of 64
            su = scales(wd->s_gu + n_out, c);
          } else {
            const int c = cur.nti * kOut + b * 128 + wn * 32 + hh * 4;
            sg = scales(wd->s_down, c);
            su = scales(wd->s_down, c + 16);
          }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          const int row0 = u * 128 + wm * (F::kUnitRows / 2) + rr;
          f32x4_t o[RF][2];
          if (split) {
            add_parts(o, u, b);
          } else {
#pragma unroll
            for (int i = 0; i < RF; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j) o[i][j] = acc[u][b][i][j];
          }
          if constexpr (GATED) {
            const int col = cur.nti * kOut + wn * (16 * NB) + b * 16 + (hh >> 1) * 8;
#pragma unroll
            for (int i = 0; i < RF; i += 2) {
              uint2 w[2];
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  float gv = o[i + q][0][e], uv = o[i + q][1][e];
                  if constexpr (FP8) {
                    gv *= sg[e];
                    uv *= su[e];
                  }
                  v[e] = gv * __builtin_amdgcn_rcpf(1.f + __expf(-gv)) * uv;
                }
                w[q] = make_uint2(pack(v[0], v[1]), pack(v[2], v[3]));
              }
              store8(w[0], w[1], row0 + (i + (hh & 1)) * 16, col);
            }
          } else {
            const int col = cur.nti * kOut + b * 128 + wn * 32 + (hh & 1) * 16 + (hh >> 1) * 8;
#pragma unroll
            for (int i = 0; i < RF; ++i) {
              uint2 w[2];
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                f32x4_t v = o[i][j];
                if constexpr (FP8) v *= j == 0 ? sg : su;
                w[j] = make_uint2(pack(v[0], v[1]), pack(v[2], v[3]));
              }
              store8(w[0], w[1], row0 + i * 16, col);
            }
          }
        }
      }
    }

    r += 1;
    if (!has_next) {
      item = nth_item(sc, r, nwg, xcd, xj);
      if (!split) {
        if (grp == 0) slot_barrier();  // the groups are in step again
        wait_vmcnt<0>();               // no load still targets the ring
      }
      return;
    }
    item = nitem;
    cur = nxt;
    split = cur.kn < KT;
    has_next = false;
    t = cur.kn;
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[u][b][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
}

// The FFN launch for bf16 or fp8 weights.
template <bool GATED, bool FP8>
__global__ __launch_bounds__(512, 2) void ffn_mfma_kernel(const FfnParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kFfnLds];
  const bool probe = p.clk != nullptr && (int)blockIdx.x < p.clk_n;
  unsigned long long clk0 = 0, rt0 = 0;
  if (probe) {
    clk0 = __builtin_amdgcn_s_memtime();
    rt0 = __builtin_amdgcn_s_memrealtime();
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_vptr)smem;
  const int nwg = gridDim.x;
  const int xcd = blockIdx.x & 7, xj = blockIdx.x >> 3;
  const const_ptr<int32_t> tot = as_const(p.tile_totals);
  Sched sc;
  sched_tiles(sc, uni(tot[0]), uni(tot[1]), uni(tot[2]), nwg);
  sched_cut(sc, (unsigned)uni((int)*as_const(p.cut)), nwg);
  int r = 0;
  int item = nth_item(sc, r, nwg, xcd, xj);
  while (item >= 0) {
    const int kind = item_kind(sc, item);
    if (kind == 0)
      run_family<GATED, FP8, 0, 2>(p, sc, smem, lds_base, nwg, xcd, xj, r, item);
    else if (kind == 1)
      run_family<GATED, FP8, 1, 2>(p, sc, smem, lds_base, nwg, xcd, xj, r, item);
    else if (kind == 2)
      run_family<GATED, FP8, 2, 2>(p, sc, smem, lds_base, nwg, xcd, xj, r, item);
    else if (kind == 4)
      run_family<GATED, FP8, 0, 1>(p, sc, smem, lds_base, nwg, xcd, xj, r, item);
    else if (kind == 5)
      run_family<GATED, FP8, 1, 1>(p, sc, smem, lds_base, nwg, xcd, xj, r, item);
    else
      run_family<GATED, FP8, 2, 1>(p, sc, smem, lds_base, nwg, xcd, xj, r, item);
  }
  if (probe) {
    const unsigned long long clk1 = __builtin_amdgcn_s_memtime(), rt1 = __builtin_amdgcn_s_memrealtime();
    if (threadIdx.x == 0) {
      p.clk[2 * blockIdx.x] = clk1 - clk0;
      p.clk[2 * blockIdx.x + 1] = rt1 - rt0;
    }
  }
}

// ---------------------------------------------------------------- f32 path
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// One 32 x 32 output tile (two in gate/up: gate and up) of a wave over kn
// values of k: v_mfma_f32_32x32x2_f32, operands straight from global memory.
// A lane reads four consecutive k of its row; lane half h of a group of 8 k
// holds k = 4h .. 4h + 3 of both operands, so every MFMA pairs equal k.
// N groups of 8 k are requested before the first is used.
template <bool GATED, int N>
__device__ __forceinline__ void f32_chunk(const float* a, const float* g, const float* u, f32x16_t& ag, f32x16_t& au) {
  float4 va[N], vg[N], vu[GATED ? N : 1];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    va[i] = *reinterpret_cast<const float4*>(a + 8 * i);
    vg[i] = *reinterpret_cast<const float4*>(g + 8 * i);
    if constexpr (GATED) vu[i] = *reinterpret_cast<const float4*>(u + 8 * i);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float av[4] = {va[i].x, va[i].y, va[i].z, va[i].w}, gv[4] = {vg[i].x, vg[i].y, vg[i].z, vg[i].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) ag = __builtin_amdgcn_mfma_f32_32x32x2f32(gv[j], av[j], ag, 0, 0, 0);
    if constexpr (GATED) {
      const float uv[4] = {vu[i].x, vu[i].y, vu[i].z, vu[i].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) au = __builtin_amdgcn_mfma_f32_32x32x2f32(uv[j], av[j], au, 0, 0, 0);
    }
  }
}

// The f32 launch.  The plan's tiles are 64 x 64; each is four work items of
// 32 x 32, of which the four waves of a workgroup take a quarter of K each and
// add their sums through LDS: launches of this path are small, and what bounds
// them is the latency of one tile's K walk.  256 tokens, d = 256, f = 512, 8
// experts: gate/up 58.8 -> 12.2 us, down 33.5 -> 7.9 us against 64 x 64 tiles
// of scalar FMAs staged through LDS.  (A wave per 32 x 32 over all of K reads
// the operands half as often; at 4096 rows of d = 512, f = 1024, 1100 tiles,
// whole layers took 274 us that way and 241 us split, 4 experts 202 and 205.)
template <bool GATED>
__global__ __launch_bounds__(256) void ffn_f32_kernel(const FfnParams p) {
  __shared__ float part[4][GATED ? 32 : 16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int items = 4 * p.tile_totals[0];
  const int K = p.K, n_out = p.n_out;
  const int r = lane & 31, h = lane >> 5;

  for (int item = blockIdx.x; item < items; item += gridDim.x) {
    const int tile = item >> 2, sub = item & 3;
    const int g = p.tile_group[tile];
    const GroupDesc gd = p.groups[g];
    const WeightDesc wd = p.wtab[g];
    const int local = tile - gd.t0[GATED ? 0 : 3];
    const int nti = local / gd.nrt[0];
    const int m0 = (local - nti * gd.nrt[0]) * kBM32 + (sub >> 1) * 32;
    const int c0 = nti * kBN32 + (sub & 1) * 32;
    if (m0 >= gd.n) continue;  // the whole workgroup
    const int kn = K / 4, k0 = wave * kn;
    const float* a = reinterpret_cast<const float*>(p.a) +
                     (int64_t)((GATED ? gd.x_row0 : gd.y_row0) + min(m0 + r, gd.n - 1)) * K + k0 + 4 * h;
    const float* wg = reinterpret_cast<const float*>(GATED ? wd.gate : wd.down) + (int64_t)(c0 + r) * K + k0 + 4 * h;
    const float* wu = GATED ? reinterpret_cast<const float*>(wd.up) + (int64_t)(c0 + r) * K + k0 + 4 * h : nullptr;
    f32x16_t ag, au;
#pragma unroll
    for (int i = 0; i < 16; ++i) ag[i] = au[i] = 0.f;
    int k = 0;  // kn is a multiple of 16
    for (; k + 64 <= kn; k += 64) f32_chunk<GATED, 8>(a + k, wg + k, wu + k, ag, au);
    for (; k < kn; k += 16) f32_chunk<GATED, 2>(a + k, wg + k, wu + k, ag, au);

    // lane: row m0 + r; register i: column c0 + 8 (i / 4) + 4 h + i % 4
    __syncthreads();  // the last item's sums are read
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      part[wave][i][lane] = ag[i];
      if constexpr (GATED) part[wave][16 + i][lane] = au[i];
    }
    __syncthreads();
    // each wave finishes four registers, adding the waves' sums in order
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float s = 0.f, u = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        s += part[w][4 * wave + i][lane];
        if constexpr (GATED) u += part[w][16 + 4 * wave + i][lane];
      }
      v[i] = GATED ? s / (1.f + expf(-s)) * u : s;
    }
    if (m0 + r < gd.n)
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.out) + (int64_t)(gd.y_row0 + m0 + r) * n_out + c0 + 4 * h +
                                 8 * wave) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

hipError_t launch_ffn(int stage, int act_dtype, int w_dtype, const GroupDesc* groups,
                      const WeightDesc* wtab, const int32_t* tile_totals, const int32_t* tile_group,
                      float* split_slots, int32_t* split_cnt, int max_tiles,
                      const void* xp, void* h, void* y, int d, int f, int num_cu,
                      unsigned long long* clk, int clk_n, hipStream_t s) {
  if (max_tiles <= 0) return hipSuccess;
  const FfnParams p{groups,
                    wtab,
                    tile_totals + 3 * stage,
                    reinterpret_cast<const uint32_t*>(tile_totals) + kCutWord + stage,
                    tile_group,
                    split_slots,
                    split_cnt,
                    stage == 0 ? xp : h,
                    stage == 0 ? h : y,
                    stage == 0 ? d : f,
                    stage == 0 ? f : d,
                    clk,
                    clk_n};
  if (act_dtype == 0) {
    const int grid = std::min(4 * std::min(max_tiles, 4 * num_cu), 8 * num_cu);
    if (stage == 0)
      ffn_f32_kernel<true><<<grid, 256, 0, s>>>(p);
    else
      ffn_f32_kernel<false><<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
  }
  // one 512-thread workgroup per CU; the tail of a launch is cut to fill the
  // whole grid, however few its tiles
  const int grid = ffn_grid(num_cu);
  if (w_dtype == 2) {
    if (stage == 0)
      ffn_mfma_kernel<true, true><<<grid, 512, 0, s>>>(p);
    else
      ffn_mfma_kernel<false, true><<<grid, 512, 0, s>>>(p);
  } else {
    if (stage == 0)
      ffn_mfma_kernel<true, false><<<grid, 512, 0, s>>>(p);
    else
      ffn_mfma_kernel<false, false><<<grid, 512, 0, s>>>(p);
  }
  return hipGetLastError();
}

}  // namespace aep
