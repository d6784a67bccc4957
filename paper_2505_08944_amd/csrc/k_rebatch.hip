// Executor re-batch kernels: drain plan + gather.
//
// plan: workgroup 0 reads the drained layer's per-expert queue depths (or one
// expert's, for a single-expert drain) with one thread per group, and writes
// counts / exclusive-scan offsets / the FFN group table (row-tile families
// and tile ranges), then the group of every tile of both FFN launches (a run
// of tiles per group, family and launch); it resets the drained queue depths
// to zero.  All workgroups clear the (token, slot) -> row map.  The launch is
// one chain of latencies (depths, scan, table), so the chain is kept short:
// scans by DPP, one barrier for up to 64 groups and no search per tile (66
// groups, 8192 tokens 11.9 -> 7.5 us; 8 groups, 4.6 us).
//
// gather: one wave per batch row.  A routed row finds its expert from the
// offsets (up to 64 experts: one lane per offset and a ballot, no LDS and no
// barrier before the row's own loads; more: binary search in LDS), reads its
// queue entry and copies the referenced row (16-byte vector loads/stores, the
// whole wave on one row, so each row is one contiguous coalesced stream; up
// to 8 loads per lane in flight before the stores); lane 0 records the row's
// token and gate weight and the (token, slot) -> row map.  Shared-expert rows
// copy every token's row in id order.  The first few workgroups choose how the
// last round of each FFN launch is cut.
#include <algorithm>

#include "ffn_sched.h"

namespace aep {

constexpr int kPlanThreads = 1024;

// Inclusive sum over the lanes of a wave: rows of 16 by shifts, then the last
// lane of the row and of the half before.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111 /* row_shr 1 */, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112 /* row_shr 2 */, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114 /* row_shr 4 */, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118 /* row_shr 8 */, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142 /* row_bcast 15 */, 0xA, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143 /* row_bcast 31 */, 0xC, 0xF, false);
  return v;
}

// Workgroup 0 plans the drain, one thread per group; every workgroup clears
// its share of the (token, slot) -> row map.
__global__ __launch_bounds__(kPlanThreads) void plan_kernel(int E, int S, int n_tokens, int k,
                                                            int only_expert, int32_t* __restrict__ depth,
                                                            int32_t* __restrict__ depth_other,
                                                            int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ offsets,
                                                            GroupDesc* __restrict__ groups,
                                                            int32_t* __restrict__ tile_totals,
                                                            int nt0, int nt1, int bm, int families,
                                                            int32_t* __restrict__ tile_group,
                                                            int64_t tile_cap,
                                                            int32_t* __restrict__ pos,
                                                            float* __restrict__ posw) {
  constexpr int kWaves = kPlanThreads / 64;
  const int tid = threadIdx.x, wave = tid >> 6;
  const int G = E + S;
  const int g = tid;
  const bool real = blockIdx.x == 0 && g < G;
  const int n = !real ? 0 : g < E ? (only_expert < 0 || g == only_expert ? depth[g] : 0) : n_tokens;

  const int64_t nk = (int64_t)n_tokens * k;
  for (int64_t i = (int64_t)blockIdx.x * kPlanThreads + tid; i < nk; i += (int64_t)gridDim.x * kPlanThreads) {
    pos[i] = -1;
    posw[i] = 0.f;
  }
  if (blockIdx.x != 0) return;

  // full blocks, and the remainder in one tile of the smallest family that
  // holds it
  const int full = n / bm, rem = n - full * bm;
  int nrt[3] = {full, 0, 0};
  if (families == 1 || rem > bm / 2)
    nrt[0] += rem > 0 ? 1 : 0;
  else if (rem > bm / 4)
    nrt[1] = 1;
  else if (rem > 0)
    nrt[2] = 1;
  // rows and row tiles per family of the groups before this one, and of all
  __shared__ int32_t wsum[kWaves][4];
  __shared__ int32_t first[3][kMaxGroups + 1];  // a group's first row tile per family
  int inc[4] = {n, nrt[0], nrt[1], nrt[2]};
  if (G > 64 || wave == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) inc[i] = wave_scan(inc[i]);
  }
  if (G > 64) {
    if ((tid & 63) == 63)
#pragma unroll
      for (int i = 0; i < 4; ++i) wsum[wave][i] = inc[i];
    __syncthreads();
    int before[4] = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
      for (int i = 0; i < 4; ++i) before[i] += w < wave ? wsum[w][i] : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) inc[i] += before[i];
  }
  if (real) {
    GroupDesc gd;
    gd.n = n;
    // shared groups all read the token rows that follow the routed ones
    const int row0 = inc[0] - n;
    gd.x_row0 = g >= E ? row0 - (g - E) * n_tokens : row0;
    gd.y_row0 = row0;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      const int t0 = inc[1 + f] - nrt[f];
      first[f][g] = t0;
      gd.t0[f] = t0 * nt0;
      gd.t0[3 + f] = t0 * nt1;
      gd.nrt[f] = nrt[f];
    }
    gd.row1 = full * bm;
    gd.pad[0] = gd.pad[1] = gd.pad[2] = 0;
    groups[g] = gd;
    counts[g] = n;
    offsets[g] = row0;
    if (g == G - 1) {
      offsets[G] = inc[0];
#pragma unroll
      for (int f = 0; f < 3; ++f) {
        first[f][G] = inc[1 + f];
        tile_totals[f] = inc[1 + f] * nt0;
        tile_totals[3 + f] = inc[1 + f] * nt1;
      }
      tile_totals[kCutWord] = tile_totals[kCutWord + 1] = (int32_t)kNoCut;
    }
    // The drained queues are empty again, in both halves of the depth
    // ping-pong: whichever half the next append reads starts from zero (so a
    // captured drain step replays correctly whatever the parity of its
    // appends).
    if (g < E && (only_expert < 0 || g == only_expert)) depth[g] = depth_other[g] = 0;
  }
  __syncthreads();
  // The group of every tile of both launches (tiles are numbered per launch,
  // family by family): a group's tiles of a family follow one another, written
  // by one wave, or by several where there are fewer groups than waves.
  const int per = G < kWaves ? kWaves / G : 1;
  for (int h = wave / per; h < G; h += kWaves / per) {
    int base = 0;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      const int lo = first[f][h], hi = first[f][h + 1], all = first[f][G];
      const int lane = (wave % per) * 64 + (tid & 63);
      for (int t = lo * nt0 + lane; t < hi * nt0; t += per * 64) tile_group[(int64_t)base * nt0 + t] = h;
      for (int t = lo * nt1 + lane; t < hi * nt1; t += per * 64) tile_group[tile_cap + (int64_t)base * nt1 + t] = h;
      base += all;
    }
  }
}

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) v4u* gsrc_t;

// N 16-byte chunks per lane of a row from chunk c0 on, every load issued
// before the first store (the source rows are global memory; the stores cannot
// alias them).  FULL: all of them exist.
template <int N, bool FULL>
__device__ __forceinline__ void copy_pass(gsrc_t src, v4u* dst, int c0, int nchunk) {
  const int c = c0 + (threadIdx.x & 63);
  v4u v[N];
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (FULL || c + 64 * i < nchunk) v[i] = src[c + 64 * i];
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (FULL || c + 64 * i < nchunk) dst[c + 64 * i] = v[i];
}

// The cuts of both FFN launches' last rounds, chosen by kCutBlocks workgroups
// in front of the gather's own: kCutSlots threads per cut, the smallest word
// wins.  A gather of few rows still waits for them a little: single-expert
// drains of a 1024-token layer, 4.9 us on average without, 6.3 with, 7.4 with
// one thread per cut.  Every FFN workgroup working it out for itself took 1.0
// us of each launch.
constexpr int kCutBlocks = 64;
static_assert(kCutBlocks * 256 == 2 * kCuts * kCutSlots && kCutSlots == 8, "threads per stage, cut and slot");
__device__ __forceinline__ void choose_cut(const CutArgs& a, int block) {
  const int stage = block & 1, id = (block >> 1) * 256 + (int)threadIdx.x, cut = id / kCutSlots;
  Sched s;
  sched_tiles(s, uni(a.tile_totals[3 * stage]), uni(a.tile_totals[3 * stage + 1]), uni(a.tile_totals[3 * stage + 2]),
              a.nwg);
  if (!cut_pays(s, a.nwg)) return;
  CutRounds q;
  const bool ok = cut_rounds(q, s, a.fp8, a.nwg, stage == 0 ? a.kt[0] : a.kt[1], a.split_bytes, cut);
  float time = ok ? cut_load(q, s, a.nwg, id % kCutSlots) : 0.f;
#pragma unroll
  for (int off = 1; off < kCutSlots; off <<= 1) time = fmaxf(time, __shfl_xor(time, off));
  uint32_t word = ok ? cut_word(time, cut) : kNoCut;
#pragma unroll
  for (int off = kCutSlots; off < 64; off <<= 1) word = min(word, (uint32_t)__shfl_xor((int)word, off));
  __shared__ uint32_t best[4];
  if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = word;
  __syncthreads();
  word = min(min(best[0], best[1]), min(best[2], best[3]));
  if (threadIdx.x == 0 && word != kNoCut) atomicMin(reinterpret_cast<uint32_t*>(a.tile_totals) + kCutWord + stage, word);
}

// LANES: E <= 64, an offset per lane.  57344 rows of 4 KB take 71 us, 3.3 TB/s
// of stores beside as much read from the Infinity Cache (a row is read once
// per selected expert); two or four rows per wave in flight took 72.
template <bool LANES>
__global__ __launch_bounds__(256) void gather_kernel(
    const QEntry* __restrict__ q, int64_t q_stride, const int32_t* __restrict__ offsets, int E,
    int64_t N, int n_tokens, int shared, const void* const* __restrict__ tok_row, char* xp,
    int64_t row_bytes, int32_t* __restrict__ row_token, float* __restrict__ row_w,
    int32_t* __restrict__ pos, float* __restrict__ posw, int k, int32_t* __restrict__ err, const CutArgs cut) {
  const int ncut = cut.nwg > 0 ? kCutBlocks : 0;
  if ((int)blockIdx.x < ncut) {
    choose_cut(cut, blockIdx.x);
    return;
  }
  __shared__ int32_t off_s[LANES ? 1 : kMaxGroups + 1];
  const int lane = threadIdx.x & 63;
  int my_off = 0;  // LANES: offsets[lane + 1], those past E equal to the last
  if constexpr (LANES) {
    my_off = offsets[min(lane + 1, E)];
  } else {
    for (int i = threadIdx.x; i <= E; i += blockDim.x) off_s[i] = offsets[i];
    __syncthreads();
  }
  const int64_t r = (int64_t)(blockIdx.x - ncut) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t R = N + (shared ? n_tokens : 0);
  if (r >= R) return;
  const int routed = LANES ? __builtin_amdgcn_readlane(my_off, 63) : off_s[E];
  if (r < N && r >= routed) return;  // N only bounds the routed rows
  const void* row;
  if (r < N) {
    int lo = 0, at;  // the row's expert, and its place in the expert's queue
    if constexpr (LANES) {
      // r < routed, so the offsets not above it are those of lo experts
      lo = __popcll(__ballot(my_off <= r));
      at = (int)r - (lo > 0 ? __builtin_amdgcn_readlane(my_off, lo - 1) : 0);
    } else {
      int hi = E;  // off_s[lo] <= r < off_s[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off_s[mid] <= r)
          lo = mid;
        else
          hi = mid;
      }
      at = (int)r - off_s[lo];
    }
    const QEntry en = q[(int64_t)lo * q_stride + at];
    row = en.row;
    if (lane == 0) {
      const int tok = en.token_slot & kTokenMask;
      const int slot = (int)((uint32_t)en.token_slot >> kTokenBits);
      row_token[r] = tok;
      row_w[r] = en.w;
      if (pos) {
        const int64_t pi = (int64_t)tok * k + slot;
        const int old = atomicExch(&pos[pi], (int)r);
        posw[pi] = en.w;
        if (old != -1) atomicOr(err, kErrCollision);
      }
    }
  } else {
    row = tok_row[r - N];
  }
  const gsrc_t src = (gsrc_t)row;
  v4u* dst = reinterpret_cast<v4u*>(xp + r * row_bytes);
  const int nchunk = (int)(row_bytes >> 4);
  int c0 = 0;
  for (; c0 + 512 <= nchunk; c0 += 512) copy_pass<8, true>(src, dst, c0, nchunk);
  if (c0 + 256 <= nchunk) {
    copy_pass<4, true>(src, dst, c0, nchunk);
    c0 += 256;
  }
  if (c0 < nchunk) copy_pass<4, false>(src, dst, c0, nchunk);
}

hipError_t launch_plan(int E, int S, int n_tokens, int k, int only_expert, int32_t* depth,
                       int32_t* depth_other, int32_t* counts, int32_t* offsets, GroupDesc* groups,
                       int32_t* tile_totals, const int* nt, int bm, int families, int32_t* tile_group, int64_t tile_cap, int32_t* pos, float* posw,
                       hipStream_t s) {
  static_assert(kMaxGroups <= kPlanThreads, "one plan thread per group");
  const int64_t nk = (int64_t)n_tokens * k;
  const unsigned nb = (unsigned)std::min<int64_t>(256, std::max<int64_t>(1, (nk + 4 * kPlanThreads - 1) / (4 * kPlanThreads)));
  plan_kernel<<<nb, kPlanThreads, 0, s>>>(E, S, n_tokens, k, only_expert, depth, depth_other, counts, offsets, groups,
                                  tile_totals, nt[0], nt[1], bm, families, tile_group, tile_cap,
                                  pos, posw);
  return hipGetLastError();
}

hipError_t launch_gather(const QEntry* q, int64_t q_stride, const int32_t* offsets, int E,
                         int64_t N, int n_tokens, int shared, const void* const* tok_row,
                         char* xp, int64_t row_bytes, int32_t* row_token, float* row_w,
                         int32_t* pos, float* posw, int k, int32_t* err, const CutArgs& cut, hipStream_t s) {
  const int64_t R = N + (shared ? n_tokens : 0);
  if (R == 0) return hipSuccess;
  const int64_t nb = (R + 3) / 4 + (cut.nwg > 0 ? kCutBlocks : 0);
  if (E <= 64)
    gather_kernel<true><<<(unsigned)nb, 256, 0, s>>>(q, q_stride, offsets, E, N, n_tokens, shared, tok_row, xp,
                                                     row_bytes, row_token, row_w, pos, posw, k, err, cut);
  else
    gather_kernel<false><<<(unsigned)nb, 256, 0, s>>>(q, q_stride, offsets, E, N, n_tokens, shared, tok_row, xp,
                                                      row_bytes, row_token, row_w, pos, posw, k, err, cut);
  return hipGetLastError();
}

}  // namespace aep
