// Token pool: the top-K merge across drains.  When a layer's experts are
// drained one at a time, a token's k rows are computed in different drains;
// each drain adds its rows, weighted by their gate weights, into the token's
// f32 pool row, and a token is released -- rounded once to the activation
// type and its pool row cleared -- when all k rows have been added.
//
// accumulate: one workgroup per batch row.  A single-expert batch holds at
// most one row per token, so no two workgroups touch the same pool row and no
// atomics are needed; the per-token count of rows still to come is decremented
// by one thread.  release: one workgroup per token id; tokens that are not
// complete are skipped after two loads.  Both are bound by the latency of a
// row's read-modify-write: a thread moves 8 consecutive elements at a time in
// 16-byte accesses, all requested before any is used (one wave per row with
// 4- and 8-byte accesses took 18.0 us per 256 rows of d = 4096 and 21.7 us
// for the release of 1024 tokens; now 5.7 and 10.0).
#include "aep_device.h"
#include "aep_internal.h"

namespace aep {

// 16 bytes at a 4-byte aligned address (caller tensors)
typedef unsigned u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kPoolU = 2;  // groups of 8 elements per thread in flight

template <bool BF16>
__global__ __launch_bounds__(256) void pool_accumulate_kernel(const void* __restrict__ y, int64_t N,
                                                              const int32_t* __restrict__ offsets,
                                                              int E, const int32_t* __restrict__ row_token,
                                                              const float* __restrict__ row_w,
                                                              float* __restrict__ pool,
                                                              int32_t* __restrict__ pend, int d) {
  const int64_t r = blockIdx.x;
  if (r >= N || r >= offsets[E]) return;
  const int tok = row_token[r];
  const float w = row_w[r];
  float* dst = pool + (int64_t)tok * d;
  const int ng = d / 8;  // d is a multiple of 64
  for (int g0 = threadIdx.x; g0 < ng; g0 += 256 * kPoolU) {
    float v[kPoolU][8];
    f32x4_a4 a[kPoolU][2];
#pragma unroll
    for (int q = 0; q < kPoolU; ++q) {
      const int g = min(g0 + 256 * q, ng - 1);
      if constexpr (BF16) {
        const u32x4_a4 u = *reinterpret_cast<const u32x4_a4*>(reinterpret_cast<const uint16_t*>(y) + r * d + 8 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[q][2 * i] = bf16_lo(u[i]);
          v[q][2 * i + 1] = bf16_hi(u[i]);
        }
      } else {
        const float* src = reinterpret_cast<const float*>(y) + r * d + 8 * g;
        const f32x4_a4 u0 = *reinterpret_cast<const f32x4_a4*>(src), u1 = *reinterpret_cast<const f32x4_a4*>(src + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[q][i] = u0[i];
          v[q][4 + i] = u1[i];
        }
      }
      a[q][0] = *reinterpret_cast<const f32x4_a4*>(dst + 8 * g);
      a[q][1] = *reinterpret_cast<const f32x4_a4*>(dst + 8 * g + 4);
    }
#pragma unroll
    for (int q = 0; q < kPoolU; ++q) {
      const int g = g0 + 256 * q;
      if (g >= ng) break;
#pragma unroll
      for (int i = 0; i < 8; ++i) a[q][i / 4][i % 4] = fmaf(w, v[q][i], a[q][i / 4][i % 4]);
      *reinterpret_cast<f32x4_a4*>(dst + 8 * g) = a[q][0];
      *reinterpret_cast<f32x4_a4*>(dst + 8 * g + 4) = a[q][1];
    }
  }
  if (threadIdx.x == 0) pend[tok] -= 1;
}

template <bool BF16>
__global__ __launch_bounds__(256) void pool_release_kernel(float* __restrict__ pool,
                                                           int32_t* __restrict__ live,
                                                           int32_t* __restrict__ pend, int n_ids,
                                                           void* __restrict__ out,
                                                           int32_t* __restrict__ ready, int d) {
  const int t = blockIdx.x;
  const bool done = live[t] != 0 && pend[t] == 0;
  if (ready && threadIdx.x == 0) ready[t] = done ? 1 : 0;
  if (!done) return;
  __syncthreads();  // live[t] is read by all before it is cleared
  float* src = pool + (int64_t)t * d;
  const int ng = d / 8;
  for (int g0 = threadIdx.x; g0 < ng; g0 += 256 * kPoolU) {
    f32x4_a4 a[kPoolU][2];
#pragma unroll
    for (int q = 0; q < kPoolU; ++q) {
      const int g = min(g0 + 256 * q, ng - 1);
      a[q][0] = *reinterpret_cast<const f32x4_a4*>(src + 8 * g);
      a[q][1] = *reinterpret_cast<const f32x4_a4*>(src + 8 * g + 4);
    }
#pragma unroll
    for (int q = 0; q < kPoolU; ++q) {
      const int g = g0 + 256 * q;
      if (g >= ng) break;
      if constexpr (BF16) {
        u32x4_a4 u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4_a4& h = a[q][i / 2];
          u[i] = f32_to_bf16_rne(h[2 * (i % 2)]) | (f32_to_bf16_rne(h[2 * (i % 2) + 1]) << 16);
        }
        *reinterpret_cast<u32x4_a4*>(reinterpret_cast<uint16_t*>(out) + (int64_t)t * d + 8 * g) = u;
      } else {
        float* o = reinterpret_cast<float*>(out) + (int64_t)t * d + 8 * g;
        *reinterpret_cast<f32x4_a4*>(o) = a[q][0];
        *reinterpret_cast<f32x4_a4*>(o + 4) = a[q][1];
      }
      const f32x4_a4 zero = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4_a4*>(src + 8 * g) = zero;
      *reinterpret_cast<f32x4_a4*>(src + 8 * g + 4) = zero;
    }
  }
  if (threadIdx.x == 0) live[t] = 0;
}

hipError_t launch_pool_accumulate(int act_dtype, const void* y, int64_t N, const int32_t* offsets,
                                  int E, const int32_t* row_token, const float* row_w, float* pool,
                                  int32_t* pend, int d, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  const unsigned nb = (unsigned)N;
  if (act_dtype == 0)
    pool_accumulate_kernel<false><<<nb, 256, 0, s>>>(y, N, offsets, E, row_token, row_w, pool, pend, d);
  else
    pool_accumulate_kernel<true><<<nb, 256, 0, s>>>(y, N, offsets, E, row_token, row_w, pool, pend, d);
  return hipGetLastError();
}

hipError_t launch_pool_release(int act_dtype, float* pool, int32_t* live, int32_t* pend, int n_ids,
                               void* out, int32_t* ready, int d, hipStream_t s) {
  const unsigned nb = (unsigned)n_ids;
  if (act_dtype == 0)
    pool_release_kernel<false><<<nb, 256, 0, s>>>(pool, live, pend, n_ids, out, ready, d);
  else
    pool_release_kernel<true><<<nb, 256, 0, s>>>(pool, live, pend, n_ids, out, ready, d);
  return hipGetLastError();
}

}  // namespace aep
