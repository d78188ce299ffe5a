// Scans within a workgroup, and a consumer's own offsets from the counts
// before it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mt_internal.h"

namespace mt {

// Inclusive scan of one value per lane across a wavefront.
template <class T>
__device__ __forceinline__ T wave_inclusive(T x) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    T y = __shfl_up(x, d, 64);
    if ((int)(threadIdx.x & 63) >= d) x += y;
  }
  return x;
}

// Exclusive scan across the workgroup (N threads) of one value per thread;
// returns the exclusive prefix and writes the total to *total.
template <int N, class T>
__device__ __forceinline__ T block_exclusive(T x, T* total) {
  __shared__ T wsum[N / 64];
  const int w = threadIdx.x >> 6;
  T inc = wave_inclusive(x);
  if ((threadIdx.x & 63) == 63) wsum[w] = inc;
  __syncthreads();
  T off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < N / 64; ++i) {
    if (i < w) off += wsum[i];
    tot += wsum[i];
  }
  __syncthreads();
  *total = tot;
  return off + inc - x;
}

// This thread's share of the sum of cnt[0 .. first) (16-byte aligned, first a
// multiple of 4) over a workgroup of N threads: 8 loads in flight (one at a
// time, whole steps of 20K to 66K slave elements took 4 to 12 us longer).
template <int N>
__device__ __forceinline__ int32_t sum_before(const int32_t* __restrict__ cnt, int32_t first) {
  constexpr int U = 8;
  int32_t part = 0;
  for (int32_t i = 4 * (int32_t)threadIdx.x; i < first; i += 4 * N * U) {
    int4 v[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int32_t k = i + 4 * N * q;
      v[q] = make_int4(0, 0, 0, 0);
      if (k < first) v[q] = *reinterpret_cast<const int4*>(cnt + k);
    }
#pragma unroll
    for (int q = 0; q < U; ++q) part += v[q].x + v[q].y + v[q].z + v[q].w;
  }
  return part;
}

// Offset of each thread's value x (of N threads, cnt[0 .. first) before
// them; cnt 16-byte aligned, first a multiple of 4): the workgroup adds up
// the counts before its own, so that no launch need scan them first.  The
// whole workgroup calls it.
template <int N>
__device__ __forceinline__ int32_t self_offset(const int32_t* __restrict__ cnt, int32_t first, int32_t x) {
  int32_t before, own;
  const int32_t part = sum_before<N>(cnt, first);
  block_exclusive<N>(part, &before);
  const int32_t off = block_exclusive<N>(x, &own);
  return before + off;
}

// Up to this many counts the kernel that uses their offsets finds them itself
// (self_offset): every workgroup reads the counts before its own from L2,
// where the scan costs a launch and the gap before it.  Whole step, wavy,
// without read-back, scan -> own offsets: 4K slave elements 213 -> 192 us,
// 10K 229 -> 214, 16K 245 -> 230, 33K 264 -> 253, 66K 320 -> 317, 90K
// 362 -> 369, 161K 515 -> 588.
constexpr int64_t SELF_OFFSETS = 67584;

// The total of a stage of the build into the device state, clamped to the
// stage's capacity (the flag records an excess); the nonzeros of the pattern
// as they are (second: of the scan's second array).
__device__ __forceinline__ void stage_total(const ScanStage& g, int64_t total, bool second) {
  DevState* st = g.st;
  if (g.stage == ScanStage::NNZ) {
    (second ? st->nnz_M : st->nnz_D) = (int32_t)total;
    return;
  }
  const bool over = total < 0 || total > g.cap;  // negative: the int32 scan overflowed (more than 2^31)
  const int32_t all = (int32_t)(total < 0 ? 0x7fffffff : total);
  const int32_t kept = (int32_t)(total < 0 ? 0 : (total < g.cap ? total : g.cap));
  if (g.stage == ScanStage::CANDIDATES) {
    st->n_cand = all;
    if (over) st->flags |= DS_CAP_CAND;
  } else if (g.stage == ScanStage::SCREENED) {
    st->need_screened = all;
    st->n_screened = kept;
    if (over) st->flags |= DS_CAP_SCREENED;
  } else {
    st->need_pairs = all;
    st->n_pairs = kept;
    if (over) st->flags |= DS_CAP_PAIRS;
  }
}

}  // namespace mt
