// Row-owner device functions of the deterministic assembly: one thread owns
// one output row (slave node) or one node's gradient and adds its
// contributions in a fixed order (incident elements ascending, then pairs in
// (slave, master) order; what depends on the slave element alone comes summed
// over its pairs).  Shared by the single-interface and batched kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mt_internal.h"

namespace mt {

// Components k0 .. k0 + N - 1 of element e, whose pairs are p0 .. p1 - 1
// (p1 > p0): its first part, then the parts of later tiles in order (one
// element in about 64 / pairs per element reaches into a second tile).
template <int N>
__device__ __forceinline__ void elem_sums(const ElemSums& E, int k0, int e, int p0, int p1, double v[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = E.v[(int64_t)(k0 + k) * E.stride + e];
  for (int t = p0 / TILE_PAIRS + 1; t <= (p1 - 1) / TILE_PAIRS; ++t)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += E.v[(int64_t)(k0 + k) * E.stride + E.n_el + t];
}

// Places of the four entries of block row j of pair (or element) i within
// their CSR row, of len columns: up to POS_PACKED columns as four bytes of
// the word at pos[4 j * stride + i], else one word each at
// pos[(4 j + l) * stride + i].  16 bytes a pair instead of 64 to write and
// to read, one load instead of four: at wavy 1024 x 1024 / 777 x 777 the
// positions 0.203 -> 0.173 ms, the assembly 0.316 -> 0.311 (0.269 since D and M
// rows are apart), the reverse sweep 0.569 -> 0.577 (its gathers wait as
// before, and unpack).
constexpr int POS_PACKED = 256;

__device__ __forceinline__ void store_pos4(int32_t* __restrict__ pos, int64_t stride, int64_t i, int j, int len,
                                           const int ix[4]) {
  if (len <= POS_PACKED) {
    pos[(int64_t)(4 * j) * stride + i] = (int32_t)((uint32_t)ix[0] | (uint32_t)ix[1] << 8 | (uint32_t)ix[2] << 16 |
                                                   (uint32_t)ix[3] << 24);
  } else {
#pragma unroll
    for (int l = 0; l < 4; ++l) pos[(int64_t)(4 * j + l) * stride + i] = ix[l];
  }
}

__device__ __forceinline__ void load_pos4(const int32_t* __restrict__ pos, int64_t stride, int64_t i, int j, int len,
                                          int ix[4]) {
  const uint32_t w = (uint32_t)pos[(int64_t)(4 * j) * stride + i];  // (both forms start here)
#pragma unroll
  for (int l = 0; l < 4; ++l) ix[l] = (int)(w >> (8 * l) & 255u);
  if (len > POS_PACKED) {
    ix[0] = (int)w;
#pragma unroll
    for (int l = 1; l < 4; ++l) ix[l] = pos[(int64_t)(4 * j + l) * stride + i];
  }
}

// The starts of the CSR rows of a slave element's four nodes, D's at
// erow[8 e ..] and M's at erow[8 e + 4 ..], with the sign bit set where the
// row has more than POS_PACKED columns (elements with pairs only): what the
// reverse sweep needs to turn places into positions, without the way over
// the connectivity and the row pointers (0.591 ms that way, 0.577 so).
__device__ __forceinline__ int row_start(int r0, int len) { return len <= POS_PACKED ? r0 : r0 | (int)0x80000000; }

// Upstream weights of the 16 block entries, r[j] the marked start of row j:
// W[4 j + l] = w[start of row j + place l].  One branch for the four rows,
// behind all loads of places.
__device__ __forceinline__ void load_weights(const double* __restrict__ w, int4 rows, const int32_t* __restrict__ pos,
                                             int64_t stride, int64_t i, double W[16]) {
  const int r[4] = {rows.x, rows.y, rows.z, rows.w};
  uint32_t word[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) word[j] = (uint32_t)pos[(int64_t)(4 * j) * stride + i];
  if ((r[0] | r[1] | r[2] | r[3]) >= 0) {
#pragma unroll
    for (int k = 0; k < 16; ++k) W[k] = w[r[k / 4] + (int)(word[k / 4] >> (8 * (k % 4)) & 255u)];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int ix[4];
      load_pos4(pos, stride, i, j, r[j] < 0 ? POS_PACKED + 1 : 0, ix);
#pragma unroll
      for (int l = 0; l < 4; ++l) W[4 * j + l] = w[(r[j] & 0x7fffffff) + ix[l]];
    }
  }
}

__device__ __forceinline__ int4 load_erow(const int32_t* __restrict__ erow, int64_t e, int m) {
  return reinterpret_cast<const int4*>(erow)[2 * e + m];
}

// The pairs that one node's row gathers, as one flat sequence k = 0 .. n-1:
// the pairs of its incident elements (ascending), each element's pairs in
// their order.  Up to four incident elements are held in registers, so the
// loads of several consecutive pairs can be issued before any of them is
// added; the additions still run in the sequence order, so the sums are the
// same bit for bit as those of the plain nested loops (used for nodes with
// more than four elements).
constexpr int ROW_RUNS = 4;

struct RowRuns {
  int e[ROW_RUNS];   // incident element
  int j[ROW_RUNS];   // local index of the node in it
  int p0[ROW_RUNS];  // first pair (or pair position) of the element
  int c1, c2, c3;    // flat index at which elements 1, 2, 3 start
  int n;             // number of pairs in all
};

// Runs of the ni <= ROW_RUNS incidences inc_list[i0 ..]; element e's pairs
// are lo[e] .. hi[e] - 1.
__device__ __forceinline__ void load_runs(int i0, int ni, const int32_t* __restrict__ inc_list,
                                          const int32_t* __restrict__ lo, const int32_t* __restrict__ hi,
                                          RowRuns& R) {
  int l[ROW_RUNS], h[ROW_RUNS];
#pragma unroll
  for (int t = 0; t < ROW_RUNS; ++t) {
    const int v = t < ni ? inc_list[i0 + t] : 0;
    R.e[t] = v >> 2;
    R.j[t] = v & 3;
  }
#pragma unroll
  for (int t = 0; t < ROW_RUNS; ++t) {
    l[t] = t < ni ? lo[R.e[t]] : 0;
    h[t] = t < ni ? hi[R.e[t]] : 0;
    R.p0[t] = l[t];
  }
  R.c1 = h[0] - l[0];
  R.c2 = R.c1 + (h[1] - l[1]);
  R.c3 = R.c2 + (h[2] - l[2]);
  R.n = R.c3 + (h[3] - l[3]);
}

// Local index j and pair p of flat position k (0 <= k < n); empty elements
// are skipped because their start equals the next one's.
__device__ __forceinline__ int run_at(const RowRuns& R, int k, int& j) {
  int base = 0, p0 = R.p0[0];
  j = R.j[0];
  if (k >= R.c1) { base = R.c1; p0 = R.p0[1]; j = R.j[1]; }
  if (k >= R.c2) { base = R.c2; p0 = R.p0[2]; j = R.j[2]; }
  if (k >= R.c3) { base = R.c3; p0 = R.p0[3]; j = R.j[3]; }
  return p0 + (k - base);
}

// pairs whose loads the gradient gathers issue together
constexpr int ROW_BATCH = 8;

// One sweep over the incident elements of row a (ascending, then their
// pairs), len columns long, for its D part (MP false; the gap is returned) or
// its M part (from the pairs' blocks blk[c * stride + p]): add(column, value)
// for every contribution, in order.
template <bool MP, class F>
__device__ __forceinline__ double row_sweep(int a, const int32_t* __restrict__ inc_off,
                                            const int32_t* __restrict__ inc_list,
                                            const int32_t* __restrict__ pair_off, int len,
                                            const int32_t* __restrict__ pos, const double* __restrict__ blk,
                                            int64_t stride, const ElemSums& E, F add) {
  double g = 0.0;
  for (int i = inc_off[a]; i < inc_off[a + 1]; ++i) {
    const int e = inc_list[i] >> 2, j = inc_list[i] & 3;
    const int p0 = pair_off[e], p1 = pair_off[e + 1];
    if (p0 == p1) continue;
    int ix[4];
    double v[4];
    if (!MP) {
      double vg[1];
      load_pos4(pos, E.n_el, e, j, len, ix);
      elem_sums<4>(E, 4 * j, e, p0, p1, v);
      elem_sums<1>(E, 16 + j, e, p0, p1, vg);
      g += vg[0];
#pragma unroll
      for (int k = 0; k < 4; ++k) add(ix[k], v[k]);
    } else {
      for (int p = p0; p < p1; ++p) {
        load_pos4(pos, stride, p, j, len, ix);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = blk[(int64_t)(j * 4 + k) * stride + p];
#pragma unroll
        for (int k = 0; k < 4; ++k) add(ix[k], v[k]);
      }
    }
  }
  return g;
}

// Row a of D with the gap (MP false) or of M, accumulated in a per-thread
// segment of cap entries, acc[i * astride], and written once; a row of up to
// ROW_WINDOWS segments in as many sweeps, a longer one in global memory.
// Every entry receives its contributions in the same order in all forms.
// (Issuing the loads of several pairs together, as the gradient gathers
// below do, measured slower here: the row's LDS updates, not its loads, set
// the pace.)
constexpr int ROW_WINDOWS = 4;

template <bool MP>
__device__ __forceinline__ void assemble_row(int a, const int32_t* __restrict__ inc_off,
                                             const int32_t* __restrict__ inc_list,
                                             const int32_t* __restrict__ pair_off,
                                             const int32_t* __restrict__ rowptr, const int32_t* __restrict__ pos,
                                             const double* __restrict__ blk, int64_t stride, const ElemSums& E,
                                             double* __restrict__ val, double* __restrict__ gap, double* acc,
                                             int astride, int cap) {
  const int r0 = rowptr[a], u = rowptr[a + 1] - r0;
  val += r0;
  double g = 0.0;
  if (u <= cap) {
    for (int i = 0; i < u; ++i) acc[i * astride] = 0.0;
    g = row_sweep<MP>(a, inc_off, inc_list, pair_off, u, pos, blk, stride, E,
                      [&](int i, double v) { acc[i * astride] += v; });
    for (int i = 0; i < u; ++i) val[i] = acc[i * astride];
  } else if (u <= ROW_WINDOWS * cap) {
    for (int w = 0; w < u; w += cap) {
      const int n = min(cap, u - w);
      for (int i = 0; i < n; ++i) acc[i * astride] = 0.0;
      g = row_sweep<MP>(a, inc_off, inc_list, pair_off, u, pos, blk, stride, E, [&](int i, double v) {
        if (i >= w && i < w + n) acc[(i - w) * astride] += v;
      });
      for (int i = 0; i < n; ++i) val[w + i] = acc[i * astride];
    }
  } else {
    for (int i = 0; i < u; ++i) val[i] = 0.0;
    g = row_sweep<MP>(a, inc_off, inc_list, pair_off, u, pos, blk, stride, E,
                      [&](int i, double v) { val[i] += v; });
  }
  if (!MP) gap[a] = g;
}

// Accumulator entries per thread of the assembly kernels: M rows of 5 x 5
// master nodes fit, and LDS leaves room for 12 wavefronts on a CU; where the
// masters are finer, rows of 6 x 6 (8 wavefronts).  Assembly alone, wavy,
// 26 -> 36 entries, by the ratio of elements per side: 0.76 270 -> 295 us
// (1024 slave elements a side), 1.0 39.7 -> 42.1, 1.2 57.9 -> 58.5, 1.3 67.6
// -> 66.7, 1.4 75.7 -> 74.7, 1.5 101 -> 84, 1.6 154 -> 94, 2.0 313 -> 156
// (400 a side; with 32 entries 102, 136 and 276 at the last three): the line
// at 1.26 in this ratio, 1.6 in the elements.
constexpr int ROW_ACC = 26;
constexpr int ROW_ACC_FINE = 36;
inline bool fine_masters(int64_t n_s_el, int64_t n_m_el) { return 10 * n_m_el > 16 * n_s_el; }

// Sum over the flat pair sequence of R of the three components
// gpair[(3 j + d) * stride + p], d = 0, 1, 2, in sequence order.
__device__ __forceinline__ void gather3(const RowRuns& R, const double* __restrict__ gpair, int64_t stride,
                                        double& g0, double& g1, double& g2) {
  constexpr int U = ROW_BATCH;
  for (int k0 = 0; k0 < R.n; k0 += U) {
    double v[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // positions past the end reload the last pair and are not added
      int j;
      const int p = run_at(R, min(k0 + u, R.n - 1), j);
#pragma unroll
      for (int d = 0; d < 3; ++d) v[u][d] = gpair[(int64_t)(3 * j + d) * stride + p];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u < R.n) {
        g0 += v[u][0];
        g1 += v[u][1];
        g2 += v[u][2];
      }
    }
  }
}

// Gradient of slave node a (structure-of-arrays gX[3 * n]): the sum over its
// incident elements, ascending.
__device__ __forceinline__ void grad_slave_row(int a, int32_t n, const int32_t* __restrict__ inc_off,
                                               const int32_t* __restrict__ inc_list,
                                               const int32_t* __restrict__ pair_off, const ElemSums& E,
                                               double* __restrict__ gX) {
  double g[3] = {0.0, 0.0, 0.0};
  for (int i = inc_off[a]; i < inc_off[a + 1]; ++i) {
    const int e = inc_list[i] >> 2, j = inc_list[i] & 3;
    const int p0 = pair_off[e], p1 = pair_off[e + 1];
    if (p0 == p1) continue;
    double v[3];
    elem_sums<3>(E, 3 * j, e, p0, p1, v);
#pragma unroll
    for (int d = 0; d < 3; ++d) g[d] += v[d];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) gX[(int64_t)d * n + a] = g[d];
}

// Gradient of master node b: the master components of the pairs are staged
// in pairs-by-master order (position k of pair p = its rank in that order),
// so the pairs of master element m are the contiguous range
// mstart[m] .. mend[m].
__device__ __forceinline__ void grad_master_row(int b, int32_t n, const int32_t* __restrict__ inc_off,
                                                const int32_t* __restrict__ inc_list,
                                                const int32_t* __restrict__ mstart, const int32_t* __restrict__ mend,
                                                const double* __restrict__ gpair, int64_t stride,
                                                double* __restrict__ gX) {
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;
  const int i0 = inc_off[b], ni = inc_off[b + 1] - i0;
  if (ni <= ROW_RUNS) {
    RowRuns R;
    load_runs(i0, ni, inc_list, mstart, mend, R);
    gather3(R, gpair, stride, g0, g1, g2);
  } else {
    for (int i = i0; i < i0 + ni; ++i) {
      const int m = inc_list[i] >> 2, l = inc_list[i] & 3;
      for (int k = mstart[m]; k < mend[m]; ++k) {
        g0 += gpair[(int64_t)(3 * l + 0) * stride + k];
        g1 += gpair[(int64_t)(3 * l + 1) * stride + k];
        g2 += gpair[(int64_t)(3 * l + 2) * stride + k];
      }
    }
  }
  gX[b] = g0;
  gX[(int64_t)n + b] = g1;
  gX[2 * (int64_t)n + b] = g2;
}

}  // namespace mt
