// Contact search on the GPU: element preparation, master elements counted
// into Cartesian bins, and the candidate lists of every slave element from its own bin and the 26 neighbouring bins
// (Alg. 2 and its bin-sizing rule, Sec. "Distributed storage: going to large
// problems").
#include <cmath>
#include <algorithm>
#include <cstring>

#include "mt_geometry.h"
#include "mt_scan.h"

namespace mt {

namespace {

constexpr int BS = 256;
constexpr int PREP_PART = 9;  // per-block partials: ext, edge, -lo xyz, hi xyz, bad (bits)

__device__ __forceinline__ unsigned long long order_key(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__host__ __device__ inline double from_order_key(unsigned long long k) {
  const unsigned long long b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  double x;
  memcpy(&x, &b, sizeof(x));
  return x;
}

template <class T>
__device__ __forceinline__ T wave_max(T x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const T y = __shfl_xor(x, d, 64);
    x = x > y ? x : y;
  }
  return x;
}

// Element preparation: bounding boxes, the grid reductions (largest box
// extent, longest slave edge, bounding box of all element boxes), for slave
// elements the precomputed frame and projected polygon of the candidate
// pass, for master elements their node coordinates gathered element by
// element (md[12 e + 3 k + d], read with 16-byte loads by the candidate
// pass).  Both sides in one launch (blockIdx.y: 0 slave, 1 master), so that
// the shorter master pass fills the slave pass's tail; within a side a
// grid-stride loop over its P.nb blocks, each writing its partials of the
// reductions to P.part[block].
struct PrepSide {
  const double* x;
  const double* y;
  const double* z;
  const int32_t* conn;
  const double* nrm;  // slave element plane normals (continuous field) or null
  double* box;
  double* sd;  // slave: frame data
  double* md;  // master: gathered node coordinates
  double* part;
  int32_t n_el, n_nodes, nb;
};

__global__ __launch_bounds__(BS) void k_prep(PrepSide s_side, PrepSide m_side) {
  const bool slave = blockIdx.y == 0;
  const PrepSide& P = slave ? s_side : m_side;
  if ((int)blockIdx.x >= P.nb) return;  // the whole block: the side has fewer blocks
  const double* __restrict__ x = P.x;
  const double* __restrict__ y = P.y;
  const double* __restrict__ z = P.z;
  const int32_t* __restrict__ conn = P.conn;
  const int32_t n_el = P.n_el, n_nodes = P.n_nodes;
  const double* __restrict__ nrm = P.nrm;
  double* __restrict__ box = P.box;
  double* __restrict__ sd = P.sd;
  double* __restrict__ md = P.md;
  double* __restrict__ part = P.part;
  __shared__ double sh[BS / 64][8];
  __shared__ int bad;  // 1: connectivity out of range, 2: a coordinate not finite
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  double ext = 0.0, edge = 0.0;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int e = blockIdx.x * BS + threadIdx.x; e < n_el; e += P.nb * BS) {
    const int4 c = load_conn(conn, e);
    const bool ok = c.x >= 0 && c.y >= 0 && c.z >= 0 && c.w >= 0 && c.x < n_nodes && c.y < n_nodes &&
                    c.z < n_nodes && c.w < n_nodes;
    if (!ok) {
      atomicOr(&bad, 1);
      continue;
    }
    double X[4][3];
    load_nodes(x, y, z, c, X);
    bool fin = true;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int d = 0; d < 3; ++d) fin = fin && isfinite(X[k][d]);
    if (!fin) atomicOr(&bad, 2);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double l = fmin(fmin(X[0][d], X[1][d]), fmin(X[2][d], X[3][d]));
      const double h = fmax(fmax(X[0][d], X[1][d]), fmax(X[2][d], X[3][d]));
      box[(int64_t)d * n_el + e] = l;
      box[(int64_t)(3 + d) * n_el + e] = h;
      ext = fmax(ext, h - l);
      lo[d] = fmin(lo[d], l);
      hi[d] = fmax(hi[d], h);
    }
    if (slave) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int k1 = (k + 1) & 3;
        const double a = X[k1][0] - X[k][0], b = X[k1][1] - X[k][1], cc = X[k1][2] - X[k][2];
        edge = fmax(edge, sqrt(a * a + b * b + cc * cc));
      }
      double f[12], hs[4], As, hmax;
      V2 S[4];
      slave_frame_p(X, nrm ? nrm + 4 * (int64_t)e : nullptr, f);
      slave_setup(X, f, S, hs, As, hmax);
#pragma unroll
      for (int k = 0; k < 12; ++k) sd[(int64_t)k * n_el + e] = f[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        sd[(int64_t)(12 + k) * n_el + e] = S[k].u;
        sd[(int64_t)(16 + k) * n_el + e] = S[k].v;
      }
      sd[(int64_t)20 * n_el + e] = As;
      sd[(int64_t)21 * n_el + e] = hmax;
    } else {
      double2* dst = reinterpret_cast<double2*>(md + (int64_t)12 * e);
#pragma unroll
      for (int k = 0; k < 6; ++k) dst[k] = make_double2(X[(2 * k) / 3][(2 * k) % 3], X[(2 * k + 1) / 3][(2 * k + 1) % 3]);
    }
  }
  double v[8] = {ext, edge, -lo[0], -lo[1], -lo[2], hi[0], hi[1], hi[2]};
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = wave_max(v[k]);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < 8; ++k) sh[w][k] = v[k];
  __syncthreads();
  if (threadIdx.x < 8) {
    double m = sh[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < BS / 64; ++i) m = fmax(m, sh[i][threadIdx.x]);
    part[(int64_t)blockIdx.x * PREP_PART + threadIdx.x] = m;
  }
  if (threadIdx.x == 8) part[(int64_t)blockIdx.x * PREP_PART + 8] = (double)bad;
}

__device__ Grid grid_from(const PrepReduce& red, double delta, double bin_size, int64_t max_cells);

// Final reduction of the per-block partials of both sides (nb_s slave
// blocks first, then nb_m master blocks) into the grid quantities and the
// search grid from them (grid_from, one thread).  Every workgroup does this
// for itself, so that all of them can clear their part of the grid's cell
// counts without another launch; the first one also writes the state (zero
// but for the grid and the flags) and zeroes the counters.  Bound by the
// latency of the partials' loads and of grid_from.
__global__ __launch_bounds__(BS) void k_prep_reduce(const double* __restrict__ part, int nb_s, int nb_m,
                                                     double delta, double bin_size, int64_t max_cells, DevState* st,
                                                     Counters* cnt, int32_t* __restrict__ cell_cnt) {
  __shared__ double sh[BS / 64][PREP_PART];
  __shared__ Grid sgrid;
  double v[PREP_PART];
#pragma unroll
  for (int k = 0; k < PREP_PART; ++k) v[k] = k == 0 || k == 1 || k == 8 ? 0.0 : -INFINITY;
  int bits = 0;
  for (int b = threadIdx.x; b < nb_s + nb_m; b += BS) {
#pragma unroll
    for (int k = 0; k < PREP_PART - 1; ++k) {
      const double x = part[(int64_t)b * PREP_PART + k];
      if (k != 1 || b < nb_s) v[k] = fmax(v[k], x);
    }
    bits |= (int)part[(int64_t)b * PREP_PART + 8];
  }
  __shared__ int sbits;
  if (threadIdx.x == 0) sbits = 0;
  if (blockIdx.x == 0) {
    static_assert(sizeof(Counters) % 4 == 0 && sizeof(DevState) % 4 == 0, "word fills");
    for (unsigned i = threadIdx.x; i < sizeof(Counters) / 4; i += BS) reinterpret_cast<int32_t*>(cnt)[i] = 0;
    for (unsigned i = threadIdx.x; i < sizeof(DevState) / 4; i += BS) reinterpret_cast<int32_t*>(st)[i] = 0;
  }
  __syncthreads();
  if (bits) atomicOr(&sbits, bits);
#pragma unroll
  for (int k = 0; k < PREP_PART; ++k) v[k] = wave_max(v[k]);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < PREP_PART; ++k) sh[threadIdx.x >> 6][k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    double r[PREP_PART];
#pragma unroll
    for (int k = 0; k < PREP_PART; ++k) {
      r[k] = sh[0][k];
#pragma unroll
      for (int i = 1; i < BS / 64; ++i) r[k] = fmax(r[k], sh[i][k]);
    }
    PrepReduce red;
    red.emax_bits = (unsigned long long)__double_as_longlong(r[0]);
    red.edge_bits = (unsigned long long)__double_as_longlong(r[1]);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      red.lo_key[d] = r[2 + d] > -INFINITY ? order_key(-r[2 + d]) : ~0ull;
      red.hi_key[d] = r[5 + d] > -INFINITY ? order_key(r[5 + d]) : 0ull;
    }
    sgrid = grid_from(red, delta, bin_size, max_cells);
    if (blockIdx.x == 0) {
      st->grid = sgrid;
      st->flags = (sbits & 2) ? DS_NONFINITE : 0u;
    }
  }
  __syncthreads();
  const int64_t nc = sgrid.ncells;
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < nc; i += (int64_t)gridDim.x * BS) cell_cnt[i] = 0;
}

// Cell index along one axis, clamped to [0, n); a NaN position (a
// non-finite coordinate, reported by the preparation) lands in cell 0.
__device__ __forceinline__ int cell_coord(double c, double lo, double inv_beta, int n) {
  double t = floor((c - lo) * inv_beta);
  t = fmax(t, 0.0);
  t = fmin(t, (double)(n - 1));
  return (int)t;
}

// ---- box prefilter ------------------------------------------------------------
// The candidate test compares (slave lo - delta) with master hi and master lo
// with (slave hi + delta) on each axis.  Master box bounds are stored as
// quantisation levels (21 bits each, one 16-byte record per master): level q
// of axis d stands for B(q) = qo + q qu, computed the same way wherever it is
// used, so B is non-decreasing in q, and a master bound x is stored as the
// largest q with B(q) <= x (then B(q) <= x < B(q + 1)).  For each slave the
// walk computes, per axis, the levels around a = lo - delta and c = hi +
// delta; a test is then decided by integer comparisons when the levels
// separate the values, and by the exact FP64 test otherwise, so the
// candidate list is the one of the exact test.
constexpr int QBITS = 21;
constexpr int64_t QMAX = (int64_t(1) << QBITS) - 1;
constexpr uint64_t QMASK = (uint64_t(1) << QBITS) - 1;
constexpr uint64_t QEXACT = uint64_t(1) << 63;  // record flag: exact test only

__device__ __forceinline__ double qlevel(const Grid& g, int d, int64_t q) { return g.qo[d] + (double)q * g.qu[d]; }

// max{q in [0, QMAX + 1] : B(q) <= x (B(q) < x when strict)}, -1 when there is
// none; x finite.  A guess, a few unit steps, then bisection.
__device__ int64_t q_max_le(const Grid& g, int d, double x, bool strict) {
  auto ok = [&](int64_t q) {
    const double b = qlevel(g, d, q);
    return strict ? b < x : b <= x;
  };
  const double f = floor((x - g.qo[d]) / g.qu[d]);
  int64_t q = (int64_t)fmin(fmax(f, -1.0), (double)(QMAX + 1));
  for (int it = 0; it < 4; ++it) {
    if (q >= 0 && !ok(q)) {
      --q;
    } else if (q <= QMAX && ok(q + 1)) {
      ++q;
    } else {
      return q;
    }
  }
  int64_t lo = -1, hi = QMAX + 2;  // ok(lo) and !ok(hi), taken as given at the ends
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (ok(mid))
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Per-slave thresholds of the prefilter: on axis d a master with levels
// (ql, qh) fails when qh < ea or ql > ecf, passes when qh > la and ql < ecp;
// anything else goes to the exact test.
struct QSlave {
  int32_t la[3], ea[3], ecp[3], ecf[3];
};

__device__ __forceinline__ QSlave q_slave(const Grid& g, const double lo[3], const double hi[3], double delta) {
  QSlave t;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double a = lo[d] - delta, c = hi[d] + delta;  // as in the exact test
    if (isfinite(a) && isfinite(c)) {
      t.la[d] = (int32_t)q_max_le(g, d, a, true);
      t.ea[d] = (int32_t)q_max_le(g, d, a, false);
      t.ecp[d] = t.ecf[d] = (int32_t)q_max_le(g, d, c, false);
    } else {  // never decided by the levels
      t.la[d] = (int32_t)QMAX + 1;
      t.ea[d] = -1;
      t.ecp[d] = -1;
      t.ecf[d] = (int32_t)QMAX + 1;
    }
  }
  return t;
}

// Search grid from the element reductions (one thread):
// beta_min = max(longest slave edge, largest box extent + delta, bin_size)
// (the paper's rule without a motion term, raised so that 27 cells are
// complete), the node bounding box expanded by beta_min, max(1, floor(L /
// beta_min)) cells per axis, the dense cell table coarsened to at most
// max_cells cells (coarser cells stay complete).
__device__ Grid grid_from(const PrepReduce& red, double delta, double bin_size, int64_t max_cells) {
  const double emax = __longlong_as_double((long long)red.emax_bits);
  const double edge = __longlong_as_double((long long)red.edge_bits);
  double beta_min = fmax(fmax(edge, emax + delta), bin_size) * (1.0 + 0x1p-20);
  if (!(beta_min > 0.0) || !isfinite(beta_min)) beta_min = 1.0;
  Grid g;
  double L[3];
  int64_t n[3];
  for (int d = 0; d < 3; ++d) {
    double lo = from_order_key(red.lo_key[d]);
    double hi = from_order_key(red.hi_key[d]);
    if (!(lo <= hi) || !isfinite(lo) || !isfinite(hi)) { lo = 0.0; hi = 0.0; }
    g.lo[d] = lo - beta_min;
    L[d] = (hi + beta_min) - g.lo[d];
    const double q = floor(L[d] / beta_min);
    n[d] = q >= 1.0 ? (q < (double)max_cells ? (int64_t)q : max_cells) : 1;
  }
  // (the product in double: three factors up to max_cells overflow int64)
  while ((double)n[0] * (double)n[1] * (double)n[2] > (double)max_cells) {
    const double f = cbrt((double)n[0] * (double)n[1] * (double)n[2] / (double)max_cells) * 1.01;
    for (int d = 0; d < 3; ++d) {
      const double q = floor((double)n[d] / f);
      n[d] = q >= 1.0 ? (int64_t)q : 1;
    }
  }
  for (int d = 0; d < 3; ++d) {
    g.n[d] = (int32_t)n[d];
    g.beta[d] = L[d] / (double)n[d];
    g.inv_beta[d] = 1.0 / g.beta[d];
  }
  g.ncells = n[0] * n[1] * n[2];
  // quantisation of the prefilter: levels from the grid's low corner in
  // steps of a power of two, QMAX + 1 of them spanning at least twice the
  // grid, so every box bound of the grid lies between levels 0 and QMAX
  for (int d = 0; d < 3; ++d) {
    g.qo[d] = g.lo[d];
    int e = 0;
    (void)frexp(2.0 * L[d] / (double)QMAX, &e);
    g.qu[d] = L[d] > 0.0 && isfinite(L[d]) ? ldexp(1.0, e) : 1.0;
  }
  // padded so that rounding in the box centres cannot move a centre across
  g.reach = (delta + 0.5 * emax) * (1.0 + 1e-9) + 1e-9 * beta_min;
  return g;
}


// Cell of each master box centre, and the master's place among those of its
// cell in arrival order (the candidate lists are ordered by master index
// afterwards, so it does not matter which order the atomics take).
__global__ __launch_bounds__(BS) void k_cell_count(const double* __restrict__ box, int32_t n,
                                                    const Grid* __restrict__ gp, int32_t* __restrict__ cell_cnt,
                                                    uint32_t* __restrict__ cell, uint32_t* __restrict__ rank) {
  const int m = blockIdx.x * BS + threadIdx.x;
  if (m >= n) return;
  const Grid& g = *gp;
  int ix[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double c = 0.5 * (box[(int64_t)d * n + m] + box[(int64_t)(3 + d) * n + m]);
    ix[d] = cell_coord(c, g.lo[d], g.inv_beta[d], g.n[d]);
  }
  const uint32_t k = (uint32_t)(ix[0] + g.n[0] * (ix[1] + g.n[1] * ix[2]));
  cell[m] = k;
  rank[m] = (uint32_t)atomicAdd(&cell_cnt[k], 1);
}

// Masters in cell order: index vals[i] and box (sbox[i] = lo xyz, hi xyz) of
// the i-th, so that the candidate walks read them contiguously.
__global__ __launch_bounds__(BS) void k_cell_place(const uint32_t* __restrict__ cell,
                                                    const uint32_t* __restrict__ rank, int32_t n,
                                                    const double* __restrict__ box_m, const Grid* __restrict__ gp,
                                                    const int32_t* __restrict__ cell_start,
                                                    uint32_t* __restrict__ vals, double* __restrict__ sbox,
                                                    uint64_t* __restrict__ qbox) {
  const int m = blockIdx.x * BS + threadIdx.x;
  if (m >= n) return;
  const int64_t i = (int64_t)cell_start[cell[m]] + rank[m];
  vals[i] = (uint32_t)m;
  double bx[6];
#pragma unroll
  for (int j = 0; j < 6; ++j) bx[j] = box_m[(int64_t)j * n + m];
  double2* dst = reinterpret_cast<double2*>(sbox + (int64_t)6 * i);
  dst[0] = make_double2(bx[0], bx[1]);
  dst[1] = make_double2(bx[2], bx[3]);
  dst[2] = make_double2(bx[4], bx[5]);
  // quantised record: lo levels in the first word, hi levels in the second
  const Grid g = *gp;
  uint64_t w[2] = {0, 0};
  bool exact = false;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const int d = j % 3;
    int64_t q = -1;
    if (isfinite(bx[j])) q = q_max_le(g, d, bx[j], false);
    if (q < 0 || q > QMAX) {
      exact = true;
      q = 0;
    }
    w[j / 3] |= (uint64_t)q << (QBITS * d);
  }
  if (exact) w[1] |= QEXACT;
  reinterpret_cast<ulonglong2*>(qbox)[i] = make_ulonglong2(w[0], w[1]);
}

struct SlaveBox {
  double lo[3], hi[3];
};

__device__ __forceinline__ SlaveBox load_box(const double* __restrict__ box, int32_t n, int e) {
  SlaveBox b;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    b.lo[d] = box[(int64_t)d * n + e];
    b.hi[d] = box[(int64_t)(3 + d) * n + e];
  }
  return b;
}

// Candidate test: closed overlap of the delta-enlarged slave box and the
// i-th master box in cell order on all three axes.
__device__ __forceinline__ bool touch(const SlaveBox& s, const double* __restrict__ sbox, int i, double delta) {
  const double2* b = reinterpret_cast<const double2*>(sbox + (int64_t)6 * i);
  const double2 b0 = b[0], b1 = b[1], b2 = b[2];
  const double mlo[3] = {b0.x, b0.y, b1.x}, mhi[3] = {b1.y, b2.x, b2.y};
  bool t = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) t = t && (s.lo[d] - delta) <= mhi[d] && mlo[d] <= (s.hi[d] + delta);
  return t;
}

// The candidate test through the quantised record first (one 16-byte load);
// the exact test only when the levels do not decide it.
__device__ __forceinline__ bool touch_q(const SlaveBox& s, const QSlave& t, const double* __restrict__ sbox,
                                        const uint64_t* __restrict__ qbox, int i, double delta) {
  const ulonglong2 rec = reinterpret_cast<const ulonglong2*>(qbox)[i];
  bool fail = false, pass = (rec.y & QEXACT) == 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int32_t ql = (int32_t)((rec.x >> (QBITS * d)) & QMASK);
    const int32_t qh = (int32_t)((rec.y >> (QBITS * d)) & QMASK);
    fail = fail || qh < t.ea[d] || ql > t.ecf[d];
    pass = pass && qh > t.la[d] && ql < t.ecp[d];
  }
  if ((rec.y & QEXACT) == 0) {
    if (fail) return false;
    if (pass) return true;
  }
  return touch(s, sbox, i, delta);
}

constexpr int CCAP = 48;  // per-thread LDS segment of the long-list fill (masters)
constexpr int CTMP = 32;  // candidates per slave kept by the count pass
// lanes per slave element (template argument G) in the count and fill passes;
// groups do not straddle a wavefront
constexpr int LANES_MANY = 2, LANES_FEW = 8;
// Up to this many slave elements 8 lanes each: two would leave SIMDs idle, and
// the passes' time is one lane's serial walk.  Whole step, wavy, without
// read-back, 2 -> 8 lanes: 16K slave elements 232 -> 224 us, 33K 254 -> 250,
// 66K 318 -> 331 (4 lanes 225, 250, 318; 16 lanes 227, 262, 364).
constexpr int32_t FEW_SLAVES = 32768;

// The 27 cells around the slave centre's cell, restricted to those that can
// hold the centre of a touching master (within g.reach of the box).
__device__ __forceinline__ void cell_window(const SlaveBox& b, const Grid& g, int c0[3], int c1[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int ic = cell_coord(0.5 * (b.lo[d] + b.hi[d]), g.lo[d], g.inv_beta[d], g.n[d]);
    c0[d] = max(ic - 1, cell_coord(b.lo[d] - g.reach, g.lo[d], g.inv_beta[d], g.n[d]));
    c1[d] = min(ic + 1, cell_coord(b.hi[d] + g.reach, g.lo[d], g.inv_beta[d], g.n[d]));
  }
}

// The cells x0 .. x1 of one (y, z) row are consecutive, so their masters are
// one run [lo, hi) of the cell-ordered list.
__device__ __forceinline__ void row_run(const int32_t* __restrict__ cell_start, int64_t row, int x0, int x1, int& lo,
                                        int& hi) {
  lo = cell_start[row + x0];
  hi = cell_start[row + x1 + 1];
}

// Candidates of one slave element: masters of its own and the 26 neighbouring
// cells whose boxes touch its delta-enlarged box, in walk order; the first
// vcap go to v[k * vs].  One lane per slave.
__device__ __forceinline__ int walk_cells(const SlaveBox& b, const double* __restrict__ sbox,
                                          const uint32_t* __restrict__ mvals, const int32_t* __restrict__ cell_start,
                                          const Grid& g, double delta, int32_t* v, int64_t vs, int vcap) {
  int c0[3], c1[3];
  cell_window(b, g, c0, c1);
  int c = 0;
  for (int zz = c0[2]; zz <= c1[2]; ++zz) {
    for (int yy = c0[1]; yy <= c1[1]; ++yy) {
      int lo, hi;
      row_run(cell_start, (int64_t)g.n[0] * (yy + (int64_t)g.n[1] * zz), c0[0], c1[0], lo, hi);
      for (int i = lo; i < hi; ++i) {
        if (touch(b, sbox, i, delta)) {
          if (c < vcap) v[c * vs] = (int)mvals[i];
          ++c;
        }
      }
    }
  }
  return c;
}

// Same walk by a group of G lanes of one wave (lane r of the group tests
// masters lo + r, lo + r + G, ...): the group's hits of one step are ranked
// by a wave ballot, so v receives the same candidates in the same order as
// the one-lane walk, and the boxes a group reads in one step are adjacent.
template <int G>
__device__ __forceinline__ int walk_cells_group(const SlaveBox& b, const double* __restrict__ sbox,
                                                const uint64_t* __restrict__ qbox,
                                                const uint32_t* __restrict__ mvals, const int32_t* __restrict__ cell_start,
                                                const Grid& g, double delta, int32_t* v, int64_t vs, int vcap, int r,
                                                int gshift) {
  int c0[3], c1[3];
  cell_window(b, g, c0, c1);
  const QSlave qs = q_slave(g, b.lo, b.hi, delta);
  const unsigned below = (1u << r) - 1u;
  int c = 0;
  for (int zz = c0[2]; zz <= c1[2]; ++zz) {
    for (int yy = c0[1]; yy <= c1[1]; ++yy) {
      int lo, hi;
      row_run(cell_start, (int64_t)g.n[0] * (yy + (int64_t)g.n[1] * zz), c0[0], c1[0], lo, hi);
      for (int i0 = lo; i0 < hi; i0 += G) {
        const int i = i0 + r;
        const bool hit = i < hi && touch_q(b, qs, sbox, qbox, i, delta);
        const unsigned m = (unsigned)(__ballot(hit) >> gshift) & ((1u << G) - 1u);
        if (hit) {
          const int k = c + __popc(m & below);
          if (k < vcap) v[k * vs] = (int)mvals[i];
        }
        c += __popc(m);
      }
    }
  }
  return c;
}

// Count pass, G lanes per slave: the number of candidates, and the first
// CTMP of them (walk order) in the lane-interleaved scratch tmp[k * n_s + s].
template <int G>
__global__ __launch_bounds__(BS) void k_cand_count(const double* __restrict__ box_s, int32_t n_s,
                                                    const double* __restrict__ sbox,
                                                    const uint64_t* __restrict__ qbox,
                                                    const uint32_t* __restrict__ mvals,
                                                    const int32_t* __restrict__ cell_start, const Grid* __restrict__ gp,
                                                    double delta, int32_t* __restrict__ count,
                                                    int32_t* __restrict__ tmp) {
  const int64_t t = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * BS + threadIdx.x;
  const int s = (int)(t / G), r = (int)(t % G);
  if (s >= n_s) return;  // whole groups leave together
  const Grid g = *gp;
  const SlaveBox b = load_box(box_s, n_s, s);
  const int c = walk_cells_group<G>(b, sbox, qbox, mvals, cell_start, g, delta, tmp + s, n_s, CTMP, r,
                                 (int)(__lane_id() & ~(G - 1)));
  if (r == 0) count[s] = c;
}

__device__ __forceinline__ void load_master_data(const double* __restrict__ md, int m, double X[4][3]) {
  const double2* src = reinterpret_cast<const double2*>(md + (int64_t)12 * m);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double2 t = src[k];
    X[(2 * k) / 3][(2 * k) % 3] = t.x;
    X[(2 * k + 1) / 3][(2 * k + 1) % 3] = t.y;
  }
}

// Screening of one candidate (master m of slave s, output slot ci) against
// the slave plane data: projection of the master nodes, degeneracy checks and
// the separating-line quick exit decide its vertex count nv_out[ci]: NV_CLIP
// where it is to be clipped (the clip overwrites it), otherwise 0.
constexpr uint8_t NV_CLIP = 255;

struct SlavePlane {
  double f[12], As;
  V2 S[4];
};

__device__ __forceinline__ void load_plane(const double* __restrict__ sd, int32_t n_s, int s, SlavePlane& P) {
#pragma unroll
  for (int k = 0; k < 12; ++k) P.f[k] = sd[(int64_t)k * n_s + s];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    P.S[k].u = sd[(int64_t)(12 + k) * n_s + s];
    P.S[k].v = sd[(int64_t)(16 + k) * n_s + s];
  }
  P.As = sd[(int64_t)20 * n_s + s];
}

struct ScreenOut {
  unsigned degen_s, degen_m;
};

__device__ __forceinline__ bool screen_one(const SlavePlane& P, int s, int m, int64_t ci,
                                           const double* __restrict__ md, double eps_a, int32_t* __restrict__ cand_s,
                                           int32_t* __restrict__ cand_m, uint8_t* __restrict__ nv_out,
                                           ScreenOut& so) {
  double Xm[4][3];
  load_master_data(md, m, Xm);
  V2 Mn[4];
  double hm[4];
  int st;
  bool flip;
  const bool clip = pair_screen(P.S, P.As, Xm, P.f, eps_a, Mn, hm, flip, st);
  nv_out[ci] = clip ? NV_CLIP : 0;
  so.degen_s += (st & PS_DEGEN_SLAVE) ? 1u : 0u;
  so.degen_m += (st & PS_DEGEN_MASTER) ? 1u : 0u;
  cand_m[ci] = m;
  cand_s[ci] = s;
  return clip;
}

__device__ __forceinline__ void count_degenerate(const ScreenOut& so, Counters* cnt) {
  // degenerate elements are rare: count them with global atomics
  if (so.degen_s) atomicAdd(&cnt->degen_slave, (unsigned long long)so.degen_s);
  if (so.degen_m) atomicAdd(&cnt->degen_master, (unsigned long long)so.degen_m);
}

// Fill pass for slaves with at most CTMP candidates, G lanes per slave: lane
// r takes the candidates r, r + G, ... of the count pass's list, finds the
// place of each in the master-sorted order by counting the smaller masters
// of the list (the masters of one slave are distinct), screens it and writes
// it there.  No lane reads what another lane wrote; the group's number of
// screened-in candidates (to scr_cnt[s]) is summed by lane shuffles.
//
// About half the time is VALU issue, the rest latency at 4 wavefronts per
// SIMD (the masters' records staged through LDS by the whole wavefront, a
// third of the cache accesses: no faster).  The screening marks the vertex
// count and keeps no array of its own.  Wavy 1024 x 1024 / 777 x 777: 0.28 ms
// and 0.040 ms for the list of the screened-in with a 4-byte flag per
// candidate, 0.25 and 0.018 ms now.
template <int G>
__device__ __forceinline__ void fill_short(int s, int r, int32_t n_s, int base, int c,
                                           const int32_t* __restrict__ tmp, int32_t* __restrict__ cand_s,
                                           int32_t* __restrict__ cand_m, const double* __restrict__ sd,
                                           const double* __restrict__ md, double eps_a, uint8_t* __restrict__ nv_out,
                                           int32_t* __restrict__ scr_cnt, Counters* cnt, int64_t cap) {
  if (base < 0 || (int64_t)base + c > cap) {  // output too short: the host sizes it, runs the pass again
    if (r == 0) scr_cnt[s] = 0;
    return;
  }
  int nscr = 0;
  if (r < c) {
    constexpr int OWN = CTMP / G;  // candidates per lane
    int own[OWN], rank[OWN];
#pragma unroll
    for (int q = 0; q < OWN; ++q) {
      const int k = r + q * G;
      own[q] = k < c ? tmp[(int64_t)k * n_s + s] : 0x7fffffff;
      rank[q] = 0;
    }
    for (int k = 0; k < c; ++k) {
      const int x = tmp[(int64_t)k * n_s + s];
#pragma unroll
      for (int q = 0; q < OWN; ++q) rank[q] += x < own[q] ? 1 : 0;
    }
    SlavePlane P;
    load_plane(sd, n_s, s, P);
    ScreenOut so{0u, 0u};
    for (int q = 0; q < OWN && r + q * G < c; ++q)
      nscr += screen_one(P, s, own[q], (int64_t)base + rank[q], md, eps_a, cand_s, cand_m, nv_out, so) ? 1 : 0;
    count_degenerate(so, cnt);
  }
  // all G lanes of the group are active here
#pragma unroll
  for (int d = 1; d < G; d <<= 1) nscr += __shfl_xor(nscr, d, 64);
  if (r == 0) scr_cnt[s] = nscr;
}

// Fill pass for slaves with more than CTMP candidates (rare), one lane per
// slave: the walk again, an insertion sort by master index in a
// lane-interleaved LDS segment (in place in the output when longer than
// CCAP; two call sites, so that each pointer has a known address space),
// then the screening.
__device__ __forceinline__ void fill_long(int s, int32_t n_s, int base, int c, int32_t* v, int vs,
                                          const double* __restrict__ box_s, const double* __restrict__ sbox,
                                          const uint32_t* __restrict__ mvals, const int32_t* __restrict__ cell_start,
                                          const Grid& g, double delta, int32_t* __restrict__ cand_s,
                                          int32_t* __restrict__ cand_m, const double* __restrict__ sd,
                                          const double* __restrict__ md, double eps_a, uint8_t* __restrict__ nv_out,
                                          ScreenOut& so, int& nscr) {
  walk_cells(load_box(box_s, n_s, s), sbox, mvals, cell_start, g, delta, v, vs, c);
  for (int i = 1; i < c; ++i) {
    const int x = v[i * vs];
    int j = i - 1;
    while (j >= 0 && v[j * vs] > x) {
      v[(j + 1) * vs] = v[j * vs];
      --j;
    }
    v[(j + 1) * vs] = x;
  }
  SlavePlane P;
  load_plane(sd, n_s, s, P);
  for (int i = 0; i < c; ++i)
    nscr += screen_one(P, s, v[i * vs], (int64_t)base + i, md, eps_a, cand_s, cand_m, nv_out, so) ? 1 : 0;
}

// One slave of the long fill: its place [base, base + c) in the output.
template <int LANES>
__device__ __forceinline__ void fill_long_slave(int s, int32_t n_s, int base, int c, int64_t cap, int32_t* lds,
                                                const double* __restrict__ box_s, const double* __restrict__ sbox,
                                                const uint32_t* __restrict__ mvals,
                                                const int32_t* __restrict__ cell_start, const Grid* __restrict__ gp,
                                                double delta, int32_t* __restrict__ cand_s,
                                                int32_t* __restrict__ cand_m, const double* __restrict__ sd,
                                                const double* __restrict__ md, double eps_a,
                                                uint8_t* __restrict__ nv_out, int32_t* __restrict__ scr_cnt,
                                                Counters* cnt) {
  if (base < 0 || (int64_t)base + c > cap) {
    scr_cnt[s] = 0;
    return;
  }
  const Grid g = *gp;
  ScreenOut so{0u, 0u};
  int nscr = 0;
  if (c <= CCAP)
    fill_long(s, n_s, base, c, lds, LANES, box_s, sbox, mvals, cell_start, g, delta, cand_s, cand_m, sd, md, eps_a,
              nv_out, so, nscr);
  else
    fill_long(s, n_s, base, c, cand_m + base, 1, box_s, sbox, mvals, cell_start, g, delta, cand_s, cand_m, sd, md,
              eps_a, nv_out, so, nscr);
  count_degenerate(so, cnt);
  scr_cnt[s] = nscr;
}

__global__ __launch_bounds__(BS) void k_cand_fill_long(const double* __restrict__ box_s, int32_t n_s,
                                                        const double* __restrict__ sbox,
                                                        const uint32_t* __restrict__ mvals,
                                                        const int32_t* __restrict__ cell_start, const Grid* __restrict__ gp,
                                                        double delta,
                                                        const int32_t* __restrict__ off, int32_t* __restrict__ cand_s,
                                                        int32_t* __restrict__ cand_m, const double* __restrict__ sd,
                                                        const double* __restrict__ md, double eps_a,
                                                        uint8_t* __restrict__ nv_out,
                                                        int32_t* __restrict__ scr_cnt, Counters* cnt,
                                                        int64_t cap) {
  __shared__ int32_t lds[CCAP * BS];
  const int s = xcd_tile(blockIdx.x, gridDim.x) * BS + threadIdx.x;
  if (s >= n_s) return;
  const int base = off[s], c = off[s + 1] - base;
  if (c > CTMP)
    fill_long_slave<BS>(s, n_s, base, c, cap, lds + threadIdx.x, box_s, sbox, mvals, cell_start, gp, delta, cand_s,
                        cand_m, sd, md, eps_a, nv_out, scr_cnt, cnt);
}

__global__ __launch_bounds__(BS) void k_cand_fill(int32_t n_s, const int32_t* __restrict__ tmp,
                                                   const int32_t* __restrict__ off, int32_t* __restrict__ cand_s,
                                                   int32_t* __restrict__ cand_m, const double* __restrict__ sd,
                                                   const double* __restrict__ md, double eps_a,
                                                   uint8_t* __restrict__ nv_out,
                                                   int32_t* __restrict__ scr_cnt, Counters* cnt, int64_t cap) {
  constexpr int G = LANES_MANY;
  const int64_t t = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * BS + threadIdx.x;
  const int s = (int)(t / G), r = (int)(t % G);
  if (s >= n_s) return;  // whole groups leave together
  const int base = off[s], c = off[s + 1] - base;
  if (c <= CTMP)  // (else k_cand_fill_long)
    fill_short<G>(s, r, n_s, base, c, tmp, cand_s, cand_m, sd, md, eps_a, nv_out, scr_cnt, cnt, cap);
}

// Both fills and the offsets in one launch, for up to SELF_OFFSETS slave
// elements: each workgroup finds its own offsets from the counts and leaves
// them in off; the first lane of a group takes a long list.
template <int G>
__global__ __launch_bounds__(BS) void k_cand_fill_self(const double* __restrict__ box_s, int32_t n_s,
                                                        const double* __restrict__ sbox,
                                                        const uint32_t* __restrict__ mvals,
                                                        const int32_t* __restrict__ cell_start,
                                                        const Grid* __restrict__ gp, double delta,
                                                        const int32_t* __restrict__ count,
                                                        const int32_t* __restrict__ tmp, int32_t* __restrict__ off,
                                                        int32_t* __restrict__ cand_s, int32_t* __restrict__ cand_m,
                                                        const double* __restrict__ sd, const double* __restrict__ md,
                                                        double eps_a, uint8_t* __restrict__ nv_out,
                                                        int32_t* __restrict__ scr_cnt, Counters* cnt,
                                                        ScanStage stage) {
  __shared__ int32_t lds[CCAP * (BS / G)];
  const int s0 = xcd_tile(blockIdx.x, gridDim.x) * (BS / G);
  if (s0 >= n_s) return;  // the whole workgroup
  const int s = s0 + (int)threadIdx.x / G, r = (int)threadIdx.x % G;
  const int c = s < n_s ? count[s] : 0;
  int base = self_offset<BS>(count, s0, r == 0 ? c : 0);
  if (r > 0) base = (int)((uint32_t)base - (uint32_t)c);
  if (s >= n_s) return;  // whole groups leave together
  if (r == 0) {
    off[s] = base;
    if (s == n_s - 1) {
      const int total = (int)((uint32_t)base + (uint32_t)c);
      off[n_s] = total;
      stage_total(stage, total, false);
    }
  }
  if (c <= CTMP)
    fill_short<G>(s, r, n_s, base, c, tmp, cand_s, cand_m, sd, md, eps_a, nv_out, scr_cnt, cnt, stage.cap);
  else if (r == 0)
    fill_long_slave<BS / G>(s, n_s, base, c, stage.cap, lds + threadIdx.x / G, box_s, sbox, mvals, cell_start, gp,
                            delta, cand_s, cand_m, sd, md, eps_a, nv_out, scr_cnt, cnt);
}

}  // namespace

int prep_blocks(int32_t n_el) { return n_el == 0 ? 0 : std::min(512, (n_el + BS - 1) / BS); }

hipError_t launch_prep(const DeviceMesh& S, const DeviceMesh& M, double* box_s, double* sd, double* box_m,
                       double* md, double* part, hipStream_t s) {
  const int nb_s = prep_blocks(S.n_el), nb_m = prep_blocks(M.n_el);
  if (nb_s == 0 && nb_m == 0) return hipSuccess;
  const PrepSide ps{S.x, S.y, S.z, S.conn, S.nrm, box_s, sd, nullptr, part, S.n_el, S.n_nodes, nb_s};
  const PrepSide pm{M.x, M.y, M.z, M.conn, nullptr, box_m, nullptr, md, part + (size_t)PREP_PART * nb_s,
                    M.n_el, M.n_nodes, nb_m};
  k_prep<<<dim3((unsigned)std::max(nb_s, nb_m), 2), BS, 0, s>>>(ps, pm);
  return hipGetLastError();
}

hipError_t launch_prep_reduce(const double* part, int nb_s, int nb_m, double delta, double bin_size,
                              int64_t max_cells, DevState* st, Counters* cnt, int32_t* cell_cnt, hipStream_t s) {
  // one workgroup per 16K cells of the capacity, at most one per compute unit
  const unsigned nb = (unsigned)std::min<int64_t>(256, std::max<int64_t>(1, max_cells >> 14));
  k_prep_reduce<<<nb, BS, 0, s>>>(part, nb_s, nb_m, delta, bin_size, max_cells, st, cnt, cell_cnt);
  return hipGetLastError();
}

hipError_t launch_cell_count(const double* box_m, int32_t n_m, const Grid* g, int32_t* cell_cnt, uint32_t* cell,
                             uint32_t* rank, hipStream_t s) {
  if (n_m == 0) return hipSuccess;
  k_cell_count<<<(n_m + BS - 1) / BS, BS, 0, s>>>(box_m, n_m, g, cell_cnt, cell, rank);
  return hipGetLastError();
}

hipError_t launch_cell_place(const uint32_t* cell, const uint32_t* rank, int32_t n, const double* box_m,
                             const Grid* g, const int32_t* cell_start, uint32_t* vals, double* sbox, uint64_t* qbox,
                             hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_cell_place<<<(n + BS - 1) / BS, BS, 0, s>>>(cell, rank, n, box_m, g, cell_start, vals, sbox, qbox);
  return hipGetLastError();
}

// Grids of the candidate passes: XCD-aware (each XCD's L2 serves a
// contiguous eighth of the slave elements, whose masters are neighbours).
unsigned group_blocks(int32_t n_s, int lanes) { return xcd_grid((unsigned)(((int64_t)n_s * lanes + BS - 1) / BS)); }

hipError_t launch_cand_count(const double* box_s, int32_t n_s, const double* sbox, const uint64_t* qbox,
                             const uint32_t* mvals,
                             const int32_t* cell_start, const Grid* g, double delta, int32_t* count, int32_t* tmp,
                             hipStream_t s) {
  if (n_s == 0) return hipSuccess;
  const bool few = n_s <= FEW_SLAVES;
  (few ? k_cand_count<LANES_FEW> : k_cand_count<LANES_MANY>)<<<group_blocks(n_s, few ? LANES_FEW : LANES_MANY), BS, 0, s>>>(
      box_s, n_s, sbox, qbox, mvals, cell_start, g, delta, count, tmp);
  return hipGetLastError();
}

hipError_t launch_cand_fill(const double* box_s, int32_t n_s, const double* sbox, const uint32_t* mvals,
                            const int32_t* cell_start, const Grid* g, double delta, const int32_t* count,
                            const int32_t* tmp, int32_t* off, const Buf& scan_tmp, int32_t* cand_s, int32_t* cand_m,
                            const double* sd, const double* md, double eps_a, uint8_t* nv, int32_t* scr_cnt,
                            Counters* cnt, const ScanStage& stage, hipStream_t s) {
  if (n_s > 0 && n_s <= SELF_OFFSETS) {
    const bool few = n_s <= FEW_SLAVES;
    auto* k = few ? k_cand_fill_self<LANES_FEW> : k_cand_fill_self<LANES_MANY>;
    k<<<group_blocks(n_s, few ? LANES_FEW : LANES_MANY), BS, 0, s>>>(box_s, n_s, sbox, mvals, cell_start, g, delta,
                                                                     count, tmp, off, cand_s, cand_m, sd, md, eps_a,
                                                                     nv, scr_cnt, cnt, stage);
    return hipGetLastError();
  }
  hipError_t e = scan_exclusive(count, off, n_s, scan_tmp, s, 0, stage);
  if (e != hipSuccess || n_s == 0) return e;
  k_cand_fill<<<group_blocks(n_s, LANES_MANY), BS, 0, s>>>(n_s, tmp, off, cand_s, cand_m, sd, md, eps_a, nv, scr_cnt, cnt,
                                               stage.cap);
  k_cand_fill_long<<<xcd_grid((unsigned)((n_s + BS - 1) / BS)), BS, 0, s>>>(box_s, n_s, sbox, mvals, cell_start, g, delta,
                                                                            off, cand_s, cand_m, sd, md, eps_a, nv,
                                                                            scr_cnt, cnt, stage.cap);
  return hipGetLastError();
}

int cand_tmp_per_slave() { return CTMP; }

}  // namespace mt
