// Backward pass of the pair evaluation: gradient of
//   L = <W_D, D> + <W_M, M> + <w_g, g>
// with respect to the 24 nodal coordinates of each pair (the linearisation
// of the mortar terms required in every nonlinear iteration): the slave
// components summed per slave element (ElemSums, component 3 * node + axis),
// the master components staged per pair in pairs-by-master order
// (gpair[(3 * node + axis) * stride + mpos[p]]), both reduced per node by the
// assembly kernels.
#include "mt_dual.h"

namespace mt {

namespace {

constexpr int BSC = 64;

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
  return x;
}

// Upstream weights of pair p gathered through the position maps.
__device__ __forceinline__ void gather_weights(int s, int64_t p, int4 csn, const int32_t* __restrict__ erow,
                                               const int32_t* __restrict__ posD,
                                               int32_t n_s, const int32_t* __restrict__ posM, int64_t stride,
                                               const double* __restrict__ W_D, const double* __restrict__ W_M,
                                               const double* __restrict__ w_g, double WD[16], double WM[16],
                                               double wg[4]) {
  load_weights(W_D, load_erow(erow, s, 0), posD, n_s, s, WD);
  load_weights(W_M, load_erow(erow, s, 1), posM, stride, p, WM);
  wg[0] = w_g[csn.x];
  wg[1] = w_g[csn.y];
  wg[2] = w_g[csn.z];
  wg[3] = w_g[csn.w];
}

// Dual basis: the dependence of the dual coefficients on the slave nodes, one
// lane per slave element, after the sweep (elem_dual_adjoint).
template <bool NODAL>
__global__ __launch_bounds__(BSC) __attribute__((amdgpu_waves_per_eu(2))) void k_elem_dual_adj(
    MeshPtrs S, const int32_t* __restrict__ pair_off, const int32_t* __restrict__ erow, const int32_t* __restrict__ posD,
    const int32_t* __restrict__ posM, int64_t stride, const double* __restrict__ W_D, const double* __restrict__ W_M,
    const double* __restrict__ w_g, const double* __restrict__ blk, ElemSums eblk, ElemSums egrad) {
  const int e = xcd_tile(blockIdx.x, gridDim.x) * BSC + threadIdx.x;
  if (e >= eblk.n_el) return;
  const int p0 = pair_off[e], p1 = pair_off[e + 1];
  if (p0 == p1) return;
  elem_dual_adjoint<NODAL>(S, e, p0, p1, erow, posD, posM, stride, W_D, W_M, w_g, blk, eblk, egrad);
}

template <int NQ, bool DUAL, bool NODAL>
__global__ __launch_bounds__(BSC) __attribute__((amdgpu_waves_per_eu(2))) void k_pair_bwd(MeshPtrs S, int32_t n_s, MeshPtrs M, KParams kp,
                                                   const int32_t* __restrict__ pair_s,
                                                   const int32_t* __restrict__ pair_m,
                                                   const int32_t* __restrict__ n_dev, PolyBuf poly,
                                                   const int32_t* __restrict__ mpos,
                                                   const int32_t* __restrict__ erow,
                                                   const int32_t* __restrict__ posD, const int32_t* __restrict__ posM,
                                                   const double* __restrict__ W_D, const double* __restrict__ W_M,
                                                   const double* __restrict__ w_g, double* __restrict__ gpair,
                                                   int64_t stride, ElemSums egrad, Counters* cnt) {
  static_assert(BSC == TILE_PAIRS, "one wavefront per tile");
  __shared__ double stash[BWD_STASH * BSC];
  const Stash st{stash + threadIdx.x, BSC};
  const int64_t n_pairs = *n_dev;
  const int64_t tile = dyn_tile(blockIdx.x, n_pairs, BSC);
  if (tile < 0) return;
  const int64_t p = tile * BSC + threadIdx.x;
  const bool valid = p < n_pairs;
  unsigned noconv = 0;
  int s = -1, prev = -1;
  double Xsb[4][3], n0b[3];
  if (valid) {
    s = pair_s[p];
    prev = p > 0 ? pair_s[p - 1] : -1;
    const int4 csn = load_conn(S.conn, s);
    double WD[16], WM[16], wg[4];
    gather_weights(s, p, csn, erow, posD, n_s, posM, stride, W_D, W_M, w_g, WD, WM, wg);
    double Xmb[4][3];
    pair_backward<NQ, DUAL, NODAL>(S, s, csn, M, load_conn(M.conn, pair_m[p]), gpoly(poly, p), gpoly_nf(poly, p), kp,
                                   st, WD, WM, wg, Xsb, Xmb, n0b, noconv);
    const int64_t q = mpos[p];
#pragma unroll
    for (int k = 0; k < 12; ++k) gpair[(int64_t)k * stride + q] = Xmb[k / 3][k % 3];
  }
  store_slave_gradient<NODAL>(Xsb, n0b, valid, s, prev, p, st, egrad);
  const unsigned long long nc = wave_sum_u64(noconv);
  if (threadIdx.x == 0 && nc) atomicAdd(&cnt->noconv, nc);
}

}  // namespace

hipError_t launch_pair_bwd(const DeviceMesh& S, const DeviceMesh& M, const KParams& kp, const int32_t* pair_s,
                           const int32_t* pair_m, const int32_t* pair_off, const int32_t* n_pairs, int64_t cap,
                           const PolyBuf& poly, const int32_t* mpos, const int32_t* erow,
                           const int32_t* posD, const int32_t* posM,
                           const double* W_D, const double* W_M, const double* w_g, const double* blk,
                           const ElemSums& eblk, double* gpair, const ElemSums& egrad, Counters* cnt, hipStream_t s) {
  if (cap == 0) return hipSuccess;
  const unsigned nb = xcd_grid((unsigned)((cap + BSC - 1) / BSC));
  const MeshPtrs ms{S.x, S.y, S.z, S.conn, S.nrm}, mm{M.x, M.y, M.z, M.conn, nullptr};
  const bool nodal = S.nrm != nullptr;
  auto* k = kp.rule == 3
                ? (kp.dual ? (nodal ? k_pair_bwd<3, true, true> : k_pair_bwd<3, true, false>)
                           : (nodal ? k_pair_bwd<3, false, true> : k_pair_bwd<3, false, false>))
                : (kp.dual ? (nodal ? k_pair_bwd<7, true, true> : k_pair_bwd<7, true, false>)
                           : (nodal ? k_pair_bwd<7, false, true> : k_pair_bwd<7, false, false>));
  hipLaunchKernelGGL(k, dim3(nb), dim3(BSC), 0, s, ms, S.n_el, mm, kp, pair_s, pair_m, n_pairs, poly, mpos, erow, posD, posM,
                     W_D, W_M, w_g, gpair, cap, egrad, cnt);
  if (kp.dual && S.n_el > 0) {
    auto* kd = nodal ? k_elem_dual_adj<true> : k_elem_dual_adj<false>;
    hipLaunchKernelGGL(kd, dim3(xcd_grid((unsigned)((S.n_el + BSC - 1) / BSC))), dim3(BSC), 0, s, ms, pair_off, erow,
                       posD, posM, cap, W_D, W_M, w_g, blk, eblk, egrad);
  }
  return hipGetLastError();
}

}  // namespace mt
