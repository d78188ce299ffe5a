// Device-wide primitives: exclusive scan and fill, written for 64-wide
// wavefronts.
#include "mt_scan.h"

namespace mt {

namespace {

constexpr int SCAN_BS = 256;
constexpr int SCAN_IPT = 8;
constexpr int SCAN_TILE = SCAN_BS * SCAN_IPT;

// n_dev (optional): a count the device holds, at most n; entries from it on
// count as zero, and the outputs behind out[*n_dev] are undefined (the tile
// that holds it is written whole, up to out[n - 1]).
template <class T>
__device__ __forceinline__ int64_t live_count(int64_t n, const int32_t* n_dev) {
  if (!n_dev) return n;
  const int64_t m = *n_dev;
  return m < 0 ? 0 : (m < n ? m : n);
}

// Exclusive scan: per-tile sums, then each tile's scan with its offset.
// Up to SCAN_SELF workgroups there is one launch: each adds up the inputs
// before its own itself (at most 64K values from L2, about 2 us, where the
// launch of the sums costs 4-5 us).  Up to SCAN_DIRECT, every workgroup adds
// up the sums before it (no third launch; the sums are a few KB); beyond, the
// sums are scanned recursively first.  No tile waits for another.
constexpr int64_t SCAN_SELF = 32;
constexpr int64_t SCAN_DIRECT = 8192;

// The SCAN_IPT values of thread's slot (zero past `live`): two 16-byte loads
// when VEC (in 16-byte aligned) and the slot is whole.
template <bool VEC>
__device__ __forceinline__ void load_slot(const int32_t* __restrict__ in, int64_t base, int64_t live,
                                          int32_t v[SCAN_IPT]) {
  static_assert(SCAN_IPT == 8, "two 16-byte vectors per thread");
  if (VEC && base + SCAN_IPT <= live) {
    const int4 a = *reinterpret_cast<const int4*>(in + base);
    const int4 b = *reinterpret_cast<const int4*>(in + base + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < SCAN_IPT; ++i) v[i] = (base + i < live) ? in[base + i] : 0;
  }
}

// Each workgroup takes `per` consecutive tiles.  A launch with gridDim.y = 2
// scans a second array of the same length (in2 into out2, its workgroup sums
// after the first array's) in the same launches.
template <bool VEC>
__global__ __launch_bounds__(SCAN_BS) void k_tile_sums(const int32_t* __restrict__ in, const int32_t* __restrict__ in2,
                                                       int64_t n, const int32_t* n_dev, int32_t* __restrict__ sums,
                                                       int per) {
  if (blockIdx.y) {
    in = in2;
    sums += gridDim.x;
  }
  const int64_t live = live_count<int32_t>(n, n_dev);
  if ((int64_t)blockIdx.x * per * SCAN_TILE >= live) {  // nothing here (the whole workgroup)
    if (threadIdx.x == 0) sums[blockIdx.x] = 0;
    return;
  }
  int32_t s = 0;
  for (int q = 0; q < per; ++q) {
    const int64_t base = ((int64_t)blockIdx.x * per + q) * SCAN_TILE + (int64_t)threadIdx.x * SCAN_IPT;
    int32_t v[SCAN_IPT];
    load_slot<VEC>(in, base, live, v);
#pragma unroll
    for (int i = 0; i < SCAN_IPT; ++i) s += v[i];
  }
  int32_t tot;
  block_exclusive<SCAN_BS>(s, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// out[i] = offset of the workgroup + exclusive prefix of in within its
// tiles; the workgroup that holds the end of the live values also writes the
// total behind them, and with a stage to the device state.  Offset of
// workgroup w: OFF_GIVEN offs[w] (scanned) or 0, OFF_SUMS the sum of
// sums[0..w) (raw workgroup sums), OFF_SELF the sum of the inputs before it.
enum { OFF_GIVEN, OFF_SUMS, OFF_SELF };

template <bool VEC, int OFF>
__global__ __launch_bounds__(SCAN_BS) void k_tile_scan(const int32_t* __restrict__ in, const int32_t* __restrict__ in2,
                                                       int64_t n, const int32_t* n_dev,
                                                       const int32_t* __restrict__ offs, int32_t* __restrict__ out,
                                                       int32_t* __restrict__ out2, int per, ScanStage stage) {
  if (blockIdx.y) {  // (the raw workgroup sums of the second array follow the first's)
    in = in2;
    out = out2;
    if (OFF == OFF_SUMS) offs += gridDim.x;
  }
  const int64_t live = live_count<int32_t>(n, n_dev);
  const int64_t w = blockIdx.x;
  const int64_t end = min(live / ((int64_t)per * SCAN_TILE), (int64_t)gridDim.x - 1);
  if (w > end) return;
  int32_t off = 0;
  if (OFF == OFF_SUMS) {
    int32_t part = 0;
    for (int64_t i = threadIdx.x; i < w; i += SCAN_BS) part += offs[i];
    block_exclusive<SCAN_BS>(part, &off);
  } else if (OFF == OFF_SELF) {
    // (w <= end: the tiles before this one hold live values only)
    int32_t part = 0;
    if (VEC) {
      part = sum_before<SCAN_BS>(in, (int32_t)(w * SCAN_TILE));
    } else {
      for (int64_t i = threadIdx.x; i < w * SCAN_TILE; i += SCAN_BS) part += in[i];
    }
    block_exclusive<SCAN_BS>(part, &off);
  } else if (offs) {
    off = offs[w];
  }
  for (int q = 0; q < per; ++q) {
    const int64_t base = (w * per + q) * SCAN_TILE + (int64_t)threadIdx.x * SCAN_IPT;
    int32_t v[SCAN_IPT];
    load_slot<VEC>(in, base, live, v);
    int32_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_IPT; ++i) s += v[i];
    int32_t tot;
    int32_t run = block_exclusive<SCAN_BS>(s, &tot) + off;
    int32_t o[SCAN_IPT];
#pragma unroll
    for (int i = 0; i < SCAN_IPT; ++i) {
      o[i] = run;
      run += v[i];
    }
    if (VEC && base + SCAN_IPT <= n) {
      *reinterpret_cast<int4*>(out + base) = make_int4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<int4*>(out + base + 4) = make_int4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
      for (int i = 0; i < SCAN_IPT; ++i)
        if (base + i < n) out[base + i] = o[i];
    }
    off += tot;
  }
  if (w == end && threadIdx.x == 0) {
    if (live == n) out[n] = off;  // (else written above: no value lies behind the live ones)
    if (stage.st) stage_total(stage, off, (blockIdx.y != 0) != stage.second);
  }
}

// Exclusive scan of n values (of the first *n_dev when given) into
// out[0..n]; with in2, also of in2 into out2 (n_dev null) in the same
// launches while the workgroup sums of both fit the direct scheme.
// max_blocks > 0 caps the workgroups of each launch (several tiles each): a
// scan queued beside a long kernel on another stream then waits for few
// dispatch slots.  No memset: the launches can be captured in a graph.
hipError_t scan_impl(const int32_t* in, int32_t* out, int64_t n, const int32_t* n_dev, int32_t* tmp, hipStream_t s,
                     const int32_t* in2 = nullptr, int32_t* out2 = nullptr, int64_t max_blocks = 0,
                     const ScanStage& stage = ScanStage{}) {
  const int64_t tiles = std::max<int64_t>(1, (n + SCAN_TILE - 1) / SCAN_TILE);
  const int per = max_blocks > 0 ? (int)((tiles + max_blocks - 1) / max_blocks) : 1;
  const int64_t blocks = (tiles + per - 1) / per;
  uintptr_t addr = reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out);
  if (in2) addr |= reinterpret_cast<uintptr_t>(in2) | reinterpret_cast<uintptr_t>(out2);
  const bool vec = (addr & 15) == 0;
  if (in2 && blocks > SCAN_DIRECT) {
    hipError_t e = scan_impl(in, out, n, n_dev, tmp, s, nullptr, nullptr, max_blocks, stage);
    ScanStage other = stage;
    other.second = true;
    return e != hipSuccess ? e : scan_impl(in2, out2, n, nullptr, tmp, s, nullptr, nullptr, max_blocks, other);
  }
  const dim3 grid((unsigned)blocks, in2 ? 2u : 1u);
  if (blocks <= SCAN_SELF && per == 1) {
    auto* k = vec ? k_tile_scan<true, OFF_SELF> : k_tile_scan<false, OFF_SELF>;
    k<<<grid, SCAN_BS, 0, s>>>(in, in2, n, n_dev, nullptr, out, out2, per, stage);
    return hipGetLastError();
  }
  int32_t* sums = tmp;  // blocks (2 blocks with in2) entries
  (vec ? k_tile_sums<true> : k_tile_sums<false>)<<<grid, SCAN_BS, 0, s>>>(in, in2, n, n_dev, sums, per);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (blocks <= SCAN_DIRECT) {
    auto* k = vec ? k_tile_scan<true, OFF_SUMS> : k_tile_scan<false, OFF_SUMS>;
    k<<<grid, SCAN_BS, 0, s>>>(in, in2, n, n_dev, sums, out, out2, per, stage);
    return hipGetLastError();
  }
  int32_t* offs = tmp + blocks;  // blocks + 1 entries
  e = scan_impl(sums, offs, blocks, nullptr, offs + blocks + 1, s);
  if (e != hipSuccess) return e;
  auto* k = vec ? k_tile_scan<true, OFF_GIVEN> : k_tile_scan<false, OFF_GIVEN>;
  k<<<(unsigned)blocks, SCAN_BS, 0, s>>>(in, nullptr, n, n_dev, offs, out, nullptr, per, stage);
  return hipGetLastError();
}

}  // namespace

int64_t scan_tmp_elems(int64_t n) {
  // per level: the tile sums and their scan (tiles + 1), while recursing
  int64_t total = 0;
  while (true) {
    const int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (tiles <= 1) break;
    total += 2 * tiles + 1;
    if (tiles <= SCAN_DIRECT) break;
    n = tiles;
  }
  return total + 1;
}

namespace {

// Grid-stride fill: at most FILL_BLOCKS workgroups, so that a fill queued
// beside a long kernel on another stream waits for few dispatch slots.
constexpr int64_t FILL_BLOCKS = 1024;
__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Several copies in one launch, a row of workgroups each: four runtime copies
// are four launches of about 2 us one after the other, and as many calls.
__global__ __launch_bounds__(256) void k_copy_i32(CopyList L) {
  const int q = blockIdx.y;
  const int32_t* __restrict__ src = L.src[q];
  int32_t* __restrict__ dst = L.dst[q];
  if (!dst) return;
  const int64_t n = L.n[q], t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  int64_t done = 0;
  if (((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0) {
    done = n & ~int64_t(3);
    for (int64_t i = t; i < n / 4; i += step)
      reinterpret_cast<int4*>(dst)[i] = reinterpret_cast<const int4*>(src)[i];
  }
  for (int64_t i = done + t; i < n; i += step) dst[i] = src[i];
}
}  // namespace

hipError_t copy_i32(const CopyList& list, hipStream_t s) {
  int64_t most = 0;
  for (int q = 0; q < 4; ++q)
    if (list.dst[q]) most = std::max(most, list.n[q]);
  if (most == 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((most + 1023) / 1024, FILL_BLOCKS);
  k_copy_i32<<<dim3((unsigned)blocks, 4), 256, 0, s>>>(list);
  return hipGetLastError();
}

hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, const Buf& tmp, hipStream_t s,
                          int64_t max_blocks, const ScanStage& stage) {
  if ((int64_t)(tmp.bytes / sizeof(int32_t)) < scan_tmp_elems(n)) return hipErrorInvalidValue;
  return scan_impl(in, out, n, nullptr, tmp.as<int32_t>(), s, nullptr, nullptr, max_blocks, stage);
}

hipError_t scan_exclusive2(const int32_t* in, int32_t* out, const int32_t* in2, int32_t* out2, int64_t n,
                           const Buf& tmp, hipStream_t s, int64_t max_blocks, const ScanStage& stage) {
  if ((int64_t)(tmp.bytes / sizeof(int32_t)) < scan_tmp_elems(n)) return hipErrorInvalidValue;
  return scan_impl(in, out, n, nullptr, tmp.as<int32_t>(), s, in2, out2, max_blocks, stage);
}

hipError_t scan_exclusive_dev(const int32_t* in, int32_t* out, const int32_t* n_dev, int64_t cap, const Buf& tmp,
                              hipStream_t s, const ScanStage& stage) {
  if ((int64_t)(tmp.bytes / sizeof(int32_t)) < scan_tmp_elems(cap)) return hipErrorInvalidValue;
  return scan_impl(in, out, cap, n_dev, tmp.as<int32_t>(), s, nullptr, nullptr, 0, stage);
}

hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill_i32<<<(unsigned)std::min<int64_t>((n + 255) / 256, FILL_BLOCKS), 256, 0, s>>>(p, v, n);
  return hipGetLastError();
}

}  // namespace mt
