// Grain bucketing of (query, probe) pairs.  Routing gives every query P grains;
// projection and scan run grain-major so that a grain's basis and Block-SoA
// codes are read once per tile of queries instead of once per query.
//
// A counting sort groups the pair ids q * P + slot by grain, grains in the
// order of their rank (Buckets::grank; the grain number where none is given).
// Inside a grain's range the pairs of probe slot 0 (each query's nearest
// grain) come first, so the scan can take slot 0 in a pass of its own whose
// results bound the other slots.  Three work-item lists are cut from the ranges
// without materialising them: the exclusive prefix ioff[L][rank] of
// ceil(pairs / tile_L) numbers list L's items, and a kernel finds the grain of
// item i by a search of ioff (or from the decoded item table).
//
// Three kernels: bucket_count_kernel takes every pair's place among its
// grain's pairs of the same kind from the counter itself (a returning atomic),
// bucket_scan_kernel turns the counts into offsets, bucket_place_kernel writes
// the pair ids, the pairs' candidate-list slots and the item table.  Batches
// of up to SMALL_PAIRS pairs do all of it in one workgroup.  Bound by launches
// and by dependent round trips, not by bytes (262,144 pairs: 3 MB).  On
// 16,384 x 16 pairs over 8,192 grains the bucketing stage takes 33 us
// (eight kernels with a histogram, a scatter and lists numbered query by query:
// 135 us), on 256 x 16 pairs 24 us (117 us).
#include <algorithm>

#include "hntl_device.h"
#include "hntl_internal.h"

namespace hntl {

namespace {

constexpr int SMALL_PAIRS = 4096;   // pairs and grains of the one-workgroup form: four pairs a
constexpr int SMALL_GRAINS = 8192;  // thread in registers, four counters a grain in the LDS (128 KiB)
constexpr int64_t ITEM_WGS = 1024;   // workgroups that write an item table (each thread strides over it)

// The pairs of a bucketing are numbered e = 0, 1, ...: every pair, or with
// PICK_SLOT0 the first of every query.
__device__ __forceinline__ int64_t pair_of(const Buckets& b, int64_t e, int P) {
  return b.pick == PICK_SLOT0 ? e * P : e;
}

// Grain of pair p, -1 for a pair that is not taken.
__device__ __forceinline__ int probe_of(const Buckets& b, const int32_t* __restrict__ probes, int64_t p, int P) {
  const int g = probes[p];
  if (g < 0 || g >= b.G) return -1;
  if (b.pick == PICK_ALL || b.pick == PICK_SLOT0) return g;
  bool take = (p % P == 0) == (b.pick == PICK_FIRST);
  if (b.pick != PICK_REST && p % P != 0)
    take = small_first_grain(probes, p / P, P, b.G, b.goff, b.need) == (b.pick == PICK_FIRST);
  return take ? g : -1;
}

// Inclusive scan over the lanes of a wave, DPP moves only.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
#define HNTL_SCAN_STEP(CTRL, ROWS) x += __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false)
  HNTL_SCAN_STEP(0x111, 0xF);  // row_shr:1, 2, 4, 8: prefixes inside each row of 16 lanes
  HNTL_SCAN_STEP(0x112, 0xF);
  HNTL_SCAN_STEP(0x114, 0xF);
  HNTL_SCAN_STEP(0x118, 0xF);
  HNTL_SCAN_STEP(0x142, 0xA);  // row_bcast:15 into rows 1 and 3
  HNTL_SCAN_STEP(0x143, 0xC);  // row_bcast:31 into rows 2 and 3
#undef HNTL_SCAN_STEP
  return x;
}

// Exclusive scan of N values per thread of a 1024-thread workgroup.
template <int N>
__device__ void block_exclusive_scan(const int (&v)[N], int (&ex)[N], int (&total)[N], int (*tmp)[16] /* N */) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  int x[N];
#pragma unroll
  for (int c = 0; c < N; ++c) x[c] = wave_inclusive_scan(v[c]);
  if (lane == 63)
#pragma unroll
    for (int c = 0; c < N; ++c) tmp[c][wave] = x[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const int t = lane < 16 ? tmp[c][lane] : 0;
    const int y = wave_inclusive_scan(t);  // lane w < 16: the waves up to w
    total[c] = __builtin_amdgcn_readlane(y, 15);
    const int before = __builtin_amdgcn_readlane(y, wave == 0 ? 0 : wave - 1);
    ex[c] = (wave == 0 ? 0 : before) + x[c] - v[c];
  }
  __syncthreads();
}

// Eight consecutive values of a 16-byte aligned array (zeros from n on).
__device__ __forceinline__ void load8(int (&v)[8], const int* a, int i, int n) {
  if (i + 8 <= n) {
    const int4 x = *reinterpret_cast<const int4*>(a + i), y = *reinterpret_cast<const int4*>(a + i + 4);
    v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
    v[4] = y.x, v[5] = y.y, v[6] = y.z, v[7] = y.w;
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = i + u < n ? a[i + u] : 0;
  }
}
__device__ __forceinline__ void store8(int* a, int i, int n, const int (&v)[8]) {
  if (i + 8 <= n) {
    *reinterpret_cast<int4*>(a + i) = make_int4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<int4*>(a + i + 4) = make_int4(v[4], v[5], v[6], v[7]);
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i + u < n) a[i + u] = v[u];
  }
}

// Offsets of every rank from the counts (one workgroup of 1,024 threads), 8,192
// ranks at a time: thread t owns ranks 8 t .. 8 t + 7 of them (16-byte accesses;
// single ones in that order touch every cache line eight times: 33 us at 8,192
// grains, this takes 9), sums its pairs, items and lists, one workgroup
// scan turns the sums into offsets, and it writes its own.  Counts come from c0 and
// c1 and start offsets go to first and lists (LDS or global); item offsets go
// to b.  With b.nsplit_rank, a grain's slot-0 and rest tiles each become nsplit
// items (one per block range of the grain) and each of its pairs owns nsplit
// candidate lists.
__device__ __forceinline__ void scan_ranks(const Buckets& b, const int* c0a, const int* c1a, bool c1_aligned,
                                           int* first, int* lists) {
  __shared__ int tmp[5][16];
  const int G = b.G;
  const int t0 = b.lists.tile[LIST_SLOT0], t1 = b.lists.tile[LIST_REST], t2 = b.lists.tile[LIST_ALL];
  int carry[5] = {0, 0, 0, 0, b.lists_from ? *b.lists_from : 0};
  for (int base = 0; base < G; base += 8192) {
    const int r0 = base + 8 * (int)threadIdx.x;
    int c0[8], c1[8], sp[8];
    load8(c0, c0a, r0, G);
    if (c1_aligned)
      load8(c1, c1a, r0, G);
    else
#pragma unroll
      for (int u = 0; u < 8; ++u) c1[u] = r0 + u < G ? c1a[r0 + u] : 0;
    if (b.nsplit_rank)
      load8(sp, b.nsplit_rank, r0, G);
    else
#pragma unroll
      for (int u = 0; u < 8; ++u) sp[u] = 1;
    int add[5][8];
    int sum[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      add[0][u] = c0[u] + c1[u];
      add[1][u] = (c0[u] + t0 - 1) / t0 * sp[u];
      add[2][u] = (c1[u] + t1 - 1) / t1 * sp[u];
      add[3][u] = (c0[u] + c1[u] + t2 - 1) / t2;
      add[4][u] = (c0[u] + c1[u]) * sp[u];
#pragma unroll
      for (int c = 0; c < 5; ++c) sum[c] += add[c][u];
    }
    int run[5], tot[5];
    block_exclusive_scan<5>(sum, run, tot, tmp);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      run[c] += carry[c];
      carry[c] += tot[c];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int v = add[c][u];
        add[c][u] = run[c];
        run[c] += v;
      }
    }
    store8(first, r0, G, add[0]);
    store8(b.lists.ioff[LIST_SLOT0], r0, G, add[1]);
    store8(b.lists.ioff[LIST_REST], r0, G, add[2]);
    store8(b.lists.ioff[LIST_ALL], r0, G, add[3]);
    if (lists) store8(lists, r0, G, add[4]);
  }
  if (threadIdx.x == 0) {
    b.lists.ioff[LIST_SLOT0][G] = carry[1];
    b.lists.ioff[LIST_REST][G] = carry[2];
    b.lists.ioff[LIST_ALL][G] = carry[3];
    if (b.lists_to) *b.lists_to = carry[4];
  }
}

// Pair p of rank r: its place in the order and its first candidate list.  start
// is the rank's first place, lists its first list, at the pair's number among
// the rank's pairs (slot 0 first).
__device__ __forceinline__ void place_pair(const Buckets& b, int p, int r, int start, int lists, int at) {
  b.order[start + at] = p;
  if (b.lbase) b.lbase[p] = lists + at * b.nsplit_rank[r];
}

// One decoded work item (see ItemDesc).
__device__ __forceinline__ void write_item(const Buckets& b, int it, int nP, int n0) {
  ItemDesc d{};
  const int G = b.G;
  // largest rank with ioff[rank] <= item
  auto rank_of = [&](const int32_t* ioff, int item) {
    int lo = 0, hi = G;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (ioff[mid] <= item)
        lo = mid;
      else
        hi = mid;
    }
    return lo;
  };
  if (it < nP) {
    const int r = rank_of(b.lists.ioff[LIST_ALL], it);
    const int tp = b.lists.tile[LIST_ALL];
    const int first = (it - b.lists.ioff[LIST_ALL][r]) * tp;
    d.g = b.gorder ? b.gorder[r] : r;
    d.off = b.gstart[r] + first;
    d.cnt = min(tp, b.cnt[r] + b.cnt[G + r] - first);
    d.c0 = d.c1 = it;
  } else {
    const bool s0 = it < nP + n0;
    const int L = s0 ? LIST_SLOT0 : LIST_REST;
    const int li = it - (s0 ? nP : nP + n0);
    const int r = rank_of(b.lists.ioff[L], li);
    const int c0 = b.cnt[r], lc = s0 ? c0 : b.cnt[G + r];
    const int qt = b.lists.tile[L];
    const int ntiles = (lc + qt - 1) / qt;
    const int k = li - b.lists.ioff[L][r];
    const int first = k % ntiles * qt;  // range-major: a range's tiles run together
    const int base = (s0 ? 0 : c0) + first;
    d.g = b.gorder ? b.gorder[r] : r;
    d.range = k / ntiles;
    d.off = b.gstart[r] + base;
    d.cnt = min(qt, lc - first);
    // a grain's projection list is its slot-0 pairs followed by the others, in
    // 16-pair items when the fused kernel projects (the only reader of c0 / c1):
    // this tile's pairs lie in items c0 .. c1 (at most two)
    const int pi0 = b.lists.ioff[LIST_ALL][r];
    d.c0 = pi0 + base / 16;
    d.c1 = pi0 + (base + d.cnt - 1) / 16;
  }
  b.items[it] = d;
}

// Every item of the table, dealt out to `stride` threads from `first` on.
__device__ __forceinline__ void write_items(const Buckets& b, int64_t first, int64_t stride) {
  const int G = b.G;
  const int nP = b.lists.ioff[LIST_ALL][G], n0 = b.lists.ioff[LIST_SLOT0][G], n1 = b.lists.ioff[LIST_REST][G];
  for (int64_t it = first; it < (int64_t)nP + n0 + n1; it += stride) write_item(b, (int)it, nP, n0);
}

// The pairs' numbers and the counts.  Up to SMALL_GRAINS grains a workgroup
// numbers its 4,096 pairs in the LDS and reserves one run per grain and kind
// with a single global atomic: 13 us for 262,144 pairs over 8,192 grains, where
// a global atomic per pair takes 31 us, and longer yet over fewer grains.
template <bool LDS>
__global__ __launch_bounds__(1024) void bucket_count_kernel(Buckets b, const int32_t* __restrict__ probes,
                                                            int64_t n, int P) {
  __shared__ int cnt[LDS ? 2 * SMALL_GRAINS : 1];
  constexpr int U = 4;
  const int G = b.G;
  const int64_t e0 = (int64_t)blockIdx.x * (U * 1024) + threadIdx.x;
  int at[U], key[U];  // key: the pair's counter
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t p = pair_of(b, e0 + u * 1024, P);
    const int g = e0 + u * 1024 < n ? probe_of(b, probes, p, P) : -1;
    key[u] = g < 0 ? -1 : (b.grank ? b.grank[g] : g) + (p % P == 0 ? 0 : G);
  }
  if constexpr (LDS) {
    for (int r = threadIdx.x; r < 2 * G; r += 1024) cnt[r] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (key[u] >= 0) at[u] = atomicAdd(&cnt[key[u]], 1);
    __syncthreads();
    for (int r = threadIdx.x; r < 2 * G; r += 1024) {
      const int n = cnt[r];
      if (n) cnt[r] = atomicAdd(&b.cnt[r], n);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (key[u] >= 0) b.slot[e0 + u * 1024] = cnt[key[u]] + at[u];
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (key[u] >= 0) b.slot[e0 + u * 1024] = atomicAdd(&b.cnt[key[u]], 1);
  }
}

__global__ __launch_bounds__(1024) void bucket_scan_kernel(Buckets b) {
  scan_ranks(b, b.cnt, b.cnt + b.G, b.G % 4 == 0, b.gstart, b.glist);
}

// Workgroups below pair_wgs place pairs, the others write the item table.
__global__ __launch_bounds__(256) void bucket_place_kernel(Buckets b, const int32_t* __restrict__ probes,
                                                           int64_t n, int P, int pair_wgs) {
  if ((int)blockIdx.x >= pair_wgs) {
    write_items(b, (int64_t)((int)blockIdx.x - pair_wgs) * 256 + threadIdx.x,
                (int64_t)((int)gridDim.x - pair_wgs) * 256);
    return;
  }
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  const int64_t p = pair_of(b, e, P);
  const int g = probe_of(b, probes, p, P);
  if (g < 0) return;
  const int r = b.grank ? b.grank[g] : g;
  const int at = b.slot[e] + ((p % P) == 0 ? 0 : b.cnt[r]);
  place_pair(b, (int)p, r, b.gstart[r], b.lbase ? b.glist[r] : 0, at);
}

__global__ __launch_bounds__(1024) void bucket_small_kernel(Buckets b, const int32_t* __restrict__ probes, int n,
                                                            int P) {
  __shared__ __align__(16) int cnt[2][SMALL_GRAINS], first[SMALL_GRAINS], lists[SMALL_GRAINS];
  constexpr int U = SMALL_PAIRS / 1024;
  const int G = b.G;
  int pair[U], rank[U], at[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = (int)threadIdx.x + u * 1024;
    pair[u] = (int)pair_of(b, e, P);
    const int g = e < n ? probe_of(b, probes, pair[u], P) : -1;
    rank[u] = g < 0 ? -1 : b.grank ? b.grank[g] : g;
  }
  for (int r = threadIdx.x; r < G; r += 1024) cnt[0][r] = cnt[1][r] = 0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (rank[u] >= 0) at[u] = atomicAdd(&cnt[pair[u] % P == 0 ? 0 : 1][rank[u]], 1);
  __syncthreads();
  scan_ranks(b, cnt[0], cnt[1], true, first, lists);
  __syncthreads();
  for (int r = threadIdx.x; r < G; r += 1024) {
    b.gstart[r] = first[r];
    b.cnt[r] = cnt[0][r];
    b.cnt[G + r] = cnt[1][r];
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (rank[u] >= 0) {
      const int p = pair[u], r = rank[u];
      place_pair(b, p, r, first[r], lists[r], at[u] + (p % P == 0 ? 0 : cnt[0][r]));
    }
  __syncthreads();  // the arrays written above are read back by other threads of this workgroup
  if (b.items) write_items(b, threadIdx.x, 1024);
}

__global__ void fill_i32_kernel(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace

// Fill with a kernel rather than hipMemsetAsync, so that captured graphs hold
// only kernel nodes.
void launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  HIP_TRY(hipGetLastError());
}

void launch_bucket(const int32_t* probes, int64_t nq, int P, const Buckets& b, hipStream_t s, bool counts_zeroed) {
  const int64_t n = b.pick == PICK_SLOT0 ? nq : nq * P;
  if (n <= 0) return;
  if (n <= SMALL_PAIRS && b.G <= SMALL_GRAINS) {
    Buckets one = b;
    // a long item table is written by many workgroups
    const bool inside = b.items && b.items_cap <= SMALL_PAIRS;
    if (!inside) one.items = nullptr;
    hipLaunchKernelGGL(bucket_small_kernel, dim3(1), dim3(1024), 0, s, one, probes, (int)n, P);
    HIP_TRY(hipGetLastError());
    if (!b.items || inside) return;
    const unsigned iwgs = (unsigned)std::min<int64_t>((b.items_cap + 255) / 256, ITEM_WGS);
    hipLaunchKernelGGL(bucket_place_kernel, dim3(iwgs), dim3(256), 0, s, b, probes, n, P, 0);
    HIP_TRY(hipGetLastError());
    return;
  }
  if (!counts_zeroed) launch_fill_i32(b.cnt, 2 * (int64_t)b.G, 0, s);
  const unsigned pwgs = (unsigned)((n + 255) / 256);
  const dim3 cgrid((unsigned)((n + 4095) / 4096));
  if (b.G <= SMALL_GRAINS)
    hipLaunchKernelGGL(bucket_count_kernel<true>, cgrid, dim3(1024), 0, s, b, probes, n, P);
  else
    hipLaunchKernelGGL(bucket_count_kernel<false>, cgrid, dim3(1024), 0, s, b, probes, n, P);
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(1024), 0, s, b);
  const unsigned iwgs = b.items ? (unsigned)std::min<int64_t>((b.items_cap + 255) / 256, ITEM_WGS) : 0;
  hipLaunchKernelGGL(bucket_place_kernel, dim3(pwgs + iwgs), dim3(256), 0, s, b, probes, n, P, (int)pwgs);
  HIP_TRY(hipGetLastError());
}

}  // namespace hntl
