// Scan dispatch by code form, and the per-grain code bounding boxes used by
// the exact pruning of the scan.
#include <algorithm>
#include <cmath>

#include "hntl_device.h"
#include "hntl_internal.h"

namespace hntl {

void launch_scan_ct0(const Index&, const float*, const float*, int, int, const Buckets&, int, uint64_t*,
                     const uint64_t*, bool, bool, unsigned long long*, hipStream_t);
void launch_scan_ct1(const Index&, const float*, const float*, int, int, const Buckets&, int, uint64_t*,
                     const uint64_t*, bool, bool, unsigned long long*, hipStream_t);
void launch_scan_ct2(const Index&, const float*, const float*, int, int, const Buckets&, int, uint64_t*,
                     const uint64_t*, bool, bool, unsigned long long*, hipStream_t);
void launch_scan_ct3(const Index&, const float*, const float*, int, int, const Buckets&, int, uint64_t*,
                     const uint64_t*, bool, bool, unsigned long long*, hipStream_t);

namespace {

// Per grain: minimum and maximum of every code coordinate, the smallest eps and
// an upper bound of the longest code over its members (one workgroup per grain).
__global__ __launch_bounds__(256) void grain_bounds_kernel(const float* __restrict__ codes,
                                                           const float* __restrict__ eps, int rp, int r,
                                                           const int32_t* __restrict__ goff,
                                                           const int32_t* __restrict__ boff, float* __restrict__ blo,
                                                           float* __restrict__ bhi, float* __restrict__ emin,
                                                           float* __restrict__ rmax) {
  __shared__ float red[256];
  const int g = blockIdx.x;
  const int b0 = boff[g], nb = boff[g + 1] - b0, ng = goff[g + 1] - goff[g];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // coordinates j = w, w + 4, ...: lanes run over members
  for (int j = w; j < rp; j += 4) {
    float mn = __builtin_inff(), mx = -__builtin_inff();
    for (int b = 0; b < nb; ++b)
      if (b * B + lane < ng) {
        const float v = codes[((size_t)(b0 + b) * rp + j) * B + lane];
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      mn = fminf(mn, __shfl_xor(mn, o, 64));
      mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
      // an empty grain gets an empty box (+inf / -inf); rank padding is exact zero
      blo[(size_t)g * rp + j] = j < r ? mn : 0.f;
      bhi[(size_t)g * rp + j] = j < r ? mx : 0.f;
    }
  }
  float e = __builtin_inff();
  for (int i = threadIdx.x; i < nb * B; i += 256)
    if (i < ng) e = fminf(e, eps[(size_t)b0 * B + i]);
  red[threadIdx.x] = e;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] = fminf(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) emin[g] = red[0];
  __syncthreads();
  float n2 = 0.f;  // the largest squared length; lanes run over members
  for (int b = w; b < nb; b += 4)
    if (b * B + lane < ng) {
      float acc = 0.f;
#pragma unroll 8  // (one load at a time: 70 us more in an append to 64 grains of 1,560 x 64)
      for (int j = 0; j < r; ++j) {
        const float v = codes[((size_t)(b0 + b) * rp + j) * B + lane];
        acc = fmaf(v, v, acc);
      }
      n2 = fmaxf(n2, acc);
    }
  red[threadIdx.x] = n2;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) rmax[g] = sqrtf(red[0]) * (1.f + 1e-5f);
}

// ---------------------------------------------- pruning before projection
// For a pair (q, g) let p = ||q - mu_g||^2, t = ||z_q|| and R >= ||z_i|| for
// every member i.  The score's tangent part is at least (t - R)^2 when t >= R, and
// eps_q = max(0, p - t^2), so
//
//   D_i >= (t - R)^2 + max(0, p - t^2) + eps_i >= (sqrt(p) - R)^2 + eps_min    for sqrt(p) > R
//
// (for t^2 <= p the left side is p + R^2 - 2 t R, smallest at t = sqrt(p); beyond
// it, it grows).  This holds for any z_q that eps_q was computed from, whatever
// the basis and the projection's precision, and needs no projection.  With
// reduced codes R covers the decoded values (BF16 2^-8 relative; FP8 2^-4
// relative plus the subnormal quantum per coordinate).  The int16 form clamps
// z_q after eps_q is taken, so it has no such bound.
//
// Margins, in roundings of u = 2^-24 (the score's own sums and p sum the same FP32
// squares (q - mu)_j^2).  The bound holds with p as the projection sums it for eps_q: four
// chains of d / 4 terms and two additions, at worst 1 - (d / 4 + 2) u of the true sum;
// the p used here (routing: 64 chains of d / 64 terms, at most four more, and six additions)
// is at worst 1 + (d / 64 + 10) u of it.  A square root halves both, so the length is at most
// (0.133 d + 6) u = 8e-9 d + 4e-7 too long, and delta = 1e-5 + 1e-8 d on both lengths covers it
// for every d (R's sum of up to 64 squares is rounded up where it is made).  ||z_q||^2
// within eps_q has eight roundings, 5e-7 p of the square at most: 4e-6 p.  The scan's sums
// over z_q - z_i are off by 70 u of the score: PRUNE_SLACK as there.
constexpr float PRUNE_SLACK = 1e-4f;

struct PruneForm {
  float rel;            // R grows by this factor ...
  const float* scales;  // ... and with FP8 codes by scales[g] * quantum
  float quantum;
  float delta;
};

__device__ __forceinline__ bool pruned(float p, float bound, float rmax, float emin, const PruneForm& f, int g) {
  const float R = rmax * f.rel + (f.scales ? f.scales[g] * f.quantum : 0.f);
  const float a = sqrtf(p) * (1.f - f.delta) - R * (1.f + f.delta);
  if (!(a > 0.f)) return false;
  return (a * a - 4e-6f * p + emin) * (1.f - PRUNE_SLACK) > bound;
}

// The query's bound as a float (+inf: none).
__device__ __forceinline__ float query_bound(const PruneArgs& a, int64_t q) {
  if (a.qbound) return a.qbound[q] == 0xFFFFFFFFu ? __builtin_inff() : ord2f(a.qbound[q]);
  return key_ceil(a.part[(size_t)q * a.P * a.C + a.C - 1]);
}

__global__ __launch_bounds__(256) void prune_pairs_kernel(PruneArgs a, int G, const float* __restrict__ rmax,
                                                          const float* __restrict__ emin, PruneForm f,
                                                          const int32_t* __restrict__ goff) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= a.nq * a.P) return;
  const int64_t q = p / a.P;
  int g = a.probes[p];
  if (p % a.P != 0 && (g < 0 || g >= G || (pruned(a.pdist[p], query_bound(a, q), rmax[g], emin[g], f, g) &&
                                           !small_first_grain(a.probes, q, a.P, G, goff, a.need))))
    g = -1;
  a.kept[p] = g;
}

// Without routing distances (learned routing, injected probes): one wave per
// query computes its pairs' ||q - mu||^2 by direct differences, four at a time.
__global__ __launch_bounds__(256) void prune_pairs_dist_kernel(PruneArgs a, int G, const float* __restrict__ rmax,
                                                               const float* __restrict__ emin, PruneForm f,
                                                               const int32_t* __restrict__ goff,
                                                               const float* __restrict__ Q, int d,
                                                               const float* __restrict__ centroids) {
  const int lane = lane_id();
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= a.nq) return;
  const float bound =
      small_first_grain(a.probes, q, a.P, G, goff, a.need) ? __builtin_inff() : query_bound(a, q);
  const int own = lane < a.P ? a.probes[q * a.P + lane] : -1;  // HNTL_MAX_P < 64
  int keep = own;
  uint64_t m = __ballot(lane > 0 && own >= 0 && own < G && bound < __builtin_inff());
  if (lane > 0 && (own < 0 || own >= G)) keep = -1;
  const float* x = Q + q * d;
  constexpr int U = 4;
  while (m) {  // wave-uniform
    int s[U], g[U];
    const float* mu[U];
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = m ? __builtin_ctzll(m) : s[0];
      m &= m - 1;
      g[u] = __builtin_amdgcn_readlane(own, s[u]);
      mu[u] = centroids + (size_t)g[u] * d;
      acc[u] = 0.f;
    }
    for (int t = lane; t < d; t += HNTL_WAVE) {
      const float v = x[t];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float df = v - mu[u][t];
        acc[u] = fmaf(df, df, acc[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float p = wave_sum(acc[u]);
      if (pruned(p, bound, rmax[g[u]], emin[g[u]], f, g[u]) && lane == s[u]) keep = -1;
    }
  }
  if (lane < a.P) a.kept[q * a.P + lane] = keep;
}

// What the pruning is likely to keep, from the grains alone (one workgroup per sampled grain
// g, `near` its P nearest centroids): a query among g's members lies about
// rho = mean(||z_i||^2 + eps_i) from mu_g, thus sqrt(||mu_g - mu_h||^2 + rho) from mu_h, and its C-th
// best score is near 1.5 rho.  kept[sample]: the other slots that the pruning's bound
// would keep then (every one where g has at most C members and leaves no bound).
constexpr int KEPT_BLOCKS = 16;  // blocks of a grain that rho is taken over, a wave each
__global__ __launch_bounds__(64 * KEPT_BLOCKS) void expected_kept_kernel(const int32_t* __restrict__ sample,
                                                            const int32_t* __restrict__ near,
                                                            const float* __restrict__ near_dist, int P, int C, int G,
                                                            const float* __restrict__ codes,
                                                            const float* __restrict__ eps, int rp, int r,
                                                            const int32_t* __restrict__ goff,
                                                            const int32_t* __restrict__ boff,
                                                            const float* __restrict__ rmax,
                                                            const float* __restrict__ emin, int* __restrict__ kept) {
  __shared__ float red[64 * KEPT_BLOCKS];
  const int g = sample[blockIdx.x];
  const int b0 = boff[g], ng = goff[g + 1] - goff[g], nb = min(boff[g + 1] - b0, KEPT_BLOCKS);
  const int lane = lane_id(), b = threadIdx.x >> 6;
  float sum = 0.f;
  if (b < nb && b * B + lane < ng) {
    sum = eps[(size_t)(b0 + b) * B + lane];
#pragma unroll 8
    for (int j = 0; j < r; ++j) {
      const float v = codes[((size_t)(b0 + b) * rp + j) * B + lane];
      sum = fmaf(v, v, sum);
    }
  }
  red[threadIdx.x] = sum;
  __syncthreads();
  for (int o = 32 * KEPT_BLOCKS; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float rho = red[0] / (float)max(1, min(ng, KEPT_BLOCKS * B));
  bool keep = false;
  if ((int)threadIdx.x >= 1 && (int)threadIdx.x < P) {
    const int h = near[blockIdx.x * P + threadIdx.x];
    keep = ng <= C;
    if (h >= 0 && h < G) {
      const float a = sqrtf(near_dist[blockIdx.x * P + threadIdx.x] + rho) - rmax[h];
      keep |= !(a > 0.f && a * a + emin[h] > 1.5f * rho);
    }
  }
  const int n = __popcll(__ballot(keep));  // HNTL_MAX_P < 64: all in the first wave
  if (threadIdx.x == 0) kept[blockIdx.x] = n;
}

__global__ void sample_rows_kernel(const float* __restrict__ X, int d, const int32_t* __restrict__ rows,
                                   float* __restrict__ out) {
  for (int j = threadIdx.x; j < d; j += blockDim.x) out[(size_t)blockIdx.x * d + j] = X[(size_t)rows[blockIdx.x] * d + j];
}

// Entry C - 1 of every query's probe-slot-0 list set to KEY_NONE: a list that
// no scan item writes (its probe is outside 0 .. G-1) then bounds nothing.
__global__ void reset_slot0_tail_kernel(uint64_t* __restrict__ part, int64_t nq, int P, int C) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nq) part[(size_t)q * P * C + C - 1] = KEY_NONE;
}

}  // namespace

void launch_reset_slot0_tail(uint64_t* part, int64_t nq, int P, int C, hipStream_t s) {
  if (nq <= 0) return;
  hipLaunchKernelGGL(reset_slot0_tail_kernel, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s, part, nq, P, C);
  HIP_TRY(hipGetLastError());
}

void launch_scan(const Index& ix, int codes, const float* T, const float* epsq, int P, int C, const Buckets& b,
                 int list, uint64_t* part, const uint64_t* bound_lists, bool prune, bool narrow,
                 unsigned long long* scored, hipStream_t s) {
  if (b.max_items[list] <= 0) return;
  if (codes == HNTL_CODES_FP32)
    launch_scan_ct0(ix, T, epsq, P, C, b, list, part, bound_lists, prune, narrow, scored, s);
  else if (codes == HNTL_CODES_BF16)
    launch_scan_ct1(ix, T, epsq, P, C, b, list, part, bound_lists, prune, narrow, scored, s);
  else if (codes == HNTL_CODES_FP8_E4M3)
    launch_scan_ct2(ix, T, epsq, P, C, b, list, part, bound_lists, prune, narrow, scored, s);
  else
    launch_scan_ct3(ix, T, epsq, P, C, b, list, part, bound_lists, prune, narrow, scored, s);
  HIP_TRY(hipGetLastError());
}

void launch_grain_bounds(Index& ix, hipStream_t s) {
  if (!ix.blo) ix.blo = dev_alloc<float>(&ix, (size_t)ix.G * ix.rp);
  if (!ix.bhi) ix.bhi = dev_alloc<float>(&ix, (size_t)ix.G * ix.rp);
  if (!ix.emin) ix.emin = dev_alloc<float>(&ix, ix.G);
  if (!ix.rmax) {
    ix.rmax = dev_alloc<float>(&ix, (size_t)ix.G + 1);
    ix.cnmax = ix.rmax + ix.G;
  }
  launch_norm_max(ix.cnorm, (int)ix.G, ix.cnmax, s);
  int64_t upto[9] = {};  // members of grains of 2^(k-1) + 1 .. 2^k
  for (uint32_t g = 0; g < ix.G; ++g) {
    const int64_t ng = ix.offsets_h[g + 1] - ix.offsets_h[g];
    int k = 0;
    while (k <= 8 && ng > (1 << k)) ++k;
    if (k <= 8) upto[k] += ng;
  }
  int64_t n = 0;
  for (int k = 0; k <= 8; ++k) {
    n += upto[k];
    ix.small_share[k] = (float)((double)n / (double)std::max<uint64_t>(ix.N, 1));
  }
  hipLaunchKernelGGL(grain_bounds_kernel, dim3(ix.G), dim3(256), 0, s, ix.codes, ix.eps, (int)ix.rp, (int)ix.r,
                     ix.goff, ix.boff, ix.blo, ix.bhi, ix.emin, ix.rmax);
  HIP_TRY(hipGetLastError());
}

// Share of the pairs of slots 1 .. P - 1 that the pruning is expected to keep, over grains
// sampled by their members.  On fourteen built indexes (patches of several
// spreads, one to eight grains a patch, a single Gaussian cloud) it was within 0.07 of the share
// that 2,000 queries kept.
float expected_kept(const Index& ix, int P, int C, hipStream_t s) {
  constexpr int S = 64;
  if (P < 2 || ix.N == 0) return 0.f;
  std::vector<int32_t> sample(S);
  for (int i = 0; i < S; ++i) {
    const int64_t at = (int64_t)((2 * i + 1) * ix.N / (2 * S));
    sample[i] = (int32_t)(std::upper_bound(ix.offsets_h.begin(), ix.offsets_h.end(), at) - ix.offsets_h.begin()) - 1;
  }
  const int G = (int)ix.G, d = (int)ix.d;
  Scratch sc(s);
  int32_t* rows = sc.get<int32_t>(S);
  float* A = sc.get<float>((size_t)S * d);
  float* an = sc.get<float>(S);
  float* D = sc.get<float>((size_t)S * G);
  int32_t* near = sc.get<int32_t>((size_t)S * P);
  float* near_dist = sc.get<float>((size_t)S * P);
  int* kept = sc.get<int>(S);
  HIP_TRY(hipMemcpyAsync(rows, sample.data(), sizeof(int32_t) * S, hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(sample_rows_kernel, dim3(S), dim3(256), 0, s, ix.centroids, d, rows, A);
  HIP_TRY(hipGetLastError());
  launch_row_norms(A, S, d, an, s);
  launch_dist_matrix(A, an, S, ix.centroids, ix.cnorm, G, d, D, s);
  launch_topk_rows(D, S, G, P, near, near_dist, s, A, an, ix.centroids, ix.cnorm, ix.cnmax, d, route_err(ROUTE_F32));
  hipLaunchKernelGGL(expected_kept_kernel, dim3(S), dim3(64 * KEPT_BLOCKS), 0, s, rows, near, near_dist, P, C, G, ix.codes, ix.eps,
                     (int)ix.rp, (int)ix.r, ix.goff, ix.boff, ix.rmax, ix.emin, kept);
  HIP_TRY(hipGetLastError());
  std::vector<int> n(S);
  HIP_TRY(hipMemcpyAsync(n.data(), kept, sizeof(int) * S, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  int64_t sum = 0;
  for (int v : n) sum += v;
  return (float)((double)sum / (double)(S * (P - 1)));
}

// Scanning slot 0 first, pruning, then bucketing, projecting and scanning what is
// left takes four more launches (10 us in a plan's graph, less where a stream of
// single launches waits for the GPU) than one projection of every pair, and what is kept
// pays them again: a second bucketing, bases and codes read twice.  Measured
// with and without on 20 to 10,000 queries over indexes of 20,000 to 400,000
// rows, uniform and Zipf sizes, grains apart and overlapping:
//  - plans, where nothing is kept: even near 64 MB of bases and query rows or 12,000 pairs
//    (100 x 12 over 1,024 x 768: 165 -> 158 us; 3,000 x 8 over 256 x 256: 220 -> 196; 100 x 8 over
//    256 x 256: 89 -> 98).  Of 2,000 x 8 pairs over 512 x 768 it gains 10 to 16% with none kept
//    and loses 8 to 10% with 0.14 kept and up to 31% with all kept (410 -> 538 us); of 10,000 x 8
//    it gains 10% with none kept, nothing with 0.4 to 0.7, and loses 3 to 14% with all.  So what is
//    dropped has to make up for the lot and a quarter of what is kept;
//  - staged searches: even near 700 pairs (100 x 8 over 256 x 768: 130 -> 119 us; 20 x 8:
//    107 -> 111) where few queries' nearest grain is too small to bound them;
//    their pairs are all left, and packed 16 or 4 to a wave they run longer
//    (3,000 x 8 over 1,024 Zipf-sized grains, 5% of the members in grains of at
//    most C: 457 -> 471), until the projection saved outweighs it.  With all kept the narrow
//    second scan still makes up for most of it (512 grains of one cloud, 256 and 768 wide: 300
//    queries 156 -> 144 and 181 -> 182 us, 10,000 468 -> 451 and 736 -> 726; at worst 148 -> 169).
bool prune_pays(const Index& ix, const hntl_search_params& sp, int64_t nq, bool plan, float kept) {
  if (sp.P < 2 || (sp.flags & HNTL_FLAG_NO_PRUNE) || sp.codes == HNTL_CODES_INT16) return false;
  // the learned router's probe budget has dropped most of them already
  if (sp.route == HNTL_ROUTE_LEARNED && sp.mass > 0.f && sp.mass < 1.f) return false;
  const int64_t rest = nq * (sp.P - 1);
  const int64_t basis = std::min<int64_t>(ix.G, rest) * ix.r * ((sp.flags & HNTL_FLAG_PROJECT_BF16) ? 2 : 4);
  const int64_t bytes = (basis + rest * 4) * ix.d;
  const double gain = 1.0 - 1.25 * kept;
  if (plan) return gain * (double)bytes >= 67108864.0 || gain * (double)rest >= 12288.0;
  int k = 0;
  while (k < 8 && (1u << k) < sp.C) ++k;
  if (ix.small_share[k] <= 0.02f) return rest >= 704;
  return bytes >= ((int64_t)128 << 20) && rest >= 8192;
}

void launch_prune_pairs(const Index& ix, int codes, const float* Q, const PruneArgs& a, hipStream_t s) {
  if (a.nq <= 0) return;
  PruneForm f{1.f, nullptr, 0.f, 1e-5f + 1e-8f * (float)ix.d};
  if (codes == HNTL_CODES_BF16) f.rel = 1.f + 0.00390625f;
  if (codes == HNTL_CODES_FP8_E4M3) f = PruneForm{1.0625f, ix.scales, sqrtf((float)ix.rp) * 0.0009765625f, f.delta};
  if (a.pdist)
    hipLaunchKernelGGL(prune_pairs_kernel, dim3((unsigned)((a.nq * a.P + 255) / 256)), dim3(256), 0, s, a, (int)ix.G,
                       ix.rmax, ix.emin, f, ix.goff);
  else
    hipLaunchKernelGGL(prune_pairs_dist_kernel, dim3((unsigned)((a.nq + 3) / 4)), dim3(256), 0, s, a, (int)ix.G,
                       ix.rmax, ix.emin, f, ix.goff, Q, (int)ix.d, ix.centroids);
  HIP_TRY(hipGetLastError());
}

}  // namespace hntl
