// Grain-major projection kernels (paper Section 2.2, eq. 1-4).  Two item
// sizes over the grain-bucketed pairs:
//   * PT (16) pairs: a single-wave workgroup per item, the basis streamed from
//     L2 (small batches, where most grains hold a pair or two);
//   * PROJECT_TILE pairs: a workgroup of PROJECT_TILE / 16 waves per item; the
//     grain's basis and centroid pass through LDS once per workgroup in depth
//     chunks, and every wave projects its 16 rows from there.
// Both give bit-identical tangents: the MFMA operands and their order per 32
// depths are those of project_wave / project_wave_bf16.
#include <type_traits>

#include "project_impl.h"

namespace hntl {

namespace {

using namespace proj_detail;

template <bool VEC, int NCT>
__global__ __launch_bounds__(64) void project_kernel(
    const float* __restrict__ Q, int d, int P, const float* __restrict__ centroids, const float* __restrict__ basis,
    int r, ListRef list, int G, const int32_t* __restrict__ gorder, const int32_t* __restrict__ order,
    float* __restrict__ T,
    float* __restrict__ epsq) {
  int rank;
  if (!item_grain(list.ioff, G, blockIdx.x, rank)) return;
  const int g = gorder ? gorder[rank] : rank;
  const int first = (blockIdx.x - list.ioff[rank]) * PT;  // within the grain's pairs
  const int cnt = min(PT, list.count(rank) - first);
  if (cnt <= 0) return;
  project_wave<VEC, NCT, true>(Q, d, P, centroids, basis, r, g, order + list.start(rank) + first, cnt, T, epsq);
}

template <int NCT>
__global__ __launch_bounds__(64) void project_bf16_kernel(
    const float* __restrict__ Q, int d, int P, const float* __restrict__ centroids,
    const uint16_t* __restrict__ basis16, int r, ListRef list, int G, const int32_t* __restrict__ gorder,
    const int32_t* __restrict__ order, float* __restrict__ T, float* __restrict__ epsq) {
  int rank;
  if (!item_grain(list.ioff, G, blockIdx.x, rank)) return;
  const int g = gorder ? gorder[rank] : rank;
  const int first = (blockIdx.x - list.ioff[rank]) * PT;
  const int cnt = min(PT, list.count(rank) - first);
  if (cnt <= 0) return;
  project_wave_bf16<NCT>(Q, d, P, centroids, basis16, r, g, order + list.start(rank) + first, cnt, T, epsq);
}

// ---- shared-basis form
constexpr int GK = 64;   // depths per LDS chunk (two 32-depth MFMA groups)
constexpr int XRUN = 4;  // consecutive items kept on one XCD

// Item of workgroup `b`: workgroups are dealt to the 8 XCDs round-robin
// (b % 8), so XCD x's k-th workgroup (k = b / 8) takes item
// ((k / XRUN) 8 + x) XRUN + k % XRUN.  Runs of XRUN consecutive items (the
// items of one grain are consecutive) then share one L2, while whole runs
// still alternate over the XCDs.  The map is a bijection on [0, 8 XRUN m) for a
// grid of 8 XRUN m workgroups.
__device__ __forceinline__ int xcd_item(int b) {
  const int x = b & 7, k = b >> 3;
  return ((k / XRUN) * 8 + x) * XRUN + k % XRUN;
}

// A workgroup of NW waves projects up to 16 NW pairs of one grain.  Per depth
// chunk k0 .. k0 + GK - 1: every thread loads its share of the 16 NCT basis rows
// (zero rows from r on, zeros from d on) and of the centroid into registers,
// then LDS; each wave reads its 16 query rows' slices straight from memory into
// registers (PD chunks are in flight while one is multiplied) and forms
// q' = q - mu in FP32.  Two LDS buffers, one barrier per chunk.  Lane (i, kq)
// feeds depth 32 h + 8 kq + e of row / basis row i of chunk half h, as in
// project_wave (FP32: 8 steps of 16x16x4, e = step) and project_wave_bf16
// (one 16x16x32 BF16 step, e = 0..7).  Needs d % 4 == 0 (FP32) or d % 8 == 0
// (BF16) and 16-byte aligned rows.
template <bool BF16, int NCT, int NW, int PD>
__global__ __launch_bounds__(64 * NW) void project_lds_kernel(
    const float* __restrict__ Q, int d, int P, const float* __restrict__ centroids, const float* __restrict__ basis,
    const uint16_t* __restrict__ basis16, int r, ListRef list, int G, const int32_t* __restrict__ gorder,
    const int32_t* __restrict__ order, float* __restrict__ T, float* __restrict__ epsq) {
  using E = std::conditional_t<BF16, uint16_t, float>;
  constexpr int ROWS = 16 * NCT;
  constexpr int EPV = 16 / (int)sizeof(E);    // elements per 16-byte vector
  constexpr int VPR = GK / EPV;               // vectors per basis row and chunk
  constexpr int RS = GK + EPV;                // padded LDS row stride (elements): rows start 16 B apart in the banks
  constexpr int NB = ROWS * VPR;              // basis vectors per chunk
  constexpr int NV = NB + GK / 4;             // + centroid vectors (FP32)
  constexpr int NT = 64 * NW;
  static_assert(NB % 64 == 0, "a wave stages basis or centroid vectors");
  constexpr int PER = (NV + NT - 1) / NT;     // vectors staged per thread and chunk
  __shared__ __align__(16) E wsh[2][ROWS * RS];
  __shared__ __align__(16) float msh[2][GK];

  const int item = xcd_item((int)blockIdx.x);
  int rank;
  if (!item_grain(list.ioff, G, item, rank)) return;  // uniform over the workgroup
  const int wave = (int)threadIdx.x >> 6, lane = lane_id();
  const int i = lane & 15, kq = lane >> 4;
  const int g = gorder ? gorder[rank] : rank;
  const int first = (item - list.ioff[rank]) * (16 * NW) + 16 * wave;  // within the grain's pairs
  const int cnt = __builtin_amdgcn_readfirstlane(min(16, list.count(rank) - first));  // <= 0: this wave only stages
  const int32_t* pairs = order + list.start(rank) + (first < 0 ? 0 : first);
  const int qrow = i < cnt ? ldg(pairs + i) / P : -1;
  const float* qp = Q + (size_t)(qrow < 0 ? 0 : qrow) * d;
  const float* mu = centroids + (size_t)g * d;
  const E* Wg = BF16 ? (const E*)(basis16 + (size_t)g * r * d) : (const E*)(basis + (size_t)g * r * d);

  using u32x4 = unsigned int __attribute__((ext_vector_type(4)));
  u32x4 st[PD][PER];
  float qv[PD][16];
  // Requests chunk k0 into register set p: the thread's share of the basis and
  // centroid (bounds-checked buffer loads: zeros past the rank and past d), the
  // lane's query slices (halves h = 0, 1, 8 floats each; depths past d repeat the
  // row's last, which meet zero basis rows and are zeroed at their use).  No
  // branches, so that the sets in flight can be counted.
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  auto request = [&](int p, int k0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int v = u * NT + (int)threadIdx.x;
      const bool basis_part = u * NT + 64 * swave < NB;  // NB is a multiple of 64: the same for the wave
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
          basis_part ? (void*)const_cast<E*>(Wg) : (void*)const_cast<float*>(mu), 0,
          basis_part ? r * d * (int)sizeof(E) : 4 * d, 0x00027000);
      const int row = v / VPR, k = k0 + (v % VPR) * EPV;
      const int at = basis_part ? (row < r && k < d ? (int)sizeof(E) * (row * d + k) : -16)
                                : (v < NV ? 4 * (k0 + (v - NB) * 4) : -16);
      st[p][u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, 0, 0);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 8; e += 4) {
        const int k = min(k0 + 32 * h + 8 * kq + e, d - 4);
        *reinterpret_cast<floatx4*>(&qv[p][8 * h + e]) = ldg(reinterpret_cast<const floatx4*>(qp + k));
      }
  };
  auto stage_store = [&](int p, int buf) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int v = u * NT + (int)threadIdx.x;
      if (v < NB)
        *reinterpret_cast<u32x4*>(&wsh[buf][(v / VPR) * RS + (v % VPR) * EPV]) = st[p][u];
      else if (v < NV)
        *reinterpret_cast<u32x4*>(&msh[buf][(v - NB) * 4]) = st[p][u];
    }
  };

  floatx4 acc[NCT];
#pragma unroll
  for (int c = 0; c < NCT; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
  float sq = 0.f;

  auto compute = [&](int buf, const float (&qv)[16], int k0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (k0 + 32 * h >= d) break;  // uniform: no zero-only MFMA group past d
      const int kl = 32 * h + 8 * kq;
      float m[8];
      *reinterpret_cast<floatx4*>(&m[0]) = *reinterpret_cast<const floatx4*>(&msh[buf][kl]);
      *reinterpret_cast<floatx4*>(&m[4]) = *reinterpret_cast<const floatx4*>(&msh[buf][kl + 4]);
      if constexpr (BF16) {
        u32x4 av;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float v0 = qrow >= 0 ? qv[8 * h + e] - m[e] : 0.f;
          const float v1 = qrow >= 0 ? qv[8 * h + e + 1] - m[e + 1] : 0.f;
          sq = fmaf(v0, v0, fmaf(v1, v1, sq));
          av[e / 2] = bf16_rne_bits(v0) | (bf16_rne_bits(v1) << 16);
        }
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
          const u32x4 bv = *reinterpret_cast<const u32x4*>(&wsh[buf][(c * 16 + i) * RS + kl]);
          acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                            __builtin_bit_cast(bf16x8, bv), acc[c], 0, 0, 0);
        }
      } else {
        float a[8], bw[NCT][8];
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
          const float* src = reinterpret_cast<const float*>(&wsh[buf][(c * 16 + i) * RS + kl]);
          *reinterpret_cast<floatx4*>(&bw[c][0]) = *reinterpret_cast<const floatx4*>(src);
          *reinterpret_cast<floatx4*>(&bw[c][4]) = *reinterpret_cast<const floatx4*>(src + 4);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          a[e] = qrow >= 0 ? qv[8 * h + e] - m[e] : 0.f;
          sq = fmaf(a[e], a[e], sq);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int c = 0; c < NCT; ++c) acc[c] = mfma16x16x4(a[e], bw[c][e], acc[c]);
      }
    }
  };

#pragma unroll
  for (int p = 0; p < PD; ++p) {
    request(p, p * GK);
    __builtin_amdgcn_sched_barrier(0);  // requested in the order of use
  }
  for (int k0 = 0; k0 < d; k0 += PD * GK) {
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      const int kc = k0 + p * GK;
      if (kc >= d) break;
      // the buffer written here was last read two chunks ago, which the barrier between closed
      const int buf = (kc / GK) & 1;
      stage_store(p, buf);
      float cur[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) cur[e] = kc + 32 * (e / 8) + 8 * kq + (e & 4) < d ? qv[p][e] : 0.f;
      __syncthreads();
      request(p, kc + PD * GK);
      if (cnt > 0) compute(buf, cur, kc);
    }
  }
  if (cnt > 0) project_store<NCT>(acc, sq, r, pairs, cnt, T, epsq);
}

}  // namespace

template <bool BF16, bool VEC, int NCT>
void launch_project_k(const Index& ix, const float* Q, int P, const Buckets& b, float* T, float* epsq,
                      hipStream_t s) {
  const ListRef list = list_ref(b, LIST_ALL);
  const int tile = b.lists.tile[LIST_ALL];
  if (tile == PROJECT_TILE && VEC) {
    constexpr int NW = PROJECT_TILE / PT, M = 8 * XRUN;
    const dim3 grid((unsigned)((b.max_items[LIST_ALL] + M - 1) / M * M)), block(64 * NW);
#define HNTL_PROJ(PD)                                                                                              \
  hipLaunchKernelGGL((project_lds_kernel<BF16, NCT, NW, PD>), grid, block, 0, s, Q, (int)ix.d, P, ix.centroids,   \
                     ix.basis, ix.basis_bf16, (int)ix.r, list, (int)ix.G, b.gorder, b.order, T, epsq)
    // Two chunks ahead where the rows are long enough for it and the registers leave
    // four waves a SIMD (BF16, or up to 32 basis rows): 3,001 queries over 1,024 grains
    // at rank 32 58 -> 51 us, BF16 at rank 48 158 -> 150; FP32 at rank 48 222 -> 237,
    // rows of 128 26 -> 32.  Four ahead lost everywhere (62, 168, 282, 44).
    if ((BF16 || NCT <= 2) && ix.d >= 4 * GK)
      HNTL_PROJ(2);
    else
      HNTL_PROJ(1);
#undef HNTL_PROJ
    return;
  }
  if (tile != PT) throw ArgError{HNTL_EDEVICE, "projection item size must be 16 pairs (or PROJECT_TILE, vector form)"};
  const dim3 grid((unsigned)b.max_items[LIST_ALL]), block(64);
  if constexpr (BF16)
    hipLaunchKernelGGL((project_bf16_kernel<NCT>), grid, block, 0, s, Q, (int)ix.d, P, ix.centroids, ix.basis_bf16,
                       (int)ix.r, list, (int)ix.G, b.gorder, b.order, T, epsq);
  else
    hipLaunchKernelGGL((project_kernel<VEC, NCT>), grid, block, 0, s, Q, (int)ix.d, P, ix.centroids, ix.basis,
                       (int)ix.r, list, (int)ix.G, b.gorder, b.order, T, epsq);
}

template <bool BF16, bool VEC>
void launch_project_w(const Index& ix, const float* Q, int P, const Buckets& b, float* T, float* epsq, hipStream_t s) {
  switch ((ix.r + 15) / 16) {
    case 1: launch_project_k<BF16, VEC, 1>(ix, Q, P, b, T, epsq, s); break;
    case 2: launch_project_k<BF16, VEC, 2>(ix, Q, P, b, T, epsq, s); break;
    case 3: launch_project_k<BF16, VEC, 3>(ix, Q, P, b, T, epsq, s); break;
    default: launch_project_k<BF16, VEC, 4>(ix, Q, P, b, T, epsq, s); break;
  }
}

int project_tile(const Index& ix, const float* Q, bool bf16) {
  const bool vec = (ix.d % (bf16 ? 8 : 4)) == 0 && ((uintptr_t)Q % 16) == 0;
  return vec ? PROJECT_TILE : PT;
}

void launch_project(const Index& ix, const float* Q, int P, const Buckets& b, float* T, float* epsq, bool bf16,
                    hipStream_t s) {
  if (b.max_items[LIST_ALL] <= 0) return;
  if (bf16) {
    if (!ix.basis_bf16) throw ArgError{HNTL_ESTATE, "BF16 projection needs the BF16 basis (build a reduced-precision code form)"};
    if ((ix.d % 8) != 0 || ((uintptr_t)Q % 16) != 0)
      throw ArgError{HNTL_EUNSUPPORTED, "BF16 projection needs d % 8 == 0 and 16-byte aligned queries"};
    launch_project_w<true, true>(ix, Q, P, b, T, epsq, s);
  } else if ((ix.d % 4) == 0 && ((uintptr_t)Q % 16) == 0) {
    launch_project_w<false, true>(ix, Q, P, b, T, epsq, s);
  } else {
    launch_project_w<false, false>(ix, Q, P, b, T, epsq, s);
  }
  HIP_TRY(hipGetLastError());
}

}  // namespace hntl
