// Learned router: a small MLP that maps a query to one score per grain, whose
// top-P grains replace centroid routing.  The paper routes by centroid
// distance (Section 2.3) and names learned partitioning as future work
// (Section 4); this is that extension.
//
//   xh = bf16((x - mean) / std)                      standardised input
//   h1 = bf16(gelu(W1 xh + b1)),  h2 = bf16(gelu(W2 h1 + b2))
//   s  = W3 h2 + b3                                   one score per grain
//
// GELU is the exact erf form (Hendrycks & Gimpel), computed with the device
// erff.  Weights are FP32 masters with BF16 copies; every GEMM takes BF16
// operands on the MFMA units (v_mfma_f32_16x16x32_bf16) and accumulates in
// FP32; bias, GELU, softmax, loss and Adam run in FP32.
//
// Training (softmax cross-entropy, Adam of Kingma & Ba with bias
// correction) targets the grain distribution of each training query's exact
// k nearest neighbours: the fraction of them in each grain.  Backward pass,
// per batch of B rows (rounding points as the forward: every GEMM operand
// rounded to BF16):
//
//   ds  = (softmax(s) - y) / B;   gW3 = bf16(ds)^T h2,  gb3 = sum_b ds
//   da2 = (bf16(ds) W3) * gelu'(a2);   gW2 = bf16(da2)^T h1,  gb2 = sum_b da2
//   da1 = (bf16(da2) W2) * gelu'(a1);  gW1 = bf16(da1)^T xh,  gb1 = sum_b da1
//
// The GEMM kernel below is the one contraction of all of this: C = A . B^T in
// the sense C[m][n] = sum_k A(m, k) B(n, k), with A and B each stored either
// k-contiguous or (transposed) m- / n-contiguous, staged through LDS.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <numeric>
#include <vector>

#include "hntl_device.h"
#include "hntl_internal.h"

namespace hntl {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float x) {
  return 0.5f * (1.f + erff(x * 0.70710678118654752f)) + x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

// ------------------------------------------------------------------ GEMM

enum { EPI_F32 = 0, EPI_BIAS_GELU = 1, EPI_GELU_GRAD = 2, EPI_BIAS_F32 = 3, EPI_DIST = 4 };
struct Epi {
  float* C;            // FP32 output (EPI_F32, EPI_BIAS_F32: the result; EPI_BIAS_GELU: pre-activation, optional)
  int ldc;
  const float* bias;   // N
  uint16_t* H;         // BF16 output (EPI_BIAS_GELU: gelu(z); EPI_GELU_GRAD: bf16(acc * gelu'(z)))
  int ldh;
  const float* Z;      // EPI_GELU_GRAD: pre-activation
  int ldz;
  float* D;            // EPI_GELU_GRAD: FP32 acc * gelu'(z)
  int ldd;
  float scale;         // EPI_BIAS_F32: result = scale * (acc + bias)
  const float* an;     // EPI_DIST: C = max(an[row] + bn[col] - 2 acc, 0)
  const float* bn;
  int64_t row_base;    // rows from *mlim - row_base on are skipped
};

// Epilogue of one output element (row < M, col < N checked by the caller).
template <int EPI>
__device__ __forceinline__ void epi_store(const Epi& e, int row, int col, float v) {
  if constexpr (EPI == EPI_F32) {
    e.C[(size_t)row * e.ldc + col] = v;
  } else if constexpr (EPI == EPI_BIAS_F32) {
    e.C[(size_t)row * e.ldc + col] = e.scale * (v + e.bias[col]);
  } else if constexpr (EPI == EPI_BIAS_GELU) {
    const float z = v + e.bias[col];
    if (e.C) e.C[(size_t)row * e.ldc + col] = z;
    e.H[(size_t)row * e.ldh + col] = to_bf16(gelu(z));
  } else if constexpr (EPI == EPI_DIST) {
    e.C[(size_t)row * e.ldc + col] = fmaxf(e.an[row] + e.bn[col] - 2.f * v, 0.f);
  } else {
    const float gz = v * gelu_grad(e.Z[(size_t)row * e.ldz + col]);
    e.D[(size_t)row * e.ldd + col] = gz;
    e.H[(size_t)row * e.ldh + col] = to_bf16(gz);
  }
}

// The same epilogue with its per-row term rt (EPI_DIST: an[row]) and per-column
// term ct (EPI_DIST: bn[col]; the bias forms: bias[col]) loaded once per row
// and column by the caller instead of once per element; same arithmetic.
template <int EPI>
__device__ __forceinline__ float epi_row_term(const Epi& e, int row) {
  if constexpr (EPI == EPI_DIST) return e.an[row];
  return 0.f;
}
template <int EPI>
__device__ __forceinline__ float epi_col_term(const Epi& e, int col) {
  if constexpr (EPI == EPI_DIST) return e.bn[col];
  if constexpr (EPI == EPI_BIAS_F32 || EPI == EPI_BIAS_GELU) return e.bias[col];
  return 0.f;
}
template <int EPI>
__device__ __forceinline__ void epi_store_t(const Epi& e, int row, int col, float v, float rt, float ct) {
  if constexpr (EPI == EPI_F32) {
    e.C[(size_t)row * e.ldc + col] = v;
  } else if constexpr (EPI == EPI_BIAS_F32) {
    e.C[(size_t)row * e.ldc + col] = e.scale * (v + ct);
  } else if constexpr (EPI == EPI_BIAS_GELU) {
    const float z = v + ct;
    if (e.C) e.C[(size_t)row * e.ldc + col] = z;
    e.H[(size_t)row * e.ldh + col] = to_bf16(gelu(z));
  } else if constexpr (EPI == EPI_DIST) {
    e.C[(size_t)row * e.ldc + col] = fmaxf(rt + ct - 2.f * v, 0.f);
  } else {
    epi_store<EPI>(e, row, col, v);
  }
}

// CT consecutive output columns of one row, with 4-byte alignment (a row of an odd
// number of columns moves the next one's).
template <class T, int CT>
struct Run {
  typedef T type __attribute__((ext_vector_type(CT), aligned(sizeof(T))));
};

// Stores a wave's RT tiles of 16 rows and its 16 CT columns from (row0, col0), lane i
// of a row holding columns CT i .. CT i + CT - 1 (B's rows go into the MFMAs in that
// order): a store instruction covers whole stretches of 64 CT bytes of four rows.
// With column 16 b + i in tile b every store touched 64 bytes of a row at a time, and
// 16,384 x 8,192 outputs took 227 us to leave (2.4 TB/s); the distances of 16,384 x
// 8,192 x 768 take 268 us (339 before), the scores over 1,024 320 (367).  The row
// and column terms are loaded before the first store: a load after a store would
// wait for it.  NT: FP32 outputs of 64 MB and more, larger than what the caches
// keep for their reader, bypass them (selection after them 227 -> 210 us, 150 ->
// 123 without distances).
template <int EPI, int RT, int CT, bool NT>
__device__ __forceinline__ void tile_store(const Epi& e, const floatx4 (&acc)[RT][CT], int row0, int col0, int M, int N) {
  const int lane = lane_id();
  const int i = lane & 15, kq = lane >> 4;
  const int col = col0 + CT * i;
  float ct[CT], rt[RT][4];
#pragma unroll
  for (int b = 0; b < CT; ++b) ct[b] = epi_col_term<EPI>(e, min(col + b, N - 1));
#pragma unroll
  for (int a = 0; a < RT; ++a)
#pragma unroll
    for (int j = 0; j < 4; ++j) rt[a][j] = epi_row_term<EPI>(e, min(row0 + 16 * a + 4 * kq + j, M - 1));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < RT; ++a)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = row0 + 16 * a + 4 * kq + j;
      if (row >= M) continue;
      if (EPI != EPI_GELU_GRAD && col + CT <= N) {
        typename Run<float, CT>::type v;
        typename Run<uint16_t, CT>::type h;
#pragma unroll
        for (int b = 0; b < CT; ++b) {
          const float x = acc[a][b][j];
          if constexpr (EPI == EPI_F32)
            v[b] = x;
          else if constexpr (EPI == EPI_BIAS_F32)
            v[b] = e.scale * (x + ct[b]);
          else if constexpr (EPI == EPI_DIST)
            v[b] = fmaxf(rt[a][j] + ct[b] - 2.f * x, 0.f);
          else {
            v[b] = x + ct[b];
            h[b] = to_bf16(gelu(v[b]));
          }
        }
        if (EPI != EPI_BIAS_GELU || e.C) {
          auto* out = reinterpret_cast<typename Run<float, CT>::type*>(e.C + (size_t)row * e.ldc + col);
          if constexpr (NT)
            __builtin_nontemporal_store(v, out);
          else
            *out = v;
        }
        if constexpr (EPI == EPI_BIAS_GELU)
          *reinterpret_cast<typename Run<uint16_t, CT>::type*>(e.H + (size_t)row * e.ldh + col) = h;
      } else {
#pragma unroll
        for (int b = 0; b < CT; ++b)
          if (col + b < N) epi_store_t<EPI>(e, row, col + b, acc[a][b][j], rt[a][j], ct[b]);
      }
    }
}

// ----------------------------------------------- small-tile GEMM, any orientation
// C(m, n) = sum_k A(m, k) B(n, k), where XT = false: X(r, k) = X[r * ld + k] (K % 8
// == 0) and XT = true: X(r, k) = X[k * ld + r] (rows % 8 == 0); ld % 8 == 0 and
// 16-byte aligned operands in both.  One workgroup of 4 waves per 64 x 64 tile of
// C, wave w owns a 32 x 32 quarter as 2 x 2 MFMA 16x16x32 tiles: lane (i = lane %
// 16, kq = lane / 16) feeds depths 8 kq .. 8 kq + 7 of row / column i and holds
// C[4 kq + j][i] of each.  Bound by latency at the sizes it is for (products that
// leave 256 x 128 tiles to a fraction of the CUs): four depth tiles of 64 are in
// flight in registers, two LDS buffers, one barrier per depth tile.  A tile row
// is 8 vectors of 8 depths; vector c of row r sits at c ^ ((r ^ r / 8) % 8), so
// neither the 16 rows of an operand read nor the writes of a transposed operand
// (8 rows apart) share banks.  A transposed operand comes in as 8 rows of two
// neighbouring depths a thread, which leave as eight 4-byte pairs.
// Training steps of 1,024 rows over 768-512-512-1024: weight gradients 15 us each,
// input gradients 17, forward products 9 (49 and 59 on 128 x 128 tiles that stored
// transposed operands element by element, 36 on 256 x 128 tiles); 256 x 8,192 x 768:
// 13 us (33 on 256 x 128 tiles).  Tiles are handed to the XCDs in contiguous runs.
constexpr int SM = 64, SK = 64, SPD = 4;

struct SFrag {
  uint4 v[2];
};

// Buffer loads of a depth tile, so that rows and depths past the end (an offset
// past the record count: zeros) need no branch and tiles in flight can be counted.
template <bool XT>
__device__ __forceinline__ void sfetch(SFrag& f, const uint16_t* __restrict__ X, int ld, int R, int K, int r0, int k0) {
  const int t = threadIdx.x;
  const uint16_t* base = X + (XT ? (size_t)k0 * ld + r0 : (size_t)r0 * ld + k0);
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, 0x7FFFFFF0, 0x00027000);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = XT ? 8 * (t & 7) : t >> 2;
    const int k = XT ? 2 * (t >> 3) + h : 16 * (t & 3) + 8 * h;
    const uint32_t off = 2u * (XT ? (uint32_t)k * ld + r : (uint32_t)r * ld + k);
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (r0 + r < R && k0 + k < K) ? off : 0xFFFFFFF0u, 0, 0);
    f.v[h] = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

__device__ __forceinline__ int svec(int r, int c) { return c ^ ((r ^ (r >> 3)) & 7); }

template <bool XT>
__device__ __forceinline__ void sstore(uint16_t (*S)[SK], const SFrag& f) {
  const int t = threadIdx.x;
  if constexpr (!XT) {
    const int r = t >> 2;
#pragma unroll
    for (int h = 0; h < 2; ++h) *reinterpret_cast<uint4*>(&S[r][8 * svec(r, 2 * (t & 3) + h)]) = f.v[h];
  } else {
    const int kp = t >> 3;
    const uint32_t lo[4] = {f.v[0].x, f.v[0].y, f.v[0].z, f.v[0].w};
    const uint32_t hi[4] = {f.v[1].x, f.v[1].y, f.v[1].z, f.v[1].w};
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = 8 * (t & 7) + u;
      // depth 2 kp in the low half, 2 kp + 1 in the high half
      const uint32_t w = u & 1 ? (lo[u / 2] >> 16) | (hi[u / 2] & 0xFFFF0000u) : (lo[u / 2] & 0xFFFFu) | (hi[u / 2] << 16);
      *reinterpret_cast<uint32_t*>(&S[r][8 * svec(r, kp >> 2) + 2 * (kp & 3)]) = w;
    }
  }
}

template <bool AT, bool BT, int EPI>
__global__ __launch_bounds__(256) void gemm_small_kernel(const uint16_t* __restrict__ A, int lda,
                                                         const uint16_t* __restrict__ B, int ldb, int M, int N, int K,
                                                         Epi e, const int32_t* __restrict__ mlim, int tiles_n,
                                                         int ntiles) {
  __shared__ __attribute__((aligned(16))) uint16_t As[2][SM][SK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][SM][SK];
  const int tile = (int)(blockIdx.x % 8) * ((int)gridDim.x / 8) + (int)blockIdx.x / 8;  // the grid is a multiple of 8
  if (tile >= ntiles) return;
  const int m0 = (tile / tiles_n) * SM, n0 = (tile % tiles_n) * SM;
  if (mlim) {
    const int lim = (int)(*mlim - e.row_base);
    if (m0 >= lim) return;
    if (lim < M) M = lim;
  }
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int i = lane & 15, kq = lane >> 4;
  floatx4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  SFrag fa[SPD], fb[SPD];
#pragma unroll
  for (int p = 0; p < SPD; ++p) {  // (tiles past K load nothing)
    sfetch<AT>(fa[p], A, lda, M, K, m0, p * SK);
    sfetch<BT>(fb[p], B, ldb, N, K, n0, p * SK);
    __builtin_amdgcn_sched_barrier(0);  // requested in the order of use
  }
  for (int k0 = 0; k0 < K; k0 += SPD * SK) {
#pragma unroll
    for (int p = 0; p < SPD; ++p) {
      if (k0 + p * SK >= K) break;
      // the buffer written here was last read two depth tiles ago, which the barrier between closed
      sstore<AT>(As[p & 1], fa[p]);
      sstore<BT>(Bs[p & 1], fb[p]);
      __syncthreads();
      sfetch<AT>(fa[p], A, lda, M, K, m0, k0 + (p + SPD) * SK);
      sfetch<BT>(fb[p], B, ldb, N, K, n0, k0 + (p + SPD) * SK);
#pragma unroll
      for (int ks = 0; ks < SK; ks += 32) {
        bf16x8 af[2], bfv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int ra = wm + 16 * t + i, rb = wn + 2 * i + t;
          af[t] = *reinterpret_cast<const bf16x8*>(&As[p & 1][ra][8 * svec(ra, ks / 8 + kq)]);
          bfv[t] = *reinterpret_cast<const bf16x8*>(&Bs[p & 1][rb][8 * svec(rb, ks / 8 + kq)]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfv[b], acc[a][b], 0, 0, 0);
      }
    }
  }
  tile_store<EPI, 2, 2, false>(e, acc, m0 + wm, n0 + wn, M, N);
}

// ------------------------------- 256 x 256 tiles, LDS filled by direct loads
// The same product as gemm_small_kernel<false, false> for large
// shapes with K % 64 == 0.  One workgroup of 8 waves (two per SIMD) per
// 256 x 256 tile of C; wave w owns rows 128 (w / 4) .. + 127 and columns
// 64 (w % 4) .. + 63 as 8 x 4 MFMA 16x16x32 tiles.  Depth tiles of 64 go from
// global memory straight into the LDS (global_load_lds_dwordx4: lane l of a
// wave instruction writes 16 bytes at the instruction's LDS base + 16 l), into
// two buffers: tile k + 1 is requested before tile k is multiplied, so its
// latency hides behind a whole tile of MFMAs, with no registers holding it.
// A row of a depth tile is 8 chunks of 16 bytes, swizzled so that the rows of one
// fragment read spread over the LDS banks (dl_pos). Rows past M
// or N load a valid clamped row (their results are never stored).  Every
// output element is accumulated in the same order as in gemm_small_kernel (depth
// tiles of 64, MFMA steps of 32), so the kernels give identical results.
constexpr int BM = 256, BN = 256;
constexpr int BIG_GROUP = 4;  // row blocks per tile group
constexpr size_t DL_STAGE = (size_t)(BM + BN) * SK * sizeof(uint16_t);  // 64 KiB
constexpr size_t BIG_LDS = 2 * DL_STAGE;

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Position of depth chunk c of row r of a 256 x 64 tile, and what sits at a
// position.  A's fragments read 16 neighbouring rows: chunk c at c ^ (r % 8) of its
// row.  B's read every fourth row: the 16 chunks of a pair of rows are permuted by
// XOR with (r / 4) % 16, so those rows too spread over the banks.
template <bool FOURTH>
__device__ __forceinline__ int dl_pos(int r, int c) {
  return FOURTH ? (r >> 1) * 16 + (((r & 1) * 8 + c) ^ ((r >> 2) & 15)) : r * 8 + (c ^ (r & 7));
}
template <bool FOURTH>
__device__ __forceinline__ void dl_at(int pos, int& r, int& c) {
  if constexpr (FOURTH) {
    const int x = (pos & 15) ^ ((pos >> 5) & 15);
    r = (pos >> 4) * 2 + (x >> 3);
    c = x & 7;
  } else {
    r = pos >> 3;
    c = (pos & 7) ^ (r & 7);
  }
}

// Requests one operand's 256 x 64 depth tile (rows r0.., depths k0..) into
// the LDS at `dst`: 2048 chunks, 4 wave instructions of 64 chunks per wave.
template <bool FOURTH>
__device__ __forceinline__ void dl_fetch(uint16_t* dst, const uint16_t* __restrict__ X, int ld, int R, int r0,
                                         int k0) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int u = h * 8 + wave;  // instruction index: LDS bytes 1024 u .. + 1023
    int row, kc;
    dl_at<FOURTH>(u * 64 + lane, row, kc);
    const int gr = min(r0 + row, R - 1);
    __builtin_amdgcn_global_load_lds((const void*)(X + (size_t)gr * ld + k0 + kc * 8),
                                     (lds_ptr_t)(dst + (size_t)u * 512), 16, 0, 0);
  }
}

// 8 bf16 of row r, depths 8 kc .. 8 kc + 7, of a swizzled depth tile.
template <bool FOURTH>
__device__ __forceinline__ bf16x8 dl_frag(const uint16_t* S, int r, int kc) {
  return *reinterpret_cast<const bf16x8*>(S + (size_t)dl_pos<FOURTH>(r, kc) * 8);
}

template <int EPI>
__global__ __launch_bounds__(512) void gemm_big_kernel(const uint16_t* __restrict__ A, int lda,
                                                       const uint16_t* __restrict__ B, int ldb, int M, int N, int K,
                                                       Epi e, const int32_t* __restrict__ mlim, int tiles_n,
                                                       int ntiles) {
  extern __shared__ __attribute__((aligned(16))) uint16_t dsm[];
  // XCD-contiguous tile order: workgroup b runs on XCD b % 8; inside an XCD's
  // range, tiles go in groups of BIG_GROUP row blocks (down a group's rows
  // first, then across its columns), so the tiles that run together on one
  // XCD read few distinct operand panels through its L2
  const int nb = (int)gridDim.x, per = nb / 8;
  const int bid = (int)blockIdx.x;
  const int tile = (nb % 8 == 0) ? (bid % 8) * per + bid / 8 : bid;
  if (tile >= ntiles) return;
  const int tiles_m = ntiles / tiles_n, in_group = BIG_GROUP * tiles_n;
  const int first = tile / in_group * BIG_GROUP, gsz = min(tiles_m - first, BIG_GROUP), r = tile % in_group;
  const int m0 = (first + r % gsz) * BM, n0 = (r / gsz) * BN;
  if (mlim) {
    const int lim = (int)(*mlim - e.row_base);
    if (m0 >= lim) return;
    if (lim < M) M = lim;
  }
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
  const int i = lane & 15, kq = lane >> 4;
  floatx4 acc[8][4];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int nk = K / SK;
  uint16_t* const st0 = dsm;
  uint16_t* const st1 = dsm + DL_STAGE / sizeof(uint16_t);
  dl_fetch<false>(st0, A, lda, M, m0, 0);
  dl_fetch<true>(st0 + BM * SK, B, ldb, N, n0, 0);
  for (int k = 0; k < nk; ++k) {
    __builtin_amdgcn_s_waitcnt(0);  // this wave's requests for tile k have landed
    __syncthreads();                // every wave's have, and every wave is done with tile k - 1
    if (k + 1 < nk) {               // the other buffer (last read for tile k - 1) takes tile k + 1
      uint16_t* nx = (k & 1) ? st0 : st1;
      dl_fetch<false>(nx, A, lda, M, m0, (k + 1) * SK);
      dl_fetch<true>(nx + BM * SK, B, ldb, N, n0, (k + 1) * SK);
    }
    const uint16_t* As = (k & 1) ? st1 : st0;
    const uint16_t* Bs = As + BM * SK;
#pragma unroll
    for (int ks = 0; ks < SK; ks += 32) {
      const int kc = (ks >> 3) + kq;
      bf16x8 bfv[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) bfv[t] = dl_frag<true>(Bs, wn + 4 * i + t, kc);
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const bf16x8 af = dl_frag<false>(As, wm + 16 * a + i, kc);
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bfv[b], acc[a][b], 0, 0, 0);
      }
    }
  }
  tile_store<EPI, 8, 4, true>(e, acc, m0 + wm, n0 + wn, M, N);
}
// 256 x 256 tiles once every CU gets one.  Three products of n rows over
// 768-1024-1024-8192: n = 16,384 524 us against 887 on 64 x 64 tiles, 8,192 328
// against 487 (the first two products on 64 x 64 in both); over 768-1024-1024-1024:
// n = 16,384 (256 tiles each) 239 against 258.  Below, 256 x 128 tiles (double
// buffered through registers) lost to 64 x 64 at every size: 10,000 rows 262 against
// 171 us, 8,192 x 8,192 412 against 333, 256 x 8,192 33 against 15.
constexpr int64_t BIG_MIN_TILES = 256;

template <bool AT, bool BT, int EPI>
void gemm(const uint16_t* A, int lda, const uint16_t* B, int ldb, int M, int N, int K, const Epi& e, hipStream_t s,
          const int32_t* mlim = nullptr) {
  if (M <= 0 || N <= 0) return;
  // rows of whole 16-byte words (the widths of a router and of split-BF16 routing are multiples of 8)
  if ((lda % 8) != 0 || (ldb % 8) != 0 || lda >= (1 << 23) || ldb >= (1 << 23) || ((uintptr_t)A % 16) != 0 ||
      ((uintptr_t)B % 16) != 0 || ((AT ? M : K) % 8) != 0 || ((BT ? N : K) % 8) != 0)
    throw ArgError{HNTL_EUNSUPPORTED, "BF16 products need 16-byte aligned rows"};
  auto tiles = [&](int tm, int tn) { return (int64_t)((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
  auto lds = [](const void* kernel, size_t bytes, bool& set) {  // more than 64 KiB of dynamic LDS
    if (set) return;
    HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    set = true;
  };
  // grids are multiples of 8 for the XCD-contiguous order
  if constexpr (!AT && !BT) {
    if ((K % SK) == 0 && tiles(BM, BN) >= BIG_MIN_TILES) {
      static bool set = false;
      lds((const void*)gemm_big_kernel<EPI>, BIG_LDS, set);
      const int nt = (int)tiles(BM, BN);
      hipLaunchKernelGGL((gemm_big_kernel<EPI>), dim3((unsigned)((nt + 7) / 8 * 8)), dim3(512), BIG_LDS, s, A, lda, B,
                         ldb, M, N, K, e, mlim, (N + BN - 1) / BN, nt);
      HIP_TRY(hipGetLastError());
      return;
    }
  }
  const int nt = (int)tiles(SM, SM);
  hipLaunchKernelGGL((gemm_small_kernel<AT, BT, EPI>), dim3((unsigned)((nt + 7) / 8 * 8)), dim3(256), 0, s, A, lda, B,
                     ldb, M, N, K, e, mlim, (N + SM - 1) / SM, nt);
  HIP_TRY(hipGetLastError());
}

// ------------------------------------------------------ elementwise kernels
__global__ void to_bf16_kernel(const float* __restrict__ x, int64_t n, uint16_t* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = to_bf16(x[i]);
}

// xh[r][j] = bf16((X[rows[r]][j] - mean[j]) / std[j]) (rows == null: r itself)
__global__ void standardize_kernel(const float* __restrict__ X, const int32_t* __restrict__ rows, int64_t n, int d,
                                   const float* __restrict__ mean, const float* __restrict__ stdv,
                                   uint16_t* __restrict__ xh, const int32_t* __restrict__ nlim) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * d) return;
  const int64_t r = i / d;
  const int j = (int)(i % d);
  if (nlim && r >= *nlim) return;
  const int64_t src = rows ? rows[r] : r;
  xh[i] = to_bf16((X[src * d + j] - mean[j]) / stdv[j]);
}

// Column mean and standard deviation (FP64 accumulation) of n x d rows, in two
// passes over the rows: the rows are cut into STAT_SPLITS runs, a workgroup
// sums 64 columns of one run (every wave its own rows, so a load is one
// 256-byte segment), and col_combine_kernel adds the runs in order.  Bound by
// the two reads of X.  A thread per column walking every row (three workgroups
// at d = 768, one load in flight each) took 8.2 ms for 16,384 x 768; the four
// launches of this take 0.03 ms.
constexpr int STAT_SPLITS = 64;
__global__ __launch_bounds__(256) void col_moment_kernel(const float* __restrict__ X, int64_t n, int d,
                                                         const double* __restrict__ mu, double* __restrict__ part) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = (int)blockIdx.x * 64 + lane;
  const int64_t per = (n + STAT_SPLITS - 1) / STAT_SPLITS;
  const int64_t r0 = (int64_t)blockIdx.y * per, r1 = r0 + per < n ? r0 + per : n;
  double s = 0.0;
  if (j < d) {
    if (mu) {
      const double m = mu[j];
#pragma unroll 8
      for (int64_t r = r0 + wave; r < r1; r += 4) {
        const double t = X[r * d + j] - m;
        s += t * t;
      }
    } else {
#pragma unroll 8
      for (int64_t r = r0 + wave; r < r1; r += 4) s += X[r * d + j];
    }
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && j < d) part[(size_t)blockIdx.y * d + j] = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
}

// mu (the mean) from the sums of the first pass, or stdv from those of the second.
__global__ void col_combine_kernel(const double* __restrict__ part, int64_t n, int d, double* __restrict__ mu,
                                   float* __restrict__ mean, float* __restrict__ stdv) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d) return;
  double s = 0.0;
  for (int k = 0; k < STAT_SPLITS; ++k) s += part[(size_t)k * d + j];
  if (mean) {
    mu[j] = s / (double)n;
    mean[j] = (float)mu[j];
  } else {
    const double sd = sqrt(s / (double)n);
    stdv[j] = (float)(sd > 1e-12 ? sd : 1.0);
  }
}

// Softmax cross-entropy of one row of scores against the target distribution
// of `kt` grain ids (each weighing 1 / kt; row rows[r] of tgt, or r itself):
// ds = (p - y) / B in FP32 and BF16, and the row's loss.  One workgroup of 256 per row.
__global__ __launch_bounds__(256) void softmax_ce_kernel(const float* __restrict__ S, int G,
                                                         const int32_t* __restrict__ tgt,
                                                         const int32_t* __restrict__ rows, int kt, float invB,
                                                         float* __restrict__ ds, uint16_t* __restrict__ dsb,
                                                         float* __restrict__ loss) {
  __shared__ float red[256];
  const int64_t r = blockIdx.x;
  const float* s = S + r * G;
  float m = -__builtin_inff();
  for (int g = threadIdx.x; g < G; g += 256) m = fmaxf(m, s[g]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  m = red[0];
  __syncthreads();
  float z = 0.f;
  for (int g = threadIdx.x; g < G; g += 256) z += expf(s[g] - m);
  red[threadIdx.x] = z;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  z = red[0];
  const float logz = logf(z);
  const int32_t* t = tgt + (rows ? (int64_t)rows[r] : r) * kt;
  const float w = 1.f / (float)kt;
  for (int g = threadIdx.x; g < G; g += 256) {
    float y = 0.f;
    for (int q = 0; q < kt; ++q) y += t[q] == g ? w : 0.f;
    const float p = expf(s[g] - m) / z;
    const float v = (p - y) * invB;
    ds[r * G + g] = v;
    dsb[r * G + g] = to_bf16(v);
  }
  if (threadIdx.x == 0) {
    float l = 0.f;
    for (int q = 0; q < kt; ++q) {
      const int g = t[q];
      if (g >= 0 && g < G) l -= w * (s[g] - m - logz);
    }
    atomicAdd(loss, l * invB);
  }
}

// out[n] = sum over rows of X[r][n] (bias gradients), added in row order: one
// thread per column keeps the chain of additions, the workgroup's other
// threads bring the rows.  A workgroup owns CS_COLS columns; chunks of CS_ROWS
// rows go through registers into the LDS, the next chunk's loads in flight
// while this one is summed.  Bound by the chain (4 cycles an addition, 2 us
// for 1,024 rows) and one memory round trip per chunk.  16 columns and not 64
// so that the 512 to 8,192 columns of a layer give a workgroup to most CUs.
// A thread per column that also loaded its own rows took 235 us a call in
// the training of a 768-512-512-1,024 router with batches of 1,024 (one load
// in flight per thread); this takes 15 us.
constexpr int CS_COLS = 16, CS_ROWS = 256, CS_PER = CS_ROWS * CS_COLS / 256;
__global__ __launch_bounds__(256) void col_sum_kernel(const float* __restrict__ X, int rows, int N,
                                                      float* __restrict__ out) {
  __shared__ float tile[CS_ROWS][CS_COLS + 1];
  const int c = threadIdx.x % CS_COLS, r0 = threadIdx.x / CS_COLS;
  const int n = blockIdx.x * CS_COLS + c;
  float v[CS_PER];
  auto load = [&](int base) {
#pragma unroll
    for (int u = 0; u < CS_PER; ++u) {
      const int r = base + r0 + u * (256 / CS_COLS);
      v[u] = (r < rows && n < N) ? X[(size_t)r * N + n] : 0.f;
    }
  };
  float acc = 0.f;
  load(0);
  for (int base = 0; base < rows; base += CS_ROWS) {
#pragma unroll
    for (int u = 0; u < CS_PER; ++u) tile[r0 + u * (256 / CS_COLS)][c] = v[u];
    __syncthreads();
    if (base + CS_ROWS < rows) load(base + CS_ROWS);
    if (threadIdx.x < CS_COLS) {
      const int m = min(CS_ROWS, rows - base);
      if (m == CS_ROWS) {
#pragma unroll 16
        for (int r = 0; r < CS_ROWS; ++r) acc += tile[r][c];
      } else {
        for (int r = 0; r < m; ++r) acc += tile[r][c];
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < CS_COLS && n < N) out[n] = acc;
}

// One Adam step of a tensor, and its BF16 copy when given.
__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1,
                            float c2, uint16_t* __restrict__ wb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  w[i] = wi;
  if (wb) wb[i] = to_bf16(wi);
}

// Max softmax probability of each row of negated scores (1 / z, z from the
// top-P pass that read the row); rows below tau are appended to the fallback
// list.  One thread per row.
__global__ __launch_bounds__(256) void fallback_select_kernel(const float2* __restrict__ znorm, int64_t rows,
                                                              float tau, int32_t* __restrict__ fb_rows,
                                                              int32_t* __restrict__ fb_count,
                                                              const int32_t* __restrict__ nlim) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows || (nlim && r >= *nlim)) return;
  if (1.f / znorm[r].y < tau) fb_rows[atomicAdd(fb_count, 1)] = (int32_t)r;
}

// Probability-mass probe budget of one learned row (one wave): with
// m = max score and z = sum_g exp(s_g - m) over all G scores, slots are kept
// up to and including the first j at which sum_{i <= j} exp(s_{p_i} - m) / z
// reaches mass; later slots become probe -1 (pdist +inf).
__global__ __launch_bounds__(256) void mass_cut_kernel(const float* __restrict__ negS, const float2* __restrict__ znorm,
                                                       int64_t rows, int G, int P, float mass,
                                                       int32_t* __restrict__ probes, float* __restrict__ pdist,
                                                       const int32_t* __restrict__ nlim) {
  const int lane = lane_id();
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows || (nlim && r >= *nlim)) return;
  const float* s = negS + r * G;  // negated scores
  // m and z of the row, from the top-P pass that read the row
  const float2 mz = znorm[r];
  const float mn = mz.x, z = mz.y;
  // lane j < P: probability of slot j; an inclusive prefix sum over the lanes
  const int32_t pj = lane < P ? probes[r * P + lane] : -1;
  float p = pj >= 0 ? expf(mn - s[pj]) / z : 0.f;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float t = __shfl_up(p, o, 64);
    if (lane >= o) p += t;
  }
  const uint64_t reached = __ballot(lane < P && p >= mass);
  if (!reached) return;
  const int cut = __builtin_ctzll(reached);  // the first slot that reaches the mass: kept
  if (lane > cut && lane < P) {
    probes[r * P + lane] = -1;
    if (pdist) pdist[r * P + lane] = __builtin_inff();
  }
}

// Copies the query rows of the fallback list into a compact block.
__global__ void gather_rows_kernel(const float* __restrict__ Q, int d, const int32_t* __restrict__ rows,
                                   const int32_t* __restrict__ count, float* __restrict__ out) {
  const int r = blockIdx.x;
  if (r >= *count) return;
  const float* src = Q + (size_t)rows[r] * d;
  for (int j = threadIdx.x; j < d; j += blockDim.x) out[(size_t)r * d + j] = src[j];
}

// Writes the centroid-routing probes of the fallback rows back in place.
__global__ void scatter_probes_kernel(const int32_t* __restrict__ rows, const int32_t* __restrict__ count, int P,
                                      const int32_t* __restrict__ src, const float* __restrict__ srcd,
                                      int32_t* __restrict__ probes, float* __restrict__ pdist) {
  const int r = blockIdx.x;
  if (r >= *count) return;
  const int q = rows[r];
  for (int j = threadIdx.x; j < P; j += blockDim.x) {
    probes[(size_t)q * P + j] = src[(size_t)r * P + j];
    if (pdist) pdist[(size_t)q * P + j] = srcd ? srcd[(size_t)r * P + j] : 0.f;
  }
}

// Grain of every original row: lab[perm[pos]] = grain holding position pos.
__global__ void row_grain_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ goff, int G, int64_t N,
                                 int32_t* __restrict__ lab) {
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= N) return;
  int lo = 0, hi = G;  // largest g with goff[g] <= pos
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (goff[mid] <= pos)
      lo = mid;
    else
      hi = mid;
  }
  lab[perm[pos]] = lo;
}

__global__ void map_ids_kernel(const int32_t* __restrict__ ids, int64_t n, const int32_t* __restrict__ lab,
                               int32_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = ids[i] >= 0 ? lab[ids[i]] : -1;
}

inline unsigned blocks(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

__host__ __device__ inline uint64_t splitmix(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
__host__ __device__ inline double uni(uint64_t seed, uint64_t stream, uint64_t i) {
  return (double)(splitmix(splitmix(seed ^ (stream * 0xD1B54A32D192ED03ull)) + i) >> 11) * (1.0 / 9007199254740992.0);
}

// Uniform weights in [-bound, bound) from the counter-based generator.  1.2 million of
// them on the host and their copy kept a training run waiting 1.7 ms.
__global__ void init_weights_kernel(float* __restrict__ w, int64_t n, uint64_t seed, uint64_t stream, double bound) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = (float)((2.0 * uni(seed, stream, (uint64_t)i) - 1.0) * bound);
}

}  // namespace

// ------------------------------------------------------------------ router
void Router::alloc(int d_, int h1_, int h2_, int G_) {
  d = d_;
  h1 = h1_;
  h2 = h2_;
  G = G_;
  const int64_t n[3] = {(int64_t)h1 * d, (int64_t)h2 * h1, (int64_t)G * h2};
  const int64_t nb[3] = {h1, h2, G};
  for (int l = 0; l < 3; ++l) {
    HIP_TRY(hipMalloc((void**)&W[l], sizeof(float) * n[l]));
    HIP_TRY(hipMalloc((void**)&b[l], sizeof(float) * nb[l]));
    HIP_TRY(hipMalloc((void**)&Wb[l], sizeof(uint16_t) * n[l]));
  }
  HIP_TRY(hipMalloc((void**)&mean, sizeof(float) * d));
  HIP_TRY(hipMalloc((void**)&stdv, sizeof(float) * d));
}

Router::~Router() {
  for (int l = 0; l < 3; ++l) {
    if (W[l]) (void)hipFree(W[l]);
    if (b[l]) (void)hipFree(b[l]);
    if (Wb[l]) (void)hipFree(Wb[l]);
  }
  if (mean) (void)hipFree(mean);
  if (stdv) (void)hipFree(stdv);
}

int64_t Router::wsize(int l) const { return l == 0 ? (int64_t)h1 * d : l == 1 ? (int64_t)h2 * h1 : (int64_t)G * h2; }
int64_t Router::bsize(int l) const { return l == 0 ? h1 : l == 1 ? h2 : G; }

void Router::refresh_bf16(hipStream_t s) {
  for (int l = 0; l < 3; ++l)
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks(wsize(l))), dim3(256), 0, s, W[l], wsize(l), Wb[l]);
  HIP_TRY(hipGetLastError());
}

// Learned routing of nq rows of Q: probes (nq x P) by descending score (ties:
// lower grain), pdist = the negated scores; rows whose largest softmax
// probability is below tau use centroid routing instead.
namespace {
// FP32 rows split into BF16 high and low parts (nearest even): an output row is
// [hi | hi | lo] (queries) or [hi | lo | hi] (centroids, corder), so that one
// product over 3d depths gives q_hi c_hi + q_hi c_lo + q_lo c_hi.
__global__ void split3_kernel(const float* __restrict__ X, int64_t rows, int d, int corder,
                              uint16_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * d) return;
  const int64_t r = i / d;
  const int k = (int)(i - r * d);
  const float x = X[i];
  const uint16_t h = to_bf16(x);
  const uint16_t l = to_bf16(x - __uint_as_float((uint32_t)h << 16));
  uint16_t* o = out + r * 3 * d;
  o[k] = h;
  o[d + k] = corder ? l : h;
  o[2 * d + k] = corder ? h : l;
}

// One wave per query row (d % 4 == 0), up to 1024 values of it in flight.  Bound by
// memory: the row is read once and its copy and operands written.  16,384 x 768
// with BF16 operands 26 us; copy, norms, conversion, batch size and counters in
// a launch each took 62.
__global__ __launch_bounds__(256) void plan_begin_kernel(PlanBegin b, bool vec4) {
  const int lane = lane_id();
  const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (tid == 0) {
    *b.nq_dev = (int32_t)b.nq;
    *b.out_dev = b.results;
  }
  for (int k = 0; k < b.fill.n; ++k)
    for (int64_t i = tid; i < b.fill.seg[k].n; i += (int64_t)gridDim.x * 256) b.fill.seg[k].p[i] = b.fill.seg[k].v;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= b.nq) return;
  const int d = b.d, w = b.prep == PREP_BF16X3 ? 3 : 1;
  const float* src = b.src + row * d;
  float* dst = b.Q + row * d;
  uint16_t* o = b.out + (size_t)row * w * d;
  float acc = 0.f;
  constexpr int U = 4;
  for (int j0 = 4 * lane; j0 < d; j0 += U * 256) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 256 * u;
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (j < d)
        v[u] = vec4 ? *reinterpret_cast<const float4*>(src + j)
                    : make_float4(src[j], src[j + 1], src[j + 2], src[j + 3]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 256 * u;
      if (j >= d) continue;
      if (src != dst) *reinterpret_cast<float4*>(dst + j) = v[u];
      float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = fmaf(x[c], x[c], acc);
      if (b.prep == PREP_NORMS) continue;
      ushort4 h, l;
      if (b.prep == PREP_STANDARDIZE) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = (x[c] - b.mean[j + c]) / b.stdv[j + c];
      }
      h = make_ushort4(to_bf16(x[0]), to_bf16(x[1]), to_bf16(x[2]), to_bf16(x[3]));
      *reinterpret_cast<ushort4*>(o + j) = h;
      if (b.prep != PREP_BF16X3) continue;
      auto low = [](float y, uint16_t hi) { return to_bf16(y - __uint_as_float((uint32_t)hi << 16)); };
      l = make_ushort4(low(x[0], h.x), low(x[1], h.y), low(x[2], h.z), low(x[3], h.w));
      *reinterpret_cast<ushort4*>(o + d + j) = h;
      *reinterpret_cast<ushort4*>(o + 2 * d + j) = l;
    }
  }
  if (b.prep != PREP_STANDARDIZE) {
    acc = wave_sum(acc);
    if (lane == 0) b.qn[row] = acc;
  }
}
std::mutex g_split_mu;
}  // namespace

void launch_plan_begin(const PlanBegin& b, hipStream_t s) {
  if (b.d % 4 != 0) throw ArgError{HNTL_EUNSUPPORTED, "plans need d % 4 == 0"};
  int64_t fill = 0;
  for (int k = 0; k < b.fill.n; ++k) fill = std::max<int64_t>(fill, b.fill.seg[k].n);
  // a workgroup per four rows, or for each 1,024 counters of a small batch
  const int64_t grid = std::max<int64_t>(std::max<int64_t>((b.nq + 3) / 4, (fill + 1023) / 1024), 1);
  hipLaunchKernelGGL(plan_begin_kernel, dim3((unsigned)grid), dim3(256), 0, s, b, (uintptr_t)b.src % 16 == 0);
  HIP_TRY(hipGetLastError());
}

void ensure_centroid_split(Index& ix, hipStream_t s) {
  std::lock_guard<std::mutex> lk(g_split_mu);
  if (ix.cent_split) return;
  if (ix.d % 8 != 0) throw ArgError{HNTL_EUNSUPPORTED, "split-BF16 routing needs d % 8 == 0"};
  uint16_t* p = dev_alloc<uint16_t>(&ix, (size_t)ix.G * 3 * ix.d);
  const int64_t n = (int64_t)ix.G * ix.d;
  hipLaunchKernelGGL(split3_kernel, dim3(blocks(n)), dim3(256), 0, s, ix.centroids, (int64_t)ix.G, (int)ix.d, 1, p);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(s));
  ix.cent_split = p;
}

void launch_dist_bf16x3(const Index& ix, const float* A, const float* an, int64_t rows, uint16_t* As, float* D,
                        hipStream_t s, const int32_t* nlim, int64_t row_base) {
  if (rows <= 0) return;
  if (!ix.cent_split) throw ArgError{HNTL_ESTATE, "split-BF16 routing: centroid split not built"};
  if (A) {
    const int64_t n = rows * ix.d;
    hipLaunchKernelGGL(split3_kernel, dim3(blocks(n)), dim3(256), 0, s, A, rows, (int)ix.d, 0, As);
    HIP_TRY(hipGetLastError());
  }
  Epi e{};
  e.C = D;
  e.ldc = (int)ix.G;
  e.an = an;
  e.bn = ix.cnorm;
  e.row_base = row_base;
  const int K3 = 3 * (int)ix.d;
  gemm<false, false, EPI_DIST>(As, K3, ix.cent_split, K3, (int)rows, (int)ix.G, K3, e, s, nlim);
}

// Plain BF16 expansion distances: <a, mu> from bf16(a) . bf16(mu) (the high
// parts of the split centroid rows, row stride 3d), FP32 accumulation.
void launch_dist_bf16(const Index& ix, const float* A, const float* an, int64_t rows, uint16_t* As, float* D,
                      hipStream_t s, const int32_t* nlim, int64_t row_base) {
  if (rows <= 0) return;
  if (!ix.cent_split) throw ArgError{HNTL_ESTATE, "BF16 routing: centroid split not built"};
  if (A) {
    const int64_t n = rows * ix.d;
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks(n)), dim3(256), 0, s, A, n, As);
    HIP_TRY(hipGetLastError());
  }
  Epi e{};
  e.C = D;
  e.ldc = (int)ix.G;
  e.an = an;
  e.bn = ix.cnorm;
  e.row_base = row_base;
  const int d = (int)ix.d;
  gemm<false, false, EPI_DIST>(As, d, ix.cent_split, 3 * d, (int)rows, (int)ix.G, d, e, s, nlim);
}

size_t RouteScratch::layout(char* base, const Index& ix, int64_t nq, int form_) {
  form = form_;
  chunk = std::min<int64_t>(std::max<int64_t>(nq, 1), std::max<int64_t>(64, ((int64_t)1 << 28) / ix.G));
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    off = (off + 255) / 256 * 256;
    char* p = base ? base + off : nullptr;
    off += std::max<size_t>(bytes, 1);
    return p;
  };
  qn = (float*)take(4 * (size_t)std::max<int64_t>(nq, 1));
  D = (float*)take(4 * (size_t)chunk * ix.G);
  const int w = form == ROUTE_BF16X3 ? 3 : form == ROUTE_BF16 ? 1 : 0;
  As = w ? (uint16_t*)take(2 * (size_t)chunk * w * ix.d) : nullptr;
  return off;
}

float route_err(int form) {
  // Bound on |expansion - exact| per entry, as a multiple of ||q||^2 + ||mu||^2
  // (|<q, mu>| <= (||q||^2 + ||mu||^2) / 2):
  //  - FP32 MFMA: products and sums in FP32 over d <= 1024 terms, about 1e-5;
  //  - split BF16: the dropped lo x lo term and the parts' own rounding (about
  //    3 x 2^-18) plus FP32 accumulation over 3d terms;
  //  - plain BF16: each operand rounded to nearest even (2^-9 relative each),
  //    2^-8 + 2^-18 of sum |q_j mu_j|, plus the FP32 accumulation.
  // Each factor also covers the FP32 norms and the final combination.
  return form == ROUTE_BF16 ? 4.0e-3f : 5.0e-5f;
}

void launch_route_centroid(const Index& ix, const float* Q, int64_t nq, int P, const RouteScratch& w,
                           int32_t* probes, float* pdist, hipStream_t s, const int32_t* nlim,
                           unsigned int* overflow, int prepared) {
  if (nq <= 0) return;
  if (w.form != ROUTE_F32 && !ix.cent_split) throw ArgError{HNTL_ESTATE, "BF16 routing: centroid split not built"};
  const int G = (int)ix.G, d = (int)ix.d;
  if (prepared < 0) launch_row_norms(Q, nq, d, w.qn, s);
  const bool operands = prepared == PREP_BF16 || prepared == PREP_BF16X3;
  for (int64_t q0 = 0; q0 < nq; q0 += w.chunk) {
    const int64_t rows = std::min<int64_t>(w.chunk, nq - q0);
    const float* Qc = Q + q0 * d;
    if (rows <= 16 || w.form == ROUTE_F32)  // a few rows: exact direct differences (FP32 MFMA expansion otherwise)
      launch_dist_matrix(Qc, w.qn + q0, rows, ix.centroids, ix.cnorm, G, d, w.D, s, nlim, q0);
    else if (w.form == ROUTE_BF16X3)
      launch_dist_bf16x3(ix, operands ? nullptr : Qc, w.qn + q0, rows, w.As, w.D, s, nlim, q0);
    else
      launch_dist_bf16(ix, operands ? nullptr : Qc, w.qn + q0, rows, w.As, w.D, s, nlim, q0);
    launch_topk_rows(w.D, rows, G, P, probes + q0 * P, pdist ? pdist + q0 * P : nullptr, s, Qc, w.qn + q0,
                     ix.centroids, ix.cnorm, ix.cnmax, d, route_err(w.form), nlim, q0, overflow);
  }
}

void launch_route_learned(const Index& ix, const float* Q, int64_t nq, int P, float tau, int32_t* probes,
                          float* pdist, const RouterScratch& w, hipStream_t s, const int32_t* nlim, float mass,
                          bool prepared) {
  const Router& rt = *ix.router;
  if (!prepared) {
    hipLaunchKernelGGL(standardize_kernel, dim3(blocks(nq * rt.d)), dim3(256), 0, s, Q, nullptr, nq, rt.d, rt.mean,
                       rt.stdv, w.xh, nlim);
    HIP_TRY(hipGetLastError());
  }
  Epi e{};
  e.bias = rt.b[0];
  e.H = w.h1;
  e.ldh = rt.h1;
  gemm<false, false, EPI_BIAS_GELU>(w.xh, rt.d, rt.Wb[0], rt.d, (int)nq, rt.h1, rt.d, e, s, nlim);
  e.bias = rt.b[1];
  e.H = w.h2;
  e.ldh = rt.h2;
  gemm<false, false, EPI_BIAS_GELU>(w.h1, rt.h1, rt.Wb[1], rt.h1, (int)nq, rt.h2, rt.h1, e, s, nlim);
  // negS = -(h2 W3^T + b3): the P smallest are the P largest scores
  Epi o{};
  o.C = w.negS;
  o.ldc = rt.G;
  o.bias = rt.b[2];
  o.scale = -1.f;
  gemm<false, false, EPI_BIAS_F32>(w.h2, rt.h2, rt.Wb[2], rt.h2, (int)nq, rt.G, rt.h2, o, s, nlim);
  const bool budget = mass > 0.f && mass < 1.f && P > 1;
  launch_topk_rows(w.negS, nq, rt.G, P, probes, pdist, s, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0.f, nlim, 0,
                   nullptr, (budget || tau > 0.f) ? w.znorm : nullptr);
  if (budget) {
    hipLaunchKernelGGL(mass_cut_kernel, dim3(blocks(nq, 4)), dim3(256), 0, s, w.negS, w.znorm, nq, rt.G, P, mass,
                       probes, pdist, nlim);
    HIP_TRY(hipGetLastError());
  }
  if (tau > 0.f) {
    launch_fill_i32(w.fb_count, 1, 0, s);
    hipLaunchKernelGGL(fallback_select_kernel, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s, w.znorm, nq, tau,
                       w.fb_rows, w.fb_count, nlim);
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)nq), dim3(256), 0, s, Q, (int)ix.d, w.fb_rows, w.fb_count,
                       w.fb_Q);
    launch_row_norms(w.fb_Q, nq, (int)ix.d, w.fb_qn, s);
    const int64_t chunk = std::max<int64_t>(64, ((int64_t)1 << 28) / ix.G);
    for (int64_t q0 = 0; q0 < nq; q0 += chunk) {
      const int64_t rows = std::min<int64_t>(chunk, nq - q0);
      launch_dist_matrix(w.fb_Q + q0 * ix.d, w.fb_qn + q0, rows, ix.centroids, ix.cnorm, (int)ix.G, (int)ix.d,
                         w.negS, s, w.fb_count, q0);  // the scores are no longer needed: reuse as scratch
      launch_topk_rows(w.negS, rows, (int)ix.G, P, w.fb_probes + q0 * P, w.fb_pdist + q0 * P, s,
                       w.fb_Q + q0 * ix.d, w.fb_qn + q0, ix.centroids, ix.cnorm, ix.cnmax, (int)ix.d, route_err(ROUTE_F32),
                       w.fb_count, q0, nullptr);
    }
    hipLaunchKernelGGL(scatter_probes_kernel, dim3((unsigned)nq), dim3(64), 0, s, w.fb_rows, w.fb_count, P,
                       w.fb_probes, w.fb_pdist, probes, pdist);
    HIP_TRY(hipGetLastError());
  }
}

// Buffers of launch_route_learned carved from one block (base == nullptr:
// sizing pass); returns the bytes used.
size_t RouterScratch::layout(char* base, const Index& ix, int64_t nq, int P) {
  const Router& rt = *ix.router;
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    off = (off + 255) / 256 * 256;
    char* p = base ? base + off : nullptr;
    off += std::max<size_t>(bytes, 1);
    return p;
  };
  xh = (uint16_t*)take(2 * (size_t)nq * rt.d);
  h1 = (uint16_t*)take(2 * (size_t)nq * rt.h1);
  h2 = (uint16_t*)take(2 * (size_t)nq * rt.h2);
  const int64_t chunk = std::min<int64_t>(nq, std::max<int64_t>(64, ((int64_t)1 << 28) / ix.G));
  negS = (float*)take(4 * (size_t)std::max<int64_t>(nq * rt.G, chunk * ix.G));
  fb_rows = (int32_t*)take(4 * (size_t)nq);
  fb_count = (int32_t*)take(4);
  fb_Q = (float*)take(4 * (size_t)nq * ix.d);
  fb_qn = (float*)take(4 * (size_t)nq);
  fb_probes = (int32_t*)take(4 * (size_t)nq * P);
  fb_pdist = (float*)take(4 * (size_t)nq * P);
  znorm = (float2*)take(sizeof(float2) * (size_t)nq);
  return off;
}

namespace {

// Training state: Adam moments, gradients, activations of one batch.
struct Trainer {
  Router& rt;
  int B;
  hipStream_t s;
  std::vector<void*> mem;
  float* m[6] = {};
  float* v[6] = {};
  float* g[6] = {};
  uint16_t *xh = nullptr, *h1 = nullptr, *h2 = nullptr, *dsb = nullptr, *da2b = nullptr, *da1b = nullptr;
  float *a1 = nullptr, *a2 = nullptr, *S = nullptr, *ds = nullptr, *da2 = nullptr, *da1 = nullptr, *loss = nullptr;
  int32_t* rows = nullptr;
  int step = 0;

  template <class T>
  T* alloc(size_t n) {
    void* p = nullptr;
    HIP_TRY(hipMalloc(&p, sizeof(T) * std::max<size_t>(n, 1)));
    mem.push_back(p);
    return (T*)p;
  }
  Trainer(Router& r, int B_, hipStream_t st) : rt(r), B(B_), s(st) {
    for (int l = 0; l < 3; ++l) {
      m[2 * l] = alloc<float>(rt.wsize(l));
      v[2 * l] = alloc<float>(rt.wsize(l));
      g[2 * l] = alloc<float>(rt.wsize(l));
      m[2 * l + 1] = alloc<float>(rt.bsize(l));
      v[2 * l + 1] = alloc<float>(rt.bsize(l));
      g[2 * l + 1] = alloc<float>(rt.bsize(l));
      HIP_TRY(hipMemsetAsync(m[2 * l], 0, sizeof(float) * rt.wsize(l), s));
      HIP_TRY(hipMemsetAsync(v[2 * l], 0, sizeof(float) * rt.wsize(l), s));
      HIP_TRY(hipMemsetAsync(m[2 * l + 1], 0, sizeof(float) * rt.bsize(l), s));
      HIP_TRY(hipMemsetAsync(v[2 * l + 1], 0, sizeof(float) * rt.bsize(l), s));
    }
    xh = alloc<uint16_t>((size_t)B * rt.d);
    h1 = alloc<uint16_t>((size_t)B * rt.h1);
    h2 = alloc<uint16_t>((size_t)B * rt.h2);
    a1 = alloc<float>((size_t)B * rt.h1);
    a2 = alloc<float>((size_t)B * rt.h2);
    S = alloc<float>((size_t)B * rt.G);
    ds = alloc<float>((size_t)B * rt.G);
    dsb = alloc<uint16_t>((size_t)B * rt.G);
    da2 = alloc<float>((size_t)B * rt.h2);
    da2b = alloc<uint16_t>((size_t)B * rt.h2);
    da1 = alloc<float>((size_t)B * rt.h1);
    da1b = alloc<uint16_t>((size_t)B * rt.h1);
    loss = alloc<float>(1);
    rows = alloc<int32_t>(B);
  }
  ~Trainer() {
    for (void* p : mem) (void)hipFree(p);
  }

  void col_sum(const float* X, int rows, int N, float* out) {
    hipLaunchKernelGGL(col_sum_kernel, dim3(blocks(N, CS_COLS)), dim3(256), 0, s, X, rows, N, out);
  }

  // Loss and gradients of the batch X[rows[0..B)] against targets tg (B x kt).
  // trows: the targets' rows (null: tg holds the batch's own); the loss is added to *lossp
  void grad(const float* X, const int32_t* d_rows, const int32_t* tg, const int32_t* trows, int kt, float* lossp) {
    const int d = rt.d, H1 = rt.h1, H2 = rt.h2, G = rt.G;
    hipLaunchKernelGGL(standardize_kernel, dim3(blocks((int64_t)B * d)), dim3(256), 0, s, X, d_rows, (int64_t)B, d,
                       rt.mean, rt.stdv, xh, nullptr);
    Epi e{};
    e.C = a1;
    e.ldc = H1;
    e.bias = rt.b[0];
    e.H = h1;
    e.ldh = H1;
    gemm<false, false, EPI_BIAS_GELU>(xh, d, rt.Wb[0], d, B, H1, d, e, s);
    e.C = a2;
    e.ldc = H2;
    e.bias = rt.b[1];
    e.H = h2;
    e.ldh = H2;
    gemm<false, false, EPI_BIAS_GELU>(h1, H1, rt.Wb[1], H1, B, H2, H1, e, s);
    Epi o{};
    o.C = S;
    o.ldc = G;
    o.bias = rt.b[2];
    o.scale = 1.f;
    gemm<false, false, EPI_BIAS_F32>(h2, H2, rt.Wb[2], H2, B, G, H2, o, s);
    hipLaunchKernelGGL(softmax_ce_kernel, dim3(B), dim3(256), 0, s, S, G, tg, trows, kt, 1.f / (float)B, ds, dsb, lossp);
    HIP_TRY(hipGetLastError());
    // layer 3: gW3[g][k] = sum_b ds[b][g] h2[b][k]; dh2 = ds W3, times gelu'(a2)
    Epi w{};
    w.C = g[4];
    w.ldc = H2;
    gemm<true, true, EPI_F32>(dsb, G, h2, H2, G, H2, B, w, s);
    col_sum(ds, B, G, g[5]);
    Epi gg{};
    gg.Z = a2;
    gg.ldz = H2;
    gg.D = da2;
    gg.ldd = H2;
    gg.H = da2b;
    gg.ldh = H2;
    gemm<false, true, EPI_GELU_GRAD>(dsb, G, rt.Wb[2], H2, B, H2, G, gg, s);
    // layer 2
    w.C = g[2];
    w.ldc = H1;
    gemm<true, true, EPI_F32>(da2b, H2, h1, H1, H2, H1, B, w, s);
    col_sum(da2, B, H2, g[3]);
    gg.Z = a1;
    gg.ldz = H1;
    gg.D = da1;
    gg.ldd = H1;
    gg.H = da1b;
    gg.ldh = H1;
    gemm<false, true, EPI_GELU_GRAD>(da2b, H2, rt.Wb[1], H1, B, H1, H2, gg, s);
    // layer 1
    w.C = g[0];
    w.ldc = d;
    gemm<true, true, EPI_F32>(da1b, H1, xh, d, H1, d, B, w, s);
    col_sum(da1, B, H1, g[1]);
    HIP_TRY(hipGetLastError());
  }

  void adam(float lr) {
    ++step;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    for (int l = 0; l < 3; ++l) {
      hipLaunchKernelGGL(adam_kernel, dim3(blocks(rt.wsize(l))), dim3(256), 0, s, rt.W[l], g[2 * l], m[2 * l],
                         v[2 * l], rt.wsize(l), lr, b1, b2, eps, c1, c2, rt.Wb[l]);
      hipLaunchKernelGGL(adam_kernel, dim3(blocks(rt.bsize(l))), dim3(256), 0, s, rt.b[l], g[2 * l + 1],
                         m[2 * l + 1], v[2 * l + 1], rt.bsize(l), lr, b1, b2, eps, c1, c2, (uint16_t*)nullptr);
    }
    HIP_TRY(hipGetLastError());
  }
};

template <class F>
hntl_status guarded_r(F&& f) {
  try {
    f();
    return HNTL_OK;
  } catch (const ArgError& e) {
    return fail(e.code, e.msg);
  } catch (const HipError& e) {
    return fail(e.code == hipErrorOutOfMemory || e.code == hipErrorMemoryAllocation ? HNTL_ENOMEM : HNTL_EDEVICE,
                e.msg);
  } catch (const std::bad_alloc&) {
    return fail(HNTL_ENOMEM, "host allocation failed");
  }
}

void init_router(Index& ix, int h1, int h2) {
  if (h1 < 1 || h2 < 1) throw ArgError{HNTL_EINVAL, "hidden sizes must be positive"};
  if (ix.d % 8 || h1 % 8 || h2 % 8 || ix.G % 8)
    throw ArgError{HNTL_EUNSUPPORTED, "the router needs d, hidden sizes and G to be multiples of 8"};
  ix.router.reset(new Router());
  ix.router->alloc((int)ix.d, h1, h2, (int)ix.G);
}

}  // namespace

}  // namespace hntl

using namespace hntl;

extern "C" {

hntl_status hntl_router_set(hntl_index* index, uint32_t h1, uint32_t h2, const float* W1, const float* b1,
                            const float* W2, const float* b2, const float* W3, const float* b3, const float* mean,
                            const float* stdv) {
  set_error("");
  if (!index || !W1 || !b1 || !W2 || !b2 || !W3 || !b3 || !mean || !stdv) return fail(HNTL_EINVAL, "null pointer");
  return guarded_r([&] {
    Index& ix = index->ix;
    HIP_TRY(hipSetDevice(ix.device));
    init_router(ix, (int)h1, (int)h2);
    Router& rt = *ix.router;
    const float* Ws[3] = {W1, W2, W3};
    const float* bs[3] = {b1, b2, b3};
    for (int l = 0; l < 3; ++l) {
      HIP_TRY(hipMemcpy(rt.W[l], Ws[l], sizeof(float) * rt.wsize(l), hipMemcpyDefault));
      HIP_TRY(hipMemcpy(rt.b[l], bs[l], sizeof(float) * rt.bsize(l), hipMemcpyDefault));
    }
    HIP_TRY(hipMemcpy(rt.mean, mean, sizeof(float) * ix.d, hipMemcpyDefault));
    HIP_TRY(hipMemcpy(rt.stdv, stdv, sizeof(float) * ix.d, hipMemcpyDefault));
    rt.refresh_bf16(nullptr);
    HIP_TRY(hipDeviceSynchronize());
    rt.trained = true;
  });
}

hntl_status hntl_router_export(const hntl_index* index, uint32_t* h1, uint32_t* h2, float* W1, float* b1, float* W2,
                               float* b2, float* W3, float* b3, float* mean, float* stdv) {
  set_error("");
  if (!index) return fail(HNTL_EINVAL, "null index");
  const Index& ix = index->ix;
  if (!ix.router) return fail(HNTL_ESTATE, "the index has no router");
  return guarded_r([&] {
    HIP_TRY(hipSetDevice(ix.device));
    const Router& rt = *ix.router;
    if (h1) *h1 = (uint32_t)rt.h1;
    if (h2) *h2 = (uint32_t)rt.h2;
    float* Ws[3] = {W1, W2, W3};
    float* bs[3] = {b1, b2, b3};
    HIP_TRY(hipDeviceSynchronize());
    for (int l = 0; l < 3; ++l) {
      if (Ws[l]) HIP_TRY(hipMemcpy(Ws[l], rt.W[l], sizeof(float) * rt.wsize(l), hipMemcpyDefault));
      if (bs[l]) HIP_TRY(hipMemcpy(bs[l], rt.b[l], sizeof(float) * rt.bsize(l), hipMemcpyDefault));
    }
    if (mean) HIP_TRY(hipMemcpy(mean, rt.mean, sizeof(float) * ix.d, hipMemcpyDefault));
    if (stdv) HIP_TRY(hipMemcpy(stdv, rt.stdv, sizeof(float) * ix.d, hipMemcpyDefault));
  });
}

hntl_status hntl_router_grad(hntl_index* index, const float* X, uint32_t n, const int32_t* targets, uint32_t kt,
                             float* loss, float* gW1, float* gb1, float* gW2, float* gb2, float* gW3, float* gb3,
                             void* stream) {
  set_error("");
  if (!index || !X || !targets) return fail(HNTL_EINVAL, "null pointer");
  Index& ix = index->ix;
  if (!ix.router) return fail(HNTL_ESTATE, "the index has no router");
  if (n == 0 || kt == 0) return fail(HNTL_EINVAL, "n and kt must be positive");
  return guarded_r([&] {
    HIP_TRY(hipSetDevice(ix.device));
    hipStream_t s = (hipStream_t)stream;
    Router& rt = *ix.router;
    Trainer tr(rt, (int)n, s);
    std::vector<int32_t> idx(n);
    std::iota(idx.begin(), idx.end(), 0);
    HIP_TRY(hipMemcpyAsync(tr.rows, idx.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
    HIP_TRY(hipMemsetAsync(tr.loss, 0, sizeof(float), s));
    tr.grad(X, tr.rows, targets, nullptr, (int)kt, tr.loss);
    float* outs[6] = {gW1, gb1, gW2, gb2, gW3, gb3};
    for (int l = 0; l < 3; ++l) {
      if (outs[2 * l]) HIP_TRY(hipMemcpyAsync(outs[2 * l], tr.g[2 * l], sizeof(float) * rt.wsize(l), hipMemcpyDefault, s));
      if (outs[2 * l + 1])
        HIP_TRY(hipMemcpyAsync(outs[2 * l + 1], tr.g[2 * l + 1], sizeof(float) * rt.bsize(l), hipMemcpyDefault, s));
    }
    if (loss) HIP_TRY(hipMemcpyAsync(loss, tr.loss, sizeof(float), hipMemcpyDefault, s));
    HIP_TRY(hipStreamSynchronize(s));
  });
}

hntl_status hntl_router_forward(const hntl_index* index, const float* Q, uint32_t nq, float* scores, void* stream) {
  set_error("");
  if (!index || !Q || !scores) return fail(HNTL_EINVAL, "null pointer");
  const Index& ix = index->ix;
  if (!ix.router) return fail(HNTL_ESTATE, "the index has no router");
  if (nq == 0) return HNTL_OK;
  return guarded_r([&] {
    HIP_TRY(hipSetDevice(ix.device));
    hipStream_t s = (hipStream_t)stream;
    const Router& rt = *ix.router;
    Scratch sc(s);
    uint16_t* xh = sc.get<uint16_t>((size_t)nq * rt.d);
    uint16_t* h1 = sc.get<uint16_t>((size_t)nq * rt.h1);
    uint16_t* h2 = sc.get<uint16_t>((size_t)nq * rt.h2);
    hipLaunchKernelGGL(standardize_kernel, dim3(blocks((int64_t)nq * rt.d)), dim3(256), 0, s, Q, nullptr,
                       (int64_t)nq, rt.d, rt.mean, rt.stdv, xh, nullptr);
    Epi e{};
    e.bias = rt.b[0];
    e.H = h1;
    e.ldh = rt.h1;
    gemm<false, false, EPI_BIAS_GELU>(xh, rt.d, rt.Wb[0], rt.d, (int)nq, rt.h1, rt.d, e, s);
    e.bias = rt.b[1];
    e.H = h2;
    e.ldh = rt.h2;
    gemm<false, false, EPI_BIAS_GELU>(h1, rt.h1, rt.Wb[1], rt.h1, (int)nq, rt.h2, rt.h1, e, s);
    Epi o{};
    o.C = scores;
    o.ldc = rt.G;
    o.bias = rt.b[2];
    o.scale = 1.f;
    gemm<false, false, EPI_BIAS_F32>(h2, rt.h2, rt.Wb[2], rt.h2, (int)nq, rt.G, rt.h2, o, s);
  });
}

hntl_status hntl_knn(const hntl_index* index, const float* Q, uint32_t nq, uint32_t k, int32_t* ids, float* dist,
                     void* stream) {
  set_error("");
  if (!index || !Q || !ids) return fail(HNTL_EINVAL, "null pointer");
  if (nq == 0) return HNTL_OK;
  const Index& ix = index->ix;
  if (!ix.X) return fail(HNTL_ESTATE, "this index holds no raw vectors");
  return guarded_r([&] {
    HIP_TRY(hipSetDevice(ix.device));
    launch_knn(Q, nq, ix.X, (int64_t)ix.N, (int)ix.d, (int)k, ids, dist, (hipStream_t)stream);
  });
}

hntl_status hntl_router_train(hntl_index* index, const float* Qtrain, uint32_t n, const int32_t* targets,
                              const hntl_router_params* rp, float* epoch_loss, void* stream) {
  set_error("");
  if (!index || !Qtrain || !rp) return fail(HNTL_EINVAL, "null pointer");
  Index& ix = index->ix;
  const uint32_t B = rp->batch ? rp->batch : 1024;
  const uint32_t kt = rp->knn ? rp->knn : 10;
  if (n < B) return fail(HNTL_EINVAL, "need at least one full batch of training queries");
  if (kt > 16) return fail(HNTL_EUNSUPPORTED, "targets from at most 16 neighbours");
  return guarded_r([&] {
    HIP_TRY(hipSetDevice(ix.device));
    hipStream_t s = (hipStream_t)stream;
    const bool keep = (rp->flags & HNTL_ROUTER_KEEP_WEIGHTS) && ix.router;
    if (!keep) {
      init_router(ix, (int)(rp->hidden1 ? rp->hidden1 : 1024), (int)(rp->hidden2 ? rp->hidden2 : 1024));
      Router& rt = *ix.router;
      // He-style uniform initialisation from the counter-based generator
      for (int l = 0; l < 3; ++l) {
        const int fan_in = l == 0 ? rt.d : l == 1 ? rt.h1 : rt.h2;
        const double bound = std::sqrt((l < 2 ? 6.0 : 3.0) / fan_in);
        hipLaunchKernelGGL(init_weights_kernel, dim3(blocks(rt.wsize(l))), dim3(256), 0, s, rt.W[l], rt.wsize(l),
                           rp->seed, (uint64_t)(10 + l), bound);
        HIP_TRY(hipMemsetAsync(rt.b[l], 0, sizeof(float) * rt.bsize(l), s));
      }
      Scratch sc(s);
      double* part = sc.get<double>((size_t)STAT_SPLITS * ix.d);
      double* mu = sc.get<double>(ix.d);
      const dim3 grid(blocks(ix.d, 64), STAT_SPLITS);
      hipLaunchKernelGGL(col_moment_kernel, grid, dim3(256), 0, s, Qtrain, (int64_t)n, (int)ix.d,
                         (const double*)nullptr, part);
      hipLaunchKernelGGL(col_combine_kernel, dim3(blocks(ix.d)), dim3(256), 0, s, part, (int64_t)n, (int)ix.d, mu,
                         rt.mean, (float*)nullptr);
      hipLaunchKernelGGL(col_moment_kernel, grid, dim3(256), 0, s, Qtrain, (int64_t)n, (int)ix.d, (const double*)mu,
                         part);
      hipLaunchKernelGGL(col_combine_kernel, dim3(blocks(ix.d)), dim3(256), 0, s, part, (int64_t)n, (int)ix.d, mu,
                         (float*)nullptr, rt.stdv);
      HIP_TRY(hipGetLastError());
      rt.refresh_bf16(s);
    }
    Router& rt = *ix.router;
    // targets: grains of each training query's exact kt nearest neighbours
    int32_t* tg = nullptr;
    std::unique_ptr<int32_t, void (*)(int32_t*)> tg_own(nullptr, [](int32_t* p) { (void)hipFree(p); });
    if (targets) {
      tg = const_cast<int32_t*>(targets);
    } else {
      if (!ix.X) throw ArgError{HNTL_ESTATE, "kNN training targets need the raw vectors (pass targets instead)"};
      int32_t *ids = nullptr, *lab = nullptr;
      HIP_TRY(hipMalloc((void**)&tg, sizeof(int32_t) * (size_t)n * kt));
      tg_own.reset(tg);
      HIP_TRY(hipMalloc((void**)&ids, sizeof(int32_t) * (size_t)n * kt));
      HIP_TRY(hipMalloc((void**)&lab, sizeof(int32_t) * ix.N));
      launch_knn(Qtrain, n, ix.X, (int64_t)ix.N, (int)ix.d, (int)kt, ids, nullptr, s);
      hipLaunchKernelGGL(row_grain_kernel, dim3(blocks((int64_t)ix.N)), dim3(256), 0, s, ix.perm, ix.goff, (int)ix.G,
                         (int64_t)ix.N, lab);
      hipLaunchKernelGGL(map_ids_kernel, dim3(blocks((int64_t)n * kt)), dim3(256), 0, s, ids, (int64_t)n * kt, lab, tg);
      HIP_TRY(hipGetLastError());
      HIP_TRY(hipStreamSynchronize(s));
      (void)hipFree(ids);
      (void)hipFree(lab);
    }
    Trainer tr(rt, (int)B, s);
    const uint32_t nb = n / B;  // full batches per epoch
    const uint32_t epochs = rp->epochs ? rp->epochs : 1;
    std::vector<int32_t> order(n);
    std::iota(order.begin(), order.end(), 0);
    // Batches are not waited for: the order of the rows, the targets and the batches'
    // losses stay on the device for an epoch (a wait, a gather of targets on the host
    // and a copy per batch left the GPU idle for 2.6 ms of a 32-batch epoch).
    int32_t* d_order = nullptr;
    float* d_loss = nullptr;
    HIP_TRY(hipMalloc((void**)&d_order, sizeof(int32_t) * n));
    std::unique_ptr<int32_t, void (*)(int32_t*)> o1(d_order, [](int32_t* p) { (void)hipFree(p); });
    HIP_TRY(hipMalloc((void**)&d_loss, sizeof(float) * nb));
    std::unique_ptr<float, void (*)(float*)> o2(d_loss, [](float* p) { (void)hipFree(p); });
    std::vector<float> loss_h(nb);
    for (uint32_t ep = 0; ep < epochs; ++ep) {
      if (!(rp->flags & HNTL_ROUTER_NO_SHUFFLE))  // Fisher-Yates from the counter-based generator
        for (uint32_t i = n - 1; i > 0; --i) {
          const uint32_t j = (uint32_t)(uni(rp->seed, 100 + ep, i) * (double)(i + 1));
          std::swap(order[i], order[std::min(j, i)]);
        }
      HIP_TRY(hipMemcpyAsync(d_order, order.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
      HIP_TRY(hipMemsetAsync(d_loss, 0, sizeof(float) * nb, s));
      for (uint32_t bi = 0; bi < nb; ++bi) {
        const int32_t* rows = d_order + (size_t)bi * B;
        tr.grad(Qtrain, rows, tg, rows, (int)kt, d_loss + bi);
        tr.adam(rp->lr > 0 ? rp->lr : 1e-3f);
      }
      HIP_TRY(hipMemcpyAsync(loss_h.data(), d_loss, sizeof(float) * nb, hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));  // also keeps the row order from being overwritten early
      double eloss = 0.0;
      for (float l : loss_h) eloss += l;
      if (epoch_loss) epoch_loss[ep] = (float)(eloss / nb);
    }
    rt.trained = true;
  });
}

}  // extern "C"
