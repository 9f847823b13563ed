// Centroid routing (paper Section 2.1 step 1 and Section 2.3): squared
// Euclidean distance from every query to every grain centroid, then the P
// nearest grains per query.  The same distance tile also serves the k-means
// assignment of the build (nearest centroid per row).
//
// Distances use the expansion ||a||^2 + ||b||^2 - 2 a.b with the a.b term on
// MFMA: FP32 (v_mfma_f32_16x16x4_f32) here, BF16 (plain or split operands) in
// router.hip.  The expansion's rounding error is harmless for the k-means
// assignment; routing bounds it per entry and re-scores every shortlist entry
// that the bound leaves in reach of the P-th by direct differences before it
// picks the P probes.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "hntl_device.h"
#include "hntl_internal.h"

namespace hntl {

namespace {

constexpr int TM = 64, TN = 64, TK = 32, LDT = TK + 1;

__global__ __launch_bounds__(256) void row_norms_kernel(const float* __restrict__ A, int64_t rows, int d,
                                                        float* __restrict__ out) {
  const int lane = lane_id();
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float* a = A + row * d;
  float acc = 0.f;
  for (int j = lane; j < d; j += HNTL_WAVE) acc = fmaf(a[j], a[j], acc);
  acc = wave_sum(acc);
  if (lane == 0) out[row] = acc;
}

// One thread's 8 floats of a TM x TK tile of row-major M (rows x d) at
// (r0, k0): row tid / 4, depths 8 (tid % 4) .. + 7 (zero outside M).
__device__ __forceinline__ void fetch_tile(float4 (&v)[2], const float* __restrict__ M, int64_t nrows, int d,
                                           int64_t r0, int k0, bool vec4) {
  const int tid = threadIdx.x;
  const int rr = tid >> 2, cc = (tid & 3) * 8;
  const int64_t gr = r0 + rr;
  if (vec4) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int gk = k0 + cc + 4 * u;
      v[u] = (gr < nrows && gk < d) ? *reinterpret_cast<const float4*>(M + gr * d + gk)
                                    : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  } else {
    float e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int gk = k0 + cc + u;
      e[u] = (gr < nrows && gk < d) ? M[gr * d + gk] : 0.f;
    }
    v[0] = make_float4(e[0], e[1], e[2], e[3]);
    v[1] = make_float4(e[4], e[5], e[6], e[7]);
  }
}

__device__ __forceinline__ void store_tile(float (*S)[LDT], const float4 (&v)[2]) {
  const int tid = threadIdx.x;
  const int rr = tid >> 2, cc = (tid & 3) * 8;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    S[rr][cc + 4 * u] = v[u].x;
    S[rr][cc + 4 * u + 1] = v[u].y;
    S[rr][cc + 4 * u + 2] = v[u].z;
    S[rr][cc + 4 * u + 3] = v[u].w;
  }
}

// One 64 x 64 tile of A.B^T accumulated over the full depth d; each of the 4
// waves owns a 32 x 32 quarter as 2 x 2 MFMA 16x16 tiles.  The next depth
// tile is fetched into registers while the MFMAs of the current one run.
__device__ __forceinline__ void tile_dot(floatx4 (&acc)[2][2], float (*As)[LDT], float (*Bs)[LDT],
                                         const float* __restrict__ A, int64_t rows, const float* __restrict__ Bm,
                                         int cols, int d, int64_t row0, int col0, bool vec4) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  float4 fa[2], fb[2];
  fetch_tile(fa, A, rows, d, row0, 0, vec4);
  fetch_tile(fb, Bm, cols, d, col0, 0, vec4);
  for (int k0 = 0; k0 < d; k0 += TK) {
    store_tile(As, fa);
    store_tile(Bs, fb);
    __syncthreads();
    if (k0 + TK < d) {
      fetch_tile(fa, A, rows, d, row0, k0 + TK, vec4);
      fetch_tile(fb, Bm, cols, d, col0, k0 + TK, vec4);
    }
#pragma unroll
    for (int kk = 0; kk < TK; kk += 4) {
      const int kr = kk + (lane >> 4);
      const float a0 = As[wr + (lane & 15)][kr];
      const float a1 = As[wr + 16 + (lane & 15)][kr];
      const float b0 = Bs[wc + (lane & 15)][kr];
      const float b1 = Bs[wc + 16 + (lane & 15)][kr];
      acc[0][0] = mfma16x16x4(a0, b0, acc[0][0]);
      acc[0][1] = mfma16x16x4(a0, b1, acc[0][1]);
      acc[1][0] = mfma16x16x4(a1, b0, acc[1][0]);
      acc[1][1] = mfma16x16x4(a1, b1, acc[1][1]);
    }
    __syncthreads();
  }
}

// ---------------------------------- FP32 products from direct LDS loads
// The products of tile_dot in another order of depths, for 16-byte aligned rows
// with d % 4 == 0 and for callers that re-score what they pick (routing, kNN).
// An RT x CT tile of A.B^T is shared by WR x WC waves of
// (RT / WR) x (CT / WC) each.  Depth chunks of 32 go from global memory
// straight into the LDS (global_load_lds_dwordx4), into two buffers: chunk
// k + 1 is requested before chunk k is multiplied, one barrier per chunk.  The
// buffers are two arrays and the loops are unrolled over them: with one array
// indexed by k % 2 the compiler cannot tell the requested half from the read
// one and waits for the request before the first LDS read (18.4 instead of
// 13.5 ms for 1,024 x 1,000,000 x 768).  A
// row of a chunk is 8 vectors of 4 depths; vector c of row r sits at position
// c ^ (r % 8), so the 16 rows of one operand read spread over the banks.  Rows
// past the end load the last row, vectors past d
// the row's first (neither reaches a result).  Bound by the FP32 MFMA units:
// 1,024 x 1,000,000 x 768 runs at the rates stated at the kernels below
// against tile_dot's 94 TFLOP/s (64 x 64 tiles, one LDS buffer filled through
// registers, two barriers per chunk).
constexpr int FK = 32;
typedef __attribute__((address_space(3))) void* lds_ptr_t;

template <int ROWS, int NW>
__device__ __forceinline__ void fetch_chunk(float* dst, const float* __restrict__ X, int64_t nrows, int d, int64_t r0,
                                            int k0) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
#pragma unroll
  for (int h = 0; h < (ROWS / 8 + NW - 1) / NW; ++h) {
    const int u = h * NW + wave;  // one instruction: 8 rows, LDS bytes 1024 u .. + 1023
    if (ROWS / 8 % NW == 0 || u < ROWS / 8) {
      const int row = u * 8 + (lane >> 3);
      const int k = k0 + ((lane & 7) ^ (row & 7)) * 4;
      const int64_t gr = r0 + row < nrows ? r0 + row : nrows - 1;
      __builtin_amdgcn_global_load_lds((const void*)(X + gr * d + (k < d ? k : 0)), (lds_ptr_t)(dst + (size_t)u * 256),
                                       16, 0, 0);
    }
  }
}

// One half (16 depths) of a chunk in a wave's registers: MT row and NT column
// groups of 16.  Lane (i, kq) holds depths 16 h + 4 kq .. + 3 of row / column i,
// one 16-byte LDS read each, free of bank conflicts, and feeds depth
// 16 h + 4 kq + e in MFMA step e.  (Dword reads in MFMA order would be merged
// by the compiler into two-address reads that lose the arrays' identity, and
// with it the overlap with the requests.)
template <int MT, int NT>
struct HalfFrag {
  floatx4 a[MT], b[NT];
  __device__ __forceinline__ void load(const float* As, const float* Bs, int wr, int wc, int h) {
    const int lane = lane_id(), i = lane & 15;
    const int x = (((lane >> 4) + 4 * h) ^ (i & 7)) * 4;
#pragma unroll
    for (int m = 0; m < MT; ++m) a[m] = *reinterpret_cast<const floatx4*>(As + (wr + 16 * m + i) * FK + x);
#pragma unroll
    for (int n = 0; n < NT; ++n) b[n] = *reinterpret_cast<const floatx4*>(Bs + (wc + 16 * n + i) * FK + x);
  }
  // zeros from depth `valid` of the chunk on (valid % 4 == 0)
  __device__ __forceinline__ void clip(int h, int valid) {
    const bool in = 16 * h + 4 * (lane_id() >> 4) < valid;
#pragma unroll
    for (int m = 0; m < MT; ++m) a[m] = in ? a[m] : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < NT; ++n) b[n] = in ? b[n] : floatx4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void mma(floatx4 (&acc)[MT][NT]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = mfma16x16x4(a[m][e], b[n][e], acc[m][n]);
  }
};

// One chunk of the stream, its first half already in f0: reads the second half
// and multiplies the first; then, with `more`, waits for the next chunk
// (requested one chunk earlier), calls request() (the chunk after it, into this
// chunk's buffer, which every wave has read by then) and reads the next
// chunk's first half; then multiplies the second half.  The barrier and the
// LDS reads that follow it so have half a chunk of MFMAs to hide behind.
// extra(): further reads of this chunk.
template <int MT, int NT, class Request, class Extra>
__device__ __forceinline__ void chunk_step(floatx4 (&acc)[MT][NT], HalfFrag<MT, NT>& f0, const float* As,
                                           const float* Bs, const float* nAs, const float* nBs, int wr, int wc,
                                           int valid, bool more, int next_valid, Request&& request, Extra&& extra) {
  HalfFrag<MT, NT> f1;
  f1.load(As, Bs, wr, wc, 1);
  if (valid < FK) f1.clip(1, valid);
  extra();
  f0.mma(acc);
  if (more) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's requests for the next chunk have landed, its reads of this one are done
    __syncthreads();                // every wave's are
    request();
    f0.load(nAs, nBs, wr, wc, 0);
    if (next_valid < FK) f0.clip(0, next_valid);
    __builtin_amdgcn_sched_barrier(0);
  }
  f1.mma(acc);
}

// Stores a wave's MT x NT MFMA tiles of distances from (row0, col0).  The norms
// are loaded before the first store: a load after a store would wait for it.
template <int MT, int NT>
__device__ __forceinline__ void store_dist(const floatx4 (&acc)[MT][NT], const float* __restrict__ an, int64_t row0,
                                           int64_t rows, const float* __restrict__ bn, int col0, int cols,
                                           float* __restrict__ D) {
  const int lane = lane_id();
  float ar[MT][4], br[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) br[n] = bn[min(col0 + n * 16 + (lane & 15), cols - 1)];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = row0 + m * 16 + 4 * (lane >> 4) + i;
      ar[m][i] = an[row < rows ? row : rows - 1];
    }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = row0 + m * 16 + 4 * (lane >> 4) + i;
      if (row >= rows) continue;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const int col = col0 + n * 16 + (lane & 15);
        if (col < cols) D[row * cols + col] = fmaxf(ar[m][i] + br[n] - 2.f * acc[m][n][i], 0.f);
      }
    }
}

// Distances on the tiles above: 10,000 x 1,024 x 768 in 155 us (101 TFLOP/s; 158 on
// tile_dot), 300 x 2,048 x 768 in 22 us (31 on tile_dot), 16,384 x 8,192 x 768 in
// 1.77 ms (117 TFLOP/s; 1.88).  Without the requests the loop runs at 137 to 143
// TFLOP/s, without the stores of D 8% faster.
template <int RT, int CT, int WR, int WC>
__global__ __launch_bounds__(64 * WR * WC) void dist_tile_kernel(const float* __restrict__ A,
                                                                 const float* __restrict__ an, int64_t rows,
                                                                 const float* __restrict__ Bm,
                                                                 const float* __restrict__ bn, int cols, int d,
                                                                 float* __restrict__ D,
                                                                 const int32_t* __restrict__ nlim, int64_t row_base) {
  constexpr int NW = WR * WC, MT = RT / WR / 16, NT = CT / WC / 16;
  __shared__ __align__(16) float buf0[(RT + CT) * FK], buf1[(RT + CT) * FK];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * RT;
  if (nlim) {  // rows from *nlim - row_base on are not part of this batch
    const int64_t lim = (int64_t)*nlim - row_base;
    if (row0 >= lim) return;
    if (lim < rows) rows = lim;
  }
  const int col0 = blockIdx.y * CT;
  const int wr = wave / WC * (RT / WR), wc = wave % WC * (CT / WC);
  floatx4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int nk = (d + FK - 1) / FK;
  auto fetch = [&](float* dst, int k) {
    if (k < nk) {
      fetch_chunk<RT, NW>(dst, A, rows, d, row0, k * FK);
      fetch_chunk<CT, NW>(dst + RT * FK, Bm, cols, d, col0, k * FK);
    }
  };
  auto none = []() {};
  HalfFrag<MT, NT> f0;
  fetch(buf0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  fetch(buf1, 1);
  f0.load(buf0, buf0 + RT * FK, wr, wc, 0);
  if (d < FK) f0.clip(0, d);
  for (int k = 0; k < nk; k += 2) {
    chunk_step(acc, f0, buf0, buf0 + RT * FK, buf1, buf1 + RT * FK, wr, wc, d - k * FK, k + 1 < nk,
               d - (k + 1) * FK, [&]() { fetch(buf0, k + 2); }, none);
    if (k + 1 >= nk) break;
    chunk_step(acc, f0, buf1, buf1 + RT * FK, buf0, buf0 + RT * FK, wr, wc, d - (k + 1) * FK, k + 2 < nk,
               d - (k + 2) * FK, [&]() { fetch(buf1, k + 3); }, none);
  }
  store_dist<MT, NT>(acc, an, row0 + wr, rows, bn, col0 + wc, cols, D);
}

// The same distances on tile_dot: short rows and rows that allow no 16-byte
// loads (odd depths, unaligned operands).
__global__ __launch_bounds__(256) void dist_matrix_kernel(const float* __restrict__ A, const float* __restrict__ an,
                                                          int64_t rows, const float* __restrict__ Bm,
                                                          const float* __restrict__ bn, int cols, int d,
                                                          float* __restrict__ D, bool vec4,
                                                          const int32_t* __restrict__ nlim, int64_t row_base) {
  __shared__ float As[TM][LDT];
  __shared__ float Bs[TN][LDT];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * TM;
  if (nlim) {  // rows from *nlim - row_base on are not part of this batch
    const int64_t lim = (int64_t)*nlim - row_base;
    if (row0 >= lim) return;
    if (lim < rows) rows = lim;
  }
  const int col0 = blockIdx.y * TN;
  floatx4 acc[2][2];
  tile_dot(acc, As, Bs, A, rows, Bm, cols, d, row0, col0, vec4);
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  store_dist<2, 2>(acc, an, row0 + wr, rows, bn, col0 + wc, cols, D);
}

// Small batches (<= 16 rows): exact distances by direct differences, one
// wave per column (centroid) held in registers (d <= 1024), every row of A
// against it.  Reads each centroid once instead of staging mostly empty
// 64-row MFMA tiles.
constexpr int DIRECT_ROWS = 16;
__global__ __launch_bounds__(256) void dist_direct_kernel(const float* __restrict__ A, int64_t rows,
                                                          const float* __restrict__ Bm, int cols, int d,
                                                          float* __restrict__ D, const int32_t* __restrict__ nlim,
                                                          int64_t row_base) {
  const int lane = lane_id();
  const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= cols) return;
  int64_t nr = rows;
  if (nlim) {
    const int64_t lim = (int64_t)*nlim - row_base;
    if (lim < nr) nr = lim;
  }
  const float* b = Bm + (size_t)col * d;
  float bv[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int j = u * HNTL_WAVE + lane;
    bv[u] = j < d ? b[j] : 0.f;
  }
  for (int64_t r = 0; r < nr; ++r) {
    const float* a = A + r * d;
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int j = u * HNTL_WAVE + lane;
      if (j < d) {
        const float df = a[j] - bv[u];
        acc = fmaf(df, df, acc);
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) D[r * cols + col] = acc;
  }
}

__global__ __launch_bounds__(256) void argmin_rows_kernel(const float* __restrict__ A, const float* __restrict__ an,
                                                          int64_t rows, const float* __restrict__ Bm,
                                                          const float* __restrict__ bn, int cols, int d,
                                                          int32_t* __restrict__ label, float* __restrict__ dmin,
                                                          bool vec4) {
  __shared__ float As[TM][LDT];
  __shared__ float Bs[TN][LDT];
  __shared__ float red_d[4][32];
  __shared__ int red_i[4][32];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * TM;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  float bd[2][4];
  int bi[2][4];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bd[rt][i] = __builtin_inff();
      bi[rt][i] = 0x7fffffff;
    }
  for (int col0 = 0; col0 < cols; col0 += TN) {
    floatx4 acc[2][2];
    tile_dot(acc, As, Bs, A, rows, Bm, cols, d, row0, col0, vec4);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t row = row0 + wr + rt * 16 + 4 * (lane >> 4) + i;
          const int col = col0 + wc + ct * 16 + (lane & 15);
          if (row < rows && col < cols) {
            const float v = fmaxf(an[row] + bn[col] - 2.f * acc[rt][ct][i], 0.f);
            if (v < bd[rt][i] || (v == bd[rt][i] && col < bi[rt][i])) {
              bd[rt][i] = v;
              bi[rt][i] = col;
            }
          }
        }
  }
  // reduce over the 16 lanes that share a row, then over the two waves that
  // share the same rows
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = bd[rt][i];
      int c = bi[rt][i];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        const float ov = __shfl_xor(v, o, 64);
        const int oc = __shfl_xor(c, o, 64);
        if (ov < v || (ov == v && oc < c)) {
          v = ov;
          c = oc;
        }
      }
      if ((lane & 15) == 0) {
        red_d[wave][rt * 16 + 4 * (lane >> 4) + i] = v;
        red_i[wave][rt * 16 + 4 * (lane >> 4) + i] = c;
      }
    }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int r = threadIdx.x;
    const int w0 = 2 * (r >> 5);
    float v = red_d[w0][r & 31];
    int c = red_i[w0][r & 31];
    const float v1 = red_d[w0 + 1][r & 31];
    const int c1 = red_i[w0 + 1][r & 31];
    if (v1 < v || (v1 == v && c1 < c)) {
      v = v1;
      c = c1;
    }
    const int64_t row = row0 + r;
    if (row < rows) {
      label[row] = c;
      if (dmin) dmin[row] = v;
    }
  }
}

// Top-P per row of D.  Without A/Bm: the P smallest entries of D.  With them
// (routing), D holds expansion distances ||a||^2 + ||b||^2 - 2 <a, b> whose
// error against the exact distance is at most err (||a||^2 + ||b||^2) per
// entry (the caller's bound for its product form).  A shortlist of the
// smallest expansion values is kept (all that the bounds leave in reach of the
// P-th, or the M smallest where those are too many); every entry j whose interval
// [D_j - bound_j, D_j + bound_j] reaches the P-th entry's upper end can still
// be among the P nearest, so exactly those are re-scored by direct
// differences ||a - b||^2 in FP32 and the P smallest exact distances are kept
// (ties: lower column).  Probe order and reported distances then carry
// direct-difference accuracy.  If the window reaches the end of the
// shortlist (entry M - 1 qualifies while columns remain beyond it), entries
// past M may qualify as well: the row is then re-read whole, and every column
// inside the window is re-scored.
//
// Rows per workgroup, one per wave.
constexpr int TOPK_ROWS = 4;

// Direct FP32 squared distance of row a and column row b (both d long), one
// wave, every lane ends with the total.
// With vec4 (d % 4 == 0, 16-byte aligned rows) lane l covers depths
// 4 l .. 4 l + 3 of every 256-wide chunk, in that order; otherwise depths l,
// l + 64, ...
__device__ __forceinline__ float wave_dist(const float* __restrict__ a, const float* __restrict__ b, int d,
                                           bool vec4) {
  float acc = 0.f;
  if (vec4) {
    for (int t = lane_id() * 4; t < d; t += 4 * HNTL_WAVE) {
      const float4 x = *reinterpret_cast<const float4*>(a + t), y = *reinterpret_cast<const float4*>(b + t);
      float df = x.x - y.x;
      acc = fmaf(df, df, acc);
      df = x.y - y.y;
      acc = fmaf(df, df, acc);
      df = x.z - y.z;
      acc = fmaf(df, df, acc);
      df = x.w - y.w;
      acc = fmaf(df, df, acc);
    }
  } else {
    for (int t = lane_id(); t < d; t += HNTL_WAVE) {
      const float df = a[t] - b[t];
      acc = fmaf(df, df, acc);
    }
  }
  return wave_sum(acc);
}

// The M smallest entries of a row of any length by a streamed top-64 list (one
// wave; lane i of the result holds the i-th smallest key).  Segments of U chunks
// of 64 columns, loaded together.  The 64 lanes' minima over a segment are 64
// entries of the row, so their maximum bounds the row's 64th smallest value (>=
// its M-th and P-th) from above: entries above the smallest such bound so far
// cannot be selected and are not offered (fewer list flushes; the selection is
// unchanged).
__device__ __forceinline__ uint64_t row_smallest(const float* __restrict__ drow, int cols, int M, uint64_t* stage,
                                                 bool znorm, float& mn, float& z) {
  const int lane = lane_id();
  WaveTop64 L;
  L.init(stage, M);
  constexpr int U = 16;
  float T = __builtin_inff();  // uniform
  // znorm (negated scores): the row's smallest value mn and z = sum exp(mn - D_c),
  // the softmax normaliser of the scores, accumulated per lane against the
  // lane's running minimum and rescaled when it drops
  float lmn = __builtin_inff(), lz = 0.f;
  for (int c0 = 0; c0 < cols; c0 += U * HNTL_WAVE) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u * HNTL_WAVE + lane;
      v[u] = c < cols ? drow[c] : __builtin_inff();
    }
    float seg = v[0];
#pragma unroll
    for (int u = 1; u < U; ++u) seg = fminf(seg, v[u]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) seg = fmaxf(seg, __shfl_xor(seg, o, 64));
    T = fminf(T, seg);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u * HNTL_WAVE + lane;
      L.offer_f(v[u], (uint32_t)c, c < cols && v[u] <= T);
    }
    if (znorm) {
      float cm = __builtin_inff();
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u * HNTL_WAVE + lane < cols) cm = fminf(cm, v[u]);
      if (cm < __builtin_inff()) {
        const float nm = fminf(lmn, cm);
        lz = lmn < __builtin_inff() ? lz * expf(nm - lmn) : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (c0 + u * HNTL_WAVE + lane < cols) lz += expf(nm - v[u]);
        lmn = nm;
      }
    }
  }
  L.finish();
  if (znorm) {
    mn = lmn;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mn = fminf(mn, __shfl_xor(mn, o, 64));
    z = wave_sum(lmn < __builtin_inff() ? lz * expf(mn - lmn) : 0.f);
  }
  return L.best;
}

// Bitonic sort of one float per lane, ascending (no NaN).
__device__ __forceinline__ float wave_sort64f(float v) {
  const int lane = lane_id();
  auto step = [&](auto jc, int k) {
    constexpr int J = decltype(jc)::value;
    const float o = __uint_as_float(lane_xor<J>(__float_as_uint(v)));
    v = (((lane & k) == 0) == ((lane & J) == 0)) ? fminf(v, o) : fmaxf(v, o);
  };
#pragma unroll
  for (int k = 2; k <= 64; k <<= 1) {
    if (k >= 64) step(std::integral_constant<int, 32>{}, k);
    if (k >= 32) step(std::integral_constant<int, 16>{}, k);
    if (k >= 16) step(std::integral_constant<int, 8>{}, k);
    if (k >= 8) step(std::integral_constant<int, 4>{}, k);
    if (k >= 4) step(std::integral_constant<int, 2>{}, k);
    step(std::integral_constant<int, 1>{}, k);
  }
  return v;
}

// The same for rows of up to 64 NCH columns, held in registers (NCH values per
// lane, every load in flight at once).  The P-th smallest of the 64 lanes'
// minima is at least the row's P-th smallest value T; every entry up to it plus
// `slack` is collected (a compare and a ballot per chunk), and one sort orders
// them.  Returns their number, or -1 if they are more than 64 (the caller
// streams the row instead); lane i < number holds the i-th smallest key.
template <int NCH>
__device__ __forceinline__ int row_window(const float* __restrict__ drow, int cols, int P, float slack,
                                          uint64_t* stage, bool znorm, float& mn, float& z, uint64_t& out) {
  const int lane = lane_id();
  float v[NCH];
  // bounds-checked buffer loads: one address register, past the row's end reads 0
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(drow), 0, 4 * cols, 0x00027000);
#pragma unroll
  for (int u = 0; u < NCH; ++u)
    v[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, 4 * lane + 4 * HNTL_WAVE * u, 0, 0));
#pragma unroll
  for (int u = 0; u < NCH; ++u)
    if (lane >= cols - u * HNTL_WAVE) v[u] = __builtin_inff();
  float own = v[0];
#pragma unroll
  for (int u = 1; u < NCH; ++u) own = fminf(own, v[u]);
  const float srt = wave_sort64f(own == own ? own : __builtin_inff());
  mn = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(srt), 0));
  if (znorm) {
    float lz = 0.f;
    if (mn < __builtin_inff()) {
#pragma unroll
      for (int u = 0; u < NCH; ++u) lz += expf(mn - v[u]);
    }
    z = wave_sum(lz);
  }
  float T = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(srt), P - 1)) + slack;
  T += 1e-6f * fabsf(T);
  if (!(T < __builtin_inff())) return -1;  // padding must not qualify
  int n = 0;
#pragma unroll
  for (int u = 0; u < NCH; ++u) {
    const bool in = v[u] <= T;
    const uint64_t m = __ballot(in);
    if (m) {
      const int at = n + mbcnt64(m);
      if (in && at < 64) stage[at] = make_key(v[u], (uint32_t)(u * HNTL_WAVE + lane));
      n += __popcll(m);
    }
  }
  if (n > 64) return -1;
  wave_sync();
  const uint64_t k = lane < n ? stage[lane] : KEY_NONE;
  wave_sync();
  out = wave_sort64(k);
  return n;
}

// Bound by memory (the row is read once: 135 us of 16,384 x 8,192 at 4 TB/s, then
// 3 KB a re-scored entry from cache) with one row per wave and its whole row in
// flight.  At 16,384 x 8,192: scores 123 us, distances with 27 re-scored entries
// a row 210 us; a streamed list (16 chunks a segment, about ten flushes a row)
// took 185 and 273.  256 such rows 29 us (49), 10,000 x 1,024 30 us (49), one row
// of 1,024 5.8 us (10.8).
// bmax: the largest bn (device).
template <int NCH>
__global__ __launch_bounds__(TOPK_ROWS * 64, NCH > 64 ? 3 : 4) void topk_rows_kernel(
    const float* __restrict__ D, int64_t rows, int cols, int P, int M, const float* __restrict__ A,
    const float* __restrict__ an, const float* __restrict__ Bm, const float* __restrict__ bn,
    const float* __restrict__ bmax, int d, float err, int32_t* __restrict__ idx, float* __restrict__ val,
    const int32_t* __restrict__ nlim, int64_t row_base, unsigned int* __restrict__ overflow,
    float2* __restrict__ znorm, bool vec4) {
  __shared__ uint64_t stage[TOPK_ROWS][64];
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = (int64_t)blockIdx.x * TOPK_ROWS + wave;
  if (row >= rows) return;
  if (nlim && row >= (int64_t)*nlim - row_base) {  // not part of this batch: no probes
    if (lane < P) {
      idx[row * P + lane] = -1;
      if (val) val[row * P + lane] = __builtin_inff();
    }
    return;
  }
  const bool exact = A != nullptr;
  const float* drow = D + row * cols;
  const float arow = exact ? an[row] : 0.f;
  float mn = __builtin_inff(), z = 0.f;
  uint64_t mine = KEY_NONE;  // lane i: the i-th smallest key of the shortlist
  int have = -1;             // its length; every entry of the window is in it (-1: only the M smallest are)
  if constexpr (NCH > 0)
    have = row_window<NCH>(drow, cols, P, exact ? 2.f * err * (arow + *bmax) : 0.f, stage[wave], znorm != nullptr, mn,
                           z, mine);
  if (have < 0) mine = row_smallest(drow, cols, exact ? M : P, stage[wave], znorm != nullptr, mn, z);
  if (znorm && lane == 0) znorm[row] = make_float2(mn, z);
  if (!exact) {
    if (lane < P) {
      idx[row * P + lane] = mine == KEY_NONE ? -1 : (int32_t)key_id(mine);
      if (val) val[row * P + lane] = mine == KEY_NONE ? __builtin_inff() : key_dist(mine);
    }
    return;
  }
  // entries j >= P qualify while D_j - bound_j <= D_{P-1} + bound_{P-1}
  const uint64_t kp = shfl_u64(mine, P - 1);
  const float hiP = key_dist(kp) + err * (arow + bn[min(key_id(kp), (uint32_t)cols - 1)]);
  const bool in = lane >= P && lane < (have < 0 ? M : 64) && mine != KEY_NONE &&
                  key_dist(mine) - err * (arow + bn[key_id(mine)]) <= hiP;
  const uint64_t qual = __ballot(in);
  const int Mr = qual ? 64 - __clzll(qual) : P;  // re-score the prefix [0, Mr)
  const float* a = A + row * d;
  uint64_t ex = KEY_NONE;
  if (have < 0 && Mr == M && M < cols) {
    // the window may extend past the shortlist: every column of the row whose
    // interval reaches hiP is re-scored, into a fresh top-P list
    if (overflow && lane == 0) atomicAdd(overflow, 1u);
    WaveTop64 X;
    wave_sync();
    X.init(stage[wave], P);
    for (int c0 = 0; c0 < cols; c0 += HNTL_WAVE) {
      const int c = c0 + lane;
      const bool w = c < cols && drow[c] - err * (arow + bn[c]) <= hiP;
      uint64_t m = __ballot(w);
      uint64_t keyc = KEY_NONE;
      while (m) {  // wave-uniform loop over the window columns of this chunk
        const int j = __builtin_ctzll(m);
        m &= m - 1;
        const float dd = wave_dist(a, Bm + (size_t)(c0 + j) * d, d, vec4);
        if (lane == j) keyc = make_key(dd, (uint32_t)(c0 + j));
      }
      X.offer(keyc, w);
    }
    X.finish();
    ex = X.best;
  } else {
    constexpr int RB = 8;  // shortlist entries re-scored together
    for (int j0 = 0; j0 < Mr; j0 += RB) {
      int cs[RB];
      const float* bp[RB];
      float acc[RB];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int j = j0 + u < Mr ? j0 + u : j0;
        // (a place without an entry reads some column, and its result is dropped below)
        cs[u] = (int)min(key_id(shfl_u64(mine, j)), (uint32_t)cols - 1);
        bp[u] = Bm + (size_t)cs[u] * d;
        acc[u] = 0.f;
      }
      if (vec4) {
        // 16-byte loads, the whole rows' in flight up to 768 depths
        constexpr int CH = NCH > 64 ? 3 : 1;
        for (int t0 = lane * 4; t0 < d; t0 += CH * 4 * HNTL_WAVE) {
          float4 av[CH], bv[CH][RB];
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            const int t = t0 + i * 4 * HNTL_WAVE;
            av[i] = t < d ? *reinterpret_cast<const float4*>(a + t) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < RB; ++u)
              bv[i][u] = t < d ? *reinterpret_cast<const float4*>(bp[u] + t) : make_float4(0.f, 0.f, 0.f, 0.f);
          }
#pragma unroll
          for (int i = 0; i < CH; ++i) {
#pragma unroll
            for (int u = 0; u < RB; ++u) {
              float df = av[i].x - bv[i][u].x;
              acc[u] = fmaf(df, df, acc[u]);
              df = av[i].y - bv[i][u].y;
              acc[u] = fmaf(df, df, acc[u]);
              df = av[i].z - bv[i][u].z;
              acc[u] = fmaf(df, df, acc[u]);
              df = av[i].w - bv[i][u].w;
              acc[u] = fmaf(df, df, acc[u]);
            }
          }
        }
      } else {
        for (int t = lane; t < d; t += HNTL_WAVE) {
          const float av = a[t];
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const float df = av - bp[u][t];
            acc[u] = fmaf(df, df, acc[u]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const float tot = wave_sum(acc[u]);
        if (lane == j0 + u && lane < Mr && mine != KEY_NONE) ex = make_key(tot, (uint32_t)cs[u]);
      }
    }
    ex = wave_sort64(ex);
  }
  // A row with fewer than P entries (its distances are NaN: a query or centroids that are not
  // finite) has fewer probes.  Never the same column twice: plans size their lists for P
  // different grains.
  if (lane < P) {
    idx[row * P + lane] = ex == KEY_NONE ? -1 : (int32_t)key_id(ex);
    if (val) val[row * P + lane] = ex == KEY_NONE ? __builtin_inff() : key_dist(ex);
  }
}

__global__ __launch_bounds__(1024) void max_kernel(const float* __restrict__ a, int n, float* __restrict__ out) {
  __shared__ float red[1024];
  float v = 0.f;
  for (int i = threadIdx.x; i < n; i += 1024) v = fmaxf(v, a[i]);
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// ------------------------------------------------------- brute-force kNN
// Exact k nearest rows of B for every row of A (the learned router's training
// targets).  Pass 1: a workgroup walks a range of columns in tiles of MFMA
// expansion distances and keeps, for each of its rows, the KNN_SHORT smallest
// (distance, column) keys.  Pass 2 merges the ranges' lists per row, re-scores
// the merged shortlist by direct differences in FP32 and keeps the k smallest
// exact distances (ties: lower column).
//
// knn_tile_kernel is pass 1 for 16-byte aligned rows.  Tiles of RT rows x 128
// columns by 8 waves, chunks of 32 depths by direct LDS loads, the chunks of
// consecutive tiles in one stream (the next tile's first chunk loads while
// this tile's candidates are taken).  A tile's values are tested in the
// accumulator registers against their row's threshold (the value of its 32nd
// best key) and the few that pass are appended to the row's stage in the LDS;
// when a stage is full its row is sorted by one wave (32 kept + 32 staged keys,
// one bitonic sort of 64) and the values that found no room are offered again.
// The squared norms of B's rows are summed from the chunks in the LDS: a pass
// of their own over B (3.1 GB at 1M x 768) cost 0.87 ms.  Bound by the FP32 MFMA
// units at 64 and 128 rows, by reading B once at 16.  Whole call over
// 1,000,000 x 768, before (64 x 64 tiles of tile_dot whose every value went
// through the LDS to a list, 128 ranges a row) and now: 1 query 2.93 -> 0.81 ms
// (3.8 TB/s), 16 3.19 -> 0.92, 64 3.33 -> 1.42, 300 6.87 -> 5.19, 1,024
// 17.8 -> 13.9 (113 TFLOP/s).
constexpr int KNN_SHORT = 32;

constexpr int KNN_COLS = 128, KNN_WAVES = 8;

// Staged keys of a row (RT = 64: 16, so that two workgroups fit a CU's LDS).
template <int RT>
constexpr int knn_stage = RT == 64 ? 16 : 32;
// (the second bound: waves per SIMD, so that the CU's LDS is what limits its workgroups)
template <int RT, int WR, int WC>
__global__ __launch_bounds__(64 * KNN_WAVES, RT == 128 ? 2 : 4) void knn_tile_kernel(const float* __restrict__ A,
                                                                  const float* __restrict__ an, int64_t rows,
                                                                  const float* __restrict__ Bm, int64_t cols, int d,
                                                                  int64_t per_split, int splits, int row_tiles,
                                                                  uint64_t* __restrict__ part) {
  constexpr int NW = KNN_WAVES, MT = RT / WR / 16, NT = KNN_COLS / WC / 16;
  constexpr int STG = knn_stage<RT>, LK = KNN_SHORT + STG;
  static_assert(WR * WC == NW && MT * NT * 4 <= 32, "one pending bit per accumulator element");
  __shared__ __align__(16) float buf0[(RT + KNN_COLS) * FK], buf1[(RT + KNN_COLS) * FK];
  __shared__ uint64_t keys[RT * LK];  // per row: sorted list, then stage
  __shared__ float bnorm[KNN_COLS], thr[RT];
  __shared__ int cnt[RT];
  // With 8 ranges or more, the row tiles of one range run on one XCD
  // (workgroup b is dealt to XCD b % 8) and share its reads of B.
  const int b = (int)blockIdx.x;
  const int rt = splits >= 8 ? (b >> 3) % row_tiles : b % row_tiles;
  const int split = splits >= 8 ? (b >> 3) / row_tiles * 8 + (b & 7) : b / row_tiles;
  if (split >= splits) return;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)rt * RT;
  const int64_t c_begin = (int64_t)split * per_split;
  const int64_t c_end = c_begin + per_split < cols ? c_begin + per_split : cols;
  const int wr = wave / WC * (RT / WR), wc = wave % WC * (KNN_COLS / WC);
  for (int e = threadIdx.x; e < RT * LK; e += 64 * NW) keys[e] = KEY_NONE;
  for (int e = threadIdx.x; e < RT; e += 64 * NW) {
    thr[e] = __builtin_inff();
    cnt[e] = 0;
  }
  float arow[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = row0 + wr + m * 16 + 4 * (lane >> 4) + i;
      arow[m][i] = row < rows ? an[row] : 0.f;
    }
  // one wave sorts a row's kept and staged keys and keeps the smallest (first: the
  // columns still to be offered begin at it)
  auto flush_row = [&](int r, uint32_t first) {
    uint64_t* kr = keys + (size_t)r * LK;
    const int n = KNN_SHORT + min(cnt[r], STG);
    wave_sync();
    uint64_t k = lane < n ? kr[lane] : KEY_NONE;
    k = wave_sort64(k);
    wave_sync();
    if (lane < KNN_SHORT) kr[lane] = k;
    const uint64_t last = lane_u64(k, KNN_SHORT - 1);
    float t = key_ceil(last);
    // Equal values of higher columns lose: with the 32nd best before the tile, the threshold is
    // the next smaller value (values are >= 0).  Where every row of B ties, each value went
    // through a sort otherwise: 512 queries over 200,000 equal rows of 128 2,190 us, so 430
    // (600 where the rows differ).
    if (last != KEY_NONE && key_id(last) < first) t = t > 0.f ? __uint_as_float(__float_as_uint(t) - 1) : -1.f;
    if (lane == 0) {
      thr[r] = t;
      cnt[r] = 0;
    }
  };
  // the wave's rows wave, wave + NW, ... whose stage holds at least `least` keys
  auto flush_rows = [&](int least, int64_t first) {
    const int own = lane < RT / NW ? cnt[wave + lane * NW] : 0;
    uint64_t m = __ballot(own >= least);
    while (m) {  // wave-uniform
      const int j = __builtin_ctzll(m);
      m &= m - 1;
      flush_row(wave + j * NW, (uint32_t)first);
    }
  };

  const int nk = (d + FK - 1) / FK;
  // chunk k of the tile at col, which for k >= nk lies in the next tile (nk
  // even: the stream of chunks goes on over the tiles; nk odd: the buffer that
  // the next tile starts with is the one its last chunk was read from, so each
  // tile starts anew)
  auto fetch = [&](float* dst, int64_t col, int k) {
    if (k >= nk) {
      col += KNN_COLS;
      k -= nk;
    }
    if (col < c_end && k < nk) {
      fetch_chunk<RT, NW>(dst, A, rows, d, row0, k * FK);
      fetch_chunk<KNN_COLS, NW>(dst + RT * FK, Bm, cols, d, col, k * FK);
    }
  };
  const int br = threadIdx.x >> 2, bq = threadIdx.x & 3;  // norms: 4 threads per row of B
  float bsum = 0.f;
  auto norm = [&](const float* Bs, int valid) {  // valid: depths of the chunk
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int pos = bq + 4 * h;
      const floatx4 v = *reinterpret_cast<const floatx4*>(Bs + br * FK + pos * 4);
      if ((pos ^ (br & 7)) * 4 < valid) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bsum = fmaf(v[e], v[e], bsum);
      }
    }
  };
  auto step = [&](floatx4(&acc)[MT][NT], const float* cur, int valid) {
    norm(cur + RT * FK, valid);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      HalfFrag<MT, NT> f;
      f.load(cur, cur + RT * FK, wr, wc, h);
      if (valid < FK) f.clip(h, valid);
      f.mma(acc);
    }
  };
  auto ready = [&]() {
    __builtin_amdgcn_s_waitcnt(0);  // this wave's requests for the chunk have landed
    __syncthreads();                // every wave's have, and every wave is done with the chunk before
  };
  const bool stream = nk % 2 == 0;
  fetch(buf0, c_begin, 0);
  for (int64_t col0 = c_begin; col0 < c_end; col0 += KNN_COLS) {
    floatx4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[m][n] = floatx4{0.f, 0.f, 0.f, 0.f};
    bsum = 0.f;
    for (int k = 0; k < nk; k += 2) {
      ready();
      if (k + 1 < nk) fetch(buf1, col0, k + 1);
      step(acc, buf0, d - k * FK);
      if (k + 1 >= nk) break;
      ready();
      if (stream || k + 2 < nk) fetch(buf0, col0, k + 2);
      step(acc, buf1, d - (k + 1) * FK);
    }
    bsum += __uint_as_float(lane_xor<1>(__float_as_uint(bsum)));
    bsum += __uint_as_float(lane_xor<2>(__float_as_uint(bsum)));
    if (bq == 0) bnorm[br] = bsum;
    __syncthreads();
    if (!stream) fetch(buf0, col0, nk);
    float bcol[NT];
    uint32_t pend = 0;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int cl = wc + n * 16 + (lane & 15);
      bcol[n] = bnorm[cl];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (col0 + cl < c_end && row0 + wr + m * 16 + 4 * (lane >> 4) + i < rows) pend |= 1u << ((m * 4 + i) * NT + n);
    }
    for (;;) {
      int over = 0;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int rl = wr + m * 16 + 4 * (lane >> 4) + i;
          const float t = thr[rl];
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const uint32_t bit = 1u << ((m * 4 + i) * NT + n);
            const float v = fmaxf(arow[m][i] + bcol[n] - 2.f * acc[m][n][i], 0.f);
            if ((pend & bit) && v <= t) {
              const int at = atomicAdd(&cnt[rl], 1);
              if (at < STG) {
                keys[(size_t)rl * LK + KNN_SHORT + at] = make_key(v, (uint32_t)(col0 + wc + n * 16 + (lane & 15)));
                pend &= ~bit;
              } else {
                over = 1;
              }
            } else {
              pend &= ~bit;  // above the threshold, which only falls
            }
          }
        }
      // every round with a full stage empties it, so the pending values shrink
      if (!__syncthreads_or(over)) break;
      flush_rows(STG, col0);
      __syncthreads();
    }
  }
  flush_rows(1, c_end);
  wave_sync();
  for (int j = 0; j < RT / NW; ++j) {
    const int r = wave + j * NW;
    const int64_t row = row0 + r;
    if (row < rows && lane < KNN_SHORT) part[((size_t)row * splits + split) * KNN_SHORT + lane] = keys[(size_t)r * LK + lane];
  }
}

// Pass 1 on tile_dot, grid (row tiles of 64, ranges): rows that allow no 16-byte loads, and
// the shapes that knn_rows leaves it.
__global__ __launch_bounds__(256) void knn_partial_kernel(const float* __restrict__ A, const float* __restrict__ an,
                                                          int64_t rows, const float* __restrict__ Bm,
                                                          const float* __restrict__ bn, int64_t cols, int d,
                                                          int64_t per_split, uint64_t* __restrict__ part, bool vec4) {
  __shared__ float tiles[2 * TM * LDT];  // As and Bs; then the 64 x 64 distance tile
  __shared__ uint64_t stage[4][16][64];
  float(*As)[LDT] = reinterpret_cast<float(*)[LDT]>(tiles);
  float(*Bs)[LDT] = reinterpret_cast<float(*)[LDT]>(tiles + TM * LDT);
  float(*Dt)[TN + 1] = reinterpret_cast<float(*)[TN + 1]>(tiles);
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * TM;
  const int64_t c_begin = (int64_t)blockIdx.y * per_split;
  const int64_t c_end = c_begin + per_split < cols ? c_begin + per_split : cols;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  WaveTop64 L[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) L[r].init(stage[wave][r], KNN_SHORT);
  for (int64_t col0 = c_begin; col0 < c_end; col0 += TN) {
    floatx4 acc[2][2];
    tile_dot(acc, As, Bs, A, rows, Bm, (int)(c_end < cols ? c_end : cols), d, row0, (int)col0, vec4);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int rl = wr + rt * 16 + 4 * (lane >> 4) + i;
          const int cl = wc + ct * 16 + (lane & 15);
          const int64_t row = row0 + rl, col = col0 + cl;
          Dt[rl][cl] = (row < rows && col < c_end) ? fmaxf(an[row] + bn[col] - 2.f * acc[rt][ct][i], 0.f)
                                                   : __builtin_inff();
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float v = Dt[16 * wave + r][lane];
      const int64_t col = col0 + lane;
      L[r].offer(make_key(v, (uint32_t)col), col < c_end);
    }
    __syncthreads();  // the next tile_dot overwrites the distance tile
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    L[r].finish();
    const int64_t row = row0 + 16 * wave + r;
    if (row < rows && lane < KNN_SHORT) part[((size_t)row * gridDim.y + blockIdx.y) * KNN_SHORT + lane] = L[r].best;
  }
}

// One wave per row: merge the splits' shortlists, exact re-score, top k.
__global__ __launch_bounds__(256) void knn_merge_kernel(const float* __restrict__ A, int64_t rows,
                                                        const float* __restrict__ Bm, int d, int splits,
                                                        const uint64_t* __restrict__ part, int k,
                                                        int32_t* __restrict__ ids, float* __restrict__ dist) {
  __shared__ uint64_t stage[4][64];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave;
  if (row >= rows) return;
  WaveTop64 L;
  L.init(stage[wave], KNN_SHORT);
  const uint64_t* src = part + (size_t)row * splits * KNN_SHORT;
  for (int e = lane; e - lane < splits * KNN_SHORT; e += HNTL_WAVE) {  // two lists at a time
    const uint64_t key = e < splits * KNN_SHORT ? src[e] : KEY_NONE;
    L.offer(key, key != KEY_NONE);
  }
  L.finish();
  const uint64_t mine = L.best;
  const float* a = A + row * d;
  uint64_t ex = KEY_NONE;
  const int have = __popcll(__ballot(lane < KNN_SHORT && mine != KEY_NONE));
  constexpr int RB = 8;  // shortlist entries re-scored together (their loads overlap)
  for (int j0 = 0; j0 < have; j0 += RB) {
    const float* bp[RB];
    uint32_t cs[RB];
    float acc[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      cs[u] = key_id(shfl_u64(mine, j0 + u < have ? j0 + u : j0));
      bp[u] = Bm + (size_t)cs[u] * d;
      acc[u] = 0.f;
    }
    for (int t = lane; t < d; t += HNTL_WAVE) {
      const float av = a[t];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const float df = av - bp[u][t];
        acc[u] = fmaf(df, df, acc[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const float tot = wave_sum(acc[u]);
      if (lane == j0 + u && lane < have) ex = make_key(tot, cs[u]);
    }
  }
  ex = wave_sort64(ex);
  if (lane < k) {
    ids[row * k + lane] = ex == KEY_NONE ? -1 : (int32_t)key_id(ex);
    if (dist) dist[row * k + lane] = ex == KEY_NONE ? __builtin_inff() : key_dist(ex);
  }
}

}  // namespace

void launch_row_norms(const float* A, int64_t rows, int d, float* out, hipStream_t s) {
  if (rows <= 0) return;
  hipLaunchKernelGGL(row_norms_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, A, rows, d, out);
  HIP_TRY(hipGetLastError());
}

void launch_dist_matrix(const float* A, const float* an, int64_t rows, const float* Bm, const float* bn, int cols,
                        int d, float* D, hipStream_t s, const int32_t* nlim, int64_t row_base) {
  if (rows <= 0 || cols <= 0) return;
  if (rows <= DIRECT_ROWS && d <= 16 * HNTL_WAVE) {
    hipLaunchKernelGGL(dist_direct_kernel, dim3((unsigned)((cols + 3) / 4)), dim3(256), 0, s, A, rows, Bm, cols, d, D,
                       nlim, row_base);
    HIP_TRY(hipGetLastError());
    return;
  }
  const bool vec4 = (d % 4) == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)Bm % 16) == 0;
  // below six chunks of depth a tile is mostly prologue and stores: tile_dot's
  // five workgroups a CU hide them better (10,000 x 1,024 x 128: 38.6 against 39.9 us)
  if (vec4 && d >= 6 * FK) {
    // 128 x 64 tiles once every CU gets eight of them (16,384 x 8,192 x 768:
    // 1.77 ms against 1.89 on 64 x 64), else 64 x 64 (10,000 x 1,024 x 768: 155
    // against 156 us; 3,001 x 1,024 x 768: 50 against 61; tile_dot: 158 and 54)
#define HNTL_DIST(RT, CT, WR, WC)                                                                                 \
  hipLaunchKernelGGL((dist_tile_kernel<RT, CT, WR, WC>),                                                          \
                     dim3((unsigned)((rows + RT - 1) / RT), (unsigned)((cols + CT - 1) / CT)), dim3(64 * WR * WC), \
                     0, s, A, an, rows, Bm, bn, cols, d, D, nlim, row_base)
    if ((rows + 127) / 128 * ((cols + 63) / 64) >= 2048)
      HNTL_DIST(128, 64, 4, 2);
    else
      HNTL_DIST(64, 64, 2, 2);
#undef HNTL_DIST
    HIP_TRY(hipGetLastError());
    return;
  }
  dim3 grid((unsigned)((rows + TM - 1) / TM), (unsigned)((cols + TN - 1) / TN));
  hipLaunchKernelGGL(dist_matrix_kernel, grid, dim3(256), 0, s, A, an, rows, Bm, bn, cols, d, D, vec4, nlim, row_base);
  HIP_TRY(hipGetLastError());
}

void launch_argmin_rows(const float* A, const float* an, int64_t rows, const float* Bm, const float* bn, int cols,
                        int d, int32_t* label, float* dmin, hipStream_t s) {
  if (rows <= 0) return;
  const bool vec4 = (d % 4) == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)Bm % 16) == 0;
  hipLaunchKernelGGL(argmin_rows_kernel, dim3((unsigned)((rows + TM - 1) / TM)), dim3(256), 0, s, A, an, rows, Bm,
                     bn, cols, d, label, dmin, vec4);
  HIP_TRY(hipGetLastError());
}

void launch_norm_max(const float* norms, int n, float* out, hipStream_t s) {
  hipLaunchKernelGGL(max_kernel, dim3(1), dim3(1024), 0, s, norms, n, out);
  HIP_TRY(hipGetLastError());
}

void launch_topk_rows(const float* D, int64_t rows, int cols, int P, int32_t* idx, float* val, hipStream_t s,
                      const float* A, const float* an, const float* Bm, const float* bn, const float* bmax, int d,
                      float err, const int32_t* nlim, int64_t row_base, unsigned int* overflow, float2* znorm) {
  if (A && (!an || !bn || !Bm || !bmax))
    throw ArgError{HNTL_EINVAL, "routing re-score needs both norm vectors, their bound and the centroids"};
  if (A && znorm) throw ArgError{HNTL_EINVAL, "the softmax normaliser is for score rows (no re-score)"};
  if (rows <= 0) return;
  if (P > HNTL_MAX_P) throw ArgError{HNTL_EUNSUPPORTED, "routing supports P <= 48"};
  // shortlist of a streamed row: the window of the P-th entry plus 48 more (one key per lane)
  const int M = A ? std::min(cols, std::min(64, P + 48)) : P;
  // float4 re-score loads where rows allow them
  const bool vec4 = A && (d % 4) == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)Bm % 16) == 0;
  dim3 grid((unsigned)((rows + TOPK_ROWS - 1) / TOPK_ROWS)), block(TOPK_ROWS * 64);
#define HNTL_TOPK(NCH)                                                                                             \
  hipLaunchKernelGGL(topk_rows_kernel<NCH>, grid, block, 0, s, D, rows, cols, P, M, A, an, Bm, bn, bmax, d, err, idx, \
                     val, nlim, row_base, overflow, znorm, vec4)
  // a row in registers up to 128 values a lane (162 VGPRs, three waves a SIMD;
  // longer rows are streamed: twice the registers would leave one)
  if (cols <= 1024)
    HNTL_TOPK(16);
  else if (cols <= 2048)
    HNTL_TOPK(32);
  else if (cols <= 4096)
    HNTL_TOPK(64);
  else if (cols <= 8192)
    HNTL_TOPK(128);
  else
    HNTL_TOPK(0);
#undef HNTL_TOPK
  HIP_TRY(hipGetLastError());
}

int pow2_at_least(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

}  // namespace hntl

namespace hntl {

namespace {

// Rows per tile of pass 1, 0: knn_partial_kernel.  Measured over 1 to 30,000 rows, 600 to
// 300,000 columns and 32 to 1,024 depths:
//  - 16 rows up to 4e9 products: a tile's first 128 columns all pass the empty lists, and 64
//    rows take 50 us to sort them in, 16 rows 5 (64 rows over 10,000 x 768: 270 and 185 us;
//    90 over 1,500 x 768: 130 us, 843 on 64 rows in ranges of eight tiles and more);
//  - 128 rows run 4% faster than twice 64 at 256 depths or more, where the padding to them
//    is no more (1,024 rows over 1,000,000 x 768: 13.9 against 14.5 ms; 300 rows 5.9 against 5.2;
//    at 64 depths the lists bound them: 5,000 over 100,000 x 64 1,465 against 1,331 us);
//  - from 448 rows of 384 depths on, up to 2,800 of its 64 x 64 tiles, knn_partial_kernel's
//    smaller workgroups fill the GPU in one round (1,500 over 5,000 x 1,024: 406 against 477 us,
//    5,000 over 1,000 x 768: 257 against 303).
int knn_rows(int64_t rows, int64_t cols, int d, bool vec4) {
  if (!vec4) return 0;
  auto tiles = [](int64_t n, int64_t t) { return (n + t - 1) / t; };
  const int64_t t64 = tiles(rows, 64) * tiles(cols, 64);
  if (d >= 384 && rows >= 448 && t64 >= 256 && t64 <= 2800) return 0;
  if (rows <= 16 || (double)rows * (double)cols * d <= 4e9) return 16;
  return d >= 256 && 100 * 128 * tiles(rows, 128) <= 103 * 64 * tiles(rows, 64) ? 128 : 64;
}

// Column ranges for rt row tiles of RT rows over `tiles` column tiles of nk depth chunks.  Each
// range starts with empty lists, which costs as much as `lists` chunks and a share of it
// again with the logarithm of its length (the values that still pass get fewer), and adds a
// list per row to merge; the rounds of workgroups should be full.  A workgroup alone on
// its CU takes 0.8 of the time of two that share it.
int64_t knn_ranges(int RT, int64_t rt, int64_t tiles, int nk) {
  const int64_t slots = RT == 128 ? 256 : 512;  // workgroups at once
  const double lists = RT == 16 ? 8.0 : 20.0;
  int64_t best = 1;
  double least = 0.0;
  for (int64_t sp = 1; sp <= tiles && (sp == 1 || rt * sp <= 4 * slots); sp += sp < 16 ? 1 : 8) {
    const int64_t len = (tiles + sp - 1) / sp;
    const int64_t wg = rt * (sp < 8 ? sp : (sp + 7) / 8 * 8);  // (from 8 on each XCD takes every eighth range)
    const double rounds = RT < 128 && wg <= 256 ? 0.8 : (double)((wg + slots - 1) / slots);
    const double cost = rounds * ((double)len * nk + lists * (1.0 + std::log((double)len))) + 0.1 * (double)sp;
    if (sp == 1 || cost < least) {
      least = cost;
      best = sp;
    }
  }
  return best;
}

}  // namespace

void launch_knn(const float* A, int64_t rows, const float* Bm, int64_t cols, int d, int k, int32_t* ids, float* dist,
                hipStream_t s) {
  if (rows <= 0) return;
  if (k < 1 || k > 16) throw ArgError{HNTL_EUNSUPPORTED, "brute-force kNN supports 1 <= k <= 16"};
  if (cols >= (1ll << 31)) throw ArgError{HNTL_EUNSUPPORTED, "brute-force kNN needs fewer than 2^31 rows"};
  float *an = nullptr, *bn = nullptr;
  uint64_t* part = nullptr;
  int64_t per;
  HIP_TRY(hipMallocAsync((void**)&an, sizeof(float) * rows, s));
  launch_row_norms(A, rows, d, an, s);
  const bool vec4 = (d % 4) == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)Bm % 16) == 0;
  const int RT = knn_rows(rows, cols, d, vec4);
  int64_t splits = 1;
  if (RT) {
    const int64_t rt = (rows + RT - 1) / RT;
    splits = knn_ranges(RT, rt, (cols + KNN_COLS - 1) / KNN_COLS, (d + FK - 1) / FK);
    per = ((cols + splits - 1) / splits + KNN_COLS - 1) / KNN_COLS * KNN_COLS;
    splits = (cols + per - 1) / per;
    HIP_TRY(hipMallocAsync((void**)&part, sizeof(uint64_t) * rows * splits * KNN_SHORT, s));
    const int64_t grid = rt * (splits >= 8 ? (splits + 7) / 8 * 8 : splits);
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * KNN_WAVES), 0, s, A, an, rows, Bm, cols, d, per,
                         (int)splits, (int)rt, part);
    };
    if (RT == 16)
      launch(knn_tile_kernel<16, 1, 8>);
    else if (RT == 64)
      launch(knn_tile_kernel<64, 2, 4>);
    else
      launch(knn_tile_kernel<128, 4, 2>);
  } else {
    const int64_t rt = (rows + TM - 1) / TM;
    splits = std::max<int64_t>(1, std::min<int64_t>((cols + TN - 1) / TN, 2048 / rt));
    per = ((cols + splits - 1) / splits + TN - 1) / TN * TN;
    splits = (cols + per - 1) / per;
    HIP_TRY(hipMallocAsync((void**)&bn, sizeof(float) * cols, s));
    HIP_TRY(hipMallocAsync((void**)&part, sizeof(uint64_t) * rows * splits * KNN_SHORT, s));
    launch_row_norms(Bm, cols, d, bn, s);
    hipLaunchKernelGGL(knn_partial_kernel, dim3((unsigned)rt, (unsigned)splits), dim3(256), 0, s, A, an, rows, Bm, bn,
                       cols, d, per, part, vec4);
  }
  HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(knn_merge_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, A, rows, Bm, d,
                     (int)splits, part, k, ids, dist);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipFreeAsync(an, s));
  if (bn) HIP_TRY(hipFreeAsync(bn, s));
  HIP_TRY(hipFreeAsync(part, s));
}

}  // namespace hntl
