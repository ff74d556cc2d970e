// NABF building blocks on the GPU (paper Sec. 4.1 "Null-space-Aware Binary
// Factorization", Algorithm nabf in App. A.1, App. A.1.4 "ADMM-SVID Framework
// in DBF", App. A.2.2-A.2.5).  Offline calibration math for one linear:
//
//   surrogate      W' = o . W . i^T with i, o the RMS of calibration inputs
//                  and output gradients
//   SVID           signs of Z and a rank-1 fit |Z| ~ a v^T (power iteration)
//   null space     P = U_hat U_hat^T from the trailing eigenvectors of a PSD
//                  C that carry at most eta of its spectral energy
//   ADMM proxies   A_hat = (W' B^T + rho (A - U)) (B B^T + rho I)^-1 and
//                  B_hat = (A^T A + rho I)^-1 (A^T W' + rho (B - U))
//   scale fits     gamma, eta of the null-space-compensated targets
//   iteration      one pass of the NABF loop over both factors
//
// Dense matrices are fp32 row-major.  Plain matrix products go to rocBLAS,
// the Cholesky and symmetric eigen factorisations to rocSOLVER (the
// eigenproblem in fp64: the cutoff compares sums of eigenvalues); every
// other step -- the power iteration, the sign packing, the energy cutoff,
// the compensation and scale fits, the factor rebuilds and dual updates,
// the surrogate statistics -- is a kernel here.  Reductions take partial
// sums per tile and add them in a fixed order, so results repeat bit for
// bit.
#include <math.h>
#include <mutex>
#include <type_traits>

#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include "af1_device.h"
#include "af1_internal.h"
#include "af1_nabf.h"

namespace af1n {
namespace {

using af1::bf16_to_f32;
using af1::f32_to_f16;
using af1::wave_sum;

constexpr double kEps = 1e-12;   // residual-energy fraction and scale fits
constexpr int kChunkLog2 = 6;
constexpr int kChunk = 1 << kChunkLog2;  // rows per partial-sum tile

// ---------------------------------------------------------------------------
// Device kernels
// ---------------------------------------------------------------------------

// Sum of v over the 64 lanes, in every lane (fixed order): four DPP steps
// within rows of 16, then the four rows.  Register moves only; the shuffles
// of wave_sum go through LDS, six dependent round trips.
template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v += dpp_f32<0xB1>(v);
  v += dpp_f32<0x4E>(v);
  v += dpp_f32<0x124>(v);
  v += dpp_f32<0x128>(v);
  const int b = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(b, 0)) +
          __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(b, 32)) +
          __int_as_float(__builtin_amdgcn_readlane(b, 48)));
}

// Sums of squares per 64-token tile of X (T x n) and G (T x m), bf16, in one
// launch: part[tile][j].  A workgroup takes 256 columns of one matrix: 32
// threads of 8 columns (16-byte loads) by 8 groups of 8 tokens, all of a
// thread's loads in flight at once (rows past T load row T - 1 and add
// nothing), the groups added in order through LDS.  Bound by memory latency:
// one 2-byte load a thread and token, each waited for in turn, took 17.4 us
// per matrix at 2048 x 4096 (16.8 MB); both together now take 7.1.
constexpr int kColsqGroups = 8;
__global__ __launch_bounds__(256) void colsq_kernel(const uint16_t *__restrict__ X, int n,
                                                    float *__restrict__ px, int xblocks,
                                                    const uint16_t *__restrict__ G, int m,
                                                    float *__restrict__ pg, int T) {
  __shared__ float red[kColsqGroups][256 + 8];
  const bool first = (int)blockIdx.x < xblocks;  // uniform
  const uint16_t *src = first ? X : G;
  const int cols = first ? n : m;
  const int c0 = 256 * ((int)blockIdx.x - (first ? 0 : xblocks));
  const int cx = threadIdx.x & 31, tg = threadIdx.x >> 5;
  const int c = c0 + 8 * cx;
  const int cl = c < cols ? c : 0;
  const int t0 = (int)blockIdx.y * kChunk + tg * (kChunk / kColsqGroups);
  uint4 v[kChunk / kColsqGroups];
#pragma unroll
  for (int q = 0; q < kChunk / kColsqGroups; ++q)
    v[q] = *reinterpret_cast<const uint4 *>(src + (size_t)min(t0 + q, T - 1) * cols + cl);
  float s[8] = {};
#pragma unroll
  for (int q = 0; q < kChunk / kColsqGroups; ++q) {
    const uint32_t d[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
    const bool use = t0 + q < T;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = __uint_as_float(d[e] << 16), b = __uint_as_float(d[e] & 0xffff0000u);
      s[2 * e] += use ? a * a : 0.f;
      s[2 * e + 1] += use ? b * b : 0.f;
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[tg][8 * cx + e] = s[e];
  __syncthreads();
  const int j = c0 + (int)threadIdx.x;
  if (j < cols) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kColsqGroups; ++k) t += red[k][threadIdx.x];
    (first ? px : pg)[(size_t)blockIdx.y * cols + j] = t;
  }
}

__device__ __forceinline__ float4 add4(const float4 &a, const float4 &b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float add4(float a, float b) { return a + b; }

// A sum of up to 16 terms, pushed in order, in pairs, pairs of pairs and so on;
// terms that are not pushed count as zeros.  Whoever adds up aligned runs of
// 1, 2, 4 or 8 of the terms first gets the same bits.
template <typename V>
struct TreeSum {
  V level[4];
  int count = 0;  // uniform
  __device__ __forceinline__ void push(V v) {
    bool held = false;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      if (held) continue;
      if (count >> l & 1) {
        v = add4(level[l], v);
      } else {
        level[l] = v;
        held = true;
      }
    }
    if (!held) total = v;  // the sixteenth term
    ++count;
  }
  __device__ __forceinline__ V sum(V zero) const {
    V v = count >> 4 ? total : zero;
#pragma unroll
    for (int l = 0; l < 4; ++l)
      if (count >> l & 1) v = add4(level[l], v);
    return v;
  }
  V total;
};

// Column sums of partial rows: out[j] = sum over the chunks of
// part[chunk][j], for up to two matrices in one launch (blocks below `split`
// take the first).  A chunk is 1 << kSubLog2 (at most 16) consecutive rows of
// part (the last one may have fewer of the `rows`), added up in pairs, pairs of
// pairs and so on (TreeSum), so that the result does not depend on how finely
// the chunks were split.  A workgroup takes
// 64 columns: 16 float4 columns by 16 chunk groups (group g adds chunks g, g +
// 16, ..., eight rows' loads or a chunk's in flight), the groups added in order through
// LDS.  kRms: out = sqrt(sum / T), the surrogate's column RMS.  One thread a
// column, each chunk waited for in turn, took 16 us at 64 rows x 2016 columns;
// 512 rows now take 4.3.
constexpr int kSumCols = 64;
struct ColSum {
  const float *part;
  float *out;
  int rows, cols;
};
template <bool kRms, int kSubLog2>
__global__ __launch_bounds__(256) void colsum_kernel(ColSum a, ColSum b, int split, int T) {
  __shared__ float4 red[16][17];
  const bool first = (int)blockIdx.x < split;  // uniform
  const ColSum p = first ? a : b;
  const int c4 = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int j = kSumCols * ((int)blockIdx.x - (first ? 0 : split)) + 4 * c4;
  const int jl = j < p.cols ? j : 0;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  constexpr int kSub = 1 << kSubLog2, kLoads = kSub > 8 ? kSub : 8;
  const int chunks = (p.rows + kSub - 1) / kSub;
  for (int c0 = g; c0 < chunks; c0 += 16 * (kLoads / kSub)) {
    float4 v[kLoads];
    // load q: a row of chunk c0 + 16 (q / kSub)
    auto row = [&](int q) { return (c0 + 16 * (q / kSub)) * kSub + q % kSub; };
#pragma unroll
    for (int q = 0; q < kLoads; ++q)
      v[q] = *reinterpret_cast<const float4 *>(p.part + (size_t)min(row(q), p.rows - 1) * p.cols +
                                               jl);
#pragma unroll
    for (int q = 0; q < kLoads; ++q)
      if (row(q) >= p.rows) v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int l = 1; l <= kSubLog2; ++l)
#pragma unroll
      for (int q = 0; q < kLoads >> l; ++q) v[q] = add4(v[2 * q], v[2 * q + 1]);
#pragma unroll
    for (int q = 0; q < kLoads / kSub; ++q) s = add4(s, v[q]);
  }
  red[g][c4] = s;
  __syncthreads();
  if (g == 0 && j < p.cols) {
    float4 t = red[0][c4];
#pragma unroll
    for (int k = 1; k < 16; ++k) {
      const float4 r = red[k][c4];
      t.x += r.x;
      t.y += r.y;
      t.z += r.z;
      t.w += r.w;
    }
    if constexpr (kRms) {
      const float f = (float)T;
      t = make_float4(sqrtf(t.x / f), sqrtf(t.y / f), sqrtf(t.z / f), sqrtf(t.w / f));
    }
    *reinterpret_cast<float4 *>(p.out + j) = t;
  }
}

// Wp[u][j] = o[u] * W[u][j] * i[j], a float4 a thread (cols % 32 == 0): 20.2
// us at 4096^2 (134 MB, 6.6 TB/s) against 28.8 with one float a thread.
__global__ __launch_bounds__(256) void surrogate_scale_kernel(const float *__restrict__ W, int64_t m,
                                                              int n, const float *__restrict__ o,
                                                              const float *__restrict__ iv,
                                                              float *__restrict__ Wp) {
  const int j = 4 * ((int)blockIdx.x * 256 + (int)threadIdx.x);
  if (j >= n) return;
  const float4 ij = *reinterpret_cast<const float4 *>(iv + j);
  for (int64_t u = blockIdx.y; u < m; u += gridDim.y) {
    const float4 v = *reinterpret_cast<const float4 *>(W + u * n + j);
    const float ou = o[u];
    *reinterpret_cast<float4 *>(Wp + u * n + j) =
        make_float4(ou * v.x * ij.x, ou * v.y * ij.y, ou * v.z * ij.z, ou * v.w * ij.w);
  }
}

__global__ __launch_bounds__(256) void fill_kernel(float *__restrict__ v, int n, float val) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j < n) v[j] = val;
}

// u[i] = sum_j |Z[i][j]| v[j]: one wave per row, 16-byte loads (cols % 32 == 0).
__global__ __launch_bounds__(256) void abs_rowdot_kernel(const float *__restrict__ Z, int64_t rows,
                                                         int cols, const float *__restrict__ v,
                                                         float *__restrict__ u) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= rows) return;
  const float4 *zr = reinterpret_cast<const float4 *>(Z + i * cols);
  const float4 *v4 = reinterpret_cast<const float4 *>(v);
  float s = 0.f;
  for (int q = lane; q < cols / 4; q += 64) {
    const float4 z = zr[q], w = v4[q];
    s += fabsf(z.x) * w.x + fabsf(z.y) * w.y + fabsf(z.z) * w.z + fabsf(z.w) * w.w;
  }
  s = wave_sum(s);
  if (lane == 0) u[i] = s;
}

// One power-iteration pass of the SVID, Z read once (kPass).  A workgroup takes
// a block of rows: for each row u = |Z_i| v (a reduction over the workgroup),
// then w += |Z_i| u from the same registers, and the block's w goes to
// part[block].  colsum_kernel adds the blocks.  A thread holds kQ float4 of
// every row (columns 4 (tid + threads q) ..), so kQ * threads * 4 >= cols;
// kR rows are reduced together (one barrier), the next kR rows loading
// meanwhile.
//
// v is the normalised w of the pass before, recomputed by every workgroup
// (each thread needs its own columns of it anyway): v = w / ||w||, kept from
// the pass before (`right`) when w is zero; w == nullptr: the constant v0.
// Workgroup 0 stores v to `right`; where the others read `right` (w zero),
// it stores the values that are there.
//
// kRowDot: left = u = |Z| v instead of w.  kLast: that, the final left, and the
// signs of Z packed as af1_pack does (eight lanes' sign nibbles make a word).
// The sums are written as fmaf, so that every mode rounds them alike.
//
// Bound by the read of Z, which the last-level cache holds between passes at
// calibration sizes.  Separate row and column passes with a finishing and a
// normalising launch read Z twice: 43.7 us a pass at 4096 x 2016 (33 MB);
// this pass takes 6.9 us there and the column sums 4.3 (kernel trace).
//
// kPassTree: kPass whose workgroups take several runs of sub_rows rows, each
// summed by itself and then as TreeSum does (the scratch has no row of part for
// every run).
constexpr int kPass = 0, kRowDot = 1, kLast = 2, kPassTree = 3;
template <int kQ, int kR, int kThreads, int kMode>
__global__ __launch_bounds__(kThreads) void svid_pass_kernel(
    const float *__restrict__ Z, int rows, int cols, int rows_wg, int sub_rows,
    const float *__restrict__ w, float v0, float *right, float *__restrict__ part,
    float *__restrict__ left, uint32_t *__restrict__ bits) {
  constexpr int kWaves = kThreads / 64;
  __shared__ float red[2][kR][kWaves];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int nf = cols / 4;  // float4 of a row
  bool live[kQ];
  int col[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    live[q] = tid + kThreads * q < nf;
    col[q] = live[q] ? 4 * (tid + kThreads * q) : 0;  // loads stay inside the arrays
  }
  const int i0 = (int)blockIdx.x * rows_wg;
  const int i1 = min(rows, i0 + rows_wg);
  auto load = [&](float4 (&z)[kR][kQ], int i) {
#pragma unroll
    for (int r = 0; r < kR; ++r)
#pragma unroll
      for (int q = 0; q < kQ; ++q)
        z[r][q] = *reinterpret_cast<const float4 *>(Z + (size_t)min(i + r, i1 - 1) * cols + col[q]);
  };
  float4 za[kR][kQ], zb[kR][kQ];
  load(za, i0);

  // v
  float4 v[kQ];
  if (w) {
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      v[q] = *reinterpret_cast<const float4 *>(w + col[q]);
      const float t = fmaf(v[q].w, v[q].w, fmaf(v[q].z, v[q].z,
                           fmaf(v[q].y, v[q].y, v[q].x * v[q].x)));
      s += live[q] ? t : 0.f;
    }
    s = wave_sum_dpp(s);
    if ((tid & 63) == 0) red[1][0][wave] = s;
    __syncthreads();
    s = red[1][0][0];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) s += red[1][0][k];
    const float norm = sqrtf(s);
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      if (s > 0.f)
        v[q] = make_float4(v[q].x / norm, v[q].y / norm, v[q].z / norm, v[q].w / norm);
      else
        v[q] = *reinterpret_cast<const float4 *>(right + col[q]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < kQ; ++q) v[q] = make_float4(v0, v0, v0, v0);
  }
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if (blockIdx.x == 0 && live[q]) *reinterpret_cast<float4 *>(right + col[q]) = v[q];
    if (!live[q]) v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }

  float4 acc[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  TreeSum<float4> tree[kMode == kPassTree ? kQ : 1];
  // rows i .. i + kR - 1 (in z); the red buffers alternate, so one barrier a
  // batch is enough
  auto batch = [&](const float4 (&z)[kR][kQ], int i, int buf) {
    float u[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        const float4 f = z[r][q];
        const float t = fmaf(fabsf(f.w), v[q].w, fmaf(fabsf(f.z), v[q].z,
                             fmaf(fabsf(f.y), v[q].y, fabsf(f.x) * v[q].x)));
        s += live[q] ? t : 0.f;
      }
      u[r] = wave_sum_dpp(s);
    }
    if ((tid & 63) == 0) {
#pragma unroll
      for (int r = 0; r < kR; ++r) red[buf][r][wave] = u[r];
    }
    // LDS only: the next batch's loads stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      float t = red[buf][r][0];
#pragma unroll
      for (int k = 1; k < kWaves; ++k) t += red[buf][r][k];
      const bool use = i + r < i1;  // uniform
      if constexpr (kMode == kRowDot || kMode == kLast) {
        if (use && tid == 0) left[i + r] = t;
#pragma unroll
        for (int q = 0; q < (kMode == kLast ? kQ : 0); ++q) {
          const float4 f = z[r][q];
          uint32_t n = (__float_as_uint(f.x) >> 31) | (__float_as_uint(f.y) >> 31) << 1 |
                       (__float_as_uint(f.z) >> 31) << 2 | (__float_as_uint(f.w) >> 31) << 3;
          n <<= 4 * (tid & 7);
          n |= __shfl_xor(n, 1, 8);
          n |= __shfl_xor(n, 2, 8);
          n |= __shfl_xor(n, 4, 8);
          if (use && live[q] && (tid & 7) == 0)
            bits[(size_t)(i + r) * (cols / 32) + col[q] / 32] = n;
        }
      } else {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          // a row past the block adds nothing (its data is another row's)
          acc[q].x = use ? fmaf(fabsf(z[r][q].x), t, acc[q].x) : acc[q].x;
          acc[q].y = use ? fmaf(fabsf(z[r][q].y), t, acc[q].y) : acc[q].y;
          acc[q].z = use ? fmaf(fabsf(z[r][q].z), t, acc[q].z) : acc[q].z;
          acc[q].w = use ? fmaf(fabsf(z[r][q].w), t, acc[q].w) : acc[q].w;
        }
      }
    }
    if constexpr (kMode == kPassTree) {
      if ((i + kR - i0) % sub_rows == 0 || i + kR >= i1) {  // a run ends (sub_rows % kR == 0)
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          tree[q].push(acc[q]);
          acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
    }
  };
  for (int i = i0; i < i1; i += 2 * kR) {
    load(zb, min(i + kR, i1 - 1));
    batch(za, i, 0);
    if (i + kR >= i1) break;
    load(za, min(i + 2 * kR, i1 - 1));
    batch(zb, i + kR, 1);
  }
  if constexpr (kMode == kPass || kMode == kPassTree) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      if constexpr (kMode == kPassTree) acc[q] = tree[q].sum(make_float4(0.f, 0.f, 0.f, 0.f));
      if (live[q])
        *reinterpret_cast<float4 *>(part + (size_t)blockIdx.x * cols + col[q]) = acc[q];
    }
  }
}

// part[chunk][j] = sum over the chunk's rows i of |Z[i][j]| u[i]; every run of
// sub_rows rows (4 to 64) is added up by itself first, the runs as TreeSum does.
// Sixteen rows' loads in flight (rows % 32 == 0).
__global__ __launch_bounds__(256) void abs_coldot_kernel(const float *__restrict__ Z, int64_t rows,
                                                         int cols, const float *__restrict__ u,
                                                         float *__restrict__ part, int sub_rows) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= cols) return;
  const int64_t i0 = (int64_t)blockIdx.y * kChunk;
  const int64_t i1 = min(rows, i0 + kChunk);
  TreeSum<float> s;
  float t = 0.f;
  for (int64_t k0 = i0; k0 < i1; k0 += 16) {
    float z[16], uu[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      z[q] = Z[(k0 + q) * cols + j];
      uu[q] = u[k0 + q];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      t = fmaf(fabsf(z[q]), uu[q], t);
      const int done = (int)(k0 - i0) + q + 1;  // uniform
      if (q % 4 == 3 && (done % sub_rows == 0 || k0 + q + 1 == i1)) {
        s.push(t);
        t = 0.f;
      }
    }
  }
  part[(size_t)blockIdx.y * cols + j] = s.sum(0.f);
}

// w[j] = sum over chunks of part[chunk][j] (in order); sq[block] = the
// block's sum of w^2 (lane order, then wave order).
__global__ __launch_bounds__(256) void coldot_finish_kernel(const float *__restrict__ part,
                                                            int chunks, int cols,
                                                            float *__restrict__ w,
                                                            float *__restrict__ sq) {
  __shared__ float red[4];
  const int j = blockIdx.x * 256 + threadIdx.x;
  float s = 0.f;
  if (j < cols) {
    for (int c = 0; c < chunks; ++c) s += part[(size_t)c * cols + j];
    w[j] = s;
  }
  const float q = wave_sum(s * s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = q;
  __syncthreads();
  if (threadIdx.x == 0) sq[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// v = w / ||w|| (||w||^2 = the block partials added in order); v is kept
// when w is zero.
__global__ __launch_bounds__(256) void normalize_kernel(const float *__restrict__ w,
                                                        const float *__restrict__ sq, int nsq,
                                                        int cols, float *__restrict__ v) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= cols) return;
  float s = 0.f;
  for (int k = 0; k < nsq; ++k) s += sq[k];
  if (s > 0.f) v[j] = w[j] / sqrtf(s);
}

__global__ __launch_bounds__(256) void to_f64_kernel(const float *__restrict__ s,
                                                     double *__restrict__ d, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
    d[k] = (double)s[k];
}

__global__ __launch_bounds__(256) void to_f32_kernel(const double *__restrict__ s,
                                                     float *__restrict__ d, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
    d[k] = (float)s[k];
}

// Residual-energy cutoff (App. A.2.3) on the ascending eigenvalues D of a
// PSD matrix.  With lambda in descending order, rho_k is the sum of the
// r - k smallest eigenvalues over (total + eps); the first k (from 0 up)
// with rho_k <= eta is the largest count c = r - k of smallest eigenvalues
// whose sum stays within eta (total + eps).  One thread, in fp64.
__global__ void cutoff_kernel(const double *__restrict__ D, int r, double eta, double eps,
                              double *__restrict__ pre, int *__restrict__ count,
                              int *__restrict__ k_out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0;
  pre[0] = 0.0;
  for (int c = 0; c < r; ++c) {
    s += D[c];
    pre[c + 1] = s;
  }
  const double thr = eta * (s + eps);
  int c = 0;
  for (int cc = r; cc >= 0; --cc)
    if (pre[cc] <= thr) {
      c = cc;
      break;
    }
  *count = c;
  if (k_out) *k_out = r - c;
}

// Zero the eigenvector columns past the selected count (column-major U).
__global__ __launch_bounds__(256) void mask_columns_kernel(double *__restrict__ U, int r,
                                                           const int *__restrict__ count) {
  const int c = *count;
  const int64_t n = (int64_t)r * r;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
    if (k / r >= c) U[k] = 0.0;
}

// G = C + rho I (copy), both r x r.
__global__ __launch_bounds__(256) void shift_copy_kernel(const float *__restrict__ C,
                                                         float *__restrict__ G, int r, float rho) {
  const int64_t n = (int64_t)r * r;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
    G[k] = C[k] + ((k / r == k % r) ? rho : 0.f);
}

// out = alpha (x - y) or x + y, elementwise.
__global__ __launch_bounds__(256) void scaled_diff_kernel(const float *__restrict__ x,
                                                          const float *__restrict__ y, float alpha,
                                                          float *__restrict__ out, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
    out[k] = alpha * (x[k] - y[k]);
}
__global__ __launch_bounds__(256) void add_kernel(const float *__restrict__ x,
                                                  const float *__restrict__ y,
                                                  float *__restrict__ out, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
    out[k] = x[k] + y[k];
}

// The binary-scaled matrix left . S . right^T at (i, j); bit 1 is -1.
__device__ __forceinline__ float bscaled(const uint32_t *__restrict__ bits,
                                         const float *__restrict__ left,
                                         const float *__restrict__ right, int64_t i, int j,
                                         int cols) {
  const uint32_t word = bits[i * (cols / 32) + (j >> 5)];
  const float v = left[i] * right[j];
  return ((word >> (j & 31)) & 1u) ? -v : v;
}

// E = hat - (left . S . right^T).
__global__ __launch_bounds__(256) void residual_kernel(const float *__restrict__ hat,
                                                       const uint32_t *__restrict__ bits,
                                                       const float *__restrict__ left,
                                                       const float *__restrict__ right,
                                                       int64_t rows, int cols,
                                                       float *__restrict__ E) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= cols) return;
  for (int64_t i = blockIdx.y; i < rows; i += gridDim.y)
    E[i * cols + j] = hat[i * cols + j] - bscaled(bits, left, right, i, j, cols);
}

// dense = left . S . right^T, and U += hat - dense (when U is given).
__global__ __launch_bounds__(256) void rebuild_kernel(const uint32_t *__restrict__ bits,
                                                      const float *__restrict__ left,
                                                      const float *__restrict__ right,
                                                      int64_t rows, int cols,
                                                      const float *__restrict__ hat,
                                                      float *__restrict__ dense,
                                                      float *__restrict__ U) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= cols) return;
  for (int64_t i = blockIdx.y; i < rows; i += gridDim.y) {
    const float q = bscaled(bits, left, right, i, j, cols);
    dense[i * cols + j] = q;
    if (U) U[i * cols + j] += hat[i * cols + j] - q;
  }
}

// Column fit partials: num = sum_i q (hat - HP), den = sum_i q^2 over a chunk
// of rows, q the binary-scaled entry.
__global__ __launch_bounds__(256) void colfit_kernel(const float *__restrict__ hat,
                                                     const float *__restrict__ HP,
                                                     const uint32_t *__restrict__ bits,
                                                     const float *__restrict__ left,
                                                     const float *__restrict__ right, int64_t rows,
                                                     int cols, float *__restrict__ pnum,
                                                     float *__restrict__ pden) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= cols) return;
  const int64_t i0 = (int64_t)blockIdx.y * kChunk;
  const int64_t i1 = min(rows, i0 + kChunk);
  float num = 0.f, den = 0.f;
  for (int64_t i = i0; i < i1; ++i) {
    const float q = bscaled(bits, left, right, i, j, cols);
    num += q * (hat[i * cols + j] - HP[i * cols + j]);
    den += q * q;
  }
  pnum[(size_t)blockIdx.y * cols + j] = num;
  pden[(size_t)blockIdx.y * cols + j] = den;
}

__global__ __launch_bounds__(256) void colfit_finish_kernel(const float *__restrict__ pnum,
                                                            const float *__restrict__ pden,
                                                            int chunks, int cols, float eps,
                                                            float *__restrict__ fit) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= cols) return;
  float num = 0.f, den = 0.f;
  for (int c = 0; c < chunks; ++c) {
    num += pnum[(size_t)c * cols + j];
    den += pden[(size_t)c * cols + j];
  }
  fit[j] = num / (den + eps);
}

// Row fit: one block per row k, fit[k] = sum_j q (hat - HP) / (sum_j q^2 + eps).
__global__ __launch_bounds__(256) void rowfit_kernel(const float *__restrict__ hat,
                                                     const float *__restrict__ HP,
                                                     const uint32_t *__restrict__ bits,
                                                     const float *__restrict__ left,
                                                     const float *__restrict__ right, int cols,
                                                     float eps, float *__restrict__ fit) {
  __shared__ float rn[4], rd[4];
  const int64_t k = blockIdx.x;
  float num = 0.f, den = 0.f;
  for (int j = threadIdx.x; j < cols; j += 256) {
    const float q = bscaled(bits, left, right, k, j, cols);
    num += q * (hat[k * cols + j] - HP[k * cols + j]);
    den += q * q;
  }
  num = wave_sum(num);
  den = wave_sum(den);
  if ((threadIdx.x & 63) == 0) {
    rn[threadIdx.x >> 6] = num;
    rd[threadIdx.x >> 6] = den;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    fit[k] = (((rn[0] + rn[1]) + rn[2]) + rn[3]) / ((((rd[0] + rd[1]) + rd[2]) + rd[3]) + eps);
}

// X[i + j * ld] /= (D[j or i] + rho): dim 0 scales the rows of a
// column-major block (index i), dim 1 its columns (index j).
__global__ __launch_bounds__(256) void inv_shift_scale_kernel(float *__restrict__ X, int64_t rows,
                                                              int64_t cols,
                                                              const double *__restrict__ D,
                                                              float rho, int dim) {
  const int64_t n = rows * cols;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) {
    const int64_t e = dim == 0 ? k % rows : k / rows;
    X[k] = (float)((double)X[k] / (D[e] + (double)rho));
  }
}

__global__ __launch_bounds__(256) void mul_kernel(float *__restrict__ x, const float *__restrict__ y,
                                                  int n) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j < n) x[j] *= y[j];
}

// Deployable scales: s_out = a / o, s_mid = m1 . m2, s_in = b / i (binary16,
// round to nearest even).
__global__ __launch_bounds__(256) void export_kernel(const float *__restrict__ a,
                                                     const float *__restrict__ m1,
                                                     const float *__restrict__ m2,
                                                     const float *__restrict__ b,
                                                     const float *__restrict__ iv,
                                                     const float *__restrict__ o, int m, int n,
                                                     int r, uint16_t *__restrict__ s_out,
                                                     uint16_t *__restrict__ s_mid,
                                                     uint16_t *__restrict__ s_in) {
  int k = blockIdx.x * 256 + threadIdx.x;
  if (k < m) {
    s_out[k] = f32_to_f16(o ? a[k] / o[k] : a[k]);
    return;
  }
  k -= m;
  if (k < r) {
    s_mid[k] = f32_to_f16(m1[k] * m2[k]);
    return;
  }
  k -= r;
  if (k < n) s_in[k] = f32_to_f16(iv ? b[k] / iv[k] : b[k]);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }
unsigned grid_cap(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}
unsigned rows_grid(int64_t rows) { return (unsigned)(rows < 65535 ? rows : 65535); }
int64_t chunks_of(int64_t rows) { return (rows + kChunk - 1) / kChunk; }
size_t al(size_t v) { return (v + 255) & ~(size_t)255; }

// One rocBLAS handle per device, created on first use.  The mutex is held
// for a whole entry point call, so concurrent calls on one device take turns
// setting the handle's stream.
struct DeviceHandle {
  std::mutex mu;
  rocblas_handle h = nullptr;
};
DeviceHandle g_handles[64];

struct Handle {
  std::unique_lock<std::mutex> lock;
  rocblas_handle h = nullptr;
  bool ok = false;
  explicit Handle(hipStream_t s) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
    lock = std::unique_lock<std::mutex>(g_handles[dev].mu);
    if (!g_handles[dev].h && rocblas_create_handle(&g_handles[dev].h) != rocblas_status_success) {
      g_handles[dev].h = nullptr;
      return;
    }
    h = g_handles[dev].h;
    ok = rocblas_set_stream(h, s) == rocblas_status_success;
  }
};

#define CHECK_HIP(x)                              \
  do {                                            \
    if ((x) != hipSuccess) return AF1_ERR_HIP;    \
  } while (0)
#define CHECK_LAUNCH() CHECK_HIP(hipGetLastError())
#define CHECK_RB(x)                                          \
  do {                                                       \
    if ((x) != rocblas_status_success) return AF1_ERR_HIP;   \
  } while (0)

const rocblas_operation kN = rocblas_operation_none, kT = rocblas_operation_transpose;

// C (m x n, column-major, ldc) = alpha op(A) op(B) + beta C.
af1_status sgemm(rocblas_handle h, rocblas_operation ta, rocblas_operation tb, int64_t m, int64_t n,
                 int64_t k, const float *A, int64_t lda, const float *B, int64_t ldb, float beta,
                 float *C, int64_t ldc) {
  const float alpha = 1.f;
  CHECK_RB(rocblas_sgemm(h, ta, tb, (rocblas_int)m, (rocblas_int)n, (rocblas_int)k, &alpha, A,
                         (rocblas_int)lda, B, (rocblas_int)ldb, &beta, C, (rocblas_int)ldc));
  return AF1_OK;
}

// ---- workspace layout (one query covers every entry point) ----------------

struct Ws {
  float *hat_a, *hat_b, *z, *e, *ep, *c, *g, *p, *svid_part, *svid_w, *svid_sq, *fit, *pnum, *pden,
      *rms_part;
  double *c64, *p64, *d, *e64, *pre;
  int *count, *info, *k;
};

size_t ws_layout(int64_t m, int64_t n, int64_t r, int64_t T, uint8_t *base, Ws *w) {
  const int64_t big = (m > n ? m : n) * r;
  const int64_t maxdim = m > n ? (m > r ? m : r) : (n > r ? n : r);
  const int64_t rows_max = maxdim;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    uint8_t *p = base ? base + off : nullptr;
    off += al(bytes);
    return p;
  };
  Ws t;
  t.hat_a = (float *)take((size_t)m * r * 4);
  t.hat_b = (float *)take((size_t)r * n * 4);
  t.z = (float *)take((size_t)big * 4);
  t.e = (float *)take((size_t)big * 4);
  t.ep = (float *)take((size_t)big * 4);
  t.c = (float *)take((size_t)r * r * 4);
  t.g = (float *)take((size_t)r * r * 4);
  t.p = (float *)take((size_t)r * r * 4);
  t.svid_part = (float *)take((size_t)chunks_of(rows_max) * maxdim * 4);
  t.svid_w = (float *)take((size_t)maxdim * 4);
  t.svid_sq = (float *)take((size_t)blocks_for(maxdim) * 4);
  t.fit = (float *)take((size_t)maxdim * 4);
  t.pnum = (float *)take((size_t)chunks_of(rows_max) * r * 4);
  t.pden = (float *)take((size_t)chunks_of(rows_max) * r * 4);
  t.rms_part = (float *)take((size_t)chunks_of(T > 0 ? T : 1) * (m + n) * 4);
  t.c64 = (double *)take((size_t)r * r * 8);
  t.p64 = (double *)take((size_t)r * r * 8);
  t.d = (double *)take((size_t)r * 8);
  t.e64 = (double *)take((size_t)r * 8);
  t.pre = (double *)take((size_t)(r + 1) * 8);
  t.count = (int *)take(4);
  t.info = (int *)take(4);
  t.k = (int *)take(4);
  if (w) *w = t;
  return off;
}

// The scratch of a stand-alone SVID of a rows x cols matrix (the power
// iteration's partial sums), laid out from the start of the workspace; it
// never exceeds the layout above for a layer that has such a factor.
size_t svid_layout(int64_t rows, int64_t cols, uint8_t *base, Ws *w) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    uint8_t *p = base ? base + off : nullptr;
    off += al(bytes);
    return p;
  };
  Ws t{};
  t.svid_part = (float *)take((size_t)chunks_of(rows) * cols * 4);
  t.svid_w = (float *)take((size_t)cols * 4);
  t.svid_sq = (float *)take((size_t)blocks_for(cols) * 4);
  if (w) *w = t;
  return off;
}

// ---- building blocks (arguments already validated) ------------------------

// log2 of the rows of a run, which svid_pass_kernel adds up row by row: one run
// a workgroup gives two workgroups per compute unit of the device (512 in all);
// at least 4 rows (below it the partial sums cost more than the read of Z:
// every workgroup writes one row of them), at most a chunk.  From the shape
// alone, so that the sums are grouped alike whatever the workspace.
constexpr int kSvidWgs = 512;
int svid_run_log2(int64_t rows) {
  int l = 2;
  while (l < kChunkLog2 && ((rows + (1 << l) - 1) >> l) > kSvidWgs) ++l;
  return l;
}

template <int kQ, int kR, int kThreads>
af1_status svid_fused(const float *Z, int64_t rows, int64_t cols, int iters, uint32_t *bits,
                      float *left, float *right, float *part, size_t part_floats, float *w,
                      hipStream_t s) {
  // Rows a workgroup: a run, or as many as leave each workgroup a row of the
  // scratch (a chunk always does).
  const int run = svid_run_log2(rows);
  int wl = run;
  auto blocks_of = [&](int l) { return (unsigned)((rows + (1 << l) - 1) >> l); };
  while (wl < kChunkLog2 && (size_t)blocks_of(wl) * cols > part_floats) ++wl;
  // Too few workgroups that way (or 1024 threads, whose registers do not hold
  // the tree): the pass ends at u, and a launch of its own, 256 columns a
  // workgroup, adds up w; the same sums (10 passes on the least scratch, apart /
  // in one: 192x4576, 3 workgroups, 122 / 368 us; 4096x2016, 64, 163 / 196;
  // 8192x1024, 128, 176 / 151; 8192x4064, 128, 473 / 286).
  const bool apart = wl > run && (blocks_of(wl) < 96 || kThreads == 1024);
  const unsigned cb = (unsigned)((cols + kSumCols - 1) / kSumCols);
  const float v0 = 1.0f / sqrtf((float)cols);
  auto pass = [&](auto mode, int l, const float *wp) {
    svid_pass_kernel<kQ, kR, kThreads, decltype(mode)::value><<<blocks_of(l), kThreads, 0, s>>>(
        Z, (int)rows, (int)cols, 1 << l, 1 << run, wp, v0, right, part, left, bits);
  };
  using std::integral_constant;
  for (int it = 0; it < iters; ++it) {
    const float *wp = it == 0 ? nullptr : w;
    if (apart) {
      pass(integral_constant<int, kRowDot>{}, run, wp);
      CHECK_LAUNCH();
      abs_coldot_kernel<<<dim3(blocks_for(cols), (unsigned)chunks_of(rows)), 256, 0, s>>>(
          Z, rows, (int)cols, left, part, 1 << run);
    } else if (wl > run) {
      if constexpr (kThreads < 1024) pass(integral_constant<int, kPassTree>{}, wl, wp);
    } else {
      pass(integral_constant<int, kPass>{}, wl, wp);
    }
    CHECK_LAUNCH();
    const int l = apart ? kChunkLog2 : wl;
    const ColSum c{part, w, (int)blocks_of(l), (int)cols};
    auto colsum = [&](auto sub) {
      colsum_kernel<false, decltype(sub)::value><<<cb, 256, 0, s>>>(c, c, (int)cb, 1);
    };
    switch (kChunkLog2 - l) {
      case 0: colsum(integral_constant<int, 0>{}); break;
      case 1: colsum(integral_constant<int, 1>{}); break;
      case 2: colsum(integral_constant<int, 2>{}); break;
      case 3: colsum(integral_constant<int, 3>{}); break;
      default: colsum(integral_constant<int, 4>{}); break;
    }
    CHECK_LAUNCH();
  }
  pass(integral_constant<int, kLast>{}, run, iters == 0 ? nullptr : w);
  CHECK_LAUNCH();
  return AF1_OK;
}

// part_floats: the floats that w.svid_part may use (at least
// chunks_of(rows) * cols).
af1_status run_svid(const float *Z, int64_t rows, int64_t cols, int iters, uint32_t *bits,
                    float *left, float *right, const Ws &w, size_t part_floats, hipStream_t s) {
  // Rows of up to 16384 columns live in the registers of one workgroup;
  // more float4 a thread first (fewer waves to reduce over), then more
  // threads.
  auto fused = [&](auto Q, auto R, auto N) {
    return svid_fused<decltype(Q)::value, decltype(R)::value, decltype(N)::value>(
        Z, rows, cols, iters, bits, left, right, w.svid_part, part_floats, w.svid_w, s);
  };
  using std::integral_constant;
  using Q1 = integral_constant<int, 1>;
  using Q2 = integral_constant<int, 2>;
  using Q4 = integral_constant<int, 4>;
  if (cols <= 1024) return fused(Q1{}, Q4{}, integral_constant<int, 256>{});
  if (cols <= 2048) return fused(Q2{}, Q4{}, integral_constant<int, 256>{});
  if (cols <= 4096) return fused(Q4{}, Q2{}, integral_constant<int, 256>{});
  if (cols <= 8192) return fused(Q4{}, Q2{}, integral_constant<int, 512>{});
  if (cols <= 16384) return fused(Q4{}, Q2{}, integral_constant<int, 1024>{});
  const unsigned cb = blocks_for(cols);
  const int64_t chunks = chunks_of(rows);
  fill_kernel<<<cb, 256, 0, s>>>(right, (int)cols, 1.0f / sqrtf((float)cols));
  CHECK_LAUNCH();
  const unsigned rowblocks = (unsigned)((rows + 3) / 4);
  for (int it = 0; it < iters; ++it) {
    abs_rowdot_kernel<<<rowblocks, 256, 0, s>>>(Z, rows, (int)cols, right, left);
    CHECK_LAUNCH();
    abs_coldot_kernel<<<dim3(cb, (unsigned)chunks), 256, 0, s>>>(Z, rows, (int)cols, left,
                                                                 w.svid_part, kChunk);
    CHECK_LAUNCH();
    coldot_finish_kernel<<<cb, 256, 0, s>>>(w.svid_part, (int)chunks, (int)cols, w.svid_w,
                                            w.svid_sq);
    CHECK_LAUNCH();
    normalize_kernel<<<cb, 256, 0, s>>>(w.svid_w, w.svid_sq, (int)cb, (int)cols, right);
    CHECK_LAUNCH();
  }
  abs_rowdot_kernel<<<rowblocks, 256, 0, s>>>(Z, rows, (int)cols, right, left);
  CHECK_LAUNCH();
  CHECK_HIP(af1::launch_pack(Z, 0, rows, cols, bits, s));
  return AF1_OK;
}

// C = U diag(D) U^T in fp64 (U column-major in w.c64, D ascending in w.d).
af1_status run_eig(rocblas_handle h, const float *C, int64_t r, const Ws &w, hipStream_t s) {
  const int64_t rr = r * r;
  to_f64_kernel<<<grid_cap(rr), 256, 0, s>>>(C, w.c64, rr);
  CHECK_LAUNCH();
  CHECK_RB(rocsolver_dsyevd(h, rocblas_evect_original, rocblas_fill_upper, (rocblas_int)r, w.c64,
                            (rocblas_int)r, w.d, w.e64, w.info));
  return AF1_OK;
}

// P from the decomposition in w.c64 / w.d (the eigenvectors are masked in
// place, so any other use of them comes first).
af1_status projector_from_eig(rocblas_handle h, int64_t r, float eta, float *P, int *k_out,
                              const Ws &w, hipStream_t s) {
  const int64_t rr = r * r;
  cutoff_kernel<<<1, 64, 0, s>>>(w.d, (int)r, (double)eta, kEps, w.pre, w.count, k_out);
  CHECK_LAUNCH();
  mask_columns_kernel<<<grid_cap(rr), 256, 0, s>>>(w.c64, (int)r, w.count);
  CHECK_LAUNCH();
  const double one = 1.0, zero = 0.0;
  CHECK_RB(rocblas_dgemm(h, kN, kT, (rocblas_int)r, (rocblas_int)r, (rocblas_int)r, &one, w.c64,
                         (rocblas_int)r, w.c64, (rocblas_int)r, &zero, w.p64, (rocblas_int)r));
  to_f32_kernel<<<grid_cap(rr), 256, 0, s>>>(w.p64, P, rr);
  CHECK_LAUNCH();
  return AF1_OK;
}

af1_status run_projector(rocblas_handle h, const float *C, int64_t r, float eta, float *P,
                         int *k_out, const Ws &w, hipStream_t s) {
  af1_status st = run_eig(h, C, r, w, s);
  if (st != AF1_OK) return st;
  return projector_from_eig(h, r, eta, P, k_out, w, s);
}

// Left proxy into out (m x r).  The Gram matrix B B^T is left in w.c.
af1_status run_admm_left(rocblas_handle h, const float *Wp, int64_t m, int64_t n, int64_t r,
                         const float *A, const float *B, const float *U, float rho, float *out,
                         const Ws &w, hipStream_t s) {
  // B row-major r x n is column-major n x r: B B^T = B_c^T B_c.
  af1_status st = sgemm(h, kT, kN, r, r, n, B, n, B, n, 0.f, w.c, r);
  if (st != AF1_OK) return st;
  shift_copy_kernel<<<grid_cap(r * r), 256, 0, s>>>(w.c, w.g, (int)r, rho);
  CHECK_LAUNCH();
  scaled_diff_kernel<<<grid_cap(m * r), 256, 0, s>>>(A, U, rho, out, m * r);
  CHECK_LAUNCH();
  // out^T (r x m, column-major) += B W'^T = B_c^T W'_c
  st = sgemm(h, kT, kN, r, m, n, B, n, Wp, n, 1.f, out, r);
  if (st != AF1_OK) return st;
  // X G = R  <=>  G X^T = R^T: a left solve on the column-major view
  CHECK_RB(rocsolver_spotrf(h, rocblas_fill_lower, (rocblas_int)r, w.g, (rocblas_int)r, w.info));
  CHECK_RB(rocsolver_spotrs(h, rocblas_fill_lower, (rocblas_int)r, (rocblas_int)m, w.g,
                            (rocblas_int)r, out, (rocblas_int)r));
  return AF1_OK;
}

// Right proxy into out (r x n).  The Gram matrix A^T A is left in w.c.
af1_status run_admm_right(rocblas_handle h, const float *Wp, int64_t m, int64_t n, int64_t r,
                          const float *A, const float *B, const float *U, float rho, float *out,
                          const Ws &w, hipStream_t s) {
  // A row-major m x r is column-major r x m: A^T A = A_c A_c^T.
  af1_status st = sgemm(h, kN, kT, r, r, m, A, r, A, r, 0.f, w.c, r);
  if (st != AF1_OK) return st;
  shift_copy_kernel<<<grid_cap(r * r), 256, 0, s>>>(w.c, w.g, (int)r, rho);
  CHECK_LAUNCH();
  scaled_diff_kernel<<<grid_cap(r * n), 256, 0, s>>>(B, U, rho, out, r * n);
  CHECK_LAUNCH();
  // out^T (n x r, column-major) += W'^T A = W'_c A_c^T
  st = sgemm(h, kN, kT, n, r, m, Wp, n, A, r, 1.f, out, n);
  if (st != AF1_OK) return st;
  // G X = R  <=>  X^T G = R^T: two right-side triangular solves with G = L L^T
  CHECK_RB(rocsolver_spotrf(h, rocblas_fill_lower, (rocblas_int)r, w.g, (rocblas_int)r, w.info));
  const float one = 1.f;
  CHECK_RB(rocblas_strsm(h, rocblas_side_right, rocblas_fill_lower, kT, rocblas_diagonal_non_unit,
                         (rocblas_int)n, (rocblas_int)r, &one, w.g, (rocblas_int)r, out,
                         (rocblas_int)n));
  CHECK_RB(rocblas_strsm(h, rocblas_side_right, rocblas_fill_lower, kN, rocblas_diagonal_non_unit,
                         (rocblas_int)n, (rocblas_int)r, &one, w.g, (rocblas_int)r, out,
                         (rocblas_int)n));
  return AF1_OK;
}

// gamma (side 0: hat is rows x r, P acts on the right) or eta (side 1: hat is
// r x cols, P acts on the left) into fit.
af1_status run_fit(rocblas_handle h, int side, const float *hat, const uint32_t *bits,
                   const float *left, const float *right, int64_t rows, int64_t cols,
                   const float *P, float *fit, const Ws &w, hipStream_t s) {
  const unsigned cb = blocks_for(cols);
  residual_kernel<<<dim3(cb, rows_grid(rows)), 256, 0, s>>>(hat, bits, left, right, rows,
                                                             (int)cols, w.e);
  CHECK_LAUNCH();
  if (side == 0) {
    // EP = E P (rows x r): column-major EP^T = P E^T (P symmetric)
    af1_status st = sgemm(h, kN, kN, cols, rows, cols, P, cols, w.e, cols, 0.f, w.ep, cols);
    if (st != AF1_OK) return st;
    const int64_t chunks = chunks_of(rows);
    colfit_kernel<<<dim3(cb, (unsigned)chunks), 256, 0, s>>>(hat, w.ep, bits, left, right, rows,
                                                              (int)cols, w.pnum, w.pden);
    CHECK_LAUNCH();
    colfit_finish_kernel<<<cb, 256, 0, s>>>(w.pnum, w.pden, (int)chunks, (int)cols, (float)kEps,
                                            fit);
    CHECK_LAUNCH();
  } else {
    // PE = P E (r x cols): column-major PE^T = E^T P
    af1_status st = sgemm(h, kN, kN, cols, rows, rows, w.e, cols, P, rows, 0.f, w.ep, cols);
    if (st != AF1_OK) return st;
    rowfit_kernel<<<(unsigned)rows, 256, 0, s>>>(hat, w.ep, bits, left, right, (int)cols,
                                                 (float)kEps, fit);
    CHECK_LAUNCH();
  }
  return AF1_OK;
}

// The proxies of one iteration, solved with the eigendecomposition of the
// Gram matrix that the null-space projector needs anyway:
// (C + rho I)^-1 = U diag(1 / (D + rho)) U^T.  w.c holds C on entry; on
// exit w.c64 / w.d hold its decomposition and w.g the fp32 eigenvectors.
af1_status proxy_by_eig(rocblas_handle h, int side, const float *Wp, int64_t m, int64_t n,
                        int64_t r, const float *A, const float *B, const float *U, float rho,
                        float *out, const Ws &w, hipStream_t s) {
  af1_status st = run_eig(h, w.c, r, w, s);
  if (st != AF1_OK) return st;
  to_f32_kernel<<<grid_cap(r * r), 256, 0, s>>>(w.c64, w.g, r * r);
  CHECK_LAUNCH();
  if (side == 0) {
    scaled_diff_kernel<<<grid_cap(m * r), 256, 0, s>>>(A, U, rho, out, m * r);
    CHECK_LAUNCH();
    st = sgemm(h, kT, kN, r, m, n, B, n, Wp, n, 1.f, out, r);   // R^T += B W'^T
    if (st != AF1_OK) return st;
    // X^T = U diag U^T R^T (column-major r x m)
    st = sgemm(h, kT, kN, r, m, r, w.g, r, out, r, 0.f, w.ep, r);
    if (st != AF1_OK) return st;
    inv_shift_scale_kernel<<<grid_cap(m * r), 256, 0, s>>>(w.ep, r, m, w.d, rho, 0);
    CHECK_LAUNCH();
    return sgemm(h, kN, kN, r, m, r, w.g, r, w.ep, r, 0.f, out, r);
  }
  scaled_diff_kernel<<<grid_cap(r * n), 256, 0, s>>>(B, U, rho, out, r * n);
  CHECK_LAUNCH();
  st = sgemm(h, kN, kT, n, r, m, Wp, n, A, r, 1.f, out, n);      // R^T += W'^T A
  if (st != AF1_OK) return st;
  // X^T = R^T U diag U^T (column-major n x r)
  st = sgemm(h, kN, kN, n, r, r, out, n, w.g, r, 0.f, w.ep, n);
  if (st != AF1_OK) return st;
  inv_shift_scale_kernel<<<grid_cap(n * r), 256, 0, s>>>(w.ep, n, r, w.d, rho, 1);
  CHECK_LAUNCH();
  return sgemm(h, kN, kT, n, r, r, w.ep, n, w.g, r, 0.f, out, n);
}

af1_status run_iteration(rocblas_handle h, const float *Wp, const af1_nabf_state *S, float rho,
                         float eta, int iters, const Ws &w, hipStream_t s) {
  const int64_t m = S->m, n = S->n, r = S->r;
  // left-factor update: C_B = B B^T gives both the proxy's solve and P_B
  af1_status st = sgemm(h, kT, kN, r, r, n, S->B, n, S->B, n, 0.f, w.c, r);
  if (st != AF1_OK) return st;
  st = proxy_by_eig(h, 0, Wp, m, n, r, S->A, S->B, S->UA, rho, w.hat_a, w, s);
  if (st != AF1_OK) return st;
  add_kernel<<<grid_cap(m * r), 256, 0, s>>>(w.hat_a, S->UA, w.z, m * r);
  CHECK_LAUNCH();
  // the SVID's partial sums go where the fit's product will (free until then)
  Ws wsv = w;
  wsv.svid_part = w.ep;
  const size_t ep_floats = (size_t)(m > n ? m : n) * r;
  st = run_svid(w.z, m, r, iters, S->A_bits, S->a, S->m1, wsv, ep_floats, s);
  if (st != AF1_OK) return st;
  st = projector_from_eig(h, r, eta, w.p, nullptr, w, s);   // null space of B B^T
  if (st != AF1_OK) return st;
  st = run_fit(h, 0, w.hat_a, S->A_bits, S->a, S->m1, m, r, w.p, w.fit, w, s);
  if (st != AF1_OK) return st;
  mul_kernel<<<blocks_for(r), 256, 0, s>>>(S->m1, w.fit, (int)r);
  CHECK_LAUNCH();
  rebuild_kernel<<<dim3(blocks_for(r), rows_grid(m)), 256, 0, s>>>(S->A_bits, S->a, S->m1, m,
                                                                   (int)r, w.hat_a, S->A, S->UA);
  CHECK_LAUNCH();
  // right-factor update with the new left factor: C_A = A^T A
  st = sgemm(h, kN, kT, r, r, m, S->A, r, S->A, r, 0.f, w.c, r);
  if (st != AF1_OK) return st;
  st = proxy_by_eig(h, 1, Wp, m, n, r, S->A, S->B, S->UB, rho, w.hat_b, w, s);
  if (st != AF1_OK) return st;
  add_kernel<<<grid_cap(r * n), 256, 0, s>>>(w.hat_b, S->UB, w.z, r * n);
  CHECK_LAUNCH();
  st = run_svid(w.z, r, n, iters, S->B_bits, S->m2, S->b, wsv, ep_floats, s);
  if (st != AF1_OK) return st;
  st = projector_from_eig(h, r, eta, w.p, nullptr, w, s);   // null space of A^T A
  if (st != AF1_OK) return st;
  st = run_fit(h, 1, w.hat_b, S->B_bits, S->m2, S->b, r, n, w.p, w.fit, w, s);
  if (st != AF1_OK) return st;
  mul_kernel<<<blocks_for(r), 256, 0, s>>>(S->m2, w.fit, (int)r);
  CHECK_LAUNCH();
  rebuild_kernel<<<dim3(blocks_for(n), rows_grid(r)), 256, 0, s>>>(S->B_bits, S->m2, S->b, r,
                                                                   (int)n, w.hat_b, S->B, S->UB);
  CHECK_LAUNCH();
  return AF1_OK;
}

// ---- validation helpers ---------------------------------------------------

bool dim_ok(int64_t d) { return d >= 32 && d <= AF1_NABF_MAX_DIM && d % 32 == 0; }

struct Span {
  uintptr_t lo, hi;
};
Span span(const void *p, uint64_t bytes) {
  const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
  return Span{lo, lo + (uintptr_t)bytes};
}
// true when any two of the non-empty spans overlap
bool any_overlap(const Span *s, int count) {
  for (int i = 0; i < count; ++i)
    for (int j = i + 1; j < count; ++j)
      if (s[i].lo != s[i].hi && s[j].lo != s[j].hi && s[i].lo < s[j].hi && s[j].lo < s[i].hi)
        return true;
  return false;
}
// rocBLAS takes 32-bit dimensions and leading dimensions; keep every matrix
// below 2^31 elements as well.
bool counts_ok(int64_t a, int64_t b) { return a * b <= (int64_t)INT32_MAX; }
bool a16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
hipStream_t as_stream(void *s) { return static_cast<hipStream_t>(s); }

}  // namespace
}  // namespace af1n

using namespace af1n;

extern "C" {

size_t af1_nabf_workspace_bytes(int64_t m, int64_t n, int64_t r, int64_t T) {
  if (!dim_ok(m) || !dim_ok(n) || !dim_ok(r) || T < 0 || T > AF1_NABF_MAX_TOKENS) return 0;
  return ws_layout(m, n, r, T, nullptr, nullptr);
}

af1_status af1_nabf_surrogate(const float *W, int64_t m, int64_t n, const uint16_t *X,
                              const uint16_t *G, int64_t T, float *Wp, float *i_vec, float *o_vec,
                              void *ws, size_t ws_bytes, void *stream) {
  if (!W || !X || !G || !Wp || !i_vec || !o_vec) return AF1_ERR_NULL;
  if (!dim_ok(m) || !dim_ok(n) || !counts_ok(m, n)) return AF1_ERR_SHAPE;
  if (T < 1 || T > AF1_NABF_MAX_TOKENS) return AF1_ERR_BATCH;
  if (!a16(W) || !a16(X) || !a16(G) || !a16(Wp) || !a16(i_vec) || !a16(o_vec) || (ws && !a16(ws)))
    return AF1_ERR_ALIGN;
  Ws w;
  const size_t need = ws_layout(m, n, 32, T, static_cast<uint8_t *>(ws), &w);
  if (!ws || ws_bytes < need) return AF1_ERR_WORKSPACE;
  if (W == Wp) return AF1_ERR_ALIAS;
  hipStream_t s = as_stream(stream);
  const int64_t chunks = chunks_of(T);
  float *px = w.rms_part, *pg = w.rms_part + chunks * n;
  const unsigned xb = blocks_for(n);
  colsq_kernel<<<dim3(xb + blocks_for(m), (unsigned)chunks), 256, 0, s>>>(
      X, (int)n, px, (int)xb, G, (int)m, pg, (int)T);
  CHECK_LAUNCH();
  const ColSum cx{px, i_vec, (int)chunks, (int)n}, cg{pg, o_vec, (int)chunks, (int)m};
  const unsigned sx = (unsigned)((n + kSumCols - 1) / kSumCols);
  const unsigned sg = (unsigned)((m + kSumCols - 1) / kSumCols);
  colsum_kernel<true, 0><<<sx + sg, 256, 0, s>>>(cx, cg, (int)sx, (int)T);
  CHECK_LAUNCH();
  surrogate_scale_kernel<<<dim3(blocks_for((n + 3) / 4), rows_grid(m)), 256, 0, s>>>(
      W, m, (int)n, o_vec, i_vec, Wp);
  CHECK_LAUNCH();
  return AF1_OK;
}

af1_status af1_svid(const float *Z, int64_t rows, int64_t cols, int32_t iters, uint32_t *bits,
                    float *left, float *right, void *ws, size_t ws_bytes, void *stream) {
  if (!Z || !bits || !left || !right) return AF1_ERR_NULL;
  if (!dim_ok(rows) || !dim_ok(cols) || !counts_ok(rows, cols) || iters < 0 ||
      iters > AF1_NABF_MAX_POWER_ITERS)
    return AF1_ERR_SHAPE;
  if (!a16(Z) || !a16(bits) || !a16(left) || !a16(right) || (ws && !a16(ws))) return AF1_ERR_ALIGN;
  Ws w;
  const size_t need = svid_layout(rows, cols, static_cast<uint8_t *>(ws), &w);
  if (!ws || ws_bytes < need) return AF1_ERR_WORKSPACE;
  // what the workspace holds past the required layout serves the partial sums
  // too: they move behind the other arrays, where the rest is theirs
  size_t part_floats = (size_t)chunks_of(rows) * cols;
  const size_t spare = (ws_bytes - need) / 4;
  if (spare > part_floats) {
    w.svid_part = reinterpret_cast<float *>(static_cast<uint8_t *>(ws) + need);
    part_floats = spare;
  }
  return run_svid(Z, rows, cols, iters, bits, left, right, w, part_floats, as_stream(stream));
}

af1_status af1_nullspace_projector(const float *C, int64_t r, float eta, float *P, int32_t *k_out,
                                   void *ws, size_t ws_bytes, void *stream) {
  if (!C || !P) return AF1_ERR_NULL;
  if (!dim_ok(r) || !(eta >= 0.f && eta <= 1.f)) return AF1_ERR_SHAPE;
  if (!a16(C) || !a16(P) || (ws && !a16(ws))) return AF1_ERR_ALIGN;
  Ws w;
  const size_t need = ws_layout(32, 32, r, 0, static_cast<uint8_t *>(ws), &w);
  if (!ws || ws_bytes < need) return AF1_ERR_WORKSPACE;
  if (C == P) return AF1_ERR_ALIAS;
  hipStream_t s = as_stream(stream);
  Handle h(s);
  if (!h.ok) return AF1_ERR_HIP;
  return run_projector(h.h, C, r, eta, P, k_out, w, s);
}

af1_status af1_admm_proxy(int32_t side, const float *Wp, int64_t m, int64_t n, int64_t r,
                          const float *A, const float *B, const float *U, float rho, float *out,
                          void *ws, size_t ws_bytes, void *stream) {
  if (side != 0 && side != 1) return AF1_ERR_SHAPE;
  if (!Wp || !A || !B || !U || !out) return AF1_ERR_NULL;
  if (!dim_ok(m) || !dim_ok(n) || !dim_ok(r) || !counts_ok(m, n) || !counts_ok(m, r) ||
      !counts_ok(r, n) || !(rho > 0.f))
    return AF1_ERR_SHAPE;
  if (!a16(Wp) || !a16(A) || !a16(B) || !a16(U) || !a16(out) || (ws && !a16(ws)))
    return AF1_ERR_ALIGN;
  Ws w;
  const size_t need = ws_layout(m, n, r, 0, static_cast<uint8_t *>(ws), &w);
  if (!ws || ws_bytes < need) return AF1_ERR_WORKSPACE;
  if (out == Wp || out == A || out == B || out == U) return AF1_ERR_ALIAS;
  hipStream_t s = as_stream(stream);
  Handle h(s);
  if (!h.ok) return AF1_ERR_HIP;
  return side == 0 ? run_admm_left(h.h, Wp, m, n, r, A, B, U, rho, out, w, s)
                   : run_admm_right(h.h, Wp, m, n, r, A, B, U, rho, out, w, s);
}

af1_status af1_scale_fit(int32_t side, const float *hat, const uint32_t *bits, const float *left,
                         const float *right, int64_t rows, int64_t cols, const float *P, float *fit,
                         void *ws, size_t ws_bytes, void *stream) {
  if (side != 0 && side != 1) return AF1_ERR_SHAPE;
  if (!hat || !bits || !left || !right || !P || !fit) return AF1_ERR_NULL;
  if (!dim_ok(rows) || !dim_ok(cols) || !counts_ok(rows, cols)) return AF1_ERR_SHAPE;
  if (!a16(hat) || !a16(bits) || !a16(left) || !a16(right) || !a16(P) || !a16(fit) ||
      (ws && !a16(ws)))
    return AF1_ERR_ALIGN;
  Ws w;
  // side 0: rows = m, cols = r; side 1: rows = r, cols = n
  const size_t need = side == 0 ? ws_layout(rows, 32, cols, 0, static_cast<uint8_t *>(ws), &w)
                                : ws_layout(32, cols, rows, 0, static_cast<uint8_t *>(ws), &w);
  if (!ws || ws_bytes < need) return AF1_ERR_WORKSPACE;
  hipStream_t s = as_stream(stream);
  Handle h(s);
  if (!h.ok) return AF1_ERR_HIP;
  return run_fit(h.h, side, hat, bits, left, right, rows, cols, P, fit, w, s);
}

af1_status af1_nabf_iteration(const float *Wp, const af1_nabf_state *S, float rho, float eta,
                              int32_t power_iters, void *ws, size_t ws_bytes, void *stream) {
  if (!Wp || !S) return AF1_ERR_NULL;
  if (!S->A || !S->B || !S->UA || !S->UB || !S->A_bits || !S->B_bits || !S->a || !S->m1 ||
      !S->m2 || !S->b)
    return AF1_ERR_NULL;
  if (!dim_ok(S->m) || !dim_ok(S->n) || !dim_ok(S->r) || !counts_ok(S->m, S->n) ||
      !counts_ok(S->m, S->r) || !counts_ok(S->r, S->n) || !(rho > 0.f) ||
      !(eta >= 0.f && eta <= 1.f) || power_iters < 0 || power_iters > AF1_NABF_MAX_POWER_ITERS)
    return AF1_ERR_SHAPE;
  const void *ptrs[] = {Wp, S->A, S->B, S->UA, S->UB, S->A_bits, S->B_bits, S->a, S->m1, S->m2,
                        S->b};
  for (const void *p : ptrs)
    if (!a16(p)) return AF1_ERR_ALIGN;
  if (ws && !a16(ws)) return AF1_ERR_ALIGN;
  Ws w;
  const size_t need = ws_layout(S->m, S->n, S->r, 0, static_cast<uint8_t *>(ws), &w);
  if (!ws || ws_bytes < need) return AF1_ERR_WORKSPACE;
  const uint64_t m = S->m, n = S->n, r = S->r;
  const Span spans[] = {span(Wp, m * n * 4),     span(S->A, m * r * 4),   span(S->B, r * n * 4),
                        span(S->UA, m * r * 4),  span(S->UB, r * n * 4),  span(S->A_bits, m * r / 8),
                        span(S->B_bits, r * n / 8), span(S->a, m * 4),    span(S->m1, r * 4),
                        span(S->m2, r * 4),      span(S->b, n * 4),       span(ws, need)};
  if (any_overlap(spans, (int)(sizeof(spans) / sizeof(spans[0])))) return AF1_ERR_ALIAS;
  hipStream_t s = as_stream(stream);
  Handle h(s);
  if (!h.ok) return AF1_ERR_HIP;
  return run_iteration(h.h, Wp, S, rho, eta, power_iters, w, s);
}

af1_status af1_nabf_export(const af1_nabf_state *S, const float *i_vec, const float *o_vec,
                           uint16_t *s_out, uint16_t *s_mid, uint16_t *s_in, void *stream) {
  if (!S || !S->a || !S->m1 || !S->m2 || !S->b || !s_out || !s_mid || !s_in) return AF1_ERR_NULL;
  if (!dim_ok(S->m) || !dim_ok(S->n) || !dim_ok(S->r)) return AF1_ERR_SHAPE;
  hipStream_t s = as_stream(stream);
  export_kernel<<<blocks_for(S->m + S->r + S->n), 256, 0, s>>>(
      S->a, S->m1, S->m2, S->b, i_vec, o_vec, (int)S->m, (int)S->n, (int)S->r, s_out, s_mid, s_in);
  CHECK_LAUNCH();
  return AF1_OK;
}

}  // extern "C"
