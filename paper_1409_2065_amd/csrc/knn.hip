// k-nearest-neighbour Gaussian-kernel weights (Methods, "Calibration of
// Weights", eq_weighting) and column standardisation on gfx950.
//
// Pipeline of cc_build_knn_weights:
//   1. observed column means; X-tilde = X with missing entries replaced by
//      them, kept in FP32 (for ranking) and FP64 (for exact distances);
//   2. Gram matrix G = X~ X~^T on the matrix cores (v_mfma_f32_16x16x4_f32),
//      d2_ij = |x_i|^2 + |x_j|^2 - 2 G_ij in FP32 for every pair;
//   3. per row, a selection in registers of the K = k + margin smallest
//      (d2, j) pairs, self excluded, ties to the lower index;
//   4. exact FP64 distances of the candidates, ranked by (d2, j), keep k;
//   5. the relation i ~_k j (either direction) as a bitmap, counted and
//      prefix-summed per row, written out as sorted edges (i < j);
//   6. exact FP64 d2 per edge, phi (literal or |phi| / lower median d2),
//      w = exp(-phi d2), optional normalisation to sum 1.
//
// Also here: the smallest k whose kNN graph is connected (Results, "Impact
// of the Constants k and phi": bisection over k with a graph search), and
// weights from the composite distance of genotypes and coordinates
// (composite_distance).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "ccmi_internal.h"

namespace ccmi {

static inline int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------- column stats
// Per column over its observed entries: the mean, and (sec not null) the
// sum of squared deviations from it or its root mean square; the count of
// non-finite observed entries is added to *nonfinite, and with skip they are
// left out of the sums.  A block of 1024 threads owns CPB columns, so a
// column's rows are read by 1024 / CPB threads at once, 8 rows of each in
// flight, and both passes (mean, then deviations) run in one launch without
// workspace.  A thread per column instead waits on one row after another:
// 1550 us on 2000 x 500 with a mask and 5900 us on 12000 x 64, against 10
// and 20 us here.  Narrow matrices take 4 columns per block so that more
// than a few blocks share the rows; from 1024 columns on, 16 (64 bytes of
// each FP32 row) already fill the chip.
constexpr int kColRows = 8;  // rows a thread has in flight

template <typename TI, int CPB>
__global__ __launch_bounds__(1024) void k_col_moments(int n, int p, const TI *X, int64_t ldx, const uint8_t *M,
                                                      int64_t ldm, int skip, double *mean, double *sec, int root,
                                                      int *nonfinite) {
  constexpr int RG = 1024 / CPB, NW = 1024 / kWave;
  __shared__ double ssum[NW][CPB];
  __shared__ int scnt[NW][CPB];
  __shared__ int sbad, sflat;
  const int c = threadIdx.x % CPB, g = threadIdx.x / CPB, wave = threadIdx.x / kWave;
  const int f = blockIdx.x * CPB + c;
  const bool col = f < p;
  const int fc = col ? f : 0;
  if (threadIdx.x == 0) sbad = sflat = 0;
  // fn(x) for every row of this thread that counts; returns the bad ones
  auto rows = [&](auto fn) {
    int bad = 0;
    for (int i0 = g; i0 < n; i0 += RG * kColRows) {
      TI x[kColRows];
      uint8_t o[kColRows];
#pragma unroll
      for (int u = 0; u < kColRows; ++u) {
        const int i = min(i0 + u * RG, n - 1);
        o[u] = M ? M[(size_t)i * ldm + fc] : (uint8_t)1;
        x[u] = X[(size_t)i * ldx + fc];
      }
#pragma unroll
      for (int u = 0; u < kColRows; ++u) {
        if (i0 + u * RG >= n || o[u] == 0) continue;
        const bool fin = isfinite((double)x[u]);
        if (!fin) ++bad;
        if (fin || !skip) fn((double)x[u]);
      }
    }
    return bad;
  };
  // a column's values within a wave combined: lanes CPB apart
  auto lanes = [&](auto v, auto op) {
#pragma unroll
    for (int off = kWave / 2; off >= CPB; off >>= 1) v = op(v, __shfl_xor(v, off, kWave));
    return v;
  };
  auto add = [](auto a, auto b) { return a + b; };
  double sum = 0.0;
  int cnt = 0;
  const int bad = rows([&](double x) { sum += x; ++cnt; });
  sum = lanes(sum, add);
  cnt = lanes(cnt, add);
  if (threadIdx.x % kWave < CPB) { ssum[wave][c] = sum; scnt[wave][c] = cnt; }
  __syncthreads();
  if (bad && col) atomicAdd(&sbad, bad);
  int tc = 0;
  double mu = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) { mu += ssum[w][c]; tc += scnt[w][c]; }
  mu = tc > 0 ? mu / tc : 0.0;
  if (threadIdx.x < CPB && col) mean[f] = mu;
  __syncthreads();
  if (threadIdx.x == 0 && sbad && nonfinite) atomicAdd(nonfinite, sbad);
  if (!sec) return;
  double ss = 0.0;
  rows([&](double x) { ss += (x - mu) * (x - mu); });
  ss = lanes(ss, add);
  if (threadIdx.x % kWave < CPB) ssum[wave][c] = ss;
  __syncthreads();
  bool flat = false;
  if (threadIdx.x < CPB && col) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += ssum[w][c];
    sec[f] = root ? (tc > 0 ? sqrt(t / tc) : 0.0) : t;
    // deviations within the rounding of the sum the mean came from
    const double r = 0x1p-52 * tc * mu;
    flat = root && t > 0.0 && t <= tc * r * r;
    if (flat) sflat = 1;
  }
  if (!root) return;
  __syncthreads();
  if (!sflat) return;
  // some column may hold one value, off whose mean it rounds: such a column
  // has a deviation of 0 exactly
  double lo = INFINITY, hi = -INFINITY;
  rows([&](double x) { lo = fmin(lo, x); hi = fmax(hi, x); });
  lo = lanes(lo, [](double a, double b) { return fmin(a, b); });
  hi = lanes(hi, [](double a, double b) { return fmax(a, b); });
  if (threadIdx.x % kWave < CPB) ssum[wave][c] = lo;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) lo = fmin(lo, ssum[w][c]);
  __syncthreads();
  if (threadIdx.x % kWave < CPB) ssum[wave][c] = hi;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) hi = fmax(hi, ssum[w][c]);
  if (flat && lo == hi) sec[f] = 0.0;
}

template <typename TI>
static void moments_launch(int64_t n, int64_t p, const TI *X, int64_t ldx, const uint8_t *M, int64_t ldm, bool skip,
                           double *mean, double *sec, bool root, int *nonfinite, hipStream_t st) {
  if (p <= 1024)
    hipLaunchKernelGGL((k_col_moments<TI, 4>), dim3((int)cdiv64(p, 4)), dim3(1024), 0, st, (int)n, (int)p, X, ldx, M,
                       ldm, skip ? 1 : 0, mean, sec, root ? 1 : 0, nonfinite);
  else
    hipLaunchKernelGGL((k_col_moments<TI, 16>), dim3((int)cdiv64(p, 16)), dim3(1024), 0, st, (int)n, (int)p, X, ldx,
                       M, ldm, skip ? 1 : 0, mean, sec, root ? 1 : 0, nonfinite);
}

void column_moments(int64_t n, int64_t p, int32_t x_dtype, const void *X, int64_t ldx, const uint8_t *mask,
                    int64_t ldm, bool skip, double *mean, double *sec, bool root, int *nonfinite, hipStream_t st) {
  if (x_dtype == CC_DTYPE_F32)
    moments_launch(n, p, (const float *)X, ldx, mask, ldm, skip, mean, sec, root, nonfinite, st);
  else
    moments_launch(n, p, (const double *)X, ldx, mask, ldm, skip, mean, sec, root, nonfinite, st);
}

template <typename TI>
__global__ void k_standardize(int n, int p, TI *X, int64_t ldx, const uint8_t *M, int64_t ldm,
                              const double *mean, const double *sd) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)n * p) return;
  const int i = (int)(idx / p), f = (int)(idx % p);
  if (M && M[(size_t)i * ldm + f] == 0) return;
  const double s = sd[f];
  const double inv = s > 0.0 ? 1.0 / s : 0.0;
  const double x = (double)X[(size_t)i * ldx + f];
  X[(size_t)i * ldx + f] = (TI)((x - mean[f]) * inv);
}

// X-tilde in FP32 (n_pad x ldk, zero padded) and FP64 (n x p), and the FP32
// squared row norms of the FP32 copy.
template <typename TI>
__global__ void k_impute(int n, int p, int n_pad, int ldk, const TI *X, int64_t ldx,
                         const uint8_t *M, int64_t ldm, const double *mean, float *Xf,
                         double *Xd) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)n_pad * ldk) return;
  const int i = (int)(idx / ldk), f = (int)(idx % ldk);
  double v = 0.0;
  if (i < n && f < p) {
    const bool obs = M ? (M[(size_t)i * ldm + f] != 0) : true;
    v = obs ? (double)X[(size_t)i * ldx + f] : mean[f];
    Xd[(size_t)i * p + f] = v;
  }
  Xf[idx] = (float)v;
}

__global__ void k_rownorm(int n_pad, int ldk, const float *Xf, float *nrm) {
  const int i = blockIdx.x;
  double acc = 0.0;
  for (int f = threadIdx.x; f < ldk; f += blockDim.x) {
    const double v = Xf[(size_t)i * ldk + f];
    acc = fma(v, v, acc);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  __shared__ double s[16];
  if (threadIdx.x % kWave == 0) s[threadIdx.x / kWave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) t += s[w];
    nrm[i] = (float)t;
  }
}

// ------------------------------------------------------------ MFMA Gram
// Output tile 64 x 64 per block of 4 waves; wave w owns rows 16w..16w+15 and
// all 64 columns as four 16 x 16 accumulators.  K is staged through LDS in
// chunks of 32 features; the next chunk's global loads are in flight while
// the current chunk's MFMAs run.  v_mfma_f32_16x16x4_f32 operand layout
// (wave64): A element (row l%16, k l/16), B element (k l/16, col l%16), and
// result register r of lane l holds (row 4*(l/16)+r, col l%16).
// When the output tiles alone cannot fill the chip, blockIdx.z splits K:
// each split writes its partial tile to part, and k_gram_combine adds the
// splits in a fixed order.  D2 and part hold the rows from row0 on (a panel
// of the matrix; rows_pad of them with padding).
constexpr int kGT = 64, kKC = 32;

typedef float floatx4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_gram_d2(int n, int n_pad, int ldk, int nsplit,
                                                 const float *Xf, const float *nrm, int row0,
                                                 int rows_pad, float *D2, int64_t ldd, float *part) {
  __shared__ float As[kGT][kKC + 1];
  __shared__ float Bs[kGT][kKC + 1];
  const int bi = row0 + blockIdx.y * kGT, bj = blockIdx.x * kGT;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int nch = ldk / kKC;
  const int per = (nch + nsplit - 1) / nsplit;
  const int c0 = blockIdx.z * per, c1 = min(nch, c0 + per);
  // 64 rows x 32 floats per operand: thread tid loads rows r and r + 32,
  // 4 consecutive floats each
  const int r = tid / 8, c4 = (tid % 8) * 4;
  float4 pa[2], pb[2];
  auto gload = [&](int ch) {
    const int k0 = ch * kKC + c4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      pa[h] = *reinterpret_cast<const float4 *>(Xf + (size_t)(bi + r + 32 * h) * ldk + k0);
      pb[h] = *reinterpret_cast<const float4 *>(Xf + (size_t)(bj + r + 32 * h) * ldk + k0);
    }
  };
  floatx4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (c0 < c1) gload(c0);
  for (int ch = c0; ch < c1; ++ch) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float *ar = &As[r + 32 * h][c4], *br = &Bs[r + 32 * h][c4];
      ar[0] = pa[h].x; ar[1] = pa[h].y; ar[2] = pa[h].z; ar[3] = pa[h].w;
      br[0] = pb[h].x; br[1] = pb[h].y; br[2] = pb[h].z; br[3] = pb[h].w;
    }
    __syncthreads();
    if (ch + 1 < c1) gload(ch + 1);
#pragma unroll
    for (int kk = 0; kk < kKC; kk += 4) {
      const float a = As[wave * 16 + lane % 16][kk + lane / 16];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float b = Bs[c * 16 + lane % 16][kk + lane / 16];
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[c], 0, 0, 0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = bi + wave * 16 + 4 * (lane / 16) + q;
      const int j = bj + c * 16 + lane % 16;
      if (nsplit > 1)
        part[((size_t)blockIdx.z * rows_pad + (i - row0)) * n_pad + j] = acc[c][q];
      else if (i < n && j < n)
        D2[(size_t)(i - row0) * ldd + j] = nrm[i] + nrm[j] - 2.0f * acc[c][q];
    }
  }
}

// d2 from the K-split partial Gram tiles, splits added in order.
__global__ void k_gram_combine(int n, int n_pad, int nsplit, const float *part, const float *nrm,
                               int row0, int rows, int rows_pad, float *D2, int64_t ldd) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)rows * n) return;
  const int r = (int)(e / n), j = (int)(e - (int64_t)r * n);
  float g = 0.f;
  for (int z = 0; z < nsplit; ++z) g += part[((size_t)z * rows_pad + r) * n_pad + j];
  D2[(size_t)r * ldd + j] = nrm[row0 + r] + nrm[j] - 2.0f * g;
}

// Monotone map of a float to an unsigned key (handles negative values).
__device__ inline uint32_t float_key(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Most candidates k_recheck takes per row (12 bytes of LDS each), and the
// largest n of the kNN builders (a row's keys fill the registers of a block).
constexpr int64_t kRecheckMaxK = 12288;
constexpr int64_t kKnnMaxN = 16384;
static_assert(kKnnMaxN <= 64 * 256, "64 keys per thread in k_row_select");
// Largest panel of the distance matrix kept at once: it stays in the last
// level cache between the product that writes it and the selection that
// reads it, and a build of 12000 rows holds 64 MiB instead of 576.
constexpr int64_t kPanelBytes = (int64_t)64 << 20;

// Inverse of float_key.
__device__ inline float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Per row: the K smallest (d2, j) pairs over the other rows j (in no
// particular order), and in dnext the FP32 d2 of the first one left out
// (infinity when none is).  Row r of the panel D2 is row row0 + r.  A block
// of 4 waves holds the row's keys in registers, PT per thread.  A K-th
// smallest key is built two bits at a time, as the largest v with fewer than
// K keys below it: a step counts the keys below three trial values with
// ballots and one barrier.
// The K-th smallest of the 256 threads' smallest keys bounds the row's K-th
// smallest from above, and little more than K keys lie below that bound: they
// go to LDS and are ranked there, by (key, j).  Only a row with more than
// kSelList such keys (K near 256 or above, many ties) takes the steps over
// all its keys.  Measured: 12000 rows 0.46 ms, 2000 rows of 2000 15 us; with
// the steps over all keys 1.90 ms and 24 us; sorting each row in LDS 7.4 ms
// and 119 us.
// todo (may be NULL): only rows with todo[i] != 0.
constexpr int kSelThreads = 256;
constexpr int kSelList = 512;

template <int PT>
__global__ __launch_bounds__(kSelThreads) void k_row_select(int n, int row0, const float *D2, int64_t ldd, int K,
                                                            int32_t *cand, const int *todo, float *dnext) {
  constexpr int NW = kSelThreads / kWave;
  __shared__ int cnts[2][NW][3];
  __shared__ uint32_t wmin[NW];
  __shared__ int fill;
  __shared__ unsigned long long list[kSelList];
  const int i = row0 + blockIdx.x;
  if (todo && !todo[i]) return;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const float *row = D2 + (size_t)blockIdx.x * ldd;
  // slots past the row, and the row itself, hold the largest key, which no
  // distance maps to
  uint32_t key[PT];
#pragma unroll
  for (int e = 0; e < PT; ++e) {
    const int j = threadIdx.x + e * kSelThreads;
    key[e] = 0xffffffffu;
    if (j < n && j != i) key[e] = min(float_key(row[j]), 0xfffffffeu);
  }
  if (threadIdx.x == 0) fill = 0;
  int buf = 0;
  // block counts of three predicates of (key, j)
  auto count3 = [&](auto p0, auto p1, auto p2, int &c0, int &c1, int &c2) {
    int a0 = 0, a1 = 0, a2 = 0;
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      const int j = threadIdx.x + e * kSelThreads;
      a0 += __popcll(__ballot(p0(key[e], j)));
      a1 += __popcll(__ballot(p1(key[e], j)));
      a2 += __popcll(__ballot(p2(key[e], j)));
    }
    if (lane == 0) { cnts[buf][wave][0] = a0; cnts[buf][wave][1] = a1; cnts[buf][wave][2] = a2; }
    __syncthreads();
    c0 = c1 = c2 = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { c0 += cnts[buf][w][0]; c1 += cnts[buf][w][1]; c2 += cnts[buf][w][2]; }
    buf ^= 1;  // the next count writes the other buffer: one barrier per count
  };
  // the K-th smallest of the threads' smallest keys
  uint32_t mine = key[0];
#pragma unroll
  for (int e = 1; e < PT; ++e) mine = min(mine, key[e]);
  uint32_t top = 0;
  for (int bit = 30; bit >= 0; bit -= 2) {
    const uint32_t t1 = top | (1u << bit), t2 = top | (2u << bit), t3 = top | (3u << bit);
    const int a1 = __popcll(__ballot(mine < t1)), a2 = __popcll(__ballot(mine < t2)), a3 = __popcll(__ballot(mine < t3));
    if (lane == 0) { cnts[buf][wave][0] = a1; cnts[buf][wave][1] = a2; cnts[buf][wave][2] = a3; }
    __syncthreads();
    int c1 = 0, c2 = 0, c3 = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { c1 += cnts[buf][w][0]; c2 += cnts[buf][w][1]; c3 += cnts[buf][w][2]; }
    buf ^= 1;
    top = c3 < K ? t3 : (c2 < K ? t2 : (c1 < K ? t1 : top));
  }
  top = min(top, 0xfffffffeu);  // fewer than K threads have a key: all keys
  uint32_t next = 0xffffffffu;  // the smallest key above the bound
#pragma unroll
  for (int e = 0; e < PT; ++e) {
    const bool sel = key[e] <= top;
    const uint64_t m = __ballot(sel);
    if (m) {
      int base = 0;
      if (lane == 0) base = atomicAdd(&fill, __popcll(m));
      base = __builtin_amdgcn_readfirstlane(base) + __popcll(m & ((1ull << lane) - 1ull));
      if (sel && base < kSelList)
        list[base] = ((unsigned long long)key[e] << 32) | (unsigned)(threadIdx.x + e * kSelThreads);
    }
    if (!sel) next = min(next, key[e]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) next = min(next, (uint32_t)__shfl_xor((int)next, off, kWave));
  if (lane == 0) wmin[wave] = next;
  __syncthreads();
  const int S = fill;
  if (S <= kSelList) {  // uniform; S >= K
    for (int c = threadIdx.x; c < S; c += kSelThreads) {
      const unsigned long long k = list[c];
      int r = 0;
      for (int o = 0; o < S; ++o) r += list[o] < k ? 1 : 0;
      if (r < K) cand[(size_t)i * K + r] = (int32_t)(k & 0xffffffffu);
      if (r == K) dnext[i] = key_float((uint32_t)(k >> 32));
    }
    if (threadIdx.x == 0 && S == K) {
#pragma unroll
      for (int w = 0; w < NW; ++w) next = min(next, wmin[w]);
      dnext[i] = K < n - 1 ? key_float(next) : INFINITY;
    }
    return;
  }
  __syncthreads();
  if (threadIdx.x == 0) fill = 0;  // used again after the next barrier
  uint32_t v = 0;
  for (int bit = 30; bit >= 0; bit -= 2) {
    const uint32_t t1 = v | (1u << bit), t2 = v | (2u << bit), t3 = v | (3u << bit);
    int c1, c2, c3;
    count3([&](uint32_t k, int) { return k < t1; }, [&](uint32_t k, int) { return k < t2; },
           [&](uint32_t k, int) { return k < t3; }, c1, c2, c3);
    v = c3 < K ? t3 : (c2 < K ? t2 : (c1 < K ? t1 : v));
  }
  // ties with the K-th key go to the lower rows: the need-th smallest row
  // among them bounds those taken
  int less, upto, unused;
  count3([&](uint32_t k, int) { return k < v; }, [&](uint32_t k, int) { return k <= v; },
         [](uint32_t, int) { return false; }, less, upto, unused);
  int jmax = n;
  if (upto > K) {  // uniform
    const int need = K - less;
    int jt = 0;
    for (int bit = 14; bit >= 0; --bit) {
      const int t = jt | (1 << bit);
      int c;
      count3([&](uint32_t k, int j) { return k == v && j < t; }, [](uint32_t, int) { return false; },
             [](uint32_t, int) { return false; }, c, unused, unused);
      if (c < need) jt = t;
    }
    jmax = jt;
  }
  next = 0xffffffffu;
#pragma unroll
  for (int e = 0; e < PT; ++e) {
    const int j = threadIdx.x + e * kSelThreads;
    const bool sel = key[e] < v || (key[e] == v && j <= jmax);
    const uint64_t m = __ballot(sel);
    if (m) {
      int base = 0;
      if (lane == 0) base = atomicAdd(&fill, __popcll(m));
      base = __builtin_amdgcn_readfirstlane(base);
      if (sel) cand[(size_t)i * K + base + __popcll(m & ((1ull << lane) - 1ull))] = j;
    }
    if (key[e] > v) next = min(next, key[e]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) next = min(next, (uint32_t)__shfl_xor((int)next, off, kWave));
  if (lane == 0) wmin[wave] = next;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < NW; ++w) next = min(next, wmin[w]);
    dnext[i] = K < n - 1 ? key_float(upto > K ? v : next) : INFINITY;
  }
}

// Largest FP32 row norm of the n rows.
__global__ __launch_bounds__(1024) void k_max_norm(int n, const float *nrm, float *nmax) {
  __shared__ float s[1024];
  float m = 0.f;
  for (int i = threadIdx.x; i < n; i += blockDim.x) m = fmaxf(m, nrm[i]);
  s[threadIdx.x] = m;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] = fmaxf(s[threadIdx.x], s[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *nmax = s[0];
}

// Order of (distance, row) pairs; a distance that is not a number comes
// after every number.
__device__ __forceinline__ bool dist_less(double a, int i, double b, int j) {
  const bool an = a == a, bn = b == b;
  if (an != bn) return an;
  return an ? (a < b || (a == b && i < j)) : i < j;
}

// How a block of 256 threads ranks K exact distances for the k smallest.
// Counting takes a step per candidate and turn of 256 candidates; finding
// them in turn measured 12 such steps each at K = 512 and 37 at 2999.  The
// first pass counts (K is about 2 k); a wide one finds a few of thousands
// (12000 rows, k = 10: 76 ms for K = 11999, by counting 3342; K = 512 1.0 and
// 1.9 ms).
static bool rank_by_counting(int K, int k) {
  const int turns = (K + 255) / 256;
  return 2 * (int64_t)turns * K <= (int64_t)k * (5 * turns + 14);
}

// Exact FP64 squared distances of the candidates, then the k best by (d2, j).
// Certificate: every row left out has an FP32 distance of at least dnext[i],
// so an exact one of at least dnext[i] - bound, with bound = bscale *
// (|x_i|^2 + max_j |x_j|^2) covering the rounding of the FP32 Gram product,
// the norms, their combination and the FP32 copy of X~.  The k best
// candidates are then the k nearest of all rows when the k-th exact distance
// lies below that; otherwise uncert[i] = 1 and the row is counted in *n_uncert.
// todo (may be NULL): only rows with todo[i] != 0.
template <bool COUNT>
__global__ __launch_bounds__(256) void k_recheck(int n, int p, const double *Xd, int K, int k,
                                                 const int32_t *cand, int32_t *knn, const int *todo,
                                                 const float *dnext, const float *nrm,
                                                 const float *nmax, double bscale, int *uncert,
                                                 int *n_uncert) {
  extern __shared__ double sd[];  // K doubles + K ints
  int *sj = reinterpret_cast<int *>(sd + K);
  __shared__ double kth;
  const int i = blockIdx.x;
  if (todo && !todo[i]) return;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
  for (int c = wave; c < K; c += nw) {
    const int j = cand[(size_t)i * K + c];
    double acc = 0.0;
#pragma unroll 4
    for (int f = lane; f < p; f += kWave) {
      const double d = Xd[(size_t)j * p + f] - Xd[(size_t)i * p + f];
      acc = fma(d, d, acc);
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    if (lane == 0) { sd[c] = acc; sj[c] = j; }
  }
  if (threadIdx.x == 0) kth = NAN;  // no candidate of that rank: not certified
  __syncthreads();
  // The k smallest (d2, j), a distance that is not a number last, by row.
  if constexpr (COUNT) {
    // a candidate's rank is the number of smaller ones; a thread per
    // candidate counts it (one thread selecting them in turn took 3/4 of this
    // kernel's time at K = 32)
    for (int c = threadIdx.x; c < K; c += blockDim.x) {
      const double d = sd[c];
      const int j = sj[c];
      const bool num = d == d;
      int r = 0;
      for (int o = 0; o < K; ++o) {
        const double od = sd[o];
        const bool less = num ? (od < d || (od == d && sj[o] < j)) : (od == od || sj[o] < j);
        r += less ? 1 : 0;
      }
      if (r < k) knn[(size_t)i * k + r] = j;
      if (r == k - 1) kth = d;
    }
  } else {
    // the block finds them in turn, each the smallest above the last
    __shared__ double wd[2][4];
    __shared__ int wj[2][4];
    double last = 0.0;
    int lj = -1;
    for (int r = 0; r < k; ++r) {
      double b = NAN;
      int bj = INT32_MAX;
      for (int c = threadIdx.x; c < K; c += blockDim.x) {
        const double d = sd[c];
        const int j = sj[c];
        if (dist_less(last, lj, d, j) && dist_less(d, j, b, bj)) { b = d; bj = j; }
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        const double ob = __shfl_xor(b, off, kWave);
        const int oj = __shfl_xor(bj, off, kWave);
        if (dist_less(ob, oj, b, bj)) { b = ob; bj = oj; }
      }
      // two sets of slots in turn: one barrier per candidate
      if (lane == 0) { wd[r & 1][wave] = b; wj[r & 1][wave] = bj; }
      __syncthreads();
      last = wd[r & 1][0];
      lj = wj[r & 1][0];
#pragma unroll
      for (int w = 1; w < 4; ++w)
        if (dist_less(wd[r & 1][w], wj[r & 1][w], last, lj)) { last = wd[r & 1][w]; lj = wj[r & 1][w]; }
      if (threadIdx.x == 0) knn[(size_t)i * k + r] = lj;
    }
    if (threadIdx.x == 0) kth = last;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double bound = bscale * ((double)nrm[i] + (double)*nmax);
    const bool ok = kth < (double)dnext[i] - bound;
    uncert[i] = ok ? 0 : 1;
    if (!ok) atomicAdd(n_uncert, 1);
  }
}

// n words of zero.
__global__ void k_zero_words(uint32_t *v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    v[i] = 0u;
}

__global__ void k_mark_pairs(int n, int k, int words, const int32_t *knn, uint32_t *bm) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * k) return;
  const int i = (int)(idx / k);
  const int j = knn[idx];
  const int a = min(i, j), b = max(i, j);
  atomicOr(&bm[(size_t)a * words + b / 32], 1u << (b % 32));
}

// Set bits of each row of the bitmap, a wave per row.
__global__ __launch_bounds__(256) void k_row_counts(int n, int words, const uint32_t *bm, int32_t *cnt) {
  const int i = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (i >= n) return;
  int c = 0;
  for (int w = threadIdx.x % kWave; w < words; w += kWave) c += __popc(bm[(size_t)i * words + w]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, kWave);
  if (threadIdx.x % kWave == 0) cnt[i] = c;
}

// Sum of the lanes below this one.
__device__ __forceinline__ int lanes_before(int v) {
  const int lane = threadIdx.x % kWave;
  int run = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int o = __shfl_up(run, off, kWave);
    if (lane >= off) run += o;
  }
  return run - v;
}

// Exclusive scan of n counts in one block: a thread's chunk, the lanes of a
// wave, the waves.  The total is at most n * k < 2^31.
__global__ __launch_bounds__(1024) void k_scan(int n, const int32_t *cnt, int32_t *off, int64_t *total) {
  __shared__ int wsum[1024 / kWave];
  const int t = threadIdx.x, nt = blockDim.x, wave = t / kWave;
  const int per = (n + nt - 1) / nt;
  const int s0 = min(n, t * per), s1 = min(n, s0 + per);
  int acc = 0;
  for (int i = s0; i < s1; ++i) acc += cnt[i];
  int run = lanes_before(acc);
  if (t % kWave == kWave - 1) wsum[wave] = run + acc;
  __syncthreads();
  for (int w = 0; w < wave; ++w) run += wsum[w];
  for (int i = s0; i < s1; ++i) { off[i] = run; run += cnt[i]; }
  if (t == nt - 1) *total = run;
}

// The edges of each row in order, a wave per row: 64 words at a time, each
// lane after the bits of the words before its own.
__global__ __launch_bounds__(256) void k_emit_edges(int n, int words, const uint32_t *bm, const int32_t *off,
                                                    int32_t *ei, int32_t *ej) {
  const int i = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (i >= n) return;
  int pos = off[i];
  for (int w0 = 0; w0 < words; w0 += kWave) {
    const int w = w0 + threadIdx.x % kWave;
    uint32_t bits = w < words ? bm[(size_t)i * words + w] : 0u;
    const int c = __popc(bits);
    const int before = lanes_before(c);
    int q = pos + before;
    while (bits) {
      const int b = __ffs(bits) - 1;
      bits &= bits - 1;
      ei[q] = i;
      ej[q] = w * 32 + b;
      ++q;
    }
    pos += __shfl(before + c, kWave - 1, kWave);
  }
}

__global__ void k_edge_d2(int E, int p, const double *Xd, const int32_t *ei, const int32_t *ej,
                          double *d2) {
  const int e = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (e >= E) return;
  const int i = ei[e], j = ej[e];
  double acc = 0.0;
  for (int f = lane; f < p; f += kWave) {
    const double d = Xd[(size_t)j * p + f] - Xd[(size_t)i * p + f];
    acc = fma(d, d, acc);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (lane == 0) d2[e] = acc;
}

// Block sums and extremes of one value per thread (1024 threads), to all.
template <typename T, typename Op>
__device__ inline T block_reduce(T v, T *red, Op op) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off, kWave));
  __syncthreads();  // red may hold an earlier result
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  v = red[0];
  for (int w = 1; w < (int)(blockDim.x / kWave); ++w) v = op(v, red[w]);
  return v;
}

// phi = c over the lower median of E >= 1 non-negative doubles (0 when the
// median is 0), by bit patterns, which order them.  One block: the range
// [lo, hi] of patterns is cut into at most 4096 equal buckets, the bucket of
// the median becomes the range, and once it holds few enough values they
// are ranked in LDS.  Distances spread evenly over the buckets, so two or
// three passes over the values do (a radix pass by bytes puts them all into
// the few bins of their exponents: 8 passes, 100 us for 23 000 values and
// 245 us for 80 000, against 18 and 48 us).
constexpr int kMedBuckets = 4096, kMedList = 1024;

__global__ __launch_bounds__(1024) void k_median_phi(int E, const double *v, double c, double *phi) {
  using u64 = unsigned long long;
  __shared__ unsigned int hist[kMedBuckets];
  __shared__ u64 list[kMedList];
  __shared__ u64 red[1024 / kWave];
  __shared__ int wsum[1024 / kWave];
  __shared__ int bucket, below, filled;
  __shared__ u64 answer;
  const int t = threadIdx.x, wave = t / kWave;
  auto key = [&](int e) { return (u64)__double_as_longlong(v[e]); };
  u64 lo = ~0ull, hi = 0ull;
#pragma unroll 4
  for (int e = t; e < E; e += 1024) { const u64 k = key(e); lo = min(lo, k); hi = max(hi, k); }
  lo = block_reduce(lo, red, [](u64 a, u64 b) { return a < b ? a : b; });
  hi = block_reduce(hi, red, [](u64 a, u64 b) { return a > b ? a : b; });
  int rank = (E - 1) / 2;
  for (;;) {  // each turn cuts the range by 4096: at most 6
    const u64 range = hi - lo;
    const int bits = range ? 64 - __clzll((long long)range) : 0;
    const int shift = bits > 12 ? bits - 12 : 0;
    for (int b = t; b < kMedBuckets; b += 1024) hist[b] = 0u;
    if (t == 0) filled = 0;
    __syncthreads();
#pragma unroll 4
    for (int e = t; e < E; e += 1024) {
      const u64 k = key(e);
      if (k >= lo && k <= hi) atomicAdd(&hist[(k - lo) >> shift], 1u);
    }
    __syncthreads();
    // each thread's 4 buckets, the counts before them, and the one with the rank
    int h[4], own = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) { h[q] = (int)hist[4 * t + q]; own += h[q]; }
    int run = lanes_before(own);
    if (t % kWave == kWave - 1) wsum[wave] = run + own;
    __syncthreads();
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (rank >= run && rank < run + h[q]) { bucket = 4 * t + q; below = run; }
      run += h[q];
    }
    __syncthreads();
    const int b = bucket, cnt = (int)hist[b];
    rank -= below;
    lo += (u64)b << shift;
    const u64 top = lo + ((1ull << shift) - 1ull);
    hi = top < hi ? top : hi;
    if (shift == 0) {  // a bucket of one value
      if (t == 0) answer = lo;
      break;
    }
    if (cnt <= kMedList) {
#pragma unroll 4
      for (int e = t; e < E; e += 1024) {
        const u64 k = key(e);
        if (k >= lo && k <= hi) list[atomicAdd(&filled, 1)] = k;
      }
      __syncthreads();
      if (t < cnt) {
        const u64 mine = list[t];
        int r = 0;
        for (int o = 0; o < cnt; ++o) r += (list[o] < mine || (list[o] == mine && o < t)) ? 1 : 0;
        if (r == rank) answer = mine;
      }
      break;
    }
    __syncthreads();  // bucket, below and hist are read before the next turn
  }
  __syncthreads();
  if (t == 0) {
    const double med = __longlong_as_double((long long)answer);
    *phi = med > 0.0 ? c / med : 0.0;
  }
}

// phi (may be NULL): the device value; else the literal c.
__global__ void k_weights(int E, const double *d2, const double *phi, double c, double *w) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < E) w[e] = exp(-(phi ? *phi : c) * d2[e]);
}

// Sum of the weights (one block, coalesced, fixed order), then the scaling.
__global__ __launch_bounds__(1024) void k_weight_sum(int E, const double *w, double *tot) {
  __shared__ double red[1024 / kWave];
  double acc = 0.0;
#pragma unroll 4
  for (int e = threadIdx.x; e < E; e += 1024) acc += w[e];
  acc = block_reduce(acc, red, [](double a, double b) { return a + b; });
  if (threadIdx.x == 0) *tot = acc;
}
__global__ void k_normalize(int E, const double *tot, double *w) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const double inv = 1.0 / *tot;
  if (e < E) w[e] *= inv;
}

// ------------------------------------------------ connectivity over k
// Directed pairs (i, q-th neighbour of i) of the k_max lists.
__global__ void k_knn_pairs(int n, int kmax, const int32_t *knn, int32_t *ei, int32_t *ej) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < (int64_t)n * kmax) {
    ei[e] = (int32_t)(e / kmax);
    ej[e] = knn[e];
  }
}

// Keep the pairs of the first k neighbours: the union graph of i ~_k j.
__global__ void k_keep_prefix(int64_t m, int kmax, int k, uint8_t *keep) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < m) keep[e] = (e % kmax) < k ? 1 : 0;
}

// ------------------------------------------------ composite distance
// Mean-imputed X in FP64 (n x p dense): missing entries take their
// observed column mean, as the kNN weights do.
template <typename TI>
__global__ void k_impute_d(int n, int p, const TI *X, int64_t ldx, const uint8_t *M, int64_t ldm,
                           const double *mean, double *Xd) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * p) return;
  const int i = (int)(e / p), f = (int)(e - (int64_t)i * p);
  Xd[e] = M[(size_t)i * ldm + f] ? (double)X[(size_t)i * ldx + f] : mean[f];
}

constexpr int kMaxCoords = 8;
struct CoordSpec {
  int q, geodesic;
  double radius, alpha;
  double period[kMaxCoords];
};

// One wave per edge: d = alpha ||x_i - x_j|| + (1 - alpha) dist_y(i, j),
// written as d^2.  dist_y is Euclidean over the coordinates, each
// difference taken modulo its period when that is positive, or with
// geodesic != 0 the great-circle distance of (latitude, longitude) in
// degrees (haversine form) times the radius.
template <typename TI>
__global__ void k_edge_composite(int E, int p, const TI *X, int64_t ldx, const double *Y,
                                 int64_t ldy, CoordSpec c, const int32_t *ei, const int32_t *ej,
                                 double *d2) {
  const int e = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (e >= E) return;
  const int i = ei[e], j = ej[e];
  double acc = 0.0;
  for (int f = lane; f < p; f += kWave) {
    const double d = (double)X[(size_t)j * ldx + f] - (double)X[(size_t)i * ldx + f];
    acc = fma(d, d, acc);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (lane != 0) return;
  const double *yi = Y + (size_t)i * ldy, *yj = Y + (size_t)j * ldy;
  double dy = 0.0;
  if (c.geodesic) {
    const double r = 3.14159265358979323846 / 180.0;
    const double la1 = yi[0] * r, la2 = yj[0] * r, dla = la2 - la1, dlo = (yj[1] - yi[1]) * r;
    const double sa = sin(0.5 * dla), so = sin(0.5 * dlo);
    const double h = fmin(fmax(sa * sa + cos(la1) * cos(la2) * so * so, 0.0), 1.0);
    dy = c.radius * 2.0 * atan2(sqrt(h), sqrt(1.0 - h));
  } else {
    double s2 = 0.0;
    for (int t = 0; t < c.q; ++t) {
      double d = fabs(yj[t] - yi[t]);
      if (c.period[t] > 0.0) {
        d = fmod(d, c.period[t]);
        d = fmin(d, c.period[t] - d);
      }
      s2 = fma(d, d, s2);
    }
    dy = sqrt(s2);
  }
  const double d = c.alpha * sqrt(acc) + (1.0 - c.alpha) * dy;
  d2[e] = d * d;
}

// ====================================================================== host
struct DevBuf {
  void *p = nullptr;
  ~DevBuf() { if (p) (void)hipFree(p); }
  cc_status alloc(size_t bytes) {
    if (bytes == 0) bytes = 8;
    if (hipMalloc(&p, bytes) != hipSuccess) {
      p = nullptr;
      set_error("hipMalloc of " + std::to_string(bytes) + " bytes failed");
      return CC_ERR_OUT_OF_MEMORY;
    }
    return CC_OK;
  }
  template <typename T> T *as() const { return reinterpret_cast<T *>(p); }
};

#define KN_TRY(x)               \
  do {                          \
    cc_status _s = (x);         \
    if (_s != CC_OK) return _s; \
  } while (0)

// One device allocation cut into aligned pieces: add() every piece, then
// alloc() once.
struct Arena {
  DevBuf buf;
  size_t total = 0;
  size_t add(size_t bytes) {
    const size_t at = total;
    total += (bytes + 255) / 256 * 256;
    return at;
  }
  cc_status alloc() { return buf.alloc(total); }
  template <typename T> T *at(size_t off) const { return reinterpret_cast<T *>((char *)buf.p + off); }
};

// Sizes and buffers of the neighbour lists (steps 1-4): X~ in FP64 (Xd,
// n x p), the k nearest neighbours of every row by (exact d2, index) (knn,
// n x k), and what ranking them takes.  plan() adds the buffers to an
// arena; rank() enqueues one ranking pass.
template <typename TI> struct KnnLists {
  int64_t n, p, n_pad, ldk, rows;  // rows: of a distance panel, a multiple of the tile
  int k, K, nsplit;
  const TI *X;
  int64_t ldx;
  const uint8_t *mask;
  int64_t ldm;
  hipStream_t st;
  Arena *ar;
  size_t mean, state, Xf, Xd, nrm, D2, cand, knn, part, dnext, nmax, uncert;

  int *bad() const { return ar->at<int>(state); }          // non-finite observed entries
  int *n_uncert() const { return ar->at<int>(state) + 1; } // rows the last pass left uncertified

  void plan(Arena &a) {
    ar = &a;
    n_pad = cdiv64(n, kGT) * kGT;
    ldk = cdiv64(p, kKC) * kKC;
    K = (int)std::min<int64_t>({n - 1, (int64_t)k + std::max(16, k), kRecheckMaxK});
    rows = std::min<int64_t>(n_pad, std::max<int64_t>(kPanelBytes / (4 * n) / kGT * kGT, kGT));
    // split the features until the launch has about 4 blocks per CU (at
    // most 8 splits)
    const int64_t tiles = (n_pad / kGT) * (rows / kGT);
    nsplit = (int)std::max<int64_t>(std::min<int64_t>(std::min<int64_t>(cdiv64(1024, tiles), 8), ldk / kKC), 1);
    mean = a.add(p * 8);
    state = a.add(64);
    Xf = a.add((size_t)n_pad * ldk * 4);
    Xd = a.add((size_t)n * p * 8);
    nrm = a.add(n_pad * 4);
    D2 = a.add((size_t)rows * n * 4);
    cand = a.add((size_t)n * K * 4);
    knn = a.add((size_t)n * k * 4);
    part = a.add(nsplit > 1 ? (size_t)nsplit * rows * n_pad * 4 : 0);
    dnext = a.add(n * 4);
    nmax = a.add(4);
    uncert = a.add(n * 4);
  }

  // Steps 1 and the norms; clears the counters.
  cc_status start() {
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, ar->at<uint32_t>(state), (int64_t)16);
    moments_launch(n, p, X, ldx, mask, ldm, true, ar->at<double>(mean), (double *)nullptr, false, bad(), st);
    hipLaunchKernelGGL((k_impute<TI>), dim3((int)cdiv64(n_pad * ldk, 256)), dim3(256), 0, st, (int)n, (int)p,
                       (int)n_pad, (int)ldk, X, ldx, mask, ldm, ar->at<double>(mean), ar->at<float>(Xf),
                       ar->at<double>(Xd));
    hipLaunchKernelGGL(k_rownorm, dim3((int)n_pad), dim3(256), 0, st, (int)n_pad, (int)ldk, ar->at<float>(Xf),
                       ar->at<float>(nrm));
    hipLaunchKernelGGL(k_max_norm, dim3(1), dim3(1024), 0, st, (int)n, ar->at<float>(nrm), ar->at<float>(nmax));
    CC_HIP(hipGetLastError());
    return CC_OK;
  }

  template <int PT> void select(int64_t row0, int64_t nr, int Kp, int32_t *cp, const int *todo) {
    hipLaunchKernelGGL((k_row_select<PT>), dim3((int)nr), dim3(kSelThreads), 0, st, (int)n, (int)row0,
                       ar->at<float>(D2), n, Kp, cp, todo, ar->at<float>(dnext));
  }

  // Steps 2-4 with Kp candidates per row, over all rows or those of todo.
  cc_status rank(int Kp, int32_t *cp, const int *todo) {
    for (int64_t row0 = 0; row0 < n; row0 += rows) {
      const int64_t nr = std::min<int64_t>(rows, n - row0);
      const int gy = (int)cdiv64(nr, kGT);
      hipLaunchKernelGGL(k_gram_d2, dim3((int)(n_pad / kGT), gy, nsplit), dim3(256), 0, st, (int)n, (int)n_pad,
                         (int)ldk, nsplit, ar->at<float>(Xf), ar->at<float>(nrm), (int)row0, (int)rows,
                         ar->at<float>(D2), n, ar->at<float>(part));
      if (nsplit > 1)
        hipLaunchKernelGGL(k_gram_combine, dim3((int)cdiv64(nr * n, 256)), dim3(256), 0, st, (int)n, (int)n_pad,
                           nsplit, ar->at<float>(part), ar->at<float>(nrm), (int)row0, (int)nr, (int)rows,
                           ar->at<float>(D2), n);
      if (n <= 256) select<1>(row0, nr, Kp, cp, todo);
      else if (n <= 1024) select<4>(row0, nr, Kp, cp, todo);
      else if (n <= 2048) select<8>(row0, nr, Kp, cp, todo);
      else if (n <= 4096) select<16>(row0, nr, Kp, cp, todo);
      else if (n <= 8192) select<32>(row0, nr, Kp, cp, todo);
      else select<64>(row0, nr, Kp, cp, todo);
    }
    // rounding bound of the FP32 distances (see k_recheck): (2 m + 24) u with
    // m the longest FP32 accumulation (ldk products and the split combine)
    const double bscale = (2.0 * (double)(ldk + nsplit) + 24.0) * std::ldexp(1.0, -24) * 1.001;
    const auto recheck = rank_by_counting(Kp, k) ? k_recheck<true> : k_recheck<false>;
    // beyond what any kernel may take, the dynamic LDS limit is set to the
    // largest size (the same value on every call, so that concurrent builds
    // agree)
    if (Kp * 12 > 64 * 1024)
      CC_HIP(hipFuncSetAttribute((const void *)recheck, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)(kRecheckMaxK * 12)));
    hipLaunchKernelGGL(recheck, dim3((int)n), dim3(256), (size_t)Kp * 12, st, (int)n, (int)p, ar->at<double>(Xd), Kp,
                       k, cp, ar->at<int32_t>(knn), todo, ar->at<float>(dnext), ar->at<float>(nrm),
                       ar->at<float>(nmax), bscale, ar->at<int>(uncert), n_uncert());
    CC_HIP(hipGetLastError());
    return CC_OK;
  }

  // After the first pass left uncertified rows: wider passes over those, 8 K
  // (at least 512) candidates, then all rows up to kRecheckMaxK (every row
  // for n up to kRecheckMaxK + 1, which certifies by construction).
  cc_status widen() {
    const int64_t widths[2] = {std::min<int64_t>({n - 1, std::max<int64_t>(8 * (int64_t)K, 512), kRecheckMaxK}),
                               std::min<int64_t>(n - 1, kRecheckMaxK)};
    int Kp = K;
    for (int64_t w : widths) {
      if (w <= Kp) continue;
      Kp = (int)w;
      DevBuf wide;
      KN_TRY(wide.alloc((size_t)n * Kp * 4));
      hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, (uint32_t *)n_uncert(), (int64_t)1);
      KN_TRY(rank(Kp, wide.as<int32_t>(), ar->at<int>(uncert)));
      int hn = 0;
      CC_HIP(hipMemcpyAsync(&hn, n_uncert(), 4, hipMemcpyDeviceToHost, st));
      CC_HIP(hipStreamSynchronize(st));
      if (hn == 0) return CC_OK;
    }
    set_error("kNN: the nearest neighbours of some rows could not be certified exact "
              "(FP32 distances too close to separate them)");
    return CC_ERR_NUMERIC;
  }
};

static cc_status non_finite_error() {
  set_error("observed X has non-finite entries");
  return CC_ERR_INVALID_ARG;
}

// Step 6 over E edges with squared distances d2 (device): phi (literal, or
// |phi| / lower median of d2 when phi < 0), w = exp(-phi d2), optional
// normalisation to sum 1; phi_used (host, may be NULL) gets phi.  work: two
// device doubles.
static cc_status finish_weights(int64_t E, const double *d2, double phi, int32_t normalize,
                                double *w, double *phi_used, double *work, hipStream_t st) {
  double hphi = phi;
  const bool med = phi < 0.0 && E > 0;
  if (phi < 0.0 && E == 0) hphi = 0.0;
  if (med) hipLaunchKernelGGL(k_median_phi, dim3(1), dim3(1024), 0, st, (int)E, d2, -phi, work);
  if (E > 0) {
    const dim3 g((int)cdiv64(E, 256));
    hipLaunchKernelGGL(k_weights, g, dim3(256), 0, st, (int)E, d2, med ? work : (const double *)nullptr, hphi, w);
    if (normalize) {
      hipLaunchKernelGGL(k_weight_sum, dim3(1), dim3(1024), 0, st, (int)E, w, work + 1);
      hipLaunchKernelGGL(k_normalize, g, dim3(256), 0, st, (int)E, work + 1, w);
    }
  }
  CC_HIP(hipGetLastError());
  if (med) CC_HIP(hipMemcpyAsync(&hphi, work, 8, hipMemcpyDeviceToHost, st));
  CC_HIP(hipStreamSynchronize(st));
  if (phi_used) *phi_used = hphi;
  return CC_OK;
}

template <typename TI>
static cc_status knn_impl(int64_t n, int64_t p, const TI *X, int64_t ldx, const uint8_t *mask,
                          int64_t ldm, int32_t k, double phi, int32_t normalize, int32_t *ei,
                          int32_t *ej, double *w, int64_t capacity, int64_t *n_edges,
                          double *phi_used, hipStream_t st) {
  const int words = (int)cdiv64(n, 32);
  Arena ar;
  KnnLists<TI> L{};
  L.n = n; L.p = p; L.k = k; L.X = X; L.ldx = ldx; L.mask = mask; L.ldm = ldm; L.st = st;
  L.plan(ar);
  const size_t bm = ar.add((size_t)n * words * 4), cnt = ar.add(n * 4), off = ar.add(n * 4),
               work = ar.add(16), d2 = ar.add((size_t)n * k * 8);
  KN_TRY(ar.alloc());
  // the total number of edges sits beside the lists' counters, so that one
  // copy brings all three to the host
  int64_t *total = ar.at<int64_t>(L.state) + 1;
  const dim3 rows4((int)cdiv64(n, 4));
  auto edges = [&]() -> cc_status {  // step 5
    const int64_t nw = n * (int64_t)words;
    hipLaunchKernelGGL(k_zero_words, dim3((int)std::min<int64_t>(cdiv64(nw, 1024), 4096)), dim3(256), 0, st,
                       ar.at<uint32_t>(bm), nw);
    hipLaunchKernelGGL(k_mark_pairs, dim3((int)cdiv64(n * k, 256)), dim3(256), 0, st, (int)n, (int)k, words,
                       ar.at<int32_t>(L.knn), ar.at<uint32_t>(bm));
    hipLaunchKernelGGL(k_row_counts, rows4, dim3(256), 0, st, (int)n, words, ar.at<uint32_t>(bm),
                       ar.at<int32_t>(cnt));
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, st, (int)n, ar.at<int32_t>(cnt), ar.at<int32_t>(off), total);
    CC_HIP(hipGetLastError());
    return CC_OK;
  };
  struct { int32_t bad, uncert; int64_t total; } h{};
  auto read = [&]() -> cc_status {
    CC_HIP(hipMemcpyAsync(&h, L.bad(), sizeof(h), hipMemcpyDeviceToHost, st));
    CC_HIP(hipStreamSynchronize(st));
    return CC_OK;
  };
  KN_TRY(L.start());
  KN_TRY(L.rank(L.K, ar.at<int32_t>(L.cand), nullptr));
  KN_TRY(edges());
  KN_TRY(read());
  if (h.bad) return non_finite_error();
  if (h.uncert) {
    KN_TRY(L.widen());
    KN_TRY(edges());
    KN_TRY(read());
  }
  const int64_t E = h.total;
  *n_edges = E;
  if (E > capacity) {
    set_error("edge capacity " + std::to_string(capacity) + " < " + std::to_string(E));
    return CC_ERR_INVALID_ARG;
  }
  hipLaunchKernelGGL(k_emit_edges, rows4, dim3(256), 0, st, (int)n, words, ar.at<uint32_t>(bm),
                     ar.at<int32_t>(off), ei, ej);
  if (E > 0) {
    hipLaunchKernelGGL(k_edge_d2, dim3((int)cdiv64(E, 4)), dim3(256), 0, st, (int)E, (int)p,
                       ar.at<double>(L.Xd), ei, ej, ar.at<double>(d2));
  }
  return finish_weights(E, ar.at<double>(d2), phi, normalize, w, phi_used, ar.at<double>(work), st);
}

template <typename TI>
static cc_status min_k_impl(int64_t n, int64_t p, const TI *X, int64_t ldx, const uint8_t *mask,
                            int64_t ldm, int32_t kmax, int32_t *k_min, int32_t *n_comp,
                            hipStream_t st) {
  Arena ar;
  KnnLists<TI> L{};
  L.n = n; L.p = p; L.k = kmax; L.X = X; L.ldx = ldx; L.mask = mask; L.ldm = ldm; L.st = st;
  L.plan(ar);
  const int64_t m = n * kmax;
  const size_t aei = ar.add(m * 4), aej = ar.add(m * 4), akeep = ar.add(m), alab = ar.add(n * 4), ancl = ar.add(4);
  KN_TRY(ar.alloc());
  KN_TRY(L.start());
  KN_TRY(L.rank(L.K, ar.at<int32_t>(L.cand), nullptr));
  int32_t h[2] = {0, 0};
  CC_HIP(hipMemcpyAsync(h, L.bad(), 8, hipMemcpyDeviceToHost, st));
  CC_HIP(hipStreamSynchronize(st));
  if (h[0]) return non_finite_error();
  if (h[1]) KN_TRY(L.widen());
  int32_t *ei = ar.at<int32_t>(aei), *ej = ar.at<int32_t>(aej), *lab = ar.at<int32_t>(alab), *ncl = ar.at<int32_t>(ancl);
  uint8_t *keep = ar.at<uint8_t>(akeep);
  hipLaunchKernelGGL(k_knn_pairs, dim3((int)cdiv64(m, 256)), dim3(256), 0, st, (int)n, (int)kmax,
                     ar.at<int32_t>(L.knn), ei, ej);
  CC_HIP(hipGetLastError());
  // components of the union graph of the first k neighbours
  auto count = [&](int k, int32_t *out) -> cc_status {
    hipLaunchKernelGGL(k_keep_prefix, dim3((int)cdiv64(m, 256)), dim3(256), 0, st, m, (int)kmax, k,
                       keep);
    CC_HIP(hipGetLastError());
    KN_TRY(components(n, m, ei, ej, keep, nullptr, lab, ncl, st));
    CC_HIP(hipMemcpyAsync(out, ncl, 4, hipMemcpyDeviceToHost, st));
    CC_HIP(hipStreamSynchronize(st));
    return CC_OK;
  };
  int32_t c = 0;
  KN_TRY(count(kmax, &c));
  *n_comp = c;
  if (c != 1) {
    *k_min = -1;
    return CC_OK;
  }
  // the graph for k is a subgraph of the one for k + 1: connectivity is
  // monotone in k, so bisection finds the smallest connected k
  int lo = 1, hi = kmax;
  while (lo < hi) {
    const int mid = lo + (hi - lo) / 2;
    KN_TRY(count(mid, &c));
    if (c == 1) hi = mid;
    else lo = mid + 1;
  }
  *k_min = hi;
  return CC_OK;
}

cc_status min_connected_k(int64_t n, int64_t p, int32_t x_dtype, const void *X, int64_t ldx,
                          const uint8_t *mask, int64_t ldm, int32_t k_max, int32_t *k_min,
                          int32_t *n_components, hipStream_t stream) {
  if (n < 2 || p < 1) { set_error("need n >= 2 and p >= 1"); return CC_ERR_INVALID_ARG; }
  if (n > kKnnMaxN) { set_error("cc_min_connected_k supports n <= 16384"); return CC_ERR_INVALID_ARG; }
  if ((int64_t)n * p > ((int64_t)1 << 31) - 1) { set_error("n * p too large"); return CC_ERR_INVALID_ARG; }
  if (k_max < 1 || k_max >= n || k_max > 1024) { set_error("need 1 <= k_max < n and k_max <= 1024"); return CC_ERR_INVALID_ARG; }
  if ((int64_t)n * k_max > ((int64_t)1 << 31) - 1) { set_error("n * k_max too large"); return CC_ERR_INVALID_ARG; }
  if (!X || !k_min || !n_components) { set_error("NULL argument"); return CC_ERR_INVALID_ARG; }
  if (x_dtype != CC_DTYPE_F32 && x_dtype != CC_DTYPE_F64) { set_error("bad x_dtype"); return CC_ERR_INVALID_ARG; }
  if (ldx < p || (mask && ldm < p)) { set_error("leading dimension < p"); return CC_ERR_INVALID_ARG; }
  if (x_dtype == CC_DTYPE_F32)
    return min_k_impl<float>(n, p, (const float *)X, ldx, mask, ldm, k_max, k_min, n_components, stream);
  return min_k_impl<double>(n, p, (const double *)X, ldx, mask, ldm, k_max, k_min, n_components, stream);
}

cc_status composite_weights(int64_t n, int64_t n_edges, const int32_t *ei, const int32_t *ej,
                            int64_t p, int32_t x_dtype, const void *X, int64_t ldx,
                            const uint8_t *mask, int64_t ldm, int32_t q,
                            const double *Y, int64_t ldy, const double *period, int32_t geodesic,
                            double radius, double alpha, double phi, int32_t normalize, double *w,
                            double *phi_used, hipStream_t st) {
  if (n < 1 || p < 0 || n_edges < 0) { set_error("need n >= 1, p >= 0, n_edges >= 0"); return CC_ERR_INVALID_ARG; }
  if (n_edges > ((int64_t)1 << 31) - 1 || n > ((int64_t)1 << 31) - 1) { set_error("n or n_edges too large"); return CC_ERR_INVALID_ARG; }
  if (n_edges > 0 && (!ei || !ej || !w)) { set_error("NULL edge or weight array"); return CC_ERR_INVALID_ARG; }
  if (p > 0 && (!X || ldx < p)) { set_error("X is NULL or ldx < p"); return CC_ERR_INVALID_ARG; }
  if (mask && p > 0 && ldm < p) { set_error("ldm < p"); return CC_ERR_INVALID_ARG; }
  if (n * p > ((int64_t)1 << 31) - 1) { set_error("n * p too large"); return CC_ERR_INVALID_ARG; }
  if (x_dtype != CC_DTYPE_F32 && x_dtype != CC_DTYPE_F64) { set_error("bad x_dtype"); return CC_ERR_INVALID_ARG; }
  if (q < 0 || q > kMaxCoords) { set_error("need 0 <= q <= 8 coordinates"); return CC_ERR_INVALID_ARG; }
  if (q > 0 && (!Y || ldy < q)) { set_error("Y is NULL or ldy < q"); return CC_ERR_INVALID_ARG; }
  if (geodesic && q != 2) { set_error("geodesic distances need q = 2 (latitude, longitude in degrees)"); return CC_ERR_INVALID_ARG; }
  if (!(alpha >= 0.0 && alpha <= 1.0)) { set_error("need 0 <= alpha <= 1"); return CC_ERR_INVALID_ARG; }
  if (!std::isfinite(phi) || !std::isfinite(radius)) { set_error("phi and radius must be finite"); return CC_ERR_INVALID_ARG; }
  CoordSpec c{};
  c.q = q;
  c.geodesic = geodesic ? 1 : 0;
  c.radius = radius > 0.0 ? radius : 1.0;
  c.alpha = alpha;
  for (int t = 0; t < q; ++t) {
    c.period[t] = period ? period[t] : 0.0;
    if (!std::isfinite(c.period[t]) || c.period[t] < 0.0) { set_error("periods must be finite and >= 0"); return CC_ERR_INVALID_ARG; }
  }
  if (n_edges > 0) {  // every endpoint in range before any launch reads rows
    std::vector<int32_t> hi(n_edges), hj(n_edges);
    CC_HIP(hipMemcpyAsync(hi.data(), ei, n_edges * 4, hipMemcpyDeviceToHost, st));
    CC_HIP(hipMemcpyAsync(hj.data(), ej, n_edges * 4, hipMemcpyDeviceToHost, st));
    CC_HIP(hipStreamSynchronize(st));
    for (int64_t e = 0; e < n_edges; ++e)
      if (hi[e] < 0 || hi[e] >= n || hj[e] < 0 || hj[e] >= n) {
        set_error("edge endpoint out of range");
        return CC_ERR_INVALID_ARG;
      }
  }
  // with a mask: distances on the mean-imputed matrix (FP64)
  DevBuf mean, bad, Xd;
  const void *Xuse = X;
  int64_t ldu = ldx;
  int32_t tuse = x_dtype;
  if (mask && p > 0 && n_edges > 0) {
    KN_TRY(mean.alloc(p * 8));
    KN_TRY(bad.alloc(4));
    KN_TRY(Xd.alloc((size_t)n * p * 8));
    CC_HIP(hipMemsetAsync(bad.p, 0, 4, st));
    const int eb = (int)cdiv64(n * p, 256);
    column_moments(n, p, x_dtype, X, ldx, mask, ldm, true, mean.as<double>(), nullptr, false, bad.as<int>(), st);
    if (x_dtype == CC_DTYPE_F32) {
      hipLaunchKernelGGL((k_impute_d<float>), dim3(eb), dim3(256), 0, st, (int)n, (int)p, (const float *)X, ldx,
                         mask, ldm, mean.as<double>(), Xd.as<double>());
    } else {
      hipLaunchKernelGGL((k_impute_d<double>), dim3(eb), dim3(256), 0, st, (int)n, (int)p, (const double *)X, ldx,
                         mask, ldm, mean.as<double>(), Xd.as<double>());
    }
    CC_HIP(hipGetLastError());
    int hbad = 0;
    CC_HIP(hipMemcpyAsync(&hbad, bad.p, 4, hipMemcpyDeviceToHost, st));
    CC_HIP(hipStreamSynchronize(st));
    if (hbad) return non_finite_error();
    Xuse = Xd.p;
    ldu = p;
    tuse = CC_DTYPE_F64;
  }
  DevBuf d2;
  KN_TRY(d2.alloc((n_edges + 2) * 8));
  if (n_edges > 0) {
    const int blocks = (int)cdiv64(n_edges, 4);
    if (tuse == CC_DTYPE_F32)
      hipLaunchKernelGGL((k_edge_composite<float>), dim3(blocks), dim3(256), 0, st, (int)n_edges,
                         (int)p, (const float *)Xuse, ldu, Y, ldy, c, ei, ej, d2.as<double>());
    else
      hipLaunchKernelGGL((k_edge_composite<double>), dim3(blocks), dim3(256), 0, st, (int)n_edges,
                         (int)p, (const double *)Xuse, ldu, Y, ldy, c, ei, ej, d2.as<double>());
    CC_HIP(hipGetLastError());
  }
  return finish_weights(n_edges, d2.as<double>(), phi, normalize, w, phi_used, d2.as<double>() + n_edges, st);
}

cc_status build_knn_weights(int64_t n, int64_t p, int32_t x_dtype, const void *X, int64_t ldx,
                            const uint8_t *mask, int64_t ldm, int32_t k, double phi,
                            int32_t normalize, int32_t *ei, int32_t *ej, double *w,
                            int64_t capacity, int64_t *n_edges, double *phi_used,
                            hipStream_t stream) {
  if (n < 2 || p < 1) { set_error("need n >= 2 and p >= 1"); return CC_ERR_INVALID_ARG; }
  if (n > kKnnMaxN) { set_error("cc_build_knn_weights supports n <= 16384"); return CC_ERR_INVALID_ARG; }
  if ((int64_t)n * p > ((int64_t)1 << 31) - 1) { set_error("n * p too large"); return CC_ERR_INVALID_ARG; }
  if (k < 1 || k >= n) { set_error("need 1 <= k < n"); return CC_ERR_INVALID_ARG; }
  if (k > kRecheckMaxK) { set_error("cc_build_knn_weights supports k <= 12288"); return CC_ERR_INVALID_ARG; }
  if (!X || !ei || !ej || !w || !n_edges) { set_error("NULL argument"); return CC_ERR_INVALID_ARG; }
  if (x_dtype != CC_DTYPE_F32 && x_dtype != CC_DTYPE_F64) { set_error("bad x_dtype"); return CC_ERR_INVALID_ARG; }
  if (ldx < p || (mask && ldm < p)) { set_error("leading dimension < p"); return CC_ERR_INVALID_ARG; }
  if (!std::isfinite(phi)) { set_error("phi must be finite"); return CC_ERR_INVALID_ARG; }
  if (capacity < 0) { set_error("capacity < 0"); return CC_ERR_INVALID_ARG; }
  if (x_dtype == CC_DTYPE_F32)
    return knn_impl<float>(n, p, (const float *)X, ldx, mask, ldm, k, phi, normalize, ei, ej, w,
                           capacity, n_edges, phi_used, stream);
  return knn_impl<double>(n, p, (const double *)X, ldx, mask, ldm, k, phi, normalize, ei, ej, w,
                          capacity, n_edges, phi_used, stream);
}

cc_status standardize_columns(int64_t n, int64_t p, int32_t x_dtype, void *X, int64_t ldx,
                              const uint8_t *mask, int64_t ldm, hipStream_t st) {
  if (n < 1 || p < 1) { set_error("need n, p >= 1"); return CC_ERR_INVALID_ARG; }
  if (!X) { set_error("X is NULL"); return CC_ERR_INVALID_ARG; }
  if (ldx < p || (mask && ldm < p)) { set_error("leading dimension < p"); return CC_ERR_INVALID_ARG; }
  if (x_dtype != CC_DTYPE_F32 && x_dtype != CC_DTYPE_F64) { set_error("bad x_dtype"); return CC_ERR_INVALID_ARG; }
  if ((int64_t)n * p > ((int64_t)1 << 31) - 1) { set_error("n * p too large"); return CC_ERR_INVALID_ARG; }
  DevBuf mean, sd, bad;
  KN_TRY(mean.alloc(p * 8));
  KN_TRY(sd.alloc(p * 8));
  KN_TRY(bad.alloc(4));
  CC_HIP(hipMemsetAsync(bad.p, 0, 4, st));
  const int eb = (int)cdiv64(n * p, 256);
  column_moments(n, p, x_dtype, X, ldx, mask, ldm, true, mean.as<double>(), sd.as<double>(), true, bad.as<int>(), st);
  int hbad = 0;
  CC_HIP(hipMemcpyAsync(&hbad, bad.p, 4, hipMemcpyDeviceToHost, st));
  CC_HIP(hipStreamSynchronize(st));
  if (hbad) return non_finite_error();
  if (x_dtype == CC_DTYPE_F32)
    hipLaunchKernelGGL((k_standardize<float>), dim3(eb), dim3(256), 0, st, (int)n, (int)p,
                       (float *)X, ldx, mask, ldm, mean.as<double>(), sd.as<double>());
  else
    hipLaunchKernelGGL((k_standardize<double>), dim3(eb), dim3(256), 0, st, (int)n, (int)p,
                       (double *)X, ldx, mask, ldm, mean.as<double>(), sd.as<double>());
  CC_HIP(hipGetLastError());
  CC_HIP(hipStreamSynchronize(st));
  return CC_OK;
}

// ------------------------------------------- standardisation without allocation
// cc_standardize_columns_noalloc keeps the column statistics in this fixed
// device array instead of memory allocated per call: the means, then the
// standard deviations (kStdMaxCols doubles each), then the count of
// non-finite observed entries.  Each GPU holds its own copy; host code uses
// the device address hipGetSymbolAddress gives on that GPU, never the
// array's name.
constexpr int64_t kStdMaxCols = 65536;
static __device__ __align__(256) double scratch[2 * kStdMaxCols + 32];

constexpr int kMaxScratchDevices = 256;
static std::mutex g_scratch_mutex;
static void *g_scratch_addr[kMaxScratchDevices];

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept.
static cc_status scratch_address(void **out) {
  int dev = 0;
  CC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxScratchDevices) {
    set_error("device index beyond the library's scratch table");
    return CC_ERR_STATE;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[dev]) {
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) {
      set_error("hipGetSymbolAddress(scratch) gave no address");
      return CC_ERR_HIP;
    }
    g_scratch_addr[dev] = ptr;
  }
  *out = g_scratch_addr[dev];
  return CC_OK;
}

__global__ void k_zero_count(int *count) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *count = 0;
}

cc_status standardize_columns_noalloc(int64_t n, int64_t p, int32_t x_dtype, void *X, int64_t ldx,
                                      const uint8_t *mask, int64_t ldm, hipStream_t st) {
  if (n < 1 || p < 1) { set_error("need n, p >= 1"); return CC_ERR_INVALID_ARG; }
  if (!X) { set_error("X is NULL"); return CC_ERR_INVALID_ARG; }
  if (ldx < p || (mask && ldm < p)) { set_error("leading dimension < p"); return CC_ERR_INVALID_ARG; }
  if (x_dtype != CC_DTYPE_F32 && x_dtype != CC_DTYPE_F64) { set_error("bad x_dtype"); return CC_ERR_INVALID_ARG; }
  if ((int64_t)n * p > ((int64_t)1 << 31) - 1) { set_error("n * p too large"); return CC_ERR_INVALID_ARG; }
  if (p > kStdMaxCols) {
    set_error("cc_standardize_columns_noalloc takes p <= " + std::to_string(kStdMaxCols) +
              " (the size of its fixed device scratch)");
    return CC_ERR_INVALID_ARG;
  }
  void *base = nullptr;
  KN_TRY(scratch_address(&base));
  double *mean = reinterpret_cast<double *>(base);
  double *sd = mean + kStdMaxCols;
  int *bad = reinterpret_cast<int *>(sd + kStdMaxCols);
  // the array keeps the last call's contents: the count starts at zero
  hipLaunchKernelGGL(k_zero_count, dim3(1), dim3(64), 0, st, bad);
  const int eb = (int)cdiv64(n * p, 256);
  column_moments(n, p, x_dtype, X, ldx, mask, ldm, true, mean, sd, true, bad, st);
  CC_HIP(hipGetLastError());
  int hbad = 0;
  CC_HIP(hipMemcpyAsync(&hbad, bad, 4, hipMemcpyDeviceToHost, st));
  CC_HIP(hipStreamSynchronize(st));
  if (hbad) return non_finite_error();
  if (x_dtype == CC_DTYPE_F32)
    hipLaunchKernelGGL((k_standardize<float>), dim3(eb), dim3(256), 0, st, (int)n, (int)p,
                       (float *)X, ldx, mask, ldm, mean, sd);
  else
    hipLaunchKernelGGL((k_standardize<double>), dim3(eb), dim3(256), 0, st, (int)n, (int)p,
                       (double *)X, ldx, mask, ldm, mean, sd);
  CC_HIP(hipGetLastError());
  CC_HIP(hipStreamSynchronize(st));
  return CC_OK;
}

}  // namespace ccmi
