// Principal components of the data and the projection of the cluster path
// onto them, on the device (Evaluation of Clusters: the path is viewed on
// principal components of the original data; Discussion: projecting on the
// GPU before any transfer saves moving U off the device for every gamma).
//
// cc_pca: X~ = X with missing entries replaced by their observed column
// means, centred by those means (C = X~ - 1 mean^T, FP64 throughout).  The
// top r right singular vectors of C come from subspace iteration on C^T C
// with s = min(r + 8, p) columns: Q <- orth(C^T (C Q)), from counter-based
// start vectors; then a Rayleigh-Ritz step: the eigenpairs of (C Q)^T (C Q)
// by cyclic Jacobi rotations give V = Q W and the singular values
// sqrt(lambda).
//
// orth between steps: with R^T R = Q^T Q (Cholesky), the step multiplies C Q
// by R^-1, which is C times the orthonormal columns.  R does not depend on
// how columns are scaled, so near convergence, where the columns are nearly
// orthogonal with norms sigma^2, it is as accurate as Gram-Schmidt.  Columns
// that are nearly dependent (a pivot small against its column: a new start,
// a spectrum that falls by orders of magnitude, fewer than s nonzero singular
// values) are orthonormalised by Gram-Schmidt instead, as the last step's
// always are.
// Each column of V is signed so that its entry of largest magnitude (the
// first such on ties) is positive.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>

#include "ccmi_internal.h"
#include "wave_ops.h"

namespace ccmi {
namespace {

constexpr int kMaxR = 16;   // principal components returned
constexpr int kMaxS = 24;   // subspace columns
constexpr int kOrthThreads = 1024;

inline int64_t cdivx(int64_t a, int64_t b) { return (a + b - 1) / b; }

__device__ inline double wsum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// C = X~ - mean (a missing entry becomes 0), n x p dense.
template <typename TI>
__global__ void k_pca_center(int n, int p, const TI *X, int64_t ldx, const uint8_t *M, int64_t ldm,
                             const double *mean, double *C) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * p) return;
  const int i = (int)(e / p), f = (int)(e - (int64_t)i * p);
  const bool obs = !M || M[(size_t)i * ldm + f];
  C[e] = obs ? (double)X[(size_t)i * ldx + f] - mean[f] : 0.0;
}

// Start vectors: SplitMix64 of the element index, mapped to [-1, 1).
__global__ void k_pca_start(int64_t m, double *Q) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= m) return;
  uint64_t z = (uint64_t)(e + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  Q[e] = (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// B = C Q R^-1 (n x s; Rinv may be NULL: the identity).  A block of 4 waves
// takes 8 rows, two per wave; Q passes through LDS in chunks of kCqChunk
// features, so each of its entries is read from L2 once per 8 rows and the
// C rows are read whole.  14.4 us at 2000 x 500 (8 MB of C): bound by the chain
// of chunks a block passes through, one wave per SIMD.
constexpr int kCqChunk = 128;

template <int S>
__global__ __launch_bounds__(256) void k_pca_cq(int n, int p, int s, const double *C, const double *Q,
                                               const double *Rinv, double *B) {
  constexpr int LD = S | 1;  // odd row stride: 64 lanes on different banks
  __shared__ double q[kCqChunk * LD];
  __shared__ double raw[8][S];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int i0 = blockIdx.x * 8 + 2 * wave;
  const double *c0 = C + (size_t)min(i0, n - 1) * p, *c1 = C + (size_t)min(i0 + 1, n - 1) * p;
  double acc[2][S];
#pragma unroll
  for (int c = 0; c < S; ++c) acc[0][c] = acc[1][c] = 0.0;
  for (int f0 = 0; f0 < p; f0 += kCqChunk) {
    const int nf = min(kCqChunk, p - f0);
    double x0[kCqChunk / kWave], x1[kCqChunk / kWave];
#pragma unroll
    for (int u = 0; u < kCqChunk / kWave; ++u) {
      const int f = lane + u * kWave;
      x0[u] = f < nf ? c0[f0 + f] : 0.0;
      x1[u] = f < nf ? c1[f0 + f] : 0.0;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kCqChunk * s; e += 256) {
      const int f = e / s, c = e - f * s;
      q[f * LD + c] = f < nf ? Q[(size_t)f0 * s + e] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCqChunk / kWave; ++u) {
#pragma unroll
      for (int c = 0; c < S; ++c) {
        if (c < s) {
          const double v = q[(lane + u * kWave) * LD + c];
          acc[0][c] = fma(x0[u], v, acc[0][c]);
          acc[1][c] = fma(x1[u], v, acc[1][c]);
        }
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int g = 0; g < S; g += 8) {
      double v[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = acc[h][g + c];
      const double t = wave_sum8_groups(v);
      if ((lane & 7) == 0) raw[2 * wave + h][g + lane / 8] = t;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 8 * s; e += 256) {
    const int r = e / s, c = e - r * s;
    const int i = blockIdx.x * 8 + r;
    if (i >= n) continue;
    double b = raw[r][c];
    if (Rinv) {
      b = 0.0;
      for (int k = 0; k <= c; ++k) b = fma(raw[r][k], Rinv[k * s + c], b);
    }
    B[(size_t)i * s + c] = b;
  }
}

// Partial sums of Q = C^T B over a chunk of `per` groups of kCtbRows rows:
// part[chunk] (p x s).  A block takes 64 features and a chunk, its 4 waves
// every fourth row; a group's rows of B are in LDS, the 16 rows of C a lane
// reads are in flight together.  Splitting the rows is what fills the chip: a
// thread per feature over all rows left 2 blocks working (1459 us a step at
// 2000 x 500, 11 us here).
constexpr int kCtbRows = 64;

template <int S>
__global__ __launch_bounds__(256) void k_pca_ctb(int n, int p, int s, int per, const double *C, const double *B,
                                                double *part) {
  __shared__ double b[kCtbRows * S];
  __shared__ double red[4][kWave][S + 1];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int f = blockIdx.x * kWave + lane;
  double acc[S];
#pragma unroll
  for (int c = 0; c < S; ++c) acc[c] = 0.0;
  for (int g = 0; g < per; ++g) {
    const int i0 = (blockIdx.y * per + g) * kCtbRows;
    if (i0 >= n) break;
    const int ni = min(kCtbRows, n - i0);
    double x[kCtbRows / 4];
#pragma unroll
    for (int u = 0; u < kCtbRows / 4; ++u) {
      const int i = 4 * u + wave;
      x[u] = (f < p && i < ni) ? C[(size_t)(i0 + i) * p + f] : 0.0;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kCtbRows * s; e += 256) {
      const int r = e / s, c = e - r * s;
      b[r * S + c] = r < ni ? B[(size_t)i0 * s + e] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCtbRows / 4; ++u) {
#pragma unroll
      for (int c = 0; c < S; ++c)
        if (c < s) acc[c] = fma(x[u], b[(4 * u + wave) * S + c], acc[c]);
    }
  }
#pragma unroll
  for (int c = 0; c < S; ++c) red[wave][lane][c] = acc[c];
  __syncthreads();
  const int nf = min(kWave, p - (int)blockIdx.x * kWave);
  double *o = part + ((size_t)blockIdx.y * p + (size_t)blockIdx.x * kWave) * s;
  for (int e = threadIdx.x; e < nf * s; e += 256) {
    const int l = e / s, c = e - l * s;
    o[e] = ((red[0][l][c] + red[1][l][c]) + red[2][l][c]) + red[3][l][c];
  }
}

// Sum of the chunks' partials (rows x s each; chunks added in order) into Q
// (NULL: not stored), and the Gram matrix of the block's 32 rows of it:
// gram[block] (s x s).  Entries (a, b) and (b, a) add the same products in
// the same order.
constexpr int kGramRows = 32;

__global__ __launch_bounds__(256) void k_pca_reduce_gram(int rows, int s, int chunks, const double *part, double *Q,
                                                        double *gram) {
  __shared__ double q[kGramRows * kMaxS];
  const int r0 = blockIdx.x * kGramRows, nr = min(kGramRows, rows - r0);
  const size_t stride = (size_t)rows * s;
  for (int e = threadIdx.x; e < nr * s; e += 256) {
    const double *src = part + (size_t)r0 * s + e;
    double t = 0.0;
#pragma unroll 8
    for (int k = 0; k < chunks; ++k) t += src[k * stride];
    q[e] = t;
    if (Q) Q[(size_t)r0 * s + e] = t;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < s * s; e += 256) {
    const int a = e / s, b = e - a * s;
    double t = 0.0;
    for (int r = 0; r < nr; ++r) t = fma(q[r * s + a], q[r * s + b], t);
    gram[(size_t)blockIdx.x * s * s + e] = t;
  }
}

// The blocks' Gram matrices added in order, by all threads of a block of
// 1024, up to 16 per entry: H in LDS.  red: 1024 doubles.
__device__ inline void sum_grams(int s, int blocks, const double *gram, double *H, double *red) {
  const int ss = s * s;
  const int per = max(1, min(16, (int)blockDim.x / ss));
  const int e = threadIdx.x % ss, g = threadIdx.x / ss;
  double t = 0.0;
  if (g < per) {
#pragma unroll 4
    for (int k = g; k < blocks; k += per) t += gram[(size_t)k * ss + e];
    red[g * ss + e] = t;
  }
  __syncthreads();
  if (g == 0) {
    for (int q = 1; q < per; ++q) t += red[q * ss + e];
    H[e] = t;
  }
  __syncthreads();
}

// Gram-Schmidt over the columns of Q (p x s): a pass takes the inner products
// with all earlier columns at once.  Two passes per column, and more while a
// pass still takes away over half of the column: what is left of a column in
// the span of the earlier ones is rounding noise, which has to be made
// orthogonal in its turn (the columns of fewer than s nonzero singular
// values; with two passes alone the noise stays in the span).  A column that
// vanishes stays zero.  One block; every thread owns the same rows
// f = tid + k * blockDim in every step.  red: (waves + 1) * kMaxS doubles.
constexpr int kOrthPasses = 6;

__device__ inline void gram_schmidt(int p, int s, double *Q, double *red) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  constexpr int NW = kOrthThreads / kWave;
  double *tot = red + NW * kMaxS;
  for (int j = 0; j < s; ++j) {
    double nn = 0.0, before = 0.0;  // squared norm of the column, and one pass ago
    for (int pass = 0;; ++pass) {
      auto products = [&](int a, int b) {
        for (int g = a; g < b; g += 8) {
          double d[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) d[k] = 0.0;
          for (int f = threadIdx.x; f < p; f += kOrthThreads) {
            const double qj = Q[(size_t)f * s + j];
#pragma unroll
            for (int k = 0; k < 8; ++k)
              if (g + k < b) d[k] = fma(Q[(size_t)f * s + g + k], qj, d[k]);
          }
          const double t = wave_sum8_groups(d);
          if ((lane & 7) == 0) red[wave * kMaxS + (g - a) + lane / 8] = t;
        }
        __syncthreads();
        if ((int)threadIdx.x < b - a) {
          double t = 0.0;
          for (int w = 0; w < NW; ++w) t += red[w * kMaxS + threadIdx.x];
          tot[a + threadIdx.x] = t;
        }
        __syncthreads();
      };
      // the norm beside the products in pass 1, by itself first from then on
      products(pass < 2 ? 0 : j, pass == 0 ? j : j + 1);
      nn = pass == 0 ? 0.0 : tot[j];
      if (pass >= 2) {  // uniform
        if (nn >= 0.25 * before || !(nn > 0.0) || pass == kOrthPasses) break;
        products(0, j);
      }
      before = nn;
      for (int f = threadIdx.x; f < p; f += kOrthThreads) {
        double qj = Q[(size_t)f * s + j];
        for (int k = 0; k < j; ++k) qj = fma(-tot[k], Q[(size_t)f * s + k], qj);
        Q[(size_t)f * s + j] = qj;
      }
      __syncthreads();  // tot is read before the next pass writes it
    }
    // still falling: nothing of it is outside the span (C^T reaches no further
    // features than the earlier columns hold)
    const double inv = nn > 0.0 && nn >= 0.25 * before ? 1.0 / sqrt(nn) : 0.0;
    for (int f = threadIdx.x; f < p; f += kOrthThreads) Q[(size_t)f * s + j] *= inv;
    __syncthreads();
  }
}

__global__ __launch_bounds__(kOrthThreads) void k_pca_orth(int p, int s, double *Q) {
  __shared__ double red[(kOrthThreads / kWave + 1) * kMaxS];
  gram_schmidt(p, s, Q, red);
}

// R^-1 of the Cholesky factor of Q^T Q (the blocks' Gram matrices added); a
// pivot below kPivot of its diagonal entry (a column whose part outside the
// earlier ones is under 1e-3 of it, where squaring would cost six digits)
// sends Q through Gram-Schmidt instead, and R^-1 is the identity.
constexpr double kPivot = 1e-6;

__global__ __launch_bounds__(kOrthThreads) void k_pca_chol(int p, int s, int blocks, const double *gram, double *Q,
                                                          double *Rinv) {
  __shared__ double H[kMaxS * kMaxS], R[kMaxS * kMaxS];
  __shared__ double red[kOrthThreads];
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  sum_grams(s, blocks, gram, H, red);
  const int t = threadIdx.x;
  // column by column: R[k][j], k <= j (lane j holds column j)
  if (t < kWave) {
    for (int k = 0; k < s; ++k) {
      double piv = H[k * s + k];
      for (int u = 0; u < k; ++u) piv = fma(-R[u * s + k], R[u * s + k], piv);
      const bool ok = piv > kPivot * H[k * s + k];
      if (!ok && t == 0) bad = 1;
      const double rk = ok ? sqrt(piv) : 1.0, inv = 1.0 / rk;
      if (t >= k && t < s) {
        double h = H[k * s + t];
        for (int u = 0; u < k; ++u) h = fma(-R[u * s + k], R[u * s + t], h);
        R[k * s + t] = t == k ? rk : h * inv;
      }
      __builtin_amdgcn_wave_barrier();
      __threadfence_block();
    }
  }
  __syncthreads();
  if (bad) {
    gram_schmidt(p, s, Q, red);
    for (int e = t; e < s * s; e += kOrthThreads) Rinv[e] = (e / s == e % s) ? 1.0 : 0.0;
    return;
  }
  // back substitution for column t of R^-1 (in H, which is free now)
  if (t < s) {
    for (int k = s - 1; k >= 0; --k) {
      double v = 0.0;
      if (k <= t) {
        v = k == t ? 1.0 : 0.0;
        for (int u = k + 1; u <= t; ++u) v = fma(-R[k * s + u], H[u * s + t], v);
        v /= R[k * s + k];
      }
      H[k * s + t] = v;
      Rinv[k * s + t] = v;
    }
  }
}

// H = B^T B from the blocks' Gram matrices.
__global__ __launch_bounds__(1024) void k_pca_gram(int s, int blocks, const double *gram, double *H) {
  __shared__ double h[kMaxS * kMaxS], red[1024];
  sum_grams(s, blocks, gram, h, red);
  for (int e = threadIdx.x; e < s * s; e += 1024) H[e] = h[e];
}

// Eigenpairs of the symmetric s x s matrix H by cyclic Jacobi rotations in
// LDS (one wave; thread t updates row or column entry t), sorted by
// decreasing eigenvalue: lam (s), W (s x s, eigenvectors in columns).
__global__ __launch_bounds__(kWave) void k_pca_eig(int s, const double *Hg, double *Wg, double *lam) {
  __shared__ double H[kMaxS][kMaxS], W[kMaxS][kMaxS];
  __shared__ int order[kMaxS];
  const int t = threadIdx.x;
  for (int e = t; e < s * s; e += kWave) {
    const int a = e / s, b = e - a * s;
    H[a][b] = Hg[e];
    W[a][b] = (a == b) ? 1.0 : 0.0;
  }
  __syncthreads();
  for (int sweep = 0; sweep < 64; ++sweep) {
    double off = 0.0, dia = 0.0;
    for (int a = 0; a < s; ++a) {
      dia = fma(H[a][a], H[a][a], dia);
      for (int b = a + 1; b < s; ++b) off = fma(H[a][b], H[a][b], off);
    }
    if (!(off > 1e-32 * dia)) break;  // the same decision in every thread
    for (int a = 0; a < s - 1; ++a) {
      for (int b = a + 1; b < s; ++b) {
        const double hab = H[a][b];
        if (hab == 0.0) continue;
        const double tau = (H[b][b] - H[a][a]) / (2.0 * hab);
        const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(fma(tau, tau, 1.0)));
        const double c = 1.0 / sqrt(fma(tt, tt, 1.0)), sn = tt * c;
        __syncthreads();
        if (t < s) {
          const double ha = H[a][t], hb = H[b][t];
          H[a][t] = c * ha - sn * hb;
          H[b][t] = sn * ha + c * hb;
        }
        __syncthreads();
        if (t < s) {
          const double ha = H[t][a], hb = H[t][b];
          H[t][a] = c * ha - sn * hb;
          H[t][b] = sn * ha + c * hb;
          const double wa = W[t][a], wb = W[t][b];
          W[t][a] = c * wa - sn * wb;
          W[t][b] = sn * wa + c * wb;
        }
        __syncthreads();
      }
    }
  }
  if (t == 0) {
    // insertion sort by decreasing eigenvalue; equal values keep their order
    for (int a = 0; a < s; ++a) order[a] = a;
    for (int a = 1; a < s; ++a) {
      const int v = order[a];
      const double key = H[v][v];
      int b = a - 1;
      while (b >= 0 && H[order[b]][order[b]] < key) {
        order[b + 1] = order[b];
        --b;
      }
      order[b + 1] = v;
    }
  }
  __syncthreads();
  for (int e = t; e < s * s; e += kWave) {
    const int a = e / s, c = e - a * s;
    Wg[e] = W[a][order[c]];
  }
  if (t < s) lam[t] = H[order[t]][order[t]];
}

// V = Q W[:, :r] (p x r).
__global__ void k_pca_rotate(int p, int s, int r, const double *Q, const double *W, double *V) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)p * r) return;
  const int f = (int)(e / r), c = (int)(e - (int64_t)f * r);
  double acc = 0.0;
  for (int u = 0; u < s; ++u) acc = fma(Q[(size_t)f * s + u], W[(size_t)u * s + c], acc);
  V[e] = acc;
}

// Sign of each column: its entry of largest magnitude (first on ties) > 0.
__global__ __launch_bounds__(kOrthThreads) void k_pca_sign(int p, int r, double *V) {
  __shared__ double bv[kOrthThreads / kWave];
  __shared__ int bi[kOrthThreads / kWave];
  __shared__ double flip;
  for (int c = 0; c < r; ++c) {
    double best = -1.0;
    int idx = p;
    for (int f = threadIdx.x; f < p; f += blockDim.x) {
      const double a = fabs(V[(size_t)f * r + c]);
      if (a > best) { best = a; idx = f; }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double ob = __shfl_xor(best, off, kWave);
      const int oi = __shfl_xor(idx, off, kWave);
      if (ob > best || (ob == best && oi < idx)) { best = ob; idx = oi; }
    }
    if (threadIdx.x % kWave == 0) { bv[threadIdx.x / kWave] = best; bi[threadIdx.x / kWave] = idx; }
    __syncthreads();
    if (threadIdx.x == 0) {
      double b = -1.0;
      int k = p;
      for (int w = 0; w < (int)(blockDim.x / kWave); ++w)
        if (bv[w] > b || (bv[w] == b && bi[w] < k)) { b = bv[w]; k = bi[w]; }
      flip = (k < p && V[(size_t)k * r + c] < 0.0) ? -1.0 : 1.0;
    }
    __syncthreads();
    const double sg = flip;
    for (int f = threadIdx.x; f < p; f += blockDim.x) V[(size_t)f * r + c] *= sg;
    __syncthreads();
  }
}

// out (n x r) = (U - center) V: one wave per row of U (row stride ld).
template <typename TS>
__global__ __launch_bounds__(256) void k_project(int n, int p, int ld, const TS *U, int r,
                                                const double *V, const double *center, double *out) {
  const int i = blockIdx.x * 4 + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (i >= n) return;
  double acc[kMaxR];
#pragma unroll
  for (int c = 0; c < kMaxR; ++c) acc[c] = 0.0;
  for (int f = lane; f < p; f += kWave) {
    const double u = (double)U[(size_t)i * ld + f] - (center ? center[f] : 0.0);
    const double *v = V + (size_t)f * r;
#pragma unroll
    for (int c = 0; c < kMaxR; ++c)
      if (c < r) acc[c] = fma(u, v[c], acc[c]);
  }
#pragma unroll
  for (int c = 0; c < kMaxR; ++c) acc[c] = wsum(acc[c]);
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < kMaxR; ++c)
      if (c < r) out[(size_t)i * r + c] = acc[c];
  }
}

struct Buf {
  void *p = nullptr;
  ~Buf() { if (p) (void)hipFree(p); }
  cc_status alloc(size_t bytes) {
    if (hipMalloc(&p, bytes ? bytes : 8) != hipSuccess) {
      p = nullptr;
      set_error("hipMalloc of " + std::to_string(bytes) + " bytes failed");
      return CC_ERR_OUT_OF_MEMORY;
    }
    return CC_OK;
  }
  double *d() const { return reinterpret_cast<double *>(p); }
};

#define PC_TRY(x)               \
  do {                          \
    cc_status _s = (x);         \
    if (_s != CC_OK) return _s; \
  } while (0)

// Row groups per chunk of k_pca_ctb: one while the launch has at most about
// 2048 blocks (8 per CU), which bounds the partials at 2048 x 64 x s and one
// p x s.
inline int64_t ctb_per(int64_t n, int64_t p) {
  return std::max<int64_t>(1, cdivx(cdivx(n, kCtbRows) * cdivx(p, kWave), 2048));
}
inline int64_t ctb_chunks(int64_t n, int64_t p) { return cdivx(cdivx(n, kCtbRows), ctb_per(n, p)); }

template <int S>
void subspace(int n, int p, int s, int iters, const double *C, double *Q, double *B, double *part, double *gram,
              double *Rinv, hipStream_t st) {
  const int chunks = (int)ctb_chunks(n, p), per = (int)ctb_per(n, p), gb = (int)cdivx(p, kGramRows);
  const dim3 gcq((int)cdivx(n, 8)), gct((int)cdivx(p, kWave), chunks);
  for (int it = 0; it < iters; ++it) {
    hipLaunchKernelGGL((k_pca_cq<S>), gcq, dim3(256), 0, st, n, p, s, C, Q, it ? Rinv : (const double *)nullptr, B);
    hipLaunchKernelGGL((k_pca_ctb<S>), gct, dim3(256), 0, st, n, p, s, per, C, B, part);
    hipLaunchKernelGGL(k_pca_reduce_gram, dim3(gb), dim3(256), 0, st, p, s, chunks, part, Q, gram);
    // the last step's columns are orthonormalised themselves
    if (it + 1 < iters)
      hipLaunchKernelGGL(k_pca_chol, dim3(1), dim3(kOrthThreads), 0, st, p, s, gb, gram, Q, Rinv);
  }
  hipLaunchKernelGGL(k_pca_orth, dim3(1), dim3(kOrthThreads), 0, st, p, s, Q);
  hipLaunchKernelGGL((k_pca_cq<S>), gcq, dim3(256), 0, st, n, p, s, C, Q, (const double *)nullptr, B);
}

template <typename TI>
cc_status pca_impl(int n, int p, const TI *X, int64_t ldx, const uint8_t *M, int64_t ldm, int r,
                   int iters, double *V, double *sval, double *center, hipStream_t st) {
  const int s = std::min(std::min(r + 8, p), kMaxS);
  const int64_t chunks = ctb_chunks(n, p), grams = std::max(cdivx(n, kGramRows), cdivx(p, kGramRows));
  Buf mean, C, Q, B, H, W, lam, part, gram;
  PC_TRY(mean.alloc((size_t)p * 8));
  PC_TRY(C.alloc((size_t)n * p * 8));
  PC_TRY(Q.alloc((size_t)p * s * 8));
  PC_TRY(B.alloc((size_t)n * s * 8));
  PC_TRY(H.alloc((size_t)s * s * 8));
  PC_TRY(W.alloc((size_t)s * s * 8));
  PC_TRY(lam.alloc((size_t)s * 8));
  PC_TRY(part.alloc((size_t)chunks * p * s * 8));
  PC_TRY(gram.alloc((size_t)grams * s * s * 8));
  column_moments(n, p, std::is_same<TI, float>::value ? CC_DTYPE_F32 : CC_DTYPE_F64, X, ldx, M, ldm, false,
                 mean.d(), nullptr, false, nullptr, st);
  hipLaunchKernelGGL((k_pca_center<TI>), dim3((int)cdivx((int64_t)n * p, 256)), dim3(256), 0, st, n,
                     p, X, ldx, M, ldm, mean.d(), C.d());
  hipLaunchKernelGGL(k_pca_start, dim3((int)cdivx((int64_t)p * s, 256)), dim3(256), 0, st,
                     (int64_t)p * s, Q.d());
  hipLaunchKernelGGL(k_pca_orth, dim3(1), dim3(kOrthThreads), 0, st, p, s, Q.d());
  CC_HIP(hipGetLastError());
  if (s <= 8) subspace<8>(n, p, s, iters, C.d(), Q.d(), B.d(), part.d(), gram.d(), W.d(), st);
  else if (s <= 16) subspace<16>(n, p, s, iters, C.d(), Q.d(), B.d(), part.d(), gram.d(), W.d(), st);
  else subspace<24>(n, p, s, iters, C.d(), Q.d(), B.d(), part.d(), gram.d(), W.d(), st);
  const int gb = (int)cdivx(n, kGramRows);
  hipLaunchKernelGGL(k_pca_reduce_gram, dim3(gb), dim3(256), 0, st, n, s, 1, B.d(), (double *)nullptr, gram.d());
  hipLaunchKernelGGL(k_pca_gram, dim3(1), dim3(1024), 0, st, s, gb, gram.d(), H.d());
  hipLaunchKernelGGL(k_pca_eig, dim3(1), dim3(kWave), 0, st, s, H.d(), W.d(), lam.d());
  hipLaunchKernelGGL(k_pca_rotate, dim3((int)cdivx((int64_t)p * r, 256)), dim3(256), 0, st, p, s, r,
                     Q.d(), W.d(), V);
  hipLaunchKernelGGL(k_pca_sign, dim3(1), dim3(kOrthThreads), 0, st, p, r, V);
  CC_HIP(hipGetLastError());
  if (center) CC_HIP(hipMemcpyAsync(center, mean.p, (size_t)p * 8, hipMemcpyDeviceToDevice, st));
  double hl[kMaxS];
  CC_HIP(hipMemcpyAsync(hl, lam.p, (size_t)s * 8, hipMemcpyDeviceToHost, st));
  CC_HIP(hipStreamSynchronize(st));
  for (int c = 0; c < r; ++c) sval[c] = std::sqrt(std::max(hl[c], 0.0));
  return CC_OK;
}

}  // namespace

cc_status pca(int64_t n, int64_t p, int32_t x_dtype, const void *X, int64_t ldx,
              const uint8_t *mask, int64_t ldm, int32_t r, int32_t iters, double *V,
              double *sval, double *center, hipStream_t stream) {
  if (n < 2 || p < 1) { set_error("need n >= 2 and p >= 1"); return CC_ERR_INVALID_ARG; }
  if (n * p > ((int64_t)1 << 31) - 1) { set_error("n * p too large"); return CC_ERR_INVALID_ARG; }
  if (r < 1 || r > kMaxR || r > p || r > n) { set_error("need 1 <= r <= min(16, n, p)"); return CC_ERR_INVALID_ARG; }
  if (iters < 0 || iters > 100000) { set_error("need 0 <= iters <= 100000"); return CC_ERR_INVALID_ARG; }
  if (!X || !V || !sval) { set_error("NULL argument"); return CC_ERR_INVALID_ARG; }
  if (x_dtype != CC_DTYPE_F32 && x_dtype != CC_DTYPE_F64) { set_error("bad x_dtype"); return CC_ERR_INVALID_ARG; }
  if (ldx < p || (mask && ldm < p)) { set_error("leading dimension < p"); return CC_ERR_INVALID_ARG; }
  const int it = iters > 0 ? iters : 100;
  if (x_dtype == CC_DTYPE_F32)
    return pca_impl<float>((int)n, (int)p, (const float *)X, ldx, mask, ldm, r, it, V, sval, center, stream);
  return pca_impl<double>((int)n, (int)p, (const double *)X, ldx, mask, ldm, r, it, V, sval, center, stream);
}

cc_status project_U(Problem *P, int32_t r, const double *V, const double *center, double *out) {
  if (r < 1 || r > kMaxR) { set_error("need 1 <= r <= 16"); return CC_ERR_INVALID_ARG; }
  if (!V || !out) { set_error("NULL argument"); return CC_ERR_INVALID_ARG; }
  const dim3 grid((unsigned)cdivx(P->n, 4));
  if (P->precision == kF32)
    hipLaunchKernelGGL((k_project<float>), grid, dim3(256), 0, P->stream, (int)P->n, (int)P->p,
                       (int)P->ld, (const float *)P->U, r, V, center, out);
  else
    hipLaunchKernelGGL((k_project<double>), grid, dim3(256), 0, P->stream, (int)P->n, (int)P->p,
                       (int)P->ld, (const double *)P->U, r, V, center, out);
  CC_HIP(hipGetLastError());
  return CC_OK;
}

}  // namespace ccmi
