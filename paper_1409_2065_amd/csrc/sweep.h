// What the sweep kernels of the solver share: storage types and vector
// accesses, block sums, block coordinates, the arithmetic of the U update and
// the end of an MM iteration.
#pragma once

#include <hip/hip_ext.h>

#include "ccmi_internal.h"
#include "wave_ops.h"

namespace ccmi {

// ------------------------------------------------------------------ traits
template <int PREC> struct Traits;
// TS: U and the stop-test snapshots; TG: the rows the pair sweeps gather;
// TA: the stored A array.  The mixed precision stores A as hi + lo: hi is
// the FP32 gather copy itself and lo (TA) the FP32 rounding of a - hi, 48
// significant bits in all, so the sweeps move 8 bytes of A per entry.
template <> struct Traits<kF32> {
  using TS = float; using TG = float; using TX = float; using TA = float;
  static constexpr bool mirror = false, hilo = false;
};
template <> struct Traits<kMixed> {
  using TS = double; using TG = float; using TX = float; using TA = float;
  static constexpr bool mirror = true, hilo = true;
};
template <> struct Traits<kF64> {
  using TS = double; using TG = double; using TX = double; using TA = double;
  static constexpr bool mirror = false, hilo = false;
};

// ------------------------------------------------------ vector load/store
// Streaming rows of the point sweep (read or written once per iteration):
// non-temporal accesses, so that they do not push the gathered neighbour
// rows out of L2.  Used by the sweep with several items per wave (wide
// rows, whose data do not stay cached); where the whole working set stays
// in the caches (narrow rows, one item per wave) they measured slower.
typedef double nt_d2 __attribute__((ext_vector_type(2)));
typedef float nt_f4 __attribute__((ext_vector_type(4)));
template <typename T, int VEC> struct NtIO {
  __device__ static void store(T *p, const double (&v)[VEC]) {
#pragma unroll
    for (int k = 0; k < VEC; ++k) __builtin_nontemporal_store((T)v[k], p + k);
  }
};
template <> struct NtIO<double, 4> {
  __device__ static void store(double *p, const double (&v)[4]) {
    nt_d2 a = {v[0], v[1]}, b = {v[2], v[3]};
    __builtin_nontemporal_store(a, reinterpret_cast<nt_d2 *>(p));
    __builtin_nontemporal_store(b, reinterpret_cast<nt_d2 *>(p + 2));
  }
  __device__ static void load(const double *p, double (&o)[4]) {
    const nt_d2 a = __builtin_nontemporal_load(reinterpret_cast<const nt_d2 *>(p));
    const nt_d2 b = __builtin_nontemporal_load(reinterpret_cast<const nt_d2 *>(p + 2));
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
  }
};
template <> struct NtIO<float, 4> {
  __device__ static void store(float *p, const double (&v)[4]) {
    nt_f4 a = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
    __builtin_nontemporal_store(a, reinterpret_cast<nt_f4 *>(p));
  }
  __device__ static void load(const float *p, float (&o)[4]) {
    const nt_f4 a = __builtin_nontemporal_load(reinterpret_cast<const nt_f4 *>(p));
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
  }
};

template <int VEC> struct VecIO;
template <> struct VecIO<4> {
  __device__ static void load(const float *p, double (&o)[4]) {
    float4 v = *reinterpret_cast<const float4 *>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
  __device__ static void load(const double *p, double (&o)[4]) {
    double2 a = *reinterpret_cast<const double2 *>(p);
    double2 b = *reinterpret_cast<const double2 *>(p + 2);
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
  }
  __device__ static void store(float *p, const double (&v)[4]) {
    *reinterpret_cast<float4 *>(p) =
        make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
  }
  __device__ static void store(double *p, const double (&v)[4]) {
    *reinterpret_cast<double2 *>(p) = make_double2(v[0], v[1]);
    *reinterpret_cast<double2 *>(p + 2) = make_double2(v[2], v[3]);
  }
};
template <> struct VecIO<2> {
  __device__ static void load(const float *p, double (&o)[2]) {
    float2 v = *reinterpret_cast<const float2 *>(p);
    o[0] = v.x; o[1] = v.y;
  }
  __device__ static void load(const double *p, double (&o)[2]) {
    double2 a = *reinterpret_cast<const double2 *>(p);
    o[0] = a.x; o[1] = a.y;
  }
  __device__ static void store(float *p, const double (&v)[2]) {
    *reinterpret_cast<float2 *>(p) = make_float2((float)v[0], (float)v[1]);
  }
  __device__ static void store(double *p, const double (&v)[2]) {
    *reinterpret_cast<double2 *>(p) = make_double2(v[0], v[1]);
  }
};
template <> struct VecIO<1> {
  __device__ static void load(const float *p, double (&o)[1]) { o[0] = *p; }
  __device__ static void load(const double *p, double (&o)[1]) { o[0] = *p; }
  __device__ static void store(float *p, const double (&v)[1]) { *p = (float)v[0]; }
  __device__ static void store(double *p, const double (&v)[1]) { *p = v[0]; }
};

// Raw mask bytes of VEC consecutive entries (byte v in bits 8v..8v+7).
template <int VEC> struct RawMask;
template <> struct RawMask<4> {
  __device__ static uint32_t load(const uint8_t *p) { return *reinterpret_cast<const uint32_t *>(p); }
};
template <> struct RawMask<2> {
  __device__ static uint32_t load(const uint8_t *p) { return *reinterpret_cast<const uint16_t *>(p); }
};
template <> struct RawMask<1> {
  __device__ static uint32_t load(const uint8_t *p) { return *p; }
};

// Raw vector loads (no conversion) for the software-pipelined gathers.
template <typename T, int VEC> struct RawIO;
template <> struct RawIO<float, 4> {
  __device__ static void load(const float *p, float (&o)[4]) {
    float4 v = *reinterpret_cast<const float4 *>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
};
template <> struct RawIO<float, 2> {
  __device__ static void load(const float *p, float (&o)[2]) {
    float2 v = *reinterpret_cast<const float2 *>(p);
    o[0] = v.x; o[1] = v.y;
  }
};
template <> struct RawIO<float, 1> {
  __device__ static void load(const float *p, float (&o)[1]) { o[0] = *p; }
};
template <> struct RawIO<double, 4> {
  __device__ static void load(const double *p, double (&o)[4]) {
    double2 a = *reinterpret_cast<const double2 *>(p);
    double2 b = *reinterpret_cast<const double2 *>(p + 2);
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
  }
};
template <> struct RawIO<double, 2> {
  __device__ static void load(const double *p, double (&o)[2]) {
    double2 a = *reinterpret_cast<const double2 *>(p);
    o[0] = a.x; o[1] = a.y;
  }
};
template <> struct RawIO<double, 1> {
  __device__ static void load(const double *p, double (&o)[1]) { o[0] = *p; }
};

template <typename T> __device__ inline double round_to(double v) { return (double)(T)v; }

// A new entry of A as the state stores it: returns the stored value, with g
// the gather copy's value and lo the stored low half (mixed precision; the
// state is exactly g + lo and g is the nearest FP32 value to it).
template <int PREC>
__device__ __forceinline__ double state_round(double a, double &g, double &lo) {
  if constexpr (Traits<PREC>::hilo) {
    g = (double)(float)a;
    lo = (double)(float)(a - g);
    return g + lo;
  } else {
    const double r = round_to<typename Traits<PREC>::TS>(a);
    g = round_to<typename Traits<PREC>::TG>(r);
    lo = 0.0;
    return r;
  }
}
// A stored entry: g the gather copy's value, r the stored TA value.
template <int PREC>
__device__ __forceinline__ double state_value(double g, double r) {
  if constexpr (Traits<PREC>::hilo) return g + r;
  else return r;
}

__device__ inline double readlane_d(double v, int k) {
  long long bits = __double_as_longlong(v);
  int lo = __builtin_amdgcn_readlane((int)(bits & 0xffffffffll), k);
  int hi = __builtin_amdgcn_readlane((int)(bits >> 32), k);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Wave sums of NV <= 9 values stored to dst[0 .. NV-1]: eight at once, the
// ninth by itself.
template <int NV>
__device__ __forceinline__ void wave_sums_store(const double (&v)[NV], double *dst) {
  static_assert(NV <= 9, "eight at once and one more");
  const int lane = threadIdx.x % kWave;
  double w[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) w[q] = q < NV ? v[q < NV ? q : 0] : 0.0;
  const double t = wave_sum8_groups(w);
  if ((lane & 7) == 0 && (lane >> 3) < NV) dst[lane >> 3] = t;
  if constexpr (NV == 9) {
    const double l = wave_sum(v[8]);
    if (lane == 0) dst[8] = l;
  }
}

// Fixed-order block reduction of NV doubles per thread: wave trees, then
// thread q < NV adds value q over the waves in order and returns it (other
// threads return 0).  scratch: (waves per block) * NV doubles.
template <int NV>
__device__ inline double block_sum(const double (&v)[NV], double *scratch) {
  wave_sums_store<NV>(v, scratch + (threadIdx.x / kWave) * NV);
  __syncthreads();
  double acc = 0.0;
  if (threadIdx.x < NV)
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) acc += scratch[w * NV + threadIdx.x];
  return acc;
}

// Fixed-order block reduction whose result every thread receives: wave
// trees, then thread q sums value q over the NW waves in order and the
// totals are broadcast through LDS.  scratch: (NW + 1) * NV doubles, not
// reused by the caller before its next barrier.
template <int NV, int NW>
__device__ inline void block_sum_all(double (&v)[NV], double *scratch) {
  wave_sums_store<NV>(v, scratch + (threadIdx.x / kWave) * NV);
  __syncthreads();
  if (threadIdx.x < NV) {
    double acc = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) acc += scratch[w * NV + threadIdx.x];
    scratch[NW * NV + threadIdx.x] = acc;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = scratch[NW * NV + q];
}

// Block coordinates within one problem's launch: b = block index, nb =
// blocks of the launch, lb = logical index.  Physical block b runs on XCD
// b % 8 (round-robin dispatch); XCD x is given the x-th contiguous eighth of
// the logical range, so each XCD sweeps a contiguous run of feature tiles.
// A single-problem launch takes them from the hardware indices, a batched
// launch from its block table (same mapping, so the same partial sums).
struct Blk {
  int b, nb, lb;
};
__device__ inline int xcd_remap(int b, int nb) {
  return nb % kXcds == 0 ? (b % kXcds) * (nb / kXcds) + b / kXcds : b;  // small grids: identity
}
__device__ inline Blk hw_blk() {
  const int b = blockIdx.x, nb = gridDim.x;
  return Blk{b, nb, xcd_remap(b, nb)};
}

// ---------------------------------------------------------------- params
struct PointArgs {
  int n, ld, ntile, nitems, chunk;
  const void *X;
  const uint8_t *M;
  void *U;
  void *A0, *A1, *G0, *G1;
  void *Usnap, *Asnap;
  int ell_s;            // ELL stride of the neighbour lists
  const int32_t *degE, *colE, *eidE;
  const double *qE;     // mu w / (rho ||b||) of the previous A, per ELL entry
  const double *s;      // state shrink factors (first iteration of a solve)
  int K;                // stop-test window
  int nblk;             // blocks of this problem's launch
  double *psum;         // this sweep's block partials
  const double *esum;   // partial rows of the previous edge stage
  int nrows;            // how many
  double *trace;
  const DevScalars *sin;  // scalars of the previous iteration
  DevScalars *sout;       // advanced scalars (block 0 writes)
  const BatchInst *bi;    // batched solves only (else null)
  // several projection sweeps per MM iteration (k_point_rhs only)
  double *H;              // h_i = sum_j s_ij (a'_i - a'_j), FP64
  void *T0;               // gather copy of the first sweep's increment A - A'
  // U stored lazily (k_point only): U is written only at missing entries,
  // into Umiss at offsets moff[item] + the entry's rank within its item
  int lazy;
  void *Umiss;
  const int32_t *moff;
};

// ------------------------------------------------------- iteration finish
// End of MM iteration h.m from the full sums v (point sums, then edge sums):
// d, the objective, the windowed stop test and the advance of the scalars.
__device__ inline void finish_scalars(DevScalars &h, const double (&v)[kIterSums], double *trace,
                                      bool writer) {
  const double uA2 = v[0], dAw = v[1], dUw = v[2], loss2 = v[3], u2 = v[4], cross = v[5];
  const double Cs = v[6], As = v[7], pen = v[8];
  const double viol = fmax(As - 2.0 * cross + Cs, 0.0);
  const double d = sqrt(uA2 + viol + h.eps);
  const double F = 0.5 * loss2 + h.mu * pen + h.rho * d;
  const int m = h.m;
  if (writer && h.record && trace) trace[m] = F;
  if (!isfinite(d) || !isfinite(F)) {
    h.status = CC_ERR_NUMERIC; h.done = 1; h.iters = m;
    return;
  }
  const int K = h.K;
  if (m >= 1) {
    // iteration m-1 of the MM loop has now finished
    h.F_last = h.F_cur;
    h.d_last = h.d_prev;
    if (m % K == 0) {
      const double r = sqrt(dUw + h.dA_prev) / (double)K;
      const double unorm = fmax(1.0, sqrt(u2));
      h.rel_last = r / unorm;
      if (h.thr > 0.0 && m - 1 >= 2 && r <= h.thr * unorm) {
        h.done = 1; h.converged = 1; h.iters = m;
        return;
      }
    }
    if (m >= h.max_iter) {
      h.done = 1; h.converged = 0; h.iters = m;
      return;
    }
  }
  h.F_cur = F;
  h.d_prev = d;
  if (m % K == K - 1) h.dA_prev = dAw;
  h.pa ^= 1;
  h.m = m + 1;
}

// Batched solves: the gamma in progress has ended (stop rule, iteration cap
// or a numeric error).  Block 0 records its fusion flags and info; every
// block then moves to the next gamma with a warm start (the state stays), as
// a single solve along a path does, or marks the path finished.
__device__ inline void next_gamma(DevScalars &h, const BatchInst &bi, const Blk blk) {
  const int k = h.path_k;
  if (blk.b == 0) {
    for (int e = threadIdx.x; e < bi.E; e += blockDim.x)
      bi.fused[(size_t)k * bi.E + e] = bi.s[e] == 0.0 ? 1 : 0;
    if (threadIdx.x == 0) {
      double *inf = bi.info + (size_t)k * kInfoVals;
      inf[0] = h.iters; inf[1] = h.converged; inf[2] = h.status;
      inf[3] = h.F_last; inf[4] = h.d_last; inf[5] = h.rel_last; inf[6] = h.mu;
      inf[7] = (double)wall_clock64();
    }
  }
  if (k + 1 < bi.n_gamma && h.status == 0) {
    h.mu = bi.mu[k + 1]; h.rho = bi.rho[k + 1]; h.eps = bi.eps[k + 1]; h.thr = bi.thr[k + 1];
    h.m = 0; h.done = 0; h.converged = 0; h.status = 0; h.iters = 0;
    h.d_prev = 0.0; h.dA_prev = 0.0; h.F_cur = 0.0;
    h.F_last = 0.0; h.d_last = 0.0; h.rel_last = 0.0;
    h.path_k = k + 1;
  } else {
    h.finished = 1;
    if (blk.b == 0 && threadIdx.x == 0) {
      *bi.t_done = wall_clock64();
      atomicAdd(bi.n_finished, 1);
    }
  }
}

// The U update of an MM iteration (Missing Data: y is x on observed entries
// and the previous u elsewhere): one fused multiply-add, so that every
// kernel that forms or rebuilds u rounds it the same way.
__device__ __forceinline__ double mm_u(double ap, double theta, double y) {
  return fma(theta, y - ap, ap);
}

// The edge stage's partial rows that a point sweep's block sums first (at
// most kEsumRows: one or two per thread), each 5 aligned 16-byte loads.  They are issued before the sweep's
// other loads, so that the finish of the previous iteration waits for them
// alone (loads retire in order); loads are unconditional (row 0 stands in
// for a missing row and is not added) so that the wait counts stay exact.
template <int NW> struct EsumLoad {
  static constexpr int kRows = (kEsumRows + NW * kWave - 1) / (NW * kWave);  // per thread
  double2 t[kRows][kEsumStride / 2];
};

template <int NW>
__device__ inline void esum_issue(const PointArgs &a, EsumLoad<NW> &L) {
#pragma unroll
  for (int r = 0; r < EsumLoad<NW>::kRows; ++r) {
    const int b = threadIdx.x + r * NW * kWave;
    const double2 *row = reinterpret_cast<const double2 *>(a.esum + (size_t)(b < a.nrows ? b : 0) * kEsumStride);
#pragma unroll
    for (int k = 0; k < kEsumStride / 2; ++k) L.t[r][k] = row[k];
  }
}

// Start of a point sweep: when a sweep is pending, sum the edge stage's
// partial rows (column-major, the same order in every block) and finish its
// iteration; block 0 stores the scalars of the iteration about to run (or
// the final ones) in the other slot.  Blocks of NW waves; red:
// (NW + 1) * kIterSums.
template <int NW, bool BATCH = false>
__device__ inline DevScalars begin_iteration(const PointArgs &a, double *red, const Blk blk,
                                             const EsumLoad<NW> &L) {
  double v[kIterSums];
#pragma unroll
  for (int q = 0; q < kIterSums; ++q) v[q] = 0.0;
  // unused when nothing is pending
#pragma unroll
  for (int r = 0; r < EsumLoad<NW>::kRows; ++r) {
    if (threadIdx.x + r * NW * kWave < a.nrows) {
#pragma unroll
      for (int k = 0; k < kEsumStride / 2; ++k) {
        v[2 * k] += L.t[r][k].x;
        if (2 * k + 1 < kIterSums) v[2 * k + 1] += L.t[r][k].y;
      }
    }
  }
  DevScalars h = *a.sin;
  const bool writer = blk.b == 0 && threadIdx.x == 0;
  if (h.pending && !h.done) {  // uniform
    block_sum_all<kIterSums, NW>(v, red);
    // uniform, and known to be: the scalars' branches and integers stay scalar
#pragma unroll
    for (int q = 0; q < kIterSums; ++q) v[q] = readlane_d(v[q], 0);
    finish_scalars(h, v, a.trace, writer);
    if constexpr (BATCH) {
      if (h.done) next_gamma(h, *a.bi, blk);
    }
  }
  h.pending = h.done ? 0 : 1;
  if (!h.done) {
    h.m_run = h.m;
    h.pa_run = h.pa;
    h.theta_run = (h.m > 0) ? h.d_prev / (h.d_prev + h.rho) : 0.0;
  }
  if (writer) *a.sout = h;
  return h;
}

// Launch on a stream.  With events given, hipExtLaunchKernel stamps them with
// the kernel's own start (e0) and end (e1), so a sampled duration is the
// kernel's execution, not the gap between two markers around it.
template <typename... KArgs, typename... Args>
static void klaunch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                    hipEvent_t e0, hipEvent_t e1, Args... args) {
  if (e0 || e1)
    hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, stream, e0, e1, 0u, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, args...);
}

}  // namespace ccmi
