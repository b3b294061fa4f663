// Small problems: the MM iterations of a solve in one workgroup.
//
// A problem whose gather copy, edge lists and q factors fit in the LDS of one
// CU, and whose sweeps one CU does in less time than two kernel launches
// take, is solved by one block that runs many iterations per launch: the
// points of an iteration at which everything must be known (the new A, the
// sums of d, the scalars they give) are three block barriers instead of kernel
// boundaries.  The gather
// copy is double-buffered in LDS, with the low half of A, the q factors, the
// edges with their weights and norms, and the neighbour lists beside it.  A
// sweep reads X and the mask from L2 while it sums neighbours; what is
// written, beside the windows of the stopping test and the state a solve may
// end with, is U where entries are missing, which every sweep reads and
// writes.
//
// The arithmetic per point and edge is that of the sweeps over many blocks
// (k_point, k_edge_items); the sums over points and over the features of an
// edge run in another (fixed) order.
//
// What bounds an iteration is one CU's FP64 arithmetic (about 17 operations
// per neighbour and four features, a square root and a division per edge)
// and its LDS reads; the barriers, block sums and scalars take 2.4 us.
// Measured per iteration, launches against this (mixed): 60 x 6 11.5 and
// 3.7 us, 200 x 10 12.4 and 7.6, 200 x 24 12.8 and 10.2, 370 x 10 12.9 and
// 10.8.  Blocks of 512 threads took 8 to 10% longer.  At 1024 threads (128
// registers each) the mixed kernel spills 17 registers and the FP64 one 4 (56
// and 20 bytes a lane), the FP32 one and all at 256 threads none.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <numeric>
#include <vector>

#include "sweep.h"

namespace ccmi {

struct ResArgs {
  int n, ld, E, ell_s, K;
  int NE;            // list entries in LDS (each point's padded to 4)
  int lel;           // log2 of the lanes that share an edge
  int iters;         // sweeps per launch
  const void *X;
  const uint8_t *M;
  void *U, *A0, *A1, *G0, *G1, *Usnap, *Asnap;
  const int32_t *degE, *colE, *eidE;
  uint32_t g4mul;         // floor(k / (ld / 4)) = umulhi(k, g4mul) for ld > 4
  const int32_t *order;   // points by decreasing degree: a wave's loops are as long
  const int32_t *estart;  // first list entry of each point
  const int32_t *ei, *ej;
  const double *w;
  double *s, *nb0, *nb1, *qe;
  double *sums;           // the pending iteration's sums between launches
  double *trace;
  DevScalars *sc;
  int prof_every;         // sample every such iteration (0: none), counted
  long long prof_iter;    // from this one
  unsigned long long *prof;  // ticks of the point phase, of the edge phase, samples
};

// Totals over the block's NW waves of their 9 sums in scratch, to every lane
// of the calling wave: 16 lanes add the waves' values by a tree.
template <int NW>
__device__ __forceinline__ void wave_totals(const double *scratch, double (&out)[kIterSums]) {
  const int lane = threadIdx.x % kWave, w = lane % 16, g = lane / 16;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const int q = 4 * r + g;
    double t = (w < NW && q < kIterSums) ? scratch[w * kIterSums + q] : 0.0;
    t += dpp<kRor + 8>(t);
    t += dpp<kRor + 4>(t);
    t += dpp<kRor + 2>(t);
    t += dpp<kRor + 1>(t);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (4 * r + k < kIterSums) out[4 * r + k < kIterSums ? 4 * r + k : 0] = readlane_d(t, 16 * k);
  }
}

// Threads take four-feature pieces of points, then edges (2^lel lanes each),
// in turn.  The scalars live in LDS: one wave finishes an iteration (a square root and
// a few divisions in FP64, which sixteen waves would queue up for on the four
// SIMDs), the others read what they need after a barrier.
template <int PREC, int NT>
__device__ __forceinline__ void resident_sweeps(const ResArgs &a) {
  using TS = typename Traits<PREC>::TS;
  using TG = typename Traits<PREC>::TG;
  using TX = typename Traits<PREC>::TX;
  using TA = typename Traits<PREC>::TA;
  constexpr bool hilo = Traits<PREC>::hilo;
  constexpr int NW = NT / kWave;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double scratch[NW * kIterSums];
  __shared__ DevScalars hs;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int nl = a.n * a.ld, G4 = a.ld / 4;
  double *q = reinterpret_cast<double *>(smem);  // E, then 0 for list padding
  TG *Gl = reinterpret_cast<TG *>(q + (a.E + 2) / 2 * 2);
  TA *lo = reinterpret_cast<TA *>(Gl + 2 * nl);  // mixed precision
  double *nb = reinterpret_cast<double *>(lo + (hilo ? nl : 0));
  double *we = nb + (a.E + 1) / 2 * 2;
  uint32_t *ent = reinterpret_cast<uint32_t *>(we + (a.E + 1) / 2 * 2);
  uint2 *pts = reinterpret_cast<uint2 *>(ent + a.NE);  // by degree: point; first entry and length
  uint32_t *ends = reinterpret_cast<uint32_t *>(pts + a.n);

  if (a.sc->done) return;
  if (tid == 0) hs = *a.sc;
  const TX *X = reinterpret_cast<const TX *>(a.X);
  TS *U = reinterpret_cast<TS *>(a.U);
  TS *Us = reinterpret_cast<TS *>(a.Usnap), *As = reinterpret_cast<TS *>(a.Asnap);

  // neighbour lists: neighbour in the upper, edge in the lower 16 bits
  for (int i = tid; i < a.n; i += NT) {
    const int d = a.degE[i], o = a.estart[i];
    const int32_t *cj = a.colE + (size_t)i * a.ell_s, *ce = a.eidE + (size_t)i * a.ell_s;
    for (int k = 0; k < d; ++k) ent[o + k] = ((uint32_t)cj[k] << 16) | (uint32_t)ce[k];
    for (int k = d; k < (d + 3) / 4 * 4; ++k) ent[o + k] = ((uint32_t)i << 16) | (uint32_t)a.E;
  }
  for (int k = tid; k < a.n; k += NT) {
    const int i = a.order[k];
    pts[k] = make_uint2((uint32_t)i, ((uint32_t)a.estart[i] << 16) | (uint32_t)a.degE[i]);
  }
  for (int e = tid; e < a.E; e += NT) {
    we[e] = a.w[e];
    ends[e] = ((uint32_t)a.ei[e] << 16) | (uint32_t)a.ej[e];
  }
  const int le = 1 << a.lel, sub = tid & (le - 1);

  int cur = 0;
  __syncthreads();
  for (int it = 0;; ++it) {
    // end of the previous sweep, start of this one
    if (wave == 0) {
      DevScalars h = hs;
      if (h.pending) {
        double v[kIterSums];
        if (it > 0) {
          wave_totals<NW>(scratch, v);
        } else {
#pragma unroll
          for (int k = 0; k < kIterSums; ++k) v[k] = a.sums[k];
        }
        finish_scalars(h, v, a.trace, lane == 0);
        h.pending = 0;
      }
      if (!h.done) {
        h.pending = 1;
        h.m_run = h.m;
        h.pa_run = h.pa;
        h.theta_run = (h.m > 0) ? h.d_prev / (h.d_prev + h.rho) : 0.0;
      }
      if (lane == 0) hs = h;
    }
    __syncthreads();
    if (hs.done) {  // uniform
      if (tid == 0) *a.sc = hs;
      return;
    }
    const int m = __builtin_amdgcn_readfirstlane(hs.m), pa = __builtin_amdgcn_readfirstlane(hs.pa);
    const double dprev = hs.d_prev, theta = hs.theta_run, dq = m > 0 ? dprev : 1.0;
    TG *Gpa = reinterpret_cast<TG *>(pa == 0 ? a.G0 : a.G1), *Gna = reinterpret_cast<TG *>(pa == 0 ? a.G1 : a.G0);
    TA *Apa = reinterpret_cast<TA *>(pa == 0 ? a.A0 : a.A1), *Ana = reinterpret_cast<TA *>(pa == 0 ? a.A1 : a.A0);
    double *nbp = pa == 0 ? a.nb0 : a.nb1, *nbn = pa == 0 ? a.nb1 : a.nb0;
    if (it == 0) {  // the state
      for (int k = 4 * tid; k < nl; k += 4 * NT) {
        TG g[4];
        RawIO<TG, 4>::load(Gpa + k, g);
        TG *d = Gl + k;
        d[0] = g[0]; d[1] = g[1]; d[2] = g[2]; d[3] = g[3];
      }
      if constexpr (hilo) {
        for (int k = 4 * tid; k < nl; k += 4 * NT) {
          TA g[4];
          RawIO<TA, 4>::load(Apa + k, g);
          lo[k] = g[0]; lo[k + 1] = g[1]; lo[k + 2] = g[2]; lo[k + 3] = g[3];
        }
      }
      for (int e = tid; e < a.E; e += NT) {
        nb[e] = nbp[e];
        // the first sweep of a solve takes c = 1 - s: min(1 q, 1) with q = 1 - s
        q[e] = m == 0 ? 1.0 - a.s[e] : a.qe[e];
      }
      if (tid == 0) q[a.E] = 0.0;
      __syncthreads();
    }
    // Sweep m.  When its end may be the solve's (the stop rule, the cap) or
    // is this launch's, the state it started from goes to global memory.
    const int K = a.K;
    const bool last = it == a.iters - 1;
    const bool keep = last || m >= hs.max_iter || (m % K == 0 && hs.thr > 0.0 && m - 1 >= 2);
    const bool snapU0 = (m == 0), winU = (m > 0) && (m % K == 0);
    const bool initA = (m == 0) && (K > 1), winA = (m % K) == (K - 1);
    const bool readU = m == 0 || a.M, storeU = keep || a.M;
    const bool sample = a.prof_every > 0 && (a.prof_iter + it) % a.prof_every == 0;
    const unsigned long long t0 = sample ? wall_clock64() : 0ull;
    const TG *Gc = Gl + cur * nl;
    TG *Gw = Gl + (cur ^ 1) * nl;
    double ps[kIterSums];
#pragma unroll
    for (int k = 0; k < kIterSums; ++k) ps[k] = 0.0;
    for (int k = tid; k < a.n * G4; k += NT) {
      const uint32_t pi = G4 > 1 ? __umulhi((uint32_t)k, a.g4mul) : (uint32_t)k;
      const uint2 pt = pts[pi];
      const int f = 4 * (k - (int)pi * G4), deg = (int)(pt.y & 0xffffu);
      const uint32_t r0 = pt.x * (uint32_t)a.ld + (uint32_t)f;
      // X, the mask and (first sweep, or missing entries) U come from L2
      // while the neighbours are summed
      TX x[4];
      TS u[4] = {(TS)0, (TS)0, (TS)0, (TS)0};
      uint32_t mk = 0xffffffffu;
      RawIO<TX, 4>::load(X + r0, x);
      if (a.M) mk = RawMask<4>::load(a.M + r0);
      if (readU) RawIO<TS, 4>::load(U + r0, u);
      double sumg[4] = {0.0, 0.0, 0.0, 0.0}, sumcg[4] = {0.0, 0.0, 0.0, 0.0}, C = 0.0;
      const uint4 *lp = reinterpret_cast<const uint4 *>(ent + (pt.y >> 16));
      for (int k4 = 0; k4 < deg; k4 += 4) {
        const uint4 e4 = lp[k4 / 4];
        const uint32_t ev[4] = {e4.x, e4.y, e4.z, e4.w};
        double qv[4];
        TG g[4][4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          qv[p] = q[ev[p] & 0xffffu];
          RawIO<TG, 4>::load(Gc + (int)(ev[p] >> 16) * a.ld + f, g[p]);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const double c = fmin(dq * qv[p], 1.0), wt = k4 + p < deg ? 1.0 : 0.0;
          C += c;
#pragma unroll
          for (int z = 0; z < 4; ++z) {
            const double xv = (double)g[p][z];
            sumg[z] = fma(wt, xv, sumg[z]);
            sumcg[z] = fma(c, xv, sumcg[z]);
          }
        }
      }
      TG gr[4];
      TA lr[4] = {(TA)0, (TA)0, (TA)0, (TA)0};
      RawIO<TG, 4>::load(Gc + r0, gr);
      if constexpr (hilo) RawIO<TA, 4>::load(lo + r0, lr);
      const double inv1d = 1.0 / (1.0 + (double)deg);
      const double S = (double)deg - C;
      double un[4], an[4], al[4], gn[4], ap[4];
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        const double gi = (double)gr[z];
        ap[z] = hilo ? state_value<PREC>(gi, (double)lr[z]) : gi;
        const bool obs = ((mk >> (8 * z)) & 0xffu) != 0u;
        const double xd = (double)x[z];
        double uu = (double)u[z];
        if (m > 0) uu = mm_u(ap[z], theta, obs ? xd : uu);
        uu = round_to<TS>(uu);
        const double jac = sumcg[z] - C * gi;
        const double hh = S * gi - (sumg[z] - sumcg[z]);
        double g, l;
        const double anew = state_round<PREC>(ap[z] + (uu - ap[z] + jac) * inv1d, g, l);
        un[z] = uu; an[z] = anew; al[z] = l; gn[z] = g;
        const double dua = uu - anew;
        ps[0] = fma(dua, dua, ps[0]);
        ps[5] = fma(hh, g, ps[5]);
        if (obs) { const double r = xd - uu; ps[3] = fma(r, r, ps[3]); }
        ps[4] = fma(uu, uu, ps[4]);
      }
      VecIO<4>::store(Gw + r0, gn);
      if (storeU) VecIO<4>::store(U + r0, un);
      if (keep) {
        Gpa[r0] = gr[0]; Gpa[r0 + 1] = gr[1]; Gpa[r0 + 2] = gr[2]; Gpa[r0 + 3] = gr[3];
        if constexpr (hilo) {
          Apa[r0] = lr[0]; Apa[r0 + 1] = lr[1]; Apa[r0 + 2] = lr[2]; Apa[r0 + 3] = lr[3];
        }
      }
      if (last) {
        VecIO<4>::store(Gna + r0, gn);
        if constexpr (hilo) VecIO<4>::store(Ana + r0, al);
      }
      if (winU) {
        double us[4];
        VecIO<4>::load(Us + r0, us);
#pragma unroll
        for (int z = 0; z < 4; ++z) { const double du = un[z] - us[z]; ps[2] = fma(du, du, ps[2]); }
      }
      if (snapU0 || winU) VecIO<4>::store(Us + r0, un);
      if (initA) VecIO<4>::store(As + r0, ap);
      if (winA) {
        double prev[4];
        if (m == 0) {
#pragma unroll
          for (int z = 0; z < 4; ++z) prev[z] = ap[z];
        } else {
          VecIO<4>::load(As + r0, prev);
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) { const double da = an[z] - prev[z]; ps[1] = fma(da, da, ps[1]); }
        VecIO<4>::store(As + r0, an);
      }
      if constexpr (hilo) VecIO<4>::store(lo + r0, al);
    }
    __syncthreads();
    const unsigned long long t1 = sample ? wall_clock64() : 0ull;
    // edges of the new A
    const double mu = hs.mu, rho = hs.rho;
    // (all lanes of a wave take as many turns: the lanes of an edge exchange)
    const int shares = a.E << a.lel;
    for (int k = wave * kWave; k < shares; k += NT) {
      const bool ok = k + lane < shares;
      const int e = ok ? (k + lane) >> a.lel : 0;
      const uint32_t ij = ends[e];
      const TG *gi = Gw + (int)(ij >> 16) * a.ld, *gj = Gw + (int)(ij & 0xffffu) * a.ld;
      double acc = 0.0;
      for (int c = sub; c < G4; c += le) {
        TG ri[4], rj[4];
        RawIO<TG, 4>::load(gi + 4 * c, ri);
        RawIO<TG, 4>::load(gj + 4 * c, rj);
#pragma unroll
        for (int z = 0; z < 4; ++z) { const double d = (double)ri[z] - (double)rj[z]; acc = fma(d, d, acc); }
      }
      if (a.lel > 0) acc += dpp<kXor1>(acc);
      if (a.lel > 1) acc += dpp<kXor2>(acc);
      if (a.lel > 2) acc += dpp_xor4(acc);
      if (ok && sub == 0) {
        const double np = nb[e], nbv = sqrt(acc);
        const double sv = m > 0 ? 1.0 - fmin(dprev * q[e], 1.0) : a.s[e];
        const double qn = nbv > 0.0 ? (mu * we[e]) / (rho * nbv) : __builtin_inf();
        ps[6] += acc;
        ps[7] += (sv * np) * (sv * np);
        ps[8] += we[e] * sv * np;
        q[e] = qn;
        nb[e] = nbv;
        if (keep) { a.s[e] = sv; nbp[e] = np; }
        if (last) { nbn[e] = nbv; a.qe[e] = qn; }
      }
    }
    cur ^= 1;
    wave_sums_store<kIterSums>(ps, scratch + wave * kIterSums);
    __syncthreads();
    if (sample && tid == 0) {
      a.prof[0] += t1 - t0;
      a.prof[1] += wall_clock64() - t1;
      a.prof[2] += 1;
    }
    if (last) {
      if (wave == 0) {
        double v[kIterSums];
        wave_totals<NW>(scratch, v);
        if (lane == 0) {
#pragma unroll
          for (int k = 0; k < kIterSums; ++k) a.sums[k] = v[k];
          *a.sc = hs;
        }
      }
      return;
    }
  }
}

template <int PREC, int NT>
__global__ __launch_bounds__(NT) void k_resident(ResArgs a) {
  resident_sweeps<PREC, NT>(a);
}

// ====================================================================== host
// Most dynamic LDS a resident block takes (static LDS beside it).
constexpr size_t kResLds = 156 * 1024;

static size_t resident_lds(int64_t n, int64_t ld, int64_t E, int64_t NE, int prec) {
  const int64_t tg = prec == kF64 ? 8 : 4, ta = prec == kMixed ? 4 : 0;
  return (size_t)((E + 2) / 2 * 2 * 8 + n * ld * (2 * tg + ta) + 2 * ((E + 1) / 2 * 2 * 8) + NE * 4 + n * 8 + E * 4);
}

// Lanes per edge: enough that an edge's loop is short, while the block's
// threads are not all taken.
static int edge_lanes_log2(int64_t E, int64_t ld, int64_t threads) {
  int l = 0;
  while (l < 3 && (ld / 4) >= (4 << l) && (E << l) < threads) ++l;
  return l;
}

// Whether a problem is solved resident, and its block.  deg: degrees of the
// points.  The limits are the LDS, 16-bit neighbours, edges and list starts,
// and the work: launches over many CUs take about 12 us an iteration
// whatever the size up to some 10^5 features, one CU's time follows the
// neighbour pieces of a sweep.  Near the limit of 17 000, resident and by
// launches (us, FP32 / mixed / FP64): 340 x 10 (14 500 to 14 900 pieces) 9.5 /
// 9.8 / 10.1 and 13.1, with a mask 9.6 / 10.0 / 10.4 and 12.9; 370 x 10 (16 000) 10.6 /
// 10.9 and 13.2, with a mask 11.1 / 11.4 and 13.6 (FP64 does not fit); 100 x 60 (15 800)
// 9.5 / 9.8 / 9.8 and 11.0 to 12.2; 40 x 250 (15 000) 10.8 / 11.4 and 11.9; beyond it 100 x 100
// (31 000) 15 and 12.
// Rows of more than 1024 features: an edge's 8 lanes walk its rows in series,
// where the launches give it a wave or a block, and points take more turns of
// the block's threads.  3 x 1100 7.1 / 7.2 / 6.5 and 11.4 to 12, 8 x 1100 10.4 / 10.8
// / 9.6 and 11.8 to 12.2, 3 x 2000 9.9 / 10.1 / 9.2 and 11.6 to 12; 10 x 1100 11.4 / 11.9 and
// 11.9 / 12.0; 5 x 2000 12.3 / 12.6 and 11.7 / 11.9, 10 x 1200 12.1 / 12.8 and 12.0, 9 x
// 1400 12.1 / 12.7 and 11.8 / 12.0, 6 x 2000 14.6 / 15.1 and 11.9, 3 x 3000 13.7 / 14.1 / 12.6
// and 11.5 to 12, 2 x 4000 15.6 / 15.7 / 14.1 and 11.6.
bool resident_plan(int64_t n, int64_t ld, int64_t E, const int32_t *deg, int prec, ResidentPlan *plan) {
  const char *env = getenv("CCMI_RESIDENT");
  if (env && atoi(env) == 0) return false;
  // a launch-shape switch asks for the sweeps over many blocks
  for (const char *v : {"CCMI_VEC", "CCMI_IPW", "CCMI_EDGE_IPW", "CCMI_POINT_WAVES", "CCMI_SLAB_F", "CCMI_EDGE_ITEMS",
                        "CCMI_EDGE_SLAB", "CCMI_EDGE_SLAB_ITEMS", "CCMI_LAZY_U"})
    if (getenv(v) && !(env && atoi(env) == 1)) return false;
  constexpr int64_t kResWork = 17000;
  if (n >= 65536 || E >= 65535 || n * ld > 65536 || 2 * E * (ld / 4) > kResWork) return false;
  if (ld > 1024 && (ld > 2048 || n * (ld / 4) > 2304)) return false;
  int64_t NE = 0;
  std::vector<int32_t> estart(n), order(n);
  for (int64_t i = 0; i < n; ++i) {
    estart[i] = (int32_t)NE;
    NE += (deg[i] + 3) / 4 * 4;
  }
  if (NE >= 65536 || resident_lds(n, ld, E, NE, prec) > kResLds) return false;
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return deg[a] > deg[b]; });
  plan->NE = NE;
  plan->lds = resident_lds(n, ld, E, NE, prec);
  const int64_t most = std::max(n * (ld / 4), E);
  plan->threads = most <= 256 ? 256 : 1024;
  plan->lel = edge_lanes_log2(E, ld, plan->threads);
  plan->estart = std::move(estart);
  plan->order = std::move(order);
  return true;
}

static ResArgs res_args(Problem *P, int iters) {
  ResArgs a{};
  a.n = (int)P->n; a.ld = (int)P->ld; a.E = (int)P->E; a.ell_s = P->ell_s; a.K = P->cur_K;
  a.g4mul = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)(P->ld / 4) + 1);
  a.NE = (int)P->res.NE; a.lel = P->res.lel; a.iters = iters;
  a.X = P->X; a.M = P->M; a.U = P->U; a.A0 = P->A[0]; a.A1 = P->A[1]; a.G0 = P->G[0]; a.G1 = P->G[1];
  a.Usnap = P->Usnap; a.Asnap = P->Asnap;
  a.degE = P->degE; a.colE = P->colE; a.eidE = P->eidE; a.order = P->res_order; a.estart = P->res_estart;
  a.ei = P->ei; a.ej = P->ej; a.w = P->w; a.s = P->s; a.nb0 = P->nb[0]; a.nb1 = P->nb[1]; a.qe = P->qe;
  a.sums = P->esum; a.trace = P->trace; a.sc = P->sc + P->slot;
  a.prof_every = P->prof_every; a.prof_iter = P->prof_iter; a.prof = P->res_prof;
  return a;
}

template <int PREC, int NT>
static cc_status launch_one(Problem *P, const ResArgs &a) {
  CC_HIP(hipFuncSetAttribute((const void *)k_resident<PREC, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kResLds));
  hipLaunchKernelGGL((k_resident<PREC, NT>), dim3(1), dim3(NT), P->res.lds, P->stream, a);
  CC_HIP(hipGetLastError());
  return CC_OK;
}

template <int PREC>
static cc_status launch_prec(Problem *P, const ResArgs &a) {
  if (P->res.threads == 256) return launch_one<PREC, 256>(P, a);
  return launch_one<PREC, 1024>(P, a);
}

// Up to `iters` sweeps of the solve in progress; ends by itself when the
// stop rule does.
cc_status resident_run(Problem *P, int iters) {
  const ResArgs a = res_args(P, iters);
  if (P->precision == kF32) return launch_prec<kF32>(P, a);
  if (P->precision == kF64) return launch_prec<kF64>(P, a);
  return launch_prec<kMixed>(P, a);
}

}  // namespace ccmi
