// Point sweep over LDS slabs: the U update and the Jacobi sweep of k_point
// over wide rows of few points, where an n x 32 tile of the gather copy fits
// in the LDS of one CU.
//
// A block stages a tile of A' for all n points and sweeps its group of points
// over it, four lanes per point and eight features per lane, gathering
// neighbour rows from LDS instead of L2; then it takes the next tile.  The
// lanes of a point load four list entries each and exchange them by DPP, so a
// q is read and its c formed once per point and not per lane.  Points are
// taken by degree, dealt over the groups, so that the lanes of a wave have
// loops of equal length and the blocks equal work.
//
// Per gathered entry and eight features a lane issues 24 FP64 operations
// (conversion, sum, weighted sum) and about 7 others, which is what bounds the
// sweep: at 1000 x 20000 (31 400 entries) 63 us of the 173, beside 80 us for
// its 400 MB at the rate of a copy (the wave-per-item sweep takes 212).  The next tile's staging, and the next point's lists and rows, load
// while the current point is summed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <numeric>
#include <type_traits>
#include <vector>

#include "sweep.h"

namespace ccmi {

constexpr int kSlabF = 32, kSlabNT = 512;  // features per tile, threads per block
constexpr int kSlabStage = 4;              // staged four-feature chunks a thread has in flight

struct SlabArgs {
  int tiles, tpb, groups, pg;
  const int2 *order;  // groups x pg: point and degree (-1: none)
};

// Value of lane U of each quad.
template <int U>
__device__ __forceinline__ int quad_lane(int v) {
  return __builtin_amdgcn_update_dpp(v, v, U * 0x55, 0xf, 0xf, false);
}
template <int U>
__device__ __forceinline__ double quad_lane(double v) {
  return __hiloint2double(quad_lane<U>(__double2hiint(v)), quad_lane<U>(__double2loint(v)));
}

template <typename T>
__device__ __forceinline__ void load4(const T *p, T *o) {
  T v[4];
  RawIO<T, 4>::load(p, v);
  o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3];
}

template <int PREC, bool MASK>
__global__ __launch_bounds__(kSlabNT) void k_point_slab(PointArgs a, SlabArgs sl) {
  using TS = typename Traits<PREC>::TS;
  using TG = typename Traits<PREC>::TG;
  using TX = typename Traits<PREC>::TX;
  using TA = typename Traits<PREC>::TA;
  constexpr bool hilo = Traits<PREC>::hilo;
  constexpr int F = kSlabF, NT = kSlabNT, LPP = 4, NV = F / LPP, NQ = NV / 4, NW = NT / kWave;
  constexpr int CPR = F / 4;  // staged chunks per row
  extern __shared__ __align__(16) unsigned char smem[];
  TG *slab = reinterpret_cast<TG *>(smem);
  int2 *pts = reinterpret_cast<int2 *>(slab + (size_t)a.n * F);
  __shared__ double scratch[NW * kPointSums];
  __shared__ double red[(NW + 1) * kIterSums];
  const Blk blk = hw_blk();
  const int tid = threadIdx.x;
  EsumLoad<NW> el;
  esum_issue<NW>(a, el);
  const int grp = blk.lb % sl.groups, tb = blk.lb / sl.groups;
  const int t0 = tb * sl.tpb, t1 = min(t0 + sl.tpb, sl.tiles);
  // The buffer of A' follows from the scalars before the finish: an
  // iteration that ends without ending the solve swaps the buffers.
  const int pa0 = (a.sin->pending && !a.sin->done) ? a.sin->pa ^ 1 : a.sin->pa;
  const TG *Gs = reinterpret_cast<const TG *>(pa0 == 0 ? a.G0 : a.G1);
  const int nch = a.n * CPR;
  TG st[kSlabStage][4];
  // chunks k0 .. k0 + kSlabStage * NT - 1 of tile t (a chunk past the end or
  // the row reads the first one; past the end it is not stored, past the row
  // its features are in the slab but no lane's sums are kept)
  auto stage_load = [&](int t, int k0) {
#pragma unroll
    for (int u = 0; u < kSlabStage; ++u) {
      const int k = k0 + u * NT + tid;
      const int f = t * F + 4 * (k % CPR);
      const bool ok = k < nch && f < a.ld;
      RawIO<TG, 4>::load(Gs + (ok ? (size_t)(k / CPR) * a.ld + f : (size_t)0), st[u]);
    }
  };
  auto stage_store = [&](int k0) {
#pragma unroll
    for (int u = 0; u < kSlabStage; ++u) {
      const int k = k0 + u * NT + tid;
      if (k < nch) {
        TG *d = slab + 4 * k;
        d[0] = st[u][0]; d[1] = st[u][1]; d[2] = st[u][2]; d[3] = st[u][3];
      }
    }
  };
  for (int p = tid; p < sl.pg; p += NT) pts[p] = sl.order[grp * sl.pg + p];
  if (t0 < t1) stage_load(t0, 0);
  const DevScalars hs = begin_iteration<NW>(a, red, blk, el);
  if (hs.done) return;
  const int m = __builtin_amdgcn_readfirstlane(hs.m), pa = __builtin_amdgcn_readfirstlane(hs.pa);
  // the first sweep of a solve takes c = 1 - s: min(1 q, 1), the lists
  // holding q = 1 - s then
  const double dprev = m > 0 ? hs.d_prev : 1.0;
  const double theta = hs.theta_run;
  const int K = a.K;
  const bool snapU0 = (m == 0), winU = (m > 0) && (m % K == 0);
  const bool initA = (m == 0) && (K > 1), winA = (m % K) == (K - 1);
  const bool lazy = a.lazy != 0;
  TS *Us = reinterpret_cast<TS *>(a.Usnap);
  TS *As = reinterpret_cast<TS *>(a.Asnap);
  const TA *Ap = reinterpret_cast<const TA *>(pa == 0 ? a.A0 : a.A1);
  TA *An = reinterpret_cast<TA *>(pa == 0 ? a.A1 : a.A0);
  TG *Gn = reinterpret_cast<TG *>(pa == 0 ? a.G1 : a.G0);
  const TX *X = reinterpret_cast<const TX *>(a.X);
  TS *U = reinterpret_cast<TS *>(a.U);
  const int fl = NV * (tid % LPP), ql = tid & 3;
  double ps[kPointSums] = {0, 0, 0, 0, 0, 0};

  for (int t = t0; t < t1; ++t) {
    if (t > t0) __syncthreads();  // the last tile's readers are done
    stage_store(0);
    for (int k0 = kSlabStage * NT; k0 < nch; k0 += kSlabStage * NT) {
      stage_load(t, k0);
      stage_store(k0);
    }
    __syncthreads();
    if (t + 1 < t1) stage_load(t + 1, 0);  // in flight during the sweep
    const int f0 = t * F + fl;
    const int nv = min(NV, a.ld - f0);  // features of this lane, a multiple of 4 (0 or less: none)
    // A point's own rows (used after its neighbour sums) and its first 32
    // list entries: 16 per group, four per lane of the quad (lists are
    // aligned to 4 entries).  Points past the group's end load point 0's.
    struct Own {
      TX x[NV];
      TA lo[NV];
      uint32_t mk[NQ];
    };
    auto own_load = [&](int i, Own &o) {
      const size_t rowc = (size_t)i * a.ld + (nv > 0 ? f0 : 0);
#pragma unroll
      for (int h = 0; h < NQ; ++h) {
        const size_t r = rowc + (4 * h < nv ? 4 * h : 0);
        load4(X + r, o.x + 4 * h);
        if constexpr (hilo) load4(Ap + r, o.lo + 4 * h);
        o.mk[h] = 0xffffffffu;
        if constexpr (MASK) o.mk[h] = RawMask<4>::load(a.M + r);
      }
    };
    auto fetch = [&](int rs, int deg, int k, int (&j)[4], double (&qv)[4]) {
      const int kk = k + 4 * ql;
      const int slot = rs + (kk < deg ? kk : 0);
      const int4 j4 = *reinterpret_cast<const int4 *>(a.colE + slot);
      const double2 q0 = *reinterpret_cast<const double2 *>(a.qE + slot);
      const double2 q1 = *reinterpret_cast<const double2 *>(a.qE + slot + 2);
      j[0] = j4.x; j[1] = j4.y; j[2] = j4.z; j[3] = j4.w;
      qv[0] = q0.x; qv[1] = q0.y; qv[2] = q1.x; qv[3] = q1.y;
    };
    int p = tid / LPP;
    int2 pt = p < sl.pg ? pts[p] : make_int2(-1, 0);
    Own own;
    int ja[4], jb[4];
    double qa[4], qb[4];
    {
      const int i = max(pt.x, 0);
      own_load(i, own);
      fetch(i * a.ell_s, pt.y, 0, ja, qa);
      fetch(i * a.ell_s, pt.y, 16, jb, qb);
    }
    while (p < sl.pg && pt.x >= 0) {  // a group's points come before its padding
      const int i = pt.x, deg = pt.y, rs = i * a.ell_s;
      const size_t row0 = (size_t)i * a.ld + f0;
      TS up[NV];
      if constexpr (MASK) {
#pragma unroll
        for (int h = 0; h < NQ; ++h) load4(U + (nv > 0 ? row0 : 0) + (4 * h < nv ? 4 * h : 0), up + 4 * h);
      }
      double sumg[NV], sumcg[NV], C = 0.0;
#pragma unroll
      for (int v = 0; v < NV; ++v) sumg[v] = sumcg[v] = 0.0;
      // four entries held by lane L of the quad, from entry k on
      auto four = [&](int k, const int (&off)[4], const double (&c)[4], auto lane_tag) {
        constexpr int L = decltype(lane_tag)::value;
        if (k >= deg) return;
        constexpr int EB = 16 / NV;  // entries in flight
#pragma unroll
        for (int e0 = 0; e0 < 4; e0 += EB) {
          TG x[EB][NV];
#pragma unroll
          for (int e = 0; e < EB; ++e) {
            const TG *src = slab + quad_lane<L>(off[e0 + e]) + fl;
#pragma unroll
            for (int h = 0; h < NV; h += 4) load4(src + h, x[e] + h);
          }
#pragma unroll
          for (int e = 0; e < EB; ++e) {
            const double wt = k + e0 + e < deg ? 1.0 : 0.0, ce = quad_lane<L>(c[e0 + e]);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              const double xv = (double)x[e][v];
              sumg[v] = fma(wt, xv, sumg[v]);
              sumcg[v] = fma(ce, xv, sumcg[v]);
            }
          }
        }
      };
      auto use = [&](int k, const int (&j)[4], const double (&qv)[4]) {
        int off[4];
        double c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = k + 4 * ql + e < deg;
          c[e] = ok ? fmin(dprev * qv[e], 1.0) : 0.0;
          off[e] = (ok ? j[e] : i) * F;  // a slot past the list: the own row, weight 0
          C += c[e];
        }
        four(k, off, c, std::integral_constant<int, 0>());
        four(k + 4, off, c, std::integral_constant<int, 1>());
        four(k + 8, off, c, std::integral_constant<int, 2>());
        four(k + 12, off, c, std::integral_constant<int, 3>());
      };
      for (int k = 0; k < deg; k += 32) {
        use(k, ja, qa);
        if (k + 16 >= deg) break;
        fetch(rs, deg, k + 32, ja, qa);
        use(k + 16, jb, qb);
        fetch(rs, deg, k + 48, jb, qb);
      }
      // the next point's loads, in flight during this one's update
      const Own cur = own;
      p += NT / LPP;
      pt = p < sl.pg ? pts[p] : make_int2(-1, 0);
      {
        const int in = max(pt.x, 0);
        own_load(in, own);
        fetch(in * a.ell_s, pt.y, 0, ja, qa);
        fetch(in * a.ell_s, pt.y, 16, jb, qb);
      }
      C += dpp<kXor1>(C);
      C += dpp<kXor2>(C);
      const double inv1d = 1.0 / (1.0 + (double)deg);
      const double S = (double)deg - C;
#pragma unroll
      for (int h = 0; h < NQ; ++h) {
        if (4 * h >= nv) break;
        const size_t row = row0 + 4 * h;
        TG gr[4];
        load4(slab + i * F + fl + 4 * h, gr);
        double u[4], an[4], al[4], gn[4], ap[4];
        if (m == 0) {
          VecIO<4>::load(U + row, u);
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            u[v] = 0.0;
            if constexpr (MASK) u[v] = (double)up[4 * h + v];
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int w = 4 * h + v;
          const double gi = (double)gr[v];
          ap[v] = hilo ? state_value<PREC>(gi, (double)cur.lo[w]) : gi;
          const bool obs = !MASK || ((cur.mk[h] >> (8 * v)) & 0xffu) != 0u;
          const double xd = (double)cur.x[w];
          double uu = u[v];
          if (m > 0) uu = mm_u(ap[v], theta, obs ? xd : uu);
          uu = round_to<TS>(uu);
          const double jac = sumcg[w] - C * gi;             // sum_j c (a'_j - a'_i)
          const double hh = S * gi - (sumg[w] - sumcg[w]);  // sum_j s (a'_i - a'_j)
          double g, l;
          const double anew = state_round<PREC>(ap[v] + (uu - ap[v] + jac) * inv1d, g, l);
          u[v] = uu; an[v] = anew; al[v] = l; gn[v] = g;
          const double dua = uu - anew;
          ps[0] = fma(dua, dua, ps[0]);
          ps[5] = fma(hh, g, ps[5]);
          if (obs) { const double r = xd - uu; ps[3] = fma(r, r, ps[3]); }
          ps[4] = fma(uu, uu, ps[4]);
        }
        if (!lazy) VecIO<4>::store(U + row, u);
        if constexpr (hilo) VecIO<4>::store(An + row, al);
        VecIO<4>::store(Gn + row, gn);
        if (winU) {
          double us[4];
          VecIO<4>::load(Us + row, us);
#pragma unroll
          for (int v = 0; v < 4; ++v) { const double du = u[v] - us[v]; ps[2] = fma(du, du, ps[2]); }
        }
        if (snapU0 || winU) VecIO<4>::store(Us + row, u);
        if (initA) VecIO<4>::store(As + row, ap);
        if (winA) {
          double prev[4];
          if (m == 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) prev[v] = ap[v];
          } else {
            VecIO<4>::load(As + row, prev);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) { const double da = an[v] - prev[v]; ps[1] = fma(da, da, ps[1]); }
          VecIO<4>::store(As + row, an);
        }
      }
    }
  }
  const double tot = block_sum<kPointSums>(ps, scratch);
  if (tid < kPointSums) a.psum[(size_t)blk.lb * 8 + tid] = tot;
}

// The lists' q of a solve's first sweep: 1 - s per entry.
__global__ void k_q_from_s(int64_t slots, const int32_t *colE, const int32_t *eidE, const double *s, double *qE) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < slots) qE[k] = colE[k] >= 0 ? 1.0 - s[eidE[k]] : 0.0;
}

// ====================================================================== host
static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
constexpr int64_t kPointSlabBytes = 140 * 1024;  // LDS of a slab and its group's points

// Few points leave most lanes of a block idle, and a small state is over
// before the staging pays (point sweep by waves and by slabs, us): 100 x
// 60000 53 and 65, 300 x 8000 31 and 22, 300 x 2000 with a mask 14 and 15,
// 1000 x 1000 with a mask 23 and 26, 1000 x 2000 41 and 26, with a mask 43
// and 33, 1000 x 20000 212 and 173.
bool slab_by_size(int64_t n, int64_t ld) { return n >= 256 && n * ld >= 1500000; }

// The split of a slab sweep; false when the slab does not fit or the
// wave-per-item sweep is as fast (or asked for).
bool slab_plan(int64_t n, int64_t ld, const int32_t *deg, int prec, SlabPlan *plan) {
  const int64_t tg = prec == kF64 ? 8 : 4;
  const char *env = getenv("CCMI_SLAB_F");
  const int want = env ? atoi(env) : -1;
  if (want == 0) return false;
  plan->forced = want > 0;
  if (!plan->forced) {
    for (const char *v : {"CCMI_VEC", "CCMI_IPW", "CCMI_POINT_WAVES"})
      if (getenv(v)) return false;
    if (!slab_by_size(n, ld)) return false;
  }
  const int64_t tiles = cdiv(ld, kSlabF), per = kSlabNT / 4;
  // A block per CU (the slab takes most of its LDS).  With more tiles than
  // CUs a block takes several; one or two groups of points, whichever leaves
  // the CUs more evenly loaded.
  const int64_t cus = 256;
  int64_t groups = 1;
  if (tiles >= cus) {
    const int64_t one = cdiv(tiles, cus) * 2, two = cdiv(2 * tiles, cus);  // rounds of half the points
    if (two < one) groups = 2;
  } else {
    groups = std::max<int64_t>(1, std::min<int64_t>(cdiv(n, per), cus / tiles));
  }
  plan->tiles = (int)tiles;
  plan->groups = (int)groups;
  plan->tpb = (int)std::max<int64_t>(1, cdiv(tiles * groups, cus));
  plan->pg = (int)cdiv(n, groups);
  plan->lds = (size_t)(n * kSlabF * tg + plan->pg * 8);
  if ((int64_t)plan->lds > kPointSlabBytes) { plan->forced = false; return false; }
  int64_t blocks = groups * cdiv(tiles, plan->tpb);
  if (blocks > kXcds) blocks = cdiv(blocks, kXcds) * kXcds;
  plan->blocks = (int)blocks;
  std::vector<int32_t> by(n);
  std::iota(by.begin(), by.end(), 0);
  std::stable_sort(by.begin(), by.end(), [&](int32_t a, int32_t b) { return deg[a] > deg[b]; });
  plan->order.assign((size_t)(2 * groups * plan->pg), -1);
  for (int64_t k = 0; k < n; ++k) {
    const int64_t r = k / groups, c = k % groups;
    const int64_t g = r % 2 ? groups - 1 - c : c;
    const size_t at = (size_t)(2 * (g * plan->pg + r));
    plan->order[at] = by[k];
    plan->order[at + 1] = deg[by[k]];
  }
  return true;
}

// The LDS limit of a problem's slab kernel: once, when it is created.
hipError_t slab_lds_limit(int prec, bool masked) {
  const void *k = masked ? (const void *)k_point_slab<kMixed, true> : (const void *)k_point_slab<kMixed, false>;
  if (prec == kF32) k = masked ? (const void *)k_point_slab<kF32, true> : (const void *)k_point_slab<kF32, false>;
  if (prec == kF64) k = masked ? (const void *)k_point_slab<kF64, true> : (const void *)k_point_slab<kF64, false>;
  return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPointSlabBytes);
}

template <int PREC, bool MASK>
static void launch_slab(Problem *P, const PointArgs &a) {
  const SlabArgs sl{P->slab.tiles, P->slab.tpb, P->slab.groups, P->slab.pg,
                    reinterpret_cast<const int2 *>(P->slab_order)};
  klaunch(k_point_slab<PREC, MASK>, dim3(P->slab.blocks), dim3(kSlabNT), P->slab.lds, P->stream, P->pev[0], P->pev[1],
          a, sl);
}

void launch_point_slab(Problem *P, const PointArgs &a) {
  if (P->precision == kF32) P->M ? launch_slab<kF32, true>(P, a) : launch_slab<kF32, false>(P, a);
  else if (P->precision == kF64) P->M ? launch_slab<kF64, true>(P, a) : launch_slab<kF64, false>(P, a);
  else P->M ? launch_slab<kMixed, true>(P, a) : launch_slab<kMixed, false>(P, a);
}

// Before the first slab sweep of a solve.
void launch_slab_start(Problem *P) {
  const int64_t slots = P->n * P->ell_s;
  hipLaunchKernelGGL(k_q_from_s, dim3((unsigned)cdiv(slots, 256)), dim3(256), 0, P->stream, slots, P->colE, P->eidE,
                     P->s, P->qE);
}

}  // namespace ccmi
