// Interior-point glue around the hot path: IPM diagonals and residuals of the
// augmented system (paper: KKT conditions with barrier homotopy, residuals
// r1..r4), the scaled KKT error, the barrier objective and constraint
// violation of the filter line search, fraction-to-boundary step lengths and
// the iterate update.  Reductions meet in a fixed tree (lanes, wavefronts,
// workgroups in order), so every scalar is reproducible run to run; what the
// host decides on goes straight into its own pinned memory (IpmDev::hs).
//
// At one scenario every kernel here is a handful of dependent loads on a few
// hundred elements, so what counts is how many launches and how many
// dependent rounds a pass over the iterate takes.  118-bus grid, one
// scenario, per iteration: residuals (17 us, one dependent chain of loads per
// term) + their u part (4) + KKT scalars (10, 60 barriers) became two
// launches of 13 and 8 us, bound-multiplier steps + step scalars +
// trial point (5 + 9 + 3) two of 5 us, the merit 5 us instead of 7.
#include "ipm.h"

#include <algorithm>

namespace rkkt {

namespace {

constexpr int kBlock = 256;
constexpr int kRed = 1024;

inline unsigned grid_for(long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

__device__ inline bool fin(double v) { return isfinite(v); }

// Sigma contribution and barrier gradient of one boxed variable
__device__ inline void box_terms(double v, double lo, double hi, double zl, double zu, double mu,
                                 double* sigma, double* bgrad, double* bdual) {
  double sg = 0.0, bg = 0.0, bd = 0.0;
  if (fin(lo)) { double dl = v - lo; sg += zl / dl; bg -= mu / dl; bd -= zl; }
  if (fin(hi)) { double du = hi - v; sg += zu / du; bg += mu / du; bd += zu; }
  *sigma = sg;
  *bgrad = bg;
  *bdual = bd;
}

// ---- reductions: the kinds of the values that a kernel reduces together
enum Red { kSum, kMax, kMin };

template <Red kR>
__device__ __forceinline__ double red2(double a, double b) {
  return kR == kSum ? a + b : kR == kMax ? fmax(a, b) : fmin(a, b);
}

// v[q] over the workgroup, every value at once: the lanes of a wavefront by a
// butterfly (the values' chains interleave), then the wavefronts in order
// through LDS; the result is in every thread
template <int kWaves, Red... kRs>
__device__ __forceinline__ void block_reduce(double (&v)[sizeof...(kRs)]) {
  constexpr int n = sizeof...(kRs);
  __shared__ double sh[kWaves][n];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    int q = 0;
    ((v[q] = red2<kRs>(v[q], __shfl_xor(v[q], o, 64)), ++q), ...);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int q = 0; q < n; ++q) sh[wv][q] = v[q];
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    int q = 0;
    ((v[q] = w == 0 ? sh[0][q] : red2<kRs>(v[q], sh[w][q]), ++q), ...);
  }
}

// value [r][n] of workgroup r's part, r over the workgroups, in every thread
template <int kWaves, Red... kRs>
__device__ __forceinline__ void parts_reduce(const double* part, int nparts, const double (&init)[sizeof...(kRs)],
                                             double (&v)[sizeof...(kRs)]) {
  constexpr int n = sizeof...(kRs);
#pragma unroll
  for (int q = 0; q < n; ++q) v[q] = init[q];
  for (int r = threadIdx.x; r < nparts; r += 64 * kWaves) {
    int q = 0;
    ((v[q] = red2<kRs>(v[q], part[(long long)r * n + q]), ++q), ...);
  }
  block_reduce<kWaves, kRs...>(v);
}

// acc + sum of a(j) b(j), j in [j0, j1) in order; the loads of kTb terms (the
// indices, then the values they name) are issued together, so a column costs
// one round of dependent loads per kTb entries
constexpr int kTb = 8;
template <typename A, typename B>
__device__ __forceinline__ double dot_terms(double acc, int j0, int j1, A a, B b) {
  for (int j = j0; j < j1; j += kTb) {
    double va[kTb], vb[kTb];
#pragma unroll
    for (int q = 0; q < kTb; ++q) {
      const int jj = min(j + q, j1 - 1);
      va[q] = a(jj);
      vb[q] = b(jj);
    }
#pragma unroll
    for (int q = 0; q < kTb; ++q)
      if (j + q < j1) acc += va[q] * vb[q];
  }
  return acc;
}

// complementarity of one boxed variable: the smallest and the largest
// (v - bound) z (every |comp - mu| follows from them, whatever mu is) and the
// sum of the bound multipliers
__device__ inline void comp_terms(double v, double lo, double hi, double zl, double zu, double* cmin,
                                  double* cmax, double* zs) {
  if (fin(lo)) {
    const double a = (v - lo) * zl;
    *cmin = fmin(*cmin, a);
    *cmax = fmax(*cmax, a);
    *zs += fabs(zl);
  }
  if (fin(hi)) {
    const double a = (hi - v) * zu;
    *cmin = fmin(*cmin, a);
    *cmax = fmax(*cmax, a);
    *zs += fabs(zu);
  }
}

// r1x, dx, Sigma_x (x part); per-scenario u gradient of the Lagrangian (u part);
// r2, ds, r4, Sigma_s (s part); the workgroup's share of the KKT scalars
__global__ __launch_bounds__(kBlock) void k_resid(DP d, IpmDev s, double mu) {
  const long long per = (long long)d.nx + d.nu + d.m;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double dmax = 0.0, pmax = 0.0, cmin = INFINITY, cmax = -INFINITY, ysum = 0.0, zs = 0.0;
  if (t < (long long)d.N * per) {
    const int k = (int)(t / per);
    int i = (int)(t % per);
    const double* ev = d.EV + (long long)k * d.n_ev;
    const double* hv = ev + d.off_h;
    const double* yk = s.y + (long long)k * d.nx;
    const double* zk = s.z + (long long)k * d.m;
    auto ht = [&](double acc, int v) {
      return dot_terms(acc, d.ht_ptr[v], d.ht_ptr[v + 1], [&](int j) { return hv[d.ht_pos[j]]; },
                       [&](int j) { return zk[d.ht_row[j]]; });
    };
    if (i < d.nx) {
      const int ih = d.pinv[i];
      const long long q = (long long)k * d.nx + i;
      double acc = dot_terms(s.gx[q], d.gxc_ptr[ih], d.gxc_ptr[ih + 1],
                             [&](int j) { return ev[d.off_gx + d.gxc_pos[j]]; },
                             [&](int j) { return yk[d.perm[d.gxc_row[j]]]; });
      acc = ht(acc, ih);
      double sg, bg, bd;
      box_terms(s.x[q], s.xl[i], s.xu[i], s.zlx[q], s.zux[q], mu, &sg, &bg, &bd);
      const double dx = acc + bd, gq = s.g[q];
      s.sx[q] = sg;
      s.r1x[q] = acc + bg;
      s.dx[q] = dx;
      s.r3[q] = gq;
      dmax = fabs(dx);
      pmax = fabs(gq);
      ysum = fabs(yk[i]);
      comp_terms(s.x[q], s.xl[i], s.xu[i], s.zlx[q], s.zux[q], &cmin, &cmax, &zs);
    } else if (i < d.nx + d.nu) {
      i -= d.nx;
      const double acc = dot_terms(s.gu[(long long)k * d.nu + i], d.guc_ptr[i], d.guc_ptr[i + 1],
                                   [&](int j) { return ev[d.off_gu + d.guc_pos[j]]; },
                                   [&](int j) { return yk[d.perm[d.guc_row[j]]]; });
      s.cu[(long long)k * d.nu + i] = ht(acc, d.nx + i);
    } else {
      i -= d.nx + d.nu;
      const long long q = (long long)k * d.m + i;
      double sg, bg, bd;
      box_terms(s.s[q], s.sl[i], s.su[i], s.zls[q], s.zus[q], mu, &sg, &bg, &bd);
      const double ds = zk[i] + bd, r4 = s.h[q] + s.s[q];
      s.ss[q] = sg;
      s.r2[q] = zk[i] + bg;
      s.ds[q] = ds;
      s.r4[q] = r4;
      dmax = fabs(ds);
      pmax = fabs(r4);
      ysum = fabs(zk[i]);
      comp_terms(s.s[q], s.sl[i], s.su[i], s.zls[q], s.zus[q], &cmin, &cmax, &zs);
    }
  }
  double v[6] = {dmax, pmax, cmin, cmax, ysum, zs};
  block_reduce<kBlock / 64, kMax, kMax, kMin, kMax, kSum, kSum>(v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 6; ++q) s.part[6LL * blockIdx.x + q] = v[q];
}

// the u part of the residuals and the KKT scalars: out [0] max dual, [1] max
// primal, [2] min comp, [3] max comp, [4] sum |y| + |z|, [5] sum |bound
// duals|.  One workgroup: lane c of a wavefront adds its column's scenario
// gradients over the wavefront's share of the scenarios, the shares meet in
// wavefront order.
__global__ __launch_bounds__(kRed) void k_resid_fin(DP d, IpmDev s, double mu, int nparts, double* out) {
  constexpr int kW = kRed / 64;
  __shared__ double sh[kW][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int per = (d.N + kW - 1) / kW, k0 = min(d.N, wv * per), k1 = min(d.N, k0 + per);
  double dmax = 0.0, cmin = INFINITY, cmax = -INFINITY, zs = 0.0;
  for (int c0 = 0; c0 < d.nu; c0 += 64) {
    const int c = c0 + lane;
    double acc = 0.0;
    if (c < d.nu)
      for (int k = k0; k < k1; k += kTb) {
        double v[kTb];
#pragma unroll
        for (int q = 0; q < kTb; ++q) v[q] = s.cu[(long long)min(k + q, k1 - 1) * d.nu + c];
#pragma unroll
        for (int q = 0; q < kTb; ++q)
          if (k + q < k1) acc += v[q];
      }
    sh[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && c < d.nu) {
      acc = sh[0][lane];
      for (int w = 1; w < kW; ++w) acc += sh[w][lane];
      double sg, bg, bd;
      box_terms(s.u[c], s.ul[c], s.uu[c], s.zlu[c], s.zuu[c], mu, &sg, &bg, &bd);
      const double du = acc + bd;
      s.sgu[c] = sg;
      s.r1u[c] = acc + bg;
      s.du[c] = du;
      dmax = fmax(dmax, fabs(du));
      comp_terms(s.u[c], s.ul[c], s.uu[c], s.zlu[c], s.zuu[c], &cmin, &cmax, &zs);
    }
    __syncthreads();
  }
  const double init[6] = {dmax, 0.0, cmin, cmax, 0.0, zs};
  double v[6];
  parts_reduce<kW, kMax, kMax, kMin, kMax, kSum, kSum>(s.part, nparts, init, v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 6; ++q) out[q] = v[q];
}

__device__ inline double logbox(double v, double lo, double hi, int* bad) {
  double r = 0.0;
  if (fin(lo)) { double a = v - lo; if (!(a > 0.0)) *bad = 1; else r += log(a); }
  if (fin(hi)) { double b = hi - v; if (!(b > 0.0)) *bad = 1; else r += log(b); }
  return r;
}

// merit of a primal point (x, u, s) with its f, g, h:
// out: [0] sum f, [1] theta = |g|_1 + |h + s|_1, [2] log-barrier sum, [3] bad (1 if outside)
// One workgroup up to kMeritPer elements per thread (the result goes to out
// itself), more workgroups above that and their parts to k_merit_fin.
constexpr int kMeritPer = 4, kMeritBlocks = 256;

inline unsigned merit_blocks(const DP& d) {
  const long long n = (long long)d.N * (d.nx + d.m) + d.nu, per = (long long)kMeritPer * kRed;
  return (unsigned)std::min<long long>(kMeritBlocks, (n + per - 1) / per);
}

__global__ __launch_bounds__(kRed) void k_merit(DP d, IpmDev s, const double* x, const double* u,
                                                const double* sv, const double* f, const double* g,
                                                const double* h, double* out) {
  int bad = 0;
  double fs = 0.0, th = 0.0, lg = 0.0;
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  const long long t0 = (long long)blockIdx.x * kRed + threadIdx.x, dt = (long long)gridDim.x * kRed;
  for (long long t = t0; t < nxN + nmN + d.nu; t += dt) {
    if (t < nxN) {
      const int i = (int)(t % d.nx);
      th += fabs(g[t]);
      lg += logbox(x[t], s.xl[i], s.xu[i], &bad);
    } else if (t < nxN + nmN) {
      const long long q = t - nxN;
      const int i = (int)(q % d.m);
      th += fabs(h[q] + sv[q]);
      lg += logbox(sv[q], s.sl[i], s.su[i], &bad);
    } else {
      const int c = (int)(t - nxN - nmN);
      lg += logbox(u[c], s.ul[c], s.uu[c], &bad);
    }
  }
  for (long long k = t0; k < d.N; k += dt) fs += f[k];
  double v[4] = {fs, th, lg, bad ? 1.0 : 0.0};
  block_reduce<kRed / 64, kSum, kSum, kSum, kMax>(v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[4LL * blockIdx.x + q] = v[q];
}

__global__ __launch_bounds__(kMeritBlocks) void k_merit_fin(IpmDev s, int nparts, double* out) {
  const double init[4] = {0.0, 0.0, 0.0, 0.0};
  double v[4];
  parts_reduce<kMeritBlocks / 64, kSum, kSum, kSum, kMax>(s.part, nparts, init, v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = v[q];
}

// bound-dual steps: p_zL = mu/(v-l) - zL - zL/(v-l) p, p_zU = mu/(u-v) - zU + zU/(u-v) p
__device__ inline void dual_step(double v, double p, double lo, double hi, double zl, double zu,
                                 double mu, double* pl, double* pu) {
  *pl = 0.0;
  *pu = 0.0;
  if (fin(lo)) { double a = v - lo; *pl = mu / a - zl - zl / a * p; }
  if (fin(hi)) { double b = hi - v; *pu = mu / b - zu + zu / b * p; }
}

__device__ inline double primal_ratio(double v, double p, double lo, double hi, double tau) {
  double a = 1.0;
  if (fin(lo) && p < 0.0) a = fmin(a, -tau * (v - lo) / p);
  if (fin(hi) && p > 0.0) a = fmin(a, tau * (hi - v) / p);
  return a;
}

__device__ inline double dual_ratio(double z, double p, double tau) {
  return p < 0.0 ? fmin(1.0, -tau * z / p) : 1.0;
}

// bound-multiplier steps and, per workgroup, the largest step lengths (primal
// and bound multipliers) and grad(phi)^T d
__global__ __launch_bounds__(kBlock) void k_step_scalars(DP d, IpmDev s, double mu, double tau) {
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double ap = 1.0, az = 1.0, dphi = 0.0;
  auto one = [&](double v, double p, double lo, double hi, double zl, double zu, double grad, double* pzl,
                 double* pzu) {
    double pl, pu, sg, bg, bd;
    dual_step(v, p, lo, hi, zl, zu, mu, &pl, &pu);
    *pzl = pl;
    *pzu = pu;
    ap = primal_ratio(v, p, lo, hi, tau);
    az = fmin(dual_ratio(zl, pl, tau), dual_ratio(zu, pu, tau));
    box_terms(v, lo, hi, 0.0, 0.0, mu, &sg, &bg, &bd);
    dphi = (grad + bg) * p;
  };
  if (t < nxN) {
    const int i = (int)(t % d.nx);
    one(s.x[t], s.px[t], s.xl[i], s.xu[i], s.zlx[t], s.zux[t], s.gx[t], &s.pzlx[t], &s.pzux[t]);
  } else if ((t -= nxN) < nmN) {
    const int i = (int)(t % d.m);
    one(s.s[t], s.ps[t], s.sl[i], s.su[i], s.zls[t], s.zus[t], 0.0, &s.pzls[t], &s.pzus[t]);
  } else if ((t -= nmN) < d.nu) {
    const int c = (int)t;
    double gsum = 0.0;
    for (int k = 0; k < d.N; k += kTb) {
      double v[kTb];
#pragma unroll
      for (int q = 0; q < kTb; ++q) v[q] = s.gu[(long long)min(k + q, d.N - 1) * d.nu + c];
#pragma unroll
      for (int q = 0; q < kTb; ++q)
        if (k + q < d.N) gsum += v[q];
    }
    one(s.u[c], s.pu[c], s.ul[c], s.uu[c], s.zlu[c], s.zuu[c], gsum, &s.pzlu[c], &s.pzuu[c]);
  }
  double v[3] = {ap, az, dphi};
  block_reduce<kBlock / 64, kMin, kMin, kSum>(v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) s.part[3LL * blockIdx.x + q] = v[q];
}

// Many parts of k_step_scalars down to one, in place, by one workgroup in the
// order in which a workgroup of k_trial adds them.  Every workgroup of k_trial
// reads all parts, work that grows with the square of their number: beyond 2048
// (of 256 elements each) this launch comes first.  118 buses x 4000 scenarios 5296
// to 5230 us per iteration; x 256 (636 parts) it would cost 3 us more than it saves.
constexpr int kTrialParts = 2048;
__global__ __launch_bounds__(kBlock) void k_step_fin(IpmDev s, int nparts) {
  const double init[3] = {1.0, 1.0, 0.0};
  double v[3];
  parts_reduce<kBlock / 64, kMin, kMin, kSum>(s.part, nparts, init, v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) s.part[q] = v[q];
}

// trial point x + alpha p.  With nparts > 0, alpha is the largest primal step
// of k_step_scalars' parts, which every workgroup reduces for itself; the
// first also reports them to the host: out [0] alpha_max primal, [1] alpha_z,
// [2] grad(phi)^T d, [3] info of the factorisation, [4], [5] device status
// (which is cleared).
__global__ __launch_bounds__(kBlock) void k_trial(DP d, IpmDev s, double alpha, int nparts, double* out) {
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (nparts > 0) {
    const double init[3] = {1.0, 1.0, 0.0};
    double v[3];
    parts_reduce<kBlock / 64, kMin, kMin, kSum>(s.part, nparts, init, v);
    alpha = v[0];
    if (t == 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q) out[q] = v[q];
      out[3] = *s.info;
      out[4] = d.status[0];
      out[5] = d.status[1];
      d.status[0] = 0;
      d.status[1] = 0;
    }
  }
  if (t < nxN) { s.xt[t] = s.x[t] + alpha * s.px[t]; return; }
  t -= nxN;
  if (t < nmN) { s.st[t] = s.s[t] + alpha * s.ps[t]; return; }
  t -= nmN;
  if (t < d.nu) s.ut[t] = s.u[t] + alpha * s.pu[t];
}

__device__ inline void safeguard(double v, double lo, double hi, double mu, double ks, double* zl,
                                 double* zu) {
  if (fin(lo)) { double a = v - lo; *zl = fmax(fmin(*zl, ks * mu / a), mu / (ks * a)); } else *zl = 0.0;
  if (fin(hi)) { double b = hi - v; *zu = fmax(fmin(*zu, ks * mu / b), mu / (ks * b)); } else *zu = 0.0;
}

// the accepted trial point becomes the iterate; y, z and the bound
// multipliers take their steps
__global__ void k_accept(DP d, IpmDev s, double alpha, double alpha_z, double mu, double ks) {
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nxN) {
    const int i = (int)(t % d.nx);
    s.x[t] = s.xt[t];
    s.y[t] += alpha * s.py[t];
    double zl = s.zlx[t] + alpha_z * s.pzlx[t], zu = s.zux[t] + alpha_z * s.pzux[t];
    safeguard(s.x[t], s.xl[i], s.xu[i], mu, ks, &zl, &zu);
    s.zlx[t] = zl;
    s.zux[t] = zu;
    return;
  }
  t -= nxN;
  if (t < nmN) {
    const int i = (int)(t % d.m);
    s.s[t] = s.st[t];
    s.z[t] += alpha * s.pz[t];
    double zl = s.zls[t] + alpha_z * s.pzls[t], zu = s.zus[t] + alpha_z * s.pzus[t];
    safeguard(s.s[t], s.sl[i], s.su[i], mu, ks, &zl, &zu);
    s.zls[t] = zl;
    s.zus[t] = zu;
    return;
  }
  t -= nmN;
  if (t < d.nu) {
    const int c = (int)t;
    s.u[c] = s.ut[c];
    double zl = s.zlu[c] + alpha_z * s.pzlu[c], zu = s.zuu[c] + alpha_z * s.pzuu[c];
    safeguard(s.u[c], s.ul[c], s.uu[c], mu, ks, &zl, &zu);
    s.zlu[c] = zl;
    s.zuu[c] = zu;
  }
}

// push v inside [lo, hi]: distance min(k1 max(1,|bound|), k2 (hi - lo))
__device__ inline double push(double v, double lo, double hi, double k1, double k2) {
  double pl = fin(lo) ? k1 * fmax(1.0, fabs(lo)) : 0.0;
  double pu = fin(hi) ? k1 * fmax(1.0, fabs(hi)) : 0.0;
  if (fin(lo) && fin(hi)) { pl = fmin(pl, k2 * (hi - lo)); pu = fmin(pu, k2 * (hi - lo)); }
  if (fin(lo)) v = fmax(v, lo + pl);
  if (fin(hi)) v = fmin(v, hi - pu);
  return v;
}

// start point: theta 0, V 1, Pg mid-range, pushed inside; y = z = 0; bound duals 1
__global__ void k_init_primal(DP d, IpmDev s, double k1, double k2) {
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nxN) {
    const int i = (int)(t % d.nx);
    double v0 = i < d.nb - 1 ? 0.0 : 1.0;
    s.x[t] = push(v0, s.xl[i], s.xu[i], k1, k2);
    s.y[t] = 0.0;
    s.zlx[t] = fin(s.xl[i]) ? 1.0 : 0.0;
    s.zux[t] = fin(s.xu[i]) ? 1.0 : 0.0;
    return;
  }
  t -= nxN;
  if (t < nmN) {
    const int i = (int)(t % d.m);
    s.z[t] = 0.0;
    s.s[t] = 0.0;
    s.zls[t] = fin(s.sl[i]) ? 1.0 : 0.0;
    s.zus[t] = fin(s.su[i]) ? 1.0 : 0.0;
    return;
  }
  t -= nmN;
  if (t < d.nu) {
    const int c = (int)t;
    double v0 = c < d.ng ? 1.0 : 0.5 * (s.ul[c] + s.uu[c]);
    s.u[c] = push(v0, s.ul[c], s.uu[c], k1, k2);
    s.zlu[c] = fin(s.ul[c]) ? 1.0 : 0.0;
    s.zuu[c] = fin(s.uu[c]) ? 1.0 : 0.0;
  }
}

__global__ void k_init_slack(DP d, IpmDev s, double k1, double k2) {
  const long long nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nmN) return;
  const int i = (int)(t % d.m);
  s.s[t] = push(-s.h[t], s.sl[i], s.su[i], k1, k2);
}

// warm start, primal part: x0, u0 pushed into the boxes
__global__ void k_warm_primal(DP d, IpmDev s, const double* x0, const double* u0, double k1, double k2) {
  const long long nxN = (long long)d.N * d.nx;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nxN) {
    const int i = (int)(t % d.nx);
    s.x[t] = push(x0[t], s.xl[i], s.xu[i], k1, k2);
  } else if (t - nxN < d.nu) {
    const int c = (int)(t - nxN);
    s.u[c] = push(u0[c], s.ul[c], s.uu[c], k1, k2);
  }
}

// warm start, dual part: y = mult y0, z = mult z0, and every bound
// multiplier from complementarity at mu0 (mu0 / gap), after the slacks
__global__ void k_warm_duals(DP d, IpmDev s, const double* y0, const double* z0, double mult, double mu0) {
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nxN) {
    const int i = (int)(t % d.nx);
    s.y[t] = mult * y0[t];
    s.zlx[t] = fin(s.xl[i]) ? mu0 / (s.x[t] - s.xl[i]) : 0.0;
    s.zux[t] = fin(s.xu[i]) ? mu0 / (s.xu[i] - s.x[t]) : 0.0;
    return;
  }
  t -= nxN;
  if (t < nmN) {
    const int i = (int)(t % d.m);
    s.z[t] = mult * z0[t];
    s.zls[t] = fin(s.sl[i]) ? mu0 / (s.s[t] - s.sl[i]) : 0.0;
    s.zus[t] = fin(s.su[i]) ? mu0 / (s.su[i] - s.s[t]) : 0.0;
    return;
  }
  t -= nmN;
  if (t < d.nu) {
    const int c = (int)t;
    s.zlu[c] = fin(s.ul[c]) ? mu0 / (s.u[c] - s.ul[c]) : 0.0;
    s.zuu[c] = fin(s.uu[c]) ? mu0 / (s.uu[c] - s.u[c]) : 0.0;
  }
}

// warm start, bound multipliers implied by stationarity (after k_resid with
// the complementarity multipliers of k_warm_duals): v = the derivative of the
// Lagrangian without bound terms (dual infeasibility plus the current bound
// terms), lower multiplier mu0 / gap + max(v, 0), upper mu0 / gap + max(-v, 0)
__device__ inline void implied_pair(double val, double lo, double hi, double v, double mu0, double* zl,
                                    double* zu) {
  *zl = fin(lo) ? mu0 / (val - lo) + fmax(v, 0.0) : 0.0;
  *zu = fin(hi) ? mu0 / (hi - val) + fmax(-v, 0.0) : 0.0;
}

__global__ void k_warm_implied(DP d, IpmDev s, double mu0) {
  const long long nxN = (long long)d.N * d.nx, nmN = (long long)d.N * d.m;
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nxN) {
    const int i = (int)(t % d.nx);
    const double v = s.dx[t] + s.zlx[t] - s.zux[t];
    implied_pair(s.x[t], s.xl[i], s.xu[i], v, mu0, &s.zlx[t], &s.zux[t]);
    return;
  }
  t -= nxN;
  if (t < nmN) {
    const int i = (int)(t % d.m);
    const double v = s.ds[t] + s.zls[t] - s.zus[t];
    implied_pair(s.s[t], s.sl[i], s.su[i], v, mu0, &s.zls[t], &s.zus[t]);
    return;
  }
  t -= nmN;
  if (t < d.nu) {
    const int c = (int)t;
    const double v = s.du[c] + s.zlu[c] - s.zuu[c];
    implied_pair(s.u[c], s.ul[c], s.uu[c], v, mu0, &s.zlu[c], &s.zuu[c]);
  }
}

// out[0] = max(max |grad_x f_i|, max |sum_i grad_u f_i|)
__global__ __launch_bounds__(kRed) void k_grad_max(DP d, IpmDev s, double* out) {
  double v[1] = {0.0};
  const long long nxN = (long long)d.N * d.nx;
  for (long long q = threadIdx.x; q < nxN; q += kRed) v[0] = fmax(v[0], fabs(s.gx[q]));
  for (int c = threadIdx.x; c < d.nu; c += kRed) {
    double acc = 0.0;
    for (int k = 0; k < d.N; ++k) acc += s.gu[(long long)k * d.nu + c];
    v[0] = fmax(v[0], fabs(acc));
  }
  block_reduce<kRed / 64, kMax>(v);
  if (threadIdx.x == 0) out[0] = v[0];
}

}  // namespace

// parts of the reductions: the largest of the workgroups' counts of k_resid
// (6 values each), k_step_scalars (3) and k_merit (4)
long long ipm_part_doubles(const DP& d) {
  const long long n = (long long)d.N * (d.nx + d.nu + d.m), n1 = (long long)d.N * (d.nx + d.m) + d.nu;
  return std::max<long long>({6LL * grid_for(n), 3LL * grid_for(n1), 4LL * kMeritBlocks});
}

void ipm_resid(const DP& d, const IpmDev& s, double mu, double* out, hipStream_t st) {
  const unsigned nb = grid_for((long long)d.N * (d.nx + d.nu + d.m));
  k_resid<<<nb, kBlock, 0, st>>>(d, s, mu);
  k_resid_fin<<<1, kRed, 0, st>>>(d, s, mu, (int)nb, out);
}

void ipm_merit(const DP& d, const IpmDev& s, bool trial, double* out, hipStream_t st) {
  const unsigned nb = merit_blocks(d);
  double* o = nb > 1 ? s.part : out;
  if (trial) k_merit<<<nb, kRed, 0, st>>>(d, s, s.xt, s.ut, s.st, s.ft, s.gt, s.ht, o);
  else k_merit<<<nb, kRed, 0, st>>>(d, s, s.x, s.u, s.s, s.f, s.g, s.h, o);
  if (nb > 1) k_merit_fin<<<1, kMeritBlocks, 0, st>>>(s, (int)nb, out);
}

void ipm_step_trial(const DP& d, const IpmDev& s, double mu, double tau, double* out, hipStream_t st) {
  const unsigned nb = grid_for((long long)d.N * (d.nx + d.m) + d.nu);
  k_step_scalars<<<nb, kBlock, 0, st>>>(d, s, mu, tau);
  const bool many = nb > (unsigned)kTrialParts;
  if (many) k_step_fin<<<1, kBlock, 0, st>>>(s, (int)nb);
  k_trial<<<nb, kBlock, 0, st>>>(d, s, 0.0, many ? 1 : (int)nb, out);
}

void ipm_trial(const DP& d, const IpmDev& s, double alpha, hipStream_t st) {
  const long long n = (long long)d.N * (d.nx + d.m) + d.nu;
  k_trial<<<grid_for(n), kBlock, 0, st>>>(d, s, alpha, 0, nullptr);
}

void ipm_accept(const DP& d, const IpmDev& s, double alpha, double alpha_z, double mu, double ks,
                hipStream_t st) {
  const long long n = (long long)d.N * (d.nx + d.m) + d.nu;
  k_accept<<<grid_for(n), kBlock, 0, st>>>(d, s, alpha, alpha_z, mu, ks);
}

void ipm_init_primal(const DP& d, const IpmDev& s, double k1, double k2, hipStream_t st) {
  const long long n = (long long)d.N * (d.nx + d.m) + d.nu;
  k_init_primal<<<grid_for(n), kBlock, 0, st>>>(d, s, k1, k2);
}

void ipm_init_slack(const DP& d, const IpmDev& s, double k1, double k2, hipStream_t st) {
  const long long n = (long long)d.N * d.m;
  k_init_slack<<<grid_for(n), kBlock, 0, st>>>(d, s, k1, k2);
}

void ipm_warm_primal(const DP& d, const IpmDev& s, const double* x0, const double* u0, double k1, double k2,
                     hipStream_t st) {
  const long long n = (long long)d.N * d.nx + d.nu;
  k_warm_primal<<<grid_for(n), kBlock, 0, st>>>(d, s, x0, u0, k1, k2);
}

void ipm_warm_implied(const DP& d, const IpmDev& s, double mu0, hipStream_t st) {
  const long long n = (long long)d.N * (d.nx + d.m) + d.nu;
  k_warm_implied<<<grid_for(n), kBlock, 0, st>>>(d, s, mu0);
}

void ipm_warm_duals(const DP& d, const IpmDev& s, const double* y0, const double* z0, double mult, double mu0,
                    hipStream_t st) {
  const long long n = (long long)d.N * (d.nx + d.m) + d.nu;
  k_warm_duals<<<grid_for(n), kBlock, 0, st>>>(d, s, y0, z0, mult, mu0);
}

void ipm_grad_max(const DP& d, const IpmDev& s, double* out, hipStream_t st) {
  k_grad_max<<<1, kRed, 0, st>>>(d, s, out);
}

}  // namespace rkkt
