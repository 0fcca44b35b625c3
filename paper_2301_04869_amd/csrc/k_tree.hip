// Reduction on the elimination tree of dense fronts (tree.h): the form that
// the adjoint closure takes when its panels do not fit on chip.
//
// A scenario's bordered system
//     [K_xx  K_xu  G_x^T]
//     [K_ux  K_uu  G_u^T]     reduced to  Z^T K Z,  Z = [-G_x^-1 G_u; I],
//     [G_x   G_u        ]
// is reduced node by node instead of column by column.  At a node with pivot
// rows J, interface rows I and control columns U (C = I and U together),
//     V = G_JJ^-1 G_JC,            G_IC <- G_IC - G_IJ V,
//     Y = K_JC - K_JJ V / 2,       K_CC <- K_CC - V^T Y - Y^T V,
// which is the same elimination (x_J = -V x_C) that the column-wise solves
// perform, with the same pivots.  G_IC and K_IC go to the parent; K_UU is
// never assembled: its updates -(V_U^T Y_U + Y_U^T V_U) of all nodes and
// scenarios are one stacked product at the end.
//
// Against the panel solves that this replaces (one 64-column panel of T and
// L_x per workgroup in device memory, every term of four triangular solves a
// 512-byte gather), a front is read and written once and all its work is
// 16 x 16 x 4 FP64 matrix products on registers: at 9241 buses, 16 scenarios
// 105 GFLOP on 1.7 GB of fronts against 335 GB of panel traffic, 5.1 ms
// (fronts 2.7, product 2.3, sum 0.1) against 90.7.
#include "device.h"

namespace rkkt {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kTT = 256;  // threads of the tree kernels (4 wavefronts)
constexpr int kTF = 512;  // threads of the pivot kernel
constexpr int kFrontKids = 32;  // children whose records it keeps in LDS
constexpr int kTld = kTreeRows + 4;  // rows of G_JJ in LDS four 8-byte banks apart

// pivot kernel of a level: 1 maps in LDS, 2 all strips in the same launch
// (levels whose nodes hold at most kFuseStrips strips: beyond, one workgroup's
// matrix cores take longer over them than a second launch over many.  Limits
// 0, 3, 6, 10, 16 at 300 buses x 16: 617, 610, 586, 577, 584 us per pass; at
// 1354 x 8: 1653, 1636, 1623, 1610, 1603; at 2869 x 8 3401 to 3379)
constexpr int kFuseStrips = 10;
int front_variant(const Tree& t, int l) {
  return (t.lev_map[l] <= kTreeMapLds ? 1 : 0) + (t.lev_cs[l] <= kFuseStrips ? 2 : 0);
}
// its LDS: G_JJ, the pool blocks and the children's maps
size_t front_lds(const Tree& t, int l) {
  const int v = front_variant(t, l), ib = t.lev_ib[l], st = v & 2 ? t.lev_cs[l] : ib;
  const size_t blocks = 2 * kTreeNB * kTreeNB + (size_t)kTreeNB * (ib + 2 * st);
  return 8 * (size_t)kTreeRows * kTld + 4 * blocks + (v & 1 ? 2 * (size_t)t.lev_map[l] + 4 : 0);
}
// the most that the device allows it next to its static arrays
constexpr int kFrontLdsMax = 120 * 1024;

__device__ inline void tree_status(const DP& d, int code, int k) {
  if (atomicCAS(d.status, 0, code) == 0) d.status[1] = k;
}

// Blocks are row-major, so register r of a lane holds row lane/16 + 4 r,
// column lane%16: the accumulator layout of v_mfma_f64_16x16x4f64, which is
// also its B operand of step r and, for the block's transpose, its A operand.
__device__ __forceinline__ v4d load_blk(const double* p, int lane) {
  v4d v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = p[64 * r + lane];
  return v;
}
__device__ __forceinline__ void store_blk(double* p, const v4d& v, int lane) {
#pragma unroll
  for (int r = 0; r < 4; ++r) p[64 * r + lane] = v[r];
}
// acc - A B, with `at` the block of A^T
__device__ __forceinline__ v4d mul_sub(const v4d& at, const v4d& b, v4d acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-at[r], b[r], acc, 0, 0, 0);
  return acc;
}
__device__ __forceinline__ v4d mul_add(const v4d& at, const v4d& b, v4d acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(at[r], b[r], acc, 0, 0, 0);
  return acc;
}

// ------------------------------------------------------- original entries
// Pool block b of scenario k: its entries of G_x, G_u (EV) or K, zeros
// elsewhere.  One wavefront per block.
__device__ __forceinline__ void tree_orig_body(const DP& d, int bx, int k) {
  __shared__ double blk[4][kTreeBlk];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = bx * 4 + wv;
  if (b >= d.tr.npool) return;
  double* s = blk[wv];
#pragma unroll
  for (int r = 0; r < 4; ++r) s[64 * r + lane] = 0.0;
  const double* ev = d.EV + (long long)k * d.n_ev;
  const double* kv = d.K + (long long)k * d.nnz_k;
  const int e1 = d.tr.optr[b + 1];
  wave_sync();
  for (int e = d.tr.optr[b] + lane; e < e1; e += 64) {
    const int at = d.tr.oent[2 * e], src = d.tr.oent[2 * e + 1];
    s[at] = src >= 0 ? ev[src] : kv[~src];
  }
  wave_sync();
  double* o = d.tr.pool + ((long long)k * d.tr.npool + b) * kTreeBlk;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[64 * r + lane] = s[64 * r + lane];
}

__device__ __forceinline__ v4d pool_blk(const double* pool, int b, int lane) {
  return b >= 0 ? load_blk(pool + (long long)b * kTreeBlk, lane) : v4d{0.0, 0.0, 0.0, 0.0};
}

// The children of a node and their row maps; kLds: maps staged in LDS.
struct Kids {
  const TreeChild* ch;
  const short *map, *smap;  // of child a: map + a * len, smap + a * us
  int n, len, us;
};
__device__ __forceinline__ Kids kids_global(const DP& d, const TreeNode& n) {
  return Kids{d.tr.children + n.child0, d.tr.rmap + n.rmap0, d.tr.smap + n.smap0, n.nchild,
              kTreeB * (n.nb + n.ib),   n.us};
}

// whether child c maps rows into the parent's block row b
__device__ __forceinline__ bool kid_has(const TreeChild& c, int b) {
  const unsigned long long m = c.blocks >> min(b, 63);
  return __builtin_amdgcn_readfirstlane((int)(m & 1)) != 0;
}

// Adds the children's updates to the NB blocks of rows from block row rb on of
// G_.U and K_.U in control strip c.  Only children that hold the strip are
// visited, and of those only the block rows that they map; all loads of a
// child are in flight together.
template <int NB>
__device__ __forceinline__ void add_ctrl(const Kids& kd, const double* slab, int rb, int c, int lane, v4d* g,
                                         v4d* kk) {
  const int lm = lane & 15, lk = lane >> 4;
  for (int a0 = 0; a0 < kd.n; a0 += 64) {
    const int cstv = a0 + lane < kd.n ? kd.smap[(a0 + lane) * kd.us + c] : -1;
    for (unsigned long long m = __ballot(cstv >= 0); m; m &= m - 1) {
      const int w = __ffsll((long long)m) - 1, a = a0 + w;
      const TreeChild& ch = kd.ch[a];
      const int cst = __builtin_amdgcn_readlane(cstv, w), ib = ch.ib;
      const short* rm = kd.map + a * kd.len + rb * kTreeB;
      const long long so = (long long)(ib + cst) * ib * kTreeBlk + lm;
      const double *gu = slab + ch.gu + so, *ku = slab + ch.ku + so;
      v4d vg[NB], vk[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        vg[b] = vk[b] = v4d{0.0, 0.0, 0.0, 0.0};
        if (kid_has(ch, rb + b))
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int ci = rm[b * kTreeB + 4 * r + lk];
            vg[b][r] = ci >= 0 ? gu[ci * kTreeB] : 0.0;
            vk[b][r] = ci >= 0 ? ku[ci * kTreeB] : 0.0;
          }
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          g[b][r] += vg[b][r];
          kk[b][r] += vk[b][r];
        }
    }
  }
}

// Adds the children's updates to one block whose rows and columns are both
// interface-mapped: element (row, col) of the parent, rows of block row rb,
// columns those of block row cb.  kG / kK: to g from G_IC, to kk from K_IC;
// kT: the block holds the transpose, element (row, col) taken from the
// child's (col, row).  Children that map nothing into the block are skipped;
// the loads of two children are in flight together.
template <bool kT, bool kG, bool kK>
__device__ __forceinline__ void add_mapped(const Kids& kd, const double* slab, int rb, int cb, int lane, v4d& g,
                                           v4d& kk) {
  const int lm = lane & 15, lk = lane >> 4;
  auto next = [&](int a) {
    while (a < kd.n && !(kid_has(kd.ch[a], rb) && kid_has(kd.ch[a], cb))) ++a;
    return a;
  };
  for (int a0 = next(0); a0 < kd.n;) {
    int a1 = next(a0 + 1);
    v4d vg[2], vk[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const int a = w == 0 ? a0 : min(a1, kd.n - 1);
      const TreeChild& ch = kd.ch[a];
      const short* rm = kd.map + a * kd.len;
      const int cj = w == 0 || a1 < kd.n ? rm[cb * kTreeB + lm] : -1;
      const long long gu = ch.gu, ku = ch.ku;
      const int pitch = ch.ib * kTreeBlk;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ci = rm[rb * kTreeB + 4 * r + lk];
        const bool in = ci >= 0 && cj >= 0;
        const int rr = kT ? cj : ci, cc = kT ? ci : cj;
        const long long at = in ? (long long)(cc >> 4) * pitch + rr * kTreeB + (cc & 15) : 0;
        if (kG) vg[w][r] = in ? slab[gu + at] : 0.0;
        if (kK) vk[w][r] = in ? slab[ku + at] : 0.0;
      }
    }
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (kG) g[r] += vg[w][r];
        if (kK) kk[r] += vk[w][r];
      }
    a0 = a1 < kd.n ? next(a1 + 1) : kd.n;
  }
}

// ------------------------------------------------------------ pivot blocks
// One Gauss-Jordan step of the in-place inverse of a 16 x 16 block held as
// x[r] = element (4 r + lane/16, lane%16): the 2 x 2 pivot block of rows and
// columns P and P + 1 (two rows per step, for half the dependent chains of a
// scalar step: 44 cycles per FP64 operation).  1/det from the reciprocal
// estimate r0 (good to about 2^-24) as r0 (1 + e + e^2), e = 1 - det r0.
// Lanes P and P + 1 of `pivots` get the two scalar pivots.
template <int P>
__device__ __forceinline__ void gj_step(double (&x)[4], double& pivots, int lane) {
  constexpr int q = P & 3, rr = P >> 2;
  const int lm = lane & 15, lk = lane >> 4;
  const double r0v = __shfl(x[rr], (q << 4) | lm), r1v = __shfl(x[rr], ((q + 1) << 4) | lm);
  const double a = readlane_d(x[rr], (q << 4) | P), b = readlane_d(x[rr], (q << 4) | (P + 1));
  const double c = readlane_d(x[rr], ((q + 1) << 4) | P), dd = readlane_d(x[rr], ((q + 1) << 4) | (P + 1));
  const double det = fma(a, dd, -(b * c));
  const double r0 = __builtin_amdgcn_rcp(det), e = fma(-det, r0, 1.0), t = fma(e, e, e);
  const double u0 = lm == P ? 1.0 : lm == P + 1 ? 0.0 : r0v, u1 = lm == P ? 0.0 : lm == P + 1 ? 1.0 : r1v;
  const double n0 = fma(dd, u0, -(b * u1)) * r0, n1 = fma(a, u1, -(c * u0)) * r0;
  const double rp0 = fma(n0, t, n0), rp1 = fma(n1, t, n1);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double f0 = row_bcast<P>(x[r]), f1 = row_bcast<P + 1>(x[r]);
    const double v = fma(-f1, rp1, fma(-f0, rp0, lm == P || lm == P + 1 ? 0.0 : x[r]));
    x[r] = r != rr ? v : lk == q ? rp0 : lk == q + 1 ? rp1 : v;
  }
  if (lm == P) pivots = a;
  if (lm == P + 1) pivots = det / a;
}

template <int... P>
__device__ __forceinline__ void gj_invert(double (&x)[4], double& pivots, int lane,
                                          std::integer_sequence<int, P...>) {
  auto one = [&](auto pc) {
    gj_step<2 * decltype(pc)::value>(x, pivots, lane);
    __builtin_amdgcn_sched_barrier(0);
  };
  (one(std::integral_constant<int, P>{}), ...);
}

// V and Y of one strip of columns whose assembled G_JC and K_JC blocks are in
// g and kj: block substitution with the node's block LU (lu(r, c): block (r,
// c) as an A operand), then K_JJ.
template <int NB, typename F>
__device__ __forceinline__ void strip_solve(const TreeNode& n, const double* slab, F lu, int lane, v4d (&g)[NB],
                                            v4d (&kj)[NB]) {
#pragma unroll
  for (int k = 1; k < NB; ++k)
#pragma unroll
    for (int j = 0; j < k; ++j) g[k] = mul_sub(lu(k, j), g[j], g[k]);
#pragma unroll
  for (int k = NB - 1; k >= 0; --k) {
#pragma unroll
    for (int j = k + 1; j < NB; ++j) g[k] = mul_sub(lu(k, j), g[j], g[k]);
    g[k] = mul_add(lu(k, k), g[k], v4d{0.0, 0.0, 0.0, 0.0});
  }
  const double* kjj = slab + n.kjj;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    v4d t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NB; ++j) t = mul_add(load_blk(kjj + (j * NB + k) * kTreeBlk, lane), g[j], t);
#pragma unroll
    for (int r = 0; r < 4; ++r) kj[k][r] = fma(-0.5, t[r], kj[k][r]);
  }
}

template <int NB>
__device__ __forceinline__ void strip_in_place(const TreeNode& n, double* slab, const double* sa, int strip, int lane) {
  v4d g[NB], kj[NB];
  double *v = slab + n.v + strip * NB * kTreeBlk, *y = slab + n.y + strip * NB * kTreeBlk;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    g[k] = load_blk(v + k * kTreeBlk, lane);
    kj[k] = load_blk(y + k * kTreeBlk, lane);
  }
  auto lu = [&](int r, int c) {
    v4d a;
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = sa[(r * kTreeB + (lane & 15)) * kTld + c * kTreeB + 4 * q + (lane >> 4)];
    return a;
  };
  strip_solve<NB>(n, slab, lu, lane, g, kj);
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    store_blk(v + k * kTreeBlk, g[k], lane);
    store_blk(y + k * kTreeBlk, kj[k], lane);
  }
}

// G_JJ in sa (row pitch kTld) by one wavefront: block LU without pivoting,
// 16 rows at a time; a pivot block is inverted in registers, the block
// products run on the matrix cores.  The pivots go to spiv.
__device__ __forceinline__ void front_factor(double* sa, double* spiv, int nb, int lane) {
  const int lm = lane & 15, lk = lane >> 4;
  for (int p = 0; p < nb; ++p) {
    const int p0 = p * kTreeB;
    double x[4], pivots = 1.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = sa[(p0 + 4 * r + lk) * kTld + p0 + lm];
    gj_invert(x, pivots, lane, std::make_integer_sequence<int, kTreeB / 2>{});
#pragma unroll
    for (int r = 0; r < 4; ++r) sa[(p0 + 4 * r + lk) * kTld + p0 + lm] = x[r];
    if (lane < kTreeB) spiv[p0 + lane] = pivots;
    // L_jp = A_jp D_p^-1, then A_ji -= L_jp A_pi along block row j
    for (int j = p + 1; j < nb; ++j) {
      v4d l = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 4; ++r)
        l = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[(j * kTreeB + lm) * kTld + p0 + 4 * r + lk], x[r], l, 0, 0, 0);
      wave_sync();
#pragma unroll
      for (int r = 0; r < 4; ++r) sa[(j * kTreeB + 4 * r + lk) * kTld + p0 + lm] = l[r];
      wave_sync();
      double la[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) la[r] = -sa[(j * kTreeB + lm) * kTld + p0 + 4 * r + lk];
      for (int i = p + 1; i < nb; ++i) {
        v4d acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = sa[(j * kTreeB + 4 * r + lk) * kTld + i * kTreeB + lm];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(la[r], sa[(p0 + 4 * r + lk) * kTld + i * kTreeB + lm], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) sa[(j * kTreeB + 4 * r + lk) * kTld + i * kTreeB + lm] = acc[r];
      }
    }
    wave_sync();
  }
}

// G_I. and K_I. of one strip and interface block row m, from the children and
// the strip's V and Y (all in the slab)
__device__ __forceinline__ void update_block(const TreeNode& n, const Kids& kd, double* slab, int strip, int m,
                                             int lane) {
  const int nb = n.nb;
  v4d ga = {0.0, 0.0, 0.0, 0.0}, ka = {0.0, 0.0, 0.0, 0.0};
  if (strip >= n.ib) add_ctrl<1>(kd, slab, nb + m, strip - n.ib, lane, &ga, &ka);
  else add_mapped<false, true, true>(kd, slab, nb + m, nb + strip, lane, ga, ka);
  const double *gt = slab + n.gijt + (long long)m * nb * kTreeBlk, *vm = slab + n.v + (long long)m * nb * kTreeBlk,
               *ym = slab + n.y + (long long)m * nb * kTreeBlk, *vs = slab + n.v + (long long)strip * nb * kTreeBlk,
               *ys = slab + n.y + (long long)strip * nb * kTreeBlk;
  for (int p = 0; p < nb; ++p) {
    const int o = p * kTreeBlk;
    const v4d v = load_blk(vs + o, lane), y = load_blk(ys + o, lane);
    ga = mul_sub(load_blk(gt + o, lane), v, ga);
    ka = mul_sub(load_blk(vm + o, lane), y, ka);
    ka = mul_sub(load_blk(ym + o, lane), v, ka);
  }
  const long long o = ((long long)strip * n.ib + m) * kTreeBlk;
  store_blk(slab + n.gu + o, ga, lane);
  store_blk(slab + n.ku + o, ka, lane);
}

// Pivot part of one node and scenario.  The children's maps go to LDS first
// (with them in global memory every child cost each block a chain of
// dependent loads: 41 against 26 us per level at 300 buses, 69 against 31 at
// 1354).  All wavefronts assemble G_JJ and K_JJ; then wavefront 0 factorises
// G_JJ while the others assemble G_IJ and the strips, whose V and Y follow:
// the interface strips only, or, for levels of narrow nodes (kAll), every
// strip and the updates for the parent too, which saves tree_cols_body's
// launch.  Bound by latency: at the upper levels one workgroup per scenario
// runs.
template <bool kMapLds, bool kAll>
__device__ __forceinline__ void tree_front_body(const DP& d, int node, int k) {
  extern __shared__ double fsm[];
  __shared__ double rmax[kTreeRows], spiv[kTreeRows];
  __shared__ TreeChild sch[kFrontKids];
  constexpr int kW = kTF / 64;
  double* sa = fsm;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lm = lane & 15, lk = lane >> 4;
  const TreeNode& n = d.tr.nodes[node];
  const int nb = n.nb, ib = n.ib, nbb = nb * nb, nstrip = kAll ? n.cs : ib;
  double* slab = d.tr.slab + (long long)k * d.tr.stride;
  const double* pool = d.tr.pool + (long long)k * d.tr.npool * kTreeBlk;
  // index data into LDS: the pool blocks (G_JJ, K_JJ, G_IJ, the strips of V,
  // those of Y), the children and their maps
  int* so = reinterpret_cast<int*>(fsm + kTreeRows * kTld);
  const int nfix = 2 * nbb + ib * nb, nst = nstrip * nb;
  for (int t = tid; t < nfix + 2 * nst; t += kTF)
    so[t] = d.tr.orig[n.oblk + (t < nfix + nst ? t : t - nst + n.cs * nb)];
  Kids kd = kids_global(d, n);
  if (kMapLds) {
    int* sm = so + nfix + 2 * nst;
    const int* src = reinterpret_cast<const int*>(kd.map);
    const int words = n.nchild * kd.len / 2;
    for (int t = tid; t < words; t += kTF) sm[t] = src[t];
    kd.map = reinterpret_cast<const short*>(sm);
    if (kAll) {
      short* ss = reinterpret_cast<short*>(sm + words);
      for (int t = tid; t < n.nchild * n.us; t += kTF) ss[t] = kd.smap[t];
      kd.smap = ss;
    }
    if (n.nchild <= kFrontKids) {
      if (tid < n.nchild) sch[tid] = kd.ch[tid];
      kd.ch = sch;
    }
  }
  __syncthreads();
  // G_JJ into LDS, K_JJ into the slab
  for (int b = wv; b < nbb; b += kW) {
    const int rb = b / nb, cb = b % nb;
    v4d g = pool_blk(pool, so[b], lane), kk = pool_blk(pool, so[nbb + b], lane);
    add_mapped<false, true, true>(kd, slab, rb, cb, lane, g, kk);
    store_blk(slab + n.kjj + b * kTreeBlk, kk, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = rb * kTreeB + 4 * r + lk, col = cb * kTreeB + lm;
      sa[row * kTld + col] = row >= n.s ? (row == col ? 1.0 : 0.0) : g[r];
    }
  }
  __syncthreads();
  if (wv == 0) {
    front_factor(sa, spiv, nb, lane);
  } else {
    // G_IJ^T, then G_J. and K_J. of the strips (in the places of V and Y)
    for (int b = wv - 1; b < ib * nb + nst; b += kW - 1) {
      v4d g = pool_blk(pool, so[2 * nbb + b], lane), kk = {0.0, 0.0, 0.0, 0.0};
      if (b < ib * nb) {
        const int ist = b / nb, kb = b % nb;
        add_mapped<true, true, false>(kd, slab, kb, nb + ist, lane, g, kk);
        store_blk(slab + n.gijt + b * kTreeBlk, g, lane);
      } else {
        const int q = b - ib * nb, ist = q / nb, kb = q % nb;
        kk = pool_blk(pool, so[nfix + nst + q], lane);
        if (kAll && ist >= ib) add_ctrl<1>(kd, slab, kb, ist - ib, lane, &g, &kk);
        else add_mapped<false, true, true>(kd, slab, kb, nb + ist, lane, g, kk);
        store_blk(slab + n.v + q * kTreeBlk, g, lane);
        store_blk(slab + n.y + q * kTreeBlk, kk, lane);
      }
    }
    // largest |entry| of every pivot row of G_x, for the pivot test
    if (wv == kW - 1 && lane < n.s) {
      const int row = d.tr.rows[n.row0 + lane];
      const double* gv = d.EV + (long long)k * d.n_ev + d.off_gx;
      double mx = 0.0;
      const int e1 = d.gx_ptr[row + 1];
      for (int e = d.gx_ptr[row]; e < e1; ++e) mx = fmax(mx, fabs(gv[e]));
      rmax[lane] = mx;
    }
  }
  __syncthreads();
  if (tid < n.s) {
    const double a = fabs(spiv[tid]);
    if (!(a > 0.0 && a >= 1e-10 * rmax[tid]) || !isfinite(a)) tree_status(d, RKKT_ERR_SINGULAR_GX, k);
  }
  for (int b = wv; b < nbb; b += kW) {
    const int r0 = b / nb * kTreeB, c0 = b % nb * kTreeB;
    double* o = slab + n.lu + b * kTreeBlk;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[64 * r + lane] = sa[(r0 + lm) * kTld + c0 + 4 * r + lk];
  }
  for (int st = wv; st < nstrip; st += kW) {
    switch (nb) {
      case 1: strip_in_place<1>(n, slab, sa, st, lane); break;
      case 2: strip_in_place<2>(n, slab, sa, st, lane); break;
      case 3: strip_in_place<3>(n, slab, sa, st, lane); break;
      default: strip_in_place<4>(n, slab, sa, st, lane); break;
    }
  }
  if (kAll) {
    __syncthreads();
    for (int t = wv; t < n.cs * ib; t += kW) update_block(n, kd, slab, t / ib, t % ib, lane);
  }
}

// --------------------------------------------------------- column strips
// One strip of a node and scenario by one wavefront, all in registers: V and
// Y of a control strip (an interface strip's are there already), then the
// strip's columns of the updated G_I. and K_I. that the parent reads.
template <int NB>
__device__ __forceinline__ void tree_strip(const DP& d, const TreeNode& n, double* slab, const double* pool,
                                           int strip, int lane) {
  v4d g[NB], kj[NB];
  const Kids kd = kids_global(d, n);
  const bool ctrl = strip >= n.ib;
  if (ctrl) {
    const int v0 = n.oblk + 2 * NB * NB + n.ib * NB + strip * NB;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      g[k] = pool_blk(pool, d.tr.orig[v0 + k], lane);
      kj[k] = pool_blk(pool, d.tr.orig[v0 + n.cs * NB + k], lane);
    }
    add_ctrl<NB>(kd, slab, 0, strip - n.ib, lane, g, kj);
    const double* lu = slab + n.lu;
    strip_solve<NB>(
        n, slab, [&](int r, int c) { return load_blk(lu + (r * NB + c) * kTreeBlk, lane); }, lane, g, kj);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      store_blk(slab + n.v + (strip * NB + k) * kTreeBlk, g[k], lane);
      store_blk(slab + n.y + (strip * NB + k) * kTreeBlk, kj[k], lane);
    }
  } else {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      g[k] = load_blk(slab + n.v + (strip * NB + k) * kTreeBlk, lane);
      kj[k] = load_blk(slab + n.y + (strip * NB + k) * kTreeBlk, lane);
    }
  }
  for (int m = 0; m < n.ib; ++m) {
    v4d ga = {0.0, 0.0, 0.0, 0.0}, ka = {0.0, 0.0, 0.0, 0.0}, bg[NB], bv[NB], by[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const long long at = (long long)(m * NB + k) * kTreeBlk;
      bg[k] = load_blk(slab + n.gijt + at, lane);
      bv[k] = load_blk(slab + n.v + at, lane);
      by[k] = load_blk(slab + n.y + at, lane);
    }
    if (ctrl) add_ctrl<1>(kd, slab, NB + m, strip - n.ib, lane, &ga, &ka);
    else add_mapped<false, true, true>(kd, slab, NB + m, NB + strip, lane, ga, ka);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      ga = mul_sub(bg[k], g[k], ga);
      ka = mul_sub(bv[k], kj[k], ka);
      ka = mul_sub(by[k], g[k], ka);
    }
    const long long o = ((long long)strip * n.ib + m) * kTreeBlk;
    store_blk(slab + n.gu + o, ga, lane);
    store_blk(slab + n.ku + o, ka, lane);
  }
}

__device__ __forceinline__ void tree_cols_body(const DP& d, int job, int k) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TreeNode& n = d.tr.nodes[d.tr.jobs[2 * job]];
  const int strip = d.tr.jobs[2 * job + 1] + wv;
  if (strip >= n.cs) return;
  double* slab = d.tr.slab + (long long)k * d.tr.stride;
  const double* pool = d.tr.pool + (long long)k * d.tr.npool * kTreeBlk;
  switch (n.nb) {
    case 1: tree_strip<1>(d, n, slab, pool, strip, lane); break;
    case 2: tree_strip<2>(d, n, slab, pool, strip, lane); break;
    case 3: tree_strip<3>(d, n, slab, pool, strip, lane); break;
    default: tree_strip<4>(d, n, slab, pool, strip, lane); break;
  }
}

// ------------------------------------------- product over control columns
// part_p[a][b] = -sum over the part's (node, scenario) units of
// V_a^T Y_b + Y_a^T V_b, one wavefront per (pair of groups of T strips, part);
// every operand block is read straight from the slab in the matrix
// instruction's own layout, one step of four rows ahead of its use, strips
// that a node does not hold from a block of zeros.  Bound by the matrix cores
// once the operands come from L2 (64 x 64 outputs per wavefront: 8 flops per
// byte; the probe of independent FP64 matrix instructions reaches 49 TFLOP/s):
// 9241 buses x 16 scenarios 95 GFLOP (79 without what fills up strips and groups)
// in 2.25 ms, 42 TFLOP/s; without the loads ahead and with every part on every
// die 4.68 ms.
template <int T>
struct ProdUnit {
  const double* slab;
  int va[T], ya[T], vb[T], yb[T], steps;
};
template <int T>
struct ProdRegs {
  double va[T], ya[T], vb[T], yb[T];
};

template <int T>
__device__ __forceinline__ void prod_load(ProdRegs<T>& x, const ProdUnit<T>& u, int st, int lane) {
  const double* p = u.slab + 64 * st;
#pragma unroll
  for (int i = 0; i < T; ++i) {
    x.va[i] = (p + u.va[i])[lane];
    x.ya[i] = (p + u.ya[i])[lane];
    x.vb[i] = (p + u.vb[i])[lane];
    x.yb[i] = (p + u.yb[i])[lane];
  }
}

template <int T>
__device__ __forceinline__ void prod_mul(const ProdRegs<T>& x, v4d (&acc)[T][T]) {
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) {
      acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.va[i], x.yb[j], acc[i][j], 0, 0, 0);
      acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.ya[i], x.vb[j], acc[i][j], 0, 0, 0);
    }
}

template <int T>
__device__ __forceinline__ void tree_product_body(const DP& d, int bx, int part) {
  const int lane = threadIdx.x & 63, q = bx * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (q >= d.tr.npair || d.tr.pair_g[2 * q] < 0) return;
  const int a = d.tr.pair_g[2 * q], b = d.tr.pair_g[2 * q + 1];
  v4d acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  // the part's units: a range of scenarios, and of the pair's nodes
  const int len = d.tr.pair_ptr[q + 1] - d.tr.pair_ptr[q], sp = d.tr.sparts, np = d.tr.parts / sp;
  const int ps = part % sp, pn = part / sp;
  const int s0 = (int)((long long)d.N * ps / sp), ns = (int)((long long)d.N * (ps + 1) / sp) - s0;
  const int l0 = d.tr.pair_ptr[q] + len * pn / np, l1 = d.tr.pair_ptr[q] + len * (pn + 1) / np;
  const int units = (l1 - l0) * ns;
  const int zero = (int)d.tr.zero;
  auto unit = [&](int u) {
    ProdUnit<T> r;
    const int li = u / ns, node = d.tr.pair_nodes[l0 + li];
    const TreeNode& n = d.tr.nodes[node];
    const int ga = d.tr.gstrip[node * d.tr.ngroup + a], gb = d.tr.gstrip[node * d.tr.ngroup + b];
    const int bs = n.nb * kTreeBlk, v0 = (int)n.v + n.ib * bs, y0 = (int)n.y + n.ib * bs;
    r.slab = d.tr.slab + (s0 + u - li * ns) * d.tr.stride;
    r.steps = 4 * n.nb;
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int ma = ga >> 16, mb = gb >> 16;
      const int ka = ((ga & 0xffff) + __popc(ma & ((1 << i) - 1))) * bs;
      const int kb = ((gb & 0xffff) + __popc(mb & ((1 << i) - 1))) * bs;
      r.va[i] = ma >> i & 1 ? v0 + ka : zero;
      r.ya[i] = ma >> i & 1 ? y0 + ka : zero;
      r.vb[i] = mb >> i & 1 ? v0 + kb : zero;
      r.yb[i] = mb >> i & 1 ? y0 + kb : zero;
    }
    return r;
  };
  if (units > 0) {
    ProdRegs<T> x, z;
    ProdUnit<T> cur = unit(0);
    prod_load<T>(x, cur, 0, lane);
    for (int u = 0; u < units; ++u) {
      const ProdUnit<T> nxt = unit(u + 1 < units ? u + 1 : u);
      for (int st = 0; st < cur.steps; st += 2) {
        prod_load<T>(z, cur, st + 1, lane);
        prod_mul<T>(x, acc);
        if (st + 2 < cur.steps) prod_load<T>(x, cur, st + 2, lane);
        else prod_load<T>(x, nxt, 0, lane);
        prod_mul<T>(z, acc);
      }
      cur = nxt;
    }
  }
  const int lm = lane & 15, lk = lane >> 4, ld = d.tr.ngroup * T * kTreeB;
  double* o = d.tr.part + (long long)part * ld * ld;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = (a * T + i) * kTreeB + 4 * r + lk, col = (b * T + j) * kTreeB + lm;
        if (col <= row) o[(long long)row * ld + col] = -acc[i][j][r];
      }
}

// K_hat (user order, both triangles) from the parts, in part order, with
// Sigma_u and delta_w on the diagonal.  One thread per entry of 16 x 16 tiles.
__device__ __forceinline__ void tree_sum_body(const DP& d, int bx, int by, const double* su, double dw, double* khat) {
  if (bx > by) return;
  const int row = by * kTreeB + (threadIdx.x >> 4), col = bx * kTreeB + (threadIdx.x & 15);
  if (row >= d.nu || col > row) return;
  const int ld = d.tr.ngroup * d.tr.T * kTreeB;
  const double* src = d.tr.part + (long long)row * ld + col;
  const long long pp = (long long)ld * ld;
  double acc = 0.0;
  for (int p = 0; p < d.tr.parts; p += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p + u < d.tr.parts ? src[(p + u) * pp] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  const int a = d.tr.uord[row], b = d.tr.uord[col];
  if (a == b) acc += su[a] + dw;
  if (!isfinite(acc)) atomicCAS(d.status, 0, RKKT_ERR_NONFINITE);
  khat[(long long)a * d.nu + b] = acc;
  khat[(long long)b * d.nu + a] = acc;
}

// K_hat += sum over scenarios of K_uu, one thread per entry of its lower triangle
__device__ __forceinline__ void tree_kuu_body(const DP& d, int bx, double* khat) {
  const int t = bx * kTT + threadIdx.x;
  if (t >= d.tr.nkuu) return;
  const int a = d.tr.kuu[3 * t], b = d.tr.kuu[3 * t + 1], e = d.tr.kuu[3 * t + 2];
  double acc = 0.0;
  for (int k = 0; k < d.N; k += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = k + u < d.N ? d.K[(long long)(k + u) * d.nnz_k + e] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  acc += khat[(long long)a * d.nu + b];
  if (!isfinite(acc)) atomicCAS(d.status, 0, RKKT_ERR_NONFINITE);
  khat[(long long)a * d.nu + b] = acc;
  khat[(long long)b * d.nu + a] = acc;
}

// ------------------------------------------------------------------ step
// The right-hand side is one more column b of the fronts: with
// V_b = G_JJ^-1 r3_J and Y_b = r1_J - K_JJ V_b / 2 a node updates
//     r3_I <- r3_I - G_IJ V_b,  r1_I <- r1_I - V_I^T Y_b - Y_I^T V_b
// on the way up, and the reduced right-hand side takes
// -(V_U^T Y_b + Y_U^T V_b) of all nodes.  On the way down
//     x_J = -(V_b + V_I x_I + V_U p_u),
//     y_J = -G_JJ^-T (Y_b + K_JJ x_J / 2 + Y_I x_I + Y_U p_u + G_IJ^T y_I),
// so a step is one sweep up and one down; the products with the control
// columns need no order and run over the whole chip.
constexpr int kTS = 64 * kTreeNB * kTreeStepNodes;  // threads of the sweeps

// value summed over the lanes of a row of 16, in every lane
__device__ __forceinline__ double sum16(double v) {
  v += __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, false);  // row_ror:8
  v += __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, false);
  v += __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, false);
  v += __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, false);
  return v;
}
// value summed over the four rows of 16 lanes
__device__ __forceinline__ double sum_rows(double v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}
// acc + sum over the block's rows of blk[row][lane%16] v[row], this lane's share
__device__ __forceinline__ double dot_rows(const v4d& blk, const double* v, int lk, double acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc = fma(blk[r], v[4 * r + lk], acc);
  return acc;
}
// acc[r] + blk[row 4 r + lane/16][lane%16] x, x the lane's column value
__device__ __forceinline__ void dot_cols(const v4d& blk, double x, v4d& acc) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] = fma(blk[r], x, acc[r]);
}
// row 4 r + lane/16 of a reduced acc (sum16 of every acc[r]) to out, 16 rows
__device__ __forceinline__ void put_rows(const v4d& acc, double* out, int lane) {
  const int lm = lane & 15, lk = lane >> 4;
  double v = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double t = sum16(acc[r]);
    if (lm == r) v = t;
  }
  if (lm < 4) out[4 * lm + lk] = v;
}

// rhat1 = r1x + H_x^T w and r3 in internal order, -H_u^T w into rpart, with
// w = Sigma_s r4 - r2 formed per use
__device__ __forceinline__ void tree_resid_body(const DP& d, int bx, int k, const double* r1x, const double* r2,
                                                const double* r3, const double* r4, const double* ss) {
  const int v = bx * kTT + threadIdx.x, nx = d.nx;
  if (v >= d.nz) return;
  const double* hv = d.EV + (long long)k * d.n_ev + d.off_h;
  const double *ssk = ss + (long long)k * d.m, *r2k = r2 + (long long)k * d.m, *r4k = r4 + (long long)k * d.m;
  const int pi = v < nx ? d.perm[v] : 0;
  double acc = v < nx ? r1x[(long long)k * nx + pi] : 0.0;
  const int j1 = d.ht_ptr[v + 1];
  for (int j = d.ht_ptr[v]; j < j1; j += 4) {
    double hj[4], wj[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int jj = min(j + u, j1 - 1), r = d.ht_row[jj];
      hj[u] = hv[d.ht_pos[jj]];
      wj[u] = ssk[r] * r4k[r] - r2k[r];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j + u < j1) acc = fma(hj[u], wj[u], acc);
  }
  if (v < nx) {
    d.rhat1[(long long)k * nx + v] = acc;
    d.qbuf[(long long)k * nx + v] = r3[(long long)k * nx + pi];
  } else {
    d.rpart[(long long)k * d.nu + v - nx] = -acc;
  }
}

// A node's block substitutions by one wavefront on a vector v of 64 in LDS,
// with the node's block LU in registers: v <- G_JJ^-1 v.
template <int NB>
__device__ __forceinline__ void pivot_solve(const v4d (&lu)[kTreeNB * kTreeNB], double* v, int lane) {
  const int lm = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int p = 1; p < NB; ++p) {
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < p; ++j) acc = dot_rows(lu[p * NB + j], v + j * kTreeB, lk, acc);
    acc = sum_rows(acc);
    if (lk == 0) v[p * kTreeB + lm] -= acc;
    wave_sync();
  }
#pragma unroll
  for (int p = NB - 1; p >= 0; --p) {
    if (p + 1 < NB) {
      double acc = 0.0;
#pragma unroll
      for (int j = p + 1; j < NB; ++j) acc = dot_rows(lu[p * NB + j], v + j * kTreeB, lk, acc);
      acc = sum_rows(acc);
      if (lk == 0) v[p * kTreeB + lm] -= acc;
      wave_sync();
    }
    const double acc = sum_rows(dot_rows(lu[p * NB + p], v + p * kTreeB, lk, 0.0));
    wave_sync();
    if (lk == 0) v[p * kTreeB + lm] = acc;
    wave_sync();
  }
}

// v <- G_JJ^-T v; s: 16 doubles of LDS
template <int NB>
__device__ __forceinline__ void pivot_solve_t(const v4d (&lu)[kTreeNB * kTreeNB], double* v, double* s, int lane) {
  const int lm = lane & 15;
#pragma unroll
  for (int p = 0; p < NB; ++p) {
    if (p > 0) {
      v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < p; ++j) dot_cols(lu[j * NB + p], -v[j * kTreeB + lm], acc);
      put_rows(acc, s, lane);
      wave_sync();
      if (lane < kTreeB) v[p * kTreeB + lane] += s[lane];
      wave_sync();
    }
    v4d z = {0.0, 0.0, 0.0, 0.0};
    dot_cols(lu[p * NB + p], v[p * kTreeB + lm], z);
    wave_sync();
    put_rows(z, v + p * kTreeB, lane);
    wave_sync();
  }
#pragma unroll
  for (int p = NB - 2; p >= 0; --p) {
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = p + 1; j < NB; ++j) dot_cols(lu[j * NB + p], -v[j * kTreeB + lm], acc);
    put_rows(acc, s, lane);
    wave_sync();
    if (lane < kTreeB) v[p * kTreeB + lane] += s[lane];
    wave_sync();
  }
}

__device__ __forceinline__ void load_lu(v4d (&lu)[kTreeNB * kTreeNB], const double* p, int nbb, int lane) {
#pragma unroll
  for (int q = 0; q < kTreeNB * kTreeNB; ++q)
    if (q < nbb) lu[q] = load_blk(p + q * kTreeBlk, lane);
}

// a value that every lane holds, in scalar registers: addresses built on it
// take no vector registers
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni(long long v) {
  return (long long)(unsigned)uni((int)v) | (long long)uni((int)(v >> 32)) << 32;
}

// The three blocks of every pivot block row j in a node's interface strip m:
// G_IJ^T, V, Y in blk[3 j ..] (past the last one the last again, without a
// branch per load)
__device__ __forceinline__ void load_strip(v4d (&blk)[3 * kTreeNB], const double* slab, const TreeNode& n,
                                           int m, int nb, int lane) {
#pragma unroll
  for (int j = 0; j < kTreeNB; ++j) {
    const long long at = (long long)(m * nb + min(j, nb - 1)) * kTreeBlk;
    blk[3 * j] = load_blk(slab + uni(n.gijt) + at, lane);
    blk[3 * j + 1] = load_blk(slab + uni(n.v) + at, lane);
    blk[3 * j + 2] = load_blk(slab + uni(n.y) + at, lane);
  }
}

// A workgroup takes kTreeStepNodes nodes at a time, kTreeNB wavefronts each,
// or one node with all its wavefronts where a level has a workgroup per node
// or one node is left.
struct SweepTurn {
  bool solo, act, own;  // one node; this wavefront has work; its group owns the block rows
  int node, cnt, me;    // place in the level; wavefronts of the node, this one among them
};
__device__ __forceinline__ SweepTurn sweep_turn(int qq, int q1, int step, int wv) {
  SweepTurn t;
  const int grp = wv / kTreeNB;
  t.solo = step == 1 || q1 - qq < 2;
  t.act = t.solo || qq + grp < q1;
  t.own = t.solo ? grp == 0 : t.act;
  t.node = t.solo ? qq : min(qq + grp, q1 - 1);
  t.cnt = t.solo ? kTreeNB * kTreeStepNodes : kTreeNB;
  t.me = t.solo ? wv : wv % kTreeNB;
  return t;
}

// Sweep up over the levels [l0, l1), workgroup bx of gx: right-hand sides by
// block rows, V_b by the first wavefront (its LU loads issued first), Y_b by
// block rows, the interface strips dealt to the wavefronts, the first one last:
// the others load their first strip and add up its children's parts while V_b
// is solved.  gx > 1 for one level only.  Bound by
// the latency of each step of the chain: with a strip's loads in its loop, one
// pivot block after the other, one child after the other, and half the
// wavefronts idle in levels of one node, a level took 12.8 us at 1354 buses (11
// now).  K_JJ is loaded behind the solve: the LU blocks' registers are free then.
__device__ __forceinline__ void tree_up_body(const DP& d, int bx, int gx, int k, int l0, int l1) {
  __shared__ double s3[kTreeStepNodes][kTreeRows], s1[kTreeStepNodes][kTreeRows];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lm = lane & 15, lk = lane >> 4, p = wv % kTreeNB;
  const double* slab = d.tr.slab + (long long)k * d.tr.stride;
  double* vec = d.tr.vec + (long long)k * d.tr.vstride;
  for (int l = l0; l < l1; ++l) {
    const int q0 = uni(d.tr.lev_ptr[l]);
    const int q1 = uni(d.tr.lev_ptr[l + 1]);
    const int step = gx > 1 && gx >= q1 - q0 ? 1 : kTreeStepNodes;
    for (int qq = q0 + bx * step; qq < q1; qq += gx * step) {
      const SweepTurn tn = sweep_turn(qq, q1, step, wv);
      const TreeNode& n = d.tr.nodes[uni(d.tr.lev_nodes[tn.node])];
      double *b3 = s3[tn.solo ? 0 : wv / kTreeNB], *b1 = s1[tn.solo ? 0 : wv / kTreeNB];
      const int nb = uni(n.nb), ib = uni(n.ib), nchild = uni(n.nchild);
      const bool row = tn.own && p < nb, pivot = tn.own && p == 0;
      const int m0 = tn.me == 0 ? tn.cnt - 1 : tn.me - 1;
      v4d lu[kTreeNB * kTreeNB], kr[kTreeNB];
      if (pivot) load_lu(lu, slab + uni(n.lu), nb * nb, lane);
      double* nv = vec + n.vec;
      // the children's parts of r3 and r1 in row r of the node
      double c3, c1;
      // (kChildren of them at a time: index loads, then value loads, in flight together)
      constexpr int kChildren = 4;
      auto children = [&](int r) {
        c3 = c1 = 0.0;
        for (int a0 = 0; a0 < nchild; a0 += kChildren) {
          int ci[kChildren], at[kChildren], ld[kChildren];
#pragma unroll
          for (int u = 0; u < kChildren; ++u) {
            const int a = min(a0 + u, nchild - 1);
            const TreeChild& ch = d.tr.children[n.child0 + a];
            ci[u] = d.tr.rmap[n.rmap0 + a * kTreeB * (nb + ib) + r];
            at[u] = ch.vec + 2 * kTreeB * ch.nb;
            ld[u] = kTreeB * ch.ib;
          }
          double v3[kChildren], v1[kChildren];
#pragma unroll
          for (int u = 0; u < kChildren; ++u) {
            v3[u] = vec[at[u] + max(ci[u], 0)];
            v1[u] = vec[at[u] + ld[u] + max(ci[u], 0)];
          }
#pragma unroll
          for (int u = 0; u < kChildren; ++u)
            if (a0 + u < nchild && ci[u] >= 0) {
              c3 += v3[u];
              c1 += v1[u];
            }
        }
      };
      if (row && lane < kTreeB) {
        const int r = p * kTreeB + lane;
        double a3 = 0.0, a1 = 0.0;
        if (r < n.s) {
          const long long at = (long long)k * d.nx + d.tr.rows[n.row0 + r];
          a3 = d.qbuf[at];
          a1 = d.rhat1[at];
        }
        children(r);
        b3[r] = a3 + c3;
        b1[r] = a1 + c1;
      }
      __syncthreads();
      if (pivot) {
        switch (nb) {
          case 1: pivot_solve<1>(lu, b3, lane); break;
          case 2: pivot_solve<2>(lu, b3, lane); break;
          case 3: pivot_solve<3>(lu, b3, lane); break;
          default: pivot_solve<4>(lu, b3, lane); break;
        }
        if (lane < nb * kTreeB) nv[lane] = b3[lane];
      } else if (tn.act && m0 < ib) {
        children((nb + m0) * kTreeB + lm);
      }
      // block rows of Y_b: by the second group where it has no node of its own
      const bool yrow = tn.solo ? !tn.own && p < nb : row;
      if (yrow)
#pragma unroll
        for (int j = 0; j < kTreeNB; ++j)
          if (j < nb) kr[j] = load_blk(slab + uni(n.kjj) + (j * nb + p) * kTreeBlk, lane);
      __syncthreads();
      if (yrow) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < kTreeNB; ++j)
          if (j < nb) acc = dot_rows(kr[j], b3 + j * kTreeB, lk, acc);
        acc = sum_rows(acc);
        if (lk == 0) {
          const double y = fma(-0.5, acc, b1[p * kTreeB + lm]);
          b1[p * kTreeB + lm] = y;
          nv[nb * kTreeB + p * kTreeB + lm] = y;
        }
      }
      __syncthreads();
      if (tn.act)
        for (int m = m0; m < ib; m += tn.cnt) {
          v4d blk[3 * kTreeNB];
          load_strip(blk, slab, n, m, nb, lane);
          if (pivot || m != m0) children((nb + m) * kTreeB + lm);
          double a3 = 0.0, a1 = 0.0;
#pragma unroll
          for (int j = 0; j < kTreeNB; ++j)
            if (j < nb) {
              a3 = dot_rows(blk[3 * j], b3 + j * kTreeB, lk, a3);
              a1 = dot_rows(blk[3 * j + 1], b1 + j * kTreeB, lk, a1);
              a1 = dot_rows(blk[3 * j + 2], b3 + j * kTreeB, lk, a1);
            }
          a3 = c3 - sum_rows(a3);
          a1 = c1 - sum_rows(a1);
          if (lk == 0) {
            double* o = nv + 2 * kTreeB * nb + m * kTreeB + lm;
            o[0] = a3;
            o[kTreeB * ib] = a1;
          }
        }
      __syncthreads();
    }
  }
}

// rpart of one control strip: the nodes that hold it, dealt to the wavefronts
__device__ __forceinline__ void tree_rhs_u_body(const DP& d, int z, int k) {
  __shared__ double red[4][kTreeB];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lm = lane & 15, lk = lane >> 4;
  const double* slab = d.tr.slab + (long long)k * d.tr.stride;
  const double* vec = d.tr.vec + (long long)k * d.tr.vstride;
  double acc = 0.0;
  const int e1 = d.tr.sn_ptr[z + 1];
  for (int e = d.tr.sn_ptr[z] + wv; e < e1; e += 4) {
    const TreeNode& n = d.tr.nodes[d.tr.sn[2 * e]];
    const int nb = n.nb;
    const long long at = (long long)(n.ib + d.tr.sn[2 * e + 1]) * nb * kTreeBlk;
    const double *vb = vec + n.vec, *yb = vb + nb * kTreeB;
    for (int p = 0; p < nb; ++p) {
      acc = dot_rows(load_blk(slab + n.v + at + p * kTreeBlk, lane), yb + p * kTreeB, lk, acc);
      acc = dot_rows(load_blk(slab + n.y + at + p * kTreeBlk, lane), vb + p * kTreeB, lk, acc);
    }
  }
  acc = sum_rows(acc);
  if (lk == 0) red[wv][lm] = acc;
  __syncthreads();
  const int p = z * kTreeB + threadIdx.x;
  if (threadIdx.x < kTreeB && p < d.nu) {
    const int t = threadIdx.x;
    d.rpart[(long long)k * d.nu + d.tr.uord[p]] += (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
  }
}

// V_U p_u and Y_U p_u of kTreeCJob control strips of a node
template <int NB>
__device__ __forceinline__ void rec_u(const DP& d, const TreeNode& n, int c0, int job, int k, const double* pu,
                                      double (*red)[2][kTreeRows], int lane, int wv) {
  const double* slab = d.tr.slab + (long long)k * d.tr.stride;
  const int lm = lane & 15;
  v4d av[NB], ay[NB];
#pragma unroll
  for (int p = 0; p < NB; ++p) av[p] = ay[p] = v4d{0.0, 0.0, 0.0, 0.0};
  const int c1 = min(n.us, c0 + kTreeCJob);
  for (int c = c0 + wv; c < c1; c += 4) {
    const int z = d.tr.strips[n.strip0 + c] * kTreeB + lm;
    const double x = z < d.nu ? pu[d.tr.uord[z]] : 0.0;
    const long long at = (long long)(n.ib + c) * NB * kTreeBlk;
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      dot_cols(load_blk(slab + n.v + at + p * kTreeBlk, lane), x, av[p]);
      dot_cols(load_blk(slab + n.y + at + p * kTreeBlk, lane), x, ay[p]);
    }
  }
#pragma unroll
  for (int p = 0; p < NB; ++p) {
    put_rows(av[p], &red[wv][0][p * kTreeB], lane);
    put_rows(ay[p], &red[wv][1][p * kTreeB], lane);
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 2 * NB * kTreeB) {
    const int h = t / (NB * kTreeB), r = t % (NB * kTreeB);
    d.tr.upart[(((long long)k * d.tr.ncjob + job) * 2 + h) * kTreeRows + r] =
        (red[0][h][r] + red[1][h][r]) + (red[2][h][r] + red[3][h][r]);
  }
}

__device__ __forceinline__ void tree_rec_u_body(const DP& d, int job, int k, const double* pu) {
  __shared__ double red[4][2][kTreeRows];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const TreeNode n = d.tr.nodes[d.tr.cjobs[2 * job]];
  const int c0 = d.tr.cjobs[2 * job + 1];
  switch (n.nb) {
    case 1: rec_u<1>(d, n, c0, job, k, pu, red, lane, wv); break;
    case 2: rec_u<2>(d, n, c0, job, k, pu, red, lane, wv); break;
    case 3: rec_u<3>(d, n, c0, job, k, pu, red, lane, wv); break;
    default: rec_u<4>(d, n, c0, job, k, pu, red, lane, wv); break;
  }
}

// Sweep down over the levels l1 - 1 .. l0, workgroups and wavefronts as in the
// sweep up: x_J and the right-hand side of y_J by block rows, y_J by the
// node's first wavefront.  Every load that does not wait for the node's own
// x_J is issued before the first barrier, the interface strips kStripsDown at a
// time; with a node to itself the second group of wavefronts takes every other
// strip.
constexpr int kStripsDown = 4;
__device__ __forceinline__ void tree_down_body(const DP& d, int bx, int gx, int k, int l0, int l1, double* px,
                                               double* py) {
  __shared__ double sx[kTreeStepNodes][kTreeRows], st[kTreeStepNodes][kTreeRows + kTreeB];
  __shared__ double sr[kTreeStepNodes * kTreeNB][2 * kTreeB];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lm = lane & 15, grp = wv / kTreeNB, p = wv % kTreeNB;
  const double* slab = d.tr.slab + (long long)k * d.tr.stride;
  const double* vec = d.tr.vec + (long long)k * d.tr.vstride;
  double* xk = d.tr.x + (long long)k * d.nx;
  double* yk = d.tr.y + (long long)k * d.nx;
  double* red = sr[wv];
  for (int l = l1 - 1; l >= l0; --l) {
    const int q0 = uni(d.tr.lev_ptr[l]), q1 = uni(d.tr.lev_ptr[l + 1]);
    const int step = gx > 1 && gx >= q1 - q0 ? 1 : kTreeStepNodes;
    for (int qq = q0 + bx * step; qq < q1; qq += gx * step) {
      const SweepTurn tn = sweep_turn(qq, q1, step, wv);
      const TreeNode& n = d.tr.nodes[uni(d.tr.lev_nodes[tn.node])];
      double *xs = sx[tn.solo ? 0 : grp], *ts = st[tn.solo ? 0 : grp];
      const int nb = uni(n.nb), ib = uni(n.ib);
      const bool row = tn.own && p < nb, pivot = tn.own && p == 0;
      v4d lu[kTreeNB * kTreeNB], kr[kTreeNB], t = {0.0, 0.0, 0.0, 0.0};
      double base = 0.0, bx0 = 0.0;
      int at = -1;
      if (row) {
#pragma unroll
        for (int j = 0; j < kTreeNB; ++j)
          if (j < nb) kr[j] = load_blk(slab + uni(n.kjj) + (p * nb + j) * kTreeBlk, lane);
        if (lane < kTreeB) {
          const double* up = d.tr.upart + ((long long)k * d.tr.ncjob + n.cjob0) * 2 * kTreeRows + p * kTreeB + lane;
          bx0 = vec[n.vec + p * kTreeB + lane];
          base = vec[n.vec + nb * kTreeB + p * kTreeB + lane];
          const int nc = n.ncjob;
          for (int c0 = 0; c0 < nc; c0 += 4) {
            double ux[4], uy[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              ux[u] = up[min(c0 + u, nc - 1) * 2 * kTreeRows];
              uy[u] = up[(min(c0 + u, nc - 1) * 2 + 1) * kTreeRows];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (c0 + u < nc) {
                bx0 += ux[u];
                base += uy[u];
              }
          }
          at = p * kTreeB + lane < n.s ? d.tr.rows[n.row0 + p * kTreeB + lane] : -1;
        }
      }
      if (tn.act && p < nb) {
        v4d acc = {0.0, 0.0, 0.0, 0.0};
        const int ms = tn.solo ? kTreeStepNodes : 1;
        for (int mb = tn.solo ? grp : 0; mb < ib; mb += kStripsDown * ms) {
          int r[kStripsDown];
          double x[kStripsDown], y[kStripsDown];
#pragma unroll
          for (int u = 0; u < kStripsDown; ++u)
            if (mb + u * ms < ib) {
              r[u] = d.tr.rows[n.row0 + n.s + min((mb + u * ms) * kTreeB + lm, n.i - 1)];
              const long long o = (long long)((mb + u * ms) * nb + p) * kTreeBlk;
              lu[3 * u] = load_blk(slab + uni(n.v) + o, lane);
              lu[3 * u + 1] = load_blk(slab + uni(n.y) + o, lane);
              lu[3 * u + 2] = load_blk(slab + uni(n.gijt) + o, lane);
            }
#pragma unroll
          for (int u = 0; u < kStripsDown; ++u)
            if (mb + u * ms < ib) {
              x[u] = xk[r[u]];
              y[u] = yk[r[u]];
            }
#pragma unroll
          for (int u = 0; u < kStripsDown; ++u)
            if (mb + u * ms < ib) {
              const bool in = (mb + u * ms) * kTreeB + lm < n.i;
              dot_cols(lu[3 * u], in ? x[u] : 0.0, acc);
              dot_cols(lu[3 * u + 1], in ? x[u] : 0.0, t);
              dot_cols(lu[3 * u + 2], in ? y[u] : 0.0, t);
            }
        }
        if (pivot) load_lu(lu, slab + uni(n.lu), nb * nb, lane);
        put_rows(acc, red, lane);
        if (!row) put_rows(t, red + kTreeB, lane);
      }
      if (tn.solo) __syncthreads();
      const double* red2 = sr[(wv + kTreeNB) % (kTreeStepNodes * kTreeNB)];  // the second group's, with solo
      if (row) {
        wave_sync();
        if (lane < kTreeB) {
          const double x = at >= 0 ? -(bx0 + red[lane] + (tn.solo ? red2[lane] : 0.0)) : 0.0;
          if (tn.solo) base += red2[kTreeB + lane];
          xs[p * kTreeB + lane] = x;
          if (at >= 0) {
            xk[at] = x;
            px[(long long)k * d.nx + d.perm[at]] = x;
          }
        }
      }
      __syncthreads();
      if (row) {
#pragma unroll
        for (int j = 0; j < kTreeNB; ++j)
          if (j < nb) dot_cols(kr[j], 0.5 * xs[j * kTreeB + lm], t);
        put_rows(t, red, lane);
        wave_sync();
        if (lane < kTreeB) ts[p * kTreeB + lane] = base + red[lane];
      }
      __syncthreads();
      if (pivot) {
        switch (nb) {
          case 1: pivot_solve_t<1>(lu, ts, ts + kTreeRows, lane); break;
          case 2: pivot_solve_t<2>(lu, ts, ts + kTreeRows, lane); break;
          case 3: pivot_solve_t<3>(lu, ts, ts + kTreeRows, lane); break;
          default: pivot_solve_t<4>(lu, ts, ts + kTreeRows, lane); break;
        }
        if (lane < n.s) {
          const int r = d.tr.rows[n.row0 + lane];
          const double v = -ts[lane];
          yk[r] = v;
          py[(long long)k * d.nx + d.perm[r]] = v;
        }
      }
      __syncthreads();
    }
  }
}

// p_s = -(r4 + H p_d), p_z = Sigma_s (H p_d + r4) - r2
__device__ __forceinline__ void tree_hp_body(const DP& d, int bx, int k, const double* r2, const double* r4,
                                             const double* ss, const double* pu, double* ps, double* pz) {
  const int r = bx * kTT + threadIdx.x;
  if (r >= d.m) return;
  const double* hv = d.EV + (long long)k * d.n_ev + d.off_h;
  const double* xk = d.tr.x + (long long)k * d.nx;
  double hp = 0.0;
  const int e1 = d.h_ptr[r + 1];
  for (int e = d.h_ptr[r]; e < e1; e += 4) {
    double h[4], x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ee = min(e + u, e1 - 1), c = d.h_col[ee];
      h[u] = hv[ee];
      x[u] = c < d.nx ? xk[c] : pu[c - d.nx];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e + u < e1) hp = fma(h[u], x[u], hp);
  }
  const long long at = (long long)k * d.m + r;
  ps[at] = -(r4[at] + hp);
  pz[at] = ss[at] * (hp + r4[at]) - r2[at];
}

__global__ __launch_bounds__(kTT) void k_tree_orig(DP d) { tree_orig_body(d, blockIdx.x, blockIdx.y); }
template <bool kMapLds, bool kAll>
__global__ __launch_bounds__(kTF) void k_tree_front(DP d, int first) {
  tree_front_body<kMapLds, kAll>(d, d.tr.lev_nodes[first + blockIdx.x], blockIdx.y);
}
__global__ __launch_bounds__(kTT) void k_tree_cols(DP d, int first) { tree_cols_body(d, first + blockIdx.x, blockIdx.y); }
template <int T>
__global__ __launch_bounds__(kTT, 2) void k_tree_product(DP d) {
  tree_product_body<T>(d, blockIdx.x / d.tr.parts, blockIdx.x % d.tr.parts);
}
__global__ __launch_bounds__(kTT) void k_tree_sum(DP d, const double* su, double dw, double* khat) {
  tree_sum_body(d, blockIdx.x, blockIdx.y, su, dw, khat);
}
__global__ __launch_bounds__(kTT) void k_tree_kuu(DP d, double* khat) { tree_kuu_body(d, blockIdx.x, khat); }
__global__ __launch_bounds__(kTT) void k_tree_resid(DP d, const double* r1x, const double* r2, const double* r3,
                                                    const double* r4, const double* ss) {
  tree_resid_body(d, blockIdx.x, blockIdx.y, r1x, r2, r3, r4, ss);
}
__global__ __launch_bounds__(kTS) void k_tree_up(DP d, int l0, int l1) {
  tree_up_body(d, blockIdx.x, gridDim.x, blockIdx.y, l0, l1);
}
__global__ __launch_bounds__(kTT) void k_tree_rhs_u(DP d) { tree_rhs_u_body(d, blockIdx.x, blockIdx.y); }
__global__ __launch_bounds__(kTT) void k_tree_rec_u(DP d, const double* pu) {
  tree_rec_u_body(d, blockIdx.x, blockIdx.y, pu);
}
__global__ __launch_bounds__(kTS) void k_tree_down(DP d, int l0, int l1, double* px, double* py) {
  tree_down_body(d, blockIdx.x, gridDim.x, blockIdx.y, l0, l1, px, py);
}
__global__ __launch_bounds__(kTT) void k_tree_hp(DP d, const double* r2, const double* r4, const double* ss,
                                                 const double* pu, double* ps, double* pz) {
  tree_hp_body(d, blockIdx.x, blockIdx.y, r2, r4, ss, pu, ps, pz);
}

#define RKKT_MULTI_ARGS \
  const DP* __restrict__ dps, const rkkt_iteration* __restrict__ its, const MultiBlk* __restrict__ blk
#define RKKT_MULTI_PROLOGUE                  \
  const MultiBlk mb = blk[blockIdx.x];       \
  const DP& d = dps[mb.inst];                \
  const rkkt_iteration& it = its[mb.inst];   \
  (void)it;

__global__ __launch_bounds__(kTT) void k_tree_orig_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_orig_body(d, mb.bx, mb.by);
}
template <bool kMapLds>
__global__ __launch_bounds__(kTF) void k_tree_front_m(RKKT_MULTI_ARGS, int level) {
  RKKT_MULTI_PROLOGUE
  tree_front_body<kMapLds, false>(d, d.tr.lev_nodes[d.tr.lev_ptr[level] + mb.bx], mb.by);
}
__global__ __launch_bounds__(kTT) void k_tree_cols_m(RKKT_MULTI_ARGS, int level) {
  RKKT_MULTI_PROLOGUE
  tree_cols_body(d, d.tr.job_ptr[level] + mb.bx, mb.by);
}
template <int T>
__global__ __launch_bounds__(kTT, 1) void k_tree_product_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_product_body<T>(d, mb.bx, mb.by);
}
__global__ __launch_bounds__(kTT) void k_tree_sum_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_sum_body(d, mb.bx, mb.by, it.sigma_u, it.delta_w, it.khat);
}
__global__ __launch_bounds__(kTT) void k_tree_kuu_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_kuu_body(d, mb.bx, it.khat);
}

__global__ __launch_bounds__(kTT) void k_tree_resid_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_resid_body(d, mb.bx, mb.by, it.r1x, it.r2, it.r3, it.r4, it.sigma_s);
}
__global__ __launch_bounds__(kTS) void k_tree_up_m(RKKT_MULTI_ARGS, int l0, int l1) {
  RKKT_MULTI_PROLOGUE
  tree_up_body(d, mb.bx, mb.gx, mb.by, l1 ? l0 : d.tr.nwide, l1 ? l1 : d.tr.nlev);
}
__global__ __launch_bounds__(kTT) void k_tree_rhs_u_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_rhs_u_body(d, mb.bx, mb.by);
}
__global__ __launch_bounds__(kTT) void k_tree_rec_u_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_rec_u_body(d, mb.bx, mb.by, it.pu);
}
__global__ __launch_bounds__(kTS) void k_tree_down_m(RKKT_MULTI_ARGS, int l0, int l1) {
  RKKT_MULTI_PROLOGUE
  tree_down_body(d, mb.bx, mb.gx, mb.by, l1 ? l0 : d.tr.nwide, l1 ? l1 : d.tr.nlev, it.px, it.py);
}
__global__ __launch_bounds__(kTT) void k_tree_hp_m(RKKT_MULTI_ARGS) {
  RKKT_MULTI_PROLOGUE
  tree_hp_body(d, mb.bx, mb.by, it.r2, it.r4, it.sigma_s, it.pu, it.ps, it.pz);
}

unsigned cdiv(long long a, long long b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

void launch_tree_reduce(const DP& d, hipStream_t s) {
  const Tree& t = *d.tr.host;
  k_tree_orig<<<dim3(cdiv(t.npool, 4), d.N), kTT, 0, s>>>(d);
  const int nlev = (int)t.lev_ptr.size() - 1;
  for (int l = 0; l < nlev; ++l) {
    const dim3 grid(t.lev_ptr[l + 1] - t.lev_ptr[l], d.N);
    const size_t lds = front_lds(t, l);
    const int v = front_variant(t, l);
    if (v == 3) k_tree_front<true, true><<<grid, kTF, lds, s>>>(d, t.lev_ptr[l]);
    else if (v == 2) k_tree_front<false, true><<<grid, kTF, lds, s>>>(d, t.lev_ptr[l]);
    else if (v == 1) k_tree_front<true, false><<<grid, kTF, lds, s>>>(d, t.lev_ptr[l]);
    else k_tree_front<false, false><<<grid, kTF, lds, s>>>(d, t.lev_ptr[l]);
    if (v & 2) continue;
    const int nj = t.job_ptr[l + 1] - t.job_ptr[l];
    if (nj > 0) k_tree_cols<<<dim3(nj, d.N), kTT, 0, s>>>(d, t.job_ptr[l]);
  }
}

void launch_tree_product(const DP& d, hipStream_t s) {
  const unsigned grid = cdiv(d.tr.npair, 4) * d.tr.parts;
  if (d.tr.T == 4) k_tree_product<4><<<grid, kTT, 0, s>>>(d);
  else k_tree_product<2><<<grid, kTT, 0, s>>>(d);
}

void launch_tree_sum(const DP& d, const double* su, double dw, double* khat, hipStream_t s) {
  k_tree_sum<<<dim3(d.tr.nstrip, d.tr.nstrip), kTT, 0, s>>>(d, su, dw, khat);
  k_tree_kuu<<<cdiv(d.tr.nkuu, kTT), kTT, 0, s>>>(d, khat);
}

// workgroups per scenario of a level's part of a sweep: one per node while all of
// them run at once (their registers leave one to a CU)
static int wide_groups(const Tree& t, int l, int n_scen) {
  const int nodes = t.lev_ptr[l + 1] - t.lev_ptr[l];
  return (long long)nodes * n_scen <= 256 ? nodes : (int)cdiv(nodes, kTreeStepNodes);
}

void launch_tree_rhs(const DP& d, const double* r1x, const double* r2, const double* r3, const double* r4,
                     const double* ss, hipStream_t s) {
  const Tree& t = *d.tr.host;
  k_tree_resid<<<dim3(cdiv(d.nz, kTT), d.N), kTT, 0, s>>>(d, r1x, r2, r3, r4, ss);
  const int nw = tree_wide_levels(t);
  for (int l = 0; l < nw; ++l) k_tree_up<<<dim3(wide_groups(t, l, d.N), d.N), kTS, 0, s>>>(d, l, l + 1);
  if (nw < d.tr.nlev) k_tree_up<<<dim3(1, d.N), kTS, 0, s>>>(d, nw, d.tr.nlev);
  k_tree_rhs_u<<<dim3(d.tr.nstrip, d.N), kTT, 0, s>>>(d);
}

void launch_tree_recover(const DP& d, const double* r2, const double* r4, const double* ss, const double* pu,
                         double* px, double* ps, double* py, double* pz, hipStream_t s) {
  const Tree& t = *d.tr.host;
  if (d.tr.ncjob > 0) k_tree_rec_u<<<dim3(d.tr.ncjob, d.N), kTT, 0, s>>>(d, pu);
  const int nw = tree_wide_levels(t);
  if (nw < d.tr.nlev) k_tree_down<<<dim3(1, d.N), kTS, 0, s>>>(d, nw, d.tr.nlev, px, py);
  for (int l = nw - 1; l >= 0; --l) k_tree_down<<<dim3(wide_groups(t, l, d.N), d.N), kTS, 0, s>>>(d, l, l + 1, px, py);
  k_tree_hp<<<dim3(cdiv(d.m, kTT), d.N), kTT, 0, s>>>(d, r2, r4, ss, pu, ps, pz);
}

// jb of a sweep's launch: first level | level after the last << 16; 0: the levels
// that one workgroup per scenario takes, whichever they are in each instance (one
// launch: one per first level, one after the other, took 213 us up and 188 down
// for 16 grids)
void launches_tree(const DP& d, std::vector<Launch>& out) {
  const Tree& t = *d.tr.host;
  const int R = kStReduce * 4096;
  out.push_back(Launch{R, kKTreeOrig, 0, (int)cdiv(t.npool, 4), d.N, kTT, 0, 0});
  const int nlev = (int)t.lev_ptr.size() - 1;
  for (int l = 0; l < nlev; ++l) {
    // never fused: an instance fused at a level where another is not would
    // make two launches of the level, one after the other (16 grids 2.88
    // against 3.05 ms per pass)
    out.push_back(Launch{R + 1 + 2 * l, kKTreeFront, front_variant(t, l) & 1, t.lev_ptr[l + 1] - t.lev_ptr[l], d.N,
                         kTF, l, (long long)front_lds(t, l)});
    const int nj = t.job_ptr[l + 1] - t.job_ptr[l];
    if (nj > 0) out.push_back(Launch{R + 2 + 2 * l, kKTreeCols, 0, nj, d.N, kTT, l, 0});
  }
  out.push_back(Launch{kStStacked * 4096, kKTreeProduct, d.tr.T == 4 ? 1 : 0, (int)cdiv(d.tr.npair, 4), d.tr.parts,
                       kTT, 0, 0});
  out.push_back(Launch{kStSum * 4096, kKTreeSum, 0, d.tr.nstrip, d.tr.nstrip, kTT, 0, 0});
  out.push_back(Launch{kStSum * 4096 + 1, kKTreeKuu, 0, (int)cdiv(d.tr.nkuu, kTT), 1, kTT, 0, 0});
  const int nw = tree_wide_levels(t);
  const int H = kStStepRhs * 4096, B = kStRecover * 4096;
  out.push_back(Launch{H, kKTreeResid, 0, (int)cdiv(d.nz, kTT), d.N, kTT, 0, 0});
  out.push_back(Launch{B, kKTreeRecU, 0, d.tr.ncjob, d.N, kTT, 0, 0});
  for (int l = 0; l < nw; ++l) {
    out.push_back(Launch{H + 1 + l, kKTreeUp, 0, wide_groups(t, l, d.N), d.N, kTS, l | (l + 1) << 16, 0});
    out.push_back(Launch{B + 2047 - l, kKTreeDown, 0, wide_groups(t, l, d.N), d.N, kTS, l | (l + 1) << 16, 0});
  }
  if (nw < nlev) {
    out.push_back(Launch{H + 2048, kKTreeUp, 0, 1, d.N, kTS, 0, 0});
    out.push_back(Launch{B + 1, kKTreeDown, 0, 1, d.N, kTS, 0, 0});
  }
  out.push_back(Launch{H + 2049, kKTreeRhsU, 0, d.tr.nstrip, d.N, kTT, 0, 0});
  out.push_back(Launch{B + 2048, kKTreeHp, 0, (int)cdiv(d.m, kTT), d.N, kTT, 0, 0});
}

bool tree_fits(const Tree& t) {
  if (t.stride >= 1ll << 31) return false;
  for (size_t l = 0; l + 1 < t.lev_ptr.size(); ++l)
    if (front_lds(t, (int)l) > (size_t)kFrontLdsMax) return false;
  return true;
}

// The pivot kernel's dynamic LDS is what tree_fits admits, beside its static
// arrays (the children's records, row maxima and pivots).
hipError_t configure_tree_kernels() {
  hipError_t e = hipSuccess;
  for (const void* fn : {(const void*)k_tree_front<true, true>, (const void*)k_tree_front<false, true>,
                         (const void*)k_tree_front<true, false>, (const void*)k_tree_front<false, false>,
                         (const void*)k_tree_front_m<true>, (const void*)k_tree_front_m<false>})
    if (e == hipSuccess) e = raise_lds(fn, kFrontLdsMax);
  return e;
}

hipError_t multi_tree(const Launch& l, unsigned nblk, long long lds, const DP* dps, const rkkt_iteration* its, const MultiBlk* blk,
                      hipStream_t s, bool prepare, bool* handled) {
  *handled = l.kernel >= kKTreeOrig && l.kernel <= kKTreeKuu;
  if (!*handled || prepare) return hipSuccess;
  switch (l.kernel) {
    case kKTreeOrig: k_tree_orig_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    case kKTreeFront:
      if (l.variant == 1) k_tree_front_m<true><<<nblk, kTF, (size_t)lds, s>>>(dps, its, blk, l.jb);
      else k_tree_front_m<false><<<nblk, kTF, (size_t)lds, s>>>(dps, its, blk, l.jb);
      break;
    case kKTreeCols: k_tree_cols_m<<<nblk, kTT, 0, s>>>(dps, its, blk, l.jb); break;
    case kKTreeProduct:
      if (l.variant) k_tree_product_m<4><<<nblk, kTT, 0, s>>>(dps, its, blk);
      else k_tree_product_m<2><<<nblk, kTT, 0, s>>>(dps, its, blk);
      break;
    case kKTreeResid: k_tree_resid_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    case kKTreeUp: k_tree_up_m<<<nblk, kTS, 0, s>>>(dps, its, blk, l.jb & 0xffff, l.jb >> 16); break;
    case kKTreeRhsU: k_tree_rhs_u_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    case kKTreeRecU: k_tree_rec_u_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    case kKTreeDown: k_tree_down_m<<<nblk, kTS, 0, s>>>(dps, its, blk, l.jb & 0xffff, l.jb >> 16); break;
    case kKTreeHp: k_tree_hp_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    case kKTreeSum: k_tree_sum_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    default: k_tree_kuu_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
  }
  return hipSuccess;
}

}  // namespace rkkt
