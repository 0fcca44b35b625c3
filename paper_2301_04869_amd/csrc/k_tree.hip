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
// 105 GFLOP on 1.7 GB of fronts against 335 GB of panel traffic, 9.4 ms
// (fronts 4.3, product 4.8, sum 0.1) against 90.7.
#include "device.h"

namespace rkkt {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kTT = 256;  // threads of the tree kernels (4 wavefronts)
constexpr int kTld = kTreeRows + 1;

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
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
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

__device__ __forceinline__ v4d pool_blk(const DP& d, const double* pool, int slot, int lane) {
  const int b = d.tr.orig[slot];
  return b >= 0 ? load_blk(pool + (long long)b * kTreeBlk, lane) : v4d{0.0, 0.0, 0.0, 0.0};
}

// adds the children's updates to one block whose rows and columns are both
// interface-mapped: element (row, col) of the parent (padded places row0 +
// lane/16 + 4 r, col0 + lane%16); kK: K_IC, else G_IC; kT: the block holds
// the transpose of the element (row, col) -> child's (col, row)
template <bool kT>
__device__ __forceinline__ void add_mapped(const DP& d, const TreeNode& n, const double* slab, int row0, int col0,
                                           int lane, bool isk, v4d& acc) {
  const int lm = lane & 15, lk = lane >> 4;
  for (int a = 0; a < n.nchild; ++a) {
    const TreeChild ch = d.tr.children[n.child0 + a];
    const TreeNode& c = d.tr.nodes[ch.node];
    const short* rm = d.tr.rmap + ch.rmap0;
    const int cj = rm[col0 + lm];
    const double* src = slab + (isk ? c.ku : c.gu);
    const int pitch = c.ib * kTreeBlk;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ci = rm[row0 + 4 * r + lk];
      if (ci >= 0 && cj >= 0) {
        const int rr = kT ? cj : ci, cc = kT ? ci : cj;
        acc[r] += src[(cc >> 4) * pitch + rr * kTreeB + (cc & 15)];
      }
    }
  }
}

// ------------------------------------------------------------ pivot blocks
// One Gauss-Jordan step of the in-place inverse of a 16 x 16 block held as
// x[r] = element (4 r + lane/16, lane%16): pivot P.  Returns the pivot.
template <int P>
__device__ __forceinline__ double gj_step(double (&x)[4], int lane) {
  constexpr int q = P & 3, rr = P >> 2;
  const int lm = lane & 15, lk = lane >> 4;
  const double rowv = __shfl(x[rr], (q << 4) | lm);
  const double piv = readlane_d(x[rr], (q << 4) | P);
  const double inv = 1.0 / piv;
  const double rp = lm == P ? inv : rowv * inv;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double f = row_bcast<P>(x[r]);
    const double v = fma(-f, rp, lm == P ? 0.0 : x[r]);
    x[r] = (r == rr && lk == q) ? rp : v;
  }
  return piv;
}

template <int... P>
__device__ __forceinline__ void gj_invert(double (&x)[4], double& pivots, int lane,
                                          std::integer_sequence<int, P...>) {
  auto one = [&](auto pc) {
    constexpr int p = decltype(pc)::value;
    const double v = gj_step<p>(x, lane);
    if ((lane & 15) == p) pivots = v;
  };
  (one(std::integral_constant<int, P>{}), ...);
}

// V and Y of one strip of columns whose assembled G_JC and K_JC blocks are in
// g and kj: block substitution with the node's block LU, then K_JJ.
template <int NB>
__device__ __forceinline__ void strip_solve(const TreeNode& n, const double* slab, int lane, v4d (&g)[NB],
                                            v4d (&kj)[NB]) {
  const double* lu = slab + n.lu;
#pragma unroll
  for (int k = 1; k < NB; ++k)
#pragma unroll
    for (int j = 0; j < k; ++j) g[k] = mul_sub(load_blk(lu + (k * NB + j) * kTreeBlk, lane), g[j], g[k]);
#pragma unroll
  for (int k = NB - 1; k >= 0; --k) {
#pragma unroll
    for (int j = k + 1; j < NB; ++j) g[k] = mul_sub(load_blk(lu + (k * NB + j) * kTreeBlk, lane), g[j], g[k]);
    g[k] = mul_add(load_blk(lu + (k * NB + k) * kTreeBlk, lane), g[k], v4d{0.0, 0.0, 0.0, 0.0});
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
__device__ __forceinline__ void istrip_solve(const DP& d, const TreeNode& n, double* slab, const double* pool,
                                             int strip, int lane) {
  v4d g[NB], kj[NB];
  const int v0 = n.oblk + 2 * NB * NB + n.ib * NB + strip * NB;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    g[k] = pool_blk(d, pool, v0 + k, lane);
    kj[k] = pool_blk(d, pool, v0 + n.cs * NB + k, lane);
    add_mapped<false>(d, n, slab, k * kTreeB, (NB + strip) * kTreeB, lane, false, g[k]);
    add_mapped<false>(d, n, slab, k * kTreeB, (NB + strip) * kTreeB, lane, true, kj[k]);
  }
  strip_solve<NB>(n, slab, lane, g, kj);
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    store_blk(slab + n.v + (strip * NB + k) * kTreeBlk, g[k], lane);
    store_blk(slab + n.y + (strip * NB + k) * kTreeBlk, kj[k], lane);
  }
}

// Pivot part of one node and scenario: assembles G_JJ, K_JJ and G_IJ,
// factorises G_JJ by 16-row blocks without pivoting (pivot blocks inverted in
// registers by one wavefront, block products on the matrix cores), tests the
// pivots, and solves the interface strips.
__device__ __forceinline__ void tree_front_body(const DP& d, int node, int k) {
  __shared__ double sa[kTreeRows * kTld];
  __shared__ double rmax[kTreeRows];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int lm = lane & 15, lk = lane >> 4;
  const TreeNode n = d.tr.nodes[node];
  const int nb = n.nb;
  double* slab = d.tr.slab + (long long)k * d.tr.stride;
  const double* pool = d.tr.pool + (long long)k * d.tr.npool * kTreeBlk;
  // G_JJ into LDS, K_JJ and G_IJ^T into the slab
  for (int b = wv; b < nb * nb; b += 4) {
    const int rb = b / nb, cb = b % nb;
    v4d g = pool_blk(d, pool, n.oblk + b, lane), kk = pool_blk(d, pool, n.oblk + nb * nb + b, lane);
    add_mapped<false>(d, n, slab, rb * kTreeB, cb * kTreeB, lane, false, g);
    add_mapped<false>(d, n, slab, rb * kTreeB, cb * kTreeB, lane, true, kk);
    store_blk(slab + n.kjj + b * kTreeBlk, kk, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = rb * kTreeB + 4 * r + lk, col = cb * kTreeB + lm;
      sa[row * kTld + col] = row >= n.s ? (row == col ? 1.0 : 0.0) : g[r];
    }
  }
  for (int b = wv; b < n.ib * nb; b += 4) {
    const int ist = b / nb, kb = b % nb;
    v4d g = pool_blk(d, pool, n.oblk + 2 * nb * nb + b, lane);
    add_mapped<true>(d, n, slab, kb * kTreeB, (nb + ist) * kTreeB, lane, false, g);
    store_blk(slab + n.gijt + b * kTreeBlk, g, lane);
  }
  // largest |entry| of every pivot row of G_x, for the pivot test
  if (tid < n.s) {
    const int row = d.tr.rows[n.row0 + tid];
    const double* gv = d.EV + (long long)k * d.n_ev + d.off_gx;
    double mx = 0.0;
    const int e1 = d.gx_ptr[row + 1];
    for (int e = d.gx_ptr[row]; e < e1; ++e) mx = fmax(mx, fabs(gv[e]));
    rmax[tid] = mx;
  }
  __syncthreads();
  for (int p = 0; p < nb; ++p) {
    const int p0 = p * kTreeB;
    if (wv == 0) {
      double x[4], pivots = 1.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = sa[(p0 + 4 * r + lk) * kTld + p0 + lm];
      gj_invert(x, pivots, lane, std::make_integer_sequence<int, kTreeB>{});
#pragma unroll
      for (int r = 0; r < 4; ++r) sa[(p0 + 4 * r + lk) * kTld + p0 + lm] = x[r];
      if (lane < kTreeB && p0 + lane < n.s) {
        const double a = fabs(pivots);
        if (!(a > 0.0 && a >= 1e-10 * rmax[p0 + lane]) || !isfinite(pivots)) tree_status(d, RKKT_ERR_SINGULAR_GX, k);
      }
    }
    __syncthreads();
    // L_jp = A_jp D_p^-1
    for (int j = p + 1 + wv; j < nb; j += 4) {
      v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[(j * kTreeB + lm) * kTld + p0 + 4 * r + lk],
                                                   sa[(p0 + 4 * r + lk) * kTld + p0 + lm], acc, 0, 0, 0);
      wave_sync();
#pragma unroll
      for (int r = 0; r < 4; ++r) sa[(j * kTreeB + 4 * r + lk) * kTld + p0 + lm] = acc[r];
    }
    __syncthreads();
    // A_ij -= L_ip A_pj
    const int m = nb - 1 - p;
    for (int t = wv; t < m * m; t += 4) {
      const int i0 = (p + 1 + t / m) * kTreeB, j0 = (p + 1 + t % m) * kTreeB;
      v4d acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = sa[(i0 + 4 * r + lk) * kTld + j0 + lm];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-sa[(i0 + lm) * kTld + p0 + 4 * r + lk],
                                                   sa[(p0 + 4 * r + lk) * kTld + j0 + lm], acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sa[(i0 + 4 * r + lk) * kTld + j0 + lm] = acc[r];
    }
    __syncthreads();
  }
  for (int b = wv; b < nb * nb; b += 4) {
    const int r0 = b / nb * kTreeB, c0 = b % nb * kTreeB;
    double* o = slab + n.lu + b * kTreeBlk;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[64 * r + lane] = sa[(r0 + lm) * kTld + c0 + 4 * r + lk];
  }
  __syncthreads();
  for (int st = wv; st < n.ib; st += 4) {
    switch (nb) {
      case 1: istrip_solve<1>(d, n, slab, pool, st, lane); break;
      case 2: istrip_solve<2>(d, n, slab, pool, st, lane); break;
      case 3: istrip_solve<3>(d, n, slab, pool, st, lane); break;
      default: istrip_solve<4>(d, n, slab, pool, st, lane); break;
    }
  }
}

// --------------------------------------------------------- column strips
// One strip of a node and scenario by one wavefront, all in registers: V and
// Y of a control strip (an interface strip's are there already), then the
// strip's columns of the updated G_I. and K_I. that the parent reads.
template <int NB>
__device__ __forceinline__ void tree_strip(const DP& d, const TreeNode& n, double* slab, const double* pool,
                                           int strip, int lane) {
  const int lm = lane & 15, lk = lane >> 4;
  v4d g[NB], kj[NB];
  const bool ctrl = strip >= n.ib;
  if (ctrl) {
    const int v0 = n.oblk + 2 * NB * NB + n.ib * NB + strip * NB;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      g[k] = pool_blk(d, pool, v0 + k, lane);
      kj[k] = pool_blk(d, pool, v0 + n.cs * NB + k, lane);
    }
    for (int a = 0; a < n.nchild; ++a) {
      const TreeChild ch = d.tr.children[n.child0 + a];
      const int cst = d.tr.smap[ch.smap0 + strip - n.ib];
      if (cst < 0) continue;
      const TreeNode& c = d.tr.nodes[ch.node];
      const long long so = (long long)(c.ib + cst) * c.ib * kTreeBlk;
      const double *gu = slab + c.gu + so, *ku = slab + c.ku + so;
      const short* rm = d.tr.rmap + ch.rmap0;
#pragma unroll
      for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ci = rm[k * kTreeB + 4 * r + lk];
          if (ci >= 0) {
            g[k][r] += gu[ci * kTreeB + lm];
            kj[k][r] += ku[ci * kTreeB + lm];
          }
        }
    }
    strip_solve<NB>(n, slab, lane, g, kj);
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
    v4d ga = {0.0, 0.0, 0.0, 0.0}, ka = {0.0, 0.0, 0.0, 0.0};
    const int row0 = (NB + m) * kTreeB;
    if (ctrl) {
      for (int a = 0; a < n.nchild; ++a) {
        const TreeChild ch = d.tr.children[n.child0 + a];
        const int cst = d.tr.smap[ch.smap0 + strip - n.ib];
        if (cst < 0) continue;
        const TreeNode& c = d.tr.nodes[ch.node];
        const long long so = (long long)(c.ib + cst) * c.ib * kTreeBlk;
        const double *gu = slab + c.gu + so, *ku = slab + c.ku + so;
        const short* rm = d.tr.rmap + ch.rmap0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ci = rm[row0 + 4 * r + lk];
          if (ci >= 0) {
            ga[r] += gu[ci * kTreeB + lm];
            ka[r] += ku[ci * kTreeB + lm];
          }
        }
      }
    } else {
      add_mapped<false>(d, n, slab, row0, (NB + strip) * kTreeB, lane, false, ga);
      add_mapped<false>(d, n, slab, row0, (NB + strip) * kTreeB, lane, true, ka);
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const long long at = (long long)(m * NB + k) * kTreeBlk;
      ga = mul_sub(load_blk(slab + n.gijt + at, lane), g[k], ga);
      ka = mul_sub(load_blk(slab + n.v + at, lane), kj[k], ka);
      ka = mul_sub(load_blk(slab + n.y + at, lane), g[k], ka);
    }
    const long long o = ((long long)strip * n.ib + m) * kTreeBlk;
    store_blk(slab + n.gu + o, ga, lane);
    store_blk(slab + n.ku + o, ka, lane);
  }
}

__device__ __forceinline__ void tree_cols_body(const DP& d, int job, int k) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const TreeNode n = d.tr.nodes[d.tr.jobs[2 * job]];
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
// instruction's own layout.
template <int T>
__device__ __forceinline__ void tree_product_body(const DP& d, int bx, int part) {
  const int lane = threadIdx.x & 63, q = bx * 4 + (threadIdx.x >> 6);
  if (q >= d.tr.npair) return;
  const int a = d.tr.pair_g[2 * q], b = d.tr.pair_g[2 * q + 1];
  v4d acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  const int l0 = d.tr.pair_ptr[q];
  const long long units = (long long)(d.tr.pair_ptr[q + 1] - l0) * d.N;
  const long long u0 = units * part / d.tr.parts, u1 = units * (part + 1) / d.tr.parts;
  for (long long u = u0; u < u1;) {
    const int li = (int)(u / d.N);
    const int node = __builtin_amdgcn_readfirstlane(d.tr.pair_nodes[l0 + li]);
    const TreeNode& n = d.tr.nodes[node];
    const int nb = n.nb, ib = n.ib;
    const int ga = __builtin_amdgcn_readfirstlane(d.tr.gstrip[(long long)node * d.tr.ngroup + a]);
    const int gb = __builtin_amdgcn_readfirstlane(d.tr.gstrip[(long long)node * d.tr.ngroup + b]);
    const int ma = ga >> 16, mb = gb >> 16;
    long long oa[T], ob[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
      oa[i] = (long long)(ib + (ga & 0xffff) + __popc(ma & ((1 << i) - 1))) * nb * kTreeBlk;
      ob[i] = (long long)(ib + (gb & 0xffff) + __popc(mb & ((1 << i) - 1))) * nb * kTreeBlk;
    }
    const long long ue = min(u1, (long long)(li + 1) * d.N);
    const long long nv = n.v, ny = n.y;
    for (; u < ue; ++u) {
      const double* slab = d.tr.slab + (u - (long long)li * d.N) * d.tr.stride;
      const double *v = slab + nv, *y = slab + ny;
      for (int st = 0; st < 4 * nb; ++st) {
        const int o = 64 * st + lane;
        double va[T], ya[T], vb[T], yb[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
          va[i] = ma >> i & 1 ? v[oa[i] + o] : 0.0;
          ya[i] = ma >> i & 1 ? y[oa[i] + o] : 0.0;
          vb[i] = mb >> i & 1 ? v[ob[i] + o] : 0.0;
          yb[i] = mb >> i & 1 ? y[ob[i] + o] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[i], yb[j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ya[i], vb[j], acc[i][j], 0, 0, 0);
          }
      }
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

__global__ __launch_bounds__(kTT) void k_tree_orig(DP d) { tree_orig_body(d, blockIdx.x, blockIdx.y); }
__global__ __launch_bounds__(kTT) void k_tree_front(DP d, int first) {
  tree_front_body(d, d.tr.lev_nodes[first + blockIdx.x], blockIdx.y);
}
__global__ __launch_bounds__(kTT) void k_tree_cols(DP d, int first) { tree_cols_body(d, first + blockIdx.x, blockIdx.y); }
template <int T>
__global__ __launch_bounds__(kTT, 1) void k_tree_product(DP d) {
  tree_product_body<T>(d, blockIdx.x, blockIdx.y);
}
__global__ __launch_bounds__(kTT) void k_tree_sum(DP d, const double* su, double dw, double* khat) {
  tree_sum_body(d, blockIdx.x, blockIdx.y, su, dw, khat);
}
__global__ __launch_bounds__(kTT) void k_tree_kuu(DP d, double* khat) { tree_kuu_body(d, blockIdx.x, khat); }

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
__global__ __launch_bounds__(kTT) void k_tree_front_m(RKKT_MULTI_ARGS, int level) {
  RKKT_MULTI_PROLOGUE
  tree_front_body(d, d.tr.lev_nodes[d.tr.lev_ptr[level] + mb.bx], mb.by);
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

unsigned cdiv(long long a, long long b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

void launch_tree_reduce(const DP& d, hipStream_t s) {
  const Tree& t = *d.tr.host;
  k_tree_orig<<<dim3(cdiv(t.npool, 4), d.N), kTT, 0, s>>>(d);
  const int nlev = (int)t.lev_ptr.size() - 1;
  for (int l = 0; l < nlev; ++l) {
    k_tree_front<<<dim3(t.lev_ptr[l + 1] - t.lev_ptr[l], d.N), kTT, 0, s>>>(d, t.lev_ptr[l]);
    const int nj = t.job_ptr[l + 1] - t.job_ptr[l];
    if (nj > 0) k_tree_cols<<<dim3(nj, d.N), kTT, 0, s>>>(d, t.job_ptr[l]);
  }
}

void launch_tree_product(const DP& d, hipStream_t s) {
  const dim3 grid(cdiv(d.tr.npair, 4), d.tr.parts);
  if (d.tr.T == 4) k_tree_product<4><<<grid, kTT, 0, s>>>(d);
  else k_tree_product<2><<<grid, kTT, 0, s>>>(d);
}

void launch_tree_sum(const DP& d, const double* su, double dw, double* khat, hipStream_t s) {
  k_tree_sum<<<dim3(d.tr.nstrip, d.tr.nstrip), kTT, 0, s>>>(d, su, dw, khat);
  k_tree_kuu<<<cdiv(d.tr.nkuu, kTT), kTT, 0, s>>>(d, khat);
}

void launches_tree(const DP& d, std::vector<Launch>& out) {
  const Tree& t = *d.tr.host;
  const int R = kStReduce * 4096;
  out.push_back(Launch{R, kKTreeOrig, 0, (int)cdiv(t.npool, 4), d.N, kTT, 0, 0});
  const int nlev = (int)t.lev_ptr.size() - 1;
  for (int l = 0; l < nlev; ++l) {
    out.push_back(Launch{R + 1 + 2 * l, kKTreeFront, 0, t.lev_ptr[l + 1] - t.lev_ptr[l], d.N, kTT, l, 0});
    const int nj = t.job_ptr[l + 1] - t.job_ptr[l];
    if (nj > 0) out.push_back(Launch{R + 2 + 2 * l, kKTreeCols, 0, nj, d.N, kTT, l, 0});
  }
  out.push_back(Launch{kStStacked * 4096, kKTreeProduct, d.tr.T == 4 ? 1 : 0, (int)cdiv(d.tr.npair, 4), d.tr.parts,
                       kTT, 0, 0});
  out.push_back(Launch{kStSum * 4096, kKTreeSum, 0, d.tr.nstrip, d.tr.nstrip, kTT, 0, 0});
  out.push_back(Launch{kStSum * 4096 + 1, kKTreeKuu, 0, (int)cdiv(d.tr.nkuu, kTT), 1, kTT, 0, 0});
}

hipError_t multi_tree(const Launch& l, unsigned nblk, const DP* dps, const rkkt_iteration* its, const MultiBlk* blk,
                      hipStream_t s, bool prepare, bool* handled) {
  *handled = l.kernel >= kKTreeOrig && l.kernel <= kKTreeKuu;
  if (!*handled || prepare) return hipSuccess;
  switch (l.kernel) {
    case kKTreeOrig: k_tree_orig_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    case kKTreeFront: k_tree_front_m<<<nblk, kTT, 0, s>>>(dps, its, blk, l.jb); break;
    case kKTreeCols: k_tree_cols_m<<<nblk, kTT, 0, s>>>(dps, its, blk, l.jb); break;
    case kKTreeProduct:
      if (l.variant) k_tree_product_m<4><<<nblk, kTT, 0, s>>>(dps, its, blk);
      else k_tree_product_m<2><<<nblk, kTT, 0, s>>>(dps, its, blk);
      break;
    case kKTreeSum: k_tree_sum_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
    default: k_tree_kuu_m<<<nblk, kTT, 0, s>>>(dps, its, blk); break;
  }
  return hipSuccess;
}

}  // namespace rkkt
