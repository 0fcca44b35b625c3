// Host analysis of the elimination tree of dense fronts (tree.h).
#include "tree.h"

#include <algorithm>
#include <iterator>
#include <set>

#include "symbolic.h"

namespace rkkt {

namespace {

int blocks(int n) { return (n + kTreeB - 1) / kTreeB; }

// Elimination order of the rows of x for the tree: weighted minimum degree
// over buses (the rows of one bus, its angle and magnitude, stay together) on
// the union of the patterns of G_x and K_xx, since K_xx couples the
// neighbours of a generator bus, which G_x does not.  up[e] lists the later
// rows (places in the order) that row e's front holds, ascending.
void order_rows(const Sym& s, std::vector<int>& order, std::vector<std::vector<int>>& up) {
  const int nx = s.nx, nb = s.nb;
  std::vector<int> bus_of(nx, -1);
  std::vector<std::vector<int>> rows(nb);
  for (int b = 0; b < nb; ++b)
    for (int v : {s.th_src[b], s.v_src[b]})
      if (v >= 0) {
        rows[b].push_back(s.pinv[v]);
        bus_of[s.pinv[v]] = b;
      }
  std::vector<std::vector<int>> adj(nb);
  auto link = [&](int r, int c) {
    const int a = bus_of[r], b = bus_of[c];
    if (a != b) {
      adj[a].push_back(b);
      adj[b].push_back(a);
    }
  };
  for (int r = 0; r < nx; ++r) {
    for (int e = s.gx_ptr[r]; e < s.gx_ptr[r + 1]; ++e) link(r, s.gx_col[e]);
    for (int e = s.k_ptr[r]; e < s.k_usplit[r]; ++e) link(r, s.k_col[e]);
  }
  for (auto& a : adj) {
    std::sort(a.begin(), a.end());
    a.erase(std::unique(a.begin(), a.end()), a.end());
  }
  auto degree = [&](int b) {
    int w = 0;
    for (int c : adj[b]) w += (int)rows[c].size();
    return w;
  };
  std::vector<int> deg(nb, 0), first(nb, -1);
  std::set<std::pair<int, int>> pq;
  for (int b = 0; b < nb; ++b)
    if (!rows[b].empty()) pq.insert({deg[b] = degree(b), b});
  order.clear();
  std::vector<std::vector<int>> fill(nb);
  std::vector<int> merged, seq;
  while (!pq.empty()) {
    const int v = pq.begin()->second;
    pq.erase(pq.begin());
    seq.push_back(v);
    first[v] = (int)order.size();
    order.insert(order.end(), rows[v].begin(), rows[v].end());
    fill[v].swap(adj[v]);
    const std::vector<int>& nv = fill[v];
    for (int w : nv) {
      merged.clear();
      std::set_union(adj[w].begin(), adj[w].end(), nv.begin(), nv.end(), std::back_inserter(merged));
      adj[w].clear();
      for (int q : merged)
        if (q != v && q != w) adj[w].push_back(q);
    }
    for (int w : nv) {
      pq.erase({deg[w], w});
      pq.insert({deg[w] = degree(w), w});
    }
  }
  up.assign(nx, {});
  for (int v : seq) {
    std::vector<int> f;
    for (int w : fill[v])
      for (int a = 0; a < (int)rows[w].size(); ++a) f.push_back(first[w] + a);
    std::sort(f.begin(), f.end());
    for (int a = (int)rows[v].size() - 1; a >= 0; --a) {
      up[first[v] + a] = f;
      f.insert(f.begin(), first[v] + a);
    }
  }
}

// Joins every row with its elimination-tree children where that adds few
// explicit zeros.  `rows[p]` lists the rows of the node whose last row is p
// (empty when p was joined into an ancestor's node); front[p] is the number
// of interface rows of that node, which joining children does not change.
// A child of s rows and front f joined into a node of sp rows and front fp
// adds s (sp + fp - f) zeros; accepted while they stay below 3/10 of the
// joined node's panel (half for joined nodes of one block row, whose blocks
// are padded anyway).
void join_rows(const std::vector<int>& par, const std::vector<int>& front, std::vector<std::vector<int>>& rows) {
  const int n = (int)par.size();
  std::vector<std::vector<int>> kids(n);
  rows.assign(n, {});
  for (int i = 0; i < n; ++i) {
    rows[i].push_back(i);
    if (par[i] >= 0) kids[par[i]].push_back(i);
  }
  for (int p = 0; p < n; ++p) {
    std::vector<int> order = kids[p];
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return front[a] > front[b]; });
    std::vector<int> left;
    for (int c : order) {
      const long long s = (long long)rows[c].size(), sp = (long long)rows[p].size();
      const long long zeros = s * (sp + front[p] - front[c]);
      const long long panel = (s + sp) * (s + sp + front[p]);
      const bool few = zeros == 0 || 10 * zeros <= 3 * panel || (s + sp <= kTreeB && 2 * zeros <= panel);
      if (s + sp <= kTreeRows && few) {
        rows[p].insert(rows[p].end(), rows[c].begin(), rows[c].end());
        rows[c].clear();
        left.insert(left.end(), kids[c].begin(), kids[c].end());
      } else {
        left.push_back(c);
      }
    }
    kids[p] = left;
    std::sort(rows[p].begin(), rows[p].end());
  }
}

}  // namespace

std::string build_tree(const Sym& s, Tree& t) {
  t = Tree();
  const int nx = s.nx, nu = s.nu;
  std::vector<int> order, at(nx);
  std::vector<std::vector<int>> up;
  order_rows(s, order, up);
  if ((int)order.size() != nx) return "internal: a row of x outside the elimination order";
  for (int e = 0; e < nx; ++e) at[order[e]] = e;
  std::vector<int> par(nx, -1), front(nx, 0);
  for (int e = 0; e < nx; ++e) {
    front[e] = (int)up[e].size();
    if (front[e] > 0) par[e] = up[e][0];
  }
  std::vector<std::vector<int>> rows;
  join_rows(par, front, rows);

  // node of every row; nodes in ascending order of their last row (children
  // before parents)
  std::vector<int> node_of(nx, -1), last;
  for (int p = 0; p < nx; ++p)
    if (!rows[p].empty()) {
      for (int r : rows[p]) node_of[r] = (int)last.size();
      last.push_back(p);
    }
  const int nn = (int)last.size();
  std::vector<int> parent(nn, -1);
  std::vector<std::vector<int>> kids(nn);
  for (int q = 0; q < nn; ++q)
    if (par[last[q]] >= 0) {
      parent[q] = node_of[par[last[q]]];
      kids[parent[q]].push_back(q);
    }
  // post-order from the roots, so that subtrees are contiguous
  std::vector<int> post, where(nn, -1);
  {
    std::vector<std::pair<int, size_t>> st;
    for (int r = 0; r < nn; ++r) {
      if (parent[r] >= 0) continue;
      st.push_back({r, 0});
      while (!st.empty()) {
        auto& top = st.back();
        if (top.second < kids[top.first].size()) {
          const int c = kids[top.first][top.second++];
          st.push_back({c, 0});
        } else {
          where[top.first] = (int)post.size();
          post.push_back(top.first);
          st.pop_back();
        }
      }
    }
  }

  // control columns of every node, renumbered as the walk meets them
  std::vector<std::vector<int>> own(nn);
  for (int r = 0; r < nx; ++r) {
    std::vector<int>& o = own[where[node_of[at[r]]]];
    for (int e = s.gu_ptr[r]; e < s.gu_ptr[r + 1]; ++e) o.push_back(s.gu_col[e]);
    for (int e = s.k_usplit[r]; e < s.k_ptr[r + 1]; ++e) o.push_back(s.k_col[e] - nx);
  }
  t.upos.assign(nu, -1);
  for (int q = 0; q < nn; ++q) {
    std::sort(own[q].begin(), own[q].end());
    for (int u : own[q])
      if (t.upos[u] < 0) {
        t.upos[u] = (int)t.uord.size();
        t.uord.push_back(u);
      }
  }
  for (int u = 0; u < nu; ++u)
    if (t.upos[u] < 0) {
      t.upos[u] = (int)t.uord.size();
      t.uord.push_back(u);
    }
  t.nstrip = blocks(nu);

  // nodes
  t.nodes.resize(nn);
  std::vector<std::vector<int>> strips(nn);
  std::vector<int> pos_in(nx, -1);  // place of a row (by its place in the order) among its node's pivot rows
  std::vector<int> erows;           // t.rows by place in the order
  for (int q = 0; q < nn; ++q) {
    const int p = last[post[q]];
    TreeNode& n = t.nodes[q];
    n.s = (int)rows[p].size();
    n.i = front[p];
    n.nb = blocks(n.s);
    n.ib = blocks(n.i);
    n.parent = parent[post[q]] >= 0 ? where[parent[post[q]]] : -1;
    n.row0 = (int)t.rows.size();
    for (int a = 0; a < n.s; ++a) pos_in[rows[p][a]] = a;
    erows.insert(erows.end(), rows[p].begin(), rows[p].end());
    erows.insert(erows.end(), up[p].begin(), up[p].end());
    for (size_t e = n.row0; e < erows.size(); ++e) t.rows.push_back(order[erows[e]]);
    n.child0 = (int)t.children.size();
    n.nchild = (int)kids[post[q]].size();
    n.level = 0;
    std::vector<char> hit(t.nstrip, 0);
    for (int u : own[q]) hit[t.upos[u] / kTreeB] = 1;
    for (int c0 : kids[post[q]]) {
      const int c = where[c0];
      t.children.push_back({c, 0, 0, t.nodes[c].ib, t.nodes[c].nb, t.nodes[c].vec, t.nodes[c].gu, t.nodes[c].ku, 0});
      n.level = std::max(n.level, t.nodes[c].level + 1);
      for (int z : strips[c]) hit[z] = 1;
    }
    for (int z = 0; z < t.nstrip; ++z)
      if (hit[z]) strips[q].push_back(z);
    n.us = (int)strips[q].size();
    n.cs = n.ib + n.us;
    n.strip0 = (int)t.strips.size();
    t.strips.insert(t.strips.end(), strips[q].begin(), strips[q].end());
    auto take = [&](long long nblk) {
      const long long o = t.stride;
      t.stride += nblk * kTreeBlk;
      return o;
    };
    n.lu = take((long long)n.nb * n.nb);
    n.kjj = take((long long)n.nb * n.nb);
    n.gijt = take((long long)n.ib * n.nb);
    n.v = take((long long)n.cs * n.nb);
    n.y = take((long long)n.cs * n.nb);
    n.gu = take((long long)n.cs * n.ib);
    n.ku = take((long long)n.cs * n.ib);
    n.vec = t.vstride;
    t.vstride += 2 * kTreeB * (n.nb + n.ib);
    n.cjob0 = (int)t.cjobs.size() / 2;
    for (int c = 0; c < n.us; c += kTreeCJob) {
      t.cjobs.push_back(q);
      t.cjobs.push_back(c);
    }
    n.ncjob = (int)t.cjobs.size() / 2 - n.cjob0;
    n.oblk = (int)t.orig.size();
    t.orig.resize(t.orig.size() + 2 * n.nb * n.nb + n.ib * n.nb + 2 * n.cs * n.nb, -1);
  }
  // place of row e of the order among a node's rows (pivot rows padded to whole blocks), -1 if absent
  auto place = [&](const TreeNode& n, int r) -> int {
    if (node_of[r] == node_of[erows[n.row0]]) return pos_in[r];
    const int* b = erows.data() + n.row0 + n.s;
    const int* e = b + n.i;
    const int* f = std::lower_bound(b, e, r);
    return f != e && *f == r ? n.nb * kTreeB + (int)(f - b) : -1;
  };
  for (int q = 0; q < nn; ++q) {
    TreeNode& n = t.nodes[q];
    n.rmap0 = (int)t.rmap.size();
    n.smap0 = (int)t.smap.size();
    for (int a = 0; a < n.nchild; ++a) {
      TreeChild& ch = t.children[n.child0 + a];
      const TreeNode& c = t.nodes[ch.node];
      ch.rmap0 = (int)t.rmap.size();
      t.rmap.resize(t.rmap.size() + kTreeB * (n.nb + n.ib), -1);
      for (int j = 0; j < c.i; ++j) {
        const int r = place(n, erows[c.row0 + c.s + j]);
        if (r < 0) return "internal: interface row of a front missing from its parent";
        t.rmap[ch.rmap0 + r] = (short)j;
        ch.blocks |= 1ull << std::min(63, r / kTreeB);
      }
      ch.smap0 = (int)t.smap.size();
      for (int z : strips[q]) {
        auto f = std::lower_bound(strips[ch.node].begin(), strips[ch.node].end(), z);
        t.smap.push_back(f != strips[ch.node].end() && *f == z ? (short)(f - strips[ch.node].begin()) : (short)-1);
      }
    }
  }

  // original entries: the node whose pivots eliminate them first
  struct Ent {
    int slot, at, src;
  };
  std::vector<Ent> ents;
  auto ustrip = [&](int q, int u) {
    return (int)(std::lower_bound(strips[q].begin(), strips[q].end(), t.upos[u] / kTreeB) - strips[q].begin());
  };
  bool ok = true;
  // block (row place, column place) of a pivot-row array with `nb` block rows, strips of columns
  auto put = [&](int slot, int row, int col, int src) { ents.push_back({slot, row % kTreeB * kTreeB + col % kTreeB, src}); };
  auto lower = [&](int r, int c) {  // post-order index of the node that owns entry (r, c)
    return std::min(where[node_of[r]], where[node_of[c]]);
  };
  for (int r = 0; r < nx; ++r) {
    const int er = at[r], qr = where[node_of[er]];
    for (int e = s.gx_ptr[r]; e < s.gx_ptr[r + 1]; ++e) {
      const int c = at[s.gx_col[e]], q = lower(er, c);
      const TreeNode& n = t.nodes[q];
      const int a = place(n, er), b = place(n, c), src = s.off_gx + e;
      if (a < 0 || b < 0) { ok = false; continue; }
      const int J = n.nb * kTreeB, nn2 = n.nb * n.nb;
      if (a < J && b < J) put(n.oblk + a / kTreeB * n.nb + b / kTreeB, a, b, src);
      else if (a < J) put(n.oblk + 2 * nn2 + n.ib * n.nb + (b - J) / kTreeB * n.nb + a / kTreeB, a, b - J, src);
      else put(n.oblk + 2 * nn2 + (a - J) / kTreeB * n.nb + b / kTreeB, b, a - J, src);
    }
    for (int e = s.k_ptr[r]; e < s.k_usplit[r]; ++e) {
      const int c = at[s.k_col[e]], q = lower(er, c);
      if (q != qr) continue;  // the mirrored entry is stored with its pivot row
      const TreeNode& n = t.nodes[q];
      const int a = place(n, er), b = place(n, c);
      if (a < 0 || b < 0) { ok = false; continue; }
      const int J = n.nb * kTreeB, nn2 = n.nb * n.nb;
      if (b < J) put(n.oblk + nn2 + a / kTreeB * n.nb + b / kTreeB, a, b, ~e);
      else put(n.oblk + 2 * nn2 + n.ib * n.nb + n.cs * n.nb + (b - J) / kTreeB * n.nb + a / kTreeB, a, b - J, ~e);
    }
    const TreeNode& n = t.nodes[qr];
    const int a = pos_in[er], v0 = n.oblk + 2 * n.nb * n.nb + n.ib * n.nb;
    for (int e = s.gu_ptr[r]; e < s.gu_ptr[r + 1]; ++e) {
      const int u = s.gu_col[e];
      put(v0 + (n.ib + ustrip(qr, u)) * n.nb + a / kTreeB, a, t.upos[u], s.off_gu + e);
    }
    for (int e = s.k_usplit[r]; e < s.k_ptr[r + 1]; ++e) {
      const int u = s.k_col[e] - nx;
      put(v0 + (n.cs + n.ib + ustrip(qr, u)) * n.nb + a / kTreeB, a, t.upos[u], ~e);
    }
  }
  if (!ok) return "internal: an entry of G_x or K lies outside the fronts";
  std::stable_sort(ents.begin(), ents.end(), [](const Ent& a, const Ent& b) { return a.slot < b.slot; });
  t.optr.push_back(0);
  for (size_t e = 0; e < ents.size();) {
    t.orig[ents[e].slot] = t.npool++;
    const int slot = ents[e].slot;
    for (; e < ents.size() && ents[e].slot == slot; ++e) {
      t.oent.push_back(ents[e].at);
      t.oent.push_back(ents[e].src);
    }
    t.optr.push_back((int)(t.oent.size() / 2));
  }

  // levels and strip jobs
  int nlev = 0;
  for (const TreeNode& n : t.nodes) nlev = std::max(nlev, n.level + 1);
  for (int l = 0; l < nlev; ++l) {
    t.lev_ptr.push_back((int)t.lev_nodes.size());
    t.job_ptr.push_back((int)t.jobs.size() / 2);
    t.lev_map.push_back(0);
    t.lev_cs.push_back(0);
    t.lev_ib.push_back(0);
    for (int q = 0; q < nn; ++q)
      if (t.nodes[q].level == l) {
        const TreeNode& n = t.nodes[q];
        t.lev_map[l] = std::max(t.lev_map[l], n.nchild * (kTreeB * (n.nb + n.ib) + n.us));
        t.lev_cs[l] = std::max(t.lev_cs[l], n.cs);
        t.lev_ib[l] = std::max(t.lev_ib[l], n.ib);
        t.lev_nodes.push_back(q);
        for (int c = 0; c < t.nodes[q].cs; c += 4) {
          t.jobs.push_back(q);
          t.jobs.push_back(c);
        }
      }
  }
  t.lev_ptr.push_back((int)t.lev_nodes.size());
  t.job_ptr.push_back((int)t.jobs.size() / 2);

  // nodes of every global strip
  {
    std::vector<std::vector<int>> of(t.nstrip);
    for (int q = 0; q < nn; ++q)
      for (int k = 0; k < (int)strips[q].size(); ++k) {
        of[strips[q][k]].push_back(q);
        of[strips[q][k]].push_back(k);
      }
    t.sn_ptr.push_back(0);
    for (auto& v : of) {
      t.sn.insert(t.sn.end(), v.begin(), v.end());
      t.sn_ptr.push_back((int)t.sn.size() / 2);
    }
  }

  // K_uu
  for (int r = nx; r < s.nz; ++r)
    for (int e = s.k_usplit[r]; e < s.k_ptr[r + 1]; ++e)
      if (s.k_col[e] <= r) {
        t.kuu.push_back(r - nx);
        t.kuu.push_back(s.k_col[e] - nx);
        t.kuu.push_back(e);
      }

  // product over the control columns: 64 x 64 outputs per wavefront (half the
  // operand traffic) from 100 strips, else 32 x 32 (four times the
  // wavefronts): at 64 strips x 8 scenarios 2170 against 2056 us per pass, at
  // 33 strips x 8 1104 against 1056
  t.T = t.nstrip >= 100 ? 4 : 2;
  t.ngroup = (t.nstrip + t.T - 1) / t.T;
  t.gstrip.assign((size_t)nn * t.ngroup, 0);
  std::vector<std::vector<int>> lists((size_t)t.ngroup * (t.ngroup + 1) / 2);
  for (int q = 0; q < nn; ++q) {
    std::vector<int> gs;
    for (int k = 0; k < (int)strips[q].size(); ++k) {
      const int g = strips[q][k] / t.T;
      int& w = t.gstrip[(size_t)q * t.ngroup + g];
      if (w == 0) {
        w = k;
        gs.push_back(g);
      }
      w |= 1 << (16 + strips[q][k] % t.T);
    }
    for (size_t a = 0; a < gs.size(); ++a)
      for (size_t b = 0; b <= a; ++b) lists[(size_t)gs[a] * (gs[a] + 1) / 2 + gs[b]].push_back(q);
  }
  t.pair_ptr.push_back(0);
  for (int a2 = 0; a2 < t.ngroup; a2 += 2)
    for (int b2 = 0; b2 <= a2; b2 += 2)
      for (int w = 0; w < 4; ++w) {
        const int a = a2 + w / 2, b = b2 + w % 2;
        const bool in = a < t.ngroup && b <= a;
        t.pair_g.push_back(in ? a : -1);
        t.pair_g.push_back(in ? b : -1);
        if (in) {
          const auto& l = lists[(size_t)a * (a + 1) / 2 + b];
          t.pair_nodes.insert(t.pair_nodes.end(), l.begin(), l.end());
        }
        t.pair_ptr.push_back((int)t.pair_nodes.size());
      }
  // parts of the contraction: about 8192 wavefronts, at most 32.  They split
  // the scenarios (by eights where there are as many: workgroups go to the
  // chip's eight dies in turn, so a part stays on one die, whose L2 holds its
  // scenarios' fronts), then the lists of nodes.
  const long long npair = (long long)t.pair_g.size() / 2;
  long long longest = 1;
  for (const auto& l : lists) longest = std::max(longest, (long long)l.size());
  const long long want = std::max(1LL, std::min(32LL, (8192 + npair - 1) / npair));
  t.sparts = (int)std::min<long long>(s.N, want);
  if (want >= 6 && s.N >= 8) t.sparts = std::min(s.N / 8, (int)(want + 4) / 8) * 8;
  t.parts = t.sparts * (int)std::min(longest, std::max(1LL, want / t.sparts));
  t.zero = t.stride;
  t.stride += kTreeNB * kTreeBlk;
  return "";
}

long long tree_bytes(const Sym& s, const Tree& t) {
  const long long ld = (long long)t.ngroup * t.T * kTreeB, ncjob = (long long)t.cjobs.size() / 2;
  return 8 * (s.N * (t.stride + (long long)t.npool * kTreeBlk + t.vstride + 2LL * s.nx + 2 * ncjob * kTreeRows) +
              t.parts * ld * ld);
}

long long panel_bytes(const Sym& s) {
  const long long ntile = (s.nu + s.col_tile - 1) / s.col_tile;
  return 8LL * s.N * (2LL * s.nx * (s.lds_reduce ? 1 : ntile * s.col_tile) + (long long)s.nu * s.nu +
                      (long long)s.f_col.size() + s.nx + s.m);
}

int tree_wide_levels(const Tree& t) {
  int l = 0;
  while (l + 1 < (int)t.lev_ptr.size() && t.lev_ptr[l + 1] - t.lev_ptr[l] > kTreeWide) ++l;
  return l;
}

}  // namespace rkkt
