// Host program: device bytes of a grid's handle on the elimination tree and with
// panels, and the rule between them.  stdin: buses, lines, generators, reference
// bus, scenarios, then the lines' ends and the generators' buses.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "symbolic.h"
#include "tree.h"

int main() {
  int nb, nl, ng, ref, N;
  if (scanf("%d %d %d %d %d", &nb, &nl, &ng, &ref, &N) != 5) return 1;
  std::vector<int> f(nl), t(nl), g(ng);
  for (int i = 0; i < nl; ++i)
    if (scanf("%d %d", &f[i], &t[i]) != 2) return 1;
  for (int& b : g)
    if (scanf("%d", &b) != 1) return 1;
  std::vector<double> one(std::max({nb, nl, ng}), 1.0);
  rkkt_network n{};
  n.n_bus = nb; n.n_line = nl; n.n_gen = ng; n.ref_bus = ref;
  n.line_from = f.data(); n.line_to = t.data(); n.gen_bus = g.data();
  n.r = n.x = n.b = n.rate = n.pmin = n.pmax = n.qmin = n.qmax = n.c2 = n.c1 = n.c0 = n.vmin = n.vmax = one.data();
  rkkt::Sym s;
  rkkt::Tree tree;
  if (!rkkt::build_symbolic(n, N, nullptr, s, true).empty() || !s.tree || !rkkt::build_tree(s, tree).empty()) return 1;
  const long long tb = rkkt::tree_bytes(s, tree), pb = rkkt::panel_bytes(s);
  long long most = 0;   // least free memory with which the tree is taken
  for (long long lo = 0, hi = 1ll << 50; lo < hi;) {
    const long long mid = lo + (hi - lo) / 2;
    if (rkkt::tree_affordable(tb, pb, mid)) hi = most = mid;
    else lo = mid + 1;
  }
  std::printf("%lld %lld %lld\n", tb, pb, most);
  return 0;
}
