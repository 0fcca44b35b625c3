// Elimination tree of dense fronts for the reduction on grids whose panels do
// not fit on chip (kernels in k_tree.hip).
//
// The filled LU pattern of G_x (internal order) is cut into nodes of at most
// kTreeRows pivot rows each, joined where the elimination tree allows it and
// little fill is added.  Every node is a dense front over its pivot rows J,
// its interface rows I (rows of ancestors that its subtree touches) and its
// control columns U (columns of u that its subtree touches).  Control columns
// are renumbered in the order in which a post-order walk meets them and kept
// in strips of 16, so a subtree's columns are a few whole strips and parent
// and child agree on what a strip holds.
#pragma once

#include <string>
#include <vector>

#include "layout.h"

namespace rkkt {

struct Sym;

constexpr int kTreeB = 16;                     // block side (one FP64 matrix instruction)
constexpr int kTreeNB = 4;                     // pivot block rows of a node, at most
constexpr int kTreeRows = kTreeB * kTreeNB;    // pivot rows of a node, at most
constexpr int kTreeBlk = kTreeB * kTreeB;      // doubles of a block
constexpr int kTreeCJob = 16;                  // control strips of a recovery job

// One node.  Blocks are 16 x 16, row-major and contiguous; nb pivot block
// rows, ib interface strips, us control strips, cs = ib + us strips in all.
// Offsets are doubles within a scenario's slab:
//   lu   [nb][nb]  block LU of G_JJ, every block transposed: (r, c) with
//                  r > c holds L_rc^T (unit block lower), r < c holds U_rc^T
//                  and r == c the transposed inverse of the pivot block
//   kjj  [nb][nb]  K_JJ
//   gijt [ib][nb]  G_IJ^T (row: pivot row, column: interface row)
//   v, y [cs][nb]  V = G_JJ^-1 G_JC and Y = K_JC - K_JJ V / 2
//   gu, ku [cs][ib]  updated G_IC and K_IC, read by the parent
struct TreeNode {
  int s, i, nb, ib, us, cs;
  int level, parent;
  int row0;        // rows[row0 ..]: internal row of every pivot row, then of every interface row
  int child0, nchild;
  int rmap0, smap0;  // maps of the first child (the others' follow)
  int strip0;      // strips[strip0 .. + us]: global strip of every control strip
  int vec;         // offset in the scenario's step vectors: V_b, Y_b (16 nb each), then the updates
                   // of r3 and r1 in the interface rows (16 ib each)
  int cjob0, ncjob;  // control-part jobs of the step's recovery
  int oblk;        // orig table: lu nb nb, kjj nb nb, gijt ib nb, v cs nb, y cs nb
  long long lu, kjj, gijt, v, y, gu, ku;
};

// A child as its parent sees it: rmap[rmap0 + r] is the child's interface
// index of the parent's padded row r (pivot block rows, then interface block
// rows) or -1; smap[smap0 + t] the child's control strip of the parent's
// control strip t or -1.  The children of a node have their maps one after the
// other.  blocks: bit b (63 for all beyond) set where a row of the
// parent's padded block row b is mapped.  ib, nb, vec, gu, ku: the child's own.
struct TreeChild {
  int node, rmap0, smap0;
  int ib, nb, vec;
  long long gu, ku;
  unsigned long long blocks;
};

struct Tree {
  std::vector<TreeNode> nodes;      // post-order
  std::vector<TreeChild> children;
  std::vector<int> rows, strips;
  std::vector<short> rmap, smap;
  long long stride = 0;             // doubles of a scenario's slab
  // original entries (G_x, G_u, K) as blocks: orig[t] is the pool block of a
  // node's block or -1; entries of pool block b are oent[2 optr[b] ..): the
  // place in the block and the source, >= 0 in EV, ~source in K
  std::vector<int> orig, optr, oent;
  int npool = 0;
  std::vector<int> lev_map;         // most shorts of row and strip maps of a node, per level
  std::vector<int> lev_cs, lev_ib;  // most strips and interface strips of a node, per level
  // nodes of every level; strip jobs of every level (node, first strip), four
  // strips each, interface strips first
  std::vector<int> lev_ptr, lev_nodes, job_ptr, jobs;
  // step: length of a scenario's vectors; recovery jobs (node, first control
  // strip), kTreeCJob strips each; nodes of every global strip with their
  // local strip, sn[2 sn_ptr[z] ..)
  int vstride = 0;
  std::vector<int> cjobs, sn_ptr, sn;
  // control columns: uord[p] = u of place p, upos the inverse; nstrip strips
  std::vector<int> uord, upos;
  int nstrip = 0;
  // K_uu entries of the lower triangle (user order): (row u, column u, K index)
  std::vector<int> kuu;
  // product over the control columns: groups of T strips; pair q = (ga, gb),
  // gb <= ga (four pairs of a workgroup share two groups on either side where
  // they can; ga -1: none), with the nodes pair_nodes[pair_ptr[q] ..) that
  // touch both; gstrip[node * ngroup + g] = first strip index | mask << 16
  // (mask 0: none); zero: offset of kTreeNB blocks of zeros in the slab
  int T = 0, ngroup = 0, parts = 1, sparts = 1;  // sparts: parts that split the scenarios
  std::vector<int> pair_g, pair_ptr, pair_nodes, gstrip;
  long long zero = 0;
};

// The pivot kernel keeps the maps of a node's children in LDS up to this many
// shorts.
constexpr int kTreeMapLds = 16384;

// Builds the tree from the filled pattern; empty string on success.
std::string build_tree(const Sym& s, Tree& t);

// Device bytes of the arrays that a handle has on the tree, or with panels in
// device memory instead.
long long tree_bytes(const Sym& s, const Tree& t);
long long panel_bytes(const Sym& s);

// Whether the tree is worth its memory with `free` bytes left on the device.
// Below about 1000 buses it takes more than the panels (200 buses x 600
// scenarios 0.87 against 0.46 GiB; at 9241 x 16 2.4 against 13), and what it
// takes in addition is missing when the handle's solve or the caller allocate
// next, so it may be a sixteenth of what is free.
constexpr bool tree_affordable(long long tree, long long panel, long long free) {
  return tree - panel <= free / 16;
}

// Levels whose nodes are spread over several workgroups per scenario in the
// step's sweeps (one launch each): the first levels, while they hold more
// than kTreeWide nodes (a level inside a longer launch costs what a launch
// does, 9-13 us, and more with several nodes: from 5 nodes on 16 grids took
// 1393 us, from 2 1358).  The rest run in one workgroup per scenario.  A
// workgroup takes one node, or kTreeStepNodes at a time with kTreeNB wavefronts
// each.
constexpr int kTreeWide = 1, kTreeStepNodes = 2;
int tree_wide_levels(const Tree& t);

}  // namespace rkkt
