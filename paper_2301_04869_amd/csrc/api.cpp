// C ABI of the reduced-KKT hot path (declared in include/rkkt.h).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <algorithm>
#include <cstring>
#include <string>
#include <tuple>
#include <type_traits>
#include <vector>

#include "device.h"
#include "rkkt.h"
#include "symbolic.h"

#include "handle.h"

namespace {

thread_local std::string g_err;

int fail(rkkt_problem* p, int code, const std::string& msg) {
  if (p) p->err = msg;
  else g_err = msg;
  return code;
}

int hip_fail(rkkt_problem* p, hipError_t e, const char* where) {
  return fail(p, RKKT_ERR_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

template <typename T>
hipError_t dalloc(rkkt_problem* p, T** out, size_t n) {
  void* ptr = nullptr;
  size_t bytes = (n ? n : 1) * sizeof(T);
  hipError_t e = hipMalloc(&ptr, bytes);
  if (e != hipSuccess) return e;
  p->allocs.push_back(ptr);
  p->bytes += (long long)bytes;
  *out = static_cast<T*>(ptr);
  return hipSuccess;
}

template <typename T>
hipError_t upload(rkkt_problem* p, const T** out, const std::vector<T>& v) {
  T* ptr = nullptr;
  hipError_t e = dalloc(p, &ptr, v.size());
  if (e != hipSuccess) return e;
  if (std::is_integral<T>::value) p->idx_bytes += (long long)(v.size() * sizeof(T));
  if (!v.empty()) e = hipMemcpy(ptr, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
  *out = ptr;
  return e;
}

void fill_dims(const rkkt::Sym& s, rkkt_dims* o, long long bytes, long long idx_bytes) {
  std::memset(o, 0, sizeof(*o));
  o->n_x = s.nx; o->n_u = s.nu; o->m = s.m; o->n_scen = s.N;
  o->n_bus = s.nb; o->n_line = s.nl; o->n_gen = s.ng;
  o->nnz_gx = (long long)s.gx_col.size();
  o->nnz_gu = (long long)s.gu_col.size();
  o->nnz_h = (long long)s.h_col.size();
  o->nnz_k = (long long)s.k_col.size();
  o->nnz_lu = (long long)s.f_col.size();
  o->lu_update_flops = s.lu_flops;
  long long nkx = 0;
  for (int r = 0; r < s.nz; ++r) nkx += s.k_usplit[r] - s.k_ptr[r];
  o->nnz_kx = nkx;
  o->n_ev = s.n_ev;
  o->n_trip = (long long)s.t_row.size();
  o->levels_up = (int)s.lvu_ptr.size() - 1;
  o->levels_down = (int)s.lvd_ptr.size() - 1;
  o->col_tile = s.col_tile;
  o->workspace_bytes = bytes;
  o->variant = s.variant;
  o->lds_reduce = s.lds_reduce ? 1 : 0;
  o->lds_group = s.lds_group ? 1 : 0;
  o->lds_step = s.lds_step ? 1 : 0;
  o->chain_rows = s.chain_t;
  o->scen_per_group = s.spw;
  for (int r = 0; r < s.nz; ++r) {
    const long long nxc = s.k_usplit[r] - s.k_ptr[r], nuc = s.k_ptr[r + 1] - s.k_usplit[r];
    if (r < s.nx) {
      o->nnz_kxx += nxc;
      o->nnz_kxu += nuc;
    } else {
      o->nnz_kuu += nuc;
    }
  }
  o->idx_bytes = idx_bytes;
  o->n_load = s.nload;
  o->sweep_form = s.sweep_form;
  o->tree = s.tree ? 1 : 0;
}

// Appends the entries of a level-sliced schedule packed as two words of
// 16-bit pairs (the form the LDS kernels stage).
void pack_entries(const rkkt::Sched& sc, std::vector<unsigned>& out) {
  const size_t n = sc.ent.size() / 4;
  for (size_t q = 0; q < n; ++q) {
    out.push_back((unsigned)sc.ent[4 * q] | ((unsigned)sc.ent[4 * q + 1] << 16));
    out.push_back((unsigned)sc.ent[4 * q + 2] | ((unsigned)sc.ent[4 * q + 3] << 16));
  }
}

// Uploads a level-sliced schedule for global-memory kernels: the pointer
// table and the entries as int4.
hipError_t upload_sched(rkkt_problem* p, const rkkt::Sched& sc, bool packed, const int** ptr,
                        const void** ent) {
  (void)packed;
  hipError_t e = upload(p, ptr, sc.ptr);
  if (e != hipSuccess) return e;
  const int* d = nullptr;
  e = upload(p, &d, sc.ent);
  *ent = d;
  return e;
}

int check_launch(rkkt_problem* p, const char* where) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(p, e, where);
  return RKKT_OK;
}

}  // namespace

extern "C" {

int rkkt_analyze(const rkkt_network* net, int n_scen, const rkkt_options* opt, rkkt_dims* out) {
  if (!net || !out) return fail(nullptr, RKKT_ERR_ARG, "rkkt_analyze: null argument");
  rkkt::Sym s;
  std::string m = rkkt::build_symbolic(*net, n_scen, opt, s);
  if (!m.empty()) return fail(nullptr, RKKT_ERR_ARG, "rkkt_analyze: " + m);
  fill_dims(s, out, 0, 0);
  return RKKT_OK;
}

int rkkt_analyze_lu(const rkkt_network* net, int n_scen, const rkkt_options* opt, int* perm,
                    int* f_ptr, int* f_col) {
  if (!net || !perm || !f_ptr || !f_col) return fail(nullptr, RKKT_ERR_ARG, "rkkt_analyze_lu: null argument");
  rkkt::Sym s;
  std::string m = rkkt::build_symbolic(*net, n_scen, opt, s);
  if (!m.empty()) return fail(nullptr, RKKT_ERR_ARG, "rkkt_analyze_lu: " + m);
  std::memcpy(perm, s.perm.data(), s.perm.size() * sizeof(int));
  std::memcpy(f_ptr, s.f_ptr.data(), s.f_ptr.size() * sizeof(int));
  std::memcpy(f_col, s.f_col.data(), s.f_col.size() * sizeof(int));
  return RKKT_OK;
}

int rkkt_analyze_schedule(const rkkt_network* net, int n_scen, const rkkt_options* opt, int which,
                          int* nphase, int* slots, int* n_ent, int* chain_rows, int* ptr, int* ent,
                          int* chain_pos, int* n_upd, int* upd) {
  if (!net || !nphase || !slots || !n_ent || !chain_rows || which < 0 || which > 4)
    return fail(nullptr, RKKT_ERR_ARG, "rkkt_analyze_schedule: bad argument");
  rkkt::Sym s;
  std::string m = rkkt::build_symbolic(*net, n_scen, opt, s);
  if (!m.empty()) return fail(nullptr, RKKT_ERR_ARG, "rkkt_analyze_schedule: " + m);
  const rkkt::Sched* sc[5] = {&s.red_up, &s.red_dn, &s.stp_up, &s.stp_dn, &s.fac};
  const rkkt::Sched& q = *sc[which];
  *nphase = q.nphase;
  *slots = q.S;
  *n_ent = (int)(q.ent.size() / 4);
  *chain_rows = s.chain_t;
  if (ptr) std::memcpy(ptr, q.ptr.data(), q.ptr.size() * sizeof(int));
  if (ent) std::memcpy(ent, q.ent.data(), q.ent.size() * sizeof(int));
  if (chain_pos) std::memcpy(chain_pos, s.chain_pos.data(), s.chain_pos.size() * sizeof(int));
  if (n_upd) *n_upd = which == 4 ? (int)s.upd_dst.size() : 0;
  if (upd && which == 4) std::memcpy(upd, s.upd_dst.data(), s.upd_dst.size() * sizeof(int));
  return RKKT_OK;
}

// no_memory: set where the device's memory did not hold a handle on the
// elimination tree
static int create_impl(const rkkt_network* net, int n_scen, const double* pd, const double* qd,
                       const rkkt_options* opt, rkkt_problem** out, bool allow_tree, bool* no_memory) {
  (void)hipGetLastError();
  if (!net || !out) return fail(nullptr, RKKT_ERR_ARG, "rkkt_create: null argument");
  *out = nullptr;
  if (net->n_load > 0 && (!pd || !qd)) return fail(nullptr, RKKT_ERR_ARG, "rkkt_create: null loads");
  rkkt_problem* p = new rkkt_problem();
  p->device = opt ? opt->device : 0;
  std::string m = rkkt::build_symbolic(*net, n_scen, opt, p->sym, true, allow_tree);
  if (!m.empty()) {
    delete p;
    return fail(nullptr, RKKT_ERR_ARG, "rkkt_create: " + m);
  }
  if (p->sym.tree) {
    m = rkkt::build_tree(p->sym, p->tree);
    if (m.empty() && !rkkt::tree_fits(p->tree)) {
      p->tree = rkkt::Tree();
      m = rkkt::build_symbolic(*net, n_scen, opt, p->sym, true, false);
    }
    if (!m.empty()) {
      delete p;
      return fail(nullptr, RKKT_ERR_ARG, "rkkt_create: " + m);
    }
  }
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) {
    int rc = hip_fail(nullptr, e, "rkkt_create: hipSetDevice");
    delete p;
    return rc;
  }
  if (p->sym.tree) {
    size_t free = 0, total = 0;
    if (hipMemGetInfo(&free, &total) == hipSuccess &&
        !rkkt::tree_affordable(rkkt::tree_bytes(p->sym, p->tree), rkkt::panel_bytes(p->sym), (long long)free)) {
      p->tree = rkkt::Tree();
      m = rkkt::build_symbolic(*net, n_scen, opt, p->sym, true, false);
      if (!m.empty()) {
        delete p;
        return fail(nullptr, RKKT_ERR_ARG, "rkkt_create: " + m);
      }
    }
  }

  const rkkt::Sym& s = p->sym;
  rkkt::DP& d = p->d;
  d.nb = s.nb; d.nl = s.nl; d.ng = s.ng; d.nload = s.nload; d.ref = s.ref; d.gref = s.gref;
  d.nx = s.nx; d.nu = s.nu; d.m = s.m; d.nz = s.nz; d.N = s.N;
  d.n_ev = s.n_ev; d.off_P = s.off_P; d.off_Q = s.off_Q; d.off_gx = s.off_gx;
  d.off_gu = s.off_gu; d.off_h = s.off_h;
  d.nnz_gx = (int)s.gx_col.size(); d.nnz_gu = (int)s.gu_col.size();
  d.nnz_h = (int)s.h_col.size(); d.nnz_k = (int)s.k_col.size(); d.nnz_f = (int)s.f_col.size();
  d.nnz_l = s.nnz_l;
  d.nlev_up = (int)s.lvu_ptr.size() - 1;
  d.nlev_dn = (int)s.lvd_ptr.size() - 1;
  d.nph_u = s.stp_up.nphase;
  d.nph_d = s.stp_dn.nphase;
  d.n_kz = (int)(s.kz_items.size() / 4);
  {
    // condensed values: enough workgroups per scenario for about 512 in all
    // (at most 16), each staging the scenario's sigma_s and H values and its
    // share of the triplets; none when that exceeds 64 KiB of LDS
    const int E = (int)s.k_col.size();
    const int G = std::min(16, std::max(1, (512 + s.N - 1) / s.N));
    const int per = (E + G - 1) / G;
    int nt = 0;
    for (int g = 0; g < G; ++g) {
      const int e0 = std::min(E, g * per), e1 = std::min(E, e0 + per);
      nt = std::max(nt, s.t_ptr[e1] - s.t_ptr[e0]);
    }
    const long long lds = 8LL * (s.m + (long long)s.h_col.size()) + 4LL * (per + 1 + 3LL * nt);
    d.cv_split = lds <= 64 * 1024 ? G : 0;
    d.cv_nt = nt;
  }
  d.kz_rounds = s.kz_rounds;
  d.nph_ru = s.red_up.nphase;
  d.nph_rd = s.red_dn.nphase;
  d.n_upd = (int)s.upd_dst.size();
  d.n_sent = (int)(s.red_up.ent.size() / 4);
  d.chain_t = s.chain_t;
  d.chain_c0 = s.nx - s.chain_t;
  d.fac_npiv = s.chain_t > 0 ? (int)s.lvu_ptr.size() - 1 - s.chain_t : (int)s.lvu_ptr.size() - 1;
  d.lu_stride = d.nnz_f + s.nx;
  d.col_tile = s.col_tile;
  d.lds_red = s.lds_reduce ? 1 : 0;
  d.lds_grp = s.lds_group ? 1 : 0;
  d.lds_stp = s.lds_step ? 1 : 0;
  d.spw = s.spw;
  d.upd_lds = s.upd_lds ? 1 : 0;
  d.variant = s.variant;
  d.tree = s.tree ? 1 : 0;
  d.nu_pad = s.nu_pad;
  d.nchunk = s.nchunk;
  // per-unit line and cost data
  std::vector<double> gs(s.nl), bs(s.nl), bc(s.nl), ca(s.ng), cb(s.ng), cc(s.ng);
  for (int l = 0; l < s.nl; ++l) {
    double den = net->r[l] * net->r[l] + net->x[l] * net->x[l];
    gs[l] = net->r[l] / den;
    bs[l] = -net->x[l] / den;
    bc[l] = 0.5 * net->b[l];
  }
  for (int g = 0; g < s.ng; ++g) {
    ca[g] = 1e4 * net->c2[g];
    cb[g] = 1e2 * net->c1[g];
    cc[g] = net->c0[g];
  }
  d.aref = ca[s.gref];
  d.bref = cb[s.gref];
  std::vector<int> load_of_bus(s.nb, -1), grow_bus(s.nx), gen_u(s.ng, -1), k_row(s.k_col.size()),
      gx_row(s.gx_col.size());
  for (int i = 0; i < s.nx; ++i)
    for (int q = s.gx_ptr[i]; q < s.gx_ptr[i + 1]; ++q) gx_row[q] = i;
  for (int j = 0; j < s.nload; ++j) load_of_bus[net->load_bus[j]] = j;
  for (int b = 0; b < s.nb; ++b) {
    if (s.prow[b] >= 0) grow_bus[s.prow[b]] = b;
    if (s.qrow[b] >= 0) grow_bus[s.qrow[b]] = b;
  }
  for (size_t j = 0; j < s.gnr.size(); ++j) gen_u[s.gnr[j]] = s.ng + (int)j;
  for (int r = 0; r < s.nz; ++r)
    for (int q = s.k_ptr[r]; q < s.k_ptr[r + 1]; ++q) k_row[q] = r;

#define UP(field, vec) \
  if ((e = upload(p, &d.field, vec)) != hipSuccess) goto hip_error;
  UP(line_f, s.line_f) UP(line_t, s.line_t) UP(line_loc, s.line_loc)
  UP(gs, gs) UP(bs, bs) UP(bc, bc)
  UP(th_src, s.th_src) UP(v_src, s.v_src) UP(prow, s.prow) UP(qrow, s.qrow) UP(pg_u, s.pg_u)
  UP(gnr, s.gnr) UP(gen_bus, s.gen_bus) UP(ca, ca) UP(cb, cb) UP(cc, cc)
  UP(load_of_bus, load_of_bus) UP(grow_bus, grow_bus) UP(gen_u, gen_u)
  UP(perm, s.perm) UP(pinv, s.pinv)
  UP(ev_ptr, s.ev_ptr) UP(ev_src, s.ev_src) UP(ev_const, s.ev_const)
  UP(gx_ptr, s.gx_ptr) UP(gx_col, s.gx_col) UP(gu_ptr, s.gu_ptr) UP(gu_col, s.gu_col)
  UP(gxc_ptr, s.gxc_ptr) UP(gxc_row, s.gxc_row) UP(gxc_pos, s.gxc_pos)
  UP(guc_ptr, s.guc_ptr) UP(guc_row, s.guc_row) UP(guc_pos, s.guc_pos)
  UP(h_ptr, s.h_ptr) UP(h_col, s.h_col) UP(ht_ptr, s.ht_ptr) UP(ht_row, s.ht_row)
  UP(ht_pos, s.ht_pos) UP(h0pos, s.h0pos)
  UP(k_ptr, s.k_ptr) UP(k_col, s.k_col) UP(k_diag, s.k_diag) UP(k_usplit, s.k_usplit)
  UP(kz_items, s.kz_items)
  UP(k_row, k_row) UP(gx_row, gx_row)
  UP(w_ptr, s.w_ptr) UP(w_src, s.w_src) UP(wp_ptr, s.wp_ptr) UP(wp_a, s.wp_a) UP(wp_b, s.wp_b)
  UP(wp_coef, s.wp_coef) UP(w_const, s.w_const)
  UP(t_ptr, s.t_ptr) UP(t_row, s.t_row) UP(t_a, s.t_a) UP(t_b, s.t_b)
  UP(f_ptr, s.f_ptr) UP(f_col, s.f_col) UP(f_diag, s.f_diag) UP(f_tpos, s.f_tpos) UP(gx2f, s.gx2f)
  UP(lvu_ptr, s.lvu_ptr) UP(lvu_rows, s.lvu_rows) UP(lvd_ptr, s.lvd_ptr) UP(lvd_rows, s.lvd_rows)
  UP(upd_dst, s.upd_dst) UP(chain_pos, s.chain_pos)
#undef UP
  // schedules: LDS images (packed entries and every index array the kernel
  // stages, in its LDS order) for the LDS kernels, int4 entries otherwise
  if (s.tree) {
    // no kernel follows them
  } else if (s.lds_reduce && s.col_tile != 64) {
    std::vector<unsigned> b;
    pack_entries(s.red_up, b);
    pack_entries(s.red_dn, b);
    for (const std::vector<int>* v : {&s.red_up.ptr, &s.red_dn.ptr, &s.k_ptr, &s.k_usplit, &s.k_col,
                                      &s.guc_ptr, &s.guc_row})
      b.insert(b.end(), v->begin(), v->end());
    if (b.size() % 2) b.push_back(0);  // whole 8-byte units
    d.blob_red_words = (int)b.size();
    if ((e = upload(p, &d.blob_red, b)) != hipSuccess) goto hip_error;
  } else {
    if ((e = upload_sched(p, s.red_up, false, &d.ru_ptr, &d.ru_ent)) != hipSuccess) goto hip_error;
    if ((e = upload_sched(p, s.red_dn, false, &d.rd_ptr, &d.rd_ent)) != hipSuccess) goto hip_error;
  }
  if (s.tree) {
    // the step sweeps the tree
  } else if (s.lds_step) {
    std::vector<unsigned> b;
    pack_entries(s.stp_up, b);
    pack_entries(s.stp_dn, b);
    b.insert(b.end(), s.stp_up.ptr.begin(), s.stp_up.ptr.end());
    b.insert(b.end(), s.stp_dn.ptr.begin(), s.stp_dn.ptr.end());
    // largest entry count of a slot, per phase (the sweep picks its code path)
    for (const rkkt::Sched* sc : {&s.stp_up, &s.stp_dn}) {
      const int S = rkkt::kGroupLds, nph = (int)(sc->ptr.size() - 1) / S;
      for (int q = 0; q < nph; ++q) {
        int mx = 0;
        for (int j = 0; j < S; ++j) mx = std::max(mx, sc->ptr[q * S + j + 1] - sc->ptr[q * S + j]);
        b.push_back((unsigned)mx);
      }
    }
    if (b.size() % 2) b.push_back(0);
    d.blob_stp_words = (int)b.size();
    if ((e = upload(p, &d.blob_stp, b)) != hipSuccess) goto hip_error;
  } else {
    if ((e = upload_sched(p, s.stp_up, false, &d.su_ptr, &d.su_ent)) != hipSuccess) goto hip_error;
    if ((e = upload_sched(p, s.stp_dn, false, &d.sd_ptr, &d.sd_ent)) != hipSuccess) goto hip_error;
  }
  if (s.tree) {
    // the fronts factorise G_x
  } else if (s.lds_group) {
    std::vector<unsigned> f;
    pack_entries(s.fac, f);
    for (const std::vector<int>* v : {&s.fac.ptr, &s.lvu_ptr, &s.lvu_rows, &s.f_diag, &s.f_ptr})
      f.insert(f.end(), v->begin(), v->end());
    if (s.upd_lds) f.insert(f.end(), s.upd_dst.begin(), s.upd_dst.end());
    if (f.size() % 2) f.push_back(0);
    d.blob_fac_words = (int)f.size();
    if ((e = upload(p, &d.blob_fac, f)) != hipSuccess) goto hip_error;
  } else {
    if ((e = upload_sched(p, s.fac, false, &d.fa_ptr, &d.fa_ent)) != hipSuccess) goto hip_error;
  }
  {
    if (s.tree) {
      const rkkt::Tree& t = p->tree;
      rkkt::TreeDP& r = d.tr;
      r.host = &t;
#define UP(field, vec) \
  if ((e = upload(p, &r.field, vec)) != hipSuccess) goto hip_error;
      UP(nodes, t.nodes) UP(children, t.children) UP(rows, t.rows) UP(strips, t.strips) UP(orig, t.orig) UP(optr, t.optr)
      UP(oent, t.oent) UP(lev_ptr, t.lev_ptr) UP(lev_nodes, t.lev_nodes) UP(job_ptr, t.job_ptr)
      UP(jobs, t.jobs) UP(uord, t.uord) UP(kuu, t.kuu) UP(pair_g, t.pair_g) UP(pair_ptr, t.pair_ptr)
      UP(pair_nodes, t.pair_nodes) UP(gstrip, t.gstrip) UP(rmap, t.rmap) UP(smap, t.smap)
      UP(cjobs, t.cjobs) UP(sn_ptr, t.sn_ptr) UP(sn, t.sn)
#undef UP
      r.npool = t.npool; r.nstrip = t.nstrip; r.T = t.T; r.ngroup = t.ngroup; r.parts = t.parts; r.sparts = t.sparts;
      r.npair = (int)t.pair_g.size() / 2;
      r.nkuu = (int)t.kuu.size() / 3;
      r.stride = t.stride;
      r.zero = t.zero;
      r.vstride = t.vstride;
      r.ncjob = (int)t.cjobs.size() / 2;
      r.nlev = (int)t.lev_ptr.size() - 1;
      r.nwide = rkkt::tree_wide_levels(t);
      const size_t ld = (size_t)t.ngroup * t.T * rkkt::kTreeB;
      if ((e = dalloc(p, &r.slab, (size_t)s.N * t.stride)) != hipSuccess) goto hip_error;
      if ((e = hipMemset2D(r.slab + t.zero, sizeof(double) * t.stride, 0,
                           sizeof(double) * rkkt::kTreeNB * rkkt::kTreeBlk, s.N)) != hipSuccess)
        goto hip_error;
      if ((e = dalloc(p, &r.pool, (size_t)s.N * t.npool * rkkt::kTreeBlk)) != hipSuccess) goto hip_error;
      if ((e = dalloc(p, &r.vec, (size_t)s.N * t.vstride)) != hipSuccess) goto hip_error;
      if ((e = dalloc(p, &r.x, (size_t)s.N * s.nx)) != hipSuccess) goto hip_error;
      if ((e = dalloc(p, &r.y, (size_t)s.N * s.nx)) != hipSuccess) goto hip_error;
      if ((e = dalloc(p, &r.upart, (size_t)s.N * r.ncjob * 2 * rkkt::kTreeRows)) != hipSuccess) goto hip_error;
      if ((e = dalloc(p, &r.part, t.parts * ld * ld)) != hipSuccess) goto hip_error;
    }
    const size_t N = s.N;
    const int ntile = (s.nu + s.col_tile - 1) / s.col_tile;
    size_t panel = d.lds_stp || d.tree ? 1 : 2 * N * (size_t)s.nx;
    if (!d.lds_red && d.variant == 1 && !d.tree) panel = std::max(panel, N * ntile * 2 * (size_t)s.nx * s.col_tile);
    // stacked panels: N n_z rows, then a slab of zero rows that the stacked
    // product's last chunk reads past the last row
    const size_t stacked = d.variant == 2 ? (N * (size_t)s.nz + rkkt::kSpSlab) * s.nu_pad : 1;
    if ((e = dalloc(p, &d.pdb, N * s.nb)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.lstat, N * s.nl)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.qdb, N * s.nb)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.LV, N * s.nl * rkkt::kLVsize)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.LH, N * s.nl * rkkt::kLHsize)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.EV, N * s.n_ev)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.W, N * s.k_col.size())) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.K, N * s.k_col.size())) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.LU, d.tree ? 1 : N * (size_t)d.lu_stride)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.part, d.variant == 1 && !d.tree ? N * s.nu * (size_t)s.nu : 1)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.panel, panel)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.Zst, stacked)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.KZst, stacked)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.gpart, d.variant == 2 ? (size_t)s.nchunk * s.nu * s.nu : 1)) != hipSuccess)
      goto hip_error;
    if (d.variant == 2) {
      // zero padding columns and the identity rows of Z, written once
      if ((e = hipMemset(d.Zst, 0, stacked * sizeof(double))) != hipSuccess) goto hip_error;
      if ((e = hipMemset(d.KZst, 0, stacked * sizeof(double))) != hipSuccess) goto hip_error;
      rkkt::launch_identity_rows(d, nullptr);
      if ((e = hipGetLastError()) != hipSuccess) goto hip_error;
      if ((e = hipDeviceSynchronize()) != hipSuccess) goto hip_error;
    }
    if ((e = dalloc(p, &d.rhat1, N * s.nx)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.wbuf, d.lds_stp || d.tree ? 1 : N * (size_t)s.m)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.rpart, N * s.nu)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.qbuf, N * s.nx)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.cw, (size_t)((s.nu + 63) / 64) * 4096)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.rinv, (size_t)((s.nu + 63) / 64) * 4096)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.ry, s.nu)) != hipSuccess) goto hip_error;
    if ((e = dalloc(p, &d.status, 2)) != hipSuccess) goto hip_error;
    if (d.tree && (e = rkkt::configure_tree_kernels()) != hipSuccess) goto hip_error;
    if ((e = rkkt::configure_lu_kernels(d)) != hipSuccess) goto hip_error;
    if ((e = rkkt::configure_dense_kernels(d)) != hipSuccess) goto hip_error;
    if ((e = rkkt::configure_eval_kernels(d)) != hipSuccess) goto hip_error;
    if ((e = hipStreamCreateWithFlags(&p->side_stream, hipStreamNonBlocking)) != hipSuccess) goto hip_error;
    for (int i = 0; i < 2; ++i) {
      if ((e = hipEventCreateWithFlags(&p->fork_ev[i], hipEventDisableTiming)) != hipSuccess) goto hip_error;
      if ((e = hipEventCreateWithFlags(&p->join_ev[i], hipEventDisableTiming)) != hipSuccess) goto hip_error;
    }
    if ((e = hipMemset(d.status, 0, 2 * sizeof(int))) != hipSuccess) goto hip_error;
    rkkt::launch_line_status(d, nullptr, nullptr);
    if ((e = hipGetLastError()) != hipSuccess) goto hip_error;
    // loads
    if (s.nload > 0) {
      double *tpd = nullptr, *tqd = nullptr;
      size_t nbytes = N * s.nload * sizeof(double);
      if ((e = hipMalloc((void**)&tpd, nbytes)) != hipSuccess) goto hip_error;
      if ((e = hipMalloc((void**)&tqd, nbytes)) != hipSuccess) { (void)hipFree(tpd); goto hip_error; }
      e = hipMemcpy(tpd, pd, nbytes, hipMemcpyHostToDevice);
      if (e == hipSuccess) e = hipMemcpy(tqd, qd, nbytes, hipMemcpyHostToDevice);
      if (e == hipSuccess) {
        rkkt::launch_bus_loads(d, tpd, tqd, nullptr);
        e = hipGetLastError();
      }
      if (e == hipSuccess) e = hipDeviceSynchronize();
      (void)hipFree(tpd);
      (void)hipFree(tqd);
      if (e != hipSuccess) goto hip_error;
    } else {
      if ((e = hipMemset(d.pdb, 0, N * s.nb * sizeof(double))) != hipSuccess) goto hip_error;
      if ((e = hipMemset(d.qdb, 0, N * s.nb * sizeof(double))) != hipSuccess) goto hip_error;
      // what was enqueued above (the tree's zero blocks, line and device status
      // among it) is done before a caller's stream, which need not wait for the
      // null stream, can read it
      if ((e = hipDeviceSynchronize()) != hipSuccess) goto hip_error;
    }
  }
  *out = p;
  return RKKT_OK;
hip_error : {
  *no_memory = e == hipErrorOutOfMemory && p->sym.tree;
  int rc = hip_fail(nullptr, e, "rkkt_create");
  if (p->side_stream) (void)hipStreamDestroy(p->side_stream);
  for (hipEvent_t ev : {p->fork_ev[0], p->fork_ev[1], p->join_ev[0], p->join_ev[1]})
    if (ev) (void)hipEventDestroy(ev);
  for (void* q : p->allocs) (void)hipFree(q);
  delete p;
  return rc;
}
}

// A handle that does not fit with the tree after all is made without it.
int rkkt_create(const rkkt_network* net, int n_scen, const double* pd, const double* qd,
                const rkkt_options* opt, rkkt_problem** out) {
  bool no_memory = false;
  const int rc = create_impl(net, n_scen, pd, qd, opt, out, true, &no_memory);
  return no_memory ? create_impl(net, n_scen, pd, qd, opt, out, false, &no_memory) : rc;
}

int rkkt_set_loads(rkkt_problem* p, const double* pd_dev, const double* qd_dev, hipStream_t stream) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p) return fail(nullptr, RKKT_ERR_ARG, "rkkt_set_loads: null handle");
  if (p->d.nload > 0 && (!pd_dev || !qd_dev)) return fail(p, RKKT_ERR_ARG, "rkkt_set_loads: null loads");
  if (p->d.nload == 0) return RKKT_OK;
  rkkt::launch_bus_loads(p->d, pd_dev, qd_dev, stream);
  return check_launch(p, "rkkt_set_loads");
}

int rkkt_set_line_status(rkkt_problem* p, const double* status_dev, hipStream_t stream) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p) return fail(nullptr, RKKT_ERR_ARG, "rkkt_set_line_status: null handle");
  if (!status_dev) return fail(p, RKKT_ERR_ARG, "rkkt_set_line_status: null status");
  rkkt::launch_line_status(p->d, status_dev, stream);
  return check_launch(p, "rkkt_set_line_status");
}

int rkkt_dims_get(const rkkt_problem* p, rkkt_dims* out) {
  if (!p || !out) return fail(nullptr, RKKT_ERR_ARG, "rkkt_dims_get: null argument");
  fill_dims(p->sym, out, p->bytes, p->idx_bytes);
  return RKKT_OK;
}

int rkkt_evaluate(rkkt_problem* p, const double* x, const double* u, const double* y,
                  const double* z, double obj_weight, double* f, double* grad_x, double* grad_u,
                  double* g, double* h, hipStream_t stream) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p) return fail(nullptr, RKKT_ERR_ARG, "rkkt_evaluate: null handle");
  if (!x || !u || !y || !z || !f || !grad_x || !grad_u || !g || !h)
    return fail(p, RKKT_ERR_ARG, "rkkt_evaluate: null array");
  if (!std::isfinite(obj_weight)) return fail(p, RKKT_ERR_ARG, "rkkt_evaluate: non-finite obj_weight");
  stage(p, RKKT_STAGE_EVALUATE, stream, [&] {
    rkkt::launch_evaluate(p->d, x, u, y, z, obj_weight, f, grad_x, grad_u, g, h, stream);
  });
  return check_launch(p, "rkkt_evaluate");
}

int rkkt_condense(rkkt_problem* p, const double* sigma_x, const double* sigma_u,
                  const double* sigma_s, double delta_w, double* khat, hipStream_t stream) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p) return fail(nullptr, RKKT_ERR_ARG, "rkkt_condense: null handle");
  if (!sigma_x || !sigma_u || !sigma_s || !khat) return fail(p, RKKT_ERR_ARG, "rkkt_condense: null array");
  if (!std::isfinite(delta_w)) return fail(p, RKKT_ERR_ARG, "rkkt_condense: non-finite delta_w");
  stage(p, RKKT_STAGE_CONDENSE_VALUES, stream,
        [&] { rkkt::launch_condense_values(p->d, sigma_x, sigma_s, delta_w, stream); });
  stage(p, RKKT_STAGE_REFACTOR, stream, [&] { rkkt::launch_refactor(p->d, stream); });
  stage(p, RKKT_STAGE_REDUCE, stream, [&] { rkkt::launch_reduce(p->d, stream); });
  if (p->d.variant == 2 || p->d.tree)
    stage(p, RKKT_STAGE_STACKED_PRODUCT, stream, [&] { rkkt::launch_stacked_product(p->d, stream); });
  stage(p, RKKT_STAGE_SCENARIO_SUM, stream,
        [&] { rkkt::launch_scenario_sum(p->d, sigma_u, delta_w, khat, stream); });
  return check_launch(p, "rkkt_condense");
}

int rkkt_factor(rkkt_problem* p, double* khat, int* info_dev, hipStream_t stream) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p) return fail(nullptr, RKKT_ERR_ARG, "rkkt_factor: null handle");
  if (!khat || !info_dev) return fail(p, RKKT_ERR_ARG, "rkkt_factor: null array");
  stage(p, RKKT_STAGE_FACTOR, stream, [&] { rkkt::launch_cholesky(p->d, khat, info_dev, stream); });
  return check_launch(p, "rkkt_factor");
}

int rkkt_step(rkkt_problem* p, const double* r1x, const double* r1u, const double* r2,
              const double* r3, const double* r4, const double* sigma_s, const double* chol,
              double* px, double* pu, double* ps, double* py, double* pz, hipStream_t stream) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p) return fail(nullptr, RKKT_ERR_ARG, "rkkt_step: null handle");
  if (!r1x || !r1u || !r2 || !r3 || !r4 || !sigma_s || !chol || !px || !pu || !ps || !py || !pz)
    return fail(p, RKKT_ERR_ARG, "rkkt_step: null array");
  stage(p, RKKT_STAGE_STEP_RHS, stream,
        [&] { rkkt::launch_step_rhs(p->d, r1x, r2, r3, r4, sigma_s, stream); });
  stage(p, RKKT_STAGE_REDUCED_SOLVE, stream,
        [&] { rkkt::launch_reduced_solve(p->d, r1u, chol, pu, stream); });
  stage(p, RKKT_STAGE_STEP_RECOVER, stream, [&] {
    rkkt::launch_step_recover(p->d, r2, r3, r4, sigma_s, pu, px, ps, py, pz, stream);
  });
  return check_launch(p, "rkkt_step");
}

int rkkt_status(rkkt_problem* p, hipStream_t stream, int* code, int* scenario) {
  if (!p || !code) return fail(p, RKKT_ERR_ARG, "rkkt_status: null argument");
  hipError_t e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_status");
  int st[2] = {0, -1};
  e = hipMemcpy(st, p->d.status, sizeof st, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_status");
  int zero[2] = {0, 0};
  e = hipMemcpy(p->d.status, zero, sizeof zero, hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_status");
  *code = st[0];
  if (scenario) *scenario = st[0] ? st[1] : -1;
  return RKKT_OK;
}

// The pass of rkkt_iterate.  With `fork`, two groups of kernels run on the
// handle's side stream, concurrently with kernels of `stream` that leave
// most compute units idle; every result is the same as with the pass on one
// stream:
//   A: g, h, f and gradients, W and K (after the line and Jacobian values,
//      which are all the refactorisation reads) beside the refactorisation;
//   B: the step's right-hand-side solves (LU factors and K only) beside the
//      stacked product, the scenario sum and the dense factorisation.
// Each group is a fork and a join of events; under graph capture they become
// concurrent branches of the graph.  No return between a fork and its join,
// so that the side stream never stays part of a capture of `stream`.
static int iterate_impl(rkkt_problem* p, const rkkt_iteration* it, hipStream_t stream, bool fork) {
  (void)hipGetLastError();  // do not report an earlier, unrelated error
  if (!p || !it) return fail(p, RKKT_ERR_ARG, "rkkt_iterate: null argument");
  if (!it->x || !it->u || !it->y || !it->z || !it->f || !it->grad_x || !it->grad_u || !it->g ||
      !it->h || !it->sigma_x || !it->sigma_u || !it->sigma_s || !it->khat || !it->chol ||
      !it->info || !it->r1x || !it->r1u || !it->r2 || !it->r3 || !it->r4 || !it->px || !it->pu ||
      !it->ps || !it->py || !it->pz)
    return fail(p, RKKT_ERR_ARG, "rkkt_iterate: null array");
  if (!std::isfinite(it->obj_weight)) return fail(p, RKKT_ERR_ARG, "rkkt_iterate: non-finite obj_weight");
  if (!std::isfinite(it->delta_w)) return fail(p, RKKT_ERR_ARG, "rkkt_iterate: non-finite delta_w");
  const rkkt::DP& d = p->d;
  hipStream_t side = fork ? p->side_stream : stream;
  auto fork_to_side = [&](int g) -> hipError_t {
    if (!fork) return hipSuccess;
    hipError_t e = hipEventRecord(p->fork_ev[g], stream);
    return e == hipSuccess ? hipStreamWaitEvent(side, p->fork_ev[g], 0) : e;
  };
  auto join_record = [&](int g) -> hipError_t {
    return fork ? hipEventRecord(p->join_ev[g], side) : hipSuccess;
  };
  auto join_wait = [&](int g, hipError_t recorded) -> hipError_t {
    if (!fork || recorded != hipSuccess) return recorded;
    return hipStreamWaitEvent(stream, p->join_ev[g], 0);
  };
  stage(p, RKKT_STAGE_EVALUATE, stream,
        [&] { rkkt::launch_evaluate_values(d, it->x, it->u, stream); });
  hipError_t e = fork_to_side(0);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_iterate: fork");
  stage(p, RKKT_STAGE_EVALUATE, side, [&] {
    rkkt::launch_evaluate_rest(d, it->x, it->u, it->y, it->z, it->obj_weight, it->f, it->grad_x,
                               it->grad_u, it->g, it->h, side);
  });
  stage(p, RKKT_STAGE_CONDENSE_VALUES, side,
        [&] { rkkt::launch_condense_values(d, it->sigma_x, it->sigma_s, it->delta_w, side); });
  hipError_t ej = join_record(0);
  stage(p, RKKT_STAGE_REFACTOR, stream, [&] { rkkt::launch_refactor(d, stream); });
  e = join_wait(0, ej);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_iterate: join");
  stage(p, RKKT_STAGE_REDUCE, stream, [&] { rkkt::launch_reduce(d, stream); });
  // group B's fork is recorded right after the reduction and the stacked
  // product is enqueued before the side stream waits on it, so the graph's
  // first child of the reduction is the stacked product
  e = fork ? hipEventRecord(p->fork_ev[1], stream) : hipSuccess;
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_iterate: fork");
  if (d.variant == 2 || d.tree)
    stage(p, RKKT_STAGE_STACKED_PRODUCT, stream, [&] { rkkt::launch_stacked_product(d, stream); });
  e = fork ? hipStreamWaitEvent(side, p->fork_ev[1], 0) : hipSuccess;
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_iterate: fork");
  stage(p, RKKT_STAGE_STEP_RHS, side, [&] {
    rkkt::launch_step_rhs(d, it->r1x, it->r2, it->r3, it->r4, it->sigma_s, side);
  });
  ej = join_record(1);
  stage(p, RKKT_STAGE_SCENARIO_SUM, stream,
        [&] { rkkt::launch_scenario_sum(d, it->sigma_u, it->delta_w, it->khat, stream); });
  stage(p, RKKT_STAGE_FACTOR, stream,
        [&] { rkkt::launch_cholesky_from(d, it->khat, it->chol, it->info, stream); });
  e = join_wait(1, ej);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_iterate: join");
  stage(p, RKKT_STAGE_REDUCED_SOLVE, stream,
        [&] { rkkt::launch_reduced_solve(d, it->r1u, it->chol, it->pu, stream); });
  stage(p, RKKT_STAGE_STEP_RECOVER, stream, [&] {
    rkkt::launch_step_recover(d, it->r2, it->r3, it->r4, it->sigma_s, it->pu, it->px, it->ps,
                              it->py, it->pz, stream);
  });
  return check_launch(p, "rkkt_iterate");
}

int rkkt_iterate(rkkt_problem* p, const rkkt_iteration* it, hipStream_t stream) {
  return iterate_impl(p, it, stream, true);
}

static void release_graph(rkkt_problem* p) {
  if (p->gexec) (void)hipGraphExecDestroy(p->gexec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  p->gexec = nullptr;
  p->graph = nullptr;
}

int rkkt_graph_capture(rkkt_problem* p, const rkkt_iteration* it) {
  if (!p || !it) return fail(p, RKKT_ERR_ARG, "rkkt_graph_capture: null argument");
  release_graph(p);
  hipError_t e;
  if (!p->cap_stream) {
    e = hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking);
    if (e != hipSuccess) return hip_fail(p, e, "rkkt_graph_capture: stream");
  }
  const bool prof = p->prof;
  p->prof = false;
  e = hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) { p->prof = prof; return hip_fail(p, e, "rkkt_graph_capture: begin"); }
  int rc = rkkt_iterate(p, it, p->cap_stream);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(p->cap_stream, &g);
  p->prof = prof;
  if (rc != RKKT_OK) { if (g) (void)hipGraphDestroy(g); return rc; }
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_graph_capture: end");
  p->graph = g;
  e = hipGraphInstantiate(&p->gexec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) { release_graph(p); return hip_fail(p, e, "rkkt_graph_capture: instantiate"); }
  return RKKT_OK;
}

int rkkt_graph_launch(rkkt_problem* p, hipStream_t stream) {
  if (!p || !p->gexec) return fail(p, RKKT_ERR_ARG, "rkkt_graph_launch: nothing captured");
  hipError_t e = hipGraphLaunch(p->gexec, stream);
  if (e != hipSuccess) return hip_fail(p, e, "rkkt_graph_launch");
  return RKKT_OK;
}

struct rkkt_batch {
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
};

int rkkt_batch_destroy(rkkt_batch* b) {
  if (!b) return RKKT_OK;
  if (b->gexec) (void)hipGraphExecDestroy(b->gexec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  delete b;
  return RKKT_OK;
}

// Switched off: a capture of several instances whose passes forked to side
// streams ended in a host segmentation fault inside this call, and its cause
// has not been shown, so the call returns an error instead of capturing.
int rkkt_batch_create(rkkt_problem* const* problems, const rkkt_iteration* its, int n,
                      rkkt_batch** out) {
  (void)problems;
  (void)its;
  (void)n;
  if (out) *out = nullptr;
  return fail(nullptr, RKKT_ERR_ARG,
              "rkkt_batch_create: switched off (a multi-instance graph capture ended in a host fault whose "
              "cause is not shown); run instances one handle at a time");
}

// ---- independent instances, one launch per kernel configuration
// The pass of every instance (rkkt_iterate on one stream) is listed as
// launches (launches_eval / _lu / _dense); launches with equal place in the
// pass, kernel, template variant, block size and panel column become one
// launch whose blocks map back to (instance, block) through a table, with
// the largest dynamic LDS of the group.  Every block runs the same code on
// the same data as in the instance's own launch, so the results are the
// same bit for bit.
struct rkkt_multi {
  struct Group {
    rkkt::Launch l;
    unsigned nblk = 0;
    long long lds = 0;
    size_t off = 0;  // first entry of its block table
  };
  std::vector<rkkt_problem*> probs;
  std::vector<Group> groups;
  rkkt::DP* dps = nullptr;
  rkkt_iteration* its = nullptr;
  rkkt::MultiBlk* blk = nullptr;
  hipStream_t cap = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
  std::string err;
};

static std::string g_multi_err;
static int multi_fail(rkkt_multi* m, int code, const std::string& msg) {
  (m ? m->err : g_multi_err) = msg;
  return code;
}
static hipError_t multi_dispatch(const rkkt_multi* m, const rkkt_multi::Group& g, hipStream_t s, bool prepare) {
  bool handled = false;
  const rkkt::MultiBlk* blk = m->blk + g.off;
  hipError_t e = rkkt::multi_eval(g.l, g.nblk, g.lds, m->dps, m->its, blk, s, prepare, &handled);
  if (!handled) e = rkkt::multi_lu(g.l, g.nblk, g.lds, m->dps, m->its, blk, s, prepare, &handled);
  if (!handled) e = rkkt::multi_tree(g.l, g.nblk, g.lds, m->dps, m->its, blk, s, prepare, &handled);
  if (!handled) e = rkkt::multi_dense(g.l, g.nblk, g.lds, m->dps, m->its, blk, s, prepare, &handled);
  if (!handled) return hipErrorInvalidValue;
  return e;
}

int rkkt_multi_destroy(rkkt_multi* m) {
  if (!m) return RKKT_OK;
  if (m->gexec) (void)hipGraphExecDestroy(m->gexec);
  if (m->graph) (void)hipGraphDestroy(m->graph);
  if (m->cap) (void)hipStreamDestroy(m->cap);
  (void)hipFree(m->dps);
  (void)hipFree(m->its);
  (void)hipFree(m->blk);
  delete m;
  return RKKT_OK;
}

const char* rkkt_multi_last_error(const rkkt_multi* m) { return m ? m->err.c_str() : g_multi_err.c_str(); }

int rkkt_multi_create(rkkt_problem* const* problems, const rkkt_iteration* its, int n, rkkt_multi** out) {
  if (!problems || !its || !out || n < 1) return multi_fail(nullptr, RKKT_ERR_ARG, "rkkt_multi_create: bad argument");
  *out = nullptr;
  for (int i = 0; i < n; ++i) {
    if (!problems[i]) return multi_fail(nullptr, RKKT_ERR_ARG, "rkkt_multi_create: null handle");
    if (problems[i]->device != problems[0]->device)
      return multi_fail(nullptr, RKKT_ERR_ARG, "rkkt_multi_create: instances on different devices");
    for (int j = 0; j < i; ++j)
      if (problems[j] == problems[i])
        return multi_fail(nullptr, RKKT_ERR_ARG,
                          "rkkt_multi_create: instance " + std::to_string(i) + " repeats the handle of instance " +
                              std::to_string(j) + " (instances of one handle share its workspace)");
    const rkkt_iteration& it = its[i];
    if (!it.x || !it.u || !it.y || !it.z || !it.f || !it.grad_x || !it.grad_u || !it.g || !it.h ||
        !it.sigma_x || !it.sigma_u || !it.sigma_s || !it.khat || !it.chol || !it.info || !it.r1x || !it.r1u ||
        !it.r2 || !it.r3 || !it.r4 || !it.px || !it.pu || !it.ps || !it.py || !it.pz)
      return multi_fail(nullptr, RKKT_ERR_ARG, "rkkt_multi_create: instance " + std::to_string(i) + ": null array");
    if (!std::isfinite(it.obj_weight) || !std::isfinite(it.delta_w))
      return multi_fail(nullptr, RKKT_ERR_ARG,
                        "rkkt_multi_create: instance " + std::to_string(i) + ": non-finite obj_weight or delta_w");
  }
  (void)hipGetLastError();
  // every instance's launches, grouped
  struct Item {
    rkkt::Launch l;
    int inst;
  };
  std::vector<Item> items;
  for (int i = 0; i < n; ++i) {
    std::vector<rkkt::Launch> ls;
    const rkkt::DP& d = problems[i]->d;
    rkkt::launches_eval(d, ls);
    rkkt::launches_lu(d, ls);
    if (d.tree) rkkt::launches_tree(d, ls);
    rkkt::launches_dense(d, ls);
    for (const auto& l : ls) items.push_back({l, i});
  }
  auto gkey = [](const rkkt::Launch& l) { return std::make_tuple(l.key, l.kernel, l.variant, l.threads, l.jb); };
  std::stable_sort(items.begin(), items.end(), [&](const Item& a, const Item& b) { return gkey(a.l) < gkey(b.l); });
  rkkt_multi* m = new rkkt_multi();
  m->probs.assign(problems, problems + n);
  std::vector<rkkt::MultiBlk> table;
  for (size_t a = 0; a < items.size();) {
    size_t b = a;
    rkkt_multi::Group g;
    g.l = items[a].l;
    g.off = table.size();
    while (b < items.size() && gkey(items[b].l) == gkey(items[a].l)) {
      const rkkt::Launch& l = items[b].l;
      for (int by = 0; by < l.gy; ++by)
        for (int bx = 0; bx < l.gx; ++bx) table.push_back({items[b].inst, bx, by, l.gx});
      g.lds = std::max(g.lds, l.lds);
      ++b;
    }
    g.nblk = (unsigned)(table.size() - g.off);
    if (g.nblk > 0) m->groups.push_back(g);
    a = b;
  }
  std::vector<rkkt::DP> hd(n);
  for (int i = 0; i < n; ++i) hd[i] = problems[i]->d;
  hipError_t e = hipSetDevice(problems[0]->device);
  if (e == hipSuccess) e = hipMalloc((void**)&m->dps, sizeof(rkkt::DP) * n);
  if (e == hipSuccess) e = hipMalloc((void**)&m->its, sizeof(rkkt_iteration) * n);
  if (e == hipSuccess) e = hipMalloc((void**)&m->blk, sizeof(rkkt::MultiBlk) * std::max<size_t>(table.size(), 1));
  if (e == hipSuccess) e = hipMemcpy(m->dps, hd.data(), sizeof(rkkt::DP) * n, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(m->its, its, sizeof(rkkt_iteration) * n, hipMemcpyHostToDevice);
  if (e == hipSuccess && !table.empty())
    e = hipMemcpy(m->blk, table.data(), sizeof(rkkt::MultiBlk) * table.size(), hipMemcpyHostToDevice);
  for (size_t q = 0; q < m->groups.size() && e == hipSuccess; ++q) e = multi_dispatch(m, m->groups[q], nullptr, true);
  if (e != hipSuccess) {
    const std::string msg = std::string("rkkt_multi_create: ") + hipGetErrorString(e);
    rkkt_multi_destroy(m);
    return multi_fail(nullptr, e == hipErrorOutOfMemory ? RKKT_ERR_NOMEM : RKKT_ERR_HIP, msg);
  }
  *out = m;
  return RKKT_OK;
}

int rkkt_multi_iterate(rkkt_multi* m, hipStream_t stream) {
  if (!m) return multi_fail(nullptr, RKKT_ERR_ARG, "rkkt_multi_iterate: null handle");
  (void)hipGetLastError();
  for (const auto& g : m->groups) {
    hipError_t e = multi_dispatch(m, g, stream, false);
    if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_iterate: ") + hipGetErrorString(e));
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_iterate: ") + hipGetErrorString(e));
  return RKKT_OK;
}

int rkkt_multi_capture(rkkt_multi* m) {
  if (!m) return multi_fail(nullptr, RKKT_ERR_ARG, "rkkt_multi_capture: null handle");
  if (m->gexec) (void)hipGraphExecDestroy(m->gexec);
  if (m->graph) (void)hipGraphDestroy(m->graph);
  m->gexec = nullptr;
  m->graph = nullptr;
  hipError_t e = hipSuccess;
  if (!m->cap) e = hipStreamCreateWithFlags(&m->cap, hipStreamNonBlocking);
  if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_capture: ") + hipGetErrorString(e));
  e = hipStreamBeginCapture(m->cap, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_capture: ") + hipGetErrorString(e));
  const int rc = rkkt_multi_iterate(m, m->cap);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(m->cap, &g);
  if (rc != RKKT_OK) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_capture: ") + hipGetErrorString(e));
  m->graph = g;
  e = hipGraphInstantiate(&m->gexec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_capture: ") + hipGetErrorString(e));
  return RKKT_OK;
}

int rkkt_multi_launch(rkkt_multi* m, hipStream_t stream) {
  if (!m || !m->gexec) return multi_fail(m, RKKT_ERR_ARG, "rkkt_multi_launch: nothing captured");
  hipError_t e = hipGraphLaunch(m->gexec, stream);
  if (e != hipSuccess) return multi_fail(m, RKKT_ERR_HIP, std::string("rkkt_multi_launch: ") + hipGetErrorString(e));
  return RKKT_OK;
}

int rkkt_multi_launches(const rkkt_multi* m) { return m ? (int)m->groups.size() : 0; }

// Launch-shape autotuner.  Stage 1 times `reps` condense calls (the
// reduction dominates them) for every reduction variant x column tile x
// schedule form of the reduction's solves (push / pull); stage
// 2 keeps the winner's variant and tile and times `reps` whole passes
// (rkkt_iterate) for every level-schedule grouping: scenarios per
// refactorisation / step workgroup (automatic, 1, 2, 4) x chain of
// single-row levels (automatic, none).  Candidates whose analysis lands on
// a shape already timed are skipped.
int rkkt_autotune(const rkkt_network* net, int n_scen, const double* pd, const double* qd,
                  const rkkt_options* opt, int reps, rkkt_options* best, double* best_ms) {
  if (!net || !best || !best_ms || reps < 1)
    return fail(nullptr, RKKT_ERR_ARG, "rkkt_autotune: bad argument");
  rkkt::Sym s0;
  std::string m = rkkt::build_symbolic(*net, n_scen, nullptr, s0);
  if (!m.empty()) return fail(nullptr, RKKT_ERR_ARG, "rkkt_autotune: " + m);
  const int N = n_scen, nx = s0.nx, nu = s0.nu, mm = s0.m;
  const rkkt_options base = opt ? *opt : rkkt_options{};
  std::vector<rkkt_options> stage1;
  const double stacked_bytes = 2.0 * 8.0 * N * (double)s0.nz * s0.nu_pad;
  for (int v : {1, 2}) {
    if (v == 2 && stacked_bytes > 4.0 * (1ull << 30)) continue;
    for (int w : {0, 8, 16, 32, 64}) {
      if (w > nu) continue;
      // schedule form: automatic, then each explicit form (a shape the
      // automatic choice already produced is skipped as seen)
      for (int form : {0, 1, 2}) {
        rkkt_options o = base;
        o.variant = v;
        o.col_tile = w;
        o.scen_per_group = 0;
        o.chain_rows = 0;
        o.sweep_form = form;
        stage1.push_back(o);
      }
    }
  }
  // fixed interior point (host), copied once; residuals all ones
  const size_t NX = (size_t)N * nx, NM = (size_t)N * mm, NU = (size_t)N * nu;
  std::vector<double> hx(NX), hu(nu), zeros_m(NM, 0.0), zeros_x(NX, 0.0);
  for (int k = 0; k < N; ++k)
    for (int i = 0; i < nx; ++i) hx[(size_t)k * nx + i] = i < s0.nb - 1 ? 0.0 : 1.0;
  for (int c = 0; c < nu; ++c) hu[c] = c < s0.ng ? 1.0 : 0.5 * (s0.ul[c] + s0.uu[c]);
  std::vector<double> ones(std::max({NX, NM, (size_t)nu}), 1.0);
  // every device array of the timed passes, carved from one allocation: the
  // sizes below, in the order they are taken, then the info word
  const size_t NN = (size_t)nu * nu;
  const size_t sizes[] = {NX, NX, NX, NX, NX, NM, NM, NM, NM, (size_t)nu, (size_t)nu, (size_t)nu,
                          (size_t)N, NX, NU, NX, NM, NN, NN, NX, (size_t)nu, NM, NX, NM};
  size_t nbuf = 0;
  for (size_t n : sizes) nbuf += n;
  double* buf = nullptr;
  hipError_t e = hipMalloc((void**)&buf, nbuf * sizeof(double) + sizeof(int));
  if (e != hipSuccess) return hip_fail(nullptr, e, "rkkt_autotune: buffers");
  double* q = buf;
  constexpr size_t kTakes = sizeof(sizes) / sizeof(sizes[0]);
  size_t taken = 0, ti = 0;
  bool layout_ok = true;
  auto take = [&](size_t n) {
    // the takes must follow `sizes` exactly (checked before any launch)
    layout_ok = layout_ok && ti < kTakes && sizes[ti] == n;
    ++ti;
    double* r = q;
    q += n;
    taken += n;
    return r;
  };
  rkkt_iteration it{};
  double *dx = take(NX), *dy = take(NX), *dsx = take(NX), *r1x = take(NX), *r3 = take(NX);
  double *dz = take(NM), *dss = take(NM), *r2 = take(NM), *r4 = take(NM);
  double *du = take(nu), *dsu = take(nu), *r1u = take(nu);
  it.x = dx; it.u = du; it.y = dy; it.z = dz; it.obj_weight = 1.0 / N;
  it.f = take(N); it.grad_x = take(NX); it.grad_u = take(NU); it.g = take(NX); it.h = take(NM);
  it.sigma_x = dsx; it.sigma_u = dsu; it.sigma_s = dss; it.delta_w = 1.0;
  it.khat = take((size_t)nu * nu); it.chol = take((size_t)nu * nu);
  it.r1x = r1x; it.r1u = r1u; it.r2 = r2; it.r3 = r3; it.r4 = r4;
  it.px = take(NX); it.pu = take(nu); it.ps = take(NM); it.py = take(NX); it.pz = take(NM);
  it.info = reinterpret_cast<int*>(q);
  if (!layout_ok || taken != nbuf || ti != kTakes) {
    (void)hipFree(buf);
    return fail(nullptr, RKKT_ERR_ARG, "rkkt_autotune: internal: buffer layout mismatch");
  }
  auto up = [&](double* d, const double* v, size_t n) {
    return hipMemcpy(d, v, n * sizeof(double), hipMemcpyHostToDevice);
  };
  for (auto pr : {std::make_pair(dx, hx.data()), std::make_pair(du, hu.data())})
    if (e == hipSuccess) e = up(pr.first, pr.second, pr.first == dx ? NX : nu);
  if (e == hipSuccess) e = up(dy, zeros_x.data(), NX);
  if (e == hipSuccess) e = up(dz, zeros_m.data(), NM);
  for (double* d : {dsx, r1x, r3})
    if (e == hipSuccess) e = up(d, ones.data(), NX);
  for (double* d : {dss, r2, r4})
    if (e == hipSuccess) e = up(d, ones.data(), NM);
  for (double* d : {dsu, r1u})
    if (e == hipSuccess) e = up(d, ones.data(), nu);
  hipEvent_t t0 = nullptr, t1 = nullptr;
  if (e == hipSuccess) e = hipEventCreate(&t0);
  if (e == hipSuccess) e = hipEventCreate(&t1);
  int rc = RKKT_OK;
  // times `reps` condense calls (whole = false) or passes (whole = true) of
  // one shape; returns the mean ms (1e300 when the shape was seen already)
  std::vector<std::vector<int>> seen;
  auto time_shape = [&](const rkkt_options& o, bool whole, rkkt_options* got) -> double {
    rkkt_problem* h = nullptr;
    rc = rkkt_create(net, n_scen, pd, qd, &o, &h);
    if (rc != RKKT_OK) return 1e300;
    const rkkt::Sym& sy = h->sym;
    // the elimination tree has no groups of scenarios and no chain
    const std::vector<int> key{whole ? 1 : 0, sy.variant, sy.col_tile, sy.tree ? 0 : sy.spw, sy.tree ? 0 : sy.chain_t,
                               sy.sweep_form, sy.lds_reduce ? 1 : 0, sy.tree ? 1 : 0};
    if (std::find(seen.begin(), seen.end(), key) != seen.end()) {
      rkkt_destroy(h);
      return 1e300;
    }
    seen.push_back(key);
    *got = o;
    got->variant = sy.variant;
    got->col_tile = sy.col_tile;
    got->sweep_form = sy.sweep_form;
    float ms = 0.f;
    rc = rkkt_evaluate(h, dx, du, dy, dz, it.obj_weight, it.f, it.grad_x, it.grad_u, it.g, it.h, nullptr);
    auto one = [&]() {
      return whole ? rkkt_iterate(h, &it, nullptr)
                   : rkkt_condense(h, dsx, dsu, dss, 1.0, it.khat, nullptr);
    };
    if (rc == RKKT_OK) rc = one();
    if (rc == RKKT_OK) e = hipEventRecord(t0, nullptr);
    for (int r = 0; r < reps && rc == RKKT_OK && e == hipSuccess; ++r) rc = one();
    if (rc == RKKT_OK && e == hipSuccess) e = hipEventRecord(t1, nullptr);
    if (rc == RKKT_OK && e == hipSuccess) e = hipEventSynchronize(t1);
    if (rc == RKKT_OK && e == hipSuccess) e = hipEventElapsedTime(&ms, t0, t1);
    if (rc != RKKT_OK) g_err = h->err;
    rkkt_destroy(h);
    return (rc == RKKT_OK && e == hipSuccess) ? ms / reps : 1e300;
  };
  rkkt_options b1 = base;
  double ms1 = 1e300;
  for (size_t ci = 0; ci < stage1.size() && e == hipSuccess && rc == RKKT_OK; ++ci) {
    rkkt_options got{};
    const double ms = time_shape(stage1[ci], false, &got);
    if (ms < ms1) { ms1 = ms; b1 = got; }
  }
  rkkt_options b2 = b1;
  double ms2 = 1e300;
  for (int spw : {0, 1, 2, 4})
    for (int chain : {0, -1}) {
      if (e != hipSuccess || rc != RKKT_OK) break;
      rkkt_options o = b1;
      o.scen_per_group = spw;
      o.chain_rows = chain;
      rkkt_options got{};
      const double ms = time_shape(o, true, &got);
      if (ms < ms2) { ms2 = ms; b2 = got; }
    }
  if (t0) (void)hipEventDestroy(t0);
  if (t1) (void)hipEventDestroy(t1);
  (void)hipFree(buf);
  if (rc != RKKT_OK) return fail(nullptr, rc, "rkkt_autotune: " + g_err);
  if (e != hipSuccess) return hip_fail(nullptr, e, "rkkt_autotune");
  *best = b2;
  *best_ms = ms2;
  return RKKT_OK;
}

int rkkt_batch_launch(rkkt_batch* b, hipStream_t stream) {
  if (!b || !b->gexec) return fail(nullptr, RKKT_ERR_ARG, "rkkt_batch_launch: no batch");
  hipError_t e = hipGraphLaunch(b->gexec, stream);
  if (e != hipSuccess) return hip_fail(nullptr, e, "rkkt_batch_launch");
  return RKKT_OK;
}

static void release_events(rkkt_problem* p) {
  for (hipEvent_t e : p->events) (void)hipEventDestroy(e);
  p->events.clear();
  p->rec_stage.clear();
  p->rec_used = 0;
  p->prof = false;
}

int rkkt_profile_begin(rkkt_problem* p, int max_records) {
  if (!p || max_records < 1) return fail(p, RKKT_ERR_ARG, "rkkt_profile_begin: bad argument");
  release_events(p);
  p->events.resize(2 * (size_t)max_records);
  for (auto& e : p->events) {
    hipError_t r = hipEventCreate(&e);
    if (r != hipSuccess) {
      e = nullptr;
      release_events(p);
      return hip_fail(p, r, "rkkt_profile_begin");
    }
  }
  p->rec_stage.assign(max_records, -1);
  p->prof = true;
  return RKKT_OK;
}

int rkkt_profile_end(rkkt_problem* p, hipStream_t stream, double* ms, int* count) {
  if (!p || !ms || !count) return fail(p, RKKT_ERR_ARG, "rkkt_profile_end: null argument");
  for (int i = 0; i < RKKT_NSTAGES; ++i) { ms[i] = 0.0; count[i] = 0; }
  hipError_t e = hipStreamSynchronize(stream);
  if (e != hipSuccess) { release_events(p); return hip_fail(p, e, "rkkt_profile_end"); }
  for (size_t r = 0; r < p->rec_used; ++r) {
    float t = 0.0f;
    e = hipEventElapsedTime(&t, p->events[2 * r], p->events[2 * r + 1]);
    if (e != hipSuccess) { release_events(p); return hip_fail(p, e, "rkkt_profile_end"); }
    ms[p->rec_stage[r]] += t;
    count[p->rec_stage[r]] += 1;
  }
  release_events(p);
  return RKKT_OK;
}

int rkkt_destroy(rkkt_problem* p) {
  if (!p) return RKKT_OK;
  release_events(p);
  release_graph(p);
  if (p->cap_stream) (void)hipStreamDestroy(p->cap_stream);
  if (p->side_stream) (void)hipStreamDestroy(p->side_stream);
  for (hipEvent_t ev : {p->fork_ev[0], p->fork_ev[1], p->join_ev[0], p->join_ev[1]})
    if (ev) (void)hipEventDestroy(ev);
  for (void* q : p->ipm_allocs) (void)hipFree(q);
  if (p->ipm_host) (void)hipHostFree(p->ipm_host);
  for (void* q : p->allocs) (void)hipFree(q);
  delete p;
  return RKKT_OK;
}

const char* rkkt_last_error(const rkkt_problem* p) {
  if (p) return p->err.c_str();
  return g_err.c_str();
}

}  // extern "C"
