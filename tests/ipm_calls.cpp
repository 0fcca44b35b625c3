// Host replay of the interior-point driver: ipm.cpp linked with stand-ins for
// the HIP runtime and the launchers that compute nothing and keep account of
// the order of calls.  Prints one line per solve: mode, the failing runtime
// call (0: none), return code, status, whether everything given to the second
// stream was waited for when the solve returned, and whether every residual
// was formed from the values of the iterate (not of a trial point).
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "handle.h"

namespace {

hipStream_t const kSt = (hipStream_t)0x10, kSide = (hipStream_t)0x20;
long long side_seq = 0, side_joined = 0;             // work given to the second stream, and waited for
std::map<hipEvent_t, long long> covers;              // event: the second stream's work it stands behind
std::map<hipStream_t, long long> knows;              // stream: the second stream's work it waits for
int calls = 0, fail_at = 0, mode = 0, iters = 0;
bool at_trial = false, resid_ok = true;
rkkt_problem* prob = nullptr;

void work(hipStream_t s) {
  if (s == kSide) ++side_seq;
}
hipError_t call() { return ++calls == fail_at ? hipErrorUnknown : hipSuccess; }
void join(long long seq) { side_joined = side_joined > seq ? side_joined : seq; }

}  // namespace

extern "C" {
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (call() != hipSuccess) return hipErrorUnknown;
  covers[e] = s == kSide ? side_seq : knows[s];
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (call() != hipSuccess) return hipErrorUnknown;
  if (s == kSt) join(knows[s] = std::max(knows[s], covers[e]));
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (call() != hipSuccess) return hipErrorUnknown;
  join(covers[e]);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (call() != hipSuccess) return hipErrorUnknown;
  if (s == kSide) join(side_seq);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return call(); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return call(); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  if (n) std::memcpy(d, s, n);
  return call();
}
hipError_t hipGetLastError() { return call(); }
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipMalloc(void** p, size_t n) { return *p = std::calloc(1, n + 64), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::calloc(1, n + 64), hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, hipSuccess; }
int rkkt_evaluate(rkkt_problem*, const double*, const double*, const double*, const double*, double, double*, double*,
                  double*, double*, double*, hipStream_t s) {
  at_trial = false;
  work(s);
  return RKKT_OK;
}
}

namespace rkkt {
long long ipm_part_doubles(const DP&) { return 1; }
void ipm_resid(const DP&, const IpmDev&, double, double* out, hipStream_t s) {
  work(s);
  resid_ok = resid_ok && !at_trial;
  for (int q = 0; q < 6; ++q) out[q] = 0.0;
  out[0] = mode == 0 && iters >= 3 ? 0.0 : 1e3;
}
// mode 0: every trial point is accepted, two convergent iterations; 1: none is
void ipm_merit(const DP&, const IpmDev&, bool trial, double* out, hipStream_t s) {
  work(s);
  out[0] = 1.0;
  out[1] = trial ? 1.0 / (2 + iters) : 10.0;
  out[2] = 0.0;
  out[3] = trial && mode == 1 ? 1.0 : 0.0;
}
void ipm_step_trial(const DP&, const IpmDev&, double, double, double* out, hipStream_t s) {
  work(s);
  out[0] = out[1] = 1.0;
  out[2] = -1.0;
  out[3] = mode == 2 ? 1.0 : 0.0;           // factorisation fails
  out[4] = mode == 3 ? -3.0 : 0.0;          // device status
  out[5] = 0.0;
}
void ipm_trial(const DP&, const IpmDev&, double, hipStream_t s) { work(s); }
void ipm_accept(const DP&, const IpmDev&, double, double, double, double, hipStream_t s) {
  work(s);
  at_trial = false;
  ++iters;
}
void ipm_init_primal(const DP&, const IpmDev&, double, double, hipStream_t s) { work(s); }
void ipm_init_slack(const DP&, const IpmDev&, double, double, hipStream_t s) { work(s); }
void ipm_warm_primal(const DP&, const IpmDev&, const double*, const double*, double, double, hipStream_t s) { work(s); }
void ipm_warm_duals(const DP&, const IpmDev&, const double*, const double*, double, double, hipStream_t s) { work(s); }
void ipm_warm_implied(const DP&, const IpmDev&, double, hipStream_t s) { work(s); }
void ipm_grad_max(const DP&, const IpmDev&, double* out, hipStream_t s) { work(s), out[0] = 1.0; }
void launch_evaluate_values(const DP&, const double* x, const double*, hipStream_t s) {
  work(s);
  at_trial = x == prob->ipm.xt;
}
void launch_assemble(const DP&, const double*, double, double*, double*, double*, double*, double*, hipStream_t s) { work(s); }
void launch_hessian(const DP&, const double*, const double*, const double*, const double*, double, hipStream_t s) { work(s); }
void launch_condense_values(const DP&, const double*, const double*, double, hipStream_t s) { work(s); }
void launch_refactor(const DP&, hipStream_t s) { work(s); }
void launch_reduce(const DP&, hipStream_t s) { work(s); }
void launch_stacked_product(const DP&, hipStream_t s) { work(s); }
void launch_scenario_sum(const DP&, const double*, double, double*, hipStream_t s) { work(s); }
void launch_cholesky_from(const DP&, const double*, double*, int*, hipStream_t s) { work(s); }
void launch_reduced_solve(const DP&, const double*, const double*, double*, hipStream_t s) { work(s); }
void launch_step_rhs(const DP&, const double*, const double*, const double*, const double*, const double*, hipStream_t s) { work(s); }
void launch_step_recover(const DP&, const double*, const double*, const double*, const double*, const double*, double*,
                         double*, double*, double*, hipStream_t s) { work(s); }
}  // namespace rkkt

int main() {
  rkkt_problem p;
  prob = &p;
  rkkt::Sym& y = p.sym;
  y.N = p.d.N = 1;
  y.nx = p.d.nx = 2;
  y.nu = p.d.nu = 1;
  y.m = p.d.m = 3;
  y.xl = y.xu = std::vector<double>(2);
  y.ul = y.uu = std::vector<double>(1);
  y.sl = y.su = std::vector<double>(3);
  int status_words[2] = {0, 0};
  p.d.status = status_words;
  p.side_stream = kSide;
  for (int i = 0; i < 2; ++i) {
    p.fork_ev[i] = (hipEvent_t)(size_t)(0x100 + i);
    p.join_ev[i] = (hipEvent_t)(size_t)(0x200 + i);
  }
  rkkt_ipm_result r;
  rkkt_solve(&p, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, &r, kSt);  // makes the workspace
  for (mode = 0; mode < 4; ++mode)
    for (fail_at = 0;; ++fail_at) {
      calls = iters = 0;
      side_seq = side_joined = 0;
      covers.clear();
      knows.clear();
      at_trial = false;
      resid_ok = true;
      const int rc = rkkt_solve(&p, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, &r, kSt);
      std::printf("%d %d %d %d %d %d\n", mode, fail_at, rc, r.status, side_joined == side_seq, resid_ok && !at_trial);
      if (fail_at > 0 && calls < fail_at) break;
    }
  return 0;
}
