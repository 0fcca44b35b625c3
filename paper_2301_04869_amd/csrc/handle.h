// Definition of the opaque handle, shared by the C ABI (api.cpp) and the
// interior-point driver (ipm.cpp).
#pragma once

#include <string>
#include <vector>

#include "device.h"
#include "ipm.h"
#include "rkkt.h"
#include "symbolic.h"
#include "tree.h"

struct rkkt_problem {
  rkkt::Sym sym;
  rkkt::Tree tree;  // empty unless sym.tree
  rkkt::DP d{};
  int device = 0;
  std::vector<void*> allocs;
  long long bytes = 0;
  long long idx_bytes = 0;  // of which shared index arrays
  std::string err;
  // stage timing (rkkt_profile_begin / rkkt_profile_end)
  bool prof = false;
  std::vector<hipEvent_t> events;  // 2 per record
  std::vector<int> rec_stage;
  size_t rec_used = 0;
  // interior-point driver workspace (allocated by the first rkkt_solve)
  bool ipm_ready = false;
  rkkt::IpmDev ipm{};
  std::vector<void*> ipm_allocs;
  double* ipm_host = nullptr;  // pinned; ipm.hs is its device address
  // captured hot-path pass
  hipStream_t cap_stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
  // second stream of rkkt_iterate and rkkt_solve and its two fork / join event
  // pairs
  hipStream_t side_stream = nullptr;
  hipEvent_t fork_ev[2] = {nullptr, nullptr}, join_ev[2] = {nullptr, nullptr};
};

// Runs `launch` between two events on `stream` when profiling is on.
template <typename F>
inline void stage(rkkt_problem* p, int id, hipStream_t stream, F&& launch) {
  if (!p->prof || 2 * (p->rec_used + 1) > p->events.size()) {
    launch();
    return;
  }
  size_t r = p->rec_used++;
  (void)hipEventRecord(p->events[2 * r], stream);
  launch();
  (void)hipEventRecord(p->events[2 * r + 1], stream);
  p->rec_stage[r] = id;
}
