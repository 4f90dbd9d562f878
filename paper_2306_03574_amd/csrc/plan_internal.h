// The plan object shared by the C ABI (abac_api.hip) and the request server
// (server.hip).  Internal: not part of the public header.
#pragma once
#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "../../include/abac.h"
#include "abac_internal.h"

using abac::DevPlan;
using abac::MinresState;
using abac::Snapshot;
using abac::kSnapRing;

struct ProfPair {
  int kid;
  hipEvent_t e0, e1;
};


struct abac_plan {
  DevPlan P;
  int prec;
  double T, alpha;
  hipStream_t stream;
  void* ws;
  size_t ws_bytes;
  bool own_ws;
  // variable-coefficient face weights (workspace region) and the preconditioner's
  // constant coefficient abar (1 for the constant-coefficient problem)
  double* coef_ws;
  double abar;
  // asynchronous solve bookkeeping
  Snapshot* h_ring;      // host-mapped pinned memory, kSnapRing * B snapshots written by the device
  int epoch;              // number of the current solve
  long long ring_posted;  // snapshots enqueued in the current solve (= device sequence number)
  const double* f;
  double* u;
  bool active;
  // kernel timing
  bool prof;
  std::vector<ProfPair> pending;
  std::vector<hipEvent_t> event_pool;
  double prof_ms[ABAC_K_COUNT];
  long long prof_n[ABAC_K_COUNT];
};

namespace abac {
// Non-blocking: whether snapshot `seq` of the current solve has been written for every
// right-hand side; if so *snaps points to them (host memory).
bool plan_peek_snapshot(const abac_plan* p, long long seq, const Snapshot** snaps);
hipError_t launch_fill_normal(double* out, unsigned long long n, unsigned long long seed, hipStream_t s);
hipError_t launch_fill_zero(double* out, unsigned long long n, hipStream_t s);
// the thread-local message abac_last_error() returns
void set_last_error(const std::string& msg);
// whether a group (abac_group_set) can take the plan as a member (its solve aside)
bool group_accepts(const abac_plan* p);
}  // namespace abac
