// A HIP runtime of host memory and launchers that only record their
// arguments, so that the library's host code (api.cpp) runs on the CPU: what
// it allocates, queues and launches is then a matter of counting.
#pragma once

#include <map>
#include <string>
#include <vector>

#include "fused2d.h"
#include "internal.h"

namespace fake {

struct Launch {
  std::string kind;           // conc, update, fields, fused2d, fused_mob, batch, ...
  nflbm::StepArgs step{};     // of conc, update, fields; the first member's of batch
  nflbm::FusedArgs fused{};   // of a fused2d launch of one simulation
  nflbm::FusedLaunch shape{};
  int nsteps = 0;             // of fused launches
};

struct State {
  std::vector<Launch> launches;
  std::map<void*, size_t> device, pinned;   // live allocations
  long long mallocs = 0, syncs = 0;         // hipMalloc and hipStreamSynchronize calls
  long long copied_after = 0;               // the waits before the last hipMemcpy
  long long events = 0;                     // live events
  size_t fail_at = 0;                       // a hipMalloc of this size fails
  bool pinned_fails = false;                // hipHostMalloc fails
  int groups_per_cu = 0;                    // occupancy of every kernel (0: not known)

  size_t device_bytes() const {
    size_t b = 0;
    for (const auto& a : device) b += a.second;
    return b;
  }
  long long count(const std::string& kind) const {
    long long c = 0;
    for (const Launch& l : launches) c += l.kind == kind;
    return c;
  }
};
State& state();

}  // namespace fake
