// What the launch plans and the kernels share: sizes of the device, and the
// fixed region at the start of a workspace.  Plain C++: a program without a
// GPU can include it.
#pragma once

#include <cstddef>

namespace pvlm {

struct DeviceInfo {
  int cus = 0;   // compute units a call may plan for: the device's, or the stream's budget
  int xcds = 0;  // accelerator complex dies (workgroup i runs on die i % xcds); 0 = unknown
  bool budgeted = false;  // the stream has a compute-unit budget (pvlm_set_stream_cu_budget)
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Every workspace starts with a fixed-size region.  Verify's statistics records
// that a captured launch waits on, from kSyncVerifyOff to kSyncTopkOff, are 0
// between calls; accept keeps its decisions at kSyncAcceptOff (written before
// they are read in every call).  Nothing else of a workspace is relied on.
// kSyncLine enters only limits on batches and groups that calls are held to.
constexpr size_t kSyncRegion = 1024 * 1024;
constexpr size_t kSyncVerifyOff = 256 * 1024;
constexpr size_t kSyncTopkOff = 768 * 1024;
constexpr size_t kSyncAcceptOff = 896 * 1024;
constexpr size_t kSyncLine = 128;

}  // namespace pvlm
