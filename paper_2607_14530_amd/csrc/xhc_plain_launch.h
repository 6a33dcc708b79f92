// Whether a single-pass launch may be a plain one (host side; Api names the HIP
// calls, so that the rule can be run without a GPU).
//
// A team waits for its members, so launches in flight together must not fill
// the chip with unfinished teams only.  Each launch has at most one (members
// are numbered as they start), which holds G - 1 workgroups at most.  HIP runs
// at most one kernel per hardware queue at a time: GPU_MAX_HW_QUEUES of them,
// 4 unless set, for all streams of the default priority without a CU mask, and
// one for cooperative launches.  With room for 8 such teams beside one more
// workgroup the launch is plain.  Everything else is cooperative, one at a time
// and no member before all can start, which costs about 20 us more (T = 16,
// C = 4096: 54 against 36 us a call, of which the kernels are 35): streams of
// another priority (queues of their own) and of a CU mask (a queue of their own,
// and perhaps fewer CUs than a team has members), a mask on the whole process,
// and streams that cannot be asked.  The queues of other processes cannot be
// counted: what that leaves open stands in xhc.h at xhc_impl.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

namespace xhc {

constexpr int kPlainLaunches = 8;   // in flight at once

struct ProcessQueues {
  int count = 4;
  bool masked = false;
};
inline ProcessQueues process_queues() {
  ProcessQueues p;
  const auto value = [](const char* name) {
    const char* v = getenv(name);
    return v && *v ? v : nullptr;
  };
  if (const char* v = value("GPU_MAX_HW_QUEUES")) p.count = atoi(v);
  p.masked = value("HSA_CU_MASK") || value("ROC_GLOBAL_CU_MASK");
  return p;
}

// (the two named streams are handles that only some calls know; neither can
// have a mask or a priority)
template <typename Api>
bool stream_has_whole_chip(hipStream_t s, int cus) {
  if (s == nullptr || s == hipStreamLegacy || s == hipStreamPerThread) return true;
  constexpr int kWords = 32;
  uint32_t mask[kWords] = {};
  int prio = 0;
  if (cus > 32 * kWords || Api::priority(s, &prio) != hipSuccess || Api::cu_mask(s, kWords, mask) != hipSuccess) {
    Api::clear_error();   // (the launch's own check would report it)
    return false;
  }
  int n = 0;
  for (uint32_t w : mask) n += __builtin_popcount(w);
  return prio == 0 && n >= cus;
}

template <typename Api>
bool plain_launch(int G, int cus, int per_cu, const ProcessQueues& p, hipStream_t s) {
  if (p.count < 1 || p.count + 1 > kPlainLaunches || p.masked) return false;
  return kPlainLaunches * (G - 1) < cus * per_cu && stream_has_whole_chip<Api>(s, cus);
}

}  // namespace xhc
