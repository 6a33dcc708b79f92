// Host build of the rule that makes a single-pass launch plain or cooperative
// (xhc_plain_launch.h) with the stream calls answered from the input.
//
// Input, one case per line: G cus per_cu stream status_priority priority
// status_mask bits (stream: 0 null, 1 legacy, 2 per-thread, 3 one of the
// caller's; a status other than 0 makes that call fail; bits: CUs in the
// mask).  Output, one line per case: plain (0 or 1), stream calls made, and
// errors they left behind.  The environment is the process's own.
#include <cstdio>

#include "xhc_plain_launch.h"

static int g_prio_status, g_prio, g_mask_status, g_bits, g_calls, g_errors;

struct FakeApi {
  static hipError_t priority(hipStream_t, int* prio) {
    ++g_calls;
    if (g_prio_status) return ++g_errors, hipErrorInvalidHandle;
    *prio = g_prio;
    return hipSuccess;
  }
  static hipError_t cu_mask(hipStream_t, int words, uint32_t* mask) {
    ++g_calls;
    if (g_mask_status) return ++g_errors, hipErrorInvalidValue;
    for (int i = 0; i < g_bits && i < 32 * words; ++i) mask[i / 32] |= 1u << (i % 32);
    return hipSuccess;
  }
  static void clear_error() { g_errors = 0; }
};

int main() {
  const xhc::ProcessQueues q = xhc::process_queues();
  int G, cus, per_cu, stream;
  while (std::scanf("%d %d %d %d %d %d %d %d", &G, &cus, &per_cu, &stream, &g_prio_status, &g_prio, &g_mask_status,
                    &g_bits) == 8) {
    g_calls = g_errors = 0;
    int own = 0;
    const hipStream_t s[] = {nullptr, hipStreamLegacy, hipStreamPerThread, reinterpret_cast<hipStream_t>(&own)};
    std::printf("%d ", xhc::plain_launch<FakeApi>(G, cus, per_cu, q, s[stream]) ? 1 : 0);
    std::printf("%d %d\n", g_calls, g_errors);
  }
  return 0;
}
