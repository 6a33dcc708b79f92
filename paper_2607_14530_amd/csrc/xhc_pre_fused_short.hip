// Instances of the single-pass pre whose last slices are short or empty.
#include "xhc_pre_fused.h"

namespace xhc {

const void* fused_kernel_short(int G) {
  switch (G) {
#define XHC_TEAM(GV) \
  case GV: return reinterpret_cast<const void*>(k_pre_fused<GV, true>);
    XHC_TEAMS(XHC_TEAM)
#undef XHC_TEAM
    default: return nullptr;
  }
}

}  // namespace xhc
