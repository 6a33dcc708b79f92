// Launch of the single-pass pre (xhc_pre_fused.h), and its instances for widths
// that fill their team.
#include "xhc_plain_launch.h"
#include "xhc_pre_fused.h"

namespace xhc {

const void* fused_kernel_exact(int G) {
  switch (G) {
#define XHC_TEAM(GV) \
  case GV: return reinterpret_cast<const void*>(k_pre_fused<GV, false>);
    XHC_TEAMS(XHC_TEAM)
#undef XHC_TEAM
    default: return nullptr;
  }
}

namespace {

// zero n1 and n2 16-byte words at p1 and p2 (one launch)
__global__ void k_zero2(uint4* __restrict__ p1, int64_t n1, uint4* __restrict__ p2, int64_t n2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint4 z = make_uint4(0, 0, 0, 0);
  if (i < n1) p1[i] = z;
  else if (i - n1 < n2) p2[i - n1] = z;
}

struct DeviceInfo {
  int cus = 0;
  int per_cu = 0;
};

constexpr size_t kTileLds = (size_t)BUFB;

bool is_short(int C) { return C != team_size(C) * FCS; }
const void* fused_kernel(int C) {
  return is_short(C) ? fused_kernel_short(team_size(C)) : fused_kernel_exact(team_size(C));
}

// CU count, and resident workgroups per CU of the instance for width C; its
// dynamic LDS limit is raised here, once per device and thread
DeviceInfo device_info(int C) {
  static thread_local int dev_cached = -1;
  static thread_local DeviceInfo info[2 * kMaxG + 2];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return DeviceInfo{};
  if (dev != dev_cached) {
    for (DeviceInfo& i : info) i = DeviceInfo{};
    dev_cached = dev;
  }
  DeviceInfo& slot = info[2 * team_size(C) + (is_short(C) ? 1 : 0)];
  if (slot.cus == 0) {
    const void* f = fused_kernel(C);
    DeviceInfo di;
    if (!f || hipDeviceGetAttribute(&di.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&di.per_cu, f, FNT, kTileLds) != hipSuccess)
      return DeviceInfo{};
    slot = di;
  }
  return slot;
}

struct StreamApi {
  static hipError_t priority(hipStream_t s, int* prio) { return hipStreamGetPriority(s, prio); }
  static hipError_t cu_mask(hipStream_t s, int words, uint32_t* mask) { return hipExtStreamGetCUMask(s, words, mask); }
  static void clear_error() { (void)hipGetLastError(); }
};

}  // namespace

// Where AUTO takes the single pass: at every width it has a team for.  It reads
// the state once where the multi-kernel path reads it twice and needs three
// launches instead of seven.  Measured multi / single pass, K_r = 4: T = 8192
// C = 2560 387 / 243 us, T = 2048 C = 2112 157 / 83 us, T = 16 C = 2560 64 / 30
// us, T = 16 C = 160 (one and a quarter slices) 48 / 30 us.
bool fused_pre_auto(const xhc_dims* d) {
  return d->state_dtype == XHC_BF16 && d->N == FN && d->k == FK && d->Kr >= 1 &&
         FK * d->Kr + FK * FK <= 16 * NOBA && d->C % 32 == 0 && team_size(d->C) <= kMaxG &&
         d->T * team_size(d->C) * NV1 < ((int64_t)1 << 31);   // 32-bit token and partial indices
}

bool fused_pre_supported(const xhc_dims* d) {
  return fused_pre_auto(d) && d->C % FCS == 0 && kMaxG % (d->C / FCS) == 0;
}

// Workspace: error counter, records (sized for up to kMaxResident co-resident
// workgroups, and no more teams than there are tiles), active partials
// [G][34][T] and their per-token sums.
constexpr int kMaxResident = 1024;
int64_t max_teams(const xhc_dims* d) {
  const int64_t ntiles = (d->T + FM - 1) / FM, most = kMaxResident / team_size(d->C);
  return ntiles < most ? ntiles : most;
}
size_t rec1_words(const xhc_dims* d) { return (size_t)max_teams(d) * RING * team_size(d->C) * FM * NV1; }
size_t rec2_words(const xhc_dims* d) { return (size_t)max_teams(d) * RING * FM * NV2; }
size_t align256(size_t b) { return (b + 255) / 256 * 256; }

size_t fused_pre_ws_bytes(const xhc_dims* d) {
  const int G = team_size(d->C);
  return 256 + align256(rec1_words(d) * 8) + align256(rec2_words(d) * 8) +
         align256((size_t)G * NV1 * d->T * sizeof(float)) + align256((size_t)NV1 * d->T * sizeof(float));
}

hipError_t launch_pre_fused(const xhc_dims* d, const void* X, const void* packed_full, const float* colsum,
                            const void* packed_act, const float* alpha, const float* b_pre, const float* b_res,
                            const float* b_post, void* input, int32_t* idx, float* p, float* Hpre, float* Hres,
                            float* Hpost, float* saved, void* ws, hipStream_t s) {
  const int G = team_size(d->C);
  const DeviceInfo di = device_info(d->C);
  if (di.cus <= 0 || di.per_cu <= 0) return hipErrorInvalidConfiguration;
  int teams = di.cus * di.per_cu / G;
  if (teams < 1) return hipErrorInvalidConfiguration;
  // (a team without a tile would only be launched and have records cleared)
  if (teams > max_teams(d)) teams = (int)max_teams(d);
  char* w = reinterpret_cast<char*>(ws);
  FusedArgs a{};
  a.X = reinterpret_cast<const uint16_t*>(X);
  a.wfull = reinterpret_cast<const uint4*>(packed_full);
  a.colsum = colsum;
  a.wact = reinterpret_cast<const uint4*>(packed_act);
  a.act_grouped = act_grouped(d->state_dtype, d->C) ? 1 : 0;
  a.alpha = alpha;
  a.b_pre = b_pre;
  a.input = reinterpret_cast<uint16_t*>(input);
  a.idx = idx;
  a.p = p;
  a.Hpre = Hpre;
  a.saved = saved;
  a.nsave = saved_floats(FN, FK, d->Kr);
  a.err = reinterpret_cast<int*>(w);
  static const ProcessQueues queues = process_queues();
  const bool plain = plain_launch<StreamApi>(G, di.cus, di.per_cu, queues, s);
  a.ticket = plain ? reinterpret_cast<int*>(w + 128) : nullptr;
  a.rec1 = reinterpret_cast<uint64_t*>(w + 256);
  a.rec2 = reinterpret_cast<uint64_t*>(w + 256 + align256(rec1_words(d) * 8));
  a.part2 = reinterpret_cast<float*>(w + 256 + align256(rec1_words(d) * 8) + align256(rec2_words(d) * 8));
  float* sums = a.part2 + align256((size_t)G * NV1 * d->T * sizeof(float)) / sizeof(float);
  a.T = d->T;
  a.C = d->C;
  a.teams = teams;
  a.m = d->m;
  a.eps = d->eps;
  a.softmax = d->router == XHC_ROUTER_SOFTMAX ? 1 : 0;
  // records start untagged: clear the error counter and the ticket (the first
  // 256 bytes) and the record slots in use, both whole 16-byte words
  const size_t used1 = (size_t)teams * RING * G * FM * NV1, used2 = (size_t)teams * RING * FM * NV2;
  const int64_t n1 = (int64_t)((256 + used1 * 8) / 16), n2 = (int64_t)((used2 * 8 + 15) / 16);
  k_zero2<<<dim3((unsigned)((n1 + n2 + 255) / 256)), dim3(256), 0, s>>>(reinterpret_cast<uint4*>(w), n1,
                                                                        reinterpret_cast<uint4*>(a.rec2), n2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  void* args[] = {&a};
  const void* f = fused_kernel(d->C);
  e = plain ? hipLaunchKernel(f, dim3(teams * G), dim3(FNT), args, kTileLds, s)
            : hipLaunchCooperativeKernel(f, dim3(teams * G), dim3(FNT), args, kTileLds, s);
  if (e != hipSuccess) return e;
  const PreRedo redo{a.err, a.X, a.wfull, a.wact, a.act_grouped, colsum, alpha, b_pre, a.input, idx, p, Hpre, d->C,
                     d->m, a.softmax};
  // active partials -> H^post, H^res (Sinkhorn + clamp); after failed waits every
  // output again
  return launch_pre_coef(a.part2, G, (int64_t)FK * d->Kr + FK * FK, d->T, FK, d->Kr, 1, d->C, alpha + 2, alpha + 1,
                         b_post, b_res, d->eps, d->sinkhorn_iters, d->clamp_delta, Hpost, Hres, sums, saved, a.nsave,
                         2 * FN, a.nsave - 2, s, &redo);
}

}  // namespace xhc
