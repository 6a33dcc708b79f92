// Mapping generation of an xHC sublayer (multi-kernel path): packing and the
// per-token finalisation of the projections.
//
//  k_pack / k_colsum   fp32 weights -> bf16 MFMA fragments; column sums of bf16(W_r)
//  k_sum_chunks        per-token sums of the split-K partials
//  k_pre_route         per token: LayerNorm / RMSNorm corrections of the raw
//                      projection (eq:fused_normalized_projection), H^pre, routing
//  k_pre_coef          per token: RMS of the active state, H^post, H^res (Sinkhorn + clamp)
#include "xhc_device.h"
#include "xhc_launch.h"

namespace xhc {
// ----------------------------------------------------------------- packing

__global__ void k_pack(int64_t K, int nob, int ncols_a, const float* __restrict__ A, int ncols_b,
                       const float* __restrict__ B, int64_t b_count, int grouped, uint4* __restrict__ out) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nfrag = (K / 32) * nob;
  if (gid >= nfrag * kWave) return;
  const int lane = (int)(gid % kWave);
  const int64_t frag = gid / kWave;
  const int ob = (int)(frag % nob);
  const int64_t kb = frag / nob;
  const int col = ob * 16 + lane % 16;
  // grouped: fragment 4G + u, lane group g holds rows 128G + 32g + 8u .. +8
  const int64_t row0 = grouped ? (kb / 4) * 128 + (lane / 16) * 32 + (kb % 4) * 8 : kb * 32 + (lane / 16) * 8;
  const int64_t nb = (int64_t)ncols_b * b_count;
  float f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t row = row0 + e;
    float v = 0.f;
    if (col < ncols_a) {
      v = A[row * ncols_a + col];
    } else if (col - ncols_a < nb) {
      const int64_t q = (col - ncols_a) / ncols_b;
      const int cc = (col - ncols_a) % ncols_b;
      v = B[(q * K + row) * ncols_b + cc];
    }
    f[e] = v;
  }
  out[gid] = pack8(f);
}

__global__ void k_colsum(int64_t K, int ncols, const float* __restrict__ W, float* __restrict__ out) {
  __shared__ float red[256];
  const int col = blockIdx.x;
  float s = 0.f;
  for (int64_t r = threadIdx.x; r < K; r += 256) s += __uint_as_float(f2bf(W[r * ncols + col]) << 16);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[col] = red[0];
}

hipError_t launch_pack(int64_t K, int64_t nout, int ncols_a, const float* A, int ncols_b, const float* B,
                       int64_t b_count, bool grouped, void* packed, hipStream_t s) {
  const int nob = (int)out_blocks(nout);
  const int64_t threads = (K / 32) * nob * kWave;
  if (threads == 0) return hipSuccess;
  k_pack<<<dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s>>>(K, nob, ncols_a, A, ncols_b, B, b_count,
                                                                       grouped ? 1 : 0,
                                                                       reinterpret_cast<uint4*>(packed));
  return hipGetLastError();
}

hipError_t launch_colsum(int64_t K, int ncols, const float* W, float* out, hipStream_t s) {
  k_colsum<<<dim3(ncols), dim3(256), 0, s>>>(K, ncols, W, out);
  return hipGetLastError();
}

// ----------------------------------------------------------------- per-token finalisation

// sums[o][t] = sum over chunks of part[chunk][o][t] (chunk order fixed), one
// thread per (o, t); the loads of all chunks are issued before the adds.
template <int B>   // chunks loaded together
__global__ __launch_bounds__(256) void k_sum_chunks(const float* __restrict__ part, int64_t nchunk, int NO,
                                                    int64_t T, float* __restrict__ sums) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)NO * T) return;
  const int64_t stride = (int64_t)NO * T;
  float s = 0.f;
  for (int64_t c0 = 0; c0 < nchunk; c0 += B) {
    float v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) v[u] = (c0 + u < nchunk) ? part[(c0 + u) * stride + i] : 0.f;
#pragma unroll
    for (int u = 0; u < B; ++u) s += v[u];
  }
  sums[i] = s;
}

// Full-state projection sums -> router logits and npre pre-maps (one thread per token).
// z^r = (x W^r - mu colsum(W^r)) / sqrt(nu - mu^2 + eps),  z^pre = x W^pre / sqrt(nu + eps).
// NB: a bound of N (16, 32 or 64).  Each batch of a token's sums (the router
// logits, then each pre-map's logits) is loaded before any of it is used
// (clamped to row N - 1 past N), so a thread waits once per batch.
template <int NB>
__global__ __launch_bounds__(64) void k_pre_route(const float* __restrict__ sums, int NO, int64_t T, int N, int m,
                                                  int k, int npre, int64_t NC, const float* __restrict__ colsum,
                                                  const float* __restrict__ alpha_pre, int alpha_stride,
                                                  const float* __restrict__ b_pre, float eps,
                                                  int32_t* __restrict__ idx, float* __restrict__ p,
                                                  float* __restrict__ Hpre, float* __restrict__ saved,
                                                  int nsave, int save_stats_at, int softmax, int save_pre) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  float zr[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) zr[i] = sums[(int64_t)(i < N ? i : N - 1) * T + t];
  const float mu = sums[(int64_t)(NO - 2) * T + t] / (float)NC;
  const float nu = sums[(int64_t)(NO - 1) * T + t] / (float)NC;
  // save_pre < 0: one record per pre-map q at saved + q T nsave (router
  // logits and statistics in each)
  const int nrec = save_pre < 0 ? npre : 1;
  if (saved)
    for (int r = 0; r < nrec; ++r) {
      saved[(r * T + t) * nsave + save_stats_at] = mu;
      saved[(r * T + t) * nsave + save_stats_at + 1] = nu;
    }
  const float r_ln = 1.0f / sqrtf(ln_variance(mu, nu) + eps);
  const float r_rms = 1.0f / sqrtf(nu + eps);
  float z[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) z[i] = (i < N) ? (zr[i] - mu * colsum[i < N ? i : 0]) * r_ln : 0.f;
  int32_t id[kMaxK];
  float pp[kMaxK];
  route_token<NB>(z, N, m, k, id, pp, softmax != 0);
  for (int j = 0; j < k; ++j) {
    idx[t * k + j] = id[j];
    p[t * k + j] = pp[j];
  }
  if (saved)
    for (int r = 0; r < nrec; ++r)
      for (int i = 0; i < N; ++i) saved[(r * T + t) * nsave + i] = z[i];
  for (int q = 0; q < npre; ++q) {
    const float a = alpha_pre[q * alpha_stride];
#pragma unroll
    for (int i = 0; i < NB; ++i) zr[i] = sums[(int64_t)(N + q * N + (i < N ? i : N - 1)) * T + t];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (i >= N) break;
      const float zp = zr[i] * r_rms;
      if (saved && save_pre < 0) saved[((int64_t)q * T + t) * nsave + N + i] = zp;
      else if (saved && q == save_pre) saved[t * nsave + N + i] = zp;
      Hpre[((int64_t)q * T + t) * N + i] = sigmoidf(a * zp + b_pre[q * N + i]);
    }
  }
}

// Active projection sums -> H^post = 2 sigma(.) and (with_res) H^res = clamp(SK(exp(.))).
__global__ __launch_bounds__(128) void k_pre_coef(const float* __restrict__ sums, int NO, int64_t T, int k, int Kq,
                                                  int with_res, int64_t kC, const float* __restrict__ alpha_post,
                                                  const float* __restrict__ alpha_res,
                                                  const float* __restrict__ b_post,
                                                  const float* __restrict__ b_res, float eps, int iters,
                                                  float delta, float* __restrict__ Hpost,
                                                  float* __restrict__ Hres, float* __restrict__ saved, int nsave,
                                                  int save_z_at, int save_stats_at) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const float nu_a = sums[(int64_t)(NO - 1) * T + t] / (float)kC;
  const float rstd = 1.0f / sqrtf(nu_a + eps);
  if (saved) {
    saved[t * nsave + save_stats_at] = nu_a;
    for (int o = 0; o < k * Kq + (with_res ? k * k : 0); ++o)
      saved[t * nsave + save_z_at + o] = sums[(int64_t)o * T + t] * rstd;
  }
  const float ap = alpha_post[0];
  for (int o = 0; o < k * Kq; ++o)
    Hpost[t * k * Kq + o] = 2.0f * sigmoidf(ap * (sums[(int64_t)o * T + t] * rstd) + b_post[o]);
  if (!with_res) return;
  const float ar = alpha_res[0];
  float M[kMaxK * kMaxK];
#pragma unroll
  for (int j = 0; j < kMaxK; ++j)
#pragma unroll
    for (int l = 0; l < kMaxK; ++l)
      M[j * kMaxK + l] = (j < k && l < k)
          ? ar * (sums[(int64_t)(k * Kq + j * k + l) * T + t] * rstd) + b_res[j * k + l] : 0.f;
  sinkhorn_clamp(M, k, iters, delta);
  for (int j = 0; j < k; ++j)
    for (int l = 0; l < k; ++l) Hres[(t * k + j) * k + l] = M[j * kMaxK + l];
}

// k = 2 and 4: the chunk sums of the active projection and the coefficients
// in one launch.  A workgroup takes 32 tokens (128 contiguous bytes of each
// output's row of partials); thread (part h, token u) sums chunk range h of
// token u (8 ranges), the ranges are added in order through LDS, and 16 lanes
// per token form the coefficients, an element of H^res each (with one thread
// per token the Sinkhorn iterations were a chain of 8 us at any T).
constexpr int kCoefTok = 32, kCoefParts = 8;   // tokens per workgroup, chunk ranges per token

// Everything xhc_pre has for token t, formed by a workgroup without the partials of
// the single pass: the full-state projection (a thread takes 8 consecutive rows
// K at a time, all 32 outputs), routing and H^pre, the dense read, then the
// active projection, whose sums go to act[o pitch] (o < 32) and act[32 pitch]
// (the square sum).  Reached only after a wait that gave up, so that a launch
// whose teams could not all run still ends in the right results; not fast (C =
// 4096: T = 16 2.7 ms, T = 16384 10 ms, against 36 and 605 us of the call), and at
// no cost where the count is zero, in registers and time.
constexpr int kRedoThreads = kCoefTok * kCoefParts;
struct RedoLds {
  float wave[kRedoThreads / kWave][34], tot[34], hpre[16];
  int32_t id[4];
};
__device__ __forceinline__ void redo_token(const PreRedo& r, int64_t t, float eps, float* saved, int nsave,
                                           RedoLds& s, float* act, int pitch) {
  constexpr int N = 16, k = 4, NO = 32;
  const int C = r.C, tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const uint16_t* x = r.X + t * N * C;
#pragma nounroll
  for (int ph = 0; ph < 2; ++ph) {   // the state's rows, then the routed ones
    const uint4* w = ph == 0 ? r.wfull : r.wact;
    const bool grouped = ph == 0 || r.act_grouped;
    float acc[NO + 2];
#pragma unroll
    for (int o = 0; o < NO + 2; ++o) acc[o] = 0.f;
    for (int K = tid * 8; K < (ph == 0 ? N : k) * C; K += kRedoThreads * 8) {
      const int j = K / C, c = K - j * C;
      float f[8];
      unpack8(*reinterpret_cast<const uint4*>(x + (int64_t)(ph == 0 ? j : s.id[j]) * C + c), f);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        acc[NO] += f[e];
        acc[NO + 1] += f[e] * f[e];
      }
      const int64_t kb = grouped ? (K >> 7) * 4 + ((K & 31) >> 3) : K >> 5;
      const int g = (grouped ? (K & 127) >> 5 : (K & 31) >> 3) * 16;
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        float wv[8];
        unpack8(w[(kb * 2 + o / 16) * kWave + g + o % 16], wv);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[o] = fmaf(f[e], wv[e], acc[o]);
      }
    }
#pragma unroll
    for (int o = 0; o < NO + 2; ++o) {
      const float v = wave_sum(acc[o]);
      if (lane == 0) s.wave[wave][o] = v;
    }
    __syncthreads();
    if (tid < NO + 2) {
      float v = 0.f;
#pragma unroll
      for (int q = 0; q < kRedoThreads / kWave; ++q) v += s.wave[q][tid];
      if (ph == 0) s.tot[tid] = v;
      else if (tid != NO) act[(tid < NO ? tid : NO) * pitch] = v;
    }
    __syncthreads();
    if (ph == 1) return;
    if (tid == 0) {
      const float NC = (float)N * (float)C, mu = s.tot[NO] / NC, nu = s.tot[NO + 1] / NC;
      const float r_ln = 1.0f / sqrtf(ln_variance(mu, nu) + eps), r_rms = 1.0f / sqrtf(nu + eps);
      float z[N], pp[kMaxK];
      int32_t id[kMaxK];
#pragma unroll
      for (int i = 0; i < N; ++i) z[i] = (s.tot[i] - mu * r.colsum[i]) * r_ln;
      route_token<N>(z, N, r.m, k, id, pp, r.softmax != 0);
      for (int j = 0; j < k; ++j) {
        s.id[j] = r.idx[t * k + j] = id[j];
        r.p[t * k + j] = pp[j];
      }
      float* sv = saved ? saved + t * nsave : nullptr;
      for (int i = 0; i < N; ++i) {
        const float zp = s.tot[N + i] * r_rms;
        s.hpre[i] = r.Hpre[t * N + i] = sigmoidf(r.alpha_pre[0] * zp + r.b_pre[i]);
        if (sv) sv[N + i] = zp;
      }
      if (sv) {
#pragma unroll
        for (int i = 0; i < N; ++i) sv[i] = z[i];
        sv[nsave - 4] = mu;
        sv[nsave - 3] = nu;
      }
    }
    __syncthreads();
    for (int c = tid * 8; c < C; c += kRedoThreads * 8) {
      float in[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int i = 0; i < N; ++i) {
        float f[8];
        unpack8(*reinterpret_cast<const uint4*>(x + (int64_t)i * C + c), f);
        const float h = s.hpre[i];
#pragma unroll
        for (int e = 0; e < 8; ++e) in[e] = fmaf(h, f[e], in[e]);
      }
      *reinterpret_cast<uint4*>(r.input + t * C + c) = pack8(in);
    }
  }
}

// SINGLE: behind a single pass, which may have failed.
template <int K, bool SINGLE>
__global__ __launch_bounds__(kCoefTok * kCoefParts) void k_pre_coef_sum(
    const float* __restrict__ part, int64_t nchunk, int NO, int64_t T, int Kq, int with_res, int64_t kC,
    const float* __restrict__ alpha_post, const float* __restrict__ alpha_res, const float* __restrict__ b_post,
    const float* __restrict__ b_res, float eps, int iters, float delta, float* __restrict__ Hpost,
    float* __restrict__ Hres, float* __restrict__ saved, int nsave, int save_z_at, int save_stats_at,
    PreRedo redo) {
  constexpr int NA = K * kMaxKr + K * K;   // outputs kept (at most)
  constexpr int GL = mix_lanes(K), NT = kCoefTok * kCoefParts;
  static_assert(NA <= 2 * GL && K * kMaxKr <= GL && K * K <= GL, "a lane keeps two outputs at most");
  __shared__ float red[kCoefParts][NA + 1][kCoefTok];
  const int nproj = K * Kq + (with_res ? K * K : 0);
  const int64_t tb = (int64_t)blockIdx.x * kCoefTok;
  {
    const int u = threadIdx.x % kCoefTok, h = threadIdx.x / kCoefTok;
    const int64_t t = tb + u;
    float acc[NA + 1];
#pragma unroll
    for (int o = 0; o <= NA; ++o) acc[o] = 0.f;
    const int64_t per = (nchunk + kCoefParts - 1) / kCoefParts;
    const int64_t c0 = h * per, c1 = (c0 + per < nchunk) ? c0 + per : nchunk;
    if (t < T) {
      const int64_t stride = (int64_t)NO * T;
      for (int64_t c = c0; c < c1; ++c) {
        const float* pc = part + c * stride + t;
        float v[NA + 1];
#pragma unroll
        for (int o = 0; o < NA; ++o) v[o] = o < nproj ? pc[(int64_t)o * T] : 0.f;
        v[NA] = pc[(int64_t)(NO - 1) * T];
#pragma unroll
        for (int o = 0; o <= NA; ++o) acc[o] += v[o];
      }
    }
#pragma unroll
    for (int o = 0; o <= NA; ++o) red[h][o][u] = acc[o];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < (NA + 1) * kCoefTok; i += NT) {
    float* r0 = &red[0][0][0] + i;
    float v = r0[0];
#pragma unroll
    for (int q = 1; q < kCoefParts; ++q) v += r0[q * (NA + 1) * kCoefTok];
    r0[0] = v;
  }
  __syncthreads();
  if constexpr (SINGLE) {
    // after failed waits the partials are not valid, and the single pass's own
    // outputs were formed from records that had not come
    __shared__ RedoLds rs;
    if (*redo.err != 0) {
      for (int u = 0; u < kCoefTok && tb + u < T; ++u)
        redo_token(redo, tb + u, eps, saved, nsave, rs, &red[0][0][u], kCoefTok);
      __syncthreads();
    }
  }
  const float ap = alpha_post[0], ar = with_res ? alpha_res[0] : 0.f;
  const int e = threadIdx.x % GL;
  for (int u = threadIdx.x / GL; u < kCoefTok; u += NT / GL) {   // (the same number of turns in every lane)
    const int64_t t = tb + u;
    const bool in = t < T;
    const float nu_a = red[0][NA][u] / (float)kC;
    const float rstd = 1.0f / sqrtf(nu_a + eps);
    if (saved && in) {
      if (e == 0) saved[t * nsave + save_stats_at] = nu_a;
#pragma unroll
      for (int o = e; o < NA; o += GL)
        if (o < nproj) saved[t * nsave + save_z_at + o] = red[0][o][u] * rstd;
    }
    if (e < K * Kq && in)
      Hpost[t * K * Kq + e] = 2.0f * sigmoidf(ap * (red[0][e][u] * rstd) + b_post[e]);
    if (!with_res) continue;
    // the W_res outputs follow the K Kq W_post outputs
    const bool used = e < K * K;
    const int er = used ? e : 0;
    const float M = sinkhorn_clamp_lanes<K>(ar * (red[0][K * Kq + er][u] * rstd) + b_res[er], used, iters, delta);
    if (used && in) Hres[t * K * K + e] = M;
  }
}

static hipError_t sum_chunks(const float* part, int64_t nchunk, int NO, int64_t T, float* sums, hipStream_t s) {
  const int64_t n = (int64_t)NO * T;
  const dim3 g((unsigned)((n + 255) / 256));
  if (nchunk <= 8) k_sum_chunks<8><<<g, dim3(256), 0, s>>>(part, nchunk, NO, T, sums);
  else k_sum_chunks<16><<<g, dim3(256), 0, s>>>(part, nchunk, NO, T, sums);
  return hipGetLastError();
}

hipError_t launch_pre_route(const float* part, int64_t nchunk, int64_t nout, int64_t T, int N, int m, int k,
                            int npre, int64_t C, const float* colsum, const float* alpha_pre, int alpha_stride,
                            const float* b_pre, float eps, int32_t* idx, float* p, float* Hpre, float* sums,
                            float* saved, int nsave, int save_stats_at, int router, hipStream_t s, int save_pre) {
  if (T == 0) return hipSuccess;
  const int NO = (int)out_blocks(nout) * 16 + 2;
  hipError_t e = sum_chunks(part, nchunk, NO, T, sums, s);
  if (e != hipSuccess) return e;
#define XHC_ROUTE(NBV)                                                                                      \
  k_pre_route<NBV><<<dim3((unsigned)((T + 63) / 64)), dim3(64), 0, s>>>(                                     \
      sums, NO, T, N, m, k, npre, (int64_t)N * C, colsum, alpha_pre, alpha_stride, b_pre, eps, idx, p, Hpre, \
      saved, nsave, save_stats_at, router == XHC_ROUTER_SOFTMAX ? 1 : 0, save_pre)
  if (N <= 16) XHC_ROUTE(16);
  else if (N <= 32) XHC_ROUTE(32);
  else XHC_ROUTE(kMaxN);
#undef XHC_ROUTE
  return hipGetLastError();
}

hipError_t launch_pre_coef(const float* part, int64_t nchunk, int64_t nout, int64_t T, int k, int Kq,
                           int with_res, int64_t C, const float* alpha_post, const float* alpha_res,
                           const float* b_post, const float* b_res, float eps, int iters, float delta,
                           float* Hpost, float* Hres, float* sums, float* saved, int nsave, int save_z_at,
                           int save_stats_at, hipStream_t s, const PreRedo* redo) {
  if (T == 0) return hipSuccess;
  const int NO = (int)out_blocks(nout) * 16 + 2;
  if ((k == 2 || k == 4) && Kq <= kMaxKr) {
    const dim3 g((unsigned)((T + kCoefTok - 1) / kCoefTok)), b(kCoefTok * kCoefParts);
#define XHC_COEF(KV, SINGLE)                                                                                      \
  k_pre_coef_sum<KV, SINGLE><<<g, b, 0, s>>>(part, nchunk, NO, T, Kq, with_res, (int64_t)k * C, alpha_post, alpha_res,      \
                                     b_post, b_res, eps, iters, delta, Hpost, Hres, saved, nsave, save_z_at,       \
                                     save_stats_at, redo ? *redo : PreRedo{})
    if (redo && (k != 4 || out_blocks(nout) != 2)) return hipErrorInvalidValue;   // (the single pass's shape)
    if (redo) XHC_COEF(4, true);
    else if (k == 4) XHC_COEF(4, false);
    else XHC_COEF(2, false);
#undef XHC_COEF
    return hipGetLastError();
  }
  if (redo) return hipErrorInvalidValue;
  hipError_t e = sum_chunks(part, nchunk, NO, T, sums, s);
  if (e != hipSuccess) return e;
  k_pre_coef<<<dim3((unsigned)((T + 127) / 128)), dim3(128), 0, s>>>(
      sums, NO, T, k, Kq, with_res, (int64_t)k * C, alpha_post, alpha_res, b_post, b_res, eps, iters, delta,
      Hpost, Hres, saved, nsave, save_z_at, save_stats_at);
  return hipGetLastError();
}

}  // namespace xhc
