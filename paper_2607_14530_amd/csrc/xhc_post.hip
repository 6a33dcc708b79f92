// Sparse write-back of an xHC sublayer (eq:aug, eq:gs, eq:sparse_write_delta,
// eq:sparse_write).
//
//  k_post_gram   MLP-type only: per token and channel chunk, the Gram matrix of
//                the components e_0 = out, e_j = DWConv_kappa_j(out) (fp32)
//  k_post_coef   per token: Gram-Schmidt in the component basis folded with p
//                and H^post into write-back weights wb[t][j][b]
//  k_post_apply  X[t, I_j, :] <- sum_l H^res[j,l] X[t, I_l, :] + sum_b wb[j][b] e_b;
//                the other N - k rows are never touched
#include "xhc_conv.h"
#include "xhc_device.h"
#include "xhc_launch.h"

namespace xhc {

// Gram partials: gpart[chunk][pair][t], pairs (a <= b) in row-major upper order.
template <typename TS, int KR>
__global__ __launch_bounds__(256) void k_post_gram(const TS* __restrict__ F, int64_t T, int64_t S, int C,
                                                   int kap0, int kap1, int kap2, const float* __restrict__ conv_w,
                                                   float* __restrict__ gpart) {
  constexpr int NP = KR * (KR + 1) / 2;
  __shared__ float red[4][NP];
  const int64_t ncb = post_chunks(C);
  const int64_t t = blockIdx.x / ncb;
  const int64_t cb = blockIdx.x % ncb;
  const int c = (int)(cb * 256 + threadIdx.x) * 8;
  const int kap[3] = {kap0, kap1, kap2};
  float g[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) g[i] = 0.f;
  if (c < C) {
    float e[KR][8];
    components<TS, KR>(F, conv_w, t, t % S, C, c, kap, e);
    int pi = 0;
#pragma unroll
    for (int a = 0; a < KR; ++a)
#pragma unroll
      for (int b = a; b < KR; ++b, ++pi)
#pragma unroll
        for (int q = 0; q < 8; ++q) g[pi] = fmaf(e[a][q], e[b][q], g[pi]);
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    float v = g[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    g[i] = v;
  }
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < NP; ++i) red[wave][i] = g[i];
  __syncthreads();
  if ((int)threadIdx.x < NP) {
    const int i = threadIdx.x;
    gpart[(cb * NP + i) * T + t] = red[0][i] + red[1][i] + red[2][i] + red[3][i];
  }
}


// Per token: G = sum over chunks; v_r = sum_b V[r][b] e_b (Gram-Schmidt, eq:gs);
// wb[j][b] = p_j sum_r H^post[j][r] V[r][b]  (p gates only the write-back term).
// out[j * Kr + b] receives token t's weights.
__device__ __forceinline__ void post_coef_token(const float* __restrict__ gpart, int64_t nchunk, int64_t T, int64_t t,
                                                int k, int Kr, int gram_schmidt, const float* __restrict__ p,
                                                const float* __restrict__ Hpost, float* __restrict__ out) {
  const int NP = Kr * (Kr + 1) / 2;
  // the chunk sums of every pair (a <= b < Kr: pair a Kr - a (a - 1) / 2 +
  // b - a in row-major upper order), each chunk's pairs loaded together (an
  // unused pair reads pair 0), summed in the order chunk 0, 1, ...
  float gs[kMaxKr][kMaxKr];
#pragma unroll
  for (int a = 0; a < kMaxKr; ++a)
#pragma unroll
    for (int b = 0; b < kMaxKr; ++b) gs[a][b] = 0.f;
  for (int64_t c = 0; c < nchunk; ++c) {
    float v[kMaxKr][kMaxKr];
#pragma unroll
    for (int a = 0; a < kMaxKr; ++a)
#pragma unroll
      for (int b = a; b < kMaxKr; ++b) {
        const int pab = (a < Kr && b < Kr) ? a * Kr - a * (a - 1) / 2 + (b - a) : 0;
        v[a][b] = gpart[(c * NP + pab) * T + t];
      }
#pragma unroll
    for (int a = 0; a < kMaxKr; ++a)
#pragma unroll
      for (int b = a; b < kMaxKr; ++b) gs[a][b] += v[a][b];
  }
  double G[kMaxKr][kMaxKr];
#pragma unroll
  for (int a = 0; a < kMaxKr; ++a)
#pragma unroll
    for (int b = a; b < kMaxKr; ++b) G[a][b] = G[b][a] = (a < Kr && b < Kr) ? (double)gs[a][b] : 0.0;
  double V[kMaxKr][kMaxKr];
  if (gram_schmidt) {
    gram_schmidt_basis(G, Kr, V);
  } else {
#pragma unroll
    for (int i = 0; i < kMaxKr; ++i)
#pragma unroll
      for (int b = 0; b < kMaxKr; ++b) V[i][b] = (i == b) ? 1.0 : 0.0;
  }
  for (int j = 0; j < k; ++j) {
    const double pj = p[t * k + j];
    for (int b = 0; b < Kr; ++b) {
      double s = 0.0;
      for (int r = 0; r < Kr; ++r) s += (double)Hpost[(t * k + j) * Kr + r] * V[r][b];
      out[j * Kr + b] = (float)(pj * s);
    }
  }
}

__global__ __launch_bounds__(128) void k_post_coef(const float* __restrict__ gpart, int64_t nchunk, int64_t T,
                                                   int k, int Kr, int gram_schmidt, const float* __restrict__ p,
                                                   const float* __restrict__ Hpost, float* __restrict__ wb) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  post_coef_token(gpart, nchunk, T, t, k, Kr, gram_schmidt, p, Hpost, wb + t * k * Kr);
}

// ------------------------------------------------------------------ run-based MLP-type kernels
// For compile-time kernel sizes (K1, K2, K3) = (4, 8, 12): a thread owns 4
// channels and walks a run of up to kRun consecutive tokens in groups of G,
// keeping the conv taps of its channels and the last 12 values of F in
// registers, so F is read once per kernel and the taps once per run.  Where a
// sequence starts the history is cleared: FIT: starts fall on group starts, the
// runs cut all tokens alike and the width in whole workgroups.  SPLIT: the same
// for the starts (or no run crosses one), but the last group may be short and the
// threads past the width work on zeros.  CROSS: starts fall anywhere.

constexpr int kRun = 64;   // tokens of a run, at most
enum RunMode { FIT, SPLIT, CROSS };

// Sequences this short, and no multiple of a group, are crossed; longer ones are
// cut each from its start.  A cut costs its run the set-up again, a crossing
// the clearing of the history (60 registers) in an instance that carries it at
// every token.  T = 8192, k = 4, cut / crossed: C = 4096 S = 2 490 / 220 us, S = 7
// 267 / 216, S = 33 196 / 210, S = 1541 188 / 218; C = 2112 S = 2 295 / 155, S = 7
// 147 / 150, S = 31 134 / 149.
constexpr int kCrossed = 8;

// the runs of a launch: units of consecutive tokens, cut into runs of rl
struct Runs {
  int64_t T, S;
  int64_t unit, rpu;   // tokens and runs of a unit
  int rl;
  __device__ __forceinline__ int64_t first(int64_t b) const { return b / rpu * unit + b % rpu * rl; }
  __device__ __forceinline__ int count(int64_t b) const {
    const int64_t t0 = first(b), next = (b / rpu + 1) * unit;
    return (int)(next - t0 < rl ? next - t0 : rl);
  }
  // tokens from t to the next sequence start after it (at most 2^30: no run is longer)
  __device__ __forceinline__ int left(int64_t t) const {
    const int64_t n = S - t % S;
    return n < (1 << 30) ? (int)n : 1 << 30;
  }
};

// Tokens per run.  A run's workgroup walks its tokens one group after the
// other, so its time is about that of its tokens in sequence; with fewer
// workgroups than the chip holds (two per CU at these register counts, 512)
// shorter runs finish sooner, until the set-up (24 taps and 12 rows of
// history a channel) is as long as the walk: 4 tokens, one group.  Sequences of
// whole groups are no matter to the cut (each cut from its start, T = 8192 k = 4
// C = 4096: S = 8 222 us against 166, S = 100 221 against 166).
static Runs make_runs(int64_t T, int64_t S, int64_t chunks, int64_t* nruns) {
  const int64_t unit = S % 4 == 0 || S < kCrossed ? T : S;   // (T is a multiple of S)
  int rl = kRun;
  while (rl > 4 && T / unit * ((unit + rl - 1) / rl) * chunks < 512) rl /= 2;
  const Runs r{T, S, unit, (unit + rl - 1) / rl, rl};
  *nruns = T / unit * r.rpu;
  return r;
}
static RunMode run_mode(int64_t S, int C, int nthr) {
  if (S % 4 != 0) return S < kCrossed ? CROSS : SPLIT;
  return C % (4 * nthr) != 0 ? SPLIT : FIT;
}

// Clears what precedes token g of a group where a sequence starts there: the
// history, and the group's earlier tokens, which have been used; the shift at
// the group's end then puts the zeros where the history has them.  left counts
// the tokens to the next start, from 0 where token g is one.
template <typename CG, int G>
__device__ __forceinline__ void start_at(CG& cg, float (&cur)[G][4], int g, int seq, int& left) {
  if (left == 0) {
    cg.reset();
#pragma unroll
    for (int h = 0; h < G; ++h)
      if (h < g) cur[h][0] = cur[h][1] = cur[h][2] = cur[h][3] = 0.f;
    left = seq;
  }
  --left;
}

// The same where starts fall on group starts.
template <typename CG>
__device__ __forceinline__ void start_at_group(CG& cg, int G, int seq, int& left) {
  if (left == 0) {
    cg.reset();
    left = seq;
  }
  left -= G;
}

// Gram partials per workgroup's channels.  Each lane forms its 4-channel
// products for G tokens; a wave sums them over its 64 lanes through an LDS
// transpose (lane v adds column v), and the waves' sums are added at the end.
template <typename TS, int K1, int K2, int K3, RunMode MODE>
__global__ __launch_bounds__(256) void k_post_gram_run(const TS* __restrict__ F, Runs runs, int C,
                                                       const float* __restrict__ conv_w,
                                                       float* __restrict__ gpart) {
  using CG = ConvGroup<K1, K2, K3>;
  constexpr int KR = CG::KR, NP = KR * (KR + 1) / 2;
  constexpr int G = 4, NV = G * NP, LD = (NV + 3) / 4 * 4 + 4;
  static_assert(NV <= kWave, "one column per lane");
  __shared__ __align__(16) float xpose[4][kWave][LD];
  __shared__ float red[kRun][4][NP];
  const int nw = blockDim.x / kWave;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int64_t cb = blockIdx.y;
  const int64_t T = runs.T, t0 = runs.first(blockIdx.x);
  const int nt = runs.count(blockIdx.x);
  int c = (int)(cb * blockDim.x + threadIdx.x) * 4;
  const bool past = MODE != FIT && c >= C;   // (reads the last channels, counts as zeros)
  if (past) c = C - 4;
  CG cg;
  cg.load_taps(conv_w, C, c);
  cg.init(F, t0, runs.S, C, c);
  if (past) cg.reset();
  const int seq = runs.left(0);
  int left = runs.left(t0);
  float* mine = &xpose[wave][lane][0];
  // F rows are loaded PF groups ahead (a lane requests 8 bytes per token of a
  // bf16 state, so one group in flight would leave the memory system mostly
  // idle)
  constexpr int PF = sizeof(TS) == 2 ? 4 : 2;
  typename Row4<TS>::raw ring[PF][G];
#pragma unroll
  for (int f = 0; f < PF; ++f)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int u = f * G + g;
      ring[f][g] = u < nt ? Row4<TS>::load(F + (t0 + u) * C + c) : Row4<TS>::zero();
    }
  for (int u1 = 0; u1 < nt; u1 += PF * G) {
#pragma unroll
    for (int f = 0; f < PF; ++f) {
      const int u0 = u1 + f * G;
      if (u0 >= nt) break;
      if (MODE != CROSS) start_at_group(cg, G, seq, left);
      float cur[G][4];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        Row4<TS>::unpack(ring[f][g], cur[g]);
        if (past) cur[g][0] = cur[g][1] = cur[g][2] = cur[g][3] = 0.f;
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int u = u0 + PF * G + g;
        ring[f][g] = u < nt ? Row4<TS>::load(F + (t0 + u) * C + c) : Row4<TS>::zero();
      }
      float part[NV];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (MODE == CROSS) start_at(cg, cur, g, seq, left);
        float e[KR][4];
        cg.components(cur, g, e);
        int pi = 0;
#pragma unroll
        for (int a = 0; a < KR; ++a)
#pragma unroll
          for (int b = a; b < KR; ++b, ++pi) {
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) v = fmaf(e[a][q], e[b][q], v);
            part[g * NP + pi] = v;
          }
      }
      cg.advance(cur);
#pragma unroll
      for (int v = 0; v < NV; v += 4)
        *reinterpret_cast<float4*>(mine + v) =
            make_float4(part[v], v + 1 < NV ? part[v + 1 < NV ? v + 1 : 0] : 0.f,
                        v + 2 < NV ? part[v + 2 < NV ? v + 2 : 0] : 0.f,
                        v + 3 < NV ? part[v + 3 < NV ? v + 3 : 0] : 0.f);
      // LDS operations of one wave complete in issue order; the fences keep the
      // compiler from moving the column reads above the row writes (or the next
      // group's writes above these reads).
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (lane < NV) {
        float sum = 0.f;
#pragma unroll 16
        for (int r = 0; r < kWave; ++r) sum += xpose[wave][r][lane];
        const int g = lane / NP, pi = lane % NP;
        if (u0 + g < nt) red[u0 + g][wave][pi] = sum;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nt * NP; i += blockDim.x) {
    const int u = i / NP, pi = i % NP;
    float v = 0.f;
    for (int w = 0; w < nw; ++w) v += red[u][w][pi];
    gpart[(cb * NP + pi) * T + t0 + u] = v;
  }
}

// Write-back Y_j = sum_l H^res_jl a_l + sum_b wb_jb e_b for the KK active rows
// (without H^res: Y_j = a_j + ...); SAVE keeps the rows read, NEXT forms the
// next sublayer's input.  The run's indices and coefficients are staged in LDS
// once, the write-back weights wb formed there from the Gram partials; the
// loads of a group of G tokens are issued together.
template <typename TS, int KK, int G, bool RES, bool SAVE, bool NEXT, RunMode MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_post_apply_run(TS* __restrict__ X, const TS* __restrict__ F, Runs runs,
                                                        int N, int C,
                                                        const float* __restrict__ conv_w,
                                                        const int32_t* __restrict__ idx,
                                                        const float* __restrict__ Hres,
                                                        const float* __restrict__ gpart, int64_t nchunk,
                                                        int gram_schmidt, const float* __restrict__ p,
                                                        const float* __restrict__ Hpost,
                                                        const float* __restrict__ Hpre_next,
                                                        const TS* __restrict__ base_next, TS* __restrict__ input_next,
                                                        TS* __restrict__ Xact_save) {
  using CG = ConvGroup<4, 8, 12>;
  using R = Row4<TS>;
  constexpr int KR = CG::KR;
  __shared__ __align__(16) float s_hr[RES ? kRun * KK * KK : 4];
  __shared__ __align__(16) float s_wb[kRun * KK * KR];
  __shared__ int32_t s_idx[kRun * KK];
  __shared__ float s_hn[NEXT ? kRun * kMaxN : 1];
  const int64_t T = runs.T, t0 = runs.first(blockIdx.x);
  const int nt = runs.count(blockIdx.x);
  int c = (int)(blockIdx.y * blockDim.x + threadIdx.x) * 4;
  const bool past = MODE != FIT && c >= C;
  if (past) c = C - 4;
  for (int i = threadIdx.x; i < nt * KK; i += blockDim.x) s_idx[i] = idx[t0 * KK + i];
  // write-back weights of the run's tokens from their Gram partials (the same
  // per-token arithmetic as k_post_coef; every channel chunk of a run forms them)
  for (int u = threadIdx.x; u < nt; u += blockDim.x)
    post_coef_token(gpart, nchunk, T, t0 + u, KK, KR, gram_schmidt, p, Hpost, s_wb + u * KK * KR);
  if (RES)
    for (int i = threadIdx.x; i < nt * KK * KK; i += blockDim.x) s_hr[i] = Hres[t0 * KK * KK + i];
  if (NEXT)
    for (int i = threadIdx.x; i < nt * N; i += blockDim.x) s_hn[i] = Hpre_next[t0 * N + i];
  CG cg;
  cg.load_taps(conv_w, C, c);
  cg.init(F, t0, runs.S, C, c);
  __syncthreads();
  if (past) return;
  const int seq = runs.left(0);
  int left = runs.left(t0);
  for (int u0 = 0; u0 < nt; u0 += G) {
    // (the branch also ends the scheduler's region: without one here the
    // write-back spilled or took one wave a SIMD, 478 us against 336 at T =
    // 16384 C = 4096)
    if (MODE == FIT && (t0 + u0) % runs.S == 0) cg.reset();
    if (MODE == SPLIT) start_at_group(cg, G, seq, left);
    int32_t rows[G][KK];
    float cur[G][4];
    typename R::raw a[G][KK], nb[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int u = MODE == FIT || u0 + g < nt ? u0 + g : nt - 1;
#pragma unroll
      for (int l = 0; l < KK; ++l) rows[g][l] = __builtin_amdgcn_readfirstlane(s_idx[u * KK + l]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int64_t tg = t0 + (MODE == FIT || u0 + g < nt ? u0 + g : nt - 1);
      R::unpack(R::load(F + tg * C + c), cur[g]);
#pragma unroll
      for (int l = 0; l < KK; ++l) a[g][l] = R::load(X + (tg * N + rows[g][l]) * (int64_t)C + c);
      if (NEXT) nb[g] = R::load(base_next + tg * C + c);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (MODE != FIT && u0 + g >= nt) break;   // (past the run: read its last token)
      const int u = u0 + g;
      const int64_t tg = t0 + u;
      if (MODE == CROSS) start_at(cg, cur, g, seq, left);
      float e[KR][4];
      cg.components(cur, g, e);
      if (SAVE) {
#pragma unroll
        for (int l = 0; l < KK; ++l) R::store_raw(Xact_save + (tg * KK + l) * (int64_t)C + c, a[g][l]);
      }
      float af[KK][4];
#pragma unroll
      for (int l = 0; l < KK; ++l) R::unpack(a[g][l], af[l]);
      float nxt[4];
      if (NEXT) R::unpack(nb[g], nxt);
      const float* hr = s_hr + (RES ? u * KK * KK : 0);
      const float* wv = s_wb + u * KK * KR;
#pragma unroll
      for (int j = 0; j < KK; ++j) {
        float y[4];
        if (RES) {
#pragma unroll
          for (int q = 0; q < 4; ++q) y[q] = 0.f;
#pragma unroll
          for (int l = 0; l < KK; ++l) {
            const float h = hr[j * KK + l];
#pragma unroll
            for (int q = 0; q < 4; ++q) y[q] = fmaf(h, af[l][q], y[q]);
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) y[q] = af[j][q];
        }
#pragma unroll
        for (int b = 0; b < KR; ++b) {
          const float w = wv[j * KR + b];
#pragma unroll
          for (int q = 0; q < 4; ++q) y[q] = fmaf(w, e[b][q], y[q]);
        }
        R::store(X + (tg * N + rows[g][j]) * (int64_t)C + c, y);
        if (NEXT) {
          R::round(y);
          const float h = s_hn[u * N + rows[g][j]];
#pragma unroll
          for (int q = 0; q < 4; ++q) nxt[q] = fmaf(h, y[q], nxt[q]);
        }
      }
      if (NEXT) R::store(input_next + tg * C + c, nxt);
    }
    cg.advance(cur);
  }
}

// Threads per workgroup of the run-based kernels for width C (4 channels
// each): the count with the fewest threads past the width, the largest of
// equals (2112: 3 x 192 threads, 2560: 5 x 128, 4096: 4 x 256).
static int run_threads(int C) {
  int best = 0, waste = 0;
  for (int n = 256; n >= kWave; n -= kWave) {
    const int over = (C + 4 * n - 1) / (4 * n) * 4 * n - C;
    if (!best || over < waste) best = n, waste = over;
  }
  return best;
}
static int64_t run_chunks(int C) { return (C + 4 * run_threads(C) - 1) / (4 * run_threads(C)); }
static bool paper_branches(int Kr, const int32_t* kappa) {
  return Kr == 4 && kappa[0] == 4 && kappa[1] == 8 && kappa[2] == 12;
}
static size_t gram_floats(int64_t chunks, int Kr, int64_t T) { return (size_t)chunks * (Kr * (Kr + 1) / 2) * T; }
static size_t bytes256(size_t floats) { return (floats * sizeof(float) + 255) / 256 * 256; }

// The run kernels serve the paper's branches at k = 2, 4 and 8, any width and
// sequence length: at T = 6164, S = 1541, N = 8, C = 2112 a Flash group's four
// write-backs take 984 us with the per-token kernels, whose every token reads up
// to 12 rows of F and 24 rows of taps, and 581 us with these; k = 8, C = 1024, T =
// 8192, S = 1024 one write-back 140 and 67 us.  The other k keep the per-token
// write-back, with the run Gram where its partials fit what they need.
// So do many tokens in sequences of one to three, of which a token reads that
// many rows and taps only, where the width fills the per-token workgroups of
// 2048 channels (per token / run, T = 8192, k = 4: C = 4096 S = 1 203 / 223 us, S
// = 2 220 / 219, C = 6144 S = 3 304 / 359; T = 2048, C = 4096, S = 1 68 / 61).
// Where the caller's workspace (or the fixed scratch) holds the per-token
// kernels' partials and not these, the per-token kernels run.
PostPlan post_plan(int64_t T, int64_t S, int C, int k, int Kr, const int32_t* kappa, size_t avail) {
  PostPlan p{};
  if (Kr == 1) return p;
  const bool even = C % 1024 == 0 || C == 256 || C == 512 || C == 768;   // whole workgroups
  const bool exact = paper_branches(Kr, kappa) && even && S % 4 == 0;
  const bool few = S <= 3 && S <= C / 2048 && C % 2048 == 0 && k <= 4 && T * C >= (int64_t)1 << 24;
  const bool run = paper_branches(Kr, kappa) && C % 4 == 0 && (k == 2 || k == 4 || k == 8) && !few;
  const size_t wb = bytes256((size_t)T * k * Kr);
  const size_t per_run = bytes256(gram_floats(run_chunks(C), Kr, T));
  const size_t per_token = bytes256(gram_floats(post_chunks(C), Kr, T));
  p.least = (exact ? per_run : per_token) + wb;
  p.bytes = run && per_run > p.least ? per_run : p.least;
  p.apply_run = run && per_run <= avail;
  p.gram_run = p.apply_run || exact;
  p.nchunk = p.gram_run ? run_chunks(C) : post_chunks(C);
  p.wb_at = p.gram_run ? per_run : per_token;
  return p;
}

hipError_t launch_post_gram(const PostPlan& plan, int state_dtype, const void* F, int64_t T, int64_t S, int C, int Kr,
                            const int32_t* kappa, const float* conv_w, float* gpart, hipStream_t s) {
  if (T == 0) return hipSuccess;
  if (plan.gram_run) {
    int64_t nruns = 0;
    const Runs runs = make_runs(T, S, plan.nchunk, &nruns);
    const int nthr = run_threads(C);
    const dim3 grid((unsigned)nruns, (unsigned)plan.nchunk);
#define XHC_GRAM_RUN(TS, MODE) \
  k_post_gram_run<TS, 4, 8, 12, MODE><<<grid, dim3(nthr), 0, s>>>(reinterpret_cast<const TS*>(F), runs, C, conv_w, gpart)
#define XHC_GRAM_MODES(TS)                            \
  switch (run_mode(S, C, nthr)) {                     \
    case FIT: XHC_GRAM_RUN(TS, FIT); break;           \
    case SPLIT: XHC_GRAM_RUN(TS, SPLIT); break;       \
    case CROSS: XHC_GRAM_RUN(TS, CROSS); break;       \
  }
    if (state_dtype == XHC_BF16) XHC_GRAM_MODES(uint16_t) else XHC_GRAM_MODES(float)
#undef XHC_GRAM_MODES
#undef XHC_GRAM_RUN
    return hipGetLastError();
  }
  const dim3 grid((unsigned)(T * post_chunks(C)));
#define XHC_GRAM(TS, KR)                                                                                   \
  k_post_gram<TS, KR><<<grid, dim3(256), 0, s>>>(reinterpret_cast<const TS*>(F), T, S, C, kappa[0], kappa[1], \
                                                 kappa[2], conv_w, gpart)
  if (state_dtype == XHC_BF16) {
    if (Kr == 2) XHC_GRAM(uint16_t, 2); else if (Kr == 3) XHC_GRAM(uint16_t, 3); else XHC_GRAM(uint16_t, 4);
  } else {
    if (Kr == 2) XHC_GRAM(float, 2); else if (Kr == 3) XHC_GRAM(float, 3); else XHC_GRAM(float, 4);
  }
#undef XHC_GRAM
  return hipGetLastError();
}

static hipError_t launch_post_coef(const float* gpart, int64_t nchunk, int64_t T, int k, int Kr, int gram_schmidt,
                            const float* p, const float* Hpost, float* wb, hipStream_t s) {
  if (T == 0) return hipSuccess;
  k_post_coef<<<dim3((unsigned)((T + 127) / 128)), dim3(128), 0, s>>>(gpart, nchunk, T, k, Kr, gram_schmidt, p,
                                                                      Hpost, wb);
  return hipGetLastError();
}

// In-place update of the k active rows of one token, 8 channels per thread.
// All k rows are read before any is written; each thread owns its channels.
// Hres == nullptr means no residual mixing (an intermediate xHC-Flash
// sublayer, eq:flash_attn_update).  With input_next, the thread also forms
// the next sublayer's input from its non-active base and the active rows as
// stored (App. E.2, eq:app_active_state_correction).
template <typename TS, int KR>
__global__ __launch_bounds__(256) void k_post_apply(TS* __restrict__ X, const TS* __restrict__ F, int64_t T,
                                                    int64_t S, int N, int C, int k, int kap0, int kap1, int kap2,
                                                    const float* __restrict__ conv_w,
                                                    const int32_t* __restrict__ idx, const float* __restrict__ p,
                                                    const float* __restrict__ Hres,
                                                    const float* __restrict__ Hpost,
                                                    const float* __restrict__ wb,
                                                    const float* __restrict__ Hpre_next,
                                                    const TS* __restrict__ base_next,
                                                    TS* __restrict__ input_next, TS* __restrict__ Xact_save) {
  const int64_t ncb = post_chunks(C);
  const int64_t t = blockIdx.x / ncb;
  const int c = (int)((blockIdx.x % ncb) * 256 + threadIdx.x) * 8;
  if (c >= C) return;
  const int kap[3] = {kap0, kap1, kap2};
  // the token's routed rows (the same in every lane), then every row load,
  // issued before anything waits for one: the rows stay raw until used, and
  // the components (F) are formed while they are in flight
  int32_t rows[kMaxK];
#pragma unroll
  for (int l = 0; l < kMaxK; ++l) rows[l] = idx[t * k + (l < k ? l : 0)];
  typename Raw8<TS>::raw ar[kMaxK] = {}, nr = {};
#pragma unroll
  for (int l = 0; l < kMaxK; ++l)
    if (l < k) ar[l] = Raw8<TS>::load(X + (t * N + rows[l]) * (int64_t)C + c);
  if (input_next) nr = Raw8<TS>::load(base_next + t * C + c);
  float e[KR][8];
  components<TS, KR>(F, conv_w, t, t % S, C, c, kap, e);
  float a[kMaxK][8];
#pragma unroll
  for (int l = 0; l < kMaxK; ++l) {
    if (l < k) {
      Raw8<TS>::unpack(ar[l], a[l]);
      if (Xact_save) Raw8<TS>::store(Xact_save + (t * k + l) * (int64_t)C + c, ar[l]);
    }
  }
  float nxt[8];
  if (input_next) Raw8<TS>::unpack(nr, nxt);
#pragma unroll
  for (int j = 0; j < kMaxK; ++j) {
    if (j >= k) break;
    float y[8];
    if (Hres) {
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = 0.f;
#pragma unroll
      for (int l = 0; l < kMaxK; ++l) {
        if (l < k) {
          const float h = Hres[(t * k + j) * k + l];
#pragma unroll
          for (int q = 0; q < 8; ++q) y[q] = fmaf(h, a[l][q], y[q]);
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = a[j][q];
    }
#pragma unroll
    for (int b = 0; b < KR; ++b) {
      const float w = (KR == 1) ? p[t * k + j] * Hpost[t * k + j] : wb[(t * k + j) * KR + b];
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = fmaf(w, e[b][q], y[q]);
    }
    Vec8<TS>::store(X + (t * N + rows[j]) * (int64_t)C + c, y);
    if (input_next) {
      Vec8<TS>::round(y);
      const float h = Hpre_next[t * N + rows[j]];
#pragma unroll
      for (int q = 0; q < 8; ++q) nxt[q] = fmaf(h, y[q], nxt[q]);
    }
  }
  if (input_next) Vec8<TS>::store(input_next + t * C + c, nxt);
}

hipError_t launch_post_apply(const PostPlan& plan, int state_dtype, void* X, const void* F, int64_t T, int64_t S, int N,
                             int C, int k, int Kr, const int32_t* kappa, const float* conv_w, const int32_t* idx,
                             const float* p, const float* Hres, const float* Hpost, const float* gpart,
                             int gram_schmidt, float* wb, const float* Hpre_next, const void* base_next,
                             void* input_next, void* Xact_save, hipStream_t s) {
  if (T == 0) return hipSuccess;
  const int64_t nchunk = plan.nchunk;
  if (plan.apply_run && (Hres != nullptr) != (input_next != nullptr)) {
    int64_t nruns = 0;
    const Runs runs = make_runs(T, S, nchunk, &nruns);
    const int nthr = run_threads(C);
    const dim3 grid((unsigned)nruns, (unsigned)nchunk);
#define XHC_APPLY_RUN(TS, KK, G, RES, SAVE, NEXT, MODE)                                                           \
  k_post_apply_run<TS, KK, G, RES, SAVE, NEXT, MODE><<<grid, dim3(nthr), 0, s>>>(                               \
      reinterpret_cast<TS*>(X), reinterpret_cast<const TS*>(F), runs, N, C, conv_w, idx, Hres, gpart, nchunk,     \
      gram_schmidt, p, Hpost, Hpre_next, reinterpret_cast<const TS*>(base_next),                                 \
      reinterpret_cast<TS*>(input_next), reinterpret_cast<TS*>(Xact_save))
#define XHC_APPLY_FORMS(TS, KK, G, MODE)                                                    \
  do {                                                                                       \
    if (input_next && Xact_save) XHC_APPLY_RUN(TS, KK, G, false, true, true, MODE);         \
    else if (input_next) XHC_APPLY_RUN(TS, KK, G, false, false, true, MODE);                \
    else if (Xact_save) XHC_APPLY_RUN(TS, KK, G, true, true, false, MODE);                  \
    else XHC_APPLY_RUN(TS, KK, G, true, false, false, MODE);                                \
  } while (0)
#define XHC_APPLY_MODES(TS, KK, G)                    \
  switch (mode) {                                     \
    case FIT: XHC_APPLY_FORMS(TS, KK, G, FIT); break; \
    case SPLIT: XHC_APPLY_FORMS(TS, KK, G, SPLIT); break; \
    case CROSS: XHC_APPLY_FORMS(TS, KK, G, CROSS); break; \
  }
#define XHC_APPLY_MODES2(TS)                                                     \
  {                                                                              \
    if (mode == CROSS) XHC_APPLY_FORMS(TS, 2, 4, CROSS);                         \
    else XHC_APPLY_FORMS(TS, 2, 4, SPLIT);   /* (a fitting one runs in it) */    \
  }
    const RunMode mode = run_mode(S, C, nthr);
    if (state_dtype == XHC_BF16) {
      if (k == 2) XHC_APPLY_MODES2(uint16_t)
      else if (k == 8) XHC_APPLY_MODES(uint16_t, 8, 2)
      else XHC_APPLY_MODES(uint16_t, 4, 4)
    } else {
      if (k == 2) XHC_APPLY_MODES2(float)
      else if (k == 8) XHC_APPLY_MODES(float, 8, 1)
      else XHC_APPLY_MODES(float, 4, 2)
    }
#undef XHC_APPLY_MODES2
#undef XHC_APPLY_MODES
#undef XHC_APPLY_FORMS
#undef XHC_APPLY_RUN
    return hipGetLastError();
  }
  if (gpart) {
    const hipError_t e = launch_post_coef(gpart, nchunk, T, k, Kr, gram_schmidt, p, Hpost, wb, s);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)(T * post_chunks(C)));
#define XHC_APPLY(TS, KR)                                                                                       \
  k_post_apply<TS, KR><<<grid, dim3(256), 0, s>>>(reinterpret_cast<TS*>(X), reinterpret_cast<const TS*>(F), T, S, \
                                                  N, C, k, kappa[0], kappa[1], kappa[2], conv_w, idx, p, Hres,   \
                                                  Hpost, wb, Hpre_next, reinterpret_cast<const TS*>(base_next),  \
                                                  reinterpret_cast<TS*>(input_next), reinterpret_cast<TS*>(Xact_save))
  if (state_dtype == XHC_BF16) {
    switch (Kr) {
      case 1: XHC_APPLY(uint16_t, 1); break;
      case 2: XHC_APPLY(uint16_t, 2); break;
      case 3: XHC_APPLY(uint16_t, 3); break;
      default: XHC_APPLY(uint16_t, 4); break;
    }
  } else {
    switch (Kr) {
      case 1: XHC_APPLY(float, 1); break;
      case 2: XHC_APPLY(float, 2); break;
      case 3: XHC_APPLY(float, 3); break;
      default: XHC_APPLY(float, 4); break;
    }
  }
#undef XHC_APPLY
  return hipGetLastError();
}

}  // namespace xhc
