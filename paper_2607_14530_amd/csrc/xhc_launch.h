// Internal launchers of the xHC kernels (host side).  Every launcher enqueues
// on `stream` and returns hipSuccess or the first launch error.  Shapes have
// been validated by the C-ABI layer before any launcher is called.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xhc.h"

namespace xhc {

constexpr int kWave = 64;
constexpr int kMaxN = 64;   // streams
constexpr int kMaxK = 8;    // active streams
constexpr int kMaxKr = 4;   // write-back components

// packed projection layout: fragments of 64 lanes x 8 bf16 (1 KiB), indexed
// [k_block (32 rows)][out_block (16 columns)][lane]; lane l of fragment
// (kb, ob) holds W[kb*32 + 8*(l/16) + e][ob*16 + l%16], e = 0..7.  Grouped
// layout (full-state weights of a bf16 state, K % 128 == 0): fragment
// 4G + u holds rows 128G + 32*(l/16) + 8u + e instead, so that a lane's four
// consecutive fragments of a group meet 64 contiguous state bytes.
inline bool full_grouped(int state_dtype, int64_t K) { return state_dtype == XHC_BF16 && K % 128 == 0; }
// the same for the active-state weights (K = k C, gathered rows): groups must
// not straddle two rows
inline bool act_grouped(int state_dtype, int C) { return state_dtype == XHC_BF16 && C % 128 == 0; }
__host__ __device__ inline int64_t out_blocks(int64_t nout) { return (nout + 15) / 16; }
inline size_t packed_frag_bytes(int64_t K, int64_t nout) { return (size_t)(K / 32) * out_blocks(nout) * 1024; }
constexpr size_t kColsumBytes = 64 * sizeof(float);

hipError_t launch_pack(int64_t K, int64_t nout, int ncols_a, const float* A, int ncols_b, const float* B,
                       int64_t b_count, bool grouped, void* packed, hipStream_t s);
hipError_t launch_colsum(int64_t K, int ncols, const float* W, float* out, hipStream_t s);

// ---- pre (multi-kernel path)
constexpr int kProjTile = 16;    // tokens per MFMA column group

// Launch plan of the split-K projection.  Wide path (bf16 state, grouped
// weight layout, full or gathered rows): 256-token workgroups, 4 consecutive
// k-blocks per step, weight fragments shared through LDS.  Other cases: each wave multiplies tg token groups of
// 16 by the same weight fragment.  A workgroup covers chunk_blocks 32-row
// blocks of K; nchunk partials are summed per token afterwards.
struct ProjPlan {
  bool wide;
  int tg;
  int64_t chunk_blocks;
  int64_t nchunk;
};
// token groups of 16 per wave of the wide path: four, or two for five and more
// output blocks (their accumulators would otherwise leave one wave per SIMD)
__host__ __device__ constexpr int wide_tg(int nob) { return nob >= 5 ? 2 : 4; }
__host__ __device__ constexpr int wide_tokens(int nob) { return 64 * wide_tg(nob); }   // per workgroup
constexpr int kWideStep = 4;   // k-blocks per step of the wide path
// steps whose weight fragments (kWideStep x nob KiB each) share one LDS fill;
// two fills alternate: four steps up to four output blocks (at most 128 KiB),
// one step from five blocks on (40 KiB at five, more workgroups per CU;
// measured faster for the router-plus-pre projection of the Flash group)
__host__ __device__ constexpr int wide_seg_steps(int nob) { return nob <= 4 ? 4 : 1; }
// fine: short chunks where few tokens run faster in them.  They leave more
// partials, so the caller sets it where its workspace holds those.
inline ProjPlan proj_plan(int state_dtype, bool gather, int64_t K, int C, int64_t nout, int64_t T, bool fine) {
  const int64_t nblk = K / 32, NO = out_blocks(nout) * 16 + 2;
  const bool wide = (gather ? act_grouped(state_dtype, C) : full_grouped(state_dtype, K)) && out_blocks(nout) <= 8;
  int tg = 4;
  while (tg > 1 && ((T + 16 * tg - 1) / (16 * tg) < 128 || NO * tg > 160)) tg /= 2;
  const int64_t wt = wide_tokens((int)out_blocks(nout));
  const int64_t tiles = wide ? (T + wt - 1) / wt : (T + 16 * tg - 1) / (16 * tg);
  // chunk granularity in k-blocks: 8 steps of the wide path, and 4 or 2 while
  // that still gives each CU one workgroup at most: a step is a round trip to
  // memory, so a workgroup's time is that of its steps (dense T = 2164 C = 128
  // 57 -> 43 us, Flash steps T = 380 C = 4096 71 -> 57 us; but T = 4782 N = 16 C =
  // 448 with 266 workgroups instead of 133 69 -> 76 us).  Not past 128 chunks, whose
  // sum then costs more than the steps saved (pre T = 9 N = 32 C = 2560 with 320
  // chunks instead of 80: 69 -> 73 us).
  const auto at_gran = [&](int64_t g) { return (nblk + g - 1) / g; };
  int64_t gran = 32;
  while (fine && wide && gran > 8 && at_gran(gran) <= 64 && tiles * at_gran(gran / 2) <= 256) gran /= 2;
  // chunks for about 1024 workgroups, 512 for five or more output blocks and
  // 256 for the gathered active rows (longer chunks, fewer weight fills and
  // pipeline starts per byte: measured faster there)
  int64_t want = ((gather ? 256 : (out_blocks(nout) >= 5 ? 512 : 1024)) + tiles - 1) / tiles;
  const int64_t most = (nblk + gran - 1) / gran;
  if (want > most) want = most;
  if (want < 1) want = 1;
  int64_t cb = (nblk + want - 1) / want;
  cb = (cb + gran - 1) / gran * gran;
  return ProjPlan{wide, tg, cb, (nblk + cb - 1) / cb};
}
inline int64_t proj_chunks(int state_dtype, bool gather, int64_t K, int C, int64_t nout, int64_t T, bool fine) {
  return proj_plan(state_dtype, gather, K, C, nout, T, fine).nchunk;
}

hipError_t launch_proj_partial(int state_dtype, const void* X, int64_t T, int N, int C, int64_t K,
                               const void* packed, int64_t nout, const int32_t* idx, int k,
                               bool fine, float* part, hipStream_t s);
// Both projections of a sublayer whose N streams are all active and fixed, in
// one read of the state: its active rows are the state's own rows in order
// (slot j is stream j), so [W_post | W_res] has the rows of [W_r | W_pre].
// Partials as of out_blocks(nout_full) + out_blocks(nout_act) output blocks.
// bf16 state, C % 128 == 0.
hipError_t launch_proj_both(const void* X, int64_t T, int N, int C, const void* packed_full, int64_t nout_full,
                            const void* packed_act, int64_t nout_act, bool fine, float* part, hipStream_t s);
hipError_t launch_pre_route(const float* part, int64_t nchunk, int64_t nout, int64_t T, int N, int m, int k,
                            int npre, int64_t C, const float* colsum, const float* alpha_pre, int alpha_stride,
                            const float* b_pre, float eps, int32_t* idx, float* p, float* Hpre, float* sums,
                            float* saved, int nsave, int save_stats_at, int router, hipStream_t s,
                            int save_pre = 0);   // which pre-map's z goes to saved[N .. 2N); -1: all, one record each
// The single pass whose partials a coefficient pass sums: its count of waits that
// gave up, and what it takes to form a token's outputs again where that is not
// zero (bf16 state, N = 16, k = 4).
struct PreRedo {
  const int* err;
  const uint16_t* X;
  const uint4 *wfull, *wact;   // the packed weights; wact grouped or plain
  int act_grouped;
  const float *colsum, *alpha_pre, *b_pre;
  uint16_t* input;
  int32_t* idx;
  float *p, *Hpre;
  int C, m, softmax;
};
hipError_t launch_pre_coef(const float* part, int64_t nchunk, int64_t nout, int64_t T, int k, int Kq,
                           int with_res, int64_t C, const float* alpha_post, const float* alpha_res,
                           const float* b_post, const float* b_res, float eps, int iters, float delta,
                           float* Hpost, float* Hres, float* sums, float* saved, int nsave, int save_z_at,
                           int save_stats_at, hipStream_t s, const PreRedo* redo = nullptr);
// out0 gets map 0 (full dense read); maps 1..nmap-1 leave out the active
// streams and go to outr + (q - 1) * T * C.
hipError_t launch_dense_read(int state_dtype, const void* X, int64_t T, int N, int C, const float* Hpre,
                             int nmap, const int32_t* idx, int k, void* out0, void* outr, hipStream_t s);

// final stream reduction and its backward (broadcast)
hipError_t launch_stream_sum(int state_dtype, const void* X, int64_t T, int N, int C, void* out, hipStream_t s);
hipError_t launch_stream_bcast(int state_dtype, const void* dout, int64_t T, int N, int C, int accumulate, void* dX,
                               hipStream_t s);

// ---- pre (fused single-pass path: bf16 state, N = 16, k = 4, C % 32 == 0, C <= 4096).
// fused_pre_auto: shapes AUTO takes it for; fused_pre_supported: those of
// impl = FUSED (C = 128 G with G dividing 32)
bool fused_pre_auto(const xhc_dims* d);
bool fused_pre_supported(const xhc_dims* d);
size_t fused_pre_ws_bytes(const xhc_dims* d);
hipError_t launch_pre_fused(const xhc_dims* d, const void* X, const void* packed_full, const float* colsum,
                            const void* packed_act, const float* alpha, const float* b_pre, const float* b_res,
                            const float* b_post, void* input, int32_t* idx, float* p, float* Hpre, float* Hres,
                            float* Hpost, float* saved, void* ws, hipStream_t s);

// ---- post
__host__ __device__ inline int64_t post_chunks(int C) { return ((int64_t)C / 8 + 255) / 256; }
// How a post with these sizes runs in a workspace of `avail` bytes: run-based
// kernels or per-token ones, the Gram partials' chunks, and where the per-token
// write-back weights lie behind them.  bytes: what the workspace query says;
// least: what has to be there.
struct PostPlan {
  bool gram_run, apply_run;
  int64_t nchunk;
  size_t bytes, least, wb_at;
};
PostPlan post_plan(int64_t T, int64_t S, int C, int k, int Kr, const int32_t* kappa, size_t avail);
hipError_t launch_post_gram(const PostPlan& plan, int state_dtype, const void* F, int64_t T, int64_t S, int C, int Kr,
                            const int32_t* kappa, const float* conv_w, float* gpart, hipStream_t s);
// The write-back of the k active rows.  For K_r > 1 gpart holds the Gram
// partials of launch_post_gram: the write-back weights are then formed from
// them (Gram-Schmidt, p, H^post) inside the run-based kernel, or into the
// workspace wb by a per-token pass before the generic one.  K_r = 1: gpart and
// wb are null.
hipError_t launch_post_apply(const PostPlan& plan, int state_dtype, void* X, const void* F, int64_t T, int64_t S, int N,
                             int C, int k, int Kr, const int32_t* kappa, const float* conv_w, const int32_t* idx,
                             const float* p, const float* Hres, const float* Hpost, const float* gpart,
                             int gram_schmidt, float* wb, const float* Hpre_next, const void* base_next,
                             void* input_next, void* Xact_save, hipStream_t s);

// ---- backward
// fine: the shorter runs and token chunks that few tokens run faster in.  They
// leave more partials, so the caller sets it where its workspace holds the
// bytes of *_ws_bytes(.., true); with the full lengths the need grows with T.
hipError_t launch_bwd_post(const xhc_dims* d, const void* dXn, void* X, const void* Xact, const void* F,
                           const float* conv_w, const int32_t* idx, const float* p, const float* Hres,
                           const float* Hpost, void* dX, void* dF, float* dHres, float* dHpost, float* dp,
                           float* dconv_w, char* ws, bool fine, hipStream_t s, bool grad_f32, bool add_dp = false);
// (X null: the saved rows are not written back into X; grad_f32: dXn and dX
// are fp32 whatever the state dtype, as the xHC-Flash active-row gradient;
// add_dp: dp is added to)
size_t bwd_post_ws_bytes(const xhc_dims* d, bool fine);
bool bwd_pre_supported(const xhc_dims* d);
size_t bwd_pre_ws_bytes(const xhc_dims* d, bool fine);
struct BwdPreWs {
  float *part, *tok, *pg, *wpart_r, *wpart_p, *wpart_a, *corr;
  uint16_t *dzf, *dza;   // packed dz' of the full-row and active-row MFMA passes
  float *srec, *sreca;   // per-token scalars of the ring passes [Tp][8]: full rows, active rows
};
// Row pass of the pre-map reverse with its inputs staged through an LDS ring
// (xhc_bwd_rows.hip): dX += (input-gradient reads, projection and
// normalisation terms) over rows x 128-channel blocks of a bf16 state, and the
// weight-gradient partials of the projection.  Weight row K = i C + c is
// channel c of row i of every token; slot j of the k-row view is row j.
constexpr int kRowRingMaxQ = 4;
struct RowRingDesc {
  const void* X;                        // bf16 state [T][N][C]
  void* dX;                             // gradient rows [T][N][C], updated in place
  bool dx_f32;                          // fp32 gradient rows (else bf16)
  int nq;                               // input gradients, 0 .. kRowRingMaxQ
  const void* din[kRowRingMaxQ];        // bf16 [T][C]
  const float* hp[kRowRingMaxQ];        // their weights: row i of token t at t hp_stride + i
  int hp_stride;
  const float* w[kRowRingMaxQ + 1];     // weight blocks [rows][win[b]] (fp32), outputs in block order
  int win[kRowRingMaxQ + 1];
  int nwin;
  float* wout[kRowRingMaxQ + 1];        // partials [chunk][rows][wout_w], outputs in blocks of wout_w
  int wout_w;
  int nout;                             // outputs
  const uint16_t* dzp;                  // packed dz' of nop outputs (rows, then 32-token transposes)
  int nop;
  const float* srec;                    // per-token r_ln, mu, m1, m2, beta (16-byte aligned rows)
  int64_t srec_stride;                  // floats
  int64_t T, tchunk;                    // tokens; tokens per partial (a multiple of 32)
  int N, C;
};
bool bwd_rows_ring_supported(int64_t rows, int C, int64_t tchunk);
hipError_t launch_bwd_rows_ring(const RowRingDesc& d, int64_t rows, hipStream_t s);
BwdPreWs bwd_pre_ws(const xhc_dims* d, char* ws, bool fine);   // layout of launch_bwd_pre's workspace
// One pre-map reverse; gradients whose pointer is null are not formed.
struct BwdPre {
  const void* X;
  const float *colsum, *W_r, *W_pre, *W_res, *W_post;   // W_res null: no residual mapping
  const float *al_pre, *al_res, *al_post;               // device scalars; null: 0
  const float* b_res;
  const float* saved;
  const int32_t* idx;
  const float *p, *Hpre, *Hpost;
  const void* d_input;
  const float* dHres;    // null: no residual mapping
  const float* dHpost;   // null: no active-row outputs
  const float* dp;       // null: no router gradient
  void* dX;
  float *dW_r, *dW_pre, *dW_res, *dW_post;
  float *dal_pre, *dal_res, *dal_post;
  float *db_pre, *db_res, *db_post;
  char* ws;
  bool fine = true;   // (the same for all that run together)
  // [T, k]: dL/dH^pre of the active streams (slot order), in place of <d input, x_i> there
  const float* dhpre_act;
  // [T, N], written here when given: Hpre with the active streams zero, the
  // weights of the dense-read term dX_i += H^pre_i d input (Hpre otherwise)
  float* hmask;
  // false leaves out every term of the dense rows (the read and the full-state
  // projection through W_r, W_pre): d_input, W_r, W_pre and colsum are then
  // not read (no router: every slot fixed), dW_r and dW_pre not written
  bool dense_rows = true;
  bool act_rows = true;    // false leaves out the active-row pass: dW_post, dW_res are not written
  bool own_rows = true;    // false: launch_bwd_rows_multi runs the row pass
  // for an fp32 view whose values are exactly bf16 and whose slot j is row j
  // (N = k: the k-row view of an xHC-Flash sublayer), the same rows as bf16
  // (read by the ring form of the active-row pass; the gradient rows stay
  // fp32), and then act_din (bf16 [T, C]), when given: that pass also adds
  // Hpre[t, j] act_din[t] to active row j (Hpre then holds [T, k] slot weights)
  const void* X_bf16;
  const void* act_din;
};
hipError_t launch_bwd_pre(const xhc_dims* d, const BwdPre& b, hipStream_t s);
// its parts around launch_bwd_rows_multi, for n = Q pre-map reverses at once:
// the token reverses (after launch_bwd_dhpre_multi) and the reductions
hipError_t launch_bwd_pre_tokens(const xhc_dims* d, const BwdPre* b, int n, hipStream_t s);
hipError_t launch_bwd_pre_reduce(const xhc_dims* d, const BwdPre* b, int n, hipStream_t s);
// The full-row pass of Q pre-map reverses of one bf16 state (N = 8 or 16, Q = 2
// or 4) in one pass: pass q's token records and weight partials live in the
// launch_bwd_pre workspace ws[q] (after launch_bwd_pre_tokens; the router's
// partials in ws[0]), hrd[q] are its dense-read weights [T, N], d_input is
// [Q, T, C]; dX accumulates every pass's row terms.
// pack_ws: a scratch buffer of bwd_rows_multi_ws_bytes (per-token inputs of the
// fused pass).
bool bwd_rows_multi_supported(const xhc_dims* d, int Q);
size_t bwd_rows_multi_ws_bytes(const xhc_dims* d, int Q);
// the <d input_q, x_i> partials of the Q passes in one read of the state,
// into each pass's workspace ws[q]
hipError_t launch_bwd_dhpre_multi(const xhc_dims* d, int Q, const void* X, const void* d_input, char* const* ws,
                                  hipStream_t s);
hipError_t launch_bwd_rows_multi(const xhc_dims* d, int Q, const void* X, void* dX, const float* W_r,
                                 const float* W_pre, const void* d_input, const float* const* hrd, char* const* ws,
                                 char* pack_ws, bool fine, hipStream_t s);

// ---- xHC-Flash backward helpers
hipError_t launch_fill0(void* p, size_t bytes, hipStream_t s);
hipError_t launch_fbwd_token(int state_dtype, int64_t T, int N, int k, int C, const int32_t* idx,
                             const float* Hpre_q, const void* din, const void* Xact, int32_t* idx_id, float* Hres_id,
                             float* Hsel, float* dhact, hipStream_t s);
hipError_t launch_fbwd_gather(int state_dtype, int64_t T, int N, int k, int C, const int32_t* idx, const void* dXn,
                              float* da, hipStream_t s);
hipError_t launch_fbwd_scatter(int state_dtype, int64_t T, int N, int k, int C, const int32_t* idx, const void* GX,
                               const float* da0, void* dX, hipStream_t s);
hipError_t launch_fbwd_finish(int state_dtype, int64_t T, int k, int C, const float* da_rev, const float* Hsel,
                              const void* din, float* da, hipStream_t s);

// per-token values xhc_pre saves for the backward: [z_r (N) | z_pre (N) |
// z_post, z_res (k*Kr + k*k) | mu | nu | nu_a | pad], z = normalised logits
__host__ __device__ inline int saved_floats(int N, int k, int Kr) { return 2 * N + k * Kr + k * k + 4; }

}  // namespace xhc
