// Host-side launchers of the Q-Delta kernels (internal to libqdelta.so).
#pragma once

#include <hip/hip_runtime.h>

#include "qd_common.h"

namespace qd {

enum Stage {
  ST_PREP_FWD = 0,
  ST_SCAN_FWD = 1,
  ST_PREP_BWD = 2,
  ST_SCAN_BWD = 3,
  ST_INTRA = 4,
  ST_STEP = 5,
  ST_REC_FWD = 6,
  ST_SEG_MAPS = 7,
  ST_SEG_COMPOSE = 8,
  ST_SEG_OUT = 9,
  ST_REC_BWD = 10,
  ST_COUNT = 11
};

// Records a HIP event on `st` before (after == 0) or after (after == 1) a
// kernel launch of `stage` while the measurement facility is active.
void prof_mark(int stage, int after, hipStream_t st);

// Chunk preparation (UT solve, WY factors) over all slots, then, if
// with_scan, the sequential forward state scan (+ chunk outputs when p.o is
// set).  in_bwd only labels the launches for the measurement facility (a
// backward that recomputes the saved context).
hipError_t launch_fwd(const Params& p, int dtype, int Dk, int Dv, int in_bwd, int with_scan,
                      hipStream_t st);

// Segment-parallel forward of a dense batch (p.n_seg segments of
// p.seg_chunks chunks per sequence; p.wSegOut, p.wSegIn set): preparation,
// segment maps, composition, outputs.
hipError_t launch_fwd_seg(const Params& p, int dtype, int Dk, int Dv, hipStream_t st);

// Workgroups of the fullest XCD when `units` are dealt to the eight XCDs
// with `tiles` workgroups each, and the rounds that many take at one
// workgroup per CU.
inline long long on_xcd(long long units, int tiles) { return (units + 7) / 8 * tiles; }
inline long long xcd_rounds(long long wgs) {
  const long long cus = device_cu_count() / 8 > 0 ? device_cu_count() / 8 : 1;
  return (wgs + cus - 1) / cus;
}
// Whether the outputs pass over `outs` segments takes 64-row tiles: a round
// of them takes 1.5 times one of 32-row tiles (2.1 us a chunk against 1.4 at
// bf16 d 128).  65536 tokens, 16 heads, 8 segments: 64-row tiles in one round
// 901 us for the call, 32-row tiles in two 985; 5 segments: 32-row tiles, one
// round either way.
inline bool seg_out_wide(long long outs, int Dv) {
  return 3 * xcd_rounds(on_xcd(outs, Dv / 64)) < 2 * xcd_rounds(on_xcd(outs, Dv / 32));
}

// Backward once the saved context (states, D, b, W, P, M) is in place:
// reverse state scan, then the intra-chunk gradient kernel.
hipError_t launch_bwd(const Params& p, int dtype, int Dk, int Dv, hipStream_t st);

// Writes 0 to one device float (a gradient with nothing to sum).
hipError_t launch_zero(float* x, hipStream_t st);

// One token of the recurrence for N sequences.
hipError_t launch_step(int N, int H, int Dk, int Dv, int dtype, const void* q, const void* k,
                       const void* v, const float* beta, const float* lam, float lam_c, const float* la,
                       float* state, void* o, hipStream_t st);

// Fully recurrent forward over whole sequences: dense (cu == nullptr, N
// sequences of T tokens) or packed (cu[N+1] on the device, T_total tokens).
hipError_t launch_rec_fwd(int N, int T, const int* cu, int T_total, int H, int Dk, int Dv,
                          int dtype, const void* q, const void* k, const void* v,
                          const float* beta, const float* lam, float lam_c, const float* la,
                          const float* S0, float* Sfin, void* o, hipStream_t st);

// The recurrent backward stores the entry state of every rec_ckpt-th block of
// 16 tokens.  The workspace holds 3 Dv + Dk floats per token and head
// (qdelta_recurrent_workspace_bytes), so the spacing is the smallest whose
// states fit: 1 at Dk = 64 with Dv = 32 or 64, 3 at Dk = 128 with Dv = 256, else 2.
__host__ __device__ constexpr int rec_ckpt(int Dk, int Dv) {
  int c = 1;
  while (16 * c * (3 * Dv + Dk) < Dv * Dk) ++c;
  return c;
}

// Arguments of the fully recurrent backward (one workgroup per (sequence,
// head) unit).
struct RecBwdArgs {
  int T;                    // dense: tokens per sequence
  const int* cu;            // varlen: cu_seqlens[N+1] (device), clamped to [0, T_total]
  int T_total;
  int H, DV;
  const void *q, *k, *v, *dO;
  const float *beta, *lam, *la, *S0, *dSfin;
  float lam_c;              // lambda when lam is nullptr
  void *dq, *dk, *dv;
  float *dbeta, *dlam, *dla, *dS0;
  float* wDL;               // per token-head gradient of a constant lambda (else nullptr)
  int skip;                 // > 0: sequences of at most so many tokens are another launch's
  float* wS;                // workspace: stored entry states, [slot][H][DV][DK] fp32 (rec_ckpt)
};

// Fully recurrent backward over `units` (sequence, head) units; when
// dlam_sum is set, the constant lambda's gradient (sum of a.wDL over
// n_tok_heads entries) is written there.
hipError_t launch_rec_bwd(const RecBwdArgs& a, int units, int dtype, int Dk, float* dlam_sum, long long n_tok_heads,
                          hipStream_t st);

// The same for sequences of at most `tokens` tokens (1 or 2; up to 4 at Dk = 64); longer ones are left alone.
hipError_t launch_rec_bwd_few(const RecBwdArgs& a, int units, int dtype, int Dk, int tokens, hipStream_t st);

// Row L2 normalisation (bwd == 0: x -> out, rn_out) or its backward
// (bwd == 1: y, rn_in, dy -> out).
hipError_t launch_l2norm(int bwd, long rows, int D, long ldx, int dtype, const void* x,
                         const void* y, const float* rn_in, float* rn_out, const void* dy, void* out,
                         hipStream_t st);

// Row L2 normalisation of two tensors of the same strided shape in one launch.
hipError_t launch_l2norm2(long rows, int D, long ldx, int dtype, const void* x, void* y, float* rn, const void* x2,
                          void* y2, float* rn2, hipStream_t st);

// Layer gates from rows of logits (ld apart) over n (token, head) pairs, and
// their backward; lam / la nullptr where not learned.  part holds gates_blocks(n) floats.
int gates_blocks(long n);
hipError_t launch_gates_fwd(long n, int H, int ld, int dtype, int bias_dtype, const void* x, const void* bias,
                            float* beta, float* lam, float* la, hipStream_t st);
hipError_t launch_gates_bwd(long n, int H, int ld, int dtype, int bias_dtype, const float* beta, const float* lam,
                            const float* la, const float* dbeta, const float* dlam, const float* dla, void* dx,
                            float* part, void* dbias, hipStream_t st);

}  // namespace qd
