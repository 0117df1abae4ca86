// Single-token Q-Delta update for N sequences (decode), Sec. 3.3
// Eq. (qdelta_decay) applied once per (sequence, head):
//
//   x = k + lambda q;  p = S x;  S <- alpha S + beta (v - alpha p) k^T;  o = S q
//
// Each state row S[v, :] is independent, so a row is owned by a group of
// Dk/4 lanes (one float4 each): the state is read once and written once with
// fully coalesced 16-byte accesses, and the two row dot products are reduced
// with DPP lane moves (one shuffle across rows of 16).  The kernel is bound by
// HBM (or MALL) bandwidth.
#include <type_traits>

#include "qd_common.h"
#include "qd_launch.h"

namespace qd {

// Sum over each aligned group of L = 16 or 32 lanes: DPP within rows of 16
// lanes, then one cross-row exchange for 32.
template <int L>
__device__ inline float row_sum(float x) {
  static_assert(L == 16 || L == 32, "lane group of 16 or 32");
  x = sum16(x);
  if (L == 32) x += __shfl_xor(x, 16, 64);
  return x;
}

// Each lane group owns RPT state rows RPB apart (RPB = rows per workgroup
// pass), so a wave has RPT independent 16-byte loads in flight instead of
// one; the per-row dot products are reduced side by side.
constexpr int STEP_RPT = 4;

template <typename E, int DK>
__global__ __launch_bounds__(NTHREADS) void k_step(int DV, int nrb, const E* __restrict__ q,
                                                  const E* __restrict__ k, const E* __restrict__ v,
                                                  const float* __restrict__ beta,
                                                  const float* __restrict__ lam, float lam_c,
                                                  const float* __restrict__ la, float* __restrict__ S,
                                                  E* __restrict__ o) {
  constexpr int LPR = DK / 4;            // lanes per state row
  constexpr int RPB = NTHREADS / LPR;    // rows per workgroup pass
  constexpr int RPT = STEP_RPT;          // passes (rows per lane group)
  const size_t u = blockIdx.x / nrb;     // (sequence, head) unit
  const int rb = blockIdx.x % nrb;       // block of RPB * RPT state rows
  const int tid = threadIdx.x;
  const int row0 = rb * RPB * RPT + tid / LPR;
  const int c0 = (tid % LPR) * 4;
  float qv[4], kv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    qv[j] = tof(q[u * DK + c0 + j]);
    kv[j] = tof(k[u * DK + c0 + j]);
  }
  const float lm = lam ? lam[u] : lam_c, bt = beta[u];
  const float al = la ? __expf(la[u]) : 1.f;
  float xv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) xv[j] = kv[j] + lm * qv[j];
  f4 s[RPT];
  float vr[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {        // rows past DV: the whole lane group skips them
    const int row = row0 + i * RPB;
    s[i] = row < DV ? *(const f4*)(S + (u * DV + row) * DK + c0) : zero4();
    vr[i] = row < DV ? tof(v[u * DV + row]) : 0.f;
  }
  float px[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    px[i] = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) px[i] += s[i][j] * xv[j];
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i) px[i] = row_sum<LPR>(px[i]);
  float oq[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const float e = bt * (vr[i] - al * px[i]);
    oq[i] = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[i][j] = al * s[i][j] + e * kv[j];
      oq[i] += s[i][j] * qv[j];
    }
    const int row = row0 + i * RPB;
    if (row < DV) *(f4*)(S + (u * DV + row) * DK + c0) = s[i];
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i) oq[i] = row_sum<LPR>(oq[i]);
  if ((tid % LPR) == 0) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int row = row0 + i * RPB;
      if (row < DV) o[u * DV + row] = fromf<E>(oq[i]);
    }
  }
}

// The same for a few tokens per sequence, the state staying in registers
// between them, from S0 (NULL: zero) to S (NULL: not wanted): sequence n spans
// tokens [cu[n], cu[n+1]) when cu is given (clamped to [0, T_total]), else
// [n T, (n + 1) T); token t of head h sits at row t H + h.
template <typename E, int DK>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(sizeof(E) == 4 ? 7 : 6))) void k_steps(
    int T, const int* __restrict__ cu, int T_total, int H, int DV, int nrb, const E* __restrict__ q,
    const E* __restrict__ k, const E* __restrict__ v, const float* __restrict__ beta, const float* __restrict__ lam,
    float lam_c, const float* __restrict__ la, const float* __restrict__ S0, float* __restrict__ S,
    E* __restrict__ o) {
  constexpr int LPR = DK / 4;            // lanes per state row
  constexpr int RPB = NTHREADS / LPR;    // rows per workgroup pass
  constexpr int RPT = STEP_RPT;          // passes (rows per lane group)
  const size_t u = blockIdx.x / nrb;     // (sequence, head) unit
  const int rb = blockIdx.x % nrb;       // block of RPB * RPT state rows
  const int tid = threadIdx.x;
  const int row0 = rb * RPB * RPT + tid / LPR;
  const int c0 = (tid % LPR) * 4;
  const int n = (int)(u / H);
  const int t0 = cu ? min(max(cu[n], 0), T_total) : n * T;
  const int t1 = cu ? min(max(cu[n + 1], t0), T_total) : t0 + T;
  size_t a = (size_t)t0 * H + u % H;     // row of the token
  // Operands of a token: loaded as they lie in memory, with no branch on the
  // row and no conversion among the loads (the compiler would wait for each by
  // itself), and converted before the stores of the token in between (a wait
  // after them would cover them too).  A long sequence among short ones walks
  // alone here, at the latency of a token: 63 sequences of one token and one
  // of 65, 16 heads, bf16, d 64: 73 us with a wait for each load, 43 so
  // (d 128: 98, 68); 64 of two tokens, d 128: 28.6, 24.2.
  typename Quad<E>::raw qr, kr;
  E vr[RPT];
  float qt[4], kt[4], vt[RPT], bt, lm, la_, bn, ln, an;
  int vz = 0;                            // the gates by vector loads too: a wait for a scalar one is a wait for all
  if constexpr (sizeof(E) == 2) asm volatile("" : "+v"(vz));
  auto load = [&]() {
    qr = *(const typename Quad<E>::raw*)(q + a * DK + c0);
    kr = *(const typename Quad<E>::raw*)(k + a * DK + c0);
#pragma unroll
    for (int i = 0; i < RPT; ++i) vr[i] = v[a * DV + min(row0 + i * RPB, DV - 1)];
    ln = (lam ? lam : beta)[a + vz];
    bn = beta[a + vz];
    an = (la ? la : beta)[a + vz];
  };
  auto take = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      qt[j] = Quad<E>::get(qr, j);
      kt[j] = Quad<E>::get(kr, j);
      asm volatile("" : "+v"(qt[j]), "+v"(kt[j])::"memory");
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      vt[i] = tof(vr[i]);
      asm volatile("" : "+v"(vt[i])::"memory");
    }
    bt = bn;
    lm = lam ? ln : lam_c;
    la_ = an;
    asm volatile("" : "+v"(bt), "+v"(lm), "+v"(la_)::"memory");
  };
  f4 s[RPT];
  if (S0) {                              // rows past DV repeat the last one, and are not stored
#pragma unroll
    for (int i = 0; i < RPT; ++i) s[i] = *(const f4*)(S0 + (u * DV + min(row0 + i * RPB, DV - 1)) * DK + c0);
  } else {
#pragma unroll
    for (int i = 0; i < RPT; ++i) s[i] = zero4();
  }
  auto token = [&](auto more) {
    const size_t at = a;
    if constexpr (decltype(more)::value) {   // the next token's operands, in flight during this one
      a += H;
      load();
    }
    const float al = la ? __expf(la_) : 1.f;
    float px[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      px[i] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) px[i] += s[i][j] * (kt[j] + lm * qt[j]);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) px[i] = row_sum<LPR>(px[i]);
    float oq[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const float e = bt * (vt[i] - al * px[i]);
      oq[i] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s[i][j] = al * s[i][j] + e * kt[j];
        oq[i] += s[i][j] * qt[j];
      }
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) oq[i] = row_sum<LPR>(oq[i]);
    if constexpr (decltype(more)::value) take();
    if ((tid % LPR) == 0) {
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int row = row0 + i * RPB;
        if (row < DV) o[at * DV + row] = fromf<E>(oq[i]);
      }
    }
  };
  if (t0 < t1) {
    load();
    take();
    for (int t = t0; t + 1 < t1; ++t) token(std::true_type());
    token(std::false_type());
  }
  if (S) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int row = row0 + i * RPB;
      if (row < DV) *(f4*)(S + (u * DV + row) * DK + c0) = s[i];
    }
  }
}

// T < 0: the decode step, S updated in place; else T tokens (or cu) from S0 to S.
static hipError_t step_at(int N, int T, const int* cu, int T_total, int H, int Dk, int Dv, int dtype, const void* q,
                          const void* k, const void* v, const float* beta, const float* lam, float lam_c,
                          const float* la, const float* S0, float* S, void* o, hipStream_t st) {
  if (N == 0) return hipSuccess;
  if (!((dtype == 1 || dtype == 0) && (Dk == 128 || Dk == 64))) return hipErrorInvalidValue;
  const int RPB = NTHREADS / (Dk / 4) * STEP_RPT;   // state rows per workgroup
  const int nrb = (Dv + RPB - 1) / RPB;
  const int stage = T < 0 ? ST_STEP : ST_REC_FWD;
  dim3 grid((unsigned)((size_t)N * H * nrb));
#define QD_STEP(ET, DKV)                                                                               \
  do {                                                                                                 \
    if (T < 0)                                                                                         \
      hipLaunchKernelGGL((k_step<ET, DKV>), grid, dim3(NTHREADS), 0, st, Dv, nrb, (const ET*)q,        \
                         (const ET*)k, (const ET*)v, beta, lam, lam_c, la, S, (ET*)o);                 \
    else                                                                                               \
      hipLaunchKernelGGL((k_steps<ET, DKV>), grid, dim3(NTHREADS), 0, st, T, cu, T_total, H, Dv, nrb,  \
                         (const ET*)q, (const ET*)k, (const ET*)v, beta, lam, lam_c, la, S0, S, (ET*)o); \
  } while (0)
  prof_mark(stage, 0, st);
  if (dtype == 1 && Dk == 128) QD_STEP(__bf16, 128);
  else if (dtype == 1 && Dk == 64) QD_STEP(__bf16, 64);
  else if (dtype == 0 && Dk == 128) QD_STEP(float, 128);
  else QD_STEP(float, 64);
  prof_mark(stage, 1, st);
#undef QD_STEP
  return hipGetLastError();
}

hipError_t launch_step(int N, int H, int Dk, int Dv, int dtype, const void* q, const void* k,
                       const void* v, const float* beta, const float* lam, float lam_c, const float* la,
                       float* state, void* o, hipStream_t st) {
  return step_at(N, -1, nullptr, 0, H, Dk, Dv, dtype, q, k, v, beta, lam, lam_c, la, nullptr, state, o, st);
}

// Fully recurrent forward over whole sequences (Sec. 3.3, Eq. (qdelta_decay)
// token by token; the paper offers this form beside the chunkwise one), in
// fp32 throughout.
//
// One wave owns 16 VB value rows of one (sequence, head) and walks its tokens
// in blocks of RTB = 16.  Within a block, with entry state S, decay products
// g_t = alpha_1..alpha_t, Gam_ti = alpha_{i+1}..alpha_t and x = k + lambda q,
// unrolling the recurrence gives
//
//   e_t = beta_t (v_t - g_t S x_t) - sum_{i<t} beta_t Gam_ti (k_i . x_t) e_i
//   o_t = g_t S q_t + sum_{i<=t} Gam_ti (k_i . q_t) e_i
//   S  <- g_C S + sum_i Gam_Ci e_i k_i^T
//
// so the products with the state, S k_t and S q_t for 16 tokens and the rank-16
// update, are fp32 matrix products (16x16x4), and only the triangular part is
// left to the vector ALU: a lane holds one value row there and substitutes
// token by token with coefficients broadcast from LDS (so a row never sees a
// later token).  The state lives in registers as S^T tiles in the matrix
// result layout, which is the layout of the operand the next block's S k_t
// takes, so it passes through no LDS.  Decays are multiplied up, never divided
// or exponentiated from sums, so alpha = 0 is exact.
//
// 64 sequences x 16 heads, d 128, bf16: 16 tokens move 151 MB and take 2.6e9
// matrix operations; vector-ALU row sums over the whole state, as in the step
// kernel, took 75 us at T = 16 and 190 us at T = 64.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int RTB = 16;
#define REC_FENCE __builtin_amdgcn_sched_barrier(0)

// State tile kt = 2 p + h holds the key columns 32 p + 8 (m >> 2) + 4 h + (m & 3)
// for m = 0..15: a lane's rows of the tile pair are eight consecutive columns,
// one 16-byte bf16 read of K or Q and 32 contiguous bytes of the state.
__device__ inline int rec_col(int kt, int m) { return 32 * (kt >> 1) + 8 * (m >> 2) + 4 * (kt & 1) + (m & 3); }

template <typename E, int DK, int VB>
struct alignas(16) RecFwdSmem {
  static constexpr int NV = 16 * VB, P = Pad<E>::v;
  static constexpr int XB = RTB * (NV + 4) * 4, QB = RTB * (DK + P) * (int)sizeof(E);
  alignas(16) E k[RTB][DK + P];
  alignas(16) char qx[QB > XB ? QB : XB];      // Q, then g_t S q_t per value row
  alignas(16) float x[RTB][NV + 4];            // right-hand sides, then Gam_Ct e_t
  alignas(16) E v[RTB][NV];
  alignas(16) float A[RTB][RTB], Pm[RTB][RTB]; // coefficients of the triangular part
  alignas(16) float gate[4][RTB];              // beta, lambda, alpha
};

// Four K (or Q) values of one row as fp32 operands of the tile pair p.
template <typename E>
__device__ inline void rec_row8(const E* src, f4& lo, f4& hi) {
  if constexpr (sizeof(E) == 2) {
    const bf8 r = *(const bf8*)src;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = (float)r[j];
      hi[j] = (float)r[4 + j];
    }
  } else {
    lo = *(const f4*)src;
    hi = *(const f4*)(src + 4);
  }
}

// K^T operand of tile kt: tokens 4 (lane >> 4) .. +3 of column rec_col(kt, lane & 15).
template <typename E>
__device__ inline f4 rec_tok4(const E* k, int ld, int kt, int lane) {
  const int g = lane >> 4, L = lane & 15;
  f4 r;
  if constexpr (sizeof(E) == 2) {
    typedef __bf16 v4b __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4b* lp;
    // LDS transpose read: lane L names the four columns from rec_col(kt, 4 (L & 3))
    // of row L >> 2 and receives column L of the group's 4 x 16 block
    const E* a = k + (size_t)(4 * g + (L >> 2)) * ld + rec_col(kt, 4 * (L & 3));
    const v4b t = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lp)(uintptr_t)(uint32_t)(uintptr_t)a);
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = (float)t[j];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = k[(size_t)(4 * g + j) * ld + rec_col(kt, L)];
  }
  return r;
}

// Value blocks per wave where the launch fills the chip: wide tiles share the
// K, Q reads and the Gram products over more rows, as many as the register
// file takes at two waves per SIMD or more (bf16, d_k 128: four take 256 and
// spill 19, 48 bytes a lane, and are still the faster: 88 us against 121 in
// 16-row tiles for 64 sequences of 64 tokens, 16 heads, d 128).
template <typename E, int DK>
constexpr int rec_wide() { return sizeof(E) == 2 && DK == 128 ? 4 : 2; }
// Waves per SIMD that the register need allows (the state takes 4 VB DK / 16
// registers of a lane, the next block's pieces and the products the rest).
template <typename E, int DK, int VB>
constexpr int rec_waves() { return sizeof(E) == 4 ? 2 : VB == 4 ? 2 : VB == 2 ? 3 : DK == 128 ? 2 : 4; }

template <typename E, int DK, int VB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(rec_waves<E, DK, VB>(), rec_waves<E, DK, VB>()))) void k_rec_fwd(
    int T, int H, int DV, int units, int ntile, const int* __restrict__ cu, int T_total, const E* __restrict__ q,
    const E* __restrict__ k, const E* __restrict__ v, const float* __restrict__ beta,
    const float* __restrict__ lam, float lam_c, const float* __restrict__ la, const float* __restrict__ S0,
    float* __restrict__ Sfin, E* __restrict__ o) {
  constexpr int NV = 16 * VB, NKT = DK / 16;
  constexpr int EPP = 16 / (int)sizeof(E);     // elements per 16-byte piece
  constexpr int QKN = RTB * DK / EPP / 64;     // pieces of one block of q (or k) per lane
  constexpr int VP = RTB * NV / EPP, VN = (VP + 63) / 64;
  typedef RecFwdSmem<E, DK, VB> SM;
  constexpr int LDK = DK + SM::P, LDX = NV + 4;
  __shared__ SM sm;
  E* const qs = (E*)sm.qx;
  float* const xq = (float*)sm.qx;
  int u, vt;                                   // all value tiles of a unit on one XCD: they share k and q
  if (!xcd_unit_tile(blockIdx.x, units, ntile, u, vt)) return;
  const int n = u / H, h = u % H, v0 = vt * NV;
  const int lane0 = threadIdx.x;
  int t0, t1;
  if (cu) {
    t0 = min(max(cu[n], 0), T_total);
    t1 = min(max(cu[n + 1], t0), T_total);
  } else {
    t0 = n * T;
    t1 = t0 + T;
  }

  // block loads one block ahead: registers, then LDS.  Tokens past the end
  // re-read the last one and value rows past DV the last piece (no branches
  // around the loads): beta = 0 and alpha = 1 there, so nothing of them reaches
  // the state or a stored output.
  u32x4 rq[QKN], rk[QKN], rv[VN];
  float rg = 0.f;
  auto load_block = [&](int tb, int lane) {
    const int g = lane >> 4, m = lane & 15;
    const float* const gsrc = g == 1 && lam ? lam : g == 2 && la ? la : beta;
#pragma unroll
    for (int j = 0; j < QKN; ++j) {
      const int idx = lane + j * 64, t = min(tb + idx / (DK / EPP), t1 - 1);
      const size_t off = ((size_t)t * H + h) * DK + (size_t)(idx % (DK / EPP)) * EPP;
      rq[j] = *(const u32x4*)(q + off);
      rk[j] = *(const u32x4*)(k + off);
    }
#pragma unroll
    for (int j = 0; j < VN; ++j) {
      const int idx = lane + j * 64, t = min(tb + (idx / (NV / EPP)) % RTB, t1 - 1);
      const int row = min(v0 + (idx % (NV / EPP)) * EPP, DV - EPP);   // DV is a multiple of 8
      rv[j] = *(const u32x4*)(v + ((size_t)t * H + h) * DV + row);
    }
    rg = gsrc[(size_t)min(tb + m, t1 - 1) * H + h];
  };
  auto store_block = [&](int tb, int lane) {
    const int g = lane >> 4, m = lane & 15;
#pragma unroll
    for (int j = 0; j < QKN; ++j) {
      const int idx = lane + j * 64, r = idx / (DK / EPP), c = (idx % (DK / EPP)) * EPP;
      *(u32x4*)(qs + r * LDK + c) = rq[j];
      *(u32x4*)&sm.k[r][c] = rk[j];
    }
#pragma unroll
    for (int j = 0; j < VN; ++j) {
      const int idx = lane + j * 64;
      if (idx < VP) *(u32x4*)(&sm.v[0][0] + idx * EPP) = rv[j];
    }
    const bool in = tb + m < t1;
    const float x = g == 0 ? (in ? rg : 0.f) : g == 1 ? (lam ? rg : lam_c) : (in && la ? __expf(rg) : 1.f);
    sm.gate[g][m] = x;                         // (row 3 is not read)
  };

  const int nblk = (t1 - t0 + RTB - 1) / RTB;
  if (nblk > 0) load_block(t0, lane0);
  // S^T tiles: s[kt][vb][j] = S[v0 + 16 vb + m][rec_col(kt, 4 g + j)]
  f4 s[NKT][VB];
  if (S0) {
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
      const float* src = S0 + ((size_t)u * DV + min(v0 + 16 * vb + (lane0 & 15), DV - 1)) * DK + 8 * (lane0 >> 4);
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) s[kt][vb] = *(const f4*)(src + 32 * (kt >> 1) + 4 * (kt & 1));
    }
  } else {
#pragma unroll
    for (int vb = 0; vb < VB; ++vb)
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) s[kt][vb] = zero4();
  }
  for (int b = 0; b < nblk; ++b) {
    const int tb = t0 + b * RTB, nt = min(RTB, t1 - tb);
    int lane = lane0;                          // laundered: addresses formed per block, not kept in registers
    asm volatile("" : "+v"(lane));
    const int g = lane >> 4, m = lane & 15;
    store_block(tb, lane);
    __syncthreads();
    // rows t = 4 g + j, columns i = m of K K^T and Q K^T; rows t, value columns of K S^T and Q S^T
    f4 kk = zero4(), qk = zero4(), sk[VB], sq[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) sk[vb] = sq[vb] = zero4();
#pragma unroll
    for (int p = 0; p < NKT / 2; ++p) {
      REC_FENCE;
      f4 ka[2], qa[2];
      rec_row8<E>(&sm.k[m][32 * p + 8 * g], ka[0], ka[1]);
      rec_row8<E>(qs + m * LDK + 32 * p + 8 * g, qa[0], qa[1]);
      if constexpr (sizeof(E) == 2) {          // products of bf16 inputs are exact in fp32
        const bf8 kr = *(const bf8*)&sm.k[m][32 * p + 8 * g], qr = *(const bf8*)(qs + m * LDK + 32 * p + 8 * g);
        kk = Mma<E>::mma(kr, kr, kk);
        qk = Mma<E>::mma(qr, kr, qk);
      }
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (sizeof(E) == 4) {
            kk = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[hh][j], ka[hh][j], kk, 0, 0, 0);
            qk = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[hh][j], ka[hh][j], qk, 0, 0, 0);
          }
#pragma unroll
          for (int vb = 0; vb < VB; ++vb) {
            sk[vb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[hh][j], s[2 * p + hh][vb][j], sk[vb], 0, 0, 0);
            sq[vb] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[hh][j], s[2 * p + hh][vb][j], sq[vb], 0, 0, 0);
          }
        }
    }
    // decay products for t = 4 g + j: gam = alpha_{m+1}..alpha_t, ge = alpha_0..alpha_t, gb = alpha_{t+1}..alpha_15
    f4 gam = {1.f, 1.f, 1.f, 1.f}, ge = gam, gb = gam;
    float gC = 1.f;
    if (la) {
      float al[RTB], pm = 1.f, suf = 1.f;
#pragma unroll
      for (int t = 0; t < RTB; t += 4) *(f4*)&al[t] = *(const f4*)&sm.gate[2][t];
#pragma unroll
      for (int t = 0; t < RTB; ++t) {
        gC *= al[t];
        pm = t > m ? pm * al[t] : 1.f;
        if (t >> 2 == g) {
          gam[t & 3] = pm;
          ge[t & 3] = gC;
        }
      }
#pragma unroll
      for (int t = RTB - 1; t >= 0; --t) {
        if (t >> 2 == g) gb[t & 3] = suf;
        suf *= al[t];
      }
    }
    const f4 be = *(const f4*)&sm.gate[0][4 * g], lm = *(const f4*)&sm.gate[1][4 * g];
    __syncthreads();                           // Q consumed: its room takes g_t S q_t
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = 4 * g + j;
      const bool in = t < nt;                  // no e past the end, whatever the repeated token holds
      sm.A[t][m] = in ? be[j] * gam[j] * (kk[j] + lm[j] * qk[j]) : 0.f;   // (right of the diagonal: not read)
      sm.Pm[t][m] = gam[j] * qk[j];
#pragma unroll
      for (int vb = 0; vb < VB; ++vb) {
        const float sqg = ge[j] * sq[vb][j];
        const float x = be[j] * (tof(sm.v[t][16 * vb + m]) - (ge[j] * sk[vb][j] + lm[j] * sqg));
        sm.x[t][16 * vb + m] = in ? x : 0.f;
        xq[t * LDX + 16 * vb + m] = sqg;
      }
    }
    __syncthreads();
    {
      // one value row per lane (with fewer rows than lanes the upper lanes
      // repeat the lower ones' work)
      const int r = lane % NV, row = v0 + r;
      float e[RTB], y[RTB];
#pragma unroll
      for (int t = 0; t < RTB; ++t) {
        REC_FENCE;
        float x0 = sm.x[t][r], x1 = 0.f, y0 = xq[t * LDX + r], y1 = 0.f;
#pragma unroll
        for (int i = 0; i < t; i += 4) {
          const f4 ac = *(const f4*)&sm.A[t][i], pc = *(const f4*)&sm.Pm[t][i];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (i + j < t) {
              (j & 1 ? x1 : x0) -= ac[j] * e[i + j];
              (j & 1 ? y1 : y0) += pc[j] * e[i + j];
            }
        }
        e[t] = x0 + x1;
        y[t] = y0 + sm.Pm[t][t] * e[t] + y1;
        asm volatile("" : "+v"(y[t]));         // formed here: sunk into the stores' branch it would hold every row of Pm
      }
      if (lane < NV && row < DV) {
        E* op = o + ((size_t)tb * H + h) * DV + row;
#pragma unroll
        for (int t = 0; t < RTB; ++t) {
          if (t < nt) *op = fromf<E>(y[t]);
          op += (size_t)H * DV;
        }
      }
#pragma unroll
      for (int t = 0; t < RTB; ++t)
        if (lane < NV) sm.x[t][r] = e[t];
    }
    __syncthreads();
    if (b + 1 < nblk) load_block(tb + RTB, lane);   // lands during the update
    // S^T <- g_C S^T + K^T diag(Gam_C) e
    f4 eb[VB];
#pragma unroll
    for (int vb = 0; vb < VB; ++vb)
#pragma unroll
      for (int j = 0; j < 4; ++j) eb[vb][j] = gb[j] * sm.x[4 * g + j][16 * vb + m];
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      if (kt % 2 == 0) REC_FENCE;
      const f4 kt4 = rec_tok4<E>(&sm.k[0][0], LDK, kt, lane);
#pragma unroll
      for (int vb = 0; vb < VB; ++vb) {
        f4 a = gC * s[kt][vb];
#pragma unroll
        for (int j = 0; j < 4; ++j) a = __builtin_amdgcn_mfma_f32_16x16x4f32(kt4[j], eb[vb][j], a, 0, 0, 0);
        s[kt][vb] = a;
      }
    }
    __syncthreads();                           // the block's LDS use is over
  }
  if (Sfin) {
#pragma unroll
    for (int vb = 0; vb < VB; ++vb) {
      const int row = v0 + 16 * vb + (lane0 & 15);
      if (row < DV) {
        float* dst = Sfin + ((size_t)u * DV + row) * DK + 8 * (lane0 >> 4);
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) *(f4*)(dst + 32 * (kt >> 1) + 4 * (kt & 1)) = s[kt][vb];
      }
    }
  }
}

hipError_t launch_rec_fwd(int N, int T, const int* cu, int T_total, int H, int Dk, int Dv,
                          int dtype, const void* q, const void* k, const void* v,
                          const float* beta, const float* lam, float lam_c, const float* la,
                          const float* S0, float* Sfin, void* o, hipStream_t st) {
  if (N == 0) return hipSuccess;
  if (!((dtype == 1 || dtype == 0) && (Dk == 128 || Dk == 64))) return hipErrorInvalidValue;
  // A few tokens per sequence go through the step kernel: many short waves
  // with one read and one write of the state overlap better than one round of
  // long ones, until its row sums cost more.  16 heads, d 128, 64 sequences:
  // bf16 T = 1 / 2 / 4 / 6 / 8: 22 / 24 / 28 / 34 / 41 us against 36 in blocks;
  // fp32 T = 4 / 6 / 8 / 10: 28 / 34 / 40 / 45 against 44; d_k 128, d_v 256, bf16
  // T = 4 / 6 / 8: 54 / 69 / 86 against 70; d 64 13 against 14 up to T = 6.  (The
  // lines stand at 4 and 6 from before the operands were loaded ahead; by these
  // times they could be at 6 and 8.)  Packed lengths are not known here: their
  // mean decides, and lower, since one long sequence walks alone: 63 of one
  // token and one of 65: d 128 bf16 67 us against 74 in blocks, fp32 68 against
  // 70, d 64 bf16 43 against 29 (one of 300: 233 against 212, fp32 245 against
  // 165, d 64 182 against 80).
  if (cu ? T_total <= 2LL * N : T >= 1 && T <= (dtype == 1 ? 4 : 6))
    return step_at(N, T, cu, T_total, H, Dk, Dv, dtype, q, k, v, beta, lam, lam_c, la, S0, Sfin, o, st);
  const int units = N * H;
  // Wide tiles once they are two waves per SIMD or more (bf16; from one per SIMD
  // on where a sequence has more than two blocks to walk) or half a wave per
  // SIMD (fp32), 16-row tiles below: there a wave's own chain of products is
  // the time.  16 heads, d 128, bf16, T = 16: 64 sequences 40.6 us in 16-row
  // tiles, 39.5 wide; 32: 23.6, 25.9; 8: 9.8, 14.8; T = 64: 64 sequences 121,
  // 88; 32: 65, 57; 16: 36, 49.  fp32, T = 16: 16 sequences 20.3, 15.4; 8: 10.8, 12.0.
  const long long t16 = (long long)units * ((Dv + 15) / 16), cus = device_cu_count();
  const bool lengthy = (cu ? T_total / N : T) > 2 * RTB;
  const bool wide = dtype == 1 ? t16 >= 32 * cus || (lengthy && t16 >= 16 * cus) : t16 >= 8 * cus;
  const int vb = !wide ? 1 : dtype == 1 && Dk == 128 ? rec_wide<__bf16, 128>() : 2;
  const int ntile = (Dv + 16 * vb - 1) / (16 * vb);
  dim3 grid((unsigned)((size_t)(units + 7) / 8 * 8 * ntile));
#define QD_REC(ET, DKV, VBV)                                                                        \
  hipLaunchKernelGGL((k_rec_fwd<ET, DKV, VBV>), grid, dim3(64), 0, st, T, H, Dv, units, ntile, cu, \
                     T_total, (const ET*)q, (const ET*)k, (const ET*)v, beta, lam, lam_c, la,  \
                     S0, Sfin, (ET*)o)
#define QD_REC_V(ET, DKV) \
  if (wide) QD_REC(ET, DKV, (rec_wide<ET, DKV>())); else QD_REC(ET, DKV, 1)
  prof_mark(ST_REC_FWD, 0, st);
  if (dtype == 1 && Dk == 128) { QD_REC_V(__bf16, 128); }
  else if (dtype == 1 && Dk == 64) { QD_REC_V(__bf16, 64); }
  else if (dtype == 0 && Dk == 128) { QD_REC_V(float, 128); }
  else { QD_REC_V(float, 64); }
  prof_mark(ST_REC_FWD, 1, st);
#undef QD_REC_V
#undef QD_REC
  return hipGetLastError();
}

}  // namespace qd
