// Backward of the fully recurrent form (Sec. 3.3, Eq. (qdelta_decay) token
// by token; the paper ships kernels for both the recurrent and the chunkwise
// form).  The paper states no backward; this is the chain rule through
//
//   x_t = k_t + lambda_t q_t,  e_t = beta_t (v_t - alpha_t S_{t-1} x_t),
//   S_t = alpha_t S_{t-1} + e_t k_t^T,  o_t = S_t q_t
//
// for L = <dO, o> + <dS_T, S_T>, in fp32, over blocks of 16 tokens (the
// recurrence unrolled within a block as in the forward, qd_step.hip).  With
// entry state S, exit-state gradient G, decay products g_t = alpha_1..alpha_t,
// Gam_ti = alpha_{i+1}..alpha_t, kb_i = Gam_Ci and rows t, i of the block:
//
//   A   = strictLower(diag(beta) Gam (.) X K^T),  M = (I + A)^{-1},  P = Gam (.) lower(Q K^T)
//   u_t = v_t - g_t S x_t,   e = M diag(beta) u
//   w   = M^T (P^T dO + diag(kb) K G^T)            (adjoint of beta u)
//   dv  = beta w
//   dA  = strictLower(-w e^T),  dG_ti = beta_t Gam_ti dA_ti,  dQK = Gam (.) lower(dO e^T)
//   dx_t = -beta_t g_t S^T w_t + sum_i dG_ti k_i
//   dq_t = g_t S^T dO_t + sum_i dQK_ti k_i + lambda_t dx_t,   dlambda_t = q_t . dx_t
//   dk_i = kb_i G^T e_i + sum_t dQK_ti q_t + sum_t dG_ti x_t + dx_i
//   dbeta_t = w_t . u_t + sum_i dA_ti Gam_ti (x_t . k_i)
//   dlog alpha_j = sum_{r>=j} (row_r - col_r of dG (.) X K^T + dQK (.) Q K^T)
//                + sum_{r>=j} g_r (dO_r . S q_r - beta_r w_r . S x_r)
//                + sum_{i<j} kb_i e_i . G k_i + g_C <G, S>
//   G  <- g_C G + sum_t g_t (dO_t - lambda_t beta_t w_t) q_t^T - sum_t g_t beta_t w_t k_t^T
//
// All contractions are fp32 matrix products (16x16x4).  One workgroup per
// (sequence, head), one wave per 16 value rows: a wave holds its rows of S and
// of G as (key x value) tiles in the matrix result layout, which is the
// operand layout of the products over the keys (S k, S q, G k) and of the
// update of G.  The products over the values (S^T w, S^T dO, G^T e) need the
// tiles the other way round and every wave's rows: S and G pass through LDS in
// pieces of 64 rows, and each wave forms its share of the key columns, so no
// sums cross waves.  Sums that do cross (w e^T, dO e^T, the token scalars)
// are added in wave order: the results are the same on every run.
//
// Sequences of more than one block are first walked forward, storing every
// rec_ckpt-th entry state; the reverse walk starts each block from the last
// stored state before it.
//
// A block is four products of 16 Dk Dv with S, two more for the gradient of the
// state before it and two with a gradient of the state after it (3.4 us each
// for 1024 units at d 128).  Bound by none of its resources alone but by the
// chain of its phases: 64 sequences x 16 heads x 16 tokens, d 128, bf16 (six
// products) keep the matrix cores 39% busy and move 169 MB at 3.0 TB/s, two
// workgroups to a CU; past one block there is one to a CU (64 tokens: 37% busy,
// 560 MB at 1.3 TB/s).  At d_v 256 sixteen waves leave 128 registers each, and
// the form of several blocks spills (63 bf16 and 51 fp32 at d_k 128, 4 at 64).
// Row sums on the vector ALU over three token sweeps took 196 us for 16 tokens
// and 680 for 64, this form takes 56 and 425.
#include "qd_common.h"
#include "qd_launch.h"

namespace qd {

namespace {

typedef unsigned int rb_u32x4 __attribute__((ext_vector_type(4)));

constexpr int RB_TB = 16;         // tokens per block

__device__ inline f4 mf(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// c += A B for 16 k values, four per lane (element j of every lane in step j)
__device__ inline f4 mf4(f4 a, f4 b, f4 c) {
#pragma unroll
  for (int j = 0; j < 4; ++j) c = mf(a[j], b[j], c);
  return c;
}

// Four consecutive values of an LDS row as fp32.
template <typename E>
__device__ inline f4 row4(const E* p) {
  if constexpr (sizeof(E) == 2) {
    const bf4 r = *(const bf4*)p;
    return f4{(float)r[0], (float)r[1], (float)r[2], (float)r[3]};
  } else {
    return *(const f4*)p;
  }
}
// Rows 4 (lane >> 4) .. +3 of column c0 + (lane & 15) of an LDS matrix.
template <typename E>
__device__ inline f4 col4(const E* p, int ld, int c0, int lane) {
  const int g = lane >> 4, L = lane & 15;
  if constexpr (sizeof(E) == 2) {
    typedef __attribute__((address_space(3))) bf4* lp;
    const E* a = p + (size_t)(4 * g + (L >> 2)) * ld + c0 + 4 * (L & 3);   // LDS transpose read
    const bf4 r = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lp)(uintptr_t)(uint32_t)(uintptr_t)a);
    return f4{(float)r[0], (float)r[1], (float)r[2], (float)r[3]};
  } else {
    f4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = p[(size_t)(4 * g + j) * ld + c0 + L];
    return r;
  }
}

// 16 token rows of D elements, staged through registers (rows past the end as zero).
template <typename E, int D, int NT>
struct Rows {
  static constexpr int VEC = 16 / (int)sizeof(E), PPR = D / VEC, PCS = RB_TB * PPR, N = (PCS + NT - 1) / NT;
  rb_u32x4 r[N];
  __device__ inline void load(const E* base, size_t stride, int tb, int t1, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = (tid + i * NT) % PCS, t = tb + idx / PPR;
      r[i] = *(const rb_u32x4*)(base + (size_t)min(t, t1 - 1) * stride + (idx % PPR) * VEC);
    }
  }
  __device__ inline void store(E* lds, int ld, int tb, int t1, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = tid + i * NT;
      if (idx < PCS)
        *(rb_u32x4*)(lds + (idx / PPR) * ld + (idx % PPR) * VEC) = tb + idx / PPR < t1 ? r[i] : rb_u32x4{0, 0, 0, 0};
    }
  }
};

// the kernel's lambdas are inlined before its arrays are given registers
#define RB_INLINE __attribute__((always_inline))

constexpr int RB_LM = 20;         // row stride of the 16 x 16 matrices

// Whether all four are finite: 0 * x is 0 for those, NaN for the others.
__device__ inline bool is_finite4(f4 x) {
  const f4 z = 0.f * x;
  return (z[0] + z[1]) + (z[2] + z[3]) == 0.f;
}

// acc + A r for a triangular 16 x 16 matrix in LDS (UPPER: zero left of the
// diagonal, else right of it) and r in the result layout.  The matrix product
// meets those zeros too, and a zero times a NaN or an infinity is a NaN: a
// wave whose r holds one goes by the sums over the triangle alone, so that no
// token reaches one on the other side of the diagonal.  (The checks of r and
// of A cost 1 to 3% of a call; checking the products instead cost 1 to 7%.)
template <bool UPPER>
__device__ inline f4 tri4(const float (*A)[RB_LM], f4 r, f4 acc, int lane) {
  const int g = lane >> 4, m = lane & 15;
  if (__all(is_finite4(r))) return mf4(*(const f4*)&A[m][4 * g], r, acc);
#pragma unroll 1
  for (int i = 0; i < RB_TB; i += 4)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float ri = lane_from(r[c], 4 * i + m);     // row i + c of this lane's column
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 4 * g + j;
        if (UPPER ? i + c >= t : i + c <= t) acc[j] += A[t][i + c] * ri;
      }
    }
  return acc;
}

}  // namespace

template <typename E, int DK, int DV>
struct alignas(16) RecBwdSmem {
  static constexpr int W = DV / 16, P = Pad<E>::v, LK = DK + P, LV = DV + P, LE = DV + 4, LX = DK + 4;
  static constexpr int PR = DV < 64 ? DV : 64;              // rows of S (or G) per piece
  static constexpr int XB = PR * LX * 4, PB = W * 2 * 64 * 16, GB = 3 * 64 * 16;
  alignas(16) E k[RB_TB][LK];
  alignas(16) E q[RB_TB][LK];
  alignas(16) E v[RB_TB][LV];
  alignas(16) E dO[RB_TB][LV];
  alignas(16) float eb[RB_TB][LE], wb[RB_TB][LE];           // e and w (token, value)
  // per-wave parts of w e^T, dO e^T and wave 0's X K^T, Q K^T, Gam; then pieces of S, G
  alignas(16) char x[XB > PB + GB ? XB : PB + GB];
  alignas(16) float M[RB_TB][RB_LM], MT[RB_TB][RB_LM], PT[RB_TB][RB_LM];
  alignas(16) float dG[RB_TB][RB_LM], dGT[RB_TB][RB_LM];    // dGT also holds A^T while M is formed
  alignas(16) float dQK[RB_TB][RB_LM], GLT[RB_TB][RB_LM];   // dQK; (dQK + diag(lambda) dG)^T
  alignas(16) float beta[RB_TB], lam[RB_TB], al[RB_TB], ge[RB_TB], gb[RB_TB];
  alignas(16) float sc[W][3][RB_TB];                        // token scalars per wave
  alignas(16) float row[RB_TB], col[RB_TB], db[RB_TB], s2[RB_TB], s3[RB_TB];
  float dl[W][RB_TB], gs[W], gC;
};

// ONE: every sequence has at most one block (T <= 16): G is then dSfin, read
// where it is used, and takes no registers, so that two workgroups share a CU
// at d 128 (under 80 KB of LDS and 128 registers each).
template <typename E, int DK, int DV, bool ONE>
__global__ __launch_bounds__(DV * 4) __attribute__((amdgpu_waves_per_eu(ONE ? 4 : 2))) void k_rec_bwd(RecBwdArgs a) {
  typedef RecBwdSmem<E, DK, DV> SM;
  constexpr int W = SM::W, NT = DV * 4, NKT = DK / 16;
  constexpr int KPW = (NKT + W - 1) / W;       // key tiles per wave in the products over the values
  constexpr int CK = rec_ckpt(DK, DV);
  __shared__ SM sm;
  const int H = a.H, unit = blockIdx.x, n = unit / H, h = unit % H;
  const int w = wave_id(threadIdx.x), v0 = 16 * w, kt0 = w * KPW;
  // laundered at every phase, so that addresses are formed where they are
  // used instead of being kept in registers through the whole loop
  int tid = threadIdx.x, lane, g, m;
  auto fresh = [&]() RB_INLINE {
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    g = lane >> 4;
    m = lane & 15;
  };
  auto sync = [&]() RB_INLINE {
    block_sync_lds();
    fresh();
  };
  fresh();
  int t0, t1;
  if (a.cu) {
    t0 = min(max(a.cu[n], 0), a.T_total);
    t1 = min(max(a.cu[n + 1], t0), a.T_total);
  } else {
    t0 = n * a.T;
    t1 = t0 + a.T;
  }
  if (a.skip > 0 && t1 - t0 <= a.skip) return;
  const int nblk = (t1 - t0 + RB_TB - 1) / RB_TB;
  const E* const qp = (const E*)a.q + (size_t)h * DK;
  const E* const kp = (const E*)a.k + (size_t)h * DK;
  const E* const vp = (const E*)a.v + (size_t)h * DV;
  const E* const op = (const E*)a.dO + (size_t)h * DV;

  // tiles: s[kt][j] = S[v0 + m][16 kt + 4 g + j]
  f4 s[NKT], gt[ONE ? 1 : NKT];
  auto load_tiles = [&](f4 (&x)[NKT], const float* src) RB_INLINE {     // src: [DV][DK] of this unit, or nullptr
    if (src) {
      src += (size_t)(v0 + m) * DK + 4 * g;
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) x[kt] = *(const f4*)(src + 16 * kt);
    } else {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) x[kt] = zero4();
    }
  };
  auto store_tiles = [&](const f4 (&x)[NKT], float* dst) RB_INLINE {
    dst += (size_t)(v0 + m) * DK + 4 * g;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) *(f4*)(dst + 16 * kt) = x[kt];
  };
  const float* const S0 = a.S0 ? a.S0 + (size_t)unit * DV * DK : nullptr;
  // entry state of block c CK (c >= 1), at token t0 + 16 c CK: no two of a batch share a multiple of 16 CK tokens
  auto ckpt = [&](int c) RB_INLINE { return a.wS + ((size_t)(t0 / (RB_TB * CK) + c - 1) * H + h) * DV * DK; };

  // one block's inputs: into registers, then into LDS
  struct Block {
    Rows<E, DK, NT> k, q;
    Rows<E, DV, NT> v, dO;
    float be, lm, al;
  };
  auto fetch = [&](Block& x, int tb, bool with_dO) RB_INLINE {
    x.k.load(kp, (size_t)H * DK, tb, t1, tid);
    x.q.load(qp, (size_t)H * DK, tb, t1, tid);
    x.v.load(vp, (size_t)H * DV, tb, t1, tid);
    if (with_dO) x.dO.load(op, (size_t)H * DV, tb, t1, tid);
    const size_t at = (size_t)min(tb + (tid & 15), t1 - 1) * H + h;
    x.be = a.beta[at];
    x.lm = a.lam ? a.lam[at] : a.lam_c;
    x.al = a.la ? a.la[at] : 0.f;
  };
  auto stage = [&](const Block& x, int tb, bool with_dO) RB_INLINE {
    x.k.store(&sm.k[0][0], SM::LK, tb, t1, tid);
    x.q.store(&sm.q[0][0], SM::LK, tb, t1, tid);
    x.v.store(&sm.v[0][0], SM::LV, tb, t1, tid);
    if (with_dO) x.dO.store(&sm.dO[0][0], SM::LV, tb, t1, tid);
    if (tid < RB_TB) {
      // gates past the end: beta 0, alpha 1 (nothing changes)
      const bool in = tb + tid < t1;
      sm.beta[tid] = in ? x.be : 0.f;
      sm.lam[tid] = x.lm;
      sm.al[tid] = in && a.la ? __expf(x.al) : 1.f;
    }
  };

  // wave 0, rows t = 4 g + j and column m: K K^T, Q K^T, the decay products;
  // A, M, and (transposed) P
  auto gram = [&]() RB_INLINE {
    f4 kk = zero4(), qk = zero4();
    if constexpr (sizeof(E) == 2) {            // products of bf16 inputs are exact in fp32
#pragma unroll
      for (int c = 0; c < DK; c += 32) {
        const bf8 kr = *(const bf8*)&sm.k[m][c + 8 * g], qr = *(const bf8*)&sm.q[m][c + 8 * g];
        kk = Mma<E>::mma(kr, kr, kk);
        qk = Mma<E>::mma(qr, kr, qk);
      }
    } else {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        const f4 kr = row4(&sm.k[m][16 * kt + 4 * g]), qr = row4(&sm.q[m][16 * kt + 4 * g]);
        kk = mf4(kr, kr, kk);
        qk = mf4(qr, kr, qk);
      }
    }
    f4 ge = {1.f, 1.f, 1.f, 1.f}, gb = ge, gam = ge;
    float gC = 1.f, pm = 1.f, suf = 1.f;
    float al[RB_TB];
#pragma unroll
    for (int t = 0; t < RB_TB; t += 4) *(f4*)&al[t] = *(const f4*)&sm.al[t];
#pragma unroll
    for (int t = 0; t < RB_TB; ++t) {
      gC *= al[t];
      pm = t > m ? pm * al[t] : 1.f;
      if (t >> 2 == g) {
        gam[t & 3] = pm;
        ge[t & 3] = gC;
      }
    }
#pragma unroll
    for (int t = RB_TB - 1; t >= 0; --t) {
      if (t >> 2 == g) gb[t & 3] = suf;
      suf *= al[t];
    }
    const f4 be = *(const f4*)&sm.beta[4 * g], lm = *(const f4*)&sm.lam[4 * g];
    f4 pt, at, xk;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = 4 * g + j;
      xk[j] = kk[j] + lm[j] * qk[j];
      at[j] = t > m ? be[j] * gam[j] * xk[j] : 0.f;
      pt[j] = t >= m ? gam[j] * qk[j] : 0.f;
    }
    const bool finite = __all(is_finite4(at));
    *(f4*)&sm.dGT[m][4 * g] = at;              // A^T
    *(f4*)&sm.PT[m][4 * g] = pt;
    f4* const keep = (f4*)(sm.x + SM::PB) + lane;
    keep[0] = xk;
    keep[64] = qk;
    keep[128] = gam;
    if (m == 0) {
      *(f4*)&sm.ge[4 * g] = ge;
      *(f4*)&sm.gb[4 * g] = gb;
      if (g == 0) sm.gC = gC;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (lane < RB_TB && finite) {
      // column m of M by substitution, column i of A read one step ahead
      float x[RB_TB];
#pragma unroll
      for (int r = 0; r < RB_TB; ++r) x[r] = r == m ? 1.f : 0.f;
      f4 cur[4], nxt[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) cur[c] = *(const f4*)&sm.dGT[0][4 * c];
#pragma unroll
      for (int i = 0; i + 1 < RB_TB; ++i) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = (i + 2) / 4; c < 4; ++c) nxt[c] = *(const f4*)&sm.dGT[i + 1][4 * c];
#pragma unroll
        for (int r = i + 1; r < RB_TB; ++r) x[r] -= cur[r >> 2][r & 3] * x[i];
#pragma unroll
        for (int c = (i + 2) / 4; c < 4; ++c) cur[c] = nxt[c];
      }
#pragma unroll
      for (int r = 0; r < RB_TB; ++r) sm.M[r][m] = x[r];
#pragma unroll
      for (int r = 0; r < RB_TB; r += 4) *(f4*)&sm.MT[m][r] = f4{x[r], x[r + 1], x[r + 2], x[r + 3]};
    } else if (lane < RB_TB) {
      // the same without the terms above the column's diagonal, whose zeros an A that is not finite must not meet
#pragma unroll 1
      for (int r = 0; r < RB_TB; ++r) {
        float x = r == m ? 1.f : 0.f;
#pragma unroll 1
        for (int i = m; i < r; ++i) x -= sm.dGT[i][r] * sm.M[i][m];
        sm.M[r][m] = x;
        sm.MT[m][r] = x;
      }
    }
  };
  // S k_t, S q_t (rows t, this wave's value columns)
  auto state_products = [&](f4& sk, f4& sq) RB_INLINE {
    sk = sq = zero4();
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      const f4 ka = row4(&sm.k[m][16 * kt + 4 * g]), qa = row4(&sm.q[m][16 * kt + 4 * g]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sk = mf(ka[j], s[kt][j], sk);
        sq = mf(qa[j], s[kt][j], sq);
      }
    }
  };
  // S over the block starting at token tb (forward)
  auto advance = [&](int tb) RB_INLINE {
    Block x;
    fetch(x, tb, false);
    sync();                                    // the LDS use of the step before is over
    stage(x, tb, false);
    sync();
    f4 sk, sq;
    if (w == 0) gram();
    state_products(sk, sq);
    sync();
    const f4 be = *(const f4*)&sm.beta[4 * g], lm = *(const f4*)&sm.lam[4 * g];
    const f4 ge = *(const f4*)&sm.ge[4 * g], gb = *(const f4*)&sm.gb[4 * g];
    f4 r, e;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = be[j] * (tof(sm.v[4 * g + j][v0 + m]) - ge[j] * (sk[j] + lm[j] * sq[j]));
    e = mf4(*(const f4*)&sm.M[m][4 * g], r, zero4());
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] *= gb[j];
    const float gC = sm.gC;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) s[kt] = mf4(col4(&sm.k[0][0], SM::LK, 16 * kt, lane), e, gC * s[kt]);
  };

  const float* const Gf = a.dSfin ? a.dSfin + (size_t)unit * DV * DK : nullptr;
  if constexpr (!ONE) load_tiles(gt, Gf);
  auto G = [&](int kt) RB_INLINE {             // tile kt of G (only while has_g)
    if constexpr (ONE) return *(const f4*)(Gf + (size_t)(v0 + m) * DK + 16 * kt + 4 * g);
    else return gt[kt];
  };
  bool has_g = a.dSfin != nullptr;             // G is not known to be zero
  const int last0 = nblk > 0 ? (nblk - 1) / CK * CK : 0;      // first block of the last group
  if constexpr (!ONE) {
    if (last0 > 0) {
      load_tiles(s, S0);
      for (int b = 0; b < last0; ++b) {
        advance(t0 + b * RB_TB);
        if ((b + 1) % CK == 0) store_tiles(s, ckpt((b + 1) / CK));
      }
    }
  }
  for (int b = nblk - 1; b >= 0; --b) {
    const int tb = t0 + b * RB_TB, nt = min(RB_TB, t1 - tb), c = b / CK;
    Block x;
    fetch(x, tb, true);
    if constexpr (ONE) {
      load_tiles(s, S0);
    } else {
      if (!(b == last0 && b == nblk - 1 && b > 0)) load_tiles(s, c > 0 ? ckpt(c) : S0);   // else just walked to it
      for (int f = c * CK; f < b; ++f) advance(t0 + f * RB_TB);
    }
    sync();
    stage(x, tb, true);
    sync();
    f4 sk, sq, gk = zero4();
    if (w == 0) gram();
    state_products(sk, sq);
    float gsum = 0.f;
    if (has_g) {
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        const f4 x = G(kt);
        gk = mf4(row4(&sm.k[m][16 * kt + 4 * g]), x, gk);
#pragma unroll
        for (int j = 0; j < 4; ++j) gsum += x[j] * s[kt][j];
      }
    }
    sync();                          // gates, M, P visible
    const f4 be = *(const f4*)&sm.beta[4 * g], lm = *(const f4*)&sm.lam[4 * g];
    const f4 ge = *(const f4*)&sm.ge[4 * g], gb = *(const f4*)&sm.gb[4 * g];
    const float gC = sm.gC;
    f4 z1, z2;
    {
      f4 u, r, dO, dd, wv;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u[j] = tof(sm.v[4 * g + j][v0 + m]) - ge[j] * (sk[j] + lm[j] * sq[j]);
        r[j] = be[j] * u[j];
        dO[j] = tof(sm.dO[4 * g + j][v0 + m]);
        dd[j] = gb[j] * gk[j];
      }
      const f4 e = tri4<false>(sm.M, r, zero4(), lane);
      dd = tri4<true>(sm.PT, dO, dd, lane);
      wv = tri4<true>(sm.MT, dd, zero4(), lane);
      f4 s1, s2, s3;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 4 * g + j;
        const float bw = be[j] * wv[j];
        sm.eb[t][v0 + m] = e[j];
        sm.wb[t][v0 + m] = wv[j];
        if (t < nt) ((E*)a.dv)[((size_t)(tb + t) * H + h) * DV + v0 + m] = fromf<E>(bw);
        s1[j] = sum16(wv[j] * u[j]);
        s2[j] = sum16(ge[j] * (dO[j] * sq[j] - bw * (sk[j] + lm[j] * sq[j])));
        s3[j] = sum16(gb[j] * e[j] * gk[j]);
        z1[j] = ge[j] * (dO[j] - lm[j] * bw);
        z2[j] = -ge[j] * bw;
      }
      if (m == 0) {
        *(f4*)&sm.sc[w][0][4 * g] = s1;
        *(f4*)&sm.sc[w][1][4 * g] = s2;
        *(f4*)&sm.sc[w][2][4 * g] = s3;
      }
      gsum = wave_sum_l(gsum, lane);
      if (lane == 0) sm.gs[w] = gsum;
      // this wave's parts of w e^T and dO e^T (its own columns, just written)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const f4 er = *(const f4*)&sm.eb[m][v0 + 4 * g];
      f4* const part = (f4*)sm.x + w * 128 + lane;
      part[0] = mf4(*(const f4*)&sm.wb[m][v0 + 4 * g], er, zero4());
      part[64] = mf4(row4(&sm.dO[m][v0 + 4 * g]), er, zero4());
    }
    sync();                          // e, w and the parts visible
    if (w == 0) {
      // dG, dQK and their transposed forms; decay and beta terms
      f4 da = zero4(), dp = zero4(), dg, dqk, gl, row, db;
#pragma unroll 4
      for (int i = 0; i < W; ++i) {
        da -= ((const f4*)sm.x)[i * 128 + lane];
        dp += ((const f4*)sm.x)[i * 128 + 64 + lane];
      }
      const f4* const keep = (const f4*)(sm.x + SM::PB) + lane;
      const f4 xk = keep[0], qk = keep[64], gam = keep[128];
      // token scalars: lane (g, t = m) adds kind g over the waves
      float sv = 0.f;
#pragma unroll
      for (int i = 0; i < W; ++i) sv += sm.sc[i][min(g, 2)][m];
      if (g == 1) sm.s2[m] = sv;
      if (g == 2) sm.s3[m] = sv;
      float cs = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 4 * g + j;
        const float dag = t > m ? da[j] * gam[j] : 0.f;
        dg[j] = be[j] * dag;
        dqk[j] = t >= m ? dp[j] * gam[j] : 0.f;
        gl[j] = dqk[j] + lm[j] * dg[j];
        sm.dG[t][m] = dg[j];
        sm.dQK[t][m] = dqk[j];
        const float tt = dg[j] * xk[j] + dqk[j] * qk[j];
        cs += tt;
        row[j] = sum16(tt);
        db[j] = sum16(dag * xk[j]);
      }
      *(f4*)&sm.dGT[m][4 * g] = dg;
      *(f4*)&sm.GLT[m][4 * g] = gl;
      cs += lane_xor(cs, 16, lane);
      cs += lane_xor(cs, 32, lane);
      if (g == 0) sm.col[m] = cs;
      if (m == 0) {
        *(f4*)&sm.row[4 * g] = row;
        *(f4*)&sm.db[4 * g] = db;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (lane < nt) {
        const size_t at = (size_t)(tb + lane) * H + h;
        a.dbeta[at] = sv + sm.db[m];
        if (a.dla) {
          float acc = 0.f;
#pragma unroll
          for (int i = 0; i < W; ++i) acc += sm.gs[i];
          acc *= gC;
#pragma unroll
          for (int r = 0; r < RB_TB; r += 4) {
            const f4 x = *(const f4*)&sm.row[r] - *(const f4*)&sm.col[r] + *(const f4*)&sm.s2[r], y = *(const f4*)&sm.s3[r];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc += r + j >= m ? x[j] : y[j];
          }
          a.dla[at] = acc;
        }
      }
    }
    sync();                          // the parts are read: their room takes the pieces
    // products over the values, this wave's key tiles (rows k, columns t = m)
    f4 aq[KPW], aw[KPW], ak[KPW];
#pragma unroll
    for (int i = 0; i < KPW; ++i) aq[i] = aw[i] = ak[i] = zero4();
    float* const X = (float*)sm.x;
    auto put_piece = [&](auto tile, int pc) RB_INLINE {
      if (v0 / SM::PR == pc) {
        float* dst = X + (v0 % SM::PR + m) * SM::LX + 4 * g;
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) *(f4*)(dst + 16 * kt) = tile(kt);
      }
    };
    auto x_col = [&](int vb, int kt) RB_INLINE {
      f4 r;
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = X[(16 * vb + 4 * g + j) * SM::LX + 16 * kt + m];
      return r;
    };
    for (int pc = 0; pc < DV / SM::PR; ++pc) {
      if (pc > 0) sync();
      put_piece([&](int kt) RB_INLINE { return s[kt]; }, pc);
      sync();
#pragma unroll
      for (int vb = 0; vb < SM::PR / 16; ++vb) {
        const int vc = pc * SM::PR + 16 * vb + 4 * g;
        const f4 zo = row4(&sm.dO[m][vc]), zw = *(const f4*)&sm.wb[m][vc];
#pragma unroll
        for (int i = 0; i < KPW; ++i)
          if (kt0 + i < NKT) {
            const f4 x = x_col(vb, kt0 + i);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              aq[i] = mf(x[j], zo[j], aq[i]);
              aw[i] = mf(x[j], zw[j], aw[i]);
            }
          }
      }
    }
    if (has_g) {
      for (int pc = 0; pc < DV / SM::PR; ++pc) {
        sync();
        put_piece(G, pc);
        sync();
#pragma unroll
        for (int vb = 0; vb < SM::PR / 16; ++vb) {
          const f4 ze = *(const f4*)&sm.eb[m][pc * SM::PR + 16 * vb + 4 * g];
#pragma unroll
          for (int i = 0; i < KPW; ++i)
            if (kt0 + i < NKT) ak[i] = mf4(x_col(vb, kt0 + i), ze, ak[i]);
        }
      }
    }
    {
      // dx, dq, dk of this wave's key tiles: lane token m, keys 16 kt + 4 g ..
      const float gm = sm.ge[m], bm = sm.beta[m], lmm = sm.lam[m], kbm = sm.gb[m];
      float dl = 0.f;
#pragma unroll
      for (int i = 0; i < KPW; ++i)
        if (kt0 + i < NKT) {
          const int kc = 16 * (kt0 + i);
          const f4 kT = col4(&sm.k[0][0], SM::LK, kc, lane), qT = col4(&sm.q[0][0], SM::LK, kc, lane);
          const f4 qr = row4(&sm.q[m][kc + 4 * g]);
          const f4 dx = mf4(kT, *(const f4*)&sm.dG[m][4 * g], (-bm * gm) * aw[i]);
          f4 dq = mf4(kT, *(const f4*)&sm.dQK[m][4 * g], gm * aq[i]);
          f4 dk = mf4(kT, *(const f4*)&sm.dGT[m][4 * g], kbm * ak[i]);
          dk = mf4(qT, *(const f4*)&sm.GLT[m][4 * g], dk);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            dl += qr[j] * dx[j];
            dq[j] += lmm * dx[j];
            dk[j] += dx[j];
          }
          if (m < nt) {
            const size_t at = ((size_t)(tb + m) * H + h) * DK + kc + 4 * g;
            *(typename Quad<E>::raw*)((E*)a.dq + at) = Quad<E>::pack(dq);
            *(typename Quad<E>::raw*)((E*)a.dk + at) = Quad<E>::pack(dk);
          }
        }
      dl += lane_xor(dl, 16, lane);
      dl += lane_xor(dl, 32, lane);
      if (lane < RB_TB) sm.dl[w][lane] = dl;
    }
    if (b > 0 || a.dS0) {
      // G <- g_C G + Q^T z1 + K^T z2 (key rows, this wave's value columns)
      float* const dst = ONE ? a.dS0 + ((size_t)unit * DV + v0 + m) * DK + 4 * g : nullptr;
#pragma unroll
      for (int kt = 0; kt < NKT; ++kt) {
        f4 x = has_g ? gC * G(kt) : zero4();
        x = mf4(col4(&sm.q[0][0], SM::LK, 16 * kt, lane), z1, x);
        x = mf4(col4(&sm.k[0][0], SM::LK, 16 * kt, lane), z2, x);
        if constexpr (ONE) *(f4*)(dst + 16 * kt) = x;
        else gt[kt] = x;
      }
      has_g = true;
    }
    sync();
    if (tid < nt) {
      float dl = 0.f;
#pragma unroll
      for (int i = 0; i < W; ++i) dl += sm.dl[i][tid];
      const size_t at = (size_t)(tb + tid) * H + h;
      if (a.dlam) a.dlam[at] = dl;
      if (a.wDL) a.wDL[at] = dl;
    }
  }
  if (a.dS0 && (!ONE || nblk == 0)) {          // (no block: G passes through)
    float* const dst = a.dS0 + ((size_t)unit * DV + v0 + m) * DK + 4 * g;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) *(f4*)(dst + 16 * kt) = ONE && !has_g ? zero4() : G(kt);
  }
}

// Sum of n floats in a fixed order (one workgroup: strided per-thread sums,
// then a tree), written to *out.
__global__ __launch_bounds__(NTHREADS) void k_sum_floats(const float* x, long long n, float* out) {
  __shared__ float part[NTHREADS];
  const int tid = threadIdx.x;
  float acc = 0.f;
  for (long long i = tid; i < n; i += NTHREADS) acc += x[i];
  part[tid] = acc;
  __syncthreads();
#pragma unroll
  for (int off = NTHREADS / 2; off >= 1; off >>= 1) {
    if (tid < off) part[tid] += part[tid + off];
    __syncthreads();
  }
  if (tid == 0) *out = part[0];
}

hipError_t launch_rec_bwd(const RecBwdArgs& a, int units, int dtype, int Dk, float* dlam_sum, long long n_tok_heads,
                          hipStream_t st) {
  if (units > 0) {
    // Sequences of a few tokens go to launch_rec_bwd_few: up to two, or four
    // at d_k 64, d_v 256 (where a workgroup here takes a whole CU) while there
    // are more of them than CUs.  The lengths of a packed batch are not known
    // here: while their mean is within that and there are more units than CUs,
    // both are launched, each for its sequences; below, where nothing but the
    // launch and the longest sequence counts, these kernels take them all
    // (packed, d 128, bf16: 64 x 16 units of one token 38 us in both launches,
    // 77 in one; 63 of one and one of 65 tokens 171, 190; 16 x 16 units, 15 of
    // one token and one of 17, 71, 47).  Past that they take a packed batch in
    // one launch also where its mean is within a block: the one-block form and
    // the other one after each other take 61 us instead of 79 where all 64
    // sequences have 3 to 16 tokens, but 327 instead of 270 where a quarter have
    // 40 and a quarter 17 (and 29 instead of 27, 104 instead of 79 at d 64).
    const bool full = units > device_cu_count();
    const int limit = Dk == 64 && a.DV == 256 && full ? 4 : 2;
    const bool few = a.cu ? full && a.T_total <= (long long)limit * (units / a.H) : a.T >= 1 && a.T <= limit;
    if (few) {
      prof_mark(ST_REC_BWD, 0, st);
      const hipError_t e = launch_rec_bwd_few(a, units, dtype, Dk, a.cu ? limit : a.T, st);
      prof_mark(ST_REC_BWD, 1, st);
      if (e != hipSuccess) return e;
    }
    RecBwdArgs b = a;
    b.skip = few ? limit : 0;
    const bool one = !a.cu && a.T <= RB_TB, rest = !few || (a.cu && a.T_total > limit);
#define QD_RB(ET, DKV, DVV)                                                                              \
  do {                                                                                                   \
    if (one) hipLaunchKernelGGL((k_rec_bwd<ET, DKV, DVV, true>), dim3(units), dim3(DVV * 4), 0, st, b);  \
    else hipLaunchKernelGGL((k_rec_bwd<ET, DKV, DVV, false>), dim3(units), dim3(DVV * 4), 0, st, b);     \
  } while (0)
#define QD_RB_V(ET, DKV)                                                                      \
  if (a.DV == 256) QD_RB(ET, DKV, 256); else if (a.DV == 128) QD_RB(ET, DKV, 128);            \
  else if (a.DV == 64) QD_RB(ET, DKV, 64); else QD_RB(ET, DKV, 32)
    if (rest) {
      prof_mark(ST_REC_BWD, 0, st);
      if (dtype == 1 && Dk == 128) { QD_RB_V(__bf16, 128); }
      else if (dtype == 1 && Dk == 64) { QD_RB_V(__bf16, 64); }
      else if (dtype == 0 && Dk == 128) { QD_RB_V(float, 128); }
      else { QD_RB_V(float, 64); }
      prof_mark(ST_REC_BWD, 1, st);
    }
#undef QD_RB_V
#undef QD_RB
  }
  if (dlam_sum) hipLaunchKernelGGL(k_sum_floats, dim3(1), dim3(NTHREADS), 0, st, a.wDL, n_tok_heads, dlam_sum);
  return hipGetLastError();
}

}  // namespace qd
