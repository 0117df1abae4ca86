// Backward of the fully recurrent form for sequences of at most NTOK (1, 2 or
// 4) tokens: the block formulas of qd_rec_bwd.hip with the token products on
// the vector ALU.  A block there has 16 tokens whatever the sequence has, and
// holds a CU with one or two workgroups; with so few tokens the call is bound
// by the states it reads and writes, so what counts is many rows in flight.
//
// One workgroup per (sequence, head).  A state row is owned by 16 lanes, which
// hold its entry state S and exit-state gradient G once: S k, S q and G k are
// row dot products, e and w follow by substitution per row (a token never
// meets another one's zero), the new G goes straight out, and the column sums
// S^T dO, S^T w and G^T e and the token products w e^T, dO e^T and <G, S> are
// kept per lane until the last row.  Sums over lanes, waves and rows are in a
// fixed order: the results are the same on every run.
//
// 64 sequences x 16 heads, bf16, one token / two: d 128 30.1 / 37.2 us against
// 54.6 / 54.9 in blocks of 16 and 58 / 66 in token sweeps; d_k 128, d_v 64
// 22.5 / 29.4 against 38.0 / 38.3 and 33.0 / 38.2; d_k 64, d_v 256 28.1 / 39.2
// against 79 / 81 and 57 / 66 (three and four tokens 55 / 58, 82 / 82, 75 / 84).
// The states alone, 134 MB at d 128, take 26 us at the rate of a large copy.
#include "qd_common.h"
#include "qd_launch.h"

namespace qd {

namespace {

__device__ inline float uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

}  // namespace

template <int DK, int NTOK>
struct alignas(16) RecFewSmem {
  static constexpr int NW = NTHREADS / 64, NP = NTOK * NTOK;
  static constexpr int NS = 3 * NTOK + 2 * NP + 1;           // s1, s2, s3, w e^T, dO e^T, <G, S>
  alignas(16) float k[NTOK][DK], q[NTOK][DK];
  alignas(16) float v[NTOK][256], dO[NTOK][256];             // v, then its gradient
  float part[NW][3 * NTOK][DK];                              // column sums per wave: S^T dO, S^T w, G^T e
  float sc[NW][NS], tot[NS];
  float kk[NTOK][NTOK], qk[NTOK][NTOK], dG[NTOK][NTOK], dQK[NTOK][NTOK], gam[NTOK][NTOK];
  float beta[NTOK], lam[NTOK], al[NTOK], ge[NTOK], kb[NTOK], dl[NTOK][2], gC;
};

template <typename E, int DK, int NTOK>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(NTOK == 4 ? 3 : 1))) void k_rec_bwd_few(
    RecBwdArgs a) {
  typedef RecFewSmem<DK, NTOK> SM;
  typedef Quad<E> QE;
  constexpr int NG = NTHREADS / 16;            // groups of 16 lanes, a row each
  constexpr int NJ = DK / 64;                  // pieces of four columns per lane: 64 j + 4 l ..
  constexpr int RC = NTOK == 4 ? 1 : 2;        // rows per lane group and pass
  constexpr int NW = SM::NW;
  __shared__ SM sm;
  const int H = a.H, DV = a.DV, unit = blockIdx.x, n = unit / H, h = unit % H;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l = tid & 15, grp = tid >> 4;
  const float* const S0 = a.S0 ? a.S0 + (size_t)unit * DV * DK : nullptr;
  const float* const Gf = a.dSfin ? a.dSfin + (size_t)unit * DV * DK : nullptr;
  float* const dS0 = a.dS0 ? a.dS0 + (size_t)unit * DV * DK : nullptr;
  auto load_rows = [&](f4 (&x)[RC][NJ], const float* src, int r0) {
    if (src) {
#pragma unroll
      for (int i = 0; i < RC; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) x[i][j] = *(const f4*)(src + (size_t)(r0 + NG * i + grp) * DK + 64 * j + 4 * l);
    } else {
#pragma unroll
      for (int i = 0; i < RC; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) x[i][j] = zero4();
    }
  };
  // the first rows are on their way while the bounds and the tokens are read
  f4 s[RC][NJ], g[RC][NJ];
  load_rows(s, S0, 0);
  load_rows(g, Gf, 0);
  int t0, t1;
  if (a.cu) {
    t0 = min(max(a.cu[n], 0), a.T_total);
    t1 = min(max(a.cu[n + 1], t0), a.T_total);
  } else {
    t0 = n * a.T;
    t1 = t0 + a.T;
  }
  const int nt = t1 - t0;
  if (nt > NTOK) return;                       // (a longer sequence of a packed batch: the other launch's)
  if (nt == 0) {                               // no token: G passes through
    if (dS0)
      for (int r0 = 0; r0 < DV; r0 += NG * RC) {
        if (r0 > 0) load_rows(g, Gf, r0);
#pragma unroll
        for (int i = 0; i < RC; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) *(f4*)(dS0 + (size_t)(r0 + NG * i + grp) * DK + 64 * j + 4 * l) = g[i][j];
      }
    return;
  }

  // tokens into LDS as fp32; those past the end as zeros with alpha 1
  auto rows_in = [&](const void* src, float* dst, int D, int ld) {
    for (int idx = tid; idx < NTOK * D / 4; idx += NTHREADS) {
      const int t = idx / (D / 4), c = 4 * (idx % (D / 4));
      f4 x = zero4();
      if (t < nt) {
        const auto r = *(const typename QE::raw*)((const E*)src + ((size_t)(t0 + t) * H + h) * D + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = QE::get(r, j);
      }
      *(f4*)(dst + t * ld + c) = x;
    }
  };
  rows_in(a.k, &sm.k[0][0], DK, DK);
  rows_in(a.q, &sm.q[0][0], DK, DK);
  rows_in(a.v, &sm.v[0][0], DV, 256);
  rows_in(a.dO, &sm.dO[0][0], DV, 256);
  if (tid < NTOK) {
    const bool in = tid < nt;
    const size_t at = (size_t)(t0 + (in ? tid : 0)) * H + h;
    sm.beta[tid] = in ? a.beta[at] : 0.f;
    sm.lam[tid] = a.lam ? a.lam[at] : a.lam_c;
    sm.al[tid] = in && a.la ? __expf(a.la[at]) : 1.f;
  }
  __syncthreads();
  if (grp < NTOK * NTOK) {                     // K K^T and Q K^T, a pair of tokens per lane group
    const int t = grp / NTOK, i = grp % NTOK;
    float x = 0.f, y = 0.f;
#pragma unroll
    for (int c = 0; c < DK / 16; ++c) {
      const float ki = sm.k[i][16 * c + l];
      x += sm.k[t][16 * c + l] * ki;
      y += sm.q[t][16 * c + l] * ki;
    }
    x = sum16(x);
    y = sum16(y);
    if (l == 0) {
      sm.kk[t][i] = x;
      sm.qk[t][i] = y;
    }
  }
  if (tid == 0) {                              // decay products: multiplied up, alpha = 0 is exact
    float p = 1.f;
    for (int t = 0; t < NTOK; ++t) sm.ge[t] = p *= sm.al[t];
    sm.gC = p;
    p = 1.f;
    for (int t = NTOK - 1; t >= 0; --t) {
      sm.kb[t] = p;
      p *= sm.al[t];
    }
    for (int i = 0; i < NTOK; ++i) {
      p = 1.f;
      for (int t = i; t < NTOK; ++t) {
        if (t > i) p *= sm.al[t];
        sm.gam[t][i] = p;
      }
    }
  }
  __syncthreads();
  // the tokens' coefficients: the same for every row, so in scalar registers
  float be[NTOK], lm[NTOK], ge[NTOK], kb[NTOK], A[NTOK][NTOK], P[NTOK][NTOK];
#pragma unroll
  for (int t = 0; t < NTOK; ++t) {
    be[t] = uniform(sm.beta[t]);
    lm[t] = uniform(sm.lam[t]);
    ge[t] = uniform(sm.ge[t]);
    kb[t] = uniform(sm.kb[t]);
#pragma unroll
    for (int i = 0; i <= t; ++i) {
      A[t][i] = i < t ? uniform(sm.beta[t] * sm.gam[t][i] * (sm.kk[t][i] + sm.lam[t] * sm.qk[t][i])) : 0.f;
      P[t][i] = uniform(sm.gam[t][i] * sm.qk[t][i]);
    }
  }
  const float gC = uniform(sm.gC);

  f4 aq[NTOK][NJ], aw[NTOK][NJ], ak[NTOK][NJ];
  float s1[NTOK], s2[NTOK], s3[NTOK], we[NTOK][NTOK], oe[NTOK][NTOK], gsum = 0.f;
#pragma unroll
  for (int t = 0; t < NTOK; ++t) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) aq[t][j] = aw[t][j] = ak[t][j] = zero4();
    s1[t] = s2[t] = s3[t] = 0.f;
#pragma unroll
    for (int i = 0; i <= t; ++i) we[t][i] = oe[t][i] = 0.f;
  }
#pragma unroll 1
  for (int r0 = 0; r0 < DV; r0 += NG * RC) {
    f4 sn[RC][NJ], gn[RC][NJ];                 // the next rows, in flight during these
    const int rn = r0 + NG * RC < DV ? r0 + NG * RC : r0;
    load_rows(sn, S0, rn);
    load_rows(gn, Gf, rn);
#pragma unroll
    for (int i = 0; i < RC; ++i) {
      if (NTOK == 4) asm volatile("" ::: "memory");   // k and q read from LDS where they are used, not kept in registers
      const int row = r0 + NG * i + grp;
      float sk[NTOK], sq[NTOK], gk[NTOK];
#pragma unroll
      for (int t = 0; t < NTOK; ++t) {
        sk[t] = sq[t] = gk[t] = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const f4 kv = *(const f4*)&sm.k[t][64 * j + 4 * l], qv = *(const f4*)&sm.q[t][64 * j + 4 * l];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            sk[t] += s[i][j][c] * kv[c];
            sq[t] += s[i][j][c] * qv[c];
            gk[t] += g[i][j][c] * kv[c];
          }
        }
        sk[t] = sum16(sk[t]);
        sq[t] = sum16(sq[t]);
        gk[t] = sum16(gk[t]);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) gsum += g[i][j][c] * s[i][j][c];
      float e[NTOK], wv[NTOK], u[NTOK], dO[NTOK];
#pragma unroll
      for (int t = 0; t < NTOK; ++t) {
        dO[t] = sm.dO[t][row];
        u[t] = sm.v[t][row] - ge[t] * (sk[t] + lm[t] * sq[t]);
        e[t] = be[t] * u[t];
#pragma unroll
        for (int p = 0; p < t; ++p) e[t] -= A[t][p] * e[p];
        if (t >= nt) e[t] = 0.f;
      }
#pragma unroll
      for (int t = NTOK - 1; t >= 0; --t) {
        wv[t] = kb[t] * gk[t];
#pragma unroll
        for (int p = t; p < NTOK; ++p)
          if (p < nt) wv[t] += P[p][t] * dO[p];
#pragma unroll
        for (int p = t + 1; p < NTOK; ++p)
          if (p < nt) wv[t] -= A[p][t] * wv[p];
        if (t >= nt) wv[t] = 0.f;
      }
#pragma unroll
      for (int t = 0; t < NTOK; ++t) {
        s1[t] += wv[t] * u[t];
        s2[t] += ge[t] * (dO[t] * sq[t] - be[t] * wv[t] * (sk[t] + lm[t] * sq[t]));
        s3[t] += kb[t] * e[t] * gk[t];
#pragma unroll
        for (int p = 0; p <= t; ++p) {
          if (p < t) we[t][p] += wv[t] * e[p];
          oe[t][p] += dO[t] * e[p];
        }
        if (l == 0 && t < nt) sm.v[t][row] = be[t] * wv[t];
      }
      if (NTOK == 4) asm volatile("" ::: "memory");
      f4 gx[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        gx[j] = gC * g[i][j];
#pragma unroll
        for (int t = 0; t < NTOK; ++t) {
          aq[t][j] += s[i][j] * dO[t];
          aw[t][j] += s[i][j] * wv[t];
          ak[t][j] += g[i][j] * e[t];
          const float z2 = -ge[t] * be[t] * wv[t], z1 = ge[t] * dO[t] + lm[t] * z2;
          const f4 kv = *(const f4*)&sm.k[t][64 * j + 4 * l], qv = *(const f4*)&sm.q[t][64 * j + 4 * l];
          if (t < nt) gx[j] += z1 * qv + z2 * kv;
        }
        if (dS0) *(f4*)(dS0 + (size_t)row * DK + 64 * j + 4 * l) = gx[j];
      }
    }
#pragma unroll
    for (int i = 0; i < RC; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        s[i][j] = sn[i][j];
        g[i][j] = gn[i][j];
      }
  }

  // sums over a wave's row groups, then over the waves in order
  auto over_groups = [&](float x) {
    x += lane_xor(x, 16, lane);
    return x + lane_xor(x, 32, lane);
  };
  auto put = [&](f4 (&x)[NTOK][NJ], int kind) {
#pragma unroll
    for (int t = 0; t < NTOK; ++t)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        f4 y;
#pragma unroll
        for (int c = 0; c < 4; ++c) y[c] = over_groups(x[t][j][c]);
        if (lane < 16) *(f4*)&sm.part[w][kind * NTOK + t][64 * j + 4 * l] = y;
      }
  };
  put(aq, 0);
  put(aw, 1);
  put(ak, 2);
  {
    const float x = over_groups(sum16(gsum));
    if (lane == 0) sm.sc[w][SM::NS - 1] = x;
#pragma unroll
    for (int t = 0; t < NTOK; ++t) {
      const float x1 = over_groups(s1[t]), x2 = over_groups(s2[t]), x3 = over_groups(s3[t]);
      if (lane == 0) {
        sm.sc[w][t] = x1;
        sm.sc[w][NTOK + t] = x2;
        sm.sc[w][2 * NTOK + t] = x3;
      }
#pragma unroll
      for (int p = 0; p < NTOK; ++p) {
        const float y1 = p < t ? over_groups(we[t][p]) : 0.f, y2 = p <= t ? over_groups(oe[t][p]) : 0.f;
        if (lane == 0) {
          sm.sc[w][3 * NTOK + t * NTOK + p] = y1;
          sm.sc[w][3 * NTOK + SM::NP + t * NTOK + p] = y2;
        }
      }
    }
  }
  __syncthreads();
  if (tid < SM::NS) {
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) x += sm.sc[i][tid];
    sm.tot[tid] = x;
  }
  __syncthreads();
  if (tid < NTOK * NTOK) {                     // dA = -w e^T below the diagonal, dO e^T on and below it
    const int t = tid / NTOK, i = tid % NTOK;
    sm.dG[t][i] = i < t ? -sm.beta[t] * sm.gam[t][i] * sm.tot[3 * NTOK + tid] : 0.f;
    sm.dQK[t][i] = i <= t ? sm.gam[t][i] * sm.tot[3 * NTOK + SM::NP + tid] : 0.f;
  }
  __syncthreads();
  for (int idx = tid; idx < nt * DK; idx += NTHREADS) {      // whole waves: DK is a multiple of 64
    const int t = idx / DK, c = idx % DK;
    float xq = 0.f, xw = 0.f, xk = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      xq += sm.part[i][t][c];
      xw += sm.part[i][NTOK + t][c];
      xk += sm.part[i][2 * NTOK + t][c];
    }
    float dx = -sm.beta[t] * sm.ge[t] * xw, dq = sm.ge[t] * xq, dk = sm.kb[t] * xk;
    for (int i = 0; i < t; ++i) dx += sm.dG[t][i] * sm.k[i][c];
    for (int i = 0; i <= t; ++i) dq += sm.dQK[t][i] * sm.k[i][c];
    dq += sm.lam[t] * dx;
    dk += dx;
    for (int r = t; r < nt; ++r) dk += sm.dQK[r][t] * sm.q[r][c];
    for (int r = t + 1; r < nt; ++r) dk += sm.dG[r][t] * (sm.k[r][c] + sm.lam[r] * sm.q[r][c]);
    const size_t at = ((size_t)(t0 + t) * H + h) * DK + c;
    ((E*)a.dq)[at] = fromf<E>(dq);
    ((E*)a.dk)[at] = fromf<E>(dk);
    const float dl = wave_sum_l(sm.q[t][c] * dx, lane);
    if (lane == 0) sm.dl[t][c / 64] = dl;
  }
  for (int idx = tid; idx < nt * DV / 4; idx += NTHREADS) {
    const int t = idx / (DV / 4), c = 4 * (idx % (DV / 4));
    *(typename QE::raw*)((E*)a.dv + ((size_t)(t0 + t) * H + h) * DV + c) = QE::pack(*(const f4*)&sm.v[t][c]);
  }
  __syncthreads();
  if (tid < nt) {
    const size_t at = (size_t)(t0 + tid) * H + h;
    const float dl = DK == 128 ? sm.dl[tid][0] + sm.dl[tid][1] : sm.dl[tid][0];
    if (a.dlam) a.dlam[at] = dl;
    if (a.wDL) a.wDL[at] = dl;
    float db = sm.tot[tid];
    for (int i = 0; i < tid; ++i)
      db -= sm.tot[3 * NTOK + tid * NTOK + i] * sm.gam[tid][i] * (sm.kk[tid][i] + sm.lam[tid] * sm.qk[tid][i]);
    a.dbeta[at] = db;
    if (a.dla) {
      auto tt = [&](int t, int i) {
        const float x = sm.dQK[t][i] * sm.qk[t][i];
        return i < t ? x + sm.dG[t][i] * (sm.kk[t][i] + sm.lam[t] * sm.qk[t][i]) : x;
      };
      float acc = sm.gC * sm.tot[SM::NS - 1];
      for (int r = 0; r < nt; ++r) {
        if (r < tid) {
          acc += sm.tot[2 * NTOK + r];
          continue;
        }
        acc += sm.tot[NTOK + r];
        for (int i = 0; i < r; ++i) acc += tt(r, i);         // (the diagonal term is in both sums)
        for (int t = r + 1; t < nt; ++t) acc -= tt(t, r);
      }
      a.dla[at] = acc;
    }
  }
}

hipError_t launch_rec_bwd_few(const RecBwdArgs& a, int units, int dtype, int Dk, int tokens, hipStream_t st) {
  const dim3 grid(units), thr(NTHREADS);
#define QD_FEW(ET, DKV)                                                                             \
  do {                                                                                              \
    if (tokens <= 1) hipLaunchKernelGGL((k_rec_bwd_few<ET, DKV, 1>), grid, thr, 0, st, a);          \
    else if (tokens <= 2) hipLaunchKernelGGL((k_rec_bwd_few<ET, DKV, 2>), grid, thr, 0, st, a);     \
    else if constexpr (DKV == 64) hipLaunchKernelGGL((k_rec_bwd_few<ET, 64, 4>), grid, thr, 0, st, a); \
  } while (0)
  if (dtype == 1 && Dk == 128) QD_FEW(__bf16, 128);
  else if (dtype == 1) QD_FEW(__bf16, 64);
  else if (Dk == 128) QD_FEW(float, 128);
  else QD_FEW(float, 64);
#undef QD_FEW
  return hipGetLastError();
}

}  // namespace qd
