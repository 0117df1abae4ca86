// Gates of the layer from its gate projection (Sec. 3.3; App. "Query-Feedback
// Coefficient"): rows of beta | lambda | alpha logits, H each (lambda and alpha
// where learned), into beta = sigmoid, lambda = sigmoid(. + b), log alpha =
// logsigmoid, and their backward with the scalar bias's gradient.
//
// The tensors are small (B4 T4096 H16: 1.6 MB of logits); as elementwise
// tensor operations the two directions are about 30 launches, 110 us of a
// training step and most of the host time of a small layer.  Here they are one
// launch forward and two backward.  The bias's gradient is summed per workgroup,
// then over the workgroups, in a fixed order.
#include "qd_common.h"
#include "qd_launch.h"

namespace qd {

namespace {

__device__ inline float sigmoid(float x) { return 1.f / (1.f + expf(-x)); }

// Sum over the workgroup in a fixed order, in thread 0.
__device__ inline float block_sum(float x, float* part) {
  part[threadIdx.x] = x;
  __syncthreads();
#pragma unroll
  for (int off = NTHREADS / 2; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
    __syncthreads();
  }
  return part[0];
}

template <typename E, typename EB>
__global__ __launch_bounds__(NTHREADS) void k_gates_fwd(long n, int H, int ld, const E* __restrict__ x,
                                                       const EB* __restrict__ bias, float* __restrict__ beta,
                                                       float* __restrict__ lam, float* __restrict__ la) {
  const float b = lam ? tof(*bias) : 0.f;
  for (long i = (long)blockIdx.x * NTHREADS + threadIdx.x; i < n; i += (long)gridDim.x * NTHREADS) {
    const E* row = x + (i / H) * ld + i % H;
    beta[i] = sigmoid(tof(row[0]));
    if (lam) lam[i] = sigmoid(tof(row[H]) + b);
    if (la) {
      const float a = tof(row[lam ? 2 * H : H]);
      la[i] = fminf(a, 0.f) - log1pf(expf(-fabsf(a)));
    }
  }
}

// dbeta, dlam, dla may be nullptr (no gradient came); part[block] receives the
// workgroup's share of the bias's gradient when lambda is learned.
template <typename E>
__global__ __launch_bounds__(NTHREADS) void k_gates_bwd(long n, int H, int ld, const float* __restrict__ beta,
                                                       const float* __restrict__ lam, const float* __restrict__ la,
                                                       const float* __restrict__ dbeta,
                                                       const float* __restrict__ dlam,
                                                       const float* __restrict__ dla, E* __restrict__ dx,
                                                       float* __restrict__ part) {
  __shared__ float red[NTHREADS];
  float sum = 0.f;
  for (long i = (long)blockIdx.x * NTHREADS + threadIdx.x; i < n; i += (long)gridDim.x * NTHREADS) {
    E* row = dx + (i / H) * ld + i % H;
    const float b = beta[i];
    row[0] = fromf<E>(dbeta ? dbeta[i] * (1.f - b) * b : 0.f);
    if (lam) {
      const float l = lam[i], d = dlam ? dlam[i] * (1.f - l) * l : 0.f;
      row[H] = fromf<E>(d);
      sum += d;
    }
    if (la) row[lam ? 2 * H : H] = fromf<E>(dla ? dla[i] * -expm1f(la[i]) : 0.f);   // 1 - alpha
  }
  if (lam) {
    sum = block_sum(sum, red);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
  }
}

template <typename EB>
__global__ __launch_bounds__(NTHREADS) void k_gates_bias(int n, const float* __restrict__ part, EB* __restrict__ out) {
  __shared__ float red[NTHREADS];
  float sum = 0.f;
  for (int i = threadIdx.x; i < n; i += NTHREADS) sum += part[i];
  sum = block_sum(sum, red);
  if (threadIdx.x == 0) *out = fromf<EB>(sum);
}

}  // namespace

// workgroups for n (token, head) pairs
int gates_blocks(long n) {
  const long b = (n + NTHREADS - 1) / NTHREADS;
  return (int)(b < 1 ? 1 : b > 1024 ? 1024 : b);
}

hipError_t launch_gates_fwd(long n, int H, int ld, int dtype, int bias_dtype, const void* x, const void* bias,
                            float* beta, float* lam, float* la, hipStream_t st) {
  const dim3 grid(gates_blocks(n)), thr(NTHREADS);
#define QD_G(ET, EB) \
  hipLaunchKernelGGL((k_gates_fwd<ET, EB>), grid, thr, 0, st, n, H, ld, (const ET*)x, (const EB*)bias, beta, lam, la)
  if (dtype == 1 && bias_dtype == 1) QD_G(__bf16, __bf16);
  else if (dtype == 1) QD_G(__bf16, float);
  else if (bias_dtype == 1) QD_G(float, __bf16);
  else QD_G(float, float);
#undef QD_G
  return hipGetLastError();
}

hipError_t launch_gates_bwd(long n, int H, int ld, int dtype, int bias_dtype, const float* beta, const float* lam,
                            const float* la, const float* dbeta, const float* dlam, const float* dla, void* dx,
                            float* part, void* dbias, hipStream_t st) {
  const int nb = gates_blocks(n);
  if (dtype == 1)
    hipLaunchKernelGGL((k_gates_bwd<__bf16>), dim3(nb), dim3(NTHREADS), 0, st, n, H, ld, beta, lam, la, dbeta, dlam,
                       dla, (__bf16*)dx, part);
  else
    hipLaunchKernelGGL((k_gates_bwd<float>), dim3(nb), dim3(NTHREADS), 0, st, n, H, ld, beta, lam, la, dbeta, dlam,
                       dla, (float*)dx, part);
  if (lam) {
    if (bias_dtype == 1)
      hipLaunchKernelGGL((k_gates_bias<__bf16>), dim3(1), dim3(NTHREADS), 0, st, nb, part, (__bf16*)dbias);
    else
      hipLaunchKernelGGL((k_gates_bias<float>), dim3(1), dim3(NTHREADS), 0, st, nb, part, (float*)dbias);
  }
  return hipGetLastError();
}

}  // namespace qd
