// steps.hip -- residuals of one primal-dual iteration for the step control (Sec. 4 uses
// the adaptive primal-dual method, which balances the primal and dual residuals by
// rescaling the steps).
//
// With dx = x_k - x_{k+1} and dy = y_k - y_{k+1} (x = (u, s), y = (v, z, p, q)):
//   r_p = T^-1 dx - K^T dy,   r_d = Sigma^-1 dy - K dx,
// and the kernel sums |r_p| and |r_d| over all entries, and the sizes of the two sides'
// variables at the new iterate, |y_{k+1}| and |x_{k+1}| (l1 norms, FP64 accumulation,
// fixed order: every thread owns a fixed set of pixels, blocks write partial sums, one
// block adds them).
#include "device_math.hpp"
#include "internal.hpp"
#include "checks.hpp"
#include "residuals.hpp"

namespace {

template <typename DT>
__global__ __launch_bounds__(RB) void k_residuals(ResPtrs R, IterArgs A) {
  residuals_body<DT>(R, A, blockIdx.x, gridDim.x);
}

// the same with the problem's parameters read from device memory (a batch's table, which
// the adaptive balance rewrites between checks while a captured graph keeps its arguments)
template <typename DT>
__global__ __launch_bounds__(RB) void k_residuals_tab(ResPtrs R, const IterArgs *__restrict__ Ap) {
  residuals_body<DT>(R, *Ap, blockIdx.x, gridDim.x);
}

// every member of a list in one launch: each block runs the lone kernel's code with its
// member's pointers, parameters, block index and block count, so the partial sums are
// bitwise those of the member's own launch
template <typename DT>
__global__ __launch_bounds__(RB) void k_residuals_batch(const ResPtrs *__restrict__ R, const IterArgs *__restrict__ A,
                                                        const int *__restrict__ mem, const int *__restrict__ first,
                                                        int nl) {
  long long blk;
  int nb;
  const int j = member_block(mem, first, nl, blk, nb);
  residuals_body<DT>(R[j], A[j], blk, nb);
}

__global__ __launch_bounds__(RB) void k_sum_quads(const double *part, int nb, double *out, const unsigned *err) {
  if (blockIdx.x == 0 && threadIdx.x == 0) out[4] = scalar_word(err);
  sum_quads_body(part, nb, out, blockIdx.x);
}
// grid (4, nl): column blockIdx.x of list entry blockIdx.y
__global__ __launch_bounds__(RB) void k_sum_quads_batch(const ResPtrs *__restrict__ R, double *const *__restrict__ out,
                                                        const int *__restrict__ mem, const int *__restrict__ first) {
  const int l = (int)blockIdx.y;
  const int j = __builtin_amdgcn_readfirstlane(mem[l]);
  const int nb = __builtin_amdgcn_readfirstlane(first[l + 1] - first[l]);
  sum_quads_body(R[j].part, nb, out[j], (int)blockIdx.x);
}

}  // namespace

hipError_t launch_residuals_batch(const ResBatch &B, hipStream_t st) {
  if (B.n[2] == 0) return hipSuccess;
  if (B.n[0] > 0)
    hipLaunchKernelGGL(k_residuals_batch<uint16_t>, dim3(B.nblk[0]), dim3(RB), 0, st, B.R, B.A, B.mem[0], B.first[0],
                       B.n[0]);
  if (B.n[1] > 0)
    hipLaunchKernelGGL(k_residuals_batch<float>, dim3(B.nblk[1]), dim3(RB), 0, st, B.R, B.A, B.mem[1], B.first[1],
                       B.n[1]);
  hipLaunchKernelGGL(k_sum_quads_batch, dim3(4, B.n[2]), dim3(RB), 0, st, B.R, B.out, B.mem[2], B.first[2]);
  return hipGetLastError();
}

int residual_blocks(const IterArgs &A) {
  const long long N = (long long)A.H * A.W;
  const long long nb = (N + RB - 1) / RB;
  return (int)(nb < 1024 ? nb : 1024);
}

hipError_t launch_residuals(bool bf16, const ResPtrs &R, const IterArgs &A, double *out, const unsigned *err,
                            hipStream_t st, const IterArgs *A_dev) {
  const int nb = residual_blocks(A);
  if (A_dev) {
    if (bf16)
      hipLaunchKernelGGL(k_residuals_tab<uint16_t>, dim3(nb), dim3(RB), 0, st, R, A_dev);
    else
      hipLaunchKernelGGL(k_residuals_tab<float>, dim3(nb), dim3(RB), 0, st, R, A_dev);
  } else if (bf16) {
    hipLaunchKernelGGL(k_residuals<uint16_t>, dim3(nb), dim3(RB), 0, st, R, A);
  } else {
    hipLaunchKernelGGL(k_residuals<float>, dim3(nb), dim3(RB), 0, st, R, A);
  }
  hipLaunchKernelGGL(k_sum_quads, dim3(4), dim3(RB), 0, st, (const double *)R.part, nb, out, err);
  return hipGetLastError();
}
