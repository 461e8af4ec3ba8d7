// Posterior prediction (Section 2.1, posterior forward formulae), with the approximated
// covariance K' of Section 3.3 in the place of the exact one:
//   mu_j  = <k_j, K'^-1 y>,      v_j = alpha - <k_j, K'^-1 k_j>,
// where k_j = k(X_train, x*_j) is the exact kernel between the training points and test point j
// and K_** has alpha on its diagonal.  The solves go through the same batched preconditioned CG
// as the loss: one single-column solve for y, then (for the variances) the cross-covariance
// columns in batches as wide as the context's vector blocks.  K_* is never stored: each batch of
// its columns is generated in fp64 straight into the right-hand-side block.
#include <algorithm>
#include <cmath>

#include "nugpr_internal.h"

namespace nugpr {

struct CrossArgs {
  double inv_ell[MAX_D];     // 1 / lengthscale per dimension
  double alpha;
  int d;
};

// U[i, col] = alpha exp(-0.5 sum_k ((x_ik - x*_jk) / ell_k)^2) for j = j0 + col, col < cnt;
// columns cnt..T-1 of the block are cleared (a zero right-hand side is skipped by the solver).
template <typename VT>
__global__ __launch_bounds__(256) void k_cross_block(CrossArgs a, const float* __restrict__ X,
                                                     const float* __restrict__ Xt, int64_t j0, int cnt,
                                                     int64_t n, int T, VT* __restrict__ U, uint64_t sys) {
  // (blockIdx.y: the block of this many columns further, in the next slot)
  U = reinterpret_cast<VT*>(reinterpret_cast<char*>(U) + blockIdx.y * sys);
  j0 += (int64_t)blockIdx.y * T;
  cnt = min(T, cnt - (int)blockIdx.y * T);
  const int rpp = 256 / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  if (myrow >= rpp) return;
  const bool live = col < cnt;
  const float* xt = Xt + (live ? (j0 + col) * (int64_t)a.d : 0);
  for (int64_t r = (int64_t)blockIdx.x * rpp + myrow; r < n; r += (int64_t)gridDim.x * rpp) {
    double v = 0.0;
    if (live) {
      const float* x = X + r * a.d;
      double q = 0.0;
      for (int k = 0; k < a.d; ++k) {
        const double t = ((double)x[k] - (double)xt[k]) * a.inv_ell[k];
        q = fma(t, t, q);
      }
      v = a.alpha * exp(-0.5 * q);
    }
    U[r * T + col] = (VT)v;
  }
}

// partial[0][block][col] = sum_i U[i,col] u[i],  partial[1][block][col] = sum_i U[i,col] S[i,col]
// (S may be null: then only the first set is written).  Fixed summation order: rows split among the workgroups as in the CG's
// dots, 256 threads, one sum over the rows of a pass.
template <typename VT>
__global__ __launch_bounds__(256) void k_predict_dots(const VT* __restrict__ U, const VT* __restrict__ u,
                                                      const VT* __restrict__ S, int64_t n, int T,
                                                      double* __restrict__ partial, uint64_t sys) {
  __shared__ double red[2][256];
  U = reinterpret_cast<const VT*>(reinterpret_cast<const char*>(U) + blockIdx.y * sys);
  if (S) S = reinterpret_cast<const VT*>(reinterpret_cast<const char*>(S) + blockIdx.y * sys);
  partial = reinterpret_cast<double*>(reinterpret_cast<char*>(partial) + blockIdx.y * sys);
  const int rpp = 256 / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  const bool live = myrow < rpp;
  const int64_t rows_per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  double s0 = 0.0, s1 = 0.0;
  if (live) {
    for (int64_t r = r0 + myrow; r < r1; r += rpp) {
      const int64_t idx = r * T + col;
      const double k = (double)U[idx];
      s0 = fma(k, (double)u[r], s0);
      if (S) s1 = fma(k, (double)S[idx], s1);
    }
  }
  red[0][tid] = s0;
  red[1][tid] = s1;
  __syncthreads();
  if (tid < T) {
    for (int w = 0; w < 2; ++w) {
      double s = 0.0;
      for (int k = 0; k < rpp; ++k) s += red[w][k * T + tid];
      partial[((int64_t)w * gridDim.x + blockIdx.x) * MAX_COLS + tid] = s;
    }
  }
}

// out[(2 system + set) * MAX_COLS + col] = the sum of that set's and column's partial sums (grid: T x 2 x systems), fixed order.  Copying the
// partial sums to the host (540 KB at 1024 workgroups) and adding them up there took longer, per batch of 17 test points
// by 1 us at 2048 training points, 13 at 32768, 49 at 131072 and 47 at 262144.
__global__ __launch_bounds__(256) void k_predict_sums(const double* __restrict__ partial, int nblocks, double* __restrict__ out, uint64_t sys) {
  __shared__ double red[256];
  const int tid = threadIdx.x;
  partial = reinterpret_cast<const double*>(reinterpret_cast<const char*>(partial) + blockIdx.z * sys);
  const double* p = partial + (int64_t)blockIdx.y * nblocks * MAX_COLS + blockIdx.x;
  double s = 0.0;
  for (int b = tid; b < nblocks; b += 256) s += p[(int64_t)b * MAX_COLS];
  red[tid] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) out[(blockIdx.z * 2 + blockIdx.y) * MAX_COLS + blockIdx.x] = red[0];
}

template <typename VT>
static int predict_t(nugpr_ctx* c, const double* theta, const float* Xt, int64_t m, double* mean, double* var,
                     int32_t* max_iters_used, hipStream_t s) {
  const Layout& L = c->L;
  const int64_t n = L.n;
  const int T = L.T;
  int worst = NUGPR_OK, mx_all = 0;
  VT *U = (VT*)c->Uv, *S = (VT*)c->Xv, *u = (VT*)c->x0;
  // u = K'^-1 y: a one-column block is just the vector
  int rc = to_internal(c, c->y, U, n, s);
  if (rc) return rc;
  int mx = 0;
  rc = run_pcg(c, U, S, 1, nullptr, nullptr, nullptr, &mx, s);
  if (rc < 0 || rc == NUGPR_INDEFINITE || rc == NUGPR_NOT_FINITE) return rc;
  worst = std::max(worst, rc);
  mx_all = std::max(mx_all, mx);
  NUGPR_HIP(hipMemcpyAsync(u, S, (size_t)n * sizeof(VT), hipMemcpyDeviceToDevice, s));

  CrossArgs a;
  const bool iso = (c->params.flags & NUGPR_ISOTROPIC) != 0;
  for (int k = 0; k < L.d; ++k) a.inv_ell[k] = 1.0 / theta[iso ? 0 : k];
  for (int k = L.d; k < MAX_D; ++k) a.inv_ell[k] = 0.0;
  a.alpha = theta[L.p - 2];
  a.d = L.d;
  const int nb = L.n_dot_blocks;
  const int rpp = 256 / T;
  const int grid = (int)std::min<int64_t>((n + rpp - 1) / rpp, 8192);
  // Blocks of T columns side by side, two or four in one set of launches, where the context can (nugpr_ctx::slots).  200 test
  // points with variances, 32768 training points, 17 columns: one after the other 5450 us, side by side 3500.
  const bool together = c->slots > 1 && c->onehot && !L.compensate;
  const uint64_t sys = L.slot_bytes;
  const Operator op{c->Kd, c->C, c->op_scale, c->op_shift};
  const Operator ops[MAX_SLOTS] = {op, op, op, op};
  int nsys = 1;
  for (int64_t j0 = 0; j0 < m; j0 += (int64_t)nsys * T) {
    const int64_t left = (m - j0 + T - 1) / T;                  // blocks
    nsys = !together || left == 1 ? 1 : left == 2 ? 2 : 4;        // (three: the last of four is empty)
    const int held = (int)std::min<int64_t>(nsys, left);
    const unsigned ny = (unsigned)nsys;
    int cnt = (int)std::min<int64_t>((int64_t)nsys * T, m - j0);
    int failed = NUGPR_OK;
    hipLaunchKernelGGL((k_cross_block<VT>), dim3(grid, ny), dim3(256), 0, s, a, c->X, Xt, j0, cnt, n, T, U, sys);
    NUGPR_HIP(hipGetLastError());
    if (var) {
      PcgOutcome out[MAX_SLOTS] = {};
      if ((rc = run_pcg_systems(c, U, S, T, ops, held, out, s))) return rc;
      for (int e = 0; e < held; ++e) {
        rc = out[e].status;
        if (rc == NUGPR_INDEFINITE || rc == NUGPR_NOT_FINITE) {
          if (e == 0) return rc;
          failed = rc;                                          // the blocks ahead of it are good: as one after the other
          cnt = e * T;
          break;
        }
        worst = std::max(worst, rc);
        mx_all = std::max(mx_all, out[e].max_it);
      }
    }
    hipLaunchKernelGGL((k_predict_dots<VT>), dim3(nb, ny), dim3(256), 0, s, U, u, var ? S : (const VT*)nullptr, n, T,
                       c->dotpart, sys);
    NUGPR_HIP(hipGetLastError());
    double* sums = c->alog;                                      // (the solver's logs are free now)
    hipLaunchKernelGGL(k_predict_sums, dim3(T, 2, ny), dim3(256), 0, s, c->dotpart, nb, sums, sys);
    NUGPR_HIP(hipGetLastError());
    NUGPR_HIP(hipMemcpyAsync(c->h_buf, sums, (size_t)nsys * 2 * MAX_COLS * sizeof(double), hipMemcpyDeviceToHost, s));
    NUGPR_HIP(hipStreamSynchronize(s));
    for (int q = 0; q < cnt; ++q) {
      const double* of = c->h_buf + (size_t)(q / T) * 2 * MAX_COLS + q % T;
      mean[j0 + q] = of[0];
      if (var) var[j0 + q] = a.alpha - of[MAX_COLS];
    }
    if (failed) return failed;
  }
  if (max_iters_used) *max_iters_used = mx_all;
  return worst;
}

int run_predict(nugpr_ctx* c, const double* theta, const float* Xt, int64_t m, double* mean, double* var,
                int32_t* max_iters_used, hipStream_t s) {
  if (c->acc64) return predict_t<double>(c, theta, Xt, m, mean, var, max_iters_used, s);
  return predict_t<float>(c, theta, Xt, m, mean, var, max_iters_used, s);
}

}  // namespace nugpr
