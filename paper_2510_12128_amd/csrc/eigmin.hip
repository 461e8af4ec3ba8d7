// lambda_0 of eq. (krep), the smallest eigenvalue of the kernel matrix C of all representatives (Section 3.3),
// for couplings too large for a dense host eigen-solve: a matrix-free, block-preconditioned Davidson
// iteration in fp64 on the device.
//
// Why not a plain Krylov (Lanczos) process: representatives of one cluster lie close together, so the low end of
// C's spectrum is a dense cluster of small eigenvalues (often down to rounding level) under a largest eigenvalue of
// order n_c r; a polynomial in C then needs thousands of steps to resolve lambda_min to 1e-10.  The same
// structure makes the remedy cheap: the small eigenvalues come from WITHIN the diagonal blocks of C, so the
// inverse of a block-diagonal part of C, in fp64, is a preconditioner that takes the cluster apart.
//
// The matrix is applied through the strip kernels that the product K' D uses for C S, on its two-term
// representation: off the diagonal C = Chi + Clo (Chi the stored fp32 entries, Clo what fp32 dropped, itself in
// fp32: together ~2^-48 relative), on the diagonal the exact scalar alpha.
// Iteration (generalised Davidson, Rayleigh-Ritz on an orthonormal basis V with thick restart):
//   (theta, y) = smallest eigenpair of H = V^T C V;  x = V y;  res = C x - theta x;
//   t = T res with T = blockdiag(B_k + mu I)^-1, B_k the 128 x 128 diagonal blocks of C recomputed in fp64
//       from the representatives and Cholesky-factored once per assembly (mu = 1e-10 alpha);
//   t is orthogonalised against V (Gram-Schmidt, twice), normalised and appended; C t is computed.
// All sums of a step are taken in a fixed order, so lambda_0 is reproducible
// to the bit.  Stop: the Ritz value theta is safe when min(|res|, 4 |res|^2 / gap) <= tol (gap: distance to the
// second Ritz value, used when it is clearly separate), or when |theta| <= tol: a kernel matrix is positive
// semi-definite, so lambda_min lies in [0, theta].  Ritz values approach lambda_min from above, so
// C - theta I misses being positive semi-definite by at most the tolerance, far below the noise variance.
// One regime converges slowly: strongly overlapping clusters with a wide lengthscale, where the small eigenvalues
// belong to modes that span many blocks.  There lambda_min is itself tiny; if the step cap is reached with
// theta <= 1e-5 alpha, theta is returned as it stands (lambda_min lies in [0, theta]; the cap makes the step
// count, and with it theta, the same smooth function of the hyperparameters on both sides of a difference
// quotient).  A run that reaches the cap with a larger theta is an error.
#include <algorithm>
#include <cmath>
#include <vector>

#include "nugpr_internal.h"

namespace nugpr {

typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int EB = 128;               // order of the preconditioner's diagonal blocks
constexpr int EBP = EB + 1;           // row stride of a block in LDS (odd: column accesses spread over the banks)
constexpr int DAV_MAX_BASIS = EIGMIN_MAX_BASIS;
constexpr int DAV_KEEP = 3;           // Ritz vectors a restart keeps
constexpr int DAV_MAX_STEPS = 150;

struct BlockKernelArgs {
  double inv_ell[MAX_D];
  double alpha, mu;
  int n, d;
};

// Inverse L^-1 of the Cholesky factor (lower, row-major EB x EB doubles per block, unit rows past the end) of
// B_k + mu I, where B_k = k(R_k, R_k) for the representatives 128 k .. 128 k + 127, evaluated in fp64 with direct
// differences.  Once per assembly; the explicit triangular inverse turns the two substitutions of every step, 256
// dependent rounds, into two products.
// One workgroup per block, so what counts is the serial chain: eight panels of 16 columns, each factored by one wave in
// registers (a lane holds rows l and l + 64; pivots and pivot rows reach the other lanes by v_readlane), the rest in 16 x 16
// blocks on the matrix cores, a block row or column per wave: the left-looking update before a panel, and the inverse by
// [L11 0; L21 L22]^-1 = [Y11 0; -Y22 L21 Y11, Y22] over blocks, pairs and fours of them.  2048 representatives: 267 us with a
// pivot's trailing update by all threads (three barriers a pivot, two a row of the inverse), now 87.
constexpr int BF_THREADS = 1024;
constexpr int BI = 16 * 17;           // an inverted diagonal block in LDS, row stride 17
constexpr int BF_LDS = (EB * EBP + EB / 16 * BI + EB) * (int)sizeof(double);
__device__ __forceinline__ double lane_double(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane), hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}
// column j of blocks of -Y22 L21 Y11 for the node of 2 H blocks from block s0 on; block (i, j) of the inverse lies where block
// (j, i) of the matrix was.  A product enters the next one as its right factor as it stands in the registers.
template <int H>
__device__ __forceinline__ void block_inverse_column(double* M, const double* inv, int s0, int j) {
  const int lane = threadIdx.x & 63, m = lane & 15, kg = lane >> 4, mid = s0 + H;
  auto yb = [&](int i, int q) { return i == q ? inv + i * BI : M + (16 * q) * EBP + 16 * i; };
  auto ldy = [&](int i, int q) { return i == q ? 17 : EBP; };
  v4d t[H];
#pragma unroll
  for (int i = 0; i < H; ++i) t[i] = (v4d){0.0, 0.0, 0.0, 0.0};
  for (int q = j; q < mid; ++q) {
    const double* y = yb(q, j);
    const int ld = ldy(q, j);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double b = y[(4 * e + kg) * ld + m];
#pragma unroll
      for (int i = 0; i < H; ++i)
        t[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(M[(16 * (mid + i) + m) * EBP + 16 * q + 4 * e + kg], b, t[i], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    v4d x = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q <= i; ++q) {
      const double* y = yb(mid + i, mid + q);
      const int ld = ldy(mid + i, mid + q);
#pragma unroll
      for (int e = 0; e < 4; ++e) x = __builtin_amdgcn_mfma_f64_16x16x4f64(-y[m * ld + 4 * e + kg], t[q][e], x, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) M[(16 * j + kg + 4 * e) * EBP + 16 * (mid + i) + m] = x[e];
  }
}
__global__ __launch_bounds__(BF_THREADS) void k_block_factor(BlockKernelArgs a, const float* __restrict__ reps,
                                                             double* __restrict__ Lout) {
  extern __shared__ __attribute__((aligned(16))) double M[];      // EB rows of EBP, eight inverted blocks, EB values
  double *inv = M + EB * EBP, *rdiag = inv + EB / 16 * BI;
  const int blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, m = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i0 = blk * EB;
  const int nb = min(EB, a.n - i0);
  for (int idx = tid; idx < EB * EB; idx += BF_THREADS) {
    const int i = idx / EB, j = idx % EB;
    double v = (i == j) ? 1.0 : 0.0;
    if (i < nb && j < nb && j <= i) {
      double q = 0.0;
      const float* ri = reps + (uint64_t)(i0 + i) * a.d;
      const float* rj = reps + (uint64_t)(i0 + j) * a.d;
      for (int k = 0; k < a.d; ++k) {
        const double t = ((double)ri[k] - (double)rj[k]) * a.inv_ell[k];
        q = fma(t, t, q);
      }
      v = a.alpha * exp(-0.5 * q) + (i == j ? a.mu : 0.0);
    }
    M[i * EBP + j] = v;
  }
  __syncthreads();
#pragma unroll 1
  for (int p = 0; p < EB / 16; ++p) {
    if (p > 0) {                                      // block (w, p) -= sum over the panels before of L(w, q) L(p, q)^T
      if (w >= p && w < EB / 16) {
        v4d x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = M[(16 * w + kg + 4 * e) * EBP + 16 * p + m];
        for (int q = 0; q < p; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            x = __builtin_amdgcn_mfma_f64_16x16x4f64(-M[(16 * w + m) * EBP + 16 * q + 4 * e + kg], M[(16 * p + m) * EBP + 16 * q + 4 * e + kg], x, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) M[(16 * w + kg + 4 * e) * EBP + 16 * p + m] = x[e];
      }
      __syncthreads();
    }
    if (w == 0) {
      // elimination without square roots; a pivot that rounding pushed below the shift is replaced by it
      double r0[16], r1[16], d0 = 1.0, d1 = 1.0;
      const bool lower = 16 * p >= 64;                // the pivots are among the rows lane + 64
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        r0[u] = M[lane * EBP + 16 * p + u];
        r1[u] = M[(lane + 64) * EBP + 16 * p + u];
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int row = 16 * p + j;
        const double pv = lower ? r1[j] : r0[j];
        double dj = lane_double(pv, row & 63);
        if (!(dj > 1e-3 * a.mu)) dj = 1e-3 * a.mu;
        d0 = lane == row ? dj : d0;
        d1 = lane + 64 == row ? dj : d1;
        const double rd = 1.0 / dj;
        const double m0 = lane > row ? r0[j] * rd : 0.0, m1 = lane + 64 > row ? r1[j] * rd : 0.0;
#pragma unroll
        for (int c = j + 1; c < 16; ++c) {
          const double x = lane_double(pv, (16 * p + c) & 63);
          r0[c] = fma(-m0, x, r0[c]);
          r1[c] = fma(-m1, x, r1[c]);
        }
      }
      const double s0 = sqrt(d0), s1 = sqrt(d1), q0 = 1.0 / s0, q1 = 1.0 / s1, qp = lower ? q1 : q0;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int col = 16 * p + u;
        const double sc = lane_double(qp, col & 63);
        if (lane >= 16 * p) M[lane * EBP + col] = lane == col ? s0 : (lane > col ? r0[u] * sc : 0.0);
        if (lane + 64 >= 16 * p) M[(lane + 64) * EBP + col] = lane + 64 == col ? s1 : (lane + 64 > col ? r1[u] * sc : 0.0);
      }
      if (lower ? lane + 64 >= 16 * p && lane + 64 < 16 * p + 16 : lane >= 16 * p && lane < 16 * p + 16) rdiag[lower ? lane + 64 : lane] = qp;
    }
    __syncthreads();
  }
  if (w < EB / 16) {                                  // inverse of diagonal block w: lane m holds column m of it
    double l[16], y[16];
    const double r = rdiag[16 * w + m];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      l[u] = M[(16 * w + m) * EBP + 16 * w + u];
      y[u] = u == m ? 1.0 : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      y[q] *= lane_double(r, q);
#pragma unroll
      for (int i = q + 1; i < 16; ++i) y[i] = fma(-lane_double(l[q], i), y[q], y[i]);
    }
    if (kg == 0) {
#pragma unroll
      for (int u = 0; u < 16; ++u) inv[w * BI + u * 17 + m] = y[u];
    }
  }
  __syncthreads();
  if (w < 4) block_inverse_column<1>(M, inv, 2 * w, 2 * w);
  __syncthreads();
  if (w < 4) block_inverse_column<2>(M, inv, 4 * (w >> 1), 4 * (w >> 1) + (w & 1));
  __syncthreads();
  if (w < 4) block_inverse_column<4>(M, inv, 0, w);
  __syncthreads();
  double* out = Lout + (uint64_t)blk * EB * EB;
  for (int idx = tid; idx < EB * EB; idx += BF_THREADS) {
    const int i = idx / EB, j = idx % EB, bi = i >> 4, bj = j >> 4;
    double v = 0.0;
    if (j <= i) v = bi == bj ? inv[bi * BI + (i & 15) * 17 + (j & 15)] : M[(16 * bj + (i & 15)) * EBP + 16 * bi + (j & 15)];
    out[idx] = v;
  }
}

// v_0: a fixed +-1 pattern (integer hash of the index), normalised
__global__ void k_eig_start(double* __restrict__ v, int n) {
  const double s = 1.0 / sqrt((double)n);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    uint32_t h = (uint32_t)i * 2654435761u;
    h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
    v[i] = (h & 1u) ? s : -s;
  }
}

struct Coef { double y[DAV_MAX_BASIS]; };

// The vector work of a step.  One workgroup per block of 128 rows (the preconditioner's blocks), eight threads a row; sums
// over all rows are left as one partial sum per workgroup and added up, in a fixed order, by every workgroup of the kernel
// that needs them.  (In single workgroups, each kernel alone on one compute unit, a step of 2048 rows took 33 us for the
// orthogonalisation, 25 for the new row, 9 + 9 for residual and correction.)
__device__ __forceinline__ double wave_total(double s) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  return s;                                           // (lane 0)
}
// partial[k][workgroup] = <V[k], x> over this workgroup's rows, k < m (x in LDS, zero past the end; a wave takes every 16th k)
__device__ __forceinline__ void row_dots(const double* __restrict__ V, const double* x, int m, int i0, int nb, int ld, double* __restrict__ partial) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int k = wave; k < m; k += 16) {
    const double* v = V + (uint64_t)k * ld + i0;
    double s = lane < nb ? v[lane] * x[lane] : 0.0;
    if (lane + 64 < nb) s = fma(v[lane + 64], x[lane + 64], s);
    s = wave_total(s);
    if (lane == 0) partial[(uint64_t)k * gridDim.x + blockIdx.x] = s;
  }
}
// h[k] = the sum of partial[k][..], k < m, in LDS (complete after the next barrier)
__device__ __forceinline__ void add_partials(const double* __restrict__ partial, int m, int nblk, double* h) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int k = wave; k < m; k += 16) {
    double s = 0.0;
    for (int q = lane; q < nblk; q += 64) s += partial[(uint64_t)k * nblk + q];
    s = wave_total(s);
    if (lane == 0) h[k] = s;
  }
}

// res = AV y - theta V y;  t = blockdiag(Y_k^T Y_k) res with Y_k = L_k^-1, two triangular products per block: rows by waves
// (shuffles), then columns by threads.  Partial sums of |res|^2 and of <V[k], t>.
__global__ __launch_bounds__(1024) void k_eig_correct(const double* __restrict__ V, const double* __restrict__ AV, Coef c, double theta, int m,
                                                      int n, int ld, const double* __restrict__ Yall, double* __restrict__ t,
                                                      double* __restrict__ res2, double* __restrict__ dots) {
  __shared__ double x[EB], z[EB], sums[1024], two[2];
  const int blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = tid & (EB - 1), part = tid >> 7;
  const int i0 = blk * EB, nb = min(EB, n - i0);
  double s = 0.0;
  if (row < nb)
    for (int k = part; k < m; k += 8) {
      const uint64_t at = (uint64_t)k * ld + i0 + row;
      s = fma(c.y[k], fma(-theta, V[at], AV[at]), s);
    }
  sums[tid] = s;
  __syncthreads();
  if (tid < EB) {
    for (int q = 1; q < 8; ++q) s += sums[tid + q * EB];
    x[tid] = s;
    const double r2 = wave_total(s * s);
    if (lane == 0) two[wave] = r2;
  }
  __syncthreads();
  if (tid == 0) res2[blk] = two[0] + two[1];
  const double* Y = Yall + (uint64_t)blk * EB * EB;
  const double x0 = x[lane], x1 = x[lane + 64];
#pragma unroll
  for (int q = 0; q < EB / 16; ++q) {                 // rows wave, wave + 16, ..
    const int i = wave + 16 * q;
    const double v = wave_total(fma(Y[i * EB + lane], x0, Y[i * EB + lane + 64] * x1));
    if (lane == 0) z[i] = v;
  }
  __syncthreads();
  s = 0.0;
#pragma unroll
  for (int q = 0; q < EB / 8; ++q) s = fma(Y[(part + 8 * q) * EB + row], z[part + 8 * q], s);
  sums[tid] = s;
  __syncthreads();
  if (tid < EB) {
    for (int q = 1; q < 8; ++q) s += sums[tid + q * EB];
    x[tid] = tid < nb ? s : 0.0;
    if (tid < nb) t[i0 + tid] = s;
  }
  __syncthreads();
  row_dots(V, x, m, i0, nb, ld, dots);
}

// One pass of classical Gram-Schmidt, all coefficients at once: t <- t - sum h_k V[k], h_k the sums of dots_in.  Two passes are
// orthogonal to rounding, as the modified form.  The first leaves the partial sums of <V[k], t>; the second (LAST) writes t as
// V[m], not yet normalised, and leaves the partial sums of |t|^2.
template <bool LAST>
__global__ __launch_bounds__(1024) void k_eig_orth(double* V, double* t, int m, int n, int ld, const double* __restrict__ dots_in,
                                                   double* __restrict__ dots_out) {
  __shared__ double x[EB], sums[1024], h[DAV_MAX_BASIS], two[2];
  const int tid = threadIdx.x, lane = tid & 63, row = tid & (EB - 1), part = tid >> 7;
  const int i0 = (int)blockIdx.x * EB, nb = min(EB, n - i0);
  double v[DAV_MAX_BASIS / 8];
#pragma unroll
  for (int q = 0; q < DAV_MAX_BASIS / 8; ++q) v[q] = row < nb && part + 8 * q < m ? V[(uint64_t)(part + 8 * q) * ld + i0 + row] : 0.0;
  add_partials(dots_in, m, (int)gridDim.x, h);
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < DAV_MAX_BASIS / 8; ++q)
    if (part + 8 * q < m) s = fma(h[part + 8 * q], v[q], s);
  sums[tid] = s;
  __syncthreads();
  if (tid < EB) {
    for (int q = 1; q < 8; ++q) s += sums[tid + q * EB];
    const double r = tid < nb ? t[i0 + tid] - s : 0.0;
    x[tid] = r;
    if (tid < nb) (LAST ? V + (uint64_t)m * ld : t)[i0 + tid] = r;
    if (LAST) {
      const double r2 = wave_total(r * r);
      if (lane == 0) two[tid >> 6] = r2;
    }
  }
  __syncthreads();
  if (LAST) {
    if (tid == 0) dots_out[blockIdx.x] = two[0] + two[1];
  } else {
    row_dots(V, x, m, i0, nb, ld, dots_out);
  }
}

// V[m] <- V[m] / |V[m]| (norm2: partial sums of the square; null: it is normalised), AV[m] = the sum of the column-slab partial sums of C V[m]
// over the same norm.  The workgroup that finishes last adds up what the host waits for, into pinned memory: out[0] = |res|^2
// (from res2, may be null), out[1] = the norm, out[8 + k] = <V[k], AV[m]>, k <= m; then, behind a system-scope fence, the
// sequence number.
__global__ __launch_bounds__(1024) void k_eig_newrow(const double* __restrict__ parts, int nparts, uint64_t stride, double* V,
                                                     double* __restrict__ AV, int m, int n, int ld, const double* __restrict__ norm2,
                                                     const double* __restrict__ res2, double* dots, double* __restrict__ out,
                                                     PcgState* __restrict__ st, HostFlags* __restrict__ flags, uint64_t seq) {
  __shared__ double x[EB], vm[EB], sums[1024], h[DAV_MAX_BASIS + 2];
  __shared__ int last;
  const int tid = threadIdx.x, row = tid & (EB - 1), part = tid >> 7, nblk = (int)gridDim.x;
  const int i0 = (int)blockIdx.x * EB, nb = min(EB, n - i0);
  double s = 0.0;
  if (row < nb)
    for (int p = part; p < nparts; p += 8) s += parts[(uint64_t)p * stride + i0 + row];
  sums[tid] = s;
  if (norm2) add_partials(norm2, 1, nblk, h);
  __syncthreads();
  const double nrm = norm2 ? sqrt(h[0]) : 1.0, inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
  if (tid < EB) {
    for (int q = 1; q < 8; ++q) s += sums[tid + q * EB];
    x[tid] = s * inv;
    vm[tid] = 0.0;
    if (tid < nb) {
      AV[(uint64_t)m * ld + i0 + tid] = s * inv;
      vm[tid] = V[(uint64_t)m * ld + i0 + tid] * inv;
      V[(uint64_t)m * ld + i0 + tid] = vm[tid];
    }
  }
  __syncthreads();
  row_dots(V, x, m, i0, nb, ld, dots);
  if (tid < 64) {                                     // <V[m], AV[m]>, from this workgroup's own copy
    const double d = wave_total(fma(vm[tid], x[tid], vm[tid + 64] * x[tid + 64]));
    if (tid == 0) dots[(uint64_t)m * nblk + blockIdx.x] = d;
  }
  __syncthreads();
  if (tid == 0) {
    __threadfence();
    last = atomicAdd(&st->check_count, 1) == nblk - 1;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  add_partials(dots, m + 1, nblk, h);
  __syncthreads();
  if (tid <= m) out[8 + tid] = h[tid];
  if (res2) {
    __syncthreads();
    add_partials(res2, 1, nblk, h);
    __syncthreads();
    if (tid == 0) out[0] = h[0];
  }
  if (tid == 0) {
    out[1] = nrm;
    st->check_count = 0;
  }
  __threadfence_system();
  __syncthreads();
  if (tid == 0) *reinterpret_cast<volatile uint64_t*>(&flags->seq) = seq;
}

// restart: V <- V Y, AV <- AV Y for the `keep` coefficient columns in c (column q at y[q * m ..]); element-wise, in place
struct RestartCoef { double y[DAV_KEEP * DAV_MAX_BASIS]; };
__global__ void k_eig_restart(double* __restrict__ V, double* __restrict__ AV, RestartCoef c, int m, int keep, int n,
                              int ld) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    double v[DAV_MAX_BASIS], av[DAV_MAX_BASIS];
    for (int k = 0; k < m; ++k) { v[k] = V[(uint64_t)k * ld + i]; av[k] = AV[(uint64_t)k * ld + i]; }
    for (int q = 0; q < keep; ++q) {
      double a = 0.0, b = 0.0;
      for (int k = 0; k < m; ++k) { a = fma(c.y[q * m + k], v[k], a); b = fma(c.y[q * m + k], av[k], b); }
      V[(uint64_t)q * ld + i] = a;
      AV[(uint64_t)q * ld + i] = b;
    }
  }
}

// what fp32 storage drops of the diagonal entries alpha - lambda_0: Chi_ii = float(alpha - lambda_0),
// Clo_ii = float((alpha - lambda_0) - Chi_ii)
__global__ void k_coupling_set_diag(float* __restrict__ Chi, float* __restrict__ Clo, uint32_t ld, int n, double value) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float hi = (float)value;
  const uint64_t at = blocked_index(ld, (uint32_t)i, (uint32_t)i);
  Chi[at] = hi;
  Clo[at] = (float)(value - (double)hi);
}

int coupling_set_diag(nugpr_ctx* c, double value, hipStream_t s) {
  const Layout& L = c->L;
  hipLaunchKernelGGL(k_coupling_set_diag, dim3((L.ncr + 255) / 256), dim3(256), 0, s, c->C, c->Clo, (uint32_t)L.ldc, L.ncr,
                     value);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

// eigen-decomposition of a small symmetric matrix (row-major m x m, overwritten) by cyclic Jacobi rotations:
// eigenvalues ascending in ev, eigenvectors in the columns of Y (row-major m x m)
static void small_sym_eigen(std::vector<double>& A, int m, std::vector<double>& ev, std::vector<double>& Y) {
  Y.assign((size_t)m * m, 0.0);
  for (int i = 0; i < m; ++i) Y[(size_t)i * m + i] = 1.0;
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int i = 0; i < m; ++i)
      for (int j = 0; j < m; ++j) (i == j ? diag : off) += A[(size_t)i * m + j] * A[(size_t)i * m + j];
    if (off <= 1e-32 * diag) break;
    const double none = 1e-33 * diag / ((double)m * m);      // entries this small, all together, pass the test above
    for (int p = 0; p < m; ++p)
      for (int q = p + 1; q < m; ++q) {
        const double apq = A[(size_t)p * m + q];
        if (apq * apq <= none) continue;
        const double tau = (A[(size_t)q * m + q] - A[(size_t)p * m + p]) / (2.0 * apq);
        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (std::fabs(tau) + std::sqrt(1.0 + tau * tau));
        const double cs = 1.0 / std::sqrt(1.0 + t * t), sn = t * cs;
        for (int k = 0; k < m; ++k) {             // columns p, q
          const double akp = A[(size_t)k * m + p], akq = A[(size_t)k * m + q];
          A[(size_t)k * m + p] = cs * akp - sn * akq;
          A[(size_t)k * m + q] = sn * akp + cs * akq;
        }
        for (int k = 0; k < m; ++k) {             // rows p, q
          const double apk = A[(size_t)p * m + k], aqk = A[(size_t)q * m + k];
          A[(size_t)p * m + k] = cs * apk - sn * aqk;
          A[(size_t)q * m + k] = sn * apk + cs * aqk;
        }
        for (int k = 0; k < m; ++k) {
          const double ykp = Y[(size_t)k * m + p], ykq = Y[(size_t)k * m + q];
          Y[(size_t)k * m + p] = cs * ykp - sn * ykq;
          Y[(size_t)k * m + q] = sn * ykp + cs * ykq;
        }
      }
  }
  std::vector<int> order(m);
  for (int i = 0; i < m; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int a, int b) { return A[(size_t)a * m + a] < A[(size_t)b * m + b]; });
  ev.resize(m);
  std::vector<double> Ys((size_t)m * m);
  for (int q = 0; q < m; ++q) {
    ev[q] = A[(size_t)order[q] * m + order[q]];
    for (int k = 0; k < m; ++k) Ys[(size_t)k * m + q] = Y[(size_t)k * m + order[q]];
  }
  Y.swap(Ys);
}

// The two lowest eigenvalues and the eigenvector y of the lowest one, for the steps that need no more: Householder reduction
// to tridiagonal form, eigenvalues by the QL iteration, the vector by inverse iteration there (Gaussian elimination with
// row exchanges) and back.  H: m x m, row stride DAV_MAX_BASIS.  At 24 x 24 39 us; all eigenvectors by Jacobi rotations 220.
int lowest_eigenpair(const std::vector<double>& H, int m, double& e0, double& e1, double* y) {
  constexpr int S = DAV_MAX_BASIS;
  y[0] = 1.0;
  e0 = H[0];
  e1 = INFINITY;
  if (m == 1) return 0;
  double A[S][S], beta[S] = {};
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) A[i][j] = H[(size_t)i * S + j];
  std::vector<double> d(m), e(m, 0.0), z;
  for (int k = 0; k + 2 < m; ++k) {                   // the reflector's vector stays in row k
    double norm2 = 0.0, tail = 0.0;
    for (int i = k + 1; i < m; ++i) norm2 += A[k][i] * A[k][i];
    for (int i = k + 2; i < m; ++i) tail += std::fabs(A[k][i]);
    if (tail == 0.0) { e[k] = A[k][k + 1]; continue; }
    const double a = A[k][k + 1] > 0.0 ? -std::sqrt(norm2) : std::sqrt(norm2);
    e[k] = a;
    A[k][k + 1] -= a;
    beta[k] = -1.0 / (a * A[k][k + 1]);               // 2 / |v|^2
    double p[S], pv = 0.0;
    for (int i = k + 1; i < m; ++i) {
      double s = 0.0;
      for (int j = k + 1; j < m; ++j) s += A[i][j] * A[k][j];
      p[i] = beta[k] * s;
      pv += p[i] * A[k][i];
    }
    for (int i = k + 1; i < m; ++i) p[i] -= 0.5 * beta[k] * pv * A[k][i];
    for (int i = k + 1; i < m; ++i)
      for (int j = k + 1; j < m; ++j) A[i][j] -= A[k][i] * p[j] + p[i] * A[k][j];
  }
  e[m - 2] = A[m - 2][m - 1];
  for (int i = 0; i < m; ++i) d[i] = A[i][i];
  std::vector<double> ev = d, off = e;
  if (tridiag_eigen_first_row(ev, off, z)) return 1;
  std::nth_element(ev.begin(), ev.begin() + 1, ev.end());
  e0 = ev[0];
  e1 = ev[1];
  double scale = 0.0;
  for (int i = 0; i < m; ++i) scale = std::max(scale, std::fabs(d[i]) + std::fabs(e[i]));
  const double tiny = std::max(2.3e-16 * scale, 1e-300);
  // T - e0 I = P^T L U: diagonal u0, first and second upper diagonals u1, u2
  double u0[S], u1[S] = {}, u2[S] = {}, mult[S] = {};
  bool swapped[S] = {};
  double p0 = d[0] - e0, p1 = e[0];
  for (int i = 0; i + 1 < m; ++i) {
    const double l = e[i], q0 = d[i + 1] - e0, q1 = i + 2 < m ? e[i + 1] : 0.0;
    if (std::fabs(l) > std::fabs(p0)) {
      swapped[i] = true;
      mult[i] = p0 / l;
      u0[i] = l; u1[i] = q0; u2[i] = q1;
      p0 = p1 - mult[i] * q0;
      p1 = -mult[i] * q1;
    } else {
      if (std::fabs(p0) < tiny) p0 = tiny;
      mult[i] = l / p0;
      u0[i] = p0; u1[i] = p1;
      p0 = q0 - mult[i] * p1;
      p1 = q1;
    }
  }
  u0[m - 1] = std::fabs(p0) < tiny ? tiny : p0;
  for (int i = 0; i < m; ++i) y[i] = 1.0 + 0.01 * i;
  for (int it = 0; it < 3; ++it) {
    for (int i = 0; i + 1 < m; ++i) {
      if (swapped[i]) std::swap(y[i], y[i + 1]);
      y[i + 1] -= mult[i] * y[i];
    }
    double norm = 0.0;
    for (int i = m - 1; i >= 0; --i) {
      double s = y[i];
      if (i + 1 < m) s -= u1[i] * y[i + 1];
      if (i + 2 < m) s -= u2[i] * y[i + 2];
      y[i] = s / u0[i];
      norm = std::max(norm, std::fabs(y[i]));
    }
    if (!(norm > 0.0) || !std::isfinite(norm)) return 1;
    double sq = 0.0;
    for (int i = 0; i < m; ++i) { y[i] /= norm; sq += y[i] * y[i]; }
    sq = 1.0 / std::sqrt(sq);
    for (int i = 0; i < m; ++i) y[i] *= sq;
  }
  for (int k = m - 3; k >= 0; --k) {
    if (beta[k] == 0.0) continue;
    double s = 0.0;
    for (int i = k + 1; i < m; ++i) s += A[k][i] * y[i];
    s *= beta[k];
    for (int i = k + 1; i < m; ++i) y[i] -= s * A[k][i];
  }
  return 0;
}

// lambda_min of the matrix whose off-diagonal part is stored in (c->C, c->Clo) (diagonal entries of both zero)
// and whose diagonal is the scalar alpha = theta[p - 2].  Scratch: the partial-sum slabs of the coupling product
// and the Davidson area of the workspace.  The host waits for the device once per step.
int coupling_lambda_min(nugpr_ctx* c, const double* theta, hipStream_t s, double* lambda_out, int* steps_out) {
  const Layout& L = c->L;
  const int n = L.ncr, ld = L.ldc;
  if (!c->acc64) { set_error("the matrix-free lambda_0 needs the fp64 arithmetic mode"); return NUGPR_ERR_INVALID; }
  const bool iso = (c->params.flags & NUGPR_ISOTROPIC) != 0;
  const double alpha = theta[L.p - 2];
  const int nblk = (n + EB - 1) / EB;
  // (the partial sums: two sets of DAV_MAX_BASIS and one of DAV_MAX_BASIS + 1 dot products, two of squares, a value per
  // block of 128 rows: at most n doubles, as n is larger than COMPENSATE_HOST_MAX)
  double *V = c->dav, *AV = V + (size_t)DAV_MAX_BASIS * ld, *sums = AV + (size_t)DAV_MAX_BASIS * ld, *tvec = sums + ld, *Lblk = tvec + ld + 64;
  static_assert((COMPENSATE_HOST_MAX + EB) / EB * (3 * DAV_MAX_BASIS + 3) <= COMPENSATE_HOST_MAX, "room for the partial sums");
  double *res2 = sums, *norm2 = res2 + nblk, *dots1 = norm2 + nblk, *dots2 = dots1 + DAV_MAX_BASIS * nblk, *dots3 = dots2 + DAV_MAX_BASIS * nblk;
  constexpr int factor_lds = BF_LDS;
  static const hipError_t lds_attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_block_factor),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, factor_lds);
  NUGPR_HIP(lds_attr);
  BlockKernelArgs ba;
  for (int k = 0; k < MAX_D; ++k) ba.inv_ell[k] = k < L.d ? 1.0 / (iso ? theta[0] : theta[k]) : 0.0;
  ba.alpha = alpha; ba.mu = 1e-10 * alpha; ba.n = n; ba.d = L.d;
  hipLaunchKernelGGL(k_block_factor, dim3(nblk), dim3(BF_THREADS), factor_lds, s, ba, c->reps, Lblk);
  hipLaunchKernelGGL(k_eig_start, dim3(64), dim3(256), 0, s, V, n);
  NUGPR_HIP(hipGetLastError());
  const uint64_t stride = (uint64_t)n;            // one column: a slab of the partial sums is n doubles
  double* parts = static_cast<double*>(c->Ppart);
  const bool together = L.T >= 2;
  const double tol = EIGMIN_REL_TOL * std::fabs(alpha);
  int rc;
  // C V[m] into AV[m] and the new row of H; returns after the host has the row
  std::vector<double> H((size_t)DAV_MAX_BASIS * DAV_MAX_BASIS, 0.0);
  auto extend = [&](int m) -> int {             // V[m] exists: AV[m] = C V[m], H[m][0..m]
    StripPort p{};
    p.A = c->C; p.in = V + (size_t)m * ld; p.out = parts; p.out_part_stride = stride; p.diag_add = alpha;
    StripPort q = p;
    q.A = c->Clo; q.diag_add = 0.0;
    // Both terms in one launch, like two systems side by side, where the partial sums of a product (of L.T columns) have room for the
    // slabs of both; k_eig_newrow adds them up.  A loss on 32 clusters of 1024 points with 64 representatives, 24 steps: 1211 / 1163 us, on uneven ones
    // 1268 / 1230 (runs of one side differ by 0.5 %).
    if (together) {
      q.out = parts + (uint64_t)L.nsP * stride;
      const StripPort both[4] = {p, p, q, q};
      if ((rc = launch_strip(c->tab_C, both, 4, 1, true, s, 2))) return rc;
    } else {
      q.accumulate = 1;
      if ((rc = launch_strip(c->tab_C, p, p, 1, true, s))) return rc;
      if ((rc = launch_strip(c->tab_C, q, q, 1, true, s))) return rc;
    }
    c->flag_seq += 1;
    hipLaunchKernelGGL(k_eig_newrow, dim3(nblk), dim3(1024), 0, s, (const double*)parts, together ? 2 * L.nsP : L.nsP, stride, V, AV, m, n, ld,
                       m > 0 ? norm2 : (const double*)nullptr, m > 0 ? res2 : (const double*)nullptr, dots3, c->h_buf, c->d_state, c->h_flags, c->flag_seq);
    NUGPR_HIP(hipGetLastError());
    if ((rc = wait_seq(&c->h_flags->seq, c->flag_seq, s))) return rc;
    for (int k = 0; k <= m; ++k) {
      const double h = c->h_buf[8 + k];
      if (!std::isfinite(h)) { set_error("lambda_0: the projected matrix is not finite"); return NUGPR_ERR_INVALID; }
      H[(size_t)m * DAV_MAX_BASIS + k] = H[(size_t)k * DAV_MAX_BASIS + m] = h;
    }
    return NUGPR_OK;
  };
  if ((rc = extend(0))) return rc;
  int m = 1, step = 0;
  double thetaR = H[0], est = INFINITY;
  bool done = false;
  std::vector<double> A, ev, Y;
  for (; step < DAV_MAX_STEPS; ++step) {
    Coef cf = {};
    double second = INFINITY;
    if (m < DAV_MAX_BASIS) {
      if (lowest_eigenpair(H, m, thetaR, second, cf.y)) { set_error("lambda_0: the projected eigen-solve did not converge"); return NUGPR_ERR_INVALID; }
    } else {
      // thick restart: the lowest Ritz vectors become the basis, H their (diagonal) Rayleigh quotients
      A.assign((size_t)m * m, 0.0);
      for (int i = 0; i < m; ++i)
        for (int j = 0; j < m; ++j) A[(size_t)i * m + j] = H[(size_t)i * DAV_MAX_BASIS + j];
      small_sym_eigen(A, m, ev, Y);
      thetaR = ev[0];
      second = ev[1];
      RestartCoef rcf;
      for (int q = 0; q < DAV_KEEP; ++q)
        for (int k = 0; k < m; ++k) rcf.y[q * m + k] = Y[(size_t)k * m + q];
      hipLaunchKernelGGL(k_eig_restart, dim3(64), dim3(256), 0, s, V, AV, rcf, m, DAV_KEEP, n, ld);
      NUGPR_HIP(hipGetLastError());
      std::fill(H.begin(), H.end(), 0.0);
      for (int q = 0; q < DAV_KEEP; ++q) H[(size_t)q * DAV_MAX_BASIS + q] = ev[q];
      m = DAV_KEEP;
      cf.y[0] = 1.0;
    }
    hipLaunchKernelGGL(k_eig_correct, dim3(nblk), dim3(1024), 0, s, (const double*)V, (const double*)AV, cf, thetaR, m, n, ld,
                       (const double*)Lblk, tvec, res2, dots1);
    hipLaunchKernelGGL((k_eig_orth<false>), dim3(nblk), dim3(1024), 0, s, V, tvec, m, n, ld, (const double*)dots1, dots2);
    hipLaunchKernelGGL((k_eig_orth<true>), dim3(nblk), dim3(1024), 0, s, V, tvec, m, n, ld, (const double*)dots2, norm2);
    NUGPR_HIP(hipGetLastError());
    if ((rc = extend(m))) return rc;              // (also brings |res|^2 and the norm of the new direction)
    const double rn = std::sqrt(std::max(c->h_buf[0], 0.0)), tn = c->h_buf[1];
    if (!std::isfinite(rn)) { set_error("lambda_0: residual not finite"); return NUGPR_ERR_INVALID; }
    est = rn;
    if (m > 1) {
      const double gap = second - thetaR;
      if (gap > 10.0 * rn) est = std::min(est, 4.0 * rn * rn / gap);
    }
    if (est <= tol || std::fabs(thetaR) <= tol) { done = true; break; }
    if (!(tn > 1e-300)) { done = est <= 1e3 * tol; break; }       // no new direction: the basis holds an invariant subspace
    m += 1;
  }
  if (steps_out) *steps_out = std::min(step + 1, DAV_MAX_STEPS);
  if (!done && std::fabs(thetaR) <= EIGMIN_PSD_TOL * std::fabs(alpha)) done = true;   // lambda_min in [0, theta], see above
  if (!done) {
    set_error("lambda_0: the eigenvalue iteration did not reach the tolerance in " + std::to_string(DAV_MAX_STEPS) + " steps");
    return NUGPR_ERR_INVALID;
  }
  *lambda_out = thetaR;
  return NUGPR_OK;
}

}  // namespace nugpr
