// Batched preconditioned CG (Sections 3.1-3.2; the vector operations of Tables 1-2) and
// the two operator applications it alternates: the block-low-rank product K' D and the
// block-Jacobi preconditioner M^-1 R.
//
// All T columns advance in lock step.  Vector blocks are n x T row-major, fp64 or fp32
// according to the context's arithmetic mode (VT below); every reduction that feeds a CG
// coefficient (the paper's batched dot products) is accumulated in fp64 in a fixed order:
// per-workgroup partial sums, which up to FUSE_BLOCKS of them (32768 points) are added up by
// every workgroup of the kernel that applies alpha or beta, and beyond by a small kernel of one
// workgroup per column (k_pcg_alpha, k_pcg_beta).  The stop test (k_pcg_check) is such a kernel
// at every size; it keeps the convergence mask on the device and stores a 16-byte flag record
// into pinned host memory (O(1) traffic, Section 4), which the host polls once per iteration,
// on problems of up to FUSE_BLOCKS partial sums one iteration late while a solve is expected to
// go on (pcg_t).
#include <algorithm>
#include <cmath>
#include <cstring>

#include "nugpr_internal.h"

namespace nugpr {

// Several systems side by side (blockIdx.y = which one): every kernel of the solver finds the blocks of system y at a fixed
// number of bytes from those of system 0 (the solver slots of the workspace), or, with 0, shares them.
template <typename P>
__device__ __forceinline__ P* of_system(P* p, uint64_t stride) {
  return reinterpret_cast<P*>(reinterpret_cast<char*>(p) + (uint64_t)blockIdx.y * stride);
}
template <typename P>
__device__ __forceinline__ const P* of_system(const P* p, uint64_t stride) {
  return reinterpret_cast<const P*>(reinterpret_cast<const char*>(p) + (uint64_t)blockIdx.y * stride);
}

// The vector kernels with dot products: workgroups of up to 512 threads, a thread owns one column of every (threads / T)-th row, four
// rows at a time with all their loads ahead of the first use.  Up to 32768 points there is one workgroup a system on a compute
// unit, so what bounds them is how many loads are in flight; beyond, HBM.  Update of two systems of 32768 x 17 values with 256
// threads and a row at a time 22.0 us, now 13.9 (1024 threads: 18.9), of one of 131072 20.8 / 21.0 (28.6), of 262144 40 / 34; the
// product's last pass 11.7 / 7.3, 14.9 / 13.2, 28 / 25.
constexpr int VB = 512;
constexpr int ROWS_AT_ONCE = 4;
// Narrow blocks: fewer threads, which the rows of a workgroup still fill, and shorter sums over them.  Eight iterations in fp64,
// 128 / 256 / 512 threads in per cent of one row at a time with 256: one column 81 / 85 / 95 at 2048 points, 88 / 95 / 102 at
// 32768, 92 / 94 / 104 at 131072; five columns 93 / 98 / 98 at 8192, 111 / 102 / 102, 98 / 96 / 100; eight 90 / 89 / 92 at 2048, 100 / 97 / 97,
// 98 / 97 / 100; nine 90 / 87 / 89, 101 / 98 / 95, 98 / 98 / 99; seventeen 91 / 88 / 88, 98 / 93 / 90, 98 / 97 / 97.
static int vector_threads(int T) { return T == 1 ? 128 : T <= 8 ? 256 : VB; }
// sums[col] of the workgroup's values (thread = row of the pass times T + column), in a fixed order: eight groups of rows,
// then the groups.  red holds the values; the result is valid for threads below T.
__device__ __forceinline__ double column_sum(double* red, int T, int tid) {
  const int rpp = (int)blockDim.x / T, g = tid / T;
  __syncthreads();
  double s = 0.0;
  if (g < 8) {
    for (int k = g; k < rpp; k += 8) s += red[k * T + tid - g * T];
  }
  __syncthreads();
  if (g < 8) red[tid] = s;
  __syncthreads();
  if (tid < T)
    for (int k = 1; k < 8 && k < rpp; ++k) s += red[k * T + tid];
  return s;
}

// ---------------------------------------------------------------------------
// per-column dot products: partial[which][block][col] = sum over the block's rows
// ---------------------------------------------------------------------------
template <int NP, typename VT>
__global__ __launch_bounds__(VB) void k_dot(const VT* __restrict__ A0, const VT* __restrict__ B0,
                                            const VT* __restrict__ A1, const VT* __restrict__ B1,
                                            int64_t n, int T, double* __restrict__ partial, uint64_t sa, uint64_t sb, uint64_t sys) {
  __shared__ double red[NP][VB];
  A0 = of_system(A0, sa); B0 = of_system(B0, sb);
  A1 = of_system(A1, sa); B1 = of_system(B1, sb);
  partial = of_system(partial, sys);
  const int rpp = (int)blockDim.x / T;          // rows per pass
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  const int64_t rows_per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  double s0 = 0.0, s1 = 0.0;
  if (myrow < rpp) {
    for (int64_t r = r0 + myrow; r < r1; r += ROWS_AT_ONCE * rpp) {
      VT a0[ROWS_AT_ONCE], b0[ROWS_AT_ONCE], a1[ROWS_AT_ONCE], b1[ROWS_AT_ONCE];
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j) {
        const int64_t idx = (r + j * rpp < r1 ? r + j * rpp : r) * T + col;
        a0[j] = A0[idx]; b0[j] = B0[idx];
        if (NP > 1) { a1[j] = A1[idx]; b1[j] = B1[idx]; }
      }
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j)
        if (r + j * rpp < r1) {
          s0 = fma((double)a0[j], (double)b0[j], s0);
          if (NP > 1) s1 = fma((double)a1[j], (double)b1[j], s1);
        }
    }
  }
  red[0][tid] = s0;
  if (NP > 1) red[NP - 1][tid] = s1;
  for (int w = 0; w < NP; ++w) {
    const double s = column_sum(red[w], T, tid);
    if (tid < T) partial[((int64_t)w * gridDim.x + blockIdx.x) * MAX_COLS + tid] = s;
  }
}

// sum over the 64 lanes of a wave by register shuffles, fixed pairing (lane, lane + 32), (lane, lane + 16), ..;
// lane 0 holds the result
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

__device__ __forceinline__ double sum_partials(const double* __restrict__ partial, int nblocks, int col,
                                               double* red, int tid) {
  // 256 threads cooperate on one column at a time, fixed order: strided partial sums per thread, shuffles
  // inside each wave, then the four wave totals through LDS
  double s = 0.0;
  for (int b = tid; b < nblocks; b += 256) s += partial[(int64_t)b * MAX_COLS + col];
  s = wave_sum(s);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  const double r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// The scalar kernels run one workgroup per column (grid = T); the cross-column
// bookkeeping (how many columns are still active, did any meet negative curvature) is
// gathered by the last workgroup of the stop test (k_pcg_check).

// start of a solve: ||b||^2 and rho_0 = <r_0, z_0>
__device__ __forceinline__ void begin_column(PcgState* st, int c, double bb, double rz, bool act) {
  st->bnorm2[c] = bb;
  st->rho[0][c] = rz;
  st->rho0[c] = rz;
  st->alpha[c] = 0.0;
  st->beta[c] = 0.0;
  st->active[c] = act ? 1 : 0;
  st->iters[c] = 0;
  st->converged[c] = (bb == 0.0) ? 1 : 0;
  st->indef[c] = 0;
}
__global__ __launch_bounds__(256) void k_pcg_begin(PcgState* __restrict__ st, const double* __restrict__ partial,
                                                   int nblocks, uint64_t sys) {
  __shared__ double red[256];
  const int tid = threadIdx.x, c = blockIdx.x;
  st = of_system(st, sys);
  partial = of_system(partial, sys);
  const double bb = sum_partials(partial, nblocks, c, red, tid);
  const double rz = sum_partials(partial + (int64_t)nblocks * MAX_COLS, nblocks, c, red, tid);
  if (tid == 0) begin_column(st, c, bb, rz, bb > 0.0 && rz == rz);
}

// the same from the values kept with the factor (which = 0: [y | L Z], 1: the probe block), where the update kernel does
// not see to it
__global__ void k_pcg_begin_known(PcgState* st, int which, int T) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= T) return;
  const double bb = st->known_bb[which][c], rz = st->known_rz[which][c];
  begin_column(st, c, bb, rz, bb > 0.0 && rz == rz);
}

__global__ __launch_bounds__(256) void k_store_known(PcgState* __restrict__ st, const double* __restrict__ partial,
                                                     int nblocks, int which) {
  __shared__ double red[256];
  const int tid = threadIdx.x, c = blockIdx.x;
  const double bb = sum_partials(partial, nblocks, c, red, tid);
  const double rz = sum_partials(partial + (int64_t)nblocks * MAX_COLS, nblocks, c, red, tid);
  if (tid == 0) { st->known_bb[which][c] = bb; st->known_rz[which][c] = rz; }
}

// alpha_c = rho_c / <d, K'd>_c for the active columns
__global__ __launch_bounds__(256) void k_pcg_alpha(PcgState* __restrict__ st, const double* __restrict__ partial,
                                                   int nblocks, int iter, double* __restrict__ alog) {
  __shared__ double red[256];
  const int tid = threadIdx.x, c = blockIdx.x;
  const double dq = sum_partials(partial, nblocks, c, red, tid);
  if (tid == 0) {
    double a = 0.0;
    if (st->active[c]) {
      if (dq > 0.0) a = st->rho[iter & 1][c] / dq;
      else { st->indef[c] = 1; st->active[c] = 0; }      // <d, K'd> <= 0 (or NaN)
    }
    st->alpha[c] = a;
    alog[(int64_t)iter * MAX_COLS + c] = a;
  }
}

// End-of-solve report, written by the device straight into pinned host memory: the per-column state, <b_c, x_c> summed from the
// per-workgroup partials (fixed order), and the first `rows` rows of the alpha / beta logs.  It comes with the stop test of the
// iteration that is expected to be the last, and of the one after it (k_pcg_check; a kernel of its own, 5 - 7 us, otherwise:
// k_pcg_tail).
struct Report {
  uint64_t seq;                    // 0: none
  int want_bx, rows;
  const double *alog, *blog;       // (of system 0, as the host's)
  PcgState* h_state;
  double *h_bx, *h_alog, *h_blog;
  uint64_t hsys;                   // bytes from a system's part of the host buffer to the next one's
};
// what state and logs a report holds, by `threads` threads; state read past what this workgroup has cached
__device__ __forceinline__ void copy_state(const PcgState* st, const Report& r, int at, int threads) {
  const int words = (int)(sizeof(PcgState) / sizeof(int32_t));
  const volatile int32_t* src = reinterpret_cast<const volatile int32_t*>(st);
  int32_t* dst = reinterpret_cast<int32_t*>(of_system(r.h_state, r.hsys));
  for (int i = at; i < words; i += threads) dst[i] = src[i];
}
__device__ __forceinline__ void copy_logs(const Report& r, uint64_t sys, int T, int at, int threads) {
  const double *alog = of_system(r.alog, sys), *blog = of_system(r.blog, sys);
  double *h_alog = of_system(r.h_alog, r.hsys), *h_blog = of_system(r.h_blog, r.hsys);
  for (int i = at; i < r.rows * T; i += threads) {
    const int e = i / T * MAX_COLS + i % T;
    h_alog[e] = alog[e];
    h_blog[e] = blog[e];
  }
}

// after the update: stop test on ||r_c|| (columns that meet it are frozen).  The workgroup that finishes
// last gathers the cross-column bookkeeping (how many columns are still active, did any meet negative
// curvature) and publishes it to the host: the flags, a system-scope fence, then the sequence number.
// With a report the workgroups share the copy of the logs, which the host then waits for with the flags.
__global__ __launch_bounds__(256) void k_pcg_check(PcgState* __restrict__ st, const double* __restrict__ partial,
                                                   int nblocks, int iter, double tol2, int T,
                                                   HostFlags* __restrict__ out, uint64_t seq, uint64_t sys, Report report) {
  __shared__ double red[256];
  __shared__ int last;
  const int tid = threadIdx.x, c = blockIdx.x;
  st = of_system(st, sys);
  partial = of_system(partial, sys);
  out += blockIdx.y;
  const double rr = sum_partials(partial, nblocks, c, red, tid);
  if (report.seq) {
    if (report.want_bx) {
      const double bx = sum_partials(partial + (int64_t)nblocks * MAX_COLS, nblocks, c, red, tid);
      if (tid == 0) of_system(report.h_bx, report.hsys)[c] = bx;
    }
    const int at = c * 256 + tid;
    copy_logs(report, sys, T, at, 256 * T);
    if (at < report.rows * T || tid == 0) __threadfence_system();      // (whoever stored something)
    __syncthreads();
  }
  if (tid == 0) {
    if (st->active[c]) {
      st->iters[c] = iter + 1;
      if (rr <= tol2 * st->bnorm2[c]) {
        st->active[c] = 0;
        st->converged[c] = 1;
      } else if (!(rr == rr)) {                // NaN residual: stop this column
        st->active[c] = 0;
        st->indef[c] = 1;
      }
    }
    __threadfence();
    last = (atomicAdd(&st->check_count, 1) == T - 1);
  }
  __syncthreads();
  if (!last) return;
  if (tid < 64) {                              // one wave, a lane per column (one after the other: 4 us)
    __threadfence();
    int act = 0, ind = 0;
    if (tid < T) {
      act = *reinterpret_cast<volatile int32_t*>(&st->active[tid]);
      ind = *reinterpret_cast<volatile int32_t*>(&st->indef[tid]);
    }
    const int n_active = __popcll(__ballot(act != 0)), indef = __ballot(ind != 0) != 0 ? 1 : 0;
    if (tid == 0) {
      st->check_count = 0;
      if (iter == 0 || st->n_active != 0) st->steps = iter + 1;     // (n_active: what the test before this one found)
      st->n_active = n_active;
      st->indefinite = indef;
      out->n_active = n_active;
      out->indefinite = indef;
      out->bad_cluster = st->bad_cluster;
      if (!report.seq) {
        __threadfence_system();
        *reinterpret_cast<volatile uint64_t*>(&out->seq) = seq;
      }
    }
  }
  if (!report.seq) return;
  __threadfence();
  __syncthreads();                             // the state is what the other workgroups and thread 0 left
  copy_state(st, report, tid, 256);
  __threadfence_system();
  __syncthreads();
  if (tid == 0) {
    *reinterpret_cast<volatile uint64_t*>(&out->tail_seq) = report.seq;
    *reinterpret_cast<volatile uint64_t*>(&out->seq) = seq;
  }
}

// beta_c = <r, z>_new / rho_c for the columns that go on
__global__ __launch_bounds__(256) void k_pcg_beta(PcgState* __restrict__ st, const double* __restrict__ partial,
                                                  int nblocks, int iter, double* __restrict__ blog) {
  __shared__ double red[256];
  const int tid = threadIdx.x, c = blockIdx.x;
  const double rz = sum_partials(partial, nblocks, c, red, tid);
  if (tid == 0) {
    double bta = 0.0;
    if (st->active[c]) {
      if (!(rz > 0.0)) {                     // preconditioned residual lost positivity (or NaN)
        st->active[c] = 0;
        st->indef[c] = 1;
      } else {
        bta = rz / st->rho[iter & 1][c];
        st->rho[(iter + 1) & 1][c] = rz;
      }
    }
    st->beta[c] = bta;
    blog[(int64_t)iter * MAX_COLS + c] = bta;
  }
}

// Problems of up to FUSE_BLOCKS partial sums per column (32768 points): the kernels that apply alpha and beta sum them
// up themselves, every workgroup in the same fixed order (35 KB of L2 reads a workgroup at 256 x 17), and the first
// one keeps the records.  That saves a launch of 3 - 5 us each; with 1024 partial sums every workgroup would read 139 KB.
// The line: a loss with them in the kernels / with launches of their own takes 254 / 261 us at 24576 points (192 sums),
// 271 / 273 at 32768 (256), 304 / 302 at 40960 (320), 372 / 351 at 65536 (512), 664 / 579 at 131072 (1024).
constexpr int FUSE_BLOCKS = 256;
__device__ __forceinline__ void sum_all_partials(const double* __restrict__ partial, int nblocks, int T, double* red, double* out) {
  const int rpp = (int)blockDim.x / T, tid = threadIdx.x, myrow = tid / T, col = tid - myrow * T;
  double s = 0.0;
  if (myrow < rpp) {
#pragma unroll 4
    for (int b = myrow; b < nblocks; b += rpp) s += partial[(int64_t)b * MAX_COLS + col];
  }
  red[tid] = s;
  s = column_sum(red, T, tid);
  if (tid < T) out[tid] = s;
  __syncthreads();
}

// X += D diag(alpha); R -= Q diag(alpha)   (alpha stays in fp64: rounding it to fp32 would scale the whole
// step coherently).  In the first step of a solve X starts from zero and R from Rin = b, neither of which is
// read or written before.  The update is fused with the two reductions that follow it: partial[0] = per-workgroup sums of r_new^2
// (the stop test) and, when B is given, partial[1] = sums of b x_new (the quadratic form of the end-of-solve
// report).  Rows are split among the workgroups as in k_dot, so the sums are those k_dot would produce.
template <typename VT>
__global__ __launch_bounds__(VB) void k_update_xr_dots(VT* __restrict__ X, VT* R, const VT* Rin,
                                                        const VT* __restrict__ D, const VT* __restrict__ Q,
                                                        const VT* __restrict__ B, PcgState* __restrict__ st,
                                                        int64_t n, int T, int first, double* __restrict__ partial,
                                                        const double* __restrict__ dqs, int iter, double* __restrict__ alog,
                                                        uint64_t sys, uint64_t s_in, uint64_t s_d, uint64_t s_b, int known) {
  __shared__ double red[2][VB];
  const PcgState* st0 = st;                    // (system 0's: keeps the values of the context's own right-hand sides)
  __shared__ double al[MAX_COLS];
  X = of_system(X, sys); R = of_system(R, sys); Q = of_system(Q, sys);
  Rin = of_system(Rin, s_in); D = of_system(D, s_d);
  if (B) B = of_system(B, s_b);
  st = of_system(st, sys); partial = of_system(partial, sys); alog = of_system(alog, sys);
  if (dqs) dqs = of_system(dqs, sys);
  const int rpp = (int)blockDim.x / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  const bool live = myrow < rpp;
  if (dqs) {                                   // the step of k_pcg_alpha (a column the first workgroup stops here has a = 0 anyway)
    sum_all_partials(dqs, (int)gridDim.x, T, &red[0][0], al);
    if (tid < T) {
      const double dq = al[tid];
      bool act;
      double rho, bb = 0.0;
      if (known >= 0) {                        // first step of such a solve: the start of k_pcg_begin_known as well
        bb = st0->known_bb[known][tid];
        rho = st0->known_rz[known][tid];
        act = bb > 0.0 && rho == rho;
      } else {
        rho = st->rho[iter & 1][tid];
        act = st->active[tid] != 0;
      }
      const double a = act && dq > 0.0 ? rho / dq : 0.0;
      al[tid] = a;
      if (blockIdx.x == 0) {
        if (known >= 0) begin_column(st, tid, bb, rho, act);
        if (act && !(dq > 0.0)) { st->indef[tid] = 1; st->active[tid] = 0; }
        st->alpha[tid] = a;
        alog[(int64_t)iter * MAX_COLS + tid] = a;
      }
    }
    __syncthreads();
  }
  const int64_t rows_per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  double s0 = 0.0, s1 = 0.0;
  if (live) {
    const double a = dqs ? al[col] : st->alpha[col];
    for (int64_t r = r0 + myrow; r < r1; r += ROWS_AT_ONCE * rpp) {
      VT d[ROWS_AT_ONCE], q[ROWS_AT_ONCE], x[ROWS_AT_ONCE], b[ROWS_AT_ONCE], ri[ROWS_AT_ONCE];
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j) {
        const int64_t idx = (r + j * rpp < r1 ? r + j * rpp : r) * T + col;
        d[j] = D[idx]; q[j] = Q[idx]; ri[j] = Rin[idx];
        if (!first) x[j] = X[idx];
        if (B) b[j] = B[idx];
      }
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j)
        if (r + j * rpp < r1) {
          const int64_t idx = (r + j * rpp) * T + col;
          const VT xn = first ? (VT)(a * (double)d[j]) : (VT)fma(a, (double)d[j], (double)x[j]);
          const VT rn = (VT)fma(-a, (double)q[j], (double)ri[j]);
          X[idx] = xn;
          R[idx] = rn;
          s0 = fma((double)rn, (double)rn, s0);
          if (B) s1 = fma((double)b[j], (double)xn, s1);
        }
    }
  }
  red[0][tid] = s0;
  red[1][tid] = s1;
  for (int w = 0; w < 2; ++w) {
    const double s = column_sum(red[w], T, tid);
    if (tid < T) partial[((int64_t)w * gridDim.x + blockIdx.x) * MAX_COLS + tid] = s;
  }
}

// D = Z + D diag(beta) for active columns, 0 for stopped ones
template <typename VT>
__global__ __launch_bounds__(VB) void k_update_d(VT* D, const VT* Din, const VT* __restrict__ Z,
                                                  PcgState* __restrict__ st, int64_t n, int T,
                                                  const double* __restrict__ rzs, int nblocks, int iter, double* __restrict__ blog,
                                                  uint64_t sys, uint64_t s_d) {
  D = of_system(D, sys); Din = of_system(Din, s_d); Z = of_system(Z, sys);
  st = of_system(st, sys); blog = of_system(blog, sys);
  if (rzs) rzs = of_system(rzs, sys);
  __shared__ double red[VB];
  __shared__ double be[MAX_COLS];
  __shared__ int goes_on[MAX_COLS];
  const int rpp = (int)blockDim.x / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  if (rzs) {                                   // the step of k_pcg_beta (beta itself can be negative: rho_0 may be, by rounding)
    sum_all_partials(rzs, nblocks, T, red, be);
    if (tid < T) {
      const double rz = be[tid];
      const bool act = st->active[tid] != 0, go = act && rz > 0.0;
      const double b = go ? rz / st->rho[iter & 1][tid] : 0.0;
      be[tid] = b;
      goes_on[tid] = go;
      if (blockIdx.x == 0) {
        if (act && !go) { st->active[tid] = 0; st->indef[tid] = 1; }
        if (go) st->rho[(iter + 1) & 1][tid] = rz;
        st->beta[tid] = b;
        blog[(int64_t)iter * MAX_COLS + tid] = b;
      }
    }
    __syncthreads();
  }
  if (myrow >= rpp) return;
  const double bta = rzs ? be[col] : st->beta[col];
  const bool act = rzs ? goes_on[col] != 0 : st->active[col] != 0;
  const int64_t step = (int64_t)gridDim.x * rpp;
  for (int64_t r = (int64_t)blockIdx.x * rpp + myrow; r < n; r += ROWS_AT_ONCE * step) {
    VT z[ROWS_AT_ONCE], d[ROWS_AT_ONCE];
#pragma unroll
    for (int j = 0; j < ROWS_AT_ONCE; ++j) {
      const int64_t idx = (r + j * step < n ? r + j * step : r) * T + col;
      z[j] = Z[idx]; d[j] = Din[idx];
    }
#pragma unroll
    for (int j = 0; j < ROWS_AT_ONCE; ++j)
      if (r + j * step < n) D[(r + j * step) * T + col] = act ? (VT)fma(bta, (double)d[j], (double)z[j]) : (VT)0;
  }
}

// The report by itself (partial: the sums of b x).  One workgroup per column (each sums its column; they share the copies); the
// workgroup that finishes last publishes the sequence number.
__global__ __launch_bounds__(256) void k_pcg_tail(PcgState* __restrict__ st, const double* __restrict__ partial,
                                                  int nblocks, int T, Report report, HostFlags* __restrict__ flags, uint64_t sys) {
  __shared__ double red[256];
  __shared__ int last;
  const int tid = threadIdx.x, c = blockIdx.x;
  st = of_system(st, sys); partial = of_system(partial, sys);
  flags += blockIdx.y;
  if (report.want_bx) {
    const double v = sum_partials(partial, nblocks, c, red, tid);
    if (tid == 0) of_system(report.h_bx, report.hsys)[c] = v;
  }
  copy_state(st, report, c * 256 + tid, 256 * T);
  copy_logs(report, sys, T, c * 256 + tid, 256 * T);
  __threadfence_system();
  __syncthreads();
  if (tid == 0) last = (atomicAdd(&st->tail_count, 1) == T - 1);
  __syncthreads();
  if (last && tid == 0) {
    st->tail_count = 0;
    __threadfence_system();
    *reinterpret_cast<volatile uint64_t*>(&flags->tail_seq) = report.seq;
  }
}

// Waits until the device has stored `want`, or a later number, in a pinned sequence slot: a short poll (the usual
// case: microseconds after the kernel ends), then an ordinary stream synchronisation.
int wait_seq(const volatile uint64_t* slot, uint64_t want, hipStream_t s) {
  for (int spin = 0; spin < 200000; ++spin) {
    if (*slot >= want) return NUGPR_OK;
    __builtin_ia32_pause();
  }
  NUGPR_HIP(hipStreamSynchronize(s));
  if (*slot < want) { set_error("the device did not report the end of a solver step"); return NUGPR_ERR_HIP; }
  return NUGPR_OK;
}

// start of a solve on a caller's right-hand sides: X = 0, R = B and, when the first direction is known
// (Z0 not null), D = Z0.  (The alpha / beta logs need no clearing: every row the host reads is written
// during the solve.)
template <typename VT>
__global__ void k_pcg_init(VT* __restrict__ X, VT* __restrict__ R, const VT* __restrict__ B,
                           const VT* __restrict__ Z0, VT* __restrict__ D, int64_t count, uint64_t sys, uint64_t s_b) {
  X = of_system(X, sys); R = of_system(R, sys); D = of_system(D, sys); B = of_system(B, s_b);
  if (Z0) Z0 = of_system(Z0, s_b);
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  if (Z0) {
    for (int64_t i = i0; i < count; i += stride) { X[i] = (VT)0; R[i] = B[i]; D[i] = Z0[i]; }
  } else {
    for (int64_t i = i0; i < count; i += stride) { X[i] = (VT)0; R[i] = B[i]; }
  }
}

template <typename SRC, typename DST>
__global__ void k_convert(const SRC* __restrict__ src, DST* __restrict__ dst, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = (DST)src[i];
}

int to_internal(nugpr_ctx* c, const float* src, void* dst, int64_t count, hipStream_t s) {
  if (c->acc64) hipLaunchKernelGGL((k_convert<float, double>), dim3(1024), dim3(256), 0, s, src, (double*)dst, count);
  else NUGPR_HIP(hipMemcpyAsync(dst, src, (size_t)count * sizeof(float), hipMemcpyDeviceToDevice, s));
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

int from_internal(nugpr_ctx* c, const void* src, float* dst, int64_t count, hipStream_t s) {
  if (c->acc64) hipLaunchKernelGGL((k_convert<double, float>), dim3(1024), dim3(256), 0, s, (const double*)src, dst, count);
  else NUGPR_HIP(hipMemcpyAsync(dst, src, (size_t)count * sizeof(float), hipMemcpyDeviceToDevice, s));
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

// ---------------------------------------------------------------------------
// operator applications on internal vector blocks
// ---------------------------------------------------------------------------
static int run_project(nugpr_ctx* c, const void* D, int T, hipStream_t s, const float* D32 = nullptr, int nsys = 1, uint64_t s_d = 0);
// Q = a Q0 + b D with the reduction that follows a product in the solver (partial as in
// k_onehot_expand_dot; may be null)
struct Combination { double a[MAX_SLOTS], b[MAX_SLOTS]; };
template <typename VT>
__global__ __launch_bounds__(VB) void k_lincomb_dot(VT* __restrict__ Q, const VT* __restrict__ Q0,
                                                     const VT* __restrict__ D, Combination of, int64_t n, int T,
                                                     double* __restrict__ partial, uint64_t sys) {
  __shared__ double red[VB];
  const double a = of.a[blockIdx.y], b = of.b[blockIdx.y];
  Q = of_system(Q, sys);
  if (partial) partial = of_system(partial, sys);
  const int rpp = (int)blockDim.x / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  const bool live = myrow < rpp;
  const int64_t rows_per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  double s0 = 0.0;
  if (live) {
    for (int64_t p = r0 + myrow; p < r1; p += ROWS_AT_ONCE * rpp) {
      VT d[ROWS_AT_ONCE], q[ROWS_AT_ONCE];
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j) {
        const int64_t idx = (p + j * rpp < r1 ? p + j * rpp : p) * T + col;
        d[j] = D[idx]; q[j] = Q0[idx];
      }
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j)
        if (p + j * rpp < r1) {
          const VT qn = (VT)fma(a, (double)q[j], b * (double)d[j]);
          Q[(p + j * rpp) * T + col] = qn;
          s0 = fma((double)d[j], (double)qn, s0);
        }
    }
  }
  red[tid] = s0;
  const double sum = column_sum(red, T, tid);
  if (partial && tid < T) partial[(int64_t)blockIdx.x * MAX_COLS + tid] = sum;
}

static int run_expand(nugpr_ctx* c, void* Q, int T, hipStream_t s, const void* D = nullptr, double* dq_partial = nullptr,
                      float* Q32 = nullptr, int parts = 1, int nsys = 1, uint64_t s_d = 0);
// How many column slabs of P the expansion adds up itself: all of them with the one-hot basis while the extra gathers
// (n T values from every slab after the first, out of L2) cost less than the launch they save.  A product with that
// launch / without it: 20.6 / 17.9 us at 0.02e6 gathers, 23.5 / 21.8 at 1e6, 42.5 / 41.2 at 2.1e6, 48.8 / 52.7 at 8.4e6.
static int fold_parts(const nugpr_ctx* c, int T) {
  return c->onehot && (double)c->L.n * T * (c->L.nsP - 1) <= 3e6 ? c->L.nsP : 1;
}

template <typename P> static P* slot_of(P* p, uint64_t stride, int e) { return (P*)((uintptr_t)p + (uint64_t)e * stride); }

// The one-hot projection (k_onehot_project): threads per representative and column, the power of two that leaves each at most eight
// points on average (one round of gathers), as far as the workgroup has them; large workgroups once an ordinary one has not.
struct ProjectShape { int block, parts, reps; };       // (reps: representatives of a workgroup)
static ProjectShape project_shape(const Layout& L, int T) {
  const int64_t want = (L.n + 8 * (int64_t)L.ncr - 1) / (8 * (int64_t)L.ncr);
  ProjectShape p;
  p.block = want > 256 / T ? 1024 : 256;
  p.parts = 1;
  while (2 * p.parts <= p.block / T && p.parts < want) p.parts *= 2;
  p.reps = p.block / T / p.parts;
  return p;
}
// Behind a projection of T columns: a byte for every odd_rows of its rows, whether a value there is not finite.
constexpr int DENSE_ODD_ROWS = TILE;
static size_t odd_offset(const nugpr_ctx* c, int T) {
  return ((size_t)c->L.ncr * T * (c->acc64 ? sizeof(double) : sizeof(float)) + 255) / 256 * 256;
}
static int odd_rows(const nugpr_ctx* c, int T) { return c->onehot ? project_shape(c->L, T).reps : DENSE_ODD_ROWS; }
// Products with C pass over items whose tiles hold no value, as the assembly of C left them (under the compensation its diagonal is
// written later), and whose vector rows are finite.  (Those of the kept projection of z_0 are: the first reduction of a solve refuses the
// others.)
static void skip_dead_items(const nugpr_ctx* c, StripPort& port, int T) {
  if (!c->c_skips) return;
  port.live = port.A == c->C ? c->c_live : port.A == c->C2 ? c->c2_live : nullptr;
  if (port.in == c->S0v) return;
  port.odd_at = (uint32_t)(odd_offset(c, T) / 256);
  port.odd_rows = (uint32_t)odd_rows(c, T);
}

// The product of `nsys` systems side by side, each with its operator; D and Q those of system 0, the others a slot further
// (the kept direction z_0 is shared).  More than one (2 or 4): one-hot basis, no compensation.  The counters and the timing
// take the first `held` of them.
static int product(nugpr_ctx* c, const Operator* ops, int nsys, int held, const void* D, void* Q, int T, hipStream_t s, double* dq_partial,
                   bool* dq_done, const float* D32, float* Q32) {
  const Layout& L = c->L;
  const uint64_t sys = L.slot_bytes;
  int rc;
  const uint64_t ppart = (uint64_t)L.ncr * T;
  // S_j = W_j^T D_j (dense W: in column slabs of W_j^T that are then added up); the projection of z_0, the
  // first direction of every solve on the context's own right-hand sides, is kept with the factor
  const bool s_known = D == c->Z0v && T == L.T && c->z0_ready && !D32;
  // The first direction again, on the blocks whose product with it is kept (base loss of a train step): the
  // operator is s K_0 + shift I for some other (s, shift), and the product a combination of what is kept.
  const bool shortcuts = !(c->params.flags & NUGPR_NO_SHORTCUTS);
  if (s_known && shortcuts && c->q0_gen == c->build_gen && Q != c->Q0v) {
    Combination of = {};
    for (int e = 0; e < nsys; ++e) {
      of.a[e] = ops[e].scale / c->q0_scale;
      of.b[e] = ops[e].shift - of.a[e] * c->q0_shift;
    }
    const dim3 nb((unsigned)L.n_dot_blocks, (unsigned)nsys);
    if (c->acc64) hipLaunchKernelGGL((k_lincomb_dot<double>), nb, dim3(vector_threads(T)), 0, s, (double*)Q, (const double*)c->Q0v, (const double*)D, of, (int64_t)L.n, T, dq_partial, sys);
    else hipLaunchKernelGGL((k_lincomb_dot<float>), nb, dim3(vector_threads(T)), 0, s, (float*)Q, (const float*)c->Q0v, (const float*)D, of, (int64_t)L.n, T, dq_partial, sys);
    NUGPR_HIP(hipGetLastError());
    if (dq_done) *dq_done = dq_partial != nullptr;
    c->stats.products_reused += held;
    return NUGPR_OK;
  }
  c->stats.products += held;
  const bool d_shared = D == c->Z0v;
  const uint64_t s_d = d_shared ? 0 : sys;
  if (!s_known && (rc = run_project(c, D, T, s, D32, nsys, s_d))) return rc;
  // Q_i = K_ii D_i   and   P = C_offdiag S (column slabs), one launch
  StripPort port[2 * MAX_SLOTS] = {};
  for (int e = 0; e < nsys; ++e) {
    StripPort &k0 = port[2 * e], &k1 = port[2 * e + 1];
    k0.A = ops[e].Kd; k0.in = slot_of(D, s_d, e); k0.out = slot_of(Q, sys, e); k0.scale = ops[e].scale; k0.diag_add = ops[e].shift;
    k1.A = ops[e].C; k1.in = s_known ? c->S0v : slot_of(c->Spart, sys, e); k1.out = slot_of(c->Ppart, sys, e);
    k1.out_part_stride = ppart; k1.scale = ops[e].scale;
    skip_dead_items(c, k1, T);
  }
  const bool timed = c->prof_on && (size_t)(2 * c->prof_used + 1) < c->prof_ev.size();
  if (timed) NUGPR_HIP(hipEventRecord(c->prof_ev[2 * c->prof_used], s));
  if ((rc = launch_strip(c->tab_KC, port, 2 * nsys, T, c->acc64, s, nsys))) return rc;
  if (timed) {
    NUGPR_HIP(hipEventRecord(c->prof_ev[2 * c->prof_used + 1], s));
    c->prof_used += 1;
    c->prof_systems += held;
  }
  if (L.compensate) {                     // the fp32 residual of C - lambda_0 I, added slab by slab
    StripPort k2 = port[1];
    k2.A = c->Clo; k2.accumulate = 1;
    if ((rc = launch_strip(c->tab_C, k2, k2, T, c->acc64, s))) return rc;
  }
  const int parts = fold_parts(c, T);
  if (L.nsP > parts && (rc = launch_sum_parts(c->Ppart, c->Ppart, (int64_t)ppart, L.nsP, ppart, c->acc64, s, nsys, sys))) return rc;
  // Q_i += W_i P_i (and, on request, the partial sums of <d, q> in the same pass)
  const bool fuse = dq_partial && c->onehot;
  if (dq_done) *dq_done = fuse;
  if ((rc = run_expand(c, Q, T, s, fuse ? D : nullptr, fuse ? dq_partial : nullptr, Q32, parts, nsys, s_d))) return rc;
  if (nsys == 1 && s_known && shortcuts && c->build_gen == c->factor_gen && c->q0_gen != c->build_gen) {
    const size_t bytes = (size_t)L.n * T * (c->acc64 ? sizeof(double) : sizeof(float));
    NUGPR_HIP(hipMemcpyAsync(c->Q0v, Q, bytes, hipMemcpyDeviceToDevice, s));
    c->q0_gen = c->build_gen;
    c->q0_scale = c->op_scale;
    c->q0_shift = c->op_shift;
  }
  return NUGPR_OK;
}

static Operator operator_in_force(const nugpr_ctx* c) { return Operator{c->Kd, c->C, c->op_scale, c->op_shift}; }

int run_matvec(nugpr_ctx* c, const void* D, void* Q, int T, hipStream_t s, double* dq_partial, bool* dq_done,
               const float* D32, float* Q32) {
  const Operator op = operator_in_force(c);
  return product(c, &op, 1, 1, D, Q, T, s, dq_partial, dq_done, D32, Q32);
}

// out = a * x  (elementwise over a vector block)
template <typename VT>
__global__ void k_scaled_copy(VT* __restrict__ out, const VT* __restrict__ x, double a, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (VT)(a * (double)x[i]);
}

// q = q + 4 a + d: the last step of Q(A) d = A(A d) + 4 A d + d (eq. (PQ)), with a = A d and q = A a on entry
template <typename VT>
__global__ void k_pade_q_combine(VT* __restrict__ q, const VT* __restrict__ a, const VT* __restrict__ d, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    q[i] = (VT)((double)q[i] + 4.0 * (double)a[i] + (double)d[i]);
}

template <typename VT>
static int scaled_copy(void* out, const void* x, double a, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL((k_scaled_copy<VT>), dim3(1024), dim3(256), 0, s, (VT*)out, (const VT*)x, a, count);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

// One-hot basis (every point belongs to exactly one representative): S = W^T D is the sum of the rows of
// D over each representative's points, in a fixed order; Q += W P adds row assign[p] of P to row p.
// Neither streams the dense W.
// ST: type of the block that is read.  Dwide (may be null): every point belongs to exactly one representative,
// so the gather visits every row of D once and can leave a copy of it in the solver's own type on the way
// (the widening of a caller's fp32 block, which the strip kernels then read, costs no pass of its own).
// A representative's points are dealt in turn to `parts` threads per column (run_project: 4 to 8 points each on average,
// more where the workgroup has no more threads or a representative more than its share), whose sums, each in ascending
// point order, are added in a fixed order: the gathers are dependent pairs of loads (point index, then row), so one thread
// per representative and column spent 125 us at 128 points each (42 us now), and the product on 8 clusters of 4096 points
// with one representative each took 722 us (117 us now).
template <typename VT, typename ST>
__global__ __launch_bounds__(1024) void k_onehot_project(const ST* __restrict__ D, VT* __restrict__ Dwide,
                                                         const int32_t* __restrict__ rep_ptr,
                                                         const int32_t* __restrict__ rep_pts, VT* __restrict__ S,
                                                         int ncr, int T, int parts, uint64_t s_d, uint64_t sys,
                                                         uint8_t* __restrict__ odd) {
  __shared__ double red[1024];
  D = of_system(D, s_d);
  S = of_system(S, sys);
  const int rpp = (int)blockDim.x / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  const int reps = rpp / parts;                  // representatives of a workgroup
  const int part = myrow % parts;
  const int a = (int)blockIdx.x * reps + myrow / parts;
  const bool live = myrow < reps * parts && a < ncr;
  double s = 0.0;
  if (live) {
    const int q0 = rep_ptr[a], q1 = rep_ptr[a + 1];
    // eight gathers in flight at a time
    for (int q = q0 + part; q < q1; q += 8 * parts) {
      int idx[8];
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) idx[j] = rep_pts[q + j * parts < q1 ? q + j * parts : q];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (double)D[(int64_t)idx[j] * T + col];
      if (Dwide) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (q + j * parts < q1) Dwide[(int64_t)idx[j] * T + col] = (VT)v[j];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) s += q + j * parts < q1 ? v[j] : 0.0;
    }
  }
  red[tid] = s;
  __syncthreads();
  bool bad = false;
  if (live && part == 0) {
    for (int k = 1; k < parts; ++k) s += red[tid + k * T];
    const VT v = (VT)s;
    S[(int64_t)a * T + col] = v;
    bad = !(v - v == (VT)0);
  }
  if (odd) {                                       // (uniform)
    const int any = __syncthreads_or(bad);
    if (tid == 0) of_system(odd, sys)[blockIdx.x] = any != 0;
  }
}
// the same bytes for a projection that exists: DENSE_ODD_ROWS rows a workgroup
template <typename VT>
__global__ __launch_bounds__(256) void k_odd_rows(const VT* __restrict__ S, int ncr, int T, uint8_t* __restrict__ odd) {
  const int64_t first = (int64_t)blockIdx.x * DENSE_ODD_ROWS * T, end = min((int64_t)ncr * T, first + (int64_t)DENSE_ODD_ROWS * T);
  bool bad = false;
  for (int64_t i = first + threadIdx.x; i < end; i += 256) bad |= !(S[i] - S[i] == (VT)0);
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) odd[blockIdx.x] = any != 0;
}

// out = Q + W P: out is Q itself, or the caller's fp32 block (the narrowing then costs no pass of its own)
// (parts: the column slabs of P = C S, a stride apart, are added up here instead of in a pass of their own)
template <typename VT>
__device__ __forceinline__ double coupling_value(const VT* __restrict__ P, int64_t at, int parts, uint64_t stride) {
  VT s = P[at];
  for (int p = 1; p < parts; ++p) s += P[(uint64_t)p * stride + at];
  return (double)s;
}
template <typename VT, typename OT>
__global__ __launch_bounds__(256) void k_onehot_expand(const VT* Q, const VT* __restrict__ P,
                                                       const int32_t* __restrict__ assign, int64_t n, int T,
                                                       OT* out, int parts, uint64_t stride) {
  const int rpp = 256 / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  if (myrow >= rpp) return;
  for (int64_t p = (int64_t)blockIdx.x * rpp + myrow; p < n; p += (int64_t)gridDim.x * rpp) {
    const int64_t idx = p * T + col;
    out[idx] = (OT)((double)Q[idx] + coupling_value(P, (int64_t)assign[p] * T + col, parts, stride));
  }
}

// the same with the reduction that follows a product in the solver: partial = per-workgroup sums of d q_new
// per column, rows split among the workgroups as in k_dot
template <typename VT>
__global__ __launch_bounds__(VB) void k_onehot_expand_dot(VT* __restrict__ Q, const VT* __restrict__ P,
                                                           const int32_t* __restrict__ assign,
                                                           const VT* __restrict__ D, int64_t n, int T,
                                                           double* __restrict__ partial, int parts, uint64_t stride, uint64_t sys, uint64_t s_d) {
  __shared__ double red[VB];
  Q = of_system(Q, sys); P = of_system(P, sys); partial = of_system(partial, sys);
  D = of_system(D, s_d);
  const int rpp = (int)blockDim.x / T;
  const int tid = threadIdx.x;
  const int myrow = tid / T, col = tid - myrow * T;
  const bool live = myrow < rpp;
  const int64_t rows_per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  double s0 = 0.0;
  if (live) {
    for (int64_t p = r0 + myrow; p < r1; p += ROWS_AT_ONCE * rpp) {
      VT d[ROWS_AT_ONCE], q[ROWS_AT_ONCE];
      int32_t a[ROWS_AT_ONCE];
      double w[ROWS_AT_ONCE];
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j) {
        const int64_t row = p + j * rpp < r1 ? p + j * rpp : p;
        a[j] = assign[row];
        d[j] = D[row * T + col]; q[j] = Q[row * T + col];
      }
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j) w[j] = coupling_value(P, (int64_t)a[j] * T + col, parts, stride);
#pragma unroll
      for (int j = 0; j < ROWS_AT_ONCE; ++j)
        if (p + j * rpp < r1) {
          const VT qn = (VT)((double)q[j] + w[j]);
          Q[(p + j * rpp) * T + col] = qn;
          s0 = fma((double)d[j], (double)qn, s0);
        }
    }
  }
  red[tid] = s0;
  const double sum = column_sum(red, T, tid);
  if (tid < T) partial[(int64_t)blockIdx.x * MAX_COLS + tid] = sum;
}

static int elementwise_grid(int64_t n, int T);

// S = W^T D into the first slab of Spart (summed over the column slabs when W is dense).  D32 (one-hot basis,
// fp64 mode only): the block is read from this fp32 array and its widened copy is written to D on the way.
static int run_project(nugpr_ctx* c, const void* D, int T, hipStream_t s, const float* D32, int nsys, uint64_t s_d) {
  const Layout& L = c->L;
  uint8_t* odd = c->c_skips ? static_cast<uint8_t*>(c->Spart) + odd_offset(c, T) : nullptr;
  if (D32 && !(c->onehot && c->acc64)) { set_error("internal: fused widening needs the one-hot basis in fp64 mode"); return NUGPR_ERR_INVALID; }
  if (c->onehot) {
    const ProjectShape shape = project_shape(L, T);
    const int parts = shape.parts;
    const dim3 grid((unsigned)((L.ncr + shape.reps - 1) / shape.reps), (unsigned)nsys), blk((unsigned)shape.block);
    const uint64_t sys = L.slot_bytes;
    if (D32) hipLaunchKernelGGL((k_onehot_project<double, float>), grid, blk, 0, s, D32, (double*)const_cast<void*>(D), c->rep_ptr, c->rep_pts, (double*)c->Spart, L.ncr, T, parts, s_d, sys, odd);
    else if (c->acc64) hipLaunchKernelGGL((k_onehot_project<double, double>), grid, blk, 0, s, (const double*)D, (double*)nullptr, c->rep_ptr, c->rep_pts, (double*)c->Spart, L.ncr, T, parts, s_d, sys, odd);
    else hipLaunchKernelGGL((k_onehot_project<float, float>), grid, blk, 0, s, (const float*)D, (float*)nullptr, c->rep_ptr, c->rep_pts, (float*)c->Spart, L.ncr, T, parts, s_d, sys, odd);
    NUGPR_HIP(hipGetLastError());
    return NUGPR_OK;
  }
  int rc;
  const uint64_t spart = (uint64_t)L.ncr * T;
  StripPort s0{};
  s0.A = c->Wt; s0.in = D; s0.out = c->Spart; s0.out_part_stride = spart;
  if ((rc = launch_strip(c->tab_WtD, s0, s0, T, c->acc64, s))) return rc;
  if (L.nsS > 1 && (rc = launch_sum_parts(c->Spart, c->Spart, (int64_t)spart, L.nsS, spart, c->acc64, s))) return rc;
  if (odd) {                                       // (over slabs that are added up)
    const dim3 grid((unsigned)((L.ncr + DENSE_ODD_ROWS - 1) / DENSE_ODD_ROWS));
    if (c->acc64) hipLaunchKernelGGL((k_odd_rows<double>), grid, dim3(256), 0, s, (const double*)c->Spart, L.ncr, T, odd);
    else hipLaunchKernelGGL((k_odd_rows<float>), grid, dim3(256), 0, s, (const float*)c->Spart, L.ncr, T, odd);
    NUGPR_HIP(hipGetLastError());
  }
  return NUGPR_OK;
}

// Q += W P with P the first slab of Ppart; with Q32 (one-hot basis, fp64 mode) the sum goes to that fp32 array instead
static int run_expand(nugpr_ctx* c, void* Q, int T, hipStream_t s, const void* D, double* dq_partial, float* Q32, int parts, int nsys, uint64_t s_d) {
  const Layout& L = c->L;
  const uint64_t stride = (uint64_t)L.ncr * T;
  if (Q32 && !(c->onehot && c->acc64 && !dq_partial)) { set_error("internal: fused narrowing needs the one-hot basis in fp64 mode"); return NUGPR_ERR_INVALID; }
  if (c->onehot && dq_partial) {
    const dim3 nb((unsigned)L.n_dot_blocks, (unsigned)nsys);
    const uint64_t sys = L.slot_bytes;
    if (c->acc64) hipLaunchKernelGGL((k_onehot_expand_dot<double>), nb, dim3(vector_threads(T)), 0, s, (double*)Q, (const double*)c->Ppart, c->assign, (const double*)D, (int64_t)L.n, T, dq_partial, parts, stride, sys, s_d);
    else hipLaunchKernelGGL((k_onehot_expand_dot<float>), nb, dim3(vector_threads(T)), 0, s, (float*)Q, (const float*)c->Ppart, c->assign, (const float*)D, (int64_t)L.n, T, dq_partial, parts, stride, sys, s_d);
    NUGPR_HIP(hipGetLastError());
    return NUGPR_OK;
  }
  if (c->onehot) {
    const int grid = elementwise_grid(L.n, T);
    if (Q32) hipLaunchKernelGGL((k_onehot_expand<double, float>), dim3(grid), dim3(256), 0, s, (const double*)Q, (const double*)c->Ppart, c->assign, (int64_t)L.n, T, Q32, parts, stride);
    else if (c->acc64) hipLaunchKernelGGL((k_onehot_expand<double, double>), dim3(grid), dim3(256), 0, s, (const double*)Q, (const double*)c->Ppart, c->assign, (int64_t)L.n, T, (double*)Q, parts, stride);
    else hipLaunchKernelGGL((k_onehot_expand<float, float>), dim3(grid), dim3(256), 0, s, (const float*)Q, (const float*)c->Ppart, c->assign, (int64_t)L.n, T, (float*)Q, parts, stride);
    NUGPR_HIP(hipGetLastError());
    return NUGPR_OK;
  }
  StripPort w0{};
  w0.A = c->Wd; w0.in = c->Ppart; w0.out = Q; w0.accumulate = 1;
  return launch_strip(c->tab_WP, w0, w0, T, c->acc64, s);
}

// Q += scale * W (C_offdiag (W^T D)): the low-rank part of the product on its own
static int run_lowrank_accumulate(nugpr_ctx* c, const void* D, void* Q, int T, hipStream_t s) {
  const Layout& L = c->L;
  int rc;
  const uint64_t ppart = (uint64_t)L.ncr * T;
  if ((rc = run_project(c, D, T, s))) return rc;
  StripPort k1{};
  k1.A = c->C; k1.in = c->Spart; k1.out = c->Ppart; k1.out_part_stride = ppart; k1.scale = c->op_scale;
  skip_dead_items(c, k1, T);
  if ((rc = launch_strip(c->tab_C, k1, k1, T, c->acc64, s))) return rc;
  if (L.compensate) {
    StripPort k2 = k1;
    k2.A = c->Clo; k2.accumulate = 1;
    if ((rc = launch_strip(c->tab_C, k2, k2, T, c->acc64, s))) return rc;
  }
  if (L.nsP > 1 && (rc = launch_sum_parts(c->Ppart, c->Ppart, (int64_t)ppart, L.nsP, ppart, c->acc64, s))) return rc;
  return run_expand(c, Q, T, s);
}

// out = A D with A = Y K' Y^T, Y = L^-1 (the paper's R^-T K' R^-1, eq. (RKR)).  Scratch: Vv, Uv.
// While the stored blocks are the ones that were factored, K_diag = s L L^T + shift I for the
// operator in force (eqs. (linear1)-(linear3)), so A D = s D + Y (shift U + s W C W^T U), U = Y^T D,
// and the block-diagonal matrix is not streamed at all.
int run_split_op(nugpr_ctx* c, const void* D, void* out, int T, hipStream_t s) {
  int rc;
  const int64_t cnt = c->L.n * T;
  StripPort up{};
  up.A = c->G; up.in = D; up.out = c->Vv;
  if ((rc = launch_strip(c->tab_upG, up, up, T, c->acc64, s))) return rc;                 // U = Y^T D
  const bool identity = c->build_gen == c->factor_gen && !c->general_route &&
                        !(c->params.flags & (NUGPR_NO_SHORTCUTS | NUGPR_PRECOND_COMPENSATED));
  StripPort lo{};
  lo.A = c->G; lo.in = c->Uv; lo.out = out;
  if (!identity) {
    if ((rc = run_matvec(c, c->Vv, c->Uv, T, s))) return rc;                              // K' U
  } else {
    rc = c->acc64 ? scaled_copy<double>(c->Uv, c->Vv, c->op_shift, cnt, s) : scaled_copy<float>(c->Uv, c->Vv, c->op_shift, cnt, s);
    if (rc) return rc;
    if ((rc = run_lowrank_accumulate(c, c->Vv, c->Uv, T, s))) return rc;
    rc = c->acc64 ? scaled_copy<double>(out, D, c->op_scale, cnt, s) : scaled_copy<float>(out, D, c->op_scale, cnt, s);
    if (rc) return rc;
    lo.accumulate = 1;
  }
  return launch_strip(c->tab_lowG, lo, lo, T, c->acc64, s);                               // Y (.)
}

// Q = (A^2 + 4 A + I) D, eq. (PQ).  Scratch: Zv (holds A D), and what run_split_op uses.
static int run_pade_q(nugpr_ctx* c, const void* D, void* Q, int T, hipStream_t s) {
  int rc;
  if ((rc = run_split_op(c, D, c->Zv, T, s))) return rc;
  if ((rc = run_split_op(c, c->Zv, Q, T, s))) return rc;
  const int64_t cnt = c->L.n * T;
  if (c->acc64)
    hipLaunchKernelGGL((k_pade_q_combine<double>), dim3(1024), dim3(256), 0, s, (double*)Q, (const double*)c->Zv, (const double*)D, cnt);
  else
    hipLaunchKernelGGL((k_pade_q_combine<float>), dim3(1024), dim3(256), 0, s, (float*)Q, (const float*)c->Zv, (const float*)D, cnt);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

// (nsys > 1: R and Z of system 0, the others a slot further; the first `held` of them are counted)
static int precond(nugpr_ctx* c, const void* R, void* Z, int T, hipStream_t s, int nsys, int held) {
  int rc;
  const uint64_t sys = c->L.slot_bytes;
  c->stats.precond_applies += held;
  StripPort a[MAX_SLOTS] = {}, b[MAX_SLOTS] = {};
  for (int e = 0; e < nsys; ++e) {
    a[e].A = c->G; a[e].in = slot_of(R, sys, e); a[e].out = slot_of(c->Vv, sys, e);
    b[e].A = c->G; b[e].in = a[e].out; b[e].out = slot_of(Z, sys, e);
  }
  if ((rc = launch_strip(c->tab_lowG, a, nsys, T, c->acc64, s, nsys))) return rc;
  return launch_strip(c->tab_upG, b, nsys, T, c->acc64, s, nsys);
}
int run_precond(nugpr_ctx* c, const void* R, void* Z, int T, hipStream_t s) { return precond(c, R, Z, T, s, 1, 1); }

static int elementwise_grid(int64_t n, int T) {
  const int rpp = 256 / T;
  int64_t g = (n + rpp - 1) / rpp;
  return (int)std::min<int64_t>(g, 4096);
}

template <typename VT>
static int dot2_t(nugpr_ctx* c, const VT* A0, const VT* B0, const VT* A1, const VT* B1, int T, double* out0,
                  double* out1, hipStream_t s) {
  const Layout& L = c->L;
  const int nb = L.n_dot_blocks;
  hipLaunchKernelGGL((k_dot<2, VT>), dim3(nb), dim3(vector_threads(T)), 0, s, A0, B0, A1, B1, (int64_t)L.n, T, c->dotpart, (uint64_t)0, (uint64_t)0, (uint64_t)0);
  NUGPR_HIP(hipGetLastError());
  NUGPR_HIP(hipMemcpyAsync(c->h_buf, c->dotpart, (size_t)2 * nb * MAX_COLS * sizeof(double), hipMemcpyDeviceToHost, s));
  NUGPR_HIP(hipStreamSynchronize(s));
  for (int col = 0; col < T; ++col) {
    double a0 = 0.0, a1 = 0.0;
    for (int b = 0; b < nb; ++b) {
      a0 += c->h_buf[(size_t)b * MAX_COLS + col];
      a1 += c->h_buf[((size_t)nb + b) * MAX_COLS + col];
    }
    out0[col] = a0;
    out1[col] = a1;
  }
  return NUGPR_OK;
}

// <A0, B0> and <A1, B1> per column, one synchronisation
int run_dot2(nugpr_ctx* c, const void* A0, const void* B0, const void* A1, const void* B1, int T, double* out0,
             double* out1, hipStream_t s) {
  if (c->acc64) return dot2_t<double>(c, (const double*)A0, (const double*)B0, (const double*)A1, (const double*)B1, T, out0, out1, s);
  return dot2_t<float>(c, (const float*)A0, (const float*)B0, (const float*)A1, (const float*)B1, T, out0, out1, s);
}

template <typename VT>
static int pcg_t(nugpr_ctx* c, const VT* B, VT* X, int T, const Operator* ops, int held, PcgOutcome* out, hipStream_t s, int system) {
  const Layout& L = c->L;
  const uint64_t sys = L.slot_bytes;
  const int nsys = held == 3 ? 4 : held;
  const unsigned ny = (unsigned)nsys;
  const bool extras = out[0].extras != nullptr;
  const int64_t n = L.n;
  const int nb = L.n_dot_blocks;
  const int vt = vector_threads(T);
  // workgroups of the direction update: four rows a thread, and where each of them adds up the partial sums first, no more than two
  // on a compute unit
  const int eg = (int)std::min<int64_t>((n + ROWS_AT_ONCE * (VB / T) - 1) / (ROWS_AT_ONCE * (VB / T)), nb <= FUSE_BLOCKS ? 512 : 4096);
  const double tol2 = c->params.tol * c->params.tol;
  const int max_iter = c->params.max_iter;
  int rc;
  VT *R = (VT*)c->Rv, *Z = (VT*)c->Zv, *D = (VT*)c->Dv, *Q = (VT*)c->Qv;
  // Without a preconditioner (the Pade system, already preconditioned) z = r throughout.
  const bool plain = system == PCG_PADE_Q;
  const VT* Zr = plain ? R : Z;
  // Solves on the two right-hand-side blocks the context owns start from values kept with the factor:
  // z_0 = M^-1 b (or b itself for the Pade system), <b, b> and <b, z_0>.  Nothing is initialised then:
  // the first update reads b in the place of r and writes x without reading it, and the first direction
  // is z_0 where it lies.
  const bool own = T == L.T && c->z0_ready && (const void*)B == (plain ? (const void*)c->Pv : (const void*)c->Bv);
  // systems side by side: their own blocks lie a slot apart; the context's right-hand sides and z_0 are shared
  const uint64_t s_b = own ? 0 : sys;
  uint64_t s_d = own ? 0 : sys;
  const VT* Dcur = D;                    // the direction the operator is applied to
  if (own) {
    if (nb > FUSE_BLOCKS) hipLaunchKernelGGL(k_pcg_begin_known, dim3(1), dim3(64), 0, s, c->d_state, plain ? 1 : 0, T);
    Dcur = plain ? B : (const VT*)c->Z0v;
  } else {
    // x_0 = 0, r_0 = b, d_0 = z_0 = M^-1 r_0 written straight into D
    hipLaunchKernelGGL((k_pcg_init<VT>), dim3(1024, ny), dim3(256), 0, s, X, R, B, plain ? B : (const VT*)nullptr, D, n * T, sys, s_b);
    if (!plain && (rc = precond(c, R, D, T, s, nsys, held))) return rc;
    hipLaunchKernelGGL((k_dot<2, VT>), dim3(nb, ny), dim3(vt), 0, s, (const VT*)R, (const VT*)R, (const VT*)R, (const VT*)D, n, T, c->dotpart, sys, sys, sys);
    hipLaunchKernelGGL(k_pcg_begin, dim3(T, ny), dim3(256), 0, s, c->d_state, c->dotpart, nb, sys);
  }
  NUGPR_HIP(hipGetLastError());
  bool first = own;
  int it = 0;
  // The first iteration is issued without asking the device whether any column is active: columns
  // that start inactive (zero right-hand side) are skipped by every kernel on their own flag, and
  // the host learns the count at the first stop test.
  for (int e = 0; e < nsys; ++e) c->h_flags[e].n_active = 1;
  const size_t cnt = (size_t)max_iter * MAX_COLS;
  PcgState* hs = reinterpret_cast<PcgState*>(c->h_buf + 2 * cnt);
  double* hdot = c->h_buf + 2 * cnt + (sizeof(PcgState) + sizeof(double) - 1) / sizeof(double);
  const uint64_t hsys = host_record_doubles(max_iter) * sizeof(double);      // a system's part of the pinned buffer
  const bool want_logs = out[0].alpha || out[0].beta || out[0].logs;
  // partial sums: sets 0 and 1 belong to the update kernel (|r|^2, <b, x>), 2 to <d, q>, 3 to <r, z>
  double *const dq_sums = c->dotpart + (size_t)2 * nb * MAX_COLS, *const rz_sums = c->dotpart + (size_t)3 * nb * MAX_COLS;
  const bool fuse = nb <= FUSE_BLOCKS;
  // Up to as many iterations as each of the last three solves of this kind and width needed, the host issues an
  // iteration while the device still works on the one before it, whose stop test it has not seen.  Should that test end
  // the solve, ONE iteration was issued in vain: every column's steps are zero in it and change nothing.  A loss gains
  // 8 - 12 us by it whatever its size (24576 points 342 us, 352 without; 131072 points 1272 / 1284), but an iteration in
  // vain costs what an iteration costs, so larger problems wait for every test.
  nugpr_ctx::IterationRecord& rec = c->recent_iters[plain ? 1 : own ? 0 : T == 1 ? 3 : 2];
  if (rec.ncols != T) { rec.ncols = T; rec.last[0] = rec.last[1] = rec.last[2] = 1; }
  const int sure = fuse ? std::min(rec.last[0], std::min(rec.last[1], rec.last[2])) : 1;
  nugpr_stats counted = c->stats, counted_before = c->stats;      // after the product of the present iteration, and the last
  // The end-of-solve report comes with the stop test of the iteration that is expected to be the last
  // one, so that it is already on the host when the stop test says "done", and with that of the iteration after it;
  // a solve that ends earlier or later than that gets the report after the loop (with one in every iteration from the expected
  // one on, a solve of k more iterations than the last would copy k rows k times over).
  const int expect = c->expect_iters[plain ? 1 : 0];
  // (its <b, x> sums were left in the second partial set by the update kernel of the same iteration)
  auto next_report = [&](int rows) {
    c->tail_seq += 1;
    return Report{c->tail_seq, extras ? 1 : 0, want_logs ? rows : 0, c->alog, c->blog, hs, hdot, c->h_buf, c->h_buf + cnt, hsys};
  };
  auto issue_tail = [&](int rows) -> int {
    if (extras)
      hipLaunchKernelGGL((k_dot<2, VT>), dim3(nb, ny), dim3(vt), 0, s, B, (const VT*)X, B, (const VT*)X, n, T, c->dotpart, s_b, sys, sys);
    hipLaunchKernelGGL(k_pcg_tail, dim3(T, ny), dim3(256), 0, s, c->d_state, c->dotpart + (size_t)nb * MAX_COLS, nb, T, next_report(rows), c->h_flags, sys);
    NUGPR_HIP(hipGetLastError());
    return NUGPR_OK;
  };
  bool tail_current = false;
  while (it < max_iter) {
    bool dq_done = false;
    if ((rc = plain ? run_pade_q(c, Dcur, Q, T, s) : product(c, ops, nsys, held, Dcur, Q, T, s, dq_sums, &dq_done, nullptr, nullptr))) return rc;
    if (!dq_done)
      hipLaunchKernelGGL((k_dot<1, VT>), dim3(nb, ny), dim3(vt), 0, s, Dcur, (const VT*)Q, Dcur, (const VT*)Q, n, T, dq_sums, s_d, sys, sys);
    if (!fuse) hipLaunchKernelGGL(k_pcg_alpha, dim3(T), dim3(256), 0, s, c->d_state, dq_sums, nb, it, c->alog);
    // the update, fused with ||r||^2 for the stop test and, in the iteration expected to be the last, <b, x>
    const bool report = it + 1 == expect || it == expect || it + 1 >= max_iter;
    hipLaunchKernelGGL((k_update_xr_dots<VT>), dim3(nb, ny), dim3(vt), 0, s, X, R, first ? B : (const VT*)R, Dcur,
                       (const VT*)Q, (report && extras) ? B : (const VT*)nullptr, c->d_state, n, T, first ? 1 : 0,
                       c->dotpart, fuse ? dq_sums : (const double*)nullptr, it, c->alog, sys, first ? s_b : sys, s_d, s_b, fuse && own && it == 0 ? (plain ? 1 : 0) : -1);
    first = false;
    // stop test first: when every column has converged the preconditioner apply is not needed
    c->flag_seq += 1;
    hipLaunchKernelGGL(k_pcg_check, dim3(T, ny), dim3(256), 0, s, c->d_state, c->dotpart, nb, it, tol2, T, c->h_flags,
                       c->flag_seq, sys, report ? next_report(it + 1) : Report{});
    NUGPR_HIP(hipGetLastError());
    tail_current = report;
    const int j = it++;
    counted_before = counted;
    counted = c->stats;
    const bool ahead = it < sure && it < max_iter;                // the stop test to wait for: this one's, or the last one's
    if (!ahead || it > 1) {
      int n_active = 0;
      for (int e = 0; e < nsys; ++e) {
        if ((rc = wait_seq(&c->h_flags[e].seq, c->flag_seq - (ahead ? 1 : 0), s))) return rc;
        n_active += c->h_flags[e].n_active;
      }
      if (n_active == 0 || it >= max_iter) break;
    }
    if (!plain && (rc = precond(c, R, Z, T, s, nsys, held))) return rc;
    hipLaunchKernelGGL((k_dot<1, VT>), dim3(nb, ny), dim3(vt), 0, s, (const VT*)R, Zr, (const VT*)R, Zr, n, T, rz_sums, sys, sys, sys);
    if (!fuse) hipLaunchKernelGGL(k_pcg_beta, dim3(T), dim3(256), 0, s, c->d_state, rz_sums, nb, j, c->blog);
    hipLaunchKernelGGL((k_update_d<VT>), dim3(eg, ny), dim3(vt), 0, s, D, Dcur, Zr, c->d_state, n, T,
                       fuse ? rz_sums : (const double*)nullptr, nb, j, c->blog, sys, s_d);
    NUGPR_HIP(hipGetLastError());
    Dcur = D;
    s_d = sys;
  }
  if (!tail_current && (rc = issue_tail(it))) return rc;
  for (int e = 0; e < nsys; ++e)
    if ((rc = wait_seq(&c->h_flags[e].tail_seq, c->tail_seq, s))) return rc;
  // NaN / Inf among the coordinates of the last assembly (found by its scaling kernel, which marks system 0's state)
  const bool bad_points = c->assembly_mark != 0 && hs->nonfinite_mark == c->assembly_mark;
  int longest = 0, in_vain = 0;
  for (int e = 0; e < held; ++e) {
    const PcgState* st = slot_of(hs, hsys, e);
    const double *dot = slot_of(hdot, hsys, e), *ha = slot_of(c->h_buf, hsys, e);
    PcgOutcome& o = out[e];
    bool all_conv = true, indefinite = false, finite = !bad_points;
    o.max_it = 0;
    o.alog = ha;
    o.blog = ha + cnt;
    for (int col = 0; col < T; ++col) {
      if (o.iters) o.iters[col] = st->iters[col];
      o.max_it = std::max(o.max_it, st->iters[col]);
      if (!st->converged[col]) all_conv = false;
      if (st->indef[col]) indefinite = true;
      // or in a right-hand side: it shows in the first dot products of its column, <b, b> and <b, M^-1 b>
      if (!std::isfinite(st->bnorm2[col]) || !std::isfinite(st->rho0[col])) finite = false;
      if (o.extras) {
        o.extras->bx[col] = dot[col];
        o.extras->rho0[col] = st->rho0[col];
      }
    }
    const int needed = std::min(std::max(st->steps, 1), it);
    longest = std::max(longest, needed);
    in_vain += it - needed;
    c->stats.pcg_solves += 1;
    c->stats.pcg_iterations += needed;
    c->stats.pcg_iterations_max = std::max<int64_t>(c->stats.pcg_iterations_max, needed);
    for (int j = 0; j < max_iter && (o.alpha || o.beta); ++j)
      for (int col = 0; col < T; ++col) {                 // rows past the last iteration were never written: zero
        if (o.alpha) o.alpha[(size_t)j * T + col] = j < it ? ha[(size_t)j * MAX_COLS + col] : 0.0;
        // (no beta follows the last iteration)
        if (o.beta) o.beta[(size_t)j * T + col] = j < it - 1 ? ha[cnt + (size_t)j * MAX_COLS + col] : 0.0;
      }
    o.status = !finite ? NUGPR_NOT_FINITE : indefinite ? NUGPR_INDEFINITE : all_conv ? NUGPR_OK : NUGPR_NOT_CONVERGED;
  }
  // The counters leave out iterations that a system did not need: the one issued ahead of its stop test, if there was one, and
  // those in which it only kept another one company.
  if (nsys == 1) {
    if (in_vain) { counted_before.pcg_solves = c->stats.pcg_solves; counted_before.pcg_iterations = c->stats.pcg_iterations; counted_before.pcg_iterations_max = c->stats.pcg_iterations_max; c->stats = counted_before; }
  } else {
    c->stats.products -= in_vain;
    c->stats.precond_applies -= in_vain;
  }
  c->expect_iters[plain ? 1 : 0] = longest;
  rec.last[2] = rec.last[1]; rec.last[1] = rec.last[0]; rec.last[0] = longest;
  return NUGPR_OK;
}

template <typename VT>
static int store_known_t(nugpr_ctx* c, hipStream_t s) {
  const Layout& L = c->L;
  const int nb = L.n_dot_blocks;
  const VT *B = (const VT*)c->Bv, *Z0 = (const VT*)c->Z0v, *P = (const VT*)c->Pv;
  const uint64_t one = 0;                // (one system)
  hipLaunchKernelGGL((k_dot<2, VT>), dim3(nb), dim3(vector_threads(L.T)), 0, s, B, B, B, Z0, (int64_t)L.n, L.T, c->dotpart, one, one, one);
  hipLaunchKernelGGL(k_store_known, dim3(L.T), dim3(256), 0, s, c->d_state, c->dotpart, nb, 0);
  if (L.t > 0) {
    hipLaunchKernelGGL((k_dot<2, VT>), dim3(nb), dim3(vector_threads(L.T)), 0, s, P, P, P, P, (int64_t)L.n, L.T, c->dotpart, one, one, one);
    hipLaunchKernelGGL(k_store_known, dim3(L.T), dim3(256), 0, s, c->d_state, c->dotpart, nb, 1);
  }
  NUGPR_HIP(hipGetLastError());
  // W^T z_0
  int rc = run_project(c, c->Z0v, L.T, s);
  if (rc) return rc;
  NUGPR_HIP(hipMemcpyAsync(c->S0v, c->Spart, (size_t)L.ncr * L.T * sizeof(VT), hipMemcpyDeviceToDevice, s));
  return NUGPR_OK;
}

// <b, b> and <b, z_0> of the context's own right-hand-side blocks, kept in the device state (called by the
// factorisation once B, z_0 = M^-1 B and the probe block exist)
int store_known_starts(nugpr_ctx* c, hipStream_t s) {
  return c->acc64 ? store_known_t<double>(c, s) : store_known_t<float>(c, s);
}

int run_pcg_systems(nugpr_ctx* c, const void* B, void* X, int T, const Operator* ops, int held, PcgOutcome* out, hipStream_t s, int system) {
  if (c->acc64) return pcg_t<double>(c, (const double*)B, (double*)X, T, ops, held, out, s, system);
  return pcg_t<float>(c, (const float*)B, (float*)X, T, ops, held, out, s, system);
}

int run_pcg(nugpr_ctx* c, const void* B, void* X, int T, int32_t* iters, double* alpha, double* beta,
            int* max_it_used, hipStream_t s, PcgExtras* extras, int system) {
  const Operator op = operator_in_force(c);
  PcgOutcome out{};
  out.iters = iters; out.alpha = alpha; out.beta = beta; out.extras = extras;
  const int rc = run_pcg_systems(c, B, X, T, &op, 1, &out, s, system);
  if (rc) return rc;
  if (max_it_used) *max_it_used = out.max_it;
  return out.status;
}

}  // namespace nugpr
